// Batched full-depth pass over many positions: the prompt pass and the
// periodic refresh of recent positions. The decode program handles one
// position per step and streams every weight once per position; here a
// chunk of positions goes through each layer together, so each weight is
// read once per chunk and the work is a tiled matrix product (positions x
// weight rows) instead of matrix-vector products.
//
// Per layer (stream order is the only synchronisation):
//   1. QKV:    Y = RMSNorm(X; g_attn) W_qkv^T, RoPE on q and k at each
//              position, k and v stored to the paged cache, q kept;
//   2. attn:   causal grouped-query attention of the chunk's queries over
//              every cached position up to their own (split over key
//              ranges when the chunk alone does not fill the device, then
//              merged in split order);
//   3. W_o:    X += O W_o^T;
//   4. gate/up: A = SiLU(RMSNorm(X; g_mlp) W_g^T) * (RMSNorm(X; g_mlp) W_u^T);
//   5. down:   X += A W_d^T.
// With bf16 weights the products run on the matrix cores (ee_mm.h): the
// producer of each vector splits it into bf16 terms once, and the residual
// products store the partial sums of their K slices, which the kernel that
// prepares the next product's input adds up in slice order. With fp32 weights
// the vector ALU computes them (k_bp_gemm), the last workgroup to finish a
// tile adding its K slices. Every result is independent of scheduling.
//
// Numerics follow the decode program: weights as stored (bf16 or fp32),
// activations and accumulation fp32, cache entries rounded to the storage
// type (round to nearest even), RMSNorm as x * rsqrt(mean(x^2) + eps) * g
// (the row's scale is applied to the finished dot products), e^x in the
// softmax and SiLU on the hardware base-2 exponential.
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "ee_internal.h"
#include "ee_mm.h"

namespace ee {

namespace {

// ---------------------------------------------------------------------------
// helpers (this file's own; the decode kernels keep theirs)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent2(float* p, float a, float b) {  // p 8-byte aligned
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p),
                     static_cast<uint64_t>(__float_as_uint(a)) | (static_cast<uint64_t>(__float_as_uint(b)) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent2(const float* p) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<uint64_t*>(const_cast<float*>(p)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float(static_cast<uint32_t>(v)), __uint_as_float(static_cast<uint32_t>(v >> 32)));
}
__device__ __forceinline__ void drain_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ float exp_hw(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

template <typename WT>
struct St;

template <>
struct St<uint16_t> {  // bf16 bit patterns
  __device__ static inline void unpack(const uint4& w, float* f) {
    f[0] = __uint_as_float(w.x << 16);
    f[1] = __uint_as_float(w.x & 0xffff0000u);
    f[2] = __uint_as_float(w.y << 16);
    f[3] = __uint_as_float(w.y & 0xffff0000u);
    f[4] = __uint_as_float(w.z << 16);
    f[5] = __uint_as_float(w.z & 0xffff0000u);
    f[6] = __uint_as_float(w.w << 16);
    f[7] = __uint_as_float(w.w & 0xffff0000u);
  }
  __device__ static inline uint32_t bits(float x) {  // round to nearest even
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
  }
  __device__ static inline void store_pair(uint16_t* p, float a, float b) {
    *reinterpret_cast<uint32_t*>(p) = bits(a) | (bits(b) << 16);
  }
  __device__ static inline float2 load_pair(const uint16_t* p) {
    const uint32_t u = *reinterpret_cast<const uint32_t*>(p);
    return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
  }
};

template <>
struct St<float> {
  static constexpr int N = 4;
  __device__ static inline void unpack(const uint4& w, float* f) {
    f[0] = __uint_as_float(w.x);
    f[1] = __uint_as_float(w.y);
    f[2] = __uint_as_float(w.z);
    f[3] = __uint_as_float(w.w);
  }
  __device__ static inline void store_pair(float* p, float a, float b) {
    *reinterpret_cast<float2*>(p) = make_float2(a, b);
  }
  __device__ static inline float2 load_pair(const float* p) { return *reinterpret_cast<const float2*>(p); }
};

__device__ __forceinline__ int64_t cache_off(const int32_t* block_table, int page_shift, int page_size, int K,
                                             int D, int64_t layer_base, int pos, int kvh) {
  const int page = block_table[pos >> page_shift];
  const int slot = pos & (page_size - 1);
  return layer_base + ((static_cast<int64_t>(page) * K + kvh) * page_size + slot) * D;
}

// Wave reductions: DPP within rows of 16 lanes, then the four row results
// by readlane; every lane gets the same value, summed in a fixed order.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_of(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ float wave_max64(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));   // lane ^ 1
  v = fmaxf(v, dpp_mov<0x4E>(v));   // lane ^ 2
  v = fmaxf(v, dpp_mov<0x141>(v));  // the other quad of the 8
  v = fmaxf(v, dpp_mov<0x140>(v));  // the other 8 of the 16
  return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 16)), fmaxf(lane_of(v, 32), lane_of(v, 48)));
}
__device__ __forceinline__ float wave_sum64(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

}  // namespace

// ---------------------------------------------------------------------------
// embedding rows of the chunk's tokens
// ---------------------------------------------------------------------------
template <typename WT>
__global__ __launch_bounds__(256) void k_bp_embed(const WT* __restrict__ E, const int32_t* __restrict__ tok, int P,
                                                  int H, int V, float* __restrict__ X, int32_t* hist, int pos0,
                                                  StepCtl* ctl) {
  const int p = blockIdx.x;
  if (p >= P) return;
  int t = tok[p];
  if (t < 0 || t >= V) {
    if (threadIdx.x == 0) atomicMax(&ctl->error, kErrToken);
    t = 0;
  }
  if (threadIdx.x == 0 && hist) hist[pos0 + p] = t;
  const WT* row = E + static_cast<int64_t>(t) * H;
  for (int i0 = 0; i0 < H; i0 += 8 * 256) {
    WT v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + threadIdx.x + 256 * u;
      v[u] = i < H ? row[i] : WT(0);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + threadIdx.x + 256 * u;
      if (i >= H) continue;
      float f;
      if constexpr (sizeof(WT) == 2) f = __uint_as_float(static_cast<uint32_t>(v[u]) << 16);
      else f = v[u];
      X[static_cast<int64_t>(p) * H + i] = f;
    }
  }
}

// ---------------------------------------------------------------------------
// tiled matrix product Y[P][N] = A[P][K] W[N][K]^T with fused RMSNorm of A
// (when gain is set) and an epilogue. Block tile BM positions x BN weight
// rows, 256 threads, each TM x 4 outputs; K in stages of BK (one 128-byte
// line of a weight row), the next stage's tiles loaded into registers while
// the current one is consumed from LDS.
// ---------------------------------------------------------------------------
enum : int { kEpiQkv = 0, kEpiResid = 1, kEpiSwiGlu = 2 };

struct GemmArgs {
  const float* A;      // [P][K] fp32
  const void* W;       // [N][K] storage type
  int P, N, K;
  int k_split;         // K elements per split (multiple of BK), splits = gridDim.z
  const float* gain;   // RMSNorm gain [K] (A is the raw residual stream) or null
  float eps;
  float* part;         // split partials [splits][P][N], then [splits][P] sums of squares
  uint32_t* tile_ctr;  // arrivals per output tile (zero before, reset by the last arrival)
  // epilogue targets
  float* Y;            // kEpiResid: X [P][N] (+=); kEpiSwiGlu: A [P][N/2]; kEpiQkv: q [P][A*D]
  u32x4* planes;       // kEpiSwiGlu on the matrix cores: term planes of A, k32_out K blocks
  int k32_out;
  // kEpiQkv: RoPE and cache
  int pos0, Aq, Kh, D;
  const float* rope_cos;
  const float* rope_sin;
  void* kpool;
  void* vpool;
  int64_t layer_base;
  const int32_t* block_table;
  int page_shift, page_size;
};

template <typename WT>
__device__ __forceinline__ void epi_pair(const GemmArgs& g, int EPI, int m, int n, float y0, float y1) {
  if (EPI == kEpiResid) {
    float2* x = reinterpret_cast<float2*>(g.Y + static_cast<int64_t>(m) * g.N + n);
    float2 v = *x;
    v.x += y0;
    v.y += y1;
    *x = v;
  } else if (EPI == kEpiSwiGlu) {
    // interleaved rows: n = 2j gate row j, n + 1 up row j
    const float s = y0 / (1.f + exp_hw(-y0));
    g.Y[static_cast<int64_t>(m) * (g.N >> 1) + (n >> 1)] = s * y1;
  } else {
    // rows of the repacked QKV matrix: q heads, k heads (RoPE pairs
    // interleaved: row 2i = dim i, row 2i+1 = dim i + D/2), v heads
    const int AD = g.Aq * g.D, KD = g.Kh * g.D;
    const int pos = g.pos0 + m;
    if (n < AD + KD) {
      const int head = n / g.D, rl = n - head * g.D, half = g.D >> 1;
      const float c = g.rope_cos[static_cast<int64_t>(pos) * half + (rl >> 1)];
      const float s = g.rope_sin[static_cast<int64_t>(pos) * half + (rl >> 1)];
      const float r0 = y0 * c - y1 * s;
      const float r1 = y1 * c + y0 * s;
      if (n < AD) {
        *reinterpret_cast<float2*>(g.Y + static_cast<int64_t>(m) * AD + n) = make_float2(r0, r1);
      } else {
        const int64_t off = cache_off(g.block_table, g.page_shift, g.page_size, g.Kh, g.D, g.layer_base, pos,
                                      head - g.Aq);
        St<WT>::store_pair(static_cast<WT*>(g.kpool) + off + rl, r0, r1);
      }
    } else {
      const int j = n - AD - KD;
      const int head = j / g.D, d = j - head * g.D;
      const int64_t off = cache_off(g.block_table, g.page_shift, g.page_size, g.Kh, g.D, g.layer_base, pos, head);
      St<WT>::store_pair(static_cast<WT*>(g.vpool) + off + d, y0, y1);
    }
  }
}

template <typename WT, int EPI, int BM, int BN, int TM>
__global__ __launch_bounds__(256) void k_bp_gemm(GemmArgs g) {
  constexpr int TN = 4;
  constexpr int EPC = St<WT>::N;           // elements per 16-byte chunk
  constexpr int BK = 128 / sizeof(WT);     // one 128-byte line of a weight row per stage
  constexpr int CPR = BK / EPC;            // chunks per row per stage (8)
  constexpr int TX = BN / TN;              // threads along N
  static_assert((BM / TM) * TX == 256, "256 threads");
  constexpr int WCH = BN * CPR / 256;      // weight chunks per thread per stage
  constexpr int AQ = BM * BK / 4;          // float4 of A per stage
  constexpr int ACH = (AQ + 255) / 256;    // float4 per thread per stage
  constexpr int LW = BN + 4;               // LDS row strides (floats)
  constexpr int LA = BM + 4;
  __shared__ float Ws[BK * LW];
  __shared__ float As[BK * LA];
  __shared__ float ss_part[BM];
  __shared__ int last_flag;

  const int tid = threadIdx.x;
  const int tx = tid % TX, ty = tid / TX;
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM;
  const int split = blockIdx.z, splits = gridDim.z;
  const int kb = split * g.k_split, ke = min(g.K, kb + g.k_split);
  const WT* W = static_cast<const WT*>(g.W);

  uint4 wr[WCH];
  float4 ar[ACH];
  float ssq[ACH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) ssq[i] = 0.f;

  auto load_stage = [&](int k0) {
#pragma unroll
    for (int i = 0; i < WCH; ++i) {
      const int c = tid + 256 * i;
      const int r = c / CPR, q = c - r * CPR;
      const int n = n0 + r, k = k0 + q * EPC;
      wr[i] = (n < g.N && k < ke) ? *reinterpret_cast<const uint4*>(W + static_cast<int64_t>(n) * g.K + k)
                                  : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      const int c = tid + 256 * i;
      const int m = c / (BK / 4), q = c - m * (BK / 4);
      const int k = k0 + 4 * q;
      ar[i] = (c < AQ && m0 + m < g.P && k < ke)
                  ? *reinterpret_cast<const float4*>(g.A + static_cast<int64_t>(m0 + m) * g.K + k)
                  : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  auto store_stage = [&](int k0) {
#pragma unroll
    for (int i = 0; i < WCH; ++i) {
      const int c = tid + 256 * i;
      const int r = c / CPR, q = c - r * CPR;
      float f[EPC];
      St<WT>::unpack(wr[i], f);
#pragma unroll
      for (int e = 0; e < EPC; ++e) Ws[(q * EPC + e) * LW + r] = f[e];
    }
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      const int c = tid + 256 * i;
      if (c < AQ) {
        const int m = c / (BK / 4), q = c - m * (BK / 4);
        const int k = k0 + 4 * q;
        float4 a = ar[i];
        if (g.gain) {
          ssq[i] = fmaf(a.x, a.x, fmaf(a.y, a.y, fmaf(a.z, a.z, fmaf(a.w, a.w, ssq[i]))));
          if (k < ke) {
            const float4 gg = *reinterpret_cast<const float4*>(g.gain + k);
            a.x *= gg.x; a.y *= gg.y; a.z *= gg.z; a.w *= gg.w;
          }
        }
        As[(4 * q + 0) * LA + m] = a.x;
        As[(4 * q + 1) * LA + m] = a.y;
        As[(4 * q + 2) * LA + m] = a.z;
        As[(4 * q + 3) * LA + m] = a.w;
      }
    }
  };

  float acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;

  if (kb < ke) load_stage(kb);
  for (int k0 = kb; k0 < ke; k0 += BK) {
    __syncthreads();
    store_stage(k0);
    __syncthreads();
    if (k0 + BK < ke) load_stage(k0 + BK);
#pragma unroll 8
    for (int k = 0; k < BK; ++k) {
      float a[TM];
      if constexpr (TM == 4) {
        const float4 av = *reinterpret_cast<const float4*>(&As[k * LA + ty * TM]);
        a[0] = av.x; a[1] = av.y; a[2] = av.z; a[3] = av.w;
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = As[k * LA + ty * TM + i];
      }
      const float4 wv = *reinterpret_cast<const float4*>(&Ws[k * LW + tx * TN]);
      const float w[TN] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
    }
  }

  // per-row sums of squares of this K-slice: the BK/4 threads of a row are
  // consecutive lanes; the first of them holds the row's sum
  if (g.gain) {
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      float v = ssq[i];
#pragma unroll
      for (int o = 1; o < BK / 4; o <<= 1) v += __shfl_xor(v, o);
      const int c = tid + 256 * i;
      if (c < AQ && (c % (BK / 4)) == 0) ss_part[c / (BK / 4)] = v;
    }
  }
  __syncthreads();

  const int64_t PN = static_cast<int64_t>(g.P) * g.N;
  if (splits > 1) {
    // publish this slice's partial tile; the last arrival merges all slices
    float* part = g.part + split * PN;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + ty * TM + i;
      if (m >= g.P) continue;
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        const int n = n0 + tx * TN + j;
        if (n < g.N) st_agent2(part + static_cast<int64_t>(m) * g.N + n, acc[i][j], acc[i][j + 1]);
      }
    }
    if (g.gain && tid < BM && m0 + tid < g.P) st_agent(g.part + splits * PN + split * g.P + m0 + tid, ss_part[tid]);
    drain_stores();
    __syncthreads();
    if (tid == 0) {
      uint32_t* ctr = g.tile_ctr + blockIdx.y * gridDim.x + blockIdx.x;
      const uint32_t old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_flag = old == static_cast<uint32_t>(splits - 1);
      if (last_flag) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last_flag) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;
    // the slices' partial sums in slice order; each group of kSG slices has
    // all its loads in flight before the first is added
    constexpr int kSG = TM >= 4 ? 2 : 8;  // 16 pairs in flight per thread
    for (int s0 = 0; s0 < splits; s0 += kSG) {
      float2 v[kSG][TM][TN / 2];
#pragma unroll
      for (int u = 0; u < kSG; ++u) {
        const float* ps = g.part + (s0 + u) * PN;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int m = m0 + ty * TM + i;
#pragma unroll
          for (int j = 0; j < TN; j += 2) {
            const int n = n0 + tx * TN + j;
            v[u][i][j / 2] = (s0 + u < splits && m < g.P && n < g.N)
                                 ? ld_agent2(ps + static_cast<int64_t>(m) * g.N + n)
                                 : make_float2(0.f, 0.f);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kSG; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; j += 2) {
            acc[i][j] += v[u][i][j / 2].x;
            acc[i][j + 1] += v[u][i][j / 2].y;
          }
    }
    if (g.gain && tid < BM && m0 + tid < g.P) {
      float t = 0.f;
      for (int s0 = 0; s0 < splits; s0 += kSG) {
        float v[kSG];
#pragma unroll
        for (int u = 0; u < kSG; ++u)
          v[u] = s0 + u < splits ? ld_agent(g.part + splits * PN + (s0 + u) * g.P + m0 + tid) : 0.f;
#pragma unroll
        for (int u = 0; u < kSG; ++u) t += v[u];
      }
      ss_part[tid] = t;
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int ml = ty * TM + i, m = m0 + ml;
    if (m >= g.P) continue;
    const float rinv = g.gain ? rsqrtf(ss_part[ml] / static_cast<float>(g.K) + g.eps) : 1.f;
#pragma unroll
    for (int j = 0; j < TN; j += 2) {
      const int n = n0 + tx * TN + j;
      if (n < g.N) epi_pair<WT>(g, EPI, m, n, acc[i][j] * rinv, acc[i][j + 1] * rinv);
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 weights: the products of ee_mm.h, their epilogues, and what runs
// between them
// ---------------------------------------------------------------------------
// tiled copy of a row-major [N][K] matrix (K a multiple of 8), padded with zeros
__global__ __launch_bounds__(256) void k_bp_tile_weights(const uint16_t* __restrict__ W, int N, int K, int k32,
                                                         int64_t chunks, u32x4* __restrict__ T) {
  for (int64_t c = blockIdx.x * 256ll + threadIdx.x; c < chunks; c += gridDim.x * 256ll) {
    const int lane = static_cast<int>(c & 63);
    const int64_t t = c >> 6;
    const int64_t n = t / k32 * 16 + (lane & 15);
    const int k = static_cast<int>(t % k32) * 32 + 8 * (lane >> 4);
    T[c] = n < N && k < K ? *reinterpret_cast<const u32x4*>(W + n * K + k) : u32x4{0u, 0u, 0u, 0u};
  }
}

// What the store of rows n .. n + 3 (of one head, n a multiple of 4) of the
// repacked QKV matrix at position p reads: the rotations of the two RoPE
// pairs and the cache row.
struct QkvEpi {
  float2 c, s;
  int64_t off;
};
__device__ __forceinline__ QkvEpi qkv_epi(const GemmArgs& g, int p, int n) {
  const int AD = g.Aq * g.D, KD = g.Kh * g.D;
  const int pos = g.pos0 + p;
  QkvEpi e{make_float2(1.f, 1.f), make_float2(0.f, 0.f), 0};
  if (n < AD + KD) {
    const int64_t i = static_cast<int64_t>(pos) * (g.D >> 1) + ((n % g.D) >> 1);
    e.c = *reinterpret_cast<const float2*>(g.rope_cos + i);
    e.s = *reinterpret_cast<const float2*>(g.rope_sin + i);
  }
  if (n >= AD) {
    const int kvh = (n - AD) % KD / g.D;
    e.off = cache_off(g.block_table, g.page_shift, g.page_size, g.Kh, g.D, g.layer_base, pos, kvh) + (n - AD) % g.D;
  }
  return e;
}
__device__ __forceinline__ void qkv_store(const GemmArgs& g, const QkvEpi& e, int p, int n, const f32x4& y) {
  const int AD = g.Aq * g.D, KD = g.Kh * g.D;
  if (n >= AD + KD) {
    uint16_t* v = static_cast<uint16_t*>(g.vpool) + e.off;
    *reinterpret_cast<uint2*>(v) = make_uint2(St<uint16_t>::bits(y[0]) | (St<uint16_t>::bits(y[1]) << 16),
                                              St<uint16_t>::bits(y[2]) | (St<uint16_t>::bits(y[3]) << 16));
    return;
  }
  const float r0 = y[0] * e.c.x - y[1] * e.s.x, r1 = y[1] * e.c.x + y[0] * e.s.x;
  const float r2 = y[2] * e.c.y - y[3] * e.s.y, r3 = y[3] * e.c.y + y[2] * e.s.y;
  if (n < AD)
    *reinterpret_cast<f32x4*>(g.Y + static_cast<int64_t>(p) * AD + n) = f32x4{r0, r1, r2, r3};
  else
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(g.kpool) + e.off) =
        make_uint2(St<uint16_t>::bits(r0) | (St<uint16_t>::bits(r1) << 16),
                   St<uint16_t>::bits(r2) | (St<uint16_t>::bits(r3) << 16));
}

// Epilogue targets of a product on the matrix cores (GemmArgs, with kEpiResid
// storing its K slices' partial sums in g.part [split][P][N] for
// k_bp_reduce_norm, and kEpiSwiGlu storing term planes).
template <int EPI, int RB, int CP, int NW, int PF, int KG>
__global__ __launch_bounds__(64 * NW * KG) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_bp_mm(MmArgs m, GemmArgs g) {
  if constexpr (EPI == kEpiQkv) {
    mm_tile<RB, CP, NW, PF, KG>(
        m, [&](int p, int n) { return qkv_epi(g, p, n); },
        [&](int, int p, int n, const f32x4& y, const QkvEpi& e) { qkv_store(g, e, p, n, y); });
  } else {
    mm_tile<RB, CP, NW, PF, KG>(
        m, [](int, int) { return 0; },
        [&](int split, int p, int n, const f32x4& y, int) {
          if constexpr (EPI == kEpiResid) {
            *reinterpret_cast<f32x4*>(g.part + (static_cast<int64_t>(split) * m.P + p) * m.N + n) = y;
          } else {
            // interleaved rows: n = 2j gate row j, n + 1 up row j
            const float a0 = y[0] / (1.f + exp_hw(-y[0])) * y[1];
            const float a1 = y[2] / (1.f + exp_hw(-y[2])) * y[3];
            const int j = n >> 1;
            uint32_t t[3];
            mm_split2(a0, a1, t);
#pragma unroll
            for (int i = 0; i < 3; ++i)
              *(reinterpret_cast<uint32_t*>(g.planes + mm_chunk(p, j & ~7, i, g.k32_out)) + ((j & 7) >> 1)) = t[i];
          }
        });
  }
}

// The residual stream after a product, and the input of the next: X += the
// product's K slices in slice order (splits may be 0), then, with a gain,
// the term planes of x * rsqrt(mean(x^2) + eps) * gain. One workgroup per
// position, thread = 8 elements (H <= 2048). The 16 positions of a block of
// planes go to workgroups of one XCD, whose L2 then merges their 16-byte
// pieces into whole lines. Bound by the reads of the slices.
constexpr int kNormThreads = 256;
__global__ __launch_bounds__(kNormThreads) void k_bp_reduce_norm(float* __restrict__ X, const float* __restrict__ part,
                                                                 int splits, int P, int H,
                                                                 const float* __restrict__ gain, float eps,
                                                                 u32x4* __restrict__ planes, int k32) {
  __shared__ float red[kNormThreads / 64];
  const int b = blockIdx.x, loc = b >> 3;
  const int p = ((loc >> 4) * 8 + (b & 7)) * 16 + (loc & 15);
  if (p >= P) return;
  const int k = 8 * threadIdx.x;
  const bool on = k < H;
  f32x4 x[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}, gv[2];
  f32x4* xp = reinterpret_cast<f32x4*>(X + static_cast<int64_t>(p) * H + k);
  if (on) {
    x[0] = xp[0];
    x[1] = xp[1];
    if (gain) {
      gv[0] = reinterpret_cast<const f32x4*>(gain + k)[0];
      gv[1] = reinterpret_cast<const f32x4*>(gain + k)[1];
    }
    // the slices' sum first, then the residual: groups of kSG slices with
    // every load of a group in flight
    if (splits > 0) {
      constexpr int kSG = 8;
      f32x4 y[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
      const int64_t PH = static_cast<int64_t>(P) * H;
      const float* q = part + static_cast<int64_t>(p) * H + k;
      for (int s0 = 0; s0 < splits; s0 += kSG) {
        f32x4 v[kSG][2];
#pragma unroll
        for (int u = 0; u < kSG; ++u) {
          const f32x4* r = reinterpret_cast<const f32x4*>(q + min(s0 + u, splits - 1) * PH);
          v[u][0] = r[0];
          v[u][1] = r[1];
        }
#pragma unroll
        for (int u = 0; u < kSG; ++u)
          if (s0 + u < splits) {
            y[0] += v[u][0];
            y[1] += v[u][1];
          }
      }
      x[0] += y[0];
      x[1] += y[1];
      xp[0] = x[0];
      xp[1] = x[1];
    }
  }
  if (!gain) return;
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) ss = fmaf(x[i >> 2][i & 3], x[i >> 2][i & 3], ss);
  ss = wave_sum64(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < kNormThreads / 64; ++w) t += red[w];
  const float r = rsqrtf(t / static_cast<float>(H) + eps);
  if (!on) return;
  uint32_t w[4][3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = 2 * i;
    mm_split2(x[e >> 2][e & 3] * r * gv[e >> 2][e & 3], x[e >> 2][(e & 3) + 1] * r * gv[e >> 2][(e & 3) + 1], w[i]);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) planes[mm_chunk(p, k, i, k32)] = u32x4{w[0][i], w[1][i], w[2][i], w[3][i]};
}

// ---------------------------------------------------------------------------
// causal grouped-query attention of a chunk of queries (positions pos0 ..
// pos0 + P - 1) over the cache. Block = (KV head, tile of 4 query
// positions, key split); its waves split the tile's queries and the KV
// head's query heads; keys in tiles of 64 staged in LDS, lane j = key j of
// the tile; online softmax per head. One split writes o directly; several
// write partial records (weighted V, max, sum) merged in split order by
// k_bp_attn_merge.
// ---------------------------------------------------------------------------
struct AttnArgs {
  const float* Q;      // [P][A*D], pair-interleaved within heads (as the cached keys)
  float* O;            // [P][A*D], natural order (fp32 weights), or
  u32x4* planes;       // its term planes (bf16 weights), k32 K blocks
  int k32;
  float* part;         // [P][A][nsplit][D + 2]
  const void* kpool;
  const void* vpool;
  int64_t layer_base;
  const int32_t* block_table;
  int page_shift, page_size;
  int P, pos0, A, K, G, D;
  int nsplit, keys_per_split;
  float scale;
};

constexpr int kKT = 64;  // keys per LDS tile

// DPL neighbouring elements (element e of query qi, e even for DPL = 2) of the attention output
template <typename WT, int DPL>
__device__ __forceinline__ void attn_store(const AttnArgs& a, int qi, int e, const float (&o)[DPL]) {
  if constexpr (sizeof(WT) == 4) {
#pragma unroll
    for (int i = 0; i < DPL; ++i) a.O[static_cast<int64_t>(qi) * a.A * a.D + e + i] = o[i];
  } else {
    uint32_t t[3];
    mm_split2(o[0], DPL == 2 ? o[DPL - 1] : 0.f, t);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      uint16_t* c = reinterpret_cast<uint16_t*>(a.planes + mm_chunk(qi, e & ~7, i, a.k32)) + (e & 7);
      if constexpr (DPL == 2) *reinterpret_cast<uint32_t*>(c) = t[i];
      else *c = static_cast<uint16_t>(t[i]);
    }
  }
}

// Block = (KV head, tile of QT query positions, key split); wave w takes
// query position w % QT and the GW query heads (w / QT) GW .. + GW - 1 of the
// KV head. With many blocks (a prompt) QT = 4 and each wave takes all G heads
// (more waves would read each key tile from LDS once per wave), at most two
// workgroups per compute unit (as LDS allows), so each wave may hold up to
// 256 registers; with few blocks (a refresh) QT = 2 and one head per wave,
// so that the G heads' dot products run on G waves per position. The first
// four waves stage each key tile in LDS.
// (fp32 caches of wide heads may need more registers: their lower bound is 1)
template <typename WT, int D, int G, int GW, int QT>
__global__ __launch_bounds__(64 * QT * (G / GW))
__attribute__((amdgpu_waves_per_eu(sizeof(WT) == 4 ? 1 : ((QT * (G / GW) + 3) / 4 > 2 ? (QT * (G / GW) + 3) / 4 : 2),
                                   (QT * (G / GW) + 3) / 4 > 2 ? (QT * (G / GW) + 3) / 4 : 2))) void k_bp_attn(AttnArgs a) {
  static_assert(G % GW == 0, "head groups cover the KV head's query heads");
  static_assert(QT * (G / GW) >= 4, "four waves stage the key tiles");
  constexpr int kQT = QT;
  constexpr int EPC = St<WT>::N;
  constexpr int CPK = D / EPC;          // 16-byte chunks per cache row
  constexpr int DPL = D / 64;           // output dimensions per lane (1 or 2)
  constexpr int KST = CPK + 1;          // key rows padded by one chunk: lane j reads row j
  __shared__ uint4 Ks[kKT * KST];
  __shared__ uint4 Vs[kKT * CPK];
  __shared__ float Qs[kQT][G][D];
  __shared__ float Ps[kQT][G][kKT];

  constexpr int HG = G / GW;            // waves per query position
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int qw = HG > 1 ? wave % kQT : wave, h0 = HG > 1 ? (wave / kQT) * GW : 0;
  const bool loader = HG > 1 ? tid < 256 : true;  // the threads that stage key tiles
  const int nqt = (a.P + kQT - 1) / kQT;
  const int item = blockIdx.x;
  const int kvh = item / (nqt * a.nsplit);
  const int rem = item - kvh * nqt * a.nsplit;
  const int qt = rem / a.nsplit, sp = rem - qt * a.nsplit;
  const int qi = qt * kQT + qw;                 // query index within the chunk
  const bool active = qi < a.P;
  const int qpos = a.pos0 + qi;                 // its position
  const int t_end = a.pos0 + min(a.P, (qt + 1) * kQT);  // keys needed by the tile: [0, t_end)
  const int kb = sp * a.keys_per_split;
  const int ke = min(t_end, kb + a.keys_per_split);

  constexpr int CPT = kKT * CPK / 256;  // chunks of K (and of V) per loading thread per tile
  // cache offsets of a tile's chunks (its page lookups)
  auto offsets = [&](int k0, int64_t (&off)[CPT]) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + 256 * i;
      const int j = c / CPK, q = c - j * CPK;
      const int key = min(k0 + j, ke - 1);
      off[i] = cache_off(a.block_table, a.page_shift, a.page_size, a.K, D, a.layer_base, key, kvh) + q * EPC;
    }
  };
  // the wave's query rows (its GW heads) and the first tile's page lookups,
  // every load in flight at once
  int64_t off[CPT];
  if (loader && kb < ke) offsets(kb, off);
  {
    constexpr int QPL = GW * D / 64;
    float qv[QPL];
#pragma unroll
    for (int u = 0; u < QPL; ++u) {
      const int i = lane + 64 * u, h = h0 + i / D, d = i % D;
      qv[u] = active ? a.Q[static_cast<int64_t>(qi) * a.A * D + (kvh * G + h) * D + d] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < QPL; ++u) {
      const int i = lane + 64 * u, h = h0 + i / D, d = i % D;
      Qs[qw][h][d] = qv[u];
    }
  }
  float m_run[GW], l_run[GW], acc[GW][DPL];
#pragma unroll
  for (int h = 0; h < GW; ++h) {
    m_run[h] = -INFINITY;
    l_run[h] = 0.f;
#pragma unroll
    for (int e = 0; e < DPL; ++e) acc[h][e] = 0.f;
  }
  const WT* kp = static_cast<const WT*>(a.kpool);
  const WT* vp = static_cast<const WT*>(a.vpool);

  for (int k0 = kb; k0 < ke; k0 += kKT) {
    // native vectors: a copy of the uint4 struct from global memory to LDS
    // through registers compiles to memory-to-memory copies through private
    // memory, which serialise the loads
    u32x4 kv[CPT], vv[CPT];
    if (loader) {
      if (k0 != kb) offsets(k0, off);
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        kv[i] = *reinterpret_cast<const u32x4*>(kp + off[i]);
        vv[i] = *reinterpret_cast<const u32x4*>(vp + off[i]);
      }
    }
    __syncthreads();  // previous tile consumed (and Qs written before the first)
    if (loader) {
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const int c = tid + 256 * i;
        const int j = c / CPK, q = c - j * CPK;
        *reinterpret_cast<u32x4*>(&Ks[j * KST + q]) = kv[i];  // keys past ke repeat key ke - 1; masked
        *reinterpret_cast<u32x4*>(&Vs[c]) = vv[i];
      }
    }
    __syncthreads();
    const int key = k0 + lane;
    const bool valid = active && key < ke && key <= qpos;
    float s[GW];
#pragma unroll
    for (int h = 0; h < GW; ++h) s[h] = 0.f;
#pragma unroll 2
    for (int q = 0; q < CPK; ++q) {
      float kf[EPC];
      St<WT>::unpack(Ks[lane * KST + q], kf);
#pragma unroll
      for (int h = 0; h < GW; ++h) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) s[h] = fmaf(Qs[qw][h0 + h][q * EPC + e], kf[e], s[h]);
      }
    }
#pragma unroll
    for (int h = 0; h < GW; ++h) {
      const float sv = valid ? s[h] * a.scale : -INFINITY;
      const float mt = wave_max64(sv);
      const float mn = fmaxf(m_run[h], mt);
      float p = 0.f, alpha = 1.f;
      if (mn != -INFINITY) {
        p = exp_hw(sv - mn);  // 0 for masked keys
        alpha = exp_hw(m_run[h] - mn);
      }
      l_run[h] = l_run[h] * alpha + wave_sum64(p);
      m_run[h] = mn;
#pragma unroll
      for (int e = 0; e < DPL; ++e) acc[h][e] *= alpha;
      Ps[qw][h0 + h][lane] = p;
    }
    __builtin_amdgcn_wave_barrier();
    // weighted values: lane owns dimensions DPL * lane .. + DPL - 1
#pragma unroll 4
    for (int j = 0; j < kKT; ++j) {
      float v[DPL];
      if constexpr (DPL == 2) {
        const float2 vv2 = St<WT>::load_pair(reinterpret_cast<const WT*>(&Vs[j * CPK]) + 2 * lane);
        v[0] = vv2.x;
        v[1] = vv2.y;
      } else {
        const WT* vr = reinterpret_cast<const WT*>(&Vs[j * CPK]);
        if constexpr (sizeof(WT) == 2) v[0] = __uint_as_float(static_cast<uint32_t>(vr[lane]) << 16);
        else v[0] = vr[lane];
      }
#pragma unroll
      for (int h = 0; h < GW; ++h) {
        const float pj = Ps[qw][h0 + h][j];
#pragma unroll
        for (int e = 0; e < DPL; ++e) acc[h][e] = fmaf(pj, v[e], acc[h][e]);
      }
    }
  }
  if (!active) return;
#pragma unroll
  for (int h = 0; h < GW; ++h) {
    const int head = kvh * G + h0 + h;
    if (a.nsplit == 1) {
      const float inv = 1.f / l_run[h];
#pragma unroll
      for (int e = 0; e < DPL; ++e) acc[h][e] *= inv;
      attn_store<WT, DPL>(a, qi, head * D + DPL * lane, acc[h]);
    } else {
      float* r = a.part + ((static_cast<int64_t>(qi) * a.A + head) * a.nsplit + sp) * (D + 2);
#pragma unroll
      for (int e = 0; e < DPL; ++e) r[DPL * lane + e] = acc[h][e];
      if (lane == 0) {
        r[D] = m_run[h];
        r[D + 1] = l_run[h];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same attention on the matrix cores, for bf16 caches. Workgroup = (KV
// head, QB blocks of 16 query positions, key split); wave = (one of the KV
// head's G query heads, one block of 16 positions), so that all G heads share
// the key and value tiles staged in LDS. Per tile of 64 keys a wave computes
// S^T = K Q^T (rows keys, columns positions) and O^T += V^T P^T: a lane then
// holds one position's scores for 16 keys, the softmax needs two exchanges
// between lanes, the scores' layout is already the second product's operand
// (the key order of its K slots is permuted alike on both sides), and the
// output's layout that of the term planes. Values are read transposed from
// LDS (ds_read_b64_tr_b16). Keys and values are exact bf16 operands; queries
// and probabilities are split exactly into three bf16 terms, so both products
// carry fp32 accumulation error only.
// A tile is 96 MFMAs (1536 cycles) per wave at D = 128 and about as much
// vector work (exponentials, the split of the probabilities), which other
// waves overlap. The vector-ALU form above is bound by its FMAs and serial
// LDS reads: 1024 queries over 1024 to 8192 keys (six heads of 128 per KV
// head) took 595 us a layer on average, this 104 (172 for the last 1024, 840
// TFLOP/s of term products); 512 queries over 512 keys 47 us, this 24 in one
// pass over the keys and less with key splits.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float max_groups(float v) {  // over the four 16-lane groups
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_groups(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int D, int G, int QB>
__global__ __launch_bounds__(64 * G * QB) __attribute__((amdgpu_waves_per_eu(2))) void k_bp_attn_mfma(AttnArgs a) {
  constexpr int NT = 64 * G * QB;
  constexpr int CPK = D / 8;        // 16-byte chunks per cache row
  constexpr int KST = CPK + 1;      // padded LDS rows: 16 lanes reading a column of 16 rows, and the
  constexpr int VST = CPK + 2;      // transposed reads of 4 rows x 32 bytes, each touch every bank once
  constexpr int KS = D / 32, DB = D / 16;
  constexpr int CPT = (kKT * CPK + NT - 1) / NT;  // chunks of K (and of V) per thread per tile
  __shared__ u32x4 Ks[kKT * KST];
  __shared__ u32x4 Vs[kKT * VST];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4, lr = lane & 15;
  const int h = wave % G, qb = wave / G;
  const int nqt = (a.P + 16 * QB - 1) / (16 * QB);
  // the last query tiles, which have the most keys, go first
  const int item = blockIdx.x;
  const int sp = item % a.nsplit, r1 = item / a.nsplit;
  const int kvh = r1 % a.K, qt = nqt - 1 - r1 / a.K;
  const int q0 = (qt * QB + qb) * 16;           // the wave's first query
  const int qi = q0 + lr, qpos = a.pos0 + qi;   // the lane's query and its position
  const int head = kvh * G + h;
  const int t_end = a.pos0 + min(a.P, (qt + 1) * QB * 16);  // keys needed by the tile: [0, t_end)
  const int kb = sp * a.keys_per_split;
  const int ke = min(t_end, kb + a.keys_per_split);

  auto offset = [&](int k0, int c) {
    const int j = c / CPK, q = c - j * CPK;
    return cache_off(a.block_table, a.page_shift, a.page_size, a.K, D, a.layer_base, min(k0 + j, ke - 1), kvh) + q * 8;
  };
  const uint16_t* kp = static_cast<const uint16_t*>(a.kpool);
  const uint16_t* vp = static_cast<const uint16_t*>(a.vpool);
  u32x4 kv[CPT], vv[CPT];
  auto load_tile = [&](int k0) {  // keys past ke repeat key ke - 1; their scores are masked
    int64_t off[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) off[i] = offset(k0, min(tid + NT * i, kKT * CPK - 1));
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      kv[i] = *reinterpret_cast<const u32x4*>(kp + off[i]);
      vv[i] = *reinterpret_cast<const u32x4*>(vp + off[i]);
    }
  };
  if (kb < ke) load_tile(kb);

  // the query's terms: k slots 8 lg .. + 7 of each 32 dimensions
  bf16x8 qf[KS][3];
  {
    const float* q = a.Q + static_cast<int64_t>(min(qi, a.P - 1)) * a.A * D + head * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(q + 32 * s + 8 * lg);
      const f32x4 x1 = *reinterpret_cast<const f32x4*>(q + 32 * s + 8 * lg + 4);
      uint32_t w[4][3];
      mm_split2(x0[0], x0[1], w[0]);
      mm_split2(x0[2], x0[3], w[1]);
      mm_split2(x1[0], x1[1], w[2]);
      mm_split2(x1[2], x1[3], w[3]);
#pragma unroll
      for (int t = 0; t < 3; ++t) qf[s][t] = __builtin_bit_cast(bf16x8, u32x4{w[0][t], w[1][t], w[2][t], w[3][t]});
    }
  }
  const float scale2 = a.scale * 1.44269504088896341f;  // scores in units of log2
  float m = -INFINITY, l = 0.f;  // running maximum of the query, the lane's share of the sum
  f32x4 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = kb; k0 < ke; k0 += kKT) {
    __syncthreads();  // the previous tile is consumed
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + NT * i;
      if (kKT * CPK % NT == 0 || c < kKT * CPK) {
        const int j = c / CPK, q = c - j * CPK;
        Ks[j * KST + q] = kv[i];
        Vs[j * VST + q] = vv[i];
      }
    }
    __syncthreads();
    if (k0 + kKT < ke) load_tile(k0 + kKT);
    if (k0 > a.pos0 + q0 + 15) continue;  // every key of the tile is past the wave's queries
    // scores: block b holds keys k0 + 16 b + 4 lg + 0..3 of the lane's query
    f32x4 s[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 kf[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) kf[b] = __builtin_bit_cast(bf16x8, Ks[(16 * b + lr) * KST + 4 * ks + lg]);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int b = 0; b < 4; ++b) s[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[b], qf[ks][t], s[b], 0, 0, 0);
    }
    if (k0 + kKT > min(ke, a.pos0 + q0 + 1)) {  // some key of the tile is past the split or a query
      const int last = min(ke - 1, qpos);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + 16 * b + 4 * lg + i > last) s[b][i] = -INFINITY;
    }
    float mt = s[0][0];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) mt = fmaxf(mt, s[b][i]);
    const float mn = fmaxf(m, max_groups(mt) * scale2);
    const float ms = mn == -INFINITY ? 0.f : mn;  // no key yet: every exponential is zero
    const float alpha = __builtin_amdgcn_exp2f(m - ms);
    m = mn;
    l *= alpha;
    // probabilities, split: operand word of keys (i, i + 1) of block b: [2 (b & 1) + i / 2] of K slots b / 2
    uint32_t pw[2][4][3];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[b][i], scale2, -ms));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[b][i + 1], scale2, -ms));
        l += p0 + p1;
        mm_split2(p0, p1, pw[b >> 1][2 * (b & 1) + (i >> 1)]);
      }
#pragma unroll
    for (int d = 0; d < DB; ++d) o[d] *= alpha;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 vf[DB];
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        // 16 lanes read keys 4 lg .. + 3 (of block 2 ks, then 2 ks + 1) x dimensions 16 d .. + 15; lane lr
        // receives dimension 16 d + lr of the four keys
        s16x4 v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int key = 32 * ks + 16 * u + 4 * lg + (lr >> 2);
          const uint16_t* src = reinterpret_cast<const uint16_t*>(&Vs[key * VST]) + 16 * d + 4 * (lr & 3);
          v[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
        }
        vf[d] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const bf16x8 pf =
            __builtin_bit_cast(bf16x8, u32x4{pw[ks][0][t], pw[ks][1][t], pw[ks][2][t], pw[ks][3][t]});
#pragma unroll
        for (int d = 0; d < DB; ++d) o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[d], pf, o[d], 0, 0, 0);
      }
    }
  }
  const float lsum = sum_groups(l);
  if (qi >= a.P) return;
  if (a.nsplit == 1) {
    const float inv = 1.f / lsum;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const int e = head * D + 16 * d + 4 * lg;
      uint32_t w[2][3];
      mm_split2(o[d][0] * inv, o[d][1] * inv, w[0]);
      mm_split2(o[d][2] * inv, o[d][3] * inv, w[1]);
#pragma unroll
      for (int t = 0; t < 3; ++t)
        *(reinterpret_cast<uint2*>(a.planes + mm_chunk(qi, e & ~7, t, a.k32)) + ((e & 7) >> 2)) =
            make_uint2(w[0][t], w[1][t]);
    }
  } else {
    float* r = a.part + ((static_cast<int64_t>(qi) * a.A + head) * a.nsplit + sp) * (D + 2);
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      *reinterpret_cast<float2*>(r + 16 * d + 4 * lg) = make_float2(o[d][0], o[d][1]);
      *reinterpret_cast<float2*>(r + 16 * d + 4 * lg + 2) = make_float2(o[d][2], o[d][3]);
    }
    if (lg == 0) *reinterpret_cast<float2*>(r + D) = make_float2(m, lsum);
  }
}

// one wave per (query, head): the splits' partial records in split order
// (maxima in units of log2 with bf16 caches, of e with fp32 caches)
template <typename WT, int D>
__global__ __launch_bounds__(256) void k_bp_attn_merge(AttnArgs a) {
  constexpr int DPL = D / 64;
  auto ex = [](float x) { return sizeof(WT) == 2 ? __builtin_amdgcn_exp2f(x) : exp_hw(x); };
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= a.P * a.A) return;
  const float* r = a.part + static_cast<int64_t>(w) * a.nsplit * (D + 2);
  float M = -INFINITY;
  float den = 0.f, num[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) num[e] = 0.f;
  // groups of 8 splits: every record of a group requested before any is used
  constexpr int kSG = 8;
  for (int s0 = 0; s0 < a.nsplit; s0 += kSG) {
    float ms[kSG], ls[kSG], vs[kSG][DPL];
#pragma unroll
    for (int u = 0; u < kSG; ++u) {
      const bool ok = s0 + u < a.nsplit;
      const float* q = r + (s0 + u) * (D + 2);
      ms[u] = ok ? q[D] : -INFINITY;
      ls[u] = ok ? q[D + 1] : 0.f;
#pragma unroll
      for (int e = 0; e < DPL; ++e) vs[u][e] = ok ? q[DPL * lane + e] : 0.f;
    }
    // running maximum over the splits so far, in split order
    float cm = M;
#pragma unroll
    for (int u = 0; u < kSG; ++u) cm = fmaxf(cm, ms[u]);
    if (cm != -INFINITY) {
      const float sc = ex(M - cm);  // 0 while nothing has been merged
      den *= sc;
#pragma unroll
      for (int e = 0; e < DPL; ++e) num[e] *= sc;
#pragma unroll
      for (int u = 0; u < kSG; ++u) {
        if (ms[u] == -INFINITY) continue;  // absent, or a split wholly past the query's position
        const float f = ex(ms[u] - cm);
        den = fmaf(f, ls[u], den);
#pragma unroll
        for (int e = 0; e < DPL; ++e) num[e] = fmaf(f, vs[u][e], num[e]);
      }
      M = cm;
    }
  }
  const int qi = w / a.A, head = w - qi * a.A;
  const float inv = 1.f / den;
#pragma unroll
  for (int e = 0; e < DPL; ++e) num[e] *= inv;
  attn_store<WT, DPL>(a, qi, head * D + DPL * lane, num);
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------
namespace {

// Splits of K so that the grid holds at least ~2 workgroups per compute unit,
// bounded by the partial workspace and by one stage per split.
void choose_split(int tiles, int P, int N, int K, int BK, size_t ws_floats, int wgs_per_cu, int n_cu, int* k_split,
                  int* splits, int max_k_split = 1 << 30) {
  // enough workgroups per compute unit (wgs_per_cu) that their weight loads
  // in flight together cover the memory latency; at most 32 slices, and
  // slices of at most max_k_split
  int s = std::max(1, (wgs_per_cu * n_cu + tiles - 1) / tiles);
  s = std::max(s, (K + max_k_split - 1) / max_k_split);
  s = std::min({s, (K + BK - 1) / BK, 32});
  const size_t per = static_cast<size_t>(P) * N + P;
  if (per > 0) s = static_cast<int>(std::min<size_t>(s, std::max<size_t>(1, ws_floats / per)));
  if (s <= 1) {
    *k_split = K;
    *splits = 1;
    return;
  }
  int ks = (K + s - 1) / s;
  ks = (ks + BK - 1) / BK * BK;
  *k_split = ks;
  *splits = (K + ks - 1) / ks;
}

// fp32 weights
template <typename WT, int EPI>
hipError_t gemm(const GemmArgs& g0, const BatchBuffers& b, int n_cu, hipStream_t s) {
  GemmArgs g = g0;
  constexpr int BK = 128 / sizeof(WT);
  if (g.P <= 16) {
    // few positions: narrow tiles (16 positions x 64 rows, one position and
    // four rows per thread) so that few K-slices fill the device and the
    // merge of a tile's slices stays short
    constexpr int BM = 16, BN = 64, TM = 1;
    const int tiles = ((g.N + BN - 1) / BN) * ((g.P + BM - 1) / BM);
    int splits;
    // a tile of 16 positions does little arithmetic per weight byte: many
    // short K-slices, so that loads of several workgroups per unit overlap
    choose_split(tiles, g.P, g.N, g.K, BK, b.gemm_ws_floats, 8, n_cu, &g.k_split, &splits);
    if (static_cast<size_t>(tiles) > b.n_tile_ctr) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_bp_gemm<WT, EPI, BM, BN, TM>), dim3((g.N + BN - 1) / BN, (g.P + BM - 1) / BM, splits),
                       dim3(256), 0, s, g);
  } else {
    constexpr int BM = 64, BN = 64, TM = 4;
    const int tiles = ((g.N + BN - 1) / BN) * ((g.P + BM - 1) / BM);
    int splits;
    choose_split(tiles, g.P, g.N, g.K, BK, b.gemm_ws_floats, 2, n_cu, &g.k_split, &splits);
    if (static_cast<size_t>(tiles) > b.n_tile_ctr) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_bp_gemm<WT, EPI, BM, BN, TM>), dim3((g.N + BN - 1) / BN, (g.P + BM - 1) / BM, splits),
                       dim3(256), 0, s, g);
  }
  return hipGetLastError();
}

// bf16 weights: the tile and K split of a product. Every candidate's time is
// estimated (microseconds; constants fitted to a sweep of tiles and splits
// over the products of three decoder widths, 16 to 1024 positions, where the
// choice costs 1.7% over the best on average):
//   * a unit runs the tile's workgroups in rounds of `occ` (what registers
//     and LDS allow); a step of a round takes the matrix-core time of its
//     workgroups or, if longer, the latency of one workgroup's step;
//   * no less than the weights' read from HBM, nor than the tiles' reads of
//     weights and activations from the caches;
//   * the stores of the outputs, and for the residual products the next
//     kernel's reads of the K slices.
struct MmTile {
  int rb, cp, nw, pf, kg, occ;
};
double mm_time(const MmTile& t, int P, int N, int K, int splits, bool resid, int n_cu) {
  const double mfma = 0.02127 * t.rb * t.cp * t.nw * t.kg;
  const double lat = (t.pf == 1 ? 0.733 : 0.262) + 0.377 * mfma / t.kg;
  const int tiles = ((N + 16 * t.rb * t.nw - 1) / (16 * t.rb * t.nw)) * ((P + 16 * t.cp - 1) / (16 * t.cp)) * splits;
  const int per_cu = (tiles + n_cu - 1) / n_cu, full = per_cu / t.occ, rest = per_cu % t.occ;
  const int steps = ((K + 63) / 64 + splits * t.kg - 1) / (splits * t.kg);
  const double round = full * std::max(t.occ * mfma, lat) + (rest ? std::max(rest * mfma, lat) : 0.0);
  const double bytes = 2.0 * N * K * ((P + 16 * t.cp - 1) / (16 * t.cp)) +
                       6.0 * P * K * ((N + 16 * t.rb * t.nw - 1) / (16 * t.rb * t.nw));
  const double out = 4.0 * splits * P * N;
  return 3.2 + std::max({round * steps, 2.0 * N * K / 5.8e6, bytes / 14.8e6}) + out / 8.5e6 + (resid ? out / 5e6 : 0.0);
}

template <int EPI, int RB, int CP, int NW, int PF, int KG>
hipError_t mm_launch(MmArgs m, const GemmArgs& g, int splits, hipStream_t s) {
  const int steps = m.k32 / 2;
  m.nN = (m.NB + RB * NW - 1) / (RB * NW);
  m.nP = (m.PB + CP - 1) / CP;
  m.steps_per_split = (steps + splits - 1) / splits;
  m.splits = (steps + m.steps_per_split - 1) / m.steps_per_split;
  const int tiles = m.nN * m.nP * m.splits;
  m.tiles_per_xcd = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_bp_mm<EPI, RB, CP, NW, PF, KG>), dim3(m.tiles_per_xcd * 8), dim3(64 * NW * KG), 0, s, m, g);
  return hipGetLastError();
}

// g: as for gemm(), with A, W unused; T the tiled weights, X the input's
// term planes. *splits receives the K slices that a residual product stored.
template <int EPI>
hipError_t gemm_mm(const GemmArgs& g, const void* T, const u32x4* X, const BatchBuffers& b, int n_cu, int* splits,
                   hipStream_t s) {
  constexpr bool kResid = EPI == kEpiResid;
  // 16 positions: the weight stream counts, four steps of it in flight. More
  // positions: 32 to 64 per workgroup. Eight waves of three row blocks share
  // the activations of 64 positions among 384 rows, the fewest cache reads.
  // The QKV product of few positions has few tiles and whole sums to finish:
  // four groups of waves share a tile's K.
  static constexpr MmTile kTiles[] = {{1, 1, 8, 4, 1, 3}, {1, 2, 4, 4, 1, 3}, {2, 2, 4, 2, 1, 4}, {3, 2, 4, 2, 1, 3},
                                      {4, 2, 4, 2, 1, 2}, {3, 3, 4, 2, 1, 2}, {3, 4, 4, 1, 1, 2}, {3, 4, 8, 1, 1, 1},
                                      {2, 4, 8, 1, 1, 1}, {1, 1, 2, 2, 4, 2}, {1, 2, 2, 2, 4, 1}};
  MmArgs m{};
  m.W = static_cast<const u32x4*>(T);
  m.X = X;
  m.P = g.P;
  m.N = g.N;
  m.NB = (g.N + 15) / 16;
  m.PB = (g.P + 15) / 16;
  m.k32 = mm_k32(g.K);
  const int steps = m.k32 / 2;
  int most = 1;
  if (kResid) {
    const size_t per = static_cast<size_t>(g.P) * g.N;
    most = static_cast<int>(std::min<size_t>(16, b.gemm_ws_floats / per));
    if (most < 1) return hipErrorInvalidValue;
  }
  int best = -1, best_s = 1;
  double best_t = 0.0;
  for (int i = 0; i < static_cast<int>(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
    const MmTile& t = kTiles[i];
    if ((t.cp == 1) != (g.P <= 16) || (t.cp == 3 && g.P > 256) || (t.kg > 1 && EPI != kEpiQkv)) continue;
    for (int sp : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16}) {
      if (sp > most || (sp > 1 && steps / sp < 4) || (t.kg > 1 && steps < 2 * t.kg)) break;
      const double us = mm_time(t, g.P, g.N, g.K, sp, kResid, n_cu);
      if (best < 0 || us < best_t) {
        best = i;
        best_s = sp;
        best_t = us;
      }
    }
  }
  if (splits) {
    const int per = (steps + best_s - 1) / best_s;
    *splits = (steps + per - 1) / per;
  }
  switch (best) {
    case 0: return mm_launch<EPI, 1, 1, 8, 4, 1>(m, g, best_s, s);
    case 1: return mm_launch<EPI, 1, 2, 4, 4, 1>(m, g, best_s, s);
    case 2: return mm_launch<EPI, 2, 2, 4, 2, 1>(m, g, best_s, s);
    case 3: return mm_launch<EPI, 3, 2, 4, 2, 1>(m, g, best_s, s);
    case 4: return mm_launch<EPI, 4, 2, 4, 2, 1>(m, g, best_s, s);
    case 5: return mm_launch<EPI, 3, 3, 4, 2, 1>(m, g, best_s, s);
    case 6: return mm_launch<EPI, 3, 4, 4, 1, 1>(m, g, best_s, s);
    case 7: return mm_launch<EPI, 3, 4, 8, 1, 1>(m, g, best_s, s);
    case 8: return mm_launch<EPI, 2, 4, 8, 1, 1>(m, g, best_s, s);
    case 9:
      if constexpr (EPI == kEpiQkv) return mm_launch<EPI, 1, 1, 2, 2, 4>(m, g, best_s, s);
      break;
    case 10:
      if constexpr (EPI == kEpiQkv) return mm_launch<EPI, 1, 2, 2, 2, 4>(m, g, best_s, s);
      break;
  }
  return hipErrorInvalidValue;
}

hipError_t reduce_norm(const BatchBuffers& b, float* X, int splits, int P, int H, const float* gain, float eps, hipStream_t s) {
  if (H > 8 * kNormThreads) return hipErrorInvalidValue;
  const int blocks = (P + 127) / 128 * 128;  // whole groups of 16 positions on each of the 8 XCDs
  hipLaunchKernelGGL(k_bp_reduce_norm, dim3(blocks), dim3(kNormThreads), 0, s, X, b.gemm_ws, splits, P, H, gain, eps,
                     static_cast<u32x4*>(b.Xp), mm_k32(H));
  return hipGetLastError();
}

// Key splits for blocks whose longest has key_tiles tiles: units run two
// workgroups at a time, a tile takes ~2.8 us (the same for one workgroup and
// for two side by side), splits add the merging launch (4.5 us) and their
// records' stores and loads.
template <int D>
hipError_t attention_mfma(AttnArgs a, const BatchBuffers& b, int n_cu, hipStream_t s) {
  const int qb = a.G >= 4 ? 1 : a.G >= 2 ? 2 : 4;  // 4 to 8 waves per workgroup
  const int blocks = a.K * ((a.P + 16 * qb - 1) / (16 * qb));
  const int t_max = a.pos0 + a.P, key_tiles = (t_max + kKT - 1) / kKT;
  const double rec = 4.0 * a.P * a.A * (D + 2);
  const int most = static_cast<int>(std::min<size_t>(key_tiles, std::max<size_t>(1, static_cast<size_t>(b.attn_ws_floats * 4.0 / rec))));
  int ns = 1;
  double best = 0.0;
  for (int n = 1; n <= std::min(most, 64); ++n) {
    const int tiles = (key_tiles + n - 1) / n;
    const double us = static_cast<double>((blocks * n + 2 * n_cu - 1) / (2 * n_cu)) * tiles * 2.8 +
                      (n > 1 ? 4.5 + 2.0 * n * rec / 4e6 : 0.0);
    if (n == 1 || us < best) {
      best = us;
      ns = n;
    }
  }
  a.keys_per_split = (key_tiles + ns - 1) / ns * kKT;
  a.nsplit = (t_max + a.keys_per_split - 1) / a.keys_per_split;
  const dim3 grid(blocks * a.nsplit), block(64 * a.G * qb);
  switch (a.G) {
#define EE_ATTN_G(GG)                                                                                         \
  case GG:                                                                                                    \
    hipLaunchKernelGGL((k_bp_attn_mfma<D, GG, (GG >= 4 ? 1 : GG >= 2 ? 2 : 4)>), grid, block, 0, s, a);        \
    break;
    EE_ATTN_G(1) EE_ATTN_G(2) EE_ATTN_G(3) EE_ATTN_G(4) EE_ATTN_G(5) EE_ATTN_G(6) EE_ATTN_G(7) EE_ATTN_G(8)
#undef EE_ATTN_G
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.nsplit == 1) return e;
  hipLaunchKernelGGL((k_bp_attn_merge<uint16_t, D>), dim3((a.P * a.A + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <typename WT, int D>
hipError_t attention(AttnArgs a, const BatchBuffers& b, int n_cu, hipStream_t s) {
  constexpr int kQT = 4;  // query positions per block of the prompt's path
  const int nqt = (a.P + kQT - 1) / kQT;
  const int t_max = a.pos0 + a.P;
  const int key_tiles = (t_max + kKT - 1) / kKT;
  int ns = std::max(1, (4 * n_cu + a.K * nqt - 1) / (a.K * nqt));
  ns = std::min(ns, key_tiles);
  const size_t per = static_cast<size_t>(a.P) * a.A * (D + 2);
  ns = static_cast<int>(std::min<size_t>(ns, std::max<size_t>(1, b.attn_ws_floats / per)));
  a.keys_per_split = (key_tiles + ns - 1) / ns * kKT;
  a.nsplit = (t_max + a.keys_per_split - 1) / a.keys_per_split;
  // few blocks: blocks of two query positions whose waves take one query
  // head each; else four positions, one wave each with all heads
  const bool split_heads = static_cast<int64_t>(a.K) * nqt * a.nsplit < 2 * n_cu && a.G >= 2;
  const dim3 grid(a.K * (split_heads ? (a.P + 1) / 2 : nqt) * a.nsplit);
  switch (a.G) {
#define EE_ATTN_G(GG)                                                                                  \
  case GG:                                                                                             \
    if (GG >= 2 && split_heads) {                                                                      \
      hipLaunchKernelGGL((k_bp_attn<WT, D, GG, 1, (GG >= 2 ? 2 : 4)>), grid, dim3(128 * GG), 0, s, a); \
    } else {                                                                                           \
      hipLaunchKernelGGL((k_bp_attn<WT, D, GG, GG, 4>), grid, dim3(64 * kQT), 0, s, a);                \
    }                                                                                                  \
    break;
    EE_ATTN_G(1) EE_ATTN_G(2) EE_ATTN_G(3) EE_ATTN_G(4) EE_ATTN_G(5) EE_ATTN_G(6) EE_ATTN_G(7) EE_ATTN_G(8)
#undef EE_ATTN_G
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.nsplit == 1) return e;
  hipLaunchKernelGGL((k_bp_attn_merge<WT, D>), dim3((a.P * a.A + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <typename WT>
hipError_t attention_d(const AttnArgs& a, const BatchBuffers& b, int n_cu, hipStream_t s) {
  switch (a.D) {
    case 32: return hipErrorInvalidValue;  // rows of at least 64 dimensions (one per lane)
    case 64:
      if constexpr (sizeof(WT) == 2) return attention_mfma<64>(a, b, n_cu, s);
      else return attention<WT, 64>(a, b, n_cu, s);
    case 128:
      if constexpr (sizeof(WT) == 2) return attention_mfma<128>(a, b, n_cu, s);
  }
  return hipErrorInvalidValue;
}

template <typename WT>
hipError_t pass(const BatchPass& bp, int pos0, const int32_t* d_tokens, int n, hipStream_t s) {
  const DevParams& p = bp.p;
  const BatchBuffers& b = bp.buf;
  hipError_t e;
  for (int c0 = 0; c0 < n; c0 += b.max_positions) {
    const int P = std::min(b.max_positions, n - c0);
    const int cpos = pos0 + c0;
    hipLaunchKernelGGL((k_bp_embed<WT>), dim3(P), dim3(256), 0, s, static_cast<const WT*>(p.embed), d_tokens + c0, P,
                       p.H, p.V, b.X, p.hist_tok, cpos, p.ctl);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if constexpr (sizeof(WT) == 2)
      if ((e = reduce_norm(b, b.X, 0, P, p.H, bp.layers[0].g_attn, p.eps, s)) != hipSuccess) return e;
    for (int l = 0; l < p.L; ++l) {
      const LayerW& lw = bp.layers[l];
      GemmArgs g{};
      g.P = P;
      g.eps = p.eps;
      g.part = b.gemm_ws;
      g.tile_ctr = b.tile_ctr;
      g.pos0 = cpos;
      g.Aq = p.A;
      g.Kh = p.K;
      g.D = p.D;
      g.rope_cos = p.rope_cos;
      g.rope_sin = p.rope_sin;
      g.kpool = p.kpool;
      g.vpool = p.vpool;
      g.layer_base = static_cast<int64_t>(l) * p.layer_stride;
      g.block_table = p.block_table;
      g.page_shift = p.page_shift;
      g.page_size = p.page_size;
      GemmArgs q = g, o = g, gu = g, dn = g;
      q.A = b.X; q.W = lw.wqkv; q.N = p.qkv_rows; q.K = p.H; q.gain = lw.g_attn; q.Y = b.Q;
      o.A = b.O; o.W = lw.wo; o.N = p.H; o.K = p.A * p.D; o.Y = b.X;
      gu.A = b.X; gu.W = lw.wgu; gu.N = 2 * p.F; gu.K = p.H; gu.gain = lw.g_mlp; gu.Y = b.Act;
      gu.planes = static_cast<u32x4*>(b.Ap); gu.k32_out = mm_k32(p.F);
      dn.A = b.Act; dn.W = lw.wd; dn.N = p.H; dn.K = p.F; dn.Y = b.X;
      AttnArgs at{};
      at.Q = b.Q; at.O = b.O; at.part = b.attn_ws;
      at.planes = static_cast<u32x4*>(b.Op); at.k32 = mm_k32(p.A * p.D);
      at.kpool = p.kpool; at.vpool = p.vpool; at.layer_base = g.layer_base;
      at.block_table = p.block_table; at.page_shift = p.page_shift; at.page_size = p.page_size;
      at.P = P; at.pos0 = cpos; at.A = p.A; at.K = p.K; at.G = p.G; at.D = p.D; at.scale = p.attn_scale;
      // After the last layer's cache entries only the final state of the
      // pass's last position is ever read, if any: one query, one row.
      float* X = b.X;
      const bool last = l + 1 == p.L;
      if (last) {
        const int64_t row = P - 1;
        X += row * p.H;
        at.Q += row * p.A * p.D;
        at.pos0 += P - 1;
        at.P = o.P = gu.P = dn.P = 1;
        o.Y = dn.Y = X;
        gu.A = X;
      }
      const bool stop = last && !(bp.head && c0 + P == n);
      if constexpr (sizeof(WT) == 2) {
        // the input's term planes are in Xp; each residual product's slices
        // are summed by the kernel that prepares the next product's input
        const LayerT& lt = bp.tiled[l];
        const u32x4* Xp = static_cast<const u32x4*>(b.Xp);
        int sp = 0;
        if ((e = gemm_mm<kEpiQkv>(q, lt.wqkv, Xp, b, bp.n_cu, nullptr, s)) != hipSuccess) return e;
        if (stop) break;
        if ((e = attention_d<WT>(at, b, bp.n_cu, s)) != hipSuccess) return e;
        if ((e = gemm_mm<kEpiResid>(o, lt.wo, static_cast<const u32x4*>(b.Op), b, bp.n_cu, &sp, s)) != hipSuccess)
          return e;
        if ((e = reduce_norm(b, X, sp, at.P, p.H, lw.g_mlp, p.eps, s)) != hipSuccess) return e;
        if ((e = gemm_mm<kEpiSwiGlu>(gu, lt.wgu, Xp, b, bp.n_cu, nullptr, s)) != hipSuccess) return e;
        if ((e = gemm_mm<kEpiResid>(dn, lt.wd, static_cast<const u32x4*>(b.Ap), b, bp.n_cu, &sp, s)) != hipSuccess)
          return e;
        const float* next = l + 1 < p.L ? bp.layers[l + 1].g_attn : nullptr;
        if ((e = reduce_norm(b, X, sp, at.P, p.H, next, p.eps, s)) != hipSuccess) return e;
      } else {
        if ((e = gemm<WT, kEpiQkv>(q, b, bp.n_cu, s)) != hipSuccess) return e;
        if (stop) break;
        if ((e = attention_d<WT>(at, b, bp.n_cu, s)) != hipSuccess) return e;
        if ((e = gemm<WT, kEpiResid>(o, b, bp.n_cu, s)) != hipSuccess) return e;
        if ((e = gemm<WT, kEpiSwiGlu>(gu, b, bp.n_cu, s)) != hipSuccess) return e;
        if ((e = gemm<WT, kEpiResid>(dn, b, bp.n_cu, s)) != hipSuccess) return e;
      }
    }
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_batched_pass(const BatchPass& bp, int pos0, const int32_t* d_tokens, int n, hipStream_t s) {
  if (n <= 0 || bp.buf.max_positions <= 0) return hipErrorInvalidValue;
  return bp.wbf16 ? pass<uint16_t>(bp, pos0, d_tokens, n, s) : pass<float>(bp, pos0, d_tokens, n, s);
}

size_t batch_tile_counters(int max_positions, int N_max) {
  // fp32 weights: tiles of 64 x 64 (more than 16 positions) and 16 x 64 (at most 16)
  return static_cast<size_t>((N_max + 63) / 64) * ((max_positions + 63) / 64);
}

size_t batch_weight_bytes(int N, int K) { return mm_weight_bytes(N, K); }
size_t batch_plane_bytes(int P, int K) { return mm_plane_bytes(P, K); }

hipError_t launch_tile_weights(const void* W, int N, int K, void* T, hipStream_t s) {
  const int64_t chunks = static_cast<int64_t>(mm_weight_bytes(N, K) / 16);
  const int blocks = static_cast<int>(std::min<int64_t>((chunks + 255) / 256, 8192));
  hipLaunchKernelGGL(k_bp_tile_weights, dim3(blocks), dim3(256), 0, s, static_cast<const uint16_t*>(W), N, K, mm_k32(K),
                     chunks, static_cast<u32x4*>(T));
  return hipGetLastError();
}

}  // namespace ee
