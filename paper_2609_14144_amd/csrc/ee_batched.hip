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
// The products run on the matrix cores (ee_mm.h): the producer of each vector
// writes it in operand order (for bf16 weights split into bf16 terms), and the
// residual products store the partial sums of their K slices, which the kernel
// that prepares the next product's input adds up in slice order. Every result
// is independent of scheduling.
//
// Numerics follow the decode program: weights as stored (bf16 or fp32),
// activations and accumulation fp32, cache entries rounded to the storage
// type (round to nearest even), RMSNorm as x * rsqrt(mean(x^2) + eps) * g,
// e^x in the softmax and SiLU on the hardware base-2 exponential.
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "ee_internal.h"
#include "ee_mm.h"
#include "ee_tiles.h"

namespace ee {

namespace {

// ---------------------------------------------------------------------------
// helpers (this file's own; the decode kernels keep theirs)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float exp_hw(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

// four neighbouring cache elements (p 8- or 16-byte aligned)
__device__ __forceinline__ uint32_t bf16_bits(float x) {  // round to nearest even
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ void store4(uint16_t* p, const f32x4& v) {
  *reinterpret_cast<uint2*>(p) =
      make_uint2(bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16));
}
__device__ __forceinline__ void store4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }

__device__ __forceinline__ int64_t cache_off(const int32_t* block_table, int page_shift, int page_size, int K,
                                             int D, int64_t layer_base, int pos, int kvh) {
  const int page = block_table[pos >> page_shift];
  const int slot = pos & (page_size - 1);
  return layer_base + ((static_cast<int64_t>(page) * K + kvh) * page_size + slot) * D;
}

// Wave sum: DPP within rows of 16 lanes, then the four row results by
// readlane; every lane gets the same value, summed in a fixed order.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_of(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
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
// the products' epilogues (ee_mm.h), and what runs between them
// ---------------------------------------------------------------------------
enum : int { kEpiQkv = 0, kEpiResid = 1, kEpiSwiGlu = 2 };

struct GemmArgs {
  int P, N, K;
  float* part;         // kEpiResid: partial sums of the K slices [split][P][N], for k_bp_reduce_norm
  u32x4* planes;       // kEpiSwiGlu: planes of SiLU(gate) * up, `blocks` K blocks
  int blocks;
  // kEpiQkv: queries [P][A*D], RoPE and cache
  float* Q;
  int pos0, Aq, Kh, D;
  const float* rope_cos;
  const float* rope_sin;
  void* kpool;
  void* vpool;
  int64_t layer_base;
  const int32_t* block_table;
  int page_shift, page_size;
};

// tiled copy of a row-major [N][K] matrix (K a multiple of 8), padded with zeros
template <typename WT>
__global__ __launch_bounds__(256) void k_bp_tile_weights(const WT* __restrict__ W, int N, int K, int blocks,
                                                         int64_t chunks, u32x4* __restrict__ T) {
  using Op = MmOp<WT>;
  for (int64_t c = blockIdx.x * 256ll + threadIdx.x; c < chunks; c += gridDim.x * 256ll) {
    const int lane = static_cast<int>(c & 63);
    const int64_t t = c >> 6;
    const int64_t n = t / blocks * 16 + (lane & 15);
    const int k = static_cast<int>(t % blocks) * Op::kBK + Op::kEl * (lane >> 4);
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
template <typename WT>
__device__ __forceinline__ void qkv_store(const GemmArgs& g, const QkvEpi& e, int p, int n, const f32x4& y) {
  const int AD = g.Aq * g.D, KD = g.Kh * g.D;
  if (n >= AD + KD) {
    store4(static_cast<WT*>(g.vpool) + e.off, y);
    return;
  }
  const f32x4 r{y[0] * e.c.x - y[1] * e.s.x, y[1] * e.c.x + y[0] * e.s.x, y[2] * e.c.y - y[3] * e.s.y,
                y[3] * e.c.y + y[2] * e.s.y};
  if (n < AD) *reinterpret_cast<f32x4*>(g.Q + static_cast<int64_t>(p) * AD + n) = r;
  else store4(static_cast<WT*>(g.kpool) + e.off, r);
}

template <typename WT, int EPI, int RB, int CP, int NW, int PF, int KG>
__global__ __launch_bounds__(64 * NW * KG) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_bp_mm(MmArgs m, GemmArgs g) {
  if constexpr (EPI == kEpiQkv) {
    mm_tile<WT, RB, CP, NW, PF, KG>(
        m, [&](int p, int n) { return qkv_epi(g, p, n); },
        [&](int, int p, int n, const f32x4& y, const QkvEpi& e) { qkv_store<WT>(g, e, p, n, y); });
  } else {
    mm_tile<WT, RB, CP, NW, PF, KG>(
        m, [](int, int) { return 0; },
        [&](int split, int p, int n, const f32x4& y, int) {
          if constexpr (EPI == kEpiResid) {
            *reinterpret_cast<f32x4*>(g.part + (static_cast<int64_t>(split) * m.P + p) * m.N + n) = y;
          } else {
            // interleaved rows: n = 2j gate row j, n + 1 up row j
            const float a[2] = {y[0] / (1.f + exp_hw(-y[0])) * y[1], y[2] / (1.f + exp_hw(-y[2])) * y[3]};
            mm_put<WT, 2>(g.planes, g.blocks, p, n >> 1, a);
          }
        });
  }
}

// The residual stream after a product, and the input of the next: X += the
// product's K slices in slice order (splits may be 0), then, with a gain,
// the planes of x * rsqrt(mean(x^2) + eps) * gain. One workgroup per
// position, thread = 8 elements (H <= 2048). The 16 positions of a block of
// planes go to workgroups of one XCD, whose L2 then merges their 16-byte
// pieces into whole lines. Bound by the reads of the slices.
constexpr int kNormThreads = 256;
template <typename WT>
__global__ __launch_bounds__(kNormThreads) void k_bp_reduce_norm(float* __restrict__ X, const float* __restrict__ part,
                                                                 int splits, int P, int H,
                                                                 const float* __restrict__ gain, float eps,
                                                                 u32x4* __restrict__ planes, int blocks) {
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
  float w[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) w[i] = x[i >> 2][i & 3] * r * gv[i >> 2][i & 3];
  mm_put<WT, 8>(planes, blocks, p, k, w);
}

// ---------------------------------------------------------------------------
// causal grouped-query attention of a chunk of queries (positions pos0 ..
// pos0 + P - 1) over the cache, on the matrix cores. With one key split the
// output's planes are written directly; several write partial records
// (weighted V, max, sum) merged in split order by k_bp_attn_merge.
// ---------------------------------------------------------------------------
struct AttnArgs {
  const float* Q;      // [P][A*D], pair-interleaved within heads (as the cached keys)
  u32x4* planes;       // planes of the output [P][A*D], `blocks` K blocks
  int blocks;
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

// Workgroup = (KV head, QB blocks of 16 query positions, key split); wave =
// (one of the KV head's G query heads, one block of 16 positions), so that all
// G heads share the key and value tiles staged in LDS. Per tile of 64 keys a
// wave computes S^T = K Q^T (rows keys, columns positions) and O^T += V^T P^T:
// a lane then holds one position's scores for 16 keys, the softmax needs two
// exchanges between lanes, the scores' layout is already the second product's
// operand (the key order of its K slots is permuted alike on both sides), and
// the output's layout that of the planes. Keys and values are exact operands;
// with bf16 caches queries and probabilities are split exactly into three bf16
// terms and values are read transposed from LDS (ds_read_b64_tr_b16), so both
// products carry fp32 accumulation error only (over that of dot products of
// one lane per key, 1 to 1024 queries: bf16 0.51 to 0.88; fp32 0.62 to 0.83
// with the scores in two chains, 0.75 to 1.02 in one).
// A tile is 96 MFMAs (1536 cycles) per wave at D = 128 in bf16 and about as
// much vector work (exponentials, the split of the probabilities), which other
// waves overlap. A vector-ALU form (dot products from LDS, one wave per
// position) was bound by its FMAs and serial LDS reads: 1024 queries over 1024
// to 8192 bf16 keys (six heads of 128 per KV head) took 595 us a layer on
// average, this 104 (172 for the last 1024, 840 TFLOP/s of term products); 512
// queries over 512 keys 47 us, this 24 in one pass over the keys and less with
// key splits; 1024 queries over 1024 fp32 keys (two heads of 64) 46 us, this
// 13.
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

template <typename WT, int D, int G, int QB>
__global__ __launch_bounds__(64 * G * QB) __attribute__((amdgpu_waves_per_eu(2))) void k_bp_attn(AttnArgs a) {
  using Op = MmOp<WT>;
  constexpr bool kBf = sizeof(WT) == 2;
  constexpr int TM = Op::kTerms;
  constexpr int NT = 64 * G * QB;
  constexpr int CPK = D / Op::kEl;  // 16-byte chunks per cache row
  constexpr int KST = CPK + 1;      // padded LDS rows: 16 lanes reading a column of 16 rows, and the
  constexpr int VST = CPK + (kBf ? 2 : 1);  // reads of 4 rows x 32 (transposed) or 64 bytes, touch each bank once
  constexpr int KS = CPK / 4, DB = D / 16;
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
    return cache_off(a.block_table, a.page_shift, a.page_size, a.K, D, a.layer_base, min(k0 + j, ke - 1), kvh) + q * Op::kEl;
  };
  const WT* kp = static_cast<const WT*>(a.kpool);
  const WT* vp = static_cast<const WT*>(a.vpool);
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

  // the query's operands: chunk 4 s + lg of its row
  u32x4 qf[KS][TM];
  {
    const float* q = a.Q + static_cast<int64_t>(min(qi, a.P - 1)) * a.A * D + head * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const float* x = q + (4 * s + lg) * Op::kEl;
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(x);
      if constexpr (kBf) {
        const f32x4 x1 = *reinterpret_cast<const f32x4*>(x + 4);
        uint32_t w[4][3];
        mm_split2(x0[0], x0[1], w[0]);
        mm_split2(x0[2], x0[3], w[1]);
        mm_split2(x1[0], x1[1], w[2]);
        mm_split2(x1[2], x1[3], w[3]);
#pragma unroll
        for (int t = 0; t < 3; ++t) qf[s][t] = u32x4{w[0][t], w[1][t], w[2][t], w[3][t]};
      } else {
        qf[s][0] = __builtin_bit_cast(u32x4, x0);
      }
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
    // scores: block b holds keys k0 + 16 b + 4 lg + 0..3 of the lane's query; with fp32 caches, where every product
    // rounds, in two chains
    f32x4 s[4], odd[kBf ? 1 : 4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (!kBf) odd[b] = s[b];
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 kf[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) kf[b] = Ks[(16 * b + lr) * KST + 4 * ks + lg];
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          f32x4& sum = kBf || ks % 2 == 0 ? s[b] : odd[kBf ? 0 : b];
          sum = Op::mma(kf[b], qf[ks][t], sum);
        }
    }
    if constexpr (!kBf) {
#pragma unroll
      for (int b = 0; b < 4; ++b) s[b] += odd[b];
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
    // probabilities; bf16: split, operand word of keys (i, i + 1) of block b: [2 (b & 1) + i / 2] of K slots b / 2
    uint32_t pw[2][4][3];
    float pf[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[b][i], scale2, -ms));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[b][i + 1], scale2, -ms));
        l += p0 + p1;
        if constexpr (kBf) {
          mm_split2(p0, p1, pw[b >> 1][2 * (b & 1) + (i >> 1)]);
        } else {
          pf[b][i] = p0;
          pf[b][i + 1] = p1;
        }
      }
#pragma unroll
    for (int d = 0; d < DB; ++d) o[d] *= alpha;
    if constexpr (kBf) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        u32x4 vf[DB];
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
          vf[d] = __builtin_bit_cast(u32x4, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int t = 0; t < TM; ++t) {
          const u32x4 pt{pw[ks][0][t], pw[ks][1][t], pw[ks][2][t], pw[ks][3][t]};
#pragma unroll
          for (int d = 0; d < DB; ++d) o[d] = Op::mma(vf[d], pt, o[d]);
        }
      }
    } else {
      // K slot lg of instruction i of block b: key 16 b + 4 lg + i
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float* src = reinterpret_cast<const float*>(&Vs[(16 * b + 4 * lg + i) * VST]) + lr;
          float v[DB];
#pragma unroll
          for (int d = 0; d < DB; ++d) v[d] = src[16 * d];
#pragma unroll
          for (int d = 0; d < DB; ++d) o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[d], pf[b][i], o[d], 0, 0, 0);
        }
    }
  }
  const float lsum = sum_groups(l);
  if (qi >= a.P) return;
  if (a.nsplit == 1) {
    const float inv = 1.f / lsum;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const float w[4] = {o[d][0] * inv, o[d][1] * inv, o[d][2] * inv, o[d][3] * inv};
      mm_put<WT, 4>(a.planes, a.blocks, qi, head * D + 16 * d + 4 * lg, w);
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
// (maxima in units of log2)
template <typename WT, int D>
__global__ __launch_bounds__(256) void k_bp_attn_merge(AttnArgs a) {
  constexpr int DPL = D / 64;
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
      const float sc = __builtin_amdgcn_exp2f(M - cm);  // 0 while nothing has been merged
      den *= sc;
#pragma unroll
      for (int e = 0; e < DPL; ++e) num[e] *= sc;
#pragma unroll
      for (int u = 0; u < kSG; ++u) {
        if (ms[u] == -INFINITY) continue;  // absent, or a split wholly past the query's position
        const float f = __builtin_amdgcn_exp2f(ms[u] - cm);
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
  mm_put<WT, DPL>(a.planes, a.blocks, qi, head * D + DPL * lane, num);
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------
namespace {

template <typename WT, int EPI, int RB, int CP, int NW, int PF, int KG>
hipError_t mm_launch(MmArgs m, const GemmArgs& g, int splits, hipStream_t s) {
  const int steps = m.blocks * MmOp<WT>::kBK / 64;
  m.nN = (m.NB + RB * NW - 1) / (RB * NW);
  m.nP = (m.PB + CP - 1) / CP;
  m.steps_per_split = (steps + splits - 1) / splits;
  m.splits = (steps + m.steps_per_split - 1) / m.steps_per_split;
  const int tiles = m.nN * m.nP * m.splits;
  m.tiles_per_xcd = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_bp_mm<WT, EPI, RB, CP, NW, PF, KG>), dim3(m.tiles_per_xcd * 8), dim3(64 * NW * KG), 0, s, m, g);
  return hipGetLastError();
}

template <typename WT, int EPI, size_t I = 0>
hipError_t mm_launch_tile(size_t i, const MmArgs& m, const GemmArgs& g, int splits, hipStream_t s) {
  constexpr size_t n = sizeof(MmTiles<WT>::t) / sizeof(MmTile);
  if constexpr (I < n) {
    if (i != I) return mm_launch_tile<WT, EPI, I + 1>(i, m, g, splits, s);
    constexpr MmTile t = MmTiles<WT>::t[I];
    if constexpr (t.kg == 1 || EPI == kEpiQkv) return mm_launch<WT, EPI, t.rb, t.cp, t.nw, t.pf, t.kg>(m, g, splits, s);
  }
  return hipErrorInvalidValue;
}

// T: the tiled weights, X: the input's planes. *splits receives the K slices
// that a residual product stored.
template <typename WT, int EPI>
hipError_t gemm(const GemmArgs& g, const void* T, const void* X, const BatchBuffers& b, int n_cu, int* splits,
                hipStream_t s) {
  constexpr bool kResid = EPI == kEpiResid;
  MmArgs m{};
  m.W = static_cast<const u32x4*>(T);
  m.X = static_cast<const u32x4*>(X);
  m.P = g.P;
  m.N = g.N;
  m.NB = (g.N + 15) / 16;
  m.PB = (g.P + 15) / 16;
  m.blocks = mm_blocks<WT>(g.K);
  const MmChoice ch = mm_choose<WT>(kResid, EPI == kEpiQkv, g.P, g.N, g.K, b.gemm_ws_floats, n_cu);
  if (!ch.splits) return hipErrorInvalidValue;
  if (splits) {
    const int steps = m.blocks * MmOp<WT>::kBK / 64, per = (steps + ch.splits - 1) / ch.splits;
    *splits = (steps + per - 1) / per;
  }
  return mm_launch_tile<WT, EPI>(ch.tile, m, g, ch.splits, s);
}

template <typename WT>
hipError_t reduce_norm(const BatchBuffers& b, float* X, int splits, int P, int H, const float* gain, float eps, hipStream_t s) {
  if (H > 8 * kNormThreads) return hipErrorInvalidValue;
  const int blocks = (P + 127) / 128 * 128;  // whole groups of 16 positions on each of the 8 XCDs
  hipLaunchKernelGGL((k_bp_reduce_norm<WT>), dim3(blocks), dim3(kNormThreads), 0, s, X, b.gemm_ws, splits, P, H, gain, eps,
                     static_cast<u32x4*>(b.Xp), mm_blocks<WT>(H));
  return hipGetLastError();
}

// Key splits for blocks whose longest has key_tiles tiles: units run two
// workgroups at a time, a tile takes ~2.8 us (the same for one workgroup and
// for two side by side), splits add the merging launch (4.5 us) and their
// records' stores and loads.
template <typename WT, int D>
hipError_t attention(AttnArgs a, const BatchBuffers& b, int n_cu, hipStream_t s) {
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
    hipLaunchKernelGGL((k_bp_attn<WT, D, GG, (GG >= 4 ? 1 : GG >= 2 ? 2 : 4)>), grid, block, 0, s, a);        \
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
  if (a.D == 64) return attention<WT, 64>(a, b, n_cu, s);
  if constexpr (sizeof(WT) == 2)
    if (a.D == 128) return attention<WT, 128>(a, b, n_cu, s);
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
    if ((e = reduce_norm<WT>(b, b.X, 0, P, p.H, bp.layers[0].g_attn, p.eps, s)) != hipSuccess) return e;
    for (int l = 0; l < p.L; ++l) {
      const LayerW& lw = bp.layers[l];
      // a matrix's tiled copy: made once, or here where the context has room for one only
      auto tiled = [&](const void* w, void* LayerT::*kept, int N, int K, const void** t) {
        *t = bp.tiled ? bp.tiled[l].*kept : bp.spare;
        return bp.tiled ? hipSuccess : launch_tile_weights(sizeof(WT) == 2, w, N, K, bp.spare, s);
      };
      const void* t = nullptr;
      GemmArgs g{};
      g.P = P;
      g.part = b.gemm_ws;
      g.Q = b.Q;
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
      q.N = p.qkv_rows; q.K = p.H;
      o.N = p.H; o.K = p.A * p.D;
      gu.N = 2 * p.F; gu.K = p.H;
      gu.planes = static_cast<u32x4*>(b.Ap); gu.blocks = mm_blocks<WT>(p.F);
      dn.N = p.H; dn.K = p.F;
      AttnArgs at{};
      at.Q = b.Q; at.part = b.attn_ws;
      at.planes = static_cast<u32x4*>(b.Op); at.blocks = mm_blocks<WT>(p.A * p.D);
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
      }
      const bool stop = last && !(bp.head && c0 + P == n);
      // the input's planes are in Xp; each residual product's slices are
      // summed by the kernel that prepares the next product's input
      int sp = 0;
      if ((e = tiled(lw.wqkv, &LayerT::wqkv, q.N, q.K, &t)) != hipSuccess) return e;
      if ((e = gemm<WT, kEpiQkv>(q, t, b.Xp, b, bp.n_cu, nullptr, s)) != hipSuccess) return e;
      if (stop) break;
      if ((e = attention_d<WT>(at, b, bp.n_cu, s)) != hipSuccess) return e;
      if ((e = tiled(lw.wo, &LayerT::wo, o.N, o.K, &t)) != hipSuccess) return e;
      if ((e = gemm<WT, kEpiResid>(o, t, b.Op, b, bp.n_cu, &sp, s)) != hipSuccess) return e;
      if ((e = reduce_norm<WT>(b, X, sp, at.P, p.H, lw.g_mlp, p.eps, s)) != hipSuccess) return e;
      if ((e = tiled(lw.wgu, &LayerT::wgu, gu.N, gu.K, &t)) != hipSuccess) return e;
      if ((e = gemm<WT, kEpiSwiGlu>(gu, t, b.Xp, b, bp.n_cu, nullptr, s)) != hipSuccess) return e;
      if ((e = tiled(lw.wd, &LayerT::wd, dn.N, dn.K, &t)) != hipSuccess) return e;
      if ((e = gemm<WT, kEpiResid>(dn, t, b.Ap, b, bp.n_cu, &sp, s)) != hipSuccess) return e;
      if ((e = reduce_norm<WT>(b, X, sp, at.P, p.H, last ? nullptr : bp.layers[l + 1].g_attn, p.eps, s)) != hipSuccess)
        return e;
    }
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_batched_pass(const BatchPass& bp, int pos0, const int32_t* d_tokens, int n, hipStream_t s) {
  if (n <= 0 || bp.buf.max_positions <= 0) return hipErrorInvalidValue;
  return bp.wbf16 ? pass<uint16_t>(bp, pos0, d_tokens, n, s) : pass<float>(bp, pos0, d_tokens, n, s);
}

namespace {
template <typename WT>
size_t weight_bytes(int N, int K) { return static_cast<size_t>((N + 15) / 16) * mm_blocks<WT>(K) * 1024; }
template <typename WT>
hipError_t tile_weights(const void* W, int N, int K, void* T, hipStream_t s) {
  const int64_t chunks = static_cast<int64_t>(weight_bytes<WT>(N, K) / 16);
  const int blocks = static_cast<int>(std::min<int64_t>((chunks + 255) / 256, 8192));
  hipLaunchKernelGGL((k_bp_tile_weights<WT>), dim3(blocks), dim3(256), 0, s, static_cast<const WT*>(W), N, K,
                     mm_blocks<WT>(K), chunks, static_cast<u32x4*>(T));
  return hipGetLastError();
}
}  // namespace

size_t batch_weight_bytes(int wbf16, int N, int K) { return wbf16 ? weight_bytes<uint16_t>(N, K) : weight_bytes<float>(N, K); }
size_t batch_plane_bytes(int wbf16, int P, int K) {
  return static_cast<size_t>((P + 15) / 16) * (wbf16 ? mm_blocks<uint16_t>(K) * 3 : mm_blocks<float>(K)) * 1024;
}
hipError_t launch_tile_weights(int wbf16, const void* W, int N, int K, void* T, hipStream_t s) {
  return wbf16 ? tile_weights<uint16_t>(W, N, K, T, s) : tile_weights<float>(W, N, K, T, s);
}

}  // namespace ee
