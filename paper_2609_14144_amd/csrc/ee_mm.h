// Matrix products of the batched full-depth pass on the matrix cores:
// Y[p][n] = sum_k X[p][k] W[n][k], weights bf16 or fp32, activations fp32.
//
// Operands lie in memory in the order in which the matrix instruction takes
// them, so that neither needs a shuffle, a conversion or a bank conflict on
// its way to the matrix cores. Both are cut into K blocks in which each lane
// of a wave holds one 16-byte chunk (8 bf16 or 4 fp32 elements) of one row:
//   * weights ("tiled copy", made once when they are loaded):
//     [N/16][K/BK][lane 64][chunk]: lane l of a 16 x BK tile holds row l % 16,
//     chunk l / 16; rows and columns padded with zeros (K to 64);
//   * activations ("planes"): [P/16][K/BK][term][lane 64][chunk], lane l
//     holding position l % 16, chunk l / 16.
// bf16 weights (v_mfma_f32_16x16x32_bf16, BK = 32): activations are three bf16
// terms into which the producer split the fp32 value exactly (the top 16
// bits, those of the remainder, the rest). The three products accumulate in
// fp32, so the result carries fp32 accumulation error only. The producer of a
// vector splits it once; splitting in the product itself repeats it for every
// row tile, and the vector ALU then takes longer than the matrix cores.
// fp32 weights (v_mfma_f32_16x16x4_f32, BK = 16, one term): a chunk's four
// elements feed four instructions, whose K slot of lane group g is element
// 4 g + j on both sides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ee {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename WT>
struct MmOp;
template <>
struct MmOp<uint16_t> {
  static constexpr int kTerms = 3, kBK = 32, kEl = 8;
  __device__ static __forceinline__ f32x4 mma(const u32x4& w, const u32x4& x, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0,
                                                   0);
  }
};
template <>
struct MmOp<float> {
  static constexpr int kTerms = 1, kBK = 16, kEl = 4;
  __device__ static __forceinline__ f32x4 mma(const u32x4& w, const u32x4& x, f32x4 c) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[j]), __uint_as_float(x[j]), c, 0, 0, 0);
    return c;
  }
};

// K blocks of a vector of K elements (whole steps of 64)
template <typename WT>
__host__ __device__ inline int mm_blocks(int K) { return (K + 63) / 64 * (64 / MmOp<WT>::kBK); }
// 16-byte chunk of term `term` of (position p, elements k .. k + kEl - 1), k a multiple of kEl
template <typename WT>
__device__ __forceinline__ int64_t mm_chunk(int p, int k, int term, int blocks) {
  using O = MmOp<WT>;
  return ((static_cast<int64_t>(p >> 4) * blocks + k / O::kBK) * O::kTerms + term) * 64 + (p & 15) +
         16 * (k % O::kBK / O::kEl);
}

// the three bf16 terms of x, each in the low 16 bits
__device__ __forceinline__ void mm_split(float x, uint32_t& t0, uint32_t& t1, uint32_t& t2) {
  const uint32_t u = __float_as_uint(x);
  const float r1 = x - __uint_as_float(u & 0xffff0000u);
  const uint32_t u1 = __float_as_uint(r1);
  const float r2 = r1 - __uint_as_float(u1 & 0xffff0000u);
  t0 = u >> 16;
  t1 = u1 >> 16;
  t2 = __float_as_uint(r2) >> 16;  // exact: r2 has at most 8 significant bits
}
// two neighbouring elements, each term packed as one 32-bit word
__device__ __forceinline__ void mm_split2(float a, float b, uint32_t (&t)[3]) {
  uint32_t x[3], y[3];
  mm_split(a, x[0], x[1], x[2]);
  mm_split(b, y[0], y[1], y[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) t[i] = x[i] | (y[i] << 16);
}
// NE neighbouring elements k .. k + NE - 1 of position p into its planes (2 or 4 of one chunk, or 8 from a
// multiple of 8 on)
template <typename WT, int NE>
__device__ __forceinline__ void mm_put(u32x4* planes, int blocks, int p, int k, const float (&v)[NE]) {
  using O = MmOp<WT>;
  if constexpr (sizeof(WT) == 4) {
#pragma unroll
    for (int i = 0; i < NE; i += NE < 4 ? NE : 4) {
      float* d = reinterpret_cast<float*>(planes + mm_chunk<WT>(p, (k + i) / O::kEl * O::kEl, 0, blocks)) + (k + i) % O::kEl;
      if constexpr (NE == 1) *d = v[0];
      else if constexpr (NE == 2) *reinterpret_cast<float2*>(d) = make_float2(v[0], v[1]);
      else *reinterpret_cast<f32x4*>(d) = f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]};
    }
  } else {
    uint32_t w[(NE + 1) / 2][3];
#pragma unroll
    for (int i = 0; i < NE; i += 2) mm_split2(v[i], NE > 1 ? v[NE > 1 ? i + 1 : 0] : 0.f, w[i / 2]);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      uint16_t* d = reinterpret_cast<uint16_t*>(planes + mm_chunk<WT>(p, k / O::kEl * O::kEl, t, blocks)) + k % O::kEl;
      if constexpr (NE == 1) *d = static_cast<uint16_t>(w[0][t]);
      else if constexpr (NE == 2) *reinterpret_cast<uint32_t*>(d) = w[0][t];
      else if constexpr (NE == 4) *reinterpret_cast<uint2*>(d) = make_uint2(w[0][t], w[1][t]);
      else *reinterpret_cast<u32x4*>(d) = u32x4{w[0][t], w[1][t], w[2][t], w[3][t]};
    }
  }
}

struct MmArgs {
  const u32x4* W;  // tiled copy
  const u32x4* X;  // planes
  int P, N;
  int NB, PB;      // 16-row and 16-position blocks
  int blocks;      // K blocks
  int nN, nP;      // tiles along N and P
  int splits, steps_per_split;  // K slices, in steps of 64
  int tiles_per_xcd;
};

// Block: KG groups of NW waves. A group's waves are stacked along N, each RB
// blocks of 16 rows; all share CP blocks of 16 positions. The groups take
// parts of the block's K slice, and their sums meet in LDS (for products with
// too few tiles to fill the device whose epilogue wants finished sums). Bound
// by the matrix cores for many positions (each wave issues 6 RB CP MFMAs of 16
// cycles per 64-wide step) and by the weight stream for few. Weights go
// straight to registers (no wave shares its rows with another of its group),
// activations through LDS, where every wave reads them: per step a wave reads
// 6 CP KB of LDS for 6 RB CP MFMAs, so RB = 3 leaves the LDS 60 to 70% busy
// and RB = 2 nearly saturates it.
// Three LDS buffers: step s is read while step s + 2 is written, and the
// first fragments of step s + 1 are already complete, so that their reads are
// issued before the one barrier per step; fragments of each group of RB x CP
// MFMAs are requested one group ahead.
// Sums: every matrix-core accumulation rounds, so the error grows with the
// number of accumulations (three per 32 elements) into one register. Groups
// of kSum steps (6 kSum accumulations) are summed from zero and then added to
// a total, about as short a chain as a K split over many waves gives; the
// additions cost the vector ALU 4% of a step's matrix-core time with groups
// of four steps, and nothing that counts where the weight stream bounds the
// tile (groups of one or two). One chain over the whole of K had 1.4 times the
// error. Within a K block the smallest term goes first: added to the large sum
// of the block's first term it would round like it, so a chain's first block
// rounds once instead of three times, at no cost. Error against 64 bits, over
// that of the product that split its activations itself (896 to 11008 wide
// products of three decoders, 13 to 1024 positions): 0.23 to 0.89, largest
// term first 0.24 to 1.03 (896 wide, 17 to 256 positions).
// With fp32 weights every product rounds, so each K block of 16 is summed from
// zero, and its sum added while the next block runs.
// A workgroup's tile follows from its XCD (blockIdx % 8): every XCD takes a
// contiguous range of tiles, position tiles fastest, so that the workgroups
// that share weight rows share an L2.
// Measured (17920 x 1536 weights, us, against the product that split its
// activations itself and read row-major weights): 1024 positions 139 against
// 233, 512 positions 77 against 143, 13 positions 15.5 against 19.
template <typename WT, int RB, int CP, int NW, int PF, int KG, typename Pre, typename Epi>
__device__ __forceinline__ void mm_tile(const MmArgs& g, Pre&& pre, Epi&& epi) {
  constexpr int NT = 64 * NW;                  // threads of a K group
  constexpr int kSum = CP <= 2 ? CP : 4;       // steps summed from zero
  using Op = MmOp<WT>;
  constexpr int KB = 64 / Op::kBK;             // K blocks per step
  constexpr int NG = KB * Op::kTerms;          // fragments of a position block per step
  constexpr int XS = CP * NG * 64;             // chunks of a step
  constexpr int XL = (XS + NT - 1) / NT;       // chunks per thread per step
  static_assert((KG - 1) * NW * RB * CP * 64 <= KG * 3 * XS, "the groups' sums fit the buffers");
  __shared__ u32x4 Xsm[KG][3][XS];
  const int lane = threadIdx.x & 63;
  const int kg = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / NT);
  const int tid = static_cast<int>(threadIdx.x) - kg * NT;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  u32x4 (*Xs)[XS] = Xsm[kg];
  const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
  const int tile = xcd * g.tiles_per_xcd + loc;
  if (loc >= g.tiles_per_xcd || tile >= g.nN * g.nP * g.splits) return;
  const int tp = tile % g.nP, tr = tile / g.nP;
  const int tn = tr % g.nN, split = tr / g.nN;
  const int nb0 = (tn * NW + wave) * RB, pb0 = tp * CP;
  const int total = g.blocks / KB;
  const int s0 = split * g.steps_per_split, slice = min(total - s0, g.steps_per_split);
  // the K group's steps; every group passes every barrier of nmax steps
  const int nmax = (slice + KG - 1) / KG;
  const int sb = s0 + slice * kg / KG, n = s0 + slice * (kg + 1) / KG - sb;

  // loads past the last row, position or step read a valid address instead;
  // what they yield is not stored
  const u32x4* wbase = g.W + static_cast<int64_t>(sb) * (KB * 64) + lane;
  int64_t wo[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) wo[r] = static_cast<int64_t>(min(nb0 + r, g.NB - 1)) * g.blocks * 64;
  // thread's chunk i of a step: c = tid + NT i of [position block][K block][term][lane]
  const u32x4* xp[XL];
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int c = min(tid + NT * i, XS - 1);
    const int pb = min(pb0 + c / (NG * 64), g.PB - 1);
    xp[i] = g.X + (static_cast<int64_t>(pb) * g.blocks + KB * sb) * (Op::kTerms * 64) + c % (NG * 64);
  }
  u32x4 xr[PF][XL];
  u32x4 wr[PF][KB][RB];
  auto load_x = [&](int st, int slot) {
    const int64_t o = static_cast<int64_t>(min(st, n - 1)) * (NG * 64);
#pragma unroll
    for (int i = 0; i < XL; ++i) xr[slot][i] = xp[i][o];
  };
  auto store_x = [&](int buf, int slot) {
#pragma unroll
    for (int i = 0; i < XL; ++i)
      if (XS % NT == 0 || tid + NT * i < XS) Xs[buf][tid + NT * i] = xr[slot][i];
  };
  auto load_w = [&](int st, int slot, int kb) {
    const u32x4* w = wbase + static_cast<int64_t>(min(st, n - 1)) * (KB * 64) + kb * 64;
#pragma unroll
    for (int r = 0; r < RB; ++r) wr[slot][kb][r] = w[wo[r]];
  };
  // sums of the current group of steps (fp32: of the latest two K blocks), and of all before them
  constexpr bool kBlockSum = sizeof(WT) == 4;
  f32x4 acc[RB][CP], odd[kBlockSum ? RB : 1][kBlockSum ? CP : 1], tot[RB][CP];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < CP; ++c) {
      acc[r][c] = tot[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (kBlockSum) odd[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  u32x4 xf[2][CP];
  // group gi = (K block gi / kTerms, its terms from the smallest on)
  auto read_f = [&](int buf, int gi, int d) {
    const int f = gi / Op::kTerms * Op::kTerms + Op::kTerms - 1 - gi % Op::kTerms;
#pragma unroll
    for (int c = 0; c < CP; ++c) xf[d][c] = Xs[buf][(c * NG + f) * 64 + lane];
  };

  // what the epilogue reads (pre(p, n)): requested here by the small tiles,
  // where a round trip after the last step would count
  constexpr bool kEarly = RB * CP <= 2;
  const int lg = lane >> 4, lr = lane & 15;
  auto out_p = [&](int c) { return (pb0 + c) * 16 + lr; };
  auto out_n = [&](int r) { return (nb0 + r) * 16 + 4 * lg; };
  decltype(pre(0, 0)) ep[kEarly ? RB : 1][kEarly ? CP : 1];
  if constexpr (kEarly) {
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < CP; ++c) ep[r][c] = pre(min(out_p(c), g.P - 1), min(out_n(r), g.N - 4));
  }
  load_x(0, 0);
#pragma unroll
  for (int i = 0; i < PF; ++i) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) load_w(i, i, kb);
    if (i == 0) {
      store_x(0, 0);
      load_x(1, 0);
      store_x(1, 0);
    }
    load_x(i + 2, i);
  }
  __syncthreads();
  read_f(0, 0, 0);
  int cur = 0, nxt = 1, fre = 2;
  constexpr int kUnroll = PF > kSum ? PF : kSum;
  static_assert(NG % 2 == 0, "the first fragments of a step go to buffer 0");
  static_assert(kUnroll % PF == 0 && kUnroll % kSum == 0, "ring slots and sums follow the unrolled steps");
  for (int st0 = 0; st0 < nmax; st0 += kUnroll) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int st = st0 + u, i = u % PF;
      if (st >= nmax) break;  // the same for every wave
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        if (gi < NG - 1) read_f(cur, gi + 1, (gi + 1) & 1);
        else read_f(nxt, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (gi == 1) {
          store_x(fre, i);
          load_x(st + 2 + PF, i);
        }
        if constexpr (kBlockSum) {
          if (KG == 1 || st < n) {
            // this block from zero while the previous block's sum is added
            auto& now = gi & 1 ? odd : acc;
            auto& before = gi & 1 ? acc : odd;
#pragma unroll
            for (int c = 0; c < CP; ++c)
#pragma unroll
              for (int r = 0; r < RB; ++r)
                now[r][c] = Op::mma(wr[i][gi][r], xf[gi & 1][c], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
            for (int c = 0; c < CP; ++c)
#pragma unroll
              for (int r = 0; r < RB; ++r) tot[r][c] += before[r][c];
          }
        } else if (KG == 1 || st < n) {
#pragma unroll
          for (int c = 0; c < CP; ++c)
#pragma unroll
            for (int r = 0; r < RB; ++r)
              acc[r][c] = Op::mma(wr[i][gi / Op::kTerms][r], xf[gi & 1][c],
                                  u % kSum == 0 && gi == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[r][c]);
        }
        if (gi % Op::kTerms == Op::kTerms - 1) load_w(st + PF, i, gi / Op::kTerms);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
      if (!kBlockSum && u % kSum == kSum - 1 && (KG == 1 || st < n)) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int c = 0; c < CP; ++c) tot[r][c] += acc[r][c];
      }
      const int t = cur;
      cur = nxt;
      nxt = fre;
      fre = t;
    }
  }
  if (kBlockSum || n % kSum != 0) {
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < CP; ++c) {
        if constexpr (kBlockSum) tot[r][c] += odd[r][c];
        else tot[r][c] += acc[r][c];
      }
  }
  if constexpr (KG > 1) {  // the groups' sums, in order (the last barrier ended every read of the buffers)
    f32x4* sums = reinterpret_cast<f32x4*>(&Xsm[0][0][0]);
    if (kg > 0) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CP; ++c) sums[(((kg - 1) * NW + wave) * RB * CP + r * CP + c) * 64 + lane] = tot[r][c];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int q = 0; q < KG - 1; ++q)
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CP; ++c) tot[r][c] += sums[((q * NW + wave) * RB * CP + r * CP + c) * 64 + lane];
  }
  // lane's outputs of (row block r, position block c): rows out_n(r) + 0..3, position out_p(c); N is a
  // multiple of 4
#pragma unroll
  for (int c = 0; c < CP; ++c) {
    if (out_p(c) >= g.P) continue;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      if (out_n(r) >= g.N) continue;
      if constexpr (kEarly) epi(split, out_p(c), out_n(r), tot[r][c], ep[r][c]);
      else epi(split, out_p(c), out_n(r), tot[r][c], pre(out_p(c), out_n(r)));
    }
  }
}

}  // namespace ee
