// Order-3 adjoint product in the symmetric form (FP32 and SPLIT_BF16).
//
// With w_t = dL/dB_t f / (N^3 n_t), L = sum_k d_k Q_k, where Q_k = sum_{i <= j <= k}
// w_ijk d_i d_j is a quadratic form of the shells up to k.  Y_k[m] = dQ_k/dd_m is one
// symmetric matrix times the fields, so that
//   a_m += d_k Y_k[m] for m <= k,   a_k += Q_k = (1/2) sum_m d_m Y_k[m]  (Euler).
// Each triplet is multiplied twice, by its two smaller sides, instead of three times
// by every side as in a_m = sum_{u <= v} W[m][(u, v)] d_u d_v, and the matrices are the
// (k, k) corner instead of every m.  For an alias-free plan the triangle bound
// k <= i + j + 2 (0-based) empties another corner: 64 shells take 211 32 x 32 x 16
// products per 32 points where the other form takes 304.
//
// Matrix products.  Y_k is computed in 32-row chains over the 16-shell chunks uc of u:
// the A operand is a weight block from LDS, B the register-held fields.  A chain's rows
// are either two blocks of 16 m of one partner (S), or one block of 16 m of the two
// partners of a pair (k, k + 1) (P), so that no row of a chain lies beyond k's block:
//   block 0 of k: P(0);  1: S(0);  2: P(0), S(1);  3: P(0), P(1), S(2).
// Rows are permuted so that lane half h, register r of either 16-row half holds
// m = 16 M + 8 h + r, the shells whose fields the lane holds: d_m Y[m] is lane-local.
#pragma once

#include "adjoint.h"

namespace ps {

static_assert(kAdjThreads == kSymCopyWords, "a round copies one word per thread");
template <int KB>
constexpr int sym_buffer_words() {
  int r = 0;
  for (int kb = 0; kb < KB; ++kb) {
    const int n = sym_rounds(kb);
    r = n > r ? n : r;
  }
  return r * kAdjThreads;
}
template <int NF, int KB>
constexpr size_t sym_lds_bytes() {
  const size_t stage = (size_t)2 * sym_buffer_words<KB>() * sizeof(uint4);
  return adj_fft_lds_bytes<NF, KB>() > stage ? adj_fft_lds_bytes<NF, KB>() : stage;
}

// The tuples of one shell ORDER times, a_k += (weight) d_k^(ORDER - 1): most of the gradient of a
// clustered field is theirs.  In the matrix products, k being the largest shell, their weight
// would be 2 w (order 4: 3 w), whose BF16 words are others than those of the whole 3 w (4 w),
// and the rounding of that one weight would set the gradient's error: 20 shells of width 2 at
// 256^3, 0.5 to 3.4 times that of a product with one row per m over 12 inputs, 0.7 to 1.1 in
// this form (128^3 x 8, order 3: 0.9 to 1.3, and 1.0).  equal[k]: the weight as its two
// words hold it, and the lo word.
// They start the accumulators, which costs no register.
template <int PREC, int KB, int ORDER>
__device__ __forceinline__ void sym_equal(float (&acc)[kAdjPB][KB][8], const AdjFields<PREC, KB>& f,
                                          const Operand<PREC> (&fop)[kAdjPB][KB], const float2* __restrict__ equal,
                                          int n_shells, int hh) {
#pragma unroll
  for (int M = 0; M < KB; ++M)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = 16 * M + 8 * hh + r;
      const float2 w = k < n_shells ? equal[k] : make_float2(0.f, 0.f);
#pragma unroll
      for (int pb = 0; pb < kAdjPB; ++pb) {
        const float x = f.F[pb][M][r];
        float y = w.x * x;
        if constexpr (PREC == kBF16) y = fmaf(-w.y, (float)fop[pb][M].lo[r], y);   // what the matrix products drop
        acc[pb][M][r] = (ORDER == 4 ? x * x : x) * y;
      }
    }
}

// COUNT blocks of a chain from chunk FROM (S: upwards; P: FROM-th below kb, downwards).
template <int PREC, int KB, int kb, bool P, int M, int T, int FROM, int COUNT>
__device__ __forceinline__ void sym_chain(f32x16 (&Y)[kAdjPB], const uint4* wv, const Operand<PREC> (&fop)[kAdjPB][KB],
                                          int lane) {
  static_for<COUNT>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int uc = P ? kb - (FROM + i) : FROM + i;
    const uint4* blk = wv + sym_index(kb, P, M, T, uc) * kSymBlockWords;
    const Operand<PREC> Wop = op_from_words<PREC>(blk[lane], blk[64 + lane]);
#pragma unroll
    for (int pb = 0; pb < kAdjPB; ++pb) {
      if constexpr (i == 0) adj_mma_first<PREC>(Y[pb], Wop, fop[pb][uc]);
      else adj_mma<PREC>(Y[pb], Wop, fop[pb][uc]);
    }
  });
}

// One 16-byte word per lane from global memory straight into LDS (consecutive lanes fill
// consecutive words from dst), without a register in between.
__device__ __forceinline__ void sym_copy(const uint4* src, uint4* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// Keeps eight accumulators in program order: without it the compiler delays the
// multiply-adds of a chain until the accumulators' next use, which keeps its Y alive and
// spills (64 shells: 267 registers).
__device__ __forceinline__ void sym_pin(float (&a)[8]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}

// The sum of a column's two lane halves, in lane half HALF; zero in the other (not multiplied by
// zero there: the sum may be infinite or NaN).
template <int HALF>
__device__ __forceinline__ float sym_half_sum(float x) {
  const unsigned own = __float_as_uint(x);
  const auto sw = __builtin_amdgcn_permlane32_swap(HALF == 0 ? own : 0u, HALF == 0 ? 0u : own, false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// a_m += d_k Y[m] and q_k += d_m Y[m] for the rows of a chain.
template <int PREC, int KB, bool P, int M, int T>
__device__ __forceinline__ void sym_add(float (&acc)[kAdjPB][KB][8], float (&q)[2][kAdjPB], const f32x16 (&Y)[kAdjPB],
                                        const float (&dk)[2][kAdjPB], const AdjFields<PREC, KB>& f) {
#pragma unroll
  for (int pb = 0; pb < kAdjPB; ++pb) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      constexpr int lo = M;
      const int Mi = P ? lo : lo + i / 8, t = P ? i / 8 : T, r = i % 8;
      acc[pb][Mi][r] = fmaf(dk[t][pb], Y[pb][i], acc[pb][Mi][r]);
      q[t][pb] = fmaf(f.F[pb][Mi][r], Y[pb][i], q[t][pb]);
    }
    sym_pin(acc[pb][M]);
    if constexpr (!P) sym_pin(acc[pb][M + 1]);
    asm volatile("" : "+v"(q[0][pb]), "+v"(q[1][pb]));
  }
}

// A workgroup of 8 waves owns 512 grid points (two 32-point column blocks per wave) and
// every m; KB = 16-shell blocks of the plan.  The partners' weights pass through LDS in
// stages of sym_stage_pairs pairs, double buffered, with one barrier per stage: the next
// stage is copied from global memory straight into LDS while one is in use.  dense: the
// plan aliases, so no block is empty by the triangle bound.
//
// 512^3, 64 unit shells, BF16: 92.3 ms with every m and a_m = sum_v d_v Y_v, 76.0 ms in
// this form (1.15 PFLOP/s issued); 128^3 x 8, 24 shells: 2.97 -> 2.19 ms.  What is left at
// 512^3: the row transform takes 8 ms, weight copies and barriers 1.5, the q products 6; the
// matrix products alone take about 52 ms at the 1.65 PFLOP/s that the power limit leaves
// for random operands.  16 waves of one column block each: 77.8 ms (before the row
// transform's paired stores: 75.4 with 8 waves).
template <int PREC, int NF, int KB>
__global__ __launch_bounds__(kAdjThreads, 1) void adjoint_sym(const float* __restrict__ D, const uint4* __restrict__ W,
                                                            const float2* __restrict__ equal, int n_shells,
                                                            int dense, long long G, float* __restrict__ A,
                                                            cplx<float>* __restrict__ H2,
                                                            const cplx<float>* __restrict__ tw, Geom g) {
  static_assert(PREC != kFP16, "the FP16 split scales every weight row by its own power of two: adjoint_gemm");
  __shared__ __attribute__((aligned(16))) unsigned char lds[sym_lds_bytes<NF, KB>()];
  auto wst = reinterpret_cast<uint4(*)[sym_buffer_words<KB>()]>(lds);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, col = lane & 31;
  const int b = blockIdx.y;
  const long long xw = (long long)blockIdx.x * kAdjPts + wave * 32 * kAdjPB + col;
  const float* Db = D + (size_t)b * n_shells * G;
  const uint4* Wb = W + (size_t)b * sym_words(n_shells);

  AdjFields<PREC, KB> f;
  adj_load_fields<PREC, KB>(f, Db, G, xw, hh, n_shells, nullptr, b);
#pragma unroll
  for (int k = 0; k < sym_rounds(0); ++k) wst[0][k * kAdjThreads + tid] = Wb[k * kAdjThreads + tid];
  Operand<PREC> fop[kAdjPB][KB];
#pragma unroll
  for (int pb = 0; pb < kAdjPB; ++pb)
#pragma unroll
    for (int uc = 0; uc < KB; ++uc) fop[pb][uc] = make_operand<PREC>(f.F[pb][uc], 1.f);

  float acc[kAdjPB][KB][8];
  sym_equal<PREC, KB, 3>(acc, f, fop, equal + b * 64, n_shells, hh);
  __syncthreads();

  // One stage: copy the next one in, then the pairs of this one.  The two buffers are
  // restrict parameters so that the compiler knows the reads of `now` not to touch the
  // words being copied; otherwise it waits for the copy at the first read.
  auto stage = [&](auto kbc, auto stc, const uint4* __restrict__ now, uint4* __restrict__ next)
      __attribute__((always_inline)) {
    constexpr int kb = decltype(kbc)::value, st = decltype(stc)::value;
    constexpr int PPS = sym_stage_pairs(kb), NST = 8 / PPS, NP = sym_p_chains(kb);
    constexpr int nkb = st + 1 < NST ? kb : kb + 1, nst = st + 1 < NST ? st + 1 : 0;
    constexpr int NR = nkb < KB ? sym_rounds(nkb) : 0;
    const uint4* src = Wb + tid;   // no further stage: words of stage 0, never read
    if constexpr (NR > 0)
      if (16 * nkb + 2 * sym_stage_pairs(nkb) * nst < n_shells)
        src += sym_base(nkb) * kSymBlockWords + nst * sym_stage_words(nkb);
#pragma unroll
    for (int k = 0; k < NR; ++k) sym_copy(src + k * kAdjThreads, next + k * kAdjThreads + 64 * wave);
    static_for<PPS>([&](auto pc) {
      constexpr int p = decltype(pc)::value;
      constexpr int kk = 2 * (PPS * st + p);     // first partner within the block
      constexpr bool first = kk == 0;
      const uint4* wv = now + p * sym_blocks(kb) * kSymBlockWords;
      float dk[2][kAdjPB], q[2][kAdjPB];
#pragma unroll
      for (int pb = 0; pb < kAdjPB; ++pb) {
        dk[0][pb] = __uint_as_float(adj_scalar<PREC, KB, kb, kk>(f, pb));
        dk[1][pb] = __uint_as_float(adj_scalar<PREC, KB, kb, kk + 1>(f, pb));
        q[0][pb] = q[1][pb] = 0.f;
      }
      static_for<NP>([&](auto mc) {
        constexpr int M = NP - 1 - decltype(mc)::value;
        f32x16 Y[kAdjPB];
        sym_chain<PREC, KB, kb, true, M, 0, 0, sym_p_chunks(kb, M, first)>(Y, wv, fop, lane);
        sym_add<PREC, KB, true, M, 0>(acc, q, Y, dk, f);
      });
      if constexpr (kb > 0) {
        static_for<2>([&](auto tc) {
          constexpr int t = decltype(tc)::value;
          f32x16 Y[kAdjPB];
          sym_chain<PREC, KB, kb, false, NP, t, 0, kb + 1>(Y, wv, fop, lane);
          sym_add<PREC, KB, false, NP, t>(acc, q, Y, dk, f);
        });
      }
      if constexpr (NP > 0 && kb > 0) {
        if (dense) {             // the chunks that the triangle bound would empty
          static_for<NP>([&](auto mc) {
            constexpr int M = decltype(mc)::value;
            constexpr int have = sym_p_chunks(kb, M, first), rest = kb + 1 - have;
            if constexpr (rest > 0) {
              f32x16 Y[kAdjPB];
              sym_chain<PREC, KB, kb, true, M, 0, have, rest>(Y, wv, fop, lane);
              sym_add<PREC, KB, true, M, 0>(acc, q, Y, dk, f);
            }
          });
        }
      }
      // a_k += (1/2) sum_m d_m Y_k[m], in the lane half that holds shell k
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int pb = 0; pb < kAdjPB; ++pb) {
          float& a = acc[pb][kb][(kk + t) % 8];
          a = fmaf(0.5f, sym_half_sum<kk / 8>(q[t][pb]), a);
        }
    });
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's part of the next stage is in LDS
    __syncthreads();                      // the next stage is complete; this one is free
  };
  int buf = 0;
  static_for<KB>([&](auto kbc) {
    constexpr int kb = decltype(kbc)::value, PPS = sym_stage_pairs(kb);
    static_for<8 / PPS>([&](auto stc) {
      if (16 * kb + 2 * PPS * decltype(stc)::value >= n_shells) return;
      stage(kbc, stc, wst[buf], wst[buf ^ 1]);
      buf ^= 1;
    });
  });
  adjoint_epilogue<NF, KB>([&](int pb, int j) { return acc[pb][j / 8][j % 8]; },
                           [&](int j) { return 16 * (j / 8) + 8 * hh + j % 8; }, lds, wave, col, b, xw, n_shells, G, A,
                           H2, tw, g);
}

// Order 4, likewise: L = sum_l d_l C_l with C_l the cubic form of the shells up to l, one
// l after the other.  C_l = (terms within shell block 0) + sum over k >= 16 of d_k Q_kl,
// Q_kl = sum_{i <= j <= k} w_ijkl d_i d_j:
//   block 0: T[m] = dC/dd_m = sum_v d_v (sum_{u <= v} W[m][(u, v)] d_u), then
//            a_m += d_l T[m] and a_l += (1/3) sum_m d_m T[m]; its partners v take P(0)
//            chains of one chunk, where the products of q would cost as much as the
//            matrix products, so the third side of a term is a row of its own here;
//   k >= 16: Y = dQ_kl/dd, a_m += d_k d_l Y[m], and q = (1/2) sum_m d_m Y[m] gives
//            a_k += d_l q and a_l += d_k q.
// pmask: per l, the pairs of partners that hold a weight (bit k / 2).  Stages are those of
// order 3, for every l in turn; a pair's blocks are stored for k / 2 <= l / 2 only.
//
// BF16, 256^3, against a_m = sum d_v d_w Y over every m: 14.8 -> 11.6 ms with 24 shells of
// width 2, 85.9 -> 40.7 ms with 40 unit shells, where the last shell blocks hold most of
// the products and a corner of k x k replaces 64 rows x every chunk.
template <int PREC, int NF, int KB>
__global__ __launch_bounds__(kAdjThreads, 1) void adjoint4_sym(const float* __restrict__ D, const uint4* __restrict__ W,
                                                             const float2* __restrict__ equal,
                                                             const int* __restrict__ pmask, int n_shells,
                                                             long long G, float* __restrict__ A,
                                                             cplx<float>* __restrict__ H2,
                                                             const cplx<float>* __restrict__ tw, Geom g) {
  static_assert(PREC != kFP16, "the FP16 split scales every weight row by its own power of two: adjoint4_gemm");
  __shared__ __attribute__((aligned(16))) unsigned char lds[sym_lds_bytes<NF, KB>()];
  auto wst = reinterpret_cast<uint4(*)[sym_buffer_words<KB>()]>(lds);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, col = lane & 31;
  const int b = blockIdx.y;
  const long long xw = (long long)blockIdx.x * kAdjPts + wave * 32 * kAdjPB + col;
  const float* Db = D + (size_t)b * n_shells * G;
  const int n_words = sym4_blocks(n_shells) * kSymBlockWords;
  const uint4* Wb = W + (size_t)b * n_words;

  AdjFields<PREC, KB> f;
  adj_load_fields<PREC, KB>(f, Db, G, xw, hh, n_shells, nullptr, b);
#pragma unroll
  for (int k = 0; k < sym_rounds(0); ++k) {
    const int i = k * kAdjThreads + tid;
    wst[0][i] = Wb[min(i, n_words - 1)];
  }
  Operand<PREC> fop[kAdjPB][KB];
#pragma unroll
  for (int pb = 0; pb < kAdjPB; ++pb)
#pragma unroll
    for (int uc = 0; uc < KB; ++uc) fop[pb][uc] = make_operand<PREC>(f.F[pb][uc], 1.f);
  float acc[kAdjPB][KB][8];
  sym_equal<PREC, KB, 4>(acc, f, fop, equal + b * 64, n_shells, hh);
  // d_l at the lane's points and the mask of l, one l ahead
  float dl_next[kAdjPB];
#pragma unroll
  for (int pb = 0; pb < kAdjPB; ++pb) dl_next[pb] = Db[xw + 32 * pb];
  int pm_next = pmask[0];
  __syncthreads();

  float dl[kAdjPB], al[kAdjPB];
  unsigned pm = 0;
  int l = 0, base = 0;    // first weight word of l
  // One stage (see adjoint_sym): words past the plan's last, and of pairs that pmask
  // excludes, are copied and never read.
  auto stage = [&](auto kbc, auto stc, const uint4* __restrict__ now, uint4* __restrict__ next)
      __attribute__((always_inline)) {
    constexpr int kb = decltype(kbc)::value, st = decltype(stc)::value;
    constexpr int PPS = sym_stage_pairs(kb), NST = 8 / PPS, NP = sym_p_chains(kb);
    constexpr int nkb = st + 1 < NST ? kb : kb + 1, nst = st + 1 < NST ? st + 1 : 0;
    auto copy = [&](int from, auto rounds) {
#pragma unroll
      for (int k = 0; k < decltype(rounds)::value; ++k)
        sym_copy(Wb + min(from + k * kAdjThreads + tid, n_words - 1), next + k * kAdjThreads + 64 * wave);
    };
    bool same = false;    // whether the next stage belongs to this l
    if constexpr (nkb < KB) {
      same = 16 * nkb + 2 * sym_stage_pairs(nkb) * nst <= l;
      if (same)
        copy(base + sym_base(nkb) * kSymBlockWords + nst * sym_stage_words(nkb),
             std::integral_constant<int, sym_rounds(nkb)>{});
    }
    if (!same) copy(base + sym4_blocks_of(l) * kSymBlockWords, std::integral_constant<int, sym_rounds(0)>{});
    if constexpr (kb == 0) {
      float T[kAdjPB][8];
#pragma unroll
      for (int pb = 0; pb < kAdjPB; ++pb)
#pragma unroll
        for (int r = 0; r < 8; ++r) T[pb][r] = 0.f;
      auto pair = [&](auto pc) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
        f32x16 Y[kAdjPB];
        sym_chain<PREC, KB, 0, true, 0, 0, 0, 1>(Y, now + p * kSymBlockWords, fop, lane);
#pragma unroll
        for (int pb = 0; pb < kAdjPB; ++pb) {
          const float d0 = __uint_as_float(adj_scalar<PREC, KB, 0, 2 * p>(f, pb));
          const float d1 = __uint_as_float(adj_scalar<PREC, KB, 0, 2 * p + 1>(f, pb));
#pragma unroll
          for (int r = 0; r < 8; ++r) T[pb][r] = fmaf(d1, Y[pb][8 + r], fmaf(d0, Y[pb][r], T[pb][r]));
          sym_pin(T[pb]);
        }
      };
      if ((pm & 0xff) == 0xff) {
        static_for<8>(pair);          // straight-line when every pair holds a weight
      } else {
        static_for<8>([&](auto pc) {
          if ((pm >> decltype(pc)::value) & 1) pair(pc);
        });
      }
#pragma unroll
      for (int pb = 0; pb < kAdjPB; ++pb) {
        float e = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          acc[pb][0][r] = fmaf(dl[pb], T[pb][r], acc[pb][0][r]);
          e = fmaf(f.F[pb][0][r], T[pb][r], e);
        }
        al[pb] = (1.0f / 3.0f) * e;
      }
    } else {
      static_for<PPS>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        constexpr int kk = 2 * (PPS * st + p);
        if (!((pm >> (8 * kb + kk / 2)) & 1)) return;
        const uint4* wv = now + p * sym_blocks(kb) * kSymBlockWords;
        float dk[2][kAdjPB], sc[2][kAdjPB], q[2][kAdjPB];
#pragma unroll
        for (int pb = 0; pb < kAdjPB; ++pb) {
          dk[0][pb] = __uint_as_float(adj_scalar<PREC, KB, kb, kk>(f, pb));
          dk[1][pb] = __uint_as_float(adj_scalar<PREC, KB, kb, kk + 1>(f, pb));
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            sc[t][pb] = dk[t][pb] * dl[pb];
            q[t][pb] = 0.f;
          }
        }
        static_for<NP>([&](auto mc) {
          constexpr int M = NP - 1 - decltype(mc)::value;
          f32x16 Y[kAdjPB];
          sym_chain<PREC, KB, kb, true, M, 0, 0, kb + 1>(Y, wv, fop, lane);
          sym_add<PREC, KB, true, M, 0>(acc, q, Y, sc, f);
        });
        static_for<2>([&](auto tc) {
          constexpr int t = decltype(tc)::value;
          f32x16 Y[kAdjPB];
          sym_chain<PREC, KB, kb, false, NP, t, 0, kb + 1>(Y, wv, fop, lane);
          sym_add<PREC, KB, false, NP, t>(acc, q, Y, sc, f);
        });
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int pb = 0; pb < kAdjPB; ++pb) {
            al[pb] = fmaf(0.5f * dk[t][pb], q[t][pb], al[pb]);   // this lane half's rows
            float& a = acc[pb][kb][(kk + t) % 8];
            a = fmaf(0.5f * dl[pb], sym_half_sum<kk / 8>(q[t][pb]), a);
          }
      });
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's part of the next stage is in LDS
    __syncthreads();                      // the next stage is complete; this one is free
  };
  int buf = 0;
  for (l = 0; l < n_shells; ++l) {
#pragma unroll
    for (int pb = 0; pb < kAdjPB; ++pb) dl[pb] = dl_next[pb];
    pm = pm_next;
    const int l1 = min(l + 1, n_shells - 1);
#pragma unroll
    for (int pb = 0; pb < kAdjPB; ++pb) dl_next[pb] = Db[(size_t)l1 * G + xw + 32 * pb];
    pm_next = pmask[l1];
    static_for<KB>([&](auto kbc) {
      constexpr int kb = decltype(kbc)::value, PPS = sym_stage_pairs(kb);
      static_for<8 / PPS>([&](auto stc) {
        if (16 * kb + 2 * PPS * decltype(stc)::value > l) return;
        stage(kbc, stc, wst[buf], wst[buf ^ 1]);
        buf ^= 1;
      });
    });
    // a_l, in the lane half that holds shell l
    const bool mine = hh == ((l >> 3) & 1);
#pragma unroll
    for (int pb = 0; pb < kAdjPB; ++pb) {
      const unsigned own = __float_as_uint(al[pb]);
      const auto sw = __builtin_amdgcn_permlane32_swap(own, own, false, false);
      al[pb] = mine ? __uint_as_float(sw[0]) + __uint_as_float(sw[1]) : 0.f;
    }
#pragma unroll
    for (int M = 0; M < KB; ++M)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool here = l >> 4 == M && (l & 7) == r;   // uniform: no indexed registers
#pragma unroll
        for (int pb = 0; pb < kAdjPB; ++pb) acc[pb][M][r] += here ? al[pb] : 0.f;
      }
    base += sym4_blocks_of(l) * kSymBlockWords;
  }
  adjoint_epilogue<NF, KB>([&](int pb, int j) { return acc[pb][j / 8][j % 8]; },
                           [&](int j) { return 16 * (j / 8) + 8 * hh + j % 8; }, lds, wave, col, b, xw, n_shells, G, A,
                           H2, tw, g);
}

template <int PREC>
hipError_t launch_adjoint_sym_prec(const float* D, const uint4* W, const float2* equal, int n_shells, int dense,
                                   long long G, float* A, cplx<float>* H2, const cplx<float>* tw, Geom g, int batch,
                                   hipStream_t st) {
  dim3 grid((unsigned)(G / kAdjPts), batch);
#define L2(NF, KB) hipLaunchKernelGGL((adjoint_sym<PREC, NF, KB>), grid, dim3(kAdjThreads), 0, st, D, W, equal, \
                                      n_shells, dense, G, A, H2, tw, g)
#define L(NF)                          \
  do {                                 \
    if (n_shells <= 16) L2(NF, 1);     \
    else if (n_shells <= 32) L2(NF, 2); \
    else if (n_shells <= 48) L2(NF, 3); \
    else L2(NF, 4);                    \
  } while (0)
  switch (g.N) {
    case 32: L(32); break;
    case 64: L(64); break;
    case 128: L(128); break;
    case 256: L(256); break;
    case 512: L(512); break;
    default: L(0); break;
  }
#undef L
#undef L2
  return hipGetLastError();
}

template <int PREC>
hipError_t launch_adjoint4_sym_prec(const float* D, const uint4* W, const float2* equal, const int* pmask,
                                    int n_shells, long long G, float* A, cplx<float>* H2, const cplx<float>* tw,
                                    Geom g, int batch, hipStream_t st) {
  dim3 grid((unsigned)(G / kAdjPts), batch);
#define L2(NF, KB) hipLaunchKernelGGL((adjoint4_sym<PREC, NF, KB>), grid, dim3(kAdjThreads), 0, st, D, W, equal, \
                                      pmask, n_shells, G, A, H2, tw, g)
#define L(NF)                           \
  do {                                  \
    if (n_shells <= 16) L2(NF, 1);      \
    else if (n_shells <= 32) L2(NF, 2); \
    else if (n_shells <= 48) L2(NF, 3); \
    else L2(NF, 4);                     \
  } while (0)
  switch (g.N) {
    case 32: L(32); break;
    case 64: L(64); break;
    case 128: L(128); break;
    case 256: L(256); break;
    case 512: L(512); break;
    default: L(0); break;
  }
#undef L
#undef L2
  return hipGetLastError();
}

}  // namespace ps
