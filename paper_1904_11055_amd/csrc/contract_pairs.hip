// Product-sum contraction, order 4 in split FP16 (up to 64 shells): pair x pair.
//
// Every pair block's operand is formed once per 32-point half stage into LDS and read from
// there by the tiles.  What bounds it is the LDS: a tile's three matrix products take 48
// cycles of one SIMD, and reading its B operand alone 16 cycles of the LDS that four SIMDs
// share; a block's forming moves 6 KB.  So a slot is several A blocks against one B block,
// whose read serves them all (neighbouring A blocks need nearly the same B blocks).
//
// Up to 28 pair blocks (29 shells): slots of two, 16 waves, both halves of a stage in LDS.
// While one half is multiplied the next is formed, by half of a SIMD's waves before they
// multiply and by the others after, so that LDS, VALU and matrix cores have work at any time;
// the B block of the next slot is read a slot ahead.  More blocks: slots of four, 8 waves with
// 160 accumulators each, one half in LDS, and groups of tiles over rectangles of blocks, each
// of which forms only what its tiles need.  (Slots of four on the small plans: 4.13 ms for 24
// shells where slots of two take 3.91.)  The staged fields are loaded a stage ahead.
//
// 256^3, against one tile per operand read and forming in a phase of its own: 9 shells 0.82 ->
// 0.70 ms, 16 shells 1.80 -> 1.44, 24 shells of width 2 5.5 -> 3.91 (matrix products alone
// 1.9), 30 unit shells 12.0 -> 10.1, 40 31.0 -> 26.1 (15); no gain at 20 and 21 (2.4, 2.8).
#include "mfma_ops.h"

namespace ps {

// W waves; slots of T A blocks against one B block; DOUBLE: both halves of a stage in LDS, for
// groups of up to k4Blocks / 2 pair blocks, else one half at a time, formed and multiplied in turn.
template <int W, int NS, int T, bool DOUBLE>
__global__ __launch_bounds__(64 * W, 1) void contract_pairs(Ctr4Params p) {
  __shared__ uint4 opHi[2][2][kMaxBlk + 1][64];   // [buffer][half][shell block][lane]; block n_blk stays zero
  __shared__ uint4 opLo[2][2][kMaxBlk + 1][64];
  constexpr int kThreads = 64 * W, kMoves = 1024 / kThreads;
  constexpr int kBlocks = DOUBLE ? k4Blocks / 2 : k4Blocks;
  __shared__ uint4 pairOp[DOUBLE ? 2 : 1][kBlocks][2][64];   // [half][pair block][hi, lo][lane]
  __shared__ float lds_scale[kMaxBlk * 16];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15;
  const int chunk = blockIdx.x, group = blockIdx.y, b = blockIdx.z;

  for (int i = tid; i < kMaxBlk * 16; i += kThreads)
    lds_scale[i] = i < p.n_shells ? ldexpf(1.0f, shell_scale_exp(p.absmax, b * p.n_shells + i)) : 0.f;
  for (int i = tid; i < 4 * (kMaxBlk + 1) * 64; i += kThreads) {
    const int bh = i / ((kMaxBlk + 1) * 64), kb = (i / 64) % (kMaxBlk + 1), ln = i % 64;
    if (kb * 16 + (ln & 15) >= p.n_shells) {
      opHi[bh >> 1][bh & 1][kb][op_slot(ln)] = make_uint4(0, 0, 0, 0);
      opLo[bh >> 1][bh & 1][kb][op_slot(ln)] = make_uint4(0, 0, 0, 0);
    }
  }

  // staging: thread t moves float4 #t (and #t + 512) of the (64 shells x 64 points) slice
  const float* src[kMoves];
  bool st_on[kMoves];
#pragma unroll
  for (int f = 0; f < kMoves; ++f) {
    const int st_row = (tid + f * kThreads) >> 4;
    st_on[f] = st_row < p.n_shells;
    src[f] = p.D + ((size_t)b * p.n_shells + (st_on[f] ? st_row : 0)) * p.G + (long long)chunk * p.ksteps * kKStep +
             (tid & 15) * 4;
  }
  float4 pre[kMoves];
  auto stage_load = [&](int ks) {
#pragma unroll
    for (int f = 0; f < kMoves; ++f)
      if (st_on[f]) pre[f] = *reinterpret_cast<const float4*>(src[f] + (size_t)ks * kKStep);
  };
  auto stage_store = [&](int buf) {
#pragma unroll
    for (int f = 0; f < kMoves; ++f) {
      if (!st_on[f]) continue;
      const int st_row = (tid + f * kThreads) >> 4, st_col = (tid & 15) * 4;
      const float sc = lds_scale[st_row];
      const float4 v = make_float4(pre[f].x * sc, pre[f].y * sc, pre[f].z * sc, pre[f].w * sc);
      uint2 hi, lo;
      split4<kFP16>(v, 1.f, hi, lo);
      const int h = st_col >> 5, kb = st_row >> 4, half = (st_col >> 2) & 1;
      const int ln = op_slot((((st_col & 31) >> 3) << 4) | (st_row & 15));
      reinterpret_cast<uint2*>(&opHi[buf][h][kb][ln])[half] = hi;
      reinterpret_cast<uint2*>(&opLo[buf][h][kb][ln])[half] = lo;
    }
  };
  stage_load(0);
  __syncthreads();
  stage_store(0);

  // the pair blocks this wave forms, of the group's own: dealt from the last wave on, so that
  // where there are fewer blocks than waves the waves that hold the tiles form none
  constexpr int kForm = (kBlocks + W - 1) / W;
  const int n_local = p.grp_nblk[group];
  int fuv[kForm];
#pragma unroll
  for (int f = 0; f < kForm; ++f) {
    const int t = W - 1 - wave + f * W;
    const int w = t < n_local ? p.pair_uv[16 * p.grp_blk[group * k4Blocks + t] + row] : 0;
    fuv[f] = (w & 0xff) | (((w >> 16) & 0xff) << 8);
  }
  auto form = [&](int buf, int h) {   // half h of the staged buffer
#pragma unroll
    for (int f = 0; f < kForm; ++f) {
      const int t = W - 1 - wave + f * W;
      if (t < n_local) {
        const Operand<kFP16> o = form_pair_f16(opHi[buf][h], opLo[buf][h], fuv[f], lane);
        op_to_words<kFP16>(o, pairOp[DOUBLE ? h : 0][t][0][lane], pairOp[DOUBLE ? h : 0][t][1][lane]);
      }
    }
  };
  // slots (see Ctr4Params)
  const size_t gw = (size_t)group * W + wave;
  int sa[NS], sb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    sa[s] = __builtin_amdgcn_readfirstlane(p.slot_a[gw * NS + s]);
    sb[s] = __builtin_amdgcn_readfirstlane(p.slot_b[gw * NS + s]);
  }
  f32x4 acc[NS][T];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int a = 0; a < T; ++a) acc[s][a] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int h) {
    auto words = [&](int i) {
      return op_from_words<kFP16>(pairOp[DOUBLE ? h : 0][i][0][lane], pairOp[DOUBLE ? h : 0][i][1][lane]);
    };
    Operand<kFP16> A[T], ahead;
    if constexpr (T == 2) ahead = words(sb[0] < 0 ? 0 : sb[0] & 0xff);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      // the slot words are re-read from SGPRs here: the LDS addresses of every slot, kept
      // over the loop, would spill
      int wb = sb[s];
      asm volatile("" : "+s"(wb));
      if (wb < 0) break;
      if (wb & 0x100) {
        int wa = sa[s];
        asm volatile("" : "+s"(wa));
#pragma unroll
        for (int a = 0; a < T; ++a) A[a] = words((wa >> (8 * a)) & 0xff);
      }
      // two tiles do not cover the latency of the next B block's reads: it is read a slot ahead
      Operand<kFP16> B;
      if constexpr (T == 2) {
        B = ahead;
        int wn = sb[s + 1 < NS ? s + 1 : s];
        asm volatile("" : "+s"(wn));
        ahead = words(wn < 0 ? 0 : wn & 0xff);
      } else {
        B = words(wb & 0xff);
      }
      if (T == 2 || (wb & 0x200))
        static_for<3>([&](auto term) {
          mma_term<kFP16, decltype(term)::value>(acc[s][0], A[0], B);
          mma_term<kFP16, decltype(term)::value>(acc[s][1], A[1], B);
        });
      if constexpr (T == 4)
        if (wb & 0x400)
          static_for<3>([&](auto term) {
            mma_term<kFP16, decltype(term)::value>(acc[s][2], A[2], B);
            mma_term<kFP16, decltype(term)::value>(acc[s][3], A[3], B);
          });
    }
  };
  // of the waves of a SIMD (w, w + 4, ...) half form while the others multiply
  const bool form_first = (wave >> 2) & 1;
  if (p.ksteps > 1) stage_load(1);
  __syncthreads();
  form(0, 0);
  __syncthreads();

  for (int ks = 0; ks < p.ksteps; ++ks) {
    const int cur = ks & 1;
    const bool more = ks + 1 < p.ksteps;
    if constexpr (DOUBLE) {
      if (form_first) form(cur, 1);
      multiply(0);
      if (!form_first) form(cur, 1);
      if (more) stage_store(cur ^ 1);
      if (ks + 2 < p.ksteps) stage_load(ks + 2);
      __syncthreads();   // half 1's operands are in LDS; half 0's are free
      if (more && form_first) form(cur ^ 1, 0);
      multiply(1);
      if (more && !form_first) form(cur ^ 1, 0);
      __syncthreads();
    } else {
      multiply(0);
      if (more) stage_store(cur ^ 1);
      if (ks + 2 < p.ksteps) stage_load(ks + 2);
      __syncthreads();
      form(cur, 1);
      __syncthreads();
      multiply(1);
      __syncthreads();
      if (more) form(cur ^ 1, 0);
      __syncthreads();
    }
  }

  float* out = p.partials + ((size_t)b * p.n_chunks + chunk) * (size_t)p.n_tiles * 256;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int a = 0; a < T; ++a) {
      const int t = p.slot_tile[(gw * NS + s) * T + a];
      if (t >= 0) *reinterpret_cast<f32x4*>(out + (size_t)t * 256 + 4 * lane) = acc[s][a];
    }
  }
}

hipError_t launch_contract_pairs(const Ctr4Params& p, int n_groups, int batch, hipStream_t st) {
  if (p.n_blk > kMaxBlk) return hipErrorInvalidValue;
  const dim3 grid(p.n_chunks, n_groups, batch);
  auto go = [&](auto kernel, int waves) { hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, st, p); };
  if (p.wide) go(contract_pairs<k4Wide.waves, k4Wide.slots, k4Wide.tiles, false>, k4Wide.waves);
  else go(contract_pairs<k4Narrow.waves, k4Narrow.slots, k4Narrow.tiles, true>, k4Narrow.waves);
  return hipGetLastError();
}

}  // namespace ps
