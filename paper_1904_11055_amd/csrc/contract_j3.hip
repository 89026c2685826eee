#include "mfma_ops.h"

namespace ps {

// ---------------------------------------------------------------------------
// Order 3, products aligned to shell blocks (FP16: up to 64 shells; FP32, BF16: up to 16).
//   S[i, j, k] = sum_x d_i d_j d_k, i <= j <= k, by the 16-shell block jb of the middle shell.
// Every 16 x 16 tile is a product operand (16 rows d_p d_j) times the plain operand of a
// shell block held in registers.  What fixes the rows of the product operand:
//   jb = 0, 1, i in block jb:  rows i <= j, columns k >= jb's block;
//   jb = 2, 3, k in block jb:  rows k >= j, columns i <= jb's block;
//   jb = 1, i in block 0:      rows i, columns k;
//   jb = 2, k in block 3:      rows k, columns i.
// In the first two a shell j fills only part of the 16 rows, so two shells whose rows add
// up to 16 share one operand (rows from either end): j = a and 14 - a of the block (for
// the second kind mirrored, 15 - a and 1 + a), a = 0..6 for wave a, and the full j = 15
// (j = 0) for wave 7.  The half-full j = 7 (j = 8) of two blocks share a ninth operand,
// whose four columns blocks go to waves 0 to 3, two each.  64 unit shells take 186 tiles
// instead of 260 with one operand per j, and 66 different operands per step instead of 96
// (512^3: 47.5 ms before).  Both rows of a product come from LDS words at lane-dependent
// slots, the rest of a 32-point step from registers.  A per-wave mask says which tiles
// hold a candidate tuple.
// ---------------------------------------------------------------------------
constexpr int kJThreads = 64 * kJWaves;
static_assert(kSlots == kSlotsHost && kSlots4 == kSlots4Host && kSlotsMax == kSlotsMaxHost && kMaxBlk == kMaxBlkHost &&
                  kCtrWaves == kCtrWavesHost,
              "host and device tile tables agree");


// NBLK: 16-shell blocks of the plan.  ALL: every wave uses every kind of product operand, so
// that a step is straight-line code; otherwise the unused ones are skipped, one branch each
// (512^3, 64 shells: 34.7 against 36.3 ms; a multipole plan of 46 fields, half of whose
// operands are unused: 0.34 against 0.27 ms with the branches).
//
// 512^3, 64 shells (the start of these measurements: 47.5 ms): 37.9 ms with shared operands,
// 34.7 with the next step's fields split in the middle of the step instead of before its
// barrier.  What is left: without staging 28 ms, without forming products 29.7, the matrix
// products alone 20.  128^3 x 8, 24 shells: 1.99 -> 0.98 ms.
//
// FP16 forms the products from the split words; FP32 and BF16, on plans of one block, from
// float32 values, which BF16 splits afterwards, as the pair tiles of contract_tiles do.
// 256^3, 13 shells, FP32: 0.89 -> 0.75 ms.
template <int PREC, int NBLK, bool ALL>
__global__ __launch_bounds__(kJThreads, 1) void contract_j3(CtrJParams p) {
  static_assert(PREC == kFP16 || (NBLK == 1 && !ALL), "FP32 and BF16: plans of one block");
  // [buffer][K-step][shell block][lane]: the operand's 16-byte words, FP16 hi and lo, else
  // the float32 values 0..3 and 4..7; BF16 keeps the split words beside them
  __shared__ uint4 opHi[2][2][kMaxBlk][64];
  __shared__ uint4 opLo[2][2][kMaxBlk][64];
  constexpr int kSp = PREC == kBF16 ? kMaxBlk * 64 : 1;
  __shared__ uint4 spHi[2][2][kSp];
  __shared__ uint4 spLo[2][2][kSp];
  __shared__ float lds_scale[kMaxBlk * 16];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int my_slot = op_slot(lane);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunk = blockIdx.x;
  const int b = blockIdx.z;

  for (int i = tid; i < kMaxBlk * 16; i += kJThreads)
    lds_scale[i] = PREC != kFP16     ? 1.f
                   : i < p.n_shells ? ldexpf(1.0f, shell_scale_exp(p.absmax, b * p.n_shells + i))
                                    : 0.f;
  for (int i = tid; i < 4 * kMaxBlk * 64; i += kJThreads) {
    const int bh = i / (kMaxBlk * 64), kb = (i / 64) % kMaxBlk, ln = i % 64;
    if (kb * 16 + (ln & 15) >= p.n_shells) {
      opHi[bh >> 1][bh & 1][kb][op_slot(ln)] = make_uint4(0, 0, 0, 0);
      opLo[bh >> 1][bh & 1][kb][op_slot(ln)] = make_uint4(0, 0, 0, 0);
      if constexpr (PREC == kBF16) {
        spHi[bh >> 1][bh & 1][kb * 64 + op_slot(ln)] = make_uint4(0, 0, 0, 0);
        spLo[bh >> 1][bh & 1][kb * 64 + op_slot(ln)] = make_uint4(0, 0, 0, 0);
      }
    }
  }
  __syncthreads();

  // staging: float4 #f of the (16 NBLK shells x 64 points) slice, f = tid, tid + kJThreads;
  // rows past the plan's shells reread shell 0 and store zeros
  constexpr int kF4 = (NBLK + 1) / 2;   // float4 per thread per stage
  const long long x_base = (long long)chunk * p.ksteps * kKStep;
  const float* src[kF4];
  float st_scale[kF4];
  bool st_on[kF4];
#pragma unroll
  for (int f = 0; f < kF4; ++f) {
    const int idx = tid + f * kJThreads, row = idx >> 4;
    st_on[f] = row < p.n_shells;
    st_scale[f] = lds_scale[row];
    src[f] = p.D + ((size_t)b * p.n_shells + (st_on[f] ? row : 0)) * p.G + x_base + (idx & 15) * 4;
  }
  float4 pre[kF4];
  auto stage_load = [&](int ks) {
#pragma unroll
    for (int f = 0; f < kF4; ++f) pre[f] = *reinterpret_cast<const float4*>(src[f] + (size_t)ks * kKStep);
  };
  auto stage_store = [&](int buf, int f) {
    const int idx = tid + f * kJThreads, row = idx >> 4, col = (idx & 15) * 4;
    const float sc = st_scale[f];
    float4 v = st_on[f] ? pre[f] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int h = col >> 5, kb = row >> 4, ln = op_slot((((col & 31) >> 3) << 4) | (row & 15)), half = (col >> 2) & 1;
    if constexpr (PREC == kFP16) v = make_float4(v.x * sc, v.y * sc, v.z * sc, v.w * sc);
    else *reinterpret_cast<float4*>(half ? &opLo[buf][h][kb][ln] : &opHi[buf][h][kb][ln]) = v;
    if constexpr (PREC != kFP32) {
      uint2 hi, lo;
      split4<PREC>(v, 1.f, hi, lo);
      reinterpret_cast<uint2*>(PREC == kFP16 ? &opHi[buf][h][kb][ln] : &spHi[buf][h][(kb * 64 + ln) % kSp])[half] = hi;
      reinterpret_cast<uint2*>(PREC == kFP16 ? &opLo[buf][h][kb][ln] : &spLo[buf][h][(kb * 64 + ln) % kSp])[half] = lo;
    }
  };
  stage_load(0);
#pragma unroll
  for (int f = 0; f < kF4; ++f) stage_store(0, f);
  __syncthreads();

  const unsigned m0 = __builtin_amdgcn_readfirstlane(p.slot_mask[wave]);
  // LDS words of the two rows of a product, by kind (block offsets are added as constants)
  const int row = lane & 15, grp = lane & 0x30;
  const int a = wave < 7 ? wave : 15;
  const bool lead = row <= a;                                   // rows of the first shell of the pair
  const int ap = op_slot(grp | (lead ? row : 15 - row)), aj = op_slot(grp | (lead ? a : 14 - a));
  const int bp = op_slot(grp | (lead ? 15 - row : row)), bj = op_slot(grp | (lead ? 15 - a : 1 + a));
  const int uj[2] = {op_slot(grp | wave), op_slot(grp | (wave + 8))};   // single shells j = wave, wave + 8
  const bool low = row < 8;
  const int xblk = wave < 2 ? (low ? 0 : 1) : (low ? 3 : 2);
  const int xp = 64 * xblk + op_slot(grp | (low == (wave < 2) ? row : 15 - row));
  const int xj = 64 * xblk + op_slot(grp | (wave < 2 ? 7 : 8));
  f32x4 acc[kJSlots];
#pragma unroll
  for (int s = 0; s < kJSlots; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int ks = 0; ks < p.ksteps; ++ks) {
    const int cur = ks & 1;
    stage_load(min(ks + 1, p.ksteps - 1));   // the last step stores a copy that nothing reads
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // the mask is re-read from an SGPR every half step (scalar bit tests) instead of being
      // kept as precomputed lane masks, which would spill into VGPR lanes
      unsigned mm = m0;
      asm volatile("" : "+s"(mm));
      mm = __builtin_amdgcn_readfirstlane(mm);
      const uint4* hi = &opHi[cur][h][0][0];
      const uint4* lo = &opLo[cur][h][0][0];
      constexpr int WP = PREC == kFP16 ? kFP16 : kFP32;           // what a product is formed from
      auto words = [&](int i) { return op_from_words<WP>(hi[i], lo[i]); };
      auto product = [&](const Operand<WP>& x, const Operand<WP>& y) {
        if constexpr (PREC == kFP16) {
          return pair_f16(x, y);
        } else {
          float z[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) z[r] = x.v[r] * y.v[r];
          return make_operand<PREC>(z, 1.f);
        }
      };
      Operand<PREC> Bop[NBLK];
#pragma unroll
      for (int kb = 0; kb < NBLK; ++kb) {
        if constexpr (PREC == kBF16)
          Bop[kb] = op_from_words<PREC>(spHi[cur][h][64 * kb + my_slot], spLo[cur][h][64 * kb + my_slot]);
        else
          Bop[kb] = words(64 * kb + my_slot);
      }
      // Slots s0 .. s0 + CNT - 1: the product operand times the blocks x0, x0 + 1, ... of the
      // plan, the products of the split in turn, so that none waits for the one before it.
      auto tiles = [&](auto s0c, auto cntc, auto x0c, auto&& form) {
        constexpr int s0 = decltype(s0c)::value, x0 = decltype(x0c)::value;
        constexpr int CNT = decltype(cntc)::value < NBLK - x0 ? decltype(cntc)::value : NBLK - x0;
        if constexpr (CNT > 0) {
          if (!ALL && (mm & (((1u << CNT) - 1) << s0)) == 0) return;
          const Operand<PREC> A = form();
          if constexpr (PREC == kFP32) {           // a tile is 256 cycles of products: worth a branch
            static_for<CNT>([&](auto c) {
              constexpr int s = s0 + decltype(c)::value;
              if ((mm >> s) & 1) mma<PREC>(acc[s], A, Bop[x0 + decltype(c)::value]);
            });
          } else {
            static_for<3>([&](auto term) {
              static_for<CNT>([&](auto c) {
                mma_term<PREC, decltype(term)::value>(acc[s0 + decltype(c)::value], A, Bop[x0 + decltype(c)::value]);
              });
            });
          }
        }
      };
      // one tile that the triangle bound empties for all but the last shell of a block
      auto corner = [&](auto sc, auto xc, auto&& form) {
        constexpr int s0 = decltype(sc)::value, x = decltype(xc)::value;
        if constexpr (x < NBLK)
          if ((mm >> s0) & 1) mma<PREC>(acc[s0], form(), Bop[x]);
      };
#define PS_C(v) std::integral_constant<int, v>{}
      auto diag0 = [&] { return product(words(ap), words(aj)); };
      tiles(PS_C(kJDiag0), PS_C(2), PS_C(0), diag0);
      tiles(PS_C(kJDiag1), PS_C(3), PS_C(1), [&] { return product(words(64 + ap), words(64 + aj)); });
      if constexpr (NBLK > 2)
        tiles(PS_C(kJDiag2), PS_C(3), PS_C(0), [&] { return product(words(128 + bp), words(128 + bj)); });
      if constexpr (NBLK > 3)
        tiles(PS_C(kJDiag3), PS_C(4), PS_C(0), [&] { return product(words(192 + bp), words(192 + bj)); });
      // the next step's fields, split under the products
      if (h == 1) stage_store(cur ^ 1, 0);
      static_for<2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if (h == 1 && q == 1 && kF4 == 2) stage_store(cur ^ 1, kF4 - 1);
        if constexpr (NBLK > 1)
          tiles(PS_C(kJLow + 3 * q), PS_C(2), PS_C(1), [&] { return product(Bop[0], words(64 + uj[q])); });
        if constexpr (NBLK > 3)
          tiles(PS_C(kJHigh + 3 * q), PS_C(3), PS_C(0), [&] { return product(Bop[3], words(128 + uj[q])); });
      });
      if ((mm >> kJShared) != 0) {
        if (wave & 1) tiles(PS_C(kJShared), PS_C(2), PS_C(2), [&] { return product(words(xp), words(xj)); });
        else tiles(PS_C(kJShared), PS_C(2), PS_C(0), [&] { return product(words(xp), words(xj)); });
      }
      corner(PS_C(kJDiag0 + 2), PS_C(2), diag0);
      corner(PS_C(kJDiag0 + 3), PS_C(3), diag0);
      if constexpr (NBLK > 3) {
        corner(PS_C(kJLow + 2), PS_C(3), [&] { return product(Bop[0], words(64 + uj[0])); });
        corner(PS_C(kJLow + 5), PS_C(3), [&] { return product(Bop[0], words(64 + uj[1])); });
      }
#undef PS_C
    }
    __syncthreads();
  }

  const int* my_tiles = p.tile_of_slot + wave * kJSlots;
  float* out = p.partials + ((size_t)b * p.n_chunks + chunk) * (size_t)p.n_tiles * 256;
#pragma unroll
  for (int s = 0; s < kJSlots; ++s) {
    if (!((m0 >> s) & 1)) continue;
    *reinterpret_cast<f32x4*>(out + (size_t)my_tiles[s] * 256 + 4 * lane) = acc[s];
  }
}

hipError_t launch_contract_j3(int prec, const CtrJParams& p, int batch, hipStream_t st) {
  dim3 grid(p.n_chunks, 1, batch);
#define L(PREC, NBLK, ALL) hipLaunchKernelGGL((contract_j3<PREC, NBLK, ALL>), grid, dim3(kJThreads), 0, st, p)
  if (prec != kFP16) {
    if (p.n_blk != 1) return hipErrorInvalidValue;
    if (prec == kFP32) L(kFP32, 1, false); else L(kBF16, 1, false);
    return hipGetLastError();
  }
  switch (p.n_blk) {
    case 1: L(kFP16, 1, false); break;
    case 2: L(kFP16, 2, false); break;
    case 3: if (p.all_used) L(kFP16, 3, true); else L(kFP16, 3, false); break;
    case 4: if (p.all_used) L(kFP16, 4, true); else L(kFP16, 4, false); break;
    default: return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

}  // namespace ps
