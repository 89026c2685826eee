// Product-sum contraction, orders 5 (pair x triple) and 6 (triple x triple).
//
// Tiles of 16 A rows x 16 B rows as in contract_tiles_lo.hip, but what bounds them is the
// VALU and the LDS: a triple row takes three row reads, 16 multiplies and the split for
// every 8 points.  So each row block is formed once per 64-point stage: the A blocks of the
// tile group into LDS, shared by the waves, and a B block in the registers of the one wave
// that holds all its tiles (a unit).  Two workgroups of 8 waves fit a CU (LDS below 64 KB:
// 11 A blocks per group), one forming while the other multiplies.  256^3, against a
// formation per tile: order 5 with 16 shells (95 tiles over 9 A and 51 B blocks) FP16 8.35 ->
// 4.75 ms, BF16 6.49 -> 4.08, FP32 8.48 -> 7.12; order 6 with 8 shells (19 tiles over 8 and 8)
// FP16 3.44 -> 1.54, FP32 4.14 -> 1.80 (units of three tiles).  What is left at order 5 is mostly LDS:
// the row reads of 102 B blocks and the A operands keep it active in 5900 of 10600 cycles per
// stage, 1300 of them bank conflicts, where the matrix cores are busy in 2300 (FP16, counters).
#include "mfma_ops.h"

namespace ps {

static_assert(kHiSlots <= kSlotsMax && kRowStride == kRowStrideHost && kHiABlocks <= 16, "slot tables");
constexpr int kHiThreads = 64 * kHiWaves;

// Product of NF staged rows, the byte offsets of the rows (in units of 16) in the 10-bit
// fields of w, split for the matrix cores.
template <int PREC, int NF>
__device__ __forceinline__ Operand<PREC> form_staged(const char* S, int w) {
  float x[8], y[8];
  load_row8(reinterpret_cast<const float*>(S + ((w & 0x3ff) << 4)), 0, x);
#pragma unroll
  for (int f = 1; f < NF; ++f) {
    load_row8(reinterpret_cast<const float*>(S + (((w >> (10 * f)) & 0x3ff) << 4)), 0, y);
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] *= y[r];
  }
  return make_operand<PREC>(x, NF == 3 ? 1.0f / (1 << kTripleShift) : 1.0f);
}

template <int PREC, int ORDER>
__global__ __launch_bounds__(kHiThreads, 4) void contract_rows(CtrParams p) {
  constexpr int kRowB = kRowStride * 4;            // bytes of a staged row
  constexpr int NA = ORDER == 6 ? 3 : 2;           // fields of an A row
  extern __shared__ __attribute__((aligned(16))) char hi_lds[];
  const int nrows = p.n_blk * 16;                  // staged rows (zero beyond n_shells); row nrows is all zero
  char* stage = hi_lds;                            // [2][nrows + 1][kRowStride] floats
  uint4* aop = reinterpret_cast<uint4*>(hi_lds + 2 * (nrows + 1) * kRowB);   // [half][A block][hi, lo][lane]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15, g = lane >> 4;
  const int chunk = blockIdx.x, group = blockIdx.y, b = blockIdx.z;

  for (int i = tid; i < 2 * (nrows + 1) * kRowStride; i += kHiThreads)
    if ((i / kRowStride) % (nrows + 1) >= p.n_shells) reinterpret_cast<float*>(stage)[i] = 0.f;

  // staging: thread t moves float4 #t of the (16 n_blk rows x 64) slice, scaled by the
  // shell's power of two (unscaled products of five or six values overflow float32)
  const int st_row = tid >> 4;
  const bool st_on = st_row < p.n_shells;
  const float st_scale = st_on ? ldexpf(1.0f, shell_scale_exp(p.absmax, b * p.n_shells + st_row)) : 0.f;
  const float* src = p.D + ((size_t)b * p.n_shells + (st_on ? st_row : 0)) * p.G +
                     (long long)chunk * p.ksteps * kKStep + (tid & 15) * 4;
  char* dst = stage + st_row * kRowB + (tid & 15) * 16;
  auto store = [&](int buf, float4 v) {
    if (st_on)
      *reinterpret_cast<float4*>(dst + buf * (nrows + 1) * kRowB) =
          make_float4(v.x * st_scale, v.y * st_scale, v.z * st_scale, v.w * st_scale);
  };
  float4 pre = *reinterpret_cast<const float4*>(src);
  store(0, pre);

  // the A rows this lane forms each stage: (block t / 2, half t % 2), t = wave + 8 f
  constexpr int kForm = (2 * kHiABlocks + kHiWaves - 1) / kHiWaves;
  const int n_a = p.grp_nblk[group];
  int aw[kForm];
#pragma unroll
  for (int f = 0; f < kForm; ++f) {
    const int t = wave + f * kHiWaves;
    aw[f] = t < 2 * n_a ? p.a_rows[16 * p.grp_blk[group * kHiABlocks + (t >> 1)] + row] : 0;
  }
  // slots: one byte each, bits 0-3 the group's A block, 6 = form B here, 7 = empty; and the
  // lane's B row of the slots that form one
  const size_t gw = (size_t)group * kHiWaves + wave;
  int un[(kHiSlots + 3) / 4], bw[kHiSlots];
#pragma unroll
  for (int i = 0; i < (kHiSlots + 3) / 4; ++i)
    un[i] = __builtin_amdgcn_readfirstlane(p.slot_uni[gw * (kSlotsMax / 4) + i]);
#pragma unroll
  for (int s = 0; s < kHiSlots; ++s) bw[s] = p.slot_lane[(gw * 16 + row) * kSlotsMax + s];
  f32x4 acc[kHiSlots];
#pragma unroll
  for (int s = 0; s < kHiSlots; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();

  for (int ks = 0; ks < p.ksteps; ++ks) {
    const char* S = stage + (ks & 1) * (nrows + 1) * kRowB + 32 * g;
    if (ks + 1 < p.ksteps) pre = *reinterpret_cast<const float4*>(src + (size_t)(ks + 1) * kKStep);
#pragma unroll
    for (int f = 0; f < kForm; ++f) {
      const int t = wave + f * kHiWaves;
      if (t < 2 * n_a) {
        const Operand<PREC> o = form_staged<PREC, NA>(S + 128 * (t & 1), aw[f]);
        uint4* w = aop + ((t & 1) * kHiABlocks + (t >> 1)) * 128 + lane;
        op_to_words<PREC>(o, w[0], w[64]);
      }
    }
    __syncthreads();                                // every A block of the stage is in LDS
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // re-read from SGPRs every half stage: kept as precomputed conditions they would spill
      int u[(kHiSlots + 3) / 4];
#pragma unroll
      for (int i = 0; i < (kHiSlots + 3) / 4; ++i) {
        u[i] = un[i];
        asm volatile("" : "+s"(u[i]));
      }
      Operand<PREC> B;
#pragma unroll
      for (int s = 0; s < kHiSlots; ++s) {
        const int info = (u[s / 4] >> (8 * (s % 4))) & 0xff;
        if (info & 0x80) break;
        if (info & 0x40) {
          int w = bw[s];
          asm volatile("" : "+v"(w));               // its row addresses are worked out here, not kept
          B = form_staged<PREC, 3>(S + 128 * h, w);
        }
        const uint4* aw4 = aop + (h * kHiABlocks + (info & 15)) * 128 + lane;
        mma<PREC>(acc[s], op_from_words<PREC>(aw4[0], aw4[64]), B);
      }
    }
    if (ks + 1 < p.ksteps) store((ks + 1) & 1, pre);
    __syncthreads();
  }

  const int* my_tiles = p.slot_tile + gw * kSlotsMax;
  float* out = p.partials + ((size_t)b * p.n_chunks + chunk) * (size_t)p.n_tiles * 256;
#pragma unroll
  for (int s = 0; s < kHiSlots; ++s) {
    if ((un[s / 4] >> (8 * (s % 4))) & 0x80) break;
    *reinterpret_cast<f32x4*>(out + (size_t)my_tiles[s] * 256 + 4 * lane) = acc[s];
  }
}

hipError_t launch_contract_hi(int prec, int order, const CtrParams& p, int n_groups, int batch, hipStream_t st) {
  if (p.n_blk > 2) return hipErrorInvalidValue;   // 32 shells: one float4 per thread and stage
  dim3 grid(p.n_chunks, n_groups, batch);
  const size_t shm = (size_t)2 * (p.n_blk * 16 + 1) * kRowStride * 4 + (size_t)2 * kHiABlocks * 128 * sizeof(uint4);
#define L(P, O) hipLaunchKernelGGL((contract_rows<P, O>), grid, dim3(kHiThreads), shm, st, p)
  if (order == 5) {
    if (prec == kFP32) L(kFP32, 5); else if (prec == kBF16) L(kBF16, 5); else L(kFP16, 5);
  } else if (order == 6) {
    if (prec == kFP32) L(kFP32, 6); else if (prec == kBF16) L(kBF16, 6); else L(kFP16, 6);
  } else {
    return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

}  // namespace ps
