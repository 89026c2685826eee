// Host-side launchers of the device kernels (fft.hip, contract.hip, util.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace ps {

// fft.hip
template <typename T, bool UNIT>
hipError_t launch_c2r_p1(const cplx<float>* box, const int16_t* shell_of_q, const int* qmax, cplx<T>* H1,
                         const cplx<T>* tw, Geom g, int nz, hipStream_t st);
template <typename T>
hipError_t launch_c2r_p2(const cplx<T>* H1, const int* qmax, cplx<T>* H2, const cplx<T>* tw, Geom g, int nz,
                         hipStream_t st);
hipError_t launch_c2r_p3(const cplx<float>* H2, const int* qmax, float* out, unsigned* absmax,
                         const cplx<float>* tw, Geom g, int nz, hipStream_t st);
hipError_t launch_c2r_p3_wedge(const cplx<double>* H2, const int* qmax, const int* rows, int nrows, double* out,
                               long long nwedge, const cplx<double>* tw, Geom g, int nz, hipStream_t st);
hipError_t launch_r2c_q3(const float* in, cplx<float>* H2, const cplx<float>* tw, Geom g, int nz, hipStream_t st);
template <bool GRAD>
hipError_t launch_r2c_q2(const cplx<float>* H2, cplx<float>* H1, const cplx<float>* tw, Geom g, int nz,
                         hipStream_t st);
template <bool MASK>
hipError_t launch_r2c_q1(const cplx<float>* H1, const int16_t* shell_of_q, const int* qmax, cplx<float>* box,
                         const cplx<float>* tw, Geom g, int nz, hipStream_t st);
constexpr int kAbsmaxSpreadHost = 256;
hipError_t launch_reduce_absmax(const unsigned* part, unsigned* absmax, int nz, hipStream_t st);
hipError_t launch_box_from_half_spectrum(const cplx<float>* hs, cplx<float>* box, Geom g, int batch,
                                         hipStream_t st);
hipError_t launch_half_spectrum_from_box(const cplx<float>* box, cplx<float>* hs, Geom g, int batch,
                                         hipStream_t st);

// contract.hip
struct CtrParams {
  const float* D;
  const int* slot_uni;     // [n_groups][waves][kSlots / 4]: one byte per slot
  const int* slot_lane;    // [n_groups][waves][16 rows][kSlots]: pair shells per lane
  const int* slot_tile;
  const unsigned* absmax;
  float* partials;
  long long G;
  int n_shells;
  int n_blk;
  int n_tiles;
  int ksteps;
  int n_chunks;
  const int* a_rows;       // orders 5 and 6: the A rows, staged row offsets of their shells (10 bits each)
  const int* grp_blk;      // orders 5 and 6: [n_groups][kHiABlocks] the group's A blocks
  const int* grp_nblk;     // [n_groups]: how many
};
constexpr int kCtrWavesHost = 16;
constexpr int kSlotsHost = 14;
constexpr int kSlots4Host = 10;
// Orders 5 and 6 (contract_tiles_hi.hip): waves of a workgroup, tiles per wave, and A row
// blocks of a tile group (formed in LDS; 4 KB each for the stage's two halves).
constexpr int kHiWaves = 8;
constexpr int kHiSlots = 14;
constexpr int kHiABlocks = 11;
constexpr int kMaxShells56 = 32;    // orders 5 and 6: shells per plan (row tables stay small)
constexpr int kSlots2Host = 4;
constexpr int kSlotsMaxHost = 16;   // per-wave stride of the slot tables
constexpr int kStagePtsHost = 64;
constexpr int kRowStrideHost = 68;   // floats per staged float32 row
constexpr int kMaxBlkHost = 4;       // the shell-block aligned order-3 kernel (<= 64 shells)
constexpr int kMaxTileBlkHost = 8;   // the tile kernel, orders 2 to 4 (<= 128 shells)
constexpr int kAdjPtsHost = 512;   // grid points per adjoint workgroup
constexpr int kCntStageHost = 32;

// Order 4 in split FP16, up to 64 shells (contract_pairs.hip): slots of `tiles` A blocks
// (aligned to that number) against one B block, `slots` per wave; k4Blocks pair blocks are what
// fits the workgroup's LDS beside the staged shell operands, one half of a stage.
struct Ctr4Shape { int waves, slots, tiles, blocks; };
constexpr int k4Blocks = 56;
constexpr Ctr4Shape k4Narrow = {16, 8, 2, k4Blocks / 2};
constexpr Ctr4Shape k4Wide = {8, 10, 4, k4Blocks};
struct Ctr4Params {
  const float* D;
  const unsigned* absmax;
  const int* pair_uv;
  const int* slot_a;       // [n_groups][waves][slots]: the group's indices of the A blocks, a byte each
  const int* slot_b;       // [n_groups][waves][slots]: bits 0-7 the B block; 8: load the A blocks; 9, 10:
                           // the first, last two tiles in use; < 0: empty
  const int* slot_tile;    // [n_groups][waves][slots][tiles]: tile ids, or -1
  const int* grp_blk;      // [n_groups][k4Blocks]: the group's pair blocks
  const int* grp_nblk;
  float* partials;
  long long G;
  int n_shells, n_blk, n_tiles, ksteps, n_chunks;
  bool wide;               // the shape of the tables
};
hipError_t launch_contract_pairs(const Ctr4Params& p, int n_groups, int batch, hipStream_t st);

hipError_t launch_contract(int prec, int order, const CtrParams& p, int n_groups, int batch, hipStream_t st);

// Order 3 with products aligned to shell blocks (contract_j3.hip): the slots of a wave, one
// 16 x 16 tile each, by the kind of product operand and the plain operand's block.
constexpr int kJWaves = 8;
constexpr int kJDiag0 = 0;     // j and i in block 0: columns k of blocks 0..3
constexpr int kJDiag1 = 4;     // j and i in block 1: columns k of blocks 1..3
constexpr int kJDiag2 = 7;     // j and k in block 2: columns i of blocks 0..2
constexpr int kJDiag3 = 10;    // j and k in block 3: columns i of blocks 0..3
constexpr int kJLow = 14;      // j = 16 + w + 8 q, i in block 0: slots 3 q + columns k of blocks 1..3
constexpr int kJHigh = 20;     // j = 32 + w + 8 q, k in block 3: slots 3 q + columns i of blocks 0..2
constexpr int kJShared = 26;   // the half-full shells of blocks 0, 1 (waves 0, 1) and 2, 3 (waves 2, 3)
constexpr int kJSlots = 28;
// The slots that contract_j3 multiplies together, by one product operand: `count` shell blocks
// from `block` on, as far as the plan's go, of plans of at least `plan_blk` blocks.
struct JGroup { int slot, count, block, plan_blk; };
constexpr JGroup kJGroups[] = {{kJDiag0, 2, 0, 1}, {kJDiag1, 3, 1, 2}, {kJDiag2, 3, 0, 3}, {kJDiag3, 4, 0, 4},
                               {kJLow, 2, 1, 2},   {kJLow + 3, 2, 1, 2}, {kJHigh, 3, 0, 4}, {kJHigh + 3, 3, 0, 4}};
// Slots multiplied alone, for the shell blocks 2 and 3 of the small shells' operands.
constexpr JGroup kJCorners[] = {{kJDiag0 + 2, 1, 2, 3}, {kJDiag0 + 3, 1, 3, 4}, {kJLow + 2, 1, 3, 4},
                                {kJLow + 5, 1, 3, 4}};
struct JPlace {
  int wave, slot, row, col;
};
// Where the candidate i <= j <= k (0-based) is accumulated.
inline JPlace jplace(int i, int j, int k) {
  const int ib = i / 16, jb = j / 16, kb = k / 16, il = i % 16, jl = j % 16, kl = k % 16;
  if (jb == 1 && ib == 0) return {jl % 8, kJLow + 3 * (jl / 8) + kb - 1, il, kl};
  if (jb == 2 && kb == 3) return {jl % 8, kJHigh + 3 * (jl / 8) + ib, kl, il};
  if (jb <= 1) {               // rows i <= j
    if (jl == 7) return {kb / 2, kJShared + kb % 2, jb == 0 ? il : 15 - il, kl};
    const int slot = jb == 0 ? kJDiag0 + kb : kJDiag1 + kb - 1;
    if (jl < 7 || jl == 15) return {jl < 7 ? jl : 7, slot, il, kl};
    return {14 - jl, slot, 15 - il, kl};
  }
  const int jm = 15 - jl;      // rows k >= j, mirrored
  if (jm == 7) return {2 + ib / 2, kJShared + ib % 2, jb == 3 ? 15 - kl : kl, il};
  const int slot = (jb == 2 ? kJDiag2 : kJDiag3) + ib;
  if (jm < 7 || jm == 15) return {jm < 7 ? jm : 7, slot, 15 - kl, il};
  return {14 - jm, slot, kl, il};
}
struct CtrJParams {
  const float* D;
  const unsigned* absmax;
  const int* tile_of_slot;   // [kJWaves][kJSlots]: compact tile id, or -1
  const unsigned* slot_mask; // [kJWaves]: bit s set when slot s holds a tile
  bool all_used;             // every wave has a tile of every kind of product operand
  float* partials;
  long long G;
  int n_shells;
  int n_blk;
  int n_tiles;
  int ksteps;
  int n_chunks;
};
hipError_t launch_contract_j3(int prec, const CtrJParams& p, int batch, hipStream_t st);
hipError_t launch_reduce_f32(const float* part, double* tmp, int n_chunks, int cpg, int n_groups, long long n_ent,
                             bool accumulate, const int* closing_of_entry, const int* bins, int order,
                             const unsigned* absmax, int n_shells, int prec, int batch, hipStream_t st);
hipError_t launch_reduce_f64(const double* part, double* tmp, int n_chunks, int cpg, int n_groups, long long n_ent,
                             int batch, hipStream_t st);
hipError_t launch_gather(const double* tmp, int n_groups, long long n_ent, const int* ent_idx, const int* bins,
                         int order, const double* fnorm, int n_closing, const unsigned* absmax, int n_shells,
                         int prec, double* out, double* raw, int* nonfinite, int batch, hipStream_t st);
hipError_t launch_counts_wedge(int order, const double* cw, long long nwedge, const unsigned char* wmult,
                               const int* cand, int n_cand, int n_shells, int stages_per_chunk, int n_chunks,
                               double2* part, hipStream_t st);
hipError_t launch_reduce_dd(const double2* part, double2* tmp, int n_chunks, int cpg, int n_groups, long long n_ent,
                            hipStream_t st);
// Adjoint products (adjoint.h).  FP16 (prec 2) scales every weight row m by its own
// power of two, found from rowmax[b][64] (float64 bits, written by the weights launch; FP32 and
// BF16 keep the weights of sym_equal there); absmax holds the per-shell field maxima of the forward's FP16 scaling.
hipError_t launch_adjoint_weights(const double* grad, const double* fnorm, const int* lookup, int n_shells,
                                  int n_closing, int prec, const unsigned* absmax, unsigned long long* rowmax,
                                  uint4* W, int batch, hipStream_t st);
// N <= 512: the adjoint kernel also runs the first (x2 -> q2) transform of its fields
// and writes H2 (A must be null); otherwise it writes the fields to A (H2 null).
inline bool adjoint_fuses_rows(int N) { return N <= 512; }
hipError_t launch_adjoint_gemm(int prec, const float* D, const uint4* W, const int* vmask, const unsigned* absmax,
                               const unsigned long long* rowmax, int n_shells, bool dense, long long G, float* A,
                               cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st);
// Order 3 in FP32 and BF16, the symmetric form (adjoint_sym.h): partners k in pairs, 32-row
// chains over the 16-shell chunks of u.  Weight blocks (32 rows x 16 u) of one pair of partners in
// shell block kb, and pairs staged together (at most 18 blocks of 2 KB per stage).
__host__ __device__ constexpr int sym_blocks(int kb) { return (kb + 1) * (kb + 1); }
__host__ __device__ constexpr int sym_stage_pairs(int kb) { return 8 >> kb; }
__host__ __device__ constexpr int sym_p_chains(int kb) { return kb == 0 ? 1 : kb == 1 ? 0 : kb - 1; }
// Blocks of all pairs of the shell blocks before kb.
__host__ __device__ constexpr int sym_base(int kb) {
  int n = 0;
  for (int i = 0; i < kb; ++i) n += 8 * sym_blocks(i);
  return n;
}

constexpr int kSymBlockWords = 2 * 64;   // 16-byte words of a block: hi and lo of its 64 lanes
constexpr int kSymCopyWords = 512;       // one word per thread: a stage is copied in whole rounds
__host__ __device__ constexpr int sym_stage_words(int kb) {
  return sym_stage_pairs(kb) * sym_blocks(kb) * kSymBlockWords;
}
__host__ __device__ constexpr int sym_rounds(int kb) {
  return (sym_stage_words(kb) + kSymCopyWords - 1) / kSymCopyWords;
}
// Weight words of one batch entry of order 3, and of what the last round of a stage reads past
// its end (the stages of block 2, 18 blocks of 128 words in five rounds).
__host__ __device__ constexpr int sym_words(int n_shells) { return sym_base((n_shells + 15) / 16) * kSymBlockWords; }
__host__ __device__ constexpr int sym_words_past(int n_shells) {
  int r = 0;
  for (int kb = 0; 16 * kb < n_shells; ++kb) {
    const int n = sym_rounds(kb) * kSymCopyWords - sym_stage_words(kb);
    r = n > r ? n : r;
  }
  return r;
}

// Position of a block within its pair: the S chains first (uc ascending), then the P
// chains from the largest uc down, the blocks that the triangle bound empties last, so
// that the others are contiguous.
__host__ __device__ constexpr int sym_index(int kb, bool pchain, int M, int t, int uc) {
  if (!pchain) return t * (kb + 1) + uc;
  if (kb == 0) return 0;
  if (kb == 2) return 6 + (2 - uc);
  if (M == 1) return uc > 0 ? 8 + (3 - uc) : 13;
  return uc > 1 ? 11 + (3 - uc) : 14 + (1 - uc);
}
// Chunks of a P chain that the triangle bound leaves, counted from uc = kb down (the
// first pair of the block reaches one more: k = 16 kb needs i + j >= k - 2).
__host__ __device__ constexpr int sym_p_chunks(int kb, int M, bool first) {
  int n = 0;
  for (int uc = 0; uc <= kb; ++uc) n += M + uc >= kb - (first ? 2 : 1);
  return n;
}

// Order 4 in the symmetric form: blocks stored for partner l (its pairs k / 2 <= l / 2), and
// of all l < n.
__host__ __device__ constexpr int sym4_blocks_of(int l) {
  return sym_base(l / 16) + (l / 2 % 8 + 1) * sym_blocks(l / 16);
}
__host__ __device__ constexpr int sym4_blocks(int n) {
  int s = 0;
  for (int l = 0; l < n; ++l) s += sym4_blocks_of(l);
  return s;
}
// Blocks of a pair that the kernel multiplies.
__host__ __device__ constexpr int sym_issued(int kb, bool first, bool dense) {
  int n = kb > 0 ? 2 * (kb + 1) : 0;
  for (int M = 0; M < sym_p_chains(kb); ++M) n += dense ? kb + 1 : sym_p_chunks(kb, M, first);
  return n;
}
// Order 4 (n_shells <= kAdj4MaxShells): W4[b][item (w, v <= w)][uc][mb][hi, lo][lane],
// item = w (w + 1) / 2 + v, over NC = 2 chunks of u and one 32-row block of m up to 32
// shells, NC = 4 chunks and two blocks above.
constexpr int kAdj4MaxShells = 64;
constexpr int kAdj3MaxShells = 64;
__host__ __device__ constexpr int adj4_chunks(int n_shells) { return n_shells <= 32 ? 2 : 4; }
__host__ __device__ constexpr int adj4_words_per_item(int n_shells) {
  return adj4_chunks(n_shells) * (adj4_chunks(n_shells) / 2) * 2 * 64;
}
hipError_t launch_adjoint4_weights(const double* grad, const double* fnorm, const int* lookup, int n_shells,
                                   int n_closing, int prec, const unsigned* absmax, unsigned long long* rowmax,
                                   uint4* W, int batch, hipStream_t st);
hipError_t launch_adjoint4_gemm(int prec, const float* D, const uint4* W, const int* imask, const int* pmask,
                                const unsigned* absmax, const unsigned long long* rowmax, int n_shells, long long G,
                                float* A, cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st);

// util.hip
constexpr size_t kStaticScratchBytes = (size_t)128 << 20;   // polyspec_forward_static's workspace
constexpr int kMaxDevices = 64;
// Device address of this device's static scratch (looked up once per device, with that
// device current).
hipError_t static_scratch_address(int device, void** ptr);
hipError_t launch_fill_u32(void* dst, unsigned value, size_t n_words, hipStream_t st);
hipError_t launch_fields_absmax(const float* x, long long G, int nz, unsigned* part, int spread, hipStream_t st);

}  // namespace ps
