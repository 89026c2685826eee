// Adjoint weights and the precision dispatch of the adjoint products: the FP16 split runs
// the kernels of adjoint.h (adjoint_fp16.hip, adjoint4_fp16.hip), FP32 and the BF16 split
// those of adjoint_sym.h (adjoint_sym_*.hip, adjoint4_sym_*.hip).
#include "adjoint_sym.h"

namespace ps {

#define PS_SYM_ARGS const float*, const uint4*, const float2*
#define PS_OUT_ARGS long long, float*, cplx<float>*, const cplx<float>*, Geom, int, hipStream_t
extern template hipError_t launch_adjoint_sym_prec<kFP32>(PS_SYM_ARGS, int, int, PS_OUT_ARGS);
extern template hipError_t launch_adjoint_sym_prec<kBF16>(PS_SYM_ARGS, int, int, PS_OUT_ARGS);
extern template hipError_t launch_adjoint4_sym_prec<kFP32>(PS_SYM_ARGS, const int*, int, PS_OUT_ARGS);
extern template hipError_t launch_adjoint4_sym_prec<kBF16>(PS_SYM_ARGS, const int*, int, PS_OUT_ARGS);
hipError_t launch_adjoint4_gemm_fp16(const float*, const uint4*, const int*, const unsigned*, const unsigned long long*,
                                     int, PS_OUT_ARGS);
hipError_t launch_adjoint_gemm_fp16(const float*, const uint4*, const int*, const unsigned*, const unsigned long long*,
                                    int, PS_OUT_ARGS);
#undef PS_OUT_ARGS
#undef PS_SYM_ARGS

// dL/dB_t f / (N^3 n_t) times the number of times m occurs in t = sort(shells), or 0
// when t does not close.
template <int ORDER>
__device__ __forceinline__ double adj_weight(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                             const int* __restrict__ lookup, int n_shells, int n_closing, int b,
                                             int m, const int (&rest)[ORDER - 1]) {
  int t[ORDER];
  t[0] = m;
#pragma unroll
  for (int j = 1; j < ORDER; ++j) t[j] = rest[j - 1];
#pragma unroll
  for (int a = 0; a < ORDER - 1; ++a)
#pragma unroll
    for (int c = 0; c < ORDER - 1 - a; ++c)
      if (t[c] > t[c + 1]) { const int x = t[c]; t[c] = t[c + 1]; t[c + 1] = x; }
  size_t key = 0;
#pragma unroll
  for (int j = 0; j < ORDER; ++j) key = key * n_shells + t[j];
  const int id = lookup[key];
  if (id < 0) return 0.0;
  int mult = 0;
#pragma unroll
  for (int j = 0; j < ORDER; ++j) mult += t[j] == m;
  return (double)mult * grad[(size_t)b * n_closing + id] * fnorm[id];
}

// Power-of-two exponent that the FP16 path folds into the weight of (m, rest): the
// row's scale e_m, the inverse of the rest's field scales, and for order 4 the 2^7
// that brings the triple products into range.
template <int ORDER>
__device__ __forceinline__ int adj_weight_exp(const unsigned* absmax, int b, int n_shells,
                                              const int (&rest)[ORDER - 1]) {
  int ex = ORDER == 4 ? kTripleShift : 0;
#pragma unroll
  for (int j = 0; j < ORDER - 1; ++j) ex -= shell_scale_exp(absmax, b * n_shells + rest[j]);
  return ex;
}

// FP16 only: rowmax[b][m] = max over the rests of |W[m][rest]| times the rest's scale
// factor (float64 bits; non-negative doubles order like their bit patterns).
// Order 3: grid (n_shells: v, batch), threads m; the rests (u <= v) of one v.
__global__ void adjoint_rowmax(const double* __restrict__ grad, const double* __restrict__ fnorm,
                               const int* __restrict__ lookup, int n_shells, int n_closing,
                               const unsigned* __restrict__ absmax, unsigned long long* __restrict__ rowmax) {
  const int m = threadIdx.x, v = blockIdx.x, b = blockIdx.y;
  if (m >= n_shells) return;
  double mx = 0.0;
  for (int u = 0; u <= v; ++u) {
    const int rest[2] = {u, v};
    const double w = adj_weight<3>(grad, fnorm, lookup, n_shells, n_closing, b, m, rest);
    if (w != 0.0) mx = fmax(mx, fabs(ldexp(w, adj_weight_exp<3>(absmax, b, n_shells, rest))));
  }
  if (mx > 0.0) atomicMax(rowmax + b * 64 + m, (unsigned long long)__double_as_longlong(mx));
}

// Order 4: grid (items (w, v <= w), batch), threads m; the rests (u <= v, v, w) of one item.
__global__ void adjoint4_rowmax(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                const int* __restrict__ lookup, int n_shells, int n_closing,
                                const unsigned* __restrict__ absmax, unsigned long long* __restrict__ rowmax) {
  const int m = threadIdx.x, it = blockIdx.x, b = blockIdx.y;
  if (m >= n_shells) return;
  int w = 0;
  while ((w + 1) * (w + 2) / 2 <= it) ++w;
  const int v = it - w * (w + 1) / 2;
  double mx = 0.0;
  for (int u = 0; u <= v; ++u) {
    const int rest[3] = {u, v, w};
    const double x = adj_weight<4>(grad, fnorm, lookup, n_shells, n_closing, b, m, rest);
    if (x != 0.0) mx = fmax(mx, fabs(ldexp(x, adj_weight_exp<4>(absmax, b, n_shells, rest))));
  }
  if (mx > 0.0) atomicMax(rowmax + b * 64 + m, (unsigned long long)__double_as_longlong(mx));
}

// Writes one weight into its operand word: lane `ln`, element r of the hi and lo
// 16-byte words at base[ln] and base[64 + ln] (float32: values 0..3 / 4..7).
__device__ __forceinline__ void adj_store_weight(uint4* base, int ln, int r, double w, int prec) {
  if (prec == kFP32) {
    float* dst = reinterpret_cast<float*>(&base[(r < 4 ? 0 : 64) + ln]);
    dst[r & 3] = (float)w;
  } else if (prec == kBF16) {
    const float x = (float)w;
    const unsigned bits = __float_as_uint(x);
    const float h = __uint_as_float(bits & 0xffff0000u);
    reinterpret_cast<unsigned short*>(&base[ln])[r] = (unsigned short)(bits >> 16);
    reinterpret_cast<unsigned short*>(&base[64 + ln])[r] = __builtin_bit_cast(unsigned short, (__bf16)(x - h));
  } else {
    const float x = (float)w;
    const _Float16 h = (_Float16)x;
    reinterpret_cast<unsigned short*>(&base[ln])[r] = __builtin_bit_cast(unsigned short, h);
    reinterpret_cast<unsigned short*>(&base[64 + ln])[r] = __builtin_bit_cast(unsigned short, (_Float16)(x - (float)h));
  }
}

// Order 3, FP16: W in operand order, [b][v][uc][mb][hi, lo][lane]: lane l holds W[m][(u, v)]
// for m = 32 mb + l % 32 and u = 16 uc + 8 (l / 32) + r, r = 0..7 (zero when u > v).
// Scaled by 2^(e_m - sigma_u - sigma_v).  grid (64: u, n_shells: v, batch), threads m.
__global__ void adjoint_weights(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                const int* __restrict__ lookup, int n_shells, int n_closing,
                                const unsigned* __restrict__ absmax, const unsigned long long* __restrict__ rowmax,
                                uint4* __restrict__ W) {
  const int m = threadIdx.x, u = blockIdx.x, v = blockIdx.y, b = blockIdx.z;
  double w = 0.0;
  if (m < n_shells && u < n_shells && u <= v) {
    const int rest[2] = {u, v};
    w = adj_weight<3>(grad, fnorm, lookup, n_shells, n_closing, b, m, rest);
    if (w != 0.0)
      w = ldexp(w, adj_row_exp(rowmax, b * 64 + m) + adj_weight_exp<3>(absmax, b, n_shells, rest));
  }
  const int uc = u >> 4, q = u & 15, hh = q >> 3, r = q & 7;
  const int ln = 32 * hh + (m & 31), mb = m >> 5;
  uint4* base = W + ((((size_t)b * n_shells + v) * 4 + uc) * kAdjMaxMb + mb) * 2 * 64;
  adj_store_weight(base, ln, r, w, kFP16);
}

// A weight of sym_equal: the value that the split's words hold, and the lo word.
__device__ __forceinline__ float2 equal_weight(double w, int prec) {
  const float x = (float)w;
  if (prec != kBF16) return make_float2(x, 0.f);
  const float h = __uint_as_float(__float_as_uint(x) & 0xffff0000u), l = (float)(__bf16)(x - h);
  return make_float2(h + l, l);
}

// Lane ln of weight block idx (sym_index) of a pair of partners in shell block kb: which of
// the two partners (t), the row m and the 16-shell chunk uc of u it holds.  Lane l is
// chain row l % 32 and u = 16 uc + 8 (l / 32) + r; row rho is 16-row half rho / 16 and
// m = 16 M + 8 (rho / 4 % 2) + 4 (rho / 8 % 2) + rho % 4.
__device__ __forceinline__ void sym_lane(int kb, int idx, int ln, int& t, int& m, int& uc) {
  const int n_p = sym_p_chains(kb);
  int M = n_p;
  bool pchain = false;
  t = uc = 0;
  if (kb > 0)
    for (int tt = 0; tt < 2; ++tt)
      for (int c = 0; c <= kb; ++c)
        if (sym_index(kb, false, n_p, tt, c) == idx) t = tt, uc = c;
  if (kb == 0 || idx >= 2 * (kb + 1))
    for (int mm = 0; mm < n_p; ++mm)
      for (int c = 0; c <= kb; ++c)
        if (sym_index(kb, true, mm, 0, c) == idx) pchain = true, M = mm, uc = c;
  const int rho = ln & 31, sub = rho >> 4;
  if (pchain) t = sub;
  m = 16 * (M + (pchain ? 0 : sub)) + 8 * ((rho >> 2) & 1) + 4 * ((rho >> 3) & 1) + (rho & 3);
}

// Order 3, symmetric form (FP32 and BF16): the matrices dQ_k/dd_m, W[b][pair][block][hi, lo]
// [lane] with the blocks of sym_index, zero outside m, u <= k.  The tuple of three times k is
// left out (sym_equal adds it): its weight 3 w goes to equal[b][k].
// grid (pairs of whole shell blocks, 16, batch), threads lane.
__global__ void adjoint_sym_weights(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                    const int* __restrict__ lookup, int n_shells, int n_closing, int prec,
                                    uint4* __restrict__ W, float2* __restrict__ equal) {
  const int ln = threadIdx.x, pair = blockIdx.x, idx = blockIdx.y, b = blockIdx.z;
  const int kb = pair / 8;
  if (idx >= sym_blocks(kb)) return;
  int k, m, uc;
  sym_lane(kb, idx, ln, k, m, uc);
  k += 2 * pair;
  uint4* base = W + (size_t)b * sym_words(n_shells) +
                (sym_base(kb) + (size_t)(pair % 8) * sym_blocks(kb) + idx) * kSymBlockWords;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int u = 16 * uc + 8 * (ln >> 5) + r;
    double w = 0.0;
    if (k < n_shells && m <= k && u <= k) {
      const size_t lo = m < u ? m : u, hi = m < u ? u : m;
      const int id = lookup[(lo * n_shells + hi) * n_shells + k];
      if (id >= 0) w = (m == u ? 2.0 : 1.0) * grad[(size_t)b * n_closing + id] * fnorm[id];
      if (m == k && u == k) {
        equal[b * 64 + k] = equal_weight(id >= 0 ? 3.0 * grad[(size_t)b * n_closing + id] * fnorm[id] : 0.0, prec);
        w = 0.0;
      }
    }
    adj_store_weight(base, ln, r, w, prec);
  }
}

// Order 4, symmetric form: W[b][l][pair][block][hi, lo][lane], pairs k / 2 <= l / 2.  Partners
// k >= 16 hold the matrices d^2 Q_kl / dd_m dd_u (m, u <= k); the partners v of shell block 0
// hold W[m][(u, v)], u <= v, of the terms within that block.
// grid (blocks of the last l, n_shells: l, batch), threads lane.
__global__ void adjoint4_sym_weights(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                     const int* __restrict__ lookup, int n_shells, int n_closing, int prec,
                                     uint4* __restrict__ W, float2* __restrict__ equal) {
  const int ln = threadIdx.x, l = blockIdx.y, b = blockIdx.z;
  if ((int)blockIdx.x >= sym4_blocks_of(l)) return;
  int kb = 0;
  while ((int)blockIdx.x >= sym_base(kb + 1)) ++kb;
  const int in_kb = blockIdx.x - sym_base(kb), pair = 8 * kb + in_kb / sym_blocks(kb), idx = in_kb % sym_blocks(kb);
  int k, m, uc;
  sym_lane(kb, idx, ln, k, m, uc);
  k += 2 * pair;
  uint4* base = W + ((size_t)b * sym4_blocks(n_shells) + sym4_blocks(l) + blockIdx.x) * kSymBlockWords;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int u = 16 * uc + 8 * (ln >> 5) + r;
    double w = 0.0;
    if (k <= l && u <= k && (kb == 0 ? m <= l : m <= k)) {
      int t[3] = {m < u ? m : u, m < u ? u : m, k};       // sorted below k; block 0: m may exceed k
      if (t[1] > t[2]) { const int x = t[1]; t[1] = t[2]; t[2] = x; }
      const int id = lookup[(((size_t)t[0] * n_shells + t[1]) * n_shells + t[2]) * n_shells + l];
      const int mult = kb == 0 ? (m == t[0]) + (m == t[1]) + (m == t[2]) : m == u ? 2 : 1;
      if (id >= 0) w = (double)mult * grad[(size_t)b * n_closing + id] * fnorm[id];
      if (m == l && u == l && k == l) {
        equal[b * 64 + l] = equal_weight(id >= 0 ? 4.0 * grad[(size_t)b * n_closing + id] * fnorm[id] : 0.0, prec);
        w = 0.0;
      }
    }
    adj_store_weight(base, ln, r, w, prec);
  }
}

// Order 4, FP16: W4[b][item (w, v <= w)][uc][mb][hi, lo][lane] (NC chunks of u, NC / 2 blocks
// of m: adj4_chunks): lane l holds row m = 32 mb + l % 32 and u = 16 uc + 8 (l / 32) + r
// (zero when u > v).  Scaled by 2^(e_m + 7 - sigma_u - sigma_v - sigma_w).
// grid (16 NC: u, items, batch), threads m (16 NC).
__global__ void adjoint4_weights(const double* __restrict__ grad, const double* __restrict__ fnorm,
                                 const int* __restrict__ lookup, int n_shells, int n_closing,
                                 const unsigned* __restrict__ absmax, const unsigned long long* __restrict__ rowmax,
                                 uint4* __restrict__ W) {
  const int m = threadIdx.x, u = blockIdx.x, it = blockIdx.y, b = blockIdx.z;
  int w = 0;
  while ((w + 1) * (w + 2) / 2 <= it) ++w;
  const int v = it - w * (w + 1) / 2;
  double val = 0.0;
  if (m < n_shells && u < n_shells && u <= v) {
    const int rest[3] = {u, v, w};
    val = adj_weight<4>(grad, fnorm, lookup, n_shells, n_closing, b, m, rest);
    if (val != 0.0)
      val = ldexp(val, adj_row_exp(rowmax, b * 64 + m) + adj_weight_exp<4>(absmax, b, n_shells, rest));
  }
  const int n_items = n_shells * (n_shells + 1) / 2;
  const int nc = adj4_chunks(n_shells), nm = nc / 2;
  const int uc = u >> 4, q = u & 15, hh = q >> 3, r = q & 7;
  const int ln = 32 * hh + (m & 31), mb = m >> 5;
  uint4* base = W + ((((size_t)b * n_items + it) * nc + uc) * nm + mb) * 2 * 64;
  adj_store_weight(base, ln, r, val, kFP16);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_adjoint_weights(const double* grad, const double* fnorm, const int* lookup, int n_shells,
                                  int n_closing, int prec, const unsigned* absmax, unsigned long long* rowmax,
                                  uint4* W, int batch, hipStream_t st) {
  if (n_shells > 64) return hipErrorInvalidValue;
  if (prec == kFP16) {
    hipError_t e = launch_fill_u32(rowmax, 0u, (size_t)batch * 64 * 2, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(adjoint_rowmax, dim3(n_shells, batch), dim3(64), 0, st, grad, fnorm, lookup, n_shells,
                       n_closing, absmax, rowmax);
  }
  if (prec == kFP16)
    hipLaunchKernelGGL(adjoint_weights, dim3(64, n_shells, batch), dim3(64), 0, st, grad, fnorm, lookup, n_shells,
                       n_closing, absmax, rowmax, W);
  else
    hipLaunchKernelGGL(adjoint_sym_weights, dim3((n_shells + 15) / 16 * 8, 16, batch), dim3(64), 0, st, grad, fnorm,
                       lookup, n_shells, n_closing, prec, W, reinterpret_cast<float2*>(rowmax));
  return hipGetLastError();
}

hipError_t launch_adjoint4_weights(const double* grad, const double* fnorm, const int* lookup, int n_shells,
                                   int n_closing, int prec, const unsigned* absmax, unsigned long long* rowmax,
                                   uint4* W, int batch, hipStream_t st) {
  if (n_shells > kAdj4MaxShells) return hipErrorInvalidValue;
  const int n_items = n_shells * (n_shells + 1) / 2;
  const int nu = 16 * adj4_chunks(n_shells);   // values of u (and of m) the operand words cover
  if (prec == kFP16) {
    hipError_t e = launch_fill_u32(rowmax, 0u, (size_t)batch * 64 * 2, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(adjoint4_rowmax, dim3(n_items, batch), dim3(nu), 0, st, grad, fnorm, lookup, n_shells,
                       n_closing, absmax, rowmax);
  }
  if (prec == kFP16)
    hipLaunchKernelGGL(adjoint4_weights, dim3(nu, n_items, batch), dim3(nu), 0, st, grad, fnorm, lookup, n_shells,
                       n_closing, absmax, rowmax, W);
  else
    hipLaunchKernelGGL(adjoint4_sym_weights, dim3(sym4_blocks_of(n_shells - 1), n_shells, batch), dim3(64), 0, st, grad,
                       fnorm, lookup, n_shells, n_closing, prec, W, reinterpret_cast<float2*>(rowmax));
  return hipGetLastError();
}

hipError_t launch_adjoint_gemm(int prec, const float* D, const uint4* W, const int* vmask, const unsigned* absmax,
                               const unsigned long long* rowmax, int n_shells, bool dense, long long G, float* A,
                               cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st) {
  const bool fused = adjoint_fuses_rows(g.N);
  if (fused == (H2 == nullptr) || fused == (A != nullptr) || n_shells > 64 || G % kAdjPts != 0)
    return hipErrorInvalidValue;
  const float2* equal = reinterpret_cast<const float2*>(rowmax);   // FP16 alone scales its rows
  if (prec == kFP32) return launch_adjoint_sym_prec<kFP32>(D, W, equal, n_shells, dense, G, A, H2, tw, g, batch, st);
  if (prec == kBF16) return launch_adjoint_sym_prec<kBF16>(D, W, equal, n_shells, dense, G, A, H2, tw, g, batch, st);
  return launch_adjoint_gemm_fp16(D, W, vmask, absmax, rowmax, n_shells, G, A, H2, tw, g, batch, st);
}

hipError_t launch_adjoint4_gemm(int prec, const float* D, const uint4* W, const int* imask, const int* pmask,
                                const unsigned* absmax, const unsigned long long* rowmax, int n_shells, long long G,
                                float* A, cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st) {
  const bool fused = adjoint_fuses_rows(g.N);
  if (fused == (H2 == nullptr) || fused == (A != nullptr) || n_shells > kAdj4MaxShells || G % kAdjPts != 0)
    return hipErrorInvalidValue;
  const float2* equal = reinterpret_cast<const float2*>(rowmax);   // FP16 alone scales its rows
  if (prec == kFP32) return launch_adjoint4_sym_prec<kFP32>(D, W, equal, pmask, n_shells, G, A, H2, tw, g, batch, st);
  if (prec == kBF16) return launch_adjoint4_sym_prec<kBF16>(D, W, equal, pmask, n_shells, G, A, H2, tw, g, batch, st);
  return launch_adjoint4_gemm_fp16(D, W, imask, absmax, rowmax, n_shells, G, A, H2, tw, g, batch, st);
}

}  // namespace ps
