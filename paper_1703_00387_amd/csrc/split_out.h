// What follows a converged single-panel split (m <= 64 rows s_j v_j^dag in X,
// their squared norms known), by the workgroup that holds it: the order and
// the count rule, the write-back of a bond update, the factors of a stand-alone
// truncation.  Shared by the direct path (eig.hip) and the Jacobi's (svd.hip).
#pragma once
#include "common.h"

struct SmallSel {
  double s2[64];    // squared values, decreasing
  int32_t perm[64]; // their rows
  SelOut o;
};

// Every thread of the workgroup (at least 64) calls it, with nrm2 visible to all.
__device__ __forceinline__ void small_select(SmallSel& Z, const double* nrm2, int m, int kmax, double eps) {
  const int j = threadIdx.x;
  if (j < 64) {   // the first wave
    double v = -2.0;
    if (j < m) {
      v = nrm2[j];
      // NaN or negative entries (non-finite input, flagged already) sort last
      if (!(v >= 0.0) || !(v <= 1.0e300)) v = -1.0;
    }
    int rank = 0;
    for (int i = 0; i < m; ++i) {
      const double w = __shfl(v, i);
      rank += (w > v) || (w == v && i < j);
    }
    if (j < m) {
      Z.s2[rank] = fmax(v, 0.0);
      Z.perm[rank] = j;
    }
  }
  __syncthreads();
  if (j < 64) {
    const double x = j < m ? Z.s2[j] : 0.0;
    double t = x;   // sum of the values from j on, smallest first
    for (int o = 1; o < 64; o <<= 1) {
      const double u = __shfl_down(t, o);
      if (j + o < 64) t += u;
    }
    const double total = __shfl(t, 0);
    int k = m;
    if (eps >= 0.0) k = 1 + __popcll(__ballot(j >= 1 && j < m && !(t <= eps * total)));
    if (k > kmax) k = kmax;
    if (k < 1) k = 1;
    const double disc = k < m ? __shfl(t, k) : 0.0;
    double kept = j < k ? x : 0.0;
    for (int o = 32; o > 0; o >>= 1) kept += __shfl_xor(kept, o);
    if (j == 0) {
      Z.o.k = k;
      Z.o.m = m;
      Z.o.disc = disc;
      Z.o.norm2 = total;
      Z.o.nk = kept > 0.0 ? sqrt(kept) : 1.0;
    }
  }
  __syncthreads();
}

// The Hastings write-back of one bond: B_{b+1} and the rows of V^dag, Lambda,
// chi, the discarded weight, and the product that makes B_b.
template <class T>
__device__ __forceinline__ void small_bond_out(const SmallSel& Z, const BondItem& it, const double2* X, int m, int n,
                                               int ld, SelOut* sel, GemmProb* prob, const DiscLog& lg) {
  const int k = Z.o.k, d = it.d, chr = n / d;
  T* const Vh = (T*)it.Vh;
  T* const Br = (T*)it.Br;
  for (int idx = threadIdx.x; idx < k * n; idx += blockDim.x) {
    const int j = idx / n, col = idx - j * n;
    const double s = sqrt(Z.s2[j]), inv = s > 0.0 ? 1.0 / s : 0.0;
    const double2 x = X[(size_t)Z.perm[j] * ld + col];
    T v;
    v.x = x.x * inv;
    v.y = x.y * inv;
    const int vv = col / chr, c = col - vv * chr;
    Br[((size_t)j * d + vv) * it.chi_max + c] = v;
    Vh[idx] = v;
  }
  if ((int)threadIdx.x < k) it.lam_m[threadIdx.x] = sqrt(Z.s2[threadIdx.x]) / Z.o.nk;
  if (threadIdx.x == 0) {
    it.chi[it.b + 1] = k;
    it.disc[it.b] += Z.o.disc;
    if (lg.log) lg.log[(long long)(*lg.step) * lg.step_stride + lg.layer_off + it.pad] = Z.o.disc;
    *sel = Z.o;
    GemmProb p;
    p.A = it.T;
    p.B = it.Vh;
    p.C = it.Bl;
    p.M = m;
    p.N = k;
    p.K = n;
    p.lda = n;
    p.ldb = n;
    p.ldc = it.chi_max;
    p.M_dev = p.N_dev = p.K_dev = nullptr;
    p.M_mul = p.N_mul = p.K_mul = 1;
    p.inv_alpha_dev = &sel->nk;
    p.alpha = 1.0;
    *prob = p;
  }
}

// Where a stand-alone truncation's results go (complex128).
struct TruncOut {
  const double2* theta;   // [m][n], the input
  double2* U;             // [m][chi_max]
  double2* Vh;            // [k][n]
  double* S;
  int32_t* k;
  double *disc, *norm2;
  int64_t chi_max;
};

// V^dag rows, values, and U = theta V / s.
__device__ __forceinline__ void small_trunc_out(const SmallSel& Z, const TruncOut& o, const double2* X, int m, int n,
                                                int ld) {
  const int k = Z.o.k;
  for (int idx = threadIdx.x; idx < k * n; idx += blockDim.x) {
    const int j = idx / n, col = idx - j * n;
    const double s = sqrt(Z.s2[j]), inv = s > 0.0 ? 1.0 / s : 0.0;
    const double2 x = X[(size_t)Z.perm[j] * ld + col];
    o.Vh[(size_t)j * n + col] = make_double2(x.x * inv, x.y * inv);
  }
  if ((int)threadIdx.x < k) o.S[threadIdx.x] = sqrt(Z.s2[threadIdx.x]);
  if (threadIdx.x == 0) {
    *o.k = k;
    *o.disc = Z.o.disc;
    *o.norm2 = Z.o.norm2;
  }
  // four adjacent lanes an entry of U; sum_c theta conj(x_c) / s^2, x = s v
  const int q = threadIdx.x & 3;
  for (int idx = threadIdx.x >> 2; idx < m * k; idx += blockDim.x >> 2) {
    const int i = idx / k, j = idx - i * k;
    const double2 *a = o.theta + (size_t)i * n, *x = X + (size_t)Z.perm[j] * ld;
    const double s = sqrt(Z.s2[j]), inv = s > 0.0 ? 1.0 / s : 0.0;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int c = q; c < n; c += 4) {
      const double2 y = a[c], v = make_double2(x[c].x * inv, x[c].y * inv);
      acc.x += y.x * v.x + y.y * v.y;
      acc.y += y.y * v.x - y.x * v.y;
    }
    acc.x += __shfl_xor(acc.x, 1);
    acc.y += __shfl_xor(acc.y, 1);
    acc.x += __shfl_xor(acc.x, 2);
    acc.y += __shfl_xor(acc.y, 2);
    if (q == 0) o.U[(size_t)i * o.chi_max + j] = make_double2(acc.x * inv, acc.y * inv);
  }
}
