// Structured effective Hamiltonian, environment updates and Lanczos vector
// kernels for the local Krylov (two-site TDVP) path.
//
// Effective Hamiltonian (Sec. "Fundamentals of the library", Fig.
// LanczosMPS): the left and right environments and the MPO matrices of the
// active sites are applied to the two-site tensor one contraction at a time,
// never forming the chi^2 d^2 square matrix:
//   X1[a',b,s,t,c]  = sum_a   L[a',b,a] x[a,s,t,c]                  (MFMA GEMM)
//   X2[a',g,s',t,c] = sum_b,s W1[b,g,s',s] X1[a',b,s,t,c]           (MPO mix)
//   X3[a',s',t',e,c]= sum_g,t W2[g,e,t',t] X2[a',g,s',t,c]          (MPO mix)
//   y[a',s',t',c']  = sum_e,c X3[a',s',t',e,c] R[c',e,c]             (MFMA GEMM)
// The Lanczos recurrence of Sec. "Krylov time evolution" (Eq.
// krylov:approx) runs on FP64 vectors: multi-vector inner products, the
// Gram-Schmidt subtraction and the final combination are wavefront
// reductions / streaming kernels; the exponential of the small tridiagonal
// matrix is a Taylor series on one wave (or the LDS Jacobi eigensolver).
#include <algorithm>
#include <type_traits>

#include "lanes.h"
#include "mfma_3m.h"
#include "jacobi_small.h"
#include "krylov_small.h"

// ---------------------------------------------------------------------------
// strided complex GEMM: C = alpha op(A) op(B), element strides, optional conj
// ---------------------------------------------------------------------------

// Tile (32 MI) x (32 NJ) per 256-thread workgroup (2 x 2 waves); the shape is
// chosen per (precision, shape class) from the table the autotuner fills.
template <class T, int MI, int NJ>
struct SGemmLds {
  static constexpr int kElems = 2 * TBK * (32 * MI + 1 + 32 * NJ + 1);
};

// Bound by the MFMA for large products (78 % of its cycles busy for complex128
// 1024 x 512 and more; 2.13 ms a product of H_eff at chi = 512, d = 2, w = 5 with four
// neighbours a thread and an even pitch, now 1.45).
// Output tile (tm, tn) of P; stage holds SGemmLds<T, MI, NJ>::kElems elements
// (two staging buffers, each an A and a B chunk).
template <class T, int MI, int NJ>
__device__ __forceinline__ void sgemm_tile(const SGemm& P, int tm, int tn, T* stage) {
  constexpr int BM = 32 * MI, BN = 32 * NJ, LDA = BM + 1, LDB = BN + 1;
  typedef typename Cx<T>::R R;
  // chunks in flight in registers: two for complex128, one for complex64
  // (measured fastest with the three accumulators of either precision)
  constexpr int kPf = sizeof(T) == 16 ? 2 : 1;
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * MI * 16, wn = (wave & 1) * NJ * 16;
  T* C = (T*)P.C;
  // three real products per complex one (mfma_3m.h)
  Acc3<T, MI, NJ> acc;
  acc_clear(acc);
  SgOperand<T, BM> oa((const T*)P.A, P.rsA, P.csA, m0, P.M);
  SgOperand<T, BN> ob((const T*)P.B, P.csB, P.rsB, n0, P.N);
  const R ca = P.conjA ? -1 : 1, cb = P.conjB ? -1 : 1;
  T va[kPf][BM / 16], vb[kPf][BN / 16];
  auto load = [&](int ci, T (&da)[BM / 16], T (&db)[BN / 16]) {
    oa.load(da, P.K - ci * TBK);
    ob.load(db, P.K - ci * TBK);
  };
  auto store = [&](int buf, const T (&da)[BM / 16], const T (&db)[BN / 16]) {
    T* As = stage + buf * TBK * (LDA + LDB);
    oa.store(As, da, ca);
    ob.store(As + TBK * LDA, db, cb);
  };
  const int nch = (P.K + TBK - 1) / TBK;
#pragma unroll
  for (int u = 0; u < kPf; ++u)
    if (u < nch) load(u, va[u], vb[u]);
  if (nch > 0) store(0, va[0], vb[0]);
  __syncthreads();
  for (int base = 0; base < nch; base += kPf) {
#pragma unroll
    for (int u = 0; u < kPf; ++u) {
      const int ci = base + u;
      if (ci < nch) {
        if (ci + kPf < nch) load(ci + kPf, va[u], vb[u]);  // chunk ci's registers were staged already
        const T* As = stage + (ci & 1) * TBK * (LDA + LDB);
        acc_chunk(As, LDA, As + TBK * LDA, LDB, acc, wm, wn, lane);
        if (ci + 1 < nch) store((ci + 1) & 1, va[(u + 1) % kPf], vb[(u + 1) % kPf]);
        __syncthreads();
      }
    }
  }
  const R alpha = P.alpha_dev ? (R)(*P.alpha_dev) : (R)P.alpha;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int row = m0 + wm + i * 16 + Cx<T>::acc_row(lane, r);
        int col = n0 + wn + j * 16 + (lane & 15);
        if (row < P.M && col < P.N) {
          T v = acc_value(acc, i, j, r);
          v.x *= alpha;
          v.y *= alpha;
          C[(long long)row * P.rsC + (long long)col * P.csC] = v;
        }
      }
}

template <class T, int MI, int NJ>
__global__ __launch_bounds__(256) void sgemm_kernel(SGemm P, int ntn) {
  __shared__ T stage[SGemmLds<T, MI, NJ>::kElems];
  sgemm_tile<T, MI, NJ>(P, blockIdx.x / ntn, blockIdx.x % ntn, stage);
}

// A batch of independent products, problem blockIdx.y; the grid covers the
// largest, tiles past a problem's dimensions return at once.
template <class T, int MI, int NJ>
__global__ __launch_bounds__(256) void sgemm_batched_kernel(const SGemm* __restrict__ probs, int ntn) {
  __shared__ T stage[SGemmLds<T, MI, NJ>::kElems];
  const SGemm P = probs[blockIdx.y];
  const int tm = blockIdx.x / ntn, tn = blockIdx.x % ntn;
  if (tm * 32 * MI >= P.M || tn * 32 * NJ >= P.N) return;
  sgemm_tile<T, MI, NJ>(P, tm, tn, stage);
}

hipError_t launch_sgemm_batched(hipStream_t s, const SGemm* probs, int n_probs, int M_max, int N_max) {
  if (n_probs <= 0 || M_max <= 0 || N_max <= 0) return hipSuccess;
  if (n_probs > 65535) return hipErrorInvalidValue;
  const bool small = gemm_small(M_max, N_max, n_probs);
  const int b = small ? 32 : 64, ntm = (M_max + b - 1) / b, ntn = (N_max + b - 1) / b;
  if (small) sgemm_batched_kernel<double2, 1, 1><<<dim3(ntm * ntn, n_probs), 256, 0, s>>>(probs, ntn);
  else sgemm_batched_kernel<double2, 2, 2><<<dim3(ntm * ntn, n_probs), 256, 0, s>>>(probs, ntn);
  return hipGetLastError();
}

// Tile shape per (precision, shape class), candidate indices of
// gemm_cand_mi / gemm_cand_nj; until the autotuner sets one (-1, reported as
// 0), 64 x 64 or by gemm_small() 32 x 32.
static int g_sgemm_choice[2][kGemmShapeClasses] = {{-1, -1, -1, -1}, {-1, -1, -1, -1}};

int gemm_shape_class(long long M, long long N) {
  if (M * N <= 64LL * 64 * 64) return 0;   // at most 64 default tiles: few workgroups
  if (M >= 2 * N) return 1;                // tall
  if (N >= 2 * M) return 2;                // wide
  return 3;
}

void set_sgemm_choice(bool c128, int shape_class, int cand) { g_sgemm_choice[c128 ? 1 : 0][shape_class] = cand; }
int get_sgemm_choice(bool c128, int shape_class) { return std::max(0, g_sgemm_choice[c128 ? 1 : 0][shape_class]); }

template <class T, int MI, int NJ>
static hipError_t sgemm_go(hipStream_t s, const SGemm& P) {
  const int ntm = (P.M + 32 * MI - 1) / (32 * MI), ntn = (P.N + 32 * NJ - 1) / (32 * NJ);
  sgemm_kernel<T, MI, NJ><<<ntm * ntn, 256, 0, s>>>(P, ntn);
  return hipGetLastError();
}

template <class T>
static hipError_t sgemm_cand(hipStream_t s, const SGemm& P, int cand) {
  switch (cand) {
    case 1: return sgemm_go<T, 4, 2>(s, P);
    case 2: return sgemm_go<T, 2, 4>(s, P);
    case 3: return sgemm_go<T, 1, 2>(s, P);
    case 4: return sgemm_go<T, 2, 1>(s, P);
    case 5: return sgemm_go<T, 1, 1>(s, P);
    default: return sgemm_go<T, 2, 2>(s, P);
  }
}

hipError_t launch_sgemm_cand(hipStream_t s, const SGemm& P, bool c128, int cand) {
  if (P.M <= 0 || P.N <= 0) return hipSuccess;
  return c128 ? sgemm_cand<double2>(s, P, cand) : sgemm_cand<float2>(s, P, cand);
}

hipError_t launch_sgemm(hipStream_t s, const SGemm& P, bool c128) {
  const int set = g_sgemm_choice[c128 ? 1 : 0][gemm_shape_class(P.M, P.N)];
  return launch_sgemm_cand(s, P, c128, set >= 0 ? set : gemm_small(P.M, P.N, 1) ? 5 : 0);
}

// ---------------------------------------------------------------------------
// MPO mix: out[o1,o2,(qo1,qo2),r] = sum_(qi1,qi2) Wm[(qo1 qo2),(qi1 qi2)] in[o1,o2,(qi1,qi2),r]
// with independent strides; Wm is built on the device from the MPO tensor.
// ---------------------------------------------------------------------------

// Wm[(qo1*O2+qo2)*(Q1*Q2) + qi1*Q2+qi2] = W[qo1*ws_o1 + qo2*ws_o2 + qi1*ws_i1 + qi2*ws_i2]
template <class T>
__global__ void wmix_build_kernel(const T* W, T* Wm, int O1, int O2, int Q1, int Q2, int ws_o1, int ws_o2,
                                  int ws_i1, int ws_i2) {
  int n = O1 * O2 * Q1 * Q2;
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    int qi = e % (Q1 * Q2), qo = e / (Q1 * Q2);
    int qo1 = qo / O2, qo2 = qo % O2, qi1 = qi / Q2, qi2 = qi % Q2;
    Wm[e] = W[qo1 * ws_o1 + qo2 * ws_o2 + qi1 * ws_i1 + qi2 * ws_i2];
  }
}

// One thread per position and group of outputs (blockIdx.y): the QI >= Q1 Q2
// inputs of the position stay in registers (zero past Q1 Q2, as Wm's rows in
// LDS), unrolled for the MPO and site dimensions in use.  A large tensor has
// one group, so every input is read once; a small one is cut into groups of
// outputs until the grid fills the chip (at chi = 10, d = 5, w = 4 one thread
// per position is two workgroups of twenty outputs each: 28 us, cut 5.4 us).
template <class T, int QI>
__global__ __launch_bounds__(256) void mix_kernel(MixDesc D, const T* __restrict__ in, const T* __restrict__ Wm,
                                                  T* __restrict__ out, int po) {
  __shared__ T Ws[32 * QI];
  typedef typename Cx<T>::R R;
  const int Qi = D.Q1 * D.Q2, Qo = D.O1 * D.O2;
  const int p0 = blockIdx.y * po, p1e = min(Qo, p0 + po);
  for (int e = threadIdx.x; e < (p1e - p0) * QI; e += blockDim.x) {
    const int p = e / QI, q = e - p * QI;
    Ws[e] = q < Qi ? Wm[(p0 + p) * Qi + q] : Cx<T>::make(0.0, 0.0);
  }
  __syncthreads();
  const long long total = (long long)D.P1 * D.P2 * D.R;
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    int r, o1, o2;
    if (total < (1u << 31)) {   // (64-bit divisions cost more than the products of a small tensor)
      const unsigned i32 = (unsigned)idx, rest = i32 / (unsigned)D.R;
      r = (int)(i32 - rest * (unsigned)D.R);
      o1 = (int)(rest / (unsigned)D.P2);
      o2 = (int)(rest - (unsigned)o1 * (unsigned)D.P2);
    } else {
      r = (int)(idx % D.R);
      const long long rest = idx / D.R;
      o2 = (int)(rest % D.P2), o1 = (int)(rest / D.P2);
    }
    const T* ip = in + o1 * D.is_o1 + o2 * D.is_o2 + r * D.is_r;
    T x[QI];
    long long at = 0;   // of input q = (q1, q2), counted up
    int q2 = 0;
#pragma unroll
    for (int q = 0; q < QI; ++q) {
      x[q] = Cx<T>::make(0.0, 0.0);
      if (q < Qi) x[q] = ip[at];
      ++q2;
      at += q2 == D.Q2 ? D.is_q1 - (D.Q2 - 1) * D.is_q2 : D.is_q2;
      if (q2 == D.Q2) q2 = 0;
    }
    T* op = out + o1 * D.os_o1 + o2 * D.os_o2 + r * D.os_r;
    int p1 = p0 / D.O2, p2 = p0 - p1 * D.O2;
    for (int p = p0; p < p1e; ++p) {
      const T* w = Ws + (p - p0) * QI;
      R ar = 0, ai = 0;
#pragma unroll
      for (int q = 0; q < QI; ++q) {
        const T wq = w[q];
        ar += wq.x * x[q].x - wq.y * x[q].y;
        ai += wq.x * x[q].y + wq.y * x[q].x;
      }
      T v;
      v.x = ar;
      v.y = ai;
      op[p1 * D.os_q1 + p2 * D.os_q2] = v;
      if (++p2 == D.O2) {
        p2 = 0;
        ++p1;
      }
    }
  }
}

hipError_t launch_wmix_build(hipStream_t s, const void* W, void* Wm, int O1, int O2, int Q1, int Q2, int ws_o1,
                             int ws_o2, int ws_i1, int ws_i2, bool c128) {
  if (c128)
    wmix_build_kernel<double2><<<1, 256, 0, s>>>((const double2*)W, (double2*)Wm, O1, O2, Q1, Q2, ws_o1, ws_o2,
                                                ws_i1, ws_i2);
  else
    wmix_build_kernel<float2><<<1, 256, 0, s>>>((const float2*)W, (float2*)Wm, O1, O2, Q1, Q2, ws_o1, ws_o2, ws_i1,
                                               ws_i2);
  return hipGetLastError();
}

template <class T>
static void mix_go(hipStream_t s, const MixDesc& D, const void* in, const void* Wm, void* out) {
  const long long total = (long long)D.P1 * D.P2 * D.R;
  const int gx = (int)std::min<long long>((total + 255) / 256, 8192), Qi = D.Q1 * D.Q2, Qo = D.O1 * D.O2;
  // at least one workgroup per CU, as long as there are outputs to deal out
  const int groups = std::max(1, std::min(Qo, (256 + gx - 1) / gx));
  const int po = (Qo + groups - 1) / groups;
  const dim3 grid(gx, (Qo + po - 1) / po);
  const T *i = (const T*)in, *w = (const T*)Wm;
  T* o = (T*)out;
  if (Qi <= 8) mix_kernel<T, 8><<<grid, 256, 0, s>>>(D, i, w, o, po);
  else if (Qi <= 12) mix_kernel<T, 12><<<grid, 256, 0, s>>>(D, i, w, o, po);
  else if (Qi <= 16) mix_kernel<T, 16><<<grid, 256, 0, s>>>(D, i, w, o, po);
  else if (Qi <= 20) mix_kernel<T, 20><<<grid, 256, 0, s>>>(D, i, w, o, po);
  else mix_kernel<T, 32><<<grid, 256, 0, s>>>(D, i, w, o, po);
}

hipError_t launch_mix(hipStream_t s, const MixDesc& D, const void* in, const void* Wm, void* out, bool c128) {
  if ((long long)D.P1 * D.P2 * D.R <= 0) return hipSuccess;
  if (c128) mix_go<double2>(s, D, in, Wm, out);
  else mix_go<float2>(s, D, in, Wm, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP64 Lanczos vector kernels
// ---------------------------------------------------------------------------
__global__ void zero_kernel(double* a, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) a[i] = 0.0;
}

// One Gram-Schmidt pass over the Krylov vectors V_i = V + i ldv, i < nv <= NB:
//   SUB : r <- r - sum_i c_i V_i, with the overlaps c of the pass before;
//   then the overlaps <V_i, r>, or (NORM) |r|^2.
// yin (first pass of a complex64 apply): r is first read from it.
// Large vectors' passes are bound by reading V once, so the subtraction and the
// next overlaps share a launch and the entries that they read.  A
// workgroup leaves its shares of the sums in part_out; whoever needs a sum adds
// the shares of the launch before, every workgroup for itself and in
// workgroup order (so the sums do not depend on scheduling): 256 shares come
// from the L2 in about 2 us, where a last workgroup adding them behind an
// agent-scope fence in every workgroup cost 25 us and more, and a launch of
// its own with one thread per overlap 180 us.
// alpha_out: the diagonal entry Re c_{nv-1}, from the shares read.
// At chi = 160, d = 5 (640,000 entries, up to 20 vectors) the passes of one
// Krylov vector took 970 us as launches of their own, 250 us with the vectors read
// twice and the sums by permutes through the LDS unit, now 140.  A short vector's
// pass (12 vectors) went from 12.3 to 3.6 us, little more than its launch.
constexpr int kGsThreads = 512;
__host__ __device__ constexpr int gs_width(int nb) { return nb <= 4 ? 8 : nb <= 8 ? 16 : nb <= 16 ? 32 : 64; }

// sum of the g shares of every value, in sums[0, NV) after the barrier inside:
// a thread's shares, then the lanes that hold the same value, then the waves
template <int NV, int NT>
__device__ __forceinline__ void gs_collect(const double* __restrict__ part, int g, double* sums) {
  constexpr int G = NT / NV, NW = NT / 64;
  __shared__ double red[NW * NV];
  const int i = threadIdx.x % NV, k0 = threadIdx.x / NV, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double a = 0.0;
#pragma unroll 16
  for (int k = k0; k < g; k += G) a += part[(size_t)k * NV + i];
  if (NV <= 2) a += lane_xor<1>(a);
  if (NV <= 4) a += lane_xor<2>(a);
  if (NV <= 8) a += lane_xor<3>(a);
  if (NV <= 16) a = swap_add<false>(a, a);
  if (NV <= 32) a = swap_add<true>(a, a);
  if (lane < NV) red[wave * NV + lane] = a;
  __syncthreads();
  if (threadIdx.x < NV) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w * NV + threadIdx.x];
    sums[threadIdx.x] = t;
  }
  __syncthreads();
}

template <int NB, bool SUB, bool NORM>
__global__ __launch_bounds__(kGsThreads) void gs_kernel(const double2* __restrict__ V, long long ldv, int nv,
                                                        double2* r, const float2* __restrict__ yin, long long n,
                                                        const double* __restrict__ part_in, int g_in,
                                                        double* __restrict__ part_out, double* alpha_out) {
  constexpr int NVI = gs_width(NB), NV = NORM ? 2 : NVI, NW = kGsThreads / 64;
  constexpr bool HOLD = NB <= 20;   // the vectors' entries stay in registers between the two uses
  __shared__ double red[NW * NV];
  __shared__ double cs[kGsThreads];
  if (SUB) {
    gs_collect<NVI, kGsThreads>(part_in, g_in, cs);
    if (alpha_out && blockIdx.x == 0 && threadIdx.x == 0) *alpha_out = cs[2 * nv - 2];
  }
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  for (long long e = (long long)blockIdx.x * kGsThreads + threadIdx.x; e < n;
       e += (long long)gridDim.x * kGsThreads) {
    // no branch between the loads, so that they are in flight together (past
    // nv the last vector again, from L1, subtracted zero times and into sums
    // that nobody reads)
    double2 v[HOLD ? NB : 1];
    if constexpr (HOLD && (SUB || !NORM)) {
#pragma unroll
      for (int i = 0; i < NB; ++i) v[i] = V[min(i, nv - 1) * ldv + e];
    }
    double2 x;
    if (!SUB && yin) {
      x = make_double2(yin[e].x, yin[e].y);
      r[e] = x;
    } else {
      x = r[e];
    }
    if (SUB) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (HOLD || i < nv) {
          const double2 vi = HOLD ? v[HOLD ? i : 0] : V[i * ldv + e];
          const double cx = i < nv ? cs[2 * i] : 0.0, cy = i < nv ? cs[2 * i + 1] : 0.0;
          x.x -= cx * vi.x - cy * vi.y;
          x.y -= cx * vi.y + cy * vi.x;
        }
      r[e] = x;
    }
    if (NORM) {
      acc[0] += x.x * x.x + x.y * x.y;
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const double2 vi = HOLD ? v[HOLD ? i : 0] : V[min(i, nv - 1) * ldv + e];
        acc[2 * i] += vi.x * x.x + vi.y * x.y;
        acc[2 * i + 1] += vi.x * x.y - vi.y * x.x;
      }
    }
  }
  wave_sums<NV>(acc, red);
  __syncthreads();
  if (threadIdx.x < NV) {
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) a += red[w * NV + threadIdx.x];
    part_out[(size_t)blockIdx.x * NV + threadIdx.x] = a;
  }
}

// y = x / |x|, |x|^2 the sum of the g shares of a norm pass, and its complex64
// copy for the apply (optional)
__global__ __launch_bounds__(256) void scale_inv_norm_kernel(const double2* x, double2* y, float2* y32, long long n,
                                                             const double* __restrict__ part, int g) {
  __shared__ double sums[256];
  gs_collect<2, 256>(part, g, sums);
  const double norm2 = sums[0];
  const double s = norm2 > 0.0 ? 1.0 / sqrt(norm2) : 0.0;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    double2 v = x[e];
    v.x *= s;
    v.y *= s;
    y[e] = v;
    if (y32) y32[e] = make_float2((float)v.x, (float)v.y);
  }
}

// x = nrm * sum_i u_i V_i
__global__ void combine_kernel(const double2* __restrict__ V, long long ldv, int nv, const double2* __restrict__ u,
                               double nrm, double2* x, long long n) {
  __shared__ double2 us[32];
  if (threadIdx.x < nv) us[threadIdx.x] = u[threadIdx.x];
  __syncthreads();
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    double2 a = make_double2(0.0, 0.0);
    for (int i = 0; i < nv; ++i) {
      double2 v = V[i * ldv + e];
      a.x += us[i].x * v.x - us[i].y * v.y;
      a.y += us[i].x * v.y + us[i].y * v.x;
    }
    x[e] = make_double2(nrm * a.x, nrm * a.y);
  }
}

// precision conversion between the FP64 Krylov vectors and the apply dtype
__global__ void c128_to_c64_kernel(const double2* a, float2* b, long long n) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    b[e] = make_float2((float)a[e].x, (float)a[e].y);
}
__global__ void c64_to_c128_kernel(const float2* a, double2* b, long long n) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    b[e] = make_double2(a[e].x, a[e].y);
}

// Tridiagonal exponential of the Lanczos matrix (one workgroup):
// u = exp(-i tau T) e_1 and err = |x| beta_{n-1} |u_{n-1}|, with |x|^2 and
// beta_{n-1}^2 from the shares of their norm passes; beta[n-1] is set here and
// stop = {err, beta_{n-1}, |x|^2} for the host.  While |tau| |T| is
// moderate, as for a time step, the first wave takes the Taylor series in
// substeps of |tau| |T| / s <= 1 (20 terms: 1 / 20! is below rounding), one
// entry of u per lane: 10 us against 60 to 107 us of the Jacobi
// diagonalisation at n = 10 to 20, which the rest keep (its cost does not
// grow with |tau| |T|).
constexpr double kTaylorMax = 40.0;
__global__ __launch_bounds__(256) void tridiag_expm_kernel(const double* alpha, double* beta, int n, double tau_re,
                                                           double tau_im, const double* __restrict__ part_x,
                                                           const double* __restrict__ part_r, int g, double2* u,
                                                           double* stop) {
  __shared__ double sums[256];
  gs_collect<2, 256>(part_x, g, sums);
  const double nx = sums[0];
  __syncthreads();
  gs_collect<2, 256>(part_r, g, sums);
  const double nr = sums[0];
  const double nrm = nx < 0.0 ? 0.0 : sqrt(nx);
  double* const err = stop;
  if (threadIdx.x == 0) {
    beta[n - 1] = sqrt(nr);
    stop[1] = sqrt(nr);
    stop[2] = nx;
  }
  __syncthreads();
  // the largest row sum of |T|, a row a lane (n <= 64)
  double bound = 0.0;
  {
    const int i = threadIdx.x & 63;
    if (i < n) bound = fmax(0.0, fabs(alpha[i]) + (i > 0 ? fabs(beta[i - 1]) : 0.0) + (i + 1 < n ? fabs(beta[i]) : 0.0));
    for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, __shfl_xor(bound, o));
  }
  bound *= sqrt(tau_re * tau_re + tau_im * tau_im);
  if (bound <= kTaylorMax) {   // uniform; false for NaN
    if (threadIdx.x >= 64) return;
    const int i = threadIdx.x;
    const double a = i < n ? alpha[i] : 0.0, bl = i > 0 && i < n ? beta[i - 1] : 0.0,
                 br = i + 1 < n ? beta[i] : 0.0;
    const int s = bound > 1.0 ? (int)ceil(bound) : 1;
    // -i tau / s
    const double fr = tau_im / s, fi = -tau_re / s;
    double yr = i == 0 ? 1.0 : 0.0, yi = 0.0;
    for (int t = 0; t < s; ++t) {
      double tr = yr, ti = yi;
#pragma unroll
      for (int k = 1; k <= 20; ++k) {
        const double ur = dpp_d<kWaveShr1>(tr), ui = dpp_d<kWaveShr1>(ti);   // lane i - 1
        const double dr = dpp_d<kWaveShl1>(tr), di = dpp_d<kWaveShl1>(ti);   // lane i + 1
        const double zr = a * tr + bl * ur + br * dr, zi = a * ti + bl * ui + br * di;
        const double ik = 1.0 / k;
        tr = (fr * zr - fi * zi) * ik;
        ti = (fr * zi + fi * zr) * ik;
        yr += tr;
        yi += ti;
      }
    }
    if (i < n) u[i] = make_double2(yr, yi);
    if (i == n - 1) *err = nrm * fabs(beta[n - 1]) * sqrt(yr * yr + yi * yi);
    return;
  }
  __shared__ double2 G[JS_N * JS_LD];
  __shared__ double2 Q[JS_N * JS_LD];
  __shared__ double4 rot[16];
  __shared__ int flag;
  tridiag_expm_block(alpha, beta, n, tau_re, tau_im, nrm, u, err, G, Q, rot, &flag);
}

static int vgrid(long long n) { return (int)std::min<long long>((n + 255) / 256, 4096); }

hipError_t launch_zero(hipStream_t s, double* a, int n) {
  zero_kernel<<<std::max(1, std::min(64, (n + 255) / 256)), 256, 0, s>>>(a, n);
  return hipGetLastError();
}
int gs_shares(long long n) { return (int)std::min<long long>((n + kGsThreads - 1) / kGsThreads, kGsBlocks); }
hipError_t launch_gs(hipStream_t s, const double2* V, long long ldv, int nv, double2* r, const void* yin, long long n,
                     bool sub, bool norm, const double* part_in, double* part_out, double* alpha_out) {
  if (nv < 1 || nv > 32 || (sub && yin)) return hipErrorInvalidValue;
  const int g = gs_shares(n);
  const float2* y = (const float2*)yin;
  auto go = [&](auto kern) { kern<<<g, kGsThreads, 0, s>>>(V, ldv, nv, r, y, n, part_in, g, part_out, alpha_out); };
  if (!sub && norm) go(gs_kernel<4, false, true>);
  else if (nv <= 4) go(!sub ? gs_kernel<4, false, false> : norm ? gs_kernel<4, true, true> : gs_kernel<4, true, false>);
  else if (nv <= 8) go(!sub ? gs_kernel<8, false, false> : norm ? gs_kernel<8, true, true> : gs_kernel<8, true, false>);
  else if (nv <= 12)
    go(!sub ? gs_kernel<12, false, false> : norm ? gs_kernel<12, true, true> : gs_kernel<12, true, false>);
  else if (nv <= 16)
    go(!sub ? gs_kernel<16, false, false> : norm ? gs_kernel<16, true, true> : gs_kernel<16, true, false>);
  else if (nv <= 20)
    go(!sub ? gs_kernel<20, false, false> : norm ? gs_kernel<20, true, true> : gs_kernel<20, true, false>);
  else go(!sub ? gs_kernel<32, false, false> : norm ? gs_kernel<32, true, true> : gs_kernel<32, true, false>);
  return hipGetLastError();
}
hipError_t launch_scale_inv_norm(hipStream_t s, const double2* x, double2* y, void* y32, long long n,
                                 const double* part) {
  scale_inv_norm_kernel<<<vgrid(n), 256, 0, s>>>(x, y, (float2*)y32, n, part, gs_shares(n));
  return hipGetLastError();
}
hipError_t launch_combine(hipStream_t s, const double2* V, long long ldv, int nv, const double2* u, double nrm,
                          double2* x, long long n) {
  combine_kernel<<<vgrid(n), 256, 0, s>>>(V, ldv, nv, u, nrm, x, n);
  return hipGetLastError();
}
hipError_t launch_convert(hipStream_t s, const void* a, void* b, long long n, bool to_c64) {
  if (to_c64)
    c128_to_c64_kernel<<<vgrid(n), 256, 0, s>>>((const double2*)a, (float2*)b, n);
  else
    c64_to_c128_kernel<<<vgrid(n), 256, 0, s>>>((const float2*)a, (double2*)b, n);
  return hipGetLastError();
}
hipError_t launch_tridiag_expm(hipStream_t s, const double* alpha, double* beta, int n, double tau_re,
                               double tau_im, const double* part_x, const double* part_r, long long len, double2* u,
                               double* stop) {
  tridiag_expm_kernel<<<1, 256, 0, s>>>(alpha, beta, n, tau_re, tau_im, part_x, part_r, gs_shares(len), u, stop);
  return hipGetLastError();
}

// b[j][i] = a[i][j], a: m x n complex128
__global__ void transpose_c128_kernel(const double2* a, double2* b, int m, int n) {
  __shared__ double2 t[32][33];
  int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  for (int k = threadIdx.y; k < 32; k += blockDim.y) {
    int i = by + k, j = bx + threadIdx.x;
    if (i < m && j < n) t[k][threadIdx.x] = a[(size_t)i * n + j];
  }
  __syncthreads();
  for (int k = threadIdx.y; k < 32; k += blockDim.y) {
    int j = bx + k, i = by + threadIdx.x;
    if (i < m && j < n) b[(size_t)j * m + i] = t[threadIdx.x][k];
  }
}

hipError_t launch_transpose_c128(hipStream_t s, const double2* a, double2* b, int m, int n) {
  dim3 grid((n + 31) / 32, (m + 31) / 32), block(32, 8);
  transpose_c128_kernel<<<grid, block, 0, s>>>(a, b, m, n);
  return hipGetLastError();
}

// normalised kept rows of a converged Jacobi matrix: row j (sorted) divided
// by s_j, written as dst[j*len + e] (row-major) or dst[e*k + j] (column-major)
template <class T>
__global__ void write_rows_kernel(const JacMat* mat, const int32_t* perm, const double* s2, const SelOut* sel, T* dst,
                                  int len, int col_major) {
  const int k = sel->k;
  const JacMat M = *mat;
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < (long long)k * len;
       idx += (long long)gridDim.x * blockDim.x) {
    int j = (int)(idx / len), e = (int)(idx % len);
    int pj = perm[j];
    pj = (pj >= 0 && pj < M.m) ? pj : 0;
    double s = sqrt(s2[j]);
    double inv = s > 0.0 ? 1.0 / s : 0.0;
    double2 x = M.X[(size_t)pj * M.ld + e];
    T v;
    v.x = x.x * inv;
    v.y = x.y * inv;
    if (col_major)
      dst[(size_t)e * k + j] = v;
    else
      dst[(size_t)j * len + e] = v;
  }
}

hipError_t launch_write_rows(hipStream_t s, const JacMat* mat, const int32_t* perm, const double* s2, const SelOut* sel,
                             void* dst, int len, int col_major, bool c128) {
  int g = std::max(1, std::min(4096, (len * 64 + 255) / 256));
  if (c128)
    write_rows_kernel<double2><<<g, 256, 0, s>>>(mat, perm, s2, sel, (double2*)dst, len, col_major);
  else
    write_rows_kernel<float2><<<g, 256, 0, s>>>(mat, perm, s2, sel, (float2*)dst, len, col_major);
  return hipGetLastError();
}
