// observables of a Hastings-form chain with FP64 accumulation.
//
// Local expectation values from the one-site reduced density matrix
// rho_i = sum lam_i^2 B_i B_i^dag, two-site expectation values from
// theta_b = lam_b B_b B_{b+1}, and the bond entropy S = -sum lam^2 ln lam^2
// (Sec. "Observables", Eq. reducedrho; Sec. "Basic concepts", bond entropy).
#include "common.h"
#include "mfma_tile.h"

__global__ void obs_zero_kernel(double* a, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) a[i] = 0.0;
}

__device__ double obs_block_sum(double v, double* red) {
  const int tid = threadIdx.x;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (tid == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += red[w];
  __syncthreads();
  return r;
}

template <class T>
__device__ __forceinline__ double2 ld2(const void* p, size_t i) {
  T v = ((const T*)p)[i];
  return make_double2((double)v.x, (double)v.y);
}

// one workgroup per site, compiled per d so that a pair's entries stay in
// registers (L = 64, chi = 256: 0.47 ms with d at run time and 256 threads, now
// 0.06; chi = 24: 7.3 us, now 4.3)
// site_out[i], or with step: site_out[(*step) * step_stride + i] (a log whose
// row the device counter selects, so a replayed graph writes the right row)
template <class T, int D>
__global__ __launch_bounds__(1024) void obs_site_kernel(mps_chain_desc c, const double2* __restrict__ op1,
                                                        double* site_out, const int32_t* step, long long step_stride) {
  __shared__ double red[16];
  const int i = blockIdx.x, cm = c.chi_max;
  const int chl = c.chi[i], chr = c.chi[i + 1];
  const size_t Boff = (size_t)i * cm * D * cm;
  const double* lam = c.lam + (size_t)i * cm;
  double2 op[D * D];
#pragma unroll
  for (int q = 0; q < D * D; ++q) op[q] = op1[q];
  double acc = 0.0;
  for (int idx = threadIdx.x; idx < chl * chr; idx += blockDim.x) {
    const int a = idx / chr, cc = idx % chr;
    double2 v[D];
#pragma unroll
    for (int s = 0; s < D; ++s) v[s] = ld2<T>(c.B, Boff + ((size_t)a * D + s) * cm + cc);
    double part = 0.0;
#pragma unroll
    for (int sp = 0; sp < D; ++sp) {
      double2 ov = make_double2(0.0, 0.0);
#pragma unroll
      for (int s = 0; s < D; ++s) ov = cadd(ov, cmul(op[sp * D + s], v[s]));
      part += v[sp].x * ov.x + v[sp].y * ov.y;  // Re(conj(v_sp) * ov)
    }
    acc += lam[a] * lam[a] * part;
  }
  const double r = obs_block_sum(acc, red);
  if (threadIdx.x == 0) site_out[(step ? (long long)(*step) * step_stride : 0) + i] = r;
}

template <class T>
static hipError_t obs_sites(hipStream_t s, const mps_chain_desc& c, const double2* op1, double* out,
                            const int32_t* step, long long stride) {
  const int nt = c.chi_max * c.chi_max > 1024 ? 1024 : 256;
  switch (c.d) {
    case 1: obs_site_kernel<T, 1><<<c.L, nt, 0, s>>>(c, op1, out, step, stride); break;
    case 2: obs_site_kernel<T, 2><<<c.L, nt, 0, s>>>(c, op1, out, step, stride); break;
    case 3: obs_site_kernel<T, 3><<<c.L, nt, 0, s>>>(c, op1, out, step, stride); break;
    case 4: obs_site_kernel<T, 4><<<c.L, nt, 0, s>>>(c, op1, out, step, stride); break;
    case 5: obs_site_kernel<T, 5><<<c.L, nt, 0, s>>>(c, op1, out, step, stride); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// <theta_b|op2|theta_b>: theta_b in tiles of AC rows a and AC columns c (all
// D x D physical indices of both, AC = 64 / D) as products B_b B_{b+1} on FP64
// MFMA, the operator applied to the tile in LDS; grid (tiles, L - 1), one
// atomic add a tile.  Bound by the MFMA: L = 64, chi = 256, d = 2 took 12.1 ms
// with a workgroup per row a and the D x D entries of theta in private memory,
// now 0.52 ms.
template <class T, int D>
__global__ __launch_bounds__(256) void obs_bond_kernel(mps_chain_desc c, const double2* __restrict__ op2,
                                                       int per_bond, int nt, double* bond_out) {
  constexpr int AC = 64 / D, DD = D * D, CL = 65;
  __shared__ union {
    struct {
      double2 a[2][TBK * CL], b[2][TBK * CL];
    } st;
    double2 th[64 * CL];
  } L;
  __shared__ double red[4];
  const int b = blockIdx.y, cm = c.chi_max;
  const int chl = c.chi[b], chm = c.chi[b + 1], chr = c.chi[b + 2];
  const int a0 = (int)(blockIdx.x / nt) * AC, c0 = (int)(blockIdx.x % nt) * AC;
  if (a0 >= chl || c0 >= chr) return;
  const size_t B0 = (size_t)b * cm * D * cm, B1 = (size_t)(b + 1) * cm * D * cm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  // rows (a, s), 16 of them a thread's apart, the lanes along be; rows be, the
  // lanes along the columns (t, c)
  const int hi = tid >> 4, lo = tid & 15;
  double2 ra[4], rb[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = hi + 16 * q;
      ra[q] = i < AC * D && a0 + i / D < chl && k0 + lo < chm ? ld2<T>(c.B, B0 + ((size_t)a0 * D + i) * cm + k0 + lo)
                                                             : make_double2(0.0, 0.0);
    }
    const int k = k0 + hi;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int col = lo + 16 * u, t = col / AC, cc = c0 + col % AC;
      rb[u] = k < chm && t < D && cc < chr ? ld2<T>(c.B, B1 + ((size_t)k * D + t) * cm + cc) : make_double2(0.0, 0.0);
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) L.st.a[buf][lo * CL + hi + 16 * q] = ra[q];
#pragma unroll
    for (int u = 0; u < 4; ++u) L.st.b[buf][hi * CL + lo + 16 * u] = rb[u];
  };
  AccTileT<double2, 2, 2> acc;
  acc_zero_t<double2, 2, 2>(acc);
  load(0);
  stage(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < chm; k0 += TBK) {
    const bool more = k0 + TBK < chm;
    if (more) load(k0 + TBK);
    mma_chunk_t<double2, 2, 2>(L.st.a[buf], CL, L.st.b[buf], CL, acc, wm, wn, lane);
    if (more) stage(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        L.th[(wm + x * 16 + Cx<double2>::acc_row(lane, r)) * CL + wn + y * 16 + (lane & 15)] =
            make_double2(acc.re[x][y][r], acc.im[x][y][r]);
  __syncthreads();
  const double2* O = op2 + (per_bond ? (size_t)b * DD * DD : 0);
  double sum = 0.0;
  for (int idx = tid; idx < AC * AC; idx += 256) {
    const int a = idx / AC, cc = idx % AC;
    if (a0 + a >= chl || c0 + cc >= chr) continue;
    double2 th[DD];
#pragma unroll
    for (int q = 0; q < DD; ++q) th[q] = L.th[(a * D + q / D) * CL + q % D * AC + cc];
    double part = 0.0;
#pragma unroll
    for (int p = 0; p < DD; ++p) {
      double2 ov = make_double2(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < DD; ++q) ov = cadd(ov, cmul(O[p * DD + q], th[q]));
      part += th[p].x * ov.x + th[p].y * ov.y;
    }
    const double la = c.lam[(size_t)b * cm + a0 + a];
    sum += la * la * part;
  }
  const double r = obs_block_sum(sum, red);
  if (tid == 0) atomicAdd(&bond_out[b], r);
}

template <class T, int D>
static void obs_bond_go(hipStream_t s, const mps_chain_desc& c, const double2* op2, int per_bond, double* out) {
  const int nt = (c.chi_max + 64 / D - 1) / (64 / D);
  obs_bond_kernel<T, D><<<dim3(nt * nt, c.L - 1), 256, 0, s>>>(c, op2, per_bond, nt, out);
}
template <class T>
static hipError_t obs_bonds(hipStream_t s, const mps_chain_desc& c, const double2* op2, int per_bond, double* out) {
  switch (c.d) {
    case 1: obs_bond_go<T, 1>(s, c, op2, per_bond, out); break;
    case 2: obs_bond_go<T, 2>(s, c, op2, per_bond, out); break;
    case 3: obs_bond_go<T, 3>(s, c, op2, per_bond, out); break;
    case 4: obs_bond_go<T, 4>(s, c, op2, per_bond, out); break;
    case 5: obs_bond_go<T, 5>(s, c, op2, per_bond, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ void obs_entropy_kernel(mps_chain_desc c, double* ent) {
  __shared__ double red[4];
  const int b = blockIdx.x, cm = c.chi_max;
  const int k = c.chi[b + 1];
  const double* lam = c.lam + (size_t)(b + 1) * cm;
  double acc = 0.0;
  for (int j = threadIdx.x; j < k; j += blockDim.x) {
    double p = lam[j] * lam[j];
    if (p > 0.0) acc -= p * log(p);
  }
  double r = obs_block_sum(acc, red);
  if (threadIdx.x == 0) ent[b] = r;
}

hipError_t launch_observe(hipStream_t s, const mps_chain_desc& c, const double2* op1, double* site_out,
                          const double2* op2, int op2_per_bond, double* bond_out, double* entropy_out) {
  if (op1 && site_out) {
    hipError_t e = c.dtype == 1 ? obs_sites<double2>(s, c, op1, site_out, nullptr, 0)
                                : obs_sites<float2>(s, c, op1, site_out, nullptr, 0);
    if (e != hipSuccess) return e;
  }
  if (op2 && bond_out && c.L > 1) {
    obs_zero_kernel<<<1, 256, 0, s>>>(bond_out, c.L - 1);
    hipError_t e = c.dtype == 1 ? obs_bonds<double2>(s, c, op2, op2_per_bond, bond_out)
                                : obs_bonds<float2>(s, c, op2, op2_per_bond, bond_out);
    if (e != hipSuccess) return e;
  }
  if (entropy_out && c.L > 1) {
    obs_entropy_kernel<<<c.L - 1, 256, 0, s>>>(c, entropy_out);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t launch_observe_log(hipStream_t s, const mps_chain_desc& c, const double2* op1, double* log,
                              const int32_t* step, long long step_stride) {
  return c.dtype == 1 ? obs_sites<double2>(s, c, op1, log, step, step_stride)
                      : obs_sites<float2>(s, c, op1, log, step, step_stride);
}
