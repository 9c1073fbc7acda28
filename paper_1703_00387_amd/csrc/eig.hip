// Rotation of a batch of matrices onto their left singular vectors by a direct
// Hermitian eigensolver, in FP64, ahead of the one-sided Jacobi.
//
// For theta' (m x n) the split needs rows s_j v_j^dag, that is U^dag theta'
// with U the eigenvectors of G = theta' theta'^dag (Sec. "Basic concepts",
// Splitting).  The block Jacobi reaches them in 8 to 12 sweeps of nb - 1
// dependent rounds each, and that chain, not its arithmetic, sets its time.
// Here the same unitary comes from
//   1. G on FP64 MFMA (lower tiles),
//   2. Householder tridiagonalisation of G / |theta'|_F^2 (tri_kernel),
//   3. the divide-and-conquer eigensolver of the real tridiagonal matrix
//      (Cuppen's rank-one tearing; the secular equation in shifted variables;
//      the vectors from the recomputed z of Gu and Eisenstat, which makes them
//      orthogonal to working precision whatever the gaps),
//   4. theta' <- Q^T (H_{m-2}^dag ... H_0^dag theta') on FP64 MFMA, the
//      reflectors in blocks of 16 (compact WY form).
// The unitary is a product of reflections, plane rotations and
// Gu-Eisenstat vectors, so it is unitary to working precision by
// construction; how well it diagonalises G is then checked: the Gram of the
// rotated rows is formed again and held to the Jacobi's own convergence test,
// |G_pq| <= max(abs_tol |X|_F^2, tol sqrt(G_pp G_qq)).  A matrix that passes
// is done (its squared row norms are the diagonal of that Gram, as after the
// Jacobi's last round); one that does not, or whose team of workgroups gave
// up waiting, goes on to the Jacobi from wherever it is.
#include <algorithm>

#include "common.h"
#include "lanes.h"
#include "mfma_tile.h"
#include "jacobi_small.h"
#include "split_out.h"

namespace {

constexpr int kLeaf = 64;     // tridiagonal blocks solved in LDS
constexpr int kWy = 16;       // reflectors per block
constexpr double kEps = 2.220446049250313e-16;
// What of the unit-trace Gram counts as zero: squares of anything above are
// normal numbers, and so are the gaps and shifts of the divide and conquer (no
// less than kEps^2 of what they came from).  Dropping it changes the matrix by
// far less than rounding does.
constexpr double kTiny = 1e-100;
// Coupling of two rows of a panel, relative to their lengths, past which the
// shorter one is cleaned of the longer (small_clean).
constexpr double kRough = 1e-11;

// A matrix being rotated and its part of the scratch.
struct EigSlot {
  Gp<double2> X;      // theta', [m][ld]
  Gp<double2> A;      // [m][m]: the Gram (lower); then the eigenvectors Q0, Q1 (real [m][m] each); then the check's Gram
  Gp<double2> V;      // Householder vectors in blocks: [block][row][16]
  Gp<double2> E;      // exchange of the tridiagonalisation; then the vectors U of a merge; then the reflected theta' [m][n]
  Gp<double2> T;      // [block][16][16] compact WY factors
  Gp<double2> tau;    // [m]
  Gp<double> d;       // [m] diagonal, then eigenvalues
  Gp<double> e;       // [m] off-diagonal
  Gp<double> f;       // [8][m] work of the merges: sorted d, z, kept d, kept z, eta, rotations c, s, deflated values
  Gp<int32_t> g;      // [8][m] work of the merges: order, kept rank, deflated rank, origin, rotation pairs, counts
  Gp<int32_t> fail;   // set when the team gave up
  double scale;    // 1 / |theta'|_F^2
  int32_t m, n, ld, active;
};

// work arrays of a merge (offsets into f and g, in units of m)
enum { F_DS = 0, F_ZS, F_DK, F_ZK, F_ETA, F_C, F_S, F_DV };
enum { G_PM = 0, G_KR, G_DR, G_ORG, G_RA, G_RB, G_CNT, G_RANK };

__device__ __forceinline__ int eig_levels(int m) {
  int l = 0;
  while ((kLeaf << l) < m) ++l;
  return l;
}
// eigenvector buffer after `level` merge levels, transposed: Qt[i][r] = entry r of vector i
__device__ __forceinline__ double* eig_q(const EigSlot& S, int level) {
  return (double*)S.A + ((level & 1) ? (size_t)S.m * S.m : 0);
}

// ---------------------------------------------------------------------------
// slots
// ---------------------------------------------------------------------------
struct EigLayout {
  size_t A, V, E, T, tau, d, e, f, g, fail, bytes;
  EigLayout(int m, int n) {
    WsPlan p;
    const size_t mm = (size_t)m * m;
    const int nblk = (m + kWy - 1) / kWy;
    A = p.take<double2>(mm);
    V = p.take<double2>((size_t)nblk * kWy * m);
    E = p.take<double2>(std::max(2 * mm, (size_t)m * n));
    T = p.take<double2>((size_t)nblk * kWy * kWy);
    tau = p.take<double2>(m);
    d = p.take<double>(m);
    e = p.take<double>(m);
    f = p.take<double>((size_t)8 * m);
    g = p.take<int32_t>((size_t)8 * m);
    fail = p.take<int32_t>(1);
    bytes = (p.off + 255) & ~size_t(255);
  }
};

__global__ void eig_slots_kernel(EigSlot* slots, const JacMat* __restrict__ mats, int n, char* base, EigLayout L,
                                 int m_cap, int n_cap, int m_lim) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const JacMat M = mats[i];
  char* w = base + (size_t)i * L.bytes;
  EigSlot S;
  S.X = M.X;
  S.A = (double2*)(w + L.A);
  S.V = (double2*)(w + L.V);
  S.E = (double2*)(w + L.E);
  S.T = (double2*)(w + L.T);
  S.tau = (double2*)(w + L.tau);
  S.d = (double*)(w + L.d);
  S.e = (double*)(w + L.e);
  S.f = (double*)(w + L.f);
  S.g = (int32_t*)(w + L.g);
  S.fail = (int32_t*)(w + L.fail);
  *S.fail = 0;
  S.m = M.m;
  S.n = M.n;
  S.ld = M.ld;
  // (matrices of one panel have a path of their own); a Gram whose entries
  // leave the comfortable range is left to the Jacobi
  S.active = M.conv == 0 && M.m > 64 && eig_takes(M.m, M.n) && M.m <= min(m_cap, m_lim) && M.n <= n_cap &&
             M.fro2 > 1e-250 && M.fro2 < 1e250;
  S.scale = S.active ? 1.0 / M.fro2 : 0.0;
  if (!S.active) S.m = S.n = 0;
  slots[i] = S;
}

// ---------------------------------------------------------------------------
// Sums over adjacent lanes (lanes.h).
// ---------------------------------------------------------------------------
// every one of NL adjacent lanes (aligned) gets the sum over them
template <int NL>
__device__ __forceinline__ double lanes_sum(double a) {
  if (NL >= 2) a += dpp_d<kXor1>(a);
  if (NL >= 4) a += dpp_d<kXor2>(a);
  if (NL >= 8) a += dpp_d<kHalfMirror>(a);   // the quads hold their sums: any lane of the other quad will do
  if (NL >= 16) a += dpp_d<kMirror>(a);
  if (NL >= 32) a += __shfl_xor(a, 16);
  if (NL >= 64) a += __shfl_xor(a, 32);
  return a;
}
template <int NL>
__device__ __forceinline__ int lanes_sum(int a) {
  if (NL >= 2) a += dpp_i<kXor1>(a);
  if (NL >= 4) a += dpp_i<kXor2>(a);
  if (NL >= 8) a += dpp_i<kHalfMirror>(a);
  if (NL >= 16) a += dpp_i<kMirror>(a);
  if (NL >= 32) a += __shfl_xor(a, 16);
  if (NL >= 64) a += __shfl_xor(a, 32);
  return a;
}
template <int NL>
__device__ __forceinline__ int lanes_max(int a) {
  if (NL >= 2) a = max(a, dpp_i<kXor1>(a));
  if (NL >= 4) a = max(a, dpp_i<kXor2>(a));
  if (NL >= 8) a = max(a, dpp_i<kHalfMirror>(a));
  if (NL >= 16) a = max(a, dpp_i<kMirror>(a));
  return a;
}
template <int NL>
__device__ __forceinline__ double lanes_prod(double a) {
  if (NL >= 2) a *= dpp_d<kXor1>(a);
  if (NL >= 4) a *= dpp_d<kXor2>(a);
  if (NL >= 8) a *= dpp_d<kHalfMirror>(a);
  if (NL >= 16) a *= dpp_d<kMirror>(a);
  if (NL >= 32) a *= __shfl_xor(a, 16);
  if (NL >= 64) a *= __shfl_xor(a, 32);
  return a;
}
__device__ __forceinline__ double lane_get(double a, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(a), lane),
                          __builtin_amdgcn_readlane(__double2loint(a), lane));
}
// the sum over a wave, uniform: rows of 16 by DPP, the four rows as scalars
__device__ __forceinline__ double wave_sum(double a) {
  a = lanes_sum<16>(a);
  return (lane_get(a, 0) + lane_get(a, 16)) + (lane_get(a, 32) + lane_get(a, 48));
}

// What a wave's lanes wrote to LDS before is what its lanes read after.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Gram of the rows, lower tiles of 32 MI: C = X X^dag (C [m][m]).  Bound by the
// FP64 MFMA: one matrix of m = 512 took 0.150 ms and of m = 2560 9.1 ms with all
// tiles 64 x 64 and on one XCD, now 0.040 and 1.47 ms.
// ---------------------------------------------------------------------------
template <int MI>
__global__ __launch_bounds__(256) void eig_gram_kernel(const EigSlot* __restrict__ slots, int n_slots, int nt_cap) {
  __shared__ DaggerLds<MI> L;
  int item, tile;
  if (!xcd_item_tile(blockIdx.x, n_slots, nt_cap * (nt_cap + 1) / 2, item, tile)) return;
  const EigSlot& S = slots[item];
  // tile -> (tm >= tn), row by row of the triangle
  int tm = (int)((sqrt(8.0 * tile + 1.0) - 1.0) * 0.5);
  while ((tm + 1) * (tm + 2) / 2 <= tile) ++tm;
  while (tm * (tm + 1) / 2 > tile) --tm;
  const int tn = tile - tm * (tm + 1) / 2;
  const int m = S.m, m0 = tm * 32 * MI, n0 = tn * 32 * MI;
  if (m0 >= m) return;
  AccTileT<double2, MI, MI> acc;
  dagger_tile<MI>(S.X, S.ld, m, S.X, S.ld, m, S.n, m0, n0, L, acc);
  dagger_out<MI>(acc, m0, n0, [&](int row, int col, double2 x) {
    if (row < m && col < m) S.A[(size_t)row * m + col] = x;
  });
}
static void gram_go(hipStream_t s, const EigSlot* slots, int n, int m_cap) {
  const int nt64 = (m_cap + 63) / 64, mi = dagger_mi((long long)n * nt64 * (nt64 + 1) / 2);
  const int nt = (m_cap + 32 * mi - 1) / (32 * mi), grid = (int)xcd_grid(n, (long long)nt * (nt + 1) / 2);
  if (mi == 1) eig_gram_kernel<1><<<grid, 256, 0, s>>>(slots, n, nt);
  else eig_gram_kernel<2><<<grid, 256, 0, s>>>(slots, n, nt);
}

// ---------------------------------------------------------------------------
// Tridiagonalisation
// ---------------------------------------------------------------------------
// A value not yet written in the exchange: a NaN with a payload that no
// computation here produces (and that publishing avoids).
constexpr unsigned long long kEmpty = 0x7ff9dead5eed0001ull;

__global__ __launch_bounds__(256) void eig_fill_kernel(const EigSlot* __restrict__ slots) {
  const EigSlot& S = slots[blockIdx.y];
  const size_t total = (size_t)4 * S.m * S.m;
  unsigned long long* p = (unsigned long long*)S.E;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) p[i] = kEmpty;
}

__device__ __forceinline__ void xch_put(double* p, double v) {
  unsigned long long b = __double_as_longlong(v);
  if (b == kEmpty) b = 0x7ff8000000000000ull;
  __hip_atomic_store((unsigned long long*)p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Polls NW words at p[o[i]] together until all are there; false when they did
// not come.  Every word carries its own arrival, so no ordering between words
// is needed, and the loads of a poll are all in flight at once.
template <int NW>
__device__ __forceinline__ bool xch_get(const double* const (&p)[NW], double (&v)[NW], bool want, int limit) {
  if (!want) return true;
  for (int it = 0; it < limit; ++it) {
    unsigned long long b[NW];
    bool all = true;
#pragma unroll
    for (int i = 0; i < NW; ++i)
      b[i] = __hip_atomic_load((const unsigned long long*)p[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      all = all && b[i] != kEmpty;
      v[i] = __longlong_as_double(b[i]);
    }
    if (all) return true;
  }
  return false;
}

// Householder reflector of (alpha; x) with |x|^2 = xn2: H = I - tau v v^dag,
// v = (1; x / (alpha - beta)), H^dag (alpha; x) = (beta; 0), beta real.
__device__ __forceinline__ void reflector(double2 alpha, double xn2, double& beta, double2& tau, double2& scl) {
  const double n2 = alpha.x * alpha.x + alpha.y * alpha.y + xn2;
  const bool none = n2 <= kTiny * kTiny;   // (the norm of a smaller column has underflown, or lost bits)
  if (none || (xn2 == 0.0 && alpha.y == 0.0)) {
    beta = none ? 0.0 : alpha.x;
    tau = make_double2(0.0, 0.0);
    scl = make_double2(0.0, 0.0);
    return;
  }
  // on every step's critical path: refined reciprocal estimates (about an ulp)
  const double ri = rsqrt_nr(n2), nrm = n2 * ri;
  beta = alpha.x >= 0.0 ? -nrm : nrm;
  const double ib = alpha.x >= 0.0 ? -ri : ri;
  tau = make_double2((beta - alpha.x) * ib, -alpha.y * ib);
  const double ax = alpha.x - beta, ay = alpha.y, id = rcp_nr(ax * ax + ay * ay);
  scl = make_double2(ax * id, -ay * id);
}

// A diagonal entry as the divide and conquer takes it (the couplings are the reflector's).
__device__ __forceinline__ double in_range(double x) { return fabs(x) < kTiny ? 0.0 : x; }

// Sums over a wave's 64 lanes of 2 NR values (the real and imaginary parts of
// NR row sums): halved over the first lane bits, then over the rest of 16
// lanes by rotations, the four 16-lane rows through LDS (part, this wave's);
// lane t < NR returns sum t.  No barrier: all of it inside the wave.
template <int NR>
__device__ __forceinline__ double2 wave_rows(double* acc, double (*part)[2 * NR]) {
  constexpr int V = 2 * NR, H = V >= 8 ? 2 : V >= 4 ? 1 : 0, K = V >> H;
  const int lane = threadIdx.x & 63, l15 = lane & 15, l4 = lane >> 4;
#pragma unroll
  for (int q = 0; q < H; ++q) {
    const int h = V >> (q + 1);
    const bool up = (lane >> q) & 1;
#pragma unroll
    for (int u = 0; u < V / 2; ++u)
      if (u < h) {
        const double lo = acc[u], hi = acc[u + h], keep = up ? hi : lo, send = up ? lo : hi;
        acc[u] = keep + (q == 0 ? dpp_d<kXor1>(send) : dpp_d<kXor2>(send));
      }
  }
#pragma unroll
  for (int u = 0; u < K; ++u) {
    if (H < 1) acc[u] += dpp_d<kXor1>(acc[u]);
    if (H < 2) acc[u] += dpp_d<kXor2>(acc[u]);
    acc[u] += dpp_d<kRor4>(acc[u]);
    acc[u] += dpp_d<kRor8>(acc[u]);
  }
  if (l15 < (1 << H)) {
    const int idx = H == 2 ? (l15 & 1) * (V / 2) + (l15 >> 1) * (V / 4) : H == 1 ? l15 * (V / 2) : 0;
#pragma unroll
    for (int u = 0; u < K; ++u) part[l4][idx + u] = acc[u];
  }
  __builtin_amdgcn_wave_barrier();
  double2 y = make_double2(0.0, 0.0);
  if (lane < NR) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      y.x += part[r][2 * lane];
      y.y += part[r][2 * lane + 1];
    }
  }
  __builtin_amdgcn_wave_barrier();
  return y;
}

// Householder tridiagonalisation, one column a step, by stages: the stage of
// COLS takes the trailing COLS rows (or all m > COLS / 2 of them) down to
// COLS / 2, the last stage (tri_last_kernel) the last 128.  A stage holds its
// matrix in the registers of a team of workgroups, EL complex elements a
// thread; as the matrix shrinks the teams do, which leaves room for more
// matrices at once (32 matrices of m = 512: 7.5 ms as one launch per class of
// m, 4.0 by stages).  Blocks of 8 rows are dealt to the team in turn, a row to
// each wave of a workgroup, and columns to the lanes in turn: the work shrinks
// evenly with the step, a wave sums its rows by itself (wave_rows), and the 8
// sums of a block of rows leave as one line.
// A step applies the last step's rank-two update and the product with the new
// vector in one pass over the registers, so memory is not read at all.  Its
// bound is latency: the one exchange between the team's workgroups (the
// product's rows, and the next column, which its owner sends as it stood
// before the update: every workgroup updates it itself), three barriers and
// the reductions between them, and the pass itself (12 FP64 FMA an element,
// 0.8 us at 16 elements).  Words are sent with agent-scope stores into a place
// of their own per step, cleared to "empty" before the launch; what else is
// stored goes out after the poll, for a load waits for the stores before it.
// Time of a step at the full stage: 512: 3.5 us at EL = 8, 4.7 at 16 (two
// workgroups to a CU either way), 5.6 at 32; 256: 2.9 us at EL = 4, 3.2 at 8, 4.6
// at 16; 1024: 5.7 us at EL = 32, 6.1 at 16; 2048: 8.8 us at EL = 32.  (A dozen
// values do not find registers at EL = 16 and 32 and are reloaded once a step.)
// With a word's sum from one workgroup's threads in four barriers,
// lane permutes through LDS and a poll per word, a step took 6.6 us at m = 512;
// a launch per step would take two launches of 5 us.
template <int COLS, int EL>
__global__ __launch_bounds__(512, EL <= 16 ? 4 : 2) void tri_kernel(const EigSlot* __restrict__ slots, int limit) {
  constexpr int NC = COLS / 64, NR = EL / NC, R = 8 * NR, TMAX = COLS / R;
  constexpr int PT = COLS >= 512 ? COLS / 512 : 1;   // vector entries per thread
  __shared__ double2 cc[COLS], ww[COLS], vv[2][COLS];
  __shared__ double part[8][4][2 * NR];
  __shared__ double redn[8], redd[8];
  __shared__ double2 yl[8 * NR];
  __shared__ double2 s_al, s_yk;
  __shared__ int s_fail;
  const EigSlot& S = slots[blockIdx.x / TMAX];
  const int q = blockIdx.x % TMAX;
  const int m = S.m;
  if (!S.active || m <= COLS / 2 || *S.fail) return;
  const int off = max(0, m - COLS), r = m - off, T = (r + R - 1) / R;   // rows and columns are counted from off
  if (q >= T) return;
  const int steps = r - COLS / 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double2* const A0 = S.A + (size_t)off * m + off;
  const double sc = off == 0 ? S.scale : 1.0;   // (an earlier stage has scaled it)
  double2 a[NR][NC];
#pragma unroll
  for (int rs = 0; rs < NR; ++rs)
#pragma unroll
    for (int cs = 0; cs < NC; ++cs) {
      const int i = (rs * T + q) * 8 + wave, j = cs * 64 + lane;
      const double f = i < r && j < r ? sc : 0.0;
      const int hi = min(max(i, j), r - 1), lo = min(min(i, j), r - 1);
      double2 x = A0[(size_t)hi * m + lo];
      x.x *= f;
      x.y *= j == i ? 0.0 : j > i ? -f : f;
      a[rs][cs] = x;
      __builtin_amdgcn_sched_barrier(0);
    }
  double2 c[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int i = tid + t * 512;
    c[t] = make_double2(0.0, 0.0);
    if (i < r) {
      c[t] = A0[(size_t)i * m];
      c[t].x *= sc;
      c[t].y *= sc;
    }
    if (i < COLS) {
      vv[1][i] = make_double2(0.0, 0.0);
      ww[i] = make_double2(0.0, 0.0);
    }
  }
  bool mine[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) mine[t] = tid + t * 512 < r && (tid + t * 512) % T == q;
  if (tid == 0) s_fail = 0;
  int k = 0;
  do {   // (as a for loop, which may be skipped, the matrix was kept twice and spilled)
    const int pb = k & 1, k1 = k + 1, kg = off + k;
    // the reflector of the column below the diagonal
    double xn = 0.0;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      if (i > k1 && i < r) xn += c[t].x * c[t].x + c[t].y * c[t].y;
      if (i == k1) s_al = c[t];
      if (i < COLS) cc[i] = c[t];
      if (i == k && q == 0) S.d[kg] = c[t].x;
    }
    xn = wave_sum(xn);
    if (lane == 0) redn[wave] = xn;
    __syncthreads();
    double xn2 = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) xn2 += redn[u];
    double beta;
    double2 tau, scl;
    reflector(s_al, xn2, beta, tau, scl);
    double2 v[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      v[t] = make_double2(0.0, 0.0);
      if (i == k1) v[t] = make_double2(1.0, 0.0);
      else if (i > k1 && i < r) v[t] = cmul(c[t], scl);
      if (i < COLS) vv[pb][i] = v[t];   // for the next step's update
    }
    // A <- A - v w^dag - w v^dag (last step's) and y = A v (this step's), rows
    // and columns past k; this step's v is formed from the column as it is read
    double acc[2 * NR];
#pragma unroll
    for (int u = 0; u < 2 * NR; ++u) acc[u] = 0.0;
    {
      const double2* const vo = vv[pb ^ 1];
      // this wave's rows of the last step's vectors: read once, then broadcast
      const int il = min(((lane & (NR - 1)) * T + q) * 8 + wave, COLS - 1);
      const double2 lv = vo[il], lw = ww[il];
      double2 rv[NR], rw[NR];
#pragma unroll
      for (int rs = 0; rs < NR; ++rs) {
        rv[rs] = make_double2(lane_get(lv.x, rs), lane_get(lv.y, rs));
        rw[rs] = make_double2(lane_get(lw.x, rs), lane_get(lw.y, rs));
      }
#pragma unroll
      for (int cs = 0; cs < NC; ++cs) {
        if ((cs + 1) * 64 > k1) {   // some column of this slot is past k
          const int j = cs * 64 + lane;
          double2 nj = cmul(cc[j], scl);
          if (j <= k1) nj = make_double2(j == k1 ? 1.0 : 0.0, 0.0);
          const double2 oj = vo[j], wj = ww[j];
#pragma unroll
          for (int rs = 0; rs < NR; ++rs) {
            if ((rs + 1) * 8 * T > k) {
              double2 x = a[rs][cs];
              x.x = fma(-rv[rs].x, wj.x, x.x);
              x.x = fma(-rv[rs].y, wj.y, x.x);
              x.x = fma(-rw[rs].x, oj.x, x.x);
              x.x = fma(-rw[rs].y, oj.y, x.x);
              x.y = fma(-rv[rs].y, wj.x, x.y);
              x.y = fma(rv[rs].x, wj.y, x.y);
              x.y = fma(-rw[rs].y, oj.x, x.y);
              x.y = fma(rw[rs].x, oj.y, x.y);
              a[rs][cs] = x;
              acc[2 * rs] = fma(x.x, nj.x, acc[2 * rs]);
              acc[2 * rs] = fma(-x.y, nj.y, acc[2 * rs]);
              acc[2 * rs + 1] = fma(x.x, nj.y, acc[2 * rs + 1]);
              acc[2 * rs + 1] = fma(x.y, nj.x, acc[2 * rs + 1]);
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the next column as it stands, from the wave that owns its row
    double* const ey = (double*)(S.E + (size_t)kg * 2 * m);
    double* const er = ey + 2 * m;
    if (k1 % 8 == wave && (k1 / 8) % T == q) {
      const int ro = (k1 / 8) / T;
      int l = lane;
      asm volatile("" : "+v"(l));   // formed here, not kept over the step
      double* const el = er + 2 * l;
#pragma unroll
      for (int cs = 0; cs < NC; ++cs) {
        double2 x = a[0][cs];
#pragma unroll
        for (int rs = 1; rs < NR; ++rs)
          if (rs == ro) x = a[rs][cs];
        const int j = cs * 64 + l;
        if (j >= k1 && j < r) {
          xch_put(el + cs * 128, x.x);
          xch_put(el + cs * 128 + 1, x.y);
        }
      }
    }
    const double2 ys = wave_rows<NR>(acc, part[wave]);
    if (lane < NR) yl[lane * 8 + wave] = ys;
    __syncthreads();
    if (tid < 16 * NR) {   // whole lines, and no load of the other waves waits behind them
      const int l = tid >> 1, i = ((l >> 3) * T + q) * 8 + (l & 7);
      if (i > k && i < r) xch_put(ey + 2 * i + (tid & 1), (tid & 1) ? yl[l].y : yl[l].x);
    }
    double2 y[PT], row[PT];
    double dot = 0.0;
    bool ok = true;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      const bool want = i > k && i < r;
      const int ii = want ? i : k1;
      const double* const at[4] = {ey + 2 * ii, ey + 2 * ii + 1, er + 2 * ii, er + 2 * ii + 1};
      double got[4] = {0.0, 0.0, 0.0, 0.0};
      ok = xch_get<4>(at, got, want, limit) && ok;
      y[t] = want ? make_double2(got[0], got[1]) : make_double2(0.0, 0.0);
      row[t] = want ? make_double2(got[2], got[3]) : make_double2(0.0, 0.0);
      dot += v[t].x * y[t].x + v[t].y * y[t].y;   // Re v^dag y (v^dag A v is real)
      if (i == k1) s_yk = y[t];
    }
    if (!ok) s_fail = 1;
    dot = wave_sum(dot);
    if (lane == 0) redd[wave] = dot;
    __syncthreads();
    if (s_fail) {   // uniform: written before the barrier only
      if (tid == 0) *S.fail = 1;
      return;
    }
    double vav = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) vav += redd[u];
    const double hv = 0.5 * (tau.x * tau.x + tau.y * tau.y) * vav;
    double2 wk = cmul(tau, s_yk);
    wk.x -= hv;   // v_{k+1} = 1
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      double2 w = cmul(tau, y[t]);
      w.x -= hv * v[t].x;
      w.y -= hv * v[t].y;
      if (i <= k || i >= r) w = make_double2(0.0, 0.0);
      if (i < COLS) ww[i] = w;
      // A_{i,k+1} = conj(row) - v_i conj(w_{k+1}) - w_i
      double2 x = make_double2(row[t].x, -row[t].y);
      x.x -= v[t].x * wk.x + v[t].y * wk.y + w.x;
      x.y -= v[t].y * wk.x - v[t].x * wk.y + w.y;
      c[t] = x;
    }
    // the vector for the later kernels, each workgroup its share of the rows
    // (here, where no load waits behind the stores)
    double2* const vg = S.V + (size_t)(kg / kWy) * m * kWy + (kg % kWy);
#pragma unroll
    for (int t = 0; t < PT; ++t)
      if (mine[t]) vg[(size_t)(off + tid + t * 512) * kWy] = v[t];
    if (q == 0) {
      if (tid < kWy && (kg / kWy) * kWy + tid < off) vg[(size_t)((kg / kWy) * kWy + tid) * kWy] = make_double2(0.0, 0.0);
      if (tid == 0) {
        S.e[kg] = beta;
        S.tau[kg] = tau;
      }
    }
  } while (++k < steps);
  // the last update, and what is left to the next stage (its lower triangle)
  __syncthreads();
  const double2* const vo = vv[(steps - 1) & 1];
  double2* const A1 = S.A + (size_t)off * m + off;
  int lane1 = lane;
  asm volatile("" : "+v"(lane1));   // so that no index is kept from the load to here
#pragma unroll
  for (int rs = 0; rs < NR; ++rs) {
    const int i = (rs * T + q) * 8 + wave;
    if (i >= steps && i < r) {
      const double2 rv = vo[i], rw = ww[i];
#pragma unroll
      for (int cs = 0; cs < NC; ++cs) {
        const int j = cs * 64 + lane1;
        if (j >= steps && j <= i) {
          const double2 wj = ww[j], oj = vo[j];
          double2 x = a[rs][cs];
          x.x -= rv.x * wj.x + rv.y * wj.y + rw.x * oj.x + rw.y * oj.y;
          x.y -= rv.y * wj.x - rv.x * wj.y + rw.y * oj.x - rw.x * oj.y;
          A1[(size_t)i * m + j] = x;
        }
      }
    }
  }
}

// The steps of a matrix of at most N rows held in the registers of one
// workgroup of NT threads (rows dealt out in turn to groups of 16 lanes, columns
// in turn to the lanes of a group).  A step is a chain, so it is kept short: a row's sums take DPP
// moves alone, and what follows the one barrier of a step (the vector
// arithmetic of the reflector and of the update, N / 64 entries a lane) every
// wave does for itself, into its own copies in LDS.
// load(i, j): the scaled matrix; out(k, i, v): entry i of the reflector of step
// k, from wave 0; out.step(k, d, e, tau) and out.last(d) from one thread.
template <int N, int NT, bool VL>   // VL: the vectors are read from where out() puts them
struct TriLds {
  double2 v[VL ? 1 : NT / 64][2][VL ? 1 : N], w[NT / 64][N], y[2][N], row[2][N];
};

template <int N, int NT, class Load, class Out>
__device__ __forceinline__ void tri_block(TriLds<N, NT, Out::kLds>& S, int m, const Load& load, const Out& out) {
  constexpr int RG = NT / 16, LRG = NT == 512 ? 5 : 4, TR = N / RG, TN = N / 16, EN = N > 64 ? N / 64 : 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rg = tid >> 4, cg = tid & 15;
  double2 a[TR][TN];
#pragma unroll
  for (int rs = 0; rs < TR; ++rs)
#pragma unroll
    for (int cs = 0; cs < TN; ++cs) a[rs][cs] = load(rs * RG + rg, cs * 16 + cg);
  double2 c[EN];
#pragma unroll
  for (int t = 0; t < EN; ++t) {
    const int i = t * 64 + lane;
    c[t] = make_double2(0.0, 0.0);
    if (i < N) {
      c[t] = load(i, 0);
      S.w[wave][i] = make_double2(0.0, 0.0);
      if constexpr (!Out::kLds) S.v[wave][1][i] = make_double2(0.0, 0.0);
    }
  }
  if constexpr (Out::kLds) {
    __syncthreads();   // the vectors take the matrix's place
#pragma unroll
    for (int t = 0; t < EN; ++t)
      if (t * 64 + lane < N) out(N, t * 64 + lane, make_double2(0.0, 0.0));   // stands before the first
  }
  auto entry = [&](const double2 (&x)[EN], int i) {   // entry i of a vector dealt to the lanes (i uniform)
    double2 z = make_double2(lane_get(x[0].x, i & 63), lane_get(x[0].y, i & 63));
#pragma unroll
    for (int t = 1; t < EN; ++t)
      if (i >> 6 == t) z = make_double2(lane_get(x[t].x, i & 63), lane_get(x[t].y, i & 63));
    return z;
  };
  for (int k = 0; k < m - 1; ++k) {
    const int b = k & 1, k1 = k + 1;
    const double2 al = entry(c, k1), dk = entry(c, k);
    double xs = 0.0;
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int i = t * 64 + lane;
      if (i > k1 && i < m) xs += c[t].x * c[t].x + c[t].y * c[t].y;
    }
    const double xn = wave_sum(xs);
    double beta;
    double2 tau, scl;
    reflector(al, xn, beta, tau, scl);
    double2 v[EN];
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int i = t * 64 + lane;
      v[t] = make_double2(0.0, 0.0);
      if (i == k1) v[t] = make_double2(1.0, 0.0);
      else if (i > k1 && i < m) v[t] = cmul(c[t], scl);
      if (i < N) {
        if constexpr (!Out::kLds) S.v[wave][b][i] = v[t];
        if (Out::kLds || wave == 0) out(k, i, v[t]);   // (in LDS: every wave the same)
      }
    }
    if (tid == 0) out.step(k, dk.x, beta, tau);
    __builtin_amdgcn_wave_barrier();
    double acc[2 * TR];
    {
      constexpr int VS = Out::kLds ? N + 1 : 1;
      const double2 *vn, *vo, *const ww = S.w[wave];
      if constexpr (Out::kLds) {
        vn = out.col(k);
        vo = out.col(k > 0 ? k - 1 : N);
      } else {
        vn = S.v[wave][b];
        vo = S.v[wave][b ^ 1];
      }
      // (what is held of the vectors over the pass: the shorter side)
      double2 rv[TR], rw[TR], cn[TN], co[TN], cw[TN];
      if constexpr (TN > 4) {
#pragma unroll
        for (int rs = 0; rs < TR; ++rs) {
          rv[rs] = vo[(rs * RG + rg) * VS];
          rw[rs] = ww[rs * RG + rg];
          acc[2 * rs] = acc[2 * rs + 1] = 0.0;
        }
#pragma unroll
        for (int cs = 0; cs < TN; ++cs)
          if (cs * 16 + 15 > k) {   // some column of this slot is past k
            const double2 nj = vn[(cs * 16 + cg) * VS], oj = vo[(cs * 16 + cg) * VS], wj = ww[cs * 16 + cg];
#pragma unroll
            for (int rs = 0; rs < TR; ++rs)
              if (rs * RG + RG - 1 > k) {
                double2 x = a[rs][cs];
                x.x -= rv[rs].x * wj.x + rv[rs].y * wj.y + rw[rs].x * oj.x + rw[rs].y * oj.y;
                x.y -= rv[rs].y * wj.x - rv[rs].x * wj.y + rw[rs].y * oj.x - rw[rs].x * oj.y;
                a[rs][cs] = x;
                acc[2 * rs] += x.x * nj.x - x.y * nj.y;
                acc[2 * rs + 1] += x.x * nj.y + x.y * nj.x;
              }
          }
      } else {
#pragma unroll
        for (int cs = 0; cs < TN; ++cs) {
          cn[cs] = vn[(cs * 16 + cg) * VS];
          co[cs] = vo[(cs * 16 + cg) * VS];
          cw[cs] = ww[cs * 16 + cg];
        }
#pragma unroll
        for (int rs = 0; rs < TR; ++rs) {
          double ax = 0.0, ay = 0.0;
          if (rs * RG + RG - 1 > k) {
            const double2 ri = vo[(rs * RG + rg) * VS], rj = ww[rs * RG + rg];
#pragma unroll
            for (int cs = 0; cs < TN; ++cs)
              if (cs * 16 + 15 > k) {
                double2 x = a[rs][cs];
                x.x -= ri.x * cw[cs].x + ri.y * cw[cs].y + rj.x * co[cs].x + rj.y * co[cs].y;
                x.y -= ri.y * cw[cs].x - ri.x * cw[cs].y + rj.y * co[cs].x - rj.x * co[cs].y;
                a[rs][cs] = x;
                ax += x.x * cn[cs].x - x.y * cn[cs].y;
                ay += x.x * cn[cs].y + x.y * cn[cs].x;
              }
          }
          acc[2 * rs] = ax;
          acc[2 * rs + 1] = ay;
        }
      }
    }
    if (rg == (k1 & (RG - 1))) {
#pragma unroll
      for (int rs = 0; rs < TR; ++rs)
        if (rs == k1 >> LRG)
#pragma unroll
          for (int cs = 0; cs < TN; ++cs) S.row[b][cs * 16 + cg] = a[rs][cs];
    }
    // row sums over 16 lanes: halved over the first lane bits (rows), then
    // summed over the rest by rotations that keep the place among four lanes
    constexpr int HB = TR >= 4 ? 2 : 1, KV = 2 * TR >> HB;
#pragma unroll
    for (int q = 0; q < HB; ++q) {
      const int h = TR >> q;
      const bool up = (lane >> q) & 1;
#pragma unroll
      for (int u = 0; u < TR; ++u)
        if (u < h) {
          const double lo = acc[u], hi = acc[u + h], keep = up ? hi : lo, send = up ? lo : hi;
          acc[u] = keep + (q == 0 ? dpp_d<kXor1>(send) : dpp_d<kXor2>(send));
        }
    }
#pragma unroll
    for (int u = 0; u < KV; ++u) {
      if (HB == 1) acc[u] += dpp_d<kXor2>(acc[u]);
      acc[u] += dpp_d<kRor4>(acc[u]);
      acc[u] += dpp_d<kRor8>(acc[u]);
    }
    if (cg < (1 << HB)) {
      const int r0 = HB == 2 ? (cg & 1) * (TR / 2) + (cg >> 1) * (TR / 4) : cg * (TR / 2);
#pragma unroll
      for (int u = 0; u < KV / 2; ++u) S.y[b][(r0 + u) * RG + rg] = make_double2(acc[2 * u], acc[2 * u + 1]);
    }
    __syncthreads();
    double2 y[EN], row[EN];
    double ds = 0.0;
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int i = t * 64 + lane;
      y[t] = row[t] = make_double2(0.0, 0.0);
      if (i < N) {
        y[t] = S.y[b][i];
        row[t] = S.row[b][i];
      }
      ds += v[t].x * y[t].x + v[t].y * y[t].y;   // v is zero up to k and past m
    }
    const double hv = 0.5 * (tau.x * tau.x + tau.y * tau.y) * wave_sum(ds);
    double2 wk = cmul(tau, entry(y, k1));
    wk.x -= hv;
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int i = t * 64 + lane;
      double2 w = cmul(tau, y[t]);
      w.x -= hv * v[t].x;
      w.y -= hv * v[t].y;
      if (i <= k || i >= m) w = make_double2(0.0, 0.0);
      if (i < N) S.w[wave][i] = w;
      c[t].x = row[t].x - (v[t].x * wk.x + v[t].y * wk.y + w.x);
      c[t].y = -row[t].y - (v[t].y * wk.x - v[t].x * wk.y + w.y);
    }
  }
  const double2 dl = entry(c, m - 1);
  if (tid == 0) out.last(dl.x);
}

// The last stage: the trailing 128 rows (or all m <= 128), one workgroup of
// 512 threads: 2.6 us a step (256 threads of twice the elements, half of them in
// AGPRs: 5.5).
__global__ __launch_bounds__(512) void tri_last_kernel(const EigSlot* __restrict__ slots) {
  constexpr int N = 128, NT = 512;
  __shared__ TriLds<N, NT, false> L;
  const EigSlot& S = slots[blockIdx.x];
  const int m = S.m;
  if (!S.active || *S.fail) return;
  const int off = max(0, m - N), r = m - off;
  const double2* const A0 = S.A + (size_t)off * m + off;
  const double sc = off == 0 ? S.scale : 1.0;
  auto load = [&](int i, int j) {
    double2 x = make_double2(0.0, 0.0);
    if (i < r && j < r) {
      x = j <= i ? A0[(size_t)i * m + j] : A0[(size_t)j * m + i];
      if (j > i) x.y = -x.y;
      if (j == i) x.y = 0.0;
      x.x *= sc;
      x.y *= sc;
    }
    return x;
  };
  struct Out {
    enum : bool { kLds = false };
    const EigSlot& S;
    int m, off, r;
    __device__ __forceinline__ void operator()(int k, int i, double2 v) const {
      const int kg = off + k;
      double2* const vg = S.V + (size_t)(kg / kWy) * m * kWy + (kg % kWy);
      if (i < r) vg[(size_t)(off + i) * kWy] = v;
      // rows of the block's first tile that lie before this stage
      if (i < kWy && (kg / kWy) * kWy + i < off) vg[(size_t)((kg / kWy) * kWy + i) * kWy] = make_double2(0.0, 0.0);
    }
    __device__ __forceinline__ void step(int k, double d, double e, double2 t) const {
      S.d[off + k] = d;
      S.e[off + k] = e;
      S.tau[off + k] = t;
    }
    __device__ __forceinline__ void last(double d) const { S.d[m - 1] = d; }
  };
  tri_block<N, NT>(L, r, load, Out{S, m, off, r});
  // the last block's unused columns
  for (int i = threadIdx.x; i < m; i += NT)
    for (int k = m - 1; k % kWy != 0; ++k) S.V[((size_t)(k / kWy) * m + i) * kWy + (k % kWy)] = make_double2(0.0, 0.0);
}

// The steps of a matrix of m > 2048 rows down to 2048, which the chip's
// registers hold: each of 256 workgroups keeps its rows (in turn) in memory,
// rewritten once per step (bound by that traffic, mostly from the last-level
// cache).
constexpr int kTriBigT = 256;
__global__ __launch_bounds__(512) void tri_sym_kernel(const EigSlot* __restrict__ slots) {
  // the upper triangle from the lower, scaled, 32 x 32 tiles through LDS
  __shared__ double2 tl[32][33];
  const EigSlot& S = slots[blockIdx.y];
  const int m = S.m;
  if (!S.active || m <= 2048) return;
  const int nt = (m + 31) / 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int t = blockIdx.x; t < nt * nt; t += gridDim.x) {
    const int bi = t / nt, bj = t % nt;
    if (bi < bj) continue;
    __syncthreads();
    for (int r = ty; r < 32; r += 16) {
      const int i = bi * 32 + r, j = bj * 32 + tx;
      double2 x = make_double2(0.0, 0.0);
      if (i < m && j < m && j <= i) {
        x = S.A[(size_t)i * m + j];
        x.x *= S.scale;
        x.y = i == j ? 0.0 : x.y * S.scale;
      }
      tl[r][tx] = x;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 16) {
      const int i = bi * 32 + r, j = bj * 32 + tx;
      if (i < m && j < m && j <= i) S.A[(size_t)i * m + j] = tl[r][tx];
      const int i2 = bj * 32 + r, j2 = bi * 32 + tx;   // transposed place
      if (i2 < m && j2 < m && i2 < j2) {
        const double2 x = tl[tx][r];
        S.A[(size_t)i2 * m + j2] = make_double2(x.x, -x.y);
      }
    }
  }
}

__global__ __launch_bounds__(512) void tri_big_kernel(const EigSlot* __restrict__ slots, int limit) {
  constexpr int MC = 4096, PT = MC / 512, RC = MC / kTriBigT;
  __shared__ double2 vo[MC];            // the last step's vector (this step's replaces it after the pass)
  __shared__ double ysum[8][RC][2];
  __shared__ double redn[2][8], redd[2][8];
  __shared__ double2 s_al, s_yk;
  __shared__ int s_fail;
  const EigSlot& S = slots[blockIdx.x / kTriBigT];
  const int q = blockIdx.x % kTriBigT, T = kTriBigT;
  const int m = S.m;
  if (!S.active || m <= 2048 || m > MC) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ double2 wrow[RC], vrow[RC];
  const int R = (m - q + T - 1) / T;    // rows i = l T + q of this workgroup
  double2 c[PT], v[PT], w[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int i = tid + t * 512;
    c[t] = i < m ? S.A[(size_t)i * m] : make_double2(0.0, 0.0);
    v[t] = w[t] = make_double2(0.0, 0.0);
  }
  if (tid < RC) wrow[tid] = vrow[tid] = make_double2(0.0, 0.0);
  if (tid == 0) s_fail = 0;
  // column 0 is read by every workgroup before any of them rewrites its rows:
  // the first pass (k = 0) has zero v and w and leaves the rows as they are
  const int steps = m - 2048;
  for (int k = 0; k < steps; ++k) {
    const int pb = k & 1;
    double xn = 0.0;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      if (i > k + 1 && i < m) xn += c[t].x * c[t].x + c[t].y * c[t].y;
      if (i == k + 1) s_al = c[t];
      if (i == k && q == 0) S.d[k] = c[t].x;
    }
    xn = wave_sum(xn);
    if (lane == 0) redn[pb][wave] = xn;
    __syncthreads();
    double xn2 = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) xn2 += redn[pb][u];
    double beta;
    double2 tau, scl;
    reflector(s_al, xn2, beta, tau, scl);
    double2 vn[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      vn[t] = make_double2(0.0, 0.0);
      if (i == k + 1) vn[t] = make_double2(1.0, 0.0);
      else if (i > k + 1 && i < m) vn[t] = cmul(c[t], scl);
      if (q == 0 && i < m) S.V[((size_t)(k / kWy) * m + i) * kWy + (k % kWy)] = vn[t];
    }
    if (q == 0 && tid == 0) {
      S.e[k] = beta;
      S.tau[k] = tau;
    }
    const int k1 = k + 1;
    double* const ey = (double*)(S.E + (size_t)k * 2 * m);
    double* const er = ey + 2 * m;
    const int l0 = k1 > q ? (k1 - q + T - 1) / T : 0;   // first row past k
    for (int l = l0; l < R; ++l) {
      const int i = l * T + q;
      double2* const ar = S.A + (size_t)i * m;
      const double2 rv = vrow[l], rw = wrow[l];
      double ax = 0.0, ay = 0.0;
      double2 x[PT];
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        const int j = tid + t * 512;
        x[t] = j > k && j < m ? ar[j] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        const int j = tid + t * 512;
        if (j > k && j < m) {
          double2 z = x[t];
          z.x -= rv.x * w[t].x + rv.y * w[t].y + rw.x * v[t].x + rw.y * v[t].y;
          z.y -= rv.y * w[t].x - rv.x * w[t].y + rw.y * v[t].x - rw.x * v[t].y;
          ar[j] = z;
          ax += z.x * vn[t].x - z.y * vn[t].y;
          ay += z.x * vn[t].y + z.y * vn[t].x;
          if (i == k1) {
            xch_put(er + 2 * j, z.x);
            xch_put(er + 2 * j + 1, z.y);
          }
        }
      }
      ax = wave_sum(ax);
      ay = wave_sum(ay);
      if (lane == 0) {
        ysum[wave][l][0] = ax;
        ysum[wave][l][1] = ay;
      }
    }
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      v[t] = vn[t];
      const int i = tid + t * 512;
      if (i < m) vo[i] = vn[t];
    }
    __syncthreads();
    if (tid < R && tid >= l0) {
      double yx = 0.0, yy = 0.0;
      for (int u = 0; u < 8; ++u) {
        yx += ysum[u][tid][0];
        yy += ysum[u][tid][1];
      }
      const int i = tid * T + q;
      xch_put(ey + 2 * i, yx);
      xch_put(ey + 2 * i + 1, yy);
    }
    if (tid < R) vrow[tid] = vo[tid * T + q];
    double2 y[PT], row[PT];
    double dot = 0.0;
    bool ok = true;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      y[t] = row[t] = make_double2(0.0, 0.0);
      if (i > k && i < m) {
        const double* const at[4] = {ey + 2 * i, ey + 2 * i + 1, er + 2 * i, er + 2 * i + 1};
        double got[4] = {0.0, 0.0, 0.0, 0.0};
        ok = xch_get<4>(at, got, true, limit) && ok;
        y[t] = make_double2(got[0], got[1]);
        row[t] = make_double2(got[2], got[3]);
        dot += v[t].x * y[t].x + v[t].y * y[t].y;
        if (i == k1) s_yk = y[t];
      }
    }
    if (!ok) s_fail = 1;
    dot = wave_sum(dot);
    if (lane == 0) redd[pb][wave] = dot;
    __syncthreads();
    if (s_fail) {
      if (tid == 0) *S.fail = 1;
      return;
    }
    double vav = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) vav += redd[pb][u];
    const double hv = 0.5 * (tau.x * tau.x + tau.y * tau.y) * vav;
    double2 wk = cmul(tau, s_yk);
    wk.x -= hv;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int i = tid + t * 512;
      double2 z = cmul(tau, y[t]);
      z.x -= hv * v[t].x;
      z.y -= hv * v[t].y;
      if (i <= k || i >= m) z = make_double2(0.0, 0.0);
      w[t] = z;
      if (i < m && i % T == q) wrow[i / T] = z;
      double2 x = make_double2(row[t].x, -row[t].y);
      x.x -= v[t].x * wk.x + v[t].y * wk.y + z.x;
      x.y -= v[t].y * wk.x - v[t].x * wk.y + z.y;
      c[t] = x;
    }
  }
  // the last update of the rows that are left
  __syncthreads();
  for (int l = 0; l < R; ++l) {
    const int i = l * T + q;
    if (i < steps) continue;
    const double2 rv = vrow[l], rw = wrow[l];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int j = tid + t * 512;
      if (j >= steps && j <= i) {
        double2 z = S.A[(size_t)i * m + j];
        z.x -= rv.x * w[t].x + rv.y * w[t].y + rw.x * v[t].x + rw.y * v[t].y;
        z.y -= rv.y * w[t].x - rv.x * w[t].y + rw.y * v[t].x - rw.x * v[t].y;
        S.A[(size_t)i * m + j] = z;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Divide and conquer on the tridiagonal matrix
// ---------------------------------------------------------------------------
// T is torn at every index: the diagonal loses |e| on both sides of a tear,
// and merging two solved blocks adds back rho u u^T with rho = |e| and
// u = (last row of one, +-first row of the other).  In the blocks'
// eigenbasis that is D + rho z z^T, whose eigenvalues are the roots of
//   1 + rho sum_j z_j^2 / (d_j - lambda) = 0,
// one between each d_j and the next (the last within rho |z|^2 of d_last).
// Entries with negligible rho |z_j|, and all but one of a group of equal d_j
// (after a rotation that zeroes z_j), are eigenvalues already (deflation).
// The tearing is Cuppen's (1981); a root's step is that of the two-pole rational
// function through value and slope of the sum's two halves (Bunch, Nielsen and
// Sorensen 1978, the "middle way" of Li, LAPACK working note 89); the vectors'
// weights are Gu's and Eisenstat's (1994).

// One thread: the sorted (ds, zs) of a merge of s entries deflated in place.
// kept rank list kr[0..K), deflated dr[0..s-K) with values dv, rotations
// (ra, rb, c, sn) in order; returns K.  The kept values ascend, by more than
// 2 tol from one to the next.
__device__ int dc_deflate(double* ds, double* zs, int s, double rho, double tol, int32_t* kr, int32_t* dr, double* dv,
                          int32_t* ra, int32_t* rb, double* rc, double* rs, int& nrot) {
  int K = 0, nd = 0, pj = -1, nr = 0;
  for (int r = 0; r < s; ++r) {
    const double z = zs[r];
    if (rho * fabs(z) <= tol) {
      dr[nd] = r;
      dv[nd++] = ds[r];
      continue;
    }
    if (pj >= 0) {
      const double zp = zs[pj], t = ds[r] - ds[pj];
      const double h2 = z * z + zp * zp;
      // |t c s| <= tol with c = z / h, s = -zp / h
      if (fabs(t * z * zp) <= tol * h2) {
        const double ih = 1.0 / sqrt(h2);
        const double c = z * ih, sn = -zp * ih;
        zs[r] = sqrt(h2);
        zs[pj] = 0.0;
        // both of the pair's values between the old ones to the last bit: as sums of
        // rounded products the kept one could fall on the value kept before it
        const double dp = ds[pj], tw = t * fmin(sn * sn, 1.0);
        ds[r] -= tw;
        ra[nr] = pj;
        rb[nr] = r;
        rc[nr] = c;
        rs[nr++] = sn;
        dr[nd] = pj;
        dv[nd++] = dp + tw;
      } else {
        kr[K++] = pj;
      }
    }
    pj = r;
  }
  if (pj >= 0) kr[K++] = pj;
  nrot = nr;
  return K;
}

// Root i (0 <= i < K) of the secular equation on kept dk (ascending), zk:
// returned as dk[org] + eta.  NL adjacent lanes (a power of two, sub = lane
// index among them) share the sums; all of them return the same values.
template <int NL, int NJ>
__device__ __forceinline__ void dc_secular(const double* dk, const double* zk, int K, int i, double rho, int sub, int& org,
                           double& eta) {
  if (K == 1) {
    org = 0;
    eta = rho * zk[0] * zk[0];
    return;
  }
  const bool last = i == K - 1;
  const double dl = dk[i], gap = last ? rho * (1.0 + 1e-10) : dk[i + 1] - dl;   // sum z_j^2 = 1 to rounding
  // this lane's poles and weights stay in registers (past K: no weight, far off)
  double dj[NJ > 0 ? NJ : 1], zj[NJ > 0 ? NJ : 1];
#pragma unroll
  for (int u = 0; u < NJ; ++u) {
    const int j = sub + u * NL;
    const bool on = j < K;
    dj[u] = on ? dk[j] : dl + 4.0 * gap;
    zj[u] = on ? zk[j] : 0.0;
  }
  // the sign at the middle of the interval says which end is nearer
  double f = 0.0;
  {
    const double mid = 0.5 * gap;
    if constexpr (NJ > 0) {
#pragma unroll
      for (int u = 0; u < NJ; ++u) f += zj[u] * zj[u] * rcp_nr((dj[u] - dl) - mid);
    } else {
#pragma unroll 4
      for (int j = sub; j < K; j += NL) {
        const double z = zk[j];
        f += z * z * rcp_nr((dk[j] - dl) - mid);
      }
    }
    f = 1.0 + rho * lanes_sum<NL>(f);
  }
  double lo, hi;   // bracket of eta, measured from dk[org]
  if (last) {
    org = i;
    lo = f <= 0.0 ? 0.5 * gap : 0.0;
    hi = f <= 0.0 ? gap : 0.5 * gap;
  } else if (f >= 0.0) {
    org = i;
    lo = 0.0;
    hi = 0.5 * gap;
  } else {
    org = i + 1;
    lo = -0.5 * gap;
    hi = 0.0;
  }
  const double d0 = dk[org];
  // poles that bound the root (the last root: the last two poles)
  const int p1 = last ? i - 1 : i, p2 = p1 + 1;
  const double e1 = dk[p1] - d0, e2 = dk[p2] - d0;
  eta = 0.5 * (lo + hi);
#pragma unroll
  for (int u = 0; u < NJ; ++u) dj[u] -= d0;
  for (int it = 0; it < 64; ++it) {
    double ps = 0.0, dps = 0.0, ph = 0.0, dph = 0.0;
    auto term = [&](double z, double d, bool left) {
      const double r = z * rcp_nr(d - eta);
      const double t = z * r, t2 = r * r;
      ps += left ? t : 0.0;
      dps += left ? t2 : 0.0;
      ph += left ? 0.0 : t;
      dph += left ? 0.0 : t2;
    };
    if constexpr (NJ > 0) {
#pragma unroll
      for (int u = 0; u < NJ; ++u) term(zj[u], dj[u], sub + u * NL <= p1);
    } else {
#pragma unroll 4
      for (int j = sub; j < K; j += NL) term(zk[j], dk[j] - d0, j <= p1);
    }
    ps = rho * lanes_sum<NL>(ps);
    dps = rho * lanes_sum<NL>(dps);
    ph = rho * lanes_sum<NL>(ph);
    dph = rho * lanes_sum<NL>(dph);
    const double fv = 1.0 + ps + ph;
    if (fv > 0.0) hi = eta;   // f increases between the poles
    else lo = eta;
    // rounding level of the sum, and of eta in it
    if (fabs(fv) <= kEps * (4.0 * (1.0 + fabs(ps) + fabs(ph)) + fabs(eta) * (dps + dph))) break;
    if (hi - lo <= 2.0 * kEps * fabs(eta)) break;
    // f ~ c + s1 / (e1 - x) + s2 / (e2 - x), matching value and slope of the two halves at eta
    const double a1 = e1 - eta, a2 = e2 - eta;
    const double c = fv - dps * a1 - dph * a2;
    // c x^2 - a x + b = 0 for the step x, with
    const double a = c * (a1 + a2) + dps * a1 * a1 + dph * a2 * a2;
    const double b = a1 * a2 * fv;
    double step;
    const double disc = a * a - 4.0 * b * c;
    if (disc >= 0.0) {
      const double rt = disc > 1e-280 ? disc * rsqrt_nr(disc) : __builtin_amdgcn_sqrt(disc);
      // the root between the poles; for the last one, the root right of both
      const bool plus = (a >= 0.0) != last;
      const double num = plus ? 2.0 * b : (last ? a + rt : a - rt), den = plus ? (last ? a - rt : a + rt) : 2.0 * c;
      step = num * rcp_nr(den);
    } else {
      step = 0.0;
    }
    double nx = eta + step;
    // a step that leaves the bracket or does not move halves it (between a
    // pole at zero and a tiny root, by the geometric mean)
    if (!(nx > lo && nx < hi) || step == 0.0) {
      // (estimates of the square roots do: some root of a wave comes here in most passes)
      if (lo > 0.0 || hi < 0.0)
        nx = copysign(__builtin_amdgcn_sqrt(fabs(lo)) * __builtin_amdgcn_sqrt(fabs(hi)), lo + hi);
      else if (lo == 0.0) nx = hi * 0.0009765625;
      else if (hi == 0.0) nx = lo * 0.0009765625;
      else nx = 0.5 * (lo + hi);
      if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
    }
    if (nx == eta || !(nx > lo && nx < hi)) break;
    eta = nx;
  }
}

// Work of the solver of a block of at most N rows in LDS.
template <int N>
struct DcLds {
  double D[N], E[N];   // diagonal (torn at every index) and the couplings of i and i + 1
  double ds[N], zs[N], dk[N], zk[N], et[N], rc[N], rs[N], dv[N], zh[N], lam[N];
  int32_t pm[N], kr[N], dr[N], ra[N], rb[N], og[N], cnt[N], nro[N], rk[N], fl[N], cl[N];
};

// The block of nn <= N rows whose torn diagonal and couplings are in L, by
// merges of 1 + 1, 2 + 2, ... rows: Q [N][N + 1] = its eigenvectors (columns,
// as L.D ascending).  256 threads, 256 / N lanes an index.  Small merges are
// chains of short dependent steps (secular iterations, barriers), so lanes of
// an index exchange by DPP, divisions are refined reciprocal estimates, and
// the serial deflation scan runs only where two kept values are close.
template <int N>
__device__ __forceinline__ void dc_solve(DcLds<N>& L, double* Q, double* U, int nn) {
  constexpr int LD = N + 1, LP = 256 / N;
  const int tid = threadIdx.x, j = tid / LP, sub = tid % LP;
  for (int t = tid; t < N * N; t += 256) Q[(t / N) * LD + t % N] = t / N == t % N ? 1.0 : 0.0;
  __syncthreads();
  // pairs in closed form: (c, -s) and (s, c) with t = tan of the rotation
  if (sub == 0 && (j & 1) == 0 && j + 1 < nn && L.E[j] != 0.0) {
    const double e = L.E[j], x = L.D[j] + fabs(e), y = L.D[j + 1] + fabs(e), ta = 0.5 * (y - x) / e;
    const double t = (ta >= 0.0 ? 1.0 : -1.0) / (fabs(ta) + sqrt(1.0 + ta * ta));
    const double c = 1.0 / sqrt(1.0 + t * t), sn = t * c, l0 = x - t * e, l1 = y + t * e;
    const int i0 = l0 <= l1 ? j : j + 1, i1 = l0 <= l1 ? j + 1 : j;
    L.D[i0] = l0;
    L.D[i1] = l1;
    Q[j * LD + i0] = c;
    Q[(j + 1) * LD + i0] = -sn;
    Q[j * LD + i1] = sn;
    Q[(j + 1) * LD + i1] = c;
  } else if (sub == 0 && (j & 1) == 0 && j + 1 < nn && L.D[j] > L.D[j + 1]) {
    const double x = L.D[j];
    L.D[j] = L.D[j + 1];
    L.D[j + 1] = x;
    Q[j * LD + j] = Q[(j + 1) * LD + j + 1] = 0.0;
    Q[(j + 1) * LD + j] = Q[j * LD + j + 1] = 1.0;
  }
  __syncthreads();
  for (int s = 4; s <= N; s <<= 1) {
    const int h = s >> 1;
    if (h >= nn) break;
    const int base = j / s * s, mid = base + h, end = min(base + s, nn), sz = end - base;
    const bool live = j < nn;              // an index of the matrix
    const bool two = mid < end;            // its block has a second half
    double rho = 0.0, sg = 1.0;
    if (two) {
      rho = 2.0 * fabs(L.E[mid - 1]);
      sg = L.E[mid - 1] < 0.0 ? -1.0 : 1.0;
    }
    if (live) {
      double zj = 0.0;
      if (two) zj = (j < mid ? Q[(mid - 1) * LD + j] : sg * Q[mid * LD + j]) * 0.70710678118654752440;
      const double dj = L.D[j];
      const int o0 = j < mid ? mid : base, o1 = j < mid ? end : mid;
      int c = 0;
      for (int o = o0 + sub; o < o1; o += LP) c += j < mid ? L.D[o] < dj : L.D[o] <= dj;
      c = lanes_sum<LP>(c);
      const int rank = base + (j < mid ? j - base : j - mid) + c;
      if (sub == 0) {
        L.ds[rank] = dj;
        L.zs[rank] = zj;
        L.pm[rank] = j;
      }
    }
    if (sub == 0) L.cl[j] = 0;
    for (int t = tid; t < N * N; t += 256) U[(t / N) * LD + t % N] = 0.0;
    __syncthreads();
    // deflation: j is a place in the merged order from here
    const double tol = live ? kEps * fmax(fmax(fabs(L.ds[base]), fabs(L.ds[end - 1])), rho) : 0.0;
    const bool small = live && rho * fabs(L.zs[j]) <= tol;
    if (sub == 0) L.fl[j] = small;
    __syncthreads();
    int before = 0;
    if (live) {
      int pj = -1;
      for (int t = base + sub; t < j; t += LP)
        if (!L.fl[t]) {
          ++before;
          pj = t;
        }
      before = lanes_sum<LP>(before);
      pj = lanes_max<LP>(pj + 1) - 1;
      if (!small && pj >= 0) {
        const double z = L.zs[j], zp = L.zs[pj];
        if (fabs((L.ds[j] - L.ds[pj]) * z * zp) <= tol * (z * z + zp * zp)) L.cl[base] = 1;
      }
    }
    __syncthreads();
    if (live && L.cl[base]) {
      if (j == base && sub == 0) {
        int nr;
        L.cnt[base] = dc_deflate(L.ds + base, L.zs + base, sz, rho, tol, L.kr + base, L.dr + base, L.dv + base,
                                 L.ra + base, L.rb + base, L.rc + base, L.rs + base, nr);
        L.nro[base] = nr;
      }
    } else if (live && sub == 0) {
      const int r = j - base;
      if (small) {
        L.dr[base + r - before] = r;
        L.dv[base + r - before] = L.ds[j];
      } else {
        L.kr[base + before] = r;
      }
      if (j == end - 1) {
        L.cnt[base] = before + !small;
        L.nro[base] = 0;
      }
    }
    __syncthreads();
    const int K = live ? L.cnt[base] : 0, ii = j - base;
    if (ii < K && sub == 0) {
      L.dk[j] = L.ds[base + L.kr[j]];
      L.zk[j] = L.zs[base + L.kr[j]];
    }
    __syncthreads();
    if (ii < K) {
      int org;
      double eta;
      const double *const dk = L.dk + base, *const zk = L.zk + base;
      if (s <= LP) dc_secular<LP, 1>(dk, zk, K, ii, rho, sub, org, eta);
      else if (s <= 2 * LP) dc_secular<LP, 2>(dk, zk, K, ii, rho, sub, org, eta);
      else if (s <= 4 * LP) dc_secular<LP, 4>(dk, zk, K, ii, rho, sub, org, eta);
      else if (s <= 8 * LP) dc_secular<LP, 8>(dk, zk, K, ii, rho, sub, org, eta);
      else dc_secular<LP, N / LP>(dk, zk, K, ii, rho, sub, org, eta);
      if (sub == 0) {
        L.og[j] = org;
        L.et[j] = eta;
        L.lam[j] = L.dk[base + org] + eta;
      }
    }
    __syncthreads();
    if (ii < K) {
      // z recomputed from the roots: z_j^2 = prod_i (lam_i - d_j) / prod_{i != j} (d_i - d_j) (/ rho)
      const double dj = L.dk[j];
      double p = 1.0;
#pragma unroll 2
      for (int i = sub; i < K; i += LP) {
        const double num = (L.dk[base + L.og[base + i]] - dj) + L.et[base + i];
        p *= i == ii ? num : num * rcp_nr(L.dk[base + i] - dj);
      }
      p = lanes_prod<LP>(p);
      if (sub == 0) L.zh[j] = copysign(sqrt(fabs(p)), L.zk[j]);
      // place of root ii among all of the block (deflated values after equal roots)
      const double l = L.lam[j];
      int c = 0;
      for (int t = sub; t < sz - K; t += LP) c += L.dv[base + t] < l;
      c = lanes_sum<LP>(c);
      if (sub == 0) L.rk[j] = base + ii + c;
    } else if (live) {
      // deflated value ii - K
      const double l = L.dv[base + ii - K];
      int c = 0;
      for (int t = sub; t < K; t += LP) c += L.lam[base + t] <= l;
      for (int t = sub; t < sz - K; t += LP) c += L.dv[base + t] < l || (L.dv[base + t] == l && t < ii - K);
      c = lanes_sum<LP>(c);
      if (sub == 0) L.rk[j] = base + c;
    }
    __syncthreads();
    if (ii < K) {
      const double d0 = L.dk[base + L.og[j]], eta = L.et[j];
      const int col = L.rk[j];
      double n2 = 0.0;
#pragma unroll 2
      for (int t = sub; t < K; t += LP) {
        const double x = L.zh[base + t] * rcp_nr((L.dk[base + t] - d0) - eta);
        n2 += x * x;
        U[L.pm[base + L.kr[base + t]] * LD + col] = x;
      }
      n2 = lanes_sum<LP>(n2);
      const double in = 1.0 / sqrt(n2);
      for (int t = sub; t < K; t += LP) U[L.pm[base + L.kr[base + t]] * LD + col] *= in;
    } else if (live && sub == 0) {
      U[L.pm[base + L.dr[base + ii - K]] * LD + L.rk[j]] = 1.0;
    }
    __syncthreads();
    // the deflating rotations, last first, on every column
    if (live && sub == 0) {
      const int nr = L.nro[base];
      for (int t = nr - 1; t >= 0; --t) {
        const int pa = L.pm[base + L.ra[base + t]], pb = L.pm[base + L.rb[base + t]];
        const double x = U[pa * LD + j], y = U[pb * LD + j];
        U[pa * LD + j] = L.rc[base + t] * x - L.rs[base + t] * y;
        U[pb * LD + j] = L.rs[base + t] * x + L.rc[base + t] * y;
      }
    }
    __syncthreads();
    // Q <- Q U (rows of a block only meet its columns): the merges of 16 and
    // more rows a half on MFMA, where a row's half bounds the sum; the others
    // an RT x RT tile a thread
    if (s >= 32) {
      const int lane = tid & 63, wave = tid >> 6, l15 = lane & 15, l4 = lane >> 4;
      const int nct = s / 16, tiles = (N / 16) * nct;
      constexpr int MT = (N / 16) * (N / 16) / 4;
      doublex4 o[MT];
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        const int t = u * 4 + wave, r0 = (t / nct) * 16, c0 = r0 / s * s + (t % nct) * 16, k0 = r0 / h * h;
        o[u] = doublex4{0.0, 0.0, 0.0, 0.0};
        if (t < tiles)
          for (int k = k0; k < k0 + h; k += 4)
            o[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(Q[(r0 + l15) * LD + k + l4], U[(k + l4) * LD + c0 + l15], o[u],
                                                        0, 0, 0);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        const int t = u * 4 + wave, r0 = (t / nct) * 16, c0 = r0 / s * s + (t % nct) * 16;
        if (t < tiles)
#pragma unroll
          for (int r = 0; r < 4; ++r) Q[(r0 + Cx<double2>::acc_row(lane, r)) * LD + c0 + l15] = o[u][r];
      }
    } else {
      constexpr int RT = N / 16;
      const int r0 = (tid >> 4) * RT, c0 = (tid & 15) * RT;
      const int w = s < RT ? RT : s, k0 = r0 / w * w;
      double o[RT][RT] = {};
      if (r0 < nn && c0 / w == r0 / w)   // other blocks' columns stay zero
        for (int k = k0; k < k0 + w; ++k) {
          double x[RT], y[RT];
#pragma unroll
          for (int u = 0; u < RT; ++u) {
            x[u] = Q[(r0 + u) * LD + k];
            y[u] = U[k * LD + c0 + u];
          }
#pragma unroll
          for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int t = 0; t < RT; ++t) o[u][t] = fma(x[u], y[t], o[u][t]);
        }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < RT; ++u)
#pragma unroll
        for (int t = 0; t < RT; ++t) Q[(r0 + u) * LD + c0 + t] = o[u][t];
    }
    if (live && sub == 0) L.D[L.rk[j]] = ii < K ? L.lam[j] : L.dv[base + ii - K];
    __syncthreads();
  }
}

// Leaves: every 64-block of T in LDS.  Results: Qt0 (the block's rows), d ascending.
__global__ __launch_bounds__(256) void dc_leaf_kernel(const EigSlot* __restrict__ slots) {
  constexpr int N = kLeaf, LD = N + 1;
  __shared__ double Q[N * LD], U[N * LD];
  __shared__ DcLds<N> L;
  const EigSlot& S = slots[blockIdx.y];
  const int m = S.m, b0 = blockIdx.x * N;
  if (!S.active || b0 >= m || *S.fail) return;
  const int nn = min(N, m - b0);
  const int tid = threadIdx.x;
  if (tid < N) {
    const int i = b0 + tid;
    double x = 0.0, ee = 0.0;
    if (tid < nn) {
      x = in_range(S.d[i]);
      if (i > 0) x -= fabs(S.e[i - 1]);
      if (i + 1 < m) {
        ee = S.e[i];
        x -= fabs(ee);
      }
    }
    L.D[tid] = x;
    L.E[tid] = ee;
  }
  dc_solve<N>(L, Q, U, nn);
  double* Qt = eig_q(S, 0);
  for (int t = tid; t < nn * nn; t += 256) {
    const int i = t / nn, r = t % nn;
    Qt[(size_t)(b0 + i) * m + b0 + r] = Q[r * LD + i];
  }
  if (tid < nn) S.d[b0 + tid] = L.D[tid];
}

// A merge block of a level: [base, base + sz) with the second half at mid.
struct DcBlock {
  int base, mid, end;
  bool on;
};
__device__ __forceinline__ DcBlock dc_block(const EigSlot& S, int level, int blk) {
  // merges of blocks of 64 << level into blocks twice as long
  DcBlock B;
  const int h = kLeaf << level;
  B.base = blk * 2 * h;
  B.mid = min(B.base + h, S.m);
  B.end = min(B.base + 2 * h, S.m);
  B.on = S.active && level < eig_levels(S.m) && B.base < S.m && *S.fail == 0;
  return B;
}

// z, merged order and deflation of one block (one workgroup).
__global__ __launch_bounds__(256) void dc_prep_kernel(const EigSlot* __restrict__ slots, int level) {
  extern __shared__ double dyn[];
  const EigSlot& S = slots[blockIdx.y];
  const DcBlock B = dc_block(S, level, blockIdx.x);
  if (!B.on) return;
  const int m = S.m, s = B.end - B.base, h = B.mid - B.base, tid = threadIdx.x;
  double* const dl = dyn;         // [s] d of the two halves
  double* const ds = dyn + s;     // [s] merged
  double* const zs = dyn + 2 * s; // [s]
  const double* Qt = eig_q(S, level);
  const double ee = B.mid < B.end ? S.e[B.mid - 1] : 0.0;
  const double rho = 2.0 * fabs(ee), sg = ee < 0.0 ? -1.0 : 1.0;
  int32_t* g = S.g + B.base;
  double* f = S.f + B.base;
  for (int j = tid; j < s; j += 256) dl[j] = S.d[B.base + j];
  __syncthreads();
  for (int j = tid; j < s; j += 256) {
    const double dj = dl[j];
    // lower bound in the other half (both ascending); ties keep the first half first
    int lo = j < h ? h : 0, hi = j < h ? s : h;
    const int o0 = lo;
    while (lo < hi) {
      const int md = (lo + hi) >> 1;
      if (j < h ? dl[md] < dj : dl[md] <= dj) lo = md + 1;
      else hi = md;
    }
    const int rank = (j < h ? j : j - h) + lo - o0;
    double z = 0.0;
    if (B.mid < B.end)
      z = (j < h ? Qt[(size_t)(B.base + j) * m + B.mid - 1] : sg * Qt[(size_t)(B.base + j) * m + B.mid]) *
          0.70710678118654752440;
    ds[rank] = dj;
    zs[rank] = z;
    g[(size_t)G_PM * m + rank] = j;
  }
  __syncthreads();
  __shared__ int sK, kept[256], lastk[256];
  const double tol = kEps * fmax(fmax(fabs(ds[0]), fabs(ds[s - 1])), rho);
  // in most merges no two kept values are close enough to be rotated: what is
  // deflated for its weight alone is then counted by all threads, each taking
  // c places in turn
  const int c = (s + 255) / 256, r0 = min(tid * c, s), r1 = min(r0 + c, s);
  int nk = 0, last = -1;
  for (int r = r0; r < r1; ++r)
    if (!(rho * fabs(zs[r]) <= tol)) {
      ++nk;
      last = r;
    }
  kept[tid] = nk;
  lastk[tid] = last;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {   // kept up to and with this thread's places, and the last of them
    const int x = tid >= o ? kept[tid - o] : 0, y = tid >= o ? lastk[tid - o] : -1;
    __syncthreads();
    kept[tid] += x;
    lastk[tid] = max(lastk[tid], y);
    __syncthreads();
  }
  int before = kept[tid] - nk, pj = tid > 0 ? lastk[tid - 1] : -1;
  bool close = false;
  {
    int q = pj;
    for (int r = r0; r < r1; ++r) {
      const double z = zs[r];
      if (rho * fabs(z) <= tol) continue;
      if (q >= 0) {
        const double zp = zs[q];
        if (fabs((ds[r] - ds[q]) * z * zp) <= tol * (z * z + zp * zp)) close = true;
      }
      q = r;
    }
  }
  if (__syncthreads_or(close)) {
    if (tid == 0) {
      int nr;
      sK = dc_deflate(ds, zs, s, rho, tol, g + (size_t)G_KR * m, g + (size_t)G_DR * m, f + (size_t)F_DV * m,
                      g + (size_t)G_RA * m, g + (size_t)G_RB * m, f + (size_t)F_C * m, f + (size_t)F_S * m, nr);
      g[(size_t)G_CNT * m] = sK | nr << 16;   // both at most 4096
    }
  } else {
    for (int r = r0; r < r1; ++r) {
      if (rho * fabs(zs[r]) <= tol) {
        g[(size_t)G_DR * m + r - before] = r;
        f[(size_t)F_DV * m + r - before] = ds[r];
      } else {
        g[(size_t)G_KR * m + before++] = r;
      }
    }
    if (tid == 0) {
      sK = kept[255];
      g[(size_t)G_CNT * m] = sK;
    }
  }
  __syncthreads();
  const int K = sK;
  for (int j = tid; j < K; j += 256) {
    const int r = g[(size_t)G_KR * m + j];
    f[(size_t)F_DK * m + j] = ds[r];
    f[(size_t)F_ZK * m + j] = zs[r];
  }
}

// Roots: one wave each.
__global__ __launch_bounds__(256) void dc_root_kernel(const EigSlot* __restrict__ slots, int level, int nblk) {
  const EigSlot& S = slots[blockIdx.y];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int h2 = kLeaf << (level + 1);
  for (int idx = blockIdx.x * 4 + wave; idx < nblk * h2; idx += gridDim.x * 4) {
    const DcBlock B = dc_block(S, level, idx / h2);
    if (!B.on) return;   // (nor is any behind it)
    const int m = S.m, i = idx % h2;
    int32_t* g = S.g + B.base;
    double* f = S.f + B.base;
    const int K = g[(size_t)G_CNT * m] & 0xffff;
    if (i >= K) continue;
    const double rho = 2.0 * fabs(S.e[B.mid - 1]);
    int org;
    double eta;
    dc_secular<64, 0>(f + (size_t)F_DK * m, f + (size_t)F_ZK * m, K, i, rho, lane, org, eta);
    if (lane == 0) {
      g[(size_t)G_ORG * m + i] = org;
      f[(size_t)F_ETA * m + i] = eta;
    }
  }
}

// z recomputed (into F_ZS) and the places of all values: one wave each.
__device__ __forceinline__ void dc_zhat(const EigSlot& S, const DcBlock& B, int ii) {
  const int lane = threadIdx.x & 63, m = S.m, s = B.end - B.base;
  int32_t* g = S.g + B.base;
  double* f = S.f + B.base;
  const int K = g[(size_t)G_CNT * m] & 0xffff;
  const double* dk = f + (size_t)F_DK * m;
  const double* et = f + (size_t)F_ETA * m;
  const double* dv = f + (size_t)F_DV * m;
  const int32_t* og = g + (size_t)G_ORG * m;
  int c = 0;
  if (ii < K) {
    const double dj = dk[ii], l = dk[og[ii]] + et[ii];
    double p = 1.0;
    for (int i = lane; i < K; i += 64) {
      const double num = (dk[og[i]] - dj) + et[i];
      p *= i == ii ? num : num * rcp_nr(dk[i] - dj);
    }
    p = lanes_prod<64>(p);
    if (lane == 0) f[(size_t)F_ZS * m + ii] = copysign(sqrt(fabs(p)), f[(size_t)F_ZK * m + ii]);
    for (int t = lane; t < s - K; t += 64) c += dv[t] < l;
    c = lanes_sum<64>(c);
    c += ii;
  } else {
    const double l = dv[ii - K];
    for (int t = lane; t < K; t += 64) c += dk[og[t]] + et[t] <= l;
    for (int t = lane; t < s - K; t += 64) c += dv[t] < l || (dv[t] == l && t < ii - K);
    c = lanes_sum<64>(c);
  }
  if (lane == 0) {
    g[(size_t)G_RANK * m + ii] = c;
    f[(size_t)F_DS * m + c] = ii < K ? dk[og[ii]] + et[ii] : dv[ii - K];   // the merged eigenvalues
  }
}
__global__ __launch_bounds__(256) void dc_zhat_kernel(const EigSlot* __restrict__ slots, int level, int nblk) {
  const EigSlot& S = slots[blockIdx.y];
  const int h2 = kLeaf << (level + 1);
  for (int idx = blockIdx.x * 4 + (threadIdx.x >> 6); idx < nblk * h2; idx += gridDim.x * 4) {
    const DcBlock B = dc_block(S, level, idx / h2);
    if (!B.on) return;
    if (idx % h2 < B.end - B.base) dc_zhat(S, B, idx % h2);
  }
}

// Vectors of the merge: column `rank` of U as row Ut[base + rank][*] (in E),
// in the halves' own order; the deflating rotations applied.  One wave each,
// its column in LDS.
__device__ __forceinline__ void dc_vec(const EigSlot& S, const DcBlock& B, int ii, double* u) {   // u: by merged rank
  const int lane = threadIdx.x & 63, m = S.m, s = B.end - B.base;
  const int32_t* g = S.g + B.base;
  const double* f = S.f + B.base;
  const int K = g[(size_t)G_CNT * m] & 0xffff, nr = g[(size_t)G_CNT * m] >> 16;
  const int32_t* kr = g + (size_t)G_KR * m;
  const int rank = g[(size_t)G_RANK * m + ii];
  if (ii == 0)
    for (int t = lane; t < s; t += 64) S.d[B.base + t] = f[(size_t)F_DS * m + t];
  for (int t = lane; t < s; t += 64) u[t] = 0.0;
  wave_fence();
  if (ii < K) {
    const double* dk = f + (size_t)F_DK * m;
    const double* zh = f + (size_t)F_ZS * m;
    const double d0 = dk[g[(size_t)G_ORG * m + ii]], eta = f[(size_t)F_ETA * m + ii];
    double n2 = 0.0;
    for (int t = lane; t < K; t += 64) {
      const double x = zh[t] * rcp_nr((dk[t] - d0) - eta);
      n2 += x * x;
      u[kr[t]] = x;
    }
    const double in = 1.0 / sqrt(wave_sum(n2));
    for (int t = lane; t < K; t += 64) u[kr[t]] = u[kr[t]] * in;
  } else if (lane == 0) {
    u[g[(size_t)G_DR * m + ii - K]] = 1.0;
  }
  wave_fence();
  if (lane == 0)
    for (int t = nr - 1; t >= 0; --t) {
      const int pa = g[(size_t)G_RA * m + t], pb = g[(size_t)G_RB * m + t];
      const double c = f[(size_t)F_C * m + t], sn = f[(size_t)F_S * m + t];
      const double x = u[pa], y = u[pb];
      u[pa] = c * x - sn * y;
      u[pb] = sn * x + c * y;
    }
  wave_fence();
  double* Ut = (double*)S.E + (size_t)(B.base + rank) * m + B.base;
  for (int t = lane; t < s; t += 64) Ut[g[(size_t)G_PM * m + t]] = u[t];
}
__global__ __launch_bounds__(256) void dc_vec_kernel(const EigSlot* __restrict__ slots, int level, int nblk,
                                                     int s_cap) {
  extern __shared__ double dyn[];
  const EigSlot& S = slots[blockIdx.y];
  const int wave = threadIdx.x >> 6, h2 = kLeaf << (level + 1);
  for (int idx = blockIdx.x * 4 + wave; idx < nblk * h2; idx += gridDim.x * 4) {
    const DcBlock B = dc_block(S, level, idx / h2);
    if (!B.on) return;
    if (idx % h2 < B.end - B.base) dc_vec(S, B, idx % h2, dyn + (size_t)wave * s_cap);
    wave_fence();   // u is this wave's again
  }
}

// One 64 x 64 tile of a real product C = A B on FP64 MFMA (row-major, any
// leading dimensions; rows of A may run backwards), 256 threads.
__device__ __forceinline__ void dgemm_tile(const double* __restrict__ A, long long lda, const double* __restrict__ B,
                                           long long ldb, double* __restrict__ C, long long ldc, int M, int N, int K,
                                           int tm, int tn, double* As, double* Bs) {
  constexpr int KC = 32, LD = 65;   // As[KC][LD], Bs[KC][LD], two buffers each; the odd pitch for the stores along k
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = tm * 64, n0 = tn * 64;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int ai = tid >> 5, ak = tid & 31;             // 64 rows x 32 k, the lanes along k
  const int bk = tid >> 6, bj = tid & 63;             // 32 k x 64 columns, the lanes along the columns
  double ra[8], rb[8];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      ra[q] = m0 + ai + 8 * q < M && k0 + ak < K ? A[(m0 + ai + 8 * q) * lda + k0 + ak] : 0.0;
      rb[q] = k0 + bk + 4 * q < K && n0 + bj < N ? B[(k0 + bk + 4 * q) * ldb + n0 + bj] : 0.0;
    }
  };
  auto stage = [&](int b) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      As[(b * KC + ak) * LD + ai + 8 * q] = ra[q];
      Bs[(b * KC + bk + 4 * q) * LD + bj] = rb[q];
    }
  };
  doublex4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  load(0);
  stage(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < K; k0 += KC) {
    const bool more = k0 + KC < K;
    if (more) load(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC / 4; ++kk) {
      const int kr = buf * KC + kk * 4 + (lane >> 4);
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = As[kr * LD + wm + i * 16 + (lane & 15)];
        b[i] = Bs[kr * LD + wn + i * 16 + (lane & 15)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm + i * 16 + Cx<double2>::acc_row(lane, r), col = n0 + wn + j * 16 + (lane & 15);
        if (row < M && col < N) C[row * ldc + col] = acc[i][j][r];
      }
}
constexpr int kDgemmLds = 2 * 32 * 65;

// Qt of the merged block: rows Ut times the two halves' Qt.  grid
// (row tiles x column tiles of the block, blocks, slots)
__global__ __launch_bounds__(256) void dc_gemm_kernel(const EigSlot* __restrict__ slots, int level, int nt) {
  __shared__ double As[kDgemmLds], Bs[kDgemmLds];
  const EigSlot& S = slots[blockIdx.z];
  const DcBlock B = dc_block(S, level, blockIdx.y);
  if (!B.on) return;
  const int m = S.m, s = B.end - B.base, h = B.mid - B.base;
  const int nt1 = (h + 63) / 64, nt2 = (s - h + 63) / 64;
  const int tm = blockIdx.x / nt, tn = blockIdx.x % nt;
  if (tm * 64 >= s || tn >= nt1 + nt2) return;
  const double* Ut = (const double*)S.E + (size_t)B.base * m + B.base;
  const double* Qi = eig_q(S, level) + (size_t)B.base * m + B.base;
  double* Qo = eig_q(S, level + 1) + (size_t)B.base * m + B.base;
  if (tn < nt1)
    dgemm_tile(Ut, m, Qi, m, Qo, m, s, h, h, tm, tn, As, Bs);
  else
    dgemm_tile(Ut + h, m, Qi + (size_t)h * m + h, m, Qo + h, m, s, s - h, s - h, tm, tn - nt1, As, Bs);
}

// theta' <- Qt Y, rows by decreasing eigenvalue (Y in E, [m][n] complex as [m][2n] real)
__global__ __launch_bounds__(256) void eig_apply_kernel(const EigSlot* __restrict__ slots, int n_slots, int ntn_cap,
                                                        int tiles_cap) {
  __shared__ double As[kDgemmLds], Bs[kDgemmLds];
  int item, tile;
  if (!xcd_item_tile(blockIdx.x, n_slots, tiles_cap, item, tile)) return;
  const EigSlot& S = slots[item];
  if (!S.active || *S.fail) return;
  const int m = S.m, tm = tile / ntn_cap, tn = tile % ntn_cap;
  if (tm * 64 >= m || tn * 64 >= 2 * S.n) return;
  const double* Qt = eig_q(S, eig_levels(m)) + (size_t)(m - 1) * m;
  dgemm_tile(Qt, -(long long)m, (const double*)S.E, 2 * S.n, (double*)S.X, 2 * S.ld, m, 2 * S.n, m, tm, tn, As, Bs);
}

// ---------------------------------------------------------------------------
// Reflectors on theta'
// ---------------------------------------------------------------------------
// Compact WY factor of block blockIdx.x: H_k ... H_{k+15} = I - V T V^dag,
// T upper triangular with T_jj = tau_j, T_{0:j,j} = -tau_j T_{0:j,0:j} (V^dag v_j).
__global__ __launch_bounds__(256) void wy_t_kernel(const EigSlot* __restrict__ slots) {
  __shared__ double2 Gw[4][kWy][kWy + 1], Tm[kWy][kWy + 1];
  const EigSlot& S = slots[blockIdx.y];
  const int m = S.m, k0 = blockIdx.x * kWy;
  if (!S.active || k0 >= m - 1 || *S.fail) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, l4 = lane >> 4;
  const int nv = min(kWy, m - 1 - k0);
  const double2* V = S.V + (size_t)blockIdx.x * m * kWy;
  // V^dag V on MFMA, the waves taking row tiles in turn (unused columns are zero)
  doublex4 re = {0.0, 0.0, 0.0, 0.0}, im = re;
  for (int t = k0 / 16 + wave; t * 16 < m; t += 4) {
    double2 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = t * 16 + 4 * r + l4;
      v[r] = row < m ? V[(size_t)row * kWy + l15] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, v[r].x, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, v[r].y, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].y, v[r].y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(-v[r].y, v[r].x, im, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) Gw[wave][l4 + 4 * r][l15] = make_double2(re[r], im[r]);
  __syncthreads();
  const int a = tid >> 4, b = tid & 15;
  const double2 g = cadd(cadd(Gw[0][a][b], Gw[1][a][b]), cadd(Gw[2][a][b], Gw[3][a][b]));
  __syncthreads();
  Gw[0][a][b] = g;
  Tm[a][b] = make_double2(0.0, 0.0);
  __syncthreads();
  if (wave == 0) {
    for (int j = 0; j < nv; ++j) {
      const double2 tj = S.tau[k0 + j];
      // T[i][j] = -tau_j sum_l T[i][l] G[l][j]: four lanes a row
      const int i = lane >> 2, q = lane & 3;
      double2 x = make_double2(0.0, 0.0);
      for (int l = q; l < j; l += 4) x = cadd(x, cmul(Tm[i][l], Gw[0][l][j]));
      x.x = lanes_sum<4>(x.x);
      x.y = lanes_sum<4>(x.y);
      x = cmul(x, tj);
      wave_fence();
      if (q == 0 && i < j) Tm[i][j] = make_double2(-x.x, -x.y);
      if (q == 0 && i == j) Tm[j][j] = tj;
      wave_fence();
    }
  }
  __syncthreads();
  S.T[(size_t)blockIdx.x * kWy * kWy + tid] = Tm[a][b];
}

// Y = H_{m-2}^dag ... H_0^dag theta', 16 columns a workgroup of 8 waves, all
// blocks of reflectors in turn: X <- X - V T^dag (V^dag X).  The strip stays
// in registers as MFMA accumulators (TPW tiles of 16 rows a wave), whose
// layout is at once the right operand's layout of the next product, so a
// strip is read and written once and only V streams (from L2, shared by the
// strips of a matrix).  TPW = 0: the strip stays in Y (m > 1024).
template <int TPW>
__global__ __launch_bounds__(512) void wy_apply_kernel(const EigSlot* __restrict__ slots, int m_lo, int m_hi,
                                                       int n_slots, int strips_cap) {
  constexpr bool REG = TPW > 0;
  constexpr int TR = REG ? TPW : 1;
  __shared__ double Pw[8][2][16][17];
  __shared__ double Ps[2][16][17];
  int item, strip;
  if (!xcd_item_tile(blockIdx.x, n_slots, strips_cap, item, strip)) return;
  const EigSlot& S = slots[item];
  const int m = S.m, n = S.n;
  if (!S.active || m <= m_lo || m > m_hi || strip * 16 >= n || *S.fail) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, l4 = lane >> 4;
  const int col = strip * 16 + l15;
  const bool cok = col < n;
  double2* const Y = S.E;
  const int ntile = (m + 15) / 16;
  doublex4 xr[TR], xi[TR];
  auto load_x = [&](const double2* src, int ld, int rt, doublex4& re, doublex4& im) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rt * 16 + 4 * r + l4;
      double2 x = make_double2(0.0, 0.0);
      if (cok && row < m) x = src[(size_t)row * ld + col];
      re[r] = x.x;
      im[r] = x.y;
    }
  };
  auto store_x = [&](int rt, const doublex4& re, const doublex4& im) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rt * 16 + 4 * r + l4;
      if (cok && row < m) Y[(size_t)row * n + col] = make_double2(re[r], im[r]);
    }
  };
  if (REG) {
#pragma unroll
    for (int t = 0; t < TR; ++t) load_x(S.X, S.ld, t * 8 + wave, xr[t], xi[t]);
  } else {
    for (int rt = wave; rt < ntile; rt += 8) {
      doublex4 re, im;
      load_x(S.X, S.ld, rt, re, im);
      store_x(rt, re, im);
    }
  }
  const int nblk = (m - 1 + kWy - 1) / kWy;
  for (int b = 0; b < nblk; ++b) {
    const int k0 = b * kWy;
    const double2* V = S.V + (size_t)b * m * kWy;
    // P = V^dag X: this wave's row tiles
    doublex4 pr = {0.0, 0.0, 0.0, 0.0}, pi = {0.0, 0.0, 0.0, 0.0};
    auto project = [&](int rt, const doublex4& re, const doublex4& im) {
      double2 v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rt * 16 + 4 * r + l4;
        v[r] = row < m ? V[(size_t)row * kWy + l15] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pr = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, re[r], pr, 0, 0, 0);
        pi = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, im[r], pi, 0, 0, 0);
        pr = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].y, im[r], pr, 0, 0, 0);
        pi = __builtin_amdgcn_mfma_f64_16x16x4f64(-v[r].y, re[r], pi, 0, 0, 0);
      }
    };
    if (REG) {
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const int rt = t * 8 + wave;
        if (rt * 16 + 15 > k0 && rt < ntile) project(rt, xr[t], xi[t]);   // V is zero up to row k0
      }
    } else {
      for (int rt = wave; rt < ntile; rt += 8) {
        if (rt * 16 + 15 <= k0) continue;
        doublex4 re, im;
        load_x(Y, n, rt, re, im);
        project(rt, re, im);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      Pw[wave][0][l4 + 4 * r][l15] = pr[r];
      Pw[wave][1][l4 + 4 * r][l15] = pi[r];
    }
    __syncthreads();
    {
      const int c = tid >> 8, i = (tid >> 4) & 15, j = tid & 15;
      double x = 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) x += Pw[u][c][i][j];
      Ps[c][i][j] = x;
    }
    __syncthreads();
    // -T^dag P, in the layout of a right operand
    doublex4 qr = {0.0, 0.0, 0.0, 0.0}, qi = {0.0, 0.0, 0.0, 0.0};
    const double2* Tb = S.T + (size_t)b * kWy * kWy;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 t = Tb[(4 * r + l4) * kWy + l15];   // T^dag[l15][4r + l4] = conj(T[4r + l4][l15])
      const double br = Ps[0][4 * r + l4][l15], bi = Ps[1][4 * r + l4][l15];
      qr = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.x, br, qr, 0, 0, 0);
      qi = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.x, bi, qi, 0, 0, 0);
      qr = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.y, bi, qr, 0, 0, 0);
      qi = __builtin_amdgcn_mfma_f64_16x16x4f64(t.y, br, qi, 0, 0, 0);
    }
    auto update = [&](int rt, doublex4& re, doublex4& im) {
      double2 v[4];
      const int row = rt * 16 + l15;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = row < m ? V[(size_t)row * kWy + 4 * r + l4] : make_double2(0.0, 0.0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, qr[r], re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].x, qi[r], im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-v[r].y, qi[r], re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r].y, qr[r], im, 0, 0, 0);
      }
    };
    if (REG) {
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const int rt = t * 8 + wave;
        if (rt * 16 + 15 > k0 && rt < ntile) update(rt, xr[t], xi[t]);
      }
    } else {
      for (int rt = wave; rt < ntile; rt += 8) {
        if (rt * 16 + 15 <= k0) continue;
        doublex4 re, im;
        load_x(Y, n, rt, re, im);
        update(rt, re, im);
        store_x(rt, re, im);
      }
    }
  }
  if (REG) {
#pragma unroll
    for (int t = 0; t < TR; ++t)
      if (t * 8 + wave < ntile) store_x(t * 8 + wave, xr[t], xi[t]);
  }
}

// ---------------------------------------------------------------------------
// Check of the rotated rows by the Jacobi's convergence test
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void eig_check_kernel(const EigSlot* __restrict__ slots,
                                                        const JacMat* __restrict__ mats, double tol, double abs_tol) {
  const EigSlot& S = slots[blockIdx.y];
  if (!S.active || *S.fail) return;
  const int m = S.m;
  const double thr_abs = abs_tol * mats[blockIdx.y].fro2;
  bool bad = false;
  for (int r = blockIdx.x; r < m; r += gridDim.x) {
    const double grr = fabs(S.A[(size_t)r * m + r].x);
    for (int c = threadIdx.x; c < r; c += 256) {
      const double2 g = S.A[(size_t)r * m + c];
      const double thr = fmax(thr_abs, tol * sqrt(grr * fabs(S.A[(size_t)c * m + c].x)));
      if (!(g.x * g.x + g.y * g.y <= thr * thr)) bad = true;
    }
  }
  if (bad) *S.fail = 2;   // rotated, not yet orthogonal
}

// done = squared norms of the rotated rows in place; conv set where the check passed
__global__ __launch_bounds__(256) void eig_done_kernel(const EigSlot* __restrict__ slots, JacMat* mats) {
  const EigSlot& S = slots[blockIdx.x];
  if (!S.active || *S.fail == 1) return;
  JacMat& M = mats[blockIdx.x];
  for (int r = threadIdx.x; r < S.m; r += 256) M.nrm2[r] = S.A[(size_t)r * S.m + r].x;
  if (threadIdx.x == 0 && *S.fail == 0) M.conv = 1;
}

// ---------------------------------------------------------------------------
// Matrices of one panel (m <= 64): all of the above in one workgroup's LDS
// ---------------------------------------------------------------------------
// The Gram (upper 16 x 16 tiles, dealt to the four waves) of the m rows of X
// in G [N][N + 1], both triangles.
template <int N>
__device__ __forceinline__ void small_gram(const double2* __restrict__ X, int m, int n, int ld, double2* G) {
  constexpr int LD = N + 1, MT = N == 64 ? 3 : 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, l4 = lane >> 4;
  // N = 64: (0,0) (0,1) (0,2) | (0,3) (1,1) (1,2) | (1,3) (2,2) | (2,3) (3,3); N = 32: (0,0) | (0,1) | (1,1) | -
  const int TI[4][3] = {{0, 0, 0}, {0, 1, 1}, {1, 2, 0}, {2, 3, 0}}, TJ[4][3] = {{0, 1, 2}, {3, 1, 2}, {3, 2, 0}, {3, 3, 0}};
  const int nt = N == 64 ? (wave < 2 ? 3 : 2) : (wave < 3 ? 1 : 0);
  int ti[MT], tj[MT];
  const double2 *ra[MT], *rb[MT];
  bool oa[MT], ob[MT];
  doublex4 re[MT], im[MT];
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    ti[u] = N == 64 ? TI[wave][u] : wave == 2;
    tj[u] = N == 64 ? TJ[wave][u] : wave >= 1;
    oa[u] = u < nt && ti[u] * 16 + l15 < m;
    ob[u] = u < nt && tj[u] * 16 + l15 < m;
    ra[u] = X + (size_t)(oa[u] ? ti[u] * 16 + l15 : 0) * ld;
    rb[u] = X + (size_t)(ob[u] ? tj[u] * 16 + l15 : 0) * ld;
    re[u] = im[u] = doublex4{0.0, 0.0, 0.0, 0.0};
  }
#pragma unroll 4
  for (int c0 = 0; c0 < n; c0 += 4) {
    const int c = c0 + l4;
    double2 a[MT], b[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      a[u] = oa[u] && c < n ? ra[u][c] : make_double2(0.0, 0.0);
      b[u] = ob[u] && c < n ? rb[u][c] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[u].x, re[u], 0, 0, 0);
      im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, b[u].x, im[u], 0, 0, 0);
      re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, b[u].y, re[u], 0, 0, 0);
      im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[u].x, b[u].y, im[u], 0, 0, 0);
    }
  }
#pragma unroll
  for (int u = 0; u < MT; ++u)
    if (u < nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = ti[u] * 16 + Cx<double2>::acc_row(lane, r), j = tj[u] * 16 + l15;
        const double x = re[u][r], y = i == j ? 0.0 : im[u][r];
        if (i <= j) {
          G[i * LD + j] = make_double2(x, y);
          G[j * LD + i] = make_double2(x, -y);
        }
      }
  __syncthreads();
}

// One matrix of at most N rows per workgroup, from the Gram to the check.  The
// reflectors (blocks of 16) and Z^T are applied to theta' on MFMA, a strip of 16
// columns per wave in registers: a product's accumulators are the next one's
// right operand.  One place in LDS holds in turn the Gram, the reflectors (the
// Gram is in registers by then; they are applied before the divide and conquer
// needs the place), Q and U, and the check's Gram: 77 KB for N = 64, so a CU holds
// two matrices at once (at 160 KB it held one: a layer of 48 chains of mixed
// lengths up to 40 at m = 48 took 604 us, now 440).
template <int N>
struct SmallLds {
  // the Gram; then V, V[i][k] = entry i of the reflector of step k (column N:
  // zeros); then Q and U of the divide and conquer; then the check's Gram
  double2 G[N * (N + 1)];
  union {
    DcLds<N> L;
    struct {
      double D[N], E[N];      // as in L
      union {
        TriLds<N, 256, true> t;
        double2 T[N == 32 ? 2 * 16 * 16 : 1];
      };
    } u;
  };
  double2 tau[N];
  int bad;
  // compact WY factor of block p: for N = 64 in the blocks of V above the
  // diagonal ones, which are zero and not read
  __device__ __forceinline__ double2& T(int p, int i, int j) {
    if (N == 32) return u.T[(p * 16 + i) * 16 + j];
    return G[((p == 0 ? 16 : 0) + i) * (N + 1) + (p == 0 ? 32 : p * 16) + j];
  }
};

template <int N>
__device__ __forceinline__ void small_tri(SmallLds<N>& S, int m, double sc) {
  constexpr int LD = N + 1;
  auto load = [&](int i, int j) {
    const double2 x = S.G[i * LD + j];
    return make_double2(x.x * sc, x.y * sc);
  };
  struct Out {
    enum : bool { kLds = true };
    SmallLds<N>& S;
    int m;
    __device__ __forceinline__ void operator()(int k, int i, double2 v) const { S.G[i * LD + k] = v; }
    __device__ __forceinline__ const double2* col(int k) const { return S.G + k; }
    __device__ __forceinline__ void step(int k, double d, double e, double2 t) const {
      S.L.D[k] = d;
      S.L.E[k] = e;
      S.tau[k] = t;
    }
    __device__ __forceinline__ void last(double d) const {
      S.L.D[m - 1] = d;
      S.L.E[m - 1] = 0.0;
    }
  };
  tri_block<N, 256>(S.u.t, m, load, Out{S, m});
  // unused columns of the last block of reflectors
  if (threadIdx.x < N)
    for (int k = max(m - 1, 0); k < N; ++k) S.G[threadIdx.x * LD + k] = make_double2(0.0, 0.0);
  __syncthreads();
}

// Compact WY factors of the blocks of reflectors, a wave each.
template <int N>
__device__ __forceinline__ void small_wy(SmallLds<N>& S, int m) {
  constexpr int LD = N + 1, NT = N / 16;
  const int lane = threadIdx.x & 63, p = threadIdx.x >> 6, l15 = lane & 15, l4 = lane >> 4;
  if (p < NT) {
    doublex4 re = {0.0, 0.0, 0.0, 0.0}, im = re;
    for (int t = p; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 v = S.G[(t * 16 + 4 * r + l4) * LD + p * 16 + l15];
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, v.x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, v.y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, v.y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, v.x, im, 0, 0, 0);
      }
    // V^dag V above the diagonal, in T's place: column j is read before T's takes it
#pragma unroll
    for (int r = 0; r < 4; ++r)
      S.T(p, l4 + 4 * r, l15) = l4 + 4 * r < l15 ? make_double2(re[r], im[r]) : make_double2(0.0, 0.0);
    __builtin_amdgcn_wave_barrier();
    const int nv = min(16, m - 1 - p * 16);
    for (int j = 0; j < 16; ++j) {
      if (j >= nv) {   // no reflector
        if (lane < 16) S.T(p, lane, j) = make_double2(0.0, 0.0);
        continue;
      }
      const double2 tj = S.tau[p * 16 + j];
      // T[i][j] = -tau_j sum_l T[i][l] F[l][j]: four lanes a row
      const int i = lane >> 2, q = lane & 3;
      double2 x = make_double2(0.0, 0.0);
      for (int l = q; l < j; l += 4) x = cadd(x, cmul(S.T(p, i, l), S.T(p, l, j)));
      x.x = lanes_sum<4>(x.x);
      x.y = lanes_sum<4>(x.y);
      x = cmul(x, tj);
      __builtin_amdgcn_wave_barrier();
      if (q == 0 && i < j) S.T(p, i, j) = make_double2(-x.x, -x.y);
      if (q == 0 && i == j) S.T(p, j, j) = tj;
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
}

// The rotation leaves rounding of |X| in every row, which for a short row is a
// part along the long ones: of 1e-16 |X| / s relative to its length s.  The
// check's Gram (S.G, rows by decreasing length) has it to rounding of the two
// rows' own lengths, so it is taken out to first order: row p loses
// G_pq / (G_qq - G_pp) of every row q at least twice as long, which is a
// rotation to second order (the long rows' own change is under their
// rounding).  The squared lengths, S.G's diagonal, stay what they are.
// It matters where a result divides by short lengths: the gradient of 12 sites
// cut at 1e-10 was 8.1e-11 off without it, 1e-12 with it and 5.3e-12 by the
// sweeps.  Where rows as short as the cut 1e-12 leaves them are resolved it costs
// 2.5 % of a layer of small bonds (48 chains, m = 48: 4.41 -> 4.52 ms a step).
template <int N>
__device__ __attribute__((noinline)) void small_clean(SmallLds<N>& S, double2* X, int m, int n, int ld) {
  constexpr int LD = N + 1, NT = N / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, l4 = lane >> 4;
  for (int t = tid; t < N * N; t += 256) {
    const int a = t / N, b = t % N;
    if (b >= a) continue;
    const double ga = S.G[a * LD + a].x, gb = S.G[b * LD + b].x;
    const bool on = a < m && 4.0 * ga < gb;
    const double f = on ? 1.0 / (gb - ga) : 0.0;
    const double2 g = S.G[a * LD + b];
    S.G[a * LD + b] = on ? make_double2(g.x * f, g.y * f) : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int c0 = wave * 16; c0 < n; c0 += 64) {
    const int col = c0 + l15;
    doublex4 xr[NT], xi[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = t * 16 + 4 * r + l4;
        double2 x = make_double2(0.0, 0.0);
        if (row < m && col < n) x = X[(size_t)row * ld + col];
        xr[t][r] = x.x;
        xi[t][r] = x.y;
      }
    // (a tile of rows takes from those up to itself: the last first, in place)
#pragma unroll
    for (int a = NT - 1; a >= 0; --a) {
      if (a * 16 >= m) continue;
      doublex4 pr = {0.0, 0.0, 0.0, 0.0}, pi = pr;
#pragma unroll
      for (int t = 0; t <= a; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = a * 16 + l15, k = t * 16 + 4 * r + l4;
          double2 v = S.G[i * LD + k];
          if (k >= i) v = make_double2(0.0, 0.0);
          pr = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, xr[t][r], pr, 0, 0, 0);
          pi = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, xi[t][r], pi, 0, 0, 0);
          pr = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, xi[t][r], pr, 0, 0, 0);
          pi = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, xr[t][r], pi, 0, 0, 0);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = a * 16 + 4 * r + l4;
        if (row < m && col < n) X[(size_t)row * ld + col] = make_double2(xr[a][r] - pr[r], xi[a][r] - pi[r]);
      }
    }
  }
  __syncthreads();
}

// M's rows rotated in place and M->nrm2 set; returns whether they passed the check (uniform).
template <int N>
__device__ __forceinline__ bool small_rotate(SmallLds<N>& S, double2* X, int m, int n, int ld, double fro2, double tol,
                                             double abs_tol) {
  constexpr int LD = N + 1, NT = N / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, l4 = lane >> 4;
  if (tid == 0) S.bad = 0;
  small_tri<N>(S, m, 1.0 / fro2);
  small_wy<N>(S, m);
  auto load = [&](int col, doublex4 (&xr)[NT], doublex4 (&xi)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = t * 16 + 4 * r + l4;
        double2 a = make_double2(0.0, 0.0);
        if (row < m && col < n) a = X[(size_t)row * ld + col];
        xr[t][r] = a.x;
        xi[t][r] = a.y;
      }
  };
  for (int c0 = wave * 16; c0 < n; c0 += 64) {
    const int col = c0 + l15;
    doublex4 xr[NT], xi[NT];
    load(col, xr, xi);
#pragma unroll
    for (int p = 0; p < NT; ++p) {
      if (p * 16 >= m - 1) continue;
      doublex4 pr = {0.0, 0.0, 0.0, 0.0}, pi = pr, qr = pr, qi = pr;
#pragma unroll
      for (int t = p; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double2 v = S.G[(t * 16 + 4 * r + l4) * LD + p * 16 + l15];
          pr = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, xr[t][r], pr, 0, 0, 0);
          pi = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, xi[t][r], pi, 0, 0, 0);
          pr = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, xi[t][r], pr, 0, 0, 0);
          pi = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, xr[t][r], pi, 0, 0, 0);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 t = S.T(p, 4 * r + l4, l15);
        qr = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.x, pr[r], qr, 0, 0, 0);
        qi = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.x, pi[r], qi, 0, 0, 0);
        qr = __builtin_amdgcn_mfma_f64_16x16x4f64(-t.y, pi[r], qr, 0, 0, 0);
        qi = __builtin_amdgcn_mfma_f64_16x16x4f64(t.y, pr[r], qi, 0, 0, 0);
      }
#pragma unroll
      for (int t = p; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double2 v = S.G[(t * 16 + l15) * LD + p * 16 + 4 * r + l4];
          xr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, qr[r], xr[t], 0, 0, 0);
          xi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, qi[r], xi[t], 0, 0, 0);
          xr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, qi[r], xr[t], 0, 0, 0);
          xi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, qr[r], xi[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = t * 16 + 4 * r + l4;
        if (row < m && col < n) X[(size_t)row * ld + col] = make_double2(xr[t][r], xi[t][r]);
      }
  }
  __syncthreads();   // V and T have been read
  double x = 0.0;
  if (tid < m) x = in_range(S.L.D[tid]) - (tid > 0 ? fabs(S.L.E[tid - 1]) : 0.0) - (tid + 1 < m ? fabs(S.L.E[tid]) : 0.0);
  __syncthreads();
  if (tid < N) S.L.D[tid] = x;
  double* const Q = (double*)S.G;
  dc_solve<N>(S.L, Q, Q + N * LD, m);
  for (int c0 = wave * 16; c0 < n; c0 += 64) {
    const int col = c0 + l15;
    doublex4 xr[NT], xi[NT];
    load(col, xr, xi);
#pragma unroll
    for (int a = 0; a < NT; ++a) {
      doublex4 pr = {0.0, 0.0, 0.0, 0.0}, pi = pr;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double q = Q[(t * 16 + 4 * r + l4) * LD + a * 16 + l15];
          pr = __builtin_amdgcn_mfma_f64_16x16x4f64(q, xr[t][r], pr, 0, 0, 0);
          pi = __builtin_amdgcn_mfma_f64_16x16x4f64(q, xi[t][r], pi, 0, 0, 0);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = a * 16 + 4 * r + l4;   // eigenvalues ascend; the rows are left in decreasing order
        if (row < m && col < n) X[(size_t)(m - 1 - row) * ld + col] = make_double2(pr[r], pi[r]);
      }
    }
  }
  __syncthreads();
  small_gram<N>(X, m, n, ld, S.G);
  const double thr_abs = abs_tol * fro2;
  bool bad = false, rough = false;
  for (int t = tid; t < N * N; t += 256) {
    const int a = t / N, b = t % N;
    if (a >= m || b >= a) continue;
    const double2 g = S.G[a * LD + b];
    const double ga = S.G[a * LD + a].x, gb = S.G[b * LD + b].x, g2 = g.x * g.x + g.y * g.y;
    const double thr = fmax(thr_abs, tol * sqrt(fabs(ga * gb)));
    if (!(g2 <= thr * thr)) bad = true;
    if (ga > thr_abs && 4.0 * ga < gb && g2 > kRough * kRough * ga * gb) rough = true;
  }
  if (bad) S.bad = 1;
  if (__syncthreads_or(rough)) small_clean<N>(S, X, m, n, ld);
  return !S.bad;
}

// A matrix takes the class of its own size, whatever else is in its batch, so
// that its result does not depend on the batch.
template <int N>
__device__ __forceinline__ bool small_class(int m) {
  return m <= N && m >= 1 && (N == 32 || m > N / 2);
}

// Matrix k of the launch is mats[list[k]] for k < *n_list, or mats[k] for
// k < n; those of this class not yet converged are rotated.
// One matrix of a list: a function of its own, so that nothing of a matrix's
// work is kept in registers over the loop of the kernel.
template <int N>
__device__ __attribute__((noinline)) void small_rotate_item(SmallLds<N>& S, JacMat* Mp, double tol, double abs_tol) {
  JacMat* const M = Gp<JacMat>(Mp);
  const int m = M->m, n = M->n, ld = M->ld;
  double2* const X = M->X;
  double* const nrm2 = M->nrm2;
  small_gram<N>(X, m, n, ld, S.G);
  // the norm from the Gram, as the kernels below take it: a matrix's bits do not
  // depend on which of them it goes through
  const int lane = threadIdx.x & 63;
  const double fro2 = wave_sum(lane < m ? S.G[lane * (N + 1) + lane].x : 0.0);
  const bool done = small_rotate<N>(S, X, m, n, ld, fro2, tol, abs_tol);
  if (threadIdx.x < m) nrm2[threadIdx.x] = S.G[threadIdx.x * (N + 1) + threadIdx.x].x;
  if (threadIdx.x == 0 && done) M->conv = 1;
  __syncthreads();
}
template <int N>
__global__ __launch_bounds__(256, 2) void small_rotate_kernel(JacMat* __restrict__ mats, int n,
                                                           const int32_t* __restrict__ list,
                                                           const int32_t* __restrict__ n_list, double tol,
                                                           double abs_tol) {
  __shared__ SmallLds<N> S;
  const int nk = list ? min(*n_list, n) : n;
  for (int k = blockIdx.x; k < nk; k += gridDim.x) {
    JacMat* M = mats + (list ? list[k] : k);
    const int m = M->m;
    const double fro2 = M->fro2;
    if (M->conv || !small_class<N>(m) || !eig_small_takes(m, M->n) || !(fro2 > 1e-250 && fro2 < 1e250)) continue;
    small_rotate_item<N>(S, M, tol, abs_tol);
  }
}

// The whole split of the bonds of this class in a layer, a workgroup each:
// descriptor, norm and range from the Gram, rotation, check, count rule and
// write-back in one launch, in place of eleven (each about 5 us on the
// device's queue whatever it does).  A bond that the direct path leaves
// (non-finite or out of range, or not orthogonal enough) keeps M.pad = 0 and
// is finished by launch_small_rest.
template <int N, class T>
__global__ __launch_bounds__(256, 2) void small_split_kernel(const BondItem* __restrict__ items, JacMat* mats,
                                                          int32_t* rowmap_ws, double* nrm_ws, int m_cap, double eps,
                                                          SelOut* sel, GemmProb* probs, uint32_t* status,
                                                          unsigned long long* stats, DiscLog lg, double tol,
                                                          double abs_tol) {
  __shared__ SmallLds<N> S;
  SmallSel& Z = *(SmallSel*)&S.L;   // the divide and conquer is done by then
  static_assert(sizeof(SmallSel) <= sizeof(DcLds<N>), "the selection fits in the solver's work");
  const int i = blockIdx.x, tid = threadIdx.x;
  const BondItem it = items[i];
  JacMat M;
  M.X = it.X;
  M.rowmap = rowmap_ws + (size_t)i * m_cap;
  M.nrm2 = nrm_ws + (size_t)i * m_cap;
  M.m = it.chi[it.b] * it.d;
  if (!small_class<N>(M.m)) return;
  M.n = it.d * it.chi[it.b + 2];
  M.ld = M.n;
  M.nb = 2;
  M.rot = 0;
  M.kmax = it.chi_max;
  M.pad = 0;
  M.conv = 0;
  M.fro2 = 0.0;
  if (stats && tid == 0) {
    const unsigned long long mm = M.m, nn = M.n;
    atomicAdd(&stats[5], 88ull * mm * nn * (mm < nn ? mm : nn));
  }
  small_gram<N>(M.X, M.m, M.n, M.ld, S.G);
  const int lane = tid & 63;
  M.fro2 = wave_sum(lane < M.m ? S.G[lane * (N + 1) + lane].x : 0.0);   // the same in every wave
  if (tid < M.m) {
    M.nrm2[tid] = S.G[tid * (N + 1) + tid].x;
    M.rowmap[tid] = tid;
  }
  M.conv = (M.fro2 == M.fro2 && M.fro2 < 1e300) ? 0 : 1;
  if (M.conv && tid == 0) atomicOr(status, MPS_DEV_NONFINITE);
  __syncthreads();
  if (!M.conv && M.fro2 > 1e-250 && M.fro2 < 1e250) {
    const bool done = small_rotate<N>(S, M.X, M.m, M.n, M.ld, M.fro2, tol, abs_tol);
    double* const nr = (double*)S.tau;   // the check's diagonal, for the selection
    if (tid < M.m) nr[tid] = M.nrm2[tid] = S.G[tid * (N + 1) + tid].x;
    __syncthreads();
    if (done) {
      M.conv = 1;
      M.pad = 1;
      small_select(Z, nr, M.m, M.kmax, eps);
      small_bond_out<T>(Z, it, M.X, M.m, M.n, M.ld, sel + i, probs + i, lg);
    }
  }
  if (tid == 0) mats[i] = M;
}

// mps_truncate of m <= N rows in one workgroup: theta copied to M.X, then as above.
template <int N>
__global__ __launch_bounds__(256, 2) void small_trunc_kernel(JacMat M, JacMat* mat, TruncOut o, double eps,
                                                          uint32_t* status, double tol, double abs_tol) {
  __shared__ SmallLds<N> S;
  SmallSel& Z = *(SmallSel*)&S.L;
  const int tid = threadIdx.x, lane = tid & 63;
  for (int e = tid; e < M.m * M.n; e += 256) M.X[e] = o.theta[e];
  __syncthreads();
  small_gram<N>(M.X, M.m, M.n, M.ld, S.G);
  M.fro2 = wave_sum(lane < M.m ? S.G[lane * (N + 1) + lane].x : 0.0);
  if (tid < M.m) {
    M.nrm2[tid] = S.G[tid * (N + 1) + tid].x;
    M.rowmap[tid] = tid;
  }
  M.conv = (M.fro2 == M.fro2 && M.fro2 < 1e300) ? 0 : 1;
  if (M.conv && tid == 0) atomicOr(status, MPS_DEV_NONFINITE);
  __syncthreads();
  if (!M.conv && M.fro2 > 1e-250 && M.fro2 < 1e250) {
    const bool done = small_rotate<N>(S, M.X, M.m, M.n, M.ld, M.fro2, tol, abs_tol);
    double* const nr = (double*)S.tau;
    if (tid < M.m) nr[tid] = M.nrm2[tid] = S.G[tid * (N + 1) + tid].x;
    __syncthreads();
    if (done) {
      M.conv = 1;
      M.pad = 1;
      small_select(Z, nr, M.m, M.kmax, eps);
      small_trunc_out(Z, o, M.X, M.m, M.n, M.ld);
    }
  }
  if (tid == 0) *mat = M;
}

}  // namespace

hipError_t launch_eig_small(hipStream_t s, JacMat* mats, int n, int m_cap, const int32_t* list, const int32_t* n_list,
                            int grid, double tol, double abs_tol) {
  if (n <= 0) return hipSuccess;
  small_rotate_kernel<32><<<grid, 256, 0, s>>>(mats, n, list, n_list, tol, abs_tol);
  if (m_cap > 32) small_rotate_kernel<64><<<grid, 256, 0, s>>>(mats, n, list, n_list, tol, abs_tol);
  return hipGetLastError();
}

hipError_t launch_small_split(hipStream_t s, const BondItem* items, JacMat* mats, int n, int m_max, int32_t* rowmap_ws,
                              double* nrm_ws, int m_cap, double eps, SelOut* sel, GemmProb* probs, uint32_t* status,
                              unsigned long long* stats, const DiscLog& lg, bool c128, double tol, double abs_tol) {
  if (n <= 0) return hipSuccess;
  auto go = [&](auto kern) {
    kern<<<n, 256, 0, s>>>(items, mats, rowmap_ws, nrm_ws, m_cap, eps, sel, probs, status, stats, lg, tol, abs_tol);
  };
  go(c128 ? small_split_kernel<32, double2> : small_split_kernel<32, float2>);
  if (m_max > 32) go(c128 ? small_split_kernel<64, double2> : small_split_kernel<64, float2>);
  return hipGetLastError();
}

hipError_t launch_small_trunc(hipStream_t s, const JacMat& M, JacMat* mat, const TruncOut& o, double eps,
                              uint32_t* status, double tol, double abs_tol) {
  if (M.m <= 32) small_trunc_kernel<32><<<1, 256, 0, s>>>(M, mat, o, eps, status, tol, abs_tol);
  else small_trunc_kernel<64><<<1, 256, 0, s>>>(M, mat, o, eps, status, tol, abs_tol);
  return hipGetLastError();
}

size_t eig_slot_bytes(int m_cap, int n_cap) { return EigLayout(m_cap, n_cap).bytes; }

hipError_t launch_eig_rotate(hipStream_t s, JacMat* mats, int n, int m_cap, int n_cap, int m_lim, char* scratch,
                             double tol, double abs_tol, int spin_limit) {
  if (n <= 0) return hipSuccess;
  if (m_cap < 1 || n_cap < 1 || m_cap > kEigMaxDim) return hipErrorInvalidValue;
  EigSlot* slots = (EigSlot*)scratch;
  const size_t head = ((size_t)n * sizeof(EigSlot) + 255) & ~size_t(255);
  const EigLayout L(m_cap, n_cap);
  eig_slots_kernel<<<(n + 63) / 64, 64, 0, s>>>(slots, mats, n, scratch + head, L, m_cap, n_cap, m_lim);
  const int nt = (m_cap + 63) / 64;
  // workgroups per matrix of the kernels that stride over one: a batch sized for
  // capacities may hold hardly any matrix of its own, and empty workgroups cost
  // (240 places of 512 rows, none taken, 0.25 ms a layer without this bound)
  auto rows = [&](int want) { return std::max(1, std::min(want, std::max(8, 8192 / n))); };
  gram_go(s, slots, n, m_cap);
  if (m_cap > 128) eig_fill_kernel<<<dim3(rows(std::min(1024, m_cap * m_cap / 512)), n), 256, 0, s>>>(slots);
  if (m_cap > 2048) {
    tri_sym_kernel<<<dim3(1024, n), 512, 0, s>>>(slots);
    tri_big_kernel<<<n * kTriBigT, 512, 0, s>>>(slots, spin_limit);
  }
  if (m_cap > 1024) tri_kernel<2048, 32><<<n * 256, 512, 0, s>>>(slots, spin_limit);
  if (m_cap > 512) tri_kernel<1024, 32><<<n * 64, 512, 0, s>>>(slots, spin_limit);
  // up to 8 matrices the teams of twice the workgroups are all resident and a
  // step is shorter (m = 512: 3.5 us against 4.7, 256: 2.9 against 3.2); more of
  // them take turns, and the larger share per workgroup wins
  if (m_cap > 256) {
    if (n <= 8) tri_kernel<512, 8><<<n * 64, 512, 0, s>>>(slots, spin_limit);
    else tri_kernel<512, 16><<<n * 32, 512, 0, s>>>(slots, spin_limit);
  }
  if (m_cap > 128) {
    if (n <= 8) tri_kernel<256, 4><<<n * 32, 512, 0, s>>>(slots, spin_limit);
    else tri_kernel<256, 8><<<n * 16, 512, 0, s>>>(slots, spin_limit);
  }
  tri_last_kernel<<<n, 512, 0, s>>>(slots);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dc_leaf_kernel<<<dim3(nt, n), 256, 0, s>>>(slots);
  for (int level = 0; (kLeaf << level) < m_cap; ++level) {
    const int h2 = kLeaf << (level + 1), nblk = (m_cap + h2 - 1) / h2, s_cap = std::min(h2, m_cap);
    const size_t lds_prep = (size_t)3 * s_cap * sizeof(double), lds_vec = (size_t)4 * s_cap * sizeof(double);
    if (lds_vec > 64 * 1024) {
      e = hipFuncSetAttribute((const void*)dc_vec_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_vec);
      if (e != hipSuccess) return e;
    }
    if (lds_prep > 64 * 1024) {
      e = hipFuncSetAttribute((const void*)dc_prep_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_prep);
      if (e != hipSuccess) return e;
    }
    dc_prep_kernel<<<dim3(nblk, n), 256, lds_prep, s>>>(slots, level);
    const int gw = rows((nblk * h2 + 3) / 4);
    dc_root_kernel<<<dim3(gw, n), 256, 0, s>>>(slots, level, nblk);
    dc_zhat_kernel<<<dim3(gw, n), 256, 0, s>>>(slots, level, nblk);
    dc_vec_kernel<<<dim3(gw, n), 256, lds_vec, s>>>(slots, level, nblk, s_cap);
    const int nts = (s_cap + 63) / 64 + 1;   // column tiles of the two halves
    dc_gemm_kernel<<<dim3(nts * nts, nblk, n), 256, 0, s>>>(slots, level, nts);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  wy_t_kernel<<<dim3((m_cap + kWy - 1) / kWy, n), 256, 0, s>>>(slots);
  const int strips = (n_cap + 15) / 16;
  const int wg = (int)xcd_grid(n, strips);
  wy_apply_kernel<1><<<wg, 512, 0, s>>>(slots, 0, 128, n, strips);
  if (m_cap > 128) wy_apply_kernel<2><<<wg, 512, 0, s>>>(slots, 128, 256, n, strips);
  if (m_cap > 256) wy_apply_kernel<4><<<wg, 512, 0, s>>>(slots, 256, 512, n, strips);
  if (m_cap > 512) wy_apply_kernel<8><<<wg, 512, 0, s>>>(slots, 512, 1024, n, strips);
  if (m_cap > 1024) wy_apply_kernel<0><<<wg, 512, 0, s>>>(slots, 1024, 1 << 30, n, strips);
  const int ntn = (2 * n_cap + 63) / 64;
  eig_apply_kernel<<<(int)xcd_grid(n, (long long)nt * ntn), 256, 0, s>>>(slots, n, ntn, nt * ntn);
  gram_go(s, slots, n, m_cap);
  eig_check_kernel<<<dim3(rows(std::min(m_cap, 256)), n), 256, 0, s>>>(slots, mats, tol, abs_tol);
  eig_done_kernel<<<n, 256, 0, s>>>(slots, mats);
  return hipGetLastError();
}

size_t eig_scratch_bytes(int n, int m_cap, int n_cap) {
  return (((size_t)n * sizeof(EigSlot) + 255) & ~size_t(255)) + (size_t)n * eig_slot_bytes(m_cap, n_cap);
}
