// 64x64 complex output tile on MFMA, one 256-thread workgroup = 4 waves,
// each wave a 32x32 quarter made of 2x2 16x16 MFMA tiles.  Two precisions:
//   complex64  : v_mfma_f32_16x16x4f32, FP32 accumulation
//   complex128 : v_mfma_f64_16x16x4f64, FP64 accumulation
// A complex product is four real products:
//   C_re += A_re B_re - A_im B_im,   C_im += A_re B_im + A_im B_re.
// Operands are staged in LDS as As[k][row] and Bs[k][col], a K-chunk of 16 at
// a time.  Lane layout of the 16x16x4 instructions (both precisions): lane l
// supplies A[l%16][l/16] and B[l/16][l%16].  Accumulator entry r of lane l is
// C[4*(l/16)+r][l%16] for f32 but C[l/16+4r][l%16] for f64 (measured on
// gfx950 with an in-bounds probe); acc_row() gives the row.
#pragma once
#include "common.h"

#define TBM 64
#define TBN 64
#define TBK 16
#define TLD 68   // LDS row pitch (complex elements) of the staged operands

typedef double doublex4 __attribute__((ext_vector_type(4)));

template <class T>
struct Cx;
template <>
struct Cx<float2> {
  typedef float R;
  typedef floatx4 V4;
  static __device__ __forceinline__ V4 mfma(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float2 make(double re, double im) { return make_float2((float)re, (float)im); }
  static __device__ __forceinline__ int acc_row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <>
struct Cx<double2> {
  typedef double R;
  typedef doublex4 V4;
  static __device__ __forceinline__ V4 mfma(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ double2 make(double re, double im) { return make_double2(re, im); }
  static __device__ __forceinline__ int acc_row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

// ---------------------------------------------------------------------------
// Tile shapes for the tuned GEMMs: 2 x 2 waves, each wave MI x NJ MFMA tiles
// of 16 x 16, so a workgroup tile is (32 MI) x (32 NJ); MI = NJ = 2 is the
// 64 x 64 tile above.
// ---------------------------------------------------------------------------
template <class T, int MI, int NJ>
struct AccTileT {
  typename Cx<T>::V4 re[MI][NJ];
  typename Cx<T>::V4 im[MI][NJ];
};

template <class T, int MI, int NJ>
__device__ __forceinline__ void acc_zero_t(AccTileT<T, MI, NJ>& a) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        a.re[i][j][r] = 0;
        a.im[i][j][r] = 0;
      }
}

// One staged K-chunk: As[TBK][lda] (rows of the tile), Bs[TBK][ldb] (columns).
template <class T, int MI, int NJ>
__device__ __forceinline__ void mma_chunk_t(const T* __restrict__ As, int lda, const T* __restrict__ Bs, int ldb,
                                            AccTileT<T, MI, NJ>& acc, int wm, int wn, int lane) {
#pragma unroll
  for (int kk = 0; kk < TBK / 4; ++kk) {
    const int kr = kk * 4 + (lane >> 4);
    T a[MI], b[NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = As[kr * lda + wm + i * 16 + (lane & 15)];
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[j] = Bs[kr * ldb + wn + j * 16 + (lane & 15)];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        acc.re[i][j] = Cx<T>::mfma(a[i].x, b[j].x, acc.re[i][j]);
        acc.re[i][j] = Cx<T>::mfma(-a[i].y, b[j].y, acc.re[i][j]);
        acc.im[i][j] = Cx<T>::mfma(a[i].x, b[j].y, acc.im[i][j]);
        acc.im[i][j] = Cx<T>::mfma(a[i].y, b[j].x, acc.im[i][j]);
      }
  }
}

// One operand's chunks of TBK x W elements (W rows of A or columns of B) on
// their way to LDS: thread t holds W / 16 of them, the lanes along whichever
// index is the nearer in memory, so a load touches whole lines; the odd LDS
// pitch W + 1 keeps the stores of either order free of bank conflicts.  (Four
// neighbours a thread, at a pitch of W + 4, touched four times the lines and
// lost a fifth of the time to conflicts.)
template <class T, int W>
struct SgOperand {
  static constexpr int E = W / 16, LD = W + 1;
  const T* base;        // the operand, for elements that are not there
  const T* p;           // this thread's first element of the next chunk
  long long ps, ks;     // to its next element; to the next chunk
  int x0, k0, dx, dk;   // its first element's place in the tile, and the steps to the next
  int left;             // rows (columns) of the tile that are there
  int l0, dl;           // LDS place and step
  __device__ __forceinline__ SgOperand(const T* q, long long xs, long long cs, int n0, int n) : base(q) {
    const int tid = threadIdx.x;
    const bool along_k = cs <= xs;
    x0 = along_k ? tid >> 4 : tid & (W - 1);
    k0 = along_k ? tid & 15 : tid / W;
    dx = along_k ? 16 : 0;
    dk = along_k ? 0 : 256 / W;
    left = n - n0;
    p = q + (long long)(n0 + x0) * xs + (long long)k0 * cs;
    ps = dx * xs + dk * cs;
    ks = TBK * cs;
    l0 = k0 * LD + x0;
    dl = dk * LD + dx;
  }
  // the next chunk, kl columns (rows of B) of which are there
  __device__ __forceinline__ void load(T (&d)[E], int kl) {
    if (left >= W && kl >= TBK) {
#pragma unroll
      for (int e = 0; e < E; ++e) d[e] = p[e * ps];
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const bool on = x0 + e * dx < left && k0 + e * dk < kl;
        const T x = *(on ? p + e * ps : base);
        d[e].x = on ? x.x : 0;
        d[e].y = on ? x.y : 0;
      }
    }
    p += ks;
  }
  __device__ __forceinline__ void store(T* lds, const T (&d)[E], typename Cx<T>::R im) const {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      T x = d[e];
      x.y *= im;
      lds[l0 + e * dl] = x;
    }
  }
};

// Tile (m0, n0) of A B^dag, both row-major (A: ma rows, B: mb rows, K columns,
// complex128), 32 MI x 32 MI, by 256 threads; the next chunk is loaded while
// the staged one is multiplied.  A product with fewer tiles than CUs is bound by
// the FP64 MFMA of the CUs that it reaches (64 cycles an instruction: a 64 x 64
// tile takes 1.7 us per chunk of 16 columns), so it is cut into tiles of 32 x 32
// (0.4 us); the order of a sum does not depend on the tile.
template <int MI>
struct DaggerLds {
  double2 a[2][TBK * (32 * MI + 1)], b[2][TBK * (32 * MI + 1)];
};
template <int MI>
__device__ __forceinline__ void dagger_tile(const double2* __restrict__ A, size_t lda, int ma,
                                            const double2* __restrict__ B, size_t ldb, int mb, int K, int m0, int n0,
                                            DaggerLds<MI>& L, AccTileT<double2, MI, MI>& acc) {
  constexpr int BM = 32 * MI, LD = BM + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BM / 2);
  SgOperand<double2, BM> oa(A, (long long)lda, 1, m0, ma), ob(B, (long long)ldb, 1, n0, mb);
  double2 ra[BM / 16], rb[BM / 16];
  acc_zero_t<double2, MI, MI>(acc);
  oa.load(ra, K);
  ob.load(rb, K);
  oa.store(L.a[0], ra, 1.0);
  ob.store(L.b[0], rb, -1.0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < K; k0 += TBK) {
    const bool more = k0 + TBK < K;
    if (more) {
      oa.load(ra, K - k0 - TBK);
      ob.load(rb, K - k0 - TBK);
    }
    mma_chunk_t<double2, MI, MI>(L.a[buf], LD, L.b[buf], LD, acc, wm, wn, lane);
    if (more) {
      oa.store(L.a[buf ^ 1], ra, 1.0);
      ob.store(L.b[buf ^ 1], rb, -1.0);
    }
    __syncthreads();
    buf ^= 1;
  }
}
// Calls out(row, column, value) for the entries of the tile at (m0, n0).
template <int MI, class Out>
__device__ __forceinline__ void dagger_out(const AccTileT<double2, MI, MI>& acc, int m0, int n0, const Out& out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * (16 * MI), wn = (wave & 1) * (16 * MI);
#pragma unroll
  for (int a = 0; a < MI; ++a)
#pragma unroll
    for (int b = 0; b < MI; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out(m0 + wm + a * 16 + Cx<double2>::acc_row(lane, r), n0 + wn + b * 16 + (lane & 15),
            make_double2(acc.re[a][b][r], acc.im[a][b][r]));
}
// 1 when tiles64 tiles of 64 x 64 leave CUs idle, else 2
inline int dagger_mi(long long tiles64) { return tiles64 < 256 ? 1 : 2; }

// The tile shapes the GEMM autotuner chooses from: (MI, NJ) of candidate c.
constexpr int kGemmCands = 6;
__host__ __device__ constexpr int gemm_cand_mi(int c) { return c == 1 ? 4 : (c == 3 || c == 5) ? 1 : 2; }
__host__ __device__ constexpr int gemm_cand_nj(int c) { return c == 2 ? 4 : (c == 4 || c == 5) ? 1 : 2; }
