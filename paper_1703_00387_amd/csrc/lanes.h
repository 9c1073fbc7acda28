// Moves between the lanes of a wave that do not go through the LDS unit: DPP
// within 16 lanes (a few cycles each, where a permute through the LDS unit takes
// its round trip), row swaps between them.
#pragma once
#include <hip/hip_runtime.h>

template <int CTRL>
__device__ __forceinline__ int dpp_i(int a) {
  return __builtin_amdgcn_update_dpp(0, a, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double a) {
  return __hiloint2double(dpp_i<CTRL>(__double2hiint(a)), dpp_i<CTRL>(__double2loint(a)));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140, kRor4 = 0x124, kRor8 = 0x128,
              kWaveShl1 = 0x130, kWaveShr1 = 0x138;   // from lane i + 1, from lane i - 1 (0 past the end)


// Sum over a wave's lanes of NV values each (a power of two, at most 64),
// halved level by level: at each a lane keeps half of its values and gets the
// other lane's part of them.  Across 32 and 16 lanes by swapping rows (the two
// halves end up side by side: two moves and one addition for two values), below
// by DPP.  Value i of wave w goes to red[w * NV + i] for after the caller's barrier.
template <int B>
__device__ __forceinline__ double lane_xor(double a) {   // the value of lane ^ (1 << B), B < 4
  return B == 0 ? dpp_d<kXor1>(a) : B == 1 ? dpp_d<kXor2>(a) : B == 2 ? dpp_d<0x1B>(dpp_d<kHalfMirror>(a)) : dpp_d<kRor8>(a);
}
template <bool ROWS32>
__device__ __forceinline__ double swap_add(double a, double b) {   // lower rows: sum of a; upper rows: of b
  const unsigned al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  const auto l = ROWS32 ? __builtin_amdgcn_permlane32_swap(al, bl, false, false)
                        : __builtin_amdgcn_permlane16_swap(al, bl, false, false);
  const auto h = ROWS32 ? __builtin_amdgcn_permlane32_swap(ah, bh, false, false)
                        : __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
template <int NV, int B>
__device__ __forceinline__ void wave_sums_low(double* v, int lane, int& idx) {
  constexpr int H = NV >> (6 - B);   // values kept at this level (lane bit B)
  if constexpr (H > 0) {
    const bool up = (lane >> B) & 1;
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const double lo = v[u], hi = v[u + H];
      v[u] = (up ? hi : lo) + lane_xor<B>(up ? lo : hi);
    }
    idx += up ? H : 0;
  } else {
    v[0] += lane_xor<B>(v[0]);
  }
}
template <int NV>
__device__ __forceinline__ void wave_sums(double* v, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int idx = 0;
  if constexpr (NV >= 2) {
#pragma unroll
    for (int u = 0; u < NV / 2; ++u) v[u] = swap_add<true>(v[u], v[u + NV / 2]);
    idx += lane & 32 ? NV / 2 : 0;
  } else {
    v[0] = swap_add<true>(v[0], v[0]);
  }
  if constexpr (NV >= 4) {
#pragma unroll
    for (int u = 0; u < NV / 4; ++u) v[u] = swap_add<false>(v[u], v[u + NV / 4]);
    idx += lane & 16 ? NV / 4 : 0;
  } else {
    v[0] = swap_add<false>(v[0], v[0]);
  }
  wave_sums_low<NV, 3>(v, lane, idx);
  wave_sums_low<NV, 2>(v, lane, idx);
  wave_sums_low<NV, 1>(v, lane, idx);
  wave_sums_low<NV, 0>(v, lane, idx);
  if ((lane & (64 / NV - 1)) == 0) red[wave * NV + idx] = v[0];
}
