// Boxes of cells in LDS for the kernels that run several relaxations of a small mesh in one launch
// (block_cycle.hip, adj_block.hip), device code.
#pragma once

#include "mr_device.h"

namespace mr {

// Box of T + 2 OFF cells per axis around a TI x TJ x TK tile, colour-split in LDS: [c][i][j][m] with
// local colour c = (i + j + k) & 1 of the local coordinates and m = k >> 1. Tile origins are even, so
// the mesh's red cells have the local colour OFF & 1.
template <int TI, int TJ, int TK, int OFF>
struct Box {
  static constexpr int RI = TI + 2 * OFF, RJ = TJ + 2 * OFF, RKH = (TK + 2 * OFF) / 2;
  static constexpr int HALF = RI * RJ * RKH;
  static constexpr int RED = OFF & 1;
  int i0, j0, k0, n, nh;   // mesh coordinates of local (0, 0, 0), mesh size

  __device__ __forceinline__ void init(int logical, int n_) {
    n = n_;
    nh = n >> 1;
    const int tk = n / TK, tj = n / TJ;
    const int a = logical % tk, r = logical / tk;
    k0 = a * TK - OFF;
    j0 = (r % tj) * TJ - OFF;
    i0 = (r / tj) * TI - OFF;
  }
  // colour-split index in the mesh of local cell (i, j, k) of local colour c
  __device__ __forceinline__ unsigned mesh(int c, int i, int j, int k) const {
    const int gi = wrapi(i0 + i, n), gj = wrapi(j0 + j, n), gk = wrapi(k0 + k, n);
    return (unsigned)(c ^ RED) * ((unsigned)n * n * nh) + ((unsigned)gi * n + gj) * (unsigned)nh + (unsigned)(gk >> 1);
  }
  // 18 neighbours of the cell at position e of its colour's half (at[own colour], at[other colour]),
  // q its parity in z
  template <typename T, typename Nb>
  static __device__ __forceinline__ void gather(const T* __restrict__ own, const T* __restrict__ other, int e, int q,
                                                Nb& t) {
    constexpr int DI = RJ * RKH, DJ = RKH;
    const T* __restrict__ o = other + e;
    const T* __restrict__ s = own + e;
    const T* __restrict__ oq = o + q;   // column of k + 1; the one before it is that of k - 1
    const T* __restrict__ sq = s + q;
    t.xm = o[-DI]; t.xp = o[DI];
    t.ym = o[-DJ]; t.yp = o[DJ];
    t.zm = oq[-1]; t.zp = oq[0];
    t.xpyp = s[DI + DJ]; t.xmym = s[-DI - DJ];
    t.xpym = s[DI - DJ]; t.xmyp = s[-DI + DJ];
    t.xpzp = sq[DI];     t.xmzm = sq[-DI - 1];
    t.xpzm = sq[DI - 1]; t.xmzp = sq[-DI];
    t.ypzp = sq[DJ];     t.ymzm = sq[-DJ - 1];
    t.ypzm = sq[DJ - 1]; t.ymzp = sq[-DJ];
  }
};

// u / D for 0 <= u < 2^13, 2 <= D < 32 (24-bit multiply; exact while u * D < 2^20).
template <int D>
__device__ __forceinline__ int div_small(int u) {
  if ((D & (D - 1)) == 0) return u / D;
  constexpr unsigned M = (1u << 20) / D + 1;
  return (int)(__umul24((unsigned)u, M) >> 20);
}

// The cells of one local colour in the tile grown by S cells on every side, dealt to NT threads.
// loc[t] of a thread's cell: position in its colour's half of the box, bit 16 its parity in z, bit 17
// set inside the tile; -1 past the end. Worked out once per launch: formed again at every use the
// divisions were a third of the half-sweeps' instructions.
constexpr int kLocQ = 1 << 16, kLocOwn = 1 << 17, kLocPos = kLocQ - 1;
template <typename T>
struct Same {
  using type = T;   // a parameter that takes its type from the others
};
template <class B, int TI, int TJ, int TK, int OFF, int S, int NT>
struct Stage {
  static constexpr int EI = TI + 2 * S, EJ = TJ + 2 * S, EKH = (TK + 2 * S) / 2;
  static constexpr int CELLS = EI * EJ * EKH;
  static constexpr int N = (CELLS + NT - 1) / NT;   // cells per thread
  static constexpr int LO = OFF - S;
  static_assert(N * NT < 8192 && B::HALF < kLocQ, "packed positions");
  int loc[N];
  // positions, and add + src of the mesh at them (and src2, when TWO)
  template <bool TWO, typename T>
  __device__ __forceinline__ void init(const B& b, int c, T add, const T* __restrict__ src,
                                       const typename Same<T>::type* __restrict__ src2, T (&v)[N], T (&v2)[N]) {
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const int u = (int)threadIdx.x + t * NT;
      const int r = div_small<EKH>(u), ri = div_small<EJ>(r);
      const int i = LO + ri, j = LO + r - ri * EJ;
      const int q = (i + j + c) & 1;                            // parity of the row's cells of this colour
      const int k = LO + ((LO + q) & 1) + 2 * (u - r * EKH);    // first cell of that parity at or after LO
      const bool in = CELLS % NT == 0 || u < CELLS;
      const bool own = (unsigned)(i - OFF) < (unsigned)TI && (unsigned)(j - OFF) < (unsigned)TJ &&
                       (unsigned)(k - OFF) < (unsigned)TK;
      loc[t] = in ? ((i * B::RJ + j) * B::RKH + (k >> 1)) | (q ? kLocQ : 0) | (own ? kLocOwn : 0) : -1;
      v[t] = add;
      v2[t] = T(0);
      if (in) {
        const unsigned g = b.mesh(c, i, j, k);
        v[t] = add + src[g];
        if (TWO) v2[t] = src2[g];
      }
    }
  }
};

// Calls f(e, c, i, j, m, q) for every cell of the box this thread loads: position e in the box, local
// colour c, row (i, j), column m, parity q in z (k = 2 m + q).
template <class B, int NT, class F>
__device__ __forceinline__ void for_box(F f) {
  constexpr int NL = (2 * B::HALF + NT - 1) / NT;
#pragma unroll
  for (int t = 0; t < NL; ++t) {
    const int e = (int)threadIdx.x + t * NT;
    if (e < 2 * B::HALF) {
      const int c = e >= B::HALF ? 1 : 0, r = e - c * B::HALF;
      const int ij = div_small<B::RKH>(r), m = r - ij * B::RKH;
      const int i = div_small<B::RJ>(ij), j = ij - i * B::RJ;
      f(e, c, i, j, m, (i + j + c) & 1);
    }
  }
}

// Sum of count values, in a fixed order, to every thread of the block.
template <int NT>
__device__ __forceinline__ double block_total(const double* __restrict__ p, int count, double (*red)[1]) {
  double v[1] = {0.0};
  for (int b = threadIdx.x; b < count; b += NT) v[0] += p[b];
  v[0] = wave_sum_full(v[0]);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = v[0];
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) s += red[w][0];
  __syncthreads();
  return s;
}

// Orders LDS accesses of the lanes of one wavefront (WAVE) or of the block.
template <bool WAVE>
__device__ __forceinline__ void tail_sync() {
  if (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

}  // namespace mr
