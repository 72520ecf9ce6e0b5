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

// u / D where u * D < 2^20 (24-bit multiply).
template <int D>
__device__ __forceinline__ int div_small(int u) {
  if ((D & (D - 1)) == 0) return u / D;
  constexpr unsigned M = (1u << 20) / D + 1;
  return (int)(__umul24((unsigned)u, M) >> 20);
}

// Loads of a whole field (at most 4 GiB) by 32-bit byte offset from scalar registers.
template <typename T>
struct Field {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Field(const T* p, int n) : r(plane_rsrc(p, (unsigned)n * n * n * (unsigned)sizeof(T))) {}
  __device__ __forceinline__ T operator[](unsigned byte_off) const {
    if constexpr (sizeof(T) == 8)
      return ld_rs(r, byte_off);
    else
      return ld_rs_f(r, byte_off);
  }
};

// The planes a thread visits in a box: first, first + G, ...; byte offset of the plane in the mesh.
template <int G>
struct PlaneWalk {
  unsigned gi, n, bytes;
  __device__ __forceinline__ PlaneWalk(int first, int n_, unsigned plane_bytes)
      : gi((unsigned)wrapi(first, n_)), n((unsigned)n_), bytes(plane_bytes) {}
  __device__ __forceinline__ unsigned off() const { return __umul24(gi, bytes); }
  __device__ __forceinline__ void next() {
    const unsigned a = gi + G;
    gi = min(a, a - n);   // one period back where that is not negative
  }
};

// The cells of one local colour in the tile grown by S cells on every side, dealt to NT threads: a thread
// keeps one position (j, m) and takes every G-th plane, so that rows, columns and their periodic images are
// worked out once per stage and a further cell costs some ten instructions (with a division and a 64-bit
// address for every cell, setting up was half of a launch's instructions).
// loc[t] of a thread's cell: position in its colour's half of the box, bit 16 its parity in z, bit 17
// set inside the tile; -1 where there is none.
constexpr int kLocQ = 1 << 16, kLocOwn = 1 << 17, kLocPos = kLocQ - 1;
template <typename T>
struct Same {
  using type = T;   // a parameter that takes its type from the others
};
template <class B, int TI, int TJ, int TK, int OFF, int S, int NT>
struct Stage {
  static constexpr int EI = TI + 2 * S, EJ = TJ + 2 * S, EKH = (TK + 2 * S) / 2;
  static constexpr int POS = EJ * EKH, G = NT / POS;
  static constexpr int N = (EI + G - 1) / G;   // cells per thread
  static constexpr int LO = OFF - S;
  static_assert(G >= 1 && NT <= 1024 && POS < 1024 && B::HALF < kLocQ, "a position per thread, packed positions");
  int loc[N];
  // positions, and add + src of the mesh at them (and src2, when TWO)
  template <bool TWO, typename T>
  __device__ __forceinline__ void init(const B& b, int c, T add, const T* __restrict__ src,
                                       const typename Same<T>::type* __restrict__ src2, T (&v)[N], T (&v2)[N]) {
    const int g = div_small<POS>((int)threadIdx.x), p = (int)threadIdx.x - g * POS;
    const int rj = div_small<EKH>(p), mm = p - rj * EKH;
    const int j = LO + rj, i0 = LO + g;
    const bool own_j = (unsigned)(j - OFF) < (unsigned)TJ;
    const unsigned plane = (unsigned)b.n * (unsigned)b.nh;
    const unsigned row = (unsigned)(c ^ B::RED) * (plane * (unsigned)b.n) + __umul24((unsigned)wrapi(b.j0 + j, b.n), (unsigned)b.nh);
    // the row's cell with the parity of the first plane (0) and with the other one (1): first of that
    // parity at or after LO, 2 mm further
    const int q0 = (i0 + j + c) & 1;
    int pos[2];
    unsigned col[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int q = q0 ^ x;
      const int k = LO + ((LO + q) & 1) + 2 * mm;
      const bool own = own_j && (unsigned)(k - OFF) < (unsigned)TK;
      pos[x] = ((i0 * B::RJ + j) * B::RKH + (k >> 1)) | (q << 16) | (own ? kLocOwn : 0);
      col[x] = (row + ((unsigned)wrapi(b.k0 + k, b.n) >> 1)) * (unsigned)sizeof(T);
    }
    const Field<T> f(src, b.n), f2(TWO ? src2 : src, b.n);
    PlaneWalk<G> w(b.i0 + i0, b.n, plane * (unsigned)sizeof(T));
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const int x = (t * G) & 1;
      const int i = i0 + t * G;
      int e = pos[x] + t * G * B::RJ * B::RKH;
      if (S > 0 && (unsigned)(i - OFF) >= (unsigned)TI) e &= ~kLocOwn;
      const bool in = g < G && ((t + 1) * G <= EI || i < LO + EI);
      loc[t] = in ? e : -1;
      const unsigned o = w.off() + col[x];
      v[t] = add + f[o];
      v2[t] = TWO ? f2[o] : T(0);
      w.next();
    }
  }
};

// Calls f(e, o, i, j, m, q) for every cell of the box this thread loads: position e in the box, byte offset o
// in a mesh of T, row (i, j), column m, parity q in z (k = 2 m + q). Dealt as a stage's cells.
template <typename T, class B, int NT, class F>
__device__ __forceinline__ void for_box(const B& b, F f) {
  constexpr int POS = B::RJ * B::RKH, G = NT / POS, N = (B::RI + G - 1) / G;
  static_assert(G >= 1 && NT <= 1024, "a position per thread");
  const int g = div_small<POS>((int)threadIdx.x), p = (int)threadIdx.x - g * POS;
  const int j = div_small<B::RKH>(p), m = p - j * B::RKH;
  if (g >= G) return;
  const unsigned plane = (unsigned)b.n * (unsigned)b.nh, half = plane * (unsigned)b.n;
  const unsigned row = __umul24((unsigned)wrapi(b.j0 + j, b.n), (unsigned)b.nh);
  const int q0 = (g + j) & 1;   // of local colour 0 in the first plane
  unsigned col[2];              // columns at parity q0 and at the other one
#pragma unroll
  for (int x = 0; x < 2; ++x)
    col[x] = (row + ((unsigned)wrapi(b.k0 + 2 * m + (q0 ^ x), b.n) >> 1)) * (unsigned)sizeof(T);
  PlaneWalk<G> w(b.i0 + g, b.n, plane * (unsigned)sizeof(T));
  const int e0 = (g * B::RJ + j) * B::RKH + m;
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const int i = g + t * G;
    if ((t + 1) * G > B::RI && i >= B::RI) break;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int x = (t * G + c) & 1;
      f(c * B::HALF + e0 + t * G * B::RJ * B::RKH, w.off() + col[x] + (unsigned)(c ^ B::RED) * half * (unsigned)sizeof(T), i,
        j, m, q0 ^ x);
    }
    w.next();
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
