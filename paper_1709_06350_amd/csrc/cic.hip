// Density assignment (the paper's footnote in Sec. I allows NGP, CIC or TSC): each particle
// spreads its mass over the 1, 8 or 27 mesh points around it with weights prod_d w_d, mesh points at
// integer coordinates, periodic wrap; then delta = rho / <rho> - 1 with <rho> = np * mass / n^3.
// Per axis, with b = floor(x) and f = x - b: NGP puts weight 1 on the nearest point (b, or b + 1
// when f >= 1/2); CIC puts 1 - f on b and f on b + 1; TSC, with i the NGP point and d = x - i,
// puts (1/2 - d)^2 / 2, 3/4 - d^2, (1/2 + d)^2 / 2 on i - 1, i, i + 1 (the quadratic B-spline).
//
// Accumulation is in unsigned 64-bit fixed point (2^40 units per particle mass): every weight is
// rounded once, the integer sums are exact and independent of the order in which atomics land,
// so the result is bitwise reproducible. Particles are processed in their input order by
// consecutive threads; for lattice-ordered catalogues (as produced by displacing a lattice)
// neighbouring lanes hit neighbouring cells, which keeps the L2 atomics local.
#include <algorithm>
#include <cmath>

#include "mr.h"
#include "mr_ctx.h"
#include "mr_device.h"
#include "mr_kernels.h"

namespace mr {

constexpr double kFixScale = 1099511627776.0;  // 2^40

__device__ __forceinline__ void wrap_coord(double x, int n, int& i0, int& i1, double& f) {
  const double dn = (double)n;
  double xw = x - dn * floor(x / dn);
  if (xw >= dn) xw -= dn;
  if (xw < 0.0) xw = 0.0;
  const double fl = floor(xw);
  i0 = (int)fl;
  if (i0 >= n) i0 = n - 1;
  f = xw - fl;
  i1 = i0 + 1 == n ? 0 : i0 + 1;
}

// The same for the three coordinates of a particle; false if one is not finite. A coordinate of [0, n) is
// its own wrapped value (x / n rounds below 1 there, so the floor is 0) and its own integer part rounded to
// zero: a particle inside the box, as nearly all are, needs no division, floor or finiteness test, which
// were half of the instructions of the counting and sorting passes.
__device__ __forceinline__ bool wrap_particle(double x, double y, double z, int n, int (&i0)[3], int (&i1)[3],
                                              double (&f)[3]) {
  const double dn = (double)n;
  if ((x >= 0.0) & (x < dn) & (y >= 0.0) & (y < dn) & (z >= 0.0) & (z < dn)) {
    const double p[3] = {x, y, z};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      i0[d] = (int)p[d];
      f[d] = p[d] - (double)i0[d];
      i1[d] = i0[d] + 1 == n ? 0 : i0[d] + 1;
    }
    return true;
  }
  if (!__builtin_isfinite(x) || !__builtin_isfinite(y) || !__builtin_isfinite(z)) return false;
  wrap_coord(x, n, i0[0], i1[0], f[0]);
  wrap_coord(y, n, i0[1], i1[1], f[1]);
  wrap_coord(z, n, i0[2], i1[2], f[2]);
  return true;
}

// A weight of [0, 1] in fixed point, rounded to nearest even: w 2^40 + 2^52 is rounded to an integer by the
// one addition, and its low 52 bits are the value (a fused multiply-add and a mask, where the conversion
// of a double to 64 bits takes eight instructions).
__device__ __forceinline__ unsigned long long fix_weight(double w) {
  const double v = __builtin_fma(w, kFixScale, 4503599627370496.0);
  return (unsigned long long)__double_as_longlong(v) & 0xfffffffffffffull;
}

// Per-axis points and weights of one coordinate for a scheme of S points (1 NGP, 2 CIC, 3 TSC).
// i0 = floor of the wrapped coordinate, i1 the point after it, f its fraction (exact).
template <int S>
__device__ __forceinline__ void axis_assign(int i0, int i1, double f, int n, int (&idx)[S], double (&w)[S]) {
  if constexpr (S == 2) {
    idx[0] = i0;
    idx[1] = i1;
    w[0] = 1.0 - f;
    w[1] = f;
  } else {
    const bool up = f >= 0.5;
    const int c = up ? i1 : i0;  // nearest point, a tie goes up
    if constexpr (S == 1) {
      idx[0] = c;
      w[0] = 1.0;
    } else {
      const double d = up ? f - 1.0 : f;  // x - c, exact
      idx[0] = c == 0 ? n - 1 : c - 1;
      idx[1] = c;
      idx[2] = c == n - 1 ? 0 : c + 1;
      const double lo = 0.5 - d, hi = 0.5 + d;
      w[0] = 0.5 * (lo * lo);
      w[1] = 0.75 - d * d;
      w[2] = 0.5 * (hi * hi);
    }
  }
}

// A particle with a non-finite coordinate deposits nothing and adds 1 to *bad_count (relaxed
// atomic: an exact integer count that needs no grid-wide reduction).
template <int S>
__global__ void __launch_bounds__(256) deposit_scatter_kernel(const double* __restrict__ pos, long long np, int n,
                                                              unsigned long long* __restrict__ grid,
                                                              double* __restrict__ bad_count) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < np; p += stride) {
    int i0[3], i1[3];
    double f[3];
    if (!wrap_particle(pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], n, i0, i1, f)) {
      __hip_atomic_fetch_add(bad_count, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      continue;
    }
    int ix[S], iy[S], iz[S];
    double wx[S], wy[S], wz[S];
    axis_assign<S>(i0[0], i1[0], f[0], n, ix, wx);
    axis_assign<S>(i0[1], i1[1], f[1], n, iy, wy);
    axis_assign<S>(i0[2], i1[2], f[2], n, iz, wz);
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < S; ++b) {
        const size_t row = ((size_t)ix[a] * n + iy[b]) * n;
#pragma unroll
        for (int d = 0; d < S; ++d) {
          const double w = wx[a] * wy[b] * wz[d];
          const unsigned long long q = fix_weight(w);
          if (q) atomicAdd(&grid[row + iz[d]], q);
        }
      }
  }
}

// The same deposit with each wave's contributions binned in LDS first. A wave takes 64 consecutive
// particles, finds the bounding box of the mesh points they reach (wrapped base indices, so a wave
// straddling the periodic seam gets a wide box) and, when the box holds at most CAP points,
// accumulates into a private LDS box with LDS atomics and then adds every non-zero box point to the
// grid with one global atomic; otherwise it adds to the grid directly. For lattice-ordered
// catalogues consecutive particles are neighbours, so a box point collects several contributions
// and the global atomics (performed beyond the L2, the bound of the plain scatter) drop by that
// factor. The integer sums per cell are the plain scatter's, so the result is bitwise identical.
__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

// lattice > 0: the catalogue holds lattice^3 particles in lattice order (k fastest) and lattice is a
// multiple of 8; a wave then takes a block of 2 (i) x 4 (j) x 8 (k) particles of the lattice, whose
// assignment points overlap along all three axes, instead of 64 consecutive particles of one row.
// Either way every particle is taken exactly once. (A 4 x 4 x 4 cube needs fewer global adds but
// timed slower, probably from more lanes meeting on the same LDS box entries.)
template <int S, int CAP>
__global__ void __launch_bounds__(256) deposit_scatter_binned_kernel(const double* __restrict__ pos, long long np, int n,
                                                                     unsigned long long* __restrict__ grid,
                                                                     double* __restrict__ bad_count, int lattice) {
  __shared__ unsigned long long boxes[4][CAP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long* box = boxes[w];
  const long long nwaves = (long long)gridDim.x * 4;
  const long long kb_n = lattice / 8, jb_n = lattice / 4;
  for (long long seg = (long long)blockIdx.x * 4 + w; seg * 64 < np; seg += nwaves) {
    long long p = seg * 64 + lane;
    if (lattice > 0) {
      const long long kb = seg % kb_n, jb = (seg / kb_n) % jb_n, ib = seg / (kb_n * jb_n);
      p = ((ib * 2 + (lane >> 5)) * lattice + jb * 4 + ((lane >> 3) & 3)) * lattice + kb * 8 + (lane & 7);
    }
    bool valid = p < np;
    int i0[3], i1[3];
    double f[3];
    if (valid && !wrap_particle(pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], n, i0, i1, f)) {
      __hip_atomic_fetch_add(bad_count, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      valid = false;
    }
    int ix[S], iy[S], iz[S];
    double wx[S], wy[S], wz[S];
    if (valid) {
      axis_assign<S>(i0[0], i1[0], f[0], n, ix, wx);
      axis_assign<S>(i0[1], i1[1], f[1], n, iy, wy);
      axis_assign<S>(i0[2], i1[2], f[2], n, iz, wz);
    }
    // first point per axis before wrapping: ix[0] for CIC and NGP; for TSC ix[0] may have wrapped
    // from -1 to n - 1, which only widens the box (then the wave takes the direct path)
    const int bx = valid ? ix[0] : 0x3fffffff, by = valid ? iy[0] : 0x3fffffff, bz = valid ? iz[0] : 0x3fffffff;
    const int lox = wave_min_i(bx), loy = wave_min_i(by), loz = wave_min_i(bz);
    const int hix = wave_max_i(valid ? bx : -1), hiy = wave_max_i(valid ? by : -1), hiz = wave_max_i(valid ? bz : -1);
    if (hix < 0) continue;  // no valid particle in this segment (wave-uniform)
    const int ex = hix - lox + S, ey = hiy - loy + S, ez = hiz - loz + S;
    const bool binned = (long long)ex * ey * ez <= CAP;  // wave-uniform
    if (binned) {
      const int vol = ex * ey * ez;
      for (int t = lane; t < vol; t += 64) box[t] = 0ull;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (valid) {
#pragma unroll
        for (int a = 0; a < S; ++a)
#pragma unroll
          for (int b = 0; b < S; ++b)
#pragma unroll
            for (int d = 0; d < S; ++d) {
              const double wgt = wx[a] * wy[b] * wz[d];
              const unsigned long long q = fix_weight(wgt);
              // local coordinates from the unwrapped neighbours of the first point
              const int l = ((bx + a - lox) * ey + (by + b - loy)) * ez + (bz + d - loz);
              if (q) atomicAdd(&box[l], q);
            }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (int t = lane; t < vol; t += 64) {
        const unsigned long long v = box[t];
        if (v) {
          const int lz = t % ez, ly = (t / ez) % ey, lx = t / (ez * ey);
          int gx = lox + lx, gy = loy + ly, gz = loz + lz;
          gx -= gx >= n ? n : 0;
          gy -= gy >= n ? n : 0;
          gz -= gz >= n ? n : 0;
          atomicAdd(&grid[((size_t)gx * n + gy) * n + gz], v);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else if (valid) {
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b) {
          const size_t row = ((size_t)ix[a] * n + iy[b]) * n;
#pragma unroll
          for (int d = 0; d < S; ++d) {
            const double wgt = wx[a] * wy[b] * wz[d];
            const unsigned long long q = fix_weight(wgt);
            if (q) atomicAdd(&grid[row + iz[d]], q);
          }
        }
    }
  }
}

// ---- deposit through particles sorted by mesh tile (any particle order) ------------------------
// The mesh is cut into tiles of 16 x 16 x 32 points (4 x 16 x 32 on small meshes). A particle belongs to the tile of the lowest
// mesh point it reaches (the first of its S points per axis, wrapped); its S^3 points then lie in
// the tile's box of (16 + S - 1) x (16 + S - 1) x (32 + S - 1) points. Counting sort of the
// particles by tile: count per (share of particles, tile), exclusive scan, scatter of the
// positions into tile order. One block per tile then accumulates its particles' contributions in
// its box in LDS (64-bit fixed point, the same rounded contribution per particle and point as the
// scatter kernels above, so the integer sums and the result are bitwise those of the scatter) and
// writes the whole box out; a last pass adds to every point of a tile the boxes of the (up to 7)
// lower neighbour tiles that reach it and writes delta. No global atomics: the result does not
// depend on particle order, and the traffic is that of reading the catalogue three times and writing it
// once, which bounds it: 256^3 particles, CIC, 484 to 499 us (604 to 619 with 256-thread blocks on contiguous ranges, a
// division per coordinate and a conversion of eight instructions per weight), of which counting takes 95
// (4.2 TB/s), sorting 155 (5.2 TB/s), accumulating 123 (205 with 8 wavefronts a compute unit, waiting on
// its LDS adds) and combining 71. 96^3 points, 0.88M particles, TSC: 80 us (180), bounded by eight launches.
constexpr int kDepTX = 16, kDepTY = 16, kDepTZ = 32;   // 4 points along x on small meshes
// Threads of the sorting and accumulating launches: two blocks fill a compute unit, except where a TSC box of a
// 16 x 16 x 32 tile takes 88 KB of LDS and one block has it to itself.
constexpr int kDepNT = 1024;
constexpr int kDepMaxBlk = 512;   // particle ranges

struct DepGeom {
  int n, sx, tnx, tny, tnz, ntiles, box;   // tile height 2^sx; points of a tile's box
};

template <int S>
struct DepBox {
  static constexpr int BY = kDepTY + S - 1, BZ = kDepTZ + S - 1;
  static constexpr int cells(int tx) { return (tx + S - 1) * BY * BZ; }
  // Where point z of row r of a box of `rows` rows is stored: the tile's own 32 points of all rows, then the
  // points past it. The tiles above in z read the latter alone, and whole lines of them.
  __device__ static int at(int rows, int r, int z) {
    return z < kDepTZ ? r * kDepTZ + z : rows * kDepTZ + r * (S - 1) + (z - kDepTZ);
  }
};

// The particle's tile and its first mesh point inside the tile (false for a non-finite position).
template <int S>
__device__ __forceinline__ bool dep_place(const double* __restrict__ pos, long long p, const DepGeom& g, int& tile,
                                          int (&ix)[S], int (&iy)[S], int (&iz)[S], double (&wx)[S], double (&wy)[S],
                                          double (&wz)[S]) {
  int i0[3], i1[3];
  double f[3];
  if (!wrap_particle(pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], g.n, i0, i1, f)) return false;
  axis_assign<S>(i0[0], i1[0], f[0], g.n, ix, wx);
  axis_assign<S>(i0[1], i1[1], f[1], g.n, iy, wy);
  axis_assign<S>(i0[2], i1[2], f[2], g.n, iz, wz);
  tile = ((ix[0] >> g.sx) * g.tny + iy[0] / kDepTY) * g.tnz + iz[0] / kDepTZ;
  return true;
}

// A slot for each active lane in its tile's counter. Neighbours in a lattice-ordered catalogue share a tile,
// and LDS atomics on one address take a turn each: the lanes of the first lane's tile, then those of the
// next one's, draw their slots with one atomic; whoever is left (another order) uses its own.
__device__ __forceinline__ unsigned dep_slot(unsigned* __restrict__ count, int tile) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int t = __builtin_amdgcn_readfirstlane(tile);
    if (tile == t) {
      const unsigned long long m = __ballot(1);
      const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      unsigned base = 0u;
      if (below == 0u) base = atomicAdd(&count[t], (unsigned)__popcll(m));
      return __builtin_amdgcn_readfirstlane(base) + below;
    }
  }
  return atomicAdd(&count[tile], 1u);
}

// hist[b][t]: particles of block b's share in tile t: the chunks b, b + nb, .. of kDepNT particles, so that the
// blocks in flight read one contiguous window of the catalogue (ranges of np / nb particles start at
// multiples of a large power of two and meet on the same memory channels).
template <int S>
__global__ void __launch_bounds__(kDepNT) dep_count_kernel(const double* __restrict__ pos, long long np, DepGeom g,
                                                        unsigned* __restrict__ hist,
                                                        double* __restrict__ bad_count) {
  extern __shared__ unsigned dep_lds[];
  for (int t = threadIdx.x; t < g.ntiles; t += blockDim.x) dep_lds[t] = 0u;
  __syncthreads();
  for (long long p = (long long)blockIdx.x * kDepNT + threadIdx.x; p < np; p += (long long)gridDim.x * kDepNT) {
    int tile, ix[S], iy[S], iz[S];
    double wx[S], wy[S], wz[S];
    if (dep_place<S>(pos, p, g, tile, ix, iy, iz, wx, wy, wz))
      (void)dep_slot(dep_lds, tile);
    else
      __hip_atomic_fetch_add(bad_count, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  unsigned* row = hist + (size_t)blockIdx.x * g.ntiles;
  for (int t = threadIdx.x; t < g.ntiles; t += blockDim.x) row[t] = dep_lds[t];
}

// hist[b][t] <- particles of tile t in blocks before b; total[t]. A block takes 16 consecutive tiles and
// splits the rows b into 64 segments, one per thread and tile, whose at most kDepMaxBlk / 64 counts stay in
// registers between the sum and the prefixes: hist is read once, in loads that do not wait for each other.
constexpr int kDepScanT = 16, kDepScanSeg = 64;
__global__ void __launch_bounds__(kDepScanT * kDepScanSeg) dep_scan_blocks_kernel(unsigned* __restrict__ hist, int nblocks,
                                                                                  int ntiles,
                                                                                  unsigned* __restrict__ total) {
  constexpr int PER = kDepMaxBlk / kDepScanSeg;
  __shared__ unsigned seg[kDepScanSeg][kDepScanT];
  const int tl = threadIdx.x % kDepScanT, w = threadIdx.x / kDepScanT;
  const int t = blockIdx.x * kDepScanT + tl;
  const int per = (nblocks + kDepScanSeg - 1) / kDepScanSeg;   // at most PER
  unsigned v[PER];
  unsigned s = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = w * per + k;
    v[k] = k < per && b < nblocks && t < ntiles ? hist[(size_t)b * ntiles + t] : 0u;
    s += v[k];
  }
  seg[w][tl] = s;
  __syncthreads();
  unsigned run = 0u;
  for (int k = 0; k < w; ++k) run += seg[k][tl];
  if (t >= ntiles) return;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = w * per + k;
    if (k < per && b < nblocks) hist[(size_t)b * ntiles + t] = run;
    run += v[k];
  }
  if (w == kDepScanSeg - 1) total[t] = run;
}

// One block of 1024 threads: start[t] = particles of tiles before t, start[ntiles] = all of them.
__global__ void __launch_bounds__(1024) dep_scan_tiles_kernel(const unsigned* __restrict__ total, int ntiles,
                                                              unsigned* __restrict__ start) {
  __shared__ unsigned part[1024];
  const int tid = threadIdx.x;
  const int per = (ntiles + 1023) / 1024;
  const int t0 = tid * per, t1 = min(ntiles, t0 + per);
  unsigned s = 0u;
  for (int t = t0; t < t1; ++t) s += total[t];
  part[tid] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {   // inclusive scan of the per-thread sums
    const unsigned v = tid >= off ? part[tid - off] : 0u;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  unsigned run = tid == 0 ? 0u : part[tid - 1];
  for (int t = t0; t < t1; ++t) {
    start[t] = run;
    run += total[t];
  }
  if (tid == 1023) start[ntiles] = part[1023];
}

// The positions of block b's particles into tile order (the order inside a tile is immaterial).
template <int S>
__global__ void __launch_bounds__(kDepNT) dep_scatter_kernel(const double* __restrict__ pos, long long np, DepGeom g,
                                                          const unsigned* __restrict__ hist,
                                                          const unsigned* __restrict__ start,
                                                          double* __restrict__ sorted) {
  extern __shared__ unsigned dep_lds[];
  const unsigned* row = hist + (size_t)blockIdx.x * g.ntiles;
  for (int t = threadIdx.x; t < g.ntiles; t += blockDim.x) dep_lds[t] = start[t] + row[t];
  __syncthreads();
  // from the end: what the counting pass read last is still in the last-level cache
  const long long step = (long long)gridDim.x * kDepNT;
  const long long rounds = (np + step - 1) / step;
  for (long long p = (rounds - 1) * step + (long long)blockIdx.x * kDepNT + threadIdx.x; p >= 0; p -= step) {
    if (p >= np) continue;
    int tile, ix[S], iy[S], iz[S];
    double wx[S], wy[S], wz[S];
    if (!dep_place<S>(pos, p, g, tile, ix, iy, iz, wx, wy, wz)) continue;
    const unsigned slot = dep_slot(dep_lds, tile);
    double* r = sorted + 3 * (size_t)slot;
    r[0] = pos[3 * p];
    r[1] = pos[3 * p + 1];
    r[2] = pos[3 * p + 2];
  }
}

// One block per tile: the tile's particles into its box (LDS), the box out to boxes[tile].
template <int S>
__global__ void __launch_bounds__(kDepNT) dep_tile_kernel(const double* __restrict__ sorted,
                                                       const unsigned* __restrict__ start, DepGeom g,
                                                       unsigned long long* __restrict__ boxes) {
  using B = DepBox<S>;
  extern __shared__ unsigned long long box[];
  const int t = blockIdx.x;
  for (int c = threadIdx.x; c < g.box; c += blockDim.x) box[c] = 0ull;
  __syncthreads();
  const int tz = t % g.tnz, ty = (t / g.tnz) % g.tny, tx = t / (g.tnz * g.tny);
  const unsigned q0 = start[t], q1 = start[t + 1];
  // a tile starts its share at a place of its own: those of a lattice catalogue are a power of two apart
  const unsigned rounds = (q1 - q0 + kDepNT - 1) / kDepNT;
  unsigned k = rounds ? (unsigned)t % rounds : 0u;
  for (unsigned r = 0; r < rounds; ++r, k = k + 1 == rounds ? 0u : k + 1) {
    const unsigned q = q0 + k * kDepNT + threadIdx.x;
    if (q >= q1) continue;
    int tile, ix[S], iy[S], iz[S];
    double wx[S], wy[S], wz[S];
    (void)dep_place<S>(sorted, (long long)q, g, tile, ix, iy, iz, wx, wy, wz);   // finite by construction
    const int lx = ix[0] - (tx << g.sx), ly = iy[0] - ty * kDepTY, lz = iz[0] - tz * kDepTZ;
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < S; ++b)
#pragma unroll
        for (int d = 0; d < S; ++d) {
          const double w = wx[a] * wy[b] * wz[d];
          const unsigned long long v = fix_weight(w);
          atomicAdd(&box[((lx + a) * B::BY + (ly + b)) * B::BZ + (lz + d)], v);
        }
  }
  __syncthreads();
  unsigned long long* out = boxes + (size_t)t * g.box;
  const int rows = g.box / B::BZ;
  for (int c = threadIdx.x; c < g.box; c += blockDim.x) {
    const int x = c - rows * kDepTZ;   // in stored order: own points first
    const int r = x < 0 ? c / kDepTZ : x / (S - 1), z = x < 0 ? c % kDepTZ : kDepTZ + x % (S - 1);
    out[c] = box[r * B::BZ + z];
  }
}

// `parts` blocks per tile: every point of the tile sums its own box and the lower neighbours' boxes that
// reach it; delta = count n^3 / (np 2^40) - 1; partials[block] = the block's sum of counts / 2^40.
// Writes nothing when a particle had a non-finite position (*bad_count != 0, complete since the
// counting launch): the call then fails and leaves delta unchanged.
template <int S>
__global__ void __launch_bounds__(256) dep_combine_kernel(const unsigned long long* __restrict__ boxes, DepGeom g,
                                                          int parts, double scale, double* __restrict__ delta,
                                                          double* __restrict__ partials, const double* bad_count) {
  using B = DepBox<S>;
  __shared__ double red[16][1];
  const int t = blockIdx.x / parts, part = blockIdx.x - t * parts;
  if (*bad_count != 0.0) {
    if (threadIdx.x == 0) partials[blockIdx.x] = 0.0;
    return;
  }
  const int tz = t % g.tnz, ty = (t / g.tnz) % g.tny, tx = t / (g.tnz * g.tny);
  const int n = g.n, rows = g.box / B::BZ;
  double acc = 0.0;
  const int per = (kDepTY * kDepTZ << g.sx) / parts;
  for (int c = part * per + threadIdx.x; c < (part + 1) * per; c += blockDim.x) {
    const int lz = c % kDepTZ, ly = (c / kDepTZ) % kDepTY, lx = c / (kDepTZ * kDepTY);
    unsigned long long v = 0ull;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int dx = k >> 2, dy = (k >> 1) & 1, dz = k & 1;
      if ((dx && lx >= S - 1) || (dy && ly >= S - 1) || (dz && lz >= S - 1)) continue;
      const int nx = tx - dx < 0 ? g.tnx - 1 : tx - dx;
      const int ny = ty - dy < 0 ? g.tny - 1 : ty - dy;
      const int nz = tz - dz < 0 ? g.tnz - 1 : tz - dz;
      const int nt = (nx * g.tny + ny) * g.tnz + nz;
      v += boxes[(size_t)nt * g.box + B::at(rows, (lx + (dx << g.sx)) * B::BY + (ly + dy * kDepTY), lz + dz * kDepTZ)];
    }
    const size_t cell = ((size_t)((tx << g.sx) + lx) * n + (ty * kDepTY + ly)) * n + (tz * kDepTZ + lz);
    const double cnt = (double)v;
    delta[cell] = cnt * scale - 1.0;
    acc += cnt * (1.0 / kFixScale);
  }
  double vv[1] = {acc};
  block_sum<1>(vv, red, threadIdx.x, blockDim.x);
  if (threadIdx.x == 0) partials[blockIdx.x] = vv[0];
}

// delta = count * n^3 / (np * 2^40) - 1; partials[block] = the block's sum of counts / 2^40. The
// partials are added by sum_partials_kernel in the next launch (fixed order, no per-block fences).
__global__ void __launch_bounds__(256) cic_normalise_kernel(const unsigned long long* __restrict__ grid, size_t cells,
                                                            double scale, double* __restrict__ delta,
                                                            double* __restrict__ partials) {
  __shared__ double red[16][1];
  double acc = 0.0;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < cells; e += (size_t)gridDim.x * blockDim.x) {
    const double cnt = (double)grid[e];
    delta[e] = cnt * scale - 1.0;
    acc += cnt * (1.0 / kFixScale);
  }
  double v[1] = {acc};
  block_sum<1>(v, red, threadIdx.x, blockDim.x);
  if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

// out[0] = sum of partials[0 .. count) in a fixed order (one block).
__global__ void __launch_bounds__(256) sum_partials_kernel(const double* __restrict__ partials, int count,
                                                           double* __restrict__ out) {
  __shared__ double red[16][1];
  double acc = 0.0;
  for (int b = threadIdx.x; b < count; b += blockDim.x) acc += partials[b];
  double v[1] = {acc};
  block_sum<1>(v, red, threadIdx.x, blockDim.x);
  if (threadIdx.x == 0) out[0] = v[0];
}

// Clears the accumulation grid; block 0 also clears the non-finite particle count.
__global__ void __launch_bounds__(256) zero_u64_kernel(unsigned long long* __restrict__ a, size_t cells,
                                                       double* __restrict__ bad_count) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *bad_count = 0.0;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < cells; e += (size_t)gridDim.x * blockDim.x) a[e] = 0ull;
}

static int blocks_for(size_t work, int cap) {
  size_t b = (work + 255) / 256;
  return (int)(b < 1 ? 1 : (b > (size_t)cap ? cap : b));
}

// The tile-sorted deposit (CIC, TSC) on meshes with n a multiple of 32 up to 512.
template <int S>
static int deposit_sorted(Ctx* c, const double* pos, long long np, double* delta_out) {
  const int n = c->n;
  // Tiles of 16 points along x, of 4 where there would be fewer tiles than compute units (below 128^3): the
  // boxes overlap more then, but every unit has one. TSC at 96^3: accumulating 34 us in 108 tiles, 20 in 432.
  const int sx = (n / kDepTX) * (n / kDepTY) * (n / kDepTZ) < 256 ? 2 : 4;
  DepGeom g{n, sx, n >> sx, n / kDepTY, n / kDepTZ, 0, DepBox<S>::cells(1 << sx)};
  g.ntiles = g.tnx * g.tny * g.tnz;
  const size_t cells = (size_t)n * n * n;
  // Particle ranges: as many blocks as the chip holds at once. Longer ranges leave longer runs per tile in the
  // sorted catalogue and fewer counters to scan.
  const int nb = (int)std::min<long long>(kDepMaxBlk, (np + kDepNT - 1) / kDepNT);
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const size_t b_hist = al((size_t)nb * g.ntiles * 4), b_tot = al((size_t)g.ntiles * 4),
               b_start = al(((size_t)g.ntiles + 1) * 4), b_sorted = al((size_t)np * 24),
               b_boxes = al((size_t)g.ntiles * DepBox<3>::cells(1 << sx) * 8);
  const size_t need = b_hist + b_tot + b_start + b_sorted + b_boxes;
  if (c->dep_bytes < need) {
    if (c->dep_mem) (void)hipFree(c->dep_mem);
    c->dep_mem = nullptr;
    c->dep_bytes = 0;
    hipError_t e = hipMalloc(&c->dep_mem, need);
    if (e != hipSuccess) return fail(MR_ENOMEM, "density assignment: %.1f MiB of sort buffers", need / 1048576.0);
    c->dep_bytes = need;
  }
  char* m = (char*)c->dep_mem;
  unsigned* hist = (unsigned*)m;
  unsigned* total = (unsigned*)(m + b_hist);
  unsigned* start = (unsigned*)(m + b_hist + b_tot);
  double* sorted = (double*)(m + b_hist + b_tot + b_start);
  unsigned long long* boxes = (unsigned long long*)(m + b_hist + b_tot + b_start + b_sorted);
  double* bad_count = c->scal + kSlotRes;
  const size_t lds = (size_t)g.ntiles * 4;
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, c->stream, (unsigned long long*)nullptr, (size_t)0, bad_count);
  hipLaunchKernelGGL(dep_count_kernel<S>, dim3(nb), dim3(kDepNT), lds, c->stream, pos, np, g, hist, bad_count);
  hipLaunchKernelGGL(dep_scan_blocks_kernel, dim3((g.ntiles + kDepScanT - 1) / kDepScanT), dim3(kDepScanT * kDepScanSeg), 0, c->stream, hist, nb,
                     g.ntiles, total);
  hipLaunchKernelGGL(dep_scan_tiles_kernel, dim3(1), dim3(1024), 0, c->stream, (const unsigned*)total, g.ntiles, start);
  hipLaunchKernelGGL(dep_scatter_kernel<S>, dim3(nb), dim3(kDepNT), lds, c->stream, pos, np, g, (const unsigned*)hist,
                     (const unsigned*)start, sorted);
  hipLaunchKernelGGL(dep_tile_kernel<S>, dim3(g.ntiles), dim3(kDepNT), (size_t)g.box * 8, c->stream, (const double*)sorted,
                     (const unsigned*)start, g, boxes);
  const double scale = (double)cells / ((double)np * kFixScale);
  // four blocks a tile where tiles are few (TSC at 96^3 31 -> 10 us); at 256^3 they cost more than they
  // give (86 us against 77)
  const int parts = g.ntiles <= 512 ? 4 : 1;
  hipLaunchKernelGGL(dep_combine_kernel<S>, dim3(g.ntiles * parts), dim3(256), 0, c->stream,
                     (const unsigned long long*)boxes, g, parts, scale, delta_out, c->partials, (const double*)bad_count);
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, c->stream, (const double*)c->partials, g.ntiles * parts,
                     c->scal + kSlotRes + 1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mr_deposit");
  double r[2];
  int rc = c->read_scalars(kSlotRes, 2, r);
  if (rc != MR_OK) return rc;
  if (r[0] != 0.0) return fail(MR_EINVAL, "mr_deposit: %.0f particles with non-finite coordinates", r[0]);
  if (!(std::fabs(r[1] - (double)np) <= 0.5 + 1e-9 * (double)np))
    return fail(MR_EINVAL, "mr_deposit: fixed-point overflow (deposited %.6g of %lld particles)", r[1], np);
  return MR_OK;
}

static bool deposit_sorted_applies(int n, long long np) {
  return n % 32 == 0 && n >= 32 && n <= 512 && np < ((long long)1 << 31);
}

int Ctx::deposit(const double* pos, long long np, double mass, int scheme, double* delta_out) {
  const size_t cells = lv[0].cells;
  (void)mass;
  if (!(opts.flags & MR_FLAG_DEPOSIT_SCATTER) && scheme != MR_DEPOSIT_NGP && deposit_sorted_applies(n, np))
    return scheme == MR_DEPOSIT_CIC ? deposit_sorted<2>(this, pos, np, delta_out)
                                    : deposit_sorted<3>(this, pos, np, delta_out);
  if (!cic_grid) {
    hipError_t e = hipMalloc((void**)&cic_grid, cells * sizeof(unsigned long long));
    if (e != hipSuccess) return fail(MR_ENOMEM, "density assignment grid: %s", hipGetErrorString(e));
  }
  double* bad_count = scal + kSlotRes;
  hipLaunchKernelGGL(zero_u64_kernel, dim3(blocks_for(cells, 1 << 16)), dim3(256), 0, stream, cic_grid, cells,
                     bad_count);
  const dim3 pg(blocks_for((size_t)np, 1 << 16));
  // CIC and TSC bin each wave's contributions in LDS (boxes of up to 1024 / 2048 mesh points);
  // NGP has one contribution per particle and little to combine.
  const dim3 wg((unsigned)std::min<long long>((np + 255) / 256, 1 << 16));
  // np = m^3 with m a multiple of 8: let each wave take a 2 x 4 x 8 block of the particle lattice
  long long m = (long long)std::llround(std::cbrt((double)np));
  while (m > 0 && m * m * m > np) --m;
  while ((m + 1) * (m + 1) * (m + 1) <= np) ++m;
  const int lattice = (m * m * m == np && m % 8 == 0 && m <= (1 << 20)) ? (int)m : 0;
  if (scheme == MR_DEPOSIT_NGP)
    hipLaunchKernelGGL(deposit_scatter_kernel<1>, pg, dim3(256), 0, stream, pos, np, n, cic_grid, bad_count);
  else if (scheme == MR_DEPOSIT_CIC)
    hipLaunchKernelGGL((deposit_scatter_binned_kernel<2, 1024>), wg, dim3(256), 0, stream, pos, np, n, cic_grid,
                       bad_count, lattice);
  else
    hipLaunchKernelGGL((deposit_scatter_binned_kernel<3, 2048>), wg, dim3(256), 0, stream, pos, np, n, cic_grid,
                       bad_count, lattice);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mr_deposit");
  double bad;
  int rc = read_scalars(kSlotRes, 1, &bad);
  if (rc != MR_OK) return rc;
  if (bad != 0.0) return fail(MR_EINVAL, "mr_deposit: %.0f particles with non-finite coordinates", bad);
  const double scale = (double)cells / ((double)np * kFixScale);
  const int nb = blocks_for(cells, kMaxReduceBlocks);
  hipLaunchKernelGGL(cic_normalise_kernel, dim3(nb), dim3(256), 0, stream, cic_grid, cells, scale, delta_out, partials);
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, stream, partials, nb, scal + kSlotRes);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mr_deposit");
  double total;
  if ((rc = read_scalars(kSlotRes, 1, &total)) != MR_OK) return rc;
  // Each particle contributes 1 up to 27 roundings of 2^-41; a wrapped 64-bit cell loses 2^24.
  if (!(std::fabs(total - (double)np) <= 0.5 + 1e-9 * (double)np))
    return fail(MR_EINVAL, "mr_deposit: fixed-point overflow (deposited %.6g of %lld particles)", total, np);
  (void)mass;
  return MR_OK;
}

// ---- Lagrangian mapping -----------------------------------------------------------------------
// q = grad Theta = x + grad theta (Theta_0 = |x|^2 / 2, Sec. II; x - q = -grad theta, Sec. III), so
// the displacement is psi = grad theta: the central difference (theta(i+1) - theta(i-1)) / 2 per
// axis on the mesh (cell units), interpolated to each particle with the CIC weights above (the
// transpose of the deposit).

// psi[(i n + j) n + k][a], a = x, y, z; one row (i, j) per block, theta in natural order. The row's
// 3n outputs are assembled in LDS and written with consecutive lanes on consecutive doubles.
constexpr int kLagRowMax = 1024;  // largest mesh a context accepts
// Block 0 also clears the non-finite particle count that the gather that follows accumulates.
__global__ void __launch_bounds__(256) lag_grad_kernel(const double* __restrict__ theta, int n,
                                                       double* __restrict__ psi, double* __restrict__ bad_count) {
  __shared__ double stage[3 * kLagRowMax];
  if (blockIdx.x == 0 && threadIdx.x == 0) *bad_count = 0.0;
  const int row = xcd_remap(blockIdx.x, gridDim.x);
  const int i = row / n, j = row - i * n;
  const int im = i == 0 ? n - 1 : i - 1, ip = i == n - 1 ? 0 : i + 1;
  const int jm = j == 0 ? n - 1 : j - 1, jp = j == n - 1 ? 0 : j + 1;
  const double* __restrict__ r0 = theta + ((size_t)i * n + j) * n;
  const double* __restrict__ rxm = theta + ((size_t)im * n + j) * n;
  const double* __restrict__ rxp = theta + ((size_t)ip * n + j) * n;
  const double* __restrict__ rym = theta + ((size_t)i * n + jm) * n;
  const double* __restrict__ ryp = theta + ((size_t)i * n + jp) * n;
  double* __restrict__ out = psi + ((size_t)i * n + j) * n * 3;
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const int km = k == 0 ? n - 1 : k - 1, kp = k == n - 1 ? 0 : k + 1;
    stage[3 * k + 0] = (rxp[k] - rxm[k]) * 0.5;
    stage[3 * k + 1] = (ryp[k] - rym[k]) * 0.5;
    stage[3 * k + 2] = (r0[kp] - r0[km]) * 0.5;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 3 * n; t += blockDim.x) out[t] = stage[t];
}

// disp[p] = sum over the 8 mesh points around x_p of w * psi (corners in x-major order). A particle
// with a non-finite coordinate is not interpolated (its output is NaN) and adds 1 to *bad_count
// with a relaxed atomic: an exact, order-independent integer count that needs no grid-wide
// reduction (whose per-block release/acquire would write back and invalidate the L2 that the
// concurrently running blocks reuse mesh lines from).
__global__ void __launch_bounds__(256) lag_gather_kernel(const double* __restrict__ pos, long long np, int n,
                                                        const double* __restrict__ psi, double* __restrict__ disp,
                                                        double* __restrict__ bad_count) {
  // consecutive particles on one XCD: lattice-ordered catalogues then reuse mesh lines in its L2
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long p = xcd_remap(blockIdx.x, gridDim.x) * (long long)blockDim.x + threadIdx.x; p < np; p += stride) {
    int i0[3], i1[3];
    double f[3];
    if (!wrap_particle(pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], n, i0, i1, f)) {
      __hip_atomic_fetch_add(bad_count, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      disp[3 * p] = disp[3 * p + 1] = disp[3 * p + 2] = __builtin_nan("");
      continue;
    }
    const int ix0 = i0[0], ix1 = i1[0], iy0 = i0[1], iy1 = i1[1], iz0 = i0[2], iz1 = i1[2];
    const double fx = f[0], fy = f[1], fz = f[2];
    const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
    const int ix[2] = {ix0, ix1}, iy[2] = {iy0, iy1}, iz[2] = {iz0, iz1};
    // all 24 loads are issued before the first use so that their latencies overlap
    double v[8][3];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int a = c >> 2, b = (c >> 1) & 1, d = c & 1;
      const double* __restrict__ src = psi + (((size_t)ix[a] * n + iy[b]) * n + iz[d]) * 3;
      v[c][0] = src[0];
      v[c][1] = src[1];
      v[c][2] = src[2];
    }
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int a = c >> 2, b = (c >> 1) & 1, d = c & 1;
      const double w = wx[a] * wy[b] * wz[d];
      a0 += w * v[c][0];
      a1 += w * v[c][1];
      a2 += w * v[c][2];
    }
    disp[3 * p] = a0;
    disp[3 * p + 1] = a1;
    disp[3 * p + 2] = a2;
  }
}

// Without the mesh field: the central differences of the 8 corners are formed at the particle from
// theta itself (32 values: per (y, z) corner pair the 4 points of the x line, per (x, z) and (x, y)
// pair the 2 outer points of the y and z lines), with the same operations in the same order as
// lag_grad_kernel followed by lag_gather_kernel, so the result is bitwise the same; theta (1/3 of the
// mesh field) is read instead of writing and reading psi.
//
// The values lie in 12 rows along z: the 4 rows of the corners give 4 consecutive points, the 8 rows
// beside them 2. They are read in pairs, 16 loads of 16 bytes; only a particle in the first or one of the
// last two cells of a row needs the single points across the seam. OFF: byte offsets in 32 bits, where
// the mesh has less than 4 GiB, go into the load as they are; 64 bits beyond. 256^3 particles on 256^3:
// 374 us, 2.5 TB/s of compulsory bytes (456 with 32 loads of 8 bytes), so the gathered loads, 16 KB a
// wavefront, bound it and not memory. Slower: blocks of 1024 (402), blocks that stay and fetch the next position (421).
struct __attribute__((packed, aligned(8))) LagPair {
  double a, b;
};

template <class OFF>
__global__ void __launch_bounds__(256) lag_gather_theta_kernel(const double* __restrict__ pos, long long np, int n,
                                                              const double* __restrict__ theta,
                                                              double* __restrict__ disp,
                                                              double* __restrict__ bad_count) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long p = xcd_remap(blockIdx.x, gridDim.x) * (long long)blockDim.x + threadIdx.x; p < np; p += stride) {
    int i0[3], i1[3];
    double f[3];
    if (!wrap_particle(pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], n, i0, i1, f)) {
      __hip_atomic_fetch_add(bad_count, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      disp[3 * p] = disp[3 * p + 1] = disp[3 * p + 2] = __builtin_nan("");
      continue;
    }
    const int xm = i0[0] == 0 ? n - 1 : i0[0] - 1, xp = i1[0] == n - 1 ? 0 : i1[0] + 1;
    const int ym = i0[1] == 0 ? n - 1 : i0[1] - 1, yp = i1[1] == n - 1 ? 0 : i1[1] + 1;
    const int z0 = i0[2];
    const OFF row_b = (OFF)n * 8, plane_b = row_b * (OFF)n;
    const OFF ox[4] = {(OFF)xm * plane_b, (OFF)i0[0] * plane_b, (OFF)i1[0] * plane_b, (OFF)xp * plane_b};
    const OFF oy[4] = {(OFF)ym * row_b, (OFF)i0[1] * row_b, (OFF)i1[1] * row_b, (OFF)yp * row_b};
    const char* __restrict__ base = reinterpret_cast<const char*>(theta);
    auto pair = [&](OFF o) { return *reinterpret_cast<const LagPair*>(base + o); };
    auto one = [&](OFF o) { return *reinterpret_cast<const double*>(base + o); };
    // the pairs that begin at z0 - 1, z0 + 1 and z0, moved inside the row at its ends
    const bool first = z0 == 0, last = z0 == n - 1, before = z0 == n - 2;
    const OFF qa = (OFF)(first ? 0 : z0 - 1) * 8;
    const OFF qb = (OFF)(last ? 0 : (before ? z0 : z0 + 1)) * 8;
    const OFF qs = (OFF)(last ? z0 - 1 : z0) * 8;
    double core[2][2][4];   // [x corner][y corner][z0 - 1 .. z0 + 2]
    double sx[2][2][2];     // [x minus / plus][y corner][z corner]
    double sy[2][2][2];     // [x corner][y minus / plus][z corner]
    LagPair ca[2][2], cb[2][2], px[2][2], py[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        ca[a][b] = pair(ox[a + 1] + oy[b + 1] + qa);
        cb[a][b] = pair(ox[a + 1] + oy[b + 1] + qb);
        px[a][b] = pair(ox[3 * a] + oy[b + 1] + qs);
        py[a][b] = pair(ox[a + 1] + oy[3 * b] + qs);
      }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        core[a][b][0] = ca[a][b].a;
        core[a][b][1] = first ? ca[a][b].a : ca[a][b].b;
        core[a][b][2] = before ? cb[a][b].b : cb[a][b].a;
        core[a][b][3] = cb[a][b].b;
        sx[a][b][0] = last ? px[a][b].b : px[a][b].a;
        sx[a][b][1] = px[a][b].b;
        sy[a][b][0] = last ? py[a][b].b : py[a][b].a;
        sy[a][b][1] = py[a][b].b;
      }
    if (first || before) {
      const OFF q = first ? row_b - 8 : (OFF)0;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const double v = one(ox[a + 1] + oy[b + 1] + q);
          if (first) core[a][b][0] = v;
          if (before) core[a][b][3] = v;
        }
    }
    if (last) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          sx[a][b][1] = one(ox[3 * a] + oy[b + 1]);
          sy[a][b][1] = one(ox[a + 1] + oy[3 * b]);
        }
    }
    const double wx[2] = {1.0 - f[0], f[0]}, wy[2] = {1.0 - f[1], f[1]}, wz[2] = {1.0 - f[2], f[2]};
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int a = c >> 2, b = (c >> 1) & 1, d = c & 1;
      // the x, y and z central differences at corner (a, b, d), as lag_grad_kernel forms them
      const double xlo = a == 0 ? sx[0][b][d] : core[0][b][d + 1], xhi = a == 0 ? core[1][b][d + 1] : sx[1][b][d];
      const double ylo = b == 0 ? sy[a][0][d] : core[a][0][d + 1], yhi = b == 0 ? core[a][1][d + 1] : sy[a][1][d];
      const double w = wx[a] * wy[b] * wz[d];
      a0 += w * ((xhi - xlo) * 0.5);
      a1 += w * ((yhi - ylo) * 0.5);
      a2 += w * ((core[a][b][d + 2] - core[a][b][d]) * 0.5);
    }
    disp[3 * p] = a0;
    disp[3 * p + 1] = a1;
    disp[3 * p + 2] = a2;
  }
}

__global__ void zero_scalar_kernel(double* __restrict__ v) { *v = 0.0; }

int Ctx::lagrangian(const double* theta, const double* pos, long long np, double* disp_out, double* psi_out) {
  double* bad_count = scal + kSlotRes;
  // one particle per thread up to 2^28 particles, a grid-stride loop beyond
  const long long gb = std::min<long long>((np + 255) / 256, 1 << 20);
  if (psi_out) {
    hipLaunchKernelGGL(lag_grad_kernel, dim3((unsigned)n * n), dim3(n < 256 ? (n < 64 ? 64 : n) : 256), 0, stream, theta,
                       n, psi_out, bad_count);
    hipLaunchKernelGGL(lag_gather_kernel, dim3((unsigned)gb), dim3(256), 0, stream, pos, np, n, psi_out, disp_out,
                       bad_count);
  } else {
    hipLaunchKernelGGL(zero_scalar_kernel, dim3(1), dim3(1), 0, stream, bad_count);
    if (lv[0].cells * sizeof(double) <= 0xffffffffull)
      hipLaunchKernelGGL(lag_gather_theta_kernel<unsigned>, dim3((unsigned)gb), dim3(256), 0, stream, pos, np, n, theta,
                         disp_out, bad_count);
    else
      hipLaunchKernelGGL(lag_gather_theta_kernel<size_t>, dim3((unsigned)gb), dim3(256), 0, stream, pos, np, n, theta,
                         disp_out, bad_count);
  }
  hipError_t e = hipGetLastError();
  double bad = 0.0;
  int rc = e == hipSuccess ? read_scalars(kSlotRes, 1, &bad) : hip_fail(e, "mr_lagrangian");
  if (rc != MR_OK) return rc;
  if (bad != 0.0) return fail(MR_EINVAL, "mr_lagrangian: %.0f particles with non-finite coordinates", bad);
  return MR_OK;
}

}  // namespace mr

extern "C" int mr_deposit(mr_ctx* h, const double* pos, int64_t np, double mass, int scheme, double* delta_out) {
  if (!h || !pos || !delta_out) return mr::fail(MR_EINVAL, "mr_deposit: null argument");
  if (np < 1) return mr::fail(MR_EINVAL, "mr_deposit: no particles");
  if (!(mass > 0.0) || !std::isfinite(mass)) return mr::fail(MR_EINVAL, "mr_deposit: mass must be positive");
  if (scheme != MR_DEPOSIT_NGP && scheme != MR_DEPOSIT_CIC && scheme != MR_DEPOSIT_TSC)
    return mr::fail(MR_EINVAL, "mr_deposit: unknown scheme %d", scheme);
  return reinterpret_cast<mr::Ctx*>(h)->deposit(pos, (long long)np, mass, scheme, delta_out);
}

extern "C" int mr_deposit_cic(mr_ctx* h, const double* pos, int64_t np, double mass, double* delta_out) {
  return mr_deposit(h, pos, np, mass, MR_DEPOSIT_CIC, delta_out);
}

extern "C" int mr_lagrangian(mr_ctx* h, const double* theta, const double* pos, int64_t np, double* disp_out,
                             double* psi_out) {
  if (!h || !theta || !pos || !disp_out) return mr::fail(MR_EINVAL, "mr_lagrangian: null argument");
  if (np < 1) return mr::fail(MR_EINVAL, "mr_lagrangian: no particles");
  return reinterpret_cast<mr::Ctx*>(h)->lagrangian(theta, pos, (long long)np, disp_out, psi_out);
}
