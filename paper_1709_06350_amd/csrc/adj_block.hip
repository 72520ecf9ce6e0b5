// The adjoint's V-cycle on its small meshes, FP64: one launch down, one launch up per level, and one
// workgroup for the levels of 12^3 cells and below, as block_cycle.hip does for the FAS cycle.
//
// A half-sweep of these levels took 7 to 12 us and a level's cycle some fifteen launches and clears
// (937 launches in a forward and backward pass at 64^3, whose gaps left the chip idle 40% of the
// time). A block holds the lambda of its tile and halo in LDS and runs two red-black sweeps with the
// residual and restriction (down, from lambda = 0 below the finest level: the first red half-sweep is
// then -h^2 rhs / 6 and the first black one needs only the face terms), or the prolongation and two
// sweeps (up). The six coefficient fields are read from memory where they are used: a box of them
// would not fit, and they come from the caches.
// lambda is kept mean-free as in adjoint.hip: each launch subtracts the mean of its input (block sums
// of the launch before); between its own two sweeps it does not, which moves the iterates by a
// multiple of a constant that the next launch takes out, with the same fixed point.
#include "adj_block.h"
#include "block_box.h"
#include "block_cycle.h"
#include "mr_kernels.h"

namespace mr {

// Coefficient values around mesh cell (gi, gj, gk): fac the face terms' (A_x at i -+ 1, A_y at j -+ 1,
// A_z at k -+ 1), edg the cross terms' (W_xy, W_xz, W_yz at ++, --, +-, -+).
struct AdjCoef {
  double fac[6], edg[12];
};

template <bool EDGES>
__device__ __forceinline__ void load_adj_coef(const double* __restrict__ coef, int n, int gi, int gj, int gk, AdjCoef& c) {
  const unsigned nh = (unsigned)n >> 1, half = (unsigned)n * n * nh, cells = 2 * half;
  const unsigned col = (unsigned)(gi + gj + gk) & 1, own = col * half, oth = half - own;
  const unsigned pi = (unsigned)n * nh;
  const unsigned i0 = gi * pi, im = (gi == 0 ? n - 1 : gi - 1) * pi, ip = (gi == n - 1 ? 0 : gi + 1) * pi;
  const unsigned j0 = gj * nh, jm = (gj == 0 ? n - 1 : gj - 1) * nh, jp = (gj == n - 1 ? 0 : gj + 1) * nh;
  const unsigned m = (unsigned)gk >> 1, q = gk & 1;
  const unsigned sp = q ? (m + 1 == nh ? 0 : m + 1) : m;   // column of k + 1
  const unsigned sm = q ? m : (m == 0 ? nh - 1 : m - 1);   // column of k - 1
  const double* __restrict__ ax = coef + oth;
  c.fac[0] = ax[im + j0 + m];
  c.fac[1] = ax[ip + j0 + m];
  c.fac[2] = ax[cells + i0 + jm + m];
  c.fac[3] = ax[cells + i0 + jp + m];
  c.fac[4] = ax[2 * cells + i0 + j0 + sm];
  c.fac[5] = ax[2 * cells + i0 + j0 + sp];
  if (EDGES) {
    const double* __restrict__ w = coef + 3 * (size_t)cells + own;
    c.edg[0] = w[ip + jp + m];
    c.edg[1] = w[im + jm + m];
    c.edg[2] = w[ip + jm + m];
    c.edg[3] = w[im + jp + m];
    const double* __restrict__ wz = w + cells;
    c.edg[4] = wz[ip + j0 + sp];
    c.edg[5] = wz[im + j0 + sm];
    c.edg[6] = wz[ip + j0 + sm];
    c.edg[7] = wz[im + j0 + sp];
    const double* __restrict__ wy = wz + cells;
    c.edg[8] = wy[i0 + jp + sp];
    c.edg[9] = wy[i0 + jm + sm];
    c.edg[10] = wy[i0 + jp + sm];
    c.edg[11] = wy[i0 + jm + sp];
  }
}

// h^2 (J^T l)_c + 6 l_c from the neighbours' lambda t.
template <bool EDGES>
__device__ __forceinline__ double adj_off(const AdjCoef& c, const Nb18& t) {
  const double off = (c.fac[0] * t.xm + c.fac[1] * t.xp) + (c.fac[2] * t.ym + c.fac[3] * t.yp) +
                     (c.fac[4] * t.zm + c.fac[5] * t.zp);
  if (!EDGES) return off;
  const double dxy = (c.edg[0] * t.xpyp + c.edg[1] * t.xmym) - (c.edg[2] * t.xpym + c.edg[3] * t.xmyp);
  const double dxz = (c.edg[4] * t.xpzp + c.edg[5] * t.xmzm) - (c.edg[6] * t.xpzm + c.edg[7] * t.xmzp);
  const double dyz = (c.edg[8] * t.ypzp + c.edg[9] * t.ymzm) - (c.edg[10] * t.ypzm + c.edg[11] * t.ymzp);
  return off - 0.5 * ((dxy + dxz) + dyz);
}

// Local (i, j, k) of position e of a box's colour half with parity q.
template <class B>
__device__ __forceinline__ void box_coords(int e, int q, int& i, int& j, int& k) {
  const int r = div_small<B::RKH>(e);
  i = div_small<B::RJ>(r);
  j = r - i * B::RJ;
  k = 2 * (e - r * B::RKH) + q;
}

// New values of local colour c on a stage; EDGES false where the own colour's lambda is zero. Adds the
// new values of the tile's own cells to acc.
template <class B, bool EDGES, bool SUM, class St>
__device__ __forceinline__ void adj_half_box(const B& b, const St& st, double* __restrict__ lam, int c,
                                             const double (&rhs)[St::N], const double* __restrict__ coef, double h2,
                                             double& acc) {
  double nv[St::N];
  double* __restrict__ own = lam + c * B::HALF;
  const double* __restrict__ other = lam + (c ^ 1) * B::HALF;
#pragma unroll
  for (int t = 0; t < St::N; ++t) {
    nv[t] = 0.0;
    if (st.loc[t] >= 0) {
      const int e = st.loc[t] & kLocPos, q = (st.loc[t] >> 16) & 1;
      int i, j, k;
      box_coords<B>(e, q, i, j, k);
      AdjCoef cf;
      load_adj_coef<EDGES>(coef, b.n, wrapi(b.i0 + i, b.n), wrapi(b.j0 + j, b.n), wrapi(b.k0 + k, b.n), cf);
      Nb18 g;
      B::gather(own, other, e, q, g);
      nv[t] = (adj_off<EDGES>(cf, g) - h2 * rhs[t]) * (1.0 / 6.0);
      if (SUM && (st.loc[t] & kLocOwn)) acc += nv[t];
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < St::N; ++t)
    if (st.loc[t] >= 0) own[st.loc[t] & kLocPos] = nv[t];
  __syncthreads();
}

template <int TI, int TJ, int TK, int NT, bool ZERO>
__global__ void __launch_bounds__(NT) adj_down_kernel(AdjDownArgs a) {
  constexpr int OFF = ZERO ? 4 : 5;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 4, NT> s4;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  constexpr int R = B::RED, K = R ^ 1;
  __shared__ double lam[2 * B::HALF];
  __shared__ double red[16][2];
  B b;
  b.init(xcd_remap(blockIdx.x, gridDim.x), a.n);
  const int tid = threadIdx.x;
  double r4[s4.N], r3[s3.N], r2[s2.N], r1[s1.N], x4[s4.N], x3[s3.N], x2[s2.N], x1[s1.N];
  s4.template init<false>(b, R, 0.0, a.rhs, nullptr, r4, x4);
  s3.template init<false>(b, K, 0.0, a.rhs, nullptr, r3, x3);
  s2.template init<false>(b, R, 0.0, a.rhs, nullptr, r2, x2);
  s1.template init<false>(b, K, 0.0, a.rhs, nullptr, r1, x1);
  const double h2 = a.h2;
  double acc = 0.0;
  if (ZERO) {
#pragma unroll
    for (int t = 0; t < s4.N; ++t)
      if (s4.loc[t] >= 0) lam[R * B::HALF + (s4.loc[t] & kLocPos)] = -h2 * r4[t] * (1.0 / 6.0);
    __syncthreads();
    adj_half_box<B, false, false>(b, s3, lam, K, r3, a.coef, h2, acc);
  } else {
    const double mu = block_total<NT>(a.mu.part, a.mu.count, reinterpret_cast<double(*)[1]>(red)) * a.mu.scale;
    const Field<double> lam_in(a.lam, a.n);
    for_box<double, B, NT>(b, [&](int e, unsigned o, int i, int j, int m, int q) { lam[e] = lam_in[o] - mu; });
    __syncthreads();
    adj_half_box<B, true, false>(b, s4, lam, R, r4, a.coef, h2, acc);
    adj_half_box<B, true, false>(b, s3, lam, K, r3, a.coef, h2, acc);
  }
  adj_half_box<B, true, true>(b, s2, lam, R, r2, a.coef, h2, acc);
  adj_half_box<B, true, true>(b, s1, lam, K, r1, a.coef, h2, acc);

  // residual of the tile, eight sons of a coarse cell on eight consecutive threads
  constexpr int TILE = TI * TJ * TK;
  static_assert(TILE <= NT && TILE % 64 == 0, "one cell of the tile per thread");
  const int son = tid & 7, cc = tid >> 3;
  const int cK = cc % (TK / 2), cJ = (cc / (TK / 2)) % (TJ / 2), cI = cc / (TK / 2 * (TJ / 2));
  const int di = OFF + 2 * cI + (son >> 2), dj = OFF + 2 * cJ + ((son >> 1) & 1), dk = OFF + 2 * cK + (son & 1);
  const int dc = (di + dj + dk) & 1;
  const bool own = tid < TILE;
  double r = 0.0;
  if (own) {
    const int e = (di * B::RJ + dj) * B::RKH + (dk >> 1);
    AdjCoef cf;
    load_adj_coef<true>(a.coef, a.n, b.i0 + di, b.j0 + dj, b.k0 + dk, cf);
    Nb18 g;
    B::gather(lam + dc * B::HALF, lam + (dc ^ 1) * B::HALF, e, dk & 1, g);
    r = a.rhs[b.mesh(dc, di, dj, dk)] - (adj_off<true>(cf, g) - 6.0 * lam[dc * B::HALF + e]) / h2;
  }
  double sr = r;
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) sr += __shfl_xor(sr, x, 64);
  if (own && son == 0) {
    const int nc = a.n >> 1;
    a.rhs_c[split_idx(nc, ((b.i0 + OFF) >> 1) + cI, ((b.j0 + OFF) >> 1) + cJ, ((b.k0 + OFF) >> 1) + cK)] = 0.125 * sr;
  }
  if (own) {
    constexpr int TKH = TK / 2;
    const int m = tid % TKH, q = tid / TKH;
    const int c = q / (TI * TJ), ij = q - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    a.lam_out[b.mesh(c, i, j, k)] = lam[c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1)];
  }
  double v[2] = {acc, r * r};
  block_sum<2>(v, red, tid, NT);
  if (tid == 0) {
    a.part_s[blockIdx.x] = v[0];
    a.part_r2[blockIdx.x] = v[1];
  }
}

template <int TI, int TJ, int TK, int NT>
__global__ void __launch_bounds__(NT) adj_up_kernel(AdjUpArgs a) {
  constexpr int OFF = 4;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  Stage<B, TI, TJ, TK, OFF, 0, NT> s0;
  constexpr int R = B::RED, K = R ^ 1;
  constexpr int QI = B::RI / 2 + 2, QJ = B::RJ / 2 + 2, QK = B::RKH + 2, NQ = QI * QJ * QK;
  __shared__ double lam[2 * B::HALF];
  __shared__ double ec[NQ];
  __shared__ double red[16][1];
  B b;
  b.init(xcd_remap(blockIdx.x, gridDim.x), a.n);
  const int tid = threadIdx.x;
  const int nc = a.n >> 1;
  for (int e = tid; e < NQ; e += NT) {
    const int r = div_small<QK>(e), k = e - r * QK;
    const int i = div_small<QJ>(r), j = r - i * QJ;
    ec[e] = a.lam_c[split_idx(nc, wrapi((b.i0 >> 1) - 1 + i, nc), wrapi((b.j0 >> 1) - 1 + j, nc),
                              wrapi((b.k0 >> 1) - 1 + k, nc))];
  }
  double r3[s3.N], r2[s2.N], r1[s1.N], r0[s0.N], x3[s3.N], x2[s2.N], x1[s1.N], x0[s0.N];
  s3.template init<false>(b, R, 0.0, a.rhs, nullptr, r3, x3);
  s2.template init<false>(b, K, 0.0, a.rhs, nullptr, r2, x2);
  s1.template init<false>(b, R, 0.0, a.rhs, nullptr, r1, x1);
  s0.template init<false>(b, K, 0.0, a.rhs, nullptr, r0, x0);
  // the weights of the interpolation add up to one, so both offsets are one constant
  const double mu = block_total<NT>(a.mu.part, a.mu.count, red) * a.mu.scale +
                    block_total<NT>(a.mu_c.part, a.mu_c.count, red) * a.mu_c.scale;   // ends in a barrier: ec is complete
  const Field<double> lam_in(a.lam, a.n);
  for_box<double, B, NT>(b, [&](int e, unsigned o, int i, int j, int m, int q) {
    const double* __restrict__ p = ec + ((i >> 1) + 1) * (QJ * QK) + ((j >> 1) + 1) * QK + m + 1;
    const int ni = (i & 1) ? QJ * QK : -QJ * QK, nj = (j & 1) ? QK : -QK, nk = q ? 1 : -1;
    auto row = [&](int s) { return 0.75 * p[s] + 0.25 * p[s + nk]; };
    const double corr = 0.75 * (0.75 * row(0) + 0.25 * row(nj)) + 0.25 * (0.75 * row(ni) + 0.25 * row(ni + nj));
    lam[e] = lam_in[o] + (corr - mu);
  });
  __syncthreads();
  double acc = 0.0;
  adj_half_box<B, true, false>(b, s3, lam, R, r3, a.coef, a.h2, acc);
  adj_half_box<B, true, false>(b, s2, lam, K, r2, a.coef, a.h2, acc);
  adj_half_box<B, true, true>(b, s1, lam, R, r1, a.coef, a.h2, acc);
  adj_half_box<B, true, true>(b, s0, lam, K, r0, a.coef, a.h2, acc);
  constexpr int TILE = TI * TJ * TK, TKH = TK / 2;
  for (int x = tid; x < TILE; x += NT) {
    const int m = x % TKH, q = x / TKH;
    const int c = q / (TI * TJ), ij = q - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    a.lam_out[b.mesh(c, i, j, k)] = lam[c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1)];
  }
  double v[1] = {acc};
  block_sum<1>(v, red, tid, NT);
  if (tid == 0) a.part_s[blockIdx.x] = v[0];
}

// ---- levels of 12^3 cells and below: one workgroup --------------------------------------------
// 8^3 or 12^3 with its coarsest 4^3 or 6^3, or a coarsest 10^3 alone, from lambda = 0. lambda is in LDS
// with a one-cell periodic halo, rhs in the registers of the cell's owner, the coefficients in LDS (the
// smaller meshes) or read from memory (12^3). The mean is taken out after every sweep (as an offset
// that the next reads subtract). The coarsest mesh is swept by one wavefront.
template <int N, bool WAVE, int W>
struct AdjTailLevel {
  using B = Box<N, N, N, 1>;
  static constexpr int HALF = N * N * N / 2, PER = (HALF + W - 1) / W;
  static constexpr int DI = B::RJ * B::RKH, DJ = B::RKH;
  double* lam;
  const double* coef;   // six fields of n^3, in memory or in LDS
  double h2;
  double mu;            // offset of both colours
  int u[PER];
  bool has[PER];
  double rhs[2][PER];

  __device__ __forceinline__ static void coords(int u, int& i, int& j, int& m) {
    m = u % (N / 2);
    const int r = u / (N / 2);
    j = r % N;
    i = r / N;
  }
  __device__ __forceinline__ void init(double* lds, const double* cf, double h2_) {
    lam = lds;
    coef = cf;
    h2 = h2_;
    mu = 0.0;
    const int lane = WAVE ? (threadIdx.x & 63) : threadIdx.x;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      has[p] = HALF % W == 0 || lane + p * W < HALF;
      u[p] = has[p] ? lane + p * W : 0;
    }
  }
  __device__ __forceinline__ double* half(int c) const { return lam + (c ^ B::RED) * B::HALF; }
  __device__ __forceinline__ static int pos(int i, int j, int k) { return ((i + 1) * B::RJ + j + 1) * B::RKH + ((k + 1) >> 1); }
  __device__ __forceinline__ double get(int c, int p) const {
    int i, j, m;
    coords(u[p], i, j, m);
    return half(c)[pos(i, j, 2 * m + ((i + j + c) & 1))];
  }
  __device__ __forceinline__ void put(int c, int p, double v) const {
    int i, j, m;
    coords(u[p], i, j, m);
    const int k = 2 * m + ((i + j + c) & 1);
    const int oi = i == 0 ? N * DI : (i == N - 1 ? -N * DI : 0), oj = j == 0 ? N * DJ : (j == N - 1 ? -N * DJ : 0),
              ok = k == 0 ? N / 2 : (k == N - 1 ? -N / 2 : 0);
    double* a = half(c) + pos(i, j, k);
    a[0] = v;
    if (ok) a[ok] = v;
    if (oj) {
      a[oj] = v;
      if (ok) a[oj + ok] = v;
    }
    if (oi) {
      a[oi] = v;
      if (ok) a[oi + ok] = v;
      if (oj) a[oi + oj] = v;
    }
  }
  // off-diagonal part at this thread's cell p of colour c; the offset mo of the other colour's stored
  // values and ms of its own are taken out
  __device__ __forceinline__ double off(int c, int p, double mo, double ms) const {
    int i, j, m;
    coords(u[p], i, j, m);
    const int k = 2 * m + ((i + j + c) & 1);
    AdjCoef cf;
    load_adj_coef<true>(coef, N, i, j, k, cf);
    Nb18 t;
    B::gather(half(c), half(c ^ 1), pos(i, j, k), (k + 1) & 1, t);
    t.xm -= mo; t.xp -= mo; t.ym -= mo; t.yp -= mo; t.zm -= mo; t.zp -= mo;
    t.xpyp -= ms; t.xmym -= ms; t.xpym -= ms; t.xmyp -= ms; t.xpzp -= ms; t.xmzm -= ms;
    t.xpzm -= ms; t.xmzp -= ms; t.ypzp -= ms; t.ymzm -= ms; t.ypzm -= ms; t.ymzp -= ms;
    return adj_off<true>(cf, t);
  }
  __device__ __forceinline__ void sweeps(int count, double (*red)[1]) {
    for (int s = 0; s < count; ++s) {
      double acc = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double nv[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) nv[p] = (off(c, p, c == 0 ? mu : 0.0, mu) - h2 * rhs[c][p]) * (1.0 / 6.0);
        tail_sync<WAVE>();
#pragma unroll
        for (int p = 0; p < PER; ++p)
          if (has[p]) {
            put(c, p, nv[p]);
            acc += nv[p];
          }
        tail_sync<WAVE>();
      }
      mu = total(acc, red) * (1.0 / (2.0 * HALF));
    }
  }
  __device__ __forceinline__ double total(double v, double (*red)[1]) const {
    v = wave_sum_full(v);
    if (WAVE) return v;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W / 64; ++w) s += red[w][0];
    __syncthreads();
    return s;
  }
};

template <int NA, int NB, int NT>
__global__ void __launch_bounds__(NT) adj_tail_kernel(AdjTailArgs a) {
  constexpr bool LDSA = NA <= 8;
  using LA = AdjTailLevel<NA, false, NT>;
  using LB = AdjTailLevel<NB == 0 ? 4 : NB, true, 64>;
  constexpr int CA = NA * NA * NA, CB = NB == 0 ? 1 : NB * NB * NB;
  __shared__ double lamA[2 * LA::B::HALF], rA[NB == 0 ? 1 : CA], cA[LDSA ? 6 * CA : 1];
  __shared__ double lamB[2 * LB::B::HALF], cB[6 * CB], ec[NB == 0 ? 1 : (NB + 2) * (NB + 2) * (NB + 2)];
  __shared__ double red[16][1];
  const int tid = threadIdx.x;
  for (int e = tid; e < 2 * LA::B::HALF; e += NT) lamA[e] = 0.0;
  if (LDSA)
    for (int e = tid; e < 6 * CA; e += NT) cA[e] = a.coef[e];
  if (NB != 0) {
    for (int e = tid; e < 6 * CB; e += NT) cB[e] = a.coef_c[e];
    for (int e = tid; e < 2 * LB::B::HALF; e += NT) lamB[e] = 0.0;
  }
  LA A;
  A.init(lamA, LDSA ? cA : a.coef, a.h2);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < LA::PER; ++p) A.rhs[c][p] = a.rhs[c * LA::HALF + A.u[p]];
  __syncthreads();
  if (NB == 0) {
    A.sweeps(a.ncoarse, red);
  } else {
    A.sweeps(a.npre, red);
    const double ih2 = 1.0 / a.h2;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < LA::PER; ++p)
        if (A.has[p])
          rA[c * LA::HALF + A.u[p]] = A.rhs[c][p] - (A.off(c, p, A.mu, A.mu) - 6.0 * (A.get(c, p) - A.mu)) * ih2;
    __syncthreads();
    if (tid < 64) {
      LB Bl;
      Bl.init(lamB, cB, 4.0 * a.h2);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p) {
          int I, J, M;
          LB::coords(Bl.u[p], I, J, M);
          const int K = 2 * M + ((I + J + c) & 1);
          double sr = 0.0;
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const int i = 2 * I + (x >> 2), j = 2 * J + ((x >> 1) & 1), k = 2 * K + (x & 1);
            sr += rA[((i + j + k) & 1) * LA::HALF + (i * NA + j) * (NA / 2) + (k >> 1)];
          }
          Bl.rhs[c][p] = 0.125 * sr;
        }
      Bl.sweeps(a.ncoarse, red);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p)
          if (Bl.has[p]) {
            int I, J, M;
            LB::coords(Bl.u[p], I, J, M);
            const int K = 2 * M + ((I + J + c) & 1);
            const double v = Bl.get(c, p) - Bl.mu;
            const int oi = I == 0 ? NB : (I == NB - 1 ? -NB : 0), oj = J == 0 ? NB : (J == NB - 1 ? -NB : 0),
                      ok = K == 0 ? NB : (K == NB - 1 ? -NB : 0);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
              if (((x & 4) && !oi) || ((x & 2) && !oj) || ((x & 1) && !ok)) continue;
              ec[((I + 1 + ((x & 4) ? oi : 0)) * (NB + 2) + J + 1 + ((x & 2) ? oj : 0)) * (NB + 2) + K + 1 +
                 ((x & 1) ? ok : 0)] = v;
            }
          }
    }
    __syncthreads();
    // the offset mu of the first level's lambda stays: its next sweep takes it out
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < LA::PER; ++p)
        if (A.has[p]) {
          int i, j, m;
          LA::coords(A.u[p], i, j, m);
          const int q = (i + j + c) & 1;
          const double* __restrict__ x = ec + (((i >> 1) + 1) * (NB + 2) + (j >> 1) + 1) * (NB + 2) + m + 1;
          const int ni = ((i & 1) ? 1 : -1) * (NB + 2) * (NB + 2), nj = ((j & 1) ? 1 : -1) * (NB + 2), nk = q ? 1 : -1;
          auto row = [&](int s) { return 0.75 * x[s] + 0.25 * x[s + nk]; };
          A.put(c, p, A.get(c, p) + 0.75 * (0.75 * row(0) + 0.25 * row(nj)) + 0.25 * (0.75 * row(ni) + 0.25 * row(ni + nj)));
        }
    __syncthreads();
    A.sweeps(a.npost, red);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < LA::PER; ++p)
      if (A.has[p]) a.lam_out[c * LA::HALF + A.u[p]] = A.get(c, p) - A.mu;
}

// ---- launchers ----------------------------------------------------------------------------

#define MR_AB_TILES(X) X(4, 4, 4, 512) X(4, 4, 8, 512) X(4, 8, 8, 512) X(8, 8, 8, 512) X(8, 8, 16, 1024)

hipError_t launch_adj_down(const AdjDownArgs& a, hipStream_t s) {
  if (!blk_level_supported(a.n)) return hipErrorInvalidValue;
  const BlkTile t = blk_tile(a.n);
#define MR_AB_GO(TI, TJ, TK, NT)                                                                                  \
  if (t.ti == TI && t.tj == TJ && t.tk == TK) {                                                                   \
    if (a.lam)                                                                                                    \
      hipLaunchKernelGGL((adj_down_kernel<TI, TJ, TK, NT, false>), dim3(blk_blocks(a.n)), dim3(NT), 0, s, a);     \
    else                                                                                                          \
      hipLaunchKernelGGL((adj_down_kernel<TI, TJ, TK, NT, true>), dim3(blk_blocks(a.n)), dim3(NT), 0, s, a);      \
    return hipGetLastError();                                                                                     \
  }
  MR_AB_TILES(MR_AB_GO)
#undef MR_AB_GO
  return hipErrorInvalidValue;
}

hipError_t launch_adj_up(const AdjUpArgs& a, hipStream_t s) {
  if (!blk_level_supported(a.n)) return hipErrorInvalidValue;
  const BlkTile t = blk_tile(a.n);
#define MR_AB_GO(TI, TJ, TK, NT)                                                                       \
  if (t.ti == TI && t.tj == TJ && t.tk == TK) {                                                        \
    hipLaunchKernelGGL((adj_up_kernel<TI, TJ, TK, NT>), dim3(blk_blocks(a.n)), dim3(NT), 0, s, a);     \
    return hipGetLastError();                                                                          \
  }
  MR_AB_TILES(MR_AB_GO)
#undef MR_AB_GO
  return hipErrorInvalidValue;
}

hipError_t launch_adj_tail(const AdjTailArgs& a, hipStream_t s) {
  if (a.n == 8)
    hipLaunchKernelGGL((adj_tail_kernel<8, 4, 256>), dim3(1), dim3(256), 0, s, a);
  else if (a.n == 12)
    hipLaunchKernelGGL((adj_tail_kernel<12, 6, 896>), dim3(1), dim3(896), 0, s, a);
  else if (a.n == 10)
    hipLaunchKernelGGL((adj_tail_kernel<10, 0, 512>), dim3(1), dim3(512), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mr
