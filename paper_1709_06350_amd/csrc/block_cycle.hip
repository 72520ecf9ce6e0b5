// The FAS cycle on its small meshes, FP64 (Sec. II.A.2-3): one launch down, one launch up per level,
// and one workgroup for the levels of 12^3 cells and below.
//
// What bounds these meshes is latency, not data: 32^3 cells are 256 KB, yet a sweep took 14 us and a
// level's cycle ten launches, because a block marched its planes one after the other (a root's
// dependency chain and a barrier per plane) and every launch waited for the one before. Here a block
// owns a TI x TJ x TK box of cells and holds the box with a halo in LDS; it computes the halo cells
// that its own cells need over two red-black sweeps redundantly (each half-sweep needs one cell less
// on every side), so that a whole pre-smoothing with its defect and restriction, or a whole
// prolongation with its post-smoothing, needs no exchange between blocks:
//   down: f = nabla^2 th - Sigma - rd on the halo (levels below the finest), red, black, red, black,
//         defect, 8-son means of theta and of the defect;
//   up:   theta + P(theta_c - theta_hat_c), red, black, red, black.
// The arithmetic per cell is that of the sweeps in sweep.hip. The uniform shift C = <Sigma + f> is
// taken once per launch from the block sums of the launch before on that level (the other sweeps
// refresh it every sweep); it moves the iterates by a constant and, through its lag, by a multiple
// of the change of <Sigma> between two cycles, and has the same fixed point. Block sums go to plain
// partial arrays that the next launch adds in a fixed order: no arrival counters.
#include "block_box.h"
#include "block_cycle.h"
#include "mr_ctx.h"
#include "mr_device.h"
#include "mr_kernels.h"

namespace mr {

// One half-sweep on a stage: new values of local colour c from the box in LDS, written back after
// every thread has read. opd: 1 + delta of this thread's cells; f: their right-hand side, from LDS
// (kLdsF) or registers (kRegF). Adds Sigma + f of the tile's own cells to acc.
enum { kNoF = 0, kLdsF = 1, kRegF = 2 };
template <class B, class St, int FMODE, bool SUM>
__device__ __forceinline__ void half_sweep_box(const St& st, double* __restrict__ th, int c, const double (&opd)[St::N],
                                               const double* __restrict__ fl, const double (&fr)[St::N], double h2,
                                               double ih2, double C, double& acc) {
  double nv[St::N];
  double* __restrict__ own = th + c * B::HALF;
  const double* __restrict__ other = th + (c ^ 1) * B::HALF;
#pragma unroll
  for (int t = 0; t < St::N; ++t) {
    nv[t] = 0.0;
    if (st.loc[t] >= 0) {
      const int e = st.loc[t] & kLocPos;
      Nb18 g;
      B::gather(own, other, e, (st.loc[t] >> 16) & 1, g);
      double S;
      const double sig = sigma_cell(g, opd[t], ih2, S);
      const double fc = FMODE == kLdsF ? fl[c * B::HALF + e] : (FMODE == kRegF ? fr[t] : 0.0);
      nv[t] = (S - h2 * (sig + fc - C)) * (1.0 / 6.0);
      if (SUM && (st.loc[t] & kLocOwn)) acc += sig + fc;
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < St::N; ++t)
    if (st.loc[t] >= 0) own[st.loc[t] & kLocPos] = nv[t];
  __syncthreads();
}

template <int TI, int TJ, int TK, int NT, bool TAU>
__global__ void __launch_bounds__(NT) blk_down_kernel(BlkDownArgs a) {
  constexpr int OFF = 5;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 4, NT> s4;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  constexpr int R = B::RED, K = R ^ 1;   // local colours of red and black
  __shared__ double th[2 * B::HALF];
  __shared__ double fl[TAU ? 2 * B::HALF : 1];
  __shared__ double red[16][3];
  B b;
  b.init(xcd_remap(blockIdx.x, gridDim.x), a.n);
  const int tid = threadIdx.x;

  // every global load of the launch is issued here: theta of the box, delta of each stage's cells,
  // the partial sums of the shift
  const Field<double> theta(a.theta, a.n);
  for_box<double, B, NT>(b, [&](int e, unsigned o, int i, int j, int m, int q) { th[e] = theta[o]; });
  double d4[s4.N], d3[s3.N], d2[s2.N], d1[s1.N], r4[s4.N], r3[s3.N], r2[s2.N], r1[s1.N];
  s4.template init<TAU>(b, R, 1.0, a.delta, a.rd, d4, r4);
  s3.template init<TAU>(b, K, 1.0, a.delta, a.rd, d3, r3);
  s2.template init<false>(b, R, 1.0, a.delta, nullptr, d2, r2);
  s1.template init<false>(b, K, 1.0, a.delta, nullptr, d1, r1);
  // the tile's cells for the defect: eight sons of a coarse cell on eight consecutive threads
  constexpr int TILE = TI * TJ * TK;
  static_assert(TILE <= NT && TILE % 64 == 0, "one cell of the tile per thread");
  const int son = tid & 7, cc = tid >> 3;
  const int cK = cc % (TK / 2), cJ = (cc / (TK / 2)) % (TJ / 2), cI = cc / (TK / 2 * (TJ / 2));
  const int di = OFF + 2 * cI + (son >> 2), dj = OFF + 2 * cJ + ((son >> 1) & 1), dk = OFF + 2 * cK + (son & 1);
  const int dc = (di + dj + dk) & 1;
  const bool own = tid < TILE;
  const double dd = own ? 1.0 + a.delta[b.mesh(dc, di, dj, dk)] : 1.0;
  const double C = block_total<NT>(a.c_part, a.c_count, reinterpret_cast<double(*)[1]>(red)) * a.c_scale;
  const double h2 = a.h2, ih2 = a.ih2;
  if (TAU) {
    // right-hand side of the cells that the first red and the first black half-sweep update
    auto tau = [&](const auto& st, int c, const auto& de, const auto& rd) {
#pragma unroll
      for (int t = 0; t < st.N; ++t) {
        if (st.loc[t] >= 0) {
          const int e = st.loc[t] & kLocPos;
          Nb18 g;
          B::gather(th + c * B::HALF, th + (c ^ 1) * B::HALF, e, (st.loc[t] >> 16) & 1, g);
          double S;
          const double sig = sigma_cell(g, de[t], ih2, S);
          fl[c * B::HALF + e] = (S - 6.0 * th[c * B::HALF + e]) * ih2 - sig - rd[t];
        }
      }
    };
    tau(s4, R, d4, r4);
    tau(s3, K, d3, r3);
    __syncthreads();
  }
  constexpr int FM = TAU ? kLdsF : kNoF;
  double acc = 0.0;
  half_sweep_box<B, decltype(s4), FM, false>(s4, th, R, d4, fl, r4, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s3), FM, false>(s3, th, K, d3, fl, r3, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s2), FM, true>(s2, th, R, d2, fl, r2, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s1), FM, true>(s1, th, K, d1, fl, r1, h2, ih2, C, acc);

  // defect of the tile, 8-son means, smoothed theta and right-hand side out
  double d = 0.0, tc = 0.0;
  if (own) {
    const int e = (di * B::RJ + dj) * B::RKH + (dk >> 1);
    Nb18 g;
    B::gather(th + dc * B::HALF, th + (dc ^ 1) * B::HALF, e, dk & 1, g);
    double S;
    const double sig = sigma_cell(g, dd, ih2, S);
    tc = th[dc * B::HALF + e];
    d = (S - 6.0 * tc) * ih2 - sig - (TAU ? fl[dc * B::HALF + e] : 0.0) + C;
  }
  double sd = d, st = tc;
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) {
    sd += __shfl_xor(sd, x, 64);
    st += __shfl_xor(st, x, 64);
  }
  if (own && son == 0) {
    const int nc = a.n >> 1, nch = nc >> 1;
    const int I = ((b.i0 + OFF) >> 1) + cI, J = ((b.j0 + OFF) >> 1) + cJ, Kc = ((b.k0 + OFF) >> 1) + cK;
    const unsigned g = (unsigned)((I + J + Kc) & 1) * ((unsigned)nc * nc * nch) + ((unsigned)I * nc + J) * (unsigned)nch +
                       (unsigned)(Kc >> 1);
    a.theta_c[g] = 0.125 * st;
    a.rd_c[g] = 0.125 * sd;
  }
  if (own) {
    // tile cells in mesh order: both colours of a row segment
    constexpr int TKH = TK / 2;
    const int m = tid % TKH, r = tid / TKH;
    const int c = r / (TI * TJ), ij = r - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    const unsigned g = b.mesh(c, i, j, k);
    const int e = c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1);
    a.theta_out[g] = th[e];
    if (TAU) a.f_out[g] = fl[e];
  }
  double v[3] = {acc, d, d * d};
  block_sum<3>(v, red, tid, NT);
  if (tid == 0) {
    a.part_c[blockIdx.x] = v[0];
    a.part_d[blockIdx.x] = v[1];
    a.part_d2[blockIdx.x] = v[2];
    if (blockIdx.x == 0 && a.c_out) *a.c_out = C;
  }
}

template <int TI, int TJ, int TK, int NT, bool HAS_F>
__global__ void __launch_bounds__(NT) blk_up_kernel(BlkUpArgs a) {
  constexpr int OFF = 4;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  Stage<B, TI, TJ, TK, OFF, 0, NT> s0;
  constexpr int R = B::RED, K = R ^ 1;
  // coarse corrections around the box: parents of the box and one cell more on every side
  constexpr int QI = B::RI / 2 + 2, QJ = B::RJ / 2 + 2, QK = B::RKH + 2, NQ = QI * QJ * QK;
  __shared__ double th[2 * B::HALF];
  __shared__ double ec[NQ];
  __shared__ double red[16][1];
  B b;
  b.init(xcd_remap(blockIdx.x, gridDim.x), a.n);
  const int tid = threadIdx.x;
  const int nc = a.n >> 1;
  for (int e = tid; e < NQ; e += NT) {
    const int r = div_small<QK>(e), k = e - r * QK;
    const int i = div_small<QJ>(r), j = r - i * QJ;
    // local origin of the box is even: parent of local 0 is (origin >> 1)
    const unsigned g = split_idx(nc, wrapi((b.i0 >> 1) - 1 + i, nc), wrapi((b.j0 >> 1) - 1 + j, nc),
                                 wrapi((b.k0 >> 1) - 1 + k, nc));
    ec[e] = a.theta_c[g] - a.that_c[g];
  }
  double d3[s3.N], d2[s2.N], d1[s1.N], d0[s0.N], f3[s3.N], f2[s2.N], f1[s1.N], f0[s0.N];
  s3.template init<HAS_F>(b, R, 1.0, a.delta, a.f, d3, f3);
  s2.template init<HAS_F>(b, K, 1.0, a.delta, a.f, d2, f2);
  s1.template init<HAS_F>(b, R, 1.0, a.delta, a.f, d1, f1);
  s0.template init<HAS_F>(b, K, 1.0, a.delta, a.f, d0, f0);
  const double C = block_total<NT>(a.c_part, a.c_count, red) * a.c_scale;   // ends in a barrier: ec is complete
  const Field<double> theta(a.theta, a.n);
  for_box<double, B, NT>(b, [&](int e, unsigned o, int i, int j, int m, int q) {
    // parent's position in ec and the neighbour towards the fine cell
    const double* __restrict__ p = ec + ((i >> 1) + 1) * (QJ * QK) + ((j >> 1) + 1) * QK + m + 1;
    const int ni = (i & 1) ? QJ * QK : -QJ * QK, nj = (j & 1) ? QK : -QK, nk = q ? 1 : -1;
    auto row = [&](int s) { return 0.75 * p[s] + 0.25 * p[s + nk]; };
    const double corr = 0.75 * (0.75 * row(0) + 0.25 * row(nj)) + 0.25 * (0.75 * row(ni) + 0.25 * row(ni + nj));
    th[e] = theta[o] + corr;
  });
  __syncthreads();
  const double h2 = a.h2, ih2 = a.ih2;
  constexpr int FM = HAS_F ? kRegF : kNoF;
  double acc = 0.0;
  half_sweep_box<B, decltype(s3), FM, false>(s3, th, R, d3, nullptr, f3, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s2), FM, false>(s2, th, K, d2, nullptr, f2, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s1), FM, true>(s1, th, R, d1, nullptr, f1, h2, ih2, C, acc);
  half_sweep_box<B, decltype(s0), FM, true>(s0, th, K, d0, nullptr, f0, h2, ih2, C, acc);
  constexpr int TILE = TI * TJ * TK, TKH = TK / 2;
  for (int x = tid; x < TILE; x += NT) {
    const int m = x % TKH, r = x / TKH;
    const int c = r / (TI * TJ), ij = r - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    a.theta_out[b.mesh(c, i, j, k)] = th[c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1)];
  }
  double v[1] = {acc};
  block_sum<1>(v, red, tid, NT);
  if (tid == 0) a.part_c[blockIdx.x] = v[0];
}

// ---- levels of 12^3 cells and below: one workgroup --------------------------------------------
// The last level above the coarsest (8^3 or 12^3) with the coarsest (4^3 or 6^3), or a coarsest level
// of 10^3 alone: FAS right-hand side, pre-relaxation, defect, restriction, the coarsest level's
// sweeps, prolongation, post-relaxation. theta is in LDS with a one-cell periodic halo (the owner of a
// cell writes its images), so a gather is one base address with constant offsets; delta and the
// right-hand side stay in the registers of the cell's owner. A coarsest mesh of 6^3 or less is swept by
// one wavefront, whose lanes exchange values through LDS without block barriers. As separate launches
// (sweeps, right-hand side, defect, 20 coarsest sweeps with two block barriers a half-sweep,
// transfers) the same work took about 140 us at 8^3.

// A mesh of N^3 cells owned by W threads (a block, or the lanes of one wavefront): cell u + p W of each
// colour belongs to thread u.
template <int N, bool WAVE, int W>
struct TailLevel {
  using B = Box<N, N, N, 1>;
  static constexpr int HALF = N * N * N / 2, PER = (HALF + W - 1) / W;
  static constexpr int DI = B::RJ * B::RKH, DJ = B::RKH;
  double* th;
  double h2, ih2;
  int e[2][PER];           // position in the colour's half of the box (c: local colour), q in bit 16
  int oi[PER], oj[PER], ok[2][PER];   // offsets of the periodic images (0: none)
  bool has[PER];
  double opd[2][PER], f[2][PER];

  __device__ __forceinline__ static void coords(int u, int& i, int& j, int& m) {
    m = u % (N / 2);
    const int r = u / (N / 2);
    j = r % N;
    i = r / N;
  }
  // mesh cell (i, j, k) of thread's cell p and mesh colour c
  __device__ __forceinline__ void init(double* lds, double h2_, double ih2_) {
    th = lds;
    h2 = h2_;
    ih2 = ih2_;
    const int lane = WAVE ? (threadIdx.x & 63) : threadIdx.x;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      has[p] = HALF % W == 0 || lane + p * W < HALF;
      int i, j, m;
      coords(has[p] ? lane + p * W : 0, i, j, m);
      oi[p] = i == 0 ? N * DI : (i == N - 1 ? -N * DI : 0);
      oj[p] = j == 0 ? N * DJ : (j == N - 1 ? -N * DJ : 0);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = 2 * m + ((i + j + c) & 1);   // local coordinates are one more
        e[c][p] = ((i + 1) * B::RJ + j + 1) * B::RKH + ((k + 1) >> 1) + (((k + 1) & 1) << 16);
        ok[c][p] = k == 0 ? N / 2 : (k == N - 1 ? -N / 2 : 0);
      }
    }
  }
  __device__ __forceinline__ double* half(int c) const { return th + (c ^ B::RED) * B::HALF; }
  __device__ __forceinline__ double get(int c, int p) const { return half(c)[e[c][p] & kLocPos]; }
  __device__ __forceinline__ void put(int c, int p, double v) const {
    double* a = half(c) + (e[c][p] & kLocPos);
    const int k = ok[c][p];
    a[0] = v;
    if (k) a[k] = v;
    if (oj[p]) {
      a[oj[p]] = v;
      if (k) a[oj[p] + k] = v;
    }
    if (oi[p]) {
      a[oi[p]] = v;
      if (k) a[oi[p] + k] = v;
      if (oj[p]) a[oi[p] + oj[p]] = v;
    }
  }
  // Sigma and the face sum of this thread's cells of colour c (several roots iterated together)
  __device__ __forceinline__ void source(int c, double (&sig)[PER], double (&S)[PER]) const {
    double pp[PER], qq[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      Nb18 t;
      B::gather(half(c), half(c ^ 1), e[c][p] & kLocPos, e[c][p] >> 16, t);
      cell_pq(t, opd[c][p], ih2, S[p], pp[p], qq[p]);
    }
    largest_roots<PER>(pp, qq, sig);
#pragma unroll
    for (int p = 0; p < PER; ++p) sig[p] -= 3.0;
  }
  // f = nabla^2 th - Sigma - f (f holds the restricted defect on entry)
  __device__ __forceinline__ void tau() {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double sig[PER], S[PER];
      source(c, sig, S);
#pragma unroll
      for (int p = 0; p < PER; ++p) f[c][p] = (S[p] - 6.0 * get(c, p)) * ih2 - sig[p] - f[c][p];
    }
  }
  // count red-black sweeps from the shift C, refreshed after every sweep
  __device__ __forceinline__ void sweeps(int count, double& C, double (*red)[1]) const {
    for (int s = 0; s < count; ++s) {
      double acc = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double sig[PER], S[PER];
        source(c, sig, S);
        tail_sync<WAVE>();   // every lane has read its neighbours before any of them is overwritten
#pragma unroll
        for (int p = 0; p < PER; ++p)
          if (has[p]) {
            acc += sig[p] + f[c][p];
            put(c, p, (S[p] - h2 * (sig[p] + f[c][p] - C)) * (1.0 / 6.0));
          }
        tail_sync<WAVE>();
      }
      C = total(acc, red) * (1.0 / (2.0 * HALF));
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

// NA: size of the first level; NB: of the coarsest level below it (0: the first is the coarsest).
template <int NA, int NB, int NT>
__global__ void __launch_bounds__(NT) blk_tail_kernel(BlkTailArgs a) {
  using LA = TailLevel<NA, false, NT>;
  using LB = TailLevel<NB == 0 ? 4 : NB, true, 64>;
  __shared__ double thA[2 * LA::B::HALF], dA[NB == 0 ? 1 : NA * NA * NA];
  __shared__ double thB[2 * LB::B::HALF], ec[NB == 0 ? 1 : (NB + 2) * (NB + 2) * (NB + 2)];
  __shared__ double red[16][1];
  const int tid = threadIdx.x;
  LA A;
  A.init(thA, a.h2, a.ih2);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < LA::PER; ++p) {
      const int g = c * LA::HALF + (A.has[p] ? tid + p * NT : 0);
      A.opd[c][p] = 1.0 + a.delta[g];
      A.f[c][p] = a.rd[g];
      const double t = a.that[g];
      if (A.has[p]) A.put(c, p, t);
    }
  double C = block_total<NT>(a.c_part, a.c_count, red) * a.c_scale;   // ends in a barrier
  A.tau();
  if (NB == 0) {
    A.sweeps(a.ncoarse, C, red);
  } else {
    A.sweeps(a.npre, C, red);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double sig[LA::PER], S[LA::PER];
      A.source(c, sig, S);
#pragma unroll
      for (int p = 0; p < LA::PER; ++p)
        if (A.has[p]) dA[c * LA::HALF + tid + p * NT] = (S[p] - 6.0 * A.get(c, p)) * A.ih2 - sig[p] - A.f[c][p] + C;
    }
    __syncthreads();
    if (tid < 64) {
      // restriction (8-son means of theta and of the defect) and the coarsest level
      LB Bl;
      Bl.init(thB, 4.0 * a.h2, 0.25 * a.ih2);
      double hat[2][LB::PER], sd = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p) {
          int I, J, M;
          LB::coords(Bl.has[p] ? tid + p * 64 : 0, I, J, M);
          const int K = 2 * M + ((I + J + c) & 1);
          double st = 0.0, sr = 0.0;
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const int i = 2 * I + (x >> 2), j = 2 * J + ((x >> 1) & 1), k = 2 * K + (x & 1);
            const int cc = (i + j + k) & 1;
            st += A.half(cc)[((i + 1) * LA::B::RJ + j + 1) * LA::B::RKH + ((k + 1) >> 1)];
            sr += dA[cc * LA::HALF + (i * NA + j) * (NA / 2) + (k >> 1)];
          }
          hat[c][p] = 0.125 * st;
          Bl.f[c][p] = 0.125 * sr;
          Bl.opd[c][p] = 1.0 + a.delta_c[c * LB::HALF + (Bl.has[p] ? tid + p * 64 : 0)];
          if (Bl.has[p]) {
            Bl.put(c, p, hat[c][p]);
            sd += Bl.f[c][p];
          }
        }
      double Cb = -wave_sum_full(sd) * (1.0 / (2.0 * LB::HALF));   // <Sigma + f> at the restricted iterate
      tail_sync<true>();
      Bl.tau();
      Bl.sweeps(a.ncoarse, Cb, red);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p)
          if (Bl.has[p]) {
            int I, J, M;
            LB::coords(tid + p * 64, I, J, M);
            const int K = 2 * M + ((I + J + c) & 1);
            const double v = Bl.get(c, p) - hat[c][p];
            // every periodic image within the one-cell halo
#pragma unroll
            for (int x = 0; x < 8; ++x) {
              const int oi = I == 0 ? NB : (I == NB - 1 ? -NB : 0), oj = J == 0 ? NB : (J == NB - 1 ? -NB : 0),
                        ok = K == 0 ? NB : (K == NB - 1 ? -NB : 0);
              if (((x & 4) && !oi) || ((x & 2) && !oj) || ((x & 1) && !ok)) continue;
              ec[((I + 1 + ((x & 4) ? oi : 0)) * (NB + 2) + J + 1 + ((x & 2) ? oj : 0)) * (NB + 2) + K + 1 +
                 ((x & 1) ? ok : 0)] = v;
            }
          }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < LA::PER; ++p)
        if (A.has[p]) {
          int i, j, m;
          LA::coords(tid + p * NT, i, j, m);
          const int q = (i + j + c) & 1;
          const double* __restrict__ x = ec + (((i >> 1) + 1) * (NB + 2) + (j >> 1) + 1) * (NB + 2) + m + 1;
          const int ni = ((i & 1) ? 1 : -1) * (NB + 2) * (NB + 2), nj = ((j & 1) ? 1 : -1) * (NB + 2), nk = q ? 1 : -1;
          auto row = [&](int s) { return 0.75 * x[s] + 0.25 * x[s + nk]; };
          A.put(c, p, A.get(c, p) + 0.75 * (0.75 * row(0) + 0.25 * row(nj)) + 0.25 * (0.75 * row(ni) + 0.25 * row(ni + nj)));
        }
    __syncthreads();
    A.sweeps(a.npost, C, red);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < LA::PER; ++p)
      if (A.has[p]) a.theta_out[c * LA::HALF + tid + p * NT] = A.get(c, p);
}

// ---- launchers ----------------------------------------------------------------------------

// Tile of a level: the smallest compiled one whose blocks are no more than the 256 compute units (a
// block's time goes with its cells and their halo, so a smaller tile is faster while units are idle;
// past that its larger halo costs more than it saves): 4^3 to 24^3, 4 x 4 x 8 at 32^3, 4 x 8 x 8 at
// 40^3, 8^3 at 48^3, 8 x 8 x 16 at 64^3. At 80^3 the largest runs twice as many: a solve takes 3.5 ms, with
// the plain launches there 4.7. 96^3 (864 blocks) stays with those: 4.4 ms either way, the adjoint 9.2 and 7.7.
BlkTile blk_tile(int n) {
  static const BlkTile tiles[] = {{4, 4, 4}, {4, 4, 8}, {4, 8, 8}, {8, 8, 8}, {8, 8, 16}};
  BlkTile best{0, 0, 0};
  for (const BlkTile& t : tiles) {
    if (n % t.ti != 0 || n % t.tj != 0 || n % t.tk != 0) continue;
    const int blocks = (n / t.ti) * (n / t.tj) * (n / t.tk);
    if (blocks <= kBlkMaxBlocks) best = t;
    if (blocks <= 256) break;
  }
  return best;
}

bool blk_level_supported(int n) { return n >= 16 && n <= kBlkMaxN && blk_tile(n).ti != 0; }

int blk_blocks(int n) {
  const BlkTile t = blk_tile(n);
  return (n / t.ti) * (n / t.tj) * (n / t.tk);
}

#define MR_BLK_GO(KERNEL, TI, TJ, TK, NT, FLAG)                                                        \
  if (t.ti == TI && t.tj == TJ && t.tk == TK) {                                                        \
    if (FLAG)                                                                                          \
      hipLaunchKernelGGL((KERNEL<TI, TJ, TK, NT, true>), dim3(blk_blocks(a.n)), dim3(NT), 0, s, a);    \
    else                                                                                               \
      hipLaunchKernelGGL((KERNEL<TI, TJ, TK, NT, false>), dim3(blk_blocks(a.n)), dim3(NT), 0, s, a);   \
    return hipGetLastError();                                                                          \
  }
#define MR_BLK_TILES(KERNEL, FLAG)        \
  MR_BLK_GO(KERNEL, 4, 4, 4, 512, FLAG)   \
  MR_BLK_GO(KERNEL, 4, 4, 8, 512, FLAG)   \
  MR_BLK_GO(KERNEL, 4, 8, 8, 512, FLAG)   \
  MR_BLK_GO(KERNEL, 8, 8, 8, 512, FLAG)   \
  MR_BLK_GO(KERNEL, 8, 8, 16, 1024, FLAG)

hipError_t launch_blk_down(const BlkDownArgs& a, hipStream_t s) {
  if (!blk_level_supported(a.n) || (a.rd != nullptr) != (a.f_out != nullptr)) return hipErrorInvalidValue;
  const BlkTile t = blk_tile(a.n);
  MR_BLK_TILES(blk_down_kernel, a.rd)
  return hipErrorInvalidValue;
}

hipError_t launch_blk_up(const BlkUpArgs& a, hipStream_t s) {
  if (!blk_level_supported(a.n)) return hipErrorInvalidValue;
  const BlkTile t = blk_tile(a.n);
  MR_BLK_TILES(blk_up_kernel, a.f)
  return hipErrorInvalidValue;
}

hipError_t launch_blk_tail(const BlkTailArgs& a, hipStream_t s) {
  if (a.n == 8 && !a.coarsest)
    hipLaunchKernelGGL((blk_tail_kernel<8, 4, 256>), dim3(1), dim3(256), 0, s, a);
  else if (a.n == 12 && !a.coarsest)
    hipLaunchKernelGGL((blk_tail_kernel<12, 6, 896>), dim3(1), dim3(896), 0, s, a);
  else if (a.n == 10 && a.coarsest)
    hipLaunchKernelGGL((blk_tail_kernel<10, 0, 512>), dim3(1), dim3(512), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mr
