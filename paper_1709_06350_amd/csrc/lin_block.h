// The FP32 linear V-cycle of the mixed-precision form on its small meshes: the device bodies shared by the
// one-mesh launches (lin_block.hip) and the multi-box launches (batched.hip).
//
// The decomposition is that of block_cycle.hip: a block holds e and the fixed-point base of its tile and
// halo in LDS and runs two red-black sweeps with the defect and restriction (down; from e = 0 the
// first red half-sweep is -h^2 (rhs - C) / 6 and the first black one needs only the face terms), or the
// prolongation with two sweeps (up); the levels of 12^3 cells and below are one workgroup, whose
// Jacobian weights are formed once and stay in the registers of the cell's owner. A sweep of 64^3 or
// 32^3 cells took two launches of 11-12 us, a level's cycle about 100 us.
// The shift C = <dSigma(e) + rhs> is taken once per launch, from the block sums of the launch before on
// that level (down from zero: from the sums of its right-hand side).
#pragma once

#include "block_box.h"
#include "mixed_device.h"

namespace mr {

// Sums that set a launch's shift: C = scale * (sum of part[0 .. count)).
struct LinShift {
  const double* part;
  int count;
  double scale;
};

struct LinDownArgs {
  const float* e;        // iterate in (null: zero)
  const float* rhs;
  const int* base;
  const float* sb;
  const double* bq;
  int n;
  float h2, ih2;
  LinShift c;
  float* e_out;
  float* rhs_c;          // 8-son mean of the defect
  double *part_c, *part_r;   // per block: dSigma + rhs of the last sweep, rhs_c
};

struct LinUpArgs {
  const float* e;
  const float* e_c;      // coarse correction
  const float* rhs;
  const int* base;
  const float* sb;
  const double* bq;
  int n;
  float h2, ih2;
  LinShift c;
  float* e_out;
  double* part_c;
};

struct LinTail2Args {
  const float* rhs;      // level of n^3 cells (8, 12, or 10 as the coarsest), e = 0 on entry
  const int *base, *base_c;
  const float *sb, *sb_c;
  const double* bq;
  int n, npre, npost, ncoarse;
  float h2;
  LinShift c;
  float* e_out;
};

// New values of local colour c on a stage (EDGES false: the own colour's e is zero). Adds dSigma + rhs of
// the tile's own cells to acc.
template <class B, bool EDGES, bool SUM, class St>
__device__ __forceinline__ void lin_half_box(const St& st, float* __restrict__ e, const float* __restrict__ bs, int c,
                                             const float (&sb)[St::N], const float (&rhs)[St::N], float bscl, float h2,
                                             float ih2, float C, double& acc) {
  float nv[St::N];
  float* __restrict__ own = e + c * B::HALF;
  const float* __restrict__ oth = e + (c ^ 1) * B::HALF;
  const float* __restrict__ bown = bs + c * B::HALF;
  const float* __restrict__ both = bs + (c ^ 1) * B::HALF;
#pragma unroll
  for (int t = 0; t < St::N; ++t) {
    nv[t] = 0.0f;
    if (st.loc[t] >= 0) {
      const int x = st.loc[t] & kLocPos, q = (st.loc[t] >> 16) & 1;
      Nb18f te, tb;
      B::gather(own, oth, x, q, te);
      if (!EDGES) te.xpyp = te.xmym = te.xpym = te.xmyp = te.xpzp = te.xmzm = te.xpzm = te.xmzp = te.ypzp = te.ymzm = te.ypzm = te.ymzp = 0.0f;
      B::gather(bown, both, x, q, tb);
      float Se;
      const float g = lin_source(tb, bown[x], bscl, sb[t], ih2, te, Se) * ih2;
      nv[t] = (Se - h2 * (g + rhs[t] - C)) * (1.0f / 6.0f);
      if (SUM && (st.loc[t] & kLocOwn)) acc += (double)(g + rhs[t]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < St::N; ++t)
    if (st.loc[t] >= 0) own[st.loc[t] & kLocPos] = nv[t];
  __syncthreads();
}

// LDS of a down or up block (floats of both boxes, coarse corrections of up).
template <int TI, int TJ, int TK, int OFF>
struct LinBoxLds {
  using B = Box<TI, TJ, TK, OFF>;
  static constexpr int QI = B::RI / 2 + 2, QJ = B::RJ / 2 + 2, QK = B::RKH + 2, NQ = QI * QJ * QK;
  float e[2 * B::HALF], bs[2 * B::HALF], ec[OFF == 4 ? NQ : 1];
  double red[16][2];
};

// blk: this block's number within its mesh, logical: its tile.
template <int TI, int TJ, int TK, int NT, bool ZERO>
__device__ void lin_down_body(const LinDownArgs& a, int logical, int blk, LinBoxLds<TI, TJ, TK, ZERO ? 4 : 5>& sh) {
  constexpr int OFF = ZERO ? 4 : 5;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 4, NT> s4;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  constexpr int R = B::RED, K = R ^ 1;
  B b;
  b.init(logical, a.n);
  const int tid = threadIdx.x;
  const Field<float> basef(reinterpret_cast<const float*>(a.base), a.n), e_in(a.e, a.n);
  for_box<float, B, NT>(b, [&](int x, unsigned o, int i, int j, int m, int q) {
    sh.bs[x] = basef[o];
    if (!ZERO) sh.e[x] = e_in[o];
  });
  float b4[s4.N], b3[s3.N], b2[s2.N], b1[s1.N], r4[s4.N], r3[s3.N], r2[s2.N], r1[s1.N];
  s4.template init<true>(b, R, 0.0f, a.sb, a.rhs, b4, r4);
  s3.template init<true>(b, K, 0.0f, a.sb, a.rhs, b3, r3);
  s2.template init<true>(b, R, 0.0f, a.sb, a.rhs, b2, r2);
  s1.template init<true>(b, K, 0.0f, a.sb, a.rhs, b1, r1);
  // the tile's cells for the defect, eight sons of a coarse cell on eight consecutive threads
  constexpr int TILE = TI * TJ * TK;
  static_assert(TILE <= NT && TILE % 64 == 0, "one cell of the tile per thread");
  const int son = tid & 7, cc = tid >> 3;
  const int cK = cc % (TK / 2), cJ = (cc / (TK / 2)) % (TJ / 2), cI = cc / (TK / 2 * (TJ / 2));
  const int di = OFF + 2 * cI + (son >> 2), dj = OFF + 2 * cJ + ((son >> 1) & 1), dk = OFF + 2 * cK + (son & 1);
  const int dc = (di + dj + dk) & 1;
  const bool own = tid < TILE;
  float ds = 0.0f, dr = 0.0f;
  if (own) {
    const unsigned g = b.mesh(dc, di, dj, dk);
    ds = a.sb[g];
    dr = a.rhs[g];
  }
  const float bscl = (float)a.bq[0], h2 = a.h2, ih2 = a.ih2;
  const float C = (float)(block_total<NT>(a.c.part, a.c.count, reinterpret_cast<double(*)[1]>(sh.red)) * a.c.scale);
  double acc = 0.0;
  if (ZERO) {
    const float g = -h2 * (1.0f / 6.0f);
#pragma unroll
    for (int t = 0; t < s4.N; ++t)
      if (s4.loc[t] >= 0) sh.e[R * B::HALF + (s4.loc[t] & kLocPos)] = g * (r4[t] - C);
    __syncthreads();
    lin_half_box<B, false, false>(s3, sh.e, sh.bs, K, b3, r3, bscl, h2, ih2, C, acc);
  } else {
    lin_half_box<B, true, false>(s4, sh.e, sh.bs, R, b4, r4, bscl, h2, ih2, C, acc);
    lin_half_box<B, true, false>(s3, sh.e, sh.bs, K, b3, r3, bscl, h2, ih2, C, acc);
  }
  lin_half_box<B, true, true>(s2, sh.e, sh.bs, R, b2, r2, bscl, h2, ih2, C, acc);
  lin_half_box<B, true, true>(s1, sh.e, sh.bs, K, b1, r1, bscl, h2, ih2, C, acc);
  float d = 0.0f;
  if (own) {
    const int x = (di * B::RJ + dj) * B::RKH + (dk >> 1), o = dc * B::HALF, p = (dc ^ 1) * B::HALF;
    Nb18f te, tb;
    B::gather(sh.e + o, sh.e + p, x, dk & 1, te);
    B::gather(sh.bs + o, sh.bs + p, x, dk & 1, tb);
    float Se;
    const float g = lin_source(tb, sh.bs[o + x], bscl, ds, ih2, te, Se) * ih2;
    d = dr + g - (Se - 6.0f * sh.e[o + x]) * ih2 - C;
  }
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) d += __shfl_xor(d, x, 64);
  d *= 0.125f;
  double sr = 0.0;
  if (own && son == 0) {
    a.rhs_c[split_idx(a.n >> 1, ((b.i0 + OFF) >> 1) + cI, ((b.j0 + OFF) >> 1) + cJ, ((b.k0 + OFF) >> 1) + cK)] = d;
    sr = (double)d;
  }
  if (own) {
    constexpr int TKH = TK / 2;
    const int m = tid % TKH, q = tid / TKH;
    const int c = q / (TI * TJ), ij = q - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    a.e_out[b.mesh(c, i, j, k)] = sh.e[c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1)];
  }
  double v[2] = {acc, sr};
  block_sum<2>(v, sh.red, tid, NT);
  if (tid == 0) {
    a.part_c[blk] = v[0];
    a.part_r[blk] = v[1];
  }
}

template <int TI, int TJ, int TK, int NT>
__device__ void lin_up_body(const LinUpArgs& a, int logical, int blk, LinBoxLds<TI, TJ, TK, 4>& sh) {
  constexpr int OFF = 4;
  using L = LinBoxLds<TI, TJ, TK, 4>;
  using B = Box<TI, TJ, TK, OFF>;
  Stage<B, TI, TJ, TK, OFF, 3, NT> s3;
  Stage<B, TI, TJ, TK, OFF, 2, NT> s2;
  Stage<B, TI, TJ, TK, OFF, 1, NT> s1;
  Stage<B, TI, TJ, TK, OFF, 0, NT> s0;
  constexpr int R = B::RED, K = R ^ 1;
  constexpr int QJ = L::QJ, QK = L::QK;
  B b;
  b.init(logical, a.n);
  const int tid = threadIdx.x, nc = a.n >> 1;
  for (int x = tid; x < L::NQ; x += NT) {
    const int r = div_small<QK>(x), k = x - r * QK;
    const int i = div_small<QJ>(r), j = r - i * QJ;
    sh.ec[x] = a.e_c[split_idx(nc, wrapi((b.i0 >> 1) - 1 + i, nc), wrapi((b.j0 >> 1) - 1 + j, nc),
                               wrapi((b.k0 >> 1) - 1 + k, nc))];
  }
  float b3[s3.N], b2[s2.N], b1[s1.N], b0[s0.N], r3[s3.N], r2[s2.N], r1[s1.N], r0[s0.N];
  s3.template init<true>(b, R, 0.0f, a.sb, a.rhs, b3, r3);
  s2.template init<true>(b, K, 0.0f, a.sb, a.rhs, b2, r2);
  s1.template init<true>(b, R, 0.0f, a.sb, a.rhs, b1, r1);
  s0.template init<true>(b, K, 0.0f, a.sb, a.rhs, b0, r0);
  const float bscl = (float)a.bq[0], h2 = a.h2, ih2 = a.ih2;
  const float C = (float)(block_total<NT>(a.c.part, a.c.count, reinterpret_cast<double(*)[1]>(sh.red)) *
                          a.c.scale);   // ends in a barrier: ec is complete
  const Field<float> basef(reinterpret_cast<const float*>(a.base), a.n), e_in(a.e, a.n);
  for_box<float, B, NT>(b, [&](int x, unsigned o, int i, int j, int m, int q) {
    const float* __restrict__ p = sh.ec + ((i >> 1) + 1) * (QJ * QK) + ((j >> 1) + 1) * QK + m + 1;
    const int ni = (i & 1) ? QJ * QK : -QJ * QK, nj = (j & 1) ? QK : -QK, nk = q ? 1 : -1;
    auto row = [&](int s) { return 0.75f * p[s] + 0.25f * p[s + nk]; };
    const float corr = 0.75f * (0.75f * row(0) + 0.25f * row(nj)) + 0.25f * (0.75f * row(ni) + 0.25f * row(ni + nj));
    sh.e[x] = e_in[o] + corr;
    sh.bs[x] = basef[o];
  });
  __syncthreads();
  double acc = 0.0;
  lin_half_box<B, true, false>(s3, sh.e, sh.bs, R, b3, r3, bscl, h2, ih2, C, acc);
  lin_half_box<B, true, false>(s2, sh.e, sh.bs, K, b2, r2, bscl, h2, ih2, C, acc);
  lin_half_box<B, true, true>(s1, sh.e, sh.bs, R, b1, r1, bscl, h2, ih2, C, acc);
  lin_half_box<B, true, true>(s0, sh.e, sh.bs, K, b0, r0, bscl, h2, ih2, C, acc);
  constexpr int TILE = TI * TJ * TK, TKH = TK / 2;
  for (int x = tid; x < TILE; x += NT) {
    const int m = x % TKH, q = x / TKH;
    const int c = q / (TI * TJ), ij = q - c * (TI * TJ);
    const int i = OFF + ij / TJ, j = OFF + ij % TJ, k = OFF + ((OFF + i + j + c) & 1) + 2 * m;
    a.e_out[b.mesh(c, i, j, k)] = sh.e[c * B::HALF + (i * B::RJ + j) * B::RKH + (k >> 1)];
  }
  double v[2] = {acc, 0.0};
  block_sum<2>(v, sh.red, tid, NT);
  if (tid == 0) a.part_c[blk] = v[0];
}

// ---- the levels of 12^3 cells and below in one workgroup ---------------------------------------
// Weights of h^2 dSigma(e) = sum_a w_a eS_a + sum_{a<b} w_ab eD_ab at a cell (see lin_source).
struct LinW {
  float x, y, z, xy, xz, yz;
};
__device__ __forceinline__ LinW lin_weights(const Nb18f& b, float bc, float bscl, float s, float ih2) {
  // dSigma is linear in e: its value on unit pair sums and cross differences
  LinW w;
  Nb18f u = {};
  float Se;
  u.xm = 1.0f;
  w.x = lin_source(b, bc, bscl, s, ih2, u, Se);
  u.xm = 0.0f;
  u.ym = 1.0f;
  w.y = lin_source(b, bc, bscl, s, ih2, u, Se);
  u.ym = 0.0f;
  u.zm = 1.0f;
  w.z = lin_source(b, bc, bscl, s, ih2, u, Se);
  u.zm = 0.0f;
  u.xpyp = 1.0f;
  w.xy = lin_source(b, bc, bscl, s, ih2, u, Se);
  u.xpyp = 0.0f;
  u.xpzp = 1.0f;
  w.xz = lin_source(b, bc, bscl, s, ih2, u, Se);
  u.xpzp = 0.0f;
  u.ypzp = 1.0f;
  w.yz = lin_source(b, bc, bscl, s, ih2, u, Se);
  return w;
}

// A mesh of N^3 cells owned by W threads (a block, or the lanes of one wavefront); e in LDS with a one-cell
// periodic halo.
template <int N, bool WAVE, int W>
struct LinTailLevel {
  using B = Box<N, N, N, 1>;
  static constexpr int HALF = N * N * N / 2, PER = (HALF + W - 1) / W;
  static constexpr int DI = B::RJ * B::RKH, DJ = B::RKH;
  float* e;
  float h2, ih2;
  int pos[2][PER];   // position in the colour's half of the box, q in bit 16
  int oi[PER], oj[PER], ok[2][PER];
  bool has[PER];
  LinW w[2][PER];
  float rhs[2][PER];

  __device__ __forceinline__ static void coords(int u, int& i, int& j, int& m) {
    m = u % (N / 2);
    const int r = u / (N / 2);
    j = r % N;
    i = r / N;
  }
  __device__ __forceinline__ void init(float* lds, float h2_) {
    e = lds;
    h2 = h2_;
    ih2 = 1.0f / h2_;
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
        const int k = 2 * m + ((i + j + c) & 1);
        pos[c][p] = ((i + 1) * B::RJ + j + 1) * B::RKH + ((k + 1) >> 1) + (((k + 1) & 1) << 16);
        ok[c][p] = k == 0 ? N / 2 : (k == N - 1 ? -N / 2 : 0);
      }
    }
  }
  __device__ __forceinline__ float* half(float* a, int c) const { return a + (c ^ B::RED) * B::HALF; }
  __device__ __forceinline__ float get(int c, int p) const { return half(e, c)[pos[c][p] & kLocPos]; }
  __device__ __forceinline__ void put(float* arr, int c, int p, float v) const {
    float* a = half(arr, c) + (pos[c][p] & kLocPos);
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
  // this thread's cells of the base into bs (then a barrier, then weights())
  __device__ __forceinline__ void load(float* bs, const int* __restrict__ base, const float* __restrict__ rhs_) {
    const int lane = WAVE ? (threadIdx.x & 63) : threadIdx.x;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        const int g = c * HALF + (has[p] ? lane + p * W : 0);
        const float v = qbits(base[g]);
        if (rhs_) rhs[c][p] = rhs_[g];
        if (has[p]) {
          put(bs, c, p, v);
          put(e, c, p, 0.0f);
        }
      }
  }
  __device__ __forceinline__ void weights(float* bs, const float* __restrict__ sb, float bscl) {
    const int lane = WAVE ? (threadIdx.x & 63) : threadIdx.x;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        Nb18f t;
        const int x = pos[c][p] & kLocPos;
        B::gather(half(bs, c), half(bs, c ^ 1), x, pos[c][p] >> 16, t);
        w[c][p] = lin_weights(t, half(bs, c)[x], bscl, sb[c * HALF + (has[p] ? lane + p * W : 0)], ih2);
      }
  }
  // dSigma(e) and the face sum at cell p of colour c
  __device__ __forceinline__ float source(int c, int p, float& S) const {
    Nb18f t;
    B::gather(half(e, c), half(e, c ^ 1), pos[c][p] & kLocPos, pos[c][p] >> 16, t);
    const float sx = t.xm + t.xp, sy = t.ym + t.yp, sz = t.zm + t.zp;
    S = sx + sy + sz;
    const float dxy = (t.xpyp + t.xmym) - (t.xpym + t.xmyp);
    const float dxz = (t.xpzp + t.xmzm) - (t.xpzm + t.xmzp);
    const float dyz = (t.ypzp + t.ymzm) - (t.ypzm + t.ymzp);
    const LinW& v = w[c][p];
    return ((v.x * sx + v.y * sy + v.z * sz) + (v.xy * dxy + v.xz * dxz + v.yz * dyz)) * ih2;
  }
  __device__ __forceinline__ void sweeps(int count, float& C, double (*red)[2]) const {
    for (int s = 0; s < count; ++s) {
      double acc = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        float nv[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
          float S;
          const float g = source(c, p, S);
          nv[p] = (S - h2 * (g + rhs[c][p] - C)) * (1.0f / 6.0f);
          if (has[p]) acc += (double)(g + rhs[c][p]);
        }
        tail_sync<WAVE>();
#pragma unroll
        for (int p = 0; p < PER; ++p)
          if (has[p]) put(e, c, p, nv[p]);
        tail_sync<WAVE>();
      }
      C = (float)(total(acc, red) * (1.0 / (2.0 * HALF)));
    }
  }
  __device__ __forceinline__ double total(double v, double (*red)[2]) const {
    v = wave_sum_full(v);
    if (WAVE) return v;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int x = 0; x < W / 64; ++x) s += red[x][0];
    __syncthreads();
    return s;
  }
};

template <int NA, int NB>
struct LinTail2Lds {
  using BA = Box<NA, NA, NA, 1>;
  using BB = Box<NB == 0 ? 4 : NB, NB == 0 ? 4 : NB, NB == 0 ? 4 : NB, 1>;
  float eA[2 * BA::HALF], bA[2 * BA::HALF], dA[NB == 0 ? 1 : NA * NA * NA];
  float eB[2 * BB::HALF], bB[2 * BB::HALF], ec[NB == 0 ? 1 : (NB + 2) * (NB + 2) * (NB + 2)];
  double red[16][2];
};

template <int NA, int NB, int NT>
__device__ void lin_tail2_body(const LinTail2Args& a, LinTail2Lds<NA, NB>& sh) {
  using LA = LinTailLevel<NA, false, NT>;
  using LB = LinTailLevel<NB == 0 ? 4 : NB, true, 64>;
  const int tid = threadIdx.x;
  const float bscl = (float)a.bq[0];
  LA A;
  LB Bl;
  A.init(sh.eA, a.h2);
  A.load(sh.bA, a.base, a.rhs);
  if (NB != 0 && tid < 64) {
    Bl.init(sh.eB, 4.0f * a.h2);
    Bl.load(sh.bB, a.base_c, nullptr);
    tail_sync<true>();
    Bl.weights(sh.bB, a.sb_c, bscl);
  }
  float C = (float)(block_total<NT>(a.c.part, a.c.count, reinterpret_cast<double(*)[1]>(sh.red)) * a.c.scale);
  A.weights(sh.bA, a.sb, bscl);   // block_total ended in a barrier
  if (NB == 0) {
    A.sweeps(a.ncoarse, C, sh.red);
  } else {
    A.sweeps(a.npre, C, sh.red);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < LA::PER; ++p) {
        float S;
        const float g = A.source(c, p, S);
        if (A.has[p]) sh.dA[c * LA::HALF + tid + p * NT] = A.rhs[c][p] + g - (S - 6.0f * A.get(c, p)) * A.ih2 - C;
      }
    __syncthreads();
    if (tid < 64) {
      double sr = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p) {
          int I, J, M;
          LB::coords(Bl.has[p] ? tid + p * 64 : 0, I, J, M);
          const int K = 2 * M + ((I + J + c) & 1);
          float s = 0.0f;
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const int i = 2 * I + (x >> 2), j = 2 * J + ((x >> 1) & 1), k = 2 * K + (x & 1);
            s += sh.dA[((i + j + k) & 1) * LA::HALF + (i * NA + j) * (NA / 2) + (k >> 1)];
          }
          Bl.rhs[c][p] = 0.125f * s;
          if (Bl.has[p]) sr += (double)(0.125f * s);
        }
      float Cb = (float)(wave_sum_full(sr) * (1.0 / (2.0 * LB::HALF)));
      Bl.sweeps(a.ncoarse, Cb, sh.red);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int p = 0; p < LB::PER; ++p)
          if (Bl.has[p]) {
            int I, J, M;
            LB::coords(tid + p * 64, I, J, M);
            const int K = 2 * M + ((I + J + c) & 1);
            const float v = Bl.get(c, p);
            const int oi = I == 0 ? NB : (I == NB - 1 ? -NB : 0), oj = J == 0 ? NB : (J == NB - 1 ? -NB : 0),
                      ok = K == 0 ? NB : (K == NB - 1 ? -NB : 0);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
              if (((x & 4) && !oi) || ((x & 2) && !oj) || ((x & 1) && !ok)) continue;
              sh.ec[((I + 1 + ((x & 4) ? oi : 0)) * (NB + 2) + J + 1 + ((x & 2) ? oj : 0)) * (NB + 2) + K + 1 +
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
          const float* __restrict__ x = sh.ec + (((i >> 1) + 1) * (NB + 2) + (j >> 1) + 1) * (NB + 2) + m + 1;
          const int ni = ((i & 1) ? 1 : -1) * (NB + 2) * (NB + 2), nj = ((j & 1) ? 1 : -1) * (NB + 2), nk = q ? 1 : -1;
          auto row = [&](int s) { return 0.75f * x[s] + 0.25f * x[s + nk]; };
          A.put(sh.eA, c, p,
                A.get(c, p) + 0.75f * (0.75f * row(0) + 0.25f * row(nj)) + 0.25f * (0.75f * row(ni) + 0.25f * row(ni + nj)));
        }
    __syncthreads();
    A.sweeps(a.npost, C, sh.red);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < LA::PER; ++p)
      if (A.has[p]) a.e_out[c * LA::HALF + tid + p * NT] = A.get(c, p);
}

// ---- tiles --------------------------------------------------------------------------------------
// Tile of a mesh: the smallest compiled one with at most 256 blocks, one per compute unit, else 8 x 8 x 16.
// All but the last have 512 threads. Levels to 96^3: mixed solves of 80^3, 96^3, 160^3 and 192^3 took 3.46,
// 4.52, 10.2 and 13.1 ms with them, 4.96, 4.96, 11.7 and 13.7 ms with the block form to 64^3 only; at
// 128^3 a cycle's two launches take 242 us against 178 us for the plain ones (the halo's share of the
// work, once every compute unit has several blocks).
constexpr int kLinBlkMaxN = 96;
constexpr int kLinBlkMaxBlocks = 1024;
#define MR_LB_TILES(X) X(4, 4, 4, 512) X(4, 4, 8, 512) X(4, 8, 8, 512) X(8, 8, 8, 512) X(8, 8, 16, 1024)
struct LinBlkTile {
  int ti, tj, tk;
};
inline LinBlkTile lin_blk_tile(int n) {
  static const int tiles[][3] = {{4, 4, 4}, {4, 4, 8}, {4, 8, 8}, {8, 8, 8}, {8, 8, 16}};
  LinBlkTile last{0, 0, 0};
  if (n < 16 || n > kLinBlkMaxN) return last;
  for (const auto& t : tiles)
    if (n % t[0] == 0 && n % t[1] == 0 && n % t[2] == 0) {
      last = LinBlkTile{t[0], t[1], t[2]};
      if ((n / t[0]) * (n / t[1]) * (n / t[2]) <= 256) break;
    }
  return last;
}
inline int lin_blk_blocks(int n) {
  const LinBlkTile t = lin_blk_tile(n);
  return t.ti ? (n / t.ti) * (n / t.tj) * (n / t.tk) : 0;
}

}  // namespace mr
