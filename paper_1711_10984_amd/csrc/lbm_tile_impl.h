// The timestep on two-dimensional tiles: one launch per step, for lattices whose strips would leave most of the
// chip idle.
//
// A workgroup owns OX x OY nodes and computes every stage of the step on them, each stage on a region that is
// wider than the next one's by a ring (mu, X on the tile and four rings; u on three; the half-step fields on two;
// M and X^{n+1/2} on one), all in LDS.  The rings are computed by the neighbouring tiles too: 1.4 to 2 times the
// arithmetic of the bare nodes.  The strips of k_step and k_wave recompute less, but a strip is a serial sweep over
// its rows: the 64 rows of a 64 x 64 lattice take two workgroups 73 us, however idle the other compute units are.
// Here a step is a chain of six stages whatever the size, bound by latency (loads, barriers, dependent arithmetic)
// while there is a workgroup per compute unit at most, and by instruction issue beyond.  One step, FP64, in us
// (centres of mass included), tiles / k_step of 64 rows / k_lb and k_fd:
//   64 x 64  6.6 / 73 / 21;   256 x 256  8.5 / 78 / 22;   512 x 256  11.8 / 78 / 23;   512 x 512  23.6 / 81 / 30
// Of the 64 x 64 step's 5.9 us inside the kernel, 1.4 are the loads, 0.6 to 1 each of the six stages and 0.9 the sums.
// What a stage leaves idle takes the work that is not on the chain: the collision runs beside s3, c^{n+1} beside
// phi^{n+1}, and the centres on a wavefront that has no part in s3 (before, the collision lengthened s2, c followed phi
// and the centres held up s4: 8.6, 10.7 and 14.2 us).
//
// The centres of mass need a sum over the whole lattice after every step.  It is taken without a launch of its
// own: a step leaves each tile's sums in memory, and the workgroups of the next step each add them up (in the
// same order, so all get the same centres) while the stages that need no centre run.  Sums and centres have two
// buffers that alternate from step to step, so that no workgroup overwrites what another one still reads.
// The last step of a sequence is followed by k_tile_final, which brings the droplet table and the step counter
// up to date.
#pragma once
#include "lbm_kernels_impl.h"

namespace lbm {
namespace {

// The centre of mass of droplet k of an instance from its tiles' sums, by one wavefront, in parts so that each runs
// while the wavefront would wait for others: begin() loads the tiles' presence bits, load() lists the tiles that hold
// the droplet and loads the sums of the first 64 of them, sum() adds up, move() gives the centre.  Tiles are taken
// TILE_CHUNK at a time; one chunk covers every lattice whose tiles fit the chip at once.  Each of the three sums has a row of 16 lanes (the last row
// repeats the third), one tile's entry to a lane: additions in twice the working precision are chains of dependent
// FP64 operations, and all three sums over all 64 lanes took the whole stage beside them (1.4 us) and more.
constexpr int TILE_UNR = 4, TILE_CHUNK = 64 * TILE_UNR;
struct TileCentre {
  const double* part;
  const uint32_t* mask;
  uint16_t* list;  // LDS, TILE_CHUNK entries of the wavefront's own
  int nt, nd, n;
  uint32_t m[TILE_UNR];
  Dd e[4];
  double v;  // the row's sum, in its last lane

  __device__ __forceinline__ void bits(int c0) {
#pragma unroll
    for (int u = 0; u < TILE_UNR; ++u) {
      const int tl = c0 + u * 64 + (int)(threadIdx.x & 63);
      m[u] = tl < nt ? mask[tl] : 0u;
    }
  }
  __device__ __forceinline__ void begin(const InstDev& I, const TileSeq& q, uint16_t* lds) {
    part = q.part_in + I.part_base[TILING_TILE];
    mask = q.mask_in + I.tile_base[TILING_TILE];
    list = lds;
    nt = I.tiles_x[TILING_TILE] * I.tiles_y[TILING_TILE];
    nd = I.ndrop;
    bits(0);
  }
  __device__ __forceinline__ void collect(int k) {
    const unsigned long long below = (1ull << (threadIdx.x & 63)) - 1ull;
    n = 0;
#pragma unroll
    for (int u = 0; u < TILE_UNR; ++u) {
      const bool has = (m[u] >> k) & 1u;
      const unsigned long long b = __ballot(has);
      if (has) list[n + __popcll(b & below)] = (uint16_t)(u * 64 + (threadIdx.x & 63));
      n += __popcll(b);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // entry j of the list, this lane's sum of it
  __device__ __forceinline__ Dd entry(int c0, int j, int k) const {
    const double* const p = part + ((int64_t)(c0 + list[j]) * nd + k) * 6 + 2 * min((int)(threadIdx.x & 63) >> 4, 2);
    return Dd{p[0], p[1]};
  }
  __device__ __forceinline__ void load(int k) {
    collect(k);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = u * 16 + (int)(threadIdx.x & 15);
      e[u] = j < n ? entry(0, j, k) : Dd{0.0, 0.0};
    }
  }
  __device__ __forceinline__ void sum(int k) {
    Dd s[1] = {e[0]};
#pragma unroll
    for (int u = 1; u < 4; ++u)
      if (u * 16 < n) dd_add(s[0], e[u]);
    for (int c0 = 0;;) {
      for (int j = (int)(threadIdx.x & 15) + (c0 == 0 ? 64 : 0); j < n; j += 16) dd_add(s[0], entry(c0, j, k));
      c0 += TILE_CHUNK;
      if (c0 >= nt) break;
      bits(c0);
      collect(k);
    }
    dd_row_sum(s);
    v = dd_value(s[0]);
  }
  __device__ __forceinline__ void move(const InstDev& I, double& cx, double& cy) const {
    const double w = lane_value(v, 15);
    if (w > 0.0) {  // without a node of the droplet its centre stays
      const double d = v / w;
      cx = wrapd(cx + lane_value(d, 31), (double)I.nx);
      cy = wrapd(cy + lane_value(d, 47), I.yper);
    }
  }
};

// One step on tiles.  MULTI: a batch, with the list of its tiles; else the lattice is `one` and block b has tile
// xcd_block() of it.  DBG: also export the stage planes of instance dbg_inst (the others are skipped), as k_step.
template <typename T, typename P, int OX, int OY, int NT, bool DBG, bool MULTI>
__global__ __launch_bounds__(NT) void k_tile(int parity, InstDev one, const TileDev* __restrict__ tiles,
                                                       const InstDev* __restrict__ insts, T* __restrict__ buf,
                                                       const DropDev* __restrict__ drops, TileSeq q,
                                                       const int64_t* __restrict__ step, double* __restrict__ dbg,
                                                       int dbg_inst) {
  constexpr int NW = NT / 64, NWO = (OX * OY + 63) / 64 < NW ? (OX * OY + 63) / 64 : NW;
  constexpr int W5 = OX + 10, H5 = OY + 10, W4 = OX + 8, H4 = OY + 8, W3 = OX + 6, H3 = OY + 6;
  constexpr int W2 = OX + 4, H2 = OY + 4, W1 = OX + 2, H1 = OY + 2;
  constexpr int R5 = (W5 * H5 + NT - 1) / NT, R3 = (W3 * H3 + NT - 1) / NT;
  __shared__ T s_phi[W5 * H5], s_c[W5 * H5];
  __shared__ T s_a[2][W4 * H4];  // mu, X; then phi and c at n + 1/2 (with their rings, W2 x H2)
  __shared__ T s_b[2][W3 * H3];  // u; then M and X^{n+1/2} (W1 x H1)
  __shared__ double s_d[TILE_DROPS][5];  // centre, disk centre, Rs^2
  __shared__ int s_src[TILE_DROPS];      // the droplet's production disk may reach the tile
  __shared__ double s_sum[NWO][TILE_DROPS][6];  // sums of the wavefronts that own nodes
  __shared__ uint32_t s_here[NWO];              // and the droplets that they met
  __shared__ double s_cv[NWO][3][64];           // a wavefront's terms of one droplet's sums
  __shared__ uint16_t s_list[NW][TILE_CHUNK];
  T* const s_mu = s_a[0];
  T* const s_X = s_a[1];
  T* const s_ph = s_a[0];
  T* const s_ch = s_a[1];
  T* const s_ux = s_b[0];
  T* const s_uy = s_b[1];
  T* const s_M = s_b[0];
  T* const s_Xh = s_b[1];

  int inst = 0, x0, y0, t;
  if constexpr (MULTI) {
    const TileDev td = tiles[blockIdx.x];
    if (td.inst < 0) return;
    if (DBG && td.inst != export_inst(dbg_inst)) return;
    inst = td.inst;
    x0 = td.x0;
    y0 = td.y0;
    t = td.t;
  }
  const InstDev& I = MULTI ? insts[inst] : one;
  if constexpr (!MULTI) {
    t = xcd_block();
    const int ty = t / I.tiles_x[TILING_TILE];
    x0 = (t - ty * I.tiles_x[TILING_TILE]) * OX;
    y0 = ty * OY;
  }
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nx = I.nx, ny = I.ny, pitch = I.pitch, nd = I.ndrop, walls = I.walls;
  const int64_t plane = I.pstride;
  const T* __restrict__ phi_in = buf + (parity ? I.off_phi[1] : I.off_phi[0]);
  const T* __restrict__ c_in = buf + (parity ? I.off_c[1] : I.off_c[0]);
  const P* __restrict__ fin = reinterpret_cast<const P*>(buf + (parity ? I.off_f[1] : I.off_f[0]));
  P* __restrict__ fout = reinterpret_cast<P*>(buf + (parity ? I.off_f[0] : I.off_f[1]));
  T* __restrict__ phi_out = buf + (parity ? I.off_phi[0] : I.off_phi[1]);
  T* __restrict__ c_out = buf + (parity ? I.off_c[0] : I.off_c[1]);

  // stored column and row of a region's node (the lattice is at least as wide and high as a tile and its rings)
  auto column = [&](int x) { return near_index(x, nx); };
  auto row = [&](int r) { return !walls ? near_index(r, ny) : r < 0 ? -1 - r : (r >= ny ? 2 * ny - 1 - r : r); };

  // ---- the droplets' presence bits, centres and parameters, one wavefront per droplet: the last wavefronts,
  // which have the least to do in the later stages
  const int k0 = NW - 1 - wv;  // this wavefront's (first) droplet
  TileCentre tc;
  DropDev dd0;
  double cx0 = 0.0, cy0 = 0.0;
  if (k0 < nd) {
    dd0 = drops[I.drop_base + k0];
    cx0 = dd0.x;
    cy0 = dd0.y;
    if (q.cen_in) {
      tc.begin(I, q, s_list[wv]);
      cx0 = q.cen_in[2 * (I.drop_base + k0)];
      cy0 = q.cen_in[2 * (I.drop_base + k0) + 1];
    }
  }
  // ---- loads: phi^n, c^n of the tile and five rings, and the populations pulled to the tile and three
  T g_phi[R5], g_c[R5];
#pragma unroll
  for (int j = 0; j < R5; ++j) {
    const int i = tid + j * NT;
    if (i >= W5 * H5) continue;
    const int ly = i / W5, lx = i - ly * W5;
    const unsigned o = (unsigned)(row(y0 + ly - 5) * pitch + column(x0 + lx - 5)) * (unsigned)sizeof(T);
    g_phi[j] = ld_col(phi_in, o);
    g_c[j] = ld_col(c_in, o);
  }
  P pf[R3][9];
  int lx3[R3], ly3[R3];
#pragma unroll
  for (int j = 0; j < R3; ++j) {
    const int i = tid + j * NT;
    if (i >= W3 * H3) continue;
    inner_first<OX, OY, 3>(i, lx3[j], ly3[j]);
    const int gx = column(x0 + lx3[j] - 3), gy = row(y0 + ly3[j] - 3);
    const int gxm = gx == 0 ? nx - 1 : gx - 1, gxp = gx == nx - 1 ? 0 : gx + 1;
    const int r0 = gy * pitch;
    const int rm = gy == 0 ? (ny - 1) * pitch : r0 - pitch, rp = gy == ny - 1 ? 0 : r0 + pitch;
    constexpr unsigned B = sizeof(P);
    const unsigned o0 = (unsigned)(r0 + gx) * B;
    pf[j][0] = ld_col(fin, o0);
    pf[j][1] = ld_col(fin + plane, (unsigned)(r0 + gxm) * B);
    pf[j][3] = ld_col(fin + 3 * plane, (unsigned)(r0 + gxp) * B);
    if (!walls) {
      pf[j][2] = ld_col(fin + 2 * plane, (unsigned)(rm + gx) * B);
      pf[j][4] = ld_col(fin + 4 * plane, (unsigned)(rp + gx) * B);
      pf[j][5] = ld_col(fin + 5 * plane, (unsigned)(rm + gxm) * B);
      pf[j][6] = ld_col(fin + 6 * plane, (unsigned)(rm + gxp) * B);
      pf[j][7] = ld_col(fin + 7 * plane, (unsigned)(rp + gxp) * B);
      pf[j][8] = ld_col(fin + 8 * plane, (unsigned)(rp + gxm) * B);
    } else {
      // behind a plate: the node's own opposite population (halfway bounce-back)
      const bool bb0 = gy == 0, bbn = gy == ny - 1;
      const unsigned pl = (unsigned)plane * B;  // an eligible lattice's nine planes are below 4 GB
      pf[j][2] = ld_col(fin, bb0 ? o0 + 4 * pl : (unsigned)(rm + gx) * B + 2 * pl);
      pf[j][4] = ld_col(fin, bbn ? o0 + 2 * pl : (unsigned)(rp + gx) * B + 4 * pl);
      pf[j][5] = ld_col(fin, bb0 ? o0 + 7 * pl : (unsigned)(rm + gxm) * B + 5 * pl);
      pf[j][6] = ld_col(fin, bb0 ? o0 + 8 * pl : (unsigned)(rm + gxp) * B + 6 * pl);
      pf[j][7] = ld_col(fin, bbn ? o0 + 5 * pl : (unsigned)(rp + gxp) * B + 7 * pl);
      pf[j][8] = ld_col(fin, bbn ? o0 + 6 * pl : (unsigned)(rp + gxm) * B + 8 * pl);
    }
  }
#pragma unroll
  for (int j = 0; j < R5; ++j)
    if (tid + j * NT < W5 * H5) {
      s_phi[tid + j * NT] = g_phi[j];
      s_c[tid + j * NT] = g_c[j];
    }
  __syncthreads();
  const bool follow = k0 < nd && q.cen_in != nullptr;
  if (follow) tc.load(k0);

  // ---- s1: mu_phi and X (Eqs. 3, 5) on the tile and four rings
  const T a = T(I.a), b = T(I.b), B0 = T(I.B0), B1 = T(I.B1), halfB1 = T(I.halfB1);
  const int64_t nplane = (int64_t)nx * ny;
  // whether the node at region position (lx, ly) of a region with `ring` rings is the tile's own
  auto owned = [&](int lx, int ly, int ring) {
    return lx >= ring && lx < OX + ring && ly >= ring && ly < OY + ring && x0 + lx - ring < nx && y0 + ly - ring < ny;
  };
  for (int i = tid; i < W4 * H4; i += NT) {
    const int ly = i / W4, lx = i - ly * W4;
    const int c5 = (ly + 1) * W5 + lx + 1;
    T gpx, gpy, gcx, gcy;
    grad9(s_phi, c5, W5, gpx, gpy);
    grad9(s_c, c5, W5, gcx, gcy);
    const T lp = lap9(s_phi, c5, W5);
    const T ph = s_phi[c5];
    const T B = B0 + B1 * s_c[c5];
    s_mu[i] = ((a * ph + b * (ph * ph * ph)) - B * lp) - B1 * (gpx * gcx + gpy * gcy);
    s_X[i] = halfB1 * (gpx * gpx + gpy * gpy);
    if (DBG && owned(lx, ly, 4)) {
      const int64_t o = (int64_t)(y0 + ly - 4) * nx + (x0 + lx - 4);
      dbg[0 * nplane + o] = (double)s_mu[i];
      dbg[1 * nplane + o] = (double)s_X[i];
    }
  }
  __syncthreads();

  // ---- s2: force (Eq. 14), density and velocity (Eq. 11) on the tile and three rings
  const T omega = T(I.omega), coef = T(I.coef);
  const T w0 = cst<T>(4.0 / 9.0), w1 = cst<T>(1.0 / 9.0), w5 = cst<T>(1.0 / 36.0);
  const T cw0 = coef * w0, cw1 = coef * w1, cw5 = coef * w5;
  const LbConst<T> lbk{w0, w1, w5, cw0, cw1, cw5, omega, T(I.wn[0]), T(I.wn[1]), T(I.wn[2]), T(I.n0)};
  T d0[9], dn0, nn0, ux0, uy0, Fx0, Fy0;
#pragma unroll
  for (int j = 0; j < R3; ++j) {
    if (tid + j * NT >= W3 * H3) continue;
    const int ly = ly3[j], lx = lx3[j], i = ly * W3 + lx;
    const int c4 = (ly + 1) * W4 + lx + 1, c5 = (ly + 2) * W5 + lx + 2;
    T gmx, gmy, gXx, gXy, gcx, gcy;
    grad9(s_mu, c4, W4, gmx, gmy);
    grad9(s_X, c4, W4, gXx, gXy);
    grad9(s_c, c5, W5, gcx, gcy);
    const T ph = s_phi[c5], cv = s_c[c5];
    const T Fx = (-(ph * gmx) - gcx) - cv * gXx;
    const T Fy = (-(ph * gmy) - gcy) - cv * gXy;
    T d[9], dn, nn, ux, uy;
    lb_moments<T, P>(pf[j], lbk, Fx, Fy, d, dn, nn, ux, uy);
    s_ux[i] = ux;
    s_uy[i] = uy;
    if (j == 0) {  // an own node's, for the collision
      for (int k = 0; k < 9; ++k) d0[k] = d[k];
      dn0 = dn;
      nn0 = nn;
      ux0 = ux;
      uy0 = uy;
      Fx0 = Fx;
      Fy0 = Fy;
    }
  }
  if (follow) tc.sum(k0);
  __syncthreads();

  // ---- the centres of mass at n, by the last wavefronts (the very last has nothing else to do here).  Theirs is the
  // longest chain, and the code is theirs alone (its instructions are fetched for them): they go first
  if (k0 < nd) __builtin_amdgcn_s_setprio(3);
  for (int k = k0; k < nd; k += NW) {
    if (k != k0) {
      dd0 = drops[I.drop_base + k];
      cx0 = dd0.x;
      cy0 = dd0.y;
      if (follow) {
        tc.begin(I, q, s_list[wv]);
        cx0 = q.cen_in[2 * (I.drop_base + k)];
        cy0 = q.cen_in[2 * (I.drop_base + k) + 1];
        tc.load(k);
        tc.sum(k);
      }
    }
    if (follow) tc.move(I, cx0, cy0);
    if (lane == 0) {
      if (t == I.tile_base[TILING_TILE]) {
        q.cen_out[2 * (I.drop_base + k)] = cx0;
        q.cen_out[2 * (I.drop_base + k) + 1] = cy0;
      }
      const double px = cx0 + (dd0.R - dd0.Rs) * dd0.ex, py = cy0 + (dd0.R - dd0.Rs) * dd0.ey;
      s_d[k][0] = cx0;
      s_d[k][1] = cy0;
      s_d[k][2] = px;
      s_d[k][3] = py;
      s_d[k][4] = dd0.Rs * dd0.Rs;
      const double hx = 0.5 * (OX - 1), hy = 0.5 * (OY - 1);
      const double sdx = fmax(0.0, fabs(minimg(x0 + hx - px, (double)nx)) - hx);
      const double sdy = fmax(0.0, fabs(minimg(y0 + hy - py, I.yper)) - hy);
      const double rr = dd0.Rs + 1e-6;
      s_src[k] = dd0.active && sdx * sdx + sdy * sdy <= rr * rr;
    }
  }
  if (k0 < nd) __builtin_amdgcn_s_setprio(0);

  constexpr int S3 = NT - (W2 * H2 + 63) / 64 * 64 - 64;
  static_assert(S3 >= 0 && OX * OY < NT, "the last wavefront has no part of the collision and of s3");
  constexpr int FIRST3 = S3 < OX * OY ? S3 : OX * OY;
  const int adv = I.advection;
  if (__builtin_amdgcn_readfirstlane(wv) != NW - 1) {
    // ---- collision (Eqs. 10, 12, 13) on the tile, by the first wavefronts while the others take s3
    if (const int x = x0 + lx3[0] - 3, y = y0 + ly3[0] - 3; tid < OX * OY && x < nx && y < ny) {
      P out[9];
      double sv[9];
      lb_collide<T, P>(d0, dn0, nn0, ux0, uy0, Fx0, Fy0, lbk, out, sv);
      const unsigned o = (unsigned)(y * pitch + x) * (unsigned)sizeof(P);
      for (int k = 0; k < 9; ++k) st_col(fout + k * plane, o, out[k]);
      if (DBG) {
        const int64_t g = (int64_t)y * nx + x;
        dbg[2 * nplane + g] = (double)Fx0;
        dbg[3 * nplane + g] = (double)Fy0;
        dbg[4 * nplane + g] = (double)nn0;
        dbg[5 * nplane + g] = (double)ux0;
        dbg[6 * nplane + g] = (double)uy0;
        if (export_all(dbg_inst))
          for (int k = 0; k < 9; ++k) dbg[(13 + k) * nplane + g] = sv[k];
      }
    }

    // ---- s3: advection half-step (Eqs. 16-17) on the tile and two rings
    for (int i = (tid + NT - FIRST3) % NT; i < W2 * H2; i += NT) {
      const int ly = i / W2, lx = i - ly * W2;
      const int c3 = (ly + 1) * W3 + lx + 1, c5 = (ly + 3) * W5 + lx + 3;
      const int r = y0 + ly - 2;
      const T uc = s_ux[c3], ue = s_ux[c3 + 1], uw = s_ux[c3 - 1], vc = s_uy[c3];
      // beyond a plate: the mirror image of the boundary row, with u_y reversed
      const T vn = (walls && r == ny - 1) ? -vc : s_uy[c3 + W3];
      const T vs = (walls && r == 0) ? -vc : s_uy[c3 - W3];
      s_ph[i] = advect_n(s_phi[c5], s_phi[c5 + 1], s_phi[c5 - 1], s_phi[c5 + W5], s_phi[c5 - W5], uc, ue, uw, vc, vn, vs,
                         adv);
      s_ch[i] = advect_n(s_c[c5], s_c[c5 + 1], s_c[c5 - 1], s_c[c5 + W5], s_c[c5 - W5], uc, ue, uw, vc, vn, vs, adv);
      if (DBG && owned(lx, ly, 2)) {
        const int64_t o = (int64_t)r * nx + (x0 + lx - 2);
        dbg[7 * nplane + o] = (double)s_ph[i];
        dbg[8 * nplane + o] = (double)s_ch[i];
      }
    }
  }
  __syncthreads();

  // ---- s4: bracket M of Eq. (18) and X^{n+1/2} on the tile and one ring
  for (int i = tid; i < W1 * H1; i += NT) {
    const int ly = i / W1, lx = i - ly * W1;
    const int c5 = (ly + 4) * W5 + lx + 4;
    const int r = y0 + ly - 1;
    // half-step fields beyond a plate: the mirror image of the boundary row
    const int m = (ly + 1) * W2, up = (walls && r == ny - 1) ? m : m + W2, dn = (walls && r == 0) ? m : m - W2;
    T gphx, gphy, gchx, gchy;
    grad9r(s_ph + up, s_ph + m, s_ph + dn, lx + 1, gphx, gphy);
    grad9r(s_ch + up, s_ch + m, s_ch + dn, lx + 1, gchx, gchy);
    const T lph = lap9r(s_ph + up, s_ph + m, s_ph + dn, lx + 1);
    const T pn = s_phi[c5];
    const T Bh = B0 + B1 * s_ch[m + lx + 1];
    const T M = ((a * s_ph[m + lx + 1] + b * (pn * pn * pn)) - Bh * lph) - B1 * (gchx * gphx + gchy * gphy);
    const T Xh = halfB1 * (gphx * gphx + gphy * gphy);
    s_M[i] = M;
    s_Xh[i] = Xh;
    if (DBG && owned(lx, ly, 1)) {
      const int64_t o = (int64_t)r * nx + (x0 + lx - 1);
      if (export_all(dbg_inst)) dbg[PLANE_M * nplane + o] = (double)M;
      dbg[PLANE_XH * nplane + o] = (double)Xh;
    }
  }
  __syncthreads();

  // ---- s5: phi^{n+1}, c^{n+1} (Eqs. 18, 19) on the tile, and the centre-of-mass sums (Sec. 4)
  const T Gamma = T(I.Gamma), D = T(I.D), gam = T(I.gamma), c0 = T(I.c0);
  const double tn = (double)(*step + q.ahead);
  const double A = I.A0 * (tn < I.t_star ? tn : I.t_star);
  // phi and the sums by the first OX x OY threads, c by the next
  static_assert(2 * OX * OY <= NT && OX * OY % 64 == 0, "two threads per node, in wavefronts of their own");
  const int own = tid < OX * OY ? tid : tid - OX * OY;
  const int lyo = own / OX, lxo = own - lyo * OX, xo = x0 + lxo, ro = y0 + lyo;
  const bool valid = tid < 2 * OX * OY && xo < nx && ro < ny;
  const bool top = walls && ro == ny - 1, bot = walls && ro == 0;
  const int m1 = (lyo + 1) * W1, m2 = (lyo + 2) * W2 + 1;
  const int u1 = top ? m1 : m1 + W1, d1 = bot ? m1 : m1 - W1, u2 = top ? m2 : m2 + W2, d2 = bot ? m2 : m2 - W2;
  const double xd = (double)xo, yd = (double)ro;
  const unsigned oo = (unsigned)(ro * pitch + xo) * (unsigned)sizeof(T);
  int kd = -1;
  double cv0 = 0.0, cv1 = 0.0, cv2 = 0.0;
  if (valid && tid >= OX * OY) {
    const T ch = s_ch[m2 + lxo + 1];
    const T lch = lap9r(s_ch + u2, s_ch + m2, s_ch + d2, lxo + 1);
    const T dv = div9r(s_ch + u2, s_ch + m2, s_ch + d2, D, s_Xh + u1, s_Xh + m1, s_Xh + d1, lxo + 1);
    int cnt = 0;
    for (int k = 0; k < nd; ++k)
      if (s_src[k]) {
        const double dx = minimg(xd - s_d[k][2], (double)nx), dy = minimg(yd - s_d[k][3], I.yper);
        if (dx * dx + dy * dy <= s_d[k][4]) ++cnt;
      }
    const double src = A * (double)cnt;
    const T cn = (((ch + D * lch) + dv) - gam * (ch - c0)) + T(src);
    st_col(c_out, oo, cn);
    if (DBG && export_all(dbg_inst)) dbg[12 * nplane + (int64_t)ro * nx + xo] = (double)cn;
  } else if (valid) {
    const T phn = s_ph[m2 + lxo + 1] + Gamma * lap9r(s_M + u1, s_M + m1, s_M + d1, lxo + 1);
    st_col(phi_out, oo, phn);
    if (DBG && export_all(dbg_inst)) dbg[11 * nplane + (int64_t)ro * nx + xo] = (double)phn;
    const double v = (double)phn;
    if (nd > 0 && v >= 0.0) {
      // nearest centre, the lowest index on ties
      int best = 0;
      double bx = minimg(xd - s_d[0][0], (double)nx), by = minimg(yd - s_d[0][1], I.yper);
      double bd = bx * bx + by * by;
      for (int k = 1; k < nd; ++k) {
        const double dx = minimg(xd - s_d[k][0], (double)nx), dy = minimg(yd - s_d[k][1], I.yper);
        const double dd = dx * dx + dy * dy;
        if (dd < bd) {
          best = k;
          bd = dd;
          bx = dx;
          by = dy;
        }
      }
      kd = best;
      cv0 = v;
      cv1 = v * bx;
      cv2 = v * by;
    }
  }
  if (nd == 0) return;
  if (wv < NWO) {
    uint32_t here = 0u;
    for (int k = 0; k < nd; ++k) {
      const bool mine = kd == k;
      if (__ballot(mine) == 0ull) continue;
      here |= 1u << k;
      // as in TileCentre: a row of lanes for each sum, four nodes to a lane
      s_cv[wv][0][lane] = mine ? cv0 : 0.0;
      s_cv[wv][1][lane] = mine ? cv1 : 0.0;
      s_cv[wv][2][lane] = mine ? cv2 : 0.0;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int i = lane >> 4;
      const double* const t = s_cv[wv][min(i, 2)] + (lane & 15);
      Dd s[1] = {{t[0], 0.0}};
      for (int u = 1; u < 4; ++u) dd_add(s[0], t[16 * u]);
      dd_row_sum(s);
      if (i < 3 && (lane & 15) == 15) {
        s_sum[wv][k][2 * i] = s[0].hi;
        s_sum[wv][k][2 * i + 1] = s[0].lo;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (lane == 0) s_here[wv] = here;
  }
  __syncthreads();
  uint32_t present = 0u;
  for (int w = 0; w < NWO; ++w) present |= s_here[w];
  if (tid == 0) q.mask_out[t] = present;
  if (tid < 3 * nd && ((present >> (tid / 3)) & 1u)) {
    const int k = tid / 3, j = tid - 3 * k;
    Dd z{0.0, 0.0};
    for (int w = 0; w < NWO; ++w)
      if ((s_here[w] >> k) & 1u) dd_add(z, Dd{s_sum[w][k][2 * j], s_sum[w][k][2 * j + 1]});
    double* const pt = q.part_out + I.part_base[TILING_TILE] + ((int64_t)(t - I.tile_base[TILING_TILE]) * nd + k) * 6;
    pt[2 * j] = z.hi;
    pt[2 * j + 1] = z.lo;
  }
}

// After the last step of a sequence: the centres from that step's sums, into the droplet table, and the step
// counter.  One wavefront per droplet.  count 0: computes and writes nothing (timing).
__global__ __launch_bounds__(64) void k_tile_final(int ndrop_total, const InstDev* __restrict__ insts,
                                                   DropDev* __restrict__ drops, TileSeq q, int64_t* __restrict__ step,
                                                   int64_t count) {
  const int g = blockIdx.x;
  if (g == 0 && threadIdx.x == 0 && count > 0) *step = *step + count;
  if (g >= ndrop_total) return;
  const InstDev& I = insts[drops[g].inst];
  __shared__ uint16_t list[TILE_CHUNK];
  const int k = g - I.drop_base;
  double cx = q.cen_in[2 * g], cy = q.cen_in[2 * g + 1];
  TileCentre tc;
  tc.begin(I, q, list);
  tc.load(k);
  tc.sum(k);
  tc.move(I, cx, cy);
  if (threadIdx.x == 0 && count > 0) {
    drops[g].x = cx;
    drops[g].y = cy;
  }
}

}  // namespace

template <typename T, typename P, int OX, int OY, int NT>
hipError_t launch_tile_sized(hipStream_t s, int parity, int ntiles_launch, const InstDev* one, const TileDev* tiles,
                             const InstDev* insts, T* buf, const DropDev* drops, const TileSeq& q, const int64_t* step,
                             double* dbg, int dbg_inst) {
  const dim3 g(ntiles_launch), b(NT);
  if (one && dbg)
    hipLaunchKernelGGL((k_tile<T, P, OX, OY, NT, true, false>), g, b, 0, s, parity, *one, tiles, insts, buf, drops, q, step,
                       dbg, dbg_inst);
  else if (one)
    hipLaunchKernelGGL((k_tile<T, P, OX, OY, NT, false, false>), g, b, 0, s, parity, *one, tiles, insts, buf, drops, q,
                       step, dbg, dbg_inst);
  else if (dbg)
    hipLaunchKernelGGL((k_tile<T, P, OX, OY, NT, true, true>), g, b, 0, s, parity, InstDev{}, tiles, insts, buf, drops, q,
                       step, dbg, dbg_inst);
  else
    hipLaunchKernelGGL((k_tile<T, P, OX, OY, NT, false, true>), g, b, 0, s, parity, InstDev{}, tiles, insts, buf, drops, q,
                       step, dbg, dbg_inst);
  return hipGetLastError();
}

template <typename T, typename P>
hipError_t launch_tile(hipStream_t s, int parity, int shape, int ntiles_launch, const InstDev* one,
                       const TileDev* tiles, const InstDev* insts, T* buf, const DropDev* drops, const TileSeq& q,
                       const int64_t* step, double* dbg, int dbg_inst) {
  if (ntiles_launch <= 0) return hipSuccess;
  auto go = [&](auto launch) {
    return launch(s, parity, ntiles_launch, one, tiles, insts, buf, drops, q, step, dbg, dbg_inst);
  };
  static_assert(TILE_NSHAPES == 3, "one launch per shape");
  constexpr TileShape A = TILE_SHAPES[0], B = TILE_SHAPES[1], C = TILE_SHAPES[2];
  switch (shape) {
    case 0: return go(launch_tile_sized<T, P, A.ox, A.oy, A.threads>);
    case 1: return go(launch_tile_sized<T, P, B.ox, B.oy, B.threads>);
    default: return go(launch_tile_sized<T, P, C.ox, C.oy, C.threads>);
  }
}

#define LBM_INSTANTIATE_TILE(T, P)                                                                                   \
  template hipError_t launch_tile<T, P>(hipStream_t, int, int, int, const InstDev*, const TileDev*, const InstDev*, \
                                        T*, const DropDev*, const TileSeq&, const int64_t*, double*, int);

}  // namespace lbm
