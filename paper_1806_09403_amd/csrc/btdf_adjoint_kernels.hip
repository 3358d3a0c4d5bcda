// btdf_adjoint_kernels.hip -- gfx950 kernels of the reverse (adjoint) step.
//
// One forward step maps the post-collision populations A_t to A_{t+1} and
// emits the body forces of eq 27. Its adjoint, for a scalar J built from the
// force history, maps dJ/dA_{t+1} to dJ/dA_t and adds the step's share of
// the parameter gradients. The state of the reverse sweep is kept in the
// form of the streamed populations: G_t = dJ/dg_t, g being the populations
// after the streaming pull of step t. dJ/dA_t is never stored: it is read
// from G_t by the transpose of the pull (pull_adj), which has the same
// shifted-read pattern as the forward pull, so the lattice kernel writes its
// planes aligned, one node per thread, as the forward lattice kernel does.
//
// Per reversed step, with the step's marker values (weights, drs ds F_l,
// rho_l, u*_l) recorded by the forward step:
//   adj_markers  16 lanes per marker, one per stencil node: each lane forms at
//                its node the forward values and dJ/df (the transposed
//                collision, as a tile does), then the marker's transposes of
//                spreading (eqs 13, 15) and eq 27 -> dJ/dF_l, of the direct
//                force (eq 20) -> dJ/drho_l, dJ/du*_l, and the position (phi')
//                and marker-velocity gradients.
//   adj_tile     64 x 4 nodes: dJ/dA_{t+1} by pull_adj (plus the channel ghost
//                columns), the transposed collision (eqs 5-7, 11) and, at
//                nodes a marker stencil covers, the transposed interpolation
//                (eqs 12, 14) of the markers' dJ/drho_l, dJ/du*_l -> G_t;
//                per-tile sums of dJ/dG and dJ/du_in.
//
// A step of a small lattice is bound by latency: a launch, then the chain of
// dependent reads of a marker (its values, the body's and the node's, the
// covering markers' weights) and of a tile that needs its results. So only
// the tiles a stencil touches wait for the markers; the others are shared out
// between both launches; a tile's populations are in flight before it stages
// its markers, and a node visits its own markers only, by a mask of bits. A
// reversed step of the 800x400 channel (126 markers) takes 15.5 us in FP32,
// with all tiles behind the markers, one pass over the tile's whole list per
// node and a marker's reads where they are used 23.4 (FP64: 21.7, was 27.4);
// of the 200x120 channel 12.7 (FP64 13.5), was 17.5 (18.0).
// After the last reversed step adj_unpull_kernel turns G_0 into dJ/dA_0.
#include <algorithm>

#include "btdf_device.h"
#include "btdf_launch.h"
#include "btdf_tile.h"

namespace btdf {

constexpr int kAdjChunk = 64;  // markers staged in LDS per pass
// Up to this many tiles untouched by stencils are shared out between the
// markers' launch and that of the tiles that wait for them. Beyond it, all but
// kAdjBeside in each have a launch of their own, whose fewer registers keep
// more loads in flight. A reversed step, shared out / with the third launch:
// 2048x1024 FP64 93.3 / 93.8 us (and 100.6 with the tiles undivided behind
// the markers), 4096x1024 FP64 174 / 188, 4096x1536 FP32 143 / 150, FP64
// 262 / 272, 4096x2048 FP32 188 / 188, FP64 374 / 354.
constexpr int kAdjApart = 28000, kAdjBeside = 1024;

// Transpose of the streaming pull, read as a pull: the adjoint of A_q at
// node (x, y) is G_q of the fluid node that read it -- the neighbour
// (x, y) + e_q, or next to a wall the bounce-back of (x, y) itself in the
// opposite direction -- and 0 when no fluid node reads it.
template <typename T>
__device__ __forceinline__ T pull_adj(const T *__restrict__ G, const LbmParams &p, int q, int x, int y) {
  int zx = x + ex(q), zy = y + ey(q);
  if (p.yper) {
    zy = zy < 0 ? zy + p.ny : (zy >= p.ny ? zy - p.ny : zy);
  } else if (zy < 0 || zy >= p.ny) {
    if (x < p.i0 || x > p.i1) return (T)0;
    return G[(long long)opp(q) * p.plane + (long long)y * p.pitch + x];
  }
  if (p.xper)
    zx = zx < 0 ? zx + p.nx : (zx >= p.nx ? zx - p.nx : zx);
  else if (zx < p.i0 || zx > p.i1)
    return (T)0;
  return G[(long long)q * p.plane + (long long)zy * p.pitch + zx];
}

// All nine of them at node (x, y) of the grid, each one load from a held
// address and a selection, so that all are in flight together.
template <typename T>
__device__ __forceinline__ void pull_adj9(const T *__restrict__ G, const LbmParams &p, int x, int y, T (&b)[9]) {
  int col[3] = {x - 1, x, x + 1}, row[3] = {y - 1, y, y + 1};
  bool in[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    in[k] = p.xper || (col[k] >= p.i0 && col[k] <= p.i1);
    col[k] = col[k] < 0 ? (p.xper ? p.nx - 1 : 0) : (col[k] >= p.nx ? (p.xper ? 0 : p.nx - 1) : col[k]);
    row[k] = row[k] < 0 ? (p.yper ? p.ny - 1 : 0) : (row[k] >= p.ny ? (p.yper ? 0 : p.ny - 1) : row[k]);
  }
#pragma unroll
  for (int q = 0; q < 9; ++q)
    b[q] = ldg(G + (long long)q * p.plane, (long long)row[1 + ey(q)] * p.pitch + col[1 + ex(q)]);
#pragma unroll
  for (int q = 0; q < 9; ++q) b[q] = in[1 + ex(q)] ? b[q] : (T)0;
  if (!p.yper && (y == 0 || y == p.ny - 1)) {
    const bool fluid = x >= p.i0 && x <= p.i1;
#pragma unroll
    for (int q = 2; q < 9; ++q) {
      if (ey(q) == 0 || y != (ey(q) < 0 ? 0 : p.ny - 1)) continue;
      b[q] = fluid ? ldg(G + (long long)opp(q) * p.plane, (long long)y * p.pitch + x) : (T)0;
    }
  }
}

// Forward values at fluid node (x, y) from the streamed deviations g and the
// total force f (eqs 9-11): rho, the full first moment m, u = (m + f/2)/rho.
struct NodeFwd {
  double rho, mx, my, ux, uy;
};
template <typename Gv>
__device__ __forceinline__ NodeFwd node_forward(const Gv gv[9], double ftx, double fty, const LbmParams &p) {
  NodeFwd n;
  double g[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) g[q] = (double)gv[q];
  const double drho = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
  n.rho = 1.0 + drho;
  // stored values are deviations from feq(1, u_ref): their first moment is m - u_ref
  n.mx = ((g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7])) + p.urx;
  n.my = ((g[2] - g[4]) + (g[5] - g[8]) + (g[6] - g[7])) + p.ury;
  n.ux = (n.mx + 0.5 * ftx) / n.rho;
  n.uy = (n.my + 0.5 * fty) / n.rho;
  return n;
}

// dJ/dB at fluid node (x, y): the transpose of the next step's pull, plus
// the zero-gradient outlet's ghost column, B(nx-1, y) = B(nx-2, y).
template <typename T>
__device__ __forceinline__ void pull_dJdB(const T *__restrict__ Gn, const LbmParams &p, int x, int y, T (&bb)[9]) {
  pull_adj9<T>(Gn, p, x, y, bb);
  if (p.outlet && x == p.nx - 2) {
    T c[9];
    pull_adj9<T>(Gn, p, x + 1, y, c);
#pragma unroll
    for (int q = 0; q < 9; ++q) bb[q] += c[q];
  }
}

// Weighted moments of dJ/dB at a node: s0 = sum w b, s1 = sum w b e,
// S2 = sum w b e e (the transposed collision needs no more of dJ/dB).
struct Mom {
  double s0 = 0.0, s1x = 0.0, s1y = 0.0, Sxx = 0.0, Sxy = 0.0, Syy = 0.0;
  __device__ __forceinline__ void add(int q, double bq) {
    const double w = wq(q);
    s0 = fma(w, bq, s0);
    if (ex(q)) s1x = fma(ex(q) * w, bq, s1x);
    if (ey(q)) s1y = fma(ey(q) * w, bq, s1y);
    if (ex(q)) Sxx = fma(w, bq, Sxx);
    if (ex(q) * ey(q)) Sxy = fma(ex(q) * ey(q) * w, bq, Sxy);
    if (ey(q)) Syy = fma(w, bq, Syy);
  }
  // the same shift added to every direction: sum w = 1, sum w e = 0, sum w e e = I/3
  __device__ __forceinline__ void add_uniform(double c) {
    s0 += c;
    Sxx += c / 3.0;
    Syy += c / 3.0;
  }
};

// Transpose of out_q = (1 - omega) g_q + omega feq_q(rho, u) + F_q(u, f),
// u = (m + f/2) / rho (eqs 5-7, 11), at one node, from the moments of
// dJ/dB. Gives dJ/df and the parts of dJ/dg_q = (1 - omega) b_q + drb + e_q.mb.
// The fused operations are spelled out, here and below: the sums cancel, so
// that the last bits of a gradient would otherwise depend on what the compiler
// fuses where. (A marker's nodes add the two parts of dJ/du_x the other way.)
struct CollideAdj {
  double fbx, fby, drb, mbx, mby;
};
template <bool MARKER>
__device__ __forceinline__ CollideAdj collide_adjoint(const NodeFwd &n, double ftx, double fty, const Mom &m,
                                                      const LbmParams &p) {
  const double omega = p.omega, guo = p.guo, ux = n.ux, uy = n.uy, inv = 1.0 / n.rho;
  const double Sux = fma(m.Sxy, uy, ux * m.Sxx), Suy = fma(m.Sxy, ux, uy * m.Syy);      // S2 u
  const double Sfx = fma(fty, m.Sxy, ftx * m.Sxx), Sfy = fma(ftx, m.Sxy, fty * m.Syy);  // S2 f
  const double su = fma(m.s1x, ux, m.s1y * uy), uSu = fma(uy, Suy, ux * Sux), uu = fma(ux, ux, uy * uy);
  // d/d rho at fixed u (times omega below)
  const double dr = fma(-1.5 * uu, m.s0, fma(4.5, uSu, fma(3.0, su, m.s0)));
  const double orho = omega * n.rho, ax = (3.0 * ux) * m.s0, ay = (3.0 * uy) * m.s0;
  const double eqx = fma(-(3.0 * ux), m.s0, fma(3.0, m.s1x, 9.0 * Sux));
  const double eqy = fma(-(3.0 * uy), m.s0, fma(3.0, m.s1y, 9.0 * Suy));
  const double gx = fma(Sfx, 9.0, -((3.0 * ftx) * m.s0)), gy = fma(Sfy, 9.0, -((3.0 * fty) * m.s0));
  const double ubx = MARKER ? fma(orho, eqx, guo * gx) : fma(guo, gx, orho * eqx);
  const double uby = fma(guo, gy, orho * eqy);
  CollideAdj r;
  r.mbx = ubx * inv;
  r.mby = uby * inv;
  r.fbx = fma(guo, fma(9.0, Sux, fma(m.s1x, 3.0, -ax)), 0.5 * r.mbx);
  r.fby = fma(guo, fma(9.0, Suy, fma(m.s1y, 3.0, -ay)), 0.5 * r.mby);
  r.drb = fma(omega, dr, -(inv * fma(uy, uby, ux * ubx)));
  return r;
}

// Sum over a wave, in lane 0, in the order of a reduction over lane distances
// 32, 16, then 8, 4, 2, 1.
__device__ __forceinline__ double wave_total(double v) {
  v += __shfl_down(v, 32, 64);
  v += __shfl_down(v, 16, 64);
  return row_sum(v);
}

// Sum over a marker's 16 lanes of the products a b, in every lane, over lane
// distances 8, 4, 2, 1; a lane's own product enters its first sum unrounded.
// (Lanes 8 apart then differ in the last bit, so the lane 4 apart is taken
// itself -- mirrored within eight lanes, then within four -- and not the one
// a rotation by 4 gives.)
__device__ __forceinline__ double lanes_dot(double a, double b) {
  const double ab = a * b;
  double v = fma(a, b, dpp<0x128>(ab));
  v += dpp<0x1B>(dpp<0x141>(v));
  v += dpp<0x4E>(v);
  v += dpp<0xB1>(v);
  return v;
}

// 16 markers of the workgroup, 16 lanes each, one per node of the up to 4 x 4
// stencil; every lane runs the sums, inactive lanes with zeros. What a marker
// needs is read in three rounds, each in flight at once: its own values and the
// sums it adds to; the body's weights, the list of markers covering the node
// and both fields there; the covering markers' weights.
template <typename T>
__device__ __forceinline__ void adj_markers(const T *__restrict__ A, const T *__restrict__ Gn, const LbmParams &p,
                                            const IbParams &ib, const AdjParams &a, int block) {
  const int tid = (int)threadIdx.x;
  const int mk = block * 16 + (tid >> 4);
  const int lane = tid & 15;
  const bool act = mk < ib.nm;
  const int l = act ? mk : ib.nm - 1;
  const int S = stencil_size(p.kind);
  const int i = lane & 3, j = lane >> 2;
  const double X = ldg(ib.X, l), Y = ldg(ib.Y, l);
  const int c0 = ldg(a.node_off, 16 * l + lane), c1 = ldg(a.node_off, 16 * l + lane + 1);
  const int b = ldg(ib.mk_body, l);
  const double s = ldg(ib.sdrs, l), U = ldg(ib.U, l), V = ldg(ib.V, l);
  const double Fx = ldg(a.Fx, l), Fy = ldg(a.Fy, l), rl = ldg(a.rho_l, l), ul = ldg(a.ux_l, l), vl = ldg(a.uy_l, l);
  typedef double pair __attribute__((ext_vector_type(2)));
  const pair xy0 = ldg(reinterpret_cast<const pair *>(a.xy_bar), l);
  const pair uv0 = ldg(reinterpret_cast<const pair *>(a.uv_bar), l);
  const pair c0b = ldg(reinterpret_cast<const pair *>(a.c_bar), l);

  const int bx = stencil_base(p.kind, X), by = stencil_base(p.kind, Y);
  const bool on = act && i < S && j < S;
  constexpr int kCover = sizeof(T) == 8 ? 2 : 4;  // covering markers in flight
  int e[kCover];
  T g[9], bb[9];
  int xx = 0, yy = 0;
  const double hx = ldg(a.hist_bar, 3 * b), hy = ldg(a.hist_bar, 3 * b + 1), hz = ldg(a.hist_bar, 3 * b + 2);
  const double cx = ldg(ib.cx, b), cy = ldg(ib.cy, b);
  double W = 0.0, dWx = 0.0, dWy = 0.0, fbx = 0.0, fby = 0.0, rk = 1.0, usx = 0.0, usy = 0.0;
  if (on) {
    // (the marker itself covers the node, so c1 > c0)
#pragma unroll
    for (int u = 0; u < kCover; ++u) e[u] = ldg(a.node_list, min(c0 + u, c1 - 1));
    xx = bx + i;
    yy = by + j;
    if (p.xper) xx = wrap_index(xx, p.nx);
    if (p.yper) yy = wrap_index(yy, p.ny);
    // the node's forward values and dJ/df, as the lattice tiles form them
    pull9<T>(A, p, xx, yy, g);
    pull_dJdB<T>(Gn, p, xx, yy, bb);
    const double rx = (double)(bx + i) - X, ry = (double)(by + j) - Y;
    const double px = phi(p.kind, rx), py = phi(p.kind, ry);
    W = px * py;
    dWx = -dphi(p.kind, rx) * py;  // d W / d X
    dWy = -px * dphi(p.kind, ry);  // d W / d Y
    if (p.inlet && xx == 1) {
      // the inlet ghost's density (the density of this node) adds one shift
      // to every direction
      const double ui = p.uin_x, vi = p.uin_y, uui = ui * ui + vi * vi;
      T gh[9];
      pull_adj9<T>(Gn, p, 0, yy, gh);
      double rbB = 0.0;
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const double eu = ex(q) * ui + ey(q) * vi;
        rbB += (double)gh[q] * wq(q) * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uui);
      }
#pragma unroll
      for (int q = 0; q < 9; ++q) bb[q] = (T)((double)bb[q] + rbB);
    }
    // the spread force, as the forward step formed it: the recorded weights and
    // drs ds F of the markers covering the node, in ascending order in the
    // population type
    const T *mw = reinterpret_cast<const T *>(p.mk_w);
    T sfx = (T)0, sfy = (T)0;
    for (int c = c0;;) {
      T w0[kCover], w1[kCover], f0[kCover], f1[kCover];
#pragma unroll
      for (int u = 0; u < kCover; ++u) {
        const T *w = mw + 10 * (long long)(e[u] >> 4);
        w0[u] = ldg(w, (e[u] >> 2) & 3);
        w1[u] = ldg(w, 4 + (e[u] & 3));
        f0[u] = ldg(w, 8);
        f1[u] = ldg(w, 9);
      }
#pragma unroll
      for (int u = 0; u < kCover; ++u) {
        const T Wk = w0[u] * w1[u], ax = fmx(Wk, f0[u], sfx), ay = fmx(Wk, f1[u], sfy);
        sfx = c + u < c1 ? ax : sfx;
        sfy = c + u < c1 ? ay : sfy;
      }
      c += kCover;
      if (c >= c1) break;
#pragma unroll
      for (int u = 0; u < kCover; ++u) e[u] = ldg(a.node_list, min(c + u, c1 - 1));
    }
    const double ftx = (double)(T)(p.Gx + (double)sfx), fty = (double)(T)(p.Gy + (double)sfy);
    const NodeFwd nf = node_forward(g, ftx, fty, p);
    Mom mo;
#pragma unroll
    for (int q = 0; q < 9; ++q) mo.add(q, (double)bb[q]);
    const CollideAdj ca = collide_adjoint<true>(nf, ftx, fty, mo, p);
    fbx = ca.fbx;
    fby = ca.fby;
    rk = nf.rho;
    usx = (nf.mx + 0.5 * p.Gx) / nf.rho;  // u* = (m + G/2) / rho
    usy = (nf.my + 0.5 * p.Gy) / nf.rho;
  }
  // spreading (eqs 13, 15): dJ/dF_l = drs ds sum_k W_lk dJ/df_k
  const double SX = lanes_dot(W, fbx), SY = lanes_dot(W, fby);
  // eq 27: F_b = -s sum F_l, T_b = -s sum (X_l - c) x F_l
  const double sh = s * hz;
  const double Fbx = fma(sh, Y - cy, fma(SX, s, -(s * hx)));
  const double Fby = fma(-sh, X - cx, fma(SY, s, -(s * hy)));
  // eq 20: F_l = 2 rho_l (U_l - u*_l)
  const double rlb = 2.0 * fma(Fbx, U - ul, Fby * (V - vl));
  const double ulb = -2.0 * rl * Fbx, vlb = -2.0 * rl * Fby;
  // positions: the weights of the spreading and of the interpolation move with X_l
  const double term = on ? fma(usy, vlb, fma(usx, ulb, fma(s, fma(fbx, Fx, fby * Fy), rk * rlb))) : 0.0;
  const double PX = lanes_dot(dWx, term), PY = lanes_dot(dWy, term);
  if (act && lane == 0) {
    reinterpret_cast<pair *>(a.xy_bar)[l] = pair{xy0.x + fma(-sh, Fy, PX), xy0.y + fma(sh, Fx, PY)};
    reinterpret_cast<pair *>(a.uv_bar)[l] = pair{fma(2.0 * rl, Fbx, uv0.x), fma(2.0 * rl, Fby, uv0.y)};
    // the body centre enters the torque only
    reinterpret_cast<pair *>(a.c_bar)[l] = pair{fma(sh, Fy, c0b.x), fma(-sh, Fx, c0b.y)};
    a.mk_adj[3 * l] = rlb;
    a.mk_adj[3 * l + 1] = ulb;
    a.mk_adj[3 * l + 2] = vlb;
  }
}

// One tile of the reversed step. FORCED: markers' stencils touch it.
//
// Loads and stores are in the population type; the arithmetic is FP64
// whatever it is: the gradients of interest are sums of large terms that
// cancel (the isotropic part of dJ/dB drops out of every moment), and a tile
// is bound by memory and its latency, not by the FP64 rate.
template <typename T, bool FORCED>
__device__ __forceinline__ void adj_tile(const T *__restrict__ A, const T *__restrict__ Gn, T *__restrict__ Go,
                                         const LbmParams &p, const AdjParams &a, int t) {
  const int tyi = t / a.ntx, txi = t - tyi * a.ntx;
  const int tid = (int)threadIdx.x;
  const int x0 = txi * kAdjTX, y0 = tyi * kAdjTY;
  const int x = x0 + (tid & (kAdjTX - 1)), y = y0 + tid / kAdjTX;
  const bool inlet = p.inlet && txi == 0;  // the tile may hold column 1
  // the tile's running sums: thread k keeps the k-th
  const double sum0 = tid < 4 ? ldg(a.part, 4 * (long long)t + tid) : 0.0;

  // Both fields of the node first, so that they are in flight while the tile
  // gathers its markers' values. A tile whose nodes and their neighbours need
  // no wrap, no wall and no ghost column (tile-uniform test) reads by direct
  // offsets; the other tiles take the general pulls.
  const bool fluid = y < p.ny && x < p.nx && x >= p.i0 && x <= p.i1;
  const bool inner = x0 - 1 >= p.i0 && x0 + kAdjTX <= p.i1 && y0 >= 1 && y0 + kAdjTY <= p.ny - 1;
  const long long node = (long long)y * p.pitch + x;
  T av[9], bb[9];
  if (inner) {
#pragma unroll
    for (int q = 0; q < 9; ++q)
      av[q] = ldg(A, (long long)q * p.plane + node - (long long)ey(q) * p.pitch - ex(q));
#pragma unroll
    for (int q = 0; q < 9; ++q)
      bb[q] = ldg(Gn, (long long)q * p.plane + node + (long long)ey(q) * p.pitch + ex(q));
  } else if (fluid) {
    pull9<T>(A, p, x, y, av);
    pull_dJdB<T>(Gn, p, x, y, bb);
  }

  // over the markers listed for the tile, in ascending order: the spread force
  // at the node as the forward step formed it, and the interpolation weights
  // applied to the markers' dJ/drho_l, dJ/du*_l. 16 lanes stage a marker and
  // mark the nodes of the tile it covers (one bit per marker), so that a node
  // visits its own markers only.
  T fibx = (T)0, fiby = (T)0;
  double Pr = 0.0, Pu = 0.0, Pv = 0.0;
  if constexpr (FORCED) {
    static_assert(kAdjChunk <= 64, "one bit per marker");
    __shared__ int s_ix[kAdjChunk], s_iy[kAdjChunk];
    __shared__ T s_w[kAdjChunk][10];
    __shared__ double s_a[kAdjChunk][3];
    __shared__ unsigned long long s_mask[kAdjTX * kAdjTY];
    const int S = stencil_size(p.kind);
    const T *mw = reinterpret_cast<const T *>(p.mk_w);
    const int m0 = ldg(a.tile_off, t), m1 = ldg(a.tile_off, t + 1);
    for (int c0 = m0; c0 < m1; c0 += kAdjChunk) {
      const int cnt = min(kAdjChunk, m1 - c0);
      const int k = tid & 15, dx = k & 3, dy = k >> 2;
      constexpr int kTurns = kAdjChunk / 16;
      int l[kTurns];
#pragma unroll
      for (int u = 0; u < kTurns; ++u) l[u] = ldg(a.tile_list, c0 + min((tid >> 4) + 16 * u, cnt - 1));
      if (c0 > m0) __syncthreads();
      s_mask[tid] = 0;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kTurns; ++u) {
        const int e = (tid >> 4) + 16 * u;
        if (e >= cnt) break;
        const int ix = ldg(p.mk_ixy, 2 * l[u]), iy = ldg(p.mk_ixy, 2 * l[u] + 1);
        if (k < 10) s_w[e][k] = ldg(mw, 10 * (long long)l[u] + k);
        if (k >= 10 && k < 13) s_a[e][k - 10] = ldg(a.mk_adj, 3 * (long long)l[u] + k - 10);
        if (k == 13) s_ix[e] = ix;
        if (k == 14) s_iy[e] = iy;
        int nx = ix + dx, ny = iy + dy;
        if (p.xper && nx >= p.nx) nx -= p.nx;
        if (p.yper && ny >= p.ny) ny -= p.ny;
        nx -= x0;
        ny -= y0;
        if (dx < S && dy < S && (unsigned)nx < (unsigned)kAdjTX && (unsigned)ny < (unsigned)kAdjTY)
          atomicOr(&s_mask[ny * kAdjTX + nx], 1ull << e);
      }
      __syncthreads();
      constexpr int kTake = sizeof(T) == 8 ? 2 : 4;  // markers in flight (as many as the registers of four waves hold)
      for (unsigned long long m = s_mask[tid]; m;) {
        int id[kTake], mx[kTake], my[kTake];
        bool on[kTake];
        T w0[kTake], w1[kTake], f0[kTake], f1[kTake];
        double ar[kTake], au[kTake], av4[kTake];
#pragma unroll
        for (int u = 0; u < kTake; ++u) {
          on[u] = m != 0;
          id[u] = on[u] ? __builtin_ctzll(m) : id[u ? u - 1 : 0];
          m &= m - 1;
        }
#pragma unroll
        for (int u = 0; u < kTake; ++u) {
          mx[u] = x - s_ix[id[u]];
          my[u] = y - s_iy[id[u]];
          f0[u] = s_w[id[u]][8];
          f1[u] = s_w[id[u]][9];
          ar[u] = s_a[id[u]][0];
          au[u] = s_a[id[u]][1];
          av4[u] = s_a[id[u]][2];
        }
#pragma unroll
        for (int u = 0; u < kTake; ++u) {
          if (mx[u] < 0) mx[u] += p.nx;  // (covered, so 0 .. 3 up to the period)
          if (my[u] < 0) my[u] += p.ny;
          w0[u] = s_w[id[u]][mx[u] & 3];
          w1[u] = s_w[id[u]][4 + (my[u] & 3)];
        }
#pragma unroll
        for (int u = 0; u < kTake; ++u) {
          const T W = w0[u] * w1[u], ax = fmx(W, f0[u], fibx), ay = fmx(W, f1[u], fiby);
          const double Wd = (double)w0[u] * (double)w1[u];
          const double br = fmx(Wd, ar[u], Pr), bu = fmx(Wd, au[u], Pu), bv = fmx(Wd, av4[u], Pv);
          fibx = on[u] ? ax : fibx;
          fiby = on[u] ? ay : fiby;
          Pr = on[u] ? br : Pr;
          Pu = on[u] ? bu : Pu;
          Pv = on[u] ? bv : Pv;
        }
      }
    }
  }

  double sGx = 0.0, sGy = 0.0, sUx = 0.0, sUy = 0.0;
  if (fluid) {
    const double ftx = FORCED ? (double)(T)(p.Gx + (double)fibx) : (double)(T)p.Gx;
    const double fty = FORCED ? (double)(T)(p.Gy + (double)fiby) : (double)(T)p.Gy;
    NodeFwd nf;
    Mom mo;
    double dr = 0.0, mx = 0.0, my = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const double v = (double)av[q];
      dr += v;
      mx += ex(q) * v;
      my += ey(q) * v;
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) mo.add(q, (double)bb[q]);
    nf.rho = 1.0 + dr;
    nf.mx = mx + p.urx;  // stored values are deviations from feq(1, u_ref)
    nf.my = my + p.ury;
    nf.ux = (nf.mx + 0.5 * ftx) / nf.rho;
    nf.uy = (nf.my + 0.5 * fty) / nf.rho;
    // the inlet ghost's density adds one shift to every direction of dJ/dB
    double shift = 0.0;
    if (inlet && x == 1) {
      // B_q(0, y) = feq_q(rho_B, u_in) - c_q with rho_B the density of column
      // 1 after collision, which the collision leaves equal to rho
      const double rB = nf.rho;
      const double ui = p.uin_x, vi = p.uin_y, uui = ui * ui + vi * vi;
      T gh[9];
      pull_adj9<T>(Gn, p, 0, y, gh);
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const double a0 = (double)gh[q];
        const double eu = ex(q) * ui + ey(q) * vi;
        shift += a0 * wq(q) * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uui);
        sUx += a0 * wq(q) * rB * (3.0 * ex(q) + 9.0 * eu * ex(q) - 3.0 * ui);
        sUy += a0 * wq(q) * rB * (3.0 * ey(q) + 9.0 * eu * ey(q) - 3.0 * vi);
      }
      mo.add_uniform(shift);
    }
    const CollideAdj ca = collide_adjoint<false>(nf, ftx, fty, mo, p);
    double drb = ca.drb, mbx = ca.mbx, mby = ca.mby;
    sGx = ca.fbx;
    sGy = ca.fby;
    if (FORCED) {
      // transposed interpolation (eqs 12, 14) through rho and u* = (m + G/2)/rho
      const double inv = 1.0 / nf.rho;
      const double usx = fma(p.Gx, 0.5, nf.mx) * inv, usy = fma(p.Gy, 0.5, nf.my) * inv;
      drb += fma(-inv, fma(Pu, usx, Pv * usy), Pr);
      mbx = fma(Pu, inv, mbx);
      mby = fma(Pv, inv, mby);
      sGx = fma(0.5 * Pu, inv, sGx);
      sGy = fma(0.5 * Pv, inv, sGy);
    }
    const double omc = 1.0 - p.omega;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
#pragma clang fp contract(off)  // (mb is added as it stands)
      Go[(long long)q * p.plane + node] = (T)(fma(omc, (double)bb[q] + shift, drb) + ex(q) * mbx + ey(q) * mby);
    }
  }

  // the tile's sums (those of the inflow only where it enters)
  __shared__ double red[4][4];
  const double v0 = wave_total(sGx), v1 = wave_total(sGy);
  const double v2 = inlet ? wave_total(sUx) : 0.0, v3 = inlet ? wave_total(sUy) : 0.0;
  if ((tid & 63) == 0) {
    red[tid >> 6][0] = v0;
    red[tid >> 6][1] = v1;
    red[tid >> 6][2] = v2;
    red[tid >> 6][3] = v3;
  }
  __syncthreads();
  if (tid < (inlet ? 4 : 2))
    a.part[4 * (long long)t + tid] = sum0 + ((red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]));
}

// The tiles no stencil touches need nothing of the markers: one launch has the
// markers (first, the longer work) and half of those tiles, the second the
// tiles that wait for the markers and the other half.
__device__ __forceinline__ int adj_open_tile(const LbmParams &p, const AdjParams &a, int first, int k, int n) {
  return ldg(a.tiles, a.n_forced + first + (p.xcd_remap ? xcd_tile(k, n) : k));
}
template <typename T>
__global__ __launch_bounds__(kAdjTX *kAdjTY, 4) void adj_marker_kernel(const T *__restrict__ A, const T *__restrict__ Gn,
                                                                    T *__restrict__ Go, LbmParams p, IbParams ib,
                                                                    AdjParams a, int marker_blocks, int open) {
  const int k = (int)blockIdx.x - marker_blocks;
  if (k < 0)
    adj_markers<T>(A, Gn, p, ib, a, (int)blockIdx.x);
  else
    adj_tile<T, false>(A, Gn, Go, p, a, adj_open_tile(p, a, 0, k, open));
}
template <typename T>
__global__ __launch_bounds__(kAdjTX *kAdjTY, 4) void adj_lattice_kernel(const T *__restrict__ A,
                                                                     const T *__restrict__ Gn, T *__restrict__ Go,
                                                                     LbmParams p, AdjParams a, int first, int open) {
  const int k = (int)blockIdx.x - a.n_forced;
  if (k < 0)
    adj_tile<T, true>(A, Gn, Go, p, a, ldg(a.tiles, (int)blockIdx.x));
  else
    adj_tile<T, false>(A, Gn, Go, p, a, adj_open_tile(p, a, first, k, open));
}

// The tiles no stencil touches, alone: fewer registers than beside the markers.
template <typename T>
__global__ __launch_bounds__(kAdjTX *kAdjTY) void adj_open_kernel(const T *__restrict__ A, const T *__restrict__ Gn,
                                                                  T *__restrict__ Go, LbmParams p, AdjParams a,
                                                                  int first, int open) {
  adj_tile<T, false>(A, Gn, Go, p, a, adj_open_tile(p, a, first, (int)blockIdx.x, open));
}

// dJ/dA_0 from G_0, all nodes (ghost columns included), packed [9][ny][nx] in FP64
template <typename T>
__global__ void adj_unpull_kernel(const T *__restrict__ G, LbmParams p, double *__restrict__ out) {
  const long long n = (long long)p.nx * p.ny;
  for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    const int y = (int)(k / p.nx), x = (int)(k - (long long)y * p.nx);
#pragma unroll
    for (int q = 0; q < 9; ++q) out[(long long)q * n + k] = (double)pull_adj<T>(G, p, q, x, y);
  }
}

// ------------------------------------------------------------------ launchers
template <typename T>
static hipError_t launch_adj_t(const void *A, const void *Gnext, void *Gout, const LbmParams &p, const IbParams &ib,
                               const AdjParams &a, hipStream_t s) {
  const int markers = (ib.nm + 15) / 16, open = a.ntx * a.nty - a.n_forced;
  const bool apart = markers == 0 || open > kAdjApart;
  const int beside = markers == 0 ? 0 : kAdjBeside;
  const int first = apart ? beside : open / 2, second = apart ? beside : open - first, rest = open - first - second;
  const dim3 block(kAdjTX * kAdjTY);
  if (markers > 0)
    hipLaunchKernelGGL(adj_marker_kernel<T>, dim3(markers + first), block, 0, s, (const T *)A, (const T *)Gnext,
                       (T *)Gout, p, ib, a, markers, first);
  if (a.n_forced + second > 0)
    hipLaunchKernelGGL(adj_lattice_kernel<T>, dim3(a.n_forced + second), block, 0, s, (const T *)A,
                       (const T *)Gnext, (T *)Gout, p, a, first, second);
  if (rest > 0)
    hipLaunchKernelGGL(adj_open_kernel<T>, dim3(rest), block, 0, s, (const T *)A, (const T *)Gnext, (T *)Gout, p, a,
                       first + second, rest);
  return hipGetLastError();
}

hipError_t launch_adj_step(int prec, const void *A, const void *Gnext, void *Gout, const LbmParams &p,
                           const IbParams &ib, const AdjParams &a, hipStream_t s) {
  return prec == 4 ? launch_adj_t<float>(A, Gnext, Gout, p, ib, a, s)
                   : launch_adj_t<double>(A, Gnext, Gout, p, ib, a, s);
}

hipError_t launch_adj_unpull(int prec, const void *G, const LbmParams &p, double *out, hipStream_t s) {
  const long long n = (long long)p.nx * p.ny;
  const int blocks = (int)std::min<long long>((n + 255) / 256, 65536);
  if (prec == 4)
    hipLaunchKernelGGL(adj_unpull_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float *)G, p, out);
  else
    hipLaunchKernelGGL(adj_unpull_kernel<double>, dim3(blocks), dim3(256), 0, s, (const double *)G, p, out);
  return hipGetLastError();
}

}  // namespace btdf
