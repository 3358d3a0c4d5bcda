// btdf_tile.h -- one tile of the lattice in one time step (device code of the
// single-step lattice kernels in btdf_kernels.hip and of the one-launch step
// in btdf_step.hip): the streaming pull, the spread gather of the tile's
// markers, the collision and the channel's ghost columns; and the per-body
// sums of eq 27.
#pragma once

#include "btdf_device.h"

namespace btdf {

// Hydrodynamic force and torque on body b (eq 27 with the body's sign): a
// workgroup of NT lanes sums its markers' forces (Fl_x, Fl_y) in a fixed
// order and writes them to the step's entry (slot) of the history ring.
template <int NT>
__device__ void body_reduce(const IbParams &ib, const double *Fl_x, const double *Fl_y, int slot, int b, int tid,
                            double (*red)[NT / 64]) {
  const int l0 = ib.body_off[b], l1 = ib.body_off[b + 1];
  const double cx = ib.cx[b], cy = ib.cy[b];
  double sfx = 0.0, sfy = 0.0, stz = 0.0;
  const bool per_marker = ib.method == 2;  // RKPM spreads with a factor per marker
  for (int l = l0 + tid; l < l1; l += NT) {
    const double Fx = Fl_x[l], Fy = Fl_y[l];
    if (per_marker) {
      const double w = ib.sdrs[l];
      sfx += w * Fx;
      sfy += w * Fy;
      stz += w * ((ib.X[l] - cx) * Fy - (ib.Y[l] - cy) * Fx);
    } else {
      sfx += Fx;
      sfy += Fy;
      stz += (ib.X[l] - cx) * Fy - (ib.Y[l] - cy) * Fx;
    }
  }
  sfx = wave_sum(sfx);
  sfy = wave_sum(sfy);
  stz = wave_sum(stz);
  const int lane = tid & 63, w = tid >> 6;
  if (lane == 0) {
    red[0][w] = sfx;
    red[1][w] = sfy;
    red[2][w] = stz;
  }
  __syncthreads();
  if (tid == 0) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int k = 0; k < NT / 64; ++k) {
      s0 += red[0][k];
      s1 += red[1][k];
      s2 += red[2][k];
    }
    const double s = per_marker ? 1.0 : ib.body_sdrs[b];
    double *h = ib.hist + ((long long)slot * ib.nb + b) * 3;
    h[0] = -s * s0;
    h[1] = -s * s1;
    h[2] = -s * s2;
  }
}

// Body b's places one step on, by one workgroup of NT threads: the centre and
// angle advance, the markers sit at c + R(theta) r with the rigid velocity.
template <int NT>
__device__ __forceinline__ void move_body(const MoveParams &mp, int b, int tid) {
#pragma clang fp contract(off)
  const double *st = mp.from.state + 4 * (long long)b;
  const bool moves = mp.moving[b] && !mp.copy;
  const double vx = st[1], vy = st[2], om = st[3];
  const double cx = moves ? mp.from.cx[b] + vx : mp.from.cx[b];
  const double cy = moves ? mp.from.cy[b] + vy : mp.from.cy[b];
  const double th = moves ? st[0] + om : st[0];
  const int l0 = mp.body_off[b], l1 = mp.body_off[b + 1];
  __syncthreads();  // every lane has read the old state
  if (tid == 0) {
    double *to = mp.to.state + 4 * (long long)b;
    mp.to.cx[b] = cx;
    mp.to.cy[b] = cy;
    to[0] = th;
    to[1] = vx;
    to[2] = vy;
    to[3] = om;
  }
  if (!moves) {
    for (int l = l0 + tid; l < l1; l += NT) {
      mp.to.X[l] = mp.from.X[l];
      mp.to.Y[l] = mp.from.Y[l];
      mp.to.U[l] = mp.from.U[l];
      mp.to.V[l] = mp.from.V[l];
    }
    return;
  }
  const double c = cos(th), s = sin(th);
  for (int l = l0 + tid; l < l1; l += NT) {
    const double rx = mp.rxy[2 * (long long)l], ry = mp.rxy[2 * (long long)l + 1];
    const double X = cx + c * rx - s * ry;
    const double Y = cy + s * rx + c * ry;
    mp.to.X[l] = X;
    mp.to.Y[l] = Y;
    mp.to.U[l] = vx - om * (Y - cy);
    mp.to.V[l] = vy + om * (X - cx);
  }
}

constexpr int kChunk = 64;  // markers staged in LDS per pass

template <typename T, bool NT>
__device__ __forceinline__ void store(T *ptr, T v) {
  const global_ptr<T> g = (global_ptr<T>)ptr;  // device memory: a global access
  if (NT)
    __builtin_nontemporal_store(v, g);
  else
    *g = v;
}

// A batch case's stop flag (nonzero once the case went unstable), read
// with an atomic load at the start of a workgroup: the read is in flight with
// the population loads and is not moved down to its use. Batch kernels pass
// the case's flag, or kNoStop when unstable cases are not masked, so the load
// needs no branch around it (whose join would wait for it at once). The
// address carries a per-lane zero the compiler cannot see through, so the
// value stays per lane instead of being moved to a scalar register (and
// waited for) right after the load.
__device__ const int kNoStop = 0;
template <bool STOP>
__device__ __forceinline__ int stop_flag(const int *stop) {
  if constexpr (STOP) {
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return __hip_atomic_load((global_ptr<const int>)stop + zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return 0;
}

// The spread force of the cnt markers staged in LDS (stencil origins, then
// wx[4], wy[4], drs ds F_x, drs ds F_y) on this thread's nodes (xb + k BX, y),
// added in ascending marker order. Each lane first tests one marker against
// the rows of its wave (WR rows from yw); the wave then walks the set bits of
// that mask, four markers at a time with their LDS reads in flight together,
// and each lane keeps the sums of the markers whose stencil covers its node.
// A loop over all markers with a branch per marker instead waited for two
// dependent LDS reads per marker (200x120 FP64 channel, 50 markers: 13.3 us a
// step then, 12.4 now; 2000x800 FP32 shedding: 28.6 and 26.2).
template <typename T, int BX, int NPT, int WR>
__device__ __forceinline__ void spread_gather(const int (&s_ix)[kChunk], const int (&s_iy)[kChunk],
                                              const T (&s_w)[kChunk][10], int cnt, int S, const LbmParams &p, int xb,
                                              int y, int yw, T (&fx)[NPT], T (&fy)[NPT]) {
  static_assert(kChunk <= 64, "one marker per lane of a wave");
  const int lane = (int)(threadIdx.y * BX + threadIdx.x) & 63;
  // rows yw .. yw + WR - 1 meet rows iy .. iy + S - 1 (mod ny) if e < S + WR - 1
  int e = yw + WR - 1 - s_iy[lane < cnt ? lane : 0];
  if (p.yper && e < 0) e += p.ny;
  unsigned long long m = __builtin_amdgcn_ballot_w64(lane < cnt && (unsigned)e < (unsigned)(S + WR - 1));
  while (m) {
    int id[4];
    bool on[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      on[u] = m != 0;
      id[u] = on[u] ? __builtin_ctzll(m) : id[u ? u - 1 : 0];
      m &= m - 1;
    }
    int dy[4];
    T wy[4], Fx[4], Fy[4];
    int ix[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      dy[u] = y - s_iy[id[u]];
      ix[u] = s_ix[id[u]];
      Fx[u] = s_w[id[u]][8];
      Fy[u] = s_w[id[u]][9];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p.yper && dy[u] < 0) dy[u] += p.ny;
      on[u] = on[u] && (unsigned)dy[u] < (unsigned)S;
      wy[u] = s_w[id[u]][4 + (dy[u] & 3)];
    }
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      int dx[4];
      T wx[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        dx[u] = xb + k * BX - ix[u];
        if (p.xper && dx[u] < 0) dx[u] += p.nx;
        wx[u] = s_w[id[u]][dx[u] & 3];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const T W = wx[u] * wy[u];
        const T ax = fmx(W, Fx[u], fx[k]), ay = fmx(W, Fy[u], fy[k]);
        const bool in = on[u] && (unsigned)dx[u] < (unsigned)S;
        fx[k] = in ? ax : fx[k];
        fy[k] = in ? ay : fy[k];
      }
    }
  }
}

// v of the lane that CTRL names (a data-parallel-primitive control word)
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over the 16 lanes of a marker, in the order of a butterfly over lane
// distances 8, 4, 2, 1 (row rotations by 8 and 4, then the quad permutations;
// after the first, lanes 8 apart hold the same value, so a rotation by 4 is
// the exchange with the lane 4 apart). Every lane ends with the sum.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp<0x128>(v);
  v += dpp<0x124>(v);
  v += dpp<0x4E>(v);
  v += dpp<0xB1>(v);
  return v;
}

// rho and the unforced velocity u* (eqs 9-10, with G/2) of one node, from its
// streamed deviations, whose first moment is m - u_ref
template <typename T>
__device__ __forceinline__ void node_moments(const T (&gq)[9], const LbmParams &p, double &rho, double &usx,
                                             double &usy) {
  double drho = 0.0, mx = 0.0, my = 0.0;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const double g = (double)gq[q];
    drho += g;
    mx += ex(q) * g;
    my += ey(q) * g;
  }
  rho = 1.0 + drho;
  const double inv = 1.0 / rho;
  usx = (mx + p.urx + 0.5 * p.Gx) * inv;
  usy = (my + p.ury + 0.5 * p.Gy) * inv;
}

// Convective outlet (d/dt + U d/dx = 0 on the ghost column, implicit upwind):
// the ghost of B is (ghost of A + U column nx-2 of B) / (1 + U), written by
// the lane that has just made column nx-2 (base: its offset, out: its
// values). The reference offsets of the stored deviations cancel (the
// weights sum to one). Here it costs nothing measurable: as a launch after
// the step it was one round trip per population on one thread per row, 9.8
// us at 401 rows and 15.3 us at 1601 (the 1601^2 far-field run: 49.5 us a
// step then, 33.0 now). The loads stay behind the collision so that the
// kernel's registers are the collision's.
template <typename T>
__device__ __forceinline__ void conv_outlet_node(const T *__restrict__ A, T *__restrict__ B, const LbmParams &p,
                                                 long long base, const T (&out)[9]) {
  const T U = (T)p.uconv, den = (T)(1.0 + p.uconv);
  T g[9];
  __builtin_amdgcn_sched_barrier(0);  // (no earlier: the loads' registers would add to the collision's)
#pragma unroll
  for (int q = 0; q < 9; ++q) g[q] = load<T>(&A[(long long)q * p.plane + base + 1]);
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    B[(long long)q * p.plane + base + 1] = (g[q] + U * out[q]) / den;
    __builtin_amdgcn_sched_barrier(0);  // one division's temporaries at a time
  }
}

// one tile t of the lattice: streaming pull, spread gather, collision; with
// STOP and *stop set, nothing is stored (a stopped batch case)
template <typename T, int BX, int BY, int NPT, bool NT, bool NTL, bool STOP = false>
__device__ __forceinline__ void lbm_tile(const T *__restrict__ A, T *__restrict__ B, const LbmParams &p, int t,
                                         const int *stop = nullptr) {
  constexpr int TX = BX * NPT;
  const int halt = stop_flag<STOP>(stop);
  __shared__ int s_ix[kChunk], s_iy[kChunk];
  __shared__ T s_w[kChunk][10];  // wx[4], wy[4], drs ds F_x, drs ds F_y
  const int tyi = t / p.ntx;
  const int txi = t - tyi * p.ntx;
  const int y = tyi * BY + (int)threadIdx.y;
  const int xb = txi * TX + (int)threadIdx.x;

  // A wave whose nodes and their neighbours need no wrap and no wall takes
  // the interior path: every pull is one load from a wave-uniform base plus
  // the lane's byte offset. A wave spans WR rows of the tile (1 if BX >= 64).
  constexpr int WR = BX >= 64 ? 1 : 64 / BX;
  constexpr int WX = BX >= 64 ? 64 : BX;
  const int yw = __builtin_amdgcn_readfirstlane(y - (BX >= 64 ? 0 : ((int)threadIdx.y % WR)));
  const int xw = __builtin_amdgcn_readfirstlane(BX >= 64 ? txi * TX + ((int)threadIdx.x & ~63) : txi * TX);
  // (a wave that holds column nx-2 of a channel also writes the outlet ghost)
  const bool interior = p.interior && yw >= 1 && yw + WR <= p.ny - 1 && xw >= 1 &&
                        xw + WX + (NPT - 1) * BX <= p.nx - 1 - (p.outlet ? 1 : 0);
  const unsigned rowoff = (unsigned)(y - yw) * (unsigned)p.pitch;

  // the pulls are issued first, so they are in flight while the tile
  // gathers its markers' forces
  T g[NPT][9];
  bool live[NPT];
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const int x = xb + k * BX;
    live[k] = y < p.ny && (interior || (x >= p.i0 && x <= p.i1));
    if (!live[k]) continue;
    // byte offset of the node from the wave's first row: one 32-bit register
    // shared by all loads and stores of the interior path
    const unsigned xoff = (rowoff + (unsigned)x) * (unsigned)sizeof(T);
    if (interior) {
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const char *base = reinterpret_cast<const char *>(A + (long long)q * p.plane +
                                                          (long long)(yw - ey(q)) * p.pitch - ex(q));
        g[k][q] = load<T, NTL>(reinterpret_cast<const T *>(base + xoff));
      }
    } else {
      pull9<T, NTL>(A, p, x, y, g[k]);
    }
  }

  T fib_x[NPT], fib_y[NPT];
#pragma unroll
  for (int k = 0; k < NPT; ++k) fib_x[k] = fib_y[k] = (T)0;

  // spread (eqs 13, 15) as a gather over the markers listed for this tile;
  // the marker kernel left each marker's weights and drs ds F_l
  const int m0 = ldg(p.tile_off, t), m1 = ldg(p.tile_off, t + 1);
  const bool forced = m1 > m0;
  if (forced) {
    const int S = stencil_size(p.kind);
    const int tid = (int)threadIdx.y * BX + (int)threadIdx.x;
    const T *mw = reinterpret_cast<const T *>(p.mk_w);
    for (int c0 = m0; c0 < m1; c0 += kChunk) {
      const int cnt = min(kChunk, m1 - c0);
      __syncthreads();
      if (tid < cnt) {
        const int l = ldg(p.tile_list, c0 + tid);
        s_ix[tid] = ldg(p.mk_ixy, 2 * l);
        s_iy[tid] = ldg(p.mk_ixy, 2 * l + 1);
#pragma unroll
        for (int k = 0; k < 10; ++k) s_w[tid][k] = ldg(mw, 10 * (long long)l + k);
      }
      __syncthreads();
      spread_gather<T, BX, NPT, WR>(s_ix, s_iy, s_w, cnt, S, p, xb, y, yw, fib_x, fib_y);
    }
  }
  if (y >= p.ny || halt) return;  // (after the gather's last barrier)

  const CollK<T> &K = coll<T>(p);
  bool bad = false;
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const int x = xb + k * BX;
    if (!live[k]) continue;
    const unsigned xoff = (rowoff + (unsigned)x) * (unsigned)sizeof(T);
    T out[9], rho;
    if (forced) {
      const ForceK<T> F = force_terms<T>(K, (T)(p.Gx + (double)fib_x[k]), (T)(p.Gy + (double)fib_y[k]));
      collide<T>(g[k], F, K, out, rho);
    } else {
      collide<T>(g[k], gforce<T>(p), K, out, rho);
    }
    bad |= !rho_ok(rho);
    if (interior) {
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        char *base = reinterpret_cast<char *>(B + (long long)q * p.plane + (long long)yw * p.pitch);
        store<T, NT>(reinterpret_cast<T *>(base + xoff), out[q]);
      }
      continue;
    }
    const long long base = (long long)y * p.pitch + x;
#pragma unroll
    for (int q = 0; q < 9; ++q) store<T, NT>(&B[(long long)q * p.plane + base], out[q]);
    if (p.inlet && x == 1) {
      // inlet ghost: equilibrium at the inflow velocity, density of column 1
      const T dr = inlet_dr<T>(out);
      const long long gb = (long long)y * p.pitch;
#pragma unroll
      for (int q = 0; q < 9; ++q) B[(long long)q * p.plane + gb] = inlet_ghost<T>(dr, p, q);
    }
    if (p.outlet && x == p.nx - 2) {
      if (p.outlet == 1) {
#pragma unroll
        for (int q = 0; q < 9; ++q) B[(long long)q * p.plane + base + 1] = out[q];
      } else {
        conv_outlet_node<T>(A, B, p, base, out);
      }
    }
  }
  if (bad) p.flag[0] = -1;
}

// ---- the one-launch step: a tile and the ring around it
constexpr int kTX = 32, kTY = 8, kHalf = kTX * kTY;  // the tile, and the threads that take its nodes
constexpr int kBlock = 2 * kHalf;  // the workgroup: as many again for the ring
constexpr int kMomX = kTX + 6, kMomY = kTY + 6;      // with the reach of a 4-point stencil around it

// All pulls of node (x, y), in the grid, with the boundary readings of
// pull(). Offsets within a plane are 32-bit: the columns and rows are wrapped
// once for all directions (at a wall they stay in the grid, and a node next to
// it replaces the three populations that came from beyond it).
template <typename T>
__device__ __forceinline__ void step_pulls(const T *__restrict__ A, const LbmParams &p, int x, int y, T (&g)[9]) {
#pragma clang fp contract(off)
  const unsigned pb = (unsigned)p.pitch * (unsigned)sizeof(T);
  int xm = x - 1, xp = x + 1, ym = y - 1, yp = y + 1;
  xm = xm < 0 ? (p.xper ? p.nx - 1 : 0) : xm;
  xp = xp >= p.nx ? (p.xper ? 0 : p.nx - 1) : xp;
  ym = ym < 0 ? (p.yper ? p.ny - 1 : 0) : ym;
  yp = yp >= p.ny ? (p.yper ? 0 : p.ny - 1) : yp;
  const unsigned row[3] = {(unsigned)ym * pb, (unsigned)y * pb, (unsigned)yp * pb};
  const unsigned col[3] = {(unsigned)xm * (unsigned)sizeof(T), (unsigned)x * (unsigned)sizeof(T),
                           (unsigned)xp * (unsigned)sizeof(T)};
#pragma unroll
  for (int q = 0; q < 9; ++q)
    g[q] = load_global<T>(reinterpret_cast<const char *>(A + (long long)q * p.plane), row[1 - ey(q)] + col[1 - ex(q)]);
  if (!p.yper && (y == 0 || y == p.ny - 1)) {
    const __attribute__((address_space(4))) T *k = (const __attribute__((address_space(4))) T *)konst<T>(p);
#pragma unroll
    for (int q = 2; q < 9; ++q) {
      if (ey(q) == 0 || y != (ey(q) > 0 ? 0 : p.ny - 1)) continue;
      if (p.slip)
        g[q] = load_global<T>(reinterpret_cast<const char *>(A + (long long)mir_y(q) * p.plane), row[1] + col[1 - ex(q)]) +
               k[27 + q];
      else
        g[q] = load_global<T>(reinterpret_cast<const char *>(A + (long long)opp(q) * p.plane), row[1] + col[1]) + k[18 + q];
    }
  }
}

// The place of a ring node: k = 0 .. 2 H (kTX + 2 H + kTY) - 1 counts the H
// rows below and above the tile, then the H columns on both sides (H = 1, 2, 3).
__device__ __forceinline__ int ring_nodes(int H) { return 2 * H * (kTX + 2 * H + kTY); }
__device__ __forceinline__ void ring_place(int k, int H, int &i, int &j) {
  const int W = kTX + 2 * H;
  // k / W for k < 2^9 and e / (2 H) for e < 48, by reciprocals
  const int rw = H == 3 ? 1725 : (H == 2 ? 1821 : 1928), rh = H == 3 ? 10923 : (H == 2 ? 16384 : 32768);
  if (k < 2 * H * W) {
    const int row = (k * rw) >> 16;
    i = k - row * W;
    j = row < H ? row : row + kTY;
  } else {
    const int e = k - 2 * H * W, row = (e * rh) >> 16, c = e - row * 2 * H;
    i = c < H ? c : c + kTX;
    j = H + row;
  }
}

// The grid node at place (i, j) of the tile (x0, y0) grown by H: past a
// periodic edge its image; false outside the fluid.
__device__ __forceinline__ bool grid_place(const LbmParams &p, int x0, int y0, int H, int i, int j, int &x, int &y) {
  x = x0 - H + i;
  y = y0 - H + j;
  if (p.xper) x = wrap_index(x, p.nx);
  if (p.yper) y = wrap_index(y, p.ny);
  return x >= p.i0 && x <= p.i1 && y >= 0 && y < p.ny;
}

}  // namespace btdf
