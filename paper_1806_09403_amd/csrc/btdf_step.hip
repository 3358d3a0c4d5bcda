// btdf_step.hip -- a whole time step in one launch (direct forcing, one pass),
// for lattices, or sets of near tiles, small enough that a step is a chain of
// latencies: a launch, a few dependent reads, and single waves working through
// the markers and the collision with their SIMDs otherwise idle.
//
// A tile that a marker stencil touches forms its markers' forces itself: it
// takes rho and u* at its nodes and the stencil's reach around them into LDS,
// interpolates them to the markers of its list and forms F_l (eqs 12, 14, 20),
// then gathers the spread force and collides as the lattice kernel does. A
// marker whose stencil touches several tiles is formed in each, from the same
// values in the same order, so all use the same bits, which are those of the
// marker kernel; the tile that holds its stencil origin stores F_l. The body
// forces (eq 27) need every F_l of the step: the next step's launch sums
// them, or step_flush_kernel after the last step. The same workgroups place
// rigidly moving bodies for the step after, in the other of two sets of places.
//
// A workgroup has eight waves. For a forced tile the first four take the
// tile's nodes and stage the markers, the other four take the ring of nodes
// around it, and all form forces; without markers the two halves take a tile
// each. (A ninth wave for the 20 ring nodes past 256 of a 4-point stencil
// gains 2% on the 200x120 channel but costs a fifth of the workgroups a CU
// holds: 57.8 -> 67.3 us a step on 2560^2 with 200 cylinders.) What a workgroup
// does is one 16-byte entry of a list made on the host (forced tiles first, as
// they take longest, and by XCD), so nothing is looked up on the way to the
// first population load.
#include "btdf_device.h"
#include "btdf_launch.h"
#include "btdf_tile.h"

namespace btdf {

namespace {

// One chunk of a tile's markers: ids, stencil origins (wrapped; and relative
// to the tile grown by the stencil's reach), delta weights (x then y),
// velocity, spreading factor; then weight products and drs ds F_l in the
// population type, as the spread takes them.
template <typename T>
struct MarkerLds {
  double ph[kChunk][8], U[kChunk], V[kChunk], sd[kChunk];
  T F[kChunk][2], w[kChunk][8];
  int l[kChunk], ix[kChunk], iy[kChunk];
};

// Stage a chunk of markers whose forces another kernel formed: weights,
// drs ds F_l and origins from the marker records, ten threads per marker.
template <typename T>
__device__ __forceinline__ void stage_records(const LbmParams &p, int c0, int cnt, int tid, MarkerLds<T> &s_k) {
  for (int k = tid; k < 16 * cnt; k += kHalf) {
    const int e = k >> 4, w = k & 15;
    const int l = ldg(p.tile_list, c0 + e);
    const T *mw = reinterpret_cast<const T *>(p.mk_w) + 10 * (long long)l;
    if (w < 8) s_k.w[e][w] = ldg(mw, w);
    if (w == 8 || w == 9) s_k.F[e][w - 8] = ldg(mw, w);
    if (w == 10) s_k.ix[e] = ldg(p.mk_ixy, 2 * l);
    if (w == 11) s_k.iy[e] = ldg(p.mk_ixy, 2 * l + 1);
  }
}

// The tile's nodes that the staged markers cover (bit e of s_mask), 16 lanes
// per marker.
template <typename T>
__device__ __forceinline__ void mark_nodes(const LbmParams &p, int x0, int y0, int S, int cnt, int tid,
                                           const MarkerLds<T> &s_k, unsigned long long (&s_mask)[kHalf]) {
  const int a = tid & 3, c = (tid >> 2) & 3;
  for (int e = tid >> 4; e < cnt; e += kBlock / 16) {
    int sx = s_k.ix[e] + a, sy = s_k.iy[e] + c;
    if (p.xper && sx >= p.nx) sx -= p.nx;
    if (p.yper && sy >= p.ny) sy -= p.ny;
    sx -= x0;
    sy -= y0;
    if (a < S && c < S && (unsigned)sx < (unsigned)kTX && (unsigned)sy < (unsigned)kTY)
      atomicOr(&s_mask[sy * kTX + sx], 1ull << e);
  }
}

// Stage a chunk of markers (list entries c0 .. c0 + cnt): eight threads per
// marker, one delta weight each, and between them its origin, velocity and
// spreading factor. Nothing here waits for populations.
template <typename T>
__device__ __forceinline__ void stage_markers(const LbmParams &p, const IbParams &ib, int S, int c0, int cnt, int tid,
                                              MarkerLds<T> &s_k) {
  for (int k = tid; k < 8 * cnt; k += kHalf) {
    const int e = k >> 3, w = k & 7, a = w & 3;
    const int l = ldg(p.tile_list, c0 + e);
    const double Z = ldg(w < 4 ? ib.X : ib.Y, l);
    const double val = ldg(a == 1 ? ib.U : (a == 2 ? ib.V : ib.sdrs), l);
    const int b = stencil_base(p.kind, Z);
    const double ph = a < S ? phi(p.kind, (double)(b + a) - Z) : 0.0;
    s_k.ph[e][w] = ph;
    s_k.w[e][w] = (T)ph;
    if (w == 0) {
      s_k.ix[e] = p.xper ? wrap_index(b, p.nx) : b;
      s_k.l[e] = l;
    }
    if (w == 4) s_k.iy[e] = p.yper ? wrap_index(b, p.ny) : b;
    if (w == 1) s_k.U[e] = val;
    if (w == 2) s_k.V[e] = val;
    if (w == 3) s_k.sd[e] = val;
  }
}

// The staged markers' forces, once rho and u* are in s_m: 16 lanes per
// marker, one per stencil node, which also marks the node of the tile it is
// (bit e of s_mask). Leaves drs ds F_l for the spread; the tile that holds
// the stencil origin stores F_l, and with record the values
// btdf_get_marker_data and the reverse sweep read. A marker whose stencil
// misses the tile (the lists of moving bodies have a margin) marks no node.
template <typename T>
__device__ __forceinline__ void marker_forces(const LbmParams &p, const IbParams &ib, int x0, int y0, int S, int cnt,
                                              bool record, int tid, const double (&s_m)[3][kMomY][kMomX],
                                              MarkerLds<T> &s_k, unsigned long long (&s_mask)[kHalf]) {
  const int node = tid & 15, a = node & 3, c = node >> 2, H = S - 1;
  for (int e = tid >> 4; e - (tid >> 4) < cnt; e += kBlock / 16) {  // (whole waves: the sums need every lane)
    const bool act = e < cnt;
    const int em = act ? e : 0;
    const int ix = s_k.ix[em], iy = s_k.iy[em];
    int rx = ix - x0 + H, ry = iy - y0 + H;
    if (p.xper) rx = rx < 0 ? rx + p.nx : (rx >= p.nx ? rx - p.nx : rx);
    if (p.yper) ry = ry < 0 ? ry + p.ny : (ry >= p.ny ? ry - p.ny : ry);
    const bool touch = act && (unsigned)rx < (unsigned)(kTX + H) && (unsigned)ry < (unsigned)(kTY + H);
    double wr = 0.0, wu = 0.0, wv = 0.0;
    if (touch && a < S && c < S) {
      const double W = s_k.ph[em][a] * s_k.ph[em][4 + c];
      wr = W * s_m[0][ry + c][rx + a];
      wu = W * s_m[1][ry + c][rx + a];
      wv = W * s_m[2][ry + c][rx + a];
      int sx = ix + a, sy = iy + c;  // the node itself, if this tile has it
      if (p.xper && sx >= p.nx) sx -= p.nx;
      if (p.yper && sy >= p.ny) sy -= p.ny;
      sx -= x0;
      sy -= y0;
      if ((unsigned)sx < (unsigned)kTX && (unsigned)sy < (unsigned)kTY) atomicOr(&s_mask[sy * kTX + sx], 1ull << e);
    }
    wr = row_sum(wr);
    wu = row_sum(wu);
    wv = row_sum(wv);
    const double Fx = 2.0 * wr * (s_k.U[em] - wu), Fy = 2.0 * wr * (s_k.V[em] - wv), sd = s_k.sd[em];
    const T fx = (T)(Fx * sd), fy = (T)(Fy * sd);
    if (act && node == 0) {
      s_k.F[e][0] = fx;
      s_k.F[e][1] = fy;
    }
    if (touch && ix >= x0 && ix < x0 + kTX && iy >= y0 && iy < y0 + kTY) {  // this tile's to store
      const int l = s_k.l[e];
      if (node == 0) {
        ib.Fx[l] = Fx;
        ib.Fy[l] = Fy;
        if (!isfinite(Fx) || !isfinite(Fy) || !(sqrt(wu * wu + wv * wv) <= 0.3)) p.flag[0] = 1 + ib.mk_body[l];
      }
      if (record) {
        T *mw = reinterpret_cast<T *>(ib.mk_w) + 10 * (long long)l;
        if (node < 8) mw[node] = s_k.w[e][node];
        if (node == 8) {
          mw[8] = fx;
          mw[9] = fy;
          ib.mk_ixy[2 * l] = ix;
          ib.mk_ixy[2 * l + 1] = iy;
        }
        if (node == 9) {
          ib.rho_l[l] = wr;
          ib.ux_l[l] = wu;
          ib.uy_l[l] = wv;
        }
      }
    }
  }
}

// The spread force (eqs 13, 15) of the chunk at node (x, y), whose covering
// markers are m: ascending, four at a time with their LDS reads in flight
// together.
template <typename T>
__device__ __forceinline__ void spread_masked(const LbmParams &p, const MarkerLds<T> &s_k, unsigned long long m, int x,
                                              int y, T &fx, T &fy) {
  while (m) {
    int id[4], dx[4], dy[4];
    bool on[4];
    T Fx[4], Fy[4], W[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      on[u] = m != 0;
      id[u] = on[u] ? __builtin_ctzll(m) : id[u ? u - 1 : 0];
      m &= m - 1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      dx[u] = x - s_k.ix[id[u]];
      dy[u] = y - s_k.iy[id[u]];
      Fx[u] = s_k.F[id[u]][0];
      Fy[u] = s_k.F[id[u]][1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (dx[u] < 0) dx[u] += p.nx;  // (covered, so the difference is 0 .. 3 up to the period)
      if (dy[u] < 0) dy[u] += p.ny;
      W[u] = s_k.w[id[u]][dx[u] & 3] * s_k.w[id[u]][4 + (dy[u] & 3)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const T ax = fmx(W[u], Fx[u], fx), ay = fmx(W[u], Fy[u], fy);
      fx = on[u] ? ax : fx;
      fy = on[u] ? ay : fy;
    }
  }
}

}  // namespace

// What a launch with moving bodies has on top (the others are spared the
// arguments: 0.1 us a launch).
template <bool MOVE>
struct Motion {};
template <>
struct Motion<true> {
  MoveParams mp;
};

// MARK: the tiles form their markers' forces; otherwise they are in the
// marker records (other forcing methods, body_kernel or the marker kernel).
// MOVE: the bodies' workgroups also place them for the next step.
template <typename T, bool MARK, bool MOVE>
__global__ __launch_bounds__(kBlock) void step_kernel(const T *__restrict__ A, T *__restrict__ B, LbmParams p,
                                                         StepWork w, IbParams ib, StepLink k, Motion<MOVE> motion) {
  const int tid = (int)threadIdx.x;
  const bool second = tid >= kHalf;
  const int ht = tid & (kHalf - 1);
  if ((int)blockIdx.x >= w.count) {  // workgroups past the tiles: the previous step's bodies, then the step counter
    const int gb = (int)blockIdx.x - w.count;
    if (second) return;
    if (gb >= (k.reduce || MOVE ? ib.nb : 0)) {
      if (tid == 0) {
        const long long n = p.step_ctr[0];
        ib.slot[k.word] = (int)(n % ib.hist_cap);
        p.step_ctr[0] = n + 1;
      }
      return;
    }
    // (moving bodies: the previous step's places are those the next step's
    // take the room of)
    __shared__ double red[3][kHalf / 64];
    if (k.reduce) {
      IbParams last = ib;
      if constexpr (MOVE) {
        last.X = motion.mp.to.X;
        last.Y = motion.mp.to.Y;
        last.cx = motion.mp.to.cx;
        last.cy = motion.mp.to.cy;
      }
      body_reduce<kHalf>(last, k.Fx, k.Fy, ib.slot[k.word ^ 1], gb, tid, red);
    }
    if constexpr (MOVE) {
      __syncthreads();
      move_body<kHalf>(motion.mp, gb, tid);
    }
    return;
  }
  // (made on the host and never written on the device: constant memory, one scalar load)
  typedef int vec4 __attribute__((ext_vector_type(4)));
  const vec4 iv = ((const __attribute__((address_space(4))) vec4 *)w.items)[blockIdx.x];
  const StepItem it{iv.x, iv.y, iv.z, iv.w};
  const bool forced = it.m1 > it.m0;
  const int tile = !forced && second ? it.t1 : it.t0;
  if (tile < 0) return;  // (the last workgroup without markers may have one tile only)
  const int x0 = (tile & 0xffff) * kTX, y0 = (tile >> 16) * kTY;
  const int x = x0 + (ht & (kTX - 1)), y = y0 + ht / kTX;
  const bool live = !(forced && second) && y < p.ny && x >= p.i0 && x <= p.i1;
  T g[9], fibx = (T)0, fiby = (T)0;
  if (!forced) {
    if (live) step_pulls<T>(A, p, x, y, g);
  } else {
    __shared__ MarkerLds<T> s_k;
    __shared__ double s_m[MARK ? 3 : 1][kMomY][kMomX];
    __shared__ unsigned long long s_mask[kHalf];
    const int S = stencil_size(p.kind), H = S - 1;
    // rho and u* at a place of the tile grown by H
    auto put = [&](int i, int j, const T(&v)[9]) {
      if constexpr (MARK) {
        double r, u, t;
        node_moments<T>(v, p, r, u, t);
        s_m[0][j][i] = r;
        s_m[1][j][i] = u;
        s_m[2][j][i] = t;
      }
    };
    if constexpr (MARK) {
      if (!second) {
        const int i = (ht & (kTX - 1)) + H, j = ht / kTX + H;
        int xw, yw;
        const bool in = grid_place(p, x0, y0, H, i, j, xw, yw);
        if (in) step_pulls<T>(A, p, xw, yw, g);
        stage_markers<T>(p, ib, S, it.m0, min(kChunk, it.m1 - it.m0), ht, s_k);
        if (in) put(i, j, g);
      } else {
        s_mask[ht] = 0;
        // two turns at a 4-point stencil (the second of 20 nodes, in one
        // wave): both turns' reads go out before the first is used
        int i, j, i2, j2, xw, yw;
        T v[9];
        ring_place(ht, H, i, j);
        const bool in = ht < ring_nodes(H) && grid_place(p, x0, y0, H, i, j, xw, yw);
        if (in) step_pulls<T>(A, p, xw, yw, g);
        ring_place(ht + kHalf, H, i2, j2);
        const bool in2 = ht + kHalf < ring_nodes(H) && grid_place(p, x0, y0, H, i2, j2, xw, yw);
        if (in2) step_pulls<T>(A, p, xw, yw, v);
        if (in) put(i, j, g);
        if (in2) put(i2, j2, v);
      }
    } else if (!second) {
      if (live) step_pulls<T>(A, p, x, y, g);
    } else {
      s_mask[ht] = 0;
      stage_records<T>(p, it.m0, min(kChunk, it.m1 - it.m0), ht, s_k);
    }
    __syncthreads();
    for (int c0 = it.m0;;) {
      const int cnt = min(kChunk, it.m1 - c0);
      if constexpr (MARK)
        marker_forces<T>(p, ib, x0, y0, S, cnt, k.record != 0, tid, s_m, s_k, s_mask);
      else
        mark_nodes<T>(p, x0, y0, S, cnt, tid, s_k, s_mask);
      __syncthreads();
      if (!second) spread_masked<T>(p, s_k, s_mask[ht], x, y, fibx, fiby);
      c0 += kChunk;
      if (c0 >= it.m1) break;
      __syncthreads();
      if (second) s_mask[ht] = 0;
      if constexpr (MARK) {
        if (!second) stage_markers<T>(p, ib, S, c0, min(kChunk, it.m1 - c0), ht, s_k);
      } else {
        if (second) stage_records<T>(p, c0, min(kChunk, it.m1 - c0), ht, s_k);
      }
      __syncthreads();
    }
  }
  if (!live) return;
  const CollK<T> &K = coll<T>(p);
  T out[9], rho;
  if (forced) {
    const ForceK<T> F = force_terms<T>(K, (T)(p.Gx + (double)fibx), (T)(p.Gy + (double)fiby));
    collide<T>(g, F, K, out, rho);
  } else {
    collide<T>(g, gforce<T>(p), K, out, rho);
  }
  const unsigned off = ((unsigned)y * (unsigned)p.pitch + (unsigned)x) * (unsigned)sizeof(T);
#pragma unroll
  for (int q = 0; q < 9; ++q)
    store_uniform<T, false>((global_ptr<char>)reinterpret_cast<char *>(B + (long long)q * p.plane), off, out[q]);
  const long long base = (long long)y * p.pitch + x;
  if (p.inlet && x == 1) {
    // inlet ghost: equilibrium at the inflow velocity, density of column 1
    const T dr = inlet_dr<T>(out);
#pragma unroll
    for (int q = 0; q < 9; ++q) B[(long long)q * p.plane + base - 1] = inlet_ghost<T>(dr, p, q);
  }
  if (p.outlet && x == p.nx - 2) {
    if (p.outlet == 1) {
#pragma unroll
      for (int q = 0; q < 9; ++q) B[(long long)q * p.plane + base + 1] = out[q];
    } else {
      conv_outlet_node<T>(A, B, p, base, out);
    }
  }
  if (!rho_ok(rho)) p.flag[0] = -1;
}

// the body forces of the step whose marker forces are in k (one workgroup per body)
__global__ __launch_bounds__(kHalf) void step_flush_kernel(IbParams ib, StepLink k, MoveParams mp) {
  __shared__ double red[3][kHalf / 64];
  body_reduce<kHalf>(ib, k.Fx, k.Fy, ib.slot[k.word], (int)blockIdx.x, (int)threadIdx.x, red);
  if (mp.nb) {
    __syncthreads();
    move_body<kHalf>(mp, (int)blockIdx.x, (int)threadIdx.x);
  }
}

// whether a launch shape's tiles are those of the one-launch step
bool variant_has_step(int variant) {
  int tx, ty;
  variant_tile(variant, &tx, &ty);
  return variant == 6 && tx == kTX && ty == kTY;
}

template <typename T, bool MARK, bool MOVE>
static void launch_step_t(const void *A, void *B, const LbmParams &p, const StepWork &w, const IbParams &ib,
                          const StepLink &k, const Motion<MOVE> &motion, int blocks, hipStream_t s) {
  hipLaunchKernelGGL((step_kernel<T, MARK, MOVE>), dim3(blocks), dim3(kBlock), 0, s, (const T *)A, (T *)B, p, w, ib,
                     k, motion);
}
template <typename T>
static void launch_step_p(bool mark, const void *A, void *B, const LbmParams &p, const StepWork &w,
                          const IbParams &ib, const StepLink &k, const MoveParams &mp, int blocks, hipStream_t s) {
  if (mp.nb)  // (only steps that form the marker forces have moving bodies)
    launch_step_t<T, true, true>(A, B, p, w, ib, k, Motion<true>{mp}, blocks, s);
  else if (mark)
    launch_step_t<T, true, false>(A, B, p, w, ib, k, Motion<false>{}, blocks, s);
  else
    launch_step_t<T, false, false>(A, B, p, w, ib, k, Motion<false>{}, blocks, s);
}

hipError_t launch_step(int prec, bool mark, const void *A, void *B, const LbmParams &p, const StepWork &w,
                       const IbParams &ib, const StepLink &k, const MoveParams &mp, hipStream_t s) {
  const int blocks = w.count + (k.count ? (k.reduce || mp.nb ? ib.nb : 0) + 1 : 0);
  if (blocks <= 0) return hipSuccess;
  if (prec == 4)
    launch_step_p<float>(mark, A, B, p, w, ib, k, mp, blocks, s);
  else
    launch_step_p<double>(mark, A, B, p, w, ib, k, mp, blocks, s);
  return hipGetLastError();
}

hipError_t launch_step_flush(const IbParams &ib, const StepLink &k, const MoveParams &mp, hipStream_t s) {
  if (ib.nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(step_flush_kernel, dim3(ib.nb), dim3(kHalf), 0, s, ib, k, mp);
  return hipGetLastError();
}

}  // namespace btdf
