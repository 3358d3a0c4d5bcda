// btdf_body.hip -- the marker forces of a step, one workgroup per body, for
// the forcing methods that couple a body's markers: the implicit method
// (eq 17: the body's inverse matrix times its direct forces) and several
// forcing passes (eqs 29-31). In launches of their own each pass was a 16-lane
// kernel of a few microseconds of latency; here the passes of a body whose
// markers share stencil nodes with no other body follow one another behind
// workgroup barriers, with the nodes' rho and u* in registers and the weights
// and forces in LDS.
//
// 16 lanes per marker, one per stencil node, 64 markers at a time; R such
// rounds are kept in registers (bodies of at most 64 R markers). The
// arithmetic and its order are those of ib_kernel, ib_pass_kernel and
// idf_kernel, so the forces are the same bits.
#include "btdf_device.h"
#include "btdf_launch.h"
#include "btdf_tile.h"

namespace btdf {

// covering markers per stencil node kept in registers with their weights
template <int R>
constexpr int body_kept() {
  return R == 1 ? 8 : (R == 2 ? 4 : 0);
}

template <typename T, int R, bool IMPLICIT>
__global__ __launch_bounds__(1024) void body_kernel(const T *__restrict__ A, LbmParams p, IbParams ib) {
  constexpr int N = 64 * R, E = IMPLICIT ? 0 : body_kept<R>();
  constexpr bool kMat = IMPLICIT && R <= 2;  // the inverse fits the LDS
  __shared__ double s_F[2][N][2];
  __shared__ double s_w[IMPLICIT ? 1 : N][9];             // x then y weights, spreading factor
  __shared__ double s_M[kMat ? N * N : 1];
  const int tid = (int)threadIdx.x, b = (int)blockIdx.x;
  const int node = tid & 15, a = node & 3, c = node >> 2, gl = tid & 48;
  const int S = stencil_size(p.kind);
  const int l0 = ib.body_off[b], n = ib.body_off[b + 1] - l0;
  if (b == 0 && tid == 0) ib.slot[0] = (int)(p.step_ctr[0] % ib.hist_cap);
  const double *M = IMPLICIT ? ib.minv + ib.minv_off[b] : nullptr;
  double rk[R], uk[R], vk[R], W[R], rl[R], U[R], V[R], sd[R];
  // interpolation and direct force (eqs 9-14, 20)
  T g[R][9];
  int bx[R], by[R];
  double X[R], Y[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = (tid >> 4) + 64 * r, l = l0 + e;
    const bool act = e < n;
    X[r] = Y[r] = U[r] = V[r] = sd[r] = 0.0;
    if (act) {
      X[r] = ib.X[l];
      Y[r] = ib.Y[l];
      U[r] = ib.U[l];
      V[r] = ib.V[l];
      sd[r] = ib.sdrs[l];
    }
    bx[r] = stencil_base(p.kind, X[r]);
    by[r] = stencil_base(p.kind, Y[r]);
    if (act && a < S && c < S) {
      int i = bx[r] + a, j = by[r] + c;
      if (p.xper) i = wrap_index(i, p.nx);
      if (p.yper) j = wrap_index(j, p.ny);
      pull9<T>(A, p, i, j, g[r]);
    }
  }
  if constexpr (kMat)  // (static data: in flight beside the populations)
    for (int k = tid; k < n * n; k += 1024) s_M[k] = M[k];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = (tid >> 4) + 64 * r, l = l0 + e;
    const bool act = e < n, on = act && a < S && c < S;
    double ph = 0.0;
    if (act && node < 8 && a < S) ph = node < 4 ? phi(p.kind, (double)(bx[r] + a) - X[r]) : phi(p.kind, (double)(by[r] + a) - Y[r]);
    const double phx = __shfl(ph, gl + a, 64), phy = __shfl(ph, gl + 4 + c, 64);
    double wr = 0.0, wu = 0.0, wv = 0.0;
    W[r] = 0.0;
    rk[r] = 1.0;
    uk[r] = vk[r] = 0.0;
    if (on) {
      node_moments<T>(g[r], p, rk[r], uk[r], vk[r]);
      W[r] = phx * phy;
      wr = W[r] * rk[r];
      wu = W[r] * uk[r];
      wv = W[r] * vk[r];
    }
    wr = row_sum(wr);
    wu = row_sum(wu);
    wv = row_sum(wv);
    rl[r] = wr;
    const double Fx = 2.0 * wr * (U[r] - wu), Fy = 2.0 * wr * (V[r] - wv);
    if (act) {
      T *mw = reinterpret_cast<T *>(ib.mk_w) + 10 * (long long)l;
      if (node < 8) {
        mw[node] = (T)ph;
        if constexpr (!IMPLICIT) s_w[e][node] = ph;
      }
      if (node == 0) {
        s_F[0][e][0] = Fx;
        s_F[0][e][1] = Fy;
        if constexpr (!IMPLICIT) s_w[e][8] = sd[r];
        ib.rho_l[l] = wr;
        ib.ux_l[l] = wu;
        ib.uy_l[l] = wv;
        ib.mk_ixy[2 * l] = p.xper ? wrap_index(bx[r], p.nx) : bx[r];
        ib.mk_ixy[2 * l + 1] = p.yper ? wrap_index(by[r], p.ny) : by[r];
        if (!isfinite(Fx) || !isfinite(Fy) || !(sqrt(wu * wu + wv * wv) <= 0.3)) p.flag[0] = 1 + b;
      }
    }
  }
  __syncthreads();
  auto leave = [&](int e, double Fx, double Fy, double s) {  // the marker's force for the lattice kernel
    const int l = l0 + e;
    T *mw = reinterpret_cast<T *>(ib.mk_w) + 10 * (long long)l;
    ib.Fx[l] = Fx;
    ib.Fy[l] = Fy;
    mw[8] = (T)(Fx * s);
    mw[9] = (T)(Fy * s);
    if (!isfinite(Fx) || !isfinite(Fy)) p.flag[0] = 1 + b;
  };
  if constexpr (IMPLICIT) {
    if (tid >= n) return;
    double fx = 0.0, fy = 0.0;
    const double *Mt = kMat ? s_M : M;
#pragma unroll 8
    for (int j = 0; j < n; ++j) {
      const double m = Mt[(long long)j * n + tid];
      fx += m * s_F[0][j][0];
      fy += m * s_F[0][j][1];
    }
    leave(tid, fx, fy, ib.sdrs[l0 + tid]);
  } else {
    // the covering markers of each node: the first E with W s in registers
    int c0[R], c1[R], id[R][E > 0 ? E : 1];
    double Wm[R][E > 0 ? E : 1];
    auto weight = [&](int v, int &m) {
      m = (v >> 4) - l0;
      return s_w[m][(v >> 2) & 3] * s_w[m][4 + (v & 3)] * s_w[m][8];
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = (tid >> 4) + 64 * r;
      const bool on = e < n && a < S && c < S;
      c0[r] = c1[r] = 0;
      if (on) {
        c0[r] = ib.cover_off[16 * (l0 + e) + node];
        c1[r] = ib.cover_off[16 * (l0 + e) + node + 1];
      }
#pragma unroll
      for (int u = 0; u < E; ++u) {
        id[r][u] = 0;
        Wm[r][u] = 0.0;
        if (c0[r] + u < c1[r]) Wm[r][u] = weight(ib.cover_list[c0[r] + u], id[r][u]);
      }
    }
    for (int k = 1; k < ib.nf; ++k) {
      const double(*fin)[2] = s_F[(k - 1) & 1];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = (tid >> 4) + 64 * r;
        double fx = 0.0, fy = 0.0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
          const double ax = fmx(Wm[r][u], fin[id[r][u]][0], fx), ay = fmx(Wm[r][u], fin[id[r][u]][1], fy);
          if (c0[r] + u < c1[r]) {
            fx = ax;
            fy = ay;
          }
        }
        for (int q = c0[r] + E; q < c1[r]; ++q) {
          int m;
          const double w = weight(ib.cover_list[q], m);
          fx = fmx(w, fin[m][0], fx);
          fy = fmx(w, fin[m][1], fy);
        }
        double wu = 0.0, wv = 0.0;
        if (e < n && a < S && c < S) {
          wu = W[r] * (uk[r] + 0.5 * fx / rk[r]);
          wv = W[r] * (vk[r] + 0.5 * fy / rk[r]);
        }
        wu = row_sum(wu);
        wv = row_sum(wv);
        if (e < n && node == 0) {
          const double Fx = fin[e][0] + 2.0 * rl[r] * (U[r] - wu);
          const double Fy = fin[e][1] + 2.0 * rl[r] * (V[r] - wv);
          s_F[k & 1][e][0] = Fx;
          s_F[k & 1][e][1] = Fy;
          if (k == ib.nf - 1)
            leave(e, Fx, Fy, sd[r]);
          else if (!isfinite(Fx) || !isfinite(Fy))
            p.flag[0] = 1 + b;
        }
      }
      __syncthreads();
    }
  }
}

template <typename T, bool IMPLICIT>
static void launch_body_t(const void *A, const LbmParams &p, const IbParams &ib, hipStream_t s) {
  const dim3 g(ib.nb), t(1024);
  if (ib.max_body <= 64)
    hipLaunchKernelGGL((body_kernel<T, 1, IMPLICIT>), g, t, 0, s, (const T *)A, p, ib);
  else if (ib.max_body <= 128)
    hipLaunchKernelGGL((body_kernel<T, 2, IMPLICIT>), g, t, 0, s, (const T *)A, p, ib);
  else
    hipLaunchKernelGGL((body_kernel<T, 4, IMPLICIT>), g, t, 0, s, (const T *)A, p, ib);
}

hipError_t launch_body(int prec, const void *A, const LbmParams &p, const IbParams &ib, hipStream_t s) {
  if (ib.nb <= 0) return hipSuccess;
  if (ib.max_body < 1 || ib.max_body > kBodyMax || (ib.method != 1 && ib.nf < 2)) return hipErrorInvalidValue;
  if (prec == 4)
    (ib.method == 1 ? launch_body_t<float, true> : launch_body_t<float, false>)(A, p, ib, s);
  else
    (ib.method == 1 ? launch_body_t<double, true> : launch_body_t<double, false>)(A, p, ib, s);
  return hipGetLastError();
}

}  // namespace btdf
