// btdf_internal.h -- host-side state of a simulation handle and the helpers
// shared by the single-case API (btdf_api.hip) and the batch API
// (btdf_batch.hip). Internal to the library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <exception>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "btdf.h"
#include "btdf_launch.h"

#define HIPCHK(call)                                                                            \
  do {                                                                                          \
    hipError_t e_ = (call);                                                                     \
    if (e_ != hipSuccess) return btdf::host::fail(BTDF_EDEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

// Pinned host memory that the force reads' report kernel writes, shared by
// all handles of the process: kPages pages in one allocation, made by the
// second read of any handle (a program that reads once does not pay for it)
// and given back with the last handle. A read holds a page for its own
// length; where all are taken (more threads reading at once) or the memory is
// not to be had, it goes by copies. (A buffer per handle, grown as needed,
// cost 64 cases of a batch 1.1 ms in their second read and 12.5 ms when they
// were destroyed, and a history longer than any before up to 0.5 ms.)
class btdf_report_pages {
 public:
  static constexpr int kPages = 4;
  static constexpr size_t kBytes = 64 * 1024;
  void enter();
  void leave();
  double *take();  // null: none
  void give(double *page);

 private:
  std::mutex mu;
  char *base = nullptr;
  unsigned taken = 0;
  int handles = 0, reads = 0;  // (reads since the memory was last to be asked for)
};
btdf_report_pages &report_pages();
// a handle's share in them
struct btdf_report_user {
  btdf_report_user() { report_pages().enter(); }
  ~btdf_report_user() { report_pages().leave(); }
  btdf_report_user(const btdf_report_user &) = delete;
  btdf_report_user &operator=(const btdf_report_user &) = delete;
};

// HIP events of the timed stepping calls: created on first use and kept
// until the handle is destroyed, so timing a run neither creates nor
// destroys events while its steps are in flight
struct btdf_event_pool {
  std::vector<hipEvent_t> ev;
  hipError_t reserve(size_t n) {
    while (ev.size() < n) {
      hipEvent_t e = nullptr;
      const hipError_t r = hipEventCreate(&e);
      if (r != hipSuccess) return r;
      ev.push_back(e);
    }
    return hipSuccess;
  }
  void release() {
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    ev.clear();
  }
};

struct btdf_sim {
  void *owner = nullptr;  // the batch this handle is a case of (null: stand-alone)
  // configuration
  int nx = 0, ny = 0;
  int bc[4] = {0, 0, 0, 0};
  int prec = 8;
  int hist_cap = 4096;
  int kind = btdf::kCos4;
  double tau = 1.0, drs = 1.0;
  double G[2] = {0, 0}, uin[2] = {0, 0};
  double rho0 = 1.0, u0[2] = {0, 0};
  hipStream_t stream = nullptr;
  // bodies (host copies)
  std::vector<double> X, Y, U, V, sdrs;
  std::vector<int> off{0};
  std::vector<double> cx, cy, bsdrs;
  std::vector<char> stage;  // host image of the body part, sent in one copy
  // lattice kernel launch shape and tiles
  // launch defaults measured fastest on the 8192^2 particle-laden workload:
  // 32x8 tiles, general pull, marker kernel before the lattice kernel
  int variant = 6, xcd_remap = 1, graph_chunk = 0, interior = 1;
  int row_pad = 0, plane_pad = 0;
  int row_align = 128;  // bytes; rows start on this boundary (0: packed rows)
  int tile_x = 64, tile_y = 4, ntx = 0, nty = 0;
  std::vector<int> tile_off, tile_list;
  std::vector<int> tile_map;  // tiles no marker touches first, then the forced tiles
  int n_free = 0, n_forced = 0;
  int nf = 1;                 // forcing passes per step
  std::vector<int> cover_off, cover_list;  // covering markers per stencil node (nf > 1)
  int method = BTDF_FORCING_DIRECT;        // how the marker force is formed and spread
  std::vector<double> minv;                // implicit: (D_I D_E)^-1 per body, column-major
  std::vector<long long> minv_off;         // implicit: start of each body's matrix in minv
  std::vector<double> s_rkpm;              // RKPM: spreading factor ds epsilon_l per marker
  std::vector<double> bds;                 // arc length per marker of each body
  int max_body = 0;                        // markers of the largest body
  bool own_bodies = false;                 // marker forces body by body (btdf_body.hip)
  std::string method_err;                  // set-up failure of the implicit / RKPM matrices
  // rigid motion (host mirror of the device integration): per body a moving
  // flag, angle, velocity and angular velocity, per marker its offset from
  // the centre at angle 0; tile lists carry a margin and are rebuilt before
  // any marker can have moved by more than it
  std::vector<int> bmoving;
  std::vector<double> theta, bvx, bvy, bom, brad;
  std::vector<double> rx, ry;
  int margin = 0;
  int64_t steps_to_rebin = 0;
  // temporal blocking: tiles taking two steps at once, then the singly stepped regions
  int tblock = 1;  // option: 0 off, 1 the default depth, 2 to 5 steps per pass
  int edge_tiles = 0;  // option: tiles within reach of a domain edge take the blocked pass
  int depth = 1;   // steps per pass of the tiles away from the bodies (set with the layout)
  bool reserve_pass = false;  // keep the blocked pass's buffers whatever the launch shape (batch cases)
  // the tile map of the pass: its groups level by level (first tile of each
  // group), then the near tiles
  std::vector<int> fmap;
  std::vector<unsigned char> near;  // per lattice tile: 1 if it steps singly
  std::vector<unsigned> rwin;       // per fmap entry of a ring group (deeper passes): the near flags around it
  int gkind[btdf::kLevels] = {};  // shape per level (set with the lists)
  int n_grp[btdf::kLevels] = {};  // groups per level
  int n_edge[btdf::kLevels] = {};  // of those, edge groups (first in the level's list)
  int n_ring[btdf::kLevels] = {};  // passes of four or five steps: groups bordering a near tile (listed first)
  bool beside = false;             // the pass's large groups run beside the near tiles' steps (pass_beside)
  long long pass_nodes = 0;        // grid nodes in the blocked pass (partial tiles counted by their nodes)
  int n_near = 0;
  // one-launch steps: what each workgroup does, over all tiles, then over the
  // pass's near tiles
  std::vector<btdf::StepItem> work;
  int n_work[2] = {0, 0}, n_work_forced[2] = {0, 0};  // entries, and those with markers
  int work_most[2] = {0, 0};                          // most markers of one entry
  int n_groups() const {
    int k = 0;
    for (int i = 0; i < btdf::kLevels; ++i) k += n_grp[i];
    return k;
  }
  int grp_start(int g) const {  // index of level g's first group in fmap
    int k = 0;
    for (int i = 0; i < g; ++i) k += n_grp[i];
    return k;
  }
  int pass_tiles() const {  // lattice tiles in the pass
    int k = 0;
    for (int i = 0; i < btdf::kLevels; ++i) k += btdf::group_tiles(gkind[i]) * n_grp[i];
    return k;
  }
  // device memory
  char *ws = nullptr;
  size_t ws_bytes = 0;
  bool ws_owned = false;
  // layout
  int pitch = 0;
  long long plane = 0;
  size_t off_pop[2] = {0, 0}, off_ctl = 0, grid_bytes = 0;
  size_t off_hist = 0, off_mk = 0, off_mkalt = 0, off_places = 0, off_mkw = 0, off_mkixy = 0, off_mkbody = 0, off_body = 0, off_boff = 0,
         off_toff = 0, off_tlist = 0, off_tmap = 0, off_coff = 0, off_clist = 0, off_mdfc = 0, off_mdff = 0,
         off_moff = 0, off_minv = 0, off_motion = 0, off_rxy = 0, off_fmap = 0, off_rwin = 0, off_near = 0, off_work = 0, off_pop3 = 0, off_pop4 = 0, off_pop5 = 0, off_pop6 = 0, total = 0;
  bool layout_ok = false;  // host layout current for bodies and tiles
  bool device_ok = false;  // body part uploaded into the workspace
  bool state_ok = false;   // populations hold a state
  bool stepped = false;    // a step ran after the state and the body part last changed
  int cur = 0;             // which population buffer holds the state
  int64_t steps = 0, hist_read = 0;
  int64_t forces_from = 0;   // first step whose ring entry matches the body set
  bool bodies_dirty = true;  // ring layout on the device predates the body set
  // graph of graph_chunk steps starting from buffer 0
  hipGraphExec_t graph = nullptr;
  int graph_depth = 0;  // steps per pass the graph was captured with (1: single steps)
  hipStream_t cap_stream = nullptr;
  // passes of four or five steps: the small groups' launches run on a second
  // stream beside the largest groups' (fork and join events)
  hipStream_t side = nullptr;
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  btdf_event_pool tev;  // events of the timed stepping calls
  btdf_report_user reports;

  int nb() const { return (int)cx.size(); }
  bool any_moving() const {
    for (int m : bmoving)
      if (m) return true;
    return false;
  }
  int nm() const { return (int)X.size(); }
  bool xper() const { return bc[0] == BTDF_PERIODIC; }
  bool yper() const { return bc[2] == BTDF_PERIODIC; }
  int i0() const { return xper() ? 0 : 1; }
  int i1() const { return xper() ? nx - 1 : nx - 2; }
  template <typename P>
  P *at(size_t o) const { return reinterpret_cast<P *>(ws + o); }
};


namespace btdf {
namespace host {

int fail(int code, const char *fmt, ...) noexcept;
inline int ok() { return BTDF_OK; }

// Every extern "C" entry runs its body through guard (guard_size for the
// size queries, which report 0): an exception thrown inside, such as a
// failed host allocation in a std::vector, becomes a status code and a
// message instead of crossing the C ABI.
template <typename F>
inline int guard(F &&body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc &) {
    return fail(BTDF_ENOMEM, "out of host memory");
  } catch (const std::exception &e) {
    return fail(BTDF_EDEVICE, "internal error: %s", e.what());
  } catch (...) {
    return fail(BTDF_EDEVICE, "internal error");
  }
}
template <typename F>
inline size_t guard_size(F &&body) noexcept {
  size_t v = 0;
  if (guard([&]() -> int {
        v = body();
        return BTDF_OK;
      }) != BTDF_OK)
    return 0;
  return v;
}
inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
bool valid_kind(int k);
void drop_graph(btdf_t *h);
void compute_layout(btdf_t *h);
void group_kinds(int variant, int prec, int d, int kind[kLevels]);
void bin_markers(const btdf_t *h, int tx, int ty, int ntx, int nty, std::vector<int> &off, std::vector<int> &list);
void cover_lists(const btdf_t *h, std::vector<int> &off, std::vector<int> &list);
// implicit / RKPM matrices of the current bodies ("" or the reason they cannot be formed)
constexpr int kMaxImplicitBody = 2048;
constexpr int kMoveMargin = 2;  // nodes a moving marker may travel between tile-list rebuilds
// Smallest lattice that blocks by default. Blocking pays from some 800 000
// nodes (FP64 640 000); per step, single / blocked, one cylinder, FP32 and
// FP64: 720^2 9.0 / 11.4 us and 14.0 / 14.8, 800^2 10.4 / 11.9 and 16.2 / 15.6,
// 900^2 12.9 / 12.6 and 19.7 / 16.1, 1000^2 14.5 / 12.6 and 23.6 / 17.0. The
// line is where it was set when both were slower and is part of the documented
// defaults (1 step per pass below it); a smaller lattice blocks when asked to.
constexpr long long kBlockMinNodes = 1ll << 20;
// steps per pass by default on a single lattice, where the launch shape has them
constexpr int kDefaultDepth = 5;
// width in tile columns of the bands down which groups two tiles tall are launched
constexpr int kSquareBand = 32;
// Most tiles with markers, and most workgroups, of the step kernel, where two
// launches in turn are as fast. Forming a marker in every tile it touches
// costs 2.5 times the marker kernel's reads, so it pays only while tiles are
// too few to fill the GPU. Per step, two launches / one, FP32 and FP64: 800^2
// with one cylinder 17.9 / 10.4 us and 26.0 / 16.1; 1024^2 with 31 of D = 24
// (350 tiles) 24.9 / 16.8 and 37.8 / 26.1, with 200 (1500) 27.4 / 24.7 and 40.1 /
// 34.4; without many markers 2000x1400 46.0 / 32.1 and 81.7 / 79.8, 2500x1800
// (9000 workgroups) 67.4 / 65.8 and 129.9 / 132.5, 3000x2000 87.8 / 89.7 and
// equal at 172.
constexpr int kStepMaxForced = 1536, kStepMaxWork = 8192;
// Most tiles with markers among a pass's near tiles whose markers the step
// kernel forms: beside the pass's groups every repeated read costs them time.
// Per step, marker kernel and step kernel / one launch, FP32 and FP64: 2048^2
// with 60 cylinders (480 tiles) equal at 33.7 us and 60.3, with 90 (643) 36.0 /
// 36.5 and 59.8 / 62.0, with 125 (937) 38.8 / 40.7 and 62.6 / 64.2, with 200
// (1434) 44.2 / 47.4 and 71.3 / 73.5; 2560^2 with 200 (1521) 53.4 / 59.6 and
// 100.9 / 102.0; with few, 2000x800 with one (25) 20.2 / 15.1 and 27.1 / 23.9.
constexpr int kStepMaxNear = 600;
// Most markers of a tile, where fewer tiles than kStepManyForced have any. A
// body traced with many markers per node makes a few tiles' chains the step's
// length, and each node of such a tile reads its own markers' values where the
// lattice kernel's waves read one marker's for all: per step, one launch / two,
// FP32 (FP64 alike), 200x120 with one body of D = 20, 207 markers in a tile
// 28.3 / 29.1 us, 302 47.7 / 40.6, 377 60.8 / 48.8; of D = 64, 285 38.6 / 38.9,
// 360 54.6 / 46.5. With 234 tiles of 279 (1024^2, 31 bodies) 38.8 / 51.5, of
// 604 93.3 / 95.6.
constexpr int kStepMaxMarkers = 288, kStepManyForced = 128;
std::string forcing_setup(btdf_t *h);
LbmParams make_params(const btdf_t *h);
IbParams make_ib(const btdf_t *h);
int ensure_device(btdf_t *h);
int check_flag(btdf_t *h);
int read_ctl(btdf_t *h, long long *ctr, int *flag);
int bind_impl(btdf_t *h, void *dev, size_t bytes);
int add_body_impl(btdf_t *h, int n, const double *xy, const double *uv, double cx, double cy, double ds,
                  int *body_id);
int destroy_impl(btdf_t *h);
// HIP events around the kernels of one step (timed stepping)
struct StepEvents {
  hipEvent_t ib0, ib1, a0, a1, b0, b1;
};
// A run of consecutive steps enqueued on one stream. One-launch steps
// (btdf_step.hip) leave their body forces to the next step's launch, so a run
// ends with finish_run; the marker forces alternate between two buffers so
// that the last step's are in the handle's own.
struct StepRun {
  int64_t left = 0;        // steps still to enqueue
  bool pending = false;    // the last one's body forces are not summed yet
  bool side = false;       // a pass's large groups are on the second stream (join_ev ends them)
  StepLink link{};
  int places = 0;          // moving bodies: which of the two sets of places the next one-launch step uses
};
// Whether a step takes one launch, over all tiles or (near) over the blocked
// pass's near tiles.
bool one_launch(const btdf_t *h, bool near);
// a one-launch step A -> B
int run_step(btdf_t *h, const LbmParams &p, const IbParams &ib, const void *A, void *B, bool near, hipStream_t s,
             StepRun *run);
StepWork step_work(const btdf_t *h, bool near);
int finish_run(btdf_t *h, const IbParams &ib, hipStream_t s, StepRun *run);
// one step from population buffer src into the other, on stream s
int enqueue_step(btdf_t *h, const LbmParams &p, const IbParams &ib, int src, hipStream_t s,
                 const StepEvents *te, StepRun *run);

}  // namespace host
}  // namespace btdf
