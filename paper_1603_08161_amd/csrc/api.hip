// Host side of the C-ABI declared in include/vd.h: the lattice handle, the
// per-frame constraint build and the flip-flop schedule of Sec. 7.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/vd.h"
#include "../../include/vd_net.h"
#include "../../include/vd_track.h"
#include "../../include/vd_fusion.h"
#include "net_kernels.h"
#include "track_kernels.h"
#include "fusion_kernels.h"
#include "vd_device.h"
#include "vd_kernels.h"

static_assert(VD_TILE_KINDS == vd::kTileKinds, "tile kinds of vd.h and the kernels differ");

namespace vd {
// Finest state as float64 AoS (kernels.hip).
template <typename T>
hipError_t launch_state_out64(const LevelView<T>& L, const double* origin, double* pos,
                              double* rot, hipStream_t s);
// Warm start's exact step (kernels.hip): float -> T copy, and d += b v with
// b = -g.v / v.Av, the line minimum of E at fixed rotations; `part` holds
// 2 * kWarmStepPartials doubles.
constexpr int kWarmStepPartials = 1024;
template <typename T>
hipError_t launch_to_type(const float* in, T* out, int64_t n, hipStream_t s);
template <typename T>
hipError_t launch_warm_step(T* d, const T* g, const float* v, const T* av, int64_t n,
                            double* part, const unsigned char* act, int64_t N, hipStream_t s);
// d += h delta, on the points of the optimised set M only when act is given
template <typename T>
hipError_t launch_add_delta_in(T* d, const float* delta, double h, int64_t n,
                               const unsigned char* act, int64_t N, hipStream_t s);
}  // namespace vd

namespace vd {
namespace {

#define VD_TRY(expr)                                  \
  do {                                                \
    if ((expr) != hipSuccess) return VD_EHIP;         \
  } while (0)

#define VD_CHECK(expr)                                \
  do {                                                \
    int rc_ = (expr);                                 \
    if (rc_ != VD_OK) return rc_;                     \
  } while (0)

inline int blocks_of(int64_t n) { return (int)((n + 255) / 256); }

// Device allocations owned by a handle.
class Pool {
 public:
  ~Pool() { release_all(); }
  template <typename P>
  int alloc(P** p, size_t count) {
    *p = nullptr;
    if (count == 0) count = 1;
    void* q = nullptr;
    if (hipMalloc(&q, count * sizeof(P)) != hipSuccess) {
      (void)hipGetLastError();
      return VD_ENOMEM;
    }
    ptrs_.push_back(q);
    *p = static_cast<P*>(q);
    return VD_OK;
  }
  void release(void* p) {
    if (!p) return;
    auto it = std::find(ptrs_.begin(), ptrs_.end(), p);
    if (it != ptrs_.end()) {
      (void)hipFree(p);
      ptrs_.erase(it);
    }
  }
  void release_all() {
    for (void* p : ptrs_) (void)hipFree(p);
    ptrs_.clear();
  }

 private:
  std::vector<void*> ptrs_;
};

// HIP-event timing of launches by kernel class (VD_FLAG_PROFILE).
class EventTimer {
 public:
  ~EventTimer() {
    for (hipEvent_t e : pool_) (void)hipEventDestroy(e);
  }
  void reset() {
    recs_.clear();
    used_ = 0;
  }
  // Runs `launch` (returning hipError_t); when `on`, brackets it with a pair
  // of events attributed to kernel class `kind`; `count` is the number of
  // launches of that class between the two events (their mean is reported).
  template <typename F>
  int timed(bool on, int kind, hipStream_t s, F&& launch, int count = 1) {
    if (!on) return launch() == hipSuccess ? VD_OK : VD_EHIP;
    while (pool_.size() < used_ + 2) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return VD_EHIP;
      pool_.push_back(e);
    }
    const int a = (int)used_, b = (int)used_ + 1;
    used_ += 2;
    if (hipEventRecord(pool_[a], s) != hipSuccess) return VD_EHIP;
    if (launch() != hipSuccess) return VD_EHIP;
    if (hipEventRecord(pool_[b], s) != hipSuccess) return VD_EHIP;
    recs_.push_back(Rec{kind, a, b, count});
    return VD_OK;
  }
  // Mean microseconds and launch counts per kind (after the stream drained).
  int collect(double* us, int* n) const {
    double sum[VD_PROF_KINDS] = {0};
    for (int k = 0; k < VD_PROF_KINDS; ++k) n[k] = 0;
    for (const Rec& r : recs_) {
      float ms = 0.0f;
      if (hipEventElapsedTime(&ms, pool_[r.a], pool_[r.b]) != hipSuccess) return VD_EHIP;
      sum[r.kind] += 1000.0 * ms;
      n[r.kind] += r.count;
    }
    for (int k = 0; k < VD_PROF_KINDS; ++k) us[k] = n[k] ? sum[k] / n[k] : 0.0;
    return VD_OK;
  }

 private:
  struct Rec {
    int kind, a, b, count;
  };
  std::vector<hipEvent_t> pool_;
  size_t used_ = 0;
  std::vector<Rec> recs_;
};

template <typename T>
struct LevelData {
  int nx = 0, ny = 0, nz = 0, N = 0, ncell = 0;
  double h = 0;
  T *d = nullptr, *r = nullptr, *r2 = nullptr, *pa = nullptr, *pb = nullptr, *ap = nullptr,
    *ap2 = nullptr, *dinv = nullptr, *bnode = nullptr, *base = nullptr, *rot = nullptr;
  int* cell_map = nullptr;
  int* node_slot = nullptr;  // node -> row of A27r (-1: no data term)
  unsigned char* act = nullptr;  // optimised set M (VD_FLAG_ACTIVE_SET), else null
  T* A27r = nullptr;         // [N][kA27Row] 27-point data blocks of A, per node slot
  Scalars* sc = nullptr;
  double* scg[2] = {nullptr, nullptr};  // CG block partials [4][max_tiles], alternating
  double* gang = nullptr;               // head and slots of one-launch CG solves
  double* pe = nullptr;                 // energy block partials [3][energy blocks]
  int cap_pe = 0;                       // doubles in pe
  // constraint rows and cell cache
  int cap_rows = 0, cap_cells = 0;
  int *row_cell = nullptr, *sorted = nullptr, *seg_start = nullptr, *active_cell = nullptr;
  // scratch of the build: sorted rows' cells, the sort, counts per block
  unsigned* keys = nullptr;
  unsigned char *sort_temp = nullptr, *touched = nullptr;
  int *heads = nullptr, *node_counts = nullptr;
  T *row_f = nullptr, *row_sn = nullptr, *row_rho = nullptr, *K = nullptr, *bcell = nullptr;
  int ntiles = 0;     // workgroups of the current tile kind
  int max_tiles = 0;  // most workgroups over all tile kinds (partials capacity)
  int tile = 0;       // tile kind of the stencil / CG kernels
  int large = -1;     // tile kind of one-launch CG solves that no other covers

  int rblocks() const { return blocks_of(cap_rows); }

  LevelView<T> view(double wr) const {
    LevelView<T> v{};
    v.nx = nx; v.ny = ny; v.nz = nz; v.N = N; v.tile = tile; v.ntiles = ntiles;
    v.rblocks = rblocks();
    v.loop_tile = large >= 0 ? large : tile;
    v.loop_tiles = large >= 0 ? tile_blocks(large, nx, ny, nz) : ntiles;
    v.h = (T)h; v.wr = (T)wr;
    v.d = d; v.r = r; v.r2 = r2; v.pa = pa; v.pb = pb; v.ap = ap; v.ap2 = ap2;
    v.dinv = dinv; v.bnode = bnode; v.base = base; v.rot = rot;
    v.scg0 = scg[0]; v.scg1 = scg[1]; v.gang = gang; v.pe = pe;
    v.cell_map = cell_map; v.K = K; v.node_slot = node_slot; v.A27r = A27r;
    v.act = act;
    v.row_cell = row_cell; v.row_f = row_f; v.row_sn = row_sn; v.row_rho = row_rho;
    v.sc = sc;
    return v;
  }
  RowView<T> rows_view(int rows, int n_dense) const {
    RowView<T> v;
    v.rows = rows; v.n_dense = n_dense; v.cell = row_cell; v.f = row_f; v.sn = row_sn;
    v.rho = row_rho; v.sorted = sorted; v.seg_start = seg_start; v.bcell = bcell;
    v.active_cell = active_cell;
    return v;
  }
};

// Single-lattice dispatches of the workgroup kinds.
template <typename T>
Dispatch<T> tiles_of(const LevelView<T>& V) { return single(V, V.ntiles); }
template <typename T>
Dispatch<T> loop_tiles_of(const LevelView<T>& V) { return single(V, V.loop_tiles); }
template <typename T>
Dispatch<T> nodes_of(const LevelView<T>& V) { return single(V, node_blocks(V.N)); }
template <typename T>
Dispatch<T> energy_of(const LevelView<T>& V) { return single(V, energy_blocks(V.rblocks, V.N)); }
template <typename T>
Dispatch<T> one_of(const LevelView<T>& V) { return single(V, 1); }

// Whether a kernel on the current device may read `bytes` at p: inside one
// allocation of this device and on a float boundary.  Anything else (another
// device's memory, host memory, a range that a copy would refuse) is left to
// the copy.
bool readable_here(const void* p, size_t bytes) {
  int dev = 0;
  hipPointerAttribute_t at{};
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  const bool ok = (uintptr_t)p % sizeof(float) == 0 && hipGetDevice(&dev) == hipSuccess &&
                  hipPointerGetAttributes(&at, p) == hipSuccess &&
                  at.type == hipMemoryTypeDevice && at.device == dev &&
                  hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) == hipSuccess &&
                  (const char*)p + bytes <= (const char*)base + size;
  if (!ok) (void)hipGetLastError();
  return ok;
}

int bits_for(int n) {
  int b = 1;
  while ((1ll << b) < (long long)n) ++b;
  return b;
}

// Camera and association thresholds of the C-ABI, checked.
int camera_of(const vd_camera* c, const vd_assoc_params* a, CamAssoc* out) {
  if (!c || !a) return VD_EINVAL;
  if (c->width < 3 || c->height < 3 || (int64_t)c->width * c->height > (1ll << 30))
    return VD_EINVAL;
  const double v[7] = {c->fx, c->fy, c->cx, c->cy, a->eps_d, a->eps_n, a->eps_v};
  for (double x : v)
    if (!std::isfinite(x)) return VD_EINVAL;
  if (!(c->fx > 0.0) || !(c->fy > 0.0) || !(a->eps_d > 0.0) || !(a->eps_n > 0.0) ||
      !(a->eps_v > 0.0))
    return VD_EINVAL;
  out->W = c->width; out->H = c->height;
  out->fx = c->fx; out->fy = c->fy; out->cx = c->cx; out->cy = c->cy;
  out->eps_d = a->eps_d; out->eps_n = a->eps_n; out->eps_v = a->eps_v;
  return VD_OK;
}

}  // namespace

class ISolver {
 public:
  virtual ~ISolver() {}
  virtual int init() = 0;
  virtual int set_constraints(const vd_constraints* c) = 0;
  virtual int solve_frame(const vd_solve_opts* o, vd_solve_report* r) = 0;
  virtual int get_energy(double out[4]) = 0;
  virtual int get_state(float* pos, float* rot, int mem) = 0;
  virtual int get_state64(double* pos, double* rot, int mem) = 0;
  virtual int set_state(const float* pos, const float* rot, int mem) = 0;
  virtual int level_info(int level, int dims[3], double* h) const = 0;
  virtual int debug_apply(int level, const float* p, float* ap, int mem) = 0;
  virtual int debug_gradient(int level, const float* pos, const float* rot, float* g, int mem) = 0;
  virtual int debug_energy(int level, const float* pos, const float* rot, double out[4], int mem) = 0;
  virtual int debug_diag(int level, float* diag, int mem) = 0;
  virtual int debug_rotations(int level, const float* pos, const float* rot_prev, float* rot_out,
                              int mem) = 0;
  virtual int debug_prolong(int level, const float* coarse, float* out, int mem) = 0;
  virtual int tune(int iters, int* tile_out, double* us_out) = 0;
  virtual int warm_features(const float* prev2, uint16_t* x, int mem) = 0;
  virtual int profile(double* us, int* n) = 0;
  virtual int abandon_loops(int on) = 0;
  virtual int set_depth_frame(const vd_depth_frame* f) = 0;
  virtual int get_pose(double* pose) = 0;
  virtual int set_pose(const double* pose) = 0;
  virtual int track_frame(const vd_track_opts* o, vd_track_report* r) = 0;
  virtual int debug_associate(const float* disp, const float* rot, float* target, float* normal,
                              float* weight, int* pixel, int mem) = 0;
  virtual int get_active(int level, unsigned char* mask, int64_t* count, int* layers) = 0;
  virtual int fuse_depth(const vd_fuse_opts* o, int64_t* n_updated) = 0;
  virtual int get_tsdf(float* D, float* W, int* frames, int mem) = 0;
  virtual int set_tsdf(const float* D, const float* W, int mem) = 0;
  virtual int extract_mesh(int64_t capacity, float* canon, float* deformed, int* cells,
                           int* edges, int64_t* n_tri, int mem) = 0;
};

template <typename T>
class Solver final : public ISolver {
 public:
  Solver(const vd_lattice_desc& d, hipStream_t s) : desc_(d), stream_(s) {}
  ~Solver() override {
    if (graph_exec_[0]) (void)hipGraphExecDestroy(graph_exec_[0]);
    if (graph_exec_[1]) (void)hipGraphExecDestroy(graph_exec_[1]);
    if (gn_graph_) (void)hipGraphExecDestroy(gn_graph_);
    if (capture_stream_) (void)hipStreamDestroy(capture_stream_);
    if (h_flags_) (void)hipHostFree(h_flags_);
    if (h_sc_) (void)hipHostFree(h_sc_);
    if (h_pose_) (void)hipHostFree(h_pose_);
    pool_.release_all();
  }

  int init() override {
    L_ = desc_.num_levels;
    lv_.resize(L_);
    int dims[3] = {desc_.dims[0], desc_.dims[1], desc_.dims[2]};
    double h = desc_.spacing;
    for (int l = L_ - 1; l >= 0; --l) {
      LevelData<T>& v = lv_[l];
      v.nx = dims[0]; v.ny = dims[1]; v.nz = dims[2];
      if (v.nx < 2 || v.ny < 2 || v.nz < 2) return VD_EINVAL;
      const int64_t N = (int64_t)v.nx * v.ny * v.nz;
      if (N > (1ll << 30)) return VD_EINVAL;
      v.N = (int)N;
      v.h = h;
      v.ncell = (v.nx - 1) * (v.ny - 1) * (v.nz - 1);
      const int want = desc_.tile[l];
      if (want < 0 || want > kTileKinds) return VD_EINVAL;
      const bool masked = (desc_.flags & VD_FLAG_ACTIVE_SET) != 0;
      v.tile = want > 0 ? want - 1 : default_tile(v.nx, v.ny, v.nz, sizeof(T) == 8, masked,
                                                   (desc_.flags & VD_FLAG_ITERATIVE) != 0);
      v.ntiles = tile_blocks(v.tile, v.nx, v.ny, v.nz);
      if (sizeof(T) == 4) v.large = large_loop_tile(v.nx, v.ny, v.nz, masked);
      for (int k = 0; k < kTileKinds; ++k)
        v.max_tiles = std::max(v.max_tiles, tile_blocks(k, v.nx, v.ny, v.nz));
      for (int k = 0; k < 3; ++k) dims[k] = (dims[k] + 1) / 2;
      h *= 2.0;
    }
    for (int l = 0; l < L_; ++l) {
      LevelData<T>& v = lv_[l];
      const size_t N = v.N;
      VD_CHECK(pool_.alloc(&v.d, 3 * N));
      VD_CHECK(pool_.alloc(&v.r, 3 * N));
      VD_CHECK(pool_.alloc(&v.pa, 3 * N));
      VD_CHECK(pool_.alloc(&v.pb, 3 * N));
      VD_CHECK(pool_.alloc(&v.ap, 6 * N));
      VD_CHECK(pool_.alloc(&v.dinv, 3 * N));
      VD_CHECK(pool_.alloc(&v.bnode, 3 * N));
      VD_CHECK(pool_.alloc(&v.base, 3 * N));
      VD_CHECK(pool_.alloc(&v.rot, 9 * N));
      VD_CHECK(pool_.alloc(&v.cell_map, (size_t)v.ncell));
      VD_CHECK(pool_.alloc(&v.node_slot, N));
      VD_CHECK(pool_.alloc(&v.node_counts, (size_t)build_node_blocks(v.N)));
      VD_CHECK(pool_.alloc(&v.A27r, (size_t)kA27Row * N));
      VD_CHECK(pool_.alloc(&v.sc, 1));
      VD_TRY(hipMemsetAsync(v.sc, 0, sizeof(Scalars), stream_));
      VD_CHECK(pool_.alloc(&v.r2, 3 * N));
      VD_CHECK(pool_.alloc(&v.ap2, 3 * N));
      if (desc_.flags & VD_FLAG_ACTIVE_SET) {
        VD_CHECK(pool_.alloc(&v.act, N));
        VD_CHECK(pool_.alloc(&v.touched, N));
        VD_TRY(hipMemsetAsync(v.act, 1, N, stream_));
      }
      VD_CHECK(pool_.alloc(&v.scg[0], 4 * (size_t)v.max_tiles));
      VD_CHECK(pool_.alloc(&v.scg[1], 4 * (size_t)v.max_tiles));
      VD_CHECK(pool_.alloc(&v.gang, kGangHead + 2 * kGangSlots * (size_t)v.max_tiles));
      VD_CHECK(ensure_partials(v, 0));
    }
    for (int k = 0; k < kLoopKinds; ++k)
      VD_TRY(cg_loop_capacity<T>(k, (desc_.flags & VD_FLAG_ACTIVE_SET) != 0, &loop_cap_[k]));
    if ((desc_.flags & VD_FLAG_PROFILE) && (desc_.flags & VD_FLAG_GRAPH))
      VD_CHECK(pool_.alloc(&stamps_, 2 * kMaxStamped));  // written by captured CG launches
    // the canonical TSDF on the finest grid (Sec. 4): D = W = 0, never observed
    VD_CHECK(pool_.alloc(&tsdf_d_, (size_t)finest().N));
    VD_CHECK(pool_.alloc(&tsdf_w_, (size_t)finest().N));
    VD_CHECK(pool_.alloc(&frames_, (size_t)finest().N));
    VD_TRY(hipMemsetAsync(tsdf_d_, 0, sizeof(float) * finest().N, stream_));
    VD_TRY(hipMemsetAsync(tsdf_w_, 0, sizeof(float) * finest().N, stream_));
    VD_TRY(hipMemsetAsync(frames_, 0, sizeof(int) * finest().N, stream_));
    if (desc_.flags & VD_FLAG_ACTIVE_SET) {
      VD_CHECK(pool_.alloc(&prev_act_, (size_t)finest().N));
      VD_CHECK(pool_.alloc(&known_, (size_t)finest().N));
      VD_CHECK(pool_.alloc(&fresh_, (size_t)finest().N));
    }
    VD_CHECK(pool_.alloc(&d_flags_, 4));
    VD_TRY(hipHostMalloc((void**)&h_flags_, 8 * sizeof(int), hipHostMallocDefault));
    VD_TRY(hipHostMalloc((void**)&h_sc_, sizeof(Scalars), hipHostMallocDefault));
    VD_TRY(hipHostMalloc((void**)&h_pose_, 12 * sizeof(double), hipHostMallocDefault));
    VD_CHECK(ensure_track(0, 0, 0));
    for (int k = 0; k < 12; ++k) h_pose_[k] = (k == 0 || k == 4 || k == 8) ? 1.0 : 0.0;
    VD_TRY(hipMemcpyAsync(pose_d_, h_pose_, 12 * sizeof(double), hipMemcpyHostToDevice, stream_));
    VD_TRY(launch_set_rest<T>(nodes_of(finest().view(desc_.w_arap)), stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  // ---------------------------------------------------------------------
  int set_constraints(const vd_constraints* c) override {
    if (!c) return VD_EINVAL;
    if (c->n_dense < 0 || c->n_sparse < 0) return VD_EINVAL;
    if (c->n_dense + 3 * c->n_sparse > (1ll << 30)) return VD_EINVAL;
    if (c->n_dense > 0 && (!c->canon || !c->target || !c->normal)) return VD_EINVAL;
    if (c->n_sparse > 0 && (!c->sparse_canon || !c->sparse_target)) return VD_EINVAL;
    if (c->mem != VD_MEM_HOST && c->mem != VD_MEM_DEVICE) return VD_EINVAL;
    const int C = (int)c->n_dense, S = (int)c->n_sparse;
    // stage the inputs (the caller's buffers are not kept)
    VD_CHECK(ensure_staging(C, S));
    const struct { float* dst; const float* src; size_t bytes; } in[6] = {
        {st_canon_, c->canon, 12ull * C},           {st_target_, c->target, 12ull * C},
        {st_normal_, c->normal, 12ull * C},         {st_weight_, c->weight, c->weight ? 4ull * C : 0},
        {st_scanon_, c->sparse_canon, 12ull * S},   {st_starget_, c->sparse_target, 12ull * S}};
    // buffers of this device are read by the kernel that checks them
    bool direct = c->mem == VD_MEM_DEVICE;
    for (const auto& x : in)
      if (direct && x.bytes) direct = readable_here(x.src, x.bytes);
    const hipMemcpyKind kind = c->mem == VD_MEM_HOST ? hipMemcpyHostToDevice
                                                     : hipMemcpyDeviceToDevice;
    for (const auto& x : in)
      if (!direct && x.bytes)
        VD_TRY(hipMemcpyAsync(x.dst, x.src, x.bytes, kind, stream_));
    RawConstraints raw;
    raw.canon = st_canon_; raw.target = st_target_; raw.normal = st_normal_;
    raw.weight = c->weight ? st_weight_ : nullptr;
    raw.sparse_canon = st_scanon_; raw.sparse_target = st_starget_;
    raw.n_dense = C; raw.n_sparse = S;
    // validate before touching any per-level structure
    RawConstraints given = raw;
    Staging st{};
    if (direct) {
      given.canon = c->canon; given.target = c->target; given.normal = c->normal;
      given.weight = c->weight;
      given.sparse_canon = c->sparse_canon; given.sparse_target = c->sparse_target;
      st = {st_canon_, st_target_, st_normal_, st_weight_, st_scanon_, st_starget_};
    }
    const LevelData<T>& c0 = lv_[0];
    h_flags_[4] = h_flags_[5] = 0;
    VD_TRY(launch_stage(given, st, c0.nx, c0.ny, c0.nz, c0.h, desc_.origin, h_flags_ + 4, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    if (h_flags_[4]) return VD_EINVAL;
    if (h_flags_[5]) return VD_ERANGE;
    have_frame_ = false;
    return build_levels(raw, C, S, true);
  }

  // Per-level rows, binning and cell cache of the staged constraints.  With
  // `structure` false only the row values are recomputed: the canonical
  // positions (hence every row's cell, the sort by cell and the cell
  // segments) are those of the previous build.
  int build_levels(const RawConstraints& raw, int C, int S, bool structure) {
    const int rows = C + 3 * S;
    if (structure) VD_CHECK(ensure_rows(rows));
    BuildLevels<T> B{};
    SortLevels so{};
    B.n = so.n = L_;
    so.rows = rows;
    so.counted = 1;
    for (int l = 0; l < L_; ++l) {
      const LevelData<T>& v = lv_[l];
      SortLevel& q = so.level[l];
      q = sort_level(v.sort_temp, v.cap_rows, bits_for(v.ncell));
      q.kin = (const unsigned*)v.row_cell;
      q.kout = v.keys;
      q.vout = v.sorted;
      so.passes = std::max(so.passes, q.passes);
      BuildLevel<T>& b = B.level[l];
      b.L = v.view(desc_.w_arap);
      b.R = v.rows_view(rows, C);
      b.ncell = v.ncell; b.cap_cells = v.cap_cells; b.cell_map = v.cell_map; b.K = v.K;
      b.node_slot = v.node_slot; b.A27r = v.A27r; b.act = v.act; b.skeys = v.keys;
      b.heads = v.heads; b.nodes = v.node_counts; b.touched = v.act ? v.touched : nullptr;
    }
    VD_TRY(launch_build<T>(raw, B, so, desc_.origin, desc_.w_dense, desc_.w_sparse, structure,
                           scan_temp_, scan_temp_bytes_, stream_));
    rows_ = rows;
    n_dense_ = C;
    have_constraints_ = true;
    energy_fresh_ = false;
    if (structure && finest().act) VD_CHECK(grow());
    return VD_OK;
  }

  // Grid growth (Sec. 8): points of the finest level's new M that were not in
  // the previous M are initialised by extrapolating the deformation field,
  // layer by layer from the points already known (the previous M, then the
  // earlier layers).  The first build has no previous M and extrapolates
  // nothing.  Waits for the stream after every layer.
  int grow() {
    LevelData<T>& F = finest();
    const size_t N = F.N;
    growth_layers_ = 0;
    if (have_prev_act_) {
      VD_CHECK(ensure_debug());
      const LevelView<T> FV = F.view(desc_.w_arap);
      VD_TRY(hipMemcpyAsync(known_, prev_act_, N, hipMemcpyDeviceToDevice, stream_));
      for (;;) {
        VD_TRY(launch_fill_int(d_flags_ + 1, 1, 0, stream_));
        VD_TRY(launch_grow_layer<T>(FV, F.act, known_, dbg_t1_, dbg_t2_, fresh_, d_flags_ + 1,
                                    stream_));
        VD_TRY(hipMemcpyAsync(h_flags_ + 1, d_flags_ + 1, sizeof(int), hipMemcpyDeviceToHost,
                              stream_));
        VD_TRY(hipStreamSynchronize(stream_));
        if (h_flags_[1] == 0) break;
        VD_TRY(launch_grow_commit<T>(FV, dbg_t1_, dbg_t2_, fresh_, known_, stream_));
        ++growth_layers_;
      }
    }
    VD_TRY(hipMemcpyAsync(prev_act_, F.act, N, hipMemcpyDeviceToDevice, stream_));
    have_prev_act_ = true;
    return VD_OK;
  }

  // ---------------------------------------------------------------------
  int solve_frame(const vd_solve_opts* o, vd_solve_report* rep) override {
    if (!have_constraints_) return VD_ESTATE;
    int reset = (o && o->reset_to_rest) ? 1 : 0;
    const bool warm = o && o->init_delta;
    const bool target = o && o->energy_target > 0.0;
    if (o && (!(o->energy_target >= 0.0) || !std::isfinite(o->energy_target) || o->max_gn < 0))
      return VD_EINVAL;
    if (warm && o->init_mem != VD_MEM_HOST && o->init_mem != VD_MEM_DEVICE) return VD_EINVAL;
    if (o && o->warm_mode != 0 && o->warm_mode != 1) return VD_EINVAL;
    double e_init[2] = {0.0, 0.0};
    int warm_used = 0, gn_done = 0, reached = 0;
    if (reset && (warm || target)) {
      VD_TRY(launch_set_rest<T>(nodes_of(finest().view(desc_.w_arap)), stream_));
      reset = 0;
    }
    if (warm) VD_CHECK(apply_warm(o->init_delta, o->init_mem, o->warm_mode, e_init, &warm_used));
    if (target) {
      const int cap = o->max_gn > 0 ? o->max_gn : desc_.gn_iters[L_ - 1];
      VD_CHECK(run_target(o->energy_target, cap, &gn_done, &reached));
    } else if (desc_.flags & VD_FLAG_GRAPH) {
      VD_CHECK(run_graph(reset));
    } else {
      VD_CHECK(enqueue_frame(reset, stream_));
    }
    energy_fresh_ = true;
    VD_TRY(launch_count_frames<T>(finest().view(desc_.w_arap), frames_, stream_));
    if (rep) {
      std::memset(rep, 0, sizeof(*rep));
      VD_TRY(hipStreamSynchronize(stream_));
      for (int l = 0; l < L_; ++l) {
        if (target && l != L_ - 1) continue;
        VD_TRY(hipMemcpy(h_sc_, lv_[l].sc, sizeof(Scalars), hipMemcpyDeviceToHost));
        if (h_sc_->guard_hits) rep->bits |= VD_REPORT_PCG_GUARD;
        if (h_sc_->bar_timeouts) rep->bits |= VD_REPORT_BARRIER_TIMEOUT;
        rep->polar_fp64 += h_sc_->polar_fp64;
        rep->polar_keep += h_sc_->polar_keep;
        for (int k = 0; k < h_sc_->n_trace && rep->n_trace < VD_MAX_TRACE; ++k)
          rep->trace[rep->n_trace++] = h_sc_->trace[k];
        if (l == L_ - 1)
          for (int k = 0; k < 4; ++k) rep->energy[k] = h_sc_->energy[k];
      }
      if (rep->polar_fp64) rep->bits |= VD_REPORT_POLAR_FP64;
      if (rep->polar_keep) rep->bits |= VD_REPORT_POLAR_KEEP;
      if (warm && !warm_used) rep->bits |= VD_REPORT_WARM_REJECTED;
      rep->init_energy[0] = e_init[0];
      rep->init_energy[1] = e_init[1];
      rep->warm_used = warm_used;
      rep->gn_done = gn_done;
      rep->target_reached = reached;
      int pn[VD_PROF_KINDS];
      VD_CHECK(timer_.collect(rep->prof_us, pn));
      for (int k = 0; k < VD_PROF_KINDS; ++k) rep->prof_n[k] = pn[k];
    }
    return VD_OK;
  }

  // Mean durations of the timed launch classes of the last frame.
  int profile(double* us, int* n) override {
    VD_TRY(hipStreamSynchronize(stream_));
    VD_CHECK(timer_.collect(us, n));
    if (n_stamped_ > 0) {  // graph frames: the finest CG blocks' clock stamps
      std::vector<unsigned long long> h(2 * n_stamped_);
      VD_TRY(hipMemcpy(h.data(), stamps_, h.size() * sizeof(unsigned long long),
                       hipMemcpyDeviceToHost));
      int khz = 0;
      int dev = 0;
      VD_TRY(hipGetDevice(&dev));
      VD_TRY(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
      if (khz <= 0) return VD_EHIP;
      double sum = 0.0;
      for (int k = 0; k < n_stamped_; ++k) sum += (double)(h[2 * k + 1] - h[2 * k]);
      us[VD_PROF_CG_A] = sum * 1000.0 / khz / ((double)n_stamped_ * stamped_launches_);
      n[VD_PROF_CG_A] = n_stamped_ * stamped_launches_;
    }
    return VD_OK;
  }

  // Features of vd_net.h for the coming frame (see vd_warm_features).
  int warm_features(const float* prev2, uint16_t* x, int mem) override {
    if (!x || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    LevelData<T>& F = finest();
    const size_t N = F.N;
    VD_CHECK(ensure_debug());
    const float* p2 = prev2;
    if (prev2 && mem == VD_MEM_HOST) {
      VD_TRY(hipMemcpyAsync(dbg_f_, prev2, 12 * N, hipMemcpyHostToDevice, stream_));
      p2 = dbg_f_;
    }
    const size_t need = 2 * (size_t)std::max(n_dense_, 1);
    if (need > feat_cap_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(feat_scratch_);
      VD_CHECK(pool_.alloc(&feat_scratch_, need));
      feat_cap_ = need;
    }
    uint16_t* xd = x;
    if (mem == VD_MEM_HOST) {
      if (!feat_x_) VD_CHECK(pool_.alloc(&feat_x_, 8 * N));
      xd = feat_x_;
    }
    VD_TRY(net::launch_features<T>(F.view(desc_.w_arap), F.rows_view(rows_, n_dense_), p2,
                                   feat_scratch_, xd, stream_));
    if (mem == VD_MEM_HOST) {
      VD_TRY(hipMemcpyAsync(x, feat_x_, 16 * N, hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
    }
    return VD_OK;
  }

  int get_energy(double out[4]) override {
    if (!out) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    LevelData<T>& F = finest();
    if (!energy_fresh_) {
      const LevelView<T> V = F.view(desc_.w_arap);
      VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 0, stream_));
      energy_fresh_ = true;
    }
    VD_TRY(hipMemcpyAsync(h_sc_, F.sc, sizeof(Scalars), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    for (int k = 0; k < 4; ++k) out[k] = h_sc_->energy[k];
    return VD_OK;
  }

  int get_state64(double* pos, double* rot, int mem) override {
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    LevelData<T>& F = finest();
    const size_t N = F.N;
    const LevelView<T> V = F.view(desc_.w_arap);
    if (mem == VD_MEM_DEVICE) {
      VD_TRY(launch_state_out64<T>(V, desc_.origin, pos, rot, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
      return VD_OK;
    }
    double* buf = nullptr;
    VD_CHECK(pool_.alloc(&buf, 12 * N));
    int rc = VD_OK;
    if (launch_state_out64<T>(V, desc_.origin, pos ? buf : nullptr, rot ? buf + 3 * N : nullptr,
                              stream_) != hipSuccess ||
        (pos && hipMemcpyAsync(pos, buf, 24 * N, hipMemcpyDeviceToHost, stream_) != hipSuccess) ||
        (rot && hipMemcpyAsync(rot, buf + 3 * N, 72 * N, hipMemcpyDeviceToHost, stream_) !=
                    hipSuccess) ||
        hipStreamSynchronize(stream_) != hipSuccess)
      rc = VD_EHIP;
    pool_.release(buf);
    return rc;
  }

  int get_state(float* pos, float* rot, int mem) override {
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    LevelData<T>& F = finest();
    const size_t N = F.N;
    if (mem == VD_MEM_DEVICE) {
      VD_TRY(launch_state_io<T>(F.view(desc_.w_arap), desc_.origin, pos, rot, nullptr, nullptr, 0,
                                d_flags_, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
      return VD_OK;
    }
    VD_CHECK(ensure_debug());
    float* dpos = pos ? dbg_f_ : nullptr;
    float* drot = rot ? dbg_f_ + 3 * N : nullptr;
    VD_TRY(launch_state_io<T>(F.view(desc_.w_arap), desc_.origin, dpos, drot, nullptr, nullptr, 0,
                              d_flags_, stream_));
    if (pos) VD_TRY(hipMemcpyAsync(pos, dpos, 12 * N, hipMemcpyDeviceToHost, stream_));
    if (rot) VD_TRY(hipMemcpyAsync(rot, drot, 36 * N, hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int set_state(const float* pos, const float* rot, int mem) override {
    if (!pos) return VD_EINVAL;
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    LevelData<T>& F = finest();
    const size_t N = F.N;
    const float* dpos = pos;
    const float* drot = rot;
    VD_CHECK(ensure_debug());
    if (mem == VD_MEM_HOST) {
      VD_TRY(hipMemcpyAsync(dbg_f_, pos, 12 * N, hipMemcpyHostToDevice, stream_));
      dpos = dbg_f_;
      if (rot) {
        VD_TRY(hipMemcpyAsync(dbg_f_ + 3 * N, rot, 36 * N, hipMemcpyHostToDevice, stream_));
        drot = dbg_f_ + 3 * N;
      }
    }
    VD_TRY(hipMemsetAsync(d_flags_, 0, sizeof(int), stream_));
    VD_TRY(launch_check_finite(dpos, 3 * N, d_flags_, stream_));
    if (drot) VD_TRY(launch_check_finite(drot, 9 * N, d_flags_, stream_));
    VD_TRY(hipMemcpyAsync(h_flags_, d_flags_, sizeof(int), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    if (h_flags_[0]) return VD_EINVAL;
    VD_TRY(launch_state_io<T>(F.view(desc_.w_arap), desc_.origin, nullptr, nullptr, dpos, drot, 1,
                              d_flags_, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    energy_fresh_ = false;
    return VD_OK;
  }

  // ---- tracking (vd_track.h) ---------------------------------------------
  int set_depth_frame(const vd_depth_frame* f) override {
    if (!f) return VD_EINVAL;
    CamAssoc cam;
    VD_CHECK(camera_of(&f->camera, &f->assoc, &cam));
    if (f->n_model < 0 || f->n_sparse < 0) return VD_EINVAL;
    if (f->n_model + 3 * f->n_sparse > (1ll << 30)) return VD_EINVAL;
    if (!f->depth || (f->n_model > 0 && (!f->model_canon || !f->model_normal)) ||
        (f->n_sparse > 0 && (!f->sparse_canon || !f->sparse_target)))
      return VD_EINVAL;
    if (f->mem != VD_MEM_HOST && f->mem != VD_MEM_DEVICE) return VD_EINVAL;
    const int C = (int)f->n_model, S = (int)f->n_sparse;
    const size_t npix = (size_t)cam.W * cam.H;
    VD_CHECK(ensure_staging(C, S));
    VD_CHECK(ensure_track(C, S, npix));
    const hipMemcpyKind kind = f->mem == VD_MEM_HOST ? hipMemcpyHostToDevice
                                                     : hipMemcpyDeviceToDevice;
    VD_TRY(hipMemcpyAsync(depth_, f->depth, 4 * npix, kind, stream_));
    if (C > 0) {
      VD_TRY(hipMemcpyAsync(st_canon_, f->model_canon, 12ull * C, kind, stream_));
      VD_TRY(hipMemcpyAsync(st_mnormal_, f->model_normal, 12ull * C, kind, stream_));
    }
    if (S > 0) {
      VD_TRY(hipMemcpyAsync(st_scanon_, f->sparse_canon, 12ull * S, kind, stream_));
      VD_TRY(hipMemcpyAsync(st_stcam_, f->sparse_target, 12ull * S, kind, stream_));
    }
    // validation: finite values, canonical points inside the coarsest level
    RawConstraints chk;
    chk.canon = st_canon_; chk.target = st_canon_; chk.normal = st_mnormal_; chk.weight = nullptr;
    chk.sparse_canon = st_scanon_; chk.sparse_target = st_stcam_;
    chk.n_dense = C; chk.n_sparse = S;
    VD_TRY(hipMemsetAsync(d_flags_, 0, sizeof(int), stream_));
    const LevelData<T>& c0 = lv_[0];
    VD_TRY(launch_validate(chk, c0.nx, c0.ny, c0.nz, c0.h, desc_.origin, d_flags_, stream_));
    VD_TRY(launch_check_finite(depth_, (int64_t)npix, d_flags_, stream_));
    VD_TRY(hipMemcpyAsync(h_flags_, d_flags_, sizeof(int), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    if (h_flags_[0] & 1) return VD_EINVAL;
    if (h_flags_[0] & 2) return VD_ERANGE;
    // the row structure of the model samples, with zero weights until the
    // first association fills them
    VD_TRY(launch_fill_float(st_target_, 3ll * C, 0.0f, stream_));
    VD_TRY(launch_fill_float(st_normal_, 3ll * C, 0.0f, stream_));
    VD_TRY(launch_fill_float(st_weight_, (int64_t)C, 0.0f, stream_));
    if (S > 0) VD_TRY(launch_to_model_frame(pose_d_, st_stcam_, st_starget_, S, stream_));
    cam_ = cam;
    have_depth_ = true;
    n_model_ = C;
    n_fsparse_ = S;
    VD_CHECK(build_levels(track_raw(), C, S, true));
    have_frame_ = true;
    return VD_OK;
  }

  int get_pose(double* pose) override {
    if (!pose) return VD_EINVAL;
    VD_TRY(hipMemcpyAsync(h_pose_, pose_d_, 12 * sizeof(double), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    std::memcpy(pose, h_pose_, 12 * sizeof(double));
    return VD_OK;
  }

  int set_pose(const double* pose) override {
    if (!pose) return VD_EINVAL;
    for (int k = 0; k < 12; ++k)
      if (!std::isfinite(pose[k])) return VD_EINVAL;
    VD_TRY(hipStreamSynchronize(stream_));
    std::memcpy(h_pose_, pose, 12 * sizeof(double));
    VD_TRY(hipMemcpyAsync(pose_d_, h_pose_, 12 * sizeof(double), hipMemcpyHostToDevice, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int track_frame(const vd_track_opts* o, vd_track_report* rep) override {
    if (!o) return VD_EINVAL;
    if (!have_frame_) return VD_ESTATE;
    if (o->rigid_iters < 0 || o->rigid_iters > VD_TRACK_MAX_ITERS || o->icp_iters < 0 ||
        o->icp_iters > VD_TRACK_MAX_ITERS)
      return VD_EINVAL;
    LevelData<T>& F = finest();
    const LevelView<T> FV = F.view(desc_.w_arap);
    if (o->reset_to_rest) VD_TRY(launch_set_rest<T>(nodes_of(FV), stream_));
    VD_TRY(launch_fill_int(kept_d_, VD_TRACK_MAX_ITERS, 0, stream_));
    const ModelView<T> mv = model_view(F.d, F.rot);
    const int G = rigid_blocks(n_model_);
    for (int it = 0; it < o->rigid_iters; ++it) {
      VD_TRY(launch_rigid_reduce_lattice<T>(cam_, depth_, mv, pose_d_, rigid_part_, G, stream_));
      VD_TRY(launch_rigid_solve(rigid_part_, G, pose_d_, rhist_d_ + 2 * it, stream_));
    }
    if (n_fsparse_ > 0)
      VD_TRY(launch_to_model_frame(pose_d_, st_stcam_, st_starget_, n_fsparse_, stream_));
    for (int it = 0; it < o->icp_iters; ++it) {
      VD_TRY(launch_assoc_lattice<T>(cam_, depth_, mv, pose_d_, st_target_, st_normal_,
                                     st_weight_, nullptr, kept_d_ + it, stream_));
      VD_CHECK(build_levels(track_raw(), n_model_, n_fsparse_, false));
      if (desc_.flags & VD_FLAG_GRAPH) {
        VD_CHECK(run_graph(0));
      } else {
        VD_CHECK(enqueue_frame(0, stream_));
      }
    }
    energy_fresh_ = o->icp_iters > 0;
    if (o->icp_iters > 0) VD_TRY(launch_count_frames<T>(FV, frames_, stream_));
    if (!rep) return VD_OK;
    std::memset(rep, 0, sizeof(*rep));
    if (!energy_fresh_) {
      VD_TRY(launch_energy<T>(energy_of(FV), one_of(FV), 0, stream_));
      energy_fresh_ = true;
    }
    VD_TRY(hipStreamSynchronize(stream_));
    VD_TRY(hipMemcpy(h_pose_, pose_d_, 12 * sizeof(double), hipMemcpyDeviceToHost));
    std::memcpy(rep->pose, h_pose_, sizeof(rep->pose));
    if (o->rigid_iters > 0)
      VD_TRY(hipMemcpy(rep->rigid_hist, rhist_d_, 2 * o->rigid_iters * sizeof(double),
                       hipMemcpyDeviceToHost));
    VD_TRY(hipMemcpy(rep->assoc_kept, kept_d_, VD_TRACK_MAX_ITERS * sizeof(int),
                     hipMemcpyDeviceToHost));
    for (int l = 0; l < L_; ++l) {
      VD_TRY(hipMemcpy(h_sc_, lv_[l].sc, sizeof(Scalars), hipMemcpyDeviceToHost));
      if (h_sc_->guard_hits) rep->bits |= VD_REPORT_PCG_GUARD;
      if (h_sc_->bar_timeouts) rep->bits |= VD_REPORT_BARRIER_TIMEOUT;
      if (h_sc_->polar_fp64) rep->bits |= VD_REPORT_POLAR_FP64;
      if (h_sc_->polar_keep) rep->bits |= VD_REPORT_POLAR_KEEP;
      if (l == L_ - 1)
        for (int k = 0; k < 4; ++k) rep->energy[k] = h_sc_->energy[k];
    }
    return VD_OK;
  }

  int debug_associate(const float* disp, const float* rot, float* target, float* normal,
                      float* weight, int* pixel, int mem) override {
    if (!disp || !rot || !target || !normal || !weight) return VD_EINVAL;
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    if (!have_frame_) return VD_ESTATE;
    VD_CHECK(ensure_debug());
    LevelData<T>& F = finest();
    const size_t N = F.N, M = n_model_;
    const hipMemcpyKind up = mem == VD_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    VD_TRY(hipMemcpyAsync(dbg_f_, disp, 12 * N, up, stream_));
    VD_TRY(launch_aos_to_soa<T>(dbg_f_, dbg_t1_, (int)N, 3, stream_));
    VD_TRY(hipMemcpyAsync(dbg_f_, rot, 36 * N, up, stream_));
    VD_TRY(launch_aos_to_soa<T>(dbg_f_, dbg_rot_, (int)N, 9, stream_));
    float *t = target, *n = normal, *w = weight;
    int* px = pixel;
    if (mem == VD_MEM_HOST) {
      if (M > dbg_assoc_cap_) {
        VD_TRY(hipStreamSynchronize(stream_));
        pool_.release(dbg_assoc_);
        VD_CHECK(pool_.alloc(&dbg_assoc_, 8 * M));
        dbg_assoc_cap_ = M;
      }
      t = dbg_assoc_;
      n = dbg_assoc_ + 3 * M;
      w = dbg_assoc_ + 6 * M;
      px = pixel ? (int*)(dbg_assoc_ + 7 * M) : nullptr;
    }
    VD_TRY(launch_assoc_lattice<T>(cam_, depth_, model_view(dbg_t1_, dbg_rot_), pose_d_, t, n, w,
                                   px, nullptr, stream_));
    if (mem == VD_MEM_HOST && M > 0) {
      VD_TRY(hipMemcpyAsync(target, t, 12 * M, hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipMemcpyAsync(normal, n, 12 * M, hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipMemcpyAsync(weight, w, 4 * M, hipMemcpyDeviceToHost, stream_));
      if (pixel) VD_TRY(hipMemcpyAsync(pixel, px, 4 * M, hipMemcpyDeviceToHost, stream_));
    }
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int get_active(int level, unsigned char* mask, int64_t* count, int* layers) override {
    if (level < 0 || level >= L_) return VD_EINVAL;
    LevelData<T>& v = lv_[level];
    std::vector<unsigned char> h(v.N, 1);
    if (v.act) {
      VD_TRY(hipMemcpyAsync(h.data(), v.act, v.N, hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
    }
    if (mask) std::memcpy(mask, h.data(), v.N);
    if (count) {
      int64_t c = 0;
      for (unsigned char b : h) c += b ? 1 : 0;
      *count = c;
    }
    if (layers) *layers = growth_layers_;
    return VD_OK;
  }

  // ---- fusion and mesh extraction (vd_fusion.h) ---------------------------
  int fuse_depth(const vd_fuse_opts* o, int64_t* n_updated) override {
    if (!o) return VD_EINVAL;
    if (!(o->tau > 0.0) || !std::isfinite(o->tau) || !(o->w_max >= 1.0) ||
        !std::isfinite(o->w_max) || o->k_min < 0)
      return VD_EINVAL;
    if (!have_depth_) return VD_ESTATE;
    const LevelData<T>& F = finest();
    FuseParams p;
    p.W = cam_.W; p.H = cam_.H;
    p.fx = cam_.fx; p.fy = cam_.fy; p.cx = cam_.cx; p.cy = cam_.cy;
    p.ox = desc_.origin[0]; p.oy = desc_.origin[1]; p.oz = desc_.origin[2]; p.h = F.h;
    p.tau = o->tau; p.w_max = o->w_max; p.k_min = o->k_min; p.all_points = o->all_points ? 1 : 0;
    if (n_updated) VD_TRY(launch_fill_int(d_flags_ + 2, 1, 0, stream_));
    VD_TRY(launch_fuse<T>(p, F.view(desc_.w_arap), depth_, pose_d_, frames_, tsdf_d_, tsdf_w_,
                          d_flags_ + 2, stream_));
    if (n_updated) {
      VD_TRY(hipMemcpyAsync(h_flags_ + 2, d_flags_ + 2, sizeof(int), hipMemcpyDeviceToHost,
                            stream_));
      VD_TRY(hipStreamSynchronize(stream_));
      *n_updated = h_flags_[2];
    }
    return VD_OK;
  }

  int get_tsdf(float* D, float* W, int* frames, int mem) override {
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    const size_t N = finest().N;
    const hipMemcpyKind k = mem == VD_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    if (D) VD_TRY(hipMemcpyAsync(D, tsdf_d_, 4 * N, k, stream_));
    if (W) VD_TRY(hipMemcpyAsync(W, tsdf_w_, 4 * N, k, stream_));
    if (frames) VD_TRY(hipMemcpyAsync(frames, frames_, 4 * N, k, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int set_tsdf(const float* D, const float* W, int mem) override {
    if (!D || !W || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
    const size_t N = finest().N;
    VD_CHECK(ensure_debug());
    const hipMemcpyKind k = mem == VD_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    VD_TRY(hipMemcpyAsync(dbg_f_, D, 4 * N, k, stream_));
    VD_TRY(hipMemcpyAsync(dbg_f_ + N, W, 4 * N, k, stream_));
    VD_TRY(hipMemsetAsync(d_flags_, 0, sizeof(int), stream_));
    VD_TRY(launch_check_finite(dbg_f_, 2 * (int64_t)N, d_flags_, stream_));
    VD_TRY(hipMemcpyAsync(h_flags_, d_flags_, sizeof(int), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    if (h_flags_[0]) return VD_EINVAL;
    std::vector<float> w(N);
    VD_TRY(hipMemcpy(w.data(), dbg_f_ + N, 4 * N, hipMemcpyDeviceToHost));
    for (float x : w)
      if (x < 0.0f) return VD_EINVAL;
    VD_TRY(hipMemcpyAsync(tsdf_d_, dbg_f_, 4 * N, hipMemcpyDeviceToDevice, stream_));
    VD_TRY(hipMemcpyAsync(tsdf_w_, dbg_f_ + N, 4 * N, hipMemcpyDeviceToDevice, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int extract_mesh(int64_t capacity, float* canon, float* deformed, int* cells, int* edges,
                   int64_t* n_tri, int mem) override {
    if (!n_tri || capacity < 0 || (capacity > 0 && !canon)) return VD_EINVAL;
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    if (mc_table_ready() != 0) return VD_EHIP;
    const LevelData<T>& F = finest();
    const int ncell = F.ncell;
    if (!mc_counts_) {
      VD_CHECK(pool_.alloc(&mc_counts_, (size_t)ncell));
      VD_CHECK(pool_.alloc(&mc_offsets_, (size_t)ncell));
      mc_scan_bytes_ = vd::scan_temp_bytes(ncell);
      VD_CHECK(pool_.alloc((unsigned char**)&mc_scan_temp_, mc_scan_bytes_));
    }
    VD_TRY(launch_mc_count(tsdf_d_, tsdf_w_, F.nx, F.ny, F.nz, mc_counts_, stream_));
    VD_TRY(exclusive_scan(mc_scan_temp_, mc_scan_bytes_, mc_counts_, mc_offsets_, ncell, stream_));
    int last[2] = {0, 0};
    VD_TRY(hipMemcpyAsync(&last[0], mc_offsets_ + ncell - 1, sizeof(int), hipMemcpyDeviceToHost,
                          stream_));
    VD_TRY(hipMemcpyAsync(&last[1], mc_counts_ + ncell - 1, sizeof(int), hipMemcpyDeviceToHost,
                          stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    const int64_t total = (int64_t)last[0] + last[1];
    *n_tri = total;
    if (total > capacity) return VD_ERANGE;
    if (total == 0) return VD_OK;
    float *dc = canon, *dd = deformed;
    int *dcell = cells, *dedge = edges;
    std::vector<void*> tmp;
    auto cleanup = [&]() {
      for (void* b : tmp) (void)hipFree(b);
    };
    if (mem == VD_MEM_HOST) {
      // temporaries of a synchronous host-bound call
      const size_t sz[4] = {36 * (size_t)total, deformed ? 36 * (size_t)total : 0,
                            cells ? 4 * (size_t)total : 0, edges ? 12 * (size_t)total : 0};
      void* bufs[4] = {nullptr, nullptr, nullptr, nullptr};
      for (int k = 0; k < 4; ++k) {
        if (!sz[k]) continue;
        if (hipMalloc(&bufs[k], sz[k]) != hipSuccess) {
          (void)hipGetLastError();
          cleanup();
          return VD_ENOMEM;
        }
        tmp.push_back(bufs[k]);
      }
      dc = (float*)bufs[0]; dd = (float*)bufs[1]; dcell = (int*)bufs[2]; dedge = (int*)bufs[3];
    }
    MeshParams mp;
    mp.ox = desc_.origin[0]; mp.oy = desc_.origin[1]; mp.oz = desc_.origin[2]; mp.h = F.h;
    hipError_t e = launch_mc_emit<T>(mp, F.view(desc_.w_arap), tsdf_d_, tsdf_w_, mc_counts_,
                                     mc_offsets_, pose_d_, dc, dd, dcell, dedge, stream_);
    if (e == hipSuccess && mem == VD_MEM_HOST) {
      e = hipMemcpyAsync(canon, dc, 36 * (size_t)total, hipMemcpyDeviceToHost, stream_);
      if (e == hipSuccess && deformed)
        e = hipMemcpyAsync(deformed, dd, 36 * (size_t)total, hipMemcpyDeviceToHost, stream_);
      if (e == hipSuccess && cells)
        e = hipMemcpyAsync(cells, dcell, 4 * (size_t)total, hipMemcpyDeviceToHost, stream_);
      if (e == hipSuccess && edges)
        e = hipMemcpyAsync(edges, dedge, 12 * (size_t)total, hipMemcpyDeviceToHost, stream_);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(stream_);
    cleanup();
    return e == hipSuccess ? VD_OK : VD_EHIP;
  }

  // ---- accessors used by the batched solve ---------------------------
  int levels() const { return L_; }
  LevelView<T> level_view(int l) const { return lv_[l].view(desc_.w_arap); }
  long generation() const { return alloc_gen_; }
  hipStream_t stream() const { return stream_; }
  bool has_constraints() const { return have_constraints_; }
  void mark_energy_fresh() { energy_fresh_ = true; }
  void mark_energy_stale() { energy_fresh_ = false; }
  const vd_lattice_desc& desc() const { return desc_; }
  int level_nodes(int l) const { return lv_[l].N; }
  int level_tile(int l) const { return lv_[l].tile; }
  // Whether a batch may run the solves of level l as one launch.  (It launches
  // all its lattices with one tile kind: none of the large.)
  bool level_loop(int l) const {
    return lv_[l].large < 0 && !(desc_.flags & VD_FLAG_ITERATIVE);
  }
  int level_tiles(int l, int kind) const {
    return tile_blocks(kind, lv_[l].nx, lv_[l].ny, lv_[l].nz);
  }
  void force_tile(int l, int kind) {
    if (lv_[l].tile == kind) return;
    lv_[l].tile = kind;
    lv_[l].ntiles = tile_blocks(kind, lv_[l].nx, lv_[l].ny, lv_[l].nz);
    desc_.tile[l] = kind + 1;
    ++alloc_gen_;
  }
  int finest_energy_host(double out[4]) {
    if (hipMemcpy(h_sc_, finest().sc, sizeof(Scalars), hipMemcpyDeviceToHost) != hipSuccess)
      return VD_EHIP;
    for (int k = 0; k < 4; ++k) out[k] = h_sc_->energy[k];
    return VD_OK;
  }

  int level_info(int level, int dims[3], double* h) const override {
    if (level < 0 || level >= L_) return VD_EINVAL;
    const LevelData<T>& v = lv_[level];
    if (dims) { dims[0] = v.nx; dims[1] = v.ny; dims[2] = v.nz; }
    if (h) *h = v.h;
    return VD_OK;
  }

  // ---- test entry points ----------------------------------------------
  int debug_apply(int level, const float* p, float* ap, int mem) override {
    if (level < 0 || level >= L_ || !p || !ap) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    VD_CHECK(ensure_debug());
    LevelData<T>& v = lv_[level];
    const int N = v.N;
    VD_CHECK(upload_aos(p, 3 * N, mem));
    VD_TRY(launch_convert<T>(dbg_f_, dbg_t1_, N, stream_));
    VD_TRY(launch_stencil<T>(kModeApply, tiles_of(v.view(desc_.w_arap)), dbg_t1_, dbg_t2_,
                             stream_));
    VD_TRY(launch_convert_back<T>(dbg_t2_, dbg_f_, N, stream_));
    return download_aos(ap, 3 * N, mem);
  }

  int debug_gradient(int level, const float* pos, const float* rot, float* g, int mem) override {
    if (level < 0 || level >= L_ || !pos || !rot || !g) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    LevelView<T> V;
    VD_CHECK(scratch_view(level, pos, rot, mem, &V));
    const int N = V.N;
    VD_TRY(launch_stencil<T>(kModeGrad, tiles_of(V), V.d, dbg_t2_, stream_));
    VD_TRY(launch_convert_back<T>(dbg_t2_, dbg_f_, N, stream_));
    return download_aos(g, 3 * N, mem);
  }

  int debug_energy(int level, const float* pos, const float* rot, double out[4], int mem) override {
    if (level < 0 || level >= L_ || !pos || !rot || !out) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    LevelView<T> V;
    VD_CHECK(scratch_view(level, pos, rot, mem, &V));
    LevelData<T>& v = lv_[level];
    VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 0, stream_));
    VD_TRY(hipMemcpyAsync(h_sc_, v.sc, sizeof(Scalars), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    for (int k = 0; k < 4; ++k) out[k] = h_sc_->energy[k];
    if (level == L_ - 1) energy_fresh_ = false;
    return VD_OK;
  }

  int debug_diag(int level, float* diag, int mem) override {
    if (level < 0 || level >= L_ || !diag) return VD_EINVAL;
    if (!have_constraints_) return VD_ESTATE;
    VD_CHECK(ensure_debug());
    LevelData<T>& v = lv_[level];
    const int N = v.N;
    std::vector<T> h(3 * (size_t)N);
    VD_TRY(hipMemcpyAsync(h.data(), v.dinv, sizeof(T) * 3 * N, hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    std::vector<float> out(3 * (size_t)N);
    for (int i = 0; i < N; ++i)
      for (int k = 0; k < 3; ++k) {
        const double di = (double)h[(size_t)k * N + i];
        out[3 * (size_t)i + k] = di > 0 ? (float)(1.0 / di) : 0.0f;
      }
    if (mem == VD_MEM_HOST) {
      std::memcpy(diag, out.data(), out.size() * sizeof(float));
    } else {
      VD_TRY(hipMemcpy(diag, out.data(), out.size() * sizeof(float), hipMemcpyHostToDevice));
    }
    return VD_OK;
  }

  int debug_rotations(int level, const float* pos, const float* rot_prev, float* rot_out,
                      int mem) override {
    if (level < 0 || level >= L_ || !pos || !rot_prev || !rot_out) return VD_EINVAL;
    LevelView<T> V;
    VD_CHECK(scratch_view(level, pos, rot_prev, mem, &V));
    const size_t N = V.N;
    VD_TRY(launch_polar<T>(nodes_of(V), stream_));
    float* drot = dbg_f_ + 3 * N;
    VD_TRY(launch_state_io<T>(V, desc_.origin, nullptr, drot, nullptr, nullptr, 0, d_flags_,
                              stream_));
    if (mem == VD_MEM_HOST) {
      VD_TRY(hipMemcpyAsync(rot_out, drot, 36 * N, hipMemcpyDeviceToHost, stream_));
    } else {
      VD_TRY(hipMemcpyAsync(rot_out, drot, 36 * N, hipMemcpyDeviceToDevice, stream_));
    }
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  int debug_prolong(int level, const float* coarse, float* out, int mem) override {
    if (level < 1 || level >= L_ || !coarse || !out) return VD_EINVAL;
    VD_CHECK(ensure_debug());
    LevelData<T>& c = lv_[level - 1];
    LevelData<T>& f = lv_[level];
    VD_CHECK(upload_aos(coarse, 3 * c.N, mem));
    VD_TRY(launch_convert<T>(dbg_f_, dbg_t1_, c.N, stream_));
    LevelView<T> Cv = c.view(desc_.w_arap), Fv = f.view(desc_.w_arap);
    Cv.d = dbg_t1_;
    Cv.base = nullptr;
    Fv.d = dbg_t2_;
    VD_TRY(launch_prolong<T>(nodes_of(Fv), nodes_of(Cv), 0, stream_));
    VD_TRY(launch_convert_back<T>(dbg_t2_, dbg_f_, f.N, stream_));
    return download_aos(out, 3 * f.N, mem);
  }

  int abandon_loops(int on) override {
    loop_ticks_ = on > 1 ? -on : on ? -1 : 0;
    ++alloc_gen_;  // captured schedules hold the old limit
    return VD_OK;
  }

  // Tile autotuner: times the CG iteration kernel with every tile kind.
  int tune(int iters, int* tile_out, double* us_out) override {
    if (!have_constraints_) return VD_ESTATE;
    if (iters < 1) return VD_EINVAL;
    const double wr = desc_.w_arap;
    hipEvent_t e0, e1;
    VD_TRY(hipEventCreate(&e0));
    VD_TRY(hipEventCreate(&e1));
    int rc = VD_OK;
    for (int l = 0; l < L_ && rc == VD_OK; ++l) {
      LevelData<T>& v = lv_[l];
      const size_t N = v.N;
      T* saved = nullptr;
      rc = pool_.alloc(&saved, 3 * N);
      if (rc != VD_OK) break;
      VD_TRY(hipMemcpyAsync(saved, v.d, 3 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
      double best = 1e300;
      int best_kind = v.tile;
      for (int kind = 0; kind < kTileKinds; ++kind) {
        v.tile = kind;
        v.ntiles = tile_blocks(kind, v.nx, v.ny, v.nz);
        const LevelView<T> V = v.view(wr);
        // the first pass warms up; the fastest of the next three counts (a
        // single timing is at the mercy of a disturbed run)
        float best_ms = 1e30f;
        for (int rep = 0; rep < 4; ++rep) {
          float ms = 0.0f;
          VD_TRY(hipMemcpyAsync(v.d, saved, 3 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
          // one position step as the solve launches it: the gradient pass
          // (which uses the same tile) and `iters` CG iterations with the
          // final step
          VD_TRY(hipEventRecord(e0, stream_));
          VD_TRY(launch_stencil<T>(kModeRhs, tiles_of(V), nullptr, nullptr, stream_));
          if (cg_loop(v)) {
            VD_TRY(launch_cg_loop<T>(iters, loop_tiles_of(V), stream_, nullptr,
                                     assemble_ticks(iters)));
          } else {
            for (int m = 0; m < iters; ++m) VD_TRY(launch_cg<T>(m, tiles_of(V), stream_));
            if (iters > 0) VD_TRY(launch_cg_final<T>(iters - 1, nodes_of(V), stream_));
          }
          VD_TRY(hipEventRecord(e1, stream_));
          VD_TRY(hipEventSynchronize(e1));
          VD_TRY(hipEventElapsedTime(&ms, e0, e1));
          if (rep > 0) best_ms = std::min(best_ms, ms);
        }
        const double us = 1000.0 * best_ms / iters;
        if (us_out) us_out[VD_TILE_KINDS * l + kind] = us;
        if (us < best) {
          best = us;
          best_kind = kind;
        }
      }
      v.tile = best_kind;
      v.ntiles = tile_blocks(best_kind, v.nx, v.ny, v.nz);
      desc_.tile[l] = best_kind + 1;
      if (tile_out) tile_out[l] = best_kind + 1;
      VD_TRY(hipMemcpyAsync(v.d, saved, 3 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(saved);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    ++alloc_gen_;  // schedules captured with the old tiles are stale
    energy_fresh_ = false;
    return rc;
  }

 private:
  LevelData<T>& finest() { return lv_[L_ - 1]; }

  // The frame's schedule (Sec. 7.1 flip-flop inside the Sec. 7.2 hierarchy),
  // queued on `s`.
  int enqueue_frame(int reset, hipStream_t s) {
    const double wr = desc_.w_arap;
    const bool trace = (desc_.flags & VD_FLAG_TRACE) != 0;
    const bool graph_prof = (desc_.flags & VD_FLAG_PROFILE) && (desc_.flags & VD_FLAG_GRAPH);
    const bool prof = (desc_.flags & VD_FLAG_PROFILE) && !graph_prof;
    timer_.reset();
    n_stamped_ = 0;
    const LevelView<T> FV = finest().view(wr);
    if (reset) VD_TRY(launch_set_rest<T>(nodes_of(FV), s));
    for (int l = 0; l < L_; ++l) VD_TRY(launch_reset_counters<T>(one_of(lv_[l].view(wr)), s));
    for (int l = 0; l < L_; ++l) {
      LevelData<T>& v = lv_[l];
      const LevelView<T> V = v.view(wr);
      const bool on = prof && l == L_ - 1;
      if (l < L_ - 1) VD_TRY(launch_inject<T>(nodes_of(V), nodes_of(FV), 1 << (L_ - 1 - l), s));
      if (l > 0) {
        const LevelView<T> C = lv_[l - 1].view(wr);
        VD_CHECK(timed(on, VD_PROF_TRANSFER, s,
                       [&] { return launch_prolong<T>(nodes_of(V), nodes_of(C), 1, s); }));
        VD_CHECK(timed(on, VD_PROF_ROTATION, s, [&] { return launch_polar<T>(nodes_of(V), s); }));
      }
      const int gn = desc_.gn_iters[l], pcg = desc_.pcg_iters[l];
      const bool loop = cg_loop(v);
      for (int k = 0; k < gn; ++k) {
        VD_CHECK(timed(on, VD_PROF_GRADIENT, s, [&] {
          return launch_stencil<T>(kModeRhs, tiles_of(V), nullptr, nullptr, s);
        }));
        if (loop && pcg > 0) {
          // captured frame: the loop itself stamps the start of iteration 1
          // and of its last step
          unsigned long long* stamp = nullptr;
          if (graph_prof && l == L_ - 1 && pcg > 1) {
            if (!stamps_) return VD_ESTATE;  // allocated at creation with both flags
            stamp = stamps_ + 2 * n_stamped_;
            if (n_stamped_ < kMaxStamped - 1) ++n_stamped_;
            stamped_launches_ = pcg - 1;
          }
          VD_CHECK(timed(on, VD_PROF_CG_LOOP, s, [&] {
            return launch_cg_loop<T>(pcg, loop_tiles_of(V), s, stamp, loop_ticks(pcg));
          }));
        } else if (graph_prof && l == L_ - 1 && pcg > 1) {
          // captured frame: the device clock at the start of CG iteration 1
          // and of the final step (first workgroup of each), written on
          // every replay, time iterations 1 .. pcg-1
          if (!stamps_) return VD_ESTATE;  // allocated at creation with both flags
          VD_TRY(launch_cg<T>(0, tiles_of(V), s));
          const int a = 2 * n_stamped_;
          for (int m = 1; m < pcg; ++m)
            VD_TRY(launch_cg<T>(m, tiles_of(V), s, m == 1 ? stamps_ + a : nullptr));
          if (n_stamped_ < kMaxStamped - 1) ++n_stamped_;
          stamped_launches_ = pcg - 1;
          VD_TRY(launch_cg_final<T>(pcg - 1, nodes_of(V), s, stamps_ + a + 1));
        } else {
          for (int m = 0; m < pcg; ++m)
            VD_CHECK(
                timed(on, VD_PROF_CG_A, s, [&] { return launch_cg<T>(m, tiles_of(V), s); }));
          if (pcg > 0)
            VD_CHECK(timed(on, VD_PROF_CG_B, s,
                           [&] { return launch_cg_final<T>(pcg - 1, nodes_of(V), s); }));
        }
        if (trace) VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 1, s));
        VD_CHECK(timed(on, VD_PROF_ROTATION, s, [&] { return launch_polar<T>(nodes_of(V), s); }));
        if (trace) VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 1, s));
      }
    }
    VD_CHECK(timed(prof, VD_PROF_ENERGY, s,
                   [&] { return launch_energy<T>(energy_of(FV), one_of(FV), 0, s); }));
    return VD_OK;
  }

  // Whether a level's CG solve runs as one launch: wherever all its tiles fit
  // on the GPU together, unless VD_FLAG_ITERATIVE asks for one launch per
  // iteration.
  bool cg_loop(const LevelData<T>& v) const {
    const int kind = v.large >= 0 ? v.large : v.tile;
    return !(desc_.flags & VD_FLAG_ITERATIVE) &&
           tile_blocks(kind, v.nx, v.ny, v.nz) <= loop_cap_[kind];
  }

  // How long a solve waits for its tiles (negative: test settings).
  int loop_ticks(int pcg) const { return loop_ticks_ < 0 ? loop_ticks_ : assemble_ticks(pcg); }

  template <typename F>
  int timed(bool on, int kind, hipStream_t s, F&& launch, int count = 1) {
    return timer_.timed(on, kind, s, launch, count);
  }

  int run_graph(int reset) {
    if (graph_gen_[reset] != alloc_gen_ || !graph_exec_[reset]) {
      if (graph_exec_[reset]) {
        VD_TRY(hipGraphExecDestroy(graph_exec_[reset]));
        graph_exec_[reset] = nullptr;
      }
      if (!capture_stream_)
        VD_TRY(hipStreamCreateWithFlags(&capture_stream_, hipStreamNonBlocking));
      VD_TRY(hipStreamSynchronize(stream_));
      hipGraph_t g = nullptr;
      VD_TRY(hipStreamBeginCapture(capture_stream_, hipStreamCaptureModeThreadLocal));
      const int rc = enqueue_frame(reset, capture_stream_);
      const hipError_t e = hipStreamEndCapture(capture_stream_, &g);
      if (rc != VD_OK) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
      }
      if (e != hipSuccess) return VD_EHIP;
      const hipError_t ei = hipGraphInstantiate(&graph_exec_[reset], g, nullptr, nullptr, 0);
      (void)hipGraphDestroy(g);
      if (ei != hipSuccess) return VD_EHIP;
      graph_gen_[reset] = alloc_gen_;
    }
    VD_TRY(hipGraphLaunch(graph_exec_[reset], stream_));
    return VD_OK;
  }

  // E_total of the finest state (waits for the stream).
  int finest_energy(double* e) {
    const LevelView<T> V = finest().view(desc_.w_arap);
    VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 0, stream_));
    VD_TRY(hipMemcpyAsync(h_sc_, V.sc, sizeof(Scalars), hipMemcpyDeviceToHost, stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    *e = h_sc_->energy[0];
    return VD_OK;
  }

  // Warm start: evaluate eq. (1) at the plain initialisation and at
  // d + h * delta (after one rotation fit), keep the lower.
  // step: 0 adds the prediction, 1 takes the exact line minimum along it
  int apply_warm(const float* delta, int mem, int step, double e[2], int* used) {
    LevelData<T>& F = finest();
    const size_t N = F.N;
    VD_CHECK(ensure_debug());
    if (!warm_d_) {
      VD_CHECK(pool_.alloc(&warm_d_, 3 * N));
      VD_CHECK(pool_.alloc(&warm_rot_, 9 * N));
    }
    if (step && !warm_g_) {
      VD_CHECK(pool_.alloc(&warm_g_, 3 * N));
      VD_CHECK(pool_.alloc(&warm_v_, 3 * N));
      VD_CHECK(pool_.alloc(&warm_av_, 3 * N));
      VD_CHECK(pool_.alloc(&warm_part_, 2 * kWarmStepPartials));
    }
    const float* dd = delta;
    if (mem == VD_MEM_HOST) {
      VD_TRY(hipMemcpyAsync(dbg_f_, delta, 12 * N, hipMemcpyHostToDevice, stream_));
      dd = dbg_f_;
    }
    VD_TRY(hipMemsetAsync(d_flags_, 0, sizeof(int), stream_));
    VD_TRY(launch_check_finite(dd, 3 * N, d_flags_, stream_));
    VD_TRY(hipMemcpyAsync(h_flags_, d_flags_, sizeof(int), hipMemcpyDeviceToHost, stream_));
    VD_CHECK(finest_energy(&e[0]));  // synchronises: h_flags_ is valid too
    if (h_flags_[0]) return VD_EINVAL;
    VD_TRY(hipMemcpyAsync(warm_d_, F.d, 3 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
    VD_TRY(hipMemcpyAsync(warm_rot_, F.rot, 9 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
    const LevelView<T> V = F.view(desc_.w_arap);
    if (step) {
      // g = J^T r at the plain state, A v, then d += b v with the exact line
      // minimum b = -g.v / v.Av at the current rotations (v in units of h)
      VD_TRY(launch_to_type<T>(dd, warm_v_, 3 * (int64_t)N, stream_));
      VD_TRY(launch_stencil<T>(kModeGrad, tiles_of(V), F.d, warm_g_, stream_));
      VD_TRY(launch_stencil<T>(kModeApply, tiles_of(V), warm_v_, warm_av_, stream_));
      VD_TRY(launch_warm_step<T>(F.d, warm_g_, dd, warm_av_, 3 * (int64_t)N, warm_part_, V.act,
                                 (int64_t)N, stream_));
    } else {
      VD_TRY(launch_add_delta_in<T>(F.d, dd, F.h, 3 * (int64_t)N, V.act, (int64_t)N, stream_));
    }
    VD_TRY(launch_polar<T>(nodes_of(V), stream_));
    VD_CHECK(finest_energy(&e[1]));
    *used = (e[1] <= e[0]) ? 1 : 0;
    if (!*used) {
      VD_TRY(hipMemcpyAsync(F.d, warm_d_, 3 * N * sizeof(T), hipMemcpyDeviceToDevice, stream_));
      VD_TRY(hipMemcpyAsync(F.rot, warm_rot_, 9 * N * sizeof(T), hipMemcpyDeviceToDevice,
                            stream_));
    }
    energy_fresh_ = false;
    return VD_OK;
  }

  // One finest-level flip-flop iteration; with `stop` every launch is
  // guarded by the device flag and the iteration ends with the target check.
  int enqueue_gn_finest(hipStream_t s, const int* stop = nullptr) {
    const LevelView<T> V = finest().view(desc_.w_arap);
    const int pcg = desc_.pcg_iters[L_ - 1];
    auto g = [&](const Dispatch<T>& D) { return guarded(D, stop); };
    VD_TRY(launch_stencil<T>(kModeRhs, g(tiles_of(V)), nullptr, nullptr, s));
    if (cg_loop(finest()) && pcg > 0) {
      VD_TRY(launch_cg_loop<T>(pcg, g(loop_tiles_of(V)), s, nullptr, loop_ticks(pcg)));
    } else {
      for (int m = 0; m < pcg; ++m) VD_TRY(launch_cg<T>(m, g(tiles_of(V)), s));
      if (pcg > 0) VD_TRY(launch_cg_final<T>(pcg - 1, g(nodes_of(V)), s));
    }
    VD_TRY(launch_polar<T>(g(nodes_of(V)), s));
    VD_TRY(launch_energy<T>(g(energy_of(V)), g(one_of(V)), 0, s));
    if (stop) VD_TRY(launch_target_step(V.sc, s));
    return VD_OK;
  }

  // Target mode: finest-level iterations until E <= target or `cap` of them,
  // decided on the device.  Every launch of an iteration is guarded by the
  // stop flag that the target check sets, so iterations queued beyond the
  // one that reaches the target cost only their empty launches.  The host
  // queues the previous call's iteration count at once (one graph launch per
  // iteration with VD_FLAG_GRAPH), waits, and then adds one iteration per
  // wait until the flag is set or `cap` are queued: one wait per frame when
  // consecutive frames need the same count, without paying for `cap` empty
  // iterations when the target comes early.
  int run_target(double target, int cap, int* done, int* reached) {
    const LevelView<T> V = finest().view(desc_.w_arap);
    const int* stop = &V.sc->stop;
    VD_TRY(launch_reset_counters<T>(one_of(V), stream_));
    VD_TRY(launch_energy<T>(energy_of(V), one_of(V), 0, stream_));
    VD_TRY(launch_target_begin(V.sc, target, stream_));
    const bool graph = (desc_.flags & VD_FLAG_GRAPH) != 0;
    if (graph && (gn_graph_gen_ != alloc_gen_ || !gn_graph_)) {
      if (gn_graph_) {
        VD_TRY(hipGraphExecDestroy(gn_graph_));
        gn_graph_ = nullptr;
      }
      if (!capture_stream_)
        VD_TRY(hipStreamCreateWithFlags(&capture_stream_, hipStreamNonBlocking));
      hipGraph_t gr = nullptr;
      VD_TRY(hipStreamBeginCapture(capture_stream_, hipStreamCaptureModeThreadLocal));
      const int rc = enqueue_gn_finest(capture_stream_, stop);
      const hipError_t ec = hipStreamEndCapture(capture_stream_, &gr);
      if (rc != VD_OK) {
        if (gr) (void)hipGraphDestroy(gr);
        return rc;
      }
      if (ec != hipSuccess) return VD_EHIP;
      const hipError_t ei = hipGraphInstantiate(&gn_graph_, gr, nullptr, nullptr, 0);
      (void)hipGraphDestroy(gr);
      if (ei != hipSuccess) return VD_EHIP;
      gn_graph_gen_ = alloc_gen_;
    }
    int queued = 0;
    int chunk = std::min(std::max(target_hint_, 1), cap);
    while (queued < cap) {
      for (int k = 0; k < chunk; ++k) {
        if (graph) VD_TRY(hipGraphLaunch(gn_graph_, stream_));
        else VD_CHECK(enqueue_gn_finest(stream_, stop));
      }
      queued += chunk;
      VD_TRY(hipMemcpyAsync(h_sc_, V.sc, sizeof(Scalars), hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
      if (h_sc_->stop) break;
      chunk = 1;
    }
    if (cap == 0) {
      VD_TRY(hipMemcpyAsync(h_sc_, V.sc, sizeof(Scalars), hipMemcpyDeviceToHost, stream_));
      VD_TRY(hipStreamSynchronize(stream_));
    }
    *done = h_sc_->gn_done;
    *reached = h_sc_->energy[0] <= target ? 1 : 0;
    target_hint_ = *done;
    return VD_OK;
  }

  int ensure_partials(LevelData<T>& v, int cap_rows) {
    const int need = 3 * energy_blocks(cap_rows, v.N);
    if (need <= v.cap_pe) return VD_OK;
    pool_.release(v.pe);
    VD_CHECK(pool_.alloc(&v.pe, (size_t)need));
    v.cap_pe = need;
    ++alloc_gen_;
    return VD_OK;
  }

  int ensure_staging(int C, int S) {
    if (C > cap_dense_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(st_canon_); pool_.release(st_target_); pool_.release(st_normal_);
      pool_.release(st_weight_);
      const size_t cap = (size_t)C + C / 4 + 64;
      VD_CHECK(pool_.alloc(&st_canon_, 3 * cap));
      VD_CHECK(pool_.alloc(&st_target_, 3 * cap));
      VD_CHECK(pool_.alloc(&st_normal_, 3 * cap));
      VD_CHECK(pool_.alloc(&st_weight_, cap));
      cap_dense_ = (int)cap;
    }
    if (S > cap_sparse_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(st_scanon_); pool_.release(st_starget_);
      const size_t cap = (size_t)S + S / 4 + 16;
      VD_CHECK(pool_.alloc(&st_scanon_, 3 * cap));
      VD_CHECK(pool_.alloc(&st_starget_, 3 * cap));
      cap_sparse_ = (int)cap;
    }
    return VD_OK;
  }

  int ensure_rows(int rows) {
    if (rows > cap_rows_ || !scan_temp_) {
      VD_TRY(hipStreamSynchronize(stream_));
      const int cap = rows + rows / 4 + 256;
      pool_.release(scan_temp_);
      scan_temp_bytes_ = vd::scan_temp_bytes(
          std::max(build_row_blocks(cap), build_node_blocks(finest().N)));
      VD_CHECK(pool_.alloc((unsigned char**)&scan_temp_, scan_temp_bytes_));
      cap_rows_ = cap;
      ++alloc_gen_;
    }
    for (int l = 0; l < L_; ++l) {
      LevelData<T>& v = lv_[l];
      if (rows > v.cap_rows || !v.row_cell) {
        const int cap = cap_rows_;
        pool_.release(v.row_cell); pool_.release(v.sorted); pool_.release(v.row_f);
        pool_.release(v.row_sn); pool_.release(v.row_rho);
        VD_CHECK(pool_.alloc(&v.row_cell, cap));
        VD_CHECK(pool_.alloc(&v.sorted, cap));
        VD_CHECK(pool_.alloc(&v.row_f, 3 * (size_t)cap));
        VD_CHECK(pool_.alloc(&v.row_sn, 3 * (size_t)cap));
        VD_CHECK(pool_.alloc(&v.row_rho, cap));
        pool_.release(v.keys); pool_.release(v.heads); pool_.release(v.sort_temp);
        VD_CHECK(pool_.alloc(&v.keys, cap));
        VD_CHECK(pool_.alloc(&v.heads, (size_t)build_row_blocks(cap)));
        VD_CHECK(pool_.alloc(&v.sort_temp, vd::sort_temp_bytes(cap)));
        v.cap_rows = cap;
        ++alloc_gen_;
      }
      const int cells = std::max(1, std::min(v.ncell, v.cap_rows));
      if (cells > v.cap_cells || !v.K) {
        pool_.release(v.K); pool_.release(v.bcell); pool_.release(v.seg_start);
        pool_.release(v.active_cell);
        VD_CHECK(pool_.alloc(&v.K, (size_t)cells * 384));
        VD_CHECK(pool_.alloc(&v.bcell, (size_t)cells * 24));
        VD_CHECK(pool_.alloc(&v.seg_start, (size_t)cells + 1));
        VD_CHECK(pool_.alloc(&v.active_cell, (size_t)cells));
        v.cap_cells = cells;
        ++alloc_gen_;
      }
      VD_CHECK(ensure_partials(v, v.cap_rows));
    }
    return VD_OK;
  }

  int ensure_debug() {
    if (dbg_f_) return VD_OK;
    const size_t N = finest().N;
    VD_CHECK(pool_.alloc(&dbg_f_, 12 * N));
    VD_CHECK(pool_.alloc(&dbg_t1_, 9 * N));
    VD_CHECK(pool_.alloc(&dbg_t2_, 9 * N));
    VD_CHECK(pool_.alloc(&dbg_rot_, 9 * N));
    return VD_OK;
  }

  ModelView<T> model_view(const T* d, const T* rot) {
    const LevelData<T>& F = finest();
    ModelView<T> m;
    m.canon = st_canon_; m.cnormal = st_mnormal_; m.M = n_model_;
    m.d = d; m.rot = rot;
    m.nx = F.nx; m.ny = F.ny; m.nz = F.nz; m.N = F.N;
    m.h = F.h; m.ox = desc_.origin[0]; m.oy = desc_.origin[1]; m.oz = desc_.origin[2];
    return m;
  }

  // The frame's rows: model samples with the association's targets,
  // normals and weights, and the sparse pairs in the lattice frame.
  RawConstraints track_raw() const {
    RawConstraints r;
    r.canon = st_canon_; r.target = st_target_; r.normal = st_normal_; r.weight = st_weight_;
    r.sparse_canon = st_scanon_; r.sparse_target = st_starget_;
    r.n_dense = n_model_; r.n_sparse = n_fsparse_;
    return r;
  }

  int ensure_track(int C, int S, size_t npix) {
    if (!pose_d_) {
      VD_CHECK(pool_.alloc(&pose_d_, 12));
      VD_CHECK(pool_.alloc(&rigid_part_, (size_t)kRigidStride * kRigidMaxBlocks));
      VD_CHECK(pool_.alloc(&rhist_d_, 2 * VD_TRACK_MAX_ITERS));
      VD_CHECK(pool_.alloc(&kept_d_, VD_TRACK_MAX_ITERS));
    }
    if (C > cap_mnormal_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(st_mnormal_);
      VD_CHECK(pool_.alloc(&st_mnormal_, 3 * (size_t)cap_dense_));
      cap_mnormal_ = cap_dense_;
    }
    if (S > cap_stcam_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(st_stcam_);
      VD_CHECK(pool_.alloc(&st_stcam_, 3 * (size_t)cap_sparse_));
      cap_stcam_ = cap_sparse_;
    }
    if (npix > depth_cap_) {
      VD_TRY(hipStreamSynchronize(stream_));
      pool_.release(depth_);
      VD_CHECK(pool_.alloc(&depth_, npix));
      depth_cap_ = npix;
    }
    return VD_OK;
  }

  int upload_aos(const float* src, size_t n, int mem) {
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    VD_TRY(hipMemcpyAsync(dbg_f_, src, n * sizeof(float),
                          mem == VD_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice,
                          stream_));
    return VD_OK;
  }

  int download_aos(float* dst, size_t n, int mem) {
    VD_TRY(hipMemcpyAsync(dst, dbg_f_, n * sizeof(float),
                          mem == VD_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice,
                          stream_));
    VD_TRY(hipStreamSynchronize(stream_));
    return VD_OK;
  }

  // A view of `level` whose d / rot are scratch copies of (pos - rest, rot).
  int scratch_view(int level, const float* pos, const float* rot, int mem, LevelView<T>* out) {
    if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
    VD_CHECK(ensure_debug());
    LevelData<T>& v = lv_[level];
    const size_t N = v.N;
    const hipMemcpyKind kind = mem == VD_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    VD_TRY(hipMemcpyAsync(dbg_f_, pos, 12 * N, kind, stream_));
    VD_TRY(hipMemcpyAsync(dbg_f_ + 3 * N, rot, 36 * N, kind, stream_));
    LevelView<T> V = v.view(desc_.w_arap);
    V.d = dbg_t1_;
    V.rot = dbg_rot_;
    VD_TRY(launch_state_io<T>(V, desc_.origin, nullptr, nullptr, dbg_f_, dbg_f_ + 3 * N, 1,
                              d_flags_, stream_));
    *out = V;
    return VD_OK;
  }

  vd_lattice_desc desc_;
  hipStream_t stream_;
  hipStream_t capture_stream_ = nullptr;
  hipGraphExec_t graph_exec_[2] = {nullptr, nullptr};
  long graph_gen_[2] = {-1, -1};
  long alloc_gen_ = 0;
  int L_ = 0;
  std::vector<LevelData<T>> lv_;
  Pool pool_;
  int* d_flags_ = nullptr;
  int* h_flags_ = nullptr;
  Scalars* h_sc_ = nullptr;
  // staging of the raw constraints
  float *st_canon_ = nullptr, *st_target_ = nullptr, *st_normal_ = nullptr, *st_weight_ = nullptr,
        *st_scanon_ = nullptr, *st_starget_ = nullptr;
  int cap_dense_ = 0, cap_sparse_ = 0;
  // sort scratch
  void* scan_temp_ = nullptr;
  size_t scan_temp_bytes_ = 0;
  int cap_rows_ = 0;
  int rows_ = 0, n_dense_ = 0;
  bool have_constraints_ = false;
  bool energy_fresh_ = false;
  EventTimer timer_;  // timing of the last profiled frame
  int loop_ticks_ = 0;  // negative: test settings of vd_debug_abandon_loops
  int loop_cap_[kLoopKinds] = {};  // most tiles of a one-launch CG solve, by tile kind
  // test scratch
  float* dbg_f_ = nullptr;
  T *dbg_t1_ = nullptr, *dbg_t2_ = nullptr, *dbg_rot_ = nullptr;
  // device clock stamps of a profiled graph frame
  static constexpr int kMaxStamped = 64;
  unsigned long long* stamps_ = nullptr;
  int n_stamped_ = 0, stamped_launches_ = 0;
  // warm start
  T *warm_d_ = nullptr, *warm_rot_ = nullptr;  // plain initialisation kept for the judge
  T *warm_g_ = nullptr, *warm_v_ = nullptr, *warm_av_ = nullptr;  // exact warm step
  double* warm_part_ = nullptr;
  hipGraphExec_t gn_graph_ = nullptr;          // one guarded finest-level iteration
  long gn_graph_gen_ = -1;
  int target_hint_ = 0;  // iterations the last target-mode call needed
  float* feat_scratch_ = nullptr;  // per-row residual pieces of the features
  size_t feat_cap_ = 0;
  uint16_t* feat_x_ = nullptr;     // features staged for a host copy
  // tracking (vd_track.h)
  CamAssoc cam_{};
  float* depth_ = nullptr;        // the frame's depth map
  size_t depth_cap_ = 0;
  float* st_mnormal_ = nullptr;   // canonical model normals
  float* st_stcam_ = nullptr;     // camera-frame sparse targets
  int cap_mnormal_ = 0, cap_stcam_ = 0;
  int n_model_ = 0, n_fsparse_ = 0;
  bool have_frame_ = false;
  double* pose_d_ = nullptr;      // global pose (R row-major, t), float64
  double* h_pose_ = nullptr;      // pinned host copy
  double* rigid_part_ = nullptr;  // rigid ICP workgroup partials
  double* rhist_d_ = nullptr;     // per rigid iteration: E, kept pairs
  int* kept_d_ = nullptr;         // kept pairs per association round
  float* dbg_assoc_ = nullptr;    // host-bound association outputs (test entry)
  size_t dbg_assoc_cap_ = 0;
  // optimised set M (VD_FLAG_ACTIVE_SET)
  unsigned char* prev_act_ = nullptr;  // the finest M of the previous build
  unsigned char* known_ = nullptr;     // grid growth: points already initialised
  unsigned char* fresh_ = nullptr;     // grid growth: the current layer
  bool have_prev_act_ = false;
  int growth_layers_ = 0;
  // canonical TSDF (vd_fusion.h)
  float* tsdf_d_ = nullptr;
  float* tsdf_w_ = nullptr;
  int* frames_ = nullptr;      // frames in a row each finest point has been in M
  bool have_depth_ = false;
  int* mc_counts_ = nullptr;   // marching cubes: triangles per cell
  int* mc_offsets_ = nullptr;  // their exclusive prefix sum
  void* mc_scan_temp_ = nullptr;
  size_t mc_scan_bytes_ = 0;
};

// ===========================================================================
// batched solve: one launch per schedule step over all lattices
// ===========================================================================

class IBatch {
 public:
  virtual ~IBatch() {}
  // Queue one frame of every lattice on `s` (graph replay or eager).
  // The most of the GPU that a lattice's one-launch solve holds (0: none).
  virtual double gang_share() = 0;
  virtual int launch(const vd_solve_opts* o, hipStream_t s) = 0;
  // Final energies (4 per lattice) after the frame finished.
  virtual int energies(double* e) = 0;
  virtual int profile(double* us, int* n) = 0;
  // Tile autotuner over the batched launches (see vd_batch_tune).
  virtual int tune(int iters, hipStream_t s, int* tile_out, double* us_out) = 0;
};

template <typename T>
class Batch final : public IBatch {
 public:
  enum Kind { kTiles = 0, kNodes = 1, kEnergy = 2, kOne = 3 };

  explicit Batch(std::vector<Solver<T>*> hs) : h_(std::move(hs)) {}
  ~Batch() override {
    for (auto& g : exec_)
      if (g) (void)hipGraphExecDestroy(g);
    if (capture_) (void)hipStreamDestroy(capture_);
    pool_.release_all();
  }

  int init() {
    n_ = (int)h_.size();
    L_ = h_[0]->levels();
    stream_ = h_[0]->stream();
    graph_ = (h_[0]->desc().flags & VD_FLAG_GRAPH) != 0;
    prof_ = !graph_ && (h_[0]->desc().flags & VD_FLAG_PROFILE) != 0;
    // one lattice with a set M and the launches are those with masks
    for (const auto* h : h_) masked_ |= (h->desc().flags & VD_FLAG_ACTIVE_SET) != 0;
    for (int k = 0; k < kTileKinds; ++k) VD_TRY(cg_loop_capacity<T>(k, masked_, &loop_cap_[k]));
    // one tile kind per level: that of the largest lattice if it was chosen
    for (int l = 0; l < L_; ++l) {
      int big = 0;
      for (int b = 1; b < n_; ++b)
        if (h_[b]->level_nodes(l) > h_[big]->level_nodes(l)) big = b;
      kinds_[l] = h_[big]->desc().tile[l] > 0 ? h_[big]->level_tile(l) : default_kind(l);
    }
    set_tiles();
    tables_.resize(L_);
    for (int l = 0; l < L_; ++l) {
      VD_CHECK(pool_.alloc(&tables_[l].views, (size_t)n_));
      for (int k = 0; k < 4; ++k) VD_CHECK(pool_.alloc(&tables_[l].starts[k], (size_t)n_ + 1));
    }
    gens_.assign(n_, -1);
    return VD_OK;
  }

  double gang_share() override {
    if (stale()) set_loops();
    double share = 0.0;
    for (int l = 0; l < L_; ++l) {
      const int kind = kinds_[l];
      for (const auto* h : h_)
        if (loops_[l]) share = std::max(share, (double)h->level_tiles(l, kind) / loop_cap_[kind]);
    }
    return share;
  }

  int launch(const vd_solve_opts* o, hipStream_t s) override {
    if (o && (o->init_delta || o->energy_target != 0.0)) return VD_EINVAL;  // single-lattice only
    for (auto* h : h_)
      if (!h->has_constraints()) return VD_ESTATE;
    const int reset = (o && o->reset_to_rest) ? 1 : 0;
    if (stale()) {
      set_tiles();
      VD_CHECK(build_tables());
      for (auto& g : exec_)
        if (g) {
          (void)hipGraphExecDestroy(g);
          g = nullptr;
        }
    }
    if (graph_) {
      if (!exec_[reset]) {
        if (!capture_) VD_TRY(hipStreamCreateWithFlags(&capture_, hipStreamNonBlocking));
        VD_TRY(hipStreamSynchronize(stream_));
        hipGraph_t g = nullptr;
        VD_TRY(hipStreamBeginCapture(capture_, hipStreamCaptureModeThreadLocal));
        const int rc = enqueue(reset, capture_);
        const hipError_t e = hipStreamEndCapture(capture_, &g);
        if (rc != VD_OK) {
          if (g) (void)hipGraphDestroy(g);
          return rc;
        }
        if (e != hipSuccess) return VD_EHIP;
        const hipError_t ei = hipGraphInstantiate(&exec_[reset], g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (ei != hipSuccess) return VD_EHIP;
      }
      VD_TRY(hipGraphLaunch(exec_[reset], s));
    } else {
      VD_CHECK(enqueue(reset, s));
    }
    for (auto* h : h_) h->mark_energy_fresh();
    return VD_OK;
  }

  int energies(double* e) override {
    for (int b = 0; b < n_; ++b) VD_CHECK(h_[b]->finest_energy_host(e + 4 * b));
    return VD_OK;
  }

 private:
  struct Tables {
    LevelView<T>* views = nullptr;
    int* starts[4] = {nullptr, nullptr, nullptr, nullptr};
    int blocks[4] = {0, 0, 0, 0};
    int masked = 0;  // some lattice restricts its solve to its set M
    LevelView<T> first{};
  };

  // Whether a handle was reallocated or re-tiled since the tables were built.
  bool stale() const {
    for (int b = 0; b < n_; ++b)
      if (gens_[b] != h_[b]->generation()) return true;
    return false;
  }

  // The batch's tiles on every handle: a launch has one tile kind, and a handle
  // may have got another since (vd_tune, another batch).
  void set_tiles() {
    for (int l = 0; l < L_; ++l)
      for (auto* h : h_) h->force_tile(l, kinds_[l]);
  }

  // A lattice of a one-launch solve waits until all its tiles are resident, and
  // tiles become resident in launch order: groups that fill the GPU (first fit,
  // largest first) leave the fewest compute units waiting for an earlier
  // lattice to end.  The groups of level l with tile kind `kind`; none where a
  // lattice does not fit or wants one launch per iteration.
  std::vector<std::vector<int>> groups_of(int l, int kind) const {
    std::vector<int> tiles(n_), by_size(n_);
    for (int b = 0; b < n_; ++b) {
      by_size[b] = b;
      tiles[b] = h_[b]->level_tiles(l, kind);
      if (!h_[b]->level_loop(l) || tiles[b] > loop_cap_[kind]) return {};
    }
    std::stable_sort(by_size.begin(), by_size.end(),
                     [&](int a, int b) { return tiles[a] > tiles[b]; });
    std::vector<std::vector<int>> groups;
    std::vector<int> left;
    for (const int b : by_size) {
      size_t g = 0;
      while (g < groups.size() && left[g] < tiles[b]) ++g;
      if (g == groups.size()) {
        groups.emplace_back();
        left.push_back(loop_cap_[kind]);
      }
      groups[g].push_back(b);
      left[g] -= tiles[b];
    }
    return groups;
  }

  // Nodes of level l, or with a tile kind the places of its tiles.
  int64_t nodes_of(int l, int kind = -1) const {
    int64_t n = 0;
    for (const auto* h : h_)
      n += kind < 0 ? h->level_nodes(l)
                    : (kind == 2 ? 1024 : 512) * (int64_t)h->level_tiles(l, kind);
    return n;
  }
  double loop_us(int l, int kind, int rounds) const {
    return batch_loop_us(kind, rounds, nodes_of(l), sizeof(T) == 8, masked_);
  }
  double iter_us(int l) const {
    return batch_iter_us(nodes_of(l), nodes_of(l, 1), sizeof(T) == 8, masked_);
  }

  // Whether the position solves of each level run as one launch: where all
  // lattices are resident together, or where the rounds that the GPU is filled
  // cost less than streaming every lattice in each iteration, by the tuner's
  // timings of the tile or else as expected.
  void set_loops() {
    loops_.assign(L_, 0);
    for (int l = 0; l < L_; ++l) {
      const int kind = kinds_[l], rounds = (int)groups_of(l, kind).size();
      if (rounds == 0) continue;
      loops_[l] = tuned_[l].kind == kind ? tuned_[l].loop
                                         : rounds == 1 || loop_us(l, kind, rounds) < iter_us(l);
    }
  }

  // The tile of level l unless the largest lattice's was chosen: the kind with
  // the fastest one-launch solves, or, where a launch per iteration is expected
  // to be faster, 8x8x8 (32x8x4 where it pads little: 12 lattices of 64^3 4.3
  // against 5.3 ms, of 48^3, a third more nodes, 1.31 against 1.23 for 8).
  int default_kind(int l) const {
    int best = -1;
    double best_us = 0.0;
    for (const int k : {7, 6, 5, 4, 3}) {
      const int rounds = (int)groups_of(l, k).size();
      if (rounds == 0) continue;
      const double us = loop_us(l, k, rounds);
      if (best < 0 || us < best_us) {
        best = k;
        best_us = us;
      }
      if (rounds == 1) return best;
    }
    if (best >= 0 && best_us < iter_us(l)) return best;
    return sizeof(T) == 4 && !masked_ && 20 * nodes_of(l, 2) <= 23 * nodes_of(l) ? 2 : 1;
  }

  // The lattices in launch order.
  std::vector<int> launch_order() const {
    std::vector<int> order;
    const int F = L_ - 1;
    if (loops_[F]) {
      for (const auto& g : groups_of(F, kinds_[F]))
        order.insert(order.end(), g.begin(), g.end());
    } else {
      for (int b = 0; b < n_; ++b) order.push_back(b);
    }
    return order;
  }

  // Device tables of the lattices' level views and the first workgroup of
  // each lattice for every workgroup kind (rebuilt when a handle reallocates).
  int build_tables() {
    set_loops();
    const std::vector<int> order = launch_order();
    for (int l = 0; l < L_; ++l) {
      std::vector<LevelView<T>> views(n_);
      std::vector<int> st[4];
      for (int k = 0; k < 4; ++k) st[k].assign(n_ + 1, 0);
      for (int b = 0; b < n_; ++b) {
        const LevelView<T> V = h_[order[b]]->level_view(l);
        views[b] = V;
        const int cnt[4] = {V.ntiles, node_blocks(V.N), energy_blocks(V.rblocks, V.N), 1};
        for (int k = 0; k < 4; ++k) st[k][b + 1] = st[k][b] + cnt[k];
      }
      Tables& t = tables_[l];
      t.first = views[0];
      t.masked = 0;
      for (const LevelView<T>& V : views) t.masked |= V.act != nullptr;
      VD_TRY(hipMemcpy(t.views, views.data(), sizeof(LevelView<T>) * n_, hipMemcpyHostToDevice));
      for (int k = 0; k < 4; ++k) {
        VD_TRY(hipMemcpy(t.starts[k], st[k].data(), sizeof(int) * (n_ + 1),
                         hipMemcpyHostToDevice));
        t.blocks[k] = st[k][n_];
      }
    }
    for (int b = 0; b < n_; ++b) gens_[b] = h_[b]->generation();
    return VD_OK;
  }

  Dispatch<T> D(int l, int kind) const {
    const Tables& t = tables_[l];
    Dispatch<T> d{};
    d.one = t.first;
    d.views = t.views;
    d.starts = t.starts[kind];
    d.n = n_;
    d.blocks = t.blocks[kind];
    d.masked = t.masked;
    return d;
  }

  int profile(double* us, int* n) override { return timer_.collect(us, n); }

  // Per level, every tile kind for all lattices of this part, in both forms of
  // the solve, timed over one batched position step (the gradient pass and
  // `iters` CG iterations) from the lattices' current state; the fastest kind
  // and form are kept and the lattices' displacements are restored.  The fastest of three timings after a
  // warm-up counts, as in the single-lattice tuner.
  int tune(int iters, hipStream_t s, int* tile_out, double* us_out) override {
    if (iters < 1) return VD_EINVAL;
    for (auto* h : h_)
      if (!h->has_constraints()) return VD_ESTATE;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    VD_TRY(hipEventCreate(&e0));
    VD_TRY(hipEventCreate(&e1));
    int rc = VD_OK;
    for (int l = 0; l < L_ && rc == VD_OK; ++l) {
      std::vector<T*> saved(n_, nullptr);
      std::vector<size_t> len(n_, 0);
      for (int b = 0; b < n_ && rc == VD_OK; ++b) {
        len[b] = 3 * (size_t)h_[b]->level_nodes(l);
        rc = pool_.alloc(&saved[b], len[b]);
        if (rc == VD_OK)
          rc = hipMemcpyAsync(saved[b], h_[b]->level_view(l).d, len[b] * sizeof(T),
                              hipMemcpyDeviceToDevice, s) == hipSuccess ? VD_OK : VD_EHIP;
      }
      auto restore = [&]() -> int {
        for (int b = 0; b < n_; ++b)
          VD_TRY(hipMemcpyAsync(h_[b]->level_view(l).d, saved[b], len[b] * sizeof(T),
                                hipMemcpyDeviceToDevice, s));
        return VD_OK;
      };
      double best = 1e300;
      int best_kind = kinds_[l];
      bool best_loop = false;
      int timed = -1;  // the kind that us_out was last written for
      for (int t = 0; t < 2 * kTileKinds && rc == VD_OK; ++t) {
        const int kind = t / 2;
        const bool loop = (t & 1) != 0;
        // (not a form expected to take half as long again as the other)
        const int rounds = (int)groups_of(l, kind).size();
        const double as_loop = rounds > 1 ? loop_us(l, kind, rounds) : 0.0;
        if (loop ? rounds == 0 || as_loop > 1.5 * iter_us(l)
                 : rounds > 0 && iter_us(l) > 1.5 * as_loop) continue;
        kinds_[l] = kind;
        set_tiles();
        tuned_[l].kind = kind;
        tuned_[l].loop = loop;
        rc = build_tables();
        float best_ms = 1e30f;
        for (int rep = 0; rep < 4 && rc == VD_OK; ++rep) {
          float ms = 0.0f;
          rc = restore();
          if (rc != VD_OK) break;
          VD_TRY(hipEventRecord(e0, s));
          VD_TRY(launch_stencil<T>(kModeRhs, D(l, kTiles), nullptr, nullptr, s));
          VD_CHECK(solve(l, iters, false, s));
          VD_TRY(hipEventRecord(e1, s));
          VD_TRY(hipEventSynchronize(e1));
          VD_TRY(hipEventElapsedTime(&ms, e0, e1));
          if (rep > 0) best_ms = std::min(best_ms, ms);
        }
        const double us = 1000.0 * best_ms / iters;
        if (us_out) {
          double& out = us_out[VD_TILE_KINDS * l + kind];
          out = timed == kind ? std::min(out, us) : us;
        }
        timed = kind;
        if (us < best) {
          best = us;
          best_kind = kind;
          best_loop = loop;
        }
      }
      kinds_[l] = best_kind;
      set_tiles();
      tuned_[l].kind = best_kind;
      tuned_[l].loop = best_loop;
      if (tile_out) tile_out[l] = best_kind + 1;
      if (rc == VD_OK) rc = restore();
      if (rc == VD_OK) rc = hipStreamSynchronize(s) == hipSuccess ? VD_OK : VD_EHIP;
      for (T* p : saved) pool_.release(p);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc == VD_OK) rc = build_tables();
    for (auto& g : exec_)  // schedules captured with the old tiles are stale
      if (g) {
        (void)hipGraphExecDestroy(g);
        g = nullptr;
      }
    for (auto* h : h_) h->mark_energy_stale();
    return rc;
  }

  // The CG solve of level l, as one launch or one per iteration.
  int solve(int l, int pcg, bool on, hipStream_t s) {
    if (pcg > 0 && loops_[l])
      return timer_.timed(on, VD_PROF_CG_LOOP, s, [&] {
        return launch_cg_loop<T>(pcg, D(l, kTiles), s, nullptr, assemble_ticks(pcg));
      });
    for (int m = 0; m < pcg; ++m)
      VD_CHECK(timer_.timed(on, VD_PROF_CG_A, s,
                            [&] { return launch_cg<T>(m, D(l, kTiles), s); }));
    if (pcg > 0)
      VD_CHECK(timer_.timed(on, VD_PROF_CG_B, s,
                            [&] { return launch_cg_final<T>(pcg - 1, D(l, kNodes), s); }));
    return VD_OK;
  }

  // The frame schedule of Solver::enqueue_frame with every launch batched.
  int enqueue(int reset, hipStream_t s) {
    const int F = L_ - 1;
    const vd_lattice_desc& dsc = h_[0]->desc();
    timer_.reset();
    if (reset) VD_TRY(launch_set_rest<T>(D(F, kNodes), s));
    for (int l = 0; l < L_; ++l) VD_TRY(launch_reset_counters<T>(D(l, kOne), s));
    for (int l = 0; l < L_; ++l) {
      const bool on = prof_ && l == F;
      if (l < F) VD_TRY(launch_inject<T>(D(l, kNodes), D(F, kNodes), 1 << (F - l), s));
      if (l > 0) {
        VD_CHECK(timer_.timed(on, VD_PROF_TRANSFER, s, [&] {
          return launch_prolong<T>(D(l, kNodes), D(l - 1, kNodes), 1, s);
        }));
        VD_CHECK(timer_.timed(on, VD_PROF_ROTATION, s,
                              [&] { return launch_polar<T>(D(l, kNodes), s); }));
      }
      const int gn = dsc.gn_iters[l], pcg = dsc.pcg_iters[l];
      for (int k = 0; k < gn; ++k) {
        VD_CHECK(timer_.timed(on, VD_PROF_GRADIENT, s, [&] {
          return launch_stencil<T>(kModeRhs, D(l, kTiles), nullptr, nullptr, s);
        }));
        VD_CHECK(solve(l, pcg, on, s));
        VD_CHECK(timer_.timed(on, VD_PROF_ROTATION, s,
                              [&] { return launch_polar<T>(D(l, kNodes), s); }));
      }
    }
    VD_CHECK(timer_.timed(prof_, VD_PROF_ENERGY, s, [&] {
      return launch_energy<T>(D(F, kEnergy), D(F, kOne), 0, s);
    }));
    return VD_OK;
  }

  std::vector<Solver<T>*> h_;
  int n_ = 0, L_ = 0;
  hipStream_t stream_ = nullptr;
  hipStream_t capture_ = nullptr;
  bool graph_ = false;
  hipGraphExec_t exec_[2] = {nullptr, nullptr};
  bool prof_ = false;
  int kinds_[VD_MAX_LEVELS] = {};  // the tile kind of each level
  bool masked_ = false;            // some lattice has an optimised set
  int loop_cap_[kTileKinds] = {};  // most tiles of a lattice's one-launch CG solve
  std::vector<char> loops_;        // per level: its CG solves are one launch
  struct Tuned {
    int kind = -1;
    bool loop = false;
  } tuned_[VD_MAX_LEVELS];         // the tuner's choice per level
  EventTimer timer_;
  std::vector<Tables> tables_;
  std::vector<long> gens_;
  Pool pool_;
};

}  // namespace vd

// ===========================================================================
// C ABI
// ===========================================================================

struct vd_lattice {
  vd::ISolver* impl;
};

// A batch holds up to two single-precision batches: the float32 lattices
// (part 0) and the float64 ones (part 1), each with the caller's positions of
// its lattices.  Part 1 runs on a library-owned stream, forked from and
// joined back into the lattices' stream, so both overlap on the GPU, or after
// part 0 where solves of both could wait for one another.
struct vd_batch {
  vd::IBatch* part[2] = {nullptr, nullptr};
  std::vector<int> index[2];
  hipStream_t stream = nullptr;  // the lattices' stream
  hipStream_t side = nullptr;    // part 1 when both parts exist
  hipEvent_t fork = nullptr, join = nullptr;
  ~vd_batch() {
    delete part[0];
    delete part[1];
    if (fork) (void)hipEventDestroy(fork);
    if (join) (void)hipEventDestroy(join);
    if (side) (void)hipStreamDestroy(side);
  }
};

namespace {

template <typename S>
int make_part(const std::vector<S*>& hs, vd::IBatch** out) {
  using T = std::remove_pointer_t<decltype(hs[0]->level_view(0).d)>;
  auto* bt = new (std::nothrow) vd::Batch<T>(hs);
  if (!bt) return VD_ENOMEM;
  const int rc = bt->init();
  if (rc != VD_OK) {
    delete bt;
    return rc;
  }
  *out = bt;
  return VD_OK;
}

int make_batch(vd_lattice* const* ls, int n, vd_batch** out) {
  std::vector<vd::Solver<float>*> h32;
  std::vector<vd::Solver<double>*> h64;
  vd_batch* h = new (std::nothrow) vd_batch;
  if (!h) return VD_ENOMEM;
  const vd_lattice_desc* d0 = nullptr;
  void* s0 = nullptr;
  for (int b = 0; b < n; ++b) {
    const vd_lattice_desc* d;
    void* st;
    if (auto* p = dynamic_cast<vd::Solver<float>*>(ls[b]->impl)) {
      h32.push_back(p);
      h->index[0].push_back(b);
      d = &p->desc();
      st = (void*)p->stream();
    } else if (auto* q = dynamic_cast<vd::Solver<double>*>(ls[b]->impl)) {
      h64.push_back(q);
      h->index[1].push_back(b);
      d = &q->desc();
      st = (void*)q->stream();
    } else {
      delete h;
      return VD_EINVAL;
    }
    if (!d0) {
      d0 = d;
      s0 = st;
    }
    bool same = d->num_levels == d0->num_levels && st == s0 &&
                ((d->flags ^ d0->flags) & VD_FLAG_GRAPH) == 0;
    for (int l = 0; l < d0->num_levels && same; ++l)
      same = d->gn_iters[l] == d0->gn_iters[l] && d->pcg_iters[l] == d0->pcg_iters[l];
    if (!same) {
      delete h;
      return VD_EINVAL;
    }
  }
  h->stream = (hipStream_t)s0;
  int rc = VD_OK;
  if (!h32.empty()) rc = make_part(h32, &h->part[0]);
  if (rc == VD_OK && !h64.empty()) rc = make_part(h64, &h->part[1]);
  if (rc == VD_OK && h->part[0] && h->part[1]) {
    if (hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&h->fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&h->join, hipEventDisableTiming) != hipSuccess)
      rc = VD_EHIP;
  }
  if (rc != VD_OK) {
    delete h;
    return rc;
  }
  *out = h;
  return VD_OK;
}

}  // namespace

extern "C" {

int vd_lattice_create(const vd_lattice_desc* d, void* stream, vd_lattice** out) {
  if (!d || !out) return VD_EINVAL;
  *out = nullptr;
  if (d->num_levels < 1 || d->num_levels > VD_MAX_LEVELS) return VD_EINVAL;
  if (!(d->spacing > 0) || !std::isfinite(d->spacing)) return VD_EINVAL;
  for (int k = 0; k < 3; ++k) {
    if (d->dims[k] < 2 || !std::isfinite(d->origin[k])) return VD_EINVAL;
  }
  if (!(d->w_dense >= 0) || !(d->w_sparse >= 0) || !(d->w_arap >= 0) ||
      !std::isfinite(d->w_dense) || !std::isfinite(d->w_sparse) || !std::isfinite(d->w_arap))
    return VD_EINVAL;
  for (int l = 0; l < d->num_levels; ++l)
    if (d->gn_iters[l] < 0 || d->pcg_iters[l] < 0) return VD_EINVAL;
  {
    int dims[3] = {d->dims[0], d->dims[1], d->dims[2]};
    for (int l = 1; l < d->num_levels; ++l)
      for (int k = 0; k < 3; ++k) dims[k] = (dims[k] + 1) / 2;
    for (int k = 0; k < 3; ++k)
      if (dims[k] < 2) return VD_EINVAL;
  }
  if (d->precision != VD_FP32_FP64RED && d->precision != VD_FP64) return VD_EINVAL;
  for (int l = 0; l < VD_MAX_LEVELS; ++l)
    if (d->tile[l] < 0 || d->tile[l] > vd::kTileKinds) return VD_EINVAL;
  vd::ISolver* impl = nullptr;
  if (d->precision == VD_FP64)
    impl = new (std::nothrow) vd::Solver<double>(*d, (hipStream_t)stream);
  else
    impl = new (std::nothrow) vd::Solver<float>(*d, (hipStream_t)stream);
  if (!impl) return VD_ENOMEM;
  const int rc = impl->init();
  if (rc != VD_OK) {
    delete impl;
    return rc;
  }
  vd_lattice* h = new (std::nothrow) vd_lattice;
  if (!h) {
    delete impl;
    return VD_ENOMEM;
  }
  h->impl = impl;
  *out = h;
  return VD_OK;
}

int vd_lattice_destroy(vd_lattice* l) {
  if (!l) return VD_OK;
  delete l->impl;
  delete l;
  return VD_OK;
}


int vd_batch_create(vd_lattice* const* ls, int32_t n, vd_batch** out) {
  if (!ls || !out || n < 1) return VD_EINVAL;
  *out = nullptr;
  for (int b = 0; b < n; ++b)
    if (!ls[b] || !ls[b]->impl) return VD_EINVAL;
  return make_batch(ls, n, out);
}

int vd_batch_solve(vd_batch* b, const vd_solve_opts* o, double* energies) {
  if (!b) return VD_EINVAL;
  if (o && (o->init_delta || o->energy_target != 0.0)) return VD_EINVAL;
  // Two solves that hold whole compute units and wait for their tiles would wait
  // for one another where together they can hold the GPU without either being
  // complete: 4 lattices of 64^3 beside 4 of 32^3 in float64 4.6 ms, one part
  // after the other 2.9.  Where that cannot be, the parts fill each other's
  // waits: 8 of 24^3 beside 8 in float64 1.3 and 1.9.
  const double a = b->part[0] && b->part[1] ? b->part[0]->gang_share() : 0.0;
  const double c = a > 0.0 ? b->part[1]->gang_share() : 0.0;
  if (c > 0.0 && a + c > 1.0) {
    for (int k = 0; k < 2; ++k) {
      const int rc = b->part[k]->launch(o, b->stream);
      if (rc != VD_OK) return rc;
    }
  } else if (b->part[0] && b->part[1]) {
    if (hipEventRecord(b->fork, b->stream) != hipSuccess ||
        hipStreamWaitEvent(b->side, b->fork, 0) != hipSuccess)
      return VD_EHIP;
    int rc = b->part[1]->launch(o, b->side);
    if (rc != VD_OK) return rc;
    rc = b->part[0]->launch(o, b->stream);
    if (rc != VD_OK) return rc;
    if (hipEventRecord(b->join, b->side) != hipSuccess ||
        hipStreamWaitEvent(b->stream, b->join, 0) != hipSuccess)
      return VD_EHIP;
  } else {
    const int rc = (b->part[0] ? b->part[0] : b->part[1])->launch(o, b->stream);
    if (rc != VD_OK) return rc;
  }
  if (!energies) return VD_OK;
  if (hipStreamSynchronize(b->stream) != hipSuccess) return VD_EHIP;
  std::vector<double> e;
  for (int k = 0; k < 2; ++k) {
    if (!b->part[k]) continue;
    e.assign(4 * b->index[k].size(), 0.0);
    const int rc = b->part[k]->energies(e.data());
    if (rc != VD_OK) return rc;
    for (size_t j = 0; j < b->index[k].size(); ++j)
      for (int q = 0; q < 4; ++q) energies[4 * b->index[k][j] + q] = e[4 * j + q];
  }
  return VD_OK;
}

int vd_batch_tune(vd_batch* b, int32_t iters, int32_t* tile_out, double* us_out) {
  if (!b || iters < 1) return VD_EINVAL;
  if (tile_out)
    for (int k = 0; k < 2 * VD_MAX_LEVELS; ++k) tile_out[k] = 0;
  for (int k = 0; k < 2; ++k) {
    if (!b->part[k]) continue;
    const int rc = b->part[k]->tune(iters, b->stream, tile_out ? tile_out + k * VD_MAX_LEVELS : nullptr,
                                    us_out ? us_out + k * VD_MAX_LEVELS * VD_TILE_KINDS : nullptr);
    if (rc != VD_OK) return rc;
  }
  return VD_OK;
}

int vd_batch_profile(vd_batch* b, double* prof_us, int32_t* prof_n) {
  if (!b || !prof_us || !prof_n) return VD_EINVAL;
  return (b->part[0] ? b->part[0] : b->part[1])->profile(prof_us, prof_n);
}

int vd_batch_destroy(vd_batch* b) {
  if (!b) return VD_OK;
  delete b;
  return VD_OK;
}

int vd_set_constraints(vd_lattice* l, const vd_constraints* c) {
  if (!l) return VD_EINVAL;
  return l->impl->set_constraints(c);
}

int vd_solve_frame(vd_lattice* l, const vd_solve_opts* o, vd_solve_report* r) {
  if (!l) return VD_EINVAL;
  return l->impl->solve_frame(o, r);
}

int vd_get_state64(vd_lattice* l, double* pos, double* rot, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->get_state64(pos, rot, mem);
}

int vd_get_energy(vd_lattice* l, double out[4]) {
  if (!l) return VD_EINVAL;
  return l->impl->get_energy(out);
}

int vd_get_state(vd_lattice* l, float* pos, float* rot, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->get_state(pos, rot, mem);
}

int vd_set_state(vd_lattice* l, const float* pos, const float* rot, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->set_state(pos, rot, mem);
}

int vd_level_info(const vd_lattice* l, int32_t level, int32_t dims[3], double* spacing) {
  if (!l) return VD_EINVAL;
  return l->impl->level_info(level, dims, spacing);
}

const char* vd_strerror(int code) {
  switch (code) {
    case VD_OK: return "ok";
    case VD_EINVAL: return "invalid argument or non-finite / negative input";
    case VD_ERANGE: return "a canonical sample lies outside the coarsest lattice";
    case VD_ENOMEM: return "device allocation failed";
    case VD_EHIP: return "HIP runtime error";
    case VD_ESTATE: return "call not valid in the current state (no constraints set?)";
    default: return "unknown status code";
  }
}

int vd_tune(vd_lattice* l, int32_t iters, int32_t* tile_out, double* us_out) {
  if (!l) return VD_EINVAL;
  return l->impl->tune(iters, tile_out, us_out);
}

int vd_get_profile(vd_lattice* l, double* prof_us, int32_t* prof_n) {
  if (!l || !prof_us || !prof_n) return VD_EINVAL;
  return l->impl->profile(prof_us, prof_n);
}

int vd_warm_features(vd_lattice* l, const float* prev2, uint16_t* x, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->warm_features(prev2, x, mem);
}

int vd_debug_apply(vd_lattice* l, int32_t level, const float* p, float* Ap, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_apply(level, p, Ap, mem);
}

int vd_debug_gradient(vd_lattice* l, int32_t level, const float* pos, const float* rot, float* g,
                      int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_gradient(level, pos, rot, g, mem);
}

int vd_debug_energy(vd_lattice* l, int32_t level, const float* pos, const float* rot,
                    double out[4], int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_energy(level, pos, rot, out, mem);
}

int vd_debug_diag(vd_lattice* l, int32_t level, float* diag, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_diag(level, diag, mem);
}

int vd_debug_rotations(vd_lattice* l, int32_t level, const float* pos, const float* rot_prev,
                       float* rot_out, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_rotations(level, pos, rot_prev, rot_out, mem);
}

int vd_debug_default_tile(const int32_t dims[3], int32_t precision, uint32_t flags) {
  if (!dims || dims[0] < 2 || dims[1] < 2 || dims[2] < 2) return VD_EINVAL;
  return 1 + vd::default_tile(dims[0], dims[1], dims[2], precision == VD_FP64,
                              (flags & VD_FLAG_ACTIVE_SET) != 0, (flags & VD_FLAG_ITERATIVE) != 0);
}

int vd_debug_abandon_loops(vd_lattice* l, int32_t on) {
  if (!l) return VD_EINVAL;
  return l->impl->abandon_loops(on);
}

int vd_debug_prolong(vd_lattice* l, int32_t level, const float* coarse, float* out, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_prolong(level, coarse, out, mem);
}

namespace {

// Device copies of a debug entry's host arguments (freed on scope exit).
struct DebugBuffers {
  std::vector<void*> bufs;
  ~DebugBuffers() {
    for (void* b : bufs) (void)hipFree(b);
  }
  void* get(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes > 0 ? bytes : 1) != hipSuccess) return nullptr;
    bufs.push_back(p);
    return p;
  }
};

}  // namespace

int vd_debug_sort_pairs(const uint32_t* keys, const int32_t* vals, uint32_t* keys_out,
                        int32_t* vals_out, int64_t n, int32_t end_bit, int32_t mem,
                        void* stream) {
  if (n < 0 || n > INT32_MAX || end_bit < 0 || end_bit > 32) return VD_EINVAL;
  if (n > 0 && (!keys || !vals || !keys_out || !vals_out)) return VD_EINVAL;
  if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
  if (n == 0) return VD_OK;
  hipStream_t s = (hipStream_t)stream;
  DebugBuffers db;
  const size_t bytes = 4 * (size_t)n;
  const size_t tb = vd::sort_temp_bytes((int)n);
  void* temp = db.get(tb);
  if (!temp) return VD_ENOMEM;
  const unsigned* kin = keys;
  const int* vin = vals;
  unsigned* kout = keys_out;
  int* vout = vals_out;
  if (mem == VD_MEM_HOST) {
    void *a = db.get(bytes), *b = db.get(bytes), *c = db.get(bytes), *d = db.get(bytes);
    if (!a || !b || !c || !d) return VD_ENOMEM;
    if (hipMemcpyAsync(a, keys, bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(b, vals, bytes, hipMemcpyHostToDevice, s) != hipSuccess)
      return VD_EHIP;
    kin = (const unsigned*)a;
    vin = (const int*)b;
    kout = (unsigned*)c;
    vout = (int*)d;
  }
  hipError_t e = vd::sort_pairs(temp, tb, kin, kout, vin, vout, (int)n, end_bit, s);
  if (e == hipSuccess && mem == VD_MEM_HOST) {
    e = hipMemcpyAsync(keys_out, kout, bytes, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(vals_out, vout, bytes, hipMemcpyDeviceToHost, s);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? VD_OK : VD_EHIP;
}

int vd_debug_exclusive_scan(const int32_t* in, int32_t* out, int64_t n, int32_t mem,
                            void* stream) {
  if (n < 0 || n > INT32_MAX || (n > 0 && (!in || !out))) return VD_EINVAL;
  if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
  if (n == 0) return VD_OK;
  hipStream_t s = (hipStream_t)stream;
  DebugBuffers db;
  const size_t bytes = 4 * (size_t)n;
  const size_t tb = vd::scan_temp_bytes((int)n);
  void* temp = db.get(tb);
  if (!temp) return VD_ENOMEM;
  const int* din = in;
  int* dout = out;
  if (mem == VD_MEM_HOST) {
    void *a = db.get(bytes), *b = db.get(bytes);
    if (!a || !b) return VD_ENOMEM;
    if (hipMemcpyAsync(a, in, bytes, hipMemcpyHostToDevice, s) != hipSuccess) return VD_EHIP;
    din = (const int*)a;
    dout = (int*)b;
  }
  hipError_t e = vd::exclusive_scan(temp, tb, din, dout, (int)n, s);
  if (e == hipSuccess && mem == VD_MEM_HOST)
    e = hipMemcpyAsync(out, dout, bytes, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? VD_OK : VD_EHIP;
}

int vd_debug_fit_rotations(const float* M, const float* R_prev, float* R, int32_t* keep,
                           int64_t n, int32_t precision, int32_t mem, void* stream) {
  if (n < 0 || (n > 0 && (!M || !R))) return VD_EINVAL;
  if (precision != VD_FP32_FP64RED && precision != VD_FP64) return VD_EINVAL;
  if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
  if (n == 0) return VD_OK;
  hipStream_t s = (hipStream_t)stream;
  float *dM = (float*)M, *dRp = (float*)R_prev, *dR = R;
  int* dk = keep;
  void* bufs[4] = {nullptr, nullptr, nullptr, nullptr};
  auto cleanup = [&]() {
    for (void* b : bufs)
      if (b) (void)hipFree(b);
  };
  if (mem == VD_MEM_HOST) {
    if (hipMalloc(&bufs[0], 36 * n) != hipSuccess || hipMalloc(&bufs[1], 36 * n) != hipSuccess ||
        hipMalloc(&bufs[2], 36 * n) != hipSuccess || hipMalloc(&bufs[3], 4 * n) != hipSuccess) {
      cleanup();
      return VD_ENOMEM;
    }
    dM = (float*)bufs[0];
    dRp = R_prev ? (float*)bufs[1] : nullptr;
    dR = (float*)bufs[2];
    dk = keep ? (int*)bufs[3] : nullptr;
    if (hipMemcpyAsync(dM, M, 36 * n, hipMemcpyHostToDevice, s) != hipSuccess ||
        (R_prev && hipMemcpyAsync(dRp, R_prev, 36 * n, hipMemcpyHostToDevice, s) != hipSuccess)) {
      cleanup();
      return VD_EHIP;
    }
  }
  hipError_t e = precision == VD_FP64 ? vd::launch_fit_batch<double>(dM, dRp, dR, dk, n, s)
                                      : vd::launch_fit_batch<float>(dM, dRp, dR, dk, n, s);
  if (e == hipSuccess && mem == VD_MEM_HOST) {
    e = hipMemcpyAsync(R, dR, 36 * n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && keep) e = hipMemcpyAsync(keep, dk, 4 * n, hipMemcpyDeviceToHost, s);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  cleanup();
  return e == hipSuccess ? VD_OK : VD_EHIP;
}

}  // extern "C"

// ---- tracking (vd_track.h) -------------------------------------------------

namespace {

int camera_check(const vd_camera* c, const vd_assoc_params* a, vd::CamAssoc* out) {
  return vd::camera_of(c, a, out);
}

// Device buffers of a synchronous stateless call, freed on scope exit.
struct Scratch {
  std::vector<void*> bufs;
  ~Scratch() {
    for (void* b : bufs) (void)hipFree(b);
  }
  template <typename P>
  P* get(size_t count) {
    void* q = nullptr;
    if (hipMalloc(&q, (count ? count : 1) * sizeof(P)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    bufs.push_back(q);
    return static_cast<P*>(q);
  }
};

}  // namespace

extern "C" {

int vd_associate(const vd_camera* cam, const float* depth, const float* points,
                 const float* normals, int64_t n, const vd_assoc_params* prm, float* target,
                 float* normal_out, float* weight, int32_t* pixel, int32_t mem, void* stream) {
  vd::CamAssoc c;
  const int rc = camera_check(cam, prm, &c);
  if (rc != VD_OK) return rc;
  if (n < 0 || n > (1ll << 30) || !depth) return VD_EINVAL;
  if (n > 0 && (!points || !normals || !target || !normal_out || !weight)) return VD_EINVAL;
  if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
  if (n == 0) return VD_OK;
  hipStream_t s = (hipStream_t)stream;
  const size_t npix = (size_t)c.W * c.H;
  const float *dd = depth, *dp = points, *dn = normals;
  float *dt = target, *dno = normal_out, *dw = weight;
  int* dpx = pixel;
  Scratch sc;
  if (mem == VD_MEM_HOST) {
    float* b = sc.get<float>(npix + 13 * (size_t)n);
    int* bp = pixel ? sc.get<int>((size_t)n) : nullptr;
    if (!b || (pixel && !bp)) return VD_ENOMEM;
    float* q = b;
    if (hipMemcpyAsync(q, depth, 4 * npix, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(q + npix, points, 12 * n, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(q + npix + 3 * n, normals, 12 * n, hipMemcpyHostToDevice, s) != hipSuccess)
      return VD_EHIP;
    dd = q;
    dp = q + npix;
    dn = q + npix + 3 * n;
    dt = q + npix + 6 * n;
    dno = q + npix + 9 * n;
    dw = q + npix + 12 * n;
    dpx = bp;
  }
  if (vd::launch_associate(c, dd, dp, dn, (int)n, dt, dno, dw, dpx, s) != hipSuccess)
    return VD_EHIP;
  if (mem == VD_MEM_HOST) {
    if (hipMemcpyAsync(target, dt, 12 * n, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(normal_out, dno, 12 * n, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(weight, dw, 4 * n, hipMemcpyDeviceToHost, s) != hipSuccess ||
        (pixel && hipMemcpyAsync(pixel, dpx, 4 * n, hipMemcpyDeviceToHost, s) != hipSuccess))
      return VD_EHIP;
  }
  return hipStreamSynchronize(s) == hipSuccess ? VD_OK : VD_EHIP;
}

int vd_rigid_pose(const vd_camera* cam, const float* depth, const float* points,
                  const float* normals, int64_t n, const vd_assoc_params* prm, int32_t iters,
                  double* pose, double* hist, int32_t mem, void* stream) {
  vd::CamAssoc c;
  const int rc = camera_check(cam, prm, &c);
  if (rc != VD_OK) return rc;
  if (n < 0 || n > (1ll << 30) || iters < 0 || !depth || !pose) return VD_EINVAL;
  if (n > 0 && (!points || !normals)) return VD_EINVAL;
  if (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE) return VD_EINVAL;
  if (mem == VD_MEM_HOST)
    for (int k = 0; k < 12; ++k)
      if (!std::isfinite(pose[k])) return VD_EINVAL;
  if (iters == 0) return VD_OK;
  hipStream_t s = (hipStream_t)stream;
  const size_t npix = (size_t)c.W * c.H;
  const int G = vd::rigid_blocks(n);
  Scratch sc;
  double* part = sc.get<double>((size_t)vd::kRigidStride * G);
  if (!part) return VD_ENOMEM;
  const float *dd = depth, *dp = points, *dn = normals;
  double *dpose = pose, *dhist = hist;
  if (mem == VD_MEM_HOST) {
    float* b = sc.get<float>(npix + 6 * (size_t)n);
    double* pb = sc.get<double>(12 + 2 * (size_t)iters);
    if (!b || !pb) return VD_ENOMEM;
    if (hipMemcpyAsync(b, depth, 4 * npix, hipMemcpyHostToDevice, s) != hipSuccess ||
        (n > 0 && hipMemcpyAsync(b + npix, points, 12 * n, hipMemcpyHostToDevice, s) != hipSuccess) ||
        (n > 0 &&
         hipMemcpyAsync(b + npix + 3 * n, normals, 12 * n, hipMemcpyHostToDevice, s) != hipSuccess) ||
        hipMemcpyAsync(pb, pose, 12 * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
      return VD_EHIP;
    dd = b;
    dp = b + npix;
    dn = b + npix + 3 * n;
    dpose = pb;
    dhist = hist ? pb + 12 : nullptr;
  }
  for (int it = 0; it < iters; ++it) {
    if (vd::launch_rigid_reduce_points(c, dd, dp, dn, (int)n, dpose, part, G, s) != hipSuccess ||
        vd::launch_rigid_solve(part, G, dpose, dhist ? dhist + 2 * it : nullptr, s) != hipSuccess)
      return VD_EHIP;
  }
  if (mem == VD_MEM_HOST) {
    if (hipMemcpyAsync(pose, dpose, 12 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        (hist && hipMemcpyAsync(hist, dhist, 2 * iters * sizeof(double), hipMemcpyDeviceToHost,
                                s) != hipSuccess))
      return VD_EHIP;
  }
  return hipStreamSynchronize(s) == hipSuccess ? VD_OK : VD_EHIP;
}

int vd_set_depth_frame(vd_lattice* l, const vd_depth_frame* f) {
  if (!l) return VD_EINVAL;
  return l->impl->set_depth_frame(f);
}

int vd_get_pose(vd_lattice* l, double pose[12]) {
  if (!l) return VD_EINVAL;
  return l->impl->get_pose(pose);
}

int vd_set_pose(vd_lattice* l, const double pose[12]) {
  if (!l) return VD_EINVAL;
  return l->impl->set_pose(pose);
}

int vd_track_frame(vd_lattice* l, const vd_track_opts* o, vd_track_report* r) {
  if (!l) return VD_EINVAL;
  return l->impl->track_frame(o, r);
}

int vd_fuse_depth(vd_lattice* l, const vd_fuse_opts* o, int64_t* n_updated) {
  if (!l) return VD_EINVAL;
  return l->impl->fuse_depth(o, n_updated);
}

int vd_get_tsdf(vd_lattice* l, float* D, float* W, int32_t* frames, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->get_tsdf(D, W, frames, mem);
}

int vd_set_tsdf(vd_lattice* l, const float* D, const float* W, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->set_tsdf(D, W, mem);
}

int vd_extract_mesh(vd_lattice* l, int64_t capacity, float* canon, float* deformed,
                    int32_t* cells, int32_t* edges, int64_t* n_triangles, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->extract_mesh(capacity, canon, deformed, cells, edges, n_triangles, mem);
}

int vd_get_active(vd_lattice* l, int32_t level, uint8_t* mask, int64_t* count,
                  int32_t* growth_layers) {
  if (!l) return VD_EINVAL;
  return l->impl->get_active(level, mask, count, growth_layers);
}

int vd_debug_associate(vd_lattice* l, const float* disp, const float* rot, float* target,
                       float* normal_out, float* weight, int32_t* pixel, int32_t mem) {
  if (!l) return VD_EINVAL;
  return l->impl->debug_associate(disp, rot, target, normal_out, weight, pixel, mem);
}

}  // extern "C"
