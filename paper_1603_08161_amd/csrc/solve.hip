// The per-frame solve kernels (Sec. 7): gradient, fused CG iterations,
// rotation fits, energy and level transfers.  Every launch takes a Dispatch:
// one lattice by value, or a device table of lattices that are all at the
// same schedule step (the batched solve), with workgroup g belonging to the
// lattice b for which starts[b] <= g < starts[b + 1].
//
// Unknowns are displacements d = t - t_hat; node vectors are SoA [3][N] in
// x-fastest order (rotations [9][N]).

#include <algorithm>

#include "vd_device.h"
#include "vd_kernels.h"

namespace vd {

namespace {

inline int blocks_for(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

__device__ __forceinline__ bool in_box(int x, int y, int z, int nx, int ny, int nz) {
  return x >= 0 && x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
}

__device__ __forceinline__ size_t rot_at(int row, int col, size_t N, size_t i) {
  return (size_t)(row * 3 + col) * N + i;
}

// The lattice of workgroup g, its local workgroup index and count.
template <typename T>
struct Where {
  LevelView<T> L;
  int b, local, count;
};

// The lattice is the number of b in 1..n-1 with starts[b] <= g (starts is
// non-decreasing): one wave-wide vector load and ballot per 64 lattices
// instead of a binary search's chain of dependent loads.
template <typename T>
__device__ __forceinline__ Where<T> locate(const Dispatch<T>& D, int g) {
  Where<T> w;
  if (D.n == 1) {
    w.L = D.one;
    w.b = 0;
    w.local = g;
    w.count = D.blocks;
    return w;
  }
  const int lane = threadIdx.x & (kWave - 1);
  int lo = 0;
  for (int base = 1; base < D.n; base += kWave) {
    const int idx = base + lane;
    lo += __popcll(__ballot(idx < D.n && glob<const int>(D.starts)[idx] <= g));
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  w.L = D.views[lo];
  w.b = lo;
  w.local = g - D.starts[lo];
  w.count = D.starts[lo + 1] - D.starts[lo];
  return w;
}

// A guarded launch (energy-target mode) returns at entry once the target
// was reached: the flag is uniform, so every workgroup leaves before any
// barrier or store.
template <typename T>
__device__ __forceinline__ bool skipped(const Dispatch<T>& D) {
  return D.stop != nullptr && *D.stop != 0;
}

template <typename T>
__device__ __forceinline__ LevelView<T> view_of(const Dispatch<T>& D, int b) {
  return D.n == 1 ? D.one : D.views[b];
}

template <typename T>
__device__ __forceinline__ int energy_blocks_dev(const LevelView<T>& L) {
  return L.rblocks + (L.N + kBlock - 1) / kBlock;
}

// Block sums of K values written to out[k * stride + local]: wave sums, then
// thread k adds the waves' k-th sums in wave order and stores the result.
template <int K, int NT = kBlock>
__device__ __forceinline__ void write_partials(double (&v)[K], double* out, int stride,
                                               int local) {
  constexpr int NW = NT / kWave;
  __shared__ double lds[K * NW];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) lds[k * NW + wid] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < K) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += lds[threadIdx.x * NW + w];
    glob(out)[(size_t)threadIdx.x * stride + local] = s;
  }
}

}  // namespace

// ===========================================================================
// tiles
// ===========================================================================

int tile_blocks(int kind, int nx, int ny, int nz) {
  auto nb = [&](int tx, int ty, int tz) {
    return ((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) * ((nz + tz - 1) / tz);
  };
  switch (kind) {
    case 1: return nb(TileM::TX, TileM::TY, TileM::TZ);
    case 2: return nb(TileW::TX, TileW::TY, TileW::TZ);
    case 3: return nb(TileX::TX, TileX::TY, TileX::TZ);
    case 4: return nb(TileZ::TX, TileZ::TY, TileZ::TZ);
    case 5: return nb(TileY::TX, TileY::TY, TileY::TZ);
    case 6: return nb(TileH::TX, TileH::TY, TileH::TZ);
    case 7: return nb(TileC::TX, TileC::TY, TileC::TZ);
    case 8: return nb(TileL4::TX, TileL4::TY, TileL4::TZ);
    case 9: return nb(TileL6::TX, TileL6::TY, TileL6::TZ);
    case 10: return nb(TileL7::TX, TileL7::TY, TileL7::TZ);
    default: return nb(TileS::TX, TileS::TY, TileS::TZ);
  }
}

// The tile of a level unless the caller or the tuner chooses one: the kind with
// the most workgroups whose tiles fit a one-launch CG solve, as smaller tiles
// spread the data rows over more compute units (us per iteration with the
// gradient pass: 32^3 in 128 tiles of 8x8x4 4.7, in 64 of 16x4x8 4.9, in 32 of
// 32x8x4 8.7; 48^3 in 216 of 16x4x8 6.7, in 108 of 32x8x4 8.1); among the
// 1024-node kinds the one that pads least.  Larger levels run one launch per
// iteration: in float32 fastest with 128-byte rows (2 x 20 iterations at 110^3:
// 3.04 ms with 32x8x4 on 256 threads, 3.23 with 8x8x8), in float64 and with
// the optimised set, whose tiles without unknowns are skipped, with 8x8x8
// (110^3: float64 7.18 against 9.29, optimised set 1.23 against 1.69, both 1.66
// against 3.51).  So do, in float64, levels of the 1024-node kinds where one
// launch per iteration is asked for (64^3: 1.68 against 1.74 ms with 32x8x4 on
// 1024 threads; in float32 1.07 against 1.02).
int default_tile(int nx, int ny, int nz, bool f64, bool masked, bool iterative) {
  const int order[] = {7, 6, 3, 5, 4};
  int best = -1;
  for (const int k : order) {
    const int n = tile_blocks(k, nx, ny, nz);
    if (n > kGangMaxTiles) continue;
    if (k == 7 || k == 6) return k;
    if (f64 && iterative) break;
    if (best < 0 || n < tile_blocks(best, nx, ny, nz)) best = k;
  }
  return best >= 0 ? best : nx >= 24 && !f64 && !masked ? 2 : 1;
}

// The tile of a one-launch CG solve on a level that is too large for every
// kind of default_tile (float32; float64 state does not fit): the smallest
// that covers it with kGangMaxTiles tiles, or -1.  One launch against one per
// iteration, frames of 3 levels with 8 x 20 iterations: 72^3 (16x16x8) 4.6
// and 5.6 ms, 84^3 (16x16x12) 5.9 and 7.6, 96^3 (16x16x14) 8.4 and 8.9; the
// optimised set at 72^3 4.4 and 5.7.  With the optimised set at 96^3 the
// largest tile spills 70 registers where the launches per iteration skip the
// tiles without unknowns: 7.4 and 6.8, so it is not used there.
int large_loop_tile(int nx, int ny, int nz, bool masked) {
  for (int k = 0; k < kTileKinds; ++k)
    if (tile_blocks(k, nx, ny, nz) <= kGangMaxTiles) return -1;
  for (int k = kTileKinds; k < kLoopKinds - (masked ? 1 : 0); ++k)
    if (tile_blocks(k, nx, ny, nz) <= kGangMaxTiles) return k;
  return -1;
}

// Costs by which a batch chooses its tiles and the form of its solves.  One
// launch over solves holds whole compute units: an iteration takes `rounds`
// times that of a full GPU, a quarter of which goes by how full the tiles and
// the rounds are.  A launch per iteration streams every node's vectors (and
// some of its tiles' empty places), in float32 more slowly once they exceed the
// last-level cache.  Fitted to batches of 2 .. 100 lattices of 8^3 .. 64^3
// nodes (ms of 2 x 15 iterations, one launch against one per iteration: 12 x
// 64^3 3.34 and 4.32, 16 x 48^3 2.12 and 2.52, 100 x 16^3 0.52 and 0.80, but 16
// x 33^3 1.41 and 1.12, 64 x 33^3 5.29 and 4.71 and, with the optimised set, 8
// x 48^3 0.94 and 0.72: lattices that leave much of their tiles, or of the GPU
// beside them, empty).
double batch_loop_us(int kind, int rounds, int64_t nodes, bool f64, bool masked) {
  const int size = kind == 0 || kind == 7 ? 0 : kind == 1 || kind == 6 ? 1 : kind == 2 ? 3 : 2;
  static const double us[2][2][4] = {{{5.8, 7.0, 9.2, 12.5}, {5.1, 6.0, 7.4, 9.2}},
                                     {{7.2, 11.4, 15.6, 20.0}, {6.2, 9.3, 11.8, 15.5}}};
  const double places = (double)rounds * kGangMaxTiles * (size == 0 ? 256 : size == 1 ? 512 : 1024);
  return rounds * us[f64][masked][size] * (0.75 + 0.25 * (double)nodes / places);
}
double batch_iter_us(int64_t nodes, int64_t places, bool f64, bool masked) {
  const double k = 1e-3 * (0.75 * (double)nodes + 0.25 * (double)places);
  if (masked) return 10.0 + k / (f64 ? 32.0 : 50.0);
  return f64 ? 8.0 + k / 13.0 : 8.0 + k / 27.0 + std::max(0.0, 1e-3 * (double)nodes - 1200.0) / 35.0;
}
int node_blocks(int N) { return blocks_for(N); }
int energy_blocks(int rblocks, int N) { return rblocks + blocks_for(N); }

template <typename TL>
struct TilePos {
  int x0, y0, z0;  // lattice coordinates of LDS index (0,0,0) (tile origin - 1)
  __device__ __forceinline__ TilePos(int nx, int ny, int local) {
    const int ntx = (nx + TL::TX - 1) / TL::TX, nty = (ny + TL::TY - 1) / TL::TY;
    const int tx = local % ntx, ty = (local / ntx) % nty, tz = local / (ntx * nty);
    x0 = tx * TL::TX - 1;
    y0 = ty * TL::TY - 1;
    z0 = tz * TL::TZ - 1;
  }
  // whether this thread owns nodes (tiles with more threads than nodes leave
  // the last threads without; they stage the halo and evaluate data blocks)
  __device__ __forceinline__ static bool owner() {
    return TL::OWNERS == TL::NT || (int)threadIdx.x < TL::OWNERS;
  }
  // LDS index of the k-th node owned by this thread
  __device__ __forceinline__ static int own(int k) {
    const int t = owner() ? (int)threadIdx.x : 0;
    const int lx = t % TL::TX + 1, ly = (t / TL::TX) % TL::TY + 1;
    const int lz = (t / (TL::TX * TL::TY)) * TL::NPT + k + 1;
    return lx + TL::HX * (ly + TL::HY * lz);
  }
};

// ===========================================================================
// the normal-equation stencil (Sec. 7.1): A p = J^T J p
// ===========================================================================
//
// A p at node i = 2 w_r sum_{j in N_i} (p_i - p_j)                (ARAP part)
//               + sum_{delta in {-1,0,1}^3} A27_i[delta] p_{i+delta}  (data part)
//
// One workgroup per tile; the tile plus a one-node halo of p is staged in LDS
// (all 27 stencil neighbours of a tile node are in it; nodes outside the
// lattice hold 0 and have zero blocks).

// ARAP part of A p at own node c (tile-local) / i (global) from the tile's p
// in LDS: 2 w_r times the 6-neighbour Laplacian.  The data part is added by
// the caller (eval_data_nodes).  With the optimised set M (sm: the tile's
// membership in LDS) only the edges inside M count: node c couples to the
// neighbours q in M.
template <typename T, typename TL>
__device__ __forceinline__ void arap_at(const LevelView<T>& L, const T (*sp)[TL::HALO], int c,
                                        int gx, int gy, int gz, T& o0, T& o1, T& o2,
                                        const unsigned char* sm = nullptr) {
  const T p0 = sp[0][c], p1 = sp[1][c], p2 = sp[2][c];
  T l0 = T(0), l1 = T(0), l2 = T(0);
  const int off[3] = {1, TL::HX, TL::HX * TL::HY};
  const int pos[3] = {gx, gy, gz};
  const int lim[3] = {L.nx, L.ny, L.nz};
  if (sm) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
      for (int sgn = -1; sgn <= 1; sgn += 2) {
        if (sgn < 0 ? pos[ax] == 0 : pos[ax] == lim[ax] - 1) continue;
        const int q = sgn < 0 ? c - off[ax] : c + off[ax];
        if (!sm[q]) continue;
        l0 += p0 - sp[0][q];
        l1 += p1 - sp[1][q];
        l2 += p2 - sp[2][q];
      }
    }
    const T w2 = T(2) * L.wr;
    o0 = w2 * l0;
    o1 = w2 * l1;
    o2 = w2 * l2;
    return;
  }
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    if (pos[ax] > 0) {
      const int q = c - off[ax];
      l0 += p0 - sp[0][q];
      l1 += p1 - sp[1][q];
      l2 += p2 - sp[2][q];
    }
    if (pos[ax] < lim[ax] - 1) {
      const int q = c + off[ax];
      l0 += p0 - sp[0][q];
      l1 += p1 - sp[1][q];
      l2 += p2 - sp[2][q];
    }
  }
  const T w2 = T(2) * L.wr;
  o0 = w2 * l0;
  o1 = w2 * l1;
  o2 = w2 * l2;
}

// ---------------------------------------------------------------------------
// data part of A p, shared by the workgroup (CG iteration and gradient pass)
// ---------------------------------------------------------------------------
//
// Only nodes near the observed surface carry data blocks, and they cluster in
// a few waves.  Evaluated by its owner, a node's 27 blocks are a long chain of
// row loads in one lane while most lanes idle, and the workgroup waits for its
// busiest wave.  Instead every wave lists its own such nodes in LDS (a segment
// per wave, in (k, lane) order) and, once the tile is staged, the workgroup's
// lanes take (node, part) items: per wave and round 21 nodes, lanes 3n, 3n+1
// and 3n+2 evaluating the blocks of dz = -1, 0, +1 of node n from that part of
// the node's row (14 16-byte loads; the row interleaves the three parts'
// chunks, so the three lanes of a node read one contiguous 48-byte span per
// load).  Lane 3n adds the three sums in fixed order and leaves the result in
// LDS for the owner.  A node's sum does not
// depend on which lane or round evaluates it, so the gradient pass and the CG
// iteration give the same bits with every tile shape.

constexpr int kPartsPerNode = 3;
constexpr int kNodesPerWave = kWave / kPartsPerNode;  // 21; lane 63 idles

template <typename T, typename TL>
struct DataShare {
  static constexpr int SEG = kWave * TL::NPT;  // list entries per wave
  static constexpr int NW = TL::NT / kWave;
  int slot[NW * SEG];
  int node[NW * SEG];  // LDS tile index of the node
  int cnt[NW];
  T d[3][NW * SEG];    // data part of A p of list entry e
};

// List the calling wave's own nodes that carry data blocks; rank[k]: entry of
// the thread's k-th node in the wave's segment (-1: none).
template <typename T, typename TL>
__device__ __forceinline__ void list_data_nodes(const int (&slot)[TL::NPT],
                                                DataShare<T, TL>& ds, int (&rank)[TL::NPT]) {
  using DS = DataShare<T, TL>;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const unsigned long long below = (1ull << lane) - 1ull;
  int base = 0;
#pragma unroll
  for (int k = 0; k < TL::NPT; ++k) {
    const unsigned long long m = __ballot(slot[k] >= 0);
    rank[k] = -1;
    if (slot[k] >= 0) {
      rank[k] = base + __popcll(m & below);
      const int e = wv * DS::SEG + rank[k];
      ds.slot[e] = slot[k];
      ds.node[e] = TilePos<TL>::own(k);
    }
    base += __popcll(m);
  }
  if (lane == 0) ds.cnt[wv] = base;
}

// Data part of A p for every listed node of the workgroup (after the barrier
// that publishes the lists and the tile's p); results in ds.d.
template <typename T, typename TL>
__device__ __forceinline__ void eval_data_nodes(const LevelView<T>& L,
                                                const T (*sp)[TL::HALO],
                                                DataShare<T, TL>& ds) {
  using DS = DataShare<T, TL>;
  constexpr int CW = 16 / (int)sizeof(T);  // entries per 16-byte chunk
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int part = lane % kPartsPerNode, nl = lane / kPartsPerNode;
  // first list position of every wave's segment (uniform: scalar registers)
  int pre[DS::NW + 1];
  pre[0] = 0;
#pragma unroll
  for (int w = 0; w < DS::NW; ++w) pre[w + 1] = pre[w] + __builtin_amdgcn_readfirstlane(ds.cnt[w]);
  const int total = pre[DS::NW];
  for (int r0 = 0; r0 < total; r0 += DS::NW * kNodesPerWave) {
    const int v = r0 + wv * kNodesPerWave + nl;
    T o0 = T(0), o1 = T(0), o2 = T(0);
    int e = -1;
    if (nl < kNodesPerWave && v < total) {
      // the segment holding list position v: the last one starting at or
      // before it (segments are in wave order)
      int u = 0, before = 0;
#pragma unroll
      for (int x = 1; x < DS::NW; ++x)
        if (v >= pre[x]) {
          u = x;
          before = pre[x];
        }
      e = u * DS::SEG + (v - before);
      const int cz = ds.node[e] + TL::HX * TL::HY * (part - 1);
      // entry x of the part: chunk 3 (x / CW) + part of the row
      const gptr<const T> __restrict__ A = glob<const T>(static_cast<const T*>(
          __builtin_assume_aligned(L.A27r + (size_t)ds.slot[e] * kA27Row + part * CW, 16)));
      auto entry = [&](int x) { return A[kPartsPerNode * CW * (x / CW) + x % CW]; };
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const int q = cz + (j % 3 - 1) + TL::HX * (j / 3 - 1);
        const T s0 = entry(6 * j), s1 = entry(6 * j + 1), s2 = entry(6 * j + 2),
                s3 = entry(6 * j + 3), s4 = entry(6 * j + 4), s5 = entry(6 * j + 5);
        const T q0 = sp[0][q], q1 = sp[1][q], q2 = sp[2][q];
        o0 += s0 * q0 + s1 * q1 + s2 * q2;
        o1 += s1 * q0 + s3 * q1 + s4 * q2;
        o2 += s2 * q0 + s4 * q1 + s5 * q2;
      }
    }
    const T a0 = __shfl_down(o0, 1, kWave), a1 = __shfl_down(o1, 1, kWave),
            a2 = __shfl_down(o2, 1, kWave);
    const T b0 = __shfl_down(o0, 2, kWave), b1 = __shfl_down(o1, 2, kWave),
            b2 = __shfl_down(o2, 2, kWave);
    if (part == 0 && e >= 0) {
      ds.d[0][e] = (o0 + a0) + b0;
      ds.d[1][e] = (o1 + a1) + b1;
      ds.d[2][e] = (o2 + a2) + b2;
    }
  }
}

// Exchange slots of a one-launch CG solve (k_cg_loop): [3 sets][4 sums][tiles]
// after the head of LevelView::gang.

__device__ __forceinline__ unsigned long long* gang_slots(const double* gang) {
  return (unsigned long long*)(gang + kGangHead);
}

// A slot that holds no sum yet.  A NaN sum is published as the canonical NaN,
// so no sum looks empty.
constexpr unsigned long long kEmptySlot = ~0ull;

// The gradient pass before a solve empties the slots (of a tile without
// unknowns: its sums, zero, for every iterate) and resets the head.  A solve
// on larger tiles has fewer: their first workgroups' slots are emptied, and
// the solve itself fills those of tiles without unknowns.
template <typename T>
__device__ __forceinline__ void gang_prepare(const LevelView<T>& L, int local, bool empty) {
  if (threadIdx.x < kGangSlots && local < L.loop_tiles) {
    const int set = threadIdx.x / 4, k = threadIdx.x % 4;
    gang_slots(L.gang)[((size_t)set * 4 + k) * L.loop_tiles + local] =
        empty && L.loop_tile == L.tile ? 0ull : kEmptySlot;
  }
  if (local == 0 && threadIdx.x < kGangHead) ((unsigned long long*)L.gang)[threadIdx.x] = 0ull;
}

// kModeRhs : p = d; g = A d - b + w_r sum_j (2I - R_i - R_j) e_ij is the
//            gradient J^T r; r = -g is stored (the CG residual r_0).
// kModeApply / kModeGrad : A p or g written to `out` (test entry points).
template <typename T, typename TL, int MODE, bool MASK>
__global__ __launch_bounds__(TL::NT) void k_stencil(Dispatch<T> D, const T* __restrict__ pin,
                                                    T* __restrict__ out) {
  if (skipped(D)) return;
  __shared__ T sp[3][TL::HALO];
  __shared__ unsigned char sm[TL::HALO];
  __shared__ DataShare<T, TL> ds;
  const Where<T> w = locate(D, xcd_remap(blockIdx.x, gridDim.x));
  const LevelView<T>& L = w.L;
  const TilePos<TL> t(L.nx, L.ny, w.local);
  const size_t N = L.N;
  const gptr<const T> __restrict__ src = glob<const T>((MODE == kModeRhs) ? L.d : pin);
  // MASK: the optimised set M (a lattice of the launch may still have none)
  const gptr<const unsigned char> __restrict__ act =
      MASK ? glob<const unsigned char>(L.act) : nullptr;
  const gptr<T> __restrict__ dst_out = glob<T>((MODE == kModeRhs) ? L.r : out);
  if (MODE == kModeRhs && act) {
    // a tile without points of M has no unknowns (its r is never read)
    int any = 0;
#pragma unroll
    for (int kk = 0; kk < TL::NPT; ++kk) {
      const int c = TilePos<TL>::own(kk);
      const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
      const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
      if ((TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz)))
        any |= act[gx + (size_t)L.nx * (gy + (size_t)L.ny * gz)];
    }
    if (!__syncthreads_or(any)) {
      gang_prepare(L, w.local, w.local != 0);
      return;
    }
  }
  if (MODE == kModeRhs) gang_prepare(L, w.local, false);
  // own nodes' data-block slots (loaded with the tile)
  int own_slot[TL::NPT];
#pragma unroll
  for (int kk = 0; kk < TL::NPT; ++kk) {
    const int c = TilePos<TL>::own(kk);
    const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    own_slot[kk] = (TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz))
                       ? glob<const int>(L.node_slot)[gx + (size_t)L.nx * (gy + (size_t)L.ny * gz)]
                       : -1;
  }
  for (int k = threadIdx.x; k < TL::HALO; k += TL::NT) {
    const int lx = k % TL::HX, ly = (k / TL::HX) % TL::HY, lz = k / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    T v0 = T(0), v1 = T(0), v2 = T(0);
    unsigned char m = 0;
    if (in_box(gx, gy, gz, L.nx, L.ny, L.nz)) {
      const size_t i = gx + (size_t)L.nx * (gy + (size_t)L.ny * gz);
      m = act ? act[i] : 1;
      // A p acts on the unknowns of M only; the gradient reads the stored
      // displacement of every point
      if (MODE != kModeApply || m) {
        v0 = src[i];
        v1 = src[N + i];
        v2 = src[2 * N + i];
      }
    }
    sp[0][k] = v0;
    sp[1][k] = v1;
    sp[2][k] = v2;
    if (MASK) sm[k] = m;
  }
  int rank[TL::NPT];
  list_data_nodes<T, TL>(own_slot, ds, rank);
  __syncthreads();
  eval_data_nodes<T, TL>(L, sp, ds);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < TL::NPT; ++kk) {
    const int c = TilePos<TL>::own(kk);
    const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    if (!(TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz))) continue;
    const size_t i = gx + (size_t)L.nx * (gy + (size_t)L.ny * gz);
    if (act && !act[i]) {
      // not an unknown: zero gradient / product
      dst_out[i] = T(0);
      dst_out[N + i] = T(0);
      dst_out[2 * N + i] = T(0);
      continue;
    }
    T o0, o1, o2;
    arap_at<T, TL>(L, sp, c, gx, gy, gz, o0, o1, o2, act ? sm : nullptr);
    if (rank[kk] >= 0) {
      const int e = (threadIdx.x / kWave) * DataShare<T, TL>::SEG + rank[kk];
      o0 += ds.d[0][e];
      o1 += ds.d[1][e];
      o2 += ds.d[2][e];
    }
    if (MODE == kModeApply) {
      dst_out[i] = o0;
      dst_out[N + i] = o1;
      dst_out[2 * N + i] = o2;
      continue;
    }
    // rotation part of the ARAP gradient: for neighbour j = i + s*axis,
    // e_ij = -s h axis and (2I - R_i - R_j) e_ij = -s h (2 axis - R_i[:,k] - R_j[:,k]).
    const gptr<const T> __restrict__ rot = glob<const T>(L.rot);
    const gptr<const T> __restrict__ bnode = glob<const T>(L.bnode);
    T q0 = T(0), q1 = T(0), q2 = T(0);
    const int pos[3] = {gx, gy, gz};
    const int lim[3] = {L.nx, L.ny, L.nz};
    const size_t stride[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const T ci0 = rot[rot_at(0, ax, N, i)], ci1 = rot[rot_at(1, ax, N, i)],
              ci2 = rot[rot_at(2, ax, N, i)];
#pragma unroll
      for (int sgn = -1; sgn <= 1; sgn += 2) {
        const int pj = pos[ax] + sgn;
        if (pj < 0 || pj >= lim[ax]) continue;
        const size_t j = sgn > 0 ? i + stride[ax] : i - stride[ax];
        const T cj0 = rot[rot_at(0, ax, N, j)], cj1 = rot[rot_at(1, ax, N, j)],
                cj2 = rot[rot_at(2, ax, N, j)];
        if (act && !act[j]) continue;  // only the edges inside M
        const T s = -T(sgn) * L.h;
        T u0 = -ci0 - cj0, u1 = -ci1 - cj1, u2 = -ci2 - cj2;
        if (ax == 0) u0 += T(2);
        if (ax == 1) u1 += T(2);
        if (ax == 2) u2 += T(2);
        q0 += s * u0;
        q1 += s * u1;
        q2 += s * u2;
      }
    }
    const T g0 = o0 - bnode[i] + L.wr * q0;
    const T g1 = o1 - bnode[N + i] + L.wr * q1;
    const T g2 = o2 - bnode[2 * N + i] + L.wr * q2;
    const T sg = (MODE == kModeGrad) ? T(1) : T(-1);
    dst_out[i] = sg * g0;
    dst_out[N + i] = sg * g1;
    dst_out[2 * N + i] = sg * g2;
  }
}

template <typename T, typename TL, bool MASK>
void launch_stencil_m(int mode, const Dispatch<T>& D, const T* pin, T* out, hipStream_t s) {
  switch (mode) {
    case kModeRhs:
      k_stencil<T, TL, kModeRhs, MASK><<<D.blocks, TL::NT, 0, s>>>(D, pin, out);
      break;
    case kModeApply:
      k_stencil<T, TL, kModeApply, MASK><<<D.blocks, TL::NT, 0, s>>>(D, pin, out);
      break;
    default: k_stencil<T, TL, kModeGrad, MASK><<<D.blocks, TL::NT, 0, s>>>(D, pin, out); break;
  }
}

template <typename T, typename TL>
void launch_stencil_t(int mode, const Dispatch<T>& D, const T* pin, T* out, hipStream_t s) {
  if (D.masked) launch_stencil_m<T, TL, true>(mode, D, pin, out, s);
  else launch_stencil_m<T, TL, false>(mode, D, pin, out, s);
}

// The tile kind is common to all lattices of a launch.
template <typename T>
hipError_t launch_stencil(int mode, const Dispatch<T>& D, const T* pin, T* out, hipStream_t s) {
  if (mode != kModeRhs && mode != kModeApply && mode != kModeGrad) return hipErrorInvalidValue;
  if (D.blocks <= 0) return hipSuccess;
  switch (D.one.tile) {
    case 1: launch_stencil_t<T, TileM>(mode, D, pin, out, s); break;
    case 2: launch_stencil_t<T, TileW>(mode, D, pin, out, s); break;
    case 3: launch_stencil_t<T, TileX>(mode, D, pin, out, s); break;
    case 4: launch_stencil_t<T, TileZ>(mode, D, pin, out, s); break;
    case 5: launch_stencil_t<T, TileY>(mode, D, pin, out, s); break;
    case 6: launch_stencil_t<T, TileH>(mode, D, pin, out, s); break;
    case 7: launch_stencil_t<T, TileC>(mode, D, pin, out, s); break;
    default: launch_stencil_t<T, TileS>(mode, D, pin, out, s); break;
  }
  return hipGetLastError();
}

// ===========================================================================
// one Jacobi-preconditioned CG iteration per launch (Sec. 7.1, position step)
// ===========================================================================
//
// Iteration m (FIRST: m = 0) reads the block partials S_{m-1} of the
// previous launch: r^T D^-1 r, p^T A p, (Ap)^T D^-1 r and (Ap)^T D^-1 Ap of
// iterate m-1.  From them
//   alpha_{m-1} = rz_{m-1} / p^T A p                    (zero if p^T A p <= 0)
//   rz_m        = rz_{m-1} - 2 alpha (Ap)^T D^-1 r + alpha^2 (Ap)^T D^-1 Ap
//   beta_m      = rz_m / rz_{m-1}                       (zero if rz_{m-1} <= 0)
// (rz_m is r_m^T D^-1 r_m expanded through r_m = r_{m-1} - alpha Ap_{m-1}, so
// one reduction phase per iteration suffices).  While staging the tile it
// forms r_m = r_{m-1} - alpha Ap_{m-1}, p_m = D^-1 r_m + beta p_{m-1}, applies
// d += alpha p_{m-1} to its own nodes, computes Ap_m and writes S_m.  Iterate
// m keeps r, p, Ap and S in buffer m % 2 of each pair (r_0 in L.r).  The
// halo inputs are loaded before the scalar reduction so that both latencies
// overlap.  The last iteration's step is applied by k_cg_final.

// A CG scalar as the sum hi + lo of two T values (lo = 0 for float64).  The
// step sizes are computed in float64 and applied to float32 vectors through
// both parts, x + s y = fma(lo, y, fma(hi, y, x)): a step size rounded to
// float32 would perturb the iterate coherently along p, and truncated CG
// amplifies such perturbations by about an order of magnitude per iteration
// once its Ritz values settle.
template <typename T>
struct Step {
  T hi, lo;
  __device__ __forceinline__ static Step of(double s) {
    Step r;
    r.hi = (T)s;
    r.lo = (T)(s - (double)r.hi);
    return r;
  }
  __device__ __forceinline__ T axpy(T x, T y) const { return fma(lo, y, fma(hi, y, x)); }
};

// alpha and beta from the sums v of the previous iterate.
template <typename T>
__device__ __forceinline__ void cg_steps(const double (&v)[4], Step<T>& alpha, Step<T>& beta,
                                         Scalars* sc, bool count_guard) {
  const double rz = v[0], pap = v[1], apdr = v[2], apdap = v[3];
  const double a = pap > 0.0 ? rz / pap : 0.0;
  double rz_new = rz - 2.0 * a * apdr + a * a * apdap;
  if (rz_new < 0.0) rz_new = 0.0;
  alpha = Step<T>::of(a);
  beta = Step<T>::of(rz > 0.0 ? rz_new / rz : 0.0);
  if (count_guard && threadIdx.x == 0 && !(pap > 0.0)) sc->guard_hits += 1;
}

template <typename T, int NT = kBlock>
__device__ __forceinline__ void cg_scalars(const double* s, int n, Step<T>& alpha, Step<T>& beta,
                                           Scalars* sc, bool count_guard) {
  double v[4];
  sum_partials_k<4, NT>(s, n, v);
  cg_steps<T>(v, alpha, beta, sc, count_guard);
}

// One CG iteration m on the tile of workgroup w (body of k_cg and of abandoned
// one-launch solves).  The own nodes' data-block slot, preconditioner,
// displacement and previous direction are loaded together with the halo,
// before the CG scalars, so that every workgroup pays one memory round trip
// before it stages the tile (a form that loaded them at their use, for more
// resident waves, was slower also on grids of several rounds of workgroups).
template <typename T, typename TL, bool FIRST, bool MASK = false>
__device__ __forceinline__ void cg_body(const Where<T>& w, int m, T (&sp)[3][TL::HALO],
                                        T (&sr)[3][TL::HALO], unsigned char (&sm)[TL::HALO],
                                        DataShare<T, TL>& ds) {
  const LevelView<T>& L = w.L;
  const TilePos<TL> t(L.nx, L.ny, w.local);
  const size_t N = L.N;
  const bool odd = (m & 1) != 0;
  const gptr<const T> __restrict__ r_in = glob<const T>((FIRST || odd) ? L.r : L.r2);
  const gptr<T> __restrict__ r_out = glob<T>(odd ? L.r2 : L.r);
  const gptr<const T> __restrict__ p_in = glob<const T>(odd ? L.pa : L.pb);
  const gptr<T> __restrict__ p_out = glob<T>(odd ? L.pb : L.pa);
  const gptr<const T> __restrict__ ap_in = glob<const T>(odd ? L.ap : L.ap2);
  const gptr<T> __restrict__ ap_out = glob<T>(odd ? L.ap2 : L.ap);
  const double* s_in = odd ? L.scg0 : L.scg1;
  double* s_out = odd ? L.scg1 : L.scg0;
  const gptr<const T> __restrict__ dinv = glob<const T>(L.dinv);
  const gptr<T> __restrict__ dvec = glob<T>(L.d);
  const gptr<const int> __restrict__ node_slot = glob<const int>(L.node_slot);
  // MASK: the optimised set M (a lattice of the launch may still have none)
  const gptr<const unsigned char> __restrict__ act =
      MASK ? glob<const unsigned char>(L.act) : nullptr;
  if (act) {
    // restricted to M: a tile without points of M has no unknowns; its
    // partials are zero.  Points outside M are read as 0 below and their
    // vectors never written.
    int any = 0;
#pragma unroll
    for (int kk = 0; kk < TL::NPT; ++kk) {
      const int c = TilePos<TL>::own(kk);
      const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
      const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
      if ((TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz)))
        any |= act[gx + (size_t)L.nx * (gy + (size_t)L.ny * gz)];
    }
    if (!__syncthreads_or(any)) {
      if (!FIRST && w.local == 0) {
        Step<T> a0, b0;
        cg_scalars<T, TL::NT>(s_in, L.ntiles, a0, b0, L.sc, true);
      }
      double zero[4] = {0.0, 0.0, 0.0, 0.0};
      write_partials<4, TL::NT>(zero, s_out, w.count, w.local);
      return;
    }
  }
  // 1. halo inputs into registers
  T hr[TL::HPT][3], hq[TL::HPT][3], hp[TL::HPT][3], ha[TL::HPT][3];
  size_t hi[TL::HPT];
  bool hin[TL::HPT];
  unsigned char hm[TL::HPT];
#pragma unroll
  for (int h = 0; h < TL::HPT; ++h) {
    const int k = threadIdx.x + h * TL::NT;
    const int lx = k % TL::HX, ly = (k / TL::HX) % TL::HY, lz = k / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    hin[h] = k < TL::HALO && in_box(gx, gy, gz, L.nx, L.ny, L.nz);
    hi[h] = hin[h] ? gx + (size_t)L.nx * (gy + (size_t)L.ny * gz) : 0;
    hm[h] = hin[h] ? (act ? act[hi[h]] : 1) : 0;
    hin[h] = hin[h] && hm[h];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      hr[h][a] = T(0);
      hq[h][a] = T(0);
      hp[h][a] = T(0);
      ha[h][a] = T(0);
    }
    if (hin[h]) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const size_t j = a * N + hi[h];
        hr[h][a] = r_in[j];
        hq[h][a] = dinv[j];
        if (!FIRST) {
          hp[h][a] = p_in[j];
          ha[h][a] = ap_in[j];
        }
      }
    }
  }
  // own nodes' data-block slot, preconditioner and displacement, loaded with
  // the halo so they are off the dependent chain of steps 3 and 4
  int own_slot[TL::NPT];
  T own_q[TL::NPT][3];
  T own_d[TL::NPT][3];
  T own_pp[TL::NPT][3];  // p of the previous iterate (the step d += alpha p)
#pragma unroll
  for (int kk = 0; kk < TL::NPT; ++kk) {
    const int c = TilePos<TL>::own(kk);
    const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    own_slot[kk] = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      own_q[kk][a] = T(0);
      own_d[kk][a] = T(0);
      own_pp[kk][a] = T(0);
    }
    if ((TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz)) &&
        (!act || act[gx + (size_t)L.nx * (gy + (size_t)L.ny * gz)])) {
      const size_t i = gx + (size_t)L.nx * (gy + (size_t)L.ny * gz);
      own_slot[kk] = node_slot[i];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        own_q[kk][a] = dinv[a * N + i];
        if (!FIRST) {
          own_d[kk][a] = dvec[a * N + i];
          own_pp[kk][a] = p_in[a * N + i];
        }
      }
    }
  }
  // 2. CG scalars of the previous iterate
  Step<T> alpha = Step<T>::of(0.0), beta = Step<T>::of(0.0);
  if (!FIRST) cg_scalars<T, TL::NT>(s_in, L.ntiles, alpha, beta, L.sc, w.local == 0);
  int rank[TL::NPT];
  list_data_nodes<T, TL>(own_slot, ds, rank);
  // 3. r_m, p_m into LDS; own nodes also store r_m, p_m and step d
#pragma unroll
  for (int h = 0; h < TL::HPT; ++h) {
    const int k = threadIdx.x + h * TL::NT;
    if (k >= TL::HALO) continue;
    T p3[3], r3[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T r = hr[h][a];
      if (!FIRST) r = alpha.axpy(r, -ha[h][a]);
      T p = hq[h][a] * r;
      if (!FIRST) p = beta.axpy(p, hp[h][a]);
      r3[a] = r;
      p3[a] = p;
      sp[a][k] = p;
      sr[a][k] = r;
    }
    if (MASK) sm[k] = hm[h];
    const int lx = k % TL::HX, ly = (k / TL::HX) % TL::HY, lz = k / (TL::HX * TL::HY);
    if (hin[h] && lx >= 1 && lx <= TL::TX && ly >= 1 && ly <= TL::TY && lz >= 1 &&
        lz <= TL::TZ) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const size_t j = a * N + hi[h];
        p_out[j] = p3[a];
        if (!FIRST) r_out[j] = r3[a];
      }
    }
  }
  __syncthreads();
  // 4. A p_m on own nodes and the block partials of S_m
  eval_data_nodes<T, TL>(L, sp, ds);
  __syncthreads();
  double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < TL::NPT; ++kk) {
    const int c = TilePos<TL>::own(kk);
    const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
    const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
    if (!(TilePos<TL>::owner() && in_box(gx, gy, gz, L.nx, L.ny, L.nz)) || (act && !sm[c])) continue;
    const size_t i = gx + (size_t)L.nx * (gy + (size_t)L.ny * gz);
    T o[3];
    arap_at<T, TL>(L, sp, c, gx, gy, gz, o[0], o[1], o[2], act ? sm : nullptr);
    const int e = (threadIdx.x / kWave) * DataShare<T, TL>::SEG + rank[kk];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (rank[kk] >= 0) o[a] += ds.d[a][e];
      const size_t j = a * N + i;
      ap_out[j] = o[a];
      if (!FIRST) dvec[j] = alpha.axpy(own_d[kk][a], own_pp[kk][a]);
      const double q = (double)own_q[kk][a], r = (double)sr[a][c],
                   p = (double)sp[a][c];
      const double ap = (double)o[a];
      part[0] += r * q * r;
      part[1] += p * ap;
      part[2] += ap * q * r;
      part[3] += ap * q * ap;
    }
  }
  write_partials<4, TL::NT>(part, s_out, w.count, w.local);
}

// Clock stamp of a launch's first workgroup at its start (graph timing).
__device__ __forceinline__ void entry_stamp(unsigned long long* stamp) {
  if (stamp != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
    *stamp = (unsigned long long)wall_clock64();
}

template <typename T, typename TL, bool FIRST, bool MASK>
__global__ __launch_bounds__(TL::NT) void k_cg(Dispatch<T> D, int m, unsigned long long* stamp) {
  if (skipped(D)) return;
  __shared__ T sp[3][TL::HALO];
  __shared__ T sr[3][TL::HALO];
  __shared__ unsigned char sm[TL::HALO];
  __shared__ DataShare<T, TL> ds;
  entry_stamp(stamp);
  const Where<T> w = locate(D, xcd_remap(blockIdx.x, gridDim.x));
  cg_body<T, TL, FIRST, MASK>(w, m, sp, sr, sm, ds);
}

// ---------------------------------------------------------------------------
// a whole CG solve in one launch
// ---------------------------------------------------------------------------
//
// One workgroup per tile for all iterations.  A workgroup keeps r, D^-1, d and
// A p of its own nodes, r and D^-1 of its halo nodes and (as far as registers
// last, up to two rounds of items) the rows of its data nodes in registers and
// p in LDS,
// and applies the scalar updates to its halo itself, so per iteration it
// exchanges only A p of the tile's surface nodes and the four block partials.
// The per-iteration launches stream every vector instead (36 MB at 64^3).
//
// Exchange without a cache flush: A p and the partials are stored and loaded
// at agent scope (past the caches that are private to a die), A p in one of
// two alternating buffers, the partials in slots that are empty until they
// are written.  A workgroup stores its surface A p, waits for those stores,
// then stores its partials; a reader that finds all partials of iterate m
// therefore finds A p_m too.  (Marks in A p itself instead of that order cost
// more than the wait, which the wave sums cover: 6.2 against 5.2 us per
// iteration at 16^3.)  Iterate m uses slot set m % 3; during iterate m a
// workgroup empties its slots of set (m + 1) % 3, which every workgroup has
// read by then: it has seen every partial of m - 1, each stored after its
// writer had read all of m - 2.
//
// Such a solve needs all tiles resident together, which concurrent work can
// prevent.  The first exchange decides: workgroup 0 of the lattice declares
// the solve running once it has seen every workgroup's first partials, and
// any workgroup that has waited `ticks` of the clock declares it abandoned (one
// compare-and-swap word, so all agree).  Once it runs every workgroup stays
// resident until its end, so no later wait can starve.  The workgroups of an
// abandoned solve, and those that start later, finish it from a ticket
// counter, one (iterate, tile) per ticket in order.  The holder of a ticket
// waits only for tickets handed out before its own, so this makes progress
// with any number of resident workgroups.  A workgroup goes through iterate 0
// before it learns that the solve is abandoned, and may do so when the tickets
// are many iterates ahead: what it then reads is no longer r_0.  So no ticket
// reads what iterate 0 of the gang stores: tickets have slot sets of their own
// and keep A p of even iterates behind ap's 3N.
//
// What bounds an iteration is the instructions of the 16 waves of a compute
// unit and the exchange's latency, so one wave alone forms the scalars, the
// four sums share their wave reductions (wave_sum4), and the stencil has no
// branches in waves away from the lattice's border.  The tiles of 2048 to
// 3584 nodes hold all of a level of up to 96^3 in the registers of the chip;
// there the rounds over the busiest tile's data nodes (940 at 96^3, 168 a
// round, 2.6 us each) are half of an iteration's 35 us, and the rows of all
// but the 16x16x8 tile are read again in every iteration.  A p packed by tile
// face instead of in node order took 5 % longer (more index arithmetic in the
// exchange), tiles dealt to the dies in turn 3 to 10 % longer.  The arithmetic
// is that of k_cg, and with the same tile kind so is the order of every sum:
// the results are the same bits.  (The large tiles have no k_cg form; they add
// the same terms up in another order.)

constexpr unsigned kSpinLimit = 1u << 18;         // polls before a wait gives up

enum GangState : unsigned { kGangForming = 0, kGangRunning = 1, kGangAbandoned = 2 };

template <typename U>
__device__ __forceinline__ U load_agent(const U* p) {
  return __hip_atomic_load(glob<U>(const_cast<U*>(p)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U>
__device__ __forceinline__ void store_agent(U* p, U v) {
  __hip_atomic_store(glob<U>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All vector-memory operations of the calling wave are complete.
__device__ __forceinline__ void wait_stores() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__device__ __forceinline__ unsigned long long slot_bits(double v) {
  return v != v ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(v);
}

// The n-th node of a tile's halo shell: the two z faces, then the rings of
// the layers between them.
template <typename TL>
__device__ __forceinline__ void shell_node(int n, int& lx, int& ly, int& lz) {
  constexpr int FACE = TL::HX * TL::HY, RING = 2 * TL::HX + 2 * TL::TY;
  if (n < 2 * FACE) {
    lz = n < FACE ? 0 : TL::HZ - 1;
    const int q = n < FACE ? n : n - FACE;
    lx = q % TL::HX;
    ly = q / TL::HX;
    return;
  }
  const int r = n - 2 * FACE;
  lz = 1 + r / RING;
  const int q = r % RING;
  if (q < 2 * TL::HX) {
    ly = q < TL::HX ? 0 : TL::HY - 1;
    lx = q % TL::HX;
  } else {
    ly = 1 + (q - 2 * TL::HX) / 2;
    lx = (q & 1) ? TL::HX - 1 : 0;
  }
}

// Waves 0 .. 3 wait for the partials of an iterate (slots s[4][n], n <= 256)
// and leave in sums[k][g] the sum of quantity k over the tiles 64 g .. 64 g +
// 63, as wave g of sum_partials_k forms it.  `limit` bounds the polls; a wait
// that gives up counts a timeout and leaves one poll to later ones.
__device__ __forceinline__ void gang_poll(const unsigned long long* s, int n, double* sums,
                                          unsigned& limit, int* timeouts) {
  const int b = threadIdx.x, lane = threadIdx.x & (kWave - 1);
  unsigned long long u[4];
  for (unsigned spins = 0;;) {
    bool all = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = b < n ? load_agent(s + k * n + b) : 0ull;
#pragma unroll
    for (int k = 0; k < 4; ++k) all &= u[k] != kEmptySlot;
    if (all) break;
    if (++spins > limit) {
      atomicAdd(timeouts, 1);
      limit = 1;
      break;
    }
  }
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = __longlong_as_double((long long)u[k]);
  const double x = wave_sum4(v);
  if (lane < 4) sums[lane * 4 + threadIdx.x / kWave] = x;
}

// Whether the solve runs as a gang (see above), decided at its first
// exchange; the same answer in every workgroup of the lattice.
__device__ __forceinline__ bool gang_assembled(double* gang, const unsigned long long* s, int n,
                                               bool first_tile, int ticks) {
  __shared__ unsigned state;
  unsigned* word = (unsigned*)gang;
  const long long t0 = wall_clock64();
  if (first_tile) {
    int late = ticks < 0 ? 1 : 0;
    if (threadIdx.x < kWave)
      for (int b = threadIdx.x; b < n && !late; b += kWave)
        while (load_agent(s + 3 * n + b) == kEmptySlot)
          if (wall_clock64() - t0 > ticks) {
            late = 1;
            break;
          }
    late = __syncthreads_or(late);
    if (threadIdx.x == 0) {
      const unsigned want = late ? kGangAbandoned : kGangRunning;
      const unsigned old = atomicCAS(word, (unsigned)kGangForming, want);
      state = old == kGangForming ? want : old;
    }
  } else if (threadIdx.x == 0) {
    unsigned v;
    while ((v = load_agent(word)) == kGangForming) {
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > ticks) {
        v = atomicCAS(word, (unsigned)kGangForming, (unsigned)kGangAbandoned);
        if (v == kGangForming) v = kGangAbandoned;
        break;
      }
    }
    state = v;
  }
  __syncthreads();
  return state == kGangRunning;
}

// Tickets of an abandoned solve (solo workgroups): the next (iterate, tile) in
// order, or -1 when all are handed out.  Waits until every ticket of the
// earlier iterates is done, then drops stale cache lines.
__device__ __forceinline__ long long take_ticket(double* gang, long long n, long long iters,
                                                 unsigned& limit, int* timeouts) {
  __shared__ long long ticket;
  unsigned long long* next = (unsigned long long*)gang + 1;
  unsigned long long* done = (unsigned long long*)gang + 2;
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long k = (long long)atomicAdd(next, 1ull);
    const bool valid = k < n * (iters + 1);
    for (unsigned spins = 0; valid && (long long)load_agent(done) < k / n * n;) {
      __builtin_amdgcn_s_sleep(4);
      if (++spins > limit) {
        atomicAdd(timeouts, 1);
        limit = 1;
        break;
      }
    }
    __threadfence();
    ticket = valid ? k : -1;
  }
  __syncthreads();
  return ticket;
}

// The calling workgroup's ticket is done: its stores first.
__device__ __forceinline__ void finish_ticket(double* gang) {
  wait_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    atomicAdd((unsigned long long*)gang + 2, 1ull);
  }
}

// For tests: waits until `tickets` tickets of an abandoned solve are done, at
// most 10 ms of the 100 MHz clock.
__device__ __forceinline__ void start_late(double* gang, unsigned tickets) {
  if (threadIdx.x == 0) {
    const long long t0 = wall_clock64();
    while (load_agent((unsigned long long*)gang + 2) < tickets &&
           wall_clock64() - t0 < 1000000)
      __builtin_amdgcn_s_sleep(1);
  }
  __syncthreads();
}

// The tile of workgroup g: lattices in dispatch order (so that a launch over
// several fills up lattice by lattice), and within a lattice a contiguous
// range of tiles per die.
template <typename T>
__device__ __forceinline__ Where<T> locate_gang(const Dispatch<T>& D) {
  Where<T> w = locate(D, blockIdx.x);
  const int first = blockIdx.x - w.local;   // the lattice's first workgroup
  const int die = blockIdx.x % kXcds;
  int before = 0;                           // tiles of the lower-numbered dies
  for (int x = 0; x < die; ++x) {
    const int lead = (x - first % kXcds + kXcds) % kXcds;  // first workgroup on die x
    if (lead < w.count) before += (w.count - lead - 1) / kXcds + 1;
  }
  w.local = before + w.local / kXcds;
  return w;
}

// One-launch solve of a tile on PT threads.  With fewer threads than owners a
// thread stands for VT owning threads of the per-iteration kernel, PT apart,
// and keeps their sums apart too.
template <typename T, typename TL_, int PT_>
struct Loop {
  using TL = TL_;
  static constexpr int PT = PT_, PW = PT / kWave;
  static constexpr int VT = TL::OWNERS > PT ? TL::OWNERS / PT : 1;
  static constexpr int NV = VT * TL::NPT;                   // own nodes per thread
  static constexpr int OW = (TL::OWNERS + kWave - 1) / kWave;  // owning waves
  static constexpr int SEG = kWave * TL::NPT;               // list entries per owning wave
  static constexpr int ENT = OW * SEG;
  static constexpr int SHELL = TL::HALO - TL::TX * TL::TY * TL::TZ;
  static constexpr int SPT = (SHELL + PT - 1) / PT;         // halo nodes per thread
  static constexpr int ROUND = PW * kNodesPerWave;          // data nodes per round
  // rounds of items whose rows stay in registers (54 values per lane each)
  static constexpr int KEEP = sizeof(T) == 8 ? (NV > 1 || SPT > 2 ? 0 : 1)
                                             : (NV > 4 ? 0 : NV > 1 ? 1 : 2);
  // the large tiles add a node's three parts up across lanes, as three arrays
  // of parts would not fit LDS beside p
  static constexpr bool LARGE = TL::TX * TL::TY * TL::TZ > 1024;
  static constexpr int PARTS = LARGE ? 1 : kPartsPerNode;
  // data nodes of the tile by owning wave, and the parts of their sums
  struct Share {
    int slot[ENT], node[ENT], cnt[OW];
    T d[PARTS][3][ENT];  // [part][component][entry]
  };
  // the calling lane's part of entry e (-1: none; whole waves call)
  __device__ __forceinline__ static void leave(Share& ls, int part, int e, const T (&o)[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (LARGE) {
        const T o1 = __shfl_down(o[a], 1, kWave), o2 = __shfl_down(o[a], 2, kWave);
        if (part == 0 && e >= 0) ls.d[0][a][e] = (o[a] + o1) + o2;
      } else if (e >= 0) {
        ls.d[part][a][e] = o[a];
      }
    }
  }
  __device__ __forceinline__ static T sum(const Share& ls, int a, int e) {
    return LARGE ? ls.d[0][a][e]
                 : (ls.d[0][a][e] + ls.d[PARTS > 1][a][e]) + ls.d[PARTS > 2 ? 2 : 0][a][e];
  }
  __device__ __forceinline__ static int owner(int j) {  // the owning thread of own node j
    return (int)threadIdx.x + (j / TL::NPT) * PT;
  }
  __device__ __forceinline__ static bool owns(int j) {
    return TL::OWNERS % PT == 0 || owner(j) < TL::OWNERS;
  }
  // layers of own node j above own node 0
  __device__ __forceinline__ static constexpr int layer(int j) {
    static_assert(VT == 1 || PT % (TL::TX * TL::TY) == 0);
    return (j / TL::NPT) * (PT / (TL::TX * TL::TY)) * TL::NPT + j % TL::NPT;
  }
  __device__ __forceinline__ static int own(int j) {  // LDS index of own node j
    const int t = owns(j) ? owner(j) : 0;
    const int lx = t % TL::TX + 1, ly = (t / TL::TX) % TL::TY + 1;
    const int lz = (t / (TL::TX * TL::TY)) * TL::NPT + j % TL::NPT + 1;
    return lx + TL::HX * (ly + TL::HY * lz);
  }
};

// Entry of list position v, or -1 past the end.
template <typename LP>
__device__ __forceinline__ int list_entry(const typename LP::Share& ls, int v) {
  int at = 0, e = -1;
  for (int u = 0; u < LP::OW; ++u) {
    const int c = ls.cnt[u];
    if (v >= at && v < at + c) e = u * LP::SEG + (v - at);
    at += c;
  }
  return e;
}

// One (node, part) item: the part's nine blocks times p.
template <typename T, int HX, int LEN, typename R>
__device__ __forceinline__ void part_product(const T (&sp)[3][LEN], int cz, R&& row, T (&o)[3]) {
  o[0] = o[1] = o[2] = T(0);
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const int q = cz + (j % 3 - 1) + HX * (j / 3 - 1);
    const T s0 = row(6 * j), s1 = row(6 * j + 1), s2 = row(6 * j + 2), s3 = row(6 * j + 3),
            s4 = row(6 * j + 4), s5 = row(6 * j + 5);
    const T q0 = sp[0][q], q1 = sp[1][q], q2 = sp[2][q];
    o[0] += s0 * q0 + s1 * q1 + s2 * q2;
    o[1] += s1 * q0 + s3 * q1 + s4 * q2;
    o[2] += s2 * q0 + s4 * q1 + s5 * q2;
  }
}

// All iterations of one CG solve and its last step.  stamp (may be null):
// two clock stamps, at the start of iteration 1 and of the last step.  LATE
// (tests): odd tiles start after -1 - ticks tickets.
template <typename T, typename LP, bool MASK, bool LATE = false>
__global__ __launch_bounds__(LP::PT) void k_cg_loop(Dispatch<T> D, int iters,
                                                    unsigned long long* stamp, int ticks) {
  if (skipped(D)) return;
  using TL = typename LP::TL;
  constexpr int NV = LP::NV, SPT = LP::SPT;
  constexpr int CW = 16 / (int)sizeof(T);  // entries per 16-byte chunk of a row
  __shared__ T sp[3][TL::HALO + 1];  // + 1: where threads past the shell write
  __shared__ unsigned char sm[TL::HALO];
  __shared__ typename LP::Share ls;
  __shared__ double sums[4 * LP::OW];   // the block's partials by owning wave
  __shared__ double gsums[16];          // the tiles' partials [4 sums][4 waves]
  __shared__ Step<T> steps[2];
  const Where<T> w = locate_gang(D);
  const LevelView<T>& L = w.L;
  const int n_tiles = L.loop_tiles;
  const size_t N = L.N;
  // (as values: a choice between two members of L would keep L in memory)
  T* const v_r = L.r;
  T* const v_r2 = L.r2;
  T* const v_pa = L.pa;
  T* const v_pb = L.pb;
  T* const v_ap = L.ap;
  T* const v_ap2 = L.ap2;
  unsigned long long* const slots = gang_slots(L.gang);
  const gptr<T> __restrict__ dvec = glob<T>(L.d);
  const gptr<const unsigned char> __restrict__ act =
      MASK ? glob<const unsigned char>(L.act) : nullptr;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int part_id = lane % kPartsPerNode, item = wv * kNodesPerWave + lane / kPartsPerNode;
  const bool has_item = lane / kPartsPerNode < kNodesPerWave;
  T r[NV][3], q[NV][3], d[NV][3], ap[NV][3];  // own nodes
  // bits 0..5: the neighbours it couples to (-x +x -y +y -z +z); bit 6: on the
  // tile's surface, neighbours read its A p; bit 7: an unknown; from bit 8:
  // 1 + the entry of its data blocks in the wave's list, 0 without
  unsigned nbr[NV];
  unsigned node0 = 0;  // global index of own node 0 (of the other own nodes: own_node)
  const unsigned plane = (unsigned)L.nx * (unsigned)L.ny;
  auto own_node = [&](int kk) { return node0 + plane * (unsigned)LP::layer(kk); };
  auto unknown = [&](int kk) { return (nbr[kk] & 128u) != 0; };
  T hr[SPT][3], hq[SPT][3];  // halo nodes
  int hnode[SPT], hc[SPT];   // global index (-1: none), LDS index
  T keep[LP::KEEP > 0 ? LP::KEEP : 1][54];  // rows of the lane's first items,
  // LDS centre and list entry (-1: none) of the kept items and of one more
  // round; the slot of the latter
  int kcz[LP::KEEP + 1], ke[LP::KEEP + 1], kslot = 0;
  int n_data = 0;
  Step<T> alpha = Step<T>::of(0.0), beta = Step<T>::of(0.0);
  unsigned limit = kSpinLimit;
  bool solo = false, load = true;
  int tile = w.local, m = 0;
  for (;;) {
    if (solo) {
      const long long k = take_ticket(L.gang, n_tiles, iters, limit, &L.sc->bar_timeouts);
      if (k < 0) return;
      m = (int)(k / n_tiles);
      tile = (int)(k % n_tiles);
      load = true;
    }
    const bool last = m == iters, odd = (m & 1) != 0;
    if (load) {
      // the tile's state: r_0 and d, or (solo) that of iterate m - 1
      load = false;
      if (LATE && !solo && (tile & 1)) start_late(L.gang, -1 - ticks);
      const TilePos<TL> t(L.nx, L.ny, tile);
      const gptr<const T> __restrict__ rin = glob<const T>(m == 0 || odd ? v_r : v_r2);
      const gptr<const T> __restrict__ pin = glob<const T>(odd ? v_pa : v_pb);
      const gptr<const T> __restrict__ apin = glob<const T>(odd ? v_ap + 3 * N : v_ap2);  // (solo)
      const gptr<const T> __restrict__ dinv = glob<const T>(L.dinv);
      int slot[NV];
#pragma unroll
      for (int kk = 0; kk < NV; ++kk) {
        const int c = LP::own(kk);
        const int lx = c % TL::HX, ly = (c / TL::HX) % TL::HY, lz = c / (TL::HX * TL::HY);
        const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
        const bool in = LP::owns(kk) && in_box(gx, gy, gz, L.nx, L.ny, L.nz);
        const size_t i = in ? gx + (size_t)L.nx * (gy + (size_t)L.ny * gz) : 0;
        const bool is = in && (!act || act[i]);
        if (kk == 0) node0 = gx + L.nx * (gy + L.ny * gz);
        // (solo: every A p is read back from memory)
        nbr[kk] = (gx > 0) | (gx < L.nx - 1) << 1 | (gy > 0) << 2 | (gy < L.ny - 1) << 3 |
                  (gz > 0) << 4 | (gz < L.nz - 1) << 5 |
                  (is && (solo || lx == 1 || lx == TL::TX || ly == 1 || ly == TL::TY ||
                          lz == 1 || lz == TL::TZ)) << 6 | is << 7;
        slot[kk] = is ? glob<const int>(L.node_slot)[i] : -1;
        if (MASK && LP::owns(kk)) sm[c] = is;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          r[kk][a] = is ? rin[a * N + i] : T(0);
          q[kk][a] = is ? dinv[a * N + i] : T(0);
          d[kk][a] = is ? dvec[a * N + i] : T(0);
          const bool past = solo && m > 0 && is;  // else A p = p = 0
          ap[kk][a] = past ? apin[a * N + i] : T(0);
          if (LP::owns(kk)) sp[a][c] = past ? pin[a * N + i] : T(0);
        }
      }
      if (MASK && act && !solo) {
        // a tile without unknowns: its slots hold zeros already, or do now
        int any = 0;
#pragma unroll
        for (int kk = 0; kk < NV; ++kk) any |= unknown(kk);
        if (!__syncthreads_or(any) && tile != 0) {
          if (LP::LARGE && threadIdx.x < kGangSlots)
            store_agent(slots + (size_t)threadIdx.x * n_tiles + tile, 0ull);
          return;
        }
      }
#pragma unroll
      for (int h = 0; h < SPT; ++h) {
        const int n = threadIdx.x + h * LP::PT;
        int lx = 0, ly = 0, lz = 0;
        shell_node<TL>(n < LP::SHELL ? n : 0, lx, ly, lz);
        const int gx = t.x0 + lx, gy = t.y0 + ly, gz = t.z0 + lz;
        const bool in = n < LP::SHELL && in_box(gx, gy, gz, L.nx, L.ny, L.nz);
        const size_t i = in ? gx + (size_t)L.nx * (gy + (size_t)L.ny * gz) : 0;
        hc[h] = n < LP::SHELL ? lx + TL::HX * (ly + TL::HY * lz) : TL::HALO;
        hnode[h] = in && (!act || act[i]) ? (int)i : -1;
        if (MASK && n < LP::SHELL) sm[hc[h]] = hnode[h] >= 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          hr[h][a] = hnode[h] >= 0 ? rin[a * N + i] : T(0);
          hq[h][a] = hnode[h] >= 0 ? dinv[a * N + i] : T(0);
          sp[a][hc[h]] = solo && m > 0 && hnode[h] >= 0 ? pin[a * N + i] : T(0);
        }
      }
      // the lists of data nodes, one per owning wave
#pragma unroll
      for (int vt = 0; vt < LP::VT; ++vt) {
        const int ow = wv + vt * LP::PW;
        if (ow >= LP::OW) continue;
        int base = 0;
#pragma unroll
        for (int z = 0; z < TL::NPT; ++z) {
          const int kk = vt * TL::NPT + z;
          const unsigned long long has = __ballot(slot[kk] >= 0);
          if (slot[kk] >= 0) {
            const int e = ow * LP::SEG + base + __popcll(has & ((1ull << lane) - 1ull));
            nbr[kk] |= (unsigned)(e + 1) << 8;
            ls.slot[e] = slot[kk];
            ls.node[e] = LP::own(kk);
          }
          base += __popcll(has);
        }
        if (lane == 0) ls.cnt[ow] = base;
      }
      __syncthreads();
      if (MASK && act) {  // only the edges inside M
        constexpr int off[3] = {1, TL::HX, TL::HX * TL::HY};
#pragma unroll
        for (int kk = 0; kk < NV; ++kk) {
          const int c = LP::own(kk);
#pragma unroll
          for (int k = 0; k < 6; ++k)
            if (!sm[c + ((k & 1) ? off[k / 2] : -off[k / 2])]) nbr[kk] &= ~(1u << k);
        }
      }
      n_data = 0;
      for (int u = 0; u < LP::OW; ++u) n_data += ls.cnt[u];
#pragma unroll
      for (int x = 0; x <= LP::KEEP; ++x) {
        ke[x] = has_item ? list_entry<LP>(ls, x * LP::ROUND + item) : -1;
        kcz[x] = ke[x] >= 0 ? ls.node[ke[x]] + TL::HX * TL::HY * (part_id - 1) : 0;
        if (x == LP::KEEP) kslot = ke[x] >= 0 ? ls.slot[ke[x]] : 0;
        if (x < LP::KEEP && ke[x] >= 0) {
          const gptr<const T> __restrict__ A = glob<const T>(static_cast<const T*>(
              __builtin_assume_aligned(L.A27r + (size_t)ls.slot[ke[x]] * kA27Row + part_id * CW,
                                       16)));
#pragma unroll
          for (int y = 0; y < 54; ++y) keep[x][y] = A[kPartsPerNode * CW * (y / CW) + y % CW];
        }
      }
    }
    if (stamp != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
      if (m == 1) stamp[0] = (unsigned long long)wall_clock64();
      if (last) stamp[1] = (unsigned long long)wall_clock64();
    }
    T ha[SPT][3];
#pragma unroll
    for (int h = 0; h < SPT; ++h) ha[h][0] = ha[h][1] = ha[h][2] = T(0);
    if (m > 0) {
      // 1. the scalars of iterate m - 1 (wave 0) and the halo's A p
      const unsigned long long* s = slots + (size_t)((m - 1) % 3 + 3 * solo) * 4 * n_tiles;
      if (m == 1 && !solo && !gang_assembled(L.gang, s, n_tiles, tile == 0, ticks)) {
        solo = true;
        continue;
      }
      if (wv < 4) gang_poll(s, n_tiles, gsums, limit, &L.sc->bar_timeouts);
      __syncthreads();
      const T* const ap_in = odd ? v_ap + (solo ? 3 * N : 0) : v_ap2;
#pragma unroll
      for (int h = 0; h < SPT; ++h) {
        if (hnode[h] < 0) continue;
#pragma unroll
        for (int a = 0; a < 3; ++a) ha[h][a] = load_agent(ap_in + a * N + (unsigned)hnode[h]);
      }
      if (wv == 0) {
        double v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          v[x] = 0.0;
#pragma unroll
          for (int g = 0; g < 4; ++g) v[x] += gsums[4 * x + g];
        }
        Step<T> al, be;
        cg_steps<T>(v, al, be, L.sc, tile == 0);
        if (lane == 0) {
          steps[0] = al;
          steps[1] = be;
        }
      }
      __syncthreads();
      alpha = steps[0];
      beta = steps[1];
    }
    // 2. r_m, p_m and the step of d (iterate 0: alpha = beta = 0, so p = D^-1 r)
    if (wv < LP::OW) {
#pragma unroll
      for (int kk = 0; kk < NV; ++kk) {
        const int c = LP::own(kk);
        T p[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = sp[a][c];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          d[kk][a] = alpha.axpy(d[kk][a], p[a]);
          r[kk][a] = alpha.axpy(r[kk][a], -ap[kk][a]);
          p[a] = beta.axpy(q[kk][a] * r[kk][a], p[a]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) sp[a][c] = p[a];
      }
    }
    if (last || solo) {
#pragma unroll
      for (int kk = 0; kk < NV; ++kk) {
        if (!unknown(kk)) continue;
        const int c = LP::own(kk);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          dvec[a * N + own_node(kk)] = d[kk][a];
          if (last) continue;
          glob<T>(odd ? v_pb : v_pa)[a * N + own_node(kk)] = sp[a][c];
          if (m > 0) glob<T>(odd ? v_r2 : v_r)[a * N + own_node(kk)] = r[kk][a];
        }
      }
      if (last) {
        if (!solo) return;
        finish_ticket(L.gang);
        continue;
      }
    }
#pragma unroll
    for (int h = 0; h < SPT; ++h) {
      T p[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) p[a] = sp[a][hc[h]];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        hr[h][a] = alpha.axpy(hr[h][a], -ha[h][a]);
        p[a] = beta.axpy(hq[h][a] * hr[h][a], p[a]);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) sp[a][hc[h]] = p[a];
    }
    __syncthreads();
    // 3. A p_m: the data part by (node, part) items, the first rounds from
    // the rows kept in registers
#pragma unroll
    for (int x = 0; x < LP::KEEP; ++x) {
      T o[3] = {T(0), T(0), T(0)};
      if (ke[x] >= 0) part_product<T, TL::HX>(sp, kcz[x], [&](int y) { return keep[x][y]; }, o);
      LP::leave(ls, part_id, ke[x], o);
    }
    for (int v0 = LP::KEEP * LP::ROUND; v0 < n_data; v0 += LP::ROUND) {
      int e = ke[LP::KEEP], cz = kcz[LP::KEEP], at = kslot;
      if (v0 > LP::KEEP * LP::ROUND) {
        e = has_item ? list_entry<LP>(ls, v0 + item) : -1;
        cz = e >= 0 ? ls.node[e] + TL::HX * TL::HY * (part_id - 1) : 0;
        at = e >= 0 ? ls.slot[e] : 0;
      }
      T o[3] = {T(0), T(0), T(0)};
      if (e >= 0) {
        const gptr<const T> __restrict__ A = glob<const T>(static_cast<const T*>(
            __builtin_assume_aligned(L.A27r + (size_t)at * kA27Row + part_id * CW, 16)));
        part_product<T, TL::HX>(sp, cz,
                                [&](int y) { return A[kPartsPerNode * CW * (y / CW) + y % CW]; },
                                o);
      }
      LP::leave(ls, part_id, e, o);
    }
    __syncthreads();
    T* const ap_out = odd ? v_ap2 : v_ap + (solo ? 3 * N : 0);
    // empty the slots of the next iterate
    if (m > 0 && !solo && threadIdx.x < 4)
      store_agent(slots + ((size_t)((m + 1) % 3) * 4 + threadIdx.x) * n_tiles + tile, kEmptySlot);
    const T w2 = T(2) * L.wr;
#pragma unroll
    for (int vt = 0; vt < LP::VT; ++vt) {
      const int ow = wv + vt * LP::PW;
      if (ow >= LP::OW) continue;
      double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int z = 0; z < TL::NPT; ++z) {
        const int kk = vt * TL::NPT + z;
        const int c = LP::own(kk);
        constexpr int off[3] = {1, TL::HX, TL::HX * TL::HY};
        T l[3] = {T(0), T(0), T(0)};
        const T p0[3] = {sp[0][c], sp[1][c], sp[2][c]};
        if (__all((nbr[kk] & 63u) == 63u)) {
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a)
              l[a] += p0[a] - sp[a][c + ((k & 1) ? off[k / 2] : -off[k / 2])];
        } else {
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              const T x = p0[a] - sp[a][c + ((k & 1) ? off[k / 2] : -off[k / 2])];
              l[a] += (nbr[kk] >> k & 1u) ? x : T(0);
            }
        }
        T dd[3] = {T(0), T(0), T(0)};
        if (nbr[kk] >> 8) {
#pragma unroll
          for (int a = 0; a < 3; ++a) dd[a] = LP::sum(ls, a, (int)(nbr[kk] >> 8) - 1);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          T o;
          {
#pragma clang fp contract(off)
            o = w2 * l[a];  // rounded before the data part, as in k_cg
            o = o + dd[a];
          }
          ap[kk][a] = unknown(kk) ? o : T(0);
          const double qd = (double)q[kk][a], rd = (double)r[kk][a], pd = (double)p0[a];
          const double ad = (double)ap[kk][a];
          part[0] += rd * qd * rd;
          part[1] += pd * ad;
          part[2] += ad * qd * rd;
          part[3] += ad * qd * ad;
        }
        if (nbr[kk] & 64u) {
#pragma unroll
          for (int a = 0; a < 3; ++a)
            store_agent(ap_out + a * N + own_node(kk), ap[kk][a]);
        }
      }
      const double x = wave_sum4(part);
      if (lane < 4) sums[lane * LP::OW + ow] = x;
    }
    // 4. the block's partials, published after A p
    wait_stores();
    __syncthreads();
    if (threadIdx.x < 4) {
      double x = 0.0;
#pragma unroll
      for (int u = 0; u < LP::OW; ++u) x += sums[threadIdx.x * LP::OW + u];
      const int set = m % 3 + 3 * solo;
      store_agent(slots + ((size_t)set * 4 + threadIdx.x) * n_tiles + tile, slot_bits(x));
    }
    if (solo) finish_ticket(L.gang);
    else ++m;
  }
}

// d += alpha p of the last CG iterate (node workgroups).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_cg_final(Dispatch<T> D, int last,
                                                     unsigned long long* stamp) {
  if (skipped(D)) return;
  entry_stamp(stamp);
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& L = w.L;
  const bool odd = (last & 1) != 0;
  Step<T> alpha, beta;
  cg_scalars<T>(odd ? L.scg1 : L.scg0, L.ntiles, alpha, beta, L.sc, w.local == 0);
  const int i = w.local * kBlock + threadIdx.x;
  if (i >= L.N || (L.act && !L.act[i])) return;
  const size_t N = L.N;
  const gptr<const T> __restrict__ p = glob<const T>(odd ? L.pb : L.pa);
  const gptr<T> __restrict__ d = glob<T>(L.d);
#pragma unroll
  for (int a = 0; a < 3; ++a) d[a * N + i] = alpha.axpy(d[a * N + i], p[a * N + i]);
}

template <typename T, typename TL>
void launch_cg_t(int m, const Dispatch<T>& D, hipStream_t s, unsigned long long* stamp) {
  if (D.masked) {
    if (m == 0) k_cg<T, TL, true, true><<<D.blocks, TL::NT, 0, s>>>(D, m, stamp);
    else k_cg<T, TL, false, true><<<D.blocks, TL::NT, 0, s>>>(D, m, stamp);
  } else {
    if (m == 0) k_cg<T, TL, true, false><<<D.blocks, TL::NT, 0, s>>>(D, m, stamp);
    else k_cg<T, TL, false, false><<<D.blocks, TL::NT, 0, s>>>(D, m, stamp);
  }
}

template <typename T>
hipError_t launch_cg(int m, const Dispatch<T>& D, hipStream_t s, unsigned long long* stamp) {
  if (D.blocks <= 0) return hipSuccess;
  switch (D.one.tile) {
    case 1: launch_cg_t<T, TileM>(m, D, s, stamp); break;
    case 2: launch_cg_t<T, TileW>(m, D, s, stamp); break;
    case 3: launch_cg_t<T, TileX>(m, D, s, stamp); break;
    case 4: launch_cg_t<T, TileZ>(m, D, s, stamp); break;
    case 5: launch_cg_t<T, TileY>(m, D, s, stamp); break;
    case 6: launch_cg_t<T, TileH>(m, D, s, stamp); break;
    case 7: launch_cg_t<T, TileC>(m, D, s, stamp); break;
    default: launch_cg_t<T, TileS>(m, D, s, stamp); break;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_cg_final(int last, const Dispatch<T>& D, hipStream_t s,
                           unsigned long long* stamp) {
  if (D.blocks <= 0) return hipSuccess;
  k_cg_final<T><<<D.blocks, kBlock, 0, s>>>(D, last, stamp);
  return hipGetLastError();
}

// Calls f(kernel, threads) with the k_cg_loop instance of a tile kind.  512
// threads leave 256 registers each, which hold two rounds of rows (336 data
// nodes) beside the state of a 1024-node tile; on 1024 threads of 128
// registers each the same state spilled.
template <typename T, bool MASK, typename F>
hipError_t with_loop_kernel(int kind, F&& f) {
  if constexpr (sizeof(T) == 4) {
    switch (kind) {
      case 8: return f(k_cg_loop<T, Loop<T, TileL4, 512>, MASK>, 512);
      case 9: return f(k_cg_loop<T, Loop<T, TileL6, 512>, MASK>, 512);
      case 10:
        if constexpr (!MASK) return f(k_cg_loop<T, Loop<T, TileL7, 512>, MASK>, 512);
    }
  }
  switch (kind) {
    case 0:
    case 7: return f(k_cg_loop<T, Loop<T, TileS, 512>, MASK>, 512);
    case 1: return f(k_cg_loop<T, Loop<T, TileM, 512>, MASK>, 512);
    case 2: return f(k_cg_loop<T, Loop<T, TileW, 256>, MASK>, 256);
    case 3: return f(k_cg_loop<T, Loop<T, TileX, 512>, MASK>, 512);
    case 4: return f(k_cg_loop<T, Loop<T, TileZ, 512>, MASK>, 512);
    case 5: return f(k_cg_loop<T, Loop<T, TileY, 512>, MASK>, 512);
    case 6: return f(k_cg_loop<T, Loop<T, TileH, 512>, MASK>, 512);
  }
  return hipErrorNotSupported;  // a large tile without an instance
}

// The same for the kinds with an instance whose odd tiles start late.
template <typename T, bool MASK, typename F>
hipError_t with_late_kernel(int kind, F&& f) {
  switch (kind) {
    case 0: return f(k_cg_loop<T, Loop<T, TileS, 512>, MASK, true>, 512);
    case 6: return f(k_cg_loop<T, Loop<T, TileH, 512>, MASK, true>, 512);
    case 8:
      if constexpr (sizeof(T) == 4) return f(k_cg_loop<T, Loop<T, TileL4, 512>, MASK, true>, 512);
  }
  return hipErrorNotSupported;
}

template <typename T>
hipError_t launch_cg_loop(int iters, const Dispatch<T>& D, hipStream_t s,
                          unsigned long long* stamp, int ticks) {
  if (D.blocks <= 0 || iters <= 0) return hipSuccess;
  auto go = [&](auto kernel, int threads) {
    kernel<<<D.blocks, threads, 0, s>>>(D, iters, stamp, ticks);
    return hipGetLastError();
  };
  if (ticks < -1)
    return D.masked ? with_late_kernel<T, true>(D.one.loop_tile, go)
                    : with_late_kernel<T, false>(D.one.loop_tile, go);
  return D.masked ? with_loop_kernel<T, true>(D.one.loop_tile, go)
                  : with_loop_kernel<T, false>(D.one.loop_tile, go);
}

template <typename T>
hipError_t cg_loop_capacity(int kind, bool masked, int* tiles) {
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  auto ask = [&](auto kernel, int threads) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0);
  };
  e = masked ? with_loop_kernel<T, true>(kind, ask) : with_loop_kernel<T, false>(kind, ask);
  if (e == hipErrorNotSupported) e = hipSuccess;  // per_cu is 0
  *tiles = std::min(cus * per_cu, kGangMaxTiles);
  return e;
}

// ===========================================================================
// energy, eq. (1): rows (dense and sparse) and ARAP edges, float64 sums
// ===========================================================================

template <typename T>
__global__ __launch_bounds__(kBlock) void k_energy(Dispatch<T> D) {
  if (skipped(D)) return;
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& L = w.L;
  double part[3] = {0.0, 0.0, 0.0};
  const size_t N = L.N;
  const T* __restrict__ d = L.d;
  if (w.local < L.rblocks) {
    const int row = w.local * kBlock + threadIdx.x;
    const int rows = L.sc->rows;
    if (row < rows) {
      const int cell = L.row_cell[row];
      const int cnx = L.nx - 1, cny = L.ny - 1;
      const int cx = cell % cnx, cy = (cell / cnx) % cny, cz = cell / (cnx * cny);
      const T* __restrict__ f = L.row_f;
      const T* __restrict__ sn = L.row_sn;
      const T fx = f[row], fy = f[(size_t)rows + row], fz = f[2 * (size_t)rows + row];
      T s0 = T(0), s1 = T(0), s2 = T(0);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const size_t m = (cx + (k & 1)) + (size_t)L.nx * ((cy + ((k >> 1) & 1)) +
                                                          (size_t)L.ny * (cz + (k >> 2)));
        const T wk = corner_weight<T>(k, fx, fy, fz);
        s0 += wk * d[m];
        s1 += wk * d[N + m];
        s2 += wk * d[2 * N + m];
      }
      const T res = sn[row] * s0 + sn[(size_t)rows + row] * s1 + sn[2 * (size_t)rows + row] * s2 -
                    L.row_rho[row];
      const double e = (double)res * (double)res;
      if (row < L.sc->n_dense) part[0] = e; else part[1] = e;
    }
  } else {
    const int i = (w.local - L.rblocks) * kBlock + threadIdx.x;
    // E_reg sums the edges inside M (all of them when the whole lattice is
    // optimised)
    if (i < L.N && (!L.act || L.act[i])) {
      const T* __restrict__ rot = L.rot;
      const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
      const int pos[3] = {x, y, z};
      const int lim[3] = {L.nx, L.ny, L.nz};
      const size_t stride[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
      double acc = 0.0;
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        // (I - R_i) e_ij with e_ij = -s h axis
        T c0 = -rot[rot_at(0, ax, N, i)], c1 = -rot[rot_at(1, ax, N, i)],
          c2 = -rot[rot_at(2, ax, N, i)];
        if (ax == 0) c0 += T(1);
        if (ax == 1) c1 += T(1);
        if (ax == 2) c2 += T(1);
#pragma unroll
        for (int sgn = -1; sgn <= 1; sgn += 2) {
          const int pj = pos[ax] + sgn;
          if (pj < 0 || pj >= lim[ax]) continue;
          const size_t j = sgn > 0 ? i + stride[ax] : i - stride[ax];
          if (L.act && !L.act[j]) continue;
          const T s = -T(sgn) * L.h;
          const T e0 = d[i] - d[j] + s * c0;
          const T e1 = d[N + i] - d[N + j] + s * c1;
          const T e2 = d[2 * N + i] - d[2 * N + j] + s * c2;
          acc += (double)e0 * e0 + (double)e1 * e1 + (double)e2 * e2;
        }
      }
      part[2] = (double)L.wr * acc;
    }
  }
  write_partials<3>(part, L.pe, w.count, w.local);
}

// One workgroup per lattice: sums its energy partials into sc->energy.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_energy_finalize(Dispatch<T> D1, int record_trace) {
  if (skipped(D1)) return;
  const LevelView<T> L = view_of(D1, blockIdx.x);
  const int n = energy_blocks_dev(L);
  double v[3];
  sum_partials_k<3>(L.pe, n, v);
  if (threadIdx.x == 0) {
    Scalars* sc = L.sc;
    sc->energy[0] = v[0] + v[1] + v[2];
    sc->energy[1] = v[0];
    sc->energy[2] = v[1];
    sc->energy[3] = v[2];
    if (record_trace && sc->n_trace < VD_MAX_TRACE) {
      sc->trace[sc->n_trace] = sc->energy[0];
      sc->n_trace += 1;
    }
  }
}

template <typename T>
hipError_t launch_energy(const Dispatch<T>& De, const Dispatch<T>& D1, int record_trace,
                         hipStream_t s) {
  if (De.blocks <= 0) return hipSuccess;
  k_energy<T><<<De.blocks, kBlock, 0, s>>>(De);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_energy_finalize<T><<<D1.blocks, kBlock, 0, s>>>(D1, record_trace);
  return hipGetLastError();
}

template <typename T>
__global__ void k_reset_counters(Dispatch<T> D1) {
  if (threadIdx.x != 0) return;
  Scalars* sc = view_of(D1, blockIdx.x).sc;
  sc->guard_hits = 0;
  sc->polar_fp64 = 0;
  sc->polar_keep = 0;
  sc->n_trace = 0;
  sc->bar_timeouts = 0;
}

__global__ void k_target_begin(Scalars* sc, double target) {
  if (threadIdx.x != 0) return;
  sc->target = target;
  sc->gn_done = 0;
  sc->stop = sc->energy[0] <= target ? 1 : 0;
}

__global__ void k_target_step(Scalars* sc) {
  if (threadIdx.x != 0 || sc->stop) return;
  sc->gn_done += 1;
  if (sc->energy[0] <= sc->target) sc->stop = 1;
}

hipError_t launch_target_begin(Scalars* sc, double target, hipStream_t s) {
  k_target_begin<<<1, 64, 0, s>>>(sc, target);
  return hipGetLastError();
}

hipError_t launch_target_step(Scalars* sc, hipStream_t s) {
  k_target_step<<<1, 64, 0, s>>>(sc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_reset_counters(const Dispatch<T>& D1, hipStream_t s) {
  k_reset_counters<T><<<D1.blocks, 64, 0, s>>>(D1);
  return hipGetLastError();
}

// ===========================================================================
// rotation step (Sec. 7.1): M_i = sum_j (t_i - t_j)(t_hat_i - t_hat_j)^T
// ===========================================================================

template <typename T>
__global__ __launch_bounds__(kBlock) void k_polar(Dispatch<T> D) {
  if (skipped(D)) return;
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& L = w.L;
  const int i = w.local * kBlock + threadIdx.x;
  if (i >= L.N || (L.act && !L.act[i])) return;  // points outside M keep R
  const size_t N = L.N;
  const T* __restrict__ d = L.d;
  T* rot = L.rot;
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const int pos[3] = {x, y, z};
  const int lim[3] = {L.nx, L.ny, L.nz};
  const size_t stride[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
  const T di0 = d[i], di1 = d[N + i], di2 = d[2 * N + i];
  T M[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) M[k] = T(0);
  const T h2 = L.h * L.h;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
    for (int sgn = -1; sgn <= 1; sgn += 2) {
      const int pj = pos[ax] + sgn;
      if (pj < 0 || pj >= lim[ax]) continue;
      const size_t j = sgn > 0 ? i + stride[ax] : i - stride[ax];
      if (L.act && !L.act[j]) continue;  // the terms of eq. (4) inside M
      // (d_i - d_j + e_ij) e_ij^T with e_ij = -s h axis: column ax gets
      // -s h (d_i - d_j) + h^2 axis
      const T s = -T(sgn) * L.h;
      M[0 * 3 + ax] += s * (di0 - d[j]);
      M[1 * 3 + ax] += s * (di1 - d[N + j]);
      M[2 * 3 + ax] += s * (di2 - d[2 * N + j]);
      M[ax * 3 + ax] += h2;
    }
  }
  T Rp[9], R[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) Rp[k] = rot[(size_t)k * N + i];
  const int code = fit_or_keep<T>(M, Rp, R);
#pragma unroll
  for (int k = 0; k < 9; ++k) rot[(size_t)k * N + i] = R[k];
  if (code == kFitFp64) atomicAdd(&L.sc->polar_fp64, 1);
  if (code == kFitKeep) atomicAdd(&L.sc->polar_keep, 1);
}

template <typename T>
hipError_t launch_polar(const Dispatch<T>& D, hipStream_t s) {
  if (D.blocks <= 0) return hipSuccess;
  k_polar<T><<<D.blocks, kBlock, 0, s>>>(D);
  return hipGetLastError();
}

// ===========================================================================
// level transfers (Sec. 7.2)
// ===========================================================================

// Level node (a,b,c) takes the finest node stride*(a,b,c): d, base and R.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_inject(Dispatch<T> D, Dispatch<T> F, int stride) {
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& Lv = w.L;
  const int i = w.local * kBlock + threadIdx.x;
  if (i >= Lv.N) return;
  const LevelView<T> Fv = view_of(F, w.b);
  const int x = i % Lv.nx, y = (i / Lv.nx) % Lv.ny, z = i / (Lv.nx * Lv.ny);
  const size_t f = (size_t)x * stride + (size_t)Fv.nx * ((size_t)y * stride + (size_t)Fv.ny * z * stride);
  const size_t N = Lv.N, NF = Fv.N;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const T v = Fv.d[k * NF + f];
    Lv.d[k * N + i] = v;
    Lv.base[k * N + i] = v;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) Lv.rot[k * N + i] = Fv.rot[k * NF + f];
}

template <typename T>
hipError_t launch_inject(const Dispatch<T>& D, const Dispatch<T>& F, int stride, hipStream_t s) {
  if (D.blocks <= 0) return hipSuccess;
  k_inject<T><<<D.blocks, kBlock, 0, s>>>(D, F, stride);
  return hipGetLastError();
}

// fine.d (+)= trilinear evaluation of (coarse.d - coarse.base) at the fine
// rest positions: fine node a sits at coarse coordinate a/2; its cell is
// clamped to the last coarse cell, so the last fine plane of an even-sized
// axis is linearly extrapolated (f = 1.5).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_prolong(Dispatch<T> D, Dispatch<T> C, int add) {
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& Fl = w.L;
  const int i = w.local * kBlock + threadIdx.x;
  if (i >= Fl.N) return;
  if (add && Fl.act && !Fl.act[i]) return;  // the increment reaches M only
  const LevelView<T> Cv = view_of(C, w.b);
  const int x = i % Fl.nx, y = (i / Fl.nx) % Fl.ny, z = i / (Fl.nx * Fl.ny);
  const int p[3] = {x, y, z};
  const int nc[3] = {Cv.nx, Cv.ny, Cv.nz};
  int cc[3];
  T f[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    int c = p[k] >> 1;
    if (c > nc[k] - 2) c = nc[k] - 2;
    cc[k] = c;
    f[k] = T(0.5) * T(p[k]) - T(c);
  }
  const size_t NC = Cv.N, NF = Fl.N;
  const T* __restrict__ cin = Cv.d;
  const T* __restrict__ cbase = Cv.base;
  T v[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const size_t m = (cc[0] + (k & 1)) +
                     (size_t)Cv.nx * ((cc[1] + ((k >> 1) & 1)) + (size_t)Cv.ny * (cc[2] + (k >> 2)));
    const T wk = corner_weight<T>(k, f[0], f[1], f[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T inc = cbase ? cin[a * NC + m] - cbase[a * NC + m] : cin[a * NC + m];
      v[a] += wk * inc;
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (add) Fl.d[a * NF + i] += v[a];
    else Fl.d[a * NF + i] = v[a];
  }
}

template <typename T>
hipError_t launch_prolong(const Dispatch<T>& Dfine, const Dispatch<T>& C, int add, hipStream_t s) {
  if (Dfine.blocks <= 0) return hipSuccess;
  k_prolong<T><<<Dfine.blocks, kBlock, 0, s>>>(Dfine, C, add);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_set_rest(Dispatch<T> D) {
  const Where<T> w = locate(D, blockIdx.x);
  const LevelView<T>& L = w.L;
  const int i = w.local * kBlock + threadIdx.x;
  if (i >= L.N) return;
  const size_t N = L.N;
#pragma unroll
  for (int k = 0; k < 3; ++k) L.d[k * N + i] = T(0);
#pragma unroll
  for (int k = 0; k < 9; ++k) L.rot[k * N + i] = (k % 4 == 0) ? T(1) : T(0);
}

template <typename T>
hipError_t launch_set_rest(const Dispatch<T>& D, hipStream_t s) {
  if (D.blocks <= 0) return hipSuccess;
  k_set_rest<T><<<D.blocks, kBlock, 0, s>>>(D);
  return hipGetLastError();
}

#define VD_INSTANTIATE_SOLVE(T)                                                                  \
  template hipError_t launch_stencil<T>(int, const Dispatch<T>&, const T*, T*, hipStream_t);    \
  template hipError_t launch_cg<T>(int, const Dispatch<T>&, hipStream_t, unsigned long long*);   \
  template hipError_t launch_cg_final<T>(int, const Dispatch<T>&, hipStream_t,                   \
                                          unsigned long long*);                                 \
  template hipError_t launch_energy<T>(const Dispatch<T>&, const Dispatch<T>&, int, hipStream_t); \
  template hipError_t launch_reset_counters<T>(const Dispatch<T>&, hipStream_t);                 \
  template hipError_t launch_cg_loop<T>(int, const Dispatch<T>&, hipStream_t,                    \
                                         unsigned long long*, int);                             \
  template hipError_t cg_loop_capacity<T>(int, bool, int*);                                      \
  template hipError_t launch_polar<T>(const Dispatch<T>&, hipStream_t);                          \
  template hipError_t launch_inject<T>(const Dispatch<T>&, const Dispatch<T>&, int, hipStream_t); \
  template hipError_t launch_prolong<T>(const Dispatch<T>&, const Dispatch<T>&, int, hipStream_t); \
  template hipError_t launch_set_rest<T>(const Dispatch<T>&, hipStream_t);

VD_INSTANTIATE_SOLVE(float)
VD_INSTANTIATE_SOLVE(double)

}  // namespace vd
