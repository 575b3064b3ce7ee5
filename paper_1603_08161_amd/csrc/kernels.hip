// HIP kernels of the lattice solver (gfx950).
//
// Unknowns are stored as displacements d_i = t_i - t_hat_i (float32 by
// default): the residuals of eqs. (2)-(4) are then differences of small
// numbers, which keeps float32 accurate even when the lattice sits far from
// the world origin.  Every node vector is SoA [3][N] in x-fastest node order.

#include <algorithm>

#include "vd_device.h"
#include "vd_kernels.h"

namespace vd {

namespace {

inline int blocks_for(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

__device__ __forceinline__ bool in_box(int x, int y, int z, int nx, int ny, int nz) {
  return x >= 0 && x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
}

// Unique (a <= b) corner pairs of a cell and the six components of a
// symmetric 3x3 block.
__constant__ unsigned char c_pair_a[36] = {0, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 2, 2, 2,
                                           2, 2, 2, 3, 3, 3, 3, 3, 4, 4, 4, 4, 5, 5, 5, 6, 6, 7};
__constant__ unsigned char c_pair_b[36] = {0, 1, 2, 3, 4, 5, 6, 7, 1, 2, 3, 4, 5, 6, 7, 2, 3, 4,
                                           5, 6, 7, 3, 4, 5, 6, 7, 4, 5, 6, 7, 5, 6, 7, 6, 7, 7};
__constant__ unsigned char c_comp_i[6] = {0, 0, 0, 1, 1, 2};
__constant__ unsigned char c_comp_j[6] = {0, 1, 2, 1, 2, 2};

// Workgroups of the cell cache per level: twice what is resident at once.
constexpr int kCellBlocks = 1536;

}  // namespace

// ===========================================================================
// constraint validation and per-level rows
// ===========================================================================

// Faults of dense sample or sparse pair i: 1 a value that is not finite or a
// negative weight, 2 a canonical point outside the coarsest level's node box.
// The values also go to st's arrays where they are not null.
__device__ __forceinline__ int sample_faults(const RawConstraints& c, const Staging& st, int i,
                                             int nx0, int ny0, int nz0, double h0, double ox,
                                             double oy, double oz) {
  int f = 0;
  const bool dense = i < c.n_dense;
  const size_t j = 3 * (size_t)(dense ? i : i - c.n_dense);
  const float* pc = (dense ? c.canon : c.sparse_canon) + j;
  const float* pt = (dense ? c.target : c.sparse_target) + j;
  const float x[3] = {pc[0], pc[1], pc[2]}, y[3] = {pt[0], pt[1], pt[2]};
  if (dense) {
    const float* pn = c.normal + j;
    const float n[3] = {pn[0], pn[1], pn[2]};
    const float w = c.weight ? c.weight[i] : 1.0f;
    if (!isfinite(n[0]) || !isfinite(n[1]) || !isfinite(n[2])) f |= 1;
    if (!isfinite(w) || w < 0.0f) f |= 1;
    if (st.normal)
      for (int k = 0; k < 3; ++k) st.normal[j + k] = n[k];
    if (st.weight && c.weight) st.weight[i] = w;
  }
  float* const sc = dense ? st.canon : st.sparse_canon;
  float* const sy = dense ? st.target : st.sparse_target;
  const double o[3] = {ox, oy, oz};
  const int n[3] = {nx0, ny0, nz0};
  for (int k = 0; k < 3; ++k) {
    if (sc) sc[j + k] = x[k];
    if (sy) sy[j + k] = y[k];
    if (!isfinite(x[k]) || !isfinite(y[k])) f |= 1;
    const double u = ((double)x[k] - o[k]) / h0;
    if (!(u >= 0.0 && u <= (double)(n[k] - 1))) f |= 2;
  }
  return f;
}

__global__ __launch_bounds__(kBlock) void k_validate(RawConstraints c, int nx0, int ny0, int nz0,
                                                     double h0, double ox, double oy, double oz,
                                                     int* flags) {
  const int total = c.n_dense + c.n_sparse;
  int f = 0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < total; i += gridDim.x * kBlock)
    f |= sample_faults(c, Staging{}, i, nx0, ny0, nz0, h0, ox, oy, oz);
  if (f) atomicOr(flags, f);
}

// Copies a frame's inputs and checks them on the way, with the faults written
// to host memory: one launch in place of six copies, a cleared flag, the check
// and a copy of the flag, whose launches cost more than the bytes (3.5 MB at
// 87 000 samples).
__global__ __launch_bounds__(kBlock) void k_stage(RawConstraints c, Staging st, int nx0, int ny0,
                                                  int nz0, double h0, double ox, double oy,
                                                  double oz, int* host_flags) {
  const int total = c.n_dense + c.n_sparse;
  int f = 0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < total; i += gridDim.x * kBlock)
    f |= sample_faults(c, st, i, nx0, ny0, nz0, h0, ox, oy, oz);
  // (plain stores of the same value: atomics may not reach host memory)
  if (f & 1) __hip_atomic_store(host_flags, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (f & 2) __hip_atomic_store(host_flags + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_validate(const RawConstraints& c, int nx0, int ny0, int nz0, double h0,
                           const double* o, int* flags, hipStream_t s) {
  const int total = c.n_dense + c.n_sparse;
  if (total == 0) return hipSuccess;
  const int grid = std::min(blocks_for(total), 4096);
  k_validate<<<grid, kBlock, 0, s>>>(c, nx0, ny0, nz0, h0, o[0], o[1], o[2], flags);
  return hipGetLastError();
}

hipError_t launch_stage(const RawConstraints& c, const Staging& st, int nx0, int ny0, int nz0,
                        double h0, const double* o, int* host_flags, hipStream_t s) {
  const int total = c.n_dense + c.n_sparse;
  if (total == 0) return hipSuccess;
  const int grid = std::min(blocks_for(total), 4096);
  k_stage<<<grid, kBlock, 0, s>>>(c, st, nx0, ny0, nz0, h0, o[0], o[1], o[2], host_flags);
  return hipGetLastError();
}

// One row per dense correspondence (eq. (2)) and three per sparse pair
// (eq. (3): a point-to-point term is the sum of three axis-aligned
// point-to-plane terms).  Row value: sn . sum_k alpha_k d_k - rho, with
// sn = sqrt(w) * normal and rho = sn . (target - canonical).  With
// `structure` also the cells' histogram of the first sort digit (block b's
// rows are those of the sort's block b) and the cleared cell map.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_rows(RawConstraints c, BuildLevels<T> B, SortLevels S,
                                                 double ox, double oy, double oz, double wd,
                                                 double ws, int structure) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  const LevelView<T>& L = V.L;
  const RowView<T>& R = V.R;
  const int rows = R.rows;
  __shared__ int h[kMaxBuckets];
  const int buckets = 1 << S.level[blockIdx.y].digit_bits;
  const bool counts = structure && (int)blockIdx.x * kRowTile < rows;
  if (structure) {
    for (int k = blockIdx.x * kBlock + threadIdx.x; k < V.ncell; k += gridDim.x * kBlock)
      V.cell_map[k] = -1;
    if (counts) {
      for (int k = threadIdx.x; k < buckets; k += kBlock) h[k] = 0;
      __syncthreads();
    }
  }
  for (int j = threadIdx.x; j < kRowTile; j += kBlock) {
    const int i = blockIdx.x * kRowTile + j;
    if (i >= rows) break;
    double x[3], sn[3], rho;
    if (i < c.n_dense) {
      const size_t b = 3 * (size_t)i;
      double n[3], tp[3];
      for (int k = 0; k < 3; ++k) {
        x[k] = c.canon[b + k];
        tp[k] = c.target[b + k];
        n[k] = c.normal[b + k];
      }
      const double ln = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
      double w = c.weight ? (double)c.weight[i] : 1.0;
      if (ln > 0.0) {
        for (int k = 0; k < 3; ++k) n[k] /= ln;
      } else {
        w = 0.0;
        n[0] = n[1] = n[2] = 0.0;
      }
      const double s = sqrt(wd * w);
      rho = 0.0;
      for (int k = 0; k < 3; ++k) {
        sn[k] = s * n[k];
        rho += sn[k] * (tp[k] - x[k]);
      }
    } else {
      const int j = i - c.n_dense;
      const int sidx = j / 3, axis = j % 3;
      const size_t b = 3 * (size_t)sidx;
      for (int k = 0; k < 3; ++k) x[k] = c.sparse_canon[b + k];
      const double s = sqrt(ws);
      sn[0] = sn[1] = sn[2] = 0.0;
      sn[axis] = s;
      rho = s * ((double)c.sparse_target[b + axis] - x[axis]);
    }
    const double o[3] = {ox, oy, oz};
    const int n[3] = {L.nx, L.ny, L.nz};
    int cc[3];
    for (int k = 0; k < 3; ++k) {
      const double u = (x[k] - o[k]) / (double)L.h;
      double fl = floor(u);
      if (fl < 0.0) fl = 0.0;
      if (fl > (double)(n[k] - 2)) fl = (double)(n[k] - 2);
      cc[k] = (int)fl;
      R.f[(size_t)k * rows + i] = (T)(u - fl);
      R.sn[(size_t)k * rows + i] = (T)sn[k];
    }
    const int cell = cc[0] + (L.nx - 1) * (cc[1] + (L.ny - 1) * cc[2]);
    R.cell[i] = cell;
    R.rho[i] = (T)rho;
    if (structure) atomicAdd(&h[cell & (buckets - 1)], 1);
  }
  if (counts) {
    __syncthreads();
    int* hist = S.level[blockIdx.y].hist + (size_t)blockIdx.x * buckets;
    for (int k = threadIdx.x; k < buckets; k += kBlock) hist[k] = h[k];
  }
}

// heads[b] = rows of block b of the sorted rows that are the first of a cell.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_heads(BuildLevels<T> B) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  const unsigned* __restrict__ keys = V.skeys;
  int heads = 0;
  for (int j = threadIdx.x; j < kRowTile; j += kBlock) {
    const int i = blockIdx.x * kRowTile + j;
    heads += i < V.R.rows && (i == 0 || keys[i] != keys[i - 1]);
  }
  int total;
  (void)block_exclusive<kBlock / kWave>(heads, &total);
  if (threadIdx.x == 0) V.heads[blockIdx.x] = total;
}

// Sum of counts[0 .. b) (all threads get it): a block adds up what the blocks
// before it counted, 4 bytes each, instead of a scan of three launches; above
// kDirectBlocks the counts are scanned first.
constexpr int kDirectBlocks = 4096;
__device__ __forceinline__ int blocks_before(const int* counts, int b, bool scanned) {
  if (scanned) return counts[b];
  int v = 0, total;
  for (int k = threadIdx.x; k < b; k += kBlock) v += counts[k];
  (void)block_exclusive<kBlock / kWave>(v, &total);
  return total;
}

// Active cells = distinct keys of the sorted rows, in their order.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_segments(BuildLevels<T> B, int scanned) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  const RowView<T>& R = V.R;
  const unsigned* __restrict__ keys = V.skeys;
  const int n = R.rows;
  if (n == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      V.L.sc->n_active = 0;
      R.seg_start[0] = 0;
    }
    return;
  }
  constexpr int PER = kRowTile / kBlock;
  const int i0 = blockIdx.x * kRowTile + threadIdx.x * PER;
  unsigned key[PER + 1];
  key[0] = i0 > 0 && i0 <= n ? keys[i0 - 1] : 0u;
  int heads = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    key[k + 1] = i0 + k < n ? keys[i0 + k] : 0u;
    heads += i0 + k < n && (i0 + k == 0 || key[k + 1] != key[k]);
  }
  int total;
  int a = blocks_before(V.heads, blockIdx.x, scanned) +
          block_exclusive<kBlock / kWave>(heads, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = i0 + k;
    if (i >= n) break;
    if (i == 0 || key[k + 1] != key[k]) {
      R.seg_start[a] = i;
      R.active_cell[a] = (int)key[k + 1];
      V.cell_map[key[k + 1]] = a;
      ++a;
    }
    if (i == n - 1) {
      R.seg_start[a] = n;
      V.L.sc->n_active = a;
    }
  }
}

// Nodes of block b (kBlock nodes) that are a corner of an active cell.
template <typename T>
__device__ __forceinline__ void count_nodes(const BuildLevel<T>& V, int b) {
  const LevelView<T>& L = V.L;
  if (b * kBlock >= L.N) return;
  const int i = b * kBlock + threadIdx.x;
  int f = 0;
  if (i < L.N) {
    const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
    const int cnx = L.nx - 1, cny = L.ny - 1, cnz = L.nz - 1;
    for (int a = 0; a < 8; ++a) {
      const int cx = x - (a & 1), cy = y - ((a >> 1) & 1), cz = z - (a >> 2);
      if (in_box(cx, cy, cz, cnx, cny, cnz) && V.cell_map[cx + cnx * (cy + cny * cz)] >= 0) f = 1;
    }
    if (V.touched) V.touched[i] = (unsigned char)f;
  }
  const int total = __syncthreads_count(f);
  if (threadIdx.x == 0) V.nodes[b] = total;
}

// B^T B and B^T b cached per active cell (the per-voxel cache of Sec. 7.1).
// Block for corners (a, b): sum over the cell's rows of
// alpha_a alpha_b sn sn^T (symmetric 3x3); rhs block of corner a:
// sum alpha_a sn rho.  One workgroup per cell; rows are staged through LDS in
// chunks of 256 as the float64 products u[3a + i] = alpha_a sn_i and rho (a
// product of two floats is exact in float64, so u_ai u_bj is the same number
// as (alpha_a alpha_b)(sn_i sn_j)); each thread owns one output entry and
// accumulates it in float64 over the rows in sorted order (deterministic).
// While a chunk is accumulated, the next chunk's rows and the row indices of
// the one after are already being loaded (cells of coarse levels hold
// thousands of rows).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_build_cells(BuildLevels<T> B, int cell_blocks) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  if ((int)blockIdx.x >= cell_blocks) {
    count_nodes(V, blockIdx.x - cell_blocks);
    return;
  }
  const RowView<T>& R = V.R;
  T* const K = V.K;
  constexpr int P = kBlock + 1;  // padded rows: conflict-free column reads
  __shared__ double s_u[25 * P];  // 24 products alpha_a sn_i, then rho
  const int n_active = V.L.sc->n_active;
  const int rows = R.rows;
  const int j = threadIdx.x;
  int ka = 0, kb = 0, ca = 0, ci = 0, kind = 2;
  if (j < 216) {
    const int p = j / 6, comp = j % 6;
    ca = c_pair_a[p];
    ci = c_comp_i[comp];
    ka = ca * 3 + ci;
    kb = c_pair_b[p] * 3 + c_comp_j[comp];
    kind = 0;
  } else if (j < 240) {
    ca = (j - 216) / 3;
    ci = (j - 216) % 3;
    ka = ca * 3 + ci;
    kb = 24;
    kind = 1;
  }
  for (int a = blockIdx.x; a < n_active; a += cell_blocks) {
    const int s0 = R.seg_start[a], s1 = R.seg_start[a + 1];
    // row of this thread in the chunk being staged (f, sn, rho) and the row
    // index of the following chunk
    int row_next = (s0 + kBlock + j < s1) ? R.sorted[s0 + kBlock + j] : 0;
    T f3[3] = {T(0), T(0), T(0)}, n3[3] = {T(0), T(0), T(0)}, rho = T(0);
    if (s0 + j < s1) {
      const int row = R.sorted[s0 + j];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        f3[k] = R.f[(size_t)k * rows + row];
        n3[k] = R.sn[(size_t)k * rows + row];
      }
      rho = R.rho[row];
    }
    double acc = 0.0;
    for (int base = s0; base < s1; base += kBlock) {
      const int cnt = min(kBlock, s1 - base);
      __syncthreads();  // the previous chunk's reads are done
      if (j < cnt) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const double w = (double)corner_weight<T>(c, f3[0], f3[1], f3[2]);
#pragma unroll
          for (int k = 0; k < 3; ++k) s_u[(c * 3 + k) * P + j] = w * (double)n3[k];
        }
        s_u[24 * P + j] = (double)rho;
      }
      __syncthreads();
      // next chunk's rows (index loaded one chunk ago), and the index after
      if (base + kBlock + j < s1) {
        const int row = row_next;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          f3[k] = R.f[(size_t)k * rows + row];
          n3[k] = R.sn[(size_t)k * rows + row];
        }
        rho = R.rho[row];
      }
      row_next = (base + 2 * kBlock + j < s1) ? R.sorted[base + 2 * kBlock + j] : 0;
      // four independent accumulators keep several LDS reads in flight
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      if (kind < 2) {
        const double* __restrict__ ua = s_u + ka * P;
        const double* __restrict__ ub = s_u + kb * P;
        int q = 0;
        // unrolled so that 16 rows' LDS reads are in flight at once (one wave
        // per SIMD: nothing else hides their latency); each accumulator still
        // adds its rows in row order
#pragma unroll 4
        for (; q + 4 <= cnt; q += 4) {
          a0 += ua[q] * ub[q];
          a1 += ua[q + 1] * ub[q + 1];
          a2 += ua[q + 2] * ub[q + 2];
          a3 += ua[q + 3] * ub[q + 3];
        }
        for (; q < cnt; ++q) a0 += ua[q] * ub[q];
      }
      acc += (a0 + a1) + (a2 + a3);
    }
    if (kind == 0) {
      const int comp = j % 6, cb = c_pair_b[j / 6];
      K[((size_t)a * 64 + ca * 8 + cb) * 6 + comp] = (T)acc;
      if (ca != cb) K[((size_t)a * 64 + cb * 8 + ca) * 6 + comp] = (T)acc;
    } else if (kind == 1) {
      R.bcell[((size_t)a * 8 + ca) * 3 + ci] = (T)acc;
    }
  }
}

// Per node: the data part of row i of A as a 27-point block stencil,
// A27[delta] = sum over adjacent active cells c (i = corner a of c, neighbour
// = corner b, delta = b - a) of K_c[a][b]; stored at the node's compact slot
// as a row A27r[slot][kA27Row]: three parts by dz (one part is one lane's
// share of the node in the stencil and CG kernels), interleaved by 16-byte
// chunks.  Also the
// Jacobi diagonal 2 w_r |N_i| + diag(A27[0]), and the data right-hand side
// b_i gathered from the cells.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_assemble_nodes(BuildLevels<T> B, int scanned) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  const LevelView<T>& L = V.L;
  const RowView<T>& R = V.R;
  if ((int)blockIdx.x * kBlock >= L.N) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // read by the energy kernel
    L.sc->rows = R.rows;
    L.sc->n_dense = R.n_dense;
  }
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const int before = blocks_before(V.nodes, blockIdx.x, scanned);
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const int nb = (x > 0) + (x < L.nx - 1) + (y > 0) + (y < L.ny - 1) + (z > 0) + (z < L.nz - 1);
  const int cnx = L.nx - 1, cny = L.ny - 1, cnz = L.nz - 1;
  int cells[8], has = 0;
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int cx = x - (a & 1), cy = y - ((a >> 1) & 1), cz = z - (a >> 2);
    cells[a] = i < L.N && in_box(cx, cy, cz, cnx, cny, cnz)
                   ? V.cell_map[cx + cnx * (cy + cny * cz)] : -1;
    has |= cells[a] >= 0;
  }
  int total;
  const int rank = block_exclusive<kBlock / kWave>(has, &total);
  if (i >= L.N) return;
  const int slot = has ? before + rank : -1;
  V.node_slot[i] = slot;
  T dg[3] = {T(0), T(0), T(0)};
  T b[3] = {T(0), T(0), T(0)};
  if (slot >= 0) {
    // each adjacent cell's block row K_c[a][*] is read once and scattered
    // into the 27 offsets delta = b - a (summed over a in ascending order)
    T acc[27][6];
#pragma unroll
    for (int dl = 0; dl < 27; ++dl)
#pragma unroll
      for (int k = 0; k < 6; ++k) acc[dl][k] = T(0);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      if (cells[a] < 0) continue;
      const T* __restrict__ row = V.K + ((size_t)cells[a] * 64 + a * 8) * 6;
#pragma unroll
      for (int bb = 0; bb < 8; ++bb) {
        const int dl = ((bb & 1) - (a & 1) + 1) + 3 * ((((bb >> 1) & 1) - ((a >> 1) & 1) + 1) +
                                                      3 * ((bb >> 2) - (a >> 2) + 1));
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[dl][k] += row[bb * 6 + k];
      }
      const T* bc = R.bcell + ((size_t)cells[a] * 8 + a) * 3;
      b[0] += bc[0];
      b[1] += bc[1];
      b[2] += bc[2];
    }
    // entry q of part m (block (dx, dy) of dz = m - 1, zero padded) at chunk
    // 3 (q / CW) + m, position q % CW
    constexpr int CW = 16 / (int)sizeof(T);
    T* __restrict__ row_out = V.A27r + (size_t)slot * kA27Row;
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int q = 0; q < kA27Part; ++q)
        row_out[(3 * (q / CW) + m) * CW + q % CW] = q < 54 ? acc[m * 9 + q / 6][q % 6] : T(0);
    dg[0] = acc[13][0];
    dg[1] = acc[13][3];
    dg[2] = acc[13][5];
  }
  const size_t N = L.N;
  T arap = T(2) * L.wr * T(nb);
  bool in_set = true;
  if (L.act) {
    // restricted to M: only the edges inside M count, so the ARAP diagonal
    // is 2 w_r |N_i and M|; points outside M are not unknowns (D^-1 = 0)
    in_set = L.act[i] != 0;
    int w = 0;
    const size_t st[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
    const int pos[3] = {x, y, z};
    const int lim[3] = {L.nx, L.ny, L.nz};
    for (int ax = 0; ax < 3; ++ax) {
      if (pos[ax] > 0) w += L.act[i - st[ax]];
      if (pos[ax] < lim[ax] - 1) w += L.act[i + st[ax]];
    }
    arap = T(2) * L.wr * T(w);
  }
  for (int k = 0; k < 3; ++k) {
    const T dk = arap + dg[k];
    L.dinv[k * N + i] = (in_set && dk > T(0)) ? T(1) / dk : T(0);
    L.bnode[k * N + i] = b[k];
  }
}

// The optimised set M: the isosurface points (corners of the cells holding
// samples) and their one-ring.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_dilate(BuildLevels<T> B) {
  const BuildLevel<T>& V = B.level[blockIdx.y];
  const LevelView<T>& L = V.L;
  const unsigned char* flags = V.touched;
  if (!V.act) return;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N) return;
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const size_t st[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
  const int pos[3] = {x, y, z};
  const int lim[3] = {L.nx, L.ny, L.nz};
  int f = flags[i];
  for (int ax = 0; ax < 3; ++ax) {
    if (pos[ax] > 0) f |= flags[i - st[ax]];
    if (pos[ax] < lim[ax] - 1) f |= flags[i + st[ax]];
  }
  V.act[i] = f ? 1 : 0;
}

int build_row_blocks(int rows) { return rows > 0 ? (rows + kRowTile - 1) / kRowTile : 1; }
int build_node_blocks(int n) { return blocks_for(n); }

template <typename T>
hipError_t launch_build(const RawConstraints& c, const BuildLevels<T>& B, const SortLevels& S,
                        const double* o, double wd, double ws, bool structure, void* temp,
                        size_t temp_bytes, hipStream_t s) {
  const int rows = B.level[0].R.rows, nb = build_row_blocks(rows);
  int cells = 0, cap = 0, nodes = 0, act = 0;
  for (int l = 0; l < B.n; ++l) {
    const BuildLevel<T>& V = B.level[l];
    cells = V.ncell > cells ? V.ncell : cells;
    cap = V.cap_cells > cap ? V.cap_cells : cap;
    nodes = V.L.N > nodes ? V.L.N : nodes;
    act |= V.act != nullptr;
  }
  // scans of counts too many to be added up by every block
  auto scan = [&](int* counts, int n) {
    return exclusive_scan(temp, temp_bytes, counts, counts, n, s);
  };
  hipError_t e = hipSuccess;
  if (rows > 0 || structure) {
    int gx = nb;  // enough workgroups to clear the cell maps
    if (structure && gx < 256) gx = std::min(256, std::max(gx, (cells + 4095) / 4096));
    k_rows<T><<<dim3(gx, B.n), kBlock, 0, s>>>(c, B, S, o[0], o[1], o[2], wd, ws, structure);
  }
  if (structure) {
    if ((e = sort_levels(S, s)) != hipSuccess) return e;
    k_heads<T><<<dim3(nb, B.n), kBlock, 0, s>>>(B);
    if (nb > kDirectBlocks)
      for (int l = 0; l < B.n; ++l)
        if ((e = scan(B.level[l].heads, nb)) != hipSuccess) return e;
    k_segments<T><<<dim3(nb, B.n), kBlock, 0, s>>>(B, nb > kDirectBlocks);
  }
  const int cb = std::min(cap, kCellBlocks), gn = blocks_for(nodes);
  k_build_cells<T><<<dim3(cb + gn, B.n), kBlock, 0, s>>>(B, cb);
  if (act) k_dilate<T><<<dim3(gn, B.n), kBlock, 0, s>>>(B);
  const bool scanned = gn > kDirectBlocks;
  if (scanned)
    for (int l = 0; l < B.n; ++l)
      if ((e = scan(B.level[l].nodes, blocks_for(B.level[l].L.N))) != hipSuccess) return e;
  k_assemble_nodes<T><<<dim3(gn, B.n), kBlock, 0, s>>>(B, scanned);
  return hipGetLastError();
}

// Grid growth, one layer (Sec. 8: points that join M for the first time are
// initialised by extrapolating the deformation field).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_grow_layer(LevelView<T> L, const unsigned char* act,
                                                       const unsigned char* known, T* tmp_d,
                                                       T* tmp_r, unsigned char* fresh,
                                                       int* count) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N) return;
  fresh[i] = 0;
  if (!act[i] || known[i]) return;
  const size_t N = L.N;
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const size_t st[3] = {1, (size_t)L.nx, (size_t)L.nx * L.ny};
  const int pos[3] = {x, y, z};
  const int lim[3] = {L.nx, L.ny, L.nz};
  double acc[3] = {0.0, 0.0, 0.0};
  int cnt = 0;
  long first = -1;
  for (int ax = 0; ax < 3; ++ax) {
    for (int sgn = -1; sgn <= 1; sgn += 2) {
      const int pj = pos[ax] + sgn;
      if (pj < 0 || pj >= lim[ax]) continue;
      const size_t j = sgn > 0 ? i + st[ax] : i - st[ax];
      if (!known[j]) continue;
      for (int k = 0; k < 3; ++k) acc[k] += (double)L.d[k * N + j];
      ++cnt;
      if (first < 0) first = (long)j;
    }
  }
  if (!cnt) return;
  for (int k = 0; k < 3; ++k) tmp_d[k * N + i] = (T)(acc[k] / cnt);
  for (int k = 0; k < 9; ++k) tmp_r[k * N + i] = L.rot[k * N + (size_t)first];
  fresh[i] = 1;
  atomicAdd(count, 1);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_grow_commit(LevelView<T> L, const T* tmp_d,
                                                        const T* tmp_r, unsigned char* fresh,
                                                        unsigned char* known) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N || !fresh[i]) return;
  const size_t N = L.N;
  for (int k = 0; k < 3; ++k) L.d[k * N + i] = tmp_d[k * N + i];
  for (int k = 0; k < 9; ++k) L.rot[k * N + i] = tmp_r[k * N + i];
  known[i] = 1;
  fresh[i] = 0;
}

template <typename T>
hipError_t launch_grow_layer(const LevelView<T>& L, const unsigned char* act,
                             const unsigned char* known, T* tmp_d, T* tmp_r,
                             unsigned char* fresh, int* count, hipStream_t s) {
  k_grow_layer<T><<<blocks_for(L.N), kBlock, 0, s>>>(L, act, known, tmp_d, tmp_r, fresh, count);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_grow_commit(const LevelView<T>& L, const T* tmp_d, const T* tmp_r,
                              unsigned char* fresh, unsigned char* known, hipStream_t s) {
  k_grow_commit<T><<<blocks_for(L.N), kBlock, 0, s>>>(L, tmp_d, tmp_r, fresh, known);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_check_finite(const float* v, int64_t n, int* flags) {
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock)
    if (!isfinite(v[i])) bad = 1;
  if (bad) atomicOr(flags, 1);
}

hipError_t launch_check_finite(const float* v, int64_t n, int* flags, hipStream_t s) {
  if (n == 0) return hipSuccess;
  int64_t g = (n + kBlock - 1) / kBlock;
  if (g > 4096) g = 4096;
  k_check_finite<<<(unsigned)g, kBlock, 0, s>>>(v, n, flags);
  return hipGetLastError();
}

// ===========================================================================
// batched rotation fit of raw matrices (test entry point)
// ===========================================================================

template <typename T>
__global__ __launch_bounds__(kBlock) void k_fit_batch(const float* M, const float* Rp, float* R,
                                                      int* keep, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  T m[9], rp[9], r[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    m[k] = (T)M[9 * i + k];
    rp[k] = Rp ? (T)Rp[9 * i + k] : ((k % 4 == 0) ? T(1) : T(0));
  }
  const int code = fit_or_keep<T>(m, rp, r);
#pragma unroll
  for (int k = 0; k < 9; ++k) R[9 * i + k] = (float)r[k];
  if (keep) keep[i] = code;
}

template <typename T>
hipError_t launch_fit_batch(const float* M, const float* R_prev, float* R, int* keep, int64_t n,
                            hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_fit_batch<T><<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(M, R_prev, R, keep, n);
  return hipGetLastError();
}

// ===========================================================================
// state helpers
// ===========================================================================

// dir 0: export positions t = t_hat + d (AoS float) and rotations (row-major
// AoS float); dir 1: import them (non-finite input sets flags bit 1).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_state_io(LevelView<T> L, double ox, double oy,
                                                     double oz, float* pos, float* rot,
                                                     const float* pos_in, const float* rot_in,
                                                     int dir, int* flags) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N) return;
  const size_t N = L.N;
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const double rest[3] = {ox + (double)L.h * x, oy + (double)L.h * y, oz + (double)L.h * z};
  if (dir == 0) {
    if (pos) {
#pragma unroll
      for (int k = 0; k < 3; ++k) pos[3 * (size_t)i + k] = (float)(rest[k] + (double)L.d[k * N + i]);
    }
    if (rot) {
#pragma unroll
      for (int k = 0; k < 9; ++k) rot[9 * (size_t)i + k] = (float)L.rot[k * N + i];
    }
  } else {
    int bad = 0;
    if (pos_in) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float v = pos_in[3 * (size_t)i + k];
        if (!isfinite(v)) bad = 1;
        L.d[k * N + i] = (T)((double)v - rest[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      float v = rot_in ? rot_in[9 * (size_t)i + k] : ((k % 4 == 0) ? 1.0f : 0.0f);
      if (!isfinite(v)) bad = 1;
      L.rot[k * N + i] = (T)v;
    }
    if (bad) atomicOr(flags, 1);
  }
}

template <typename T>
hipError_t launch_state_io(const LevelView<T>& L, const double* o, float* pos, float* rot,
                           const float* pos_in, const float* rot_in, int dir, int* flags,
                           hipStream_t s) {
  k_state_io<T><<<blocks_for(L.N), kBlock, 0, s>>>(L, o[0], o[1], o[2], pos, rot, pos_in, rot_in,
                                                    dir, flags);
  return hipGetLastError();
}

// Finest state as float64 AoS: positions t_hat + d, rotations row-major.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_state_out64(LevelView<T> L, double ox, double oy,
                                                        double oz, double* pos, double* rot) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N) return;
  const size_t N = L.N;
  const int x = i % L.nx, y = (i / L.nx) % L.ny, z = i / (L.nx * L.ny);
  const double rest[3] = {ox + (double)L.h * x, oy + (double)L.h * y, oz + (double)L.h * z};
  if (pos) {
#pragma unroll
    for (int k = 0; k < 3; ++k) pos[3 * (size_t)i + k] = rest[k] + (double)L.d[k * N + i];
  }
  if (rot) {
#pragma unroll
    for (int k = 0; k < 9; ++k) rot[9 * (size_t)i + k] = (double)L.rot[k * N + i];
  }
}

template <typename T>
hipError_t launch_state_out64(const LevelView<T>& L, const double* o, double* pos, double* rot,
                              hipStream_t s) {
  k_state_out64<T><<<blocks_for(L.N), kBlock, 0, s>>>(L, o[0], o[1], o[2], pos, rot);
  return hipGetLastError();
}

// AoS float xyz <-> SoA T (used by the test entry points)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_add_delta(T* d, const float* delta, T h, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) d[i] += h * (T)delta[i];
}

template <typename T>
hipError_t launch_add_delta(T* d, const float* delta, double h, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_add_delta<T><<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(d, delta, (T)h, n);
  return hipGetLastError();
}

// Exact step of a warm start along its predicted direction v (not in the
// paper): with the rotations fixed E is quadratic in the displacement,
// E(d + b v) = E(d) + 2 b g.v + b^2 v.Av with g = J^T r and A = J^T J
// (Sec. 7.1), smallest at b = -g.v / v.Av.  k_warm_dots writes the block
// partials of g.v and v.Av in float64; k_warm_step re-reduces them in every
// block in the same order and applies d += b v (b = 0 when v.Av <= 0).
constexpr int kWarmDotBlocks = 1024;  // partial pairs at most (the caller's buffer)

template <typename T>
__global__ __launch_bounds__(kBlock) void k_warm_dots(const T* __restrict__ g,
                                                      const float* __restrict__ v,
                                                      const T* __restrict__ av, int64_t n,
                                                      double* part) {
  double acc[2] = {0.0, 0.0};
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * kBlock) {
    const double vk = (double)v[k];
    acc[0] += (double)g[k] * vk;
    acc[1] += (double)av[k] * vk;
  }
  write_block_partials<2>(acc, part, gridDim.x);
}

// act (null: every point): with the optimised set M only its points move.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_warm_step(T* d, const float* __restrict__ v,
                                                      int64_t n, const double* part,
                                                      int nblocks,
                                                      const unsigned char* __restrict__ act,
                                                      int64_t N) {
  double s[2];
  sum_partials_k<2>(part, nblocks, s);
  const double b = s[1] > 0.0 ? -s[0] / s[1] : 0.0;
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * kBlock)
    if (!act || act[k % N]) d[k] = (T)((double)d[k] + b * (double)v[k]);
}

// d += h delta on the points of the optimised set M only.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_add_delta_in(T* d, const float* __restrict__ delta,
                                                         T h, int64_t n,
                                                         const unsigned char* __restrict__ act,
                                                         int64_t N) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n && act[i % N]) d[i] += h * (T)delta[i];
}

template <typename T>
hipError_t launch_add_delta_in(T* d, const float* delta, double h, int64_t n,
                               const unsigned char* act, int64_t N, hipStream_t s) {
  if (!act) return launch_add_delta<T>(d, delta, h, n, s);
  if (n == 0) return hipSuccess;
  k_add_delta_in<T><<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(d, delta, (T)h, n,
                                                                            act, N);
  return hipGetLastError();
}

// The direction as T (the A p pass reads T) and the step; `part` holds
// 2 * kWarmDotBlocks doubles.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_to_type(const float* __restrict__ in, T* out,
                                                    int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) out[i] = (T)in[i];
}

template <typename T>
hipError_t launch_to_type(const float* in, T* out, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_to_type<T><<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(in, out, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_warm_step(T* d, const T* g, const float* v, const T* av, int64_t n,
                            double* part, const unsigned char* act, int64_t N, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t want = (n + kBlock - 1) / kBlock;
  const int nb = (int)(want < kWarmDotBlocks ? want : kWarmDotBlocks);
  k_warm_dots<T><<<nb, kBlock, 0, s>>>(g, v, av, n, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_warm_step<T><<<nb, kBlock, 0, s>>>(d, v, n, part, nb, act, N);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_convert(const float* in, T* out, int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) out[(size_t)k * n + i] = (T)in[3 * (size_t)i + k];
}
template <typename T>
__global__ __launch_bounds__(kBlock) void k_convert_back(const T* in, float* out, int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) out[3 * (size_t)i + k] = (float)in[(size_t)k * n + i];
}
template <typename T>
hipError_t launch_convert(const float* in, T* out, int n, hipStream_t s) {
  k_convert<T><<<blocks_for(n), kBlock, 0, s>>>(in, out, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_convert_back(const T* in, float* out, int n, hipStream_t s) {
  k_convert_back<T><<<blocks_for(n), kBlock, 0, s>>>(in, out, n);
  return hipGetLastError();
}

// ---- explicit instantiations -----------------------------------------------
#define VD_INSTANTIATE(T)                                                                        \
  template hipError_t launch_build<T>(const RawConstraints&, const BuildLevels<T>&,              \
                                      const SortLevels&, const double*, double, double, bool,   \
                                      void*, size_t, hipStream_t);                              \
  template hipError_t launch_grow_layer<T>(const LevelView<T>&, const unsigned char*,           \
                                           const unsigned char*, T*, T*, unsigned char*, int*,  \
                                           hipStream_t);                                         \
  template hipError_t launch_grow_commit<T>(const LevelView<T>&, const T*, const T*,            \
                                            unsigned char*, unsigned char*, hipStream_t);       \
  template hipError_t launch_state_io<T>(const LevelView<T>&, const double*, float*, float*,    \
                                         const float*, const float*, int, int*, hipStream_t);   \
  template hipError_t launch_state_out64<T>(const LevelView<T>&, const double*, double*,        \
                                            double*, hipStream_t);                              \
  template hipError_t launch_convert<T>(const float*, T*, int, hipStream_t);                    \
  template hipError_t launch_add_delta<T>(T*, const float*, double, int64_t, hipStream_t);      \
  template hipError_t launch_to_type<T>(const float*, T*, int64_t, hipStream_t);                \
  template hipError_t launch_warm_step<T>(T*, const T*, const float*, const T*, int64_t,        \
                                          double*, const unsigned char*, int64_t, hipStream_t); \
  template hipError_t launch_add_delta_in<T>(T*, const float*, double, int64_t,                 \
                                             const unsigned char*, int64_t, hipStream_t);       \
  template hipError_t launch_convert_back<T>(const T*, float*, int, hipStream_t);               \
  template hipError_t launch_fit_batch<T>(const float*, const float*, float*, int*, int64_t,    \
                                          hipStream_t);

VD_INSTANTIATE(float)
VD_INSTANTIATE(double)

}  // namespace vd
