// Stable key/value sort and integer exclusive prefix sums on the device: the
// binning of constraint rows by lattice cell (the rows of a cell become one
// contiguous segment, Sec. 7.1's per-cell B^T B blocks), the slots of the
// nodes that carry data blocks, and the output offsets of marching cubes.
//
// Sort: least-significant-digit radix sort over digits of up to 10 bits (two
// passes up to 2^20 cells).  Each pass counts the digits of every block of
// 1024 rows, turns the counts of each digit into running counts over the
// blocks, and scatters: a block scans the digits' totals for each digit's
// first output position.  Inside a block the rows form 16 chunks of 64, one
// per wave at a time; the lanes of a chunk find the lanes holding the same
// digit with one ballot per digit bit, which gives each row its rank among
// the equal digits before it in the chunk, and a per-digit prefix over the
// chunks orders the chunks.  Every row thus keeps the input order among equal
// digits, so each pass is stable and the sort orders by key with ties in
// input order.  One launch of a step covers the sorts of several lattice
// levels: these sorts are bound by their launches (three levels of 30k rows:
// 40 launches of 2 .. 6 us each with one level and 8-bit digits at a time,
// 5 with all levels and the first count in the kernel that writes the keys).
//
// Scan: block sums of 1024 elements, a one-workgroup exclusive scan of the
// block sums, then each block's own exclusive scan offset by its sum.
//
// Integer arithmetic only: both are exact, and the results do not depend on
// the order in which the hardware schedules the workgroups.
#include <algorithm>

#include "vd_device.h"
#include "vd_kernels.h"

namespace vd {

namespace {

constexpr int kThreads = 256;                 // 4 waves
constexpr int kWaves = kThreads / kWave;
constexpr int kSortTile = 1024;               // rows per block and pass
constexpr int kChunks = kSortTile / kWave;    // 16 chunks of 64 rows
constexpr int kChunksPerWave = kChunks / kWaves;
constexpr int kScanTile = 1024;               // elements per scan block
constexpr int kPerThread = kScanTile / kThreads;
static_assert(kSortTile == kRowTile, "the first pass is counted by the rows' kernel");

inline int ceil_div(int64_t n, int d) { return (int)((n + d - 1) / d); }
inline size_t aligned(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// sums[b] = sum of in[b * kScanTile .. (b + 1) * kScanTile) (within n).
__global__ __launch_bounds__(kThreads) void k_scan_block_sums(const int* __restrict__ in,
                                                              int64_t n, int* __restrict__ sums) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
  int v = 0;
#pragma unroll
  for (int k = 0; k < kPerThread; ++k)
    if (base + k < n) v += in[base + k];
  int total;
  (void)block_exclusive<kWaves>(v, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// In-place exclusive scan of the nb block sums (one workgroup, in order).
__global__ __launch_bounds__(kThreads) void k_scan_sums(int* sums, int nb) {
  int carry = 0;
  for (int c0 = 0; c0 < nb; c0 += kScanTile) {
    const int base = c0 + threadIdx.x * kPerThread;
    int v[kPerThread], s = 0;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      v[k] = base + k < nb ? sums[base + k] : 0;
      s += v[k];
    }
    int total;
    int run = carry + block_exclusive<kWaves>(s, &total);
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      if (base + k < nb) sums[base + k] = run;
      run += v[k];
    }
    carry += total;
  }
}

// out = exclusive prefix sum of in, given the scanned block sums.  out may be
// in: a thread reads its elements before it writes them.
__global__ __launch_bounds__(kThreads) void k_scan_apply(const int* in, int64_t n,
                                                         const int* __restrict__ sums, int* out) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
  int v[kPerThread], s = 0;
#pragma unroll
  for (int k = 0; k < kPerThread; ++k) {
    v[k] = base + k < n ? in[base + k] : 0;
    s += v[k];
  }
  int total;
  int run = sums[blockIdx.x] + block_exclusive<kWaves>(s, &total);
#pragma unroll
  for (int k = 0; k < kPerThread; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
}

// Where the pass of a level reads and writes: the last pass lands in the
// output, the ones before alternate.  A level with fewer passes than the
// others joins the last ones; -1: it has no part in this launch.
__device__ __forceinline__ int level_pass(const SortLevels& S, const SortLevel& V, int step) {
  return step - (S.passes - V.passes);
}
__device__ __forceinline__ bool to_out(const SortLevel& V, int p) {
  return ((V.passes - p) & 1) == 1;
}
__device__ __forceinline__ const unsigned* source(const SortLevel& V, int p) {
  return p == 0 ? V.kin : to_out(V, p) ? V.ktmp : V.kout;
}

// hist[b][d] = rows of block b whose digit is d.
__global__ __launch_bounds__(kThreads) void k_digit_hist(SortLevels S, int step) {
  const SortLevel& V = S.level[blockIdx.y];
  const int p = level_pass(S, V, step);
  if (p < 0 || (p == 0 && S.counted)) return;
  __shared__ int h[kMaxBuckets];
  const int buckets = 1 << V.digit_bits;
  for (int d = threadIdx.x; d < buckets; d += kThreads) h[d] = 0;
  __syncthreads();
  const unsigned* keys = source(V, p);
  const int base = blockIdx.x * kSortTile, shift = p * V.digit_bits;
  for (int j = threadIdx.x; j < kSortTile; j += kThreads) {
    const int r = base + j;
    if (r < S.rows) atomicAdd(&h[(keys[r] >> shift) & (buckets - 1)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < buckets; d += kThreads)
    V.hist[(size_t)blockIdx.x * buckets + d] = h[d];
}

// hist[b][d] -> sum of hist[0 .. b - 1][d]; total[d] = sum over all blocks.  A
// workgroup takes 32 digits (128-byte rows of the table), its 32 groups of 32
// threads a contiguous range of the blocks each.
__global__ __launch_bounds__(1024) void k_digit_scan(SortLevels S, int step) {
  const SortLevel& V = S.level[blockIdx.y];
  const int buckets = 1 << V.digit_bits, d = blockIdx.x * 32 + threadIdx.x % 32;
  if (level_pass(S, V, step) < 0 || (int)blockIdx.x * 32 >= buckets) return;
  __shared__ int part[32][32];
  const int g = threadIdx.x / 32, nb = (S.rows + kSortTile - 1) / kSortTile;
  const int per = (nb + 31) / 32, b0 = min(nb, g * per), b1 = min(nb, b0 + per);
  const bool ok = d < buckets;
  int sum = 0;
  for (int b = b0; b < b1; ++b) sum += ok ? V.hist[(size_t)b * buckets + d] : 0;
  part[g][threadIdx.x % 32] = sum;
  __syncthreads();
  int run = 0;
  for (int k = 0; k < g; ++k) run += part[k][threadIdx.x % 32];
  if (!ok) return;
  for (int b = b0; b < b1; ++b) {
    const int v = V.hist[(size_t)b * buckets + d];
    V.hist[(size_t)b * buckets + d] = run;
    run += v;
  }
  if (g == 31) V.total[d] = run;
}

// Stable scatter of block b's rows to (rows of smaller digits) + hist[b][digit]
// + (rows of the same digit before them in the block).
__global__ __launch_bounds__(kThreads) void k_digit_scatter(SortLevels S, int step) {
  const SortLevel& V = S.level[blockIdx.y];
  const int p = level_pass(S, V, step);
  if (p < 0) return;
  // rows per (chunk, digit), then their prefix
  __shared__ unsigned short cnt[kChunks][kMaxBuckets];
  __shared__ int first[kMaxBuckets];
  const int bits = V.digit_bits, buckets = 1 << bits, shift = p * bits, n = S.rows;
  const unsigned* __restrict__ kin = source(V, p);
  const int* __restrict__ vin = p == 0 ? V.vin : to_out(V, p) ? V.vtmp : V.vout;
  unsigned* __restrict__ kout = to_out(V, p) ? V.kout : V.ktmp;
  int* __restrict__ vout = to_out(V, p) ? V.vout : V.vtmp;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const unsigned long long below = (1ull << lane) - 1ull;
  const int base = blockIdx.x * kSortTile;
  unsigned key[kChunksPerWave];
  int val[kChunksPerWave], rank[kChunksPerWave];
  bool ok[kChunksPerWave];
#pragma unroll
  for (int q = 0; q < kChunksPerWave; ++q) {
    const int r = base + (wv + q * kWaves) * kWave + lane;  // chunks in row order
    ok[q] = r < n;
    key[q] = ok[q] ? kin[r] : 0u;
    val[q] = !ok[q] ? 0 : vin ? vin[r] : r;
  }
  constexpr int PER = kMaxBuckets / kThreads;
  int t[PER], sum = 0, all;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int d = threadIdx.x * PER + k;
    t[k] = d < buckets ? V.total[d] : 0;
    sum += t[k];
  }
  int run = block_exclusive<kWaves>(sum, &all);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int d = threadIdx.x * PER + k;
    if (d < buckets) first[d] = run;
    run += t[k];
  }
  for (int d = threadIdx.x; d < buckets; d += kThreads) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c) cnt[c][d] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kChunksPerWave; ++q) {
    const int c = wv + q * kWaves;
    const int d = (int)((key[q] >> shift) & (unsigned)(buckets - 1));
    // lanes of the chunk with the same digit: agree on every digit bit
    unsigned long long peers = __ballot(ok[q]);
    for (int bit = 0; bit < bits; ++bit) {
      const bool set = ((d >> bit) & 1) != 0;
      const unsigned long long m = __ballot(ok[q] && set);
      peers &= set ? m : ~m;
    }
    rank[q] = __popcll(peers & below);
    if (ok[q] && rank[q] == 0) cnt[c][d] = (unsigned short)__popcll(peers);
  }
  __syncthreads();
  // per digit: where the chunk's rows start
  for (int d = threadIdx.x; d < buckets; d += kThreads) {
    first[d] += V.hist[(size_t)blockIdx.x * buckets + d];
    int before = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int v = cnt[c][d];
      cnt[c][d] = (unsigned short)before;
      before += v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kChunksPerWave; ++q) {
    if (!ok[q]) continue;
    const int d = (int)((key[q] >> shift) & (unsigned)(buckets - 1));
    const int pos = first[d] + cnt[wv + q * kWaves][d] + rank[q];
    kout[pos] = key[q];
    vout[pos] = val[q];
  }
}

hipError_t scan_with(int* sums, const int* in, int* out, int64_t n, hipStream_t s) {
  const int nb = ceil_div(n, kScanTile);
  k_scan_block_sums<<<nb, kThreads, 0, s>>>(in, n, sums);
  k_scan_sums<<<1, kThreads, 0, s>>>(sums, nb);
  k_scan_apply<<<nb, kThreads, 0, s>>>(in, n, sums, out);
  return hipGetLastError();
}

}  // namespace

size_t sort_temp_bytes(int n) {
  if (n <= 0) return 0;
  const size_t table = (size_t)kMaxBuckets * (ceil_div(n, kSortTile) + 1);
  return aligned(4 * table) + 2 * aligned(4 * (size_t)n);
}

// Lays out a sort of up to cap rows in temp.
SortLevel sort_level(void* temp, int cap, int end_bit) {
  SortLevel V{};
  V.passes = (end_bit + kMaxDigitBits - 1) / kMaxDigitBits;
  V.digit_bits = V.passes ? (end_bit + V.passes - 1) / V.passes : 0;
  char* p = (char*)temp;
  V.total = (int*)p;
  V.hist = V.total + kMaxBuckets;
  p += aligned(4 * (size_t)kMaxBuckets * (ceil_div(cap, kSortTile) + 1));
  V.ktmp = (unsigned*)p;
  V.vtmp = (int*)(p + aligned(4 * (size_t)cap));
  return V;
}

hipError_t sort_levels(const SortLevels& S, hipStream_t s) {
  if (S.rows <= 0) return hipSuccess;
  const int nb = ceil_div(S.rows, kSortTile);
  int buckets = 0;
  for (int l = 0; l < S.n; ++l) buckets = std::max(buckets, 1 << S.level[l].digit_bits);
  for (int step = 0; step < S.passes; ++step) {
    if (step > 0 || !S.counted) k_digit_hist<<<dim3(nb, S.n), kThreads, 0, s>>>(S, step);
    k_digit_scan<<<dim3(ceil_div(buckets, 32), S.n), 1024, 0, s>>>(S, step);
    k_digit_scatter<<<dim3(nb, S.n), kThreads, 0, s>>>(S, step);
  }
  return hipGetLastError();
}

hipError_t sort_pairs(void* temp, size_t bytes, const unsigned* kin, unsigned* kout,
                      const int* vin, int* vout, int n, int end_bit, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (n < 0 || end_bit < 0 || end_bit > 32 || !temp || bytes < sort_temp_bytes(n))
    return hipErrorInvalidValue;
  SortLevels S{};
  S.n = 1;
  S.rows = n;
  SortLevel& V = S.level[0];
  V = sort_level(temp, n, end_bit);
  S.passes = V.passes;
  if (S.passes == 0) {  // every key is 0: the order is the input order
    hipError_t e = hipMemcpyAsync(kout, kin, 4 * (size_t)n, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(vout, vin, 4 * (size_t)n, hipMemcpyDeviceToDevice, s);
    return e;
  }
  V.kin = kin;
  V.vin = vin;
  V.kout = kout;
  V.vout = vout;
  return sort_levels(S, s);
}

size_t scan_temp_bytes(int n) { return aligned(4 * (size_t)ceil_div(n > 0 ? n : 1, kScanTile)); }

hipError_t exclusive_scan(void* temp, size_t bytes, const int* in, int* out, int n,
                          hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (n < 0 || !temp || bytes < scan_temp_bytes(n)) return hipErrorInvalidValue;
  return scan_with((int*)temp, in, out, n, s);
}

}  // namespace vd
