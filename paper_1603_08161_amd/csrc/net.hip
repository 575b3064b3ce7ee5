// Learned warm start: the 3-D convolutional encoder-decoder of vd_net.h on
// the gfx950 matrix cores, its training (loss, backward, Adam) and the input
// feature build from a lattice's constraint rows.
//
// Every convolution is an implicit GEMM on channels-last bfloat16 tensors:
// rows are output voxels, columns output channels, and the reduction index
// k = tap * c_in + channel runs over the 27 taps and the input channels.  A
// wavefront issues v_mfma_f32_16x16x32_bf16 on 16-voxel x 16-channel tiles:
// each lane reads 8 consecutive k of one voxel (8 channels of one tap, a
// single 16-byte LDS read, since every channel count is a multiple of 8) and
// the matching 8 k of one output channel from the pre-packed weights.  The
// same kernel runs the backward data pass (flipped, transposed weights; a
// stride-2 layer reads its output gradient at (o + tap - 1) / 2 where that is
// even).
// Weight gradients are a split-K GEMM over voxels with both operands read
// transposed from LDS, followed by a fixed-order reduction of the partials.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/vd_net.h"
#include "net_kernels.h"
#include "vd_device.h"

namespace vd {
namespace net {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest even (NaN kept quiet).
__host__ __device__ inline uint16_t f2bf(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__host__ __device__ inline float bf2f(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

__device__ inline bool bf_pos(uint16_t b) { return !(b & 0x8000u) && (b & 0x7fffu); }

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Source coordinate of output coordinate o at tap t along one axis; false
// where the tap falls into the zero padding.
__device__ inline bool src_coord(int mode, int stride, int o, int t, int n_src, int n_out,
                                 int& q) {
  if (mode == kGatherPlain) {
    q = stride * o + t - 1;
    return q >= 0 && q < n_src;
  }
  q = o + t - 1;
  if (mode == kGatherUp) {
    const bool ok = q >= 0 && q < n_out;
    q >>= 1;
    return ok;
  }
  // kGatherTransposed2: input gradient of a stride-2 convolution
  const bool ok = q >= 0 && !(q & 1) && (q >> 1) < n_src;
  q >>= 1;
  return ok;
}

// 8 consecutive k (one tap, 8 channels) of output voxel (b, z, y, x).
__device__ inline uint4 gather8(const ConvArgs& A, int b, int z, int y, int x, int k0) {
  uint4 zero = {0u, 0u, 0u, 0u};
  if (k0 >= A.ktot) return zero;
  const int t = k0 >> A.lcin;
  int c = k0 & (A.cin - 1);
  const int tz = t / 9, ty = (t / 3) % 3, tx = t % 3;
  int qz, qy, qx;
  if (!src_coord(A.mode, A.stride, z, tz, A.sd, A.od, qz)) return zero;
  if (!src_coord(A.mode, A.stride, y, ty, A.sh, A.oh, qy)) return zero;
  if (!src_coord(A.mode, A.stride, x, tx, A.sw, A.ow, qx)) return zero;
  const uint16_t* base = A.a;
  int C = A.ca;
  if (c >= A.ca) {
    base = A.b;
    C = A.cb;
    c -= A.ca;
  }
  const size_t v = (((size_t)b * A.sd + qz) * A.sh + qy) * A.sw + qx;
  return *reinterpret_cast<const uint4*>(base + v * C + c);
}

// ---------------------------------------------------------------------------
// convolution (forward and backward data)
// ---------------------------------------------------------------------------

// A workgroup computes a brick of 16 x BY x BZ output voxels for NB blocks of
// 16 output channels.  It stages the brick's input with its halo in LDS, one
// plane per group of 8 channels, so that the 16 voxels of a fragment are 256
// contiguous bytes whatever the tap.  Its four waves hold MB = BY BZ / 4 rows
// of 16 voxels each; the weights of a 32-wide chunk of k are loaded once for
// them, and with the brick's extents known to the compiler a fragment's
// address is one register and an immediate.  The products are taken
// transposed (weights as the first operand), which leaves four consecutive
// output channels of a voxel in a lane: 8-byte stores.  Chunks run in order, so
// the sums do not depend on the brick.
//
// What bounds it: one KB of LDS per matrix op with 16 output channels (about 3
// us for a 16 -> 16 layer at 64^3), the staging's round trip and the launch.
// Gathering every tap from memory, or staging rows of 128 voxels with weights
// loaded once per two fragments, took 413 us per forward pass at 64^3 (33 us
// for that layer).

// Four output channels co .. co + 3 of voxel m at (b, n): bias, skip addend,
// ReLU / ReLU mask, bfloat16 or float32 output.
__device__ __forceinline__ void conv_store(const ConvArgs& A, f32x4 v, int m, int b, int n, int co) {
  if (A.bias) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (co + r < A.cout) v[r] += A.bias[co + r];
  }
  if (A.out_f32) {
    const int64_t npb = (int64_t)A.od * A.oh * A.ow;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (co + r < A.cout) A.out_f32[((int64_t)b * A.cout + co + r) * npb + n] = v[r];
    return;
  }
  // channels [0, c0) go to dst0, [c0, c0 + c1) to dst1 (multiples of 16)
  const bool lower = co < A.c0;
  const int c = lower ? A.c0 : A.c1, cc = lower ? co : co - A.c0;
  if (cc >= c) return;
  const size_t e = (size_t)m * c + cc;
  const uint16_t* const add = lower ? A.add0 : A.add1;
  const uint16_t* const mask = lower ? A.mask0 : A.mask1;
  if (add) {
    const uint2 s = *reinterpret_cast<const uint2*>(add + e);
    v[0] += bf2f((uint16_t)s.x);
    v[1] += bf2f((uint16_t)(s.x >> 16));
    v[2] += bf2f((uint16_t)s.y);
    v[3] += bf2f((uint16_t)(s.y >> 16));
  }
  if (A.relu) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
  }
  if (mask) {
    const uint2 s = *reinterpret_cast<const uint2*>(mask + e);
    if (!bf_pos((uint16_t)s.x)) v[0] = 0.f;
    if (!bf_pos((uint16_t)(s.x >> 16))) v[1] = 0.f;
    if (!bf_pos((uint16_t)s.y)) v[2] = 0.f;
    if (!bf_pos((uint16_t)(s.y >> 16))) v[3] = 0.f;
  }
  uint2 o;
  o.x = f2bf(v[0]) | (uint32_t)f2bf(v[1]) << 16;
  o.y = f2bf(v[2]) | (uint32_t)f2bf(v[3]) << 16;
  *reinterpret_cast<uint2*>((lower ? A.dst0 : A.dst1) + e) = o;
}

constexpr int kConvX = 16;  // brick extent along x

template <int CIN, int NB, int S, int BY, int BZ>
__global__ __launch_bounds__(kBlock) void k_conv(ConvArgs A) {
  constexpr int HX = S * (kConvX - 1) + 3, HY = S * (BY - 1) + 3, HZ = S * (BZ - 1) + 3;
  constexpr int VOX = HX * HY * HZ, CG = CIN / 8, MB = BY * BZ / 4;
  constexpr int NCH = (27 * CIN + 31) / 32;
  __shared__ uint4 s_in[CG * VOX];  // [channel group][z][y][x]
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int q = blockIdx.x;
  const int nbx = (A.ow + kConvX - 1) / kConvX, nby = (A.oh + BY - 1) / BY,
            nbz = (A.od + BZ - 1) / BZ;
  const int ox = q % nbx * kConvX;
  q /= nbx;
  const int oy = q % nby * BY;
  q /= nby;
  const int oz = q % nbz * BZ, b = q / nbz;
  const int j0 = blockIdx.y * NB;
  // limits of the input coordinates (up-sampled and transposed layers: of the
  // fine grid)
  const bool plain = A.mode == kGatherPlain, odd_zero = A.mode == kGatherTransposed2;
  const int half = plain ? 0 : 1;
  const unsigned nx = A.mode == kGatherUp ? A.ow : A.sw << half,
                 ny = A.mode == kGatherUp ? A.oh : A.sh << half,
                 nz = A.mode == kGatherUp ? A.od : A.sd << half;
#pragma unroll
  for (int it = 0; it < (CG * VOX + kBlock - 1) / kBlock; ++it) {  // all loads in flight
    const int i = threadIdx.x + it * kBlock;
    if (i >= CG * VOX) break;
    const int v = i / CG, g = i % CG;
    const int px = S * ox + v % HX - 1, py = S * oy + v / HX % HY - 1,
              pz = S * oz + v / (HX * HY) - 1;
    uint4 val = {0u, 0u, 0u, 0u};
    if ((unsigned)px < nx && (unsigned)py < ny && (unsigned)pz < nz &&
        !(odd_zero && ((px | py | pz) & 1))) {
      const int sv = ((b * A.sd + (pz >> half)) * A.sh + (py >> half)) * A.sw + (px >> half);
      const int c = 8 * g;
      val = *reinterpret_cast<const uint4*>(c < A.ca ? A.a + (size_t)sv * A.ca + c
                                                     : A.b + (size_t)sv * A.cb + c - A.ca);
    }
    s_in[g * VOX + v] = val;
  }
  __syncthreads();
  f32x4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the wave's first row, and the lane's voxel and channel group in it
  const int y0 = wave * MB % BY, z0 = wave * MB / BY, quarter = lane >> 4;
  const int base = ((S * z0 * HY + S * y0) * HX + S * (lane & 15)) +
                   (CIN >= 32 ? quarter : CIN == 16 ? quarter & 1 : 0) * VOX;
  const uint4* __restrict__ W = A.w + (size_t)j0 * kWave + lane;
  auto tap = [](int t) { return ((t / 9) * HY + (t / 3) % 3) * HX + t % 3; };
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    bf16x8 bw[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) bw[j] = as_bf16x8(W[(ch * A.nb + j) * kWave]);
    // the lane's k: taps t .. t + 32 / CIN - 1 by lane quarter
    const int t = ch * 32 / CIN;
    int at = base;
    bool pad = false;  // past the last tap
    if (CIN >= 32) {
      at += tap(t) + (CIN == 64 ? (ch & 1) * 4 * VOX : 0);
    } else if (CIN == 16) {
      at += quarter < 2 ? tap(t) : tap(t + 1 < 27 ? t + 1 : t);
      pad = t + 1 >= 27 && quarter >= 2;
    } else {
      const int far = quarter < 2 ? (quarter == 0 ? tap(t) : tap(t + 1))
                                  : (quarter == 2 ? tap(t + 2) : tap(t + 3 < 27 ? t + 3 : t));
      at += far;
      pad = t + 3 >= 27 && quarter == 3;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      uint4 x = s_in[at + i * S * HX];
      if (pad) x = uint4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[j], as_bf16x8(x), acc[i][j], 0, 0, 0);
    }
  }
  // lane: voxel lane % 16 of its row, channels 4 (lane / 16) .. + 3 of a block
  const int x = ox + (lane & 15), z = oz + z0;
  if (x >= A.ow || z >= A.od) return;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int y = oy + y0 + i;
    if (y >= A.oh) continue;
    const int n = (z * A.oh + y) * A.ow + x;
    const int m = b * (A.od * A.oh * A.ow) + n;
#pragma unroll
    for (int j = 0; j < NB; ++j) conv_store(A, acc[i][j], m, b, n, (j0 + j) * 16 + 4 * quarter);
  }
}

// ---------------------------------------------------------------------------
// weight gradients: dW[k][co] = sum_v X[v][k] dY[v][co], k = tap * c_in + ci,
// plus the bias row k = 27 c_in (X = 1)
// ---------------------------------------------------------------------------
//
// Voxels are split into chunks; a chunk's sum runs over its voxels in linear
// order, 32 per matrix op, and the chunks are added in order, so every path
// below gives the same bits.
//
// Path of grids whose rows fit in LDS (k_wgrad): workgroup (chunk, tap plane
// and 16 input channels), all columns.  It stages blocks of 32 KS voxels: dY as it
// lies in memory, and the input rows that the block's nine taps of plane tz
// touch, channels-last.  Its eight waves share the taps.  The transposing LDS
// read (ds_read_b64_tr_b16) gives a lane four voxels of its channel from
// voxel-major rows at any addresses, so a tap is an address offset and a block
// may cross rows and planes.  The next block's loads are in flight while the
// current one is computed.  Every input is loaded three times (once per tap
// plane) instead of 27.
//
// What bounds it: the LDS reads of the operands, 18 + 16 CO half-kilobyte
// reads per 32 voxels and workgroup.  Gathering 8 channels per lane and tap
// from memory and transposing through 2-byte LDS stores (k_wgrad_gather, still
// the path of wider rows) took 755 us for the layers of 16 columns at 64^3,
// batch 4, on average, against 185 us here (32 columns: 197 and 66 us); the
// training step went from 6.69 to 3.16 ms.

typedef short s16x4 __attribute__((ext_vector_type(4)));
constexpr int kWgThreads = 512;
constexpr int kWgLoads = 8;  // 16-byte loads per thread and block

// Four voxels of the calling lane's channel; `row` is the lane's own address:
// voxel (lane % 16) / 4 of the four, channel 4 (lane % 4).
__device__ __forceinline__ s16x4 read_tr(const uint16_t* row) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)const_cast<uint16_t*>(row));
}

__device__ __forceinline__ bf16x8 join8(s16x4 lo, s16x4 hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A voxel's place in a staged block: its x and the LDS line of tap row ty = 0.
// Lines are the input rows of the block's planes in order, each plane's from
// the row above its first output row (in the block) to the one below its
// last: plane p's are y = -1 .. S oh + 1 - S, LP = S oh + 3 - S of them.
template <int S>
struct WgPlace {
  int x, y, line;
  // the voxel `ahead` after (x0, y0), the block's first
  __device__ __forceinline__ void at(int x0, int y0, int ahead, int ow, int oh) {
    x = x0 + ahead;
    y = y0;
    line = 0;
    while (x >= ow) wrap(ow, oh);
  }
  __device__ __forceinline__ void wrap(int ow, int oh) {  // past a row's end
    const bool r = x >= ow;
    x -= r ? ow : 0;
    line += r ? S : 0;
    y += r ? 1 : 0;
    const bool pl = y == oh;
    y = pl ? 0 : y;
    line += pl ? 3 - S : 0;
  }
  __device__ __forceinline__ void step(int ow, int oh) {
    x += 32;
    wrap(ow, oh);
    if (ow < 32)
      while (x >= ow) wrap(ow, oh);
  }
};

template <int CO, int S>
__global__ __launch_bounds__(kWgThreads) void k_wgrad(ConvArgs A, WgradArgs G) {
  extern __shared__ __attribute__((aligned(16))) uint16_t wg_lds[];
  const int W = S * (A.ow - 1) + 3, LP = S * A.oh + 3 - S;
  uint16_t* const ys = wg_lds;                             // [32 KS][CO * 16]
  uint16_t* const xs = wg_lds + 32 * G.ksteps * CO * 16;   // [lines][W][16]
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int chunk = blockIdx.x, tz = blockIdx.y % 3, ci0 = blockIdx.y / 3 * 16;
  // (at most 2^28 voxels: 32-bit indices)
  const int v_begin = chunk * (int)G.vox_per_chunk;
  const int v_end = min(v_begin + (int)G.vox_per_chunk, A.batch * A.od * A.oh * A.ow);
  // source of the 16 channels (a concatenation's boundary is a multiple of 16)
  const uint16_t* src = A.a;
  int C = A.ca, cc = ci0;
  if (cc >= A.ca) {
    src = A.b;
    C = A.cb;
    cc -= A.ca;
  }
  const int nch8 = C - cc >= 16 ? 2 : 1;  // 16-byte groups that exist
  const int block_vox = 32 * G.ksteps;
  // the wave's taps (ty, tx) of plane tz: wave, and 8 for wave 0; wave 1 of
  // the first plane and channels sums the bias row instead
  const bool second = wave == 0, bias = wave == 1 && blockIdx.y == 0;
  const int off0 = (wave / 3 * W + wave % 3) * 16, off1 = (2 * W + 2) * 16;
  f32x4 acc[2][CO];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < CO; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const short one = (lane & 15) == 0 ? (short)0x3f80 : (short)0;  // bfloat16 1, first row
  const s16x4 ones = {one, one, one, one};
  const int sub = (lane & 15) >> 2, quad = (lane & 3) * 4, first = 8 * (lane >> 4) + sub;
  const int ny = block_vox * CO * 2;  // 16-byte groups of a block's dY
  uint4 pre[kWgLoads];
  // the input line and x of each of the thread's loads: line << 16 | x, -1: none
  int place[kWgLoads];
#pragma unroll
  for (int i = 0; i < kWgLoads; ++i) {
    const int q = threadIdx.x + i * kWgThreads - ny, l = (q >> 1) / W;
    place[i] = q >= 0 && l < G.lines && (q & 1) < nch8 ? l << 16 | ((q >> 1) - l * W) : -1;
  }
  // limits of the input coordinates (up-sampled layers: of the fine grid)
  const bool up = A.mode == kGatherUp;
  const unsigned nx = up ? A.ow : A.sw, nyl = up ? A.oh : A.sh, nz = up ? A.od : A.sd;
  const bool many_planes = G.lines + S * A.oh > 2 * LP;
  // block starts: the block being fetched, then (one behind) the one computed
  int fx = v_begin % A.ow, fy = v_begin / A.ow % A.oh, fz = v_begin / (A.ow * A.oh) % A.od,
      fb = v_begin / (A.ow * A.oh * A.od);
  auto fetch = [&](int v) {
#pragma unroll
    for (int i = 0; i < kWgLoads; ++i) {
      const int q = threadIdx.x + i * kWgThreads;
      const uint16_t* p = nullptr;
      if (q < ny) {
        const int m = v + q / (CO * 2), c = q % (CO * 2) * 8;
        if (m < v_end && c < G.cdy) p = G.dy + (size_t)m * G.cdy + c;
      } else if (place[i] >= 0) {
        int py = (place[i] >> 16) + S * fy, z = fz, b = fb;
        do {  // into the next plane
          const bool w = py >= LP;
          py -= w ? LP : 0;
          z += w ? 1 : 0;
          const bool nb = z == A.od;
          z = nb ? 0 : z;
          b += nb ? 1 : 0;
        } while (many_planes && py >= LP);
        int px = (place[i] & 0xffff) - 1, pz = S * z + tz - 1;
        --py;
        if ((unsigned)px < nx && (unsigned)py < nyl && (unsigned)pz < nz && b < A.batch) {
          px >>= up;
          py >>= up;
          pz >>= up;
          const int sv = ((b * A.sd + pz) * A.sh + py) * A.sw + px;
          p = src + (size_t)sv * C + cc + 8 * ((q - ny) & 1);
        }
      }
      pre[i] = p ? *reinterpret_cast<const uint4*>(p) : uint4{0u, 0u, 0u, 0u};
    }
  };
  WgPlace<S> lo, hi;
  // operands of one step at the places lo, hi
  struct Frags {
    bf16x8 b[CO], a0, a1;
  };
  auto read = [&](int s) {
    Frags f;
    const uint16_t* yrow = ys + (32 * s + first) * CO * 16 + quad;
    const uint16_t* xlo = xs + (lo.line * W + S * lo.x) * 16 + quad;
    const uint16_t* xhi = xs + (hi.line * W + S * hi.x) * 16 + quad;
#pragma unroll
    for (int j = 0; j < CO; ++j)
      f.b[j] = join8(read_tr(yrow + 16 * j), read_tr(yrow + 4 * CO * 16 + 16 * j));
    f.a0 = join8(read_tr(xlo + off0), read_tr(xhi + off0));
    f.a1 = second ? join8(read_tr(xlo + off1), read_tr(xhi + off1)) : join8(ones, ones);
    return f;
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int j = 0; j < CO; ++j)
      acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a0, f.b[j], acc[0][j], 0, 0, 0);
    if (second || bias) {
#pragma unroll
      for (int j = 0; j < CO; ++j)
        acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a1, f.b[j], acc[1][j], 0, 0, 0);
    }
  };
  fetch(v_begin);
  for (int v = v_begin; v < v_end; v += block_vox) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWgLoads; ++i) {
      const int q = threadIdx.x + i * kWgThreads;
      if (q < ny + G.lines * W * 2) *reinterpret_cast<uint4*>(wg_lds + 8 * q) = pre[i];
    }
    __syncthreads();
    lo.at(fx, fy, first, A.ow, A.oh);
    hi.at(fx, fy, first + 4, A.ow, A.oh);
    if (v + block_vox < v_end) {
      fx += block_vox;
      const int rows = fx / A.ow;
      fx -= rows * A.ow;
      fy += rows;
      while (fy >= A.oh) {
        fy -= A.oh;
        if (++fz == A.od) {
          fz = 0;
          ++fb;
        }
      }
      fetch(v + block_vox);
    }
    const int left = (v_end - v + 31) / 32;
    const int steps = min(left, G.ksteps);
    // the next step's reads are issued before a step's products
    Frags f = read(0);
    for (int s = 0; s < steps; s += 2) {
      lo.step(A.ow, A.oh);
      hi.step(A.ow, A.oh);
      Frags g = f;
      if (s + 1 < steps) g = read(s + 1);
      multiply(f);
      if (s + 1 >= steps) break;
      lo.step(A.ow, A.oh);
      hi.step(A.ow, A.oh);
      if (s + 2 < steps) f = read(s + 2);
      multiply(g);
    }
  }
  float* out = G.partial + (size_t)chunk * G.mpad * G.npad;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t == 1 && !second && !bias) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ci = ci0 + 4 * (lane >> 4) + r;
      const bool is_bias = t == 1 && bias;
      if (is_bias ? ci > 0 : ci >= A.cin) continue;
      const int row = is_bias ? 27 * A.cin : (tz * 9 + (t == 0 ? wave : 8)) * A.cin + ci;
#pragma unroll
      for (int j = 0; j < CO; ++j)
        out[(size_t)row * G.npad + j * 16 + (lane & 15)] = acc[t][j][r];
    }
  }
}

// Grids whose rows do not fit: workgroup (mtile, chunk) sums the voxels of its
// chunk for 64 rows k and all columns; partials [chunk][mpad][npad].

constexpr int kWgVox = 32;          // voxels per LDS stage (one MFMA K step)
constexpr int kWgPitch = kWgVox + 8;  // bf16 per LDS row (80 bytes, 16-aligned)

template <int NB>
__global__ __launch_bounds__(kBlock) void k_wgrad_gather(ConvArgs A, WgradArgs G) {
  __shared__ __attribute__((aligned(16))) uint16_t xt[64 * kWgPitch];
  __shared__ __attribute__((aligned(16))) uint16_t gt[64 * kWgPitch];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int mtile = blockIdx.x, chunk = blockIdx.y;
  const int64_t M = (int64_t)A.batch * A.od * A.oh * A.ow;
  const int64_t v_begin = (int64_t)chunk * G.vox_per_chunk;
  int64_t v_end = v_begin + G.vox_per_chunk;
  if (v_end > M) v_end = M;
  f32x4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sv = threadIdx.x & (kWgVox - 1);  // staging: voxel within the stage
  const int sg = threadIdx.x / kWgVox;        // staging: group of 8 rows / columns
  const int row0 = mtile * 64 + 8 * sg;
  for (int64_t v0 = v_begin; v0 < v_end; v0 += kWgVox) {
    const int64_t m = v0 + sv;
    uint4 xv = {0u, 0u, 0u, 0u}, gv = {0u, 0u, 0u, 0u};
    if (m < v_end) {
      int64_t r = m;
      const int x = (int)(r % A.ow);
      r /= A.ow;
      const int y = (int)(r % A.oh);
      r /= A.oh;
      const int z = (int)(r % A.od);
      const int b = (int)(r / A.od);
      if (row0 < A.ktot)
        xv = gather8(A, b, z, y, x, row0);
      else if (row0 == A.ktot)
        xv.x = 0x3f80u;  // bfloat16 1.0 in element 0: the bias row
      if (8 * sg < G.cdy) gv = *reinterpret_cast<const uint4*>(G.dy + (size_t)m * G.cdy + 8 * sg);
    }
    const uint16_t* xe = reinterpret_cast<const uint16_t*>(&xv);
    const uint16_t* ge = reinterpret_cast<const uint16_t*>(&gv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xt[(8 * sg + e) * kWgPitch + sv] = xe[e];
      gt[(8 * sg + e) * kWgPitch + sv] = ge[e];
    }
    __syncthreads();
    const bf16x8 af =
        as_bf16x8(*reinterpret_cast<const uint4*>(&xt[(wave * 16 + (lane & 15)) * kWgPitch +
                                                       8 * (lane >> 4)]));
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bf16x8 bf = as_bf16x8(
          *reinterpret_cast<const uint4*>(&gt[(j * 16 + (lane & 15)) * kWgPitch + 8 * (lane >> 4)]));
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc[j], 0, 0, 0);
    }
    __syncthreads();
  }
  float* out = G.partial + (size_t)chunk * G.mpad * G.npad;
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = mtile * 64 + wave * 16 + 4 * (lane >> 4) + r;
      out[(size_t)row * G.npad + j * 16 + (lane & 15)] = acc[j][r];
    }
}

// grad[p] = sum over chunks (in order) of the partial at (row, co), one thread
// per entry in the partials' order.
__global__ __launch_bounds__(kWave) void k_wgrad_reduce(const float* __restrict__ partial,
                                                        int nchunks, int mpad, int npad, int cin,
                                                        int cout, float* grad) {
  const int e = blockIdx.x * kWave + threadIdx.x;
  const int row = e / npad, co = e - row * npad;
  if (row > 27 * cin || co >= cout) return;
  const float* p = partial + (size_t)row * npad + co;
  float s = 0.f;
#pragma unroll 16
  for (int c = 0; c < nchunks; ++c) s += p[(size_t)c * mpad * npad];
  if (row == 27 * cin) {
    grad[(size_t)cout * cin * 27 + co] = s;
  } else {
    const int t = row / cin, ci = row - t * cin;
    grad[((size_t)co * cin + ci) * 27 + t] = s;
  }
}

// ---------------------------------------------------------------------------
// weight packing: float32 master -> MFMA operand order [chunk][nb][lane][8]
// ---------------------------------------------------------------------------

// Forward: k = t * cin + ci, column co; W[co][ci][t].
__global__ __launch_bounds__(kBlock) void k_pack_fwd(const float* __restrict__ W, int cin, int cout,
                                                     int nchunk, int nb, uint16_t* out) {
  const int total = nchunk * nb * kWave * 8;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= total) return;
  const int e = i & 7, lane = (i >> 3) & (kWave - 1);
  const int rest = i / (8 * kWave);
  const int j = rest % nb, ch = rest / nb;
  const int k = ch * 32 + 8 * (lane >> 4) + e;
  const int co = j * 16 + (lane & 15);
  float v = 0.f;
  if (k < 27 * cin && co < cout) {
    const int t = k / cin, ci = k - t * cin;
    v = W[((size_t)co * cin + ci) * 27 + t];
  }
  out[i] = f2bf(v);
}

// Backward data: a convolution of the output gradient (cdy channels, cout of
// them real) producing the cin input channels, taps flipped: W[co][ci][26 - t].
__global__ __launch_bounds__(kBlock) void k_pack_dgrad(const float* __restrict__ W, int cin,
                                                       int cout, int cdy, int nchunk, int nb,
                                                       uint16_t* out) {
  const int total = nchunk * nb * kWave * 8;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= total) return;
  const int e = i & 7, lane = (i >> 3) & (kWave - 1);
  const int rest = i / (8 * kWave);
  const int j = rest % nb, ch = rest / nb;
  const int k = ch * 32 + 8 * (lane >> 4) + e;
  const int n = j * 16 + (lane & 15);
  float v = 0.f;
  if (k < 27 * cdy && n < cin) {
    const int t = k / cdy, co = k - t * cdy;
    if (co < cout) v = W[((size_t)co * cin + n) * 27 + (26 - t)];
  }
  out[i] = f2bf(v);
}

// ---------------------------------------------------------------------------
// up-sampling backward, loss, Adam
// ---------------------------------------------------------------------------

// g[w][c] = (src[w][c] > 0) * sum of dup over the fine voxels v with v/2 = w.
__global__ __launch_bounds__(kBlock) void k_upsum(const uint16_t* __restrict__ dup, int fd, int fh,
                                                  int fw, const uint16_t* __restrict__ src, int cd,
                                                  int chh, int cw, int C, int batch, uint16_t* g) {
  const int64_t total = (int64_t)batch * cd * chh * cw * C;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % C);
  int64_t r = i / C;
  const int x = (int)(r % cw);
  r /= cw;
  const int y = (int)(r % chh);
  r /= chh;
  const int z = (int)(r % cd);
  const int b = (int)(r / cd);
  float s = 0.f;
  for (int dz = 0; dz < 2; ++dz) {
    const int fz = 2 * z + dz;
    if (fz >= fd) continue;
    for (int dy = 0; dy < 2; ++dy) {
      const int fy = 2 * y + dy;
      if (fy >= fh) continue;
      for (int dx = 0; dx < 2; ++dx) {
        const int fx = 2 * x + dx;
        if (fx >= fw) continue;
        s += bf2f(dup[((((size_t)b * fd + fz) * fh + fy) * fw + fx) * C + c]);
      }
    }
  }
  g[i] = bf_pos(src[i]) ? f2bf(s) : (uint16_t)0;
}

// dout[m][0..7] = 2 (out - target) / M for the 3 real channels, 0 otherwise;
// block partials of sum (out - target)^2.
__global__ __launch_bounds__(kBlock) void k_mse(const float* __restrict__ out,
                                                const float* __restrict__ target, int64_t npb,
                                                int batch, uint16_t* dout, double* part) {
  const int64_t M = npb * batch;
  const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double v[1] = {0.0};
  if (m < M) {
    const int64_t b = m / npb, n = m - b * npb;
    uint4 w = {0u, 0u, 0u, 0u};
    uint16_t* we = reinterpret_cast<uint16_t*>(&w);
    const float scale = (float)(2.0 / (double)M);
    for (int c = 0; c < 3; ++c) {
      const size_t e = (size_t)(b * 3 + c) * npb + n;
      const float d = out[e] - target[e];
      v[0] += (double)d * d;
      we[c] = f2bf(scale * d);
    }
    *reinterpret_cast<uint4*>(dout + (size_t)m * 8) = w;
  }
  write_block_partials<1>(v, part, 0);
}

__global__ void k_mse_finalize(const double* part, int n, double inv_m, double* loss) {
  const double s = sum_partials(part, n);
  if (threadIdx.x == 0) *loss = s * inv_m;
}

// One Adam step.  ob1 = 1 - beta1 and ob2 = 1 - beta2 arrive rounded from
// their float64 values: 1.f - 0.999f would lose four digits to cancellation
// (a 1.3e-5 relative error in every second-moment update).
__global__ __launch_bounds__(kBlock) void k_adam(float* p, const float* __restrict__ g, float* m1,
                                                 float* m2, int64_t n, float lr, float b1,
                                                 float ob1, float b2, float ob2, float eps,
                                                 float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + ob1 * gi;
  const float b = b2 * m2[i] + ob2 * gi * gi;
  m1[i] = a;
  m2[i] = b;
  p[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

__global__ __launch_bounds__(kBlock) void k_check_finite_f(const float* v, int64_t n, int* flag) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n && !(fabsf(v[i]) <= 3.0e38f)) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------
// features (channels of vd_net.h) from a lattice's finest level
// ---------------------------------------------------------------------------

// Per dense row: sqrt(w) * (w-weighted residual) pieces: a = |sn| * r',
// b = |sn|^2 with r' = sn . sum_k alpha_k d_k - rho.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_row_residual(LevelView<T> L, int rows, int n_dense,
                                                         float* ra, float* rb) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n_dense) return;
  const int cell = L.row_cell[i];
  const int cnx = L.nx - 1, cny = L.ny - 1;
  const int cx = cell % cnx, cy = (cell / cnx) % cny, cz = cell / (cnx * cny);
  const T f[3] = {L.row_f[i], L.row_f[(size_t)rows + i], L.row_f[2 * (size_t)rows + i]};
  const T sn[3] = {L.row_sn[i], L.row_sn[(size_t)rows + i], L.row_sn[2 * (size_t)rows + i]};
  T s[3] = {0, 0, 0};
  for (int k = 0; k < 8; ++k) {
    const int dx = k & 1, dy = (k >> 1) & 1, dz = k >> 2;
    const T a = (dx ? f[0] : 1 - f[0]) * (dy ? f[1] : 1 - f[1]) * (dz ? f[2] : 1 - f[2]);
    const size_t node = (size_t)(cx + dx) + L.nx * ((size_t)(cy + dy) + (size_t)L.ny * (cz + dz));
    for (int c = 0; c < 3; ++c) s[c] += a * L.d[(size_t)c * L.N + node];
  }
  const T r = sn[0] * s[0] + sn[1] * s[1] + sn[2] * s[2] - L.row_rho[i];
  const T w2 = sn[0] * sn[0] + sn[1] * sn[1] + sn[2] * sn[2];
  ra[i] = (float)(sqrt(w2) * r);
  rb[i] = (float)w2;
}

// One thread per node: gathers the rows of the (up to) 8 cells around it in
// cell order, then the rows of each cell in sorted order.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_features(LevelView<T> L, RowView<T> R,
                                                     const float* __restrict__ ra,
                                                     const float* __restrict__ rb,
                                                     const float* __restrict__ prev2, int n_dense,
                                                     uint16_t* x) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= L.N) return;
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  const int ix = i % nx, iy = (i / nx) % ny, iz = i / (nx * ny);
  const int cnx = nx - 1, cny = ny - 1, cnz = nz - 1;
  const int rows = R.rows;
  double num = 0.0, den = 0.0;
  for (int k = 0; k < 8; ++k) {
    const int dx = k & 1, dy = (k >> 1) & 1, dz = k >> 2;  // corner of node i in the cell
    const int cx = ix - dx, cy = iy - dy, cz = iz - dz;
    if (cx < 0 || cy < 0 || cz < 0 || cx >= cnx || cy >= cny || cz >= cnz) continue;
    const int a = L.cell_map[cx + cnx * (cy + cny * cz)];
    if (a < 0) continue;
    for (int s = R.seg_start[a]; s < R.seg_start[a + 1]; ++s) {
      const int row = R.sorted[s];
      if (row >= n_dense) continue;
      const T fx = R.f[row], fy = R.f[(size_t)rows + row], fz = R.f[2 * (size_t)rows + row];
      const double al = (double)((dx ? fx : 1 - fx) * (dy ? fy : 1 - fy) * (dz ? fz : 1 - fz));
      num += al * ra[row];
      den += al * rb[row];
    }
  }
  const double inv_h = 1.0 / (double)L.h;
  float ch[8];
  for (int c = 0; c < 3; ++c) {
    const double d1 = (double)L.d[(size_t)c * L.N + i];
    ch[c] = (float)(d1 * inv_h);
    ch[3 + c] = prev2 ? (float)((d1 - (double)prev2[(size_t)c * L.N + i]) * inv_h) : 0.f;
  }
  ch[6] = den > 0.0 ? (float)(num / den * inv_h) : 0.f;
  ch[7] = den > 0.0 ? 1.f : 0.f;
  uint4 w;
  uint16_t* we = reinterpret_cast<uint16_t*>(&w);
  for (int c = 0; c < 8; ++c) we[c] = f2bf(ch[c]);
  *reinterpret_cast<uint4*>(x + (size_t)i * 8) = w;
}

template <typename T>
hipError_t launch_features(const LevelView<T>& L, const RowView<T>& R, const float* prev2,
                           float* scratch, uint16_t* x, hipStream_t s) {
  float* ra = scratch;
  float* rb = scratch + (R.n_dense > 0 ? R.n_dense : 1);
  if (R.n_dense > 0)
    k_row_residual<T><<<(R.n_dense + kBlock - 1) / kBlock, kBlock, 0, s>>>(L, R.rows, R.n_dense,
                                                                          ra, rb);
  k_features<T><<<(L.N + kBlock - 1) / kBlock, kBlock, 0, s>>>(L, R, ra, rb, prev2, R.n_dense, x);
  return hipGetLastError();
}

template hipError_t launch_features<float>(const LevelView<float>&, const RowView<float>&,
                                           const float*, float*, uint16_t*, hipStream_t);
template hipError_t launch_features<double>(const LevelView<double>&, const RowView<double>&,
                                            const float*, float*, uint16_t*, hipStream_t);

// ---------------------------------------------------------------------------
// host side: the network handle
// ---------------------------------------------------------------------------

namespace {

struct LayerDef {
  int ca, cb, cout, stride, up, relu;
};

// The 11 layers of vd_net.h in parameter order.
constexpr LayerDef kLayers[kNumLayers] = {
    {8, 0, 16, 1, 0, 1},   {16, 0, 16, 1, 0, 1},  {16, 0, 32, 2, 0, 1}, {32, 0, 32, 1, 0, 1},
    {32, 0, 64, 2, 0, 1},  {64, 0, 64, 1, 0, 1},  {64, 0, 32, 1, 1, 1}, {32, 32, 32, 1, 0, 1},
    {32, 0, 16, 1, 1, 1},  {16, 16, 16, 1, 0, 1}, {16, 0, 3, 1, 0, 0}};
enum { E0A, E0, E1A, E1, E2A, E2, U1, D1, U0, D0, HEAD };

int log2i(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}
int round_up(int v, int m) { return (v + m - 1) / m * m; }
int64_t layer_params(const LayerDef& d) { return (int64_t)d.cout * (d.ca + d.cb) * 27 + d.cout; }

struct Dims {
  int d, h, w;
  int64_t n() const { return (int64_t)d * h * w; }
};

}  // namespace

class Net {
 public:
  Net(int nx, int ny, int nz, int max_batch, hipStream_t s)
      : max_batch_(max_batch), stream_(s) {
    dims_[0] = Dims{nz, ny, nx};
    dims_[1] = Dims{(nz + 1) / 2, (ny + 1) / 2, (nx + 1) / 2};
    dims_[2] = Dims{(dims_[1].d + 1) / 2, (dims_[1].h + 1) / 2, (dims_[1].w + 1) / 2};
  }
  ~Net() {
    for (void* p : ptrs_) (void)hipFree(p);
  }

  // Floats of wpart_: what the weight gradients of any layer and any batch of
  // up to max_batch_ samples store.  (The chunks of a smaller batch can be
  // more than those of the largest, as their length is rounded up.)
  int64_t wpart_capacity() const {
    int64_t n = 1;
    for (int l = 0; l < kNumLayers; ++l) {
      const WgPlan p = wg_plan(l, max_batch_);
      n = std::max(n, (int64_t)p.most_chunks * p.mpad * p.npad);
    }
    return n;
  }

  // Most floats that a batch's weight gradients store in wpart_.
  int64_t wpart_need(int batch) const {
    int64_t n = 0;
    for (int l = 0; l < kNumLayers; ++l) n = std::max(n, wg_plan(l, batch).partials());
    return n;
  }

  static int64_t param_count() {
    int64_t n = 0;
    for (const LayerDef& d : kLayers) n += layer_params(d);
    return n;
  }

  int init() {
    const int64_t P = param_count();
    int64_t off = 0;
    for (int l = 0; l < kNumLayers; ++l) {
      off_[l] = off;
      off += layer_params(kLayers[l]);
    }
    VD_NET_CHECK(alloc(&params_, P));
    VD_NET_CHECK(alloc(&grad_, P));
    VD_NET_CHECK(alloc(&m1_, P));
    VD_NET_CHECK(alloc(&m2_, P));
    VD_NET_CHECK(alloc(&flag_, 1));
    if (hipMemsetAsync(params_, 0, P * sizeof(float), stream_) != hipSuccess ||
        hipMemsetAsync(m1_, 0, P * sizeof(float), stream_) != hipSuccess ||
        hipMemsetAsync(m2_, 0, P * sizeof(float), stream_) != hipSuccess)
      return VD_EHIP;
    // packed weights
    for (int l = 0; l < kNumLayers; ++l) {
      const LayerDef& d = kLayers[l];
      const int cin = d.ca + d.cb;
      const int nchunk = (27 * cin + 31) / 32, nb = (d.cout + 15) / 16;
      wf_n_[l] = (size_t)nchunk * nb * kWave * 8;
      VD_NET_CHECK(alloc(&wf_[l], wf_n_[l]));
      const int cdy = round_up(d.cout, 8);
      const int nchunk_b = (27 * cdy + 31) / 32, nb_b = (cin + 15) / 16;
      wb_n_[l] = (size_t)nchunk_b * nb_b * kWave * 8;
      VD_NET_CHECK(alloc(&wb_[l], wb_n_[l]));
    }
    // activations and gradients
    const int B = max_batch_;
    const int64_t n0 = dims_[0].n() * B, n1 = dims_[1].n() * B, n2 = dims_[2].n() * B;
    struct Want {
      uint16_t** p;
      int64_t n;
    } want[] = {
        {&x_, n0 * 8},      {&a_[E0A], n0 * 16}, {&a_[E0], n0 * 16}, {&a_[E1A], n1 * 32},
        {&a_[E1], n1 * 32}, {&a_[E2A], n2 * 64}, {&a_[E2], n2 * 64}, {&a_[U1], n1 * 32},
        {&a_[D1], n1 * 32}, {&a_[U0], n0 * 16},  {&a_[D0], n0 * 16},
        // gradients w.r.t. pre-activations, skip parts and up-sampled inputs
        {&dout_, n0 * 8},   {&g_[D0], n0 * 16},  {&g_[U0], n0 * 16}, {&skip0_, n0 * 16},
        {&dup0_, n0 * 32},  {&g_[D1], n1 * 32},  {&g_[U1], n1 * 32}, {&skip1_, n1 * 32},
        {&dup1_, n1 * 64},  {&g_[E2], n2 * 64},  {&g_[E2A], n2 * 64}, {&g_[E1], n1 * 32},
        {&g_[E1A], n1 * 32}, {&g_[E0], n0 * 16}, {&g_[E0A], n0 * 16},
    };
    for (const Want& w : want) VD_NET_CHECK(alloc(w.p, w.n));
    VD_NET_CHECK(alloc(&out_, n0 * 3));
    VD_NET_CHECK(alloc(&tgt_, n0 * 3));
    mse_blocks_ = (int)((n0 + kBlock - 1) / kBlock);
    VD_NET_CHECK(alloc(&mse_part_, mse_blocks_));
    VD_NET_CHECK(alloc(&loss_, 1));
    VD_NET_CHECK(alloc(&wpart_, wpart_capacity()));
    return pack() == hipSuccess ? VD_OK : VD_EHIP;
  }

  int set_params(const float* p, int mem) {
    const int64_t P = param_count();
    if (mem == VD_MEM_HOST) {
      if (hipMemcpyAsync(params_, p, P * 4, hipMemcpyHostToDevice, stream_) != hipSuccess)
        return VD_EHIP;
    } else {
      if (hipMemcpyAsync(params_, p, P * 4, hipMemcpyDeviceToDevice, stream_) != hipSuccess)
        return VD_EHIP;
    }
    if (hipMemsetAsync(flag_, 0, sizeof(int), stream_) != hipSuccess) return VD_EHIP;
    k_check_finite_f<<<(unsigned)((P + kBlock - 1) / kBlock), kBlock, 0, stream_>>>(params_, P,
                                                                                   flag_);
    int h = 0;
    if (hipMemcpyAsync(&h, flag_, sizeof(int), hipMemcpyDeviceToHost, stream_) != hipSuccess ||
        hipStreamSynchronize(stream_) != hipSuccess)
      return VD_EHIP;
    if (h) return VD_EINVAL;
    if (hipMemsetAsync(m1_, 0, P * 4, stream_) != hipSuccess) return VD_EHIP;
    if (hipMemsetAsync(m2_, 0, P * 4, stream_) != hipSuccess) return VD_EHIP;
    step_ = 0;
    return pack() == hipSuccess ? VD_OK : VD_EHIP;
  }

  int get_params(float* p, int mem) {
    const int64_t P = param_count();
    const hipMemcpyKind kind = mem == VD_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    if (hipMemcpyAsync(p, params_, P * 4, kind, stream_) != hipSuccess) return VD_EHIP;
    return hipStreamSynchronize(stream_) == hipSuccess ? VD_OK : VD_EHIP;
  }

  // Copies (host) or aliases (device) the input, runs the forward pass.
  int forward(const uint16_t* x, int batch, float* out, int mem) {
    VD_NET_CHECK(check_batch(batch));
    const uint16_t* xd = x;
    if (mem == VD_MEM_HOST) {
      if (hipMemcpyAsync(x_, x, dims_[0].n() * batch * 16, hipMemcpyHostToDevice, stream_) !=
          hipSuccess)
        return VD_EHIP;
      xd = x_;
    }
    float* od = mem == VD_MEM_HOST ? out_ : out;
    if (run_forward(xd, batch, od) != hipSuccess) return VD_EHIP;
    if (mem == VD_MEM_HOST) {
      if (hipMemcpyAsync(out, out_, dims_[0].n() * batch * 12, hipMemcpyDeviceToHost, stream_) !=
          hipSuccess)
        return VD_EHIP;
      if (hipStreamSynchronize(stream_) != hipSuccess) return VD_EHIP;
    }
    return VD_OK;
  }

  // Forward + loss + backward; the gradient lands in grad_.
  int gradients(const uint16_t* x, const float* target, int batch, int mem) {
    VD_NET_CHECK(check_batch(batch));
    const uint16_t* xd = x;
    const float* td = target;
    if (mem == VD_MEM_HOST) {
      const int64_t n = dims_[0].n() * batch;
      if (hipMemcpyAsync(x_, x, n * 16, hipMemcpyHostToDevice, stream_) != hipSuccess ||
          hipMemcpyAsync(tgt_, target, n * 12, hipMemcpyHostToDevice, stream_) != hipSuccess)
        return VD_EHIP;
      xd = x_;
      td = tgt_;
    }
    if (run_forward(xd, batch, out_) != hipSuccess) return VD_EHIP;
    if (run_backward(xd, td, batch) != hipSuccess) return VD_EHIP;
    return VD_OK;
  }

  int copy_grad(float* g, int mem) {
    const int64_t P = param_count();
    const hipMemcpyKind kind = mem == VD_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    if (hipMemcpyAsync(g, grad_, P * 4, kind, stream_) != hipSuccess) return VD_EHIP;
    return hipStreamSynchronize(stream_) == hipSuccess ? VD_OK : VD_EHIP;
  }

  int read_loss(double* loss) {
    if (hipMemcpyAsync(loss, loss_, sizeof(double), hipMemcpyDeviceToHost, stream_) != hipSuccess)
      return VD_EHIP;
    return hipStreamSynchronize(stream_) == hipSuccess ? VD_OK : VD_EHIP;
  }

  int adam(float lr) {
    ++step_;
    const double b1 = 0.9, b2 = 0.999;
    const float eps = 1e-8f;
    const float c1 = (float)(1.0 - std::pow(b1, (double)step_));
    const float c2 = (float)(1.0 - std::pow(b2, (double)step_));
    const int64_t P = param_count();
    k_adam<<<(unsigned)((P + kBlock - 1) / kBlock), kBlock, 0, stream_>>>(
        params_, grad_, m1_, m2_, P, lr, (float)b1, (float)(1.0 - b1), (float)b2,
        (float)(1.0 - b2), eps, c1, c2);
    if (hipGetLastError() != hipSuccess) return VD_EHIP;
    return pack() == hipSuccess ? VD_OK : VD_EHIP;
  }

 private:
  struct WgPlan {
    int mpad, npad, nb, mtiles, nchunks;
    int most_chunks;  // nchunks of no smaller batch is above this
    int64_t vox_per_chunk;
    int64_t partials() const { return (int64_t)nchunks * mpad * npad; }
  };

  template <typename P>
  int alloc(P** p, int64_t count) {
    void* q = nullptr;
    if (hipMalloc(&q, (size_t)std::max<int64_t>(count, 1) * sizeof(P)) != hipSuccess) {
      (void)hipGetLastError();
      return VD_ENOMEM;
    }
    ptrs_.push_back(q);
    *p = static_cast<P*>(q);
    return VD_OK;
  }

  int check_batch(int batch) const {
    return (batch >= 1 && batch <= max_batch_) ? VD_OK : VD_EINVAL;
  }

  int level_in(int l) const {  // grid level of a layer's input
    static const int lv[kNumLayers] = {0, 0, 0, 1, 1, 2, 2, 1, 1, 0, 0};
    return lv[l];
  }
  int level_out(int l) const {
    static const int lv[kNumLayers] = {0, 0, 1, 1, 2, 2, 1, 1, 0, 0, 0};
    return lv[l];
  }

  WgPlan wg_plan(int l, int batch) const {
    const LayerDef& d = kLayers[l];
    const int cin = d.ca + d.cb;
    WgPlan p;
    p.mpad = round_up(27 * cin + 1, 64);
    p.nb = (d.cout + 15) / 16;
    p.npad = 16 * p.nb;
    p.mtiles = p.mpad / 64;
    const int64_t M = dims_[level_out(l)].n() * batch;
    const int64_t steps = (M + kWgVox - 1) / kWgVox;
    int64_t nch = (512 + p.mtiles - 1) / p.mtiles;
    if (nch > steps) nch = steps;
    if (nch < 1) nch = 1;
    p.most_chunks = (int)nch;
    p.vox_per_chunk = (steps + nch - 1) / nch * kWgVox;
    p.nchunks = (int)((M + p.vox_per_chunk - 1) / p.vox_per_chunk);
    return p;
  }

  // Geometry and sources of layer l's forward convolution.
  ConvArgs fwd_args(int l, const uint16_t* x, int batch) const {
    const LayerDef& d = kLayers[l];
    ConvArgs A{};
    static const int src_a[kNumLayers] = {-1, E0A, E0, E1A, E1, E2A, E2, U1, D1, U0, D0};
    static const int src_b[kNumLayers] = {-1, -1, -1, -1, -1, -1, -1, E1, -1, E0, -1};
    A.a = src_a[l] < 0 ? x : a_[src_a[l]];
    A.ca = d.ca;
    A.b = src_b[l] < 0 ? nullptr : a_[src_b[l]];
    A.cb = d.cb;
    A.cin = d.ca + d.cb;
    A.lcin = log2i(A.cin);
    A.ktot = 27 * A.cin;
    A.nchunk = (A.ktot + 31) / 32;
    A.mode = d.up ? kGatherUp : kGatherPlain;
    A.stride = d.stride;
    const Dims& si = dims_[level_in(l)];
    const Dims& so = dims_[level_out(l)];
    A.sd = si.d; A.sh = si.h; A.sw = si.w;
    A.od = so.d; A.oh = so.h; A.ow = so.w;
    A.batch = batch;
    A.cout = d.cout;
    A.nb = (d.cout + 15) / 16;
    A.w = reinterpret_cast<const uint4*>(wf_[l]);
    A.bias = params_ + off_[l] + (int64_t)d.cout * A.cin * 27;
    A.relu = d.relu;
    if (l == HEAD) {
      A.out_f32 = nullptr;  // set by the caller
    } else {
      A.dst0 = const_cast<uint16_t*>(a_[l]);
      A.c0 = d.cout;
    }
    return A;
  }

  // Bricks: 512 voxels (8 rows x 4 planes) where that leaves more than 600
  // workgroups, else 128, else 64 with the output channels split over
  // workgroups too: a workgroup waits for its staging, and only others on its
  // compute unit cover that, while small bricks load more halo (64 input
  // channels or stride 2: at most 128 voxels, for their LDS).  Forward pass at
  // 64^3 / 57x41x50 with two samples: 181 / 210 us with lines at 256 and 128
  // workgroups, 165 / 178 with 600 for the first, 157 / 192 with 600 for the
  // second; the batch-4 training step is the same with each.
  template <int CIN, int NB, int S>
  hipError_t launch_conv_t(const ConvArgs& A) {
    auto run = [&](auto kernel, int by, int bz, int groups) {
      const int64_t n = (int64_t)((A.ow + kConvX - 1) / kConvX) * ((A.oh + by - 1) / by) *
                        ((A.od + bz - 1) / bz) * A.batch;
      kernel<<<dim3((unsigned)n, groups), kBlock, 0, stream_>>>(A);
      return hipGetLastError();
    };
    const int64_t rows = (int64_t)((A.ow + kConvX - 1) / kConvX) * A.oh * A.od * A.batch;
    if constexpr (S == 1 && CIN < 64) {
      if (rows / 32 > 600) return run(k_conv<CIN, NB, S, 8, 4>, 8, 4, 1);
    }
    if (rows / 8 > 600) return run(k_conv<CIN, NB, S, 4, 2>, 4, 2, 1);
    return run(k_conv<CIN, 1, S, 4, 1>, 4, 1, NB);
  }

  hipError_t launch_conv(const ConvArgs& A) {
    switch (1000 * A.stride + 10 * A.cin + A.nb) {
      case 1081: return launch_conv_t<8, 1, 1>(A);
      case 1161: return launch_conv_t<16, 1, 1>(A);
      case 1162: return launch_conv_t<16, 2, 1>(A);
      case 1321: return launch_conv_t<32, 1, 1>(A);
      case 1322: return launch_conv_t<32, 2, 1>(A);
      case 1324: return launch_conv_t<32, 4, 1>(A);
      case 1642: return launch_conv_t<64, 2, 1>(A);
      case 1644: return launch_conv_t<64, 4, 1>(A);
      case 2162: return launch_conv_t<16, 2, 2>(A);
      case 2324: return launch_conv_t<32, 4, 2>(A);
      default: return hipErrorInvalidValue;
    }
  }

  hipError_t run_forward(const uint16_t* x, int batch, float* out) {
    for (int l = 0; l < kNumLayers; ++l) {
      ConvArgs A = fwd_args(l, x, batch);
      if (l == HEAD) A.out_f32 = out;
      const hipError_t e = launch_conv(A);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }

  // Input gradient of layer l as a convolution of its output gradient gy
  // (cdy channels) over grid `out_level`.
  ConvArgs dgrad_args(int l, const uint16_t* gy, int batch) const {
    const LayerDef& d = kLayers[l];
    ConvArgs A{};
    const int cdy = round_up(d.cout, 8);
    A.a = gy;
    A.ca = cdy;
    A.cin = cdy;
    A.lcin = log2i(cdy);
    A.ktot = 27 * cdy;
    A.nchunk = (A.ktot + 31) / 32;
    A.stride = 1;
    const Dims& gd = dims_[level_out(l)];
    // the data gradient lives on the forward input grid (the up-sampled one
    // for the up layers)
    const Dims& xd = d.up ? dims_[level_out(l)] : dims_[level_in(l)];
    A.mode = d.stride == 2 ? kGatherTransposed2 : kGatherPlain;
    A.sd = gd.d; A.sh = gd.h; A.sw = gd.w;
    A.od = xd.d; A.oh = xd.h; A.ow = xd.w;
    A.batch = batch;
    A.cout = d.ca + d.cb;
    A.nb = (A.cout + 15) / 16;
    A.w = reinterpret_cast<const uint4*>(wb_[l]);
    return A;
  }

  // The staged block of k_wgrad: the most 32-voxel steps (at most 16) whose
  // dY and input lines a workgroup loads at once, 64 KB, so that two workgroups
  // fit a compute unit's LDS.  Returns the LDS bytes, 0 where not even one step
  // fits (rows of some 600 voxels) and k_wgrad_gather runs instead.
  static size_t wgrad_block(const ConvArgs& A, int co, WgradArgs* G) {
    const int S = A.stride, W = S * (A.ow - 1) + 3;
    for (int ks = 16; ks >= 1; ks /= 2) {
      // voxels of a block lie in at most this many rows and planes
      const int64_t rows = (32 * ks + A.ow - 2) / A.ow + 1;
      const int64_t planes = (rows + A.oh - 2) / A.oh + 1;
      const int64_t lines = S * (rows - 1) + (3 - S) * (planes - 1) + 3;
      const int64_t groups = 32 * ks * co * 2 + lines * W * 2;
      if (groups > kWgLoads * kWgThreads) continue;
      G->ksteps = ks;
      G->lines = (int)lines;
      return (size_t)groups * 16;
    }
    return 0;
  }

  hipError_t launch_wgrad(int l, const uint16_t* x, const uint16_t* gy, int batch) {
    const WgPlan p = wg_plan(l, batch);
    if (p.partials() > wpart_capacity()) return hipErrorInvalidValue;
    const ConvArgs A = fwd_args(l, x, batch);
    WgradArgs G{};
    G.dy = gy;
    G.cdy = round_up(kLayers[l].cout, 8);
    G.mpad = p.mpad;
    G.npad = p.npad;
    G.vox_per_chunk = p.vox_per_chunk;
    G.partial = wpart_;
    const size_t lds = wgrad_block(A, p.nb, &G);
    if (lds > 0) {
      const dim3 grid(p.nchunks, 3 * ((A.cin + 15) / 16));
      auto run = [&](auto kernel) { kernel<<<grid, kWgThreads, lds, stream_>>>(A, G); };
      switch (10 * A.stride + p.nb) {
        case 11: run(k_wgrad<1, 1>); break;
        case 12: run(k_wgrad<2, 1>); break;
        case 14: run(k_wgrad<4, 1>); break;
        case 22: run(k_wgrad<2, 2>); break;
        case 24: run(k_wgrad<4, 2>); break;
        default: return hipErrorInvalidValue;
      }
    } else {
      const dim3 grid(p.mtiles, p.nchunks);
      switch (p.nb) {
        case 1: k_wgrad_gather<1><<<grid, kBlock, 0, stream_>>>(A, G); break;
        case 2: k_wgrad_gather<2><<<grid, kBlock, 0, stream_>>>(A, G); break;
        case 4: k_wgrad_gather<4><<<grid, kBlock, 0, stream_>>>(A, G); break;
        default: return hipErrorInvalidValue;
      }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const LayerDef& d = kLayers[l];
    k_wgrad_reduce<<<(unsigned)((p.mpad * p.npad + kWave - 1) / kWave), kWave, 0, stream_>>>(
        wpart_, p.nchunks, p.mpad, p.npad, d.ca + d.cb, d.cout, grad_ + off_[l]);
    return hipGetLastError();
  }

  hipError_t launch_upsum(const uint16_t* dup, int fine_level, const uint16_t* src, int level,
                          int C, int batch, uint16_t* g) {
    const Dims& f = dims_[fine_level];
    const Dims& c = dims_[level];
    const int64_t total = c.n() * batch * C;
    k_upsum<<<(unsigned)((total + kBlock - 1) / kBlock), kBlock, 0, stream_>>>(
        dup, f.d, f.h, f.w, src, c.d, c.h, c.w, C, batch, g);
    return hipGetLastError();
  }

#define VD_NET_HIP(expr)                 \
  do {                                   \
    const hipError_t e_ = (expr);        \
    if (e_ != hipSuccess) return e_;     \
  } while (0)

  hipError_t run_backward(const uint16_t* x, const float* target, int batch) {
    const int64_t npb = dims_[0].n();
    const int64_t M = npb * batch;
    const unsigned mb = (unsigned)((M + kBlock - 1) / kBlock);
    k_mse<<<mb, kBlock, 0, stream_>>>(out_, target, npb, batch, dout_, mse_part_);
    VD_NET_HIP(hipGetLastError());
    k_mse_finalize<<<1, kBlock, 0, stream_>>>(mse_part_, (int)mb, 1.0 / (double)M, loss_);
    VD_NET_HIP(hipGetLastError());
    ConvArgs A;
    // head
    VD_NET_HIP(launch_wgrad(HEAD, x, dout_, batch));
    A = dgrad_args(HEAD, dout_, batch);
    A.dst0 = g_[D0]; A.c0 = 16; A.mask0 = a_[D0];
    VD_NET_HIP(launch_conv(A));
    // d0 = relu(conv([u0, e0]))
    VD_NET_HIP(launch_wgrad(D0, x, g_[D0], batch));
    A = dgrad_args(D0, g_[D0], batch);
    A.dst0 = g_[U0]; A.c0 = 16; A.mask0 = a_[U0];
    A.dst1 = skip0_; A.c1 = 16;
    VD_NET_HIP(launch_conv(A));
    // u0 = relu(conv(up(d1)))
    VD_NET_HIP(launch_wgrad(U0, x, g_[U0], batch));
    A = dgrad_args(U0, g_[U0], batch);
    A.dst0 = dup0_; A.c0 = 32;
    VD_NET_HIP(launch_conv(A));
    VD_NET_HIP(launch_upsum(dup0_, 0, a_[D1], 1, 32, batch, g_[D1]));
    // d1 = relu(conv([u1, e1]))
    VD_NET_HIP(launch_wgrad(D1, x, g_[D1], batch));
    A = dgrad_args(D1, g_[D1], batch);
    A.dst0 = g_[U1]; A.c0 = 32; A.mask0 = a_[U1];
    A.dst1 = skip1_; A.c1 = 32;
    VD_NET_HIP(launch_conv(A));
    // u1 = relu(conv(up(e2)))
    VD_NET_HIP(launch_wgrad(U1, x, g_[U1], batch));
    A = dgrad_args(U1, g_[U1], batch);
    A.dst0 = dup1_; A.c0 = 64;
    VD_NET_HIP(launch_conv(A));
    VD_NET_HIP(launch_upsum(dup1_, 1, a_[E2], 2, 64, batch, g_[E2]));
    // e2
    VD_NET_HIP(launch_wgrad(E2, x, g_[E2], batch));
    A = dgrad_args(E2, g_[E2], batch);
    A.dst0 = g_[E2A]; A.c0 = 64; A.mask0 = a_[E2A];
    VD_NET_HIP(launch_conv(A));
    // e2a (stride 2): its input e1 also feeds d1 through the skip
    VD_NET_HIP(launch_wgrad(E2A, x, g_[E2A], batch));
    A = dgrad_args(E2A, g_[E2A], batch);
    A.dst0 = g_[E1]; A.c0 = 32; A.mask0 = a_[E1]; A.add0 = skip1_;
    VD_NET_HIP(launch_conv(A));
    // e1
    VD_NET_HIP(launch_wgrad(E1, x, g_[E1], batch));
    A = dgrad_args(E1, g_[E1], batch);
    A.dst0 = g_[E1A]; A.c0 = 32; A.mask0 = a_[E1A];
    VD_NET_HIP(launch_conv(A));
    // e1a (stride 2): its input e0 also feeds d0 through the skip
    VD_NET_HIP(launch_wgrad(E1A, x, g_[E1A], batch));
    A = dgrad_args(E1A, g_[E1A], batch);
    A.dst0 = g_[E0]; A.c0 = 16; A.mask0 = a_[E0]; A.add0 = skip0_;
    VD_NET_HIP(launch_conv(A));
    // e0
    VD_NET_HIP(launch_wgrad(E0, x, g_[E0], batch));
    A = dgrad_args(E0, g_[E0], batch);
    A.dst0 = g_[E0A]; A.c0 = 16; A.mask0 = a_[E0A];
    VD_NET_HIP(launch_conv(A));
    // e0a (the input needs no gradient)
    VD_NET_HIP(launch_wgrad(E0A, x, g_[E0A], batch));
    return hipSuccess;
  }

  hipError_t pack() {
    for (int l = 0; l < kNumLayers; ++l) {
      const LayerDef& d = kLayers[l];
      const int cin = d.ca + d.cb;
      const float* W = params_ + off_[l];
      const int nchunk = (27 * cin + 31) / 32, nb = (d.cout + 15) / 16;
      k_pack_fwd<<<(unsigned)((wf_n_[l] + kBlock - 1) / kBlock), kBlock, 0, stream_>>>(
          W, cin, d.cout, nchunk, nb, wf_[l]);
      VD_NET_HIP(hipGetLastError());
      const int cdy = round_up(d.cout, 8);
      const int nchunk_b = (27 * cdy + 31) / 32, nb_b = (cin + 15) / 16;
      k_pack_dgrad<<<(unsigned)((wb_n_[l] + kBlock - 1) / kBlock), kBlock, 0, stream_>>>(
          W, cin, d.cout, cdy, nchunk_b, nb_b, wb_[l]);
      VD_NET_HIP(hipGetLastError());
    }
    return hipSuccess;
  }

  Dims dims_[3];
  int max_batch_;
  hipStream_t stream_;
  std::vector<void*> ptrs_;
  int64_t off_[kNumLayers] = {};
  float *params_ = nullptr, *grad_ = nullptr, *m1_ = nullptr, *m2_ = nullptr;
  int* flag_ = nullptr;
  uint16_t* wf_[kNumLayers] = {};
  uint16_t* wb_[kNumLayers] = {};
  size_t wf_n_[kNumLayers] = {}, wb_n_[kNumLayers] = {};
  uint16_t* x_ = nullptr;
  uint16_t* a_[kNumLayers] = {};
  uint16_t* g_[kNumLayers] = {};
  uint16_t *dout_ = nullptr, *skip0_ = nullptr, *skip1_ = nullptr, *dup0_ = nullptr,
           *dup1_ = nullptr;
  float *out_ = nullptr, *tgt_ = nullptr, *wpart_ = nullptr;
  double *mse_part_ = nullptr, *loss_ = nullptr;
  int mse_blocks_ = 0;
  int64_t step_ = 0;
};

}  // namespace net
}  // namespace vd

struct vd_net {
  vd::net::Net* impl;
};

extern "C" {

int64_t vd_net_param_count(void) { return vd::net::Net::param_count(); }

int vd_net_create(int32_t nx, int32_t ny, int32_t nz, int32_t max_batch, void* stream,
                  vd_net** out) {
  if (!out) return VD_EINVAL;
  *out = nullptr;
  if (nx < 1 || ny < 1 || nz < 1 || max_batch < 1) return VD_EINVAL;
  if ((int64_t)nx * ny * nz * max_batch > (int64_t)1 << 28) return VD_EINVAL;
  vd::net::Net* impl =
      new (std::nothrow) vd::net::Net(nx, ny, nz, max_batch, static_cast<hipStream_t>(stream));
  if (!impl) return VD_ENOMEM;
  const int rc = impl->init();
  if (rc != VD_OK) {
    delete impl;
    return rc;
  }
  vd_net* h = new (std::nothrow) vd_net{impl};
  if (!h) {
    delete impl;
    return VD_ENOMEM;
  }
  *out = h;
  return VD_OK;
}

int vd_debug_net_partials(int32_t nx, int32_t ny, int32_t nz, int32_t max_batch, int32_t batch,
                          int64_t* need, int64_t* have) {
  if (nx < 1 || ny < 1 || nz < 1 || batch < 1 || batch > max_batch || !need || !have)
    return VD_EINVAL;
  if ((int64_t)nx * ny * nz * max_batch > (int64_t)1 << 28) return VD_EINVAL;
  const vd::net::Net plan(nx, ny, nz, max_batch, nullptr);
  *need = plan.wpart_need(batch);
  *have = plan.wpart_capacity();
  return VD_OK;
}

int vd_net_destroy(vd_net* n) {
  if (!n) return VD_OK;
  delete n->impl;
  delete n;
  return VD_OK;
}

int vd_net_set_params(vd_net* n, const float* params, int32_t mem) {
  if (!n || !params || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
  return n->impl->set_params(params, mem);
}

int vd_net_get_params(vd_net* n, float* params, int32_t mem) {
  if (!n || !params || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
  return n->impl->get_params(params, mem);
}

int vd_net_forward(vd_net* n, const uint16_t* x, int32_t batch, float* out, int32_t mem) {
  if (!n || !x || !out || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
  return n->impl->forward(x, batch, out, mem);
}

int vd_net_gradients(vd_net* n, const uint16_t* x, const float* target, int32_t batch, float* grad,
                     double* loss, int32_t mem) {
  if (!n || !x || !target || !grad || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE))
    return VD_EINVAL;
  int rc = n->impl->gradients(x, target, batch, mem);
  if (rc != VD_OK) return rc;
  rc = n->impl->copy_grad(grad, mem);
  if (rc != VD_OK) return rc;
  return loss ? n->impl->read_loss(loss) : VD_OK;
}

int vd_net_train_step(vd_net* n, const uint16_t* x, const float* target, int32_t batch, float lr,
                      int32_t mem, double* loss) {
  if (!n || !x || !target || (mem != VD_MEM_HOST && mem != VD_MEM_DEVICE)) return VD_EINVAL;
  if (!(lr >= 0.0f) || !std::isfinite(lr)) return VD_EINVAL;
  int rc = n->impl->gradients(x, target, batch, mem);
  if (rc != VD_OK) return rc;
  if (loss) {
    rc = n->impl->read_loss(loss);
    if (rc != VD_OK) return rc;
  }
  return n->impl->adam(lr);
}

}  // extern "C"
