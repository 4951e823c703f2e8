// gfx950 kernels of the fluence denoiser: BF16 MFMA convolutions with FP32
// accumulation (forward, input gradient, weight gradient) and the
// element-wise steps around them.
//
// Activations are channels-last BF16 arrays [voxel][channel], voxels
// x-fastest.  A convolution is an implicit GEMM: rows m are the voxels of
// the grid the kernel iterates, columns n the output channels, and the
// reduction index k = tap * Cin + ci walks the input channels of every tap.
// The A operand is gathered from the activation array on the fly (zero
// outside the volume), the B operand is the weight matrix packed as BF16
// rows Bt[n][k] (k contiguous, padded with zeros to the tile sizes).
// Four gather geometries cover the forward pass and the input gradient of
// all three layer kinds:
//   kConv3   y[v] += x[v + d(t)] W[t]        (3x3x3, stride 1, zero pad)
//   kConv3T  y[v] += x[v - d(t)] W[t]        (its input gradient)
//   kDown    y[v] += x[2v + e(t)] W[t]       (2x2x2, stride 2)
//   kUp      y[2v + e(c)] = x[v] W[c]        (2x2x2 transposed, one parity
//                                             class c per grid z-slice)
// The down layer's input gradient is a kUp product and the up layer's a
// kDown product, each with transposed weights.
//
// Kernels: conv_kernel is the generic implicit GEMM (every geometry);
// 3x3x3 products get dedicated kernels that stage operands in LDS --
// conv3_resident_kernel (exactly 32 gathered channels on large grids: the
// weights stay in LDS, input planes stream in by direct global-to-LDS
// loads), conv3_brick_kernel (other multiples of 32 gathered channels),
// conv3_scalar_kernel (one gathered channel) -- and up_kernel the stride-2 up
// products.  Weight gradients: wgrad_brick_kernel (3x3x3) and
// wgrad_pair_kernel (stride 2) for channels in eights,
// wgrad_onechannel_kernel, wgrad_slab_kernel for other output channels, and
// wgrad_kernel for the rest.  Products that launch too few workgroups split their
// reduction and finish in split_reduce_kernel / wgrad_reduce_kernel, which
// add FP32 partial sums in a fixed order.
//
// MFMA v_mfma_f32_16x16x32_bf16: lane l supplies A[l % 16][8(l / 16) + j]
// and B[8(l / 16) + j][l % 16] (j = 0..7) and receives
// D[4(l / 16) + i][l % 16] (i = 0..3).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "nn_internal.hpp"

namespace mcx {
namespace nn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

constexpr int kBM = 64;   // rows per workgroup tile (4 waves x 16)
constexpr int kBK = 32;   // reduction step
constexpr int kPadK = 8;  // LDS row padding (bf16 elements)

// float -> bf16 bits, round to nearest even: the kernels run with FP32
// denormals kept and round-to-nearest-even, so gfx950's conversion
// instruction gives exactly that rounding, denormals included (NaN stays NaN)
__device__ __forceinline__ uint16_t to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
__device__ __forceinline__ float from_bf16(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// voxel index of the A operand for row m (grid coordinates z, y, x) and
// tap t, or -1 when it lies outside the input volume
__device__ __forceinline__ int64_t gather_at(const ConvArgs& a, int z, int y, int x, int t) {
  int iz, iy, ix;
  if (a.geo == kConv3 || a.geo == kConv3T) {
    const int s = a.geo == kConv3 ? 1 : -1;
    iz = z + s * (t / 9 - 1);
    iy = y + s * ((t / 3) % 3 - 1);
    ix = x + s * (t % 3 - 1);
    if (iz < 0 || iy < 0 || ix < 0 || iz >= a.in_d || iy >= a.in_h || ix >= a.in_w) return -1;
  } else if (a.geo == kDown) {
    iz = 2 * z + (t >> 2);
    iy = 2 * y + ((t >> 1) & 1);
    ix = 2 * x + (t & 1);
  } else {
    iz = z;
    iy = y;
    ix = x;
  }
  return (static_cast<int64_t>(iz) * a.in_h + iy) * a.in_w + ix;
}

// ------------------------------------------------------------ forward GEMM
// One workgroup: 64 rows x 16*NB columns; wave w owns rows 16w..16w+15.
// KS reduction steps of 32 are staged per pair of barriers.
template <int NB, bool kVec, int KS>
__global__ void __launch_bounds__(256) conv_kernel(ConvArgs a) {
  __shared__ uint16_t sA[kBM][KS * kBK + kPadK];
  __shared__ uint16_t sB[16 * NB][KS * kBK + kPadK];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t m0 = static_cast<int64_t>(blockIdx.x) * kBM;
  const int n0 = blockIdx.y * 16 * NB;
  const int cls = blockIdx.z;  // parity class of kUp, else 0
  const int64_t M = static_cast<int64_t>(a.batch) * a.d * a.h * a.w;  // the images' rows
  const int koff = a.geo == kUp ? cls * a.cin : 0;

  // this thread's A row and 8-wide k chunk for the loads
  const int lr = tid >> 2, lc = (tid & 3) * 8;
  const int64_t lm = m0 + lr;
  int lz = 0, ly = 0, lx = 0;
  const uint16_t* x_img = a.x;  // the row's image
  if (lm < M) {
    lx = static_cast<int>(lm % a.w);
    ly = static_cast<int>((lm / a.w) % a.h);
    lz = static_cast<int>(lm / (static_cast<int64_t>(a.w) * a.h));
    if (a.batch > 1) {
      const int img = lz / a.d;
      lz -= img * a.d;
      x_img += static_cast<int64_t>(img) * a.in_d * a.in_h * a.in_w * a.cin;
    }
  }

  floatx4 acc[NB], tot[NB];  // the current range's sums, those of the ranges before it
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = tot[j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // this thread's 8 k of row lr of the A tile at reduction step k0
  auto load_a = [&](int k0) -> uint4 {
    const int k = k0 + lc;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (lm >= M) return v;
    if constexpr (kVec) {
      if (k < a.k) {
        const int t = k / a.cin, ci = k - t * a.cin;
        const int64_t src = gather_at(a, lz, ly, lx, t);
        if (src >= 0) v = *reinterpret_cast<const uint4*>(x_img + src * a.cin + ci);
      }
    } else {
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        e[j] = 0;
        const int kk = k + j;
        if (kk < a.k) {
          const int t = kk / a.cin, ci = kk - t * a.cin;
          const int64_t src = gather_at(a, lz, ly, lx, t);
          if (src >= 0) e[j] = x_img[src * a.cin + ci];
        }
      }
      v = make_uint4(e[0] | (uint32_t(e[1]) << 16), e[2] | (uint32_t(e[3]) << 16),
                     e[4] | (uint32_t(e[5]) << 16), e[6] | (uint32_t(e[7]) << 16));
    }
    return v;
  };
  // this thread's 8 k of one B row (threads 0 .. 64*NB-1), Bt[n][koff + k]
  const bool has_b = tid < 16 * NB * 4;
  const int br = tid >> 2, bc = (tid & 3) * 8;
  const uint16_t* brow = a.bt + static_cast<int64_t>(n0 + br) * a.kpad + koff;
  auto load_b = [&](int k0) -> uint4 {
    const int k = k0 + bc;
    if (k + 8 <= a.k && (koff & 7) == 0) return *reinterpret_cast<const uint4*>(brow + k);
    uint16_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = (k + j < a.k) ? brow[k + j] : 0;
    return make_uint4(e[0] | (uint32_t(e[1]) << 16), e[2] | (uint32_t(e[3]) << 16),
                      e[4] | (uint32_t(e[5]) << 16), e[6] | (uint32_t(e[7]) << 16));
  };

  // software pipeline: the next stage's global loads are in flight while
  // the matrix cores work on the current stage's tiles
  constexpr int kStage = KS * kBK;
  // kDown in a.ranges > 1 ranges (each a multiple of kStage; the last ends at
  // a.k): all of them, or with gridDim.z = a.ranges this workgroup's
  int k_begin = 0, k_end = a.k, range_len = a.k;
  if (a.geo != kUp && a.ranges > 1) {
    range_len = (a.k / a.ranges + kStage - 1) / kStage * kStage;
    if (gridDim.z > 1) {
      k_begin = static_cast<int>(blockIdx.z) * range_len;
      k_end = min(a.k, k_begin + range_len);
    }
  }
  int range_end = k_begin + range_len;
  uint4 va[KS], vb[KS];
#pragma unroll
  for (int q = 0; q < KS; ++q) {
    va[q] = k_begin + q * kBK < k_end ? load_a(k_begin + q * kBK) : make_uint4(0u, 0u, 0u, 0u);
    vb[q] = has_b && k_begin + q * kBK < k_end ? load_b(k_begin + q * kBK)
                                               : make_uint4(0u, 0u, 0u, 0u);
  }
  for (int k0 = k_begin; k0 < k_end; k0 += kStage) {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      *reinterpret_cast<uint4*>(&sA[lr][q * kBK + lc]) = va[q];
      if (has_b) *reinterpret_cast<uint4*>(&sB[br][q * kBK + bc]) = vb[q];
    }
    __syncthreads();
    if (k0 + kStage < k_end) {
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        const int kn = k0 + kStage + q * kBK;
        va[q] = kn < k_end ? load_a(kn) : make_uint4(0u, 0u, 0u, 0u);
        if (has_b) vb[q] = kn < k_end ? load_b(kn) : make_uint4(0u, 0u, 0u, 0u);
      }
    }
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      if (k0 + q * kBK >= k_end) break;
      const bf16x8 af =
          *reinterpret_cast<const bf16x8*>(&sA[wave * 16 + (lane & 15)][q * kBK + (lane >> 4) * 8]);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const bf16x8 bf =
            *reinterpret_cast<const bf16x8*>(&sB[j * 16 + (lane & 15)][q * kBK + (lane >> 4) * 8]);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc[j], 0, 0, 0);
      }
    }
    if (k0 + kStage == range_end && range_end < k_end) {  // the next range starts from zero
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        tot[j] = k0 + kStage == range_len ? acc[j] : tot[j] + acc[j];
        acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      range_end += range_len;
    }
    __syncthreads();
  }
  if (k_end > k_begin + range_len) {  // several ranges, added in order
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = tot[j] + acc[j];
  }

  // epilogue: bias, skip, ReLU, store; with gridDim.z = S > 1 (kDown only)
  // the raw sums of this reduction range go to part[z][m][cout] instead
  const bool split = a.geo != kUp && gridDim.z > 1;
  float* part = split ? a.part + static_cast<int64_t>(blockIdx.z) * M * a.cout : nullptr;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + wave * 16 + (lane >> 4) * 4 + i;
    if (m >= M) continue;
    int64_t o = m;
    if (a.geo == kUp) {
      // grids hold at most 2^30 voxels: 32-bit arithmetic
      const uint32_t mm = static_cast<uint32_t>(m);
      const uint32_t x = mm % static_cast<uint32_t>(a.w);
      const uint32_t rest = mm / static_cast<uint32_t>(a.w);
      const uint32_t y = rest % static_cast<uint32_t>(a.h);
      const uint32_t z = rest / static_cast<uint32_t>(a.h);
      o = (static_cast<int64_t>(2 * z + (cls >> 2)) * (2 * a.h) + 2 * y + ((cls >> 1) & 1)) *
              (2 * a.w) + 2 * x + (cls & 1);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = n0 + j * 16 + (lane & 15);
      if (n >= a.cout) continue;
      if (split) {
        part[o * a.cout + n] = acc[j][i];
        continue;
      }
      float v = acc[j][i] + (a.bias ? a.bias[n] : 0.f);
      if (a.skip) v += from_bf16(a.skip[o * a.cout + n]);
      if (a.relu) v = fmaxf(v, 0.f);
      if (a.y_f32)
        static_cast<float*>(a.y)[o * a.cout + n] = v;
      else
        static_cast<uint16_t*>(a.y)[o * a.cout + n] = to_bf16(v);
    }
  }
}

// ------------------------------------------------------- 2x2x2 stride-2 up
// kUp with cin a multiple of 32 and cout one of 8: a wave owns 16 R voxels of
// the small grid, 32 output channels and a range of the parity classes.  The
// voxels are the columns of the matrix product and the channels its rows,
// so a lane's sums are 8 channels of one output voxel (row 4 g + i of the two
// products is channel 8 g + 4 j + i): bias, skip and ReLU are applied and 16
// bytes stored from registers, and the two x classes fill whole cache lines.
// The voxels' channels (KC chunks of 32; 0: any number, read again for each
// class) stay in registers for all classes; weights come from L1 and L2.
// No LDS, no barrier.
// What bounds it: at full resolution the bytes of skip and output, 3.6 of
// the 4.8 TB/s that a large copy reaches.  Measured: eight images of 32^3
// 64 -> 32 224 -> 84 us, one 22.8 -> 12.4 (the generic kernel stored 2 bytes a
// lane and each class half lines), 16^3 128 -> 64 12.2 -> 7.7.
template <int KC, int R>
__global__ void __launch_bounds__(256) up_kernel(ConvArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int64_t M = static_cast<int64_t>(a.batch) * a.d * a.h * a.w;
  const int64_t m0 = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * (16 * R);
  if (m0 >= M) return;
  const int n0 = blockIdx.y * 32, n = n0 + 8 * g;
  const bool has_n = n < a.cout;
  const int nc = 8 / static_cast<int>(gridDim.z);
  const int chunks = KC > 0 ? KC : a.cin / kBK;

  const uint16_t* xp[R];
  int64_t ob[R];  // output voxel of class 0, or -1 past the rows
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int64_t m = m0 + 16 * q + r;
    const uint32_t mm = static_cast<uint32_t>(m < M ? m : M - 1);  // at most 2^30 voxels
    const uint32_t x = mm % static_cast<uint32_t>(a.w), t = mm / static_cast<uint32_t>(a.w);
    const uint32_t y = t % static_cast<uint32_t>(a.h), z = t / static_cast<uint32_t>(a.h);
    xp[q] = a.x + static_cast<int64_t>(mm) * a.cin + 8 * g;
    ob[q] = m < M && has_n
                ? (static_cast<int64_t>(2 * z) * (2 * a.h) + 2 * y) * (2 * a.w) + 2 * x
                : -1;
  }
  bf16x8 xf[KC > 0 ? KC : 1][R];
  if constexpr (KC > 0) {
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int q = 0; q < R; ++q) xf[c][q] = *reinterpret_cast<const bf16x8*>(xp[q] + c * kBK);
  }
  const uint16_t* wp[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    wp[j] = a.bt + static_cast<int64_t>(n0 + 8 * (r >> 2) + 4 * j + (r & 3)) * a.kpad + 8 * g;
  float bias[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) bias[i] = a.bias && has_n ? a.bias[n + i] : 0.f;

  for (int cls = blockIdx.z * nc; cls < (static_cast<int>(blockIdx.z) + 1) * nc; ++cls) {
    const int64_t oc = (static_cast<int64_t>(cls >> 2) * (2 * a.h) + ((cls >> 1) & 1)) * (2 * a.w) +
                       (cls & 1);
    uint4 sk[R];
    if (a.skip) {
#pragma unroll
      for (int q = 0; q < R; ++q)
        sk[q] = ob[q] >= 0 ? *reinterpret_cast<const uint4*>(a.skip + (ob[q] + oc) * a.cout + n)
                           : make_uint4(0u, 0u, 0u, 0u);
    }
    floatx4 acc[R][2];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q][0] = acc[q][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int c, const bf16x8 (&v)[R]) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 wf = *reinterpret_cast<const bf16x8*>(wp[j] + cls * a.cin + c * kBK);
#pragma unroll
        for (int q = 0; q < R; ++q)
          acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, v[q], acc[q][j], 0, 0, 0);
      }
    };
    if constexpr (KC > 0) {
#pragma unroll
      for (int c = 0; c < KC; ++c) step(c, xf[c]);
    } else {
      for (int c = 0; c < chunks; ++c) {
#pragma unroll
        for (int q = 0; q < R; ++q)
          xf[0][q] = *reinterpret_cast<const bf16x8*>(xp[q] + c * kBK);
        step(c, xf[0]);
      }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (ob[q] < 0) continue;
      const int64_t e0 = (ob[q] + oc) * a.cout + n;
      float v[8];
      const uint16_t* sh = reinterpret_cast<const uint16_t*>(&sk[q]);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = acc[q][i >> 2][i & 3] + bias[i];
        if (a.skip) v[i] += from_bf16(sh[i]);
        if (a.relu) v[i] = fmaxf(v[i], 0.f);
      }
      if (a.y_f32) {
        float4* y = reinterpret_cast<float4*>(static_cast<float*>(a.y) + e0);
        y[0] = make_float4(v[0], v[1], v[2], v[3]);
        y[1] = make_float4(v[4], v[5], v[6], v[7]);
      } else {
        uint4 o;
        uint16_t* oh = reinterpret_cast<uint16_t*>(&o);
#pragma unroll
        for (int i = 0; i < 8; ++i) oh[i] = to_bf16(v[i]);
        *reinterpret_cast<uint4*>(static_cast<uint16_t*>(a.y) + e0) = o;
      }
    }
  }
}

// ------------------------------------------------- 3x3x3 conv from an LDS brick
// The source of the zero padding of direct global-to-LDS loads: 64 KB of
// zeros, each lane reading its own 16 bytes (offset by workgroup and load),
// so that zero chunks spread over many cache lines instead of sending every
// compute unit to one address.
constexpr int kZeroChunks = 4096;
__device__ __align__(16) uint4 g_zero16[kZeroChunks];

__device__ __forceinline__ void load_lds16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)(src),
                                   (__attribute__((address_space(3))) void*)(dst), 16, 0, 0);
}

// Wait until at most N of this wave's global memory operations are
// outstanding (they complete in order); other counters are not waited for.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "six bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Where the 16-byte chunk j of a row of 64 bytes lies: slot j ^ row_slot(row
// index / 4) for weight rows, j ^ plane_slot(y) for voxel rows of planes 6
// voxels wide.  16-byte LDS reads are served 16 lanes at a time (lanes 0-3,
// 12-15, 20-27, then 4-11, 16-19, 28-31, and so in the upper half: measured,
// no bank conflicts this way against one in two reads when the slots follow
// the rows as if lanes 0-15 went together), and these spread each such group
// over all 64 banks.
__device__ __forceinline__ int row_slot(int q) { return ((q ^ (q >> 1)) & 1) << 1 | ((q >> 1) & 1); }
__device__ __forceinline__ int plane_slot(int y) { return (y & 1) << 1; }

// A workgroup barrier that waits for this wave's LDS operations but not, as
// __syncthreads does, for all its global loads: those in flight towards LDS
// are waited for by count (wait_vm) where they are due.
__device__ __forceinline__ void barrier_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// bits 0 .. n - 1: which of the positions p0 .. p0 + n - 1 are outside [0, size)
__device__ __forceinline__ uint32_t outside(int p0, int n, int size) {
  uint32_t m = 0;
  for (int i = 0; i < n; ++i) m |= p0 + i < 0 || p0 + i >= size ? 1u << i : 0u;
  return m;
}

// kConv3 / kConv3T with cin a multiple of 32: a workgroup owns 16 NB output
// channels and walks the 4 x 4 x 4MZ tiles of output voxels blockIdx.x,
// + gridDim.x, ... of all images.  Per chunk of 32 input channels the
// 6 x 6 x (4MZ + 2) input brick (tile plus halo, zero outside the volume) is
// staged in LDS, and the chunk's weights pass through a ring of stages of
// three taps (one dz, dy).  Four compute waves, kWN of them side by side along
// the channels, take their fragments of voxels from the brick and of weights
// from the stage and issue no global loads; two loader waves stream the
// weights (three stages ahead) and the next chunk's brick, also across tiles,
// by direct global-to-LDS loads, each waiting only for the loads of the stage
// that is due.  One barrier per stage.
// What bounds it: for many images the matrix instructions, 0.73 of the 1.12
// PFLOP/s that a large matrix product reaches; for one image filling and
// draining the pipeline.  Measured: a barrier for every plane of 9 taps and
// weights loaded by the waves that compute, 32^3 64 -> 64 30 us; the loader
// waves 20.2; eight images with a workgroup for each tile 134, walking the tiles
// (the next one's bricks loading meanwhile) with 4 x 4 x 16 voxels, 16-byte stores
// and fragments read across the stages 79.  16^3 128 -> 128: 63 -> 39 for
// eight, 16.6 for one; 8^3 256 -> 256: 34 and 10.3 + 4.6.
// Layouts: brick voxel v at v * 64 bytes, its 16-byte chunk j in slot
// j ^ plane_slot(y); weight row n at n * 64 bytes, chunk j in slot
// j ^ row_slot((n >> kShift) & 3).  The channels are the product's rows and the voxels
// its columns, as in up_kernel: with two channel blocks per wave a lane's sums
// are 8 consecutive channels of one voxel (row 4 g + i of block j of a pair is
// channel 8 g + 4 j + i), with one block 4.
// The chunks are reduced in a.ranges equal ranges whose sums are added in
// order.  With gridDim.z = a.ranges > 1 each grid z index takes one of them
// and stores its raw sums to the workspace part[z][out voxel][cout] for
// split_reduce_kernel to finish; with gridDim.z == 1 a workgroup takes all.
template <int NB, int MZ>
struct Brick {
  static constexpr int kBZ = 4 * MZ + 2;
  static constexpr int kPieces = 36 * kBZ * 4;               // 16-byte pieces of a brick
  static constexpr int kBrickLoads = (kPieces + 63) / 64;    // wave loads of a brick
  static constexpr int kBrickBytes = kBrickLoads * 1024;
  static constexpr int kStageLoads = 3 * NB;                 // wave loads of a stage
  static constexpr int kStageBytes = kStageLoads * 1024;
  static constexpr int kRing = 4;
  static constexpr int kWN = NB == 4 && MZ < 4 ? 2 : 1;      // compute waves along the channels
  static constexpr int kSW = MZ * kWN;                       // z-slices per wave
  static constexpr int kCW = NB / kWN;                       // 16-channel blocks per wave
  static constexpr int kShift = kCW >= 2 ? 3 : 2;
};

// The workgroup's i-th tile: its first voxel (bx, by, bz) and image
template <int MZ>
__device__ __forceinline__ void brick_tile(const ConvArgs& a, int i, int& img, int& bx, int& by,
                                           int& bz) {
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2;
  const int ntile = tx_n * ty_n * ((a.d + 4 * MZ - 1) / (4 * MZ));
  const int t = blockIdx.x + i * gridDim.x;
  img = t / ntile;
  const int tile = t - img * ntile;
  bx = (tile % tx_n) * 4;
  by = ((tile / tx_n) % ty_n) * 4;
  bz = (tile / (tx_n * ty_n)) * (4 * MZ);
}

// Loader wave LW (0 or 1) of a workgroup: every other wave load.
template <int NB, int MZ, int LW>
__device__ __forceinline__ void brick_loader(const ConvArgs& a, char* s_br, char* s_w, int lane,
                                             int n0, int c_begin, int nchunks, int ntiles) {
  using K = Brick<NB, MZ>;
  constexpr int kB = (K::kBrickLoads + 1 - LW) / 2;  // this wave's loads of a brick
  constexpr int kW = (K::kStageLoads + 1 - LW) / 2;  // and of a stage
  // Per brick load: this lane's offset from the tile's first voxel, and the
  // brick position as one bit for each of x, y and z (bit 31: no such
  // piece), which a tile's mask of what lies outside the volume tells apart
  // in two instructions.
  const uint16_t* zero = reinterpret_cast<const uint16_t*>(g_zero16) +
                         ((blockIdx.x * 64 + lane) & (kZeroChunks - 1)) * 8;
  int64_t rel[kB];
  uint32_t pos[kB];
#pragma unroll
  for (int k = 0; k < kB; ++k) {
    const int p = (2 * k + LW) * 64 + lane;
    const int v = p >> 2, x = v % 6, y = (v / 6) % 6, z = v / 36;
    const int j = (p & 3) ^ plane_slot(y);
    rel[k] = ((static_cast<int64_t>(z - 1) * a.in_h + (y - 1)) * a.in_w + (x - 1)) * a.cin + j * 8;
    pos[k] = p < K::kPieces ? 1u << x | 1u << (6 + y) | 1u << (12 + z) : 1u << 31;
  }
  // the next brick: chunk b_chunk of tile b_tile, into buffer b_buf
  const uint16_t* x0 = nullptr;
  uint32_t out = 0;
  int b_tile = 0, b_chunk = 0, b_buf = 0;
  auto load_brick = [&]() {
    if (b_chunk == 0) {
      int img, bx, by, bz;
      brick_tile<MZ>(a, b_tile, img, bx, by, bz);
      x0 = a.x + (((static_cast<int64_t>(img) * a.in_d + bz) * a.in_h + by) * a.in_w + bx) * a.cin +
           c_begin;
      out = 1u << 31 | outside(bx - 1, 6, a.in_w) | outside(by - 1, 6, a.in_h) << 6 |
            outside(bz - 1, K::kBZ, a.in_d) << 12;
    }
    const uint16_t* xc = x0 + b_chunk * 32;
    char* dst = s_br + b_buf * K::kBrickBytes;
#pragma unroll
    for (int k = 0; k < kB; ++k)
      load_lds16(pos[k] & out ? zero : xc + rel[k], dst + (2 * k + LW) * 1024);
    b_buf ^= 1;
    if (++b_chunk == nchunks) {
      b_chunk = 0;
      ++b_tile;
    }
  };
  // weights: row lane / 4 of each 16 of the workgroup's 16 NB rows
  uint32_t off[NB];
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    const int n = 16 * rb + (lane >> 2);
    off[rb] = static_cast<uint32_t>(n0 + n) * static_cast<uint32_t>(a.kpad) +
              ((lane & 3) ^ row_slot((n >> K::kShift) & 3)) * 8;
  }
  // the next stage: taps 3 w_row .. of chunk w_chunk, into slot w_slot
  int w_row = 0, w_chunk = 0, w_slot = 0;
  auto load_stage = [&]() {
    char* dst = s_w + w_slot * K::kStageBytes;
#pragma unroll
    for (int k = 0; k < kW; ++k) {
      const int b = 2 * k + LW, dx = b / NB, rb = b % NB;
      const uint16_t* base = a.bt + (3 * w_row + dx) * a.cin + c_begin + w_chunk * 32;
      load_lds16(base + off[rb], dst + b * 1024);
    }
    w_slot = (w_slot + 1) & (K::kRing - 1);
    if (++w_row == 9) {
      w_row = 0;
      if (++w_chunk == nchunks) w_chunk = 0;
    }
  };
  const int C = ntiles * nchunks, S = 9 * C;
  load_brick();
#pragma unroll
  for (int s = 0; s < 3; ++s) load_stage();
  wait_vm<2 * kW>();
  barrier_lds();  // the first stage has landed
  int chunk = 0, js = 0;  // s = 9 chunk + js, chunks counted over all tiles
  for (int s = 0; s < S; ++s) {
    // stages up to s + 1 have landed once at most the loads of stage s + 2,
    // and of a brick asked for just before it (at js == 0), are outstanding
    if (s + 2 >= S)
      wait_vm<0>();
    else if (js == 1 && chunk + 1 < C)
      wait_vm<kW + kB>();
    else
      wait_vm<kW>();
    barrier_lds();
    if (js == 0 && chunk + 1 < C) load_brick();
    if (s + 3 < S) load_stage();
    if (++js == 9) {
      js = 0;
      ++chunk;
    }
  }
}

// N (4 or 8) consecutive channels of output voxel o: bias, skip, ReLU and
// store, or the raw sums to part.  vec: channels in eights, aligned operands.
template <int N>
__device__ __forceinline__ void put_channels(const ConvArgs& a, const floatx4 (&sum)[N / 4],
                                             int64_t o, int n, float* part, bool vec) {
  const int64_t e0 = o * a.cout + n;
  if (vec) {
    if (n >= a.cout) return;
    if (part) {
#pragma unroll
      for (int j = 0; j < N / 4; ++j) *reinterpret_cast<floatx4*>(part + e0 + 4 * j) = sum[j];
      return;
    }
    float v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = sum[i >> 2][i & 3] + (a.bias ? a.bias[n + i] : 0.f);
    typedef uint32_t words __attribute__((ext_vector_type(N / 2)));
    if (a.skip) {
      const words sk = *reinterpret_cast<const words*>(a.skip + e0);
#pragma unroll
      for (int i = 0; i < N; ++i)
        v[i] += from_bf16(static_cast<uint16_t>(i & 1 ? sk[i >> 1] >> 16 : sk[i >> 1] & 0xffffu));
    }
    if (a.relu) {
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = fmaxf(v[i], 0.f);
    }
    if (a.y_f32) {
#pragma unroll
      for (int j = 0; j < N / 4; ++j)
        *reinterpret_cast<floatx4*>(static_cast<float*>(a.y) + e0 + 4 * j) =
            floatx4{v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
    } else {
      words u;
#pragma unroll
      for (int i = 0; i < N; i += 2) u[i >> 1] = to_bf16(v[i]) | uint32_t(to_bf16(v[i + 1])) << 16;
      *reinterpret_cast<words*>(static_cast<uint16_t*>(a.y) + e0) = u;
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (n + i >= a.cout) return;
    float v = sum[i >> 2][i & 3];
    if (part) {
      part[e0 + i] = v;
      continue;
    }
    v += a.bias ? a.bias[n + i] : 0.f;
    if (a.skip) v += from_bf16(a.skip[e0 + i]);
    if (a.relu) v = fmaxf(v, 0.f);
    if (a.y_f32)
      static_cast<float*>(a.y)[e0 + i] = v;
    else
      static_cast<uint16_t*>(a.y)[e0 + i] = to_bf16(v);
  }
}

template <int NB, int MZ>
__global__ void __launch_bounds__(384) conv3_brick_kernel(ConvArgs a, int vec) {
  using K = Brick<NB, MZ>;
  __shared__ __align__(16) char s_br[2 * K::kBrickBytes];
  __shared__ __align__(16) char s_w[K::kRing * K::kStageBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles = a.batch * ((a.w + 3) >> 2) * ((a.h + 3) >> 2) * ((a.d + 4 * MZ - 1) / (4 * MZ));
  const int ntiles = (tiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  const int n0 = blockIdx.y * 16 * NB;
  const int split_len = a.cin / static_cast<int>(gridDim.z);  // a multiple of kBK
  const int c_begin = static_cast<int>(blockIdx.z) * split_len;
  const int nchunks = split_len / kBK;
  if (wave == 4) {
    brick_loader<NB, MZ, 0>(a, s_br, s_w, lane, n0, c_begin, nchunks, ntiles);
    return;
  }
  if (wave == 5) {
    brick_loader<NB, MZ, 1>(a, s_br, s_w, lane, n0, c_begin, nchunks, ntiles);
    return;
  }

  const int sgn = a.geo == kConv3 ? 1 : -1;
  const int r = lane & 15;            // this lane's voxel (r & 3, r >> 2) of a slice
  const int ox = r & 3, oy = r >> 2;
  const int g = lane >> 4;            // and its 16-byte chunk of the 32 channels
  const int z0 = wave / K::kWN * K::kSW;          // the wave's first slice
  const int cb = wave % K::kWN * K::kCW;          // and 16-channel block
  // byte offsets in a stage of this lane's weight rows
  int wo[K::kCW];
#pragma unroll
  for (int c = 0; c < K::kCW; ++c) {
    const int n = K::kCW >= 2 ? 16 * cb + 32 * (c >> 1) + 8 * (r >> 2) + 4 * (c & 1) + (r & 3)
                              : 16 * cb + r;
    wo[c] = n * 64 + ((g ^ row_slot((n >> K::kShift) & 3)) << 4);
  }
  const int64_t vox = static_cast<int64_t>(a.d) * a.h * a.w;
  float* part = gridDim.z > 1 ? a.part + static_cast<int64_t>(blockIdx.z) * a.batch * vox * a.cout
                              : nullptr;
  const int range_chunks = gridDim.z > 1 ? nchunks : nchunks / a.ranges;

  // this lane's voxel offset for dy = -1, 0, 1 (in the taps' order)
  int ao[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int yy = oy + 1 + sgn * (k - 1);
    ao[k] = ((z0 + 1) * 36 + yy * 6 + ox + 1) * 64 + ((g ^ plane_slot(yy)) << 4);
  }
  bf16x8 af[2][K::kSW], bf[2][K::kCW];
  auto read = [&](const char* br, int slot, int t, bf16x8 (&fa)[K::kSW], bf16x8 (&fb)[K::kCW]) {
    const char* wst = s_w + slot * K::kStageBytes + (t % 3) * 16 * NB * 64;
    const char* ab = br + sgn * ((t / 9 - 1) * 36 + (t % 3 - 1)) * 64 + ao[(t / 3) % 3];
#pragma unroll
    for (int c = 0; c < K::kCW; ++c) fb[c] = *reinterpret_cast<const bf16x8*>(wst + wo[c]);
#pragma unroll
    for (int q = 0; q < K::kSW; ++q) fa[q] = *reinterpret_cast<const bf16x8*>(ab + q * 36 * 64);
  };
  int slot = 0, buf = 0;
  barrier_lds();  // the first stage has landed
  read(s_br, 0, 0, af[0], bf[0]);
  for (int ti = 0; ti < ntiles; ++ti) {
    // the current range's sums, those of the ranges before it
    floatx4 acc[K::kSW][K::kCW], tot[K::kSW][K::kCW];
#pragma unroll
    for (int q = 0; q < K::kSW; ++q)
#pragma unroll
      for (int c = 0; c < K::kCW; ++c) acc[q][c] = tot[q][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    int range_left = range_chunks;
    for (int chunk = 0; chunk < nchunks; ++chunk) {
      if (range_left == 0) {  // the next range starts from zero
#pragma unroll
        for (int q = 0; q < K::kSW; ++q)
#pragma unroll
          for (int c = 0; c < K::kCW; ++c) {
            tot[q][c] = chunk == range_chunks ? acc[q][c] : tot[q][c] + acc[q][c];
            acc[q][c] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
        range_left = range_chunks;
      }
      --range_left;
      // taps t = 3 row + dx; each one's fragments are read while the tap
      // before runs, across stages and chunks
      const char* br = s_br + buf * K::kBrickBytes;
#pragma unroll
      for (int t = 0; t < 27; ++t) {
        if (t % 3 == 0) barrier_lds();  // this stage and the next have landed
        if (t < 26) {
          if (t % 3 == 2) slot = (slot + 1) & (K::kRing - 1);
          read(br, slot, t + 1, af[(t + 1) & 1], bf[(t + 1) & 1]);
        } else {
          slot = (slot + 1) & (K::kRing - 1);
          buf ^= 1;
          if (chunk + 1 < nchunks || ti + 1 < ntiles)
            read(s_br + buf * K::kBrickBytes, slot, 0, af[1], bf[1]);
        }
        __builtin_amdgcn_sched_barrier(0);  // those reads ahead of the matrix instructions
#pragma unroll
        for (int q = 0; q < K::kSW; ++q)
#pragma unroll
          for (int c = 0; c < K::kCW; ++c)
            acc[q][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[t & 1][c], af[t & 1][q],
                                                                acc[q][c], 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < K::kSW; ++q) af[0][q] = af[1][q];
#pragma unroll
      for (int c = 0; c < K::kCW; ++c) bf[0][c] = bf[1][c];
    }
    if (range_chunks < nchunks) {  // several ranges, added in order
#pragma unroll
      for (int q = 0; q < K::kSW; ++q)
#pragma unroll
        for (int c = 0; c < K::kCW; ++c) acc[q][c] = tot[q][c] + acc[q][c];
    }
    // epilogue: this lane's voxel of each of the wave's slices
    int img, bx, by, bz;
    brick_tile<MZ>(a, ti, img, bx, by, bz);
    const int x = bx + ox, y = by + oy;
#pragma unroll
    for (int q = 0; q < K::kSW; ++q) {
      const int z = bz + z0 + q;
      if (x >= a.w || y >= a.h || z >= a.d) continue;
      const int64_t o = img * vox + (static_cast<int64_t>(z) * a.h + y) * a.w + x;
      if constexpr (K::kCW >= 2) {
#pragma unroll
        for (int c = 0; c < K::kCW; c += 2) {
          const floatx4 v[2] = {acc[q][c], acc[q][c + 1]};
          put_channels<8>(a, v, o, n0 + 16 * (cb + c) + 8 * g, part, vec);
        }
      } else {
        const floatx4 v[1] = {acc[q][0]};
        put_channels<4>(a, v, o, n0 + 16 * cb + 4 * g, part, vec);
      }
    }
  }
}

// --------------------------------- 3x3x3 conv, 32 input channels, weights resident
// kConv3 / kConv3T with cin == 32 on large grids (the full-resolution layers):
// the reduction is one chunk of 32 channels, so a workgroup's weights (27
// taps x 16 NB output channels) fit in LDS and stay there while the
// workgroup walks its columns of tiles (columns blockIdx.x, blockIdx.x +
// gridDim.x, ... of all images, each of 4 x 4 x 8-voxel tiles stacked along z).  Waves 0-3
// compute (wave w: z-slices 2w, 2w + 1 of the tile, NB 16-column MFMA blocks
// each) and leave each tile's outputs in LDS; wave 4 streams the input
// planes of the column (6 x 6 voxels of 32 channels, z = -1 .. 8 per tile
// count + 1) into a ring of plane slots with direct global-to-LDS loads,
// A tiles ahead (a tile reuses two planes of the previous one and loads
// eight; zeros outside the volume come from g_zero16); waves 5 and 6
// write the previous tile's outputs from LDS to global memory.  The compute
// waves issue no global memory operation; each data wave waits only for its
// own transfers (the plane wave for all but the newest A - 1 tiles' loads,
// which complete in issue order): one barrier per tile, which does not wait
// for transfers (barrier_lds).  What bounds a tile are the compute waves'
// fragment reads from LDS, 4 KB per 4 matrix instructions with both operands
// read for every tap, so the weights of most taps stay in registers, and the
// plane wave's address arithmetic, so a plane's addresses are the last ones'
// plus a plane.  Measured at 64^3, 32 -> 32 channels: 24.5 -> 21.6 us with the
// weights in registers, -> 21 with the cheap addresses; input gradient folded
// (kGrad) 26.5 -> 25.3; eight images 148 -> 137, where the matrix instructions
// alone take 103 at the rate of a large product; 32 -> 16 channels, eight images,
// 116 -> 89.  Plane layout: voxel
// (y, x) of the plane at (y * 6 + x) * 64 bytes, its 16-byte chunk j
// (channels 8j .. 8j + 7) in slot j ^ plane_slot(y); the weights of output
// channel n likewise at n * 64 bytes, chunk j in slot j ^ row_slot((n >> 2) & 3).
constexpr int kResPlane = 36 * 64;  // bytes per plane slot

// Byte offset of byte `byte` of local voxel vl's outputs in an output tile
// of the resident kernel (rows of NB 16 outputs of ES bytes).  For NB == 2
// the rows and 16-byte chunks are permuted within each group of 16 voxels
// by g = (vl >> 2) & 3, the group of lanes that writes them in the
// epilogue (lanes 16 g .. 16 g + 15), so that each epilogue write
// instruction hits 64 different banks: BF16 rows (64 bytes) go to row
// vl ^ g with the two 32-byte halves swapped for odd g; FP32 rows (128
// bytes) to row vl ^ (g >> 1) with the halves swapped for odd g.
template <int NB, int ES>
__device__ __forceinline__ int sout_off(int vl, int byte) {
  if constexpr (NB != 2) {
    return vl * (16 * NB * ES) + byte;
  } else {
    const int g = (vl >> 2) & 3;
    if constexpr (ES == 2)
      return (vl ^ g) * 64 + (byte ^ ((g & 1) << 5));
    else
      return (vl ^ (g >> 1)) * 128 + (byte ^ ((g & 1) << 6));
  }
}

// Makes the compiler produce v here (an empty instruction that takes it as
// input): loads of values used only under a condition are otherwise moved
// into the conditional code, one load and one wait at a time.
__device__ __forceinline__ void pin(const uint4& v) {
  asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
}

// tiles of planes in flight: all that fit in LDS beside the weights and
// two output tiles (three, or two for 32 FP32 output columns)
constexpr int res_ahead(int nb, bool f32) { return nb == 2 && f32 ? 2 : 3; }
// taps whose weights the compute waves hold in registers: what 256 registers
// per lane leave room for
constexpr int res_taps(int nb) { return nb == 2 ? 18 : 27; }
// taps between reading a fragment from LDS and using it: a tap's 2 NB matrix
// instructions take 64 or 32 cycles, an LDS read about 150
constexpr int kAhead = 3;

// kGrad: an input gradient with the next backward step folded in
// (ConvArgs::gmask): the compute waves leave FP32 sums in LDS, the output
// waves apply the ReLU mask, round to BF16, store, and sum each channel's
// BF16 values; the workgroup's sums go to gpart.
template <int NB, bool kF32, bool kGrad>
__global__ void __launch_bounds__(448) conv3_resident_kernel(ConvArgs a) {
  constexpr int NC = 16 * NB;                 // output channels of the workgroup
  constexpr int ES = kF32 || kGrad ? 4 : 2;   // bytes per output in LDS
  constexpr int A = res_ahead(NB, kF32 || kGrad);
  constexpr int kRing = 8 * A + 10;           // plane slots: tiles k .. k + A
  __shared__ uint4 sW[27][NC][4];
  __shared__ uint4 sRing[kRing * kResPlane / 16];
  __shared__ uint4 sOut[2][128 * NC * ES / 16];  // 128 voxels x NC outputs
  __shared__ float sBias[NC];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2, tz_n = (a.d + 7) >> 3;
  const int ncol = tx_n * ty_n;  // columns of an image
  const int64_t in_vox = static_cast<int64_t>(a.in_d) * a.in_h * a.in_w;
  const int64_t out_vox = static_cast<int64_t>(a.d) * a.h * a.w;
  const int n0 = blockIdx.y * NC;
  const int ncols = min(NC, a.cout - n0);

  // weights and bias, once.  The weights by direct global-to-LDS loads of
  // 64 slots (1 KB) each, all in flight together, from every wave but the
  // plane wave (which starts on the first column's planes meanwhile): lane
  // L of block bl fills slot 64 bl + L, i.e. row (16 bl + L / 4) of the
  // flattened [27][NC] rows, chunk slot L % 4, with the chunk
  // (L % 4) ^ row_slot((row >> 2) & 3) of that row.
  if (wave != 4) {
    const int w6 = wave < 4 ? wave : wave - 1;
    for (int bl = w6; bl < 27 * NC / 16; bl += 6) {
      const int fr = 16 * bl + (lane >> 2), tt = fr / NC, row = fr % NC;
      const int j = (lane & 3) ^ row_slot((row >> 2) & 3);
      __builtin_amdgcn_global_load_lds(
          (__attribute__((address_space(1))) void*)(a.bt + static_cast<int64_t>(n0 + row) * a.kpad +
                                                     tt * 32 + j * 8),
          (__attribute__((address_space(3))) void*)(reinterpret_cast<char*>(sW) + bl * 1024), 16, 0,
          0);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wave's weight transfers have landed
  }
  for (int i = tid; i < NC; i += blockDim.x) sBias[i] = (a.bias && i < ncols) ? a.bias[n0 + i] : 0.f;

  // wave 4: the planes of a column, z = -1, 0, ..., each into the next ring
  // slot (z + 1) % kRing in three loads of 64 lanes (144 chunks: the last load
  // has 16 lanes).  Per load the lane's address of the next plane; in the
  // volume's x and y it moves by a plane, elsewhere it stays on zeros.
  int64_t rel[3];
  uint32_t pos[3];  // the chunk's voxel in the plane, one bit for x and one for y
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int c = k * 64 + lane;  // chunk slot within the plane
    const int vp = c >> 2, y = vp / 6, x = vp % 6, j = (c & 3) ^ plane_slot(y);
    rel[k] = (static_cast<int64_t>(y - 1) * a.in_w + (x - 1)) * 32 + j * 8;
    pos[k] = 1u << x | 1u << (6 + y);
  }
  const uint16_t* zero = reinterpret_cast<const uint16_t*>(g_zero16) +
                         ((blockIdx.x * 64 + lane) & (kZeroChunks - 1)) * 8;
  const uint16_t* next[3];
  int64_t step[3];
  int p_z = 0, p_slot = 0;  // the next plane and its slot
  auto start_column = [&](int64_t v0, int bx, int by) {
    const uint32_t out = outside(bx - 1, 6, a.in_w) | outside(by - 1, 6, a.in_h) << 6;
    const int64_t plane = static_cast<int64_t>(a.in_h) * a.in_w * 32;
    const uint16_t* x0 = a.x + (v0 + static_cast<int64_t>(by) * a.in_w + bx) * 32 - plane;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      next[k] = pos[k] & out ? zero : x0 + rel[k];
      step[k] = pos[k] & out ? 0 : plane;
    }
    p_z = -1;
    p_slot = 0;
  };
  auto load_plane = [&]() {
    const bool zin = p_z >= 0 && p_z < a.in_d;
    char* slot = reinterpret_cast<char*>(sRing) + p_slot * kResPlane;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k < 2 || lane < 16) load_lds16(zin ? next[k] : zero, slot + k * 1024);
      next[k] += step[k];
    }
    ++p_z;
    if (++p_slot == kRing) p_slot = 0;
  };
  // waves 5 and 6: the outputs of the tile at (bx, by, bz) from sOut[b] to
  // y, every other 64 pieces each
  const int s0 = lane + 64 * (wave - 5);
  // kGrad: this lane's channel sums, and the ReLU mask of its pieces of
  // the next tile to store (loaded a tile ahead: the output path is the
  // kernel's bound)
  constexpr int kGP = NC * 2 / 16;  // 16-byte BF16 pieces per voxel
  float gsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint4 gm[kGP];
  auto piece = [&](int64_t v0, int bx, int by, int bz, int mm, int64_t& e0) {
    const int i = s0 + 128 * mm;
    const int vl = i / kGP, k = i % kGP;
    const int x = bx + (vl & 3), y = by + ((vl >> 2) & 3), z = bz + (vl >> 4);
    e0 = (v0 + (static_cast<int64_t>(z) * a.h + y) * a.w + x) * a.cout + n0 + k * 8;
    return x < a.w && y < a.h && z < a.d;
  };
  auto load_mask = [&](int64_t v0, int bx, int by, int bz) {
#pragma unroll
    for (int mm = 0; mm < kGP; ++mm) {
      int64_t e0;
      gm[mm] = piece(v0, bx, by, bz, mm, e0) ? *reinterpret_cast<const uint4*>(a.gmask + e0)
                                          : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  auto store_out = [&](int64_t v0, int bx, int by, int bz, int b) {
    const char* src = reinterpret_cast<const char*>(sOut[b]);
    if constexpr (kGrad) {
      // 16-byte BF16 pieces of 8 channels (NC == cout): a lane always has
      // channels 8 (lane % 4) .. + 7; their FP32 sums (32 bytes at byte 32 i
      // of the tile for piece i) are read from LDS first
      float fv[kGP][8];
#pragma unroll
      for (int mm = 0; mm < kGP; ++mm) {
        const int i = s0 + 128 * mm;  // piece i: voxel i / kGP, channels 8 (i % kGP) ..
        const uint4* q = reinterpret_cast<const uint4*>(src + sout_off<NB, 4>(i / kGP, (i % kGP) * 32));
        *reinterpret_cast<uint4*>(&fv[mm][0]) = q[0];
        *reinterpret_cast<uint4*>(&fv[mm][4]) = q[1];
      }
#pragma unroll
      for (int mm = 0; mm < kGP; ++mm) {
        pin(*reinterpret_cast<uint4*>(&fv[mm][0]));
        pin(*reinterpret_cast<uint4*>(&fv[mm][4]));
      }
#pragma unroll
      for (int mm = 0; mm < kGP; ++mm) {
        int64_t e0;
        if (!piece(v0, bx, by, bz, mm, e0)) continue;
        const float* f = fv[mm];
        const uint16_t* mh = reinterpret_cast<const uint16_t*>(&gm[mm]);
        uint4 o;
        uint16_t* oh = reinterpret_cast<uint16_t*>(&o);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float v = f[j];
          if (!(from_bf16(mh[j]) > 0.f)) v = 0.f;
          oh[j] = to_bf16(v);
          gsum[j] += from_bf16(oh[j]);
        }
        *reinterpret_cast<uint4*>(static_cast<uint16_t*>(a.y) + e0) = o;
      }
      return;
    }
    const int out_bytes = ncols * ES;
    if (ncols == NC && (a.cout * ES) % 16 == 0) {  // whole rows of 16-byte pieces
      constexpr int per = NC * ES / 16;
      // all of this lane's pieces from LDS first: one wait for the LDS
      // reads (which queue behind the compute waves' fragment reads), not
      // one per piece
      uint4 v[per];
#pragma unroll
      for (int mm = 0; mm < per; ++mm)  // piece i = s0 + 128 mm at byte 16 i of the tile
        v[mm] = *reinterpret_cast<const uint4*>(
            src + sout_off<NB, ES>((s0 + 128 * mm) / per, (s0 + 128 * mm) % per * 16));
#pragma unroll
      for (int mm = 0; mm < per; ++mm) pin(v[mm]);
#pragma unroll
      for (int mm = 0; mm < per; ++mm) {  // 128 * per pieces, 128 per step
        const int i = s0 + 128 * mm;
        const int vl = i / per, k = i % per;
        const int x = bx + (vl & 3), y = by + ((vl >> 2) & 3), z = bz + (vl >> 4);
        if (x >= a.w || y >= a.h || z >= a.d) continue;
        const int64_t o = v0 + (static_cast<int64_t>(z) * a.h + y) * a.w + x;
        *reinterpret_cast<uint4*>(static_cast<char*>(a.y) + (o * a.cout + n0) * ES + k * 16) =
            v[mm];
      }
    } else if (out_bytes % 16 == 0 && (a.cout * ES) % 16 == 0) {
      const int per = out_bytes / 16;
      for (int i = s0; i < 128 * per; i += 128) {
        const int vl = i / per, k = i % per;
        const int x = bx + (vl & 3), y = by + ((vl >> 2) & 3), z = bz + (vl >> 4);
        if (x >= a.w || y >= a.h || z >= a.d) continue;
        const int64_t o = v0 + (static_cast<int64_t>(z) * a.h + y) * a.w + x;
        *reinterpret_cast<uint4*>(static_cast<char*>(a.y) + (o * a.cout + n0) * ES + k * 16) =
            *reinterpret_cast<const uint4*>(src + sout_off<NB, ES>(vl, k * 16));
      }
    } else {
      for (int i = s0; i < 128 * ncols; i += 128) {
        const int vl = i / ncols, n = i % ncols;
        const int x = bx + (vl & 3), y = by + ((vl >> 2) & 3), z = bz + (vl >> 4);
        if (x >= a.w || y >= a.h || z >= a.d) continue;
        const int64_t o = v0 + (static_cast<int64_t>(z) * a.h + y) * a.w + x;
        if constexpr (kF32)
          static_cast<float*>(a.y)[o * a.cout + n0 + n] =
              *reinterpret_cast<const float*>(src + sout_off<NB, ES>(vl, n * 4));
        else
          static_cast<uint16_t*>(a.y)[o * a.cout + n0 + n] =
              *reinterpret_cast<const uint16_t*>(src + sout_off<NB, ES>(vl, n * 2));
      }
    }
  };

  // The three kinds of wave meet at the same barriers: one before the first
  // column (the weights have landed), per column one once the first tile's
  // planes have, one per tile, and one after the column's last outputs.
  barrier_lds();
  if (wave == 4) {
    for (int gc = blockIdx.x; gc < ncol * a.batch; gc += gridDim.x) {
      const int img = gc / ncol, col = gc - img * ncol;
      const int bx = (col % tx_n) * 4, by = (col / tx_n) * 4;
      start_column(img * in_vox, bx, by);
      // planes -1 .. 8 min(tz_n, A): the first A tiles; wait for tile 0's
      // (all loads but those of the tiles after it, 24 per tile)
      const int zend = 8 * min(tz_n, A);
      for (int z = -1; z <= zend; ++z) load_plane();
      const int first = min(tz_n, A) - 1;
      if (first >= 2)
        wait_vm<48>();
      else if (first == 1)
        wait_vm<24>();
      else
        wait_vm<0>();
      barrier_lds();
      for (int k = 0; k < tz_n; ++k) {
        // the eight new planes of tile k + A (their slots held planes no tile
        // from k on needs); then wait until tile k + 1's planes have arrived:
        // all loads but those of the tiles after it (24 per tile)
        const int last = min(k + A, tz_n - 1);  // the newest tile loaded
        if (k + A < tz_n)
          for (int z = 0; z < 8; ++z) load_plane();
        const int pending = last - (k + 1);  // tiles whose loads may stay in flight
        if (pending >= 2)
          wait_vm<48>();
        else if (pending == 1)
          wait_vm<24>();
        else
          wait_vm<0>();
        barrier_lds();
      }
      barrier_lds();
    }
  } else if (wave >= 5) {
    for (int gc = blockIdx.x; gc < ncol * a.batch; gc += gridDim.x) {
      const int img = gc / ncol, col = gc - img * ncol;
      const int bx = (col % tx_n) * 4, by = (col / tx_n) * 4;
      const int64_t v0 = img * out_vox;
      barrier_lds();
      for (int k = 0; k < tz_n; ++k) {
        if (k > 0) store_out(v0, bx, by, 8 * (k - 1), (k - 1) & 1);
        if constexpr (kGrad) load_mask(v0, bx, by, 8 * k);  // for the store of tile k
        barrier_lds();
      }
      // the column's last tile; the ring and the output tiles are reused next
      store_out(v0, bx, by, 8 * (tz_n - 1), (tz_n - 1) & 1);
      barrier_lds();
    }
  } else {
    const int sgn = a.geo == kConv3 ? 1 : -1;
    const int r = lane & 15;
    const int ox = r & 3, oy = r >> 2;
    const int kq = lane >> 4;  // this lane's 16-byte chunk of the 32 channels
    const int wslot = kq ^ row_slot(r >> 2);
    const char* ring = reinterpret_cast<const char*>(sRing);
    // The fragment reads bound the tile (4 KB per 4 matrix instructions of
    // a wave), so the B fragments of the first kRT taps stay in registers for
    // every tile, as many as fit beside the sums and the fragments in
    // flight; only the other taps' are read with each tile.
    constexpr int kRT = res_taps(NB);
    bf16x8 breg[kRT][NB];
#pragma unroll
    for (int tt = 0; tt < kRT; ++tt)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        breg[tt][j] = *reinterpret_cast<const bf16x8*>(&sW[tt][16 * j + r][wslot]);
    for (int gc = blockIdx.x; gc < ncol * a.batch; gc += gridDim.x) {
      barrier_lds();
      for (int k = 0; k < tz_n; ++k) {
        floatx4 acc[2][NB];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[q][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        // fragments of tap tt: A from the planes (voxel of row r shifted by
        // the tap), B from the weights; those of the tap kAhead further on are
        // read while this tap's matrix instructions run
        auto read_a = [&](int tt, bf16x8 (&af)[2]) {
          const int dz = sgn * (tt / 9 - 1), dy = sgn * ((tt / 3) % 3 - 1), dx = sgn * (tt % 3 - 1);
          const int yy = oy + 1 + dy;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int zs = (8 * k + wave * 2 + q + 1 + dz) % kRing;  // plane z = 8k + zi - 1
            af[q] = *reinterpret_cast<const bf16x8*>(
                ring + zs * kResPlane + (yy * 6 + ox + 1 + dx) * 64 + ((kq ^ plane_slot(yy)) << 4));
          }
        };
        auto read_b = [&](int tt, bf16x8 (&bc)[NB]) {
#pragma unroll
          for (int j = 0; j < NB; ++j)
            bc[j] = *reinterpret_cast<const bf16x8*>(&sW[tt][16 * j + r][wslot]);
        };
        bf16x8 bc[kAhead + 1][NB], af[kAhead + 1][2];
        static_assert(kRT >= kAhead, "the first taps' weights are in registers");
#pragma unroll
        for (int tt = 0; tt < kAhead; ++tt) read_a(tt, af[tt]);
#pragma unroll
        for (int tt = 0; tt < 27; ++tt) {
          const int cur = tt % (kAhead + 1), next = tt + kAhead;
          if (next < 27) {
            read_a(next, af[next % (kAhead + 1)]);
            if (next >= kRT) read_b(next, bc[next % (kAhead + 1)]);
          }
          __builtin_amdgcn_sched_barrier(0);  // keep those reads ahead of the MFMAs below
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  af[cur][q], tt < kRT ? breg[tt < kRT ? tt : 0][j] : bc[cur][j], acc[q][j], 0, 0, 0);
        }
        // epilogue into sOut: row 4 (lane >> 4) + e of slice 2 wave + q is
        // local voxel (x, y, z) = (rr & 3, rr >> 2, 2 wave + q)
        char* dst = reinterpret_cast<char*>(sOut[k & 1]);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int nl = j * 16 + (lane & 15);
            const int vl0 = ((wave * 2 + q) * 4 + (lane >> 4)) * 4;  // the voxel of e = 0
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = acc[q][j][e] + sBias[nl];
              if (a.relu) v[e] = fmaxf(v[e], 0.f);
            }
            if constexpr (kF32 || kGrad) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                *reinterpret_cast<float*>(dst + sout_off<NB, 4>(vl0 + e, nl * 4)) = v[e];
            } else {
              // two adjacent channels of one voxel per 32-bit write: lanes
              // 2m and 2m + 1 (channels nl, nl + 1) swap one value, the even
              // lane then holds voxel e0's pair, the odd lane voxel e0 + 1's
              const bool odd = lane & 1;
#pragma unroll
              for (int e0 = 0; e0 < 4; e0 += 2) {
                const float send = odd ? v[e0] : v[e0 + 1];
                const float recv = __int_as_float(
                    __builtin_amdgcn_mov_dpp(__float_as_int(send), 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
                floatx2 pr;
                pr.x = odd ? recv : v[e0];
                pr.y = odd ? v[e0 + 1] : recv;
                *reinterpret_cast<uint32_t*>(dst + sout_off<NB, 2>(vl0 + e0 + (odd ? 1 : 0), (nl & ~1) * 2)) =
                    __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2v));
              }
            }
          }
        barrier_lds();
      }
      barrier_lds();
    }
  }
  if constexpr (kGrad) {
    // the workgroup's channel sums, added in a fixed order
    __shared__ float sRed[2][64][8];
    if (wave >= 5)
#pragma unroll
      for (int j = 0; j < 8; ++j) sRed[wave - 5][lane][j] = gsum[j];
    __syncthreads();
    if (tid < NC) {
      const int k = tid >> 3, j = tid & 7;
      float sum = 0.f;
      for (int w = 0; w < 2; ++w)
        for (int l = k; l < 64; l += 4) sum += sRed[w][l][j];
      a.gpart[static_cast<int64_t>(blockIdx.x) * a.cout + n0 + tid] = sum;
    }
  }
}

// ------------------------------------------ 3x3x3 conv with one gathered channel
// kConv3 / kConv3T with cin == 1 (the input layer's forward pass, the output
// layer's input gradient): the 27 taps are the reduction axis (one MFMA
// step, taps 27..31 zero).  A workgroup owns a 16 x 4 x 4 tile (wave w: the
// z-slice w, four rows of 16 voxels) and 32 NP output channels; the tile's
// 18 x 6 x 6 input brick is staged in LDS and the weights' fragments are read
// once from the packed weights (kpad >= 32, zero beyond tap 26).  As in
// up_kernel the voxels are the product's columns and a lane's sums 8 channels
// of one voxel: with `vec` (channels in eights, aligned) 16 bytes are stored
// at a time, 1 KB of consecutive memory per row and 32 channels.
// What bounds it: writing the output.  With 2-byte stores of 4 x 4 patches 32
// BF16 channels of eight 64^3 images took 94 us, one image 15.6; now 40 and
// 10.5 (134 MB: 28 us at the rate of a large copy).
template <int NP>
__global__ void __launch_bounds__(256) conv3_scalar_kernel(ConvArgs a, int vec) {
  __shared__ uint16_t sB[648];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int tx_n = (a.w + 15) >> 4, ty_n = (a.h + 3) >> 2;
  const int ntile = tx_n * ty_n * ((a.d + 3) >> 2);
  const int img = blockIdx.x / ntile, tile = blockIdx.x - img * ntile;
  const int bx = (tile % tx_n) * 16;
  const int by = ((tile / tx_n) % ty_n) * 4;
  const int bz = (tile / (tx_n * ty_n)) * 4;
  const int n0 = blockIdx.y * 32 * NP;
  const int sgn = a.geo == kConv3 ? 1 : -1;
  const int r = lane & 15, g = lane >> 4;
  const uint16_t* x_img = a.x + static_cast<int64_t>(img) * a.in_d * a.in_h * a.in_w;
  const int64_t o_img = static_cast<int64_t>(img) * a.d * a.h * a.w;
  for (int v = tid; v < 648; v += 256) {
    const int gx = bx + v % 18 - 1, gy = by + (v / 18) % 6 - 1, gz = bz + v / 108 - 1;
    uint16_t val = 0;
    if (gx >= 0 && gy >= 0 && gz >= 0 && gx < a.in_w && gy < a.in_h && gz < a.in_d)
      val = x_img[(static_cast<int64_t>(gz) * a.in_h + gy) * a.in_w + gx];
    sB[v] = val;
  }
  // rows 4 g' + i of product j are channels 8 g' + 4 j + i
  bf16x8 wf[NP][2];
  float bias[NP][8];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wf[p][j] = *reinterpret_cast<const bf16x8*>(
          a.bt + static_cast<int64_t>(n0 + 32 * p + 8 * (r >> 2) + 4 * j + (r & 3)) * a.kpad + 8 * g);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int n = n0 + 32 * p + 8 * g + i;
      bias[p][i] = a.bias && n < a.cout ? a.bias[n] : 0.f;
    }
  }
  int off[8];  // the brick positions of this lane's taps 8 g + j
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int t = min(8 * g + j, 26);
    const int dz = sgn * (t / 9 - 1), dy = sgn * ((t / 3) % 3 - 1), dx = sgn * (t % 3 - 1);
    off[j] = ((wave + 1 + dz) * 6 + 1 + dy) * 18 + r + 1 + dx;
  }
  __syncthreads();
  const int x = bx + r, z = bz + __builtin_amdgcn_readfirstlane(wave);
  if (z >= a.d) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int y = by + q;
    if (y >= a.h) break;
    bf16x8 vf;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t e = sB[off[j] + 18 * q];
      vf[j] = __builtin_bit_cast(__bf16, 8 * g + j < 27 ? e : static_cast<uint16_t>(0));
    }
    const int64_t o = o_img + (static_cast<int64_t>(z) * a.h + y) * a.w + x;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      floatx4 acc[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[p][j], vf,
                                                         floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const int n = n0 + 32 * p + 8 * g;
      const int64_t e0 = o * a.cout + n;
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = acc[i >> 2][i & 3] + bias[p][i];
      if (x >= a.w) continue;  // (every lane takes part in the matrix products)
      if (vec) {
        if (n >= a.cout) continue;
        if (a.skip) {
          const uint4 sk = *reinterpret_cast<const uint4*>(a.skip + e0);
          const uint16_t* sh = reinterpret_cast<const uint16_t*>(&sk);
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] += from_bf16(sh[i]);
        }
        if (a.relu) {
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = fmaxf(v[i], 0.f);
        }
        if (a.y_f32) {
          float4* dst = reinterpret_cast<float4*>(static_cast<float*>(a.y) + e0);
          dst[0] = make_float4(v[0], v[1], v[2], v[3]);
          dst[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
          uint4 u;
          uint16_t* uh = reinterpret_cast<uint16_t*>(&u);
#pragma unroll
          for (int i = 0; i < 8; ++i) uh[i] = to_bf16(v[i]);
          *reinterpret_cast<uint4*>(static_cast<uint16_t*>(a.y) + e0) = u;
        }
        continue;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (n + i >= a.cout) continue;
        if (a.skip) v[i] += from_bf16(a.skip[e0 + i]);
        if (a.relu) v[i] = fmaxf(v[i], 0.f);
        if (a.y_f32)
          static_cast<float*>(a.y)[e0 + i] = v[i];
        else
          static_cast<uint16_t*>(a.y)[e0 + i] = to_bf16(v[i]);
      }
    }
  }
}

// ------------------------------------- 3x3x3 conv with few channels in eights
// kConv3 / kConv3T with cin = 8, 16, 24, 40, 48 or 56: the reduction runs over
// (tap, channel) in steps of 32, lane group g of step s taking the 8 channels
// q % (cin / 8) of tap q / (cin / 8), q = 4 s + g.  A workgroup owns a 4 x 4 x 4
// tile (wave w: the z-slice w) and 16 NB output channels; the tile's brick is
// staged in LDS, where those 8 channels of a shifted voxel are 16 bytes, and
// the weights' fragments of kSteps steps at a time are read straight from the
// packed weights, all in flight together.  Rows and columns as in the brick
// kernel.
// What bounds it: on small grids the latency of its one or two rounds of loads,
// where the generic kernel waits for each of its stages.  Measured, generic and
// this, us: 24^3 8 -> 8 7.0 and 4.5, 12^3 16 -> 16 9.9 and 6.0.
template <int NB>
__global__ void __launch_bounds__(256) conv3_eights_kernel(ConvArgs a, int vec) {
  constexpr int kSteps = 7;
  __shared__ uint4 s_br[216 * 7];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2;
  const int ntile = tx_n * ty_n * ((a.d + 3) >> 2);
  const int img = blockIdx.x / ntile, tile = blockIdx.x - img * ntile;
  const int bx = (tile % tx_n) * 4;
  const int by = ((tile / tx_n) % ty_n) * 4;
  const int bz = (tile / (tx_n * ty_n)) * 4;
  const int n0 = blockIdx.y * 16 * NB;
  const int sgn = a.geo == kConv3 ? 1 : -1;
  const int r = lane & 15, g = lane >> 4;
  const int c8 = a.cin >> 3;                 // 1 .. 7
  const int inv = 65536 / c8 + 1;            // (n * inv) >> 16 = n / c8 for n < 1512
  const int steps = (27 * c8 + 3) >> 2;
  const uint16_t* x_img = a.x + static_cast<int64_t>(img) * a.in_d * a.in_h * a.in_w * a.cin;

  const uint16_t* wp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = NB >= 2 ? 32 * (j >> 1) + 8 * (r >> 2) + 4 * (j & 1) + (r & 3) : r;
    wp[j] = a.bt + static_cast<int64_t>(n0 + n) * a.kpad + 8 * g;
  }
  bf16x8 wf[kSteps][NB];
  auto load_w = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        wf[u][j] = *reinterpret_cast<const bf16x8*>(wp[j] + min(s0 + u, steps - 1) * kBK);
  };
  load_w(0);
  for (int p = tid; p < 216 * c8; p += 256) {
    const int v = (p * inv) >> 16, c = p - v * c8;
    const int gx = bx + v % 6 - 1, gy = by + (v / 6) % 6 - 1, gz = bz + v / 36 - 1;
    uint4 val = make_uint4(0u, 0u, 0u, 0u);
    if (gx >= 0 && gy >= 0 && gz >= 0 && gx < a.in_w && gy < a.in_h && gz < a.in_d)
      val = *reinterpret_cast<const uint4*>(
          x_img + ((static_cast<int64_t>(gz) * a.in_h + gy) * a.in_w + gx) * a.cin + c * 8);
    s_br[p] = val;
  }
  __syncthreads();
  const int center = ((wave + 1) * 6 + (r >> 2) + 1) * 6 + (r & 3) + 1;
  floatx4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < steps; s0 += kSteps) {
    if (s0 > 0) load_w(s0);
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      if (s0 + u >= steps) break;
      const int q = 4 * (s0 + u) + g, t = (q * inv) >> 16, c = q - t * c8;
      uint4 xv = make_uint4(0u, 0u, 0u, 0u);
      if (t < 27)
        xv = s_br[(center + sgn * ((t / 9 - 1) * 36 + ((t / 3) % 3 - 1) * 6 + t % 3 - 1)) * c8 + c];
      const bf16x8 xf = __builtin_bit_cast(bf16x8, xv);
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u][j], xf, acc[j], 0, 0, 0);
    }
  }
  const int x = bx + (r & 3), y = by + (r >> 2), z = bz + wave;
  if (x >= a.w || y >= a.h || z >= a.d) return;
  const int64_t o = ((static_cast<int64_t>(img) * a.d + z) * a.h + y) * a.w + x;
  if constexpr (NB >= 2) {
#pragma unroll
    for (int j = 0; j < NB; j += 2) {
      const floatx4 v[2] = {acc[j], acc[j + 1]};
      put_channels<8>(a, v, o, n0 + 16 * j + 8 * g, nullptr, vec);
    }
  } else {
    const floatx4 v[1] = {acc[0]};
    put_channels<4>(a, v, o, n0 + 4 * g, nullptr, vec);
  }
}

// Finish a split product: y[o][n] = [relu](sum over splits of part[s][o][n]
// + bias[n] [+ skip[o][n]]), splits summed in order.
__global__ void __launch_bounds__(256) split_reduce_kernel(ConvArgs a, int nsplit) {
  const int64_t n_out = static_cast<int64_t>(a.batch) * a.d * a.h * a.w * a.cout;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n_out;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int n = static_cast<int>(i % a.cout);
    float v = a.part[i];
    for (int sp = 1; sp < nsplit; ++sp) v += a.part[sp * n_out + i];
    v += a.bias ? a.bias[n] : 0.f;
    if (a.skip) v += from_bf16(a.skip[i]);
    if (a.relu) v = fmaxf(v, 0.f);
    if (a.y_f32)
      static_cast<float*>(a.y)[i] = v;
    else
      static_cast<uint16_t*>(a.y)[i] = to_bf16(v);
  }
}

// ------------------------------------------------------------ weight GEMM
// gw[p][n] += sum over the workgroup's voxels of A(m, p) gy(m, n), with
// p = t * cin + ci.  kConv3 / kDown: m runs over the output grid, A is x
// gathered at the tap; kUp: m runs over the input grid, A = x[m] and gy is
// read at the parity-class position of tap t (all rows of a tile share t).
// kVec, vec_gy: x, gy in 16-byte pieces (channels in eights, aligned).
template <int NB, bool kVec>
__global__ void __launch_bounds__(256) wgrad_kernel(WgradArgs a, bool vec_gy) {
  __shared__ uint16_t sA[kBM][kBK + kPadK];       // [p][m]
  __shared__ uint16_t sB[16 * NB][kBK + kPadK];   // [n][m]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t M = static_cast<int64_t>(a.d) * a.h * a.w;
  const int64_t mb = static_cast<int64_t>(blockIdx.x) * a.m_per_block;
  const int64_t me = mb + a.m_per_block < M ? mb + a.m_per_block : M;
  const int n0 = blockIdx.z * 16 * NB;
  const int P = a.taps * a.cin;
  // rows of this tile
  int p0, t_up = 0, prow_lim;
  if (a.geo == kUp) {
    const int tiles = (a.cin + kBM - 1) / kBM;
    t_up = blockIdx.y / tiles;
    p0 = t_up * a.cin + (blockIdx.y % tiles) * kBM;
    prow_lim = t_up * a.cin + a.cin;
  } else {
    p0 = blockIdx.y * kBM;
    prow_lim = P;
  }

  floatx4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int64_t m0 = mb; m0 < me; m0 += kBK) {
    // A: 64 rows (p) x 32 voxels, loaded 8 rows of one voxel per thread
    {
      const int mm = tid >> 3, rc = (tid & 7) * 8;
      const int64_t m = m0 + mm;
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = 0;
      if (m < me) {
        const int x = static_cast<int>(m % a.w);
        const int y = static_cast<int>((m / a.w) % a.h);
        const int z = static_cast<int>(m / (static_cast<int64_t>(a.w) * a.h));
        const int p = p0 + rc;
        if constexpr (kVec) {
          if (p < prow_lim) {
            const int t = p / a.cin, ci = p - t * a.cin;
            const int64_t src = a.geo == kUp ? m : gather_at(a.g, z, y, x, t);
            if (src >= 0) {
              const uint4 v = *reinterpret_cast<const uint4*>(a.x + src * a.cin + ci);
              e[0] = v.x & 0xffff; e[1] = v.x >> 16; e[2] = v.y & 0xffff; e[3] = v.y >> 16;
              e[4] = v.z & 0xffff; e[5] = v.z >> 16; e[6] = v.w & 0xffff; e[7] = v.w >> 16;
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int pj = p + j;
            if (pj < prow_lim) {
              const int t = pj / a.cin, ci = pj - t * a.cin;
              const int64_t src = a.geo == kUp ? m : gather_at(a.g, z, y, x, t);
              if (src >= 0) e[j] = a.x[src * a.cin + ci];
            }
          }
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) sA[rc + j][mm] = e[j];
    }
    // B: 16*NB channels x 32 voxels of gy
    for (int i = tid; i < 2 * NB * kBK; i += 256) {
      const int nc = (i % (2 * NB)) * 8, mm = i / (2 * NB);
      const int64_t m = m0 + mm;
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = 0;
      if (m < me) {
        int64_t gi = m;
        if (a.geo == kUp) {
          const int x = static_cast<int>(m % a.w);
          const int y = static_cast<int>((m / a.w) % a.h);
          const int z = static_cast<int>(m / (static_cast<int64_t>(a.w) * a.h));
          gi = (static_cast<int64_t>(2 * z + (t_up >> 2)) * (2 * a.h) + 2 * y + ((t_up >> 1) & 1)) *
                   (2 * a.w) + 2 * x + (t_up & 1);
        }
        const uint16_t* row = a.gy + gi * a.cout + n0 + nc;
        if (vec_gy && n0 + nc + 8 <= a.cout) {
          const uint4 v = *reinterpret_cast<const uint4*>(row);
          e[0] = v.x & 0xffff; e[1] = v.x >> 16; e[2] = v.y & 0xffff; e[3] = v.y >> 16;
          e[4] = v.z & 0xffff; e[5] = v.z >> 16; e[6] = v.w & 0xffff; e[7] = v.w >> 16;
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) e[j] = (n0 + nc + j < a.cout) ? row[j] : 0;
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) sB[nc + j][mm] = e[j];
    }
    __syncthreads();
    const bf16x8 af = *reinterpret_cast<const bf16x8*>(&sA[wave * 16 + (lane & 15)][(lane >> 4) * 8]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bf16x8 bf = *reinterpret_cast<const bf16x8*>(&sB[j * 16 + (lane & 15)][(lane >> 4) * 8]);
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc[j], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = n0 + j * 16 + (lane & 15);
    if (n >= a.cout) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = p0 + wave * 16 + (lane >> 4) * 4 + i;
      if (p < prow_lim && acc[j][i] != 0.f)
        unsafeAtomicAdd(a.gw + static_cast<int64_t>(p) * a.cout + n, acc[j][i]);
    }
  }
}

// ---------------------------------------- 3x3x3 weight gradient from a slab
// kConv3 layers with cin a multiple of 32 whose other operands the kernels with
// transposing reads below do not take (16-byte pieces of 8 output channels).
// A workgroup owns one chunk of 32 input channels (blockIdx.y % chunks), one plane dz = blockIdx.y / chunks
// of taps (the 9 taps t = 9 dz + 3 dy + dx) and 32 NBW output channels
// (blockIdx.z), and walks the 4 x 4 x kSlabTZ voxel tiles blockIdx.x,
// blockIdx.x + gridDim.x, ...  Per tile it stages the kSlabTZ x 6 x 6 slab of x
// the plane's taps read (zero outside the volume), transposed to channel
// rows in three copies, one per tap column dx, each holding the 4 x
// positions dx .. dx + 3 of every (z, y) row of the slab -- so that an A
// fragment (8 voxels: two rows of 4 in x) is two aligned 8-byte reads --
// and the tile's gy transposed to [n][m]; wave w then accumulates the 16
// input channels 16 (w & 1).. and 16 NBW output channels of its half
// (w >> 1) for all 9 taps, with the tile's 16 kSlabTZ voxels on the MFMA's
// reduction axis (kSlabTZ / 2 steps of 32: tiles of 8 z-slices halve the
// staging round trips -- global loads, the transpose, two barriers -- per
// matrix instruction against 4).  The sums are stored to
// part[blockIdx.x][t][ci][n] and wgrad_reduce_kernel adds them to gw in a
// fixed order.
__device__ __forceinline__ uint4 load8(const uint16_t* p, bool vec) {
  if (vec) return *reinterpret_cast<const uint4*>(p);
  return make_uint4(p[0] | uint32_t(p[1]) << 16, p[2] | uint32_t(p[3]) << 16,
                    p[4] | uint32_t(p[5]) << 16, p[6] | uint32_t(p[7]) << 16);
}
constexpr int kSlabTZ = 8;                     // z-slices per tile
constexpr int kSlabRow = kSlabTZ * 6 * 4 + 4;  // one channel's (z, y, 4 x) of a copy, padded
// vec_x: x aligned, and read in 16-byte pieces.
template <int NBW>
__global__ void __launch_bounds__(256) wgrad_slab_kernel(WgradArgs a, bool vec_x) {
  __shared__ __align__(16) uint16_t sXT[3][32][kSlabRow];  // copy dx, channel, (z, y, x - dx)
  __shared__ uint16_t sG[32 * NBW][16 * kSlabTZ + kPadK];  // output channel, tile voxel
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int chunks = a.cin / kBK;
  const int c0 = static_cast<int>(blockIdx.y % chunks) * kBK;
  const int dz = static_cast<int>(blockIdx.y / chunks);
  const int n0 = static_cast<int>(blockIdx.z) * 32 * NBW;
  const int cb = wave & 1;
  const int nw = (wave >> 1) * 16 * NBW;  // this wave's first channel within the group
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2, tz_n = (a.d + kSlabTZ - 1) / kSlabTZ;
  const int tiles = tx_n * ty_n * tz_n;
  const int P = a.taps * a.cin;

  floatx4 acc[9][NBW];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < NBW; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // This thread's staging loads of one tile, held in registers so that the
  // next tile's loads are in flight while the current one is computed:
  // slab item tid (< kSlabTZ * 6 * 4): one (z, y) row of the slab and
  // 8-channel chunk, its 6 voxels; output-gradient items tid + 256 u: one
  // voxel of the tile and 8 output channels.
  constexpr int kXI = kSlabTZ * 6 * 4;
  constexpr int kGI = 16 * kSlabTZ * 4 * NBW / 256;
  static_assert(kXI <= 256 && kGI * 256 == 16 * kSlabTZ * 4 * NBW, "staging items per thread");
  uint4 xv[6], gv[kGI];
  auto load = [&](int tile) {
    const int bx = (tile % tx_n) * 4;
    const int by = ((tile / tx_n) % ty_n) * 4;
    const int bz = (tile / (tx_n * ty_n)) * kSlabTZ;
    if (tid < kXI) {
      const int oc = tid & 3, yy = (tid >> 2) % 6, zz = (tid >> 2) / 6;
      const int gy = by + yy - 1, gz = bz + zz + dz - 1;
      const bool row_in = gy >= 0 && gz >= 0 && gy < a.g.in_h && gz < a.g.in_d;
#pragma unroll
      for (int xx = 0; xx < 6; ++xx) {
        const int gx = bx + xx - 1;
        xv[xx] = make_uint4(0u, 0u, 0u, 0u);
        if (row_in && gx >= 0 && gx < a.g.in_w)
          xv[xx] = load8(
              a.x + ((static_cast<int64_t>(gz) * a.g.in_h + gy) * a.g.in_w + gx) * a.cin + c0 +
              oc * 8, vec_x);
      }
    }
#pragma unroll
    for (int u = 0; u < kGI; ++u) {
      const int i = tid + 256 * u;
      const int m = i / (4 * NBW), nc = (i % (4 * NBW)) * 8;
      const int x = bx + (m & 3), y = by + ((m >> 2) & 3), z = bz + (m >> 4);
      gv[u] = make_uint4(0u, 0u, 0u, 0u);
      if (x < a.w && y < a.h && z < a.d) {
        const uint16_t* row =
            a.gy + ((static_cast<int64_t>(z) * a.h + y) * a.w + x) * a.cout + n0 + nc;
        uint32_t h[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = (n0 + nc + j < a.cout) ? row[j] : 0u;
        gv[u] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                           h[6] | (h[7] << 16));
      }
    }
  };
  // the registers into LDS: each channel of the slab row as its 4-voxel runs
  // starting at x = 0, 1, 2; the output gradient transposed to [n][m]
  auto store = [&]() {
    if (tid < kXI) {
      const int oc = tid & 3, yy = (tid >> 2) % 6, zz = (tid >> 2) / 6;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        uint32_t e[6];  // channel oc * 8 + c of the row's 6 voxels
#pragma unroll
        for (int xx = 0; xx < 6; ++xx) {
          const uint32_t w32 = (&xv[xx].x)[c >> 1];
          e[xx] = (c & 1) ? (w32 >> 16) : (w32 & 0xffffu);
        }
#pragma unroll
        for (int d0 = 0; d0 < 3; ++d0)
          *reinterpret_cast<uint2*>(&sXT[d0][oc * 8 + c][(zz * 6 + yy) * 4]) =
              make_uint2(e[d0] | (e[d0 + 1] << 16), e[d0 + 2] | (e[d0 + 3] << 16));
      }
    }
#pragma unroll
    for (int u = 0; u < kGI; ++u) {
      const int i = tid + 256 * u;
      const int m = i / (4 * NBW), nc = (i % (4 * NBW)) * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t w32 = (&gv[u].x)[j >> 1];
        sG[nc + j][m] = static_cast<uint16_t>((j & 1) ? (w32 >> 16) : (w32 & 0xffffu));
      }
    }
  };

  if (static_cast<int>(blockIdx.x) < tiles) load(blockIdx.x);
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    __syncthreads();  // the previous tile's fragments have been read
    store();
    __syncthreads();
    if (tile + static_cast<int>(gridDim.x) < tiles) load(tile + gridDim.x);
    // B fragments: voxels 32 ks + 8 g .. + 7 of output channel nw + 16 j + r
    bf16x8 bf[kSlabTZ / 2][NBW];
#pragma unroll
    for (int ks = 0; ks < kSlabTZ / 2; ++ks)
#pragma unroll
      for (int j = 0; j < NBW; ++j)
        bf[ks][j] = *reinterpret_cast<const bf16x8*>(&sG[nw + 16 * j + r][32 * ks + 8 * g]);
    // A fragments: channel 16 cb + r of the slab at voxel m + tap offset,
    // m = 32 ks + 8 g + j: x = j & 3, y = 2 (g & 1) + (j >> 2), z = 2 ks + (g >> 1);
    // slab rows y0 + dy and y0 + dy + 1 of copy dx
    const int ci = cb * 16 + r;
#pragma unroll
    for (int ks = 0; ks < kSlabTZ / 2; ++ks) {
      const int zz = 2 * ks + (g >> 1);
      const int y0 = 2 * (g & 1);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int dy = t / 3, dx = t % 3;
        const uint16_t* row = &sXT[dx][ci][(zz * 6 + y0 + dy) * 4];
        const uint2 lo = *reinterpret_cast<const uint2*>(row);
        const uint2 hi = *reinterpret_cast<const uint2*>(row + 4);
        const bf16x8 af = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
        for (int j = 0; j < NBW; ++j)
          acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf[ks][j], acc[t][j], 0, 0, 0);
      }
    }
  }
  // lane (r, g) holds D[4 g + i][r]: input channel c0 + 16 cb + 4 g + i, output channel
  float* out = a.part + static_cast<int64_t>(blockIdx.x) * P * a.cout;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      const int n = n0 + nw + 16 * j + r;
      if (n >= a.cout) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = (9 * dz + t) * a.cin + c0 + 16 * cb + 4 * g + i;
        out[static_cast<int64_t>(p) * a.cout + n] = acc[t][j][i];
      }
    }
}

// ------------------------------------ weight gradients, operands by transposing reads
// gw[t][ci][n] = sum_m x(m, t, ci) gy(m, t, n): both operands of the matrix
// product run along voxels, which are the slow axis of x and gy.  Tiles are
// copied to LDS as they are, [voxel][32 channels], by loader waves with direct
// global-to-LDS loads, and gfx950's transposing LDS reads form the fragments:
// of 16 lanes, lane 4 a + b reads 8 bytes, channels 4 b .. 4 b + 3 of the
// voxel given by its address, and lane i receives channel i of the four
// voxels a.  The voxels' addresses are free, so taps and classes are
// offsets.  A 16-byte piece j of voxel v is in slot j ^ 2 s(v), where s differs
// between the voxels that a half-wave reads 256 bytes apart: the 32 lanes
// fall on 64 different banks.
__device__ __forceinline__ bf16x8 read_tr(const char* lo, const char* hi) {
  typedef short shortx4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) shortx4* lds;
  struct {
    shortx4 a, b;
  } v = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)(lo)),
         __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)(hi))};
  return __builtin_bit_cast(bf16x8, v);
}

// this lane's byte offset in a transposing read of voxels 64 bytes apart
__device__ __forceinline__ int tr_lane(int lane) {
  return ((lane >> 2) & 3) * 64 + (lane & 3) * 8;
}

// floats of one group's sums: the weights' and, with gb, the bias gradient
__host__ __device__ __forceinline__ int64_t wgrad_floats(const WgradArgs& a) {
  return static_cast<int64_t>(a.taps) * a.cin * a.cout + (a.gb ? a.cout : 0);
}

// Output channel n's sum over the workgroup's tiles of gy.  It comes from the
// matrix products with a fragment of ones beside gy's, where each column is
// the sum; a kernel of its own read gy again, 10 us at 64^3 x 32.
__device__ __forceinline__ void wgrad_put_bias(const WgradArgs& a, int n, float v) {
  if (n >= a.cout) return;
  if (gridDim.x > 1)
    a.part[blockIdx.x * wgrad_floats(a) + static_cast<int64_t>(a.taps) * a.cin * a.cout + n] = v;
  else
    a.gb[n] = a.overwrite ? v : a.gb[n] + v;
}
__device__ __forceinline__ bf16x8 ones8() {
  const uint32_t two = 0x3f803f80u;  // 1.0 twice
  return __builtin_bit_cast(bf16x8, make_uint4(two, two, two, two));
}

// A workgroup's sums, N groups of four output channels at the elements
// at(0) .. at(N - 1) of gw, or nowhere (-1).  Several workgroups along the
// tiles store to part[blockIdx.x] for wgrad_reduce_kernel; a single one
// finishes gw itself, reading all of it before it stores any.
template <int N, typename At, typename Sum>
__device__ __forceinline__ void wgrad_put(const WgradArgs& a, At at, Sum sum) {
  if (gridDim.x > 1) {
    float* out = a.part + blockIdx.x * wgrad_floats(a);
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (at(k) >= 0) *reinterpret_cast<floatx4*>(out + at(k)) = sum(k);
    return;
  }
  float old[N][4];
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) old[k][i] = !a.overwrite && at(k) >= 0 ? a.gw[at(k) + i] : 0.f;
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (at(k) >= 0)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a.gw[at(k) + i] = a.overwrite ? sum(k)[i] : old[k][i] + sum(k)[i];
}

// The loader waves' protocol: stage s of nt in slot s % 3 of the ring, two
// stages ahead; kL loads a stage.  The compute waves meet the same barrier
// before each stage.
template <int kL, typename Load>
__device__ __forceinline__ void stream_stages(int nt, Load load) {
  load(0, 0);
  if (nt > 1) load(1, 1);
  for (int s = 0, slot = 2; s < nt; ++s) {
    if (s + 1 < nt)
      wait_vm<kL>();
    else
      wait_vm<0>();
    barrier_lds();  // stage s has landed; the slot of stage s - 1 is free
    if (s + 2 < nt) load(s + 2, slot);
    slot = slot == 2 ? 0 : slot + 1;
  }
}

// 3x3x3 layers with cin and cout multiples of 8.  A workgroup owns 32 input
// channels, 32 output channels and all 27 taps, or with kPlane one plane dz
// of 9 (three workgroups), and walks the 4 x 4 x 8-voxel tiles blockIdx.x,
// + gridDim.x, ...: per tile the 6 x 6 x 10 brick of x and the tile of gy.
// The compute waves share the taps.  Where tiles end past the volume (kEdge), the
// activations that the zero gradients there meet are read from a block of
// zeros: an infinite one, inside the volume, would make sums NaN that it is no
// part of.  That is a choice of address for each two slices (62 x 62 x 63, 32 -> 32:
// 42.3 us a call with the zeros left out, 43.7; masking the fragments 48).
// What bounds it: a tile's 31 KB arrive in 1.2 us where its matrix
// instructions take 0.75; below four tiles a workgroup the partial sums, 28 MB
// for 256 workgroups with all taps.  The slab kernel copied the tiles through
// registers, transposing 2 bytes at a time.  Measured with the reductions, slab
// and this, us: 64^3 32 -> 32 33.0 + 11.7 and 21.7 + 6.4, 32^3 64 -> 64 23.1 +
// 7.7 and 16.0 + 6.4, 16^3 128 -> 128 15.4 + 10.7 and 16.3 + 4.8, 8^3 256 -> 256
// 12.5 + 10.1 and 15.7.  Voxel k = 8 g + j of reduction step ks is
// (x, y, z) = (j & 3, 2 (g & 1) + (j >> 2), 2 ks + (g >> 1)).
struct WBrick {
  static constexpr int kPieces = 360 * 4;               // 16-byte pieces of a brick
  static constexpr int kBrickLoads = 23, kLoads = 31;   // wave loads: brick, then gy
  static constexpr int kStageBytes = kLoads * 1024;
  // zeros as far as a tap's reads reach: two planes, three rows and three voxels
  static constexpr int kZeroBytes = 384 * 16;
  static_assert((2 * 36 + 3 * 6 + 2 + 1) * 64 <= kZeroBytes, "one chunk a thread covers them");
};

template <int LW>
__device__ __forceinline__ void wbrick_loader(const WgradArgs& a, char* s_st, int lane, int c0,
                                              int n0, int tx_n, int ty_n, int nt) {
  using K = WBrick;
  constexpr int kL = (K::kLoads + 1 - LW) / 2;
  const uint16_t* zero = reinterpret_cast<const uint16_t*>(g_zero16) +
                         ((blockIdx.x * 64 + lane) & (kZeroChunks - 1)) * 8;
  // Per load: the offset from the tile's first voxel, and the brick position
  // as one bit for each of x, y and z (bit 31: no such piece), which a tile's
  // mask of what lies outside the volume tells apart in two instructions.
  int64_t rel[kL];
  uint32_t pos[kL];
#pragma unroll
  for (int k = 0; k < kL; ++k) {
    const int b = 2 * k + LW;
    int x, y, z;
    if (b < K::kBrickLoads) {
      const int p = b * 64 + lane, v = p >> 2;
      x = v % 6, y = (v / 6) % 6, z = v / 36;
      const int c = c0 + (((p & 3) ^ (y & 2)) << 3);
      rel[k] = ((static_cast<int64_t>(z - 1) * a.h + (y - 1)) * a.w + (x - 1)) * a.cin + c;
      pos[k] = p < K::kPieces && c < a.cin ? 0u : 1u << 31;
    } else {
      const int p = (b - K::kBrickLoads) * 64 + lane, v = p >> 2;
      x = v & 3, y = (v >> 2) & 3, z = v >> 4;
      const int n = n0 + (((p & 3) ^ (y & 2)) << 3);
      rel[k] = ((static_cast<int64_t>(z) * a.h + y) * a.w + x) * a.cout + n;
      pos[k] = n < a.cout ? 0u : 1u << 31;
      ++x, ++y, ++z;
    }
    if (!pos[k]) pos[k] = 1u << x | 1u << (6 + y) | 1u << (12 + z);
  }
  stream_stages<kL>(nt, [&](int s, int slot) {
    const int tile = blockIdx.x + s * gridDim.x;
    const int bx = (tile % tx_n) * 4, by = ((tile / tx_n) % ty_n) * 4, bz = (tile / (tx_n * ty_n)) * 8;
    const uint32_t out = 1u << 31 | outside(bx - 1, 6, a.w) | outside(by - 1, 6, a.h) << 6 |
                         outside(bz - 1, 10, a.d) << 12;
    const int64_t v0 = (static_cast<int64_t>(bz) * a.h + by) * a.w + bx;
    const uint16_t* x0 = a.x + v0 * a.cin;
    const uint16_t* g0 = a.gy + v0 * a.cout;
#pragma unroll
    for (int k = 0; k < kL; ++k) {
      const int b = 2 * k + LW;
      load_lds16(pos[k] & out ? zero : (b < K::kBrickLoads ? x0 : g0) + rel[k],
                 s_st + slot * K::kStageBytes + b * 1024);
    }
  });
}

template <bool kPlane, bool kEdge, int W>
__device__ __forceinline__ void wbrick_compute(const WgradArgs& a, const char* s_st, int lane,
                                               int c0, int n0, int dz0, int tx_n, int ty_n,
                                               int nt) {
  using K = WBrick;
  // the last wave, which has the fewest taps, sums gy for the bias gradient
  const bool bias = W == 3 && a.gb && c0 == 0 && dz0 == 0;
  floatx4 sum[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
  constexpr int kT0 = kPlane ? (9 * W + 3) / 4 : 7 * W;  // the wave's taps kT0 .. kT0 + kNT - 1
  constexpr int kNT = kPlane ? (9 * W + 12) / 4 - kT0 : (W < 3 ? 7 : 6);
  const int r = lane & 15, g = lane >> 4;
  const int xo = tr_lane(lane) + ((g >> 1) * 36 + (g & 1) * 12 + dz0 * 36) * 64;
  const int go = tr_lane(lane) + ((g >> 1) * 16 + (g & 1) * 8) * 64 + K::kBrickLoads * 1024;
  floatx4 acc[kNT][2][2];
#pragma unroll
  for (int t = 0; t < kNT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[t][q >> 1][q & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0, slot = 0; s < nt; ++s) {
    barrier_lds();  // stage s has landed
    const char* st = s_st + slot * K::kStageBytes;
    // the two 16-channel halves, as they lie for even y >> 1
    const char* xh[2] = {st + xo + (g & 1) * 32, st + xo + ((g & 1) ^ 1) * 32};
    const char* gh[2] = {st + go + (g & 1) * 32, st + go + ((g & 1) ^ 1) * 32};
    // kEdge: whether the voxels this lane reads, of its two rows, and how many
    // of the tile's slices lie in the volume; the others are read from the zeros
    bool in_row[2] = {true, true};
    int in_z = 8;
    if constexpr (kEdge) {
      const int tile = blockIdx.x + s * gridDim.x;
      const int x = a.w - (tile % tx_n) * 4 - ((lane >> 2) & 3);
      const int y = a.h - ((tile / tx_n) % ty_n) * 4 - 2 * (g & 1);
      in_row[0] = x > 0 && y > 0;
      in_row[1] = x > 0 && y > 1;
      in_z = a.d - (tile / (tx_n * ty_n)) * 8 - (g >> 1);
    }
    const char* xr[2][2] = {{xh[0], xh[1]}, {xh[0], xh[1]}};  // row, half: of the step
    auto read_x = [&](int i, bf16x8 (&f)[2]) {  // tap i % kNT of step i / kNT
      const int ks = i / kNT, t = kT0 + i % kNT, dz = t / 9, dy = (t / 3) % 3, dx = t % 3;
      if (kEdge && i % kNT == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          xr[q >> 1][q & 1] = in_row[q >> 1] && 2 * ks < in_z
                                  ? xh[q & 1] : s_st + 3 * K::kStageBytes - 2 * ks * 36 * 64;
      }
      const int o = ((2 * ks + dz) * 36 + dy * 6 + dx) * 64;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        f[cb] = read_tr(xr[0][cb ^ (dy >> 1)] + o, xr[1][cb ^ ((dy + 1) >> 1)] + o + 6 * 64);
    };
    bf16x8 xf[2][2], gf[2];
    read_x(0, xf[0]);
#pragma unroll
    for (int i = 0; i < 4 * kNT; ++i) {
      const int t = i % kNT;
      if (t == 0) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          gf[nb] = read_tr(gh[nb] + (i / kNT) * 2048, gh[nb] + (i / kNT) * 2048 + 256);
        if (bias) {
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            sum[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[nb], ones8(), sum[nb], 0, 0, 0);
        }
      }
      if (i + 1 < 4 * kNT) read_x(i + 1, xf[(i + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);  // those reads ahead of the matrix instructions
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          acc[t][nb][cb] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[nb], xf[i & 1][cb], acc[t][nb][cb], 0, 0, 0);
    }
    slot = slot == 2 ? 0 : slot + 1;
  }
  if (bias && r == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) wgrad_put_bias(a, n0 + (i >> 2) * 16 + 4 * g + (i & 3), sum[i >> 2][i & 3]);
  }
  // lane (r, g) holds output channels 16 nb + 4 g .. + 3 of input channel 16 cb + r
  wgrad_put<4 * kNT>(
      a,
      [&](int k) -> int64_t {
        const int n = n0 + ((k >> 1) & 1) * 16 + 4 * g, ci = c0 + (k & 1) * 16 + r;
        return n < a.cout && ci < a.cin
                   ? (static_cast<int64_t>(9 * dz0 + kT0 + (k >> 2)) * a.cin + ci) * a.cout + n
                   : -1;
      },
      [&](int k) { return acc[k >> 2][(k >> 1) & 1][k & 1]; });
}

// blockIdx.y: 32 input channels (kPlane: times 3, plus dz), blockIdx.z: 32 output channels
template <bool kPlane, bool kEdge>
__global__ void __launch_bounds__(384) wgrad_brick_kernel(WgradArgs a) {
  __shared__ __align__(16) char s_st[3 * WBrick::kStageBytes + (kEdge ? WBrick::kZeroBytes : 0)];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2, tiles = tx_n * ty_n * ((a.d + 7) >> 3);
  const int nt = (tiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  const int dz0 = kPlane ? blockIdx.y % 3 : 0;
  const int c0 = (kPlane ? blockIdx.y / 3 : blockIdx.y) * 32, n0 = blockIdx.z * 32;
  if constexpr (kEdge)  // ahead of the first stage's barrier
    *reinterpret_cast<uint4*>(s_st + 3 * WBrick::kStageBytes + threadIdx.x * 16) =
        make_uint4(0u, 0u, 0u, 0u);
  switch (wave) {
    case 0: wbrick_compute<kPlane, kEdge, 0>(a, s_st, lane, c0, n0, dz0, tx_n, ty_n, nt); break;
    case 1: wbrick_compute<kPlane, kEdge, 1>(a, s_st, lane, c0, n0, dz0, tx_n, ty_n, nt); break;
    case 2: wbrick_compute<kPlane, kEdge, 2>(a, s_st, lane, c0, n0, dz0, tx_n, ty_n, nt); break;
    case 3: wbrick_compute<kPlane, kEdge, 3>(a, s_st, lane, c0, n0, dz0, tx_n, ty_n, nt); break;
    case 4: wbrick_loader<0>(a, s_st, lane, c0, n0, tx_n, ty_n, nt); break;
    default: wbrick_loader<1>(a, s_st, lane, c0, n0, tx_n, ty_n, nt); break;
  }
}

// 2x2x2 stride-2 layers with cin and cout multiples of 8: of each voxel m of the
// small grid, the operand on the large grid (kDown: x, kUp: gy) has the 8
// voxels 2 m + e(t), one per tap.  A workgroup owns 32 channels of the large
// operand (blockIdx.y), 16 NS of the small one (blockIdx.z) and all taps, and
// walks the tiles of 64 consecutive m blockIdx.x, + gridDim.x, ...; the large
// operand is staged by tap.  Compute wave w has taps 2 w and 2 w + 1; s(v) is
// bit 3 of v = 32 ks + 8 g + j.
// What bounds it: reading the large operand (17 MB at 64^3 x 32: 4 us) and the
// partial sums (17 MB).  The generic kernel reads it again for every 64 rows of
// gw and adds to gw with atomics.  Measured, generic and this with its
// reduction, us: down 64^3 -> 32^3, 32 -> 64 30 and 9.7 + 4.7, 32^3 -> 16^3,
// 64 -> 128 27 and 9.5 + 4.3, up 32^3 -> 64^3, 64 -> 32 41 and 9.5 + 4.7.
template <int NS>
struct WPair {
  static constexpr int kStageBytes = 32768 + NS * 2048;  // [tap][64 voxels], [NS / 2][64 voxels]
};

template <bool kUpGeo, int NS, int LW>
__device__ __forceinline__ void wpair_loader(const WgradArgs& a, char* s_st, int lane, int b0,
                                             int s0, int nt) {
  const uint16_t* zero = reinterpret_cast<const uint16_t*>(g_zero16) + lane * 8;
  const int64_t M = static_cast<int64_t>(a.d) * a.h * a.w;
  const uint16_t* big = kUpGeo ? a.gy : a.x;
  const uint16_t* small = kUpGeo ? a.x : a.gy;
  const int bc = kUpGeo ? a.cout : a.cin, sc = kUpGeo ? a.cin : a.cout;
  const int64_t row = 2 * a.w, plane = row * (2 * a.h);
  stream_stages<16 + NS>(nt, [&](int s, int slot) {
    const int64_t m0 = (blockIdx.x + static_cast<int64_t>(s) * gridDim.x) * 64;
    char* st = s_st + slot * WPair<NS>::kStageBytes;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int v = (2 * LW + q) * 16 + (lane >> 2);
      const int j = (lane & 3) ^ ((v >> 2) & 2);
      const int64_t m = m0 + v;
      const uint32_t mm = static_cast<uint32_t>(m < M ? m : 0);  // at most 2^30 voxels
      const uint32_t x = mm % static_cast<uint32_t>(a.w), t = mm / static_cast<uint32_t>(a.w);
      const uint32_t y = t % static_cast<uint32_t>(a.h), z = t / static_cast<uint32_t>(a.h);
      const uint16_t* pb = big + (2 * z * plane + 2 * y * row + 2 * x) * bc + b0 + 8 * j;
      const uint16_t* ps = small + static_cast<int64_t>(mm) * sc + s0 + 8 * j;
      const bool in_b = m < M && b0 + 8 * j < bc;
      char* dst = st + (2 * LW + q) * 1024;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        load_lds16(in_b ? pb + ((e >> 2) * plane + ((e >> 1) & 1) * row + (e & 1)) * bc : zero,
                   dst + e * 4096);
#pragma unroll
      for (int h = 0; h < NS / 2; ++h)
        load_lds16(m < M && s0 + 32 * h + 8 * j < sc ? ps + 32 * h : zero, dst + (8 + h) * 4096);
    }
  });
}

template <bool kUpGeo, int NS>
__global__ void __launch_bounds__(384) wgrad_pair_kernel(WgradArgs a) {
  __shared__ __align__(16) char s_st[3 * WPair<NS>::kStageBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t M = static_cast<int64_t>(a.d) * a.h * a.w;
  const int tiles = static_cast<int>((M + 63) / 64);
  const int nt = (tiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  const int b0 = blockIdx.y * 32, s0 = blockIdx.z * 16 * NS;
  if (wave == 4) {
    wpair_loader<kUpGeo, NS, 0>(a, s_st, lane, b0, s0, nt);
    return;
  }
  if (wave == 5) {
    wpair_loader<kUpGeo, NS, 1>(a, s_st, lane, b0, s0, nt);
    return;
  }
  const int r = lane & 15, g = lane >> 4;
  const int lo = tr_lane(lane) + g * 512;
  // the bias gradient: gy is the large operand (each wave sums its taps') or
  // the small one (the first wave does)
  constexpr int kSums = kUpGeo ? 2 : NS;
  const bool bias = a.gb && (kUpGeo ? s0 == 0 : b0 == 0 && wave == 0);
  floatx4 sum[kSums];
#pragma unroll
  for (int q = 0; q < kSums; ++q) sum[q] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 acc[2][NS][2];  // tap, small and large 16-channel block
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int q = 0; q < 2 * NS; ++q) acc[e][q >> 1][q & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0, slot = 0; s < nt; ++s) {
    barrier_lds();  // stage s has landed
    const char* st = s_st + slot * WPair<NS>::kStageBytes + lo;
    const char* h[2] = {st + (g & 1) * 32, st + ((g & 1) ^ 1) * 32};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 sf[NS], bf[2][2];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const char* p = h[q] + (2 * wave + e) * 4096 + ks * 2048;
          bf[e][q] = read_tr(p, p + 256);
        }
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        const char* p = h[q & 1] + (8 + (q >> 1)) * 4096 + ks * 2048;
        sf[q] = read_tr(p, p + 256);
      }
      if (bias) {
#pragma unroll
        for (int q = 0; q < kSums; ++q) {
          if constexpr (kUpGeo) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
              sum[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[e][q], ones8(), sum[q], 0, 0, 0);
          } else {
            sum[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sf[q], ones8(), sum[q], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc[e][q][c] =
                kUpGeo ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[e][c], sf[q], acc[e][q][c], 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_16x16x32_bf16(sf[q], bf[e][c], acc[e][q][c], 0, 0, 0);
    }
    slot = slot == 2 ? 0 : slot + 1;
  }
  if constexpr (kUpGeo) {
    // the waves' sums in order, through the first stage's memory: the loader
    // waves have ended, every compute wave has read its last fragments
    if (a.gb && s0 == 0) {
      float* sh = reinterpret_cast<float*>(s_st);
      barrier_lds();
      if (r == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          sh[wave * 32 + (i >> 2) * 16 + 4 * g + (i & 3)] = sum[i >> 2][i & 3];
      }
      barrier_lds();
      if (wave == 0 && lane < 32) {
        float t = sh[lane];
        for (int w = 1; w < 4; ++w) t += sh[w * 32 + lane];
        wgrad_put_bias(a, b0 + lane, t);
      }
    }
  } else if (bias && r == 0) {
#pragma unroll
    for (int i = 0; i < 4 * NS; ++i)
      wgrad_put_bias(a, s0 + (i >> 2) * 16 + 4 * g + (i & 3), sum[i >> 2][i & 3]);
  }
  // lane (r, g): four output channels of one input channel, as above
  wgrad_put<4 * NS>(
      a,
      [&](int k) -> int64_t {
        const int e = k / (2 * NS), q = (k >> 1) % NS, c = k & 1;
        const int n = (kUpGeo ? b0 + 16 * c : s0 + 16 * q) + 4 * g;
        const int ci = (kUpGeo ? s0 + 16 * q : b0 + 16 * c) + r;
        return n < a.cout && ci < a.cin
                   ? (static_cast<int64_t>(2 * wave + e) * a.cin + ci) * a.cout + n
                   : -1;
      },
      [&](int k) { return acc[k / (2 * NS)][(k >> 1) % NS][k & 1]; });
}

// ------------------------------------- 3x3x3 weight gradients with one channel
// Taps as a matrix axis (27 of 32 used).  kConv3 layers with cin == 1:
// gw[t][n] = sum_m x[m + d(t)] gy[m][n], rows t, columns n; with cout == 1:
// gw[t][ci] = sum_m x[m][ci] gy[m - d(t)], rows ci, columns t (the same sum
// with m shifted; x and gy are zero outside the volume).  A workgroup
// walks 4 x 4 x 4 tiles blockIdx.x, + gridDim.x, ... and owns 32 columns
// (cin == 1: output channels 32 blockIdx.z ..) or 32 rows (cout == 1: input
// channels 32 blockIdx.z ..); wave w computes the 16 x 16 block (w & 1,
// w >> 1).  Per tile the single-channel side is staged as a 6 x 6 x 6
// brick and the other side transposed to [channel][voxel]; sums go to
// part[blockIdx.x][t][ci][n] for wgrad_reduce_kernel.
template <bool kCin1>
__global__ void __launch_bounds__(256) wgrad_onechannel_kernel(WgradArgs a) {
  __shared__ uint16_t sB[216];                 // brick of the one-channel side
  __shared__ uint16_t sT[32][64 + kPadK];      // [channel][tile voxel] of the other side
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int rb = wave & 1, cb = wave >> 1;     // row block, column block
  const int c0 = static_cast<int>(blockIdx.z) * 32;  // first channel of the many-channel side
  const int cmany = kCin1 ? a.cout : a.cin;
  const int tx_n = (a.w + 3) >> 2, ty_n = (a.h + 3) >> 2, tz_n = (a.d + 3) >> 2;
  const int tiles = tx_n * ty_n * tz_n;
  const int sgn = kCin1 ? 1 : -1;  // brick offset of tap t: x at m + d(t), or gy at m - d(t)
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int bx = (tile % tx_n) * 4;
    const int by = ((tile / tx_n) % ty_n) * 4;
    const int bz = (tile / (tx_n * ty_n)) * 4;
    __syncthreads();
    if (tid < 216) {
      const int v = tid;
      const int gx = bx + v % 6 - 1, gy = by + (v / 6) % 6 - 1, gz = bz + v / 36 - 1;
      uint16_t val = 0;
      if (gx >= 0 && gy >= 0 && gz >= 0 && gx < a.w && gy < a.h && gz < a.d) {
        const int64_t o = (static_cast<int64_t>(gz) * a.h + gy) * a.w + gx;
        val = kCin1 ? a.x[o] : a.gy[o];
      }
      sB[v] = val;
    }
    for (int i = tid; i < 64 * 4; i += 256) {
      const int m = i >> 2, cc = (i & 3) * 8;
      const int x = bx + (m & 3), y = by + ((m >> 2) & 3), z = bz + (m >> 4);
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = 0;
      if (x < a.w && y < a.h && z < a.d) {
        const int64_t o = (static_cast<int64_t>(z) * a.h + y) * a.w + x;
        const uint16_t* row = (kCin1 ? a.gy : a.x) + o * cmany + c0 + cc;
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = (c0 + cc + j < cmany) ? row[j] : 0;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) sT[cc + j][m] = e[j];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      // voxels m = 32 ks + 8 g + j: x = j & 3, y = 2 (g & 1) + (j >> 2), z = 2 ks + (g >> 1)
      const int zz = 2 * ks + (g >> 1), y0 = 2 * (g & 1);
      // brick side: tap t = 16 (kCin1 ? rb : cb) + r at the 8 voxels
      const int t = 16 * (kCin1 ? rb : cb) + r;
      bf16x8 br;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        uint16_t e = 0;
        if (t < 27) {
          const int dz = sgn * (t / 9 - 1), dy = sgn * ((t / 3) % 3 - 1), dx = sgn * (t % 3 - 1);
          e = sB[((zz + 1 + dz) * 6 + (y0 + (j >> 2) + 1 + dy)) * 6 + ((j & 3) + 1 + dx)];
        }
        br[j] = __builtin_bit_cast(__bf16, e);
      }
      // channel side: channel 16 (kCin1 ? cb : rb) + r at the 8 voxels
      const bf16x8 ch = *reinterpret_cast<const bf16x8*>(
          &sT[16 * (kCin1 ? cb : rb) + r][32 * ks + 8 * g]);
      acc = kCin1 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(br, ch, acc, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(ch, br, acc, 0, 0, 0);
    }
  }
  // lane (r, g) holds D[4 g + i][r] of block (rb, cb)
  float* out = a.part + static_cast<int64_t>(blockIdx.x) * 27 * a.cin * a.cout;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 16 * rb + 4 * g + i, col = 16 * cb + r;
    const int t = kCin1 ? row : col;
    const int c = c0 + (kCin1 ? col : row);
    if (t < 27 && c < cmany) out[static_cast<int64_t>(t) * cmany + c] = acc[i];
  }
}

// sum i of a reduction: of the weights' (i < nw) or of the bias gradient
__device__ __forceinline__ void wgrad_finish(float* gw, int64_t nw, float* gb, int64_t i, float v,
                                             int overwrite) {
  float* p = i < nw ? gw + i : gb + (i - nw);
  *p = overwrite ? v : *p + v;
}

// the same for fewer than 8 workgroups: one thread per i
__global__ void wgrad_reduce_few_kernel(const float* part, int groups, int64_t n, float* gw,
                                        int64_t nw, float* gb, int overwrite) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    float v = part[i];
#pragma unroll 7
    for (int k = 1; k < groups; ++k) v += part[k * n + i];
    wgrad_finish(gw, nw, gb, i, v, overwrite);
  }
}

// gw[i] += (overwrite: =) sum over the workgroups k < groups of part[k][i]: a workgroup
// takes E = 256 / KL consecutive i; thread (q, il) sums k = q, q + KL, ...
// for i = E blockIdx.x + il, and the KL sums of each i are added in q order
template <int KL>
__global__ void __launch_bounds__(256) wgrad_reduce_kernel(const float* part, int groups,
                                                           int64_t n, float* gw, int64_t nw,
                                                           float* gb, int overwrite) {
  constexpr int E = 256 / KL;
  __shared__ float sh[KL][E + 1];
  const int il = threadIdx.x % E, q = threadIdx.x / E;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * E + il;
  float v = 0.f;
  if (i < n)
#pragma unroll 8
    for (int k = q; k < groups; k += KL) v += part[k * n + i];
  sh[q][il] = v;
  __syncthreads();
  if (q == 0 && i < n) {
    float t = sh[0][il];
#pragma unroll
    for (int k = 1; k < KL; ++k) t += sh[k][il];
    wgrad_finish(gw, nw, gb, i, t, overwrite);
  }
}

// ------------------------------------------------------------ element-wise

// Bt[n][t * cin + ci] (fwd) and Bt[ci][t * cout + n] (bwd, transposed) from
// w[t][ci][n], for every job in one launch: a workgroup takes one 32 x 32
// tile (ci, n) of one tap, reads it once and writes it to both (either may
// be null); tiles cover the rows up to a multiple of 64, zero beyond the
// weights, and the tiles at the end of the last tap also zero the columns up
// to kpad.  Bound by launches and by 2-byte scattered writes before: two
// launches per layer, one thread per weight, 130 us for the 16 layers of the
// (32, 64, 128, 256) network, 21 us as one launch.
__global__ void __launch_bounds__(256) pack_kernel(const PackJob* jobs, int njobs, PackJob one) {
  __shared__ uint16_t sh[32][34];
  int b = static_cast<int>(blockIdx.x);
  PackJob J = one;
  if (jobs) {
    int k = 0;
    while (k + 1 < njobs && b >= jobs[k].tiles()) b -= jobs[k++].tiles();
    J = jobs[k];
  }
  const int tn = PackJob::side(J.cout), tc = PackJob::side(J.cin);
  const int n0 = (b % tn) * 32, c0 = (b / tn % tc) * 32, t = b / (tn * tc);
  const int col = static_cast<int>(threadIdx.x) & 31, row = static_cast<int>(threadIdx.x) >> 5;
  const float* w = J.w + static_cast<int64_t>(t) * J.cin * J.cout;
#pragma unroll
  for (int i = row; i < 32; i += 8)
    sh[i][col] = c0 + i < J.cin && n0 + col < J.cout
                     ? to_bf16(w[static_cast<int64_t>(c0 + i) * J.cout + n0 + col]) : 0;
  __syncthreads();
  const bool last = t == J.taps - 1;
  if (J.fwd && c0 < J.cin) {
    const int k = t * J.cin + c0 + col;
    const bool end = last && c0 + 32 >= J.cin;  // up to 31 columns of zeros follow
    const bool here = c0 + col < J.cin || (end && k < J.fwd_kpad);
    const bool past = end && k + 32 < J.fwd_kpad;
#pragma unroll
    for (int i = row; i < 32; i += 8) {
      uint16_t* p = J.fwd + static_cast<int64_t>(n0 + i) * J.fwd_kpad + k;
      if (here) p[0] = sh[col][i];
      if (past) p[32] = 0;
    }
  }
  if (J.bwd && n0 < J.cout) {
    const int k = t * J.cout + n0 + col;
    const bool end = last && n0 + 32 >= J.cout;  // up to 31 columns of zeros follow
    const bool here = n0 + col < J.cout || (end && k < J.bwd_kpad);
    const bool past = end && k + 32 < J.bwd_kpad;
#pragma unroll
    for (int i = row; i < 32; i += 8) {
      uint16_t* p = J.bwd + static_cast<int64_t>(c0 + i) * J.bwd_kpad + k;
      if (here) p[0] = sh[i][col];
      if (past) p[32] = 0;
    }
  }
}

__global__ void zero2_kernel(double* acc, float* fmax) {
  acc[0] = 0.0;
  acc[1] = 0.0;
  fmax[0] = 0.f;
}

__global__ void fill_f32_kernel(float* p, int64_t n, float v) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

__global__ void fill2_f32_kernel(float* p, int64_t n, float* q, int64_t m) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n + m;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (i < n)
      p[i] = 0.f;
    else
      q[i - n] = 0.f;
  }
}

// u = (ln max(phi, eps) - shift) / scale, in FP32 and as BF16
__global__ void to_log_kernel(const float* phi, int64_t n, float eps, float shift, float inv_scale,
                              float* u, uint16_t* u16) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const float v = (logf(fmaxf(phi[i], eps)) - shift) * inv_scale;
    if (u) u[i] = v;
    if (u16) u16[i] = to_bf16(v);
  }
}

// the input voxel of output voxel (x, y, z) under the symmetry op (see mirror_xy_kernel)
__device__ __forceinline__ int64_t mirror_source(int x, int y, int64_t z, int nx, int ny, int op) {
  int sx = (op & 4) ? y : x;
  int sy = (op & 4) ? x : y;
  if (op & 1) sx = nx - 1 - sx;
  if (op & 2) sy = ny - 1 - sy;
  return (z * ny + sy) * nx + sx;
}

// out[z][y][x] = in[z][y'][x'], (x', y') = (op & 4 ? (y, x) : (x, y)) with
// x' mirrored when op & 1 and y' when op & 2: the eight symmetries of a
// square cross-section (the swap needs nx == ny)
__global__ void mirror_xy_kernel(const float* in, float* out, int nx, int ny, int64_t n, int op) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int x = static_cast<int>(i % nx);
    const int64_t r = i / nx;
    const int y = static_cast<int>(r % ny);
    const int64_t z = r / ny;
    out[i] = in[mirror_source(x, y, z, nx, ny, op)];
  }
}

// The network's inputs for the symmetries op0 .. op0 + nop - 1, one image
// each: to_log_kernel of mirror_xy_kernel's images.  u (FP32): that of the
// volume itself.
__global__ void __launch_bounds__(256) sym_inputs_kernel(const float* phi, int nx, int ny,
                                                         int64_t n, int op0, float eps, float shift,
                                                         float inv_scale, float* u,
                                                         uint16_t* u16) {
  const int op = op0 + blockIdx.y;
  uint16_t* out = u16 + blockIdx.y * n;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int x = static_cast<int>(i % nx);
    const int64_t r = i / nx;
    const int y = static_cast<int>(r % ny);
    const float v = (logf(fmaxf(phi[mirror_source(x, y, r / ny, nx, ny, op)], eps)) - shift) *
                    inv_scale;
    out[i] = to_bf16(v);
    if (op == 0) u[i] = v;
  }
}

// The outputs r + u of the symmetries op0 .. op0 + nop - 1, mapped back to
// the volume and added in order (an image's u, mapped back, is the volume's);
// acc holds the sum of the symmetries before op0, and receives the sum unless
// `last`: then the mean in u space and its fluence are written.
__global__ void __launch_bounds__(256) sym_outputs_kernel(const float* r, const float* u, int nx,
                                                          int ny, int64_t n, int op0, int nop,
                                                          float* acc, int last, float inv_nsym,
                                                          float scale, float shift, float* out_u,
                                                          float* phi) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int x = static_cast<int>(i % nx);
    const int64_t t = i / nx;
    const int y = static_cast<int>(t % ny);
    const int64_t z = t / ny;
    const float ui = u[i];
    float sum = op0 > 0 ? acc[i] : 0.f;
    for (int k = 0; k < nop; ++k) {
      // the inverse of op: a flip is its own inverse; with the swap, the
      // flips of x and y exchange
      const int op = op0 + k;
      const int inv = (op & 4) ? (4 | ((op & 1) << 1) | ((op & 2) >> 1)) : op;
      const float v = r[k * n + mirror_source(x, y, z, nx, ny, inv)] + ui;
      sum = op == 0 ? v : sum + v;
    }
    if (!last) {
      acc[i] = sum;
      continue;
    }
    const float v = sum * inv_nsym;
    if (out_u) out_u[i] = v;
    if (phi) phi[i] = expf(v * scale + shift);
  }
}

// phi_out = exp((r + u) * scale + shift): output of the residual network
__global__ void from_log_kernel(const float* r, const float* u, int64_t n, float scale, float shift,
                                float* out_u, float* phi) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const float v = r[i] + u[i];
    if (out_u) out_u[i] = v;
    if (phi) phi[i] = expf(v * scale + shift);
  }
}

// g16 = bf16((g + skip16) * (y16 > 0)); g may be FP32 or absent (skip
// only).  With `partial` set (and 256 a multiple of cout, so that a thread
// sees one channel in every grid-stride step) each block also writes its
// per-channel sums of g16 to partial[block][cout] for bias_sum_kernel.
__global__ void __launch_bounds__(256) relu_grad_kernel(const float* g, const uint16_t* skip16,
                                                        const uint16_t* y16, int64_t n, int cout,
                                                        uint16_t* g16, float* partial) {
  __shared__ float sh[256];
  float s = 0.f;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    float v = g ? g[i] : 0.f;
    if (skip16) v += from_bf16(skip16[i]);
    if (y16 && !(from_bf16(y16[i]) > 0.f)) v = 0.f;
    const uint16_t h = to_bf16(v);
    g16[i] = h;
    s += from_bf16(h);
  }
  if (!partial) return;
  // thread j's sums are of channel j % cout (cout a power of two dividing
  // 256): halve the block's 256 sums down to cout, pairing threads of one
  // channel (a tree, not one thread adding 256 / cout values in a row)
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off >= cout; off >>= 1) {
    if (static_cast<int>(threadIdx.x) < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (static_cast<int>(threadIdx.x) < cout)
    partial[static_cast<int64_t>(blockIdx.x) * cout + threadIdx.x] = sh[threadIdx.x];
}

// gb[c] += sum over blocks of partial[block][c]; one workgroup per channel
__global__ void __launch_bounds__(256) bias_sum_kernel(const float* partial, int blocks, int cout,
                                                       float* gb) {
  __shared__ float sh[4];
  const int c = blockIdx.x;
  float t = 0.f;
  for (int b = threadIdx.x; b < blocks; b += blockDim.x)
    t += partial[static_cast<int64_t>(b) * cout + c];
  for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) gb[c] += sh[0] + sh[1] + sh[2] + sh[3];
}

// the bias_sum_kernel sums of several layers in one launch: workgroup x
// takes channel x of the concatenated channels of `jobs`
__global__ void __launch_bounds__(256) bias_sums_kernel(const BiasJob* jobs, int njobs,
                                                        const float* partial, float* grads) {
  __shared__ float sh[4];
  int c = blockIdx.x, j = 0;
  while (j + 1 < njobs && c >= jobs[j].cout) c -= jobs[j++].cout;
  const BiasJob J = jobs[j];
  const float* p = partial + J.partial_off;
  float t = 0.f;
  for (int b = threadIdx.x; b < J.blocks; b += blockDim.x)
    t += p[static_cast<int64_t>(b) * J.cout + c];
  for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) grads[J.gb_off + c] += sh[0] + sh[1] + sh[2] + sh[3];
}

// block-wide sum of one double per thread (256 threads), returned to thread 0
__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) r += sh[w];
  __syncthreads();
  return r;
}

// masked squared error of out against target (both in u space): sum and
// count into acc[0..1] (FP64, one atomic per block), and the unnormalised
// gradient 2 (out - t) per masked voxel (zero elsewhere)
__global__ void __launch_bounds__(256) mse_kernel(const float* out, const float* target_u,
                                                  const float* target_phi, float rel_floor,
                                                  const float* phi_max, int64_t n, float* grad,
                                                  double* acc) {
  __shared__ double sh[4];
  double s = 0.0, c = 0.0;
  const float thr = rel_floor * phi_max[0];
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const bool on = target_phi[i] >= thr;
    const float d = on ? out[i] - target_u[i] : 0.f;
    grad[i] = 2.f * d;
    s += static_cast<double>(d) * d;
    c += on ? 1.0 : 0.0;
  }
  s = block_sum(s, sh);
  c = block_sum(c, sh);
  if (threadIdx.x == 0) {
    unsafeAtomicAdd(acc, s);
    unsafeAtomicAdd(acc + 1, c);
  }
}

__global__ void __launch_bounds__(256) max_kernel(const float* x, int64_t n, float* out) {
  __shared__ float sh[4];
  float m = 0.f;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    m = fmaxf(m, x[i]);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_down(m, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) m = fmaxf(m, sh[w]);
    atomicMax(reinterpret_cast<int*>(out), __float_as_int(m));  // m >= 0
  }
}

// grad *= 1 / count (count from acc[1])
__global__ void scale_grad_kernel(float* g, int64_t n, const double* acc) {
  const float s = acc[1] > 0.0 ? static_cast<float>(1.0 / acc[1]) : 0.f;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    g[i] *= s;
}

// gb[n] += sum over voxels of gy[m][n]: each block sums a range of rows and
// ends with one atomic per channel.  The memory side takes atomics on one
// address one at a time, so launch_bias_grad keeps the blocks few; with
// cout a multiple of 8 (kVec) a thread reads 8 channels of a row at once.
// 64^3 x 32: 21.7 us with 1024 blocks of 2-byte loads, 10 us.
template <bool kVec>
__global__ void __launch_bounds__(256) bias_grad_kernel(const uint16_t* gy, int64_t m, int cout,
                                                        int64_t rows_per_block, float* gb) {
  constexpr int W = kVec ? 8 : 1;  // channels per thread
  __shared__ float sh[256][W + 1];
  const int groups = cout / W;                       // threads' worth of channels in a row
  const int lanes_c = groups < 256 ? groups : 256;   // threads per row
  const int phases = 256 / lanes_c;                  // rows in flight
  const int tid = threadIdx.x;
  const int64_t r0 = blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < m ? r0 + rows_per_block : m;
  for (int c0 = 0; c0 < groups; c0 += lanes_c) {
    float s[W];
#pragma unroll
    for (int k = 0; k < W; ++k) s[k] = 0.f;
    const int c = c0 + tid % lanes_c;
    const int ph = tid / lanes_c;
    if (ph < phases && c < groups) {
#pragma unroll 4
      for (int64_t r = r0 + ph; r < r1; r += phases) {
        if constexpr (kVec) {
          const uint4 v = *reinterpret_cast<const uint4*>(gy + r * cout + c * 8);
          const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            s[2 * k] += __uint_as_float(w4[k] << 16);
            s[2 * k + 1] += __uint_as_float(w4[k] & 0xffff0000u);
          }
        } else {
          s[0] += from_bf16(gy[r * cout + c]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < W; ++k) sh[tid][k] = s[k];
    __syncthreads();
    // thread i adds channel i % W of the row's group i / W over the phases
    for (int i = tid; i < lanes_c * W; i += 256) {
      const int g = i / W, k = i % W;
      if (c0 + g >= groups) break;
      float t = 0.f;
#pragma unroll 8
      for (int p = 0; p < phases; ++p) t += sh[p * lanes_c + g][k];
      unsafeAtomicAdd(gb + (c0 + g) * W + k, t);
    }
    __syncthreads();
  }
}

// per-block sums of squares of g (for the global gradient norm)
__global__ void __launch_bounds__(256) sumsq_kernel(const float* g, int64_t n, double* partial) {
  __shared__ double sh[4];
  double s = 0.0;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    s += static_cast<double>(g[i]) * g[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Adam with bias-corrected moments on g * scale, where scale also clips
// the global norm: scale = gs * min(1, max_norm / (gs * |g|)) when
// max_norm > 0 (|g|^2 = sum of the `blocks` partial sums, which every block
// adds for itself: by all its threads -- one thread adding the 1024 in a row
// made a step of 5.4e6 parameters 187 us, 28 us now).  The update is
// bound by memory: seven floats per parameter.
__global__ void __launch_bounds__(256) adam_kernel(float* p, const float* g, float* m, float* v, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2, float gs,
                            float max_norm, const double* partial, int blocks) {
  __shared__ float s_scale;
  __shared__ double sh[4];
  double ss = 0.0;
  if (max_norm > 0.f) {
    for (int b = threadIdx.x; b < blocks; b += blockDim.x) ss += partial[b];
    ss = block_sum(ss, sh);
  }
  if (threadIdx.x == 0) {
    float sc = gs;
    if (max_norm > 0.f) {
      const double norm = gs * sqrt(ss);
      if (norm > max_norm) sc = static_cast<float>(gs * (max_norm / norm));
    }
    s_scale = sc;
  }
  __syncthreads();
  const float scale = s_scale;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const float gi = g[i] * scale;
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

int blocks_for(int64_t n, int per = 256, int cap = 8192) {
  const int64_t b = (n + per - 1) / per;
  return static_cast<int>(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

// --------------------------------------------------------------- launchers

namespace {

constexpr int64_t kSplitTargetGroups = 1024;  // about four workgroups per CU
constexpr int64_t kSplitBelowGroups = 512;    // split only launches smaller than this
constexpr int64_t kDeepTileGroups = 1024;     // 4 x 4 x 8 tiles when at least this many

int conv_nb(const ConvArgs& a) { return a.cout > 32 ? 4 : (a.cout > 16 ? 2 : 1); }

// the generic kernel takes operands at any address
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

bool uses_brick(const ConvArgs& a) {
  return (a.geo == kConv3 || a.geo == kConv3T) && a.cin % kBK == 0 && aligned16(a.x);
}

int64_t brick_tiles(const ConvArgs& a, int mz);
int64_t brick_ngroups(const ConvArgs& a);
// Few channels, whose weights a workgroup reads for its 64 voxels alone: where
// these are few (blocks of 8 channels x 16), or the reads of the whole launch.
// Measured, single layers, us, generic and this: 64^3 24 -> 16 (3 blocks) 78 and
// 53, 8 -> 64 68 and 59, 16 -> 32 (4) 71 and 77; 24^3 56 -> 56 (216 workgroups, 28
// blocks) 53 and 46, 32^3 56 -> 32 (512, 14) 51 and 46, 40 -> 64 (512, 20) 49 and 55.
bool uses_eights(const ConvArgs& a) {
  if ((a.geo != kConv3 && a.geo != kConv3T) || a.cin % 8 != 0 || a.cin % kBK == 0 || a.cin > 56 ||
      !aligned16(a.x))
    return false;
  const int blocks = a.cin / 8 * conv_nb(a);
  return a.cin == 8 || blocks <= 3 ||
         brick_tiles(a, 1) * brick_ngroups(a) * blocks <= 512 * 14;
}

bool uses_up(const ConvArgs& a) {
  return a.geo == kUp && a.cin % kBK == 0 && a.cout % 8 == 0 && aligned16(a.x) &&
         aligned16(a.y) && aligned16(a.skip);
}

// 64 voxels a wave where that leaves 512 workgroups, the classes apart if
// need be, else 32; the classes split until there are 512.  Measured (us, 256 /
// 512 / 1024 / 2048 workgroups): 32^3 64 -> 32 14.9 / 12.4 / 13.5 / 15.3, eight
// images of 16^3 128 -> 64 37.0 / 29.5 / 32.3 / 38.6; eight of 8^3 256 -> 128
// with 64 voxels 17.9, with 32 20.9.
template <int KC>
void launch_up(const ConvArgs& a, hipStream_t s) {
  const int64_t M = static_cast<int64_t>(a.batch) * a.d * a.h * a.w;
  const int nb = (a.cout + 31) / 32;
  const bool wide = (M + 255) / 256 * nb * 8 >= 512;
  const int64_t rows = (M + (wide ? 255 : 127)) / (wide ? 256 : 128);
  int z = 1;
  while (z < 8 && rows * nb * z < 512) z *= 2;
  const dim3 grid(static_cast<unsigned>(rows), static_cast<unsigned>(nb), static_cast<unsigned>(z));
  if (wide)
    up_kernel<KC, 4><<<grid, 256, 0, s>>>(a);
  else
    up_kernel<KC, 2><<<grid, 256, 0, s>>>(a);
}

// The resident-weights kernel: 3x3x3 layers gathering exactly 32 channels,
// without a skip input, on grids of at least kResidentTiles 4 x 4 x 8 tiles
// (the full-resolution layers; smaller grids keep the brick kernel, whose
// split reductions fill the chip).  Its output waves store 16-byte pieces: an
// output off that alignment goes to the brick kernel (64^3 32 -> 32: 69 us for
// 39, and 79 with this kernel's stores by element).
constexpr int64_t kResidentTiles = 1024;
bool uses_resident(const ConvArgs& a) {
  return (a.geo == kConv3 || a.geo == kConv3T) && a.cin == 32 && !a.skip && aligned16(a.x) &&
         aligned16(a.y) && aligned16(a.gmask) && brick_tiles(a, 2) >= kResidentTiles;
}

// 4 x 4 columns of all images, each a workgroup's unit of work
int64_t resident_columns(const ConvArgs& a) {
  return static_cast<int64_t>(a.batch) * ((a.w + 3) / 4) * ((a.h + 3) / 4);
}

// compute units of the current device (queried once)
int device_cus() {
  static int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

// tiles of all images
int64_t brick_tiles(const ConvArgs& a, int mz) {
  return static_cast<int64_t>(a.batch) * ((a.w + 3) / 4) * ((a.h + 3) / 4) *
         ((a.d + 4 * mz - 1) / (4 * mz));
}

int64_t brick_ngroups(const ConvArgs& a) {
  const int nb = conv_nb(a);
  return (a.cout + 16 * nb - 1) / (16 * nb);
}

// z-slices of a tile in fours: two when the launch keeps at least
// kDeepTileGroups workgroups with them
int deep_mz(const ConvArgs& a) {
  return brick_tiles(a, 2) * brick_ngroups(a) >= kDeepTileGroups ? 2 : 1;
}
// four, for 64 channels, when every CU has a workgroup and at most a fifth of
// the slices is padding (eight images of 16^3 128 -> 128: 59.9 us with one, 41.4
// with four; of 32^3 64 -> 64 87.5 with two, 85.6)
int brick_mz(const ConvArgs& a) {
  if (conv_nb(a) == 4 && brick_tiles(a, 4) * brick_ngroups(a) >= 256 &&
      5 * ((a.d + 15) / 16 * 16) <= 6 * a.d)
    return 4;
  return deep_mz(a);
}

// Ranges of the brick kernel's input-channel chunks, whose sums are added in
// order: chosen from one image, so that an image's results do not depend on
// how many share the launch.  For products of fewer than two workgroups per
// CU, enough ranges to fill the chip, a divisor of the chunk count.
int brick_ranges(ConvArgs a) {
  a.batch = 1;
  const int64_t groups = brick_tiles(a, deep_mz(a)) * brick_ngroups(a);
  if (groups >= kSplitBelowGroups) return 1;
  const int chunks = a.cin / kBK;
  int sp = static_cast<int>(std::min<int64_t>(chunks, (kSplitTargetGroups + groups - 1) / groups));
  while (sp > 1 && chunks % sp != 0) --sp;
  return sp;
}

// the same for the generic kernel's reduction of kDown products (the other
// geometries have one range), at least one stage of 128 each
int generic_ranges(ConvArgs a) {
  if (a.geo != kDown || a.cin % 8 != 0) return 1;
  const int64_t M = static_cast<int64_t>(a.d) * a.h * a.w;
  const int64_t groups = (M + kBM - 1) / kBM * ((a.cout + 16 * conv_nb(a) - 1) / (16 * conv_nb(a)));
  if (groups >= kSplitBelowGroups) return 1;
  return std::max(1, static_cast<int>(std::min<int64_t>(
                         a.k / (4 * kBK), (kSplitTargetGroups + groups - 1) / groups)));
}

int64_t out_floats(const ConvArgs& a) {
  return static_cast<int64_t>(a.batch) * a.d * a.h * a.w * a.cout;
}

// Whether the ranges go to workgroups of their own (and their sums through
// the workspace): only where the launch has few workgroups without that.
// Measured: 16^3 128 -> 128 (128 workgroups, 4 ranges) 15.1 + 4.6 us spread,
// 17.0 not; 8^3 (32 workgroups, 8 ranges) 10.8 + 4.6 us spread, and the two
// 256 -> 256 layers with the down layer before them 34 us longer if not; the
// generic kernel with 128 workgroups (4 ranges) 7.0 + 4.6 us and 13.4.
bool spread_ranges(const ConvArgs& a, int ranges) {
  if (ranges <= 1) return false;
  if (uses_brick(a)) return brick_tiles(a, brick_mz(a)) * brick_ngroups(a) < 128;
  const int nc = 16 * conv_nb(a);
  return (out_floats(a) / a.cout + kBM - 1) / kBM * ((a.cout + nc - 1) / nc) < 256;
}

}  // namespace

// the folded input gradient: resident-weights kConv3T products of 32
// channels to 32, without bias or ReLU of their own
bool conv_folds_grad(const ConvArgs& a) {
  return a.geo == kConv3T && uses_resident(a) && a.cout == 32 && !a.bias && !a.relu && !a.y_f32;
}

int conv_fold_rows(const ConvArgs& a) {
  return static_cast<int>(std::min<int64_t>(resident_columns(a), device_cus()));
}

int64_t conv_workspace_floats(const ConvArgs& a) {
  const int ranges = uses_brick(a) ? brick_ranges(a) : generic_ranges(a);
  return spread_ranges(a, ranges) ? ranges * out_floats(a) : 0;
}

hipError_t launch_conv(const ConvArgs& args, hipStream_t s) {
  ConvArgs a = args;
  const int nb = conv_nb(a);
  if ((a.geo == kConv3 || a.geo == kConv3T) && a.cin == 1) {
    const int64_t tiles = static_cast<int64_t>(a.batch) * ((a.w + 15) / 16) * ((a.h + 3) / 4) *
                          ((a.d + 3) / 4);
    const int np = a.cout > 32 ? 2 : 1;
    const dim3 grid(static_cast<unsigned>(tiles),
                    static_cast<unsigned>((a.cout + 32 * np - 1) / (32 * np)), 1);
    const int vec = a.cout % 8 == 0 && aligned16(a.y) && aligned16(a.skip);
    if (np == 2)
      conv3_scalar_kernel<2><<<grid, 256, 0, s>>>(a, vec);
    else
      conv3_scalar_kernel<1><<<grid, 256, 0, s>>>(a, vec);
    return hipGetLastError();
  }
  if (a.gmask && (!conv_folds_grad(a) || !a.gpart)) return hipErrorInvalidValue;
  if (uses_resident(a)) {
    const int nbr = a.cout > 16 ? 2 : 1;
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>(resident_columns(a), device_cus())),
                    static_cast<unsigned>((a.cout + 16 * nbr - 1) / (16 * nbr)), 1);
    if (a.gmask)  // conv_folds_grad: 32 output channels, BF16
      conv3_resident_kernel<2, false, true><<<grid, 448, 0, s>>>(a);
    else if (nbr == 2 && a.y_f32)
      conv3_resident_kernel<2, true, false><<<grid, 448, 0, s>>>(a);
    else if (nbr == 2)
      conv3_resident_kernel<2, false, false><<<grid, 448, 0, s>>>(a);
    else if (a.y_f32)
      conv3_resident_kernel<1, true, false><<<grid, 448, 0, s>>>(a);
    else
      conv3_resident_kernel<1, false, false><<<grid, 448, 0, s>>>(a);
    return hipGetLastError();
  }
  if (uses_brick(a)) {
    const int mz = brick_mz(a);
    a.ranges = brick_ranges(a);
    const int sp = spread_ranges(a, a.ranges) && a.part && a.part_cap >= a.ranges * out_floats(a)
                       ? a.ranges
                       : 1;
    // as many workgroups as the chip holds at once (by LDS two per CU, one with
    // deeper tiles of 64 channels), each with its share of the tiles
    const int64_t slots = device_cus() * (nb == 4 && mz > 1 ? 1 : 2);
    const int64_t others = brick_ngroups(a) * sp;
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>(
                        brick_tiles(a, mz), std::max<int64_t>(1, slots / others))),
                    static_cast<unsigned>(brick_ngroups(a)), static_cast<unsigned>(sp));
    const int vec = a.cout % 8 == 0 && aligned16(a.y) && aligned16(a.skip);
    if (nb == 4 && mz == 4)
      conv3_brick_kernel<4, 4><<<grid, 384, 0, s>>>(a, vec);
    else if (nb == 4 && mz == 2)
      conv3_brick_kernel<4, 2><<<grid, 384, 0, s>>>(a, vec);
    else if (nb == 4)
      conv3_brick_kernel<4, 1><<<grid, 384, 0, s>>>(a, vec);
    else if (nb == 2 && mz == 2)
      conv3_brick_kernel<2, 2><<<grid, 384, 0, s>>>(a, vec);
    else if (nb == 2)
      conv3_brick_kernel<2, 1><<<grid, 384, 0, s>>>(a, vec);
    else if (mz == 2)
      conv3_brick_kernel<1, 2><<<grid, 384, 0, s>>>(a, vec);
    else
      conv3_brick_kernel<1, 1><<<grid, 384, 0, s>>>(a, vec);
    if (sp > 1) split_reduce_kernel<<<blocks_for(out_floats(a)), 256, 0, s>>>(a, sp);
    return hipGetLastError();
  }
  if (uses_eights(a)) {
    const dim3 grid(static_cast<unsigned>(brick_tiles(a, 1)),
                    static_cast<unsigned>(brick_ngroups(a)), 1);
    const int vec = a.cout % 8 == 0 && aligned16(a.y) && aligned16(a.skip);
    if (nb == 4)
      conv3_eights_kernel<4><<<grid, 256, 0, s>>>(a, vec);
    else if (nb == 2)
      conv3_eights_kernel<2><<<grid, 256, 0, s>>>(a, vec);
    else
      conv3_eights_kernel<1><<<grid, 256, 0, s>>>(a, vec);
    return hipGetLastError();
  }
  if (uses_up(a)) {
    if (a.cin == 32)
      launch_up<1>(a, s);
    else if (a.cin == 64)
      launch_up<2>(a, s);
    else if (a.cin == 128)
      launch_up<4>(a, s);
    else if (a.cin == 256)
      launch_up<8>(a, s);
    else
      launch_up<0>(a, s);
    return hipGetLastError();
  }
  a.ranges = generic_ranges(a);
  const int sp = spread_ranges(a, a.ranges) && a.part && a.part_cap >= a.ranges * out_floats(a)
                     ? a.ranges
                     : 1;
  const int64_t M = static_cast<int64_t>(a.batch) * a.d * a.h * a.w;
  const dim3 grid(static_cast<unsigned>((M + kBM - 1) / kBM),
                  static_cast<unsigned>((a.cout + 16 * nb - 1) / (16 * nb)),
                  a.geo == kUp ? 8 : static_cast<unsigned>(sp));
  const bool vec = a.cin % 8 == 0 && aligned16(a.x);
  const bool deep = a.k >= 4 * kBK;  // four reduction steps per stage
#define MCX_CONV(NB)                                                   \
  if (vec && deep)                                                     \
    conv_kernel<NB, true, 4><<<grid, 256, 0, s>>>(a);                  \
  else if (vec)                                                        \
    conv_kernel<NB, true, 1><<<grid, 256, 0, s>>>(a);                  \
  else                                                                 \
    conv_kernel<NB, false, 1><<<grid, 256, 0, s>>>(a);
  if (nb == 4) { MCX_CONV(4) } else if (nb == 2) { MCX_CONV(2) } else { MCX_CONV(1) }
#undef MCX_CONV
  if (sp > 1) split_reduce_kernel<<<blocks_for(out_floats(a)), 256, 0, s>>>(a, sp);
  return hipGetLastError();
}

namespace {

constexpr int64_t kSlabTargetGroups = 512;
constexpr int64_t kSlabMaxPart = int64_t(8) << 20;  // floats of partial sums at most

bool uses_onechannel(const WgradArgs& a) {
  return a.geo == kConv3 && (a.cin == 1 || (a.cout == 1 && a.cin > 1));
}
// the kernels with transposing reads take 16-byte pieces of both operands
bool uses_tr(const WgradArgs& a) {
  return !uses_onechannel(a) && a.cin % 8 == 0 && a.cout % 8 == 0 && aligned16(a.x) &&
         aligned16(a.gy);
}
bool uses_slab(const WgradArgs& a) {
  return a.geo == kConv3 && a.cin % kBK == 0 && !uses_onechannel(a) && !uses_tr(a);
}

// their workgroups along the voxel tiles: one workgroup per CU in all
// (kTrGroups), at most one per tile, with the partial sums within `cap` floats
constexpr int64_t kTrGroups = 256;
int tr_ns(const WgradArgs& a) { return (a.geo == kUp ? a.cin : a.cout) > 32 ? 4 : 2; }
int64_t tr_tiles(const WgradArgs& a) {
  return a.geo == kConv3
             ? static_cast<int64_t>((a.w + 3) / 4) * ((a.h + 3) / 4) * ((a.d + 7) / 8)
             : (static_cast<int64_t>(a.d) * a.h * a.w + 63) / 64;
}
// workgroups for one of the tile groups, each with all the taps
int64_t tr_blocks(const WgradArgs& a) {
  if (a.geo == kConv3) return static_cast<int64_t>((a.cin + 31) / 32) * ((a.cout + 31) / 32);
  const int bc = a.geo == kUp ? a.cout : a.cin, sc = a.geo == kUp ? a.cin : a.cout;
  const int ns = 16 * tr_ns(a);
  return static_cast<int64_t>((bc + 31) / 32) * ((sc + ns - 1) / ns);
}
// A plane of taps per workgroup, a third of the partial sums for three times
// the loads, where a workgroup has at most two tiles.  Measured with the
// reduction, us, planes and not: 8^3 256 -> 256 15.7 and 24.3, 16^3 128 -> 128
// 21.1 and 26.6, 32^3 64 -> 64 (four tiles) 23.8 and 22.7.
bool tr_plane(const WgradArgs& a) {
  return a.geo == kConv3 && tr_tiles(a) * tr_blocks(a) <= 2 * kTrGroups;
}
int tr_groups(const WgradArgs& a, int64_t cap) {
  const int64_t other = tr_blocks(a) * (tr_plane(a) ? 3 : 1);
  int64_t G = std::min<int64_t>(tr_tiles(a), std::max<int64_t>(1, kTrGroups / other));
  const int64_t per = wgrad_floats(a);
  while (G > 1 && G * per > cap) G = (G + 1) / 2;
  return static_cast<int>(G);
}
// floats of their partial sums (one group needs none)
int64_t tr_part(const WgradArgs& a) {
  const int G = tr_groups(a, kSlabMaxPart);
  return G > 1 ? G * wgrad_floats(a) : 0;
}

// tile groups of the one-channel kernels: about kSlabTargetGroups in all
int onechannel_groups(const WgradArgs& a, int64_t cap) {
  const int64_t tiles = static_cast<int64_t>((a.w + 3) / 4) * ((a.h + 3) / 4) * ((a.d + 3) / 4);
  const int cmany = a.cin == 1 ? a.cout : a.cin;
  const int64_t other = (cmany + 31) / 32;
  int64_t G = std::min<int64_t>(tiles, (kSlabTargetGroups + other - 1) / other);
  const int64_t per = static_cast<int64_t>(a.taps) * a.cin * a.cout;
  while (G > 1 && G * per > cap) G = (G + 1) / 2;
  return static_cast<int>(G < 1 ? 1 : G);
}
int slab_nbw(const WgradArgs& a) { return a.cout > 32 ? 2 : 1; }

// workgroups along the voxel tiles: about kSlabKernelGroups in all (three
// per CU: the slab kernel's loads are latency-bound), at most one per tile,
// with the partial sums within `cap` floats
constexpr int64_t kSlabKernelGroups = 768;
int slab_groups(const WgradArgs& a, int64_t cap) {
  const int64_t tiles =
      static_cast<int64_t>((a.w + 3) / 4) * ((a.h + 3) / 4) * ((a.d + kSlabTZ - 1) / kSlabTZ);
  const int nbw = slab_nbw(a);
  const int64_t other = static_cast<int64_t>(a.cin / kBK) * 3 * ((a.cout + 32 * nbw - 1) / (32 * nbw));
  int64_t G = std::min<int64_t>(tiles, (kSlabKernelGroups + other - 1) / other);
  const int64_t per = static_cast<int64_t>(a.taps) * a.cin * a.cout;
  while (G > 1 && G * per > cap) G = (G + 1) / 2;
  return static_cast<int>(G < 1 ? 1 : G);
}

}  // namespace

namespace {

// the reduction of a's partial sums of G groups into gw and gb
hipError_t launch_wgrad_reduce(const WgradArgs& a, int G, hipStream_t s) {
  const int ow = a.overwrite ? 1 : 0;
  const int64_t n = wgrad_floats(a), nw = static_cast<int64_t>(a.taps) * a.cin * a.cout;
  if (G < 8)
    wgrad_reduce_few_kernel<<<blocks_for(n), 256, 0, s>>>(a.part, G, n, a.gw, nw, a.gb, ow);
  else if (G >= 64 && n < 8192)  // fewer than 256 workgroups with 8 lanes per i
    wgrad_reduce_kernel<32><<<static_cast<unsigned>((n + 7) / 8), 256, 0, s>>>(a.part, G, n, a.gw,
                                                                              nw, a.gb, ow);
  else
    wgrad_reduce_kernel<8><<<static_cast<unsigned>((n + 31) / 32), 256, 0, s>>>(a.part, G, n, a.gw,
                                                                              nw, a.gb, ow);
  return hipGetLastError();
}

}  // namespace

int64_t wgrad_workspace_floats(const WgradArgs& a) {
  if (uses_onechannel(a))
    return onechannel_groups(a, kSlabMaxPart) * static_cast<int64_t>(a.taps) * a.cin * a.cout;
  if (uses_tr(a)) return tr_part(a);
  if (!uses_slab(a)) return 0;
  return slab_groups(a, kSlabMaxPart) * static_cast<int64_t>(a.taps) * a.cin * a.cout;
}

bool wgrad_folds_bias(const WgradArgs& a) { return uses_tr(a); }

bool wgrad_overwrites(const WgradArgs& a) {
  return (uses_onechannel(a) || uses_tr(a) || uses_slab(a)) && wgrad_workspace_floats(a) <= kSlabMaxPart;
}

hipError_t launch_wgrad(const WgradArgs& a, hipStream_t s) {
  if (uses_onechannel(a) && a.part) {
    const int64_t per = static_cast<int64_t>(a.taps) * a.cin * a.cout;
    const int G = onechannel_groups(a, a.part_cap);
    if (static_cast<int64_t>(G) * per <= a.part_cap) {
      const int cmany = a.cin == 1 ? a.cout : a.cin;
      const dim3 grid(static_cast<unsigned>(G), 1, static_cast<unsigned>((cmany + 31) / 32));
      if (a.cin == 1)
        wgrad_onechannel_kernel<true><<<grid, 256, 0, s>>>(a);
      else
        wgrad_onechannel_kernel<false><<<grid, 256, 0, s>>>(a);
      return launch_wgrad_reduce(a, G, s);
    }
  }
  if (uses_tr(a)) {
    const int G = tr_groups(a, a.part ? a.part_cap : 0);
    const auto g = [&](int rows, int cols) {
      return dim3(static_cast<unsigned>(G), static_cast<unsigned>(rows),
                  static_cast<unsigned>(cols));
    };
    const int ns = tr_ns(a), cb = (a.cin + 31) / 32, nb = (a.cout + 31) / 32;
    const bool edge = a.w % 4 != 0 || a.h % 4 != 0 || a.d % 8 != 0;
    if (a.geo == kConv3 && tr_plane(a) && edge)
      wgrad_brick_kernel<true, true><<<g(3 * cb, nb), 384, 0, s>>>(a);
    else if (a.geo == kConv3 && tr_plane(a))
      wgrad_brick_kernel<true, false><<<g(3 * cb, nb), 384, 0, s>>>(a);
    else if (a.geo == kConv3 && edge)
      wgrad_brick_kernel<false, true><<<g(cb, nb), 384, 0, s>>>(a);
    else if (a.geo == kConv3)
      wgrad_brick_kernel<false, false><<<g(cb, nb), 384, 0, s>>>(a);
    else if (a.geo == kUp && ns == 4)
      wgrad_pair_kernel<true, 4><<<g(nb, (a.cin + 63) / 64), 384, 0, s>>>(a);
    else if (a.geo == kUp)
      wgrad_pair_kernel<true, 2><<<g(nb, 1), 384, 0, s>>>(a);
    else if (ns == 4)
      wgrad_pair_kernel<false, 4><<<g(cb, (a.cout + 63) / 64), 384, 0, s>>>(a);
    else
      wgrad_pair_kernel<false, 2><<<g(cb, 1), 384, 0, s>>>(a);
    if (G == 1) return hipGetLastError();
    return launch_wgrad_reduce(a, G, s);
  }
  if (uses_slab(a) && a.part) {
    const int64_t per = static_cast<int64_t>(a.taps) * a.cin * a.cout;
    const int G = slab_groups(a, a.part_cap);
    if (static_cast<int64_t>(G) * per <= a.part_cap) {
      const int nbw = slab_nbw(a);
      const dim3 grid(static_cast<unsigned>(G), static_cast<unsigned>(a.cin / kBK * 3),
                      static_cast<unsigned>((a.cout + 32 * nbw - 1) / (32 * nbw)));
      if (nbw == 2)
        wgrad_slab_kernel<2><<<grid, 256, 0, s>>>(a, aligned16(a.x));
      else
        wgrad_slab_kernel<1><<<grid, 256, 0, s>>>(a, aligned16(a.x));
      return launch_wgrad_reduce(a, G, s);
    }
  }
  const int64_t M = static_cast<int64_t>(a.d) * a.h * a.w;
  const int nb = a.cout > 32 ? 4 : (a.cout > 16 ? 2 : 1);
  const int P = a.taps * a.cin;
  const int ptiles = a.geo == kUp ? a.taps * ((a.cin + kBM - 1) / kBM) : (P + kBM - 1) / kBM;
  const dim3 grid(static_cast<unsigned>((M + a.m_per_block - 1) / a.m_per_block),
                  static_cast<unsigned>(ptiles),
                  static_cast<unsigned>((a.cout + 16 * nb - 1) / (16 * nb)));
  const bool vec = a.cin % 8 == 0 && aligned16(a.x);
  const bool vec_gy = a.cout % 8 == 0 && aligned16(a.gy);
#define MCX_WG(NB)                                                     \
  if (vec)                                                             \
    wgrad_kernel<NB, true><<<grid, 256, 0, s>>>(a, vec_gy);            \
  else                                                                 \
    wgrad_kernel<NB, false><<<grid, 256, 0, s>>>(a, vec_gy);
  if (nb == 4) { MCX_WG(4) } else if (nb == 2) { MCX_WG(2) } else { MCX_WG(1) }
#undef MCX_WG
  return hipGetLastError();
}

hipError_t launch_pack(const PackJob* dev_jobs, int njobs, int tiles, hipStream_t s) {
  pack_kernel<<<tiles, 256, 0, s>>>(dev_jobs, njobs, PackJob{});
  return hipGetLastError();
}

hipError_t launch_pack(const PackJob& job, hipStream_t s) {
  pack_kernel<<<job.tiles(), 256, 0, s>>>(nullptr, 1, job);
  return hipGetLastError();
}

hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t s) {
  fill_f32_kernel<<<blocks_for(n), 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill2(float* p, int64_t n, float* q, int64_t m, hipStream_t s) {
  if (n + m == 0) return hipSuccess;
  fill2_f32_kernel<<<blocks_for(n + m), 256, 0, s>>>(p, n, q, m);
  return hipGetLastError();
}

hipError_t launch_to_log(const float* phi, int64_t n, float* u, uint16_t* u16, hipStream_t s) {
  to_log_kernel<<<blocks_for(n), 256, 0, s>>>(phi, n, kEps, kLogShift, 1.f / kLogScale, u, u16);
  return hipGetLastError();
}

hipError_t launch_mirror_xy(const float* in, float* out, int nx, int ny, int nz, int op,
                            hipStream_t s) {
  const int64_t n = static_cast<int64_t>(nx) * ny * nz;
  mirror_xy_kernel<<<blocks_for(n), 256, 0, s>>>(in, out, nx, ny, n, op);
  return hipGetLastError();
}

hipError_t launch_sym_inputs(const float* phi, int nx, int ny, int nz, int op0, int nop, float* u,
                             uint16_t* u16, hipStream_t s) {
  const int64_t n = static_cast<int64_t>(nx) * ny * nz;
  const dim3 grid(static_cast<unsigned>(blocks_for(n)), static_cast<unsigned>(nop), 1);
  sym_inputs_kernel<<<grid, 256, 0, s>>>(phi, nx, ny, n, op0, kEps, kLogShift, 1.f / kLogScale, u,
                                         u16);
  return hipGetLastError();
}

hipError_t launch_sym_outputs(const float* r, const float* u, int nx, int ny, int nz, int op0,
                              int nop, int nsym, float* acc, float* out_u, float* phi,
                              hipStream_t s) {
  const int64_t n = static_cast<int64_t>(nx) * ny * nz;
  sym_outputs_kernel<<<blocks_for(n), 256, 0, s>>>(
      r, u, nx, ny, n, op0, nop, acc, op0 + nop == nsym, 1.f / static_cast<float>(nsym), kLogScale,
      kLogShift, out_u, phi);
  return hipGetLastError();
}

hipError_t launch_from_log(const float* r, const float* u, int64_t n, float* out_u, float* phi,
                           hipStream_t s) {
  from_log_kernel<<<blocks_for(n), 256, 0, s>>>(r, u, n, kLogScale, kLogShift, out_u, phi);
  return hipGetLastError();
}

hipError_t launch_mse(const float* out, const float* target_u, const float* target_phi,
                      float rel_floor, int64_t n, float* grad, double* acc, float* phi_max,
                      hipStream_t s) {
  // at most 128 blocks: each ends with atomics on one address (one per
  // block for the maximum, two for the sums), which the memory side takes
  // one at a time
  zero2_kernel<<<1, 1, 0, s>>>(acc, phi_max);
  max_kernel<<<blocks_for(n, 256, 128), 256, 0, s>>>(target_phi, n, phi_max);
  mse_kernel<<<blocks_for(n, 256, 128), 256, 0, s>>>(out, target_u, target_phi, rel_floor,
                                                    phi_max, n, grad, acc);
  scale_grad_kernel<<<blocks_for(n), 256, 0, s>>>(grad, n, acc);
  return hipGetLastError();
}

hipError_t launch_bias_grad(const uint16_t* gy, int64_t m, int cout, float* gb, hipStream_t s) {
  const int64_t blocks = m < 512 ? 1 : (m / 256 < 256 ? m / 256 : 256);
  const int64_t per = (m + blocks - 1) / blocks;
  if (cout % 8 == 0 && aligned16(gy))
    bias_grad_kernel<true><<<static_cast<int>(blocks), 256, 0, s>>>(gy, m, cout, per, gb);
  else
    bias_grad_kernel<false><<<static_cast<int>(blocks), 256, 0, s>>>(gy, m, cout, per, gb);
  return hipGetLastError();
}

hipError_t launch_relu_grad(const float* g, const uint16_t* skip16, const uint16_t* y16, int64_t n,
                            int cout, uint16_t* g16, float* gb, float* partial, hipStream_t s) {
  const int blocks = blocks_for(n, 256, kBiasBlocks);
  const bool fused = gb && partial && cout <= 256 && 256 % cout == 0;
  relu_grad_kernel<<<blocks, 256, 0, s>>>(g, skip16, y16, n, cout, g16,
                                          fused ? partial : nullptr);
  if (fused) {
    bias_sum_kernel<<<cout, 256, 0, s>>>(partial, blocks, cout, gb);
    return hipGetLastError();
  }
  if (gb) return launch_bias_grad(g16, n / cout, cout, gb, s);
  return hipGetLastError();
}

bool relu_grad_defers(int cout) { return cout <= 256 && 256 % cout == 0; }

int relu_grad_blocks(int64_t n) { return blocks_for(n, 256, kBiasBlocks); }

hipError_t launch_relu_grad_deferred(const float* g, const uint16_t* skip16, const uint16_t* y16,
                                     int64_t n, int cout, uint16_t* g16, float* gb, float* partial,
                                     hipStream_t s) {
  if (!relu_grad_defers(cout)) return launch_relu_grad(g, skip16, y16, n, cout, g16, gb, nullptr, s);
  relu_grad_kernel<<<relu_grad_blocks(n), 256, 0, s>>>(g, skip16, y16, n, cout, g16, partial);
  return hipGetLastError();
}

hipError_t launch_bias_sums(const BiasJob* jobs, int njobs, int channels, const float* partial,
                            float* grads, hipStream_t s) {
  if (njobs > 0 && channels > 0)
    bias_sums_kernel<<<channels, 256, 0, s>>>(jobs, njobs, partial, grads);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, int step,
                       float grad_scale, float max_norm, double* partial, hipStream_t s) {
  const double c1 = 1.0 - std::pow(0.9, step), c2 = 1.0 - std::pow(0.999, step);
  int blocks = 0;
  if (max_norm > 0.f) {
    blocks = blocks_for(n, 256, kNormBlocks);
    sumsq_kernel<<<blocks, 256, 0, s>>>(g, n, partial);
  }
  adam_kernel<<<blocks_for(n, 256, 2048), 256, 0, s>>>(p, g, m, v, n, lr, 0.9f, 0.999f, 1e-8f,
                                            static_cast<float>(c1), static_cast<float>(c2),
                                            grad_scale, max_norm, partial, blocks);
  return hipGetLastError();
}

}  // namespace nn
}  // namespace mcx
