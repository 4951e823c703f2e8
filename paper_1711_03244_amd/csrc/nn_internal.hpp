// Internal interfaces of the denoiser kernels (nn_kernels.hip) used by the
// denoiser runtime (nn_runtime.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcx {
namespace nn {

// log-space input transform u = (ln max(phi, kEps) - kLogShift) / kLogScale
constexpr float kEps = 1e-12f;
constexpr float kLogShift = -16.f;
constexpr float kLogScale = 4.f;

enum Geometry : int32_t { kConv3 = 0, kConv3T = 1, kDown = 2, kUp = 3 };

// One implicit-GEMM convolution.  Rows m run over the d x h x w grid
// (kConv3/kConv3T: the output grid = input grid; kDown: the output grid;
// kUp: the input grid, the output being twice as large per axis).
struct ConvArgs {
  int32_t geo;
  int32_t d, h, w;            // grid of rows
  int32_t in_d, in_h, in_w;   // grid of x (for bounds of kConv3/kConv3T)
  int32_t cin, cout;          // channels of x and of y
  int32_t k;                  // reduction length: taps * cin (kUp: cin)
  int32_t kpad;               // row length of bt
  const uint16_t* x;          // BF16 [voxel][cin]
  const uint16_t* bt;         // BF16 [>= cout rounded to 64][kpad]
  const float* bias;          // [cout] or null
  const uint16_t* skip;       // BF16 [out voxel][cout] added before ReLU, or null
  void* y;                    // BF16 or FP32 [out voxel][cout]
  int32_t y_f32, relu;
  float* part;                // FP32 workspace for split reductions, or null
  int64_t part_cap;           // its size in floats
  int32_t batch = 1;          // images: x, skip and y hold that many volumes one after another
  int32_t ranges = 1;         // ranges of the reduction, added in order (set by launch_conv)
  // An input gradient with the next step of the backward pass folded in
  // (conv_folds_grad): when gmask is set, y receives the BF16 gradient of
  // the layer below's pre-activation, bf16(sum * (gmask > 0)), and
  // gpart[workgroup][cout] the per-workgroup channel sums of those BF16
  // values (its bias gradient, for launch_bias_sums).
  const uint16_t* gmask = nullptr;  // BF16 [out voxel][cout]: the layer below's output
  float* gpart = nullptr;
};

// Whether launch_conv can fold the ReLU mask, BF16 rounding and bias sums
// into this input-gradient product (see ConvArgs::gmask), and
// the number of channel-sum rows it then writes to gpart.
bool conv_folds_grad(const ConvArgs& a);
int conv_fold_rows(const ConvArgs& a);

// Weight gradient gw[t][ci][n] += sum_m A(m, t, ci) gy(m, n) (FP32 atomics).
struct WgradArgs {
  int32_t geo;                // kConv3, kDown or kUp (the layer's forward geometry)
  int32_t d, h, w;            // grid of m: the output grid (kConv3, kDown), the input grid (kUp)
  int32_t taps, cin, cout;
  int64_t m_per_block;        // voxels per workgroup (multiple of 32)
  ConvArgs g;                 // geometry fields for the gather (geo, in_d, in_h, in_w)
  const uint16_t* x;          // BF16 [voxel][cin], the layer input
  const uint16_t* gy;         // BF16 [voxel][cout], gradient of the layer output
  float* gw;                  // FP32 [taps][cin][cout], accumulated
  float* part;                // FP32 workspace for per-workgroup partial sums, or null
  int64_t part_cap;           // its size in floats
  bool overwrite = false;     // gw (and gb) receive the sum instead (wgrad_overwrites)
  float* gb = nullptr;        // also gb[n] += sum_m gy(m, n), where wgrad_folds_bias
};

hipError_t launch_conv(const ConvArgs& a, hipStream_t s);
// floats of split-reduction workspace launch_conv would use for `a` (0: none;
// the results are the same without it)
int64_t conv_workspace_floats(const ConvArgs& a);
hipError_t launch_wgrad(const WgradArgs& a, hipStream_t s);
// floats of workspace launch_wgrad uses for `a` (0: it needs none)
int64_t wgrad_workspace_floats(const WgradArgs& a);
// whether launch_wgrad can take the bias gradient along (WgradArgs::gb; to be
// set before wgrad_workspace_floats)
bool wgrad_folds_bias(const WgradArgs& a);
// whether launch_wgrad with its workspace can store to gw instead of adding
bool wgrad_overwrites(const WgradArgs& a);
// One layer's weights w[taps][cin][cout] (FP32) to pack into BF16 rows:
// forward Bt[n][t * cin + ci] (cout rows rounded up to 64) and transposed
// Bt[ci][t * cout + n] (cin rows rounded up to 64), each kpad columns; what
// lies outside the weights is zeroed.  Either target may be null.
struct PackJob {
  const float* w = nullptr;
  uint16_t* fwd = nullptr;
  uint16_t* bwd = nullptr;
  int32_t taps = 0, cin = 0, cout = 0;
  int32_t fwd_kpad = 0, bwd_kpad = 0;
  // 32-wide tiles along `c` channels, up to a multiple of 64
  __host__ __device__ static int side(int c) { return (c + 63) / 64 * 2; }
  __host__ __device__ int tiles() const { return taps * side(cin) * side(cout); }
};
// all jobs of a device array (`tiles` in all), or one given by value
hipError_t launch_pack(const PackJob* dev_jobs, int njobs, int tiles, hipStream_t s);
hipError_t launch_pack(const PackJob& job, hipStream_t s);
hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t s);
// zero p[0, n) and q[0, m) in one launch (none when both are empty)
hipError_t launch_fill2(float* p, int64_t n, float* q, int64_t m, hipStream_t s);
hipError_t launch_to_log(const float* phi, int64_t n, float* u, uint16_t* u16, hipStream_t s);
hipError_t launch_mirror_xy(const float* in, float* out, int nx, int ny, int nz, int op,
                            hipStream_t s);
// BF16 log-space inputs u16[k][voxel] of phi under the symmetries op0 + k, k < nop
// (as launch_mirror_xy), and for op 0 phi's own in FP32, u
hipError_t launch_sym_inputs(const float* phi, int nx, int ny, int nz, int op0, int nop, float* u,
                             uint16_t* u16, hipStream_t s);
// The network outputs r[k][voxel] of those inputs plus u, mapped back and
// added to acc (which the first op starts); when op0 + nop == nsym instead
// out_u = the sum / nsym and phi = its fluence (either may be null).
hipError_t launch_sym_outputs(const float* r, const float* u, int nx, int ny, int nz, int op0,
                              int nop, int nsym, float* acc, float* out_u, float* phi,
                              hipStream_t s);
hipError_t launch_from_log(const float* r, const float* u, int64_t n, float* out_u, float* phi,
                           hipStream_t s);
// g16 = bf16((g + skip16) * (y16 > 0)) over n = voxels * cout values;
// with gb set, also gb[c] += sum over voxels of g16[.][c] (through
// `partial`, kBiasBlocks * cout floats of scratch)
constexpr int kBiasBlocks = 2048;
hipError_t launch_relu_grad(const float* g, const uint16_t* skip16, const uint16_t* y16, int64_t n,
                            int cout, uint16_t* g16, float* gb, float* partial, hipStream_t s);
// The same with the bias sums deferred: when relu_grad_defers(cout), the
// per-block channel sums go to partial[relu_grad_blocks(n)][cout] and a
// later launch_bias_sums adds them to the gradients; otherwise the bias
// gradient is added at once, as launch_relu_grad does.
bool relu_grad_defers(int cout);
int relu_grad_blocks(int64_t n);
hipError_t launch_relu_grad_deferred(const float* g, const uint16_t* skip16, const uint16_t* y16,
                                     int64_t n, int cout, uint16_t* g16, float* gb, float* partial,
                                     hipStream_t s);
// One deferred bias sum: grads[gb_off + c] += sum over b < blocks of
// partial[partial_off + b * cout + c], c < cout.
struct BiasJob {
  int64_t partial_off;
  int64_t gb_off;
  int32_t blocks;
  int32_t cout;
};
// all jobs (a device array) in one launch; channels = sum of their couts
hipError_t launch_bias_sums(const BiasJob* jobs, int njobs, int channels, const float* partial,
                            float* grads, hipStream_t s);
// masked MSE in u space; target voxels with phi >= rel_floor * max(phi)
// count; grad = 2 (out - t) / count there.  acc[0] = sum of squares,
// acc[1] = count (FP64); phi_max: one float of scratch
hipError_t launch_mse(const float* out, const float* target_u, const float* target_phi,
                      float rel_floor, int64_t n, float* grad, double* acc, float* phi_max,
                      hipStream_t s);
hipError_t launch_bias_grad(const uint16_t* gy, int64_t m, int cout, float* gb, hipStream_t s);
// Adam step on grad_scale * g, clipped to global norm max_norm (> 0);
// partial: kNormBlocks doubles of scratch
constexpr int kNormBlocks = 1024;
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, int step,
                       float grad_scale, float max_norm, double* partial, hipStream_t s);

}  // namespace nn
}  // namespace mcx
