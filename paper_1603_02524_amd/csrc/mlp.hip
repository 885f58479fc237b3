// Overlap-weight network: forward, backward and Adam kernels (FP32, gfx950).
//
// x (IN) -> tanh(W1 x + b1) (HID) -> tanh(W2 h1 + b2) (HID) -> W3 h2 + b3 (OUT).
// Parameter layout: W1 (HID x IN, row-major), b1, W2 (HID x HID), b2, W3 (OUT x HID), b3.
// Loss L = (1/B) sum_b sum_o (y_bo - t_bo)^2.  All reductions over the batch run
// in a fixed order, so gradients are reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>
#include <string>

#include "../../include/dgmg.h"

void dgmg_set_global_error(const std::string& msg);

namespace {

constexpr int IN = DGMG_MLP_IN, HID = DGMG_MLP_HIDDEN, OUT = DGMG_MLP_OUT;
constexpr int OW1 = 0, OB1 = OW1 + HID * IN, OW2 = OB1 + HID, OB2 = OW2 + HID * HID, OW3 = OB2 + HID,
              OB3 = OW3 + OUT * HID, NPAR = OB3 + OUT;
static_assert(NPAR == DGMG_MLP_PARAMS, "parameter count");

// 16x16x4 FP32 matrix product: A[i][k] from lane i + 16 k, B[k][j] from lane
// j + 16 k; result register r of lane l holds D[4 (l / 16) + r][l % 16].  The
// contraction index may be dealt to (lane group, step) in any order that A and
// B share: k = 16 (l / 16) + step makes a lane's 16 values consecutive.
typedef float acc4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ acc4 mfma(float a, float b, acc4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int TH = 256;      // block size: 4 waves, one per 16 hidden units
constexpr int FS = 16;       // samples of a forward block
constexpr int GS = 64;       // samples of a tile of the gradient
constexpr int HP = HID + 4;  // LDS pitch of a row of hidden values (rows stay 16-byte aligned)
static_assert(HID == 64 && TH / 64 * 16 == HID, "one wave per 16 hidden units");

// Forward pass of FS samples per block; work holds h1 and h2 (B x 2 HID).  The
// second layer runs on the matrix cores (W2 as the A operand, the samples as
// the columns).  Bound by latency (6144 samples: 379 KB, 65 MFLOP): 6.5 us, against
// 19.4 us for one wave per sample reading its rows of W2 from global memory.
__global__ void __launch_bounds__(TH) k_mlp_forward(const float* __restrict__ p, const float* __restrict__ X, int B,
                                                    float* __restrict__ Y, float* __restrict__ work) {
  __shared__ float xs[FS][IN];
  __shared__ __align__(16) float h1[FS][HP], h2[FS][HP];
  const int tid = threadIdx.x, b0 = blockIdx.x * FS, n = B - b0 < FS ? B - b0 : FS;
  const int lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  if (tid < FS * IN) xs[tid / IN][tid % IN] = tid < n * IN ? X[(size_t)b0 * IN + tid] : 0.0f;
  float w2[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) w2[k] = p[OW2 + (16 * wave + li) * HID + 16 * lk + k];
  {
    const int j = lane;
    float w1[IN];
#pragma unroll
    for (int k = 0; k < IN; ++k) w1[k] = p[OW1 + j * IN + k];
    const float b1 = p[OB1 + j];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < FS / 4; ++q) {
      const int s = wave + 4 * q;
      float a = b1;
#pragma unroll
      for (int k = 0; k < IN; ++k) a += w1[k] * xs[s][k];
      a = tanhf(a);
      h1[s][j] = a;
      if (s < n) work[(size_t)(b0 + s) * 2 * HID + j] = a;
    }
  }
  acc4 acc;
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] = p[OB2 + 16 * wave + 4 * lk + r];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) acc = mfma(w2[k], h1[li][16 * lk + k], acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int j = 16 * wave + 4 * lk + r;
    const float h = tanhf(acc[r]);
    h2[li][j] = h;
    if (li < n) work[(size_t)(b0 + li) * 2 * HID + HID + j] = h;
  }
  __syncthreads();
  // output o of sample s: 8 lanes of 8 products each
  const int s = tid / 16, o = (tid / 8) % OUT, part = tid & 7;
  float y = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) y += p[OW3 + o * HID + 8 * part + k] * h2[s][8 * part + k];
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) y += __shfl_xor(y, m, 64);
  if (part == 0 && s < n) Y[(size_t)(b0 + s) * OUT + o] = p[OB3 + o] + y;
}

// Number of partial gradients: one per GS samples, as many as fit the caller's
// scratch of B (2 HID + OUT) floats (always at least one sample chunk; a single
// chunk writes the gradient itself and needs no scratch).
int grad_chunks(int B) {
  const int64_t fit = (int64_t)B * (2 * HID + OUT) / NPAR, want = ((int64_t)B + GS - 1) / GS;
  return (int)(fit < 1 ? 1 : (want < fit ? want : fit));
}

// Gradient over one chunk of samples per block, in tiles of GS: the deltas of a
// tile stay in LDS, both 64 x 64 x 64 contractions (the delta of layer 1 and the
// gradient of W2) run on the matrix cores, the sums of the small layers on the
// VALU.  The sums over the batch run in a fixed order (tile by tile, then chunk by
// chunk in k_mlp_grad_sum).  One thread per parameter walking the whole batch, as
// before, left 19 blocks of one serial chain each: 1566 us at 6144 samples,
// against 17.5 us for this kernel and 4.0 us for the sum of its partials.
__global__ void __launch_bounds__(TH) k_mlp_grad(const float* __restrict__ p, const float* __restrict__ X,
                                                 const float* __restrict__ T, int B, int per,
                                                 const float* __restrict__ Y, const float* __restrict__ work,
                                                 float* __restrict__ out) {
  __shared__ __align__(16) float h1[GS][HP], h2[GS][HP], d2[GS][HP];
  __shared__ float xs[GS][IN], dy[GS][OUT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int first = blockIdx.x * per, last = B - first < per ? B : first + per;
  float* __restrict__ g = out + (size_t)blockIdx.x * NPAR;
  float w2t[16];  // column 16 wave + li of W2
#pragma unroll
  for (int k = 0; k < 16; ++k) w2t[k] = p[OW2 + (16 * lk + k) * HID + 16 * wave + li];
  acc4 gw2[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) gw2[c] = acc4{0, 0, 0, 0};
  // the small sums: W1 (HID x IN), b1, b2, W3 (OUT x HID), b3
  constexpr int NS = HID * IN + 2 * HID + OUT * HID + OUT, NQ = (NS + TH - 1) / TH;
  float small[NQ];
#pragma unroll
  for (int c = 0; c < NQ; ++c) small[c] = 0.0f;
  for (int b0 = first; b0 < last; b0 += GS) {
    const int n = last - b0 < GS ? last - b0 : GS;
    for (int q = tid; q < GS * HID; q += TH) {
      const int s = q / HID, j = q % HID;
      const bool ok = s < n;
      const float* w = work + (size_t)(b0 + (ok ? s : 0)) * 2 * HID;
      h1[s][j] = ok ? w[j] : 0.0f;
      h2[s][j] = ok ? w[HID + j] : 0.0f;
    }
    for (int q = tid; q < GS * IN; q += TH) xs[q / IN][q % IN] = q < n * IN ? X[(size_t)b0 * IN + q] : 0.0f;
    if (tid < GS * OUT)
      dy[tid / OUT][tid % OUT] =
          tid < n * OUT ? 2.0f * (Y[(size_t)b0 * OUT + tid] - T[(size_t)b0 * OUT + tid]) / (float)B : 0.0f;
    __syncthreads();
    {
      const int j = lane;
      float w3[OUT];
#pragma unroll
      for (int o = 0; o < OUT; ++o) w3[o] = p[OW3 + o * HID + j];
      for (int s = wave; s < GS; s += TH / 64) {
        float a = 0.0f;
#pragma unroll
        for (int o = 0; o < OUT; ++o) a += dy[s][o] * w3[o];
        const float h = h2[s][j];
        d2[s][j] = s < n ? a * (1.0f - h * h) : 0.0f;  // (the padding is 0 whatever the weights)
      }
    }
    __syncthreads();
    // W2 gradient: rows j = 16 wave + .., columns k, contraction over the samples
    for (int k = 0; k < GS / 4; ++k) {
      const int s = 4 * k + lk;
      const float a = d2[s][16 * wave + li];
#pragma unroll
      for (int c = 0; c < 4; ++c) gw2[c] = mfma(a, h1[s][16 * c + li], gw2[c]);
    }
    __syncthreads();
    // h1[s][k] <- d1[s][k] = (1 - h1^2) sum_j d2[s][j] W2[j][k]: rows k = 16 wave + .., columns s
#pragma unroll
    for (int c = 0; c < GS / 16; ++c) {
      acc4 a = acc4{0, 0, 0, 0};
      const int s = 16 * c + li;
#pragma unroll
      for (int k = 0; k < 16; ++k) a = mfma(w2t[k], d2[s][16 * lk + k], a);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * wave + 4 * lk + r;
        const float h = h1[s][k];
        h1[s][k] = s < n ? a[r] * (1.0f - h * h) : 0.0f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
      const int q = tid + c * TH;
      if (q >= NS) break;
      float s = 0.0f;
      if (q < HID * IN) {
        for (int b = 0; b < GS; ++b) s += h1[b][q / IN] * xs[b][q % IN];
      } else if (q < HID * IN + 2 * HID) {
        const int j = q - HID * IN;
        float(*d)[HP] = j < HID ? h1 : d2;
        for (int b = 0; b < GS; ++b) s += d[b][j % HID];
      } else if (q < NS - OUT) {
        const int j = q - HID * IN - 2 * HID;
        for (int b = 0; b < GS; ++b) s += dy[b][j / HID] * h2[b][j % HID];
      } else {
        for (int b = 0; b < GS; ++b) s += dy[b][q - (NS - OUT)];
      }
      small[c] += s;
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) g[OW2 + (16 * wave + 4 * lk + r) * HID + 16 * c + li] = gw2[c][r];
#pragma unroll
  for (int c = 0; c < NQ; ++c) {
    const int q = tid + c * TH;
    if (q >= NS) break;
    int at;  // q counts W1, b1, b2, W3, b3 without W2
    if (q < OW2) at = q;
    else at = OB2 + (q - OW2);
    g[at] = small[c];
  }
}

// g = the partial gradients summed in order of their chunks: 64 parameters per
// block, four thread groups taking a quarter of the chunks each, then their sums
// in order.
__global__ void __launch_bounds__(TH) k_mlp_grad_sum(const float* __restrict__ part, int nc, float* __restrict__ g) {
  __shared__ float red[4][64];
  const int q = blockIdx.x * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  const int lo = (int)((int64_t)nc * w / 4), hi = (int)((int64_t)nc * (w + 1) / 4);
  float s = 0.0f;
  if (q < NPAR) {
    int c = lo;
    for (; c + 8 <= hi; c += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(c + u) * NPAR + q];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; c < hi; ++c) s += part[(size_t)c * NPAR + q];
  }
  red[w][threadIdx.x & 63] = s;
  __syncthreads();
  if (w == 0 && q < NPAR) g[q] = ((red[0][q & 63] + red[1][q & 63]) + red[2][q & 63]) + red[3][q & 63];
}

__global__ void __launch_bounds__(256) k_mlp_adam(float* __restrict__ p, const float* __restrict__ g,
                                                  float* __restrict__ m, float* __restrict__ v, int n, float c1,
                                                  float c2, float lr, float b1, float b2, float eps) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const float gq = g[q];
  const float mq = b1 * m[q] + (1.0f - b1) * gq;
  const float vq = b2 * v[q] + (1.0f - b2) * gq * gq;
  m[q] = mq;
  v[q] = vq;
  p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

int launch_status() { return hipGetLastError() == hipSuccess ? DGMG_OK : DGMG_EHIP; }

// Work area of dgmg_mlp_forward_noalloc: the hidden activations h1, h2 of up to
// DGMG_MLP_NOALLOC_MAX_ROWS samples (4 MiB).  Every GPU the library runs on
// holds its own copy until the process ends.  In host code the array's name is
// only a stand-in: kernels receive the device address looked up once per device
// with hipGetSymbolAddress (mlp_fwd_scratch_ptr below).
constexpr int MAX_DEVICES = 64;
static __device__ __align__(256) float mlp_fwd_scratch[(size_t)DGMG_MLP_NOALLOC_MAX_ROWS * 2 * HID];

std::mutex g_scratch_mu;
float* g_scratch_dev[MAX_DEVICES] = {};

// Device address of this device's mlp_fwd_scratch, looked up with the device
// current on its first use and kept per device.
int mlp_fwd_scratch_ptr(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    dgmg_set_global_error(std::string("mlp_forward_noalloc: hipGetDevice: ") + hipGetErrorString(e));
    return DGMG_EHIP;
  }
  if (dev < 0 || dev >= MAX_DEVICES) {
    dgmg_set_global_error("mlp_forward_noalloc: device index beyond the supported 64");
    return DGMG_EUNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(mlp_fwd_scratch));
    if (e != hipSuccess || !p) {
      dgmg_set_global_error(std::string("mlp_forward_noalloc: hipGetSymbolAddress: ") +
                            (e != hipSuccess ? hipGetErrorString(e) : "null address"));
      return DGMG_EHIP;
    }
    g_scratch_dev[dev] = (float*)p;
  }
  *out = g_scratch_dev[dev];
  return DGMG_OK;
}

}  // namespace

extern "C" {

int dgmg_mlp_param_count(void) { return NPAR; }

int dgmg_mlp_forward(const float* params, const float* X, int B, float* Y, float* work, void* stream) {
  if (!params || !X || !Y || !work || B < 0) return DGMG_EINVAL;
  if (B == 0) return DGMG_OK;
  hipLaunchKernelGGL(k_mlp_forward, dim3((B + FS - 1) / FS), dim3(TH), 0, (hipStream_t)stream, params, X, B, Y, work);
  return launch_status();
}

int dgmg_mlp_forward_noalloc(const float* params, const float* X, int B, float* Y, void* stream) {
  if (!params || !X || !Y || B < 0) {
    dgmg_set_global_error("mlp_forward_noalloc: null pointer or negative row count");
    return DGMG_EINVAL;
  }
  if (B > DGMG_MLP_NOALLOC_MAX_ROWS) {
    dgmg_set_global_error("mlp_forward_noalloc: " + std::to_string(B) + " rows exceed the maximum of " +
                          std::to_string(DGMG_MLP_NOALLOC_MAX_ROWS) + " (use dgmg_mlp_forward with a work buffer)");
    return DGMG_EINVAL;
  }
  if (B == 0) return DGMG_OK;
  float* work = nullptr;
  int rc = mlp_fwd_scratch_ptr(&work);
  if (rc) return rc;
  hipLaunchKernelGGL(k_mlp_forward, dim3((B + FS - 1) / FS), dim3(TH), 0, (hipStream_t)stream, params, X, B, Y, work);
  return launch_status();
}

int dgmg_mlp_backward(const float* params, const float* X, const float* T, int B, const float* Y,
                      const float* work, float* grad, float* scratch, void* stream) {
  if (!params || !X || !T || !Y || !work || !grad || !scratch || B < 1) return DGMG_EINVAL;
  const int want = grad_chunks(B), per = (B + want - 1) / want, nc = (B + per - 1) / per;
  float* out = nc > 1 ? scratch : grad;
  hipLaunchKernelGGL(k_mlp_grad, dim3(nc), dim3(TH), 0, (hipStream_t)stream, params, X, T, B, per, Y, work, out);
  if (nc > 1)
    hipLaunchKernelGGL(k_mlp_grad_sum, dim3((NPAR + 63) / 64), dim3(TH), 0, (hipStream_t)stream, scratch, nc, grad);
  return launch_status();
}

int dgmg_mlp_adam(float* params, const float* grad, float* m, float* v, int n, int t, float lr, float b1,
                  float b2, float eps, void* stream) {
  if (!params || !grad || !m || !v || n < 0 || t < 1) return DGMG_EINVAL;
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_mlp_adam, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, params, grad, m, v, n,
                     c1, c2, lr, b1, b2, eps);
  return launch_status();
}

}  // extern "C"
