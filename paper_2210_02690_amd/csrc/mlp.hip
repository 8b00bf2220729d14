// Learned Newton initial guess: BF16 multilayer perceptron (forward, mean-squared-error
// gradient, Adam) on the matrix cores, and the patch gather / average kernels around it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <new>
#include <string>

#include "vk_mlp.h"

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float bf2f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }

__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return 0x7FC0;  // NaN stays NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

constexpr int MAX_LAYERS = 9;

// The network as its kernels see it.  Products run on v_mfma_f32_16x16x16_bf16: lane l supplies
// A(m, k) and B(k, n) for m, n = l % 16 and k = 4 (l / 16) .. + 3 of every 16-deep step and holds
// D(4 (l / 16) + i, l % 16), i < 4, in FP32.  Everything a lane reads for one step is one 8-byte word:
//   wf / wt  the BF16 weights in the order the forward (W^T) and the backward (W) products read them,
//            [column tile][16-deep step][lane][4], zero where a tile sticks out of the matrix;
//   ta / tz  per layer the inputs (features, then hidden activations) and the pre-activation gradients
//            of the batch, [16-sample tile][feature, padded to 16][16 samples]: the layout the
//            accumulators already have, and the one the weight gradients (sums over samples) read.
struct net_desc {
  int32_t L;                      // layers (n_hidden + 1)
  int32_t fi[MAX_LAYERS], fo[MAX_LAYERS];
  int64_t w[MAX_LAYERS], b[MAX_LAYERS];    // W_l and b_l in the packed parameters
  int64_t wf[MAX_LAYERS], wt[MAX_LAYERS];  // offsets in the two weight copies
  int64_t ta[MAX_LAYERS], tz[MAX_LAYERS];  // offsets of layer l's input and output gradient
};

__host__ __device__ inline int tiles16(int n) { return (n + 15) >> 4; }

// One workgroup takes 16 samples through the whole network, its activations in LDS: the layers need
// no other samples, so the forward pass, the loss, and (GRAD) the chain of pre-activation gradients are
// one launch (they were 4 + 3 products, the error kernel and a copy).  A wavefront owns every
// (wavefronts)-th 16-column tile of a layer; each product is one accumulator over k ascending, as
// before, so activations and gradients round as they did.  At these sizes the layers are a chain of
// L2 round trips, so a tile's weight words are all requested (8 steps at a time) before the first
// product.  One optimiser step of the 84-128-128-128-42 network on 512 samples (this kernel,
// grad_kernel, Adam, two parameter copies): 256 us in 21 launches -> 29 us in 4.
template <bool GRAD>
__global__ __launch_bounds__(512) void net_kernel(net_desc net, int32_t batch, int32_t ldk,
                                                  const uint16_t* __restrict__ x, const int32_t* __restrict__ rows,
                                                  const uint16_t* __restrict__ wf, const uint16_t* __restrict__ wt,
                                                  const float* __restrict__ theta, float* __restrict__ y,
                                                  const float* __restrict__ target, float scale, uint16_t* ta,
                                                  uint16_t* tz, float* __restrict__ part) {
  extern __shared__ __align__(16) uint16_t sm[];  // two buffers of 16 rows x ldk (ldk = 4 mod 16)
  __shared__ float red[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int l16 = lane & 15, q = lane >> 4;
  const int64_t mt = blockIdx.x;
  const int m0 = (int)mt * 16;
  uint16_t* buf[2] = {sm, sm + 16 * ldk};
  {
    const int n_in = net.fi[0], kp = 16 * tiles16(n_in);
    for (int m = wave; m < 16; m += nw) {
      const bool ok = m0 + m < batch;
      const int64_t r = ok ? (rows ? (int64_t)rows[m0 + m] : (int64_t)(m0 + m)) : 0;
      for (int k = lane; k < kp; k += 64) buf[0][m * ldk + k] = (ok && k < n_in) ? x[r * n_in + k] : (uint16_t)0;
    }
    __syncthreads();
    if (GRAD) {
      bf16x4* t = reinterpret_cast<bf16x4*>(ta + net.ta[0] + mt * kp * 16);
      for (int e = tid; e < kp * 4; e += blockDim.x) {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (short)buf[0][(4 * (e & 3) + i) * ldk + (e >> 2)];
        t[e] = v;
      }
    }
  }
  // one 16 x 16 tile: rows of `in` times column tile nt of the weight copy w, ks steps deep
  auto product = [&](const uint16_t* in, const uint16_t* w, int nt, int ks) {
    const bf16x4* wp = reinterpret_cast<const bf16x4*>(w) + (int64_t)nt * ks * 64 + lane;
    const uint16_t* ap = in + l16 * ldk + 4 * q;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    int s = 0;
    for (; s + 8 <= ks; s += 8) {
      bf16x4 bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) bv[u] = wp[(s + u) * 64];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4*>(ap + (s + u) * 16), bv[u], acc,
                                                        0, 0, 0);
    }
    for (; s < ks; ++s)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4*>(ap + s * 16), wp[s * 64], acc, 0,
                                                      0, 0);
    return acc;
  };
  int cur = 0;
  float loss = 0.0f;
  for (int l = 0; l < net.L; ++l) {
    const int N = net.fo[l], nts = tiles16(N), ks = tiles16(net.fi[l]);
    const bool last = l + 1 == net.L;
    uint16_t* dst = buf[cur ^ 1];
    for (int nt = wave; nt < nts; nt += nw) {
      const f32x4 acc = product(buf[cur], wf + net.wf[l], nt, ks);
      const int n = nt * 16 + l16;
      const float bias = n < N ? theta[net.b[l] + n] : 0.0f;
      bf16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + 4 * q + i;
        const bool ok = n < N && m < batch;
        uint16_t h = 0;
        if (!last) {
          if (ok) h = f2bf(tanhf(acc[i] + bias));
        } else if (ok) {
          const float v = acc[i] + bias;
          if (GRAD) {
            const int64_t tr = rows ? (int64_t)rows[m] : (int64_t)m;
            const float d = v - target[tr * N + n];
            loss += d * d;
            h = f2bf(scale * d);
          } else {
            y[(int64_t)m * N + n] = v;
          }
        }
        dst[(4 * q + i) * ldk + n] = h;
        o[i] = (short)h;
      }
      if (GRAD) {
        uint16_t* t = last ? tz + net.tz[l] : ta + net.ta[l + 1];
        *reinterpret_cast<bf16x4*>(t + (mt * nts * 16 + n) * 16 + 4 * q) = o;
      }
    }
    cur ^= 1;
    __syncthreads();
  }
  if (!GRAD) return;
  // dz_{l-1}(m, i) = (sum_j dz_l[m, j] W_l[j, i]) (1 - a(m, i)^2); the activation words were written by
  // this lane (same tile, same wavefront)
  for (int l = net.L - 1; l >= 1; --l) {
    const int N = net.fi[l], nts = tiles16(N), ks = tiles16(net.fo[l]);
    uint16_t* dst = buf[cur ^ 1];
    for (int nt = wave; nt < nts; nt += nw) {
      const int n = nt * 16 + l16;
      const int64_t at = (mt * nts * 16 + n) * 16 + 4 * q;
      const bf16x4 av = *reinterpret_cast<const bf16x4*>(ta + net.ta[l] + at);
      const f32x4 acc = product(buf[cur], wt + net.wt[l], nt, ks);
      bf16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = bf2f((uint16_t)av[i]);
        const uint16_t h = (n < N && m0 + 4 * q + i < batch) ? f2bf(acc[i] * (1.0f - a * a)) : (uint16_t)0;
        dst[(4 * q + i) * ldk + n] = h;
        o[i] = (short)h;
      }
      *reinterpret_cast<bf16x4*>(tz + net.tz[l - 1] + at) = o;
    }
    cur ^= 1;
    __syncthreads();
  }
  for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
  if (lane == 0) red[wave] = loss;
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    for (int w = 0; w < nw; ++w) t += red[w];
    part[blockIdx.x] = t;
  }
}

// All weight and bias gradients, and the loss, in one launch: blockIdx.y = layer (y = L: the loss),
// a wavefront per 16 x 16 tile of dW_l(j, i) = sum_m dz[m, j] a[m, i], one accumulator over the samples
// in order; the tiles of the first input columns also sum dz over the samples (db: four at a time, then in 64
// bits, since one wavefront adds up a batch of up to 2^20).  Both operands of 16 samples are one 8-byte word per lane, 8 steps in flight (per layer and 512 samples, a product with
// scalar 2-byte loads, one round trip per step, took 44 us and the bias sums 4.7 us).
__global__ __launch_bounds__(64) void grad_kernel(net_desc net, int32_t batch, const uint16_t* __restrict__ ta,
                                                  const uint16_t* __restrict__ tz, const float* __restrict__ part,
                                                  float inv_count, float* __restrict__ grad, float* __restrict__ grad_out,
                                                  float* __restrict__ loss_out) {
  const int l = blockIdx.y, lane = threadIdx.x;
  const int mts = (batch + 15) >> 4;
  if (l == net.L) {
    if (blockIdx.x != 0 || !loss_out) return;
    float s = 0.0f;
    for (int i = lane; i < mts; i += 64) s += part[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) loss_out[0] = s * inv_count;
    return;
  }
  const int l16 = lane & 15, q = lane >> 4;
  const int fi = net.fi[l], fo = net.fo[l], it_n = tiles16(fi), jt_n = tiles16(fo);
  const int jt = (int)blockIdx.x / it_n, it = (int)blockIdx.x - jt * it_n;
  if (jt >= jt_n) return;
  const int sa = jt_n * 64, sb = it_n * 64;  // words per 16-sample tile
  const bf16x4* ap = reinterpret_cast<const bf16x4*>(tz + net.tz[l]) + (jt * 16 + l16) * 4 + q;
  const bf16x4* bp = reinterpret_cast<const bf16x4*>(ta + net.ta[l]) + (it * 16 + l16) * 4 + q;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  double db = 0.0;
  auto step = [&](bf16x4 a, bf16x4 b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
    if (it == 0)
      db += (double)((bf2f((uint16_t)a[0]) + bf2f((uint16_t)a[1])) + (bf2f((uint16_t)a[2]) + bf2f((uint16_t)a[3])));
  };
  int s = 0;
  for (; s + 8 <= mts; s += 8) {
    bf16x4 a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a[u] = ap[(int64_t)(s + u) * sa];
      b[u] = bp[(int64_t)(s + u) * sb];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) step(a[u], b[u]);
  }
  for (; s < mts; ++s) step(ap[(int64_t)s * sa], bp[(int64_t)s * sb]);
  const int i = it * 16 + l16;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int j = jt * 16 + 4 * q + v;
    if (j >= fo || i >= fi) continue;
    const int64_t at = net.w[l] + (int64_t)j * fi + i;
    grad[at] = acc[v];
    if (grad_out) grad_out[at] = acc[v];
  }
  if (it == 0) {
    db += __shfl_xor(db, 16, 64);
    db += __shfl_xor(db, 32, 64);
    const int j = jt * 16 + l16;
    if (q == 0 && j < fo) {
      grad[net.b[l] + j] = (float)db;
      if (grad_out) grad_out[net.b[l] + j] = (float)db;
    }
  }
}

// parameter p rounded to BF16 goes to its place in both weight copies (biases have none)
__device__ inline void store_weight(const net_desc& net, int64_t p, float v, uint16_t* __restrict__ wf,
                                    uint16_t* __restrict__ wt) {
  int l = 0;
  while (l + 1 < net.L && p >= net.w[l + 1]) ++l;
  if (p >= net.b[l]) return;
  const int fi = net.fi[l], fo = net.fo[l], e = (int)(p - net.w[l]);
  const int j = e / fi, i = e - j * fi;
  const uint16_t h = f2bf(v);
  // forward: k = i, n = j; backward: k = j, n = i
  wf[net.wf[l] + (((int64_t)(j >> 4) * tiles16(fi) + (i >> 4)) * 64 + (j & 15) + 16 * ((i & 15) >> 2)) * 4 + (i & 3)] = h;
  wt[net.wt[l] + (((int64_t)(i >> 4) * tiles16(fo) + (j >> 4)) * 64 + (i & 15) + 16 * ((j & 15) >> 2)) * 4 + (j & 3)] = h;
}

__global__ void adam_kernel(net_desc net, int64_t P, float* __restrict__ theta, float* __restrict__ m1,
                            float* __restrict__ m2, const float* __restrict__ g, uint16_t* __restrict__ wf,
                            uint16_t* __restrict__ wt, float lr, float b1, float b2, float eps, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float m = b1 * m1[i] + (1.0f - b1) * gi;
    const float v = b2 * m2[i] + (1.0f - b2) * gi * gi;
    m1[i] = m;
    m2[i] = v;
    const float th = theta[i] - lr * (m * c1) / (sqrtf(v * c2) + eps);
    theta[i] = th;
    store_weight(net, i, th, wf, wt);
  }
}

// both weight copies zero (their padding stays so)
__global__ void clear_weights_kernel(int64_t n, uint64_t* __restrict__ w) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) w[i] = 0;
}

__global__ void set_params_kernel(net_desc net, int64_t P, const float* __restrict__ src, float* __restrict__ theta,
                                  float* __restrict__ m1, float* __restrict__ m2, uint16_t* __restrict__ wf,
                                  uint16_t* __restrict__ wt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
    const float v = src[i];
    theta[i] = v;
    m1[i] = 0.0f;
    m2[i] = 0.0f;
    store_weight(net, i, v, wf, wt);
  }
}

__global__ void copy_f32_kernel(int64_t n, const float* __restrict__ src, float* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void features_kernel(int32_t n_cells, int32_t n_K, const int32_t* __restrict__ dofs,
                                const double* __restrict__ X1, const double* __restrict__ X2,
                                const double* __restrict__ B, const float* __restrict__ mean,
                                const float* __restrict__ inv_std, uint16_t* __restrict__ out) {
  const int64_t w = 2 * (int64_t)n_K;
  const int64_t total = (int64_t)n_cells * w;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = i / w;
    const int j = (int)(i - c * w);
    const int jl = j < n_K ? j : j - n_K;
    const int32_t d = dofs[c * n_K + jl];
    const double x = X2[d] - (j < n_K ? X1 : B)[d];
    out[i] = f2bf((float)(x - (double)mean[j]) * inv_std[j]);
  }
}

__global__ void targets_kernel(int32_t n_cells, int32_t n_K, const int32_t* __restrict__ dofs,
                               const double* __restrict__ X, const double* __restrict__ base,
                               const float* __restrict__ mean, const float* __restrict__ inv_std,
                               float* __restrict__ out) {
  const int64_t total = (int64_t)n_cells * n_K;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(i % n_K);
    const int32_t d = dofs[i];
    out[i] = (float)((X[d] - base[d] - (double)mean[j]) * (double)inv_std[j]);
  }
}

__global__ void average_kernel(int64_t n, const int64_t* __restrict__ ptr, const int64_t* __restrict__ list,
                               int32_t n_K, const float* __restrict__ pred, const float* __restrict__ mean,
                               const float* __restrict__ sd, const double* __restrict__ base,
                               double* __restrict__ out) {
  for (int64_t mu = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; mu < n; mu += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e0 = ptr[mu], e1 = ptr[mu + 1];
    double s = 0.0;
    for (int64_t e = e0; e < e1; ++e) {
      const int64_t idx = list[e];
      const int j = (int)(idx % n_K);
      s += (double)pred[idx] * (double)sd[j] + (double)mean[j];
    }
    out[mu] = base[mu] + (e1 > e0 ? s / (double)(e1 - e0) : 0.0);
  }
}

struct ext_coef {
  double e[64];
};

__global__ void extrapolate_kernel(int64_t ns, int32_t nt, ext_coef E, const double* __restrict__ X,
                                   double* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
    double x[8];
    for (int b = 0; b < nt; ++b) x[b] = X[b * ns + i];
    for (int a = 0; a < nt; ++a) {
      double s = 0.0;
      for (int b = 0; b < nt; ++b) s += E.e[a * 8 + b] * x[b];
      out[a * ns + i] = s;
    }
  }
}

inline unsigned grid_for(int64_t work, int per, unsigned cap = 4096) {
  int64_t g = (work + per - 1) / per;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

char g_mlp_create_err[256] = "";

}  // namespace

struct vk_mlp {
  hipStream_t stream = nullptr;
  std::string err;
  int32_t n_in = 0, width = 0, n_hidden = 0, n_out = 0, max_batch = 0;
  net_desc net{};
  int64_t P = 0;
  int64_t n_wf = 0, n_wt = 0, n_ta = 0, n_tz = 0;  // elements of the weight copies and batch arrays
  int32_t wide = 0;                                // widest layer, padded to 16
  // workspace
  bool ready = false;
  float* theta = nullptr;
  float* m1 = nullptr;
  float* m2 = nullptr;
  float* grad = nullptr;
  uint16_t* wf = nullptr;  // weights in the forward products' order; wt follows it
  uint16_t* wt = nullptr;
  uint16_t* ta = nullptr;  // the batch's layer inputs and pre-activation gradients (gradient calls)
  uint16_t* tz = nullptr;
  float* part = nullptr;   // squared error per 16 samples
  int64_t step = 0;
  bool have_grad = false;
};

namespace {

vk_status mfail(vk_mlp* c, vk_status st, const std::string& msg) {
  c->err = msg;
  return st;
}

vk_status mfail_hip(vk_mlp* c, hipError_t e, const char* what) {
  (void)hipGetLastError();
  c->err = std::string(what) + ": " + hipGetErrorString(e);
  return VK_ERR_HIP;
}

#define MLP_TRY(expr)                                     \
  do {                                                    \
    hipError_t _e = (expr);                               \
    if (_e != hipSuccess) return mfail_hip(c, _e, #expr); \
  } while (0)

#define MLP_LAUNCHED(what)                               \
  do {                                                   \
    hipError_t _e = hipGetLastError();                   \
    if (_e != hipSuccess) return mfail_hip(c, _e, what); \
  } while (0)

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

size_t plan(vk_mlp* c, char* base) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    char* p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  const size_t P = (size_t)c->P;
  c->theta = reinterpret_cast<float*>(take(P * 4));
  c->m1 = reinterpret_cast<float*>(take(P * 4));
  c->m2 = reinterpret_cast<float*>(take(P * 4));
  c->grad = reinterpret_cast<float*>(take(P * 4));
  c->wf = reinterpret_cast<uint16_t*>(take((size_t)(c->n_wf + c->n_wt) * 2));
  c->wt = c->wf ? c->wf + c->n_wf : nullptr;
  c->ta = reinterpret_cast<uint16_t*>(take((size_t)c->n_ta * 2));
  c->tz = reinterpret_cast<uint16_t*>(take((size_t)c->n_tz * 2));
  c->part = reinterpret_cast<float*>(take((size_t)((c->max_batch + 15) / 16) * 4));
  return off;
}

vk_status check_ready(vk_mlp* c) {
  if (!c) return VK_ERR_ARG;
  if (!c->ready) return mfail(c, VK_ERR_WORKSPACE, "workspace not set");
  return VK_OK;
}

// The network over `batch` samples: y (forward), or with a target the loss parts, the layer inputs and
// the pre-activation gradients the weight gradients are formed from.  Eight wavefronts per 16 samples
// where a layer has that many column tiles (one tile each), else four.
hipError_t run_net(vk_mlp* c, int32_t batch, const uint16_t* x, const int32_t* rows, float* y, const float* target,
                   float scale) {
  const unsigned grid = (unsigned)((batch + 15) / 16);
  const unsigned nt = c->wide > 64 ? 512 : 256;
  const int32_t ldk = c->wide + 4;  // rows 8 bytes apart modulo 32: the lanes' 8-byte reads spread over the banks
  const size_t lds = (size_t)2 * 16 * ldk * sizeof(uint16_t);
  if (lds > 65000) {  // layers about 1 000 wide: beyond what a launch may take unasked (the same limit from every thread)
    constexpr int limit = 2 * 16 * (1024 + 4) * (int)sizeof(uint16_t);
    const void* f = target ? reinterpret_cast<const void*>(net_kernel<true>) : reinterpret_cast<const void*>(net_kernel<false>);
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, limit);
    if (e != hipSuccess) return e;
  }
  if (target)
    net_kernel<true><<<grid, nt, lds, c->stream>>>(c->net, batch, ldk, x, rows, c->wf, c->wt, c->theta, nullptr, target,
                                                   scale, c->ta, c->tz, c->part);
  else
    net_kernel<false><<<grid, nt, lds, c->stream>>>(c->net, batch, ldk, x, rows, c->wf, c->wt, c->theta, y, nullptr,
                                                    0.0f, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

}  // namespace

extern "C" {

vk_status vk_mlp_create(vk_mlp** out, int32_t n_in, int32_t width, int32_t n_hidden, int32_t n_out,
                        int32_t max_batch, void* hip_stream) {
  if (!out) {
    snprintf(g_mlp_create_err, sizeof(g_mlp_create_err), "null output pointer");
    return VK_ERR_ARG;
  }
  *out = nullptr;
  if (n_hidden < 1 || n_hidden > 8 || n_in < 1 || n_in > 1024 || width < 1 || width > 1024 || n_out < 1 ||
      n_out > 1024 || max_batch < 1 || max_batch > (1 << 20)) {
    snprintf(g_mlp_create_err, sizeof(g_mlp_create_err), "layer sizes or max_batch out of range");
    return VK_ERR_ARG;
  }
  vk_mlp* c = new (std::nothrow) vk_mlp;
  if (!c) {
    snprintf(g_mlp_create_err, sizeof(g_mlp_create_err), "host allocation failed");
    return VK_ERR_ARG;
  }
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  c->n_in = n_in;
  c->width = width;
  c->n_hidden = n_hidden;
  c->n_out = n_out;
  c->max_batch = max_batch;
  int64_t off = 0;
  const int64_t mts = (max_batch + 15) / 16;
  net_desc& d = c->net;
  d.L = n_hidden + 1;
  for (int l = 0; l < d.L; ++l) {
    const int32_t fi = l == 0 ? n_in : width, fo = l == n_hidden ? n_out : width;
    const int64_t ti = tiles16(fi), to = tiles16(fo);
    d.fi[l] = fi;
    d.fo[l] = fo;
    d.w[l] = off;
    d.b[l] = off + (int64_t)fi * fo;
    off = d.b[l] + fo;
    d.wf[l] = c->n_wf;
    c->n_wf += ti * to * 256;
    d.wt[l] = c->n_wt;
    c->n_wt += ti * to * 256;
    d.ta[l] = c->n_ta;
    c->n_ta += mts * ti * 256;
    d.tz[l] = c->n_tz;
    c->n_tz += mts * to * 256;
    const int32_t wide = 16 * (int32_t)(ti > to ? ti : to);
    if (wide > c->wide) c->wide = wide;
  }
  // (together the two also hold a batch of outputs, see vk_mlp_forward)
  c->n_tz = std::max(c->n_tz, mts * 16 * 2 * (int64_t)n_out - c->n_ta);
  c->P = off;
  *out = c;
  return VK_OK;
}

void vk_mlp_destroy(vk_mlp* mlp) {
  if (!mlp) return;
  if (mlp->stream) (void)hipStreamSynchronize(mlp->stream);
  else (void)hipDeviceSynchronize();
  delete mlp;
}

const char* vk_mlp_last_error(const vk_mlp* mlp) { return mlp ? mlp->err.c_str() : g_mlp_create_err; }

int64_t vk_mlp_param_count(const vk_mlp* mlp) { return mlp ? mlp->P : 0; }

size_t vk_mlp_workspace_bytes(const vk_mlp* mlp) {
  if (!mlp) return 0;
  vk_mlp tmp = *mlp;
  return plan(&tmp, nullptr);
}

vk_status vk_mlp_set_workspace(vk_mlp* c, void* dev, size_t bytes) {
  if (!c) return VK_ERR_ARG;
  c->ready = false;
  if (!dev) return mfail(c, VK_ERR_ARG, "null workspace");
  if (reinterpret_cast<uintptr_t>(dev) % 256 != 0) return mfail(c, VK_ERR_ARG, "workspace must be 256-byte aligned");
  if (bytes < vk_mlp_workspace_bytes(c)) return mfail(c, VK_ERR_WORKSPACE, "workspace smaller than required");
  plan(c, static_cast<char*>(dev));
  c->ready = true;
  c->step = 0;
  c->have_grad = false;
  return VK_OK;
}

vk_status vk_mlp_set_params(vk_mlp* c, const float* params) {
  vk_status st = check_ready(c);
  if (st != VK_OK) return st;
  if (!params) return mfail(c, VK_ERR_ARG, "null parameter vector");
  const int64_t words = (c->n_wf + c->n_wt) / 4;
  clear_weights_kernel<<<grid_for(words, 256), 256, 0, c->stream>>>(words, reinterpret_cast<uint64_t*>(c->wf));
  MLP_LAUNCHED("clear_weights_kernel");
  set_params_kernel<<<grid_for(c->P, 256), 256, 0, c->stream>>>(c->net, c->P, params, c->theta, c->m1, c->m2, c->wf,
                                                                c->wt);
  MLP_LAUNCHED("set_params_kernel");
  c->step = 0;
  c->have_grad = false;
  return VK_OK;
}

vk_status vk_mlp_get_params(vk_mlp* c, float* params) {
  vk_status st = check_ready(c);
  if (st != VK_OK) return st;
  if (!params) return mfail(c, VK_ERR_ARG, "null output");
  copy_f32_kernel<<<grid_for(c->P, 256), 256, 0, c->stream>>>(c->P, c->theta, params);
  MLP_LAUNCHED("copy_f32_kernel");
  return VK_OK;
}

vk_status vk_mlp_forward(vk_mlp* c, int32_t batch, const uint16_t* x, const int32_t* rows, float* y) {
  vk_status st = check_ready(c);
  if (st != VK_OK) return st;
  if (batch < 0 || batch > c->max_batch) return mfail(c, VK_ERR_ARG, "batch exceeds max_batch");
  if (batch == 0) return VK_OK;
  if (!x || !y) return mfail(c, VK_ERR_ARG, "null input or output");
  // Workgroups write their samples' y while others still read x and rows: an output that may share memory
  // with them (with rows, x reaches to no known end) goes through the batch arrays.
  const char *yb = reinterpret_cast<const char*>(y), *ye = reinterpret_cast<const char*>(y + (int64_t)batch * c->n_out);
  auto apart = [&](const void* first, const void* last) {
    return ye <= static_cast<const char*>(first) || (last && yb >= static_cast<const char*>(last));
  };
  if (apart(x, rows ? nullptr : x + (int64_t)batch * c->n_in) && (!rows || apart(rows, rows + batch))) {
    MLP_TRY(run_net(c, batch, x, rows, y, nullptr, 0.0f));
    return VK_OK;
  }
  float* staged = reinterpret_cast<float*>(c->ta);
  MLP_TRY(run_net(c, batch, x, rows, staged, nullptr, 0.0f));
  const int64_t n = (int64_t)batch * c->n_out;
  copy_f32_kernel<<<grid_for(n, 256), 256, 0, c->stream>>>(n, staged, y);
  MLP_LAUNCHED("copy_f32_kernel");
  return VK_OK;
}

vk_status vk_mlp_gradient(vk_mlp* c, int32_t batch, const uint16_t* x, const int32_t* rows, const float* target,
                          float* loss, float* grad) {
  vk_status st = check_ready(c);
  if (st != VK_OK) return st;
  if (batch < 1 || batch > c->max_batch) return mfail(c, VK_ERR_ARG, "batch must be in [1, max_batch]");
  if (!x || !target) return mfail(c, VK_ERR_ARG, "null input or target");
  const float count = (float)batch * (float)c->n_out;
  MLP_TRY(run_net(c, batch, x, rows, nullptr, target, 2.0f / count));
  unsigned tiles = 1;
  for (int l = 0; l < c->net.L; ++l)
    tiles = std::max(tiles, (unsigned)(tiles16(c->net.fi[l]) * tiles16(c->net.fo[l])));
  grad_kernel<<<dim3(tiles, (unsigned)c->net.L + 1), 64, 0, c->stream>>>(c->net, batch, c->ta, c->tz, c->part,
                                                                         1.0f / count, c->grad, grad, loss);
  MLP_LAUNCHED("grad_kernel");
  c->have_grad = true;
  return VK_OK;
}

vk_status vk_mlp_adam(vk_mlp* c, float lr, float beta1, float beta2, float eps) {
  vk_status st = check_ready(c);
  if (st != VK_OK) return st;
  if (!c->have_grad) return mfail(c, VK_ERR_STATE, "no gradient since the parameters were set");
  if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
    return mfail(c, VK_ERR_ARG, "Adam hyper-parameters out of range");
  ++c->step;
  const double c1 = 1.0 / (1.0 - std::pow((double)beta1, (double)c->step));
  const double c2 = 1.0 / (1.0 - std::pow((double)beta2, (double)c->step));
  adam_kernel<<<grid_for(c->P, 256), 256, 0, c->stream>>>(c->net, c->P, c->theta, c->m1, c->m2, c->grad, c->wf, c->wt,
                                                           lr, beta1, beta2, eps, (float)c1, (float)c2);
  MLP_LAUNCHED("adam_kernel");
  return VK_OK;
}

vk_status vk_mlp_patch_features(vk_mlp* c, int32_t n_cells, int32_t n_K, const int32_t* cell_dofs, const double* X1,
                                const double* X2, const double* B, const float* mean, const float* inv_std,
                                uint16_t* out) {
  if (!c) return VK_ERR_ARG;
  if (n_cells < 0 || n_K < 1) return mfail(c, VK_ERR_ARG, "bad patch sizes");
  if (n_cells == 0) return VK_OK;
  if (!cell_dofs || !X1 || !X2 || !B || !mean || !inv_std || !out) return mfail(c, VK_ERR_ARG, "null array");
  const int64_t total = (int64_t)n_cells * 2 * n_K;
  features_kernel<<<grid_for(total, 256), 256, 0, c->stream>>>(n_cells, n_K, cell_dofs, X1, X2, B, mean, inv_std,
                                                               out);
  MLP_LAUNCHED("features_kernel");
  return VK_OK;
}

vk_status vk_mlp_patch_targets(vk_mlp* c, int32_t n_cells, int32_t n_K, const int32_t* cell_dofs, const double* X,
                               const double* base, const float* mean, const float* inv_std, float* out) {
  if (!c) return VK_ERR_ARG;
  if (n_cells < 0 || n_K < 1) return mfail(c, VK_ERR_ARG, "bad patch sizes");
  if (n_cells == 0) return VK_OK;
  if (!cell_dofs || !X || !base || !mean || !inv_std || !out) return mfail(c, VK_ERR_ARG, "null array");
  const int64_t total = (int64_t)n_cells * n_K;
  targets_kernel<<<grid_for(total, 256), 256, 0, c->stream>>>(n_cells, n_K, cell_dofs, X, base, mean, inv_std, out);
  MLP_LAUNCHED("targets_kernel");
  return VK_OK;
}

vk_status vk_mlp_patch_average(vk_mlp* c, int64_t n, const int64_t* dof_ptr, const int64_t* dof_list, int32_t n_K,
                               const float* pred, const float* mean, const float* std, const double* base,
                               double* out) {
  if (!c) return VK_ERR_ARG;
  if (n < 0 || n_K < 1) return mfail(c, VK_ERR_ARG, "bad sizes");
  if (n == 0) return VK_OK;
  if (!dof_ptr || !dof_list || !pred || !mean || !std || !base || !out) return mfail(c, VK_ERR_ARG, "null array");
  average_kernel<<<grid_for(n, 256), 256, 0, c->stream>>>(n, dof_ptr, dof_list, n_K, pred, mean, std, base, out);
  MLP_LAUNCHED("average_kernel");
  return VK_OK;
}

vk_status vk_mlp_slab_extrapolate(vk_mlp* c, int64_t n_space, int32_t n_time, const double* E, const double* X,
                                  double* out) {
  if (!c) return VK_ERR_ARG;
  if (n_space < 0 || n_time < 1 || n_time > 8) return mfail(c, VK_ERR_ARG, "n_time must be in [1, 8]");
  if (!E || !X || !out) return mfail(c, VK_ERR_ARG, "null array");
  if (X == out) return mfail(c, VK_ERR_ARG, "out must not alias X");
  if (n_space == 0) return VK_OK;
  ext_coef co{};
  for (int a = 0; a < n_time; ++a)
    for (int b = 0; b < n_time; ++b) co.e[a * 8 + b] = E[a * n_time + b];
  extrapolate_kernel<<<grid_for(n_space, 256), 256, 0, c->stream>>>(n_space, n_time, co, X, out);
  MLP_LAUNCHED("extrapolate_kernel");
  return VK_OK;
}

}  // extern "C"
