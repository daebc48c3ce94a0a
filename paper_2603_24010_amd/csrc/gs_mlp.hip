// Training and batch evaluation of the Newton guess network on the GPU.
//
// Training is plain mini-batch gradient descent with Adam (Kingma and Ba,
// 2015) on the mean squared error, in binary32 on the matrix cores; every
// reduction has a fixed order, so a run is bitwise repeatable.  Batch evaluation uses the same device routine as the
// strict step (bfloat16 weights, binary32 sums).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "gapsim.h"
#include "gs_internal.h"
#include "gs_mlp_dev.h"

namespace gs {

// ---------------------------------------------------------------------------
// One optimiser step is two kernels.  k_train_rows takes a tile of batch rows
// through the whole network and back, the tile's activations in LDS from the
// gather to the last layer's derivative, and leaves what the weight gradients
// contract over (inputs, activations, derivatives) in the workspace.
// k_train_update sums one 16 x 16 block of a weight gradient over the batch per
// workgroup and applies Adam to it.  What bounds a step at the usual batches is
// latency: 14.6 GFLOP in 64 steps of batch 1024 is 1.5 us of matrix work a step.
// At batch 1024 (64 row tiles, 160 blocks) the two kernels take 19.7 and 8.3 us
// and a step 30.4 us, launches included; one kernel per GEMM, column sum and
// reduction (22 launches) took 157 us.
//
// All products run on the matrix cores in binary32 (v_mfma_f32_16x16x4_f32:
// binary32 products and sums).  Lane l gives A(l % 16, l / 16) and B(l / 16, l
// % 16); its accumulator r holds D(4 (l / 16) + r, l % 16).  The order of a
// sum over k is free but fixed: where k runs along memory, the four MFMAs of a
// 16-wide step take k = 4 (l / 16) + j, j = 0..3, so that a lane reads four
// consecutive values.
// ---------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ inline float gelu_both(float z, float *grad) {
  const float Phi = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
  *grad = Phi + z * (0.39894228040143268f * expf(-0.5f * z * z));
  return gelu_f32(z);
}

// four consecutive floats from 4-byte aligned memory (the caller's arrays)
__device__ inline v4f ld4(const float *a) {
  v4f v;
  __builtin_memcpy(&v, a, 16);
  return v;
}

constexpr int TRW = 8;              // waves of k_train_rows: one 16-wide column block each
constexpr int TRT = TRW * 64;       // its threads
constexpr int TLD = MLP_H + 4;      // row stride of the LDS tiles (spreads rows over the banks)
constexpr int TRM = 16;             // batch rows per row block
constexpr int TRAIN_MB1_MAX = 4096; // largest batch with one row block per workgroup
static_assert(TRW * 16 == MLP_H, "a wave per column block");

// what k_train_rows leaves for the weight gradients (rows of the batch)
struct TrainRows {
  float *x, *a1, *a2, *a3;   // inputs and activations: [B][48], [B][128] x 3
  float *d1, *d2, *d3, *dy;  // derivatives by the pre-activations: [B][128] x 3, [B][3]
  float *loss;               // sum of squared errors per workgroup
  unsigned int *bad;
};

template <int MB>
constexpr size_t train_rows_lds() {
  return ((size_t)MB * TRM * (5 * TLD + 3 * MLP_OUT)) * 4;
}

// W (row-major [128][K], K a multiple of 16) for one column block of the
// forward product: lane l's values of row n0 + l % 16
template <int K>
__device__ inline void load_fwd(const float *W, int n0, v4f *w) {
  const int c = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int k = 0; k < K / 16; ++k) w[k] = ld4(W + (size_t)(n0 + c) * K + 16 * k + 4 * q);
}

// the same for the backward product: lane l's values of column k0 + l % 16
__device__ inline void load_bwd(const float *W, int k0, v4f *w) {
  const int c = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int n = 0; n < MLP_H / 16; ++n)
#pragma unroll
    for (int j = 0; j < 4; ++j) w[n][j] = W[(size_t)(16 * n + 4 * q + j) * MLP_H + k0 + c];
}

// acc[m] = rows of block m of the LDS tile A times the loaded block
template <int MB, int K>
__device__ inline void mul_block(const float *A, const v4f *w, v4f *acc) {
  const int c = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int m = 0; m < MB; ++m) acc[m] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < K / 16; ++k) {
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const v4f a = *(const v4f *)(A + (m * TRM + c) * TLD + 16 * k + 4 * q);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], w[k][j], acc[m], 0, 0, 0);
    }
  }
}

// MB row blocks of 16 per workgroup
template <int MB>
__global__ __launch_bounds__(TRT, 2) void k_train_rows(const float *x, const float *t, long long n,
                                                       const int32_t *order, long long off, int B, const float *th,
                                                       TrainRows o) {
  constexpr int R = MB * TRM;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  float *A0 = (float *)lds_raw;        // [R][TLD] x 2: a layer's input, its output
  float *A1 = A0 + R * TLD;
  float *G1 = A1 + R * TLD;            // [R][TLD] x 3: GELU' of the pre-activations
  float *G2 = G1 + R * TLD, *G3 = G2 + R * TLD;
  float *sdy = G3 + R * TLD;           // [R][3]
  float *st = sdy + R * MLP_OUT;       // [R][3] targets
  float *se = st + R * MLP_OUT;        // [R][3] squared errors
  const int tid = threadIdx.x, wv = tid >> 6, c = tid & 15, q = (tid >> 4) & 3;
  const int n0 = wv * 16;
  const int r0 = blockIdx.x * R;
  const float *W1 = th + MLP_OFF_W1, *W2 = th + MLP_OFF_W2, *W3 = th + MLP_OFF_W3, *W4 = th + MLP_OFF_W4;
  v4f w1[MLP_IN / 16], wa[MLP_H / 16], wb[MLP_H / 16];
  load_fwd<MLP_IN>(W1, n0, w1);
  load_fwd<MLP_H>(W2, n0, wa);
  // the batch's rows (past its end the last one, whose derivative is zeroed);
  // an index outside [0, n) is replaced by 0 and counted
  for (int e = tid; e < R * (MLP_IN + MLP_OUT); e += TRT) {
    const int r = e / (MLP_IN + MLP_OUT), f = e % (MLP_IN + MLP_OUT);
    const int b = min(r0 + r, B - 1);
    long long i = order[off + b];
    if (i < 0 || i >= n) {
      if (f == 0 && r0 + r < B) atomicAdd(o.bad, 1u);
      i = 0;
    }
    if (f < MLP_IN) {
      const float v = x[i * MLP_IN + f];
      A0[r * TLD + f] = v;
      if (r0 + r < B) o.x[(size_t)b * MLP_IN + f] = v;
    } else {
      st[r * MLP_OUT + f - MLP_IN] = t[i * MLP_OUT + f - MLP_IN];
    }
  }
  __syncthreads();
  // a hidden layer's epilogue: bias, GELU to LDS and the workspace, GELU' to LDS
  v4f acc[MB];
  auto hidden = [&](const float *bias, float *out, float *g, float *global) {
    const float bj = bias[n0 + c];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = m * TRM + 4 * q + i;
        float gr;
        const float v = gelu_both(acc[m][i] + bj, &gr);
        out[r * TLD + n0 + c] = v;
        g[r * TLD + n0 + c] = gr;
        if (r0 + r < B) global[(size_t)(r0 + r) * MLP_H + n0 + c] = v;
      }
  };
  mul_block<MB, MLP_IN>(A0, w1, acc);
  load_fwd<MLP_H>(W3, n0, wb);
  hidden(th + MLP_OFF_B1, A1, G1, o.a1);
  __syncthreads();
  mul_block<MB, MLP_H>(A1, wa, acc);
  load_bwd(W3, n0, wa);
  hidden(th + MLP_OFF_B2, A0, G2, o.a2);
  __syncthreads();
  mul_block<MB, MLP_H>(A0, wb, acc);
  load_bwd(W2, n0, wb);
  hidden(th + MLP_OFF_B3, A1, G3, o.a3);
  __syncthreads();
  // the output layer: eight lanes per output, sixteen inputs each
  const float inv = 1.0f / (float)(B * MLP_OUT);
  for (int e = tid; e < R * MLP_OUT * 8; e += TRT) {
    const int p = e & 7, r = (e >> 3) / MLP_OUT, u = (e >> 3) % MLP_OUT;
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += A1[r * TLD + 16 * p + k] * W4[u * MLP_H + 16 * p + k];
    s += __shfl_xor(s, 4, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 1, 64);
    if (p == 0) {
      const bool in = r0 + r < B;
      const float d = in ? s + th[MLP_OFF_B4 + u] - st[r * MLP_OUT + u] : 0.0f;
      se[r * MLP_OUT + u] = d * d;
      sdy[r * MLP_OUT + u] = 2.0f * d * inv;
      if (in) o.dy[(size_t)(r0 + r) * MLP_OUT + u] = 2.0f * d * inv;
    }
  }
  __syncthreads();
  if (wv == 0) {
    float s = 0.0f;
    for (int e = tid; e < R * MLP_OUT; e += 64) s += se[e];
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) s += __shfl_xor(s, k, 64);
    if (tid == 0) o.loss[blockIdx.x] = s;
  }
  // back: d3 = (dy W4) GELU'(z3), then d2 and d1 through W3 and W2
  for (int e = tid; e < R * MLP_H; e += TRT) {
    const int r = e / MLP_H, k = e % MLP_H;
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < MLP_OUT; ++u) s += sdy[r * MLP_OUT + u] * W4[u * MLP_H + k];
    s *= G3[r * TLD + k];
    A0[r * TLD + k] = s;
    if (r0 + r < B) o.d3[(size_t)(r0 + r) * MLP_H + k] = s;
  }
  __syncthreads();
  auto back = [&](float *out, const float *g, float *global) {
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = m * TRM + 4 * q + i;
        const float v = acc[m][i] * g[r * TLD + n0 + c];
        if (out) out[r * TLD + n0 + c] = v;
        if (r0 + r < B) global[(size_t)(r0 + r) * MLP_H + n0 + c] = v;
      }
  };
  mul_block<MB, MLP_H>(A0, wa, acc);
  back(A1, G2, o.d2);
  __syncthreads();
  mul_block<MB, MLP_H>(A1, wb, acc);
  back(nullptr, G1, o.d1);
}

// Adam on one parameter (Kingma and Ba, bias-corrected moments)
struct AdamK {
  float lr, b1, b2, eps, c1, c2;
};
__device__ inline void adam_one(float *th, float *m, float *v, int i, float g, const AdamK &k) {
  const float mi = k.b1 * m[i] + (1.0f - k.b1) * g;
  const float vi = k.b2 * v[i] + (1.0f - k.b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  th[i] -= k.lr * (mi / k.c1) / (sqrtf(vi / k.c2) + k.eps);
}

// The weight-gradient blocks: 8 x 8 for W2 and W3, 8 x 3 for W1, 1 x 8 for W4.
// A small block spreads the parameters over the most workgroups: at the usual
// batches each has little to contract.
constexpr int UB2 = 64, UB1 = 24, UB4 = 8, UBLOCKS = 2 * UB2 + UB1 + UB4;
constexpr int UPW = 16;  // waves of k_train_update, each with a slice of the batch
constexpr int UPT = UPW * 64;
constexpr int UPU = 8;   // MFMAs of 4 batch rows whose loads are in flight together

// dW[j][k] = sum_b d[b][j] a[b][k] for one block, summed over the waves' slices
// in slice order, then Adam; the blocks of the first column also do the bias
// (the same sum with a = 1).  The last step's gradient goes to grad when set.
// Workgroup 0 adds up the batch loss.
__global__ __launch_bounds__(UPT) void k_train_update(TrainRows o, int B, int ntiles, float *th, float *m, float *v,
                                                      AdamK ak, float *grad, float *loss) {
  __shared__ float part[UPW][16 * 16];
  __shared__ float partb[UPW][16];
  const int tid = threadIdx.x, wv = tid >> 6, c = tid & 15, q = (tid >> 4) & 3;
  int bl = blockIdx.x;
  const float *d, *a;
  int ldd = MLP_H, lda = MLP_H, j0, k0, ow, ob, K = MLP_H, J = MLP_H;
  if (bl < UB2) {
    d = o.d3, a = o.a2, ow = MLP_OFF_W3, ob = MLP_OFF_B3, j0 = bl / 8 * 16, k0 = bl % 8 * 16;
  } else if ((bl -= UB2) < UB2) {
    d = o.d2, a = o.a1, ow = MLP_OFF_W2, ob = MLP_OFF_B2, j0 = bl / 8 * 16, k0 = bl % 8 * 16;
  } else if ((bl -= UB2) < UB1) {
    d = o.d1, a = o.x, ow = MLP_OFF_W1, ob = MLP_OFF_B1, j0 = bl / 3 * 16, k0 = bl % 3 * 16, K = lda = MLP_IN;
  } else {
    bl -= UB1;
    d = o.dy, a = o.a3, ow = MLP_OFF_W4, ob = MLP_OFF_B4, j0 = 0, k0 = bl * 16, J = ldd = MLP_OUT;
  }
  // this wave's rows: a whole number of MFMA steps of four
  const int per = ((B + UPW - 1) / UPW + 3) / 4 * 4;
  const int b0 = min(wv * per, B), b1 = min(B, b0 + per);
  const float *dl = d + min(j0 + c, J - 1), *al = a + k0 + c;
  const bool jin = j0 + c < J;
  v4f acc = {0.0f, 0.0f, 0.0f, 0.0f}, accb = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int b = b0; b < b1; b += 4 * UPU) {
    float dv[UPU], av[UPU];
#pragma unroll
    for (int i = 0; i < UPU; ++i) {
      const int r = min(b + 4 * i + q, B - 1);
      dv[i] = dl[(size_t)r * ldd];
      av[i] = al[(size_t)r * lda];
    }
#pragma unroll
    for (int i = 0; i < UPU; ++i) {
      const float dd = jin && b + 4 * i + q < b1 ? dv[i] : 0.0f;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dd, av[i], acc, 0, 0, 0);
      if (k0 == 0) accb = __builtin_amdgcn_mfma_f32_16x16x4f32(dd, 1.0f, accb, 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    part[wv][(4 * q + i) * 16 + c] = acc[i];
    if (c == 0) partb[wv][4 * q + i] = accb[i];
  }
  __syncthreads();
  if (tid < 256) {
    const int j = j0 + tid / 16, k = k0 + tid % 16;
    if (j < J) {
      float g = 0.0f;
#pragma unroll
      for (int w = 0; w < UPW; ++w) g += part[w][tid];
      const int i = ow + j * K + k;
      adam_one(th, m, v, i, g, ak);
      if (grad) grad[i] = g;
    }
  } else if (tid < 256 + 16 && k0 == 0) {
    const int j = j0 + tid - 256;
    if (j < J) {
      float g = 0.0f;
#pragma unroll
      for (int w = 0; w < UPW; ++w) g += partb[w][tid - 256];
      adam_one(th, m, v, ob + j, g, ak);
      if (grad) grad[ob + j] = g;
    }
  }
  if (blockIdx.x == 0 && loss) {
    __syncthreads();
    float *red = &part[0][0];  // [UPT]
    float s = 0.0f;
    for (int e = tid; e < ntiles; e += UPT) s += o.loss[e];
    red[tid] = s;
    __syncthreads();
    for (int k = UPT / 2; k > 0; k >>= 1) {
      if (tid < k) red[tid] += red[tid + k];
      __syncthreads();
    }
    if (tid == 0) *loss = red[0] * (1.0f / (float)(B * MLP_OUT));
  }
}

__global__ __launch_bounds__(256) void k_mlp_forward(const uint16_t *W, const float *x, float *y) {
  __shared__ float s_x[MLP_IN], s_h0[MLP_H], s_h1[MLP_H], s_y[MLP_OUT];
  const long b = blockIdx.x;
  if (threadIdx.x < MLP_IN) s_x[threadIdx.x] = x[b * MLP_IN + threadIdx.x];
  mlp_eval_block(W, s_x, s_h0, s_h1, s_y);
  if (threadIdx.x < MLP_OUT) y[b * MLP_OUT + threadIdx.x] = s_y[threadIdx.x];
}

hipError_t launch_mlp_forward(const uint16_t *W, const float *x, long long n, float *y, hipStream_t s) {
  for (long long b0 = 0; b0 < n; b0 += (1 << 30)) {
    const long long nb = n - b0 < (1 << 30) ? n - b0 : (1 << 30);
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned int)nb), dim3(256), 0, s, W, x + b0 * MLP_IN,
                       y + b0 * MLP_OUT);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// the workspace of a batch of B rows; returns its floats (work may be null)
static size_t ws_map(void *work, int B, TrainRows *o) {
  float *f = (float *)work;
  size_t used = 0;
  auto take = [&](size_t n) {
    float *r = f ? f + used : nullptr;
    used += (n + 63) / 64 * 64;
    return r;
  };
  o->bad = (unsigned int *)take(64);
  o->x = take((size_t)B * MLP_IN);
  for (float **p : {&o->a1, &o->a2, &o->a3, &o->d1, &o->d2, &o->d3}) *p = take((size_t)B * MLP_H);
  o->dy = take((size_t)B * MLP_OUT);
  o->loss = take((size_t)(B + TRM - 1) / TRM);
  return used;
}

template <int MB>
static hipError_t train_rows(const float *x, const float *t, long long n, const int32_t *order, long long off, int B,
                             const float *th, const TrainRows &o, hipStream_t s, int *ntiles) {
  constexpr size_t lds = train_rows_lds<MB>();
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute((const void *)k_train_rows<MB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  *ntiles = (B + MB * TRM - 1) / (MB * TRM);
  hipLaunchKernelGGL(k_train_rows<MB>, dim3(*ntiles), dim3(TRT), lds, s, x, t, n, order, off, B, th, o);
  return hipGetLastError();
}

// one optimiser step on the batch at order[off .. off + B)
static hipError_t train_step(const float *x, const float *t, long long n, const int32_t *order, long long off, int B,
                             float *th, float *m, float *v, long long step, float lr, float b1, float b2, float eps,
                             float *loss, float *grad, const TrainRows &o, hipStream_t s) {
  // one row block per workgroup while that leaves CUs idle, else two, which
  // read the weights half as often
  int ntiles = 0;
  hipError_t e = B <= TRAIN_MB1_MAX ? train_rows<1>(x, t, n, order, off, B, th, o, s, &ntiles)
                                    : train_rows<2>(x, t, n, order, off, B, th, o, s, &ntiles);
  if (e != hipSuccess) return e;
  const double c1 = 1.0 - std::pow((double)b1, (double)step), c2 = 1.0 - std::pow((double)b2, (double)step);
  const AdamK ak{lr, b1, b2, eps, (float)c1, (float)c2};
  hipLaunchKernelGGL(k_train_update, dim3(UBLOCKS), dim3(UPT), 0, s, o, B, ntiles, th, m, v, ak, grad, loss);
  return hipGetLastError();
}

}  // namespace gs

using namespace gs;

extern "C" size_t gs_mlp_train_workspace(int32_t batch) {
  if (batch < 1) return 0;
  TrainRows o;
  return ws_map(nullptr, batch, &o) * sizeof(float);
}

extern "C" gs_status gs_mlp_train(const float *x, const float *t, int64_t n, const int32_t *order, int64_t n_order,
                                  int32_t batch, float *theta, float *adam_m, float *adam_v, int64_t step0,
                                  double lr, double beta1, double beta2, double eps, float *loss, float *grad_last,
                                  void *work, size_t work_bytes, void *hip_stream) {
  if (!x || !t || !order || !theta || !adam_m || !adam_v || !work) return GS_EINVAL;
  if (n < 1 || n_order < 0 || batch < 1 || batch > (1 << 20) || step0 < 0) return GS_EINVAL;
  if (!(lr > 0.0) || !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
    return GS_EINVAL;
  if (work_bytes < gs_mlp_train_workspace(batch)) return GS_EINVAL;
  hipStream_t s = (hipStream_t)hip_stream;
  TrainRows w;
  (void)ws_map(work, batch, &w);
  if (hipMemsetAsync(w.bad, 0, 4, s) != hipSuccess) return GS_EDEVICE;
  const long long steps = n_order / batch;
  for (long long k = 0; k < steps; ++k) {
    if (train_step(x, t, n, order, k * batch, batch, theta, adam_m, adam_v, step0 + k + 1, (float)lr,
                   (float)beta1, (float)beta2, (float)eps, loss ? loss + k : nullptr,
                   k == steps - 1 ? grad_last : nullptr, w, s) != hipSuccess)
      return GS_EDEVICE;
  }
  unsigned int bad = 0;
  if (hipMemcpyAsync(&bad, w.bad, 4, hipMemcpyDeviceToHost, s) != hipSuccess) return GS_EDEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return GS_EDEVICE;
  return bad ? GS_EINVAL : GS_OK;
}
