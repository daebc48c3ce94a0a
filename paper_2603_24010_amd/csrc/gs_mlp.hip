// Training and batch evaluation of the Newton guess network on the GPU.
//
// Training is plain mini-batch gradient descent with Adam (Kingma and Ba,
// 2015) on the mean squared error, in binary32 on the matrix cores; every
// reduction has a fixed order, so a run is bitwise repeatable.  Batch evaluation uses
// the strict step's device routine for few rows and the matrix cores for many
// (bfloat16 weights, binary32 activations and sums in both).
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
// At batch 1024 (64 row tiles, 160 blocks) the two kernels take 16.2 and 8.2 us
// (19.7 with the library's erff and expf, and indices, rows and biases fetched one
// after the other where they are used) and a step 25.5 us, launches included; one
// kernel per GEMM, column sum and reduction (22 launches) took 157 us.
//
// All products run on the matrix cores in binary32 (v_mfma_f32_16x16x4_f32:
// binary32 products and sums).  Lane l gives A(l % 16, l / 16) and B(l / 16, l
// % 16); its accumulator r holds D(4 (l / 16) + r, l % 16).  The order of a
// sum over k is free but fixed: where k runs along memory, the four MFMAs of a
// 16-wide step take k = 4 (l / 16) + j, j = 0..3, so that a lane reads four
// consecutive values.
// ---------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));

// Phi(z), the normal distribution function, in some twenty instructions without a
// branch (the library's erff has two, and a wave takes both): Phi(-t) = 2^-(1 + t
// P(t)) for t >= 0, where t P(t) = -log2 erfc(t / sqrt 2) is nearly a parabola.  P is
// the minimax polynomial of degree 9 on [0, 5.5] for the absolute error of Phi
// (1.6e-9), constant past it (Phi(-5.5) = 1.9e-8).  Against 64 bits in the 2-norm, for
// normal z of scale 0.05, 0.2, 0.5, 1 and 3: GELU 4.3, 4.3, 3.8, 3.3 and 2.6e-8, its
// derivative 4.4, 4.4, 4.2, 4.1 and 3.9e-8; with the library's erff and expf 3.7, 3.9,
// 4.2, 3.9 and 2.9e-8, and 3.9, 3.9, 3.9, 4.1 and 4.0e-8.  So small z lose a little and
// larger ones gain; over 42 training runs (batches 64 to 4096, 16 to 64 steps) the weights
// are off by 1.71e-7 with either and the gradient by 2.93e-7, 2.98e-7 with the library's.
__device__ inline float normal_cdf(float z) {
  const float t = fabsf(z), u = fminf(t, 5.5f);
  float h = 3.639413037603845e-08f;
  h = __builtin_fmaf(h, u, -1.0236597063340014e-06f);
  h = __builtin_fmaf(h, u, 1.2430210517777596e-05f);
  h = __builtin_fmaf(h, u, -8.325302042067051e-05f);
  h = __builtin_fmaf(h, u, 0.0002973641094285995f);
  h = __builtin_fmaf(h, u, -2.5722472855704837e-05f);
  h = __builtin_fmaf(h, u, -0.006927415728569031f);
  h = __builtin_fmaf(h, u, 0.052434973418712616f);
  h = __builtin_fmaf(h, u, 0.45922109484672546f);
  h = __builtin_fmaf(h, u, 1.1511043310165405f);
  const float a = 0.5f * __builtin_amdgcn_exp2f(-t * h);
  return z >= 0.0f ? 1.0f - a : a;
}

__device__ inline float gelu_both(float z, float *grad) {
  const float Phi = normal_cdf(z);
  // (2^x: -z^2 / (2 ln 2))
  *grad = Phi + z * (0.39894228040143268f * __builtin_amdgcn_exp2f(-0.72134752044448170f * z * z));
  return z * Phi;
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
constexpr int TRAIN_CUS = 256;      // workgroups of k_train_rows that run at once at full speed (one a CU)
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
  // (the last update wrote the parameters from every XCD: each first read of them is a
  // trip to memory, so the small ones go out now too, not where they are used)
  __shared__ float sW4[MLP_OUT * MLP_H];
  const float w4v = tid < MLP_OUT * MLP_H ? W4[tid] : 0.0f;
  const float b1 = th[MLP_OFF_B1 + n0 + c], b2 = th[MLP_OFF_B2 + n0 + c], b3 = th[MLP_OFF_B3 + n0 + c];
  float b4[MLP_OUT];
#pragma unroll
  for (int u = 0; u < MLP_OUT; ++u) b4[u] = th[MLP_OFF_B4 + u];
  load_fwd<MLP_IN>(W1, n0, w1);
  load_fwd<MLP_H>(W2, n0, wa);
  // the batch's rows (past its end the last one, whose derivative is zeroed);
  // an index outside [0, n) is replaced by 0 and counted
  // (an index, then the row it names: each of the two trips is made once, for all of a
  // thread's words together)
  constexpr int RW = MLP_IN + MLP_OUT, NE = (R * RW + TRT - 1) / TRT;
  long long idx[NE];
  float val[NE];
#pragma unroll
  for (int u = 0; u < NE; ++u) idx[u] = order[off + min(r0 + min((tid + u * TRT) / RW, R - 1), B - 1)];
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    const int f = (tid + u * TRT) % RW;
    const bool ok = idx[u] >= 0 && idx[u] < n;
    const long long i = ok ? idx[u] : 0;
    idx[u] = ok ? 0 : 1;  // (from here: whether it was out of range)
    val[u] = *(f < MLP_IN ? x + i * MLP_IN + f : t + i * MLP_OUT + f - MLP_IN);
  }
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    const int e = tid + u * TRT, r = e / RW, f = e % RW;
    if (e >= R * RW) break;
    if (idx[u] && f == 0 && r0 + r < B) atomicAdd(o.bad, 1u);
    if (f < MLP_IN) {
      A0[r * TLD + f] = val[u];
      if (r0 + r < B) o.x[(size_t)(r0 + r) * MLP_IN + f] = val[u];
    } else {
      st[r * MLP_OUT + f - MLP_IN] = val[u];
    }
  }
  static_assert(MLP_OUT * MLP_H <= TRT, "a word per thread");
  if (tid < MLP_OUT * MLP_H) sW4[tid] = w4v;
  lds_barrier();
  // a hidden layer's epilogue: bias, GELU to LDS and the workspace, GELU' to LDS
  v4f acc[MB];
  auto hidden = [&](float bj, float *out, float *g, float *global) {
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
  hidden(b1, A1, G1, o.a1);
  lds_barrier();
  mul_block<MB, MLP_H>(A1, wa, acc);
  load_bwd(W3, n0, wa);
  hidden(b2, A0, G2, o.a2);
  lds_barrier();
  mul_block<MB, MLP_H>(A0, wb, acc);
  load_bwd(W2, n0, wb);
  hidden(b3, A1, G3, o.a3);
  lds_barrier();
  // the output layer: eight lanes per output, sixteen inputs each
  const float inv = 1.0f / (float)(B * MLP_OUT);
  for (int e = tid; e < R * MLP_OUT * 8; e += TRT) {
    const int p = e & 7, r = (e >> 3) / MLP_OUT, u = (e >> 3) % MLP_OUT;
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += A1[r * TLD + 16 * p + k] * sW4[u * MLP_H + 16 * p + k];
    s += __shfl_xor(s, 4, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 1, 64);
    if (p == 0) {
      const bool in = r0 + r < B;
      const float d = in ? s + (u == 0 ? b4[0] : u == 1 ? b4[1] : b4[2]) - st[r * MLP_OUT + u] : 0.0f;
      se[r * MLP_OUT + u] = d * d;
      sdy[r * MLP_OUT + u] = 2.0f * d * inv;
      if (in) o.dy[(size_t)(r0 + r) * MLP_OUT + u] = 2.0f * d * inv;
    }
  }
  lds_barrier();
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
    for (int u = 0; u < MLP_OUT; ++u) s += sdy[r * MLP_OUT + u] * sW4[u * MLP_H + k];
    s *= G3[r * TLD + k];
    A0[r * TLD + k] = s;
    if (r0 + r < B) o.d3[(size_t)(r0 + r) * MLP_H + k] = s;
  }
  lds_barrier();
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
  lds_barrier();
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
  lds_barrier();
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
    lds_barrier();
    float *red = &part[0][0];  // [UPT]
    float s = 0.0f;
    for (int e = tid; e < ntiles; e += UPT) s += o.loss[e];
    red[tid] = s;
    lds_barrier();
    for (int k = UPT / 2; k > 0; k >>= 1) {
      if (tid < k) red[tid] += red[tid + k];
      lds_barrier();
    }
    if (tid == 0) *loss = red[0] * (1.0f / (float)(B * MLP_OUT));
  }
}

// ---------------------------------------------------------------------------
// Batch evaluation.  k_mlp_forward: one row per workgroup with the strict step's
// device routine, for few rows.  k_mlp_tiles: persistent workgroups take tiles
// of 32 rows through the network on the matrix cores; every wave holds the
// weights of its 16 outputs of each layer in registers for the whole launch
// (the row kernel reads all of them again for every row, which bounds it), and
// only activations pass through LDS.
// The weights are bfloat16, so a binary32 activation is split exactly into three
// bfloat16 terms, 8 significant bits each (hi + mid + lo), and the three
// products, each exact, are summed in binary32 by v_mfma_f32_16x16x32_bf16, the
// smallest first.  Errors against 64 bits (2-norm, 32 to 1e6 rows): 4.1e-8, the
// row kernel's 5.1e-8.  92000 rows take 45 us (423 us by rows), 1e6 rows 0.42 ms
// (4.5 ms): the activations' reads from LDS, GELU with the splits, and the barriers
// between the layers share that.  (Waves of 32 outputs, which read half as much, took
// 6% off 92000 rows and added 5% at 2048.)
// Lane l gives A(l % 16, 8 (l / 16) + i) and B(8 (l / 16) + i, l % 16), i =
// 0..7, and holds D(4 (l / 16) + r, l % 16): A rows are outputs, B columns batch
// rows, so that a lane ends up with four consecutive outputs of one row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mlp_forward(const uint16_t *W, const float *x, float *y) {
  __shared__ float s_x[MLP_IN], s_h0[MLP_H], s_h1[MLP_H], s_y[MLP_OUT];
  const long b = blockIdx.x;
  MlpWeights<256> mw;
  mw.load(W);
  if (threadIdx.x < MLP_IN) s_x[threadIdx.x] = x[b * MLP_IN + threadIdx.x];
  mw.eval(s_x, s_h0, s_h1, s_y);
  if (threadIdx.x < MLP_OUT) y[b * MLP_OUT + threadIdx.x] = s_y[threadIdx.x];
}

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
// The row kernel up to here: 5.5 us at 512 rows against the tiles' 7.5, 6.9 and 7.6 at
// 768, 7.9 and 7.6 at 896, 13.5 and 7.6 at 2048 (launches included)
constexpr long long FORWARD_ROWS_MAX = 768;
constexpr int FTW = 8, FTT = FTW * 64;  // waves (one 16-output block each) and threads
constexpr int FTR = 32;                 // rows per tile: two blocks of 16
constexpr int FTLD = MLP_H + 8;         // row stride of an activation plane in LDS (bfloat16)
constexpr int FTP = FTR * FTLD;         // one plane; three per buffer, two buffers
static_assert(FTW * 16 == MLP_H, "a wave per output block");

// Two values as three pairs of bfloat16, x = hi + mid + lo exactly (truncation leaves
// 8 of 24 significant bits to each); infinities and NaN stay in hi, a NaN by its quiet
// bit (results of arithmetic have it set; see quiet for others).
__device__ inline void split3(float x0, float x1, uint32_t *hi, uint32_t *mid, uint32_t *lo) {
  const float x[2] = {x0, x1};
  float r1[2], r2[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float d = x[i] - __uint_as_float(__float_as_uint(x[i]) & 0xFFFF0000u);
    r1[i] = d == d ? d : 0.0f;
    r2[i] = r1[i] - __uint_as_float(__float_as_uint(r1[i]) & 0xFFFF0000u);
  }
  // the upper halves of both
  *hi = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u);
  *mid = __builtin_amdgcn_perm(__float_as_uint(r1[1]), __float_as_uint(r1[0]), 0x07060302u);
  *lo = __builtin_amdgcn_perm(__float_as_uint(r2[1]), __float_as_uint(r2[0]), 0x07060302u);
}

__device__ inline float quiet(float x) { return x != x ? __uint_as_float(0x7FC00000u) : x; }

__device__ inline v8bf ld8(const uint16_t *a) {
  v8bf v;
  __builtin_memcpy(&v, a, 16);
  return v;
}

// one layer of K = 32 S inputs (zero-padded) for the wave's output block and
// both row blocks
template <int S>
__device__ inline void tile_layer(const uint16_t *src, const v8bf *w, v4f *acc) {
  const int c = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int m = 0; m < 2; ++m) acc[m] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int pl = 2; pl >= 0; --pl)
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const v8bf b = *(const v8bf *)(src + pl * FTP + (16 * m + c) * FTLD + 32 * s + 8 * q);
        acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], b, acc[m], 0, 0, 0);
      }
}

__global__ __launch_bounds__(FTT, 4) void k_mlp_tiles(const uint16_t *W, const float *x, long long n, float *y) {
  __shared__ __align__(16) uint16_t buf[2][3 * FTP];
  const int tid = threadIdx.x, wv = tid >> 6, c = tid & 15, q = (tid >> 4) & 3;
  const int o0 = wv * 16;
  // the weights: rows o0 + c of each layer (the first layer's inputs past 48
  // and the last layer's outputs past 3 are zero)
  v8bf w1[2], w2[4], w3[4], w4[4];
  const v8bf zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = 32 * s + 8 * q;
    const v8bf v = ld8(W + MLP_OFF_W1 + (o0 + c) * MLP_IN + (k < MLP_IN ? k : 0));
    w1[s] = k < MLP_IN ? v : zero;
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 32 * s + 8 * q;
    w2[s] = ld8(W + MLP_OFF_W2 + (o0 + c) * MLP_H + k);
    w3[s] = ld8(W + MLP_OFF_W3 + (o0 + c) * MLP_H + k);
    const v8bf v = ld8(W + MLP_OFF_W4 + (c < MLP_OUT ? c : 0) * MLP_H + k);
    w4[s] = c < MLP_OUT ? v : zero;
  }
  float b1[4], b2[4], b3[4], b4[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    b1[r] = bf16_to_f32(W[MLP_OFF_B1 + o0 + 4 * q + r]);
    b2[r] = bf16_to_f32(W[MLP_OFF_B2 + o0 + 4 * q + r]);
    b3[r] = bf16_to_f32(W[MLP_OFF_B3 + o0 + 4 * q + r]);
    b4[r] = bf16_to_f32(W[MLP_OFF_B4 + min(r, MLP_OUT - 1)]);
  }
  const long long tiles = (n + FTR - 1) / FTR;
  // a tile's inputs: 4 per thread of its 32 x 64 (zero-padded), rows past n
  // repeating the last
  auto load_x = [&](long long t, float *v) {
    const int r = tid >> 4, f = 4 * (tid & 15);
    const long long row = min(t * FTR + r, n - 1);
    const v4f a = ld4(x + row * MLP_IN + (f < MLP_IN ? f : 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = f < MLP_IN ? quiet(a[i]) : 0.0f;
  };
  // four consecutive values of row r, from column k, to a buffer's planes
  auto put = [&](uint16_t *dst, int r, int k, const float *v) {
    uint32_t *d = (uint32_t *)(dst + r * FTLD + k);
#pragma unroll
    for (int i = 0; i < 2; ++i) split3(v[2 * i], v[2 * i + 1], &d[i], &d[FTP / 2 + i], &d[FTP + i]);
  };
  v4f acc[2];
  auto hidden = [&](uint16_t *dst, const float *bias) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = acc[m][r] + bias[r];
        v[r] = z * normal_cdf(z);
      }
      put(dst, 16 * m + c, o0 + 4 * q, v);
    }
    lds_barrier();
  };
  float xv[4];
  if ((long long)blockIdx.x < tiles) load_x(blockIdx.x, xv);
  for (long long t = blockIdx.x; t < tiles; t += gridDim.x) {
    put(buf[0], tid >> 4, 4 * (tid & 15), xv);
    if (t + gridDim.x < tiles) load_x(t + gridDim.x, xv);
    lds_barrier();
    tile_layer<2>(buf[0], w1, acc);
    hidden(buf[1], b1);
    tile_layer<4>(buf[1], w2, acc);
    hidden(buf[0], b2);
    tile_layer<4>(buf[0], w3, acc);
    hidden(buf[1], b3);
    if (wv < 2) {  // the three outputs of row block wv
      tile_layer<4>(buf[1], w4, acc);
      const long long row = t * FTR + 16 * wv + c;
      const v4f a = wv == 0 ? acc[0] : acc[1];
      if (q == 0 && row < n)
#pragma unroll
        for (int r = 0; r < MLP_OUT; ++r) y[row * MLP_OUT + r] = a[r] + b4[r];
    }
    // (the next tile's inputs go to buf[0], which every wave is done with; the
    // layer after them is written to buf[1] behind the barrier in between)
  }
}

// finite: no weight is infinite in bfloat16.  (The tiles' lower terms are mostly zero,
// and zero times an infinite weight is NaN where the whole activation's product is not.)
hipError_t launch_mlp_forward(const uint16_t *W, bool finite, const float *x, long long n, float *y, int ncu,
                              hipStream_t s) {
  if (n > FORWARD_ROWS_MAX && finite) {
    const long long tiles = (n + FTR - 1) / FTR;
    const unsigned int grid = (unsigned int)(tiles < 2ll * ncu ? tiles : 2ll * ncu);
    hipLaunchKernelGGL(k_mlp_tiles, dim3(grid), dim3(FTT), 0, s, W, x, n, y);
    return hipGetLastError();
  }
  constexpr long long MOST = 1 << 23;  // rows a launch (2^31 threads)
  for (long long b = 0; b < n; b += MOST) {
    const long long nb = n - b < MOST ? n - b : MOST;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned int)nb), dim3(256), 0, s, W, x + b * MLP_IN, y + b * MLP_OUT);
    const hipError_t e = hipGetLastError();
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
  // one row block per workgroup, or two where that gives each CU one workgroup and one
  // would give it two (two read the weights half as often, but past that leave a second
  // round of large workgroups on few CUs).  A step in us with one and with two: batch 4096
  // 45.8 and 52.5, 4600 56.0 and 54.8, 8192 72.9 and 71.1, 10000 91.1 and 98.5, 16384 128
  // and 128, 32768 239 and 243
  const int blocks = (B + TRM - 1) / TRM;
  int ntiles = 0;
  hipError_t e = blocks > TRAIN_CUS && blocks <= 2 * TRAIN_CUS
                     ? train_rows<2>(x, t, n, order, off, B, th, o, s, &ntiles)
                     : train_rows<1>(x, t, n, order, off, B, th, o, s, &ntiles);
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
