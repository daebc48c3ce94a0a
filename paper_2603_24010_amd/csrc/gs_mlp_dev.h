// Device side of the Newton guess network: 48 -> 128 -> 128 -> 128 -> 3, GELU
// hidden layers, linear output; weights in bfloat16, products and sums in
// binary32.  One workgroup evaluates one input vector; every (output, part)
// partial sum has a fixed order, and the eight parts of an output are combined by
// the same butterfly, so the result does not depend on the workgroup size.
#ifndef GS_MLP_DEV_H
#define GS_MLP_DEV_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gs {

constexpr int MLP_IN = 48;
constexpr int MLP_H = 128;
constexpr int MLP_OUT = 3;
constexpr int MLP_NPARAM = 39683;
// flat layout: W1[128][48] b1 W2[128][128] b2 W3[128][128] b3 W4[3][128] b4
constexpr int MLP_OFF_W1 = 0;
constexpr int MLP_OFF_B1 = MLP_OFF_W1 + MLP_H * MLP_IN;
constexpr int MLP_OFF_W2 = MLP_OFF_B1 + MLP_H;
constexpr int MLP_OFF_B2 = MLP_OFF_W2 + MLP_H * MLP_H;
constexpr int MLP_OFF_W3 = MLP_OFF_B2 + MLP_H;
constexpr int MLP_OFF_B3 = MLP_OFF_W3 + MLP_H * MLP_H;
constexpr int MLP_OFF_W4 = MLP_OFF_B3 + MLP_H;
constexpr int MLP_OFF_B4 = MLP_OFF_W4 + MLP_OUT * MLP_H;
static_assert(MLP_OFF_B4 + MLP_OUT == MLP_NPARAM, "layout");
// normalisation block (binary64): x_mean[48] x_scale[48] y_mean[3] y_scale[3]
constexpr int MLP_NORM = 2 * MLP_IN + 2 * MLP_OUT;

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline float gelu_f32(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

// One workgroup's evaluation of one input, the weights in the registers of its
// BS threads: thread t's items t, t + BS, ... of a layer are output q / 8, part
// q % 8, which sums inputs [part K / 8, (part + 1) K / 8) in order.  load()
// issues every weight's load (16-byte ones where a part is 16 inputs), so that
// the network costs the caller one round trip, behind work of its own, instead
// of one per layer: in the strict step's field solve the network took 4.5 us
// with its loads in the layers.
template <int BS>
struct MlpWeights {
  static constexpr int IT = MLP_H * 8 / BS;  // items per thread of a hidden layer
  static_assert(MLP_H * 8 % BS == 0 && BS >= MLP_H, "whole items");
  template <int N>
  struct Part {
    uint16_t w[N];
  };
  Part<MLP_IN / 8> w1[IT];
  Part<16> w2[IT], w3[IT], w4;
  uint16_t b[3][IT], b4;

  __device__ inline void load(const uint16_t *W) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int q = t + k * BS, j = q >> 3, part = q & 7;
      __builtin_memcpy(&w1[k], W + MLP_OFF_W1 + j * MLP_IN + part * (MLP_IN / 8), MLP_IN / 8 * 2);
      __builtin_memcpy(&w2[k], W + MLP_OFF_W2 + j * MLP_H + part * 16, 32);
      __builtin_memcpy(&w3[k], W + MLP_OFF_W3 + j * MLP_H + part * 16, 32);
      b[0][k] = W[MLP_OFF_B1 + j];
      b[1][k] = W[MLP_OFF_B2 + j];
      b[2][k] = W[MLP_OFF_B3 + j];
    }
    const int j = t < MLP_OUT * 8 ? t >> 3 : 0;
    __builtin_memcpy(&w4, W + MLP_OFF_W4 + j * MLP_H + (t & 7) * 16, 32);
    b4 = W[MLP_OFF_B4 + j];
  }

  template <int N>
  static __device__ inline float part_sum(const uint16_t *w, const float *x) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) s += bf16_to_f32(w[i]) * x[i];
    return s;
  }
  // the sum of the eight parts of an output (consecutive lanes), the same in all
  // of them: + lane ^ 4, + lane ^ 2, + lane ^ 1, with lane ^ 4 as the mirror of
  // eight lanes and then of four (DPP moves; LDS permutes cost a round trip each)
  template <int CTRL>
  static __device__ inline float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
  }
  static __device__ inline float parts(float s) {
    s += dpp<0x1B>(dpp<0x141>(s));  // quad_perm 3 2 1 0 of row_half_mirror
    s += dpp<0x4E>(s);              // quad_perm 2 3 0 1
    s += dpp<0xB1>(s);              // quad_perm 1 0 3 2
    return s;
  }
  // a hidden layer of 8 N inputs: the lanes of parts 0 .. IT - 1 finish one of
  // the thread's outputs each, so that GELU is evaluated once
  template <int N, class WT>
  __device__ inline void hidden(const WT *w, const uint16_t *bias, const float *in, float *out) {
    static_assert(IT <= 8, "an output per lane of a group");
    const int part = threadIdx.x & 7;
    float x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = in[part * N + i];
    float z = 0.0f;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const float s = parts(part_sum<N>((const uint16_t *)&w[k], x)) + bf16_to_f32(bias[k]);
      z = part == k ? s : z;
    }
    if (part < IT) out[(threadIdx.x + part * BS) >> 3] = gelu_f32(z);
    lds_barrier();
  }

  // y = net(x): x[48] in LDS (already normalised), h0/h1 scratch of 128 floats
  // in LDS, y[3] in LDS.  Every thread of the workgroup calls it.
  __device__ inline void eval(const float *x, float *h0, float *h1, float *y) {
    lds_barrier();
    hidden<MLP_IN / 8>(w1, b[0], x, h0);
    hidden<16>(w2, b[1], h0, h1);
    hidden<16>(w3, b[2], h1, h0);
    if (threadIdx.x < 64) {
      const float s = parts(part_sum<16>(w4.w, h0 + (threadIdx.x & 7) * 16));
      if (threadIdx.x < MLP_OUT * 8 && (threadIdx.x & 7) == 0) y[threadIdx.x >> 3] = s + bf16_to_f32(b4);
    }
    lds_barrier();
  }
};

}  // namespace gs
#endif
