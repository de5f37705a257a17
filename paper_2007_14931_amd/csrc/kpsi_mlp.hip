// Learned efficiency: a 4 -> 64 -> 64 -> 1 network (SiLU, SiLU, sigmoid) trained on accept
// labels with binary cross-entropy and Adam, and evaluated once per normalisation event.
// The 64x64 layer (forward, weight gradient and input gradient) runs on BF16 matrix cores
// (v_mfma_f32_16x16x32_bf16: 16x16 outputs, 32-deep products, 8 operands per lane) with FP32
// accumulation; the 4-wide input layer and the output layer run on the vector ALUs in FP32.
// Master weights are FP32; the Adam step also writes the BF16 copies of the 64x64 layer in both
// layouts, which the gradient kernel loads into registers as operands.
//
// Parameter layout (4545 floats): W1[64][4], b1[64], W2[64][64] (row = output), b2[64],
// w3[64], b3.  Network input: u = (2 (m - lo)/(hi - lo) - 1, cos theta_K*, cos theta_J/psi,
// phi/pi).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kpsi_internal.h"
#include "kpsi_silu.h"

namespace kpsi {

namespace nn {

constexpr int P_W1 = 0, P_B1 = 256, P_W2 = 320, P_B2 = 4416, P_W3 = 4480, P_B3 = 4544;
constexpr int TE = 64;   // events per tile

typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// float -> bf16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned short bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float silu(float z) {
  const float d = 1.0f + __expf(-z);
  return silu_of(z, d, __builtin_amdgcn_rcpf(d));
}
__device__ __forceinline__ void silu_both(float z, float& sl, float& ds) {
  const float d = 1.0f + __expf(-z);
  silu_both_of(z, d, __builtin_amdgcn_rcpf(d), sl, ds);
}
// Sum over the 16 lanes of a row, in every lane (quad permutations, then the mirrored half rows and
// rows: their lanes hold equal values by then).
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum(float x) {
  x += dpp<0xB1>(x);
  x += dpp<0x4E>(x);
  x += dpp<0x141>(x);
  return x + dpp<0x140>(x);
}
// Eight consecutive FP32 weights (16-byte aligned) as a BF16 operand.
__device__ __forceinline__ bf8_t to_bf8(const float* p) {
  const f4_t lo = *reinterpret_cast<const f4_t*>(p), hi = *reinterpret_cast<const f4_t*>(p + 4);
  bf8_t v;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = (__bf16)lo[j];
    v[4 + j] = (__bf16)hi[j];
  }
  return v;
}
// Input layer in registers, for the features f(c) = 32 (c / 8) + 8 lg + c % 8 of a lane (the order
// of the matrix cores' operands); W1 rounded to BF16 like W2.
struct L1Weights {
  float w[16][4], b[16];
  __device__ __forceinline__ void load(const float* params, int lg) {
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const int f = 32 * (c >> 3) + 8 * lg + (c & 7);
      const f4_t v = *reinterpret_cast<const f4_t*>(params + P_W1 + 4 * f);
#pragma unroll
      for (int k = 0; k < 4; ++k) w[c][k] = (float)(__bf16)v[k];
      b[c] = params[P_B1 + f];
    }
  }
  __device__ __forceinline__ float z(int c, const float* u) const {
    float x = b[c];
#pragma unroll
    for (int k = 0; k < 4; ++k) x = __builtin_fmaf(w[c][k], u[k], x);
    return x;
  }
};

// Row strides of the LDS tiles: 16-byte rows for the vector accesses, and rows 4 and 8 apart start
// in other banks.
constexpr int SF = 68, SH = 72;
struct __align__(16) Smem {
  float D1[TE * SF];                // silu'(z1) [event][feature]
  unsigned short H1[2][TE * SH];    // h1 [event][feature]
  unsigned short DZT[2][64 * SH];   // dz2 [output][event]
  f4_t U[TE];                       // network inputs
  float red[4][28 * 16];            // per-wavefront sums of the thin layers
  float sc[4][2];                   // and of b3 and the loss
};

// eight consecutive bf16 of an LDS row (16-byte aligned) as an MFMA operand: one 16-byte read
__device__ __forceinline__ bf8_t ld8(const unsigned short* p) { return *reinterpret_cast<const bf8_t*>(p); }

// Four values down the column (lane % 16) of the 4 x 16 block of 16-bit values whose rows start at p
// in steps of `stride`, for each group of 16 lanes its own block: the transposing LDS read, for which
// lane t of a group passes row t / 4, columns 4 (t % 4) on.
typedef short s4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s4_t ld4t(const unsigned short* p, int stride, int l16) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s4_t*)(p + stride * (l16 >> 2) + 4 * (l16 & 3)));
}
// Operand whose eight k values are the rows 0..7 of such a block.
__device__ __forceinline__ bf8_t ld8t(const unsigned short* p, int stride, int l16) {
  const s4_t lo = ld4t(p, stride, l16), hi = ld4t(p + 4 * stride, stride, l16);
  return __builtin_bit_cast(bf8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Orders the LDS accesses of one wavefront's lanes (they execute in order; this holds the compiler).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// a and b, c and d summed over the four 16-lane rows as (row 0 + row 1) + (row 2 + row 3): row k of
// the result holds the sum of the k-th value.
__device__ __forceinline__ float rows_sum4(float a, float b, float c, float d) {
  auto pair = [](float x, float y, auto f) {
    const auto r = f(__float_as_uint(x), __float_as_uint(y));
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  auto s16 = [](unsigned x, unsigned y) { return __builtin_amdgcn_permlane16_swap(x, y, false, false); };
  auto s32 = [](unsigned x, unsigned y) { return __builtin_amdgcn_permlane32_swap(x, y, false, false); };
  return pair(pair(a, b, s16), pair(c, d, s16), s32);
}

__device__ __forceinline__ float input_map(const MlpArgs& a, int k, double x) {
  if (k == 0) return (float)(2.0 * (x - a.lo) / (a.hi - a.lo) - 1.0);
  if (k == 3) return (float)(x * 0.31830988618379067154);
  return (float)x;
}

}  // namespace nn

// Per-block gradient of the summed BCE (no 1/n) over the events [blk*per, (blk+1)*per),
// written block-major to partial[block * 4546 + v] (one contiguous record per block, so the
// writes are coalesced); v = 4545 is the loss.
//
// A block takes 64 events at a time, wavefront w the events 16 w .. 16 w + 15 of them.  The input
// layer is computed in the operand layout of the matrix cores (as in mlp_eval_kernel), the weights
// stay in registers, and each sigmoid is evaluated once for both silu and silu'.  LDS carries what
// changes hands: silu' of the first layer within the wavefront, and h1 and dz2, between the
// wavefronts, for the weight gradient, which contracts over all 64 events; these are read back
// transposed.  One barrier per 64 events (two buffers).  Bound by the latency of a step that has
// 128 events per compute unit (the weights, the chain of layers, the records): 24.9 -> 14.0 us
// for 32768 events (the weights staged through LDS by every block, 128-byte LDS rows, three
// barriers per 64 events and 60 at the end, each sigmoid evaluated three times).
__global__ __launch_bounds__(256, 1) void mlp_grad_kernel(MlpArgs a) {
  using namespace nn;
  __shared__ Smem s;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, lg = lane >> 4;
  const int64_t begin = (int64_t)blockIdx.x * a.per_block;
  const int64_t end = begin + a.per_block < a.n ? begin + a.per_block : a.n;
  // observables of event 16 w + l16 and label of event 16 w + 4 lg + l16 % 4 of a tile
  double x[4] = {0.0, 0.0, 0.0, 0.0};
  float y = 0.f;
  auto fetch = [&](int64_t e0) {
    const int64_t e = e0 + 16 * w + l16, ey = e0 + 16 * w + 4 * lg + (l16 & 3);
    if (e < end) {
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = a.obs[k][e];
    }
    if (ey < end) y = (float)a.label[ey];
  };
  fetch(begin);
  L1Weights w1;
  w1.load(a.params, lg);
  bf8_t w2[4][2], w2t[4][2];   // W2[16 nt + l16][k] and W2[k][16 nt + l16], k = 32 kk + 8 lg + j
  float b2[4], w3[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int o = 16 * nt + l16;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      w2[nt][kk] = ld8(a.w2h + 64 * o + 32 * kk + 8 * lg);
      w2t[nt][kk] = ld8(a.w2h + 4096 + 64 * o + 32 * kk + 8 * lg);
    }
    b2[nt] = a.params[P_B2 + o];
    w3[nt] = (float)(__bf16)a.params[P_W3 + o];
  }
  const float b3 = a.params[P_B3];
  float gW2[4][4];        // dW2[o = 16 w + 4 lg + r][i = 16 nt + l16]
  float gb2[4], gw3[4];   // outputs 16 nt + l16 (this lane's events)
  float gb1[4], gW1[4][4];
  float gb3 = 0.f, loss = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    gb2[i] = gw3[i] = gb1[i] = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) { gW2[i][k] = 0.f; gW1[i][k] = 0.f; }
  }
  int buf = 0;
  for (int64_t e0 = begin; e0 < end; e0 += TE, buf ^= 1) {
    unsigned short* H1 = s.H1[buf];
    unsigned short* DZT = s.DZT[buf];
    // ---- input layer: event 16 w + l16, features 32 kk + 8 lg + j
    f4_t u;
    const bool in = e0 + 16 * w + l16 < end;
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = in ? input_map(a, k, x[k]) : 0.0f;
    const float yl = y;
    const bool ok = e0 + 16 * w + 4 * lg + (l16 & 3) < end;   // the event of yl
    if (e0 + TE < end) fetch(e0 + TE);
    if (lg == 0) s.U[16 * w + l16] = u;
    const float uf[4] = {u[0], u[1], u[2], u[3]};
    bf8_t h[2];
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
      f4_t d1;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = 4 * c4 + j;
        float sl, ds;
        silu_both(w1.z(c, uf), sl, ds);
        d1[j] = ds;
        h[c >> 3][c & 7] = (__bf16)sl;
      }
      *reinterpret_cast<f4_t*>(&s.D1[(16 * w + l16) * SF + 32 * (c4 >> 1) + 8 * lg + 4 * (c4 & 1)]) = d1;
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) *reinterpret_cast<bf8_t*>(&H1[(16 * w + l16) * SH + 32 * kk + 8 * lg]) = h[kk];
    // ---- 64x64 layer: z2 of events 16 w + 4 lg + r, outputs 16 nt + l16
    float sl2[4][4], ds2[4][4], z3p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f4_t z2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) z2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h[kk], w2[nt][kk], z2, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        silu_both(z2[r] + b2[nt], sl2[nt][r], ds2[nt][r]);
        z3p[r] = __builtin_fmaf(w3[nt], sl2[nt][r], z3p[r]);
      }
    }
    // ---- output layer: each lane takes the event 4 lg + l16 % 4, then hands it to its quad
#pragma unroll
    for (int r = 0; r < 4; ++r) z3p[r] = row_sum(z3p[r]);
    const float zlo = (l16 & 1) ? z3p[1] : z3p[0], zhi = (l16 & 1) ? z3p[3] : z3p[2];
    const float z3 = ((l16 & 2) ? zhi : zlo) + b3;
    const float p = 1.0f / (1.0f + __expf(-z3)), d_not = 1.0f + __expf(z3);
    const float p_not = quotient(1.0f, d_not, newton_rcp(d_not, __builtin_amdgcn_rcpf(d_not)));
    const float dz = ok ? p - yl : 0.0f;
    // (p_not and not 1 - p, which is 0 for z3 > 17: its logarithm is then -inf, and times a label's 0 no number)
    const float term = ok ? -(yl * __logf(fmaxf(p, 1e-12f)) + (1.0f - yl) * __logf(fmaxf(p_not, 1e-12f))) : 0.0f;
    const float dz3[4] = {dpp<0x00>(dz), dpp<0x55>(dz), dpp<0xAA>(dz), dpp<0xFF>(dz)};
    const float tr[4] = {dpp<0x00>(term), dpp<0x55>(term), dpp<0xAA>(term), dpp<0xFF>(term)};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      loss += tr[r];
      gb3 += dz3[r];
    }
    // ---- back to z2: dz2 = dz3 w3 silu'(z2); bias and w3 gradients
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      bf4_t dq;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        gw3[nt] = __builtin_fmaf(dz3[r], sl2[nt][r], gw3[nt]);
        const float dw = dz3[r] * w3[nt];
        gb2[nt] = __builtin_fmaf(dw, ds2[nt][r], gb2[nt]);
        dq[r] = (__bf16)(dw * ds2[nt][r]);
      }
      *reinterpret_cast<bf4_t*>(&DZT[(16 * nt + l16) * SH + 16 * w + 4 * lg]) = dq;
    }
    wave_sync();
    // ---- dh1[e][i] = sum_o dz2[e][o] W2[o][i] for the wavefront's events, then the input layer
    bf8_t dz2[2];   // event l16, outputs 32 kk + 8 lg + j
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) dz2[kk] = ld8t(&DZT[(32 * kk + 8 * lg) * SH + 16 * w], SH, l16);
    f4_t ur[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) ur[r] = s.U[16 * w + 4 * lg + r];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f4_t dh = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) dh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dz2[kk], w2t[nt][kk], dh, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float d1 = s.D1[(16 * w + 4 * lg + r) * SF + 16 * nt + l16];
        gb1[nt] = __builtin_fmaf(dh[r], d1, gb1[nt]);
        const float dz1 = dh[r] * d1;
#pragma unroll
        for (int k = 0; k < 4; ++k) gW1[nt][k] = __builtin_fmaf(dz1, ur[r][k], gW1[nt][k]);
      }
    }
    __syncthreads();
    // ---- dW2[o][i] += sum_e dz2[e][o] h1[e][i]: wavefront w owns the outputs 16 w ..
    bf8_t dv[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) dv[kk] = ld8(&DZT[(16 * w + l16) * SH + 32 * kk + 8 * lg]);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf8_t hv = ld8t(&H1[(32 * kk + 8 * lg) * SH + 16 * nt], SH, l16);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dv[kk], hv, acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) gW2[nt][r] += acc[r];
    }
  }
  // ---- block record.  dW2 entries have a unique owner lane; the others are summed over the rows of
  // the wavefront, then the four wavefronts in order.
  float* rec = a.partial + (int64_t)blockIdx.x * MLP_NV;
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) rec[P_W2 + (16 * w + 4 * lg + r) * 64 + 16 * nt + l16] = gW2[nt][r];
  auto put4 = [&](int g, const float* v) { s.red[w][64 * g + lane] = rows_sum4(v[0], v[1], v[2], v[3]); };
  put4(0, gb2);
  put4(1, gw3);
  put4(2, gb1);
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) put4(3 + nt, gW1[nt]);
  // b3 and loss: every lane of a row holds the row's sum
  gb3 += __shfl_xor(gb3, 32, 64);
  gb3 += __shfl_xor(gb3, 16, 64);
  loss += __shfl_xor(loss, 32, 64);
  loss += __shfl_xor(loss, 16, 64);
  if (lane == 0) {
    s.sc[w][0] = gb3;
    s.sc[w][1] = loss;
  }
  __syncthreads();
  for (int i = t; i < 28 * 16; i += 256) {
    const int j = i >> 4, f = i & 15;   // value j of unit f
    const int v = j < 4    ? P_B2 + 16 * j + f
                  : j < 8  ? P_W3 + 16 * (j - 4) + f
                  : j < 12 ? P_B1 + 16 * (j - 8) + f
                           : P_W1 + 4 * (16 * ((j - 12) >> 2) + f) + (j & 3);
    rec[v] = ((s.red[0][i] + s.red[1][i]) + s.red[2][i]) + s.red[3][i];
  }
  if (t < 2) rec[t == 0 ? P_B3 : 4545] = ((s.sc[0][t] + s.sc[1][t]) + s.sc[2][t]) + s.sc[3][t];
}

// Adam step of parameter i at the gradient g, on the FP32 master parameters; also the BF16 copies of
// the updated 64x64 layer in both layouts (as launch_mlp_bf16 writes them).
__device__ __forceinline__ void adam_step(const AdamArgs& a, int i, double g) {
  const float gi = (float)g;
  const float mi = __builtin_fmaf(a.b1, a.m[i], (1.0f - a.b1) * gi);
  const float vi = __builtin_fmaf(a.b2, a.v[i], (1.0f - a.b2) * gi * gi);
  a.m[i] = mi;
  a.v[i] = vi;
  const float pi = a.p[i] - a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
  a.p[i] = pi;
  const int k = i - nn::P_W2;
  if (k >= 0 && k < 4096) {
    const unsigned short h = nn::bf16(pi);
    a.w2h[k] = h;
    a.w2h[4096 + (k & 63) * 64 + (k >> 6)] = h;
  }
}

// Sum of block-major partials in FP64, fixed order: value v = scale * sum_b partial[b * nv + v].
// A workgroup takes 16 consecutive values and 16 chains of blocks: chain 4 s + q sums the blocks
// s + 4 q + 16 k (s, q = 0..3; of an incomplete last 16, chain 4 s takes the blocks s mod 4), eight
// reads in flight, and the chains are combined in a fixed order.  The values go to out, or, while
// training (ADAM), each parameter's update follows at once and the loss goes to loss: 7.0 us and a
// launch of 4.8 us for 256 records in one of 4.5 us (64 values a workgroup and four reads in
// flight before).
template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_reduce_kernel(const float* __restrict__ partial, int nb, int nv,
                                                         double scale, double* __restrict__ out, AdamArgs ad) {
  __shared__ double red[16][16];
  const int vl = threadIdx.x & 15, chain = threadIdx.x >> 4, sg = chain >> 2, q = chain & 3;
  const int v = blockIdx.x * 16 + vl;
  double x = 0.0;
  if (v < nv) {
    const int K = nb > sg + 12 ? (nb - sg - 13) / 16 + 1 : 0;   // whole sixteens of this s
    const float* p = partial + (int64_t)(sg + 4 * q) * nv + v;
    const int64_t step = (int64_t)16 * nv;
    int k = 0;
    for (; k + 8 <= K; k += 8) {
      float f[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = p[(k + i) * step];
#pragma unroll
      for (int i = 0; i < 8; ++i) x += (double)f[i];
    }
    for (; k < K; ++k) x += (double)p[k * step];
    if (q == 0)
      for (int b = sg + 16 * K; b < nb; b += 4) x += (double)partial[(int64_t)b * nv + v];
  }
  red[chain][vl] = x;
  __syncthreads();
  if (chain == 0 && v < nv) {
    double y[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      y[g] = (red[4 * g][vl] + red[4 * g + 1][vl]) + (red[4 * g + 2][vl] + red[4 * g + 3][vl]);
    const double r = scale * (((y[0] + y[1]) + y[2]) + y[3]);
    if constexpr (ADAM) {
      if (v == nv - 1) *ad.loss = r;
      else adam_step(ad, v, r);
    } else {
      out[v] = r;
    }
  }
}

// Probabilities of the network for n events.
//
// One wavefront takes 64 events at a time, with no LDS and no barrier: lane l evaluates the input
// layer for event l % 16 of a group of 16 and the features 32 kk + 8 (l / 16) + j, which is the
// layout in which the matrix cores read them as the A operand, and the weights of all layers stay
// in registers over the events of the wavefront.  Bound by the vector instructions of the 128
// sigmoids per event: 140 us of kernel, 153 us per call for 2e6 events.  (4% of that are the Newton steps
// of the first layer's reciprocals, without which one quotient in about 2^20 is not correctly rounded.  335 us
// per call with the layers passed through LDS by a workgroup per 64 events, a barrier between them, whole
// IEEE divisions and the double exponential of four events per 16 lanes evaluated in each of them.)
__global__ __launch_bounds__(256, 2) void mlp_eval_kernel(MlpArgs a) {
  using namespace nn;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  L1Weights w1;
  w1.load(a.params, lg);
  bf8_t w2[4][2];   // W2[16 nt + l16][32 kk + 8 lg + j]
  float b2[4], w3[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int o = 16 * nt + l16;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) w2[nt][kk] = to_bf8(a.params + P_W2 + 64 * o + 32 * kk + 8 * lg);
    b2[nt] = a.params[P_B2 + o];
    w3[nt] = (float)(__bf16)a.params[P_W3 + o];
  }
  const float b3 = a.params[P_B3];
  const int64_t tiles = (a.n + 63) / 64, stride = (int64_t)gridDim.x * 4;
  int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  double x[4] = {0.0, 0.0, 0.0, 0.0};   // observables of event 64 tile + lane
  auto fetch = [&](int64_t t) {
    const int64_t e = 64 * t + lane;
    if (e < a.n) {
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = a.obs[k][e];
    }
  };
  if (tile < tiles) fetch(tile);
  for (; tile < tiles; tile += stride) {
    float u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = input_map(a, k, x[k]);
    if (tile + stride < tiles) fetch(tile + stride);
    float z3 = 0.f;   // of event 16 (l16 / 4) + 4 lg + l16 % 4
#pragma unroll 1
    for (int mt = 0; mt < 4; ++mt) {
      float um[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) um[k] = __shfl(u[k], 16 * mt + l16, 64);
      bf8_t h[2];
#pragma unroll
      for (int c = 0; c < 16; ++c) h[c >> 3][c & 7] = (__bf16)silu(w1.z(c, um));
      float z3p[4] = {0.f, 0.f, 0.f, 0.f};   // events 4 lg + r of the group
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        f4_t z2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) z2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h[kk], w2[nt][kk], z2, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) z3p[r] += w3[nt] * silu(z2[r] + b2[nt]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) z3p[r] = row_sum(z3p[r]);
      const float lo = (l16 & 1) ? z3p[1] : z3p[0], hi = (l16 & 1) ? z3p[3] : z3p[2];
      const float v = (l16 & 2) ? hi : lo;
      z3 = (l16 >> 2) == mt ? v : z3;
    }
    const int64_t e = 64 * tile + 16 * (l16 >> 2) + 4 * lg + (l16 & 3);
    if (e < a.n) a.out[e] = 1.0 / (1.0 + exp(-(double)(z3 + b3)));
  }
}

// Accept labels: label_e = [u_e < eps_true(x_e)], u_e from Philox counter (e, 0, 3).
__device__ __forceinline__ void philox_c(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
    c[1] = (uint32_t)p1;
    c[3] = (uint32_t)p0;
    c[0] = n0;
    c[2] = n2;
  }
}

#pragma clang fp contract(off)
__global__ __launch_bounds__(256) void label_kernel(LabelArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  uint32_t c[4] = {(uint32_t)(a.e0 + e), (uint32_t)((uint64_t)(a.e0 + e) >> 32), 0u, 3u};
  philox_c(c, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  const double u = (double)(((uint64_t)(c[0] >> 5) << 26) | (uint64_t)(c[1] >> 6)) * (1.0 / 9007199254740992.0);
  const double x[4] = {2.0 * (a.obs[0][e] - a.lo) / (a.hi - a.lo) - 1.0, a.obs[1][e], a.obs[2][e],
                       a.obs[3][e] / 3.14159265358979323846};
  double eps = 0.9;
  for (int d = 0; d < 4; ++d) {
    const double v = x[d];
    const double P1 = v, P2 = 0.5 * (3.0 * v * v - 1.0), P3 = 0.5 * (5.0 * v * v * v - 3.0 * v);
    const double num = a.coef[3 * d] * P1 + a.coef[3 * d + 1] * P2 + a.coef[3 * d + 2] * P3;
    const double den = fabs(a.coef[3 * d]) + fabs(a.coef[3 * d + 1]) + fabs(a.coef[3 * d + 2]);
    const double tt = den > 0.0 ? num / den : 0.0;
    eps *= 1.0 - a.delta * (1.0 - tt) / 2.0;
  }
  if (a.eps_out) a.eps_out[e] = eps;
  a.label[e] = (u < eps) ? 1 : 0;
}
#pragma clang fp contract(on)

// Histogram counts: generated and accepted events per bin of a 4D grid (integer atomics,
// so the counts are exact and order-independent).
__global__ __launch_bounds__(256) void hist_count_kernel(HistCountArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  int64_t idx = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const double x = a.obs[d][e];
    int b = (int)floor((x - a.lo[d]) / (a.hi[d] - a.lo[d]) * a.nb[d]);
    b = b < 0 ? 0 : (b >= a.nb[d] ? a.nb[d] - 1 : b);
    idx = idx * a.nb[d] + b;
  }
  atomicAdd(&a.gen[idx], 1u);
  if (a.label[e]) atomicAdd(&a.acc[idx], 1u);
}

// BF16 copies of the 64x64 layer's weights: w2h[0, 4096) = W2[o][i], w2h[4096, 8192) = W2[o][i] at [i][o].
__global__ __launch_bounds__(256) void mlp_bf16_kernel(const float* __restrict__ params, unsigned short* __restrict__ w2h) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= 4096) return;
  const unsigned short h = nn::bf16(params[nn::P_W2 + i]);
  w2h[i] = h;
  w2h[4096 + (i & 63) * 64 + (i >> 6)] = h;
}

hipError_t launch_mlp_bf16(const float* params, unsigned short* w2h, hipStream_t st) {
  hipLaunchKernelGGL(mlp_bf16_kernel, dim3(16), dim3(256), 0, st, params, w2h);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpArgs& a, int nb, hipStream_t st) {
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(nb), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_mlp_reduce(const float* partial, int nb, int nv, double scale, double* out, const AdamArgs* ad,
                             hipStream_t st) {
  if (nv != MLP_NV) return hipErrorInvalidValue;   // the block records are MLP_NV values long
  const dim3 grid((nv + 15) / 16);
  if (ad) hipLaunchKernelGGL(mlp_reduce_kernel<true>, grid, dim3(256), 0, st, partial, nb, nv, scale, out, *ad);
  else hipLaunchKernelGGL(mlp_reduce_kernel<false>, grid, dim3(256), 0, st, partial, nb, nv, scale, out, AdamArgs{});
  return hipGetLastError();
}
hipError_t launch_mlp_eval(const MlpArgs& a, int nb, hipStream_t st) {
  hipLaunchKernelGGL(mlp_eval_kernel, dim3(nb), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_labels(const LabelArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(label_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_hist_count(const HistCountArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(hist_count_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace kpsi
