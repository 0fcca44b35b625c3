// Kernels of the warm-start perceptron: BF16 products on the matrix cores
// with FP32 accumulation and fused epilogues, the output-layer gradient and
// loss, and the Adam step.
//
// GELU in the erf form, g(a) = a Phi(a) = a (1 + erf(a / sqrt 2)) / 2, with
// g'(a) = Phi(a) + a phi(a); loss 1/(2B) sum ||y - t||^2, so the output
// gradient is (y - t) / B; Adam as published by Kingma and Ba.
//
// Products.  Every product of a layer is C[m][n] = sum_k A[m][k] B[n][k] with
// both operands stored k-contiguous in BF16 (row pitch a multiple of 8
// elements, so 8 consecutive k are one aligned 16-byte load):
//   forward   Z_l  = A_l W_l + b_l   A = A_l [B][fi],   B = W_l^T [fo][fi]
//   dW        dW_l = A_l^T dZ_l      A = A_l^T [fi][B], B = dZ_l^T [fo][B]
//   dA        dA   = dZ_l W_l^T      A = dZ_l [B][fo],  B = W_l [fi][fo]
// so the parameters keep two BF16 copies per layer (W_l and W_l^T) and the
// forward and backward epilogues write each activation and output gradient in
// both orientations.  The transposed activations carry one extra row of ones
// (row fi of A_l^T): the dW product over fi + 1 rows then also yields the
// bias gradient, the column sums of dZ_l, in the row that follows W_l in the
// parameter layout.
//
// Each 32 x 32 output tile is 2 x 2 blocks of v_mfma_f32_16x16x32_bf16 (A
// operand: lane holds row lane % 16, k group lane / 16 of 8 consecutive k;
// B operand: column lane % 16, the same k group; result register r of a
// lane: row 4 (lane / 16) + r, column lane % 16).  Operands come straight
// from global memory (each 16-byte fragment is used by two products), four k
// steps' fragments in flight.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "mlp_dev.h"

namespace rkkt {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kT = 256;
inline unsigned blocks(long long n) { return (unsigned)((n + kT - 1) / kT); }

// FP32 -> BF16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ float gelu(float a) { return 0.5f * a * (1.0f + erff(a * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float a) {
  return 0.5f * (1.0f + erff(a * 0.70710678118654752f)) + a * expf(-0.5f * a * a) * 0.39894228040143268f;
}

// sum over the kT threads of a workgroup in halving steps (thread 0 returns it)
__device__ __forceinline__ float block_sum(float v, float* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = kT / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}

// values k + 2 q, k + 2 q + 1 (q = 0..3) of a fragment that has nv <= 8 valid
// ones left, the others zero
__device__ __forceinline__ uint4 keep_first(uint4 v, int nv) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = 2 * q < nv ? 0x0000ffffu : 0u;
    const uint32_t hi = 2 * q + 1 < nv ? 0xffff0000u : 0u;
    w[q] &= lo | hi;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// A fragment as loaded (8 consecutive k of one row, from kk on) and as the
// products take it.  Loading neither masks nor converts, so nothing waits for
// a load before its k step comes up; a granule past K loads the row's last one
// and is masked then.
//   BF16 rows: the pitch is at least K rounded up to 8, so every granule that
//   starts below K lies inside the row.
struct FragBf16 {
  uint4 v;
  __device__ __forceinline__ void load(const uint16_t* row, int kk, int K) {
    v = *reinterpret_cast<const uint4*>(row + min(kk, (K + 7) / 8 * 8 - 8));
  }
  __device__ __forceinline__ uint4 get() const { return v; }
};

//   FP32 rows (the network's input, pitch K, aligned to 4 bytes): rounded to
//   BF16 when taken.
struct FragF32 {
  float v[8];
  __device__ __forceinline__ void load(const float* row, int kk, int K) {
    if (kk + 8 <= K) {
      __builtin_memcpy(v, row + kk, sizeof(v));
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = row[min(kk + j, K - 1)];
    }
  }
  __device__ __forceinline__ uint4 get() const {
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = (uint32_t)to_bf16(v[2 * q]) | ((uint32_t)to_bf16(v[2 * q + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
};

__device__ __forceinline__ f32x4 mfma(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                 c, 0, 0, 0);
}

// One workgroup of four wavefronts per 32 x 32 output tile: wavefront w
// takes the k steps w, w + 4, ... (so each wavefront's chain of dependent
// loads is a quarter of K long), the four partial tiles are added in LDS in
// wavefront order, and wavefront w then applies the epilogue to block
// (w / 2, w % 2) of the tile.
constexpr int kGemmWaves = 4;
constexpr int kGemmT = 64 * kGemmWaves;
constexpr int kAhead = 4;

template <int EPI, typename FragA>
__device__ void gemm_tile(const MlpGemm& g, int bx, int by, int nbx, f32x4 (*part)[4][64]) {
  constexpr bool kF32 = sizeof(FragA) != sizeof(FragBf16);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = by * 32, n0 = bx * 32;
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const std::conditional_t<kF32, float, uint16_t>* pa[2];
  const uint16_t* pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const long long m = min(m0 + 16 * i + r16, g.M - 1);
    if constexpr (kF32)
      pa[i] = g.x + m * g.lda;
    else
      pa[i] = g.A + m * g.lda;
    pb[i] = g.B + (long long)min(n0 + 16 * i + r16, g.N - 1) * g.ldb;
  }
  // the epilogue of this wavefront: block (i, j) = (w / 2, w % 2), the lane
  // holds rows mr .. mr + 3 of column nc; what it reads is loaded here
  constexpr bool kHalf = EPI == kMlpBiasGelu || EPI == kMlpGeluBack || EPI == kMlpOutGrad;
  const int mr = m0 + 16 * (w >> 1) + 4 * (lane >> 4);
  const int nc = n0 + 16 * (w & 1) + r16;
  float bias = 0.0f, zin[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (EPI == kMlpBiasGelu || EPI == kMlpBiasOut || EPI == kMlpOutGrad) bias = g.bias[min(nc, g.N - 1)];
  if (EPI == kMlpGeluBack || EPI == kMlpOutGrad) {
#pragma unroll
    for (int r = 0; r < 4; ++r) zin[r] = g.zin[(long long)min(mr + r, g.M - 1) * g.ldz + min(nc, g.N - 1)];
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int kStride = 32 * kGemmWaves;
  // kAhead k steps of every operand in flight: K up to 128 kAhead is one wait
  // (one step ahead: forward of 256 rows 21.3 us, gradients 49.3; four: 19.5
  // and 46.3)
  FragA fa[kAhead][2];
  FragBf16 fb[kAhead][2];
#pragma unroll
  for (int s = 0; s < kAhead; ++s)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (s == 0 || 32 * w + s * kStride < g.K) {
        fa[s][i].load(pa[i], 32 * w + s * kStride + kq, g.K);
        fb[s][i].load(pb[i], 32 * w + s * kStride + kq, g.K);
      }
  auto step = [&](int k0, int s) {
    uint4 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = fa[s][i].get();
      b[i] = fb[s][i].get();
    }
    if (k0 + 32 > g.K) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = keep_first(a[i], g.K - k0 - kq);
        b[i] = keep_first(b[i], g.K - k0 - kq);
      }
    }
    // the input's transposed copy (operand of dW_0): the tiles of a row of
    // tiles all pass over its k steps and share them out
    if (kF32 && g.xt && (k0 >> 5) % nbx == bx) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m = m0 + 16 * i + r16;
        const uint32_t v[4] = {a[i].x, a[i].y, a[i].z, a[i].w};
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (m < g.M && k0 + kq + j < g.K)
            g.xt[(long long)(k0 + kq + j) * g.ldt + m] = (uint16_t)(v[j >> 1] >> (16 * (j & 1)));
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a[i], b[j], acc[i][j]);
    const int kn = k0 + kAhead * kStride;
    if (kn < g.K) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[s][i].load(pa[i], kn + kq, g.K);
        fb[s][i].load(pb[i], kn + kq, g.K);
      }
    }
  };
  for (int kb = 32 * w; kb < g.K; kb += kAhead * kStride) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
      if (s == 0 || kb + s * kStride < g.K) step(kb + s * kStride, s);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) part[w][2 * i + j][lane] = acc[i][j];
  __syncthreads();
  f32x4 t = part[0][w][lane];
#pragma unroll
  for (int q = 1; q < kGemmWaves; ++q) t += part[q][w][lane];
  float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t h[4];
  // values first, then the stores: a wait for a load also waits for every
  // store before it
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (EPI == kMlpGeluBack) h[r] = to_bf16(t[r] * gelu_grad(zin[r]));  // dZ_{l-1} = dA g'(Z_{l-1})
    if (EPI == kMlpBiasGelu || EPI == kMlpBiasOut || EPI == kMlpOutGrad) t[r] += bias;
    if (EPI == kMlpBiasGelu) h[r] = to_bf16(gelu(t[r]));
    if (EPI == kMlpOutGrad) {  // dZ = (Y - T) / B
      const float e = t[r] - zin[r];
      h[r] = to_bf16(e * g.inv_b);
      d[r] = mr + r < g.M && nc < g.N ? e : 0.0f;
    }
  }
  if (nc < g.N) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mr + r;
      if (m < g.M) {
        if (EPI == kMlpStore || (EPI == kMlpBiasGelu && g.zout)) g.zout[(long long)m * g.ldz + nc] = t[r];
        if (EPI == kMlpBiasOut) g.y[(long long)m * g.N + nc] = t[r];
        if (kHalf) g.hout[(long long)m * g.ldh + nc] = (uint16_t)h[r];
      }
    }
    if (kHalf && g.tout) {
      uint16_t* tp = g.tout + (long long)nc * g.ldt + mr;
      if (mr + 3 < g.M) {
        *reinterpret_cast<uint2*>(tp) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
          if (mr + r < g.M) tp[r] = (uint16_t)h[r];
      }
    }
  }
  if (EPI == kMlpOutGrad) {
    // the tile's sum of (Y - T)^2: a thread takes column tx's rows ty, ty + 8,
    // ty + 16, ty + 24 (zero outside the batch), then halving steps
    float* red = reinterpret_cast<float*>(part);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(mr - m0 + r) * 33 + nc - n0] = d[r];
    __syncthreads();
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    float sq = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) sq = fmaf(red[(ty + 8 * q) * 33 + tx], red[(ty + 8 * q) * 33 + tx], sq);
    __syncthreads();
    const float sum = block_sum(sq, red);
    if (threadIdx.x == 0) g.lpart[by * nbx + bx] = sum;
  }
}

template <int EPI, typename FragA>
__global__ __launch_bounds__(kGemmT) void k_gemm(MlpGemm g) {
  __shared__ f32x4 part[kGemmWaves][4][64];
  gemm_tile<EPI, FragA>(g, blockIdx.x, blockIdx.y, gridDim.x, part);
}

// Everything of the backward pass that follows from dZ_l, in one launch: first
// the tiles of dZ_{l-1} (the next launch waits for them), then those of
// [dW_l; db_l], then, with a loss, one workgroup that adds its partial sums.
// The gradients of 256 rows are bound by their launches (15 of them, 68.5 us):
// with these merged, the input converted where it is read, the output gradient
// in the last layer's epilogue and the gradients written to the caller's array
// it is 8, 46.3 us.
__global__ __launch_bounds__(kGemmT) void k_back(MlpGemm ga, int na, int nax, MlpGemm gw, int nw, int nwx,
                                                 const float* __restrict__ lpart, int np, float inv_b,
                                                 float* __restrict__ loss) {
  __shared__ f32x4 part[kGemmWaves][4][64];
  const int b = blockIdx.x;
  if (b < na) {
    gemm_tile<kMlpGeluBack, FragBf16>(ga, b % nax, b / nax, nax, part);
  } else if (b < na + nw) {
    gemm_tile<kMlpStore, FragBf16>(gw, (b - na) % nwx, (b - na) / nwx, nwx, part);
  } else {
    // loss = 0.5 inv_b sum of the partials, in a fixed order
    float sum = 0.0f;
    for (int i = threadIdx.x; i < np; i += kGemmT) sum += lpart[i];
    sum = block_sum(sum, reinterpret_cast<float*>(part));
    if (threadIdx.x == 0) *loss = 0.5f * inv_b * sum;
  }
}

// x [rows][cols] FP32 -> BF16 row-major (pitch ldh) and transposed (pitch ldt)
__global__ void k_input_bf16(const float* __restrict__ x, int rows, int cols, uint16_t* __restrict__ h, int ldh,
                             uint16_t* __restrict__ t, int ldt) {
  const long long i = (long long)blockIdx.x * kT + threadIdx.x;
  if (i >= (long long)rows * cols) return;
  const int r = (int)(i / cols), c = (int)(i % cols);
  const uint16_t v = to_bf16(x[i]);
  h[(long long)r * ldh + c] = v;
  if (t) t[(long long)c * ldt + r] = v;
}

// BF16 copies of parameter i: W_l entries into W_l [fi][pitch fo] and
// W_l^T [fo][pitch fi], biases nowhere (they stay FP32)
__device__ __forceinline__ void store_copies(const MlpLayers& L, long long i, float p, uint16_t* __restrict__ wb,
                                             uint16_t* __restrict__ wt) {
  for (int l = 0; l < L.n; ++l) {
    const long long rel = i - L.woff[l];
    const long long nw = (long long)L.fi[l] * L.fo[l];
    if (rel >= 0 && rel < nw) {
      const int r = (int)(rel / L.fo[l]), c = (int)(rel % L.fo[l]);
      const uint16_t v = to_bf16(p);
      wb[L.wb_off[l] + (long long)r * L.fo_p[l] + c] = v;
      wt[L.wt_off[l] + (long long)c * L.fi_p[l] + r] = v;
      return;
    }
  }
}

__global__ void k_param_copies(const float* __restrict__ p, long long n, MlpLayers L, uint16_t* __restrict__ wb,
                               uint16_t* __restrict__ wt) {
  const long long i = (long long)blockIdx.x * kT + threadIdx.x;
  if (i < n) store_copies(L, i, p[i], wb, wt);
}

// Adam on the master parameters, then their BF16 copies
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long long n, float lr, float b1, float b2, float c1, float c2,
                       float eps, MlpLayers L, uint16_t* __restrict__ wb, uint16_t* __restrict__ wt) {
  const long long i = (long long)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  store_copies(L, i, pi, wb, wt);
}

__global__ void k_fill_bf16(uint16_t* __restrict__ d, long long n, uint16_t v) {
  const long long i = (long long)blockIdx.x * kT + threadIdx.x;
  if (i < n) d[i] = v;
}

}  // namespace

void mlp_gemm(int epi, const MlpGemm& g, hipStream_t st) {
  const dim3 grid((unsigned)((g.N + 31) / 32), (unsigned)((g.M + 31) / 32));
  switch (epi) {
    case kMlpBiasGelu:
      if (g.x)
        k_gemm<kMlpBiasGelu, FragF32><<<grid, kGemmT, 0, st>>>(g);
      else
        k_gemm<kMlpBiasGelu, FragBf16><<<grid, kGemmT, 0, st>>>(g);
      break;
    case kMlpBiasOut: k_gemm<kMlpBiasOut, FragBf16><<<grid, kGemmT, 0, st>>>(g); break;
    default: k_gemm<kMlpOutGrad, FragBf16><<<grid, kGemmT, 0, st>>>(g); break;
  }
}

void mlp_back(const MlpGemm* ga, const MlpGemm& gw, const float* lpart, int np, float inv_b, float* loss,
              hipStream_t st) {
  const int nax = ga ? (ga->N + 31) / 32 : 1, na = ga ? nax * ((ga->M + 31) / 32) : 0;
  const int nwx = (gw.N + 31) / 32, nw = nwx * ((gw.M + 31) / 32);
  k_back<<<na + nw + (loss ? 1 : 0), kGemmT, 0, st>>>(ga ? *ga : MlpGemm{}, na, nax, gw, nw, nwx, lpart, np,
                                                      inv_b, loss);
}

void mlp_input_bf16(const float* x, int rows, int cols, uint16_t* h, int ldh, uint16_t* t, int ldt,
                    hipStream_t st) {
  k_input_bf16<<<blocks((long long)rows * cols), kT, 0, st>>>(x, rows, cols, h, ldh, t, ldt);
}

int mlp_out_grad_tiles(int rows, int cols) { return ((rows + 31) / 32) * ((cols + 31) / 32); }

void mlp_param_copies(const float* p, long long n, const MlpLayers& L, uint16_t* wb, uint16_t* wt,
                      hipStream_t st) {
  k_param_copies<<<blocks(n), kT, 0, st>>>(p, n, L, wb, wt);
}

void mlp_adam(float* p, const float* g, float* m, float* v, long long n, float lr, int t, const MlpLayers& L,
              uint16_t* wb, uint16_t* wt, hipStream_t st) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  k_adam<<<blocks(n), kT, 0, st>>>(p, g, m, v, n, lr, b1, b2, c1, c2, 1e-8f, L, wb, wt);
}

void mlp_fill_bf16(uint16_t* d, long long n, float v, hipStream_t st) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  k_fill_bf16<<<blocks(n), kT, 0, st>>>(d, n, (uint16_t)(u >> 16));
}

}  // namespace rkkt
