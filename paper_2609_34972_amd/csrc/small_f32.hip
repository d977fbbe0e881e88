// fp32 build kernels for calls too small to fill the chip with 64 x 64 tiles (see small_f32.hpp): there a
// handful of blocks walks the reduction one K tile after another, each waiting out a global load, an LDS
// write and a barrier. Here an output tile is 16 tokens x 16 columns, fragments come straight from global
// memory (float4 per lane: K step r of a 16-deep group takes k = 4 (lane / 16) + r, for both operands), and
// the four waves of a block split the reduction, or take four column tiles where it is short (r).
// The weights are the MFMA's A operand, so a lane ends with one token and four consecutive columns.
#include "small_f32.hpp"

#include "dv_device.hpp"

namespace dv {

namespace {

constexpr int NW = 4;      // waves per block
constexpr int BATCH = 8;   // 16-deep groups loaded before their MFMAs

// acc += W[n][k] X[m][k] over k0 <= k < k1 (multiples of 16); wrow and xrow are this lane's rows.
__device__ __forceinline__ f32x4 dot16(const float* wrow, const float* xrow, int k0, int k1, f32x4 acc) {
  const int ko = 4 * ((threadIdx.x & 63) >> 4);
  for (int k = k0; k < k1; k += 16 * BATCH) {
    f32x4 w[BATCH], x[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int kk = k + 16 * u;
      w[u] = kk < k1 ? *(const f32x4*)(wrow + kk + ko) : f32x4{};
      x[u] = kk < k1 ? *(const f32x4*)(xrow + kk + ko) : f32x4{};
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][r], x[u][r], acc, 0, 0, 0);
  }
  return acc;
}

// This wave's quarter of a d-long reduction.
__device__ __forceinline__ void quarter(int d, int wave, int& k0, int& k1) {
  const int q = (d / 16 + NW - 1) / NW * 16;
  k0 = min(wave * q, d);
  k1 = min(k0 + q, d);
}

// The sum of the waves' tiles, in wave 0 (the others return false).
__device__ __forceinline__ bool sum_waves(f32x4& acc, f32x4 (&red)[NW][WAVE], int wave, int lane) {
  red[wave][lane] = acc;
  __syncthreads();
  if (wave != 0) return false;
#pragma unroll
  for (int w = 1; w < NW; ++w) acc += red[w][lane];
  return true;
}

template <int ACT>
__global__ __launch_bounds__(NW * WAVE) void k_small_down(const float* __restrict__ E, const float* __restrict__ Dw,
                                                          float* __restrict__ Z, int T, int d, int r) {
  __shared__ f32x4 red[NW][WAVE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.x * 16, m = blockIdx.y * 16 + (lane & 15);
  int k0, k1;
  quarter(d, wave, k0, k1);
  f32x4 acc = dot16(Dw + (int64_t)(n0 + (lane & 15)) * d, E + (int64_t)min(m, T - 1) * d, k0, k1, f32x4{});
  if (!sum_waves(acc, red, wave, lane) || m >= T) return;
  const int n = n0 + 4 * (lane >> 4), l = n / r;  // r % 16 == 0: the tile lies in one layer
  f32x4 z;
#pragma unroll
  for (int u = 0; u < 4; ++u) z[u] = ACT == 0 ? silu(acc[u]) : gelu(acc[u]);
  *(f32x4*)(Z + ((int64_t)l * T + m) * r + (n - l * r)) = z;
}

// Four waves, 16 columns each: 64 columns of M * gamma for 16 tokens of one layer, and their sums of squares.
__global__ __launch_bounds__(NW * WAVE) void k_small_up(const float* __restrict__ E, const float* __restrict__ Z,
                                                        const float* __restrict__ Uw, const float* __restrict__ gamma,
                                                        float* __restrict__ Mg, float* __restrict__ ssq, int T, int d,
                                                        int r, int l0) {
  __shared__ float red[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lz = blockIdx.z, l = l0 + lz;
  const int n0 = blockIdx.x * 64 + wave * 16, m = blockIdx.y * 16 + (lane & 15), mc = min(m, T - 1);
  const int n = n0 + 4 * (lane >> 4);
  const f32x4 e = *(const f32x4*)(E + (int64_t)mc * d + n), g = *(const f32x4*)(gamma + (int64_t)l * d + n);
  const f32x4 acc = dot16(Uw + ((int64_t)l * d + n0 + (lane & 15)) * r, Z + ((int64_t)l * T + mc) * r, 0, r, f32x4{});
  f32x4 o;
  float ss = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float x = acc[u] + e[u];
    ss += x * x;
    o[u] = x * g[u];
  }
  if (m < T) *(f32x4*)(Mg + ((int64_t)lz * T + m) * d + n) = o;
  ss += shfl_xor(ss, 16);
  ss += shfl_xor(ss, 32);
  if (lane < 16) red[wave][lane] = ss;
  __syncthreads();
  if (wave == 0 && lane < 16 && m < T)
    ssq[((int64_t)lz * gridDim.x + blockIdx.x) * T + m] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

__global__ __launch_bounds__(NW * WAVE) void k_small_kv(const float* __restrict__ Mg, const float* __restrict__ ssq,
                                                        const float* __restrict__ Wk, const float* __restrict__ Wv,
                                                        float* __restrict__ Kv, float* __restrict__ Vv, int B_, int Nv,
                                                        int d, int Hkv, int hd, int l0, int np, float eps) {
  __shared__ f32x4 red[NW][WAVE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int T = B_ * Nv, kv = Hkv * hd;
  const int lz = blockIdx.z, l = l0 + lz;
  const int n0 = blockIdx.x * 16, m = blockIdx.y * 16 + (lane & 15), mc = min(m, T - 1);
  const bool is_k = n0 < kv;  // kv % 64 == 0: the tile lies in one head of K or of V
  const int o0 = is_k ? n0 : n0 - kv;
  const float* W = (is_k ? Wk : Wv) + ((int64_t)l * kv + o0 + (lane & 15)) * d;
  float s = 0.f;  // row scale: the partial sums of squares, lane group q taking q, q + 4, ...
  if (wave == 0)
    for (int p = lane >> 4; p < np; p += 4) s += ssq[((int64_t)lz * np + p) * T + mc];
  int k0, k1;
  quarter(d, wave, k0, k1);
  f32x4 acc = dot16(W, Mg + ((int64_t)lz * T + mc) * d, k0, k1, f32x4{});
  if (!sum_waves(acc, red, wave, lane)) return;
  s += shfl_xor(s, 16);
  s += shfl_xor(s, 32);
  if (m >= T) return;
  const int o = o0 + 4 * (lane >> 4), h = o / hd, c = o - h * hd, b = m / Nv, i = m - b * Nv;
  *(f32x4*)((is_k ? Kv : Vv) + ((((int64_t)l * B_ + b) * Hkv + h) * Nv + i) * hd + c) =
      acc * rsqrtf(s / (float)d + eps);
}

inline unsigned blocks16(int64_t n) { return (unsigned)((n + 15) / 16); }

}  // namespace

hipError_t launch_small_down(const float* E, const float* Dw, float* Z, int T, int d, int L, int r, int act,
                             hipStream_t s) {
  const dim3 grid(blocks16((int64_t)L * r), blocks16(T));
  if (act == 0)
    k_small_down<0><<<grid, NW * WAVE, 0, s>>>(E, Dw, Z, T, d, r);
  else
    k_small_down<1><<<grid, NW * WAVE, 0, s>>>(E, Dw, Z, T, d, r);
  return hipGetLastError();
}

hipError_t launch_small_up(const float* E, const float* Z, const float* Uw, const float* gamma, float* Mg, float* ssq,
                           int T, int d, int r, int l0, int nl, hipStream_t s) {
  k_small_up<<<dim3(d / 64, blocks16(T), nl), NW * WAVE, 0, s>>>(E, Z, Uw, gamma, Mg, ssq, T, d, r, l0);
  return hipGetLastError();
}

hipError_t launch_small_kv(const float* Mg, const float* ssq, const float* Wk, const float* Wv, float* Kv, float* Vv,
                           int B_, int Nv, int d, int Hkv, int hd, int l0, int nl, int np, float eps, hipStream_t s) {
  k_small_kv<<<dim3(2 * Hkv * hd / 16, blocks16((int64_t)B_ * Nv), nl), NW * WAVE, 0, s>>>(Mg, ssq, Wk, Wv, Kv, Vv, B_,
                                                                                          Nv, d, Hkv, hd, l0, np, eps);
  return hipGetLastError();
}

}  // namespace dv
