// fp32 build kernels for calls too small to fill the chip with 64 x 64 tiles (see small_f32.hpp): there a
// handful of blocks walks the reduction one K tile after another, each waiting out a global load, an LDS
// write and a barrier, on 32x32x2 MFMAs. Here an output tile is 16 tokens x 16 columns, a wave each, and its
// fragments come straight from global memory (float4 per lane), the next 128 of K ahead of the products of
// these.
// Every sum is the 64 x 64-tile kernels' to the bit, so which kernel a launch takes shows in no output: the
// rule that chooses counts a launch's tiles, and with them its tokens and layers. MFMAs add their K steps as a
// chain of fused multiply-adds; mfma_k16 walks a 16-deep group as k = 0, 8, 1, 9, .. 7, 15, and so do the
// four 16x16x4 products of dot16. (With the reduction split over four waves the chain was a quarter as
// long, but the bits depended on the launch.) Bound by the loads' latency and that chain: K/V of 64 tokens, 4
// layers of d = 256, 512 columns 14.2 -> 7.7 us, a launch of about 4 included; d = 4096 125 -> 76.
// The weights are the MFMA's A operand, so a lane ends with one token and four consecutive columns.
#include "small_f32.hpp"

#include "dv_device.hpp"

namespace dv {

namespace {

constexpr int BATCH = 8;  // 16-deep groups in flight ahead of the MFMAs

// A lane's share of a 16-deep group, k = 8 (q % 2) + 4 (q / 2) .. + 3 for q = lane / 16, as the operands of
// the four products: product i takes k = 8 (q % 2) + 2 i + q / 2, in the order of q. Lanes q and q + 2
// exchange halves.
__device__ __forceinline__ f32x4 chain_order(f32x4 v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2]), __float_as_uint(v[3]), false, false);
  return f32x4{__uint_as_float(a[0]), __uint_as_float(b[0]), __uint_as_float(a[1]), __uint_as_float(b[1])};
}

struct Batch {
  f32x4 w[BATCH], x[BATCH];
};

// sum of W[n][k] X[m][k] over k < K (a multiple of 16); wrow and xrow are this lane's rows.
__device__ __forceinline__ f32x4 dot16(const float* wrow, const float* xrow, int K) {
  const int q = (threadIdx.x & 63) >> 4, ko = 8 * (q & 1) + 4 * (q >> 1);
  f32x4 acc = {};
  auto load = [&](Batch& t, int k) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int kk = min(k + 16 * u, K - 16) + ko;  // (past the end: the last group again, not multiplied)
      t.w[u] = *(const f32x4*)(wrow + kk);
      t.x[u] = *(const f32x4*)(xrow + kk);
    }
  };
  auto group = [&](const Batch& t, int u) {
    const f32x4 w = chain_order(t.w[u]), x = chain_order(t.x[u]);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], x[r], acc, 0, 0, 0);
  };
  auto mma = [&](const Batch& t, int k) {
    if (k + 16 * BATCH <= K) {
#pragma unroll
      for (int u = 0; u < BATCH; ++u) group(t, u);
    } else {
#pragma unroll
      for (int u = 0; u < BATCH; ++u)
        if (k + 16 * u < K) group(t, u);
    }
  };
  constexpr int S = 16 * BATCH;
  Batch b0, b1;
  if (K <= S / 2) {  // a short reduction (r): only its own groups
#pragma unroll
    for (int u = 0; u < BATCH / 2; ++u)
      if (16 * u < K) {
        b0.w[u] = *(const f32x4*)(wrow + 16 * u + ko);
        b0.x[u] = *(const f32x4*)(xrow + 16 * u + ko);
      }
    mma(b0, 0);
    return acc;
  }
  // The loads are unconditional, so that the waits for one batch leave the next in flight.
  load(b0, 0);
  for (int k = 0; k < K; k += 2 * S) {
    load(b1, k + S);
    mma(b0, k);
    load(b0, k + 2 * S);
    mma(b1, k + S);
  }
  return acc;
}

// One wave a block: 16 tokens x 16 of the L * r columns.
template <int ACT>
__global__ __launch_bounds__(WAVE) void k_small_down(const float* __restrict__ E, const float* __restrict__ Dw,
                                                     float* __restrict__ Z, int T, int d, int r) {
  const int lane = threadIdx.x;
  const int n0 = blockIdx.x * 16, m = blockIdx.y * 16 + (lane & 15);
  const f32x4 acc = dot16(Dw + (int64_t)(n0 + (lane & 15)) * d, E + (int64_t)min(m, T - 1) * d, d);
  if (m >= T) return;
  const int n = n0 + 4 * (lane >> 4), l = n / r;  // r % 16 == 0: the tile lies in one layer
  f32x4 z;
#pragma unroll
  for (int u = 0; u < 4; ++u) z[u] = ACT == 0 ? silu(acc[u]) : gelu(acc[u]);
  *(f32x4*)(Z + ((int64_t)l * T + m) * r + (n - l * r)) = z;
}

// Four waves, 16 columns each: 64 columns of M * gamma for 16 tokens of one layer, and their sums of squares.
constexpr int UP_W = 4;
__global__ __launch_bounds__(UP_W * WAVE) void k_small_up(const float* __restrict__ E, const float* __restrict__ Z,
                                                          const float* __restrict__ Uw, const float* __restrict__ gamma,
                                                          float* __restrict__ Mg, float* __restrict__ ssq, int T, int d,
                                                          int r, int l0) {
  __shared__ float red[UP_W][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lz = blockIdx.z, l = l0 + lz;
  const int n0 = blockIdx.x * 64 + wave * 16, m = blockIdx.y * 16 + (lane & 15), mc = min(m, T - 1);
  const int n = n0 + 4 * (lane >> 4);
  const f32x4 e = *(const f32x4*)(E + (int64_t)mc * d + n), g = *(const f32x4*)(gamma + (int64_t)l * d + n);
  const f32x4 acc = dot16(Uw + ((int64_t)l * d + n0 + (lane & 15)) * r, Z + ((int64_t)l * T + mc) * r, r);
  f32x4 o;
  float ss;
  {
    // The squares are rounded, then added in pairs of columns 1, 2, 4, 8, 16 and 32 apart, as the tile
    // kernel's lanes do: no fused multiply-add.
#pragma clang fp contract(off)
    float sq[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float x = acc[u] + e[u];
      sq[u] = x * x;
      o[u] = x * g[u];
    }
    ss = (sq[0] + sq[1]) + (sq[2] + sq[3]);
  }
  if (m < T) *(f32x4*)(Mg + ((int64_t)lz * T + m) * d + n) = o;
  ss += shfl_xor(ss, 16);
  ss += shfl_xor(ss, 32);
  if (lane < 16) red[wave][lane] = ss;
  __syncthreads();
  if (wave == 0 && lane < 16 && m < T)
    ssq[((int64_t)lz * gridDim.x + blockIdx.x) * T + m] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// One wave a block: 16 tokens x 16 of the 2 Hkv hd columns of one layer.
__global__ __launch_bounds__(WAVE) void k_small_kv(const float* __restrict__ Mg, const float* __restrict__ ssq,
                                                   const float* __restrict__ Wk, const float* __restrict__ Wv,
                                                   float* __restrict__ Kv, float* __restrict__ Vv, int B_, int Nv,
                                                   int d, int Hkv, int hd, int l0, int np, float eps) {
  const int lane = threadIdx.x;
  const int T = B_ * Nv, kv = Hkv * hd;
  const int lz = blockIdx.z, l = l0 + lz;
  const int n0 = blockIdx.x * 16, m = blockIdx.y * 16 + (lane & 15), mc = min(m, T - 1);
  const bool is_k = n0 < kv;  // kv % 64 == 0: the tile lies in one head of K or of V
  const int o0 = is_k ? n0 : n0 - kv;
  const float* W = (is_k ? Wk : Wv) + ((int64_t)l * kv + o0 + (lane & 15)) * d;
  // Row scale from the partial sums of squares, added in order; the first are requested ahead of the products.
  const float* part = ssq + (int64_t)lz * np * T + mc;
  constexpr int PRE = 16;
  float p0[PRE];
#pragma unroll
  for (int p = 0; p < PRE; ++p) p0[p] = p < np ? part[(int64_t)p * T] : 0.f;
  const f32x4 acc = dot16(W, Mg + ((int64_t)lz * T + mc) * d, d);
  float s = 0.f;
#pragma unroll
  for (int p = 0; p < PRE; ++p) s += p0[p];
#pragma unroll 8
  for (int p = PRE; p < np; ++p) s += part[(int64_t)p * T];
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
    k_small_down<0><<<grid, WAVE, 0, s>>>(E, Dw, Z, T, d, r);
  else
    k_small_down<1><<<grid, WAVE, 0, s>>>(E, Dw, Z, T, d, r);
  return hipGetLastError();
}

hipError_t launch_small_up(const float* E, const float* Z, const float* Uw, const float* gamma, float* Mg, float* ssq,
                           int T, int d, int r, int l0, int nl, hipStream_t s) {
  k_small_up<<<dim3(d / 64, blocks16(T), nl), UP_W * WAVE, 0, s>>>(E, Z, Uw, gamma, Mg, ssq, T, d, r, l0);
  return hipGetLastError();
}

hipError_t launch_small_kv(const float* Mg, const float* ssq, const float* Wk, const float* Wv, float* Kv, float* Vv,
                           int B_, int Nv, int d, int Hkv, int hd, int l0, int nl, int np, float eps, hipStream_t s) {
  k_small_kv<<<dim3(2 * Hkv * hd / 16, blocks16((int64_t)B_ * Nv), nl), WAVE, 0, s>>>(Mg, ssq, Wk, Wv, Kv, Vv, B_,
                                                                                          Nv, d, Hkv, hd, l0, np, eps);
  return hipGetLastError();
}

}  // namespace dv
