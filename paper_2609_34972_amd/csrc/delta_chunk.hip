// bf16 kernels of the gated delta-rule write (see delta_rule.hip for the recurrence and its chunked
// form). With D = diag(gamma_C / gamma), T = (I + A)^-1 and R = D T diag(beta), a chunk is
//     X = V - diag(gamma) (K S_0),   U = R X,   S_C = gamma_C S_0 + K^T U,
// so all that has to be prepared per chunk and value head is R (64 x 64, lower triangular) and
// gamma: K and V enter the products as they are, and the keys that several value heads share are
// read where they lie. (The fp32 kernels store W = T diag(beta gamma) K, diag(gamma_C / gamma) K and
// T diag(beta) V instead: 48 KiB a chunk in bf16 against 6.25 KiB here.)
//
//   k_gdr_tri    R and gamma of every chunk and value head, one wave each.
//   k_gdr_scan   the chunks of a segment in order; a wave keeps 32 columns of the fp32 state.
//   k_gdr_join   S <- Phi_g S + Psi_g over the segments of a long sequence.
//
// Row order. Item 8 q + e of lane half h of a 32 x 32 accumulator is row 16 q + 8 (e / 4) + 4 h + e % 4.
// The rows of an A operand may be any rows of the matrix, so lane x % 32 = x takes matrix row pi(x),
// pi swapping bits 2 and 3 (an involution): then item 8 q + e of half h is matrix row 16 q + 8 h + e,
// and the items of an accumulator, rounded to bf16, are the B fragment of the next product's K step q
// in natural order (lane half h: k = 16 q + 8 h .. + 7), which the A operands meet with plain
// 16-byte reads of their rows.
#include "delta_rule.hpp"

#include <cfloat>

#include "dv_device.hpp"
#include "gemm_pipe.hpp"

namespace dv {

namespace gdc {
constexpr int C = 64;
// Chunk record: R rows 0..31, columns 0..31 (64-byte rows), then rows 32..63 (128-byte rows), then
// gamma (64 floats). 16-byte pieces of a row are XOR-swizzled by the row, as they lie in LDS.
constexpr int R1 = 2048, GAM = 6144, REC = 6400;
constexpr int REC_INS = 7, REC_LDS = REC_INS * 1024;
static_assert(REC == kGdrRecBytes, "record size");
__device__ __forceinline__ int pi(int x) { return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1); }
__device__ __forceinline__ int r0_off(int row, int c) { return row * 64 + ((c ^ ((row >> 2) & 3)) << 4); }
// Keys of the 16-byte pieces of a K, V, Phi or R row in LDS: bijections of the row's low bits, so
// that 16 rows read at one piece, and the 4 rows x 4 pieces that a lane half of a transpose read
// takes, fall in distinct bank groups.
template <int D>
__device__ __forceinline__ int row_key(int row) {
  static_assert(D == 64 || D == 128, "rows of 128 or 256 bytes");
  return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : ((row & 2) << 1) | ((row >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int row_off(int row, int c) { return row * D * 2 + ((c ^ row_key<D>(row)) << 4); }
}  // namespace gdc

__device__ __forceinline__ bf16x8 lds_b8(const unsigned char* p) { return __builtin_bit_cast(bf16x8, *(const u32x4*)p); }

// ------------------------------------------------------------------ R and gamma

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 d) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d, 0, 0, 0); }

// d += X Y for 16 x 16 fp32 blocks, X at x in LDS (pitch MP). K step r takes k = 4 (lane / 16) + r, so
// X comes as one 16-byte read per lane and an accumulator block is Y as it stands (item r).
template <int MP>
__device__ __forceinline__ f32x4 mul16(const float* x, f32x4 y, f32x4 d) {
  const int lane = threadIdx.x & 63;
  const f32x4 a = *(const f32x4*)(x + (lane & 15) * MP + 4 * (lane >> 4));
#pragma unroll
  for (int r = 0; r < 4; ++r) d = mfma4(a[r], y[r], d);
  return d;
}
// A 16 x 16 block of LDS as the Y operand of mul16, and back.
template <int MP>
__device__ __forceinline__ f32x4 get16(const float* y) {
  const int lane = threadIdx.x & 63;
  f32x4 v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = y[(4 * (lane >> 4) + r) * MP + (lane & 15)];
  return v;
}
template <int MP>
__device__ __forceinline__ void put16(float* y, f32x4 v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) y[(4 * (lane >> 4) + r) * MP + (lane & 15)] = v[r];
}

// One wave per (chunk, value head): K K^T on MFMA, A and T = (I + A)^-1 in fp32 in LDS (the diagonal
// 16 x 16 blocks by forward substitution, a column per lane, the others on fp32 MFMA), R in bf16.
// The waves of a block share nothing, so the ten that LDS lets on a CU run at different phases. Blocks
// are dealt so that each XCD takes consecutive (chunk, head) pairs and the heads of a key head find
// their K in its L2. Bound by latency and the loads: 42 us for 8192 chunk-heads of the 16384-token video,
// of which 22 for an empty body with the loads, 3 A, 5 the diagonal blocks, 7 the other blocks, 8 R
// (the kernel that also formed W, Uv and the scaled K took 185 us).
// Orders this wave's LDS writes before its later reads (its lanes exchange data through LDS).
__device__ __forceinline__ void wave_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

constexpr int TRI_W = 2;  // waves per block

template <int DK>
__global__ __launch_bounds__(64 * TRI_W) void k_gdr_tri(const bf16* __restrict__ k, const float* __restrict__ alpha,
                                                const float* __restrict__ beta, int Hk, int Hv, int N, int NC,
                                                int n, unsigned char* __restrict__ recs) {
  using namespace gdc;
  constexpr int NKS = DK / 16;
  constexpr int P0 = 36, P1 = 68;            // pitches of rows 0..31 (columns 0..31) and 32..63
  constexpr int MB = 32 * P0, WB = MB + 32 * P1 + 2 * C;
  __shared__ __align__(16) float smem[TRI_W * WB];
  const int lane = threadIdx.x & 63, wave = wave_index();
  float *M0 = smem + wave * WB, *M1 = M0 + MB, *g = M1 + 32 * P1, *bet = g + C;
  const int per = gridDim.x / 8, full = per * 8;
  const int id = blockIdx.x, q = (id < full ? (id % 8) * per + id / 8 : id) * TRI_W + wave;
  if (q >= n) return;  // waves share nothing: no block barrier follows
  const int hv = q % Hv, bc = q / Hv, c = bc % NC, b = bc / NC;
  const int hk = hv / (Hv / Hk);
  const int64_t t0 = (int64_t)c * C, seq = (int64_t)b * Hv + hv;
  const int nval = (int)min((int64_t)C, (int64_t)N - t0);
  const int h = lane >> 5, rr = lane & 31;
  const auto rk = buffer_rsrc(k + (((int64_t)b * Hk + hk) * N + t0) * DK, nval * DK * 2);

  float la = 0.f, be = 0.f;
  if (lane < nval) {
    la = alpha[seq * N + t0 + lane];
    be = beta[seq * N + t0 + lane];
  }
  bf16x8 f[2][NKS];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      f[t][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, rr * DK * 2 + h * 16, t * 32 * DK * 2 + ks * 32, 0));
  // g = prefix sum of log2 alpha (tokens past N: alpha = 1, beta = 0, k = 0)
  float x = lane < nval ? __builtin_amdgcn_logf(fmaxf(la, FLT_MIN)) : 0.f;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  const float gt = x, gC = __shfl(x, 63, WAVE);
  g[lane] = gt;
  bet[lane] = be;
  wave_sync();
  // A[t][s] = beta_t 2^(g_t - g_s) k_t.k_s below the diagonal, 0 on and above it (lower tiles)
#pragma unroll
  for (int tile = 0; tile < 3; ++tile) {
    const int ti = tile == 0 ? 0 : 1, si = tile == 2 ? 1 : 0;
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) mfma_k16(acc, f[ti][ks], f[si][ks]);
    const int s = si * 32 + rr;
    const float gs = g[s];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const int tb = ti * 32 + i4 * 8 + h * 4;
      const f32x4 g4 = *(const f32x4*)(g + tb), b4 = *(const f32x4*)(bet + tb);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = b4[e] * __builtin_amdgcn_exp2f(g4[e] - gs) * acc[i4 * 4 + e];
        (tile == 0 ? M0 + (tb + e) * P0 : M1 + (tb - 32 + e) * P1)[s] = s < tb + e ? a : 0.f;
      }
    }
  }
  wave_sync();
  {  // the four diagonal blocks: lane 16 b + j solves column j of block b
    const int j = lane & 15, pitch = h ? P1 : P0;
    float* D = (h ? M1 + 32 : M0) + ((lane >> 4) & 1) * 16 * (pitch + 1);  // this lane's diagonal block
    float col[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float x4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s4 = 0; s4 < i; s4 += 4) {
        const f32x4 a4 = *(const f32x4*)(D + i * pitch + s4);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (s4 + u < i) x4[u] -= a4[u] * col[s4 + u];
      }
      col[i] = i < j ? 0.f : (i == j ? 1.f : (x4[0] + x4[1]) + (x4[2] + x4[3]));
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) D[i * pitch + j] = col[i];
  }
  wave_sync();
  // T_(2p+1)(2p) = -D_(2p+1) (A_(2p+1)(2p) D_(2p)) in each half p
  const f32x4 d0 = get16<P0>(M0), d1 = get16<P0>(M0 + 16 * P0 + 16), d2 = get16<P1>(M1 + 32);
  const f32x4 t10 = -mul16<P0>(M0 + 16 * P0 + 16, mul16<P0>(M0 + 16 * P0, d0, f32x4{}), f32x4{});
  const f32x4 t32 = -mul16<P1>(M1 + 16 * P1 + 48, mul16<P1>(M1 + 16 * P1 + 32, d2, f32x4{}), f32x4{});
  // T21 = -T22 (A21 T11) over 16 x 16 blocks; T11 and T22 are lower triangular
  f32x4 xx[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const float* a21 = M1 + 16 * a * P1;
    xx[a][0] = mul16<P1>(a21 + 16, t10, mul16<P1>(a21, d0, f32x4{}));
    xx[a][1] = mul16<P1>(a21 + 16, d1, f32x4{});
  }
  wave_sync();
  put16<P0>(M0 + 16 * P0, t10);
  put16<P1>(M1 + 16 * P1 + 32, t32);
  wave_sync();
#pragma unroll
  for (int bb = 0; bb < 2; ++bb) {
    put16<P1>(M1 + 16 * bb, -mul16<P1>(M1 + 32, xx[0][bb], f32x4{}));
    put16<P1>(M1 + 16 * P1 + 16 * bb,
              -mul16<P1>(M1 + 16 * P1 + 48, xx[1][bb], mul16<P1>(M1 + 16 * P1 + 32, xx[0][bb], f32x4{})));
  }
  wave_sync();
  // R[t][s] = 2^(g_C - g_t) T[t][s] beta_s
  unsigned char* rec = recs + (seq * NC + c) * REC;
#pragma unroll
  for (int u = 0; u < 6; ++u) {
    const int idx = lane + (u < 2 ? u : u - 2) * 64;
    const int row = u < 2 ? idx >> 2 : 32 + (idx >> 3), cc = u < 2 ? idx & 3 : idx & 7;
    const float dt = __builtin_amdgcn_exp2f(gC - g[row]);
    bf16x8 y;
#pragma unroll
    for (int e4 = 0; e4 < 2; ++e4) {
      const f32x4 m4 = *(const f32x4*)((u < 2 ? M0 + row * P0 : M1 + (row - 32) * P1) + cc * 8 + e4 * 4), b4 = *(const f32x4*)(bet + cc * 8 + e4 * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e4 * 4 + e] = (bf16)(m4[e] * (dt * b4[e]));
    }
    *(u32x4*)(rec + (u < 2 ? r0_off(row, cc) : R1 + row_off<64>(row - 32, cc))) = __builtin_bit_cast(u32x4, y);
  }
  *(float*)(rec + GAM + lane * 4) = __builtin_amdgcn_exp2f(gt);
}

// ------------------------------------------------------------------ chunk scan

// Transposed reads with their wait in one assembly block (no read is in flight outside it): 4 rows x
// 4 columns of 16-bit values per 16 lanes each, at the given bases plus constant offsets.
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void tr_read8(uint32_t lo, uint32_t hi, s16x4 (&v)[8]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%10\n\t"
      "ds_read_b64_tr_b16 %1, %9 offset:%10\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %6, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(lo), "v"(hi), "n"(O0), "n"(O1), "n"(O2), "n"(O3)
      : "memory");
}
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void tr_read16(const uint32_t (&lo)[2], const uint32_t (&hi)[2], s16x4 (&v)[16]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16 offset:%20\n\t"
      "ds_read_b64_tr_b16 %1, %17 offset:%20\n\t"
      "ds_read_b64_tr_b16 %2, %16 offset:%21\n\t"
      "ds_read_b64_tr_b16 %3, %17 offset:%21\n\t"
      "ds_read_b64_tr_b16 %4, %16 offset:%22\n\t"
      "ds_read_b64_tr_b16 %5, %17 offset:%22\n\t"
      "ds_read_b64_tr_b16 %6, %16 offset:%23\n\t"
      "ds_read_b64_tr_b16 %7, %17 offset:%23\n\t"
      "ds_read_b64_tr_b16 %8, %18 offset:%20\n\t"
      "ds_read_b64_tr_b16 %9, %19 offset:%20\n\t"
      "ds_read_b64_tr_b16 %10, %18 offset:%21\n\t"
      "ds_read_b64_tr_b16 %11, %19 offset:%21\n\t"
      "ds_read_b64_tr_b16 %12, %18 offset:%22\n\t"
      "ds_read_b64_tr_b16 %13, %19 offset:%22\n\t"
      "ds_read_b64_tr_b16 %14, %18 offset:%23\n\t"
      "ds_read_b64_tr_b16 %15, %19 offset:%23\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]),
        "=&v"(v[8]), "=&v"(v[9]), "=&v"(v[10]), "=&v"(v[11]), "=&v"(v[12]), "=&v"(v[13]), "=&v"(v[14]), "=&v"(v[15])
      : "v"(lo[0]), "v"(hi[0]), "v"(lo[1]), "v"(hi[1]), "n"(O0), "n"(O1), "n"(O2), "n"(O3)
      : "memory");
}
__device__ __forceinline__ bf16x8 tr_frag(s16x4 a, s16x4 b) {
  const s16x4 v[2] = {a, b};
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ bf16x8 acc_bf8(const f32x16& a, int q) {
  bf16x8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (bf16)a[8 * q + e];
  return x;
}

template <int DK, int DV>
struct ScanLds {
  static constexpr int K = 0, V = 64 * DK * 2, R = V + 64 * DV * 2, STAGE = R + gdc::REC_LDS;
  static constexpr int NS = 4;
  static constexpr int BYTES = NS * STAGE;
  static constexpr int KI = 64 * DK * 2 / 1024, VI = 64 * DV * 2 / 1024;
  static_assert(BYTES <= 160 * 1024, "fits LDS");
};

// 1 KiB straight into LDS at dst, from byte voff (per lane) + soff of src; past `bytes` zeros.
__device__ __forceinline__ void copy_kib(const void* src, int bytes, unsigned char* dst, int voff, int soff) {
  const auto rs = buffer_rsrc(src, bytes);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, voff, soff, 0, 0);
}
// 1 KiB of D-wide rows (row block blk): lanes pick the 16-byte piece that belongs at their LDS slot.
template <int D>
__device__ __forceinline__ void copy_rows(const void* src, int bytes, unsigned char* dst, int blk) {
  constexpr int PR = D * 2 / 16;  // pieces per row
  const int lane = threadIdx.x & 63, r = lane / PR, row = blk * (64 / PR) + r;
  copy_kib(src, bytes, dst + blk * 1024, r * D * 2 + (((lane % PR) ^ gdc::row_key<D>(row)) << 4), blk * 1024);
}

// Block: the chunks of one segment of one (sequence, value head), waves 0..3 on 32 columns each of the
// state. SEG (long sequences, several segments): waves 4..7 carry 32 columns each of the segment's
// transition matrix Phi, from I and without V, on the same chunks in LDS; the first segment starts from
// S itself and needs none. Four stages, three chunks in flight. Bound by the chain of products of a
// chunk: 38 MFMAs of 32 cycles and about 250 VALU instructions a wave, 1.4 us a chunk with one wave per
// SIMD (of it 0.64 us if only the loads are left in, 1.1 without them), 2.1 to 2.5 with the Phi waves beside
// them. Raising one wave's priority, so that the two of a SIMD fall out of step, measured equal.
template <int DK, int DV, bool SEG>
__global__ __launch_bounds__(SEG ? 512 : 256) __attribute__((amdgpu_waves_per_eu(SEG ? 2 : 1, SEG ? 2 : 1))) void k_gdr_scan(
    const bf16* __restrict__ k, const bf16* __restrict__ v, float* __restrict__ S, int Hk, int Hv, int N, GdrWs ws) {
  using namespace gdc;
  typedef ScanLds<DK, DV> L;
  constexpr int NW = SEG ? 8 : 4, NKT = DK / 32;
  constexpr int RI = (REC_INS + NW - 1) / NW, CNT = L::KI / NW + L::VI / NW + RI;
  static_assert(L::KI % NW == 0 && L::VI % NW == 0 && 2 * CNT < 64, "every wave copies the same number of KiB");
  extern __shared__ __align__(16) unsigned char smem[];
  const int P = ws.P;
  const int per = gridDim.x / 8, full = per * 8;
  const int id = blockIdx.x, blk = id < full ? (id % 8) * per + id / 8 : id;
  const int hv = blk % Hv, bs = blk / Hv, seg = bs % P, b = bs / P;
  const int hk = hv / (Hv / Hk);
  const int NC = (N + C - 1) / C;
  const int c_begin = seg * ws.cps, c_end = min(NC, c_begin + ws.cps);
  const int64_t seq = (int64_t)b * Hv + hv;
  const bf16* kh = k + ((int64_t)b * Hk + hk) * N * DK;
  const bf16* vh = v + seq * N * DV;
  const unsigned char* recs = (const unsigned char*)ws.rec_ + seq * NC * REC;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int h = lane >> 5, rr = lane & 31, prow = pi(rr);
  const bool phi = SEG && wave >= 4;
  const int n0 = (wave & 3) * 32;
  const bool active = phi ? seg > 0 && n0 < DK : n0 < DV;

  f32x16 st[NKT];
#pragma unroll
  for (int kt = 0; kt < NKT; ++kt) st[kt] = f32x16{};
  if (active) {
    if (phi) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) st[kt][i] = kt * 32 + pi(acc_row(lane, i)) == n0 + rr ? 1.f : 0.f;
    } else if (seg == 0) {
      const float* Sg = S + seq * DK * DV + n0 + rr;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) st[kt][i] = Sg[(kt * 32 + pi(acc_row(lane, i))) * DV];
    }
  }

  auto issue = [&](int c, int stage) {
    unsigned char* d = smem + stage * L::STAGE;
    const int nval = min(C, N - c * C);
    const bf16 *kc = kh + (int64_t)c * C * DK, *vc = vh + (int64_t)c * C * DV;
#pragma unroll
    for (int j = 0; j < L::KI / NW; ++j) copy_rows<DK>(kc, nval * DK * 2, d + L::K, j * NW + wave);
#pragma unroll
    for (int j = 0; j < L::VI / NW; ++j) copy_rows<DV>(vc, nval * DV * 2, d + L::V, j * NW + wave);
#pragma unroll
    for (int j = 0; j < RI; ++j) {  // (past the record's end: the last KiB again)
      const int i = min(j * NW + wave, REC_INS - 1);
      copy_kib(recs + (int64_t)c * REC, REC, d + L::R + i * 1024, lane * 16, i * 1024);
    }
  };

  // Lane addresses of the transposed reads, relative to a stage. A read takes, per 16 lanes, source
  // row lane % 16 / 4 of four token rows and four 8-byte pieces; half 0 / 1: tokens 8 h .. + 3 / + 4 .. + 7
  // of a 16-token step. K: column dk = 32 kt + 16 (lane / 16 % 2) + pi order; V: column n0 + lane % 32.
  uint32_t ka[2][NKT], va[2];
  {
    const int r = (lane & 15) >> 2, p = lane & 3, g1 = (lane >> 4) & 1;
    const int sw = ((p & 1) << 1) | (p >> 1);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int row = 8 * h + 4 * hf + r;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) ka[hf][kt] = L::K + row_off<DK>(row, 4 * kt + 2 * g1 + (sw >> 1)) + (sw & 1) * 8;
      va[hf] = L::V + row_off<DV>(row, (n0 < DV ? n0 / 8 : 0) + 2 * g1 + (p >> 1)) + (p & 1) * 8;
    }
  }
  const uint32_t lds0 = lds_addr(smem);

#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (c_begin + j < c_end) issue(c_begin + j, j);
  for (int c = c_begin; c < c_end; ++c) {
    const int stage = (c - c_begin) & 3;
    // Chunk c has landed for this wave (the two after it may be in flight); the barrier makes that true
    // of every wave and ends every wave's reads of the stage that chunk c + 3 goes to.
    if (c + 2 < c_end) pipe_sync<waitcnt_imm(2 * CNT, 0)>();
    else if (c + 1 < c_end) pipe_sync<waitcnt_imm(CNT, 0)>();
    else pipe_sync<waitcnt_imm(0, 0)>();
    if (c + 3 < c_end) issue(c + 3, (stage + 3) & 3);
    if (!active) continue;
    const unsigned char* sm = smem + stage * L::STAGE;
    const uint32_t so = lds0 + stage * L::STAGE;
    const float* gam = (const float*)(sm + L::R + GAM);
    // K S for the two token tiles; every LDS read of the product and V's are issued before it
    bf16x8 kf[2][NKT][2];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) kf[tt][kt][q] = lds_b8(sm + L::K + row_off<DK>(tt * 32 + prow, 4 * kt + 2 * q + h));
    bf16x8 sb[NKT][2];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int q = 0; q < 2; ++q) sb[kt][q] = acc_bf8(st[kt], q);
    s16x4 vv[8];
    if (!phi) {
      tr_read8<0, 16 * DV * 2, 32 * DV * 2, 48 * DV * 2>(so + va[0], so + va[1], vv);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) vv[i] = s16x4{};
    }
    f32x16 u[2] = {f32x16{}, f32x16{}};
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int q = 0; q < 2; ++q) mfma_k16(u[tt], kf[tt][kt][q], sb[kt][q]);
    // K's first transposed fragments, requested behind the last of these MFMAs instead of after U's (six
    // layers of 16384 tokens, 32 heads: 768 -> 762 us)
    s16x4 kv[2][16];
    auto read_kt = [&](int k2) {
      const uint32_t lo[2] = {so + ka[0][k2], so + ka[0][k2 + 1]}, hi[2] = {so + ka[1][k2], so + ka[1][k2 + 1]};
      tr_read16<0, 16 * DK * 2, 32 * DK * 2, 48 * DK * 2>(lo, hi, kv[(k2 / 2) & 1]);
    };
    read_kt(0);
    // X = V - gamma (K S)
    bf16x8 xb[2][2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const bf16x8 ve = tr_frag(vv[(tt * 2 + q) * 2], vv[(tt * 2 + q) * 2 + 1]);
        const f32x4 g0 = *(const f32x4*)(gam + tt * 32 + q * 16 + h * 8), g1 = *(const f32x4*)(gam + tt * 32 + q * 16 + h * 8 + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) xb[tt][q][e] = (bf16)fmaf(e < 4 ? -g0[e] : -g1[e - 4], u[tt][8 * q + e], (float)ve[e]);
      }
    // U = R X (R's upper right tile is zero)
    f32x16 w[2] = {f32x16{}, f32x16{}};
#pragma unroll
    for (int q = 0; q < 2; ++q) mfma_k16(w[0], lds_b8(sm + L::R + r0_off(prow, 2 * q + h)), xb[0][q]);
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        mfma_k16(w[1], lds_b8(sm + L::R + R1 + row_off<64>(prow, 4 * ss + 2 * q + h)), xb[ss][q]);
    // S = gamma_C S + K^T U
    const float gc = gam[63];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) st[kt] *= gc;
    bf16x8 ub[2][2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int q = 0; q < 2; ++q) ub[tt][q] = acc_bf8(w[tt], q);
#pragma unroll
    for (int k2 = 0; k2 < NKT; k2 += 2) {
      const s16x4(&f)[16] = kv[(k2 / 2) & 1];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
          mfma_k16(st[k2 + kk], tr_frag(f[kk * 8 + x * 2], f[kk * 8 + x * 2 + 1]), ub[x >> 1][x & 1]);
      if (k2 + 2 < NKT) read_kt(k2 + 2);
    }
  }
  if (!active) return;
  if (phi) {
    bf16* out = (bf16*)ws.phi + (seq * P + seg) * DK * DK + n0 + rr;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) out[(kt * 32 + pi(acc_row(lane, i))) * DK] = (bf16)st[kt][i];
    return;
  }
  float* out = (SEG ? ws.psi + (seq * P + seg) * DK * DV : S + seq * DK * DV) + n0 + rr;
#pragma unroll
  for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
    for (int i = 0; i < 16; ++i) out[(kt * 32 + pi(acc_row(lane, i))) * DV] = st[kt][i];
}

// ------------------------------------------------------------------ segments in order

// S <- Phi_g S + Psi_g for g = 1 .. P - 1, from S = Psi_0; grid (DV / 32, Hv, B), one wave and 32 state
// columns a block. Phi enters the product in bf16, as it is stored; two LDS buffers of it, and Psi one step
// ahead. A step is bounded by its loads, so the columns of a head are spread over CUs although each of
// them then reads all of Phi (32 KiB of 48 a step).
template <int DK, int DV>
__global__ __launch_bounds__(64) void k_gdr_join(float* __restrict__ S, int Hv, GdrWs ws) {
  using namespace gdc;
  constexpr int NKT = DK / 32, BYTES = DK * DK * 2, INS = BYTES / 1024;
  __shared__ __align__(16) unsigned char smem[2 * BYTES];
  const int P = ws.P;
  const int64_t seq = (int64_t)blockIdx.z * Hv + blockIdx.y;
  const int lane = threadIdx.x;
  const int h = lane >> 5, rr = lane & 31, prow = pi(rr), n0 = blockIdx.x * 32;
  const float* psi = ws.psi + seq * P * DK * DV + n0 + rr;
  f32x16 st[NKT], ps[NKT];
  auto load_psi = [&](int g, f32x16 (&x)[NKT]) {
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) x[kt][i] = psi[(int64_t)g * DK * DV + (kt * 32 + pi(acc_row(lane, i))) * DV];
  };
  auto issue = [&](int g) {
    const bf16* src = (const bf16*)ws.phi + (seq * P + g) * DK * DK;
    for (int i = 0; i < INS; ++i) copy_rows<DK>(src, BYTES, smem + (g & 1) * BYTES, i);
  };
  load_psi(0, st);
  load_psi(1, ps);
  issue(1);
  for (int g = 1; g < P; ++g) {
    pipe_sync<waitcnt_imm(0, 0)>();
    if (g + 1 < P) issue(g + 1);
    const unsigned char* sm = smem + (g & 1) * BYTES;
    bf16x8 sb[NKT][2];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      sb[kt][0] = acc_bf8(st[kt], 0);
      sb[kt][1] = acc_bf8(st[kt], 1);
      st[kt] = ps[kt];
    }
    if (g + 1 < P) load_psi(g + 1, ps);
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int k2 = 0; k2 < NKT; ++k2)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          mfma_k16(st[kt], lds_b8(sm + row_off<DK>(kt * 32 + prow, 4 * k2 + 2 * q + h)), sb[k2][q]);
  }
  float* Sg = S + seq * DK * DV + n0 + rr;
#pragma unroll
  for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
    for (int i = 0; i < 16; ++i) Sg[(kt * 32 + pi(acc_row(lane, i))) * DV] = st[kt][i];
}

// ------------------------------------------------------------------ host side

template <int DK, int DV>
static hipError_t chunk_launch(const bf16* k, const bf16* v, const float* alpha, const float* beta, float* S, int B,
                               int Hk, int Hv, int N, GdrWs ws, hipStream_t s, const LaunchEvents& ev) {
  typedef ScanLds<DK, DV> L;
  static bool once = [] {
    (void)hipFuncSetAttribute((const void*)k_gdr_scan<DK, DV, false>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    (void)hipFuncSetAttribute((const void*)k_gdr_scan<DK, DV, true>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    return true;
  }();
  (void)once;
  const int NC = (N + gdc::C - 1) / gdc::C;
  record(ev.gdr_prep[0], s);
  const int n = B * Hv * NC;
  k_gdr_tri<DK><<<(n + TRI_W - 1) / TRI_W, 64 * TRI_W, 0, s>>>(k, alpha, beta, Hk, Hv, N, NC, n, (unsigned char*)ws.rec_);
  record(ev.gdr_prep[1], s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  record(ev.gdr_scan[0], s);
  const unsigned grid = (unsigned)((int64_t)B * Hv * ws.P);
  if (ws.P > 1) {
    k_gdr_scan<DK, DV, true><<<grid, 512, L::BYTES, s>>>(k, v, S, Hk, Hv, N, ws);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_gdr_join<DK, DV><<<dim3(DV / 32, Hv, B), 64, 0, s>>>(S, Hv, ws);
  } else {
    k_gdr_scan<DK, DV, false><<<grid, 256, L::BYTES, s>>>(k, v, S, Hk, Hv, N, ws);
  }
  record(ev.gdr_scan[1], s);
  return hipGetLastError();
}

hipError_t launch_delta_chunk(const void* k, const void* v, const float* alpha, const float* beta, float* S, int B,
                              int Hk, int Hv, int N, int dk, int dv, GdrWs ws, hipStream_t s, const LaunchEvents& ev) {
  const bf16 *kb = (const bf16*)k, *vb = (const bf16*)v;
  if (dk == 128 && dv == 128) return chunk_launch<128, 128>(kb, vb, alpha, beta, S, B, Hk, Hv, N, ws, s, ev);
  if (dk == 128) return chunk_launch<128, 64>(kb, vb, alpha, beta, S, B, Hk, Hv, N, ws, s, ev);
  if (dv == 128) return chunk_launch<64, 128>(kb, vb, alpha, beta, S, B, Hk, Hv, N, ws, s, ev);
  return chunk_launch<64, 64>(kb, vb, alpha, beta, S, B, Hk, Hv, N, ws, s, ev);
}

}  // namespace dv
