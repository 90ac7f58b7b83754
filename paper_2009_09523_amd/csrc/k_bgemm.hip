// Batched small GEMM with arbitrary strides and mixed operand types on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation).  Used for the per-(sequence, head)
// contractions of self-attention (scores, probabilities x values, and their backward products), where
// every matrix is a strided window of a larger activation tensor.
//   C[b][m,n] = alpha * sum_k A[b][m,k] * B[b][n,k]
// with X[b][i,k] at X + (b / inner) * x.outer + (b % inner) * x.inner + i * x.rs + k * x.cs.
//
// These products are small (64 x 64 x 64 for each of some ten heads), so what bounds them is the trip to
// memory and how many wavefronts share it.  A wavefront owns one tile of 16 x 16 (or 32 x 32) outputs and
// takes its operands from memory straight into the registers that the matrix instruction reads, four
// chunks of 16 contraction elements in flight: a contraction of 64 is one trip.  No LDS, no barrier;
// neighbouring wavefronts share their operands through the caches.  (64 x 64 tiles of one workgroup,
// staged 16 elements at a time through LDS, on the vector ALUs: 14.8 us for 8 to 16 heads of 64 x 64 x 64; this: 4.3 to 4.8 us.)
#include <algorithm>

#include "vf_device.h"

namespace vf {
namespace {

constexpr int NT = 256, WAVES = NT / 64;
constexpr int kGridRows = 65535;             // batches of one launch
constexpr int CHUNK_K = 16, DEPTH = 4;       // contraction elements of a chunk, chunks in flight

// Four consecutive contraction elements of one operand row: fp32 or bf16, as one vector or one by one.
enum { F32_VEC, F32_ANY, BF16_VEC, BF16_ANY };
template <int KIND> struct Quad;
template <> struct Quad<F32_VEC> {
  float4 v;
  __device__ __forceinline__ void load(const void* p, int64_t row, int64_t, int k, int K) {
    v = *reinterpret_cast<const float4*>(static_cast<const float*>(p) + row + min(k, K - 4));
  }
  __device__ __forceinline__ float get(int i) const { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
};
template <> struct Quad<F32_ANY> {
  float v[4];
  __device__ __forceinline__ void load(const void* p, int64_t row, int64_t cs, int k, int K) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = static_cast<const float*>(p)[row + (int64_t)min(k + i, K - 1) * cs];
  }
  __device__ __forceinline__ float get(int i) const { return v[i]; }
};
template <> struct Quad<BF16_VEC> {
  uint2 v;
  __device__ __forceinline__ void load(const void* p, int64_t row, int64_t, int k, int K) {
    v = *reinterpret_cast<const uint2*>(static_cast<const bf16_t*>(p) + row + min(k, K - 4));
  }
  __device__ __forceinline__ float get(int i) const {
    const uint32_t w = i < 2 ? v.x : v.y;
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
template <> struct Quad<BF16_ANY> {
  bf16_t v[4];
  __device__ __forceinline__ void load(const void* p, int64_t row, int64_t cs, int k, int K) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = static_cast<const bf16_t*>(p)[row + (int64_t)min(k + i, K - 1) * cs];
  }
  __device__ __forceinline__ float get(int i) const { return bf16_to_f32(v[i]); }
};

typedef float acc4 __attribute__((ext_vector_type(4)));

// TW x TW tiles of 16 x 16 per wavefront.  Lane l holds operand row l % 16; of a chunk's sixteen contraction
// elements it holds 4 (l / 16) .. + 3 (both operands alike, so element i of all lanes makes one matrix step).
// Rows beyond the matrix are clamped (their products never stored), elements beyond K are zero in both operands.
template <int TW, int KA, int KB>
__global__ __launch_bounds__(NT) void bgemm_kernel(BMat A, BMat B, BMat C, int M, int N, int K, int inner,
                                                   float alpha, int tiles, int tn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.y, t = blockIdx.x * WAVES + wave;
  if (t >= tiles) return;
  const int m0 = (t / tn) * 16 * TW, n0 = (t % tn) * 16 * TW;
  const int bo = b / inner, bi = b - bo * inner;
  const int r16 = lane & 15, g4 = (lane >> 4) * 4;
  int64_t arow[TW], brow[TW];
#pragma unroll
  for (int j = 0; j < TW; ++j) {
    arow[j] = (int64_t)bo * A.outer + (int64_t)bi * A.inner + (int64_t)min(m0 + 16 * j + r16, M - 1) * A.rs;
    brow[j] = (int64_t)bo * B.outer + (int64_t)bi * B.inner + (int64_t)min(n0 + 16 * j + r16, N - 1) * B.rs;
  }
  Quad<KA> a[DEPTH][TW];
  Quad<KB> q[DEPTH][TW];
  auto load = [&](int k0, int slot) {
#pragma unroll
    for (int j = 0; j < TW; ++j) {
      a[slot][j].load(A.p, arow[j], A.cs, k0 + g4, K);
      q[slot][j].load(B.p, brow[j], B.cs, k0 + g4, K);
    }
  };
  acc4 acc[TW][TW];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = acc4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < DEPTH; ++u) load(u * CHUNK_K, u);
  for (int k0 = 0; k0 < K; k0 += DEPTH * CHUNK_K) {
    const bool more = k0 + DEPTH * CHUNK_K < K;
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      const int k = k0 + u * CHUNK_K + g4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float av[TW], bv[TW];
#pragma unroll
        for (int j = 0; j < TW; ++j) {
          av[j] = a[u][j].get(i);
          bv[j] = q[u][j].get(i);
          if (A.round_bf16) av[j] = round_bf16(av[j]);
          if (B.round_bf16) bv[j] = round_bf16(bv[j]);
          if (k + i >= K) av[j] = bv[j] = 0.f;
        }
#pragma unroll
        for (int x = 0; x < TW; ++x)
#pragma unroll
          for (int y = 0; y < TW; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[x], bv[y], acc[x][y], 0, 0, 0);
      }
      if (more) load(k0 + (DEPTH + u) * CHUNK_K, u);
    }
  }
  // accumulator register r of a lane: row 4 (lane / 16) + r, column lane % 16
  const int64_t cbase = (int64_t)bo * C.outer + (int64_t)bi * C.inner;
#pragma unroll
  for (int x = 0; x < TW; ++x)
#pragma unroll
    for (int y = 0; y < TW; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * x + g4 + r, n = n0 + 16 * y + r16;
        if (m >= M || n >= N) continue;
        const float v = alpha * acc[x][y][r];
        const int64_t idx = cbase + (int64_t)m * C.rs + (int64_t)n * C.cs;
        if (C.is_bf16) static_cast<bf16_t*>(const_cast<void*>(C.p))[idx] = f32_to_bf16(v);
        else           static_cast<float*>(const_cast<void*>(C.p))[idx] = v;
      }
}

// Vector reads need contiguous contraction elements, whole groups of four, and every row aligned for them.
int kind_of(const BMat& x, int K) {
  const bool vec = x.cs == 1 && K % 4 == 0 && x.rs % 4 == 0 && x.outer % 4 == 0 && x.inner % 4 == 0 &&
                   (reinterpret_cast<uintptr_t>(x.p) & (x.is_bf16 ? 7 : 15)) == 0;
  return x.is_bf16 ? (vec ? BF16_VEC : BF16_ANY) : (vec ? F32_VEC : F32_ANY);
}

}  // namespace

int launch_bgemm(const BMat& A, const BMat& B, const BMat& C, int M, int N, int K, int batch, int inner,
                 float alpha, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0 || batch <= 0 || inner <= 0 || !A.p || !B.p || !C.p) return VF_EINVAL;
  if (batch > kGridRows) {      // (rows of a grid: a unit of several nodes may hold more heads than that)
    const int run = kGridRows / inner;          // whole steps of `outer`
    if (run < 1) return VF_EINVAL;
    auto from = [](BMat x, int64_t step) {
      x.p = static_cast<const char*>(x.p) + step * x.outer * (x.is_bf16 ? 2 : 4);
      return x;
    };
    for (int64_t o = 0; o * inner < batch; o += run)
      VF_TRY(launch_bgemm(from(A, o), from(B, o), from(C, o), M, N, K, (int)std::min<int64_t>((int64_t)run * inner, batch - o * inner),
                          inner, alpha, s));
    return VF_OK;
  }
  // 32 x 32 outputs per wavefront (half the operand reads per output) as soon as that leaves four wavefronts for
  // each of the 256 compute units
  const int64_t big = (int64_t)batch * ((M + 31) / 32) * ((N + 31) / 32);
  const int tw = big >= 1024 ? 2 : 1, side = 16 * tw;
  const int tn = (N + side - 1) / side;
  const int64_t all = (int64_t)((M + side - 1) / side) * tn;
  if (all > 0x7fffff00) return VF_EINVAL;
  const int tiles = (int)all;
  const dim3 grid((tiles + WAVES - 1) / WAVES, batch);
  const int ka = kind_of(A, K), kb = kind_of(B, K);
#define VF_BG(KA, KB)                                                                                          \
  case KA * 4 + KB:                                                                                            \
    if (tw == 2) bgemm_kernel<2, KA, KB><<<grid, NT, 0, s>>>(A, B, C, M, N, K, inner, alpha, tiles, tn);   \
    else         bgemm_kernel<1, KA, KB><<<grid, NT, 0, s>>>(A, B, C, M, N, K, inner, alpha, tiles, tn);   \
    break;
#define VF_BG4(KA) VF_BG(KA, F32_VEC) VF_BG(KA, F32_ANY) VF_BG(KA, BF16_VEC) VF_BG(KA, BF16_ANY)
  switch (ka * 4 + kb) { VF_BG4(F32_VEC) VF_BG4(F32_ANY) VF_BG4(BF16_VEC) VF_BG4(BF16_ANY) }
#undef VF_BG4
#undef VF_BG
  VF_LAUNCH_CHECK();
  return VF_OK;
}

}  // namespace vf
