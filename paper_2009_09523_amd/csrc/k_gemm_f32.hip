// fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32 and 16x16x4: fp32 operands, fp32 fused
// multiply-adds) for the fp32 workloads.  acc[m,n] = sum_k A[m*sam + k*sak] * B[n*sbn + k*sbk], each operand
// contiguous along k or along its rows.
//
// An fp32 workload's products are small (16 to 512 rows, 10 to 1024 columns, contractions of 16 to 4096), so
// what bounds them is the number of dependent trips to memory and how many compute units have a tile, not
// flops: 64 x 64 tiles staged through LDS 16 contraction elements at a time made K / 16 trips one after the
// other on a handful of workgroups (104 us for 256 x 256 x 1024, 714 us for 36 x 256 x 4099).
// Here a workgroup's wavefronts cut the contraction among themselves: each takes its slice of k for the WHOLE
// tile, operands straight from memory into the MFMA registers (nothing is shared between wavefronts, so LDS
// would only add a round trip), two groups of 32 or 64 contraction elements in flight; the partial tiles are
// then added through LDS in wavefront order, so results do not depend on scheduling.  The same products now
// take 4.9 us and, with the operands in cache, 15 us (24 us inside a step); 2048 x 1024 x 1024 runs at 81 TFLOP/s.
// Where there are tiles enough for every wavefront to have one of its own, and for operands out of 32-bit reach,
// see launch_operands and launch_gemm_f32.
#include "vf_device.h"

namespace vf {
namespace {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x16v __attribute__((ext_vector_type(16)));

constexpr int GU = 4;        // chunks of the contraction per group
constexpr uint32_t kOutside = 0x80000000u;   // an offset beyond every buffer: the load returns 0

// One lane's part of an operand: T row tiles of MS rows, this lane's row of each.  A chunk is 4 * 64 / MS
// contraction elements: the q-th copy of the rows among the lanes (q = lane / MS) holds elements 4 q .. 4 q + 3
// of it, and MFMA step s contracts element s of every copy (any assignment of k to steps will do as long as
// both operands use the same one).  A group is GU chunks.  KC: the operand is contiguous along k; VEC: in
// 16-byte vectors (rows 16-byte aligned, K % 4 == 0).  Loads go through a buffer descriptor over the operand
// from the workgroup's first row on: what lies outside the matrix (rows, or k at and beyond K) is asked for
// beyond the buffer's end and comes back as 0, so there are neither branches nor selections around the loads
// and the compiler keeps a whole group's in flight.
template <int MS, int T, bool KC, bool VEC>
struct Operand {
  static constexpr int CK = 4 * (64 / MS);
  __amdgpu_buffer_rsrc_t buf;
  uint32_t pitch;                                        // bytes
  int K, kl;                                             // kl: this lane's first element of a chunk
  uint32_t off[T];                                       // of this lane's row (and of its first element's row of k)
  __device__ __forceinline__ void init(const float* p, int64_t ld, int r0, int nrows, int K_, int lane) {
    K = K_;
    kl = 4 * (lane / MS);
    pitch = (uint32_t)ld * 4u;
    const float* base = p + (KC ? (int64_t)r0 * ld : (int64_t)r0);
    // bytes from the first row to the operand's end (the host keeps what a workgroup can reach below 2 GiB)
    const int64_t span = (KC ? (int64_t)(nrows - 1 - r0) * ld + K : (int64_t)(K - 1) * ld + (nrows - r0)) * 4;
    buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)min(span, (int64_t)0x7fffffff), 0x00020000);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int r = MS * t + lane % MS;
      off[t] = r0 + r < nrows ? (KC ? (uint32_t)r * pitch + (uint32_t)kl * 4u : (uint32_t)r * 4u + (uint32_t)kl * pitch) : kOutside;
    }
  }
  // The group of contraction elements k0 .. k0 + GU * CK - 1 (k0 the same for the whole wavefront).
  __device__ __forceinline__ void load(float (&v)[GU][T][4], int k0) const {
    const int left = K - k0 - kl;                        // elements of this lane from its first one on
    // (a chunk that starts past the end: nothing is fetched, and its scalar offset stays inside the buffer, so that
    // the bounds check -- lane offset against the buffer's size, with or without the scalar offset -- is the same)
#pragma unroll
    for (int u = 0; u < GU; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if (KC && VEC) {
          typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
          const u32x4v q = __builtin_amdgcn_raw_buffer_load_b128(buf, CK * u < left ? off[t] : kOutside,
                                                              min(k0 + CK * u, K - 1) * 4, 0);
#pragma unroll
          for (int s = 0; s < 4; ++s) v[u][t][s] = __uint_as_float(q[s]);
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const uint32_t o = CK * u + s < left ? off[t] + (KC ? 4u * s : pitch * s) : kOutside;
            const uint32_t so = (uint32_t)min(k0 + CK * u, K - 1) * (KC ? 4u : pitch);
            v[u][t][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, o, so, 0));
          }
        }
      }
  }
};

template <int MS> struct Mfma;
template <> struct Mfma<32> {
  typedef f32x16v acc_t;
  static constexpr int R = 16;
  static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <> struct Mfma<16> {
  typedef f32x4v acc_t;
  static constexpr int R = 4;
  static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};

// blockIdx.z selects the contraction slice [z * kslab, (z + 1) * kslab); slice z writes its partial product
// to slab z of C (the consumer adds the slabs in order), the bias goes to slab 0.  Wavefront w of a
// workgroup takes the elements [w * kwave, (w + 1) * kwave) of the slice (kwave and kslab multiples of a group).
template <int MS, int TM, int TN, int NW, bool AKC, bool BKC, bool VEC>
__global__ __launch_bounds__(NW * 64) void gemm_f32_mfma_kernel(const float* __restrict__ A, int64_t lda,
                                                                const float* __restrict__ B, int64_t ldb,
                                                                int M, int N, int K, int kslab, int kwave,
                                                                int64_t slab_stride, Epilogue ep) {
  typedef Mfma<MS> MF;
  constexpr int R = MF::R;
  constexpr int E = TM * TN * MS * MS;                   // elements of the tile
  constexpr int GK = GU * 4 * (64 / MS);                 // contraction elements of a group
  __shared__ float part[NW > 1 ? NW * E : 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.y * (MS * TM), n0 = blockIdx.x * (MS * TN);
  const int kend_slab = min(K, (int)(blockIdx.z + 1) * kslab);
  const int kbeg = (int)blockIdx.z * kslab + wave * kwave;
  const int kend = min(kend_slab, kbeg + kwave);

  typename MF::acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < R; ++r) acc[i][j][r] = 0.f;

  const int groups = kend > kbeg ? (kend - kbeg + GK - 1) / GK : 0;
  if (groups > 0) {
    Operand<MS, TM, AKC, VEC> oa;
    Operand<MS, TN, BKC, VEC> ob;
    oa.init(A, lda, m0, M, K, lane);
    ob.init(B, ldb, n0, N, K, lane);
    float a0[GU][TM][4], b0[GU][TN][4], a1[GU][TM][4], b1[GU][TN][4];
    auto multiply = [&](const float (&a)[GU][TM][4], const float (&b)[GU][TN][4]) {
#pragma unroll
      for (int u = 0; u < GU; ++u)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = MF::mul(a[u][i][s], b[u][j][s], acc[i][j]);
    };
    // two groups in flight: the loads of group g + 2 are issued as soon as group g has been multiplied (past the
    // operand's end they fetch nothing and return 0; past the slice's end they are not used)
    oa.load(a0, kbeg);
    ob.load(b0, kbeg);
    if (groups > 1) {
      oa.load(a1, kbeg + GK);
      ob.load(b1, kbeg + GK);
      int k = kbeg;
      for (int g = 0; g + 2 <= groups; g += 2, k += 2 * GK) {
        __builtin_amdgcn_sched_barrier(0);
        multiply(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        oa.load(a0, min(k + 2 * GK, K));
        ob.load(b0, min(k + 2 * GK, K));
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        oa.load(a1, min(k + 3 * GK, K));
        ob.load(b1, min(k + 3 * GK, K));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (groups & 1) multiply(a0, b0);
  }

  // Partial tiles through LDS as the registers hold them, added in wavefront order.
  if (NW > 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < R; ++r) part[wave * E + ((i * TN + j) * R + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
  }
  float* C = static_cast<float*>(ep.C) + (int64_t)blockIdx.z * slab_stride;
  const bool first_slice = blockIdx.z == 0;
  constexpr int NT = NW * 64;
  constexpr int PER = (E + NT - 1) / NT;
  float add[PER];
  int mm[PER], nn[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * NT + tid;
    const int f = e / 64, r = f % R, i = f / R / TN, j = f / R % TN;
    mm[p] = m0 + MS * i + MF::row(r, lane);
    nn[p] = n0 + MS * j + lane % MS;
    if (E % NT && e >= E) mm[p] = M;
    const int m = min(mm[p], M - 1), n = min(nn[p], N - 1);
    add[p] = (ep.bias && first_slice) ? ep.bias[n] : 0.f;
    if (ep.R) add[p] = fmaf(ep.beta, ep.R[(int64_t)m * ep.ldr + n], add[p]);
  }
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * NT + tid;
    if (mm[p] >= M || nn[p] >= N) continue;
    float sum;
    if (NW > 1) {
      sum = part[e];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += part[w * E + e];
    } else {
      sum = acc[p / R / TN][p / R % TN][p % R];            // (element e of the tile is this lane's p-th)
    }
    C[(int64_t)mm[p] * ep.ldc + nn[p]] = fmaf(ep.alpha, sum, add[p]);
  }
}

// The general form: any strides, 64-bit addresses.  64 x 64 tiles of 256 threads, 16 contraction elements at a time
// through LDS, products on the vector ALUs.
constexpr int TT = 64, TK = 16, TILED_NT = 256;

// Loads a [64 x TK] tile (row r, element k) into dst[k][r].  When the k stride is 1 consecutive threads walk k,
// otherwise they walk rows, so that the unit-stride index is the fastest across a wavefront.
__device__ __forceinline__ void load_tile(const float* __restrict__ base, int64_t srow, int64_t sk, int row0, int nrows,
                                          int k0, int K, float (*dst)[TT + 4], int tid) {
  if (sk == 1) {
#pragma unroll
    for (int i = 0; i < TT * TK / TILED_NT; ++i) {
      const int e = tid + i * TILED_NT;
      const int k = e % TK, r = e / TK;
      const int gr = row0 + r, gk = k0 + k;
      dst[k][r] = gr < nrows && gk < K ? base[(int64_t)gr * srow + gk] : 0.f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < TT * TK / TILED_NT; ++i) {
      const int e = tid + i * TILED_NT;
      const int r = e % TT, k = e / TT;
      const int gr = row0 + r, gk = k0 + k;
      dst[k][r] = gr < nrows && gk < K ? base[(int64_t)gr * srow + (int64_t)gk * sk] : 0.f;
    }
  }
}

__global__ __launch_bounds__(TILED_NT) void gemm_f32_tiled_kernel(const float* __restrict__ A, int64_t sam, int64_t sak,
                                                                  const float* __restrict__ B, int64_t sbn, int64_t sbk,
                                                                  int M, int N, int K, int kslab, int64_t slab_stride,
                                                                  Epilogue ep) {
  __shared__ float As[TK][TT + 4];
  __shared__ float Bs[TK][TT + 4];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int m0 = blockIdx.y * TT, n0 = blockIdx.x * TT;
  float acc[4][4] = {};
  const int kbeg = blockIdx.z * kslab;
  const int kend = min(K, kbeg + kslab);
  for (int k0 = kbeg; k0 < kend; k0 += TK) {
    load_tile(A, sam, sak, m0, M, k0, kend, As, tid);
    load_tile(B, sbn, sbk, n0, N, k0, kend, Bs, tid);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  float* C = static_cast<float*>(ep.C) + (int64_t)blockIdx.z * slab_stride;
  const bool first_slice = blockIdx.z == 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      float add = (ep.bias && first_slice) ? ep.bias[n] : 0.f;
      if (ep.R) add = fmaf(ep.beta, ep.R[(int64_t)m * ep.ldr + n], add);
      C[(int64_t)m * ep.ldc + n] = fmaf(ep.alpha, acc[i][j], add);
    }
  }
}

int launch_tiled(const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbn, int64_t sbk, int M, int N, int K,
                 int nsplit, int64_t slab_stride, const Epilogue& ep, hipStream_t s) {
  const int kslab = ((K + nsplit - 1) / nsplit + TK - 1) / TK * TK;
  dim3 grid((N + TT - 1) / TT, (M + TT - 1) / TT, nsplit);
  gemm_f32_tiled_kernel<<<grid, TILED_NT, 0, s>>>(A, sam, sak, B, sbn, sbk, M, N, K, kslab, slab_stride, ep);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

struct F32Shape {
  const float* A; int64_t lda; const float* B; int64_t ldb; int M, N, K, nsplit; int64_t slab;
};

template <int MS, int TM, int TN, int NW, bool AKC, bool BKC, bool VEC>
int launch_tile(const F32Shape& g, const Epilogue& ep, hipStream_t s) {
  constexpr int GK = GU * 4 * (64 / MS);
  const int kslab = ((g.K + g.nsplit - 1) / g.nsplit + GK - 1) / GK * GK;
  const int kwave = ((kslab + NW - 1) / NW + GK - 1) / GK * GK;
  dim3 grid((g.N + MS * TN - 1) / (MS * TN), (g.M + MS * TM - 1) / (MS * TM), g.nsplit);
  gemm_f32_mfma_kernel<MS, TM, TN, NW, AKC, BKC, VEC><<<grid, NW * 64, 0, s>>>(g.A, g.lda, g.B, g.ldb, g.M, g.N, g.K,
                                                                                   kslab, kwave, g.slab, ep);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

// Which tile on how many wavefronts: measured back to back with launch (2.5 us of it), us per product, the
// neighbouring choices beside the one taken (M x N x K):
//   few tiles       16 x 256 x 784: 16/16 4.2, 16/4 4.9, 32/16 8.4;  100 x 500 x 1000: 4.8, 5.5, 11.3
//   short k         784 x 256 x 16: 16/4 3.0, 16/16 5.7, 32/4 3.6
//   more tiles      256 x 1024 x 256: 32/16 4.2, 32/4 5.2, 16/4 5.0;  256 x 4099 x 36: 32/4 6.1, 32/8 7.9, 16/4 8.0
//                   512 x 1024 x 1024: 32/8 17.1, 32/16 22.6, 64/4 26.9;  2048 x 1152 x 384: 32/4 29.8, 32/8 37.0
//   64 x 64         300 x 30522 x 384: 64/4 111, 32/16 147, 32/4 156;  2048 x 1024 x 1024: 53, 88, 56
// More than 512 tiles of 64 x 64 (two workgroups per compute unit, one round): the chip is full whatever the tile,
// and wavefronts that share a tile wait for one another -- with a contraction of a group or two most of them have
// nothing to multiply at all.  So up to 32 elements (80, 128 with many more tiles), where writing the result is all
// there is, the tiled kernel's sixteen elements per trip waste the least, and then one wavefront owns a tile of its
// own (no LDS, no barrier) until the contraction is long enough for 64/4.  The tiled kernel also takes operands that
// are contiguous along k but allow no vector reads: four scalar loads per lane over 32 rows each are bound by the
// cache lines they touch.  us, tiled | 64/4 | taken; rows: a weight gradient (both operands contiguous along their
// rows, result accumulated), k: both contiguous along k, fwd: one and one:
//   rows  4096 x 4096 x 16: 37 | 86 | tiled       x 128: 83 | 105 | 32/4 75       x 256: 140 | 166 | 32/1 126
//         1001 x 2051 x 24: 14.2 | 21.7 | tiled   x 80: 20.6 | 24.2 | 32/4 16.0   2048 x 2048 x 200: 40 | 39 | 32/1 35
//   k     4096 x 4096 x 16: 30 | 52 | tiled       2048 x 2048 x 128: 26 | 25 | 32/1 23      x 256: 47 | 47 | 32x64/1 33
//         8192 x 8192 x 128: 233 | 348 | tiled    x 256: 434 | 657 | 32x64/1 420            x 255: 426 | 1113 | tiled
//         2048 x 2048 x 1024: 177 | 101 | 32x64/1 98   x 4096: 630 | 297 | 64/4 (32x64/1: 350)
//         2051 x 3001 x 201: 55 | 99 | tiled      1001 x 2051 x 99: 21.6 | 19.8 | 32/4 18.9  x 513: 117 | 82 | 64/4
//   fwd   4096 x 4096 x 255: 128 | 203 | tiled    2051 x 3001 x 255: 65 | 84 | 32x64/1 61   x 99: 35 | 34 | 32/4 32
template <bool AKC, bool BKC, bool VEC>
int launch_operands(const F32Shape& g, const Epilogue& ep, hipStream_t s) {
  auto tiles = [&](int t) { return (int64_t)((g.M + t - 1) / t) * ((g.N + t - 1) / t) * g.nsplit; };
  const int K = g.K / g.nsplit;
  const int64_t t64 = tiles(64);
  if (t64 > 512) {
    constexpr bool along_k = AKC && BKC, scalar_k = !VEC && (AKC || BKC);
    const bool scalar_tiled = along_k ? (t64 >= 1536 || (K > (t64 < 1024 ? 112 : 80) && K <= (t64 < 1024 ? 256 : 640)))
                                      : t64 >= 4096 && (K <= 640 || t64 >= 8192);
    if (K <= (t64 < 1024 ? 32 : t64 <= 4096 ? 80 : 128) || (scalar_k && scalar_tiled))
      return launch_tiled(g.A, AKC ? g.lda : 1, AKC ? 1 : g.lda, g.B, BKC ? g.ldb : 1, BKC ? 1 : g.ldb, g.M, g.N, g.K, g.nsplit,
                          g.slab, ep, s);
    if (K <= (scalar_k ? 112 : 128))
      return along_k && !scalar_k ? launch_tile<32, 1, 1, 1, AKC, BKC, VEC>(g, ep, s) : launch_tile<32, 1, 1, 4, AKC, BKC, VEC>(g, ep, s);
    if ((along_k && !scalar_k && t64 >= 1024 && K <= 1024) || (scalar_k && !along_k && K <= 640))
      return launch_tile<32, 1, 2, 1, AKC, BKC, VEC>(g, ep, s);
    if (!along_k && !scalar_k && K <= (t64 < 1024 ? 256 : 512)) return launch_tile<32, 1, 1, 1, AKC, BKC, VEC>(g, ep, s);
    return launch_tile<32, 2, 2, 4, AKC, BKC, VEC>(g, ep, s);
  }
  if (t64 == 512)
    return K <= 32 ? launch_tile<32, 1, 1, 1, AKC, BKC, VEC>(g, ep, s) : launch_tile<32, 2, 2, 4, AKC, BKC, VEC>(g, ep, s);
  if (tiles(32) > 1024) {      // (up to 512 tiles of 64 x 64: the same two reasons, tiled | 32/4 | taken)
    // rows  1210 x 1300 x 8: 10.6 | 12.1 | tiled      k  1210 x 1300 x 255: 43 | 58 | 32x64/1 37   x 1025: 220 | 149 | 111
    if (!AKC && !BKC && K <= 16)
      return launch_tiled(g.A, 1, g.lda, g.B, 1, g.ldb, g.M, g.N, g.K, g.nsplit, g.slab, ep, s);
    if (AKC && BKC && !VEC && K > 128) return launch_tile<32, 1, 2, 1, AKC, BKC, VEC>(g, ep, s);
  }
  if (tiles(16) <= (K <= 128 ? 1024 : 512))
    return K >= 512 ? launch_tile<16, 1, 1, 16, AKC, BKC, VEC>(g, ep, s) : launch_tile<16, 1, 1, 4, AKC, BKC, VEC>(g, ep, s);
  if (K <= 128 || tiles(32) > 1024) return launch_tile<32, 1, 1, 4, AKC, BKC, VEC>(g, ep, s);
  return tiles(32) > 256 ? launch_tile<32, 1, 1, 8, AKC, BKC, VEC>(g, ep, s) : launch_tile<32, 1, 1, 16, AKC, BKC, VEC>(g, ep, s);
}

}  // namespace

// Slices of the contraction beyond what a workgroup's wavefronts take: only for very long contractions
// of few tiles (the input gradient of a wide output layer).
int gemm_f32_pick_split(int M, int N, int K) {
  const int64_t tiles = (int64_t)((M + 31) / 32) * ((N + 31) / 32);
  int split = 1;
  while (tiles * split < 128 && K / (split * 2) >= 1024 && split < 32) split *= 2;
  return split;
}

int launch_gemm_f32(const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbn,
                    int64_t sbk, int M, int N, int K, int nsplit, int64_t slab_stride,
                    const Epilogue& ep, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0 || !A || !B || !ep.C || ep.c_is_bf16 || nsplit < 1) return VF_EINVAL;
  if (nsplit > 1 && ep.R) return VF_EINVAL;
  const bool akc = sak == 1, bkc = sbk == 1;
  if ((!akc && sam != 1) || (!bkc && sbn != 1)) return VF_EINVAL;
  F32Shape g{A, akc ? sam : sak, B, bkc ? sbn : sbk, M, N, K, nsplit, slab_stride};
  // What a workgroup's loads reach: 64 rows of an operand contiguous along k (pitches of 32 MB and more are out of
  // reach), or the whole contraction of one contiguous along its rows (any weight of 2 GiB and more).  Out of
  // 32-bit reach the tiled kernel takes them (64 x 32768 x 16384, a weight of 2 GiB: 3.9 ms; one thread per output
  // 27 ms).
  auto near = [&](bool kc, int64_t ld, int rows) { return (kc ? 64 * ld + K : (int64_t)K * ld + rows) * 4 < ((int64_t)1 << 31); };
  if (!near(akc, g.lda, M) || !near(bkc, g.ldb, N)) {
    return launch_tiled(A, sam, sak, B, sbn, sbk, M, N, K, nsplit, slab_stride, ep, s);
  }
  auto al = [](const float* p, int64_t ld) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && (ld & 3) == 0; };
  const bool vec = (K & 3) == 0 && (!akc || al(A, g.lda)) && (!bkc || al(B, g.ldb));
  if (akc && bkc) return vec ? launch_operands<true, true, true>(g, ep, s) : launch_operands<true, true, false>(g, ep, s);
  if (akc) return vec ? launch_operands<true, false, true>(g, ep, s) : launch_operands<true, false, false>(g, ep, s);
  if (!bkc) return launch_operands<false, false, false>(g, ep, s);
  return launch_operands<false, true, false>(g, ep, s);
}

}  // namespace vf
