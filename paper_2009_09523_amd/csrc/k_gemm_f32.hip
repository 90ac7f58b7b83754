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
#include <algorithm>

#include "vf_device.h"

namespace vf {
namespace {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x16v __attribute__((ext_vector_type(16)));

constexpr int GU = 4;        // chunks of the contraction per group
// Contractions from which rows that allow no aligned vectors are read with unaligned ones (36 x 256 x 4099 in four slices:
// scalar loads 24.4 us, unaligned vectors 9.5; 100 x 500 x 10: 6.0, 9.3).
constexpr int kUnalignedK = 64;
constexpr uint32_t kOutside = 0x80000000u;   // an offset beyond every buffer: the load returns 0

// One lane's part of an operand: T row tiles of MS rows, this lane's row of each.  A chunk is 4 * 64 / MS
// contraction elements: the q-th copy of the rows among the lanes (q = lane / MS) holds elements 4 q .. 4 q + 3
// of it, and MFMA step s contracts element s of every copy (any assignment of k to steps will do as long as
// both operands use the same one).  A group is G chunks.  KC: the operand is contiguous along k; VEC: in
// 16-byte vectors, 1 (rows 16-byte aligned, K % 4 == 0) or 2 (any rows of at least four elements).  Loads go through a buffer descriptor over the operand
// from the workgroup's first row on: what lies outside the matrix (rows, or k at and beyond K) is asked for
// beyond the buffer's end and comes back as 0, so there are neither branches nor selections around the loads
// and the compiler keeps a whole group's in flight.
template <int MS, int T, bool KC, int VEC, int G>
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
  // The group of contraction elements k0 .. k0 + G * CK - 1 (k0 the same for the whole wavefront).
  __device__ __forceinline__ void load(float (&v)[G][T][4], int k0) const {
    const int left = K - k0 - kl;                        // elements of this lane from its first one on
    // (a chunk that starts past the end: nothing is fetched, and its scalar offset stays inside the buffer, so that
    // the bounds check -- lane offset against the buffer's size, with or without the scalar offset -- is the same)
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if (KC && VEC == 1) {
          typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
          const u32x4v q = __builtin_amdgcn_raw_buffer_load_b128(buf, CK * u < left ? off[t] : kOutside,
                                                              min(k0 + CK * u, K - 1) * 4, 0);
#pragma unroll
          for (int s = 0; s < 4; ++s) v[u][t][s] = __uint_as_float(q[s]);
        } else if (KC && VEC == 2) {
          typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
          const int rest = left - CK * u;                // elements from this vector's first one to the end of the row
          // (a vector that reaches past the row's end is read so that it ends there, and moved into place: rows need no
          // alignment beyond their elements' own, and the contraction no multiple of 4)
          const uint32_t back = rest < 4 ? 16u - 4u * (uint32_t)max(rest, 0) : 0u;
          const uint32_t o = rest > 0 && off[t] != kOutside ? off[t] + 4u * (uint32_t)min(k0 + CK * u, K - 1) - back : kOutside;
          const u32x4v q = __builtin_amdgcn_raw_buffer_load_b128(buf, o, 0, 0);
          v[u][t][0] = __uint_as_float(rest >= 4 ? q[0] : rest == 3 ? q[1] : rest == 2 ? q[2] : q[3]);
          v[u][t][1] = __uint_as_float(rest >= 4 ? q[1] : rest == 3 ? q[2] : rest == 2 ? q[3] : 0u);
          v[u][t][2] = __uint_as_float(rest >= 4 ? q[2] : rest == 3 ? q[3] : 0u);
          v[u][t][3] = __uint_as_float(rest >= 4 ? q[3] : 0u);
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

// A wavefront's share of a tile's product: the contraction elements [kbeg, kend), added to acc.
template <int MS, int TM, int TN, bool AKC, bool BKC, int VEC, int G>
__device__ __forceinline__ void slice_product(typename Mfma<MS>::acc_t (&acc)[TM][TN], const float* __restrict__ A, int64_t lda,
                                              const float* __restrict__ B, int64_t ldb, int M, int N, int K, int m0, int n0,
                                              int kbeg, int kend, int lane) {
  constexpr int GK = G * 4 * (64 / MS);                  // contraction elements of a group
  const int groups = kend > kbeg ? (kend - kbeg + GK - 1) / GK : 0;
  if (groups <= 0) return;
  Operand<MS, TM, AKC, VEC, G> oa;
  Operand<MS, TN, BKC, VEC, G> ob;
  oa.init(A, lda, m0, M, K, lane);
  ob.init(B, ldb, n0, N, K, lane);
  float a0[G][TM][4], b0[G][TN][4], a1[G][TM][4], b1[G][TN][4];
  auto multiply = [&](const float (&a)[G][TM][4], const float (&b)[G][TN][4]) {
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<MS>::mul(a[u][i][s], b[u][j][s], acc[i][j]);
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

// blockIdx.z selects the contraction slice [z * kslab, (z + 1) * kslab); slice z writes its partial product
// to slab z of C (the consumer adds the slabs in order), the bias goes to slab 0.  Wavefront w of a
// workgroup takes the elements [w * kwave, (w + 1) * kwave) of the slice (kwave and kslab multiples of a group).
// GELU: the epilogue's activation is GELU instead of ReLU (in a kernel of its own: its registers would cost the others a
// workgroup per compute unit, 100 x 1000 x 784 in a step 8.8 -> 11 us).
template <int MS, int TM, int TN, int NW, bool AKC, bool BKC, int VEC, bool GELU>
__global__ __launch_bounds__(NW * 64) void gemm_f32_mfma_kernel(const float* __restrict__ A, int64_t lda,
                                                                const float* __restrict__ B, int64_t ldb,
                                                                int M, int N, int K, int kslab, int kwave,
                                                                int64_t slab_stride, Epilogue ep) {
  typedef Mfma<MS> MF;
  constexpr int R = MF::R;
  constexpr int E = TM * TN * MS * MS;                   // elements of the tile
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

  slice_product<MS, TM, TN, AKC, BKC, VEC, GU>(acc, A, lda, B, ldb, M, N, K, m0, n0, kbeg, kend, lane);

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
  float add[PER], gate[PER];
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
    gate[p] = ep.gate ? ep.gate[(int64_t)m * ep.ldg + n] : 0.f;
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
    const float v = fmaf(ep.alpha, sum, add[p]);
    C[(int64_t)mm[p] * ep.ldc + nn[p]] = !ep.gate ? v : GELU ? v * gelu_df(gate[p]) : gate[p] > 0.f ? v : 0.f;
    if (ep.act) ep.act[(int64_t)mm[p] * ep.ldact + nn[p]] = GELU ? gelu_f(v) : fmaxf(v, 0.f);
  }
}

// ---- one node's product with its BatchNorm pass ---------------------------------------------------
// A node of up to 128 rows: a workgroup takes ALL its rows of 16 columns (TM tiles of 16 rows), so the columns' sums over
// the node stay inside it and the BatchNorm + ReLU pass needs no launch of its own (4 us behind a product of 5 to 10).
// Eight wavefronts cut the contraction among themselves as above; bound by the trips to memory and, with only N / 16
// workgroups, by the fp32 matrix rate of their compute units, hence the limit on rows times contraction (f32_bn_takes).
// The arithmetic is that of bn_relu_fwd_kernel / bn_relu_bwd_kernel.
constexpr int BN_NW = 8;

template <int TM, bool BKC, int VEC, bool BWD>
__global__ __launch_bounds__(BN_NW * 64) void gemm_f32_bn_kernel(const float* __restrict__ A, int64_t lda,
                                                                 const float* __restrict__ B, int64_t ldb, int R, int N,
                                                                 int K, int kwave, F32BnArgs f) {
  constexpr int E = TM * 256, NT = BN_NW * 64, PER = E / NT;
  __shared__ float part[BN_NW * E];
  __shared__ float red[2][BN_NW][16];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * 16, n = n0 + (lane & 15), nc = min(n, N - 1);
  // element p of this thread: element p * NT + tid of the tile in register order (tile row f / 4, register f % 4)
  int mm[PER];
  float zz[PER];
  const float g = f.gamma[nc], b = f.beta[nc];
  float mean = 0.f, rstd = 1.f, rm = 0.f, rv = 0.f;
  if (BWD) { mean = f.mean[nc]; rstd = f.rstd[nc]; }
  else if (f.run_mean) { rm = f.run_mean[nc]; rv = f.run_var[nc]; }
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * BN_NW + wave;
    mm[p] = 16 * (e >> 2) + 4 * (lane >> 4) + (e & 3);
    zz[p] = BWD ? f.z[(int64_t)min(mm[p], R - 1) * f.ldz + nc] : 0.f;
  }
  f32x4v acc[TM][1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][0][r] = 0.f;
  slice_product<16, TM, 1, true, BKC, VEC, 2>(acc, A, lda, B, ldb, R, N, K, 0, n0, wave * kwave, min(K, (wave + 1) * kwave), lane);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave * E + (i * 4 + r) * 64 + lane] = acc[i][0][r];
  __syncthreads();
  float v[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    v[p] = part[p * NT + tid];
#pragma unroll
    for (int w = 1; w < BN_NW; ++w) v[p] += part[w * E + p * NT + tid];
  }
  // sum over the node's rows of this thread's column, to every thread of the column
  auto column_sum = [&](float s, int k) {
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < 16) red[k][wave][lane] = s;
    __syncthreads();
    float t = red[k][0][lane & 15];
#pragma unroll
    for (int w = 1; w < BN_NW; ++w) t += red[k][w][lane & 15];
    return t;
  };
  const bool mine = n < N;
  if (!BWD) {
    float s = 0.f;
#pragma unroll
    for (int p = 0; p < PER; ++p) s += mm[p] < R ? v[p] : 0.f;
    mean = column_sum(s, 0) / (float)R;
    float q = 0.f;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const float d = mm[p] < R ? v[p] - mean : 0.f;
      q = fmaf(d, d, q);
    }
    const float var = column_sum(q, 1) / (float)R;
    rstd = 1.0f / sqrtf(var + f.eps);
    if (mine && tid < 16) {
      f.mean[n] = mean; f.rstd[n] = rstd;
      if (f.run_mean) {
        f.run_mean[n] = fmaf(f.run_mix, mean - rm, rm);
        f.run_var[n] = fmaf(f.run_mix, var - rv, rv);
      }
    }
#pragma unroll
    for (int p = 0; p < PER; ++p)
      if (mine && mm[p] < R) {
        f.z[(int64_t)mm[p] * f.ldz + n] = v[p];
        f.out[(int64_t)mm[p] * f.ldo + n] = fmaxf(bn_pre(g, (v[p] - mean) * rstd, b), 0.f);
      }
    return;
  }
  float sg = 0.f, sb = 0.f;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const float xhat = (zz[p] - mean) * rstd;
    const bool on = mm[p] < R && bn_pre(g, xhat, b) > 0.f;
    zz[p] = mm[p] < R ? xhat : 0.f;
    v[p] = on ? v[p] : 0.f;
    sg = fmaf(v[p], zz[p], sg);
    sb += v[p];
  }
  sg = column_sum(sg, 0);
  sb = column_sum(sb, 1);
  if (mine && tid < 16) {
    grad_store(f.gout_g, n, sg);
    grad_store(f.gout_b, n, sb);
  }
  const float invR = 1.0f / (float)R, kk = g * rstd;
#pragma unroll
  for (int p = 0; p < PER; ++p)
    if (mine && mm[p] < R) f.out[(int64_t)mm[p] * f.ldo + n] = bn_dz(kk, v[p], zz[p], sg, sb, invR);
}

// ---- the last layer's product with the loss -------------------------------------------------------------
// Few classes (TN tiles of 16): a workgroup takes all logits of 16 rows, so the softmax cross-entropy needs no launch of its
// own.  The logits pass through LDS; 32 lanes take a row.  What is computed is what softmax_xent_kernel computes.
template <int TN, int VEC>
__global__ __launch_bounds__(512) void gemm_f32_xent_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ B,
                                                            int64_t ldb, int R, int N, int K, int kwave,
                                                            const float* __restrict__ bias, const int32_t* __restrict__ labels,
                                                            float* __restrict__ z, int64_t ldz, float* __restrict__ dz,
                                                            int64_t lddz, float* __restrict__ rowloss) {
  constexpr int NW = 8, E = TN * 256, NT = NW * 64, PER = (E + NT - 1) / NT, CPL = (16 * TN + 31) / 32;
  __shared__ float part[NW * E];
  __shared__ float logit[16][16 * TN + 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * 16;
  const int row = tid >> 5, l = tid & 31, m = m0 + row, mc = min(m, R - 1);
  const int label = min(max(labels[mc], 0), N - 1);
  float bb[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) bb[p] = bias[min(16 * (((p * NT + tid) >> 6) >> 2) + (lane & 15), N - 1)];
  f32x4v acc[1][TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[0][j][r] = 0.f;
  slice_product<16, 1, TN, true, false, VEC, TN <= 2 ? 4 : 2>(acc, A, lda, B, ldb, R, N, K, m0, 0, wave * kwave,
                                                              min(K, (wave + 1) * kwave), lane);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave * E + (j * 4 + r) * 64 + lane] = acc[0][j][r];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * NT + tid;
    if (E % NT && e >= E) break;
    float v = part[e];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += part[w * E + e];
    const int f = e >> 6;
    logit[4 * (lane >> 4) + (f & 3)][16 * (f >> 2) + (lane & 15)] = v + bb[p];
  }
  __syncthreads();
  float v[CPL], mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    const int c = l + 32 * k;
    v[k] = c < N ? logit[row][c] : -INFINITY;
    if (c < N && m < R) z[(int64_t)m * ldz + c] = v[k];
    mx = fmaxf(mx, v[k]);
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    v[k] = expf(v[k] - mx);                              // exp(-inf) = 0 for the padding
    sum += v[k];
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  const float inv = 1.0f / sum, invR = 1.0f / (float)R;
  if (m >= R) return;
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    const int c = l + 32 * k;
    if (c < N) dz[(int64_t)m * lddz + c] = (v[k] * inv - (c == label ? 1.f : 0.f)) * invR;
  }
  if (l == 0) rowloss[m] = logf(sum) + mx - logit[row][label];
}

// ---- the weight and bias gradients of a unit in one launch ------------------------------------------
// They depend on nothing but the unit's activations and output gradients and none of them fills the chip (784 x 256 x 64 is
// 3.6 us, most of it launch): one grid holds the tiles of all layers, a workgroup finding its job from the running totals.
// A job without A is a bias gradient: the sums over the unit's rows of 32 columns of B.  The last workgroup does the loss
// bookkeeping of the step if there is any to do (as loss_reduce_nodes_kernel).
template <int MS>
__global__ __launch_bounds__(256) void gemm_f32_jobs_kernel(F32Jobs jobs, const float* __restrict__ rowloss, LossNodes ln,
                                                            float* __restrict__ node_loss, float* __restrict__ total) {
  typedef Mfma<MS> MF;
  constexpr int R = MF::R, E = MS * MS, NW = 4, PER = E / 256 ? E / 256 : 1;
  __shared__ float part[NW * E];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int j = 0;                                              // (no chain of loads: the totals come with one or two)
#pragma unroll
  for (int i = 0; i < kF32Jobs; ++i) j += (int)blockIdx.x >= jobs.end[i] ? 1 : 0;
  if (j == jobs.count) {
    float acc = ln.first == 0 ? 0.f : *total;
    for (int i = 0; i < ln.count; ++i) {
      float s = 0.f;
      for (int r = tid; r < ln.rows[i]; r += 256) s += rowloss[ln.off[i] + r];
      s = wave_sum(s);
      __syncthreads();
      if (lane == 0) part[wave] = s;
      __syncthreads();
      const float L = (part[0] + part[1] + part[2] + part[3]) / (float)ln.rows[i];
      if (tid == 0) node_loss[ln.first + i] = L;
      acc = fmaf(ln.w[i], L, acc);
    }
    if (tid == 0) *total = acc;
    return;
  }
  const F32Job& job = jobs.job[j];
  const int t = (int)blockIdx.x - (j ? jobs.end[j - 1] : 0);
  const int N = job.N, K = jobs.rows;
  if (!job.A) {
    const int n = t * 32 + (tid & 31), r0 = tid >> 5, nc = min(n, N - 1);
    float s = 0.f;
    int r = r0;
    for (; r + 24 < K; r += 32) {                        // four rows' loads in flight together
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = job.B[(int64_t)(r + 8 * q) * job.ldb + nc];
#pragma unroll
      for (int q = 0; q < 4; ++q) s += x[q];
    }
    for (; r < K; r += 8) s += job.B[(int64_t)r * job.ldb + nc];
    part[r0 * 32 + (tid & 31)] = s;
    __syncthreads();
    if (tid < 32 && n < N) {
      s = part[tid];
#pragma unroll
      for (int q = 1; q < 8; ++q) s += part[q * 32 + tid];
      grad_store(job.out, n, s);
    }
    return;
  }
  const int tiles_n = (N + MS - 1) / MS;
  const int m0 = t / tiles_n * MS, n0 = t % tiles_n * MS;
  typename MF::acc_t acc[1][1];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[0][0][r] = 0.f;
  slice_product<MS, 1, 1, false, false, 0, GU>(acc, job.A, job.lda, job.B, job.ldb, job.M, N, K, m0, n0, wave * jobs.kwave,
                                                   min(K, (wave + 1) * jobs.kwave), lane);
#pragma unroll
  for (int r = 0; r < R; ++r) part[wave * E + r * 64 + lane] = acc[0][0][r];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * 256 + tid, m = m0 + MF::row(e / 64, lane), n = n0 + lane % MS;
    if (m >= job.M || n >= N) continue;
    float sum = part[e];
#pragma unroll
    for (int w = 1; w < NW; ++w) sum += part[w * E + e];
    grad_store(job.out, (int64_t)m * N + n, sum);
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
      const float v = fmaf(ep.alpha, acc[i][j], add);
      const float gate = ep.gate ? ep.gate[(int64_t)m * ep.ldg + n] : 0.f;
      C[(int64_t)m * ep.ldc + n] = !ep.gate ? v : ep.gelu ? v * gelu_df(gate) : gate > 0.f ? v : 0.f;
      if (ep.act) ep.act[(int64_t)m * ep.ldact + n] = ep.gelu ? gelu_f(v) : fmaxf(v, 0.f);
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

template <int MS, int TM, int TN, int NW, bool AKC, bool BKC, int VEC>
int launch_tile(const F32Shape& g, const Epilogue& ep, hipStream_t s) {
  constexpr int GK = GU * 4 * (64 / MS);
  const int kslab = ((g.K + g.nsplit - 1) / g.nsplit + GK - 1) / GK * GK;
  const int kwave = ((kslab + NW - 1) / NW + GK - 1) / GK * GK;
  dim3 grid((g.N + MS * TN - 1) / (MS * TN), (g.M + MS * TM - 1) / (MS * TM), g.nsplit);
  if constexpr (AKC)                                     // (no weight gradient has an activation)
    if (ep.gelu) {
      gemm_f32_mfma_kernel<MS, TM, TN, NW, AKC, BKC, VEC, true><<<grid, NW * 64, 0, s>>>(g.A, g.lda, g.B, g.ldb, g.M, g.N, g.K,
                                                                                         kslab, kwave, g.slab, ep);
      VF_LAUNCH_CHECK();
      return VF_OK;
    }
  if (ep.gelu) return VF_EINVAL;
  gemm_f32_mfma_kernel<MS, TM, TN, NW, AKC, BKC, VEC, false><<<grid, NW * 64, 0, s>>>(g.A, g.lda, g.B, g.ldb, g.M, g.N, g.K,
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
template <bool AKC, bool BKC, int VEC>
int launch_operands(const F32Shape& g, const Epilogue& ep, hipStream_t s) {
  auto tiles = [&](int t) { return (int64_t)((g.M + t - 1) / t) * ((g.N + t - 1) / t) * g.nsplit; };
  const int K = g.K / g.nsplit;
  const int64_t t64 = tiles(64);
  if constexpr (VEC == 2) {
    if (t64 >= 512 || tiles(32) > 1024) return launch_operands<AKC, BKC, 0>(g, ep, s);   // (what was measured above)
  } else if (t64 > 512) {
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
  if constexpr (VEC != 2) {
    if (t64 == 512)
      return K <= 32 ? launch_tile<32, 1, 1, 1, AKC, BKC, VEC>(g, ep, s) : launch_tile<32, 2, 2, 4, AKC, BKC, VEC>(g, ep, s);
    if (tiles(32) > 1024) {    // (up to 512 tiles of 64 x 64: the same two reasons, tiled | 32/4 | taken)
      // rows  1210 x 1300 x 8: 10.6 | 12.1 | tiled      k  1210 x 1300 x 255: 43 | 58 | 32x64/1 37   x 1025: 220 | 149 | 111
      if (!AKC && !BKC && K <= 16)
        return launch_tiled(g.A, 1, g.lda, g.B, 1, g.ldb, g.M, g.N, g.K, g.nsplit, g.slab, ep, s);
      if (AKC && BKC && !VEC && K > 128) return launch_tile<32, 1, 2, 1, AKC, BKC, VEC>(g, ep, s);
    }
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
  const int vec = (K & 3) == 0 && (!akc || al(A, g.lda)) && (!bkc || al(B, g.ldb)) ? 1 : K >= kUnalignedK ? 2 : 0;
#define VF_F32_OPS(A_, B_) \
  return vec == 1 ? launch_operands<A_, B_, 1>(g, ep, s) : vec == 2 ? launch_operands<A_, B_, 2>(g, ep, s) : launch_operands<A_, B_, 0>(g, ep, s)
  if (akc && bkc) VF_F32_OPS(true, true);
  if (akc) VF_F32_OPS(true, false);
#undef VF_F32_OPS
  if (!bkc) return launch_operands<false, false, 0>(g, ep, s);
  return launch_operands<false, true, 0>(g, ep, s);
}

// What a workgroup's loads reach in 32-bit byte offsets: 64 (128) rows of an operand contiguous along k, or the whole
// contraction of one contiguous along its rows.
static bool near32(bool kc, int64_t ld, int rows, int K) {
  return (kc ? 128 * ld + K : (int64_t)K * ld + rows) * 4 < ((int64_t)1 << 31);
}

// Rows (rounded up to 32) times contraction that a workgroup of the fused kernel takes: a node's product is cut by columns
// only, so with long contractions of many rows its few workgroups cost more than the BatchNorm launch they save.  Steps of
// K-N-N-10 networks of three nodes, launches apart | fused (us): 16 rows, N = 64, K = 1000 115 | 86; 32 rows, N = 1000,
// K = 1000 193 | 180; 64 rows, N = 256, K = 256 124 | 104, K = 512 111 | 118; 100 rows, N = 500, K = 64 131 | 129, K = 256 136 | 171.
// And while the columns are not so many that a compute unit has several workgroups, each reading all rows again (rows times
// columns; forward, where the columns are strided, also columns times contraction).  Forward, K-N-10, three nodes: 8 rows,
// K = 1024, N = 8192 216 | 199, N = 16384 304 | 316; 64 rows, K = 256, N = 16384 222 | 219; 128 rows, K = 128, N = 8192
// 150 | 148, N = 16384 226 | 242.  Backward, 64-N-K: 8 rows, K = 1024, N = 16384 403 | 392; 96 rows, K = 170, N = 16384
// 354 | 324; 128 rows, K = 128, N = 16384 318 | 319.
bool f32_bn_takes(int R, int N, int K, int64_t lda, int64_t ldb, bool backward) {
  if (R < 1 || R > 128 || N < 1 || K < 1) return false;
  const int64_t rows = (R + 31) / 32 * 32;
  if (rows * N > (backward ? 3 << 19 : 1 << 20) || (!backward && (int64_t)N * K > 1 << 23)) return false;
  return rows * K <= (R <= 32 ? 32768 : 16384) && near32(true, lda, R, K) && near32(backward, ldb, N, K);
}

int launch_gemm_f32_bn(const float* A, int64_t lda, const float* B, int64_t ldb, int R, int N, int K, bool backward,
                       const F32BnArgs& f, hipStream_t s) {
  if (!A || !B || !f.gamma || !f.beta || !f.mean || !f.rstd || !f.z || !f.out || (f.run_mean == nullptr) != (f.run_var == nullptr) ||
      (backward && (!f.gout_g.dst || !f.gout_b.dst)) || !f32_bn_takes(R, N, K, lda, ldb, backward))
    return VF_EINVAL;
  auto al = [](const float* p, int64_t ld) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && (ld & 3) == 0; };
  const int vec = (K & 3) == 0 && al(A, lda) && (!backward || al(B, ldb)) ? 1 : K >= kUnalignedK ? 2 : 0;
  const int kwave = ((K + BN_NW - 1) / BN_NW + 31) / 32 * 32;
  const int grid = (N + 15) / 16;
#define VF_F32BN2(TM, VEC)                                                                                              \
  if (backward) gemm_f32_bn_kernel<TM, true, VEC, true><<<grid, BN_NW * 64, 0, s>>>(A, lda, B, ldb, R, N, K, kwave, f); \
  else gemm_f32_bn_kernel<TM, false, VEC, false><<<grid, BN_NW * 64, 0, s>>>(A, lda, B, ldb, R, N, K, kwave, f)
#define VF_F32BN(TM) if (vec == 1) { VF_F32BN2(TM, 1); } else if (vec) { VF_F32BN2(TM, 2); } else { VF_F32BN2(TM, 0); }
  switch ((R + 31) / 32) {
    case 1: VF_F32BN(2) break;
    case 2: VF_F32BN(4) break;
    case 3: VF_F32BN(6) break;
    default: VF_F32BN(8) break;
  }
#undef VF_F32BN
#undef VF_F32BN2
  VF_LAUNCH_CHECK();
  return VF_OK;
}

// Classes (rounded up to 16) times contraction that a workgroup of the kernel with the loss takes: it is cut by rows only.
bool f32_xent_takes(int R, int N, int K, int64_t lda, int64_t ldb) {
  return R >= 1 && N >= 1 && K >= 1 && N <= 128 && (int64_t)((N + 15) / 16 * 16) * K <= 32768 && near32(true, lda, R, K) &&
         near32(false, ldb, N, K);
}

int launch_gemm_f32_xent(const float* A, int64_t lda, const float* B, int64_t ldb, int R, int N, int K, const float* bias,
                         const int32_t* labels, float* z, int64_t ldz, float* dz, int64_t lddz, float* rowloss, hipStream_t s) {
  if (!A || !B || !bias || !labels || !z || !dz || !rowloss || !f32_xent_takes(R, N, K, lda, ldb)) return VF_EINVAL;
  const int vec = (K & 3) == 0 && (lda & 3) == 0 && (reinterpret_cast<uintptr_t>(A) & 15) == 0 ? 1 : K >= kUnalignedK ? 2 : 0;
  const int tn = (N + 15) / 16, gk = (tn <= 2 ? 4 : 2) * 16;
  const int kwave = ((K + 7) / 8 + gk - 1) / gk * gk;
  const int grid = (R + 15) / 16;
#define VF_XENT(TN)                                                                                                        \
  if (vec == 1) gemm_f32_xent_kernel<TN, 1><<<grid, 512, 0, s>>>(A, lda, B, ldb, R, N, K, kwave, bias, labels, z, ldz, dz, lddz, rowloss); \
  else if (vec) gemm_f32_xent_kernel<TN, 2><<<grid, 512, 0, s>>>(A, lda, B, ldb, R, N, K, kwave, bias, labels, z, ldz, dz, lddz, rowloss); \
  else gemm_f32_xent_kernel<TN, 0><<<grid, 512, 0, s>>>(A, lda, B, ldb, R, N, K, kwave, bias, labels, z, ldz, dz, lddz, rowloss)
  if (tn <= 1) { VF_XENT(1); }
  else if (tn <= 2) { VF_XENT(2); }
  else if (tn <= 4) { VF_XENT(4); }
  else { VF_XENT(8); }
#undef VF_XENT
  VF_LAUNCH_CHECK();
  return VF_OK;
}

// Up to 512 contraction elements and as many tiles as a launch of one layer takes without sharing wavefronts out
// differently (launch_operands); 16 x 16 tiles while they are few.
bool f32_jobs_take(const F32Jobs& jobs) {
  if (jobs.count < 1 || jobs.count > kF32Jobs || jobs.rows < 1 || jobs.rows > 512) return false;
  int64_t t64 = 0;
  for (int j = 0; j < jobs.count; ++j) {
    const F32Job& g = jobs.job[j];
    if (!g.B || !g.out.dst || g.N < 1 || !near32(false, g.ldb, g.N, jobs.rows)) return false;
    if (g.A && (g.M < 1 || !near32(false, g.lda, g.M, jobs.rows))) return false;
    if (g.A) t64 += (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64);
  }
  return t64 <= 512;
}

int launch_gemm_f32_jobs(F32Jobs jobs, const float* rowloss, const LossNodes& ln, float* node_loss, float* total, hipStream_t s) {
  if (!f32_jobs_take(jobs) || ln.count < 0 || ln.count > kLossNodes || (ln.count && (!rowloss || !node_loss || !total)))
    return VF_EINVAL;
  int64_t t16 = 0;
  for (int j = 0; j < jobs.count; ++j)
    if (jobs.job[j].A) t16 += (int64_t)((jobs.job[j].M + 15) / 16) * ((jobs.job[j].N + 15) / 16);
  const int ms = t16 <= (jobs.rows <= 128 ? 1024 : 512) ? 16 : 32;
  int end = 0;
  for (int j = 0; j < jobs.count; ++j) {
    const F32Job& g = jobs.job[j];
    end += g.A ? ((g.M + ms - 1) / ms) * ((g.N + ms - 1) / ms) : (g.N + 31) / 32;
    jobs.end[j] = end;
  }
  for (int j = jobs.count; j < kF32Jobs; ++j) jobs.end[j] = 0x7fffffff;
  const int gk = GU * 4 * (64 / ms);
  jobs.kwave = ((jobs.rows + 3) / 4 + gk - 1) / gk * gk;
  const int grid = end + (ln.count ? 1 : 0);
  if (ms == 16) gemm_f32_jobs_kernel<16><<<grid, 256, 0, s>>>(jobs, rowloss, ln, node_loss, total);
  else gemm_f32_jobs_kernel<32><<<grid, 256, 0, s>>>(jobs, rowloss, ln, node_loss, total);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

}  // namespace vf
