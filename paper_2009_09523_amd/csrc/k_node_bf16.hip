// One node's bf16 input-gradient product with the BatchNorm + ReLU backward pass (or the ReLU's alone) of the layer it
// arrives at in the same launch, for nodes of up to 128 rows that go through the passes alone.
//
// A workgroup takes ALL the node's rows (TM tiles of 16) of 16 columns, so the columns' sums over the node stay inside it:
// no slabs of partial products, no kernel that reads them.  Its eight wavefronts deal the contraction out among themselves,
// operands straight from memory into the registers of v_mfma_f32_16x16x32_bf16 (every element of the node's rows is used
// once per workgroup, so LDS would only add a trip), two groups of 64 contraction elements in flight; the partial tiles are
// added through LDS in wavefront order.  What bounds it is how fast a compute unit pulls the node's rows out of its XCD's L2,
// for small layers the trips to memory.  The arithmetic behind the product is that of bn_relu_bwd_kernel.
// (The same for the forward pass saved as much again, but adds the products up in another order than units of several nodes
// do, and single bf16 roundings of activations that fall the other way move a node's loss by 1e-5.)
#include <algorithm>

#include "vf_device.h"

namespace vf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NW = 8, NTN = NW * 64;
constexpr int GC = 2;                       // chunks of 32 contraction elements per group
constexpr uint32_t kOutside = 0x80000000u;  // an offset beyond every buffer: the load returns 0

__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand(const bf16_t* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, (int)min(bytes, (int64_t)0x7fffffff), 0x00020000);
}

template <int TM>
__global__ __launch_bounds__(NTN) void gemm_bf16_node_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                             const bf16_t* __restrict__ B, int64_t ldb, int R, int N, int K8,
                                                             NodeBnArgs f) {
  constexpr int E = TM * 256, PER = E / NTN;
  __shared__ float part[NW * E];
  __shared__ float red[2][NW][16];
  __shared__ __attribute__((aligned(16))) bf16_t tile[16][TM * 16 + 8];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  // the workgroups that an XCD receives in a row (b, b + 8, ..) take neighbouring columns
  const int per = (gridDim.x + 7) >> 3;
  const int blk = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  const int n0 = blk * 16, n = n0 + lr, nc = min(n, N - 1);
  if (n0 >= N) return;

  // element p of this thread: element p * NTN + tid of the tile in register order (tile row e / 4, register e % 4)
  int mm[PER];
  float zz[PER];
  const bool bn = f.gamma != nullptr;
  float g = 1.f, b = 0.f, mean = 0.f, rstd = 1.f;
  if (bn) {
    g = round_bf16(f.gamma[nc]); b = round_bf16(f.beta[nc]);
    mean = f.mean[nc]; rstd = f.rstd[nc];
  }
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int e = p * NW + wave;
    mm[p] = 16 * (e >> 2) + 4 * lq + (e & 3);
    zz[p] = f.z[(int64_t)min(mm[p], R - 1) * f.ldz + nc];
  }

  f32x4 acc[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // wavefront w takes the groups w, w + 8, ... (side by side the eight read a run of lines)
  constexpr int GK = 32 * GC;
  const int kbeg = wave * GK;
  if (kbeg < K8) {
    const auto ra = operand(A, ((int64_t)(R - 1) * lda + K8) * 2), rb = operand(B + (int64_t)n0 * ldb, ((int64_t)(min(16, N - n0) - 1) * ldb + K8) * 2);
    uint32_t oa[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) oa[i] = 16 * i + lr < R ? (uint32_t)((16 * i + lr) * lda + 8 * lq) * 2u : kOutside;
    const uint32_t ob = n < N ? (uint32_t)(lr * ldb + 8 * lq) * 2u : kOutside;
    u32x4 a0[GC][TM], b0[GC], a1[GC][TM], b1[GC];
    auto load = [&](u32x4 (&a)[GC][TM], u32x4 (&bb)[GC], int k) {
#pragma unroll
      for (int u = 0; u < GC; ++u) {
        // (past the contraction nothing is fetched, and the scalar offset stays inside the buffer)
        const bool on = k + 32 * u + 8 * lq < K8;
        const int so = min(k + 32 * u, K8 - 8) * 2;
        bb[u] = __builtin_amdgcn_raw_buffer_load_b128(rb, on ? ob : kOutside, so, 0);
#pragma unroll
        for (int i = 0; i < TM; ++i) a[u][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, on ? oa[i] : kOutside, so, 0);
      }
    };
    auto multiply = [&](const u32x4 (&a)[GC][TM], const u32x4 (&bb)[GC]) {
#pragma unroll
      for (int u = 0; u < GC; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][i]), __builtin_bit_cast(bf16x8, bb[u]), acc[i], 0, 0, 0);
    };
    constexpr int STEP = NW * GK;
    const int groups = (K8 - kbeg + STEP - 1) / STEP;
    load(a0, b0, kbeg);
    if (groups > 1) {
      load(a1, b1, kbeg + STEP);
      int k = kbeg;
      for (int q = 0; q + 2 <= groups; q += 2, k += 2 * STEP) {
        __builtin_amdgcn_sched_barrier(0);
        multiply(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        load(a0, b0, k + 2 * STEP);
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        load(a1, b1, k + 3 * STEP);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (groups & 1) multiply(a0, b0);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave * E + (i * 4 + r) * 64 + lane] = acc[i][r];
  __syncthreads();
  float v[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    v[p] = part[p * NTN + tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) v[p] += part[w * E + p * NTN + tid];
  }
  // sum over the node's rows of this thread's column, to every thread of the column
  auto column_sum = [&](float s, int k) {
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < 16) red[k][wave][lane] = s;
    __syncthreads();
    float t = red[k][0][lr];
#pragma unroll
    for (int w = 1; w < NW; ++w) t += red[k][w][lr];
    return t;
  };
  const bool mine = n < N;
  float sg = 0.f, sb = 0.f;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const float xhat = (zz[p] - mean) * rstd;
    const float pre = bn ? bn_pre(g, xhat, b) : zz[p];
    const bool on = mm[p] < R;
    v[p] = on && pre > 0.f ? v[p] : 0.f;
    zz[p] = on ? xhat : 0.f;
    sg = fmaf(v[p], zz[p], sg);
    sb += v[p];
  }
  sg = column_sum(sg, 0);
  sb = column_sum(sb, 1);
  if (mine && tid < 16) {
    if (bn) grad_store(f.gout_g, n, sg);
    if (f.gout_b.dst) grad_store(f.gout_b, n, sb);
  }
  const float invR = 1.0f / (float)R, kk = g * rstd;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    float d = 0.f;
    if (mm[p] < R) {
      d = bn ? bn_dz(kk, v[p], zz[p], sg, sb, invR) : v[p];
      if (mine) f.out[(int64_t)mm[p] * f.ldo + n] = f32_to_bf16(d);
    }
    tile[lr][mm[p]] = f32_to_bf16(d * f.tscale);
  }
  // the transposed copy: 16 columns x TM * 2 vectors of eight rows (rows past R are padding up to a multiple of 8: zeros)
  __syncthreads();
  if (tid < 16 * TM * 2) {
    const int col = tid / (TM * 2), r = tid % (TM * 2) * 8;
    if (n0 + col < N && r < R)
      *reinterpret_cast<u32x4*>(&f.outT[(int64_t)(n0 + col) * f.ldt + r]) = *reinterpret_cast<const u32x4*>(&tile[col][r]);
  }
}

}  // namespace

// Rows (rounded up to 32) times contraction up to which one launch beats the sliced product and the kernel behind it: every
// workgroup reads all of the node's rows.  Steps of four nodes on K-N-K-64 networks, apart | fused (us): 11 rows, N = 256,
// K = 256 232 | 200; 32 rows, N = 512, K = 1024 249 | 224; 64 rows, N = 512, K = 256 220 | 196; 128 rows, N = 512, K = 256
// 228 | 210, N = 256, K = 1024 240 | 248, N = K = 4096 656 | 728.
constexpr int64_t kNodeWork = 49152;
// Rows times columns, and columns times contraction, up to which it does: beyond, a compute unit has several workgroups.
// 64-N-K, four nodes: 32 rows, K = 768, N = 8192 346 | 332, N = 16384 406 | 407, K = 1536 496 | 489, 632 | 656; 64 rows,
// K = 384, N = 8192 206 | 201, N = 16384 326 | 331; 128 rows, K = 384, N = 4096 191 | 185, N = 8192 231 | 241, N = 16384
// 303 | 339.
constexpr int64_t kNodeOut = 1 << 19, kNodeWeights = 1 << 24;

bool node_bn_bwd_takes(const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int R, int N, int K, const NodeBnArgs& f) {
  if (R < 1 || R > 128 || N < 1 || K < 1 || !A || !B || !f.z || !f.out || !f.outT) return false;
  const int64_t K8 = (K + 7) & ~7;
  const int64_t rows = (R + 31) / 32 * 32;
  if (rows * K8 > kNodeWork || rows * N > kNodeOut || N * K8 > kNodeWeights) return false;
  if ((lda & 7) || (ldb & 7) || lda < K8 || ldb < K8 || (f.ldt & 7) || f.ldt < ((R + 7) & ~7)) return false;
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!al(A) || !al(B) || !al(f.outT)) return false;
  if (128 * lda * 2 >= ((int64_t)1 << 31) || 16 * ldb * 2 >= ((int64_t)1 << 31)) return false;
  return !f.gamma || (f.beta && f.mean && f.rstd && f.gout_g.dst);
}

int launch_node_bn_bwd(const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int R, int N, int K, const NodeBnArgs& f,
                   hipStream_t s) {
  if (!node_bn_bwd_takes(A, lda, B, ldb, R, N, K, f)) return VF_EINVAL;
  const int K8 = (K + 7) & ~7;
  const int grid = ((N + 15) / 16 + 7) / 8 * 8;
#define VF_NODE(TM) gemm_bf16_node_kernel<TM><<<grid, NTN, 0, s>>>(A, lda, B, ldb, R, N, K8, f);
  switch ((R + 31) / 32) {
    case 1: VF_NODE(2) break;
    case 2: VF_NODE(4) break;
    case 3: VF_NODE(6) break;
    default: VF_NODE(8) break;
  }
#undef VF_NODE
  VF_LAUNCH_CHECK();
  return VF_OK;
}

}  // namespace vf
