// Layout kernels: bf16 transposes and the fp32 -> bf16 weight copies the GEMMs read.
#include "vf_device.h"

namespace vf {
namespace {

constexpr int TS = 32;   // tile side; 256 threads = 32 x 8
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// out[c*ldo + r] = in[r*ldi + c]
__global__ __launch_bounds__(256) void transpose_kernel(const bf16_t* __restrict__ in, int64_t ldi,
                                                        bf16_t* __restrict__ out, int64_t ldo, int R, int C) {
  __shared__ bf16_t tile[TS][TS + 2];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = blockIdx.y * TS, c0 = blockIdx.x * TS;
#pragma unroll
  for (int i = 0; i < TS; i += 8) {
    int r = r0 + ty + i, c = c0 + tx;
    if (r < R && c < C) tile[ty + i][tx] = in[(int64_t)r * ldi + c];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TS; i += 8) {
    int c = c0 + ty + i, r = r0 + tx;
    if (r < R && c < C) out[(int64_t)c * ldo + r] = tile[tx][ty + i];
  }
}

// out[c*ldo + r] = in[r*ldi + c] for bf16, 64x64 tiles, 16 bytes per lane on both sides (eight
// lanes cover 128 contiguous bytes of an input row, and of an output row).  Loads go to clamped,
// always valid addresses and come first, so both of a thread's loads are in flight together.
// Requires ldi % 8 == 0, ldi >= C rounded up to 8 (what lies there is read and dropped), ldo % 8 == 0, 16-byte aligned
// bases, and output rows that may be written up to R rounded to 8 (the rows past R receive copies of row R-1).
__device__ __forceinline__ void transpose64_body(const bf16_t* __restrict__ in, int64_t ldi,
                                                 bf16_t* __restrict__ out, int64_t ldo, int R, int C, int bx, int by) {
  __shared__ __attribute__((aligned(16))) bf16_t tile[64][kTransposePitch];
  const int r0 = by * 64, c0 = bx * 64;
  const int v = threadIdx.x & 7, row = threadIdx.x >> 3;     // 8 vectors per row, 32 rows per pass
  u32x4 x[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    x[i] = *reinterpret_cast<const u32x4*>(&in[(int64_t)min(r0 + row + 32 * i, R - 1) * ldi + min(c0 + 8 * v, ((C + 7) & ~7) - 8)]);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(&tile[row + 32 * i][8 * v + 2 * e]) = x[i][e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int col = (threadIdx.x >> 3) + 32 * i;             // output row = input column
    const int rb = 8 * (threadIdx.x & 7);                    // eight input rows -> one 16-byte vector
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = (uint32_t)tile[rb + 2 * e][col] | ((uint32_t)tile[rb + 2 * e + 1][col] << 16);
    if (c0 + col < C && r0 + rb < R)
      *reinterpret_cast<u32x4*>(&out[(int64_t)(c0 + col) * ldo + r0 + rb]) = o;
  }
}

__global__ __launch_bounds__(256) void transpose64_kernel(const bf16_t* __restrict__ in, int64_t ldi,
                                                          bf16_t* __restrict__ out, int64_t ldo, int R, int C) {
  transpose64_body(in, ldi, out, ldo, R, C, blockIdx.x, blockIdx.y);
}
// Several matrices of R rows in one launch: blockIdx.x runs over the column tiles of all of them.
__global__ __launch_bounds__(256) void transpose64_jobs_kernel(TransposeJobs tj) {
  int j = 0, first = 0;
  while (j < tj.count - 1 && (int)blockIdx.x >= first + (tj.C[j] + 63) / 64) { first += (tj.C[j] + 63) / 64; ++j; }
  transpose64_body(tj.in[j], tj.ldi[j], tj.out[j], tj.ldo, tj.R, tj.C[j], blockIdx.x - first, blockIdx.y);
}

// fp32 [R, C] -> bf16 natural copy [R, ldn] and transposed copy [C, ldt], 64x64 tiles, of several matrices in one launch
// (blockIdx.x runs over their tiles; up to 17 launches of 5 us otherwise).  Every thread reads 16 bytes and writes 8 bytes at a time in both
// orientations; rows of C elements that are no multiple of 4, or unaligned, are read element by element (768 x 30522: 54 us by 32 x 32
// tiles of single elements; with sixteen matrices of 28 million elements beside it 74 here).  Requires ldn, ldt % 4 == 0, ldn >= C rounded up to 4, ldt >= R rounded up to 4
// (the padding receives zeros), nat and tr 8-byte aligned.  MAX is 1 where a matrix goes alone (an MLP's layers): the list of
// sixteen is 1.1 KB of arguments, which cost the host 1 us a launch (98 rows of seven layers, bound by launches: 293 | 287 us).
template <int MAX>
__global__ __launch_bounds__(256) void cast_weight_kernel(CastJobList<MAX> jobs) {
  __shared__ bf16_t tile[64][64 + 2];
  int j = 0;
#pragma unroll
  for (int i = 0; i < MAX && MAX > 1; ++i) j += (int)blockIdx.x >= jobs.end[i] ? 1 : 0;
  const CastJob& job = jobs.job[j];
  const int R = job.R, C = job.C;
  const float* __restrict__ in = job.in;
  const int t = (int)blockIdx.x - (j ? jobs.end[j - 1] : 0), tiles_c = (C + 63) / 64;
  const int q = threadIdx.x & 15, g = threadIdx.x >> 4;      // 16 quads per row, 16 row groups
  const int r0 = t / tiles_c * 64, c0 = t % tiles_c * 64;
  // loads at clamped (always valid) positions first, all in flight together
  float4 vin[4];
  if (job.vec) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      vin[i] = load4_stream(&in[(int64_t)min(r0 + g + 16 * i, R - 1) * C + min(c0 + 4 * q, C - 4)]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* p = &in[(int64_t)min(r0 + g + 16 * i, R - 1) * C];
      const int c = c0 + 4 * q;
      vin[i] = make_float4(p[min(c, C - 1)], p[min(c + 1, C - 1)], p[min(c + 2, C - 1)], p[min(c + 3, C - 1)]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = g + 16 * i, r = r0 + rl, c = c0 + 4 * q;
    const float v[4] = {vin[i].x, vin[i].y, vin[i].z, vin[i].w};
    bf16_t h[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) h[u] = r < R && c + u < C ? f32_to_bf16(v[u]) : (bf16_t)0;
    if (r < R && c < C) {
      uint2 pk;
      pk.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
      pk.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
      *reinterpret_cast<uint2*>(&job.nat[(int64_t)r * job.ldn + c]) = pk;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) tile[rl][4 * q + u] = h[u];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int cl = g + 16 * i, c = c0 + cl, r = r0 + 4 * q;
    if (c < C && r < R) {      // R % 4 == 0 is not required: rows past R inside the quad are padding of ldt
      uint2 pk;
      pk.x = (uint32_t)tile[4 * q][cl] | ((uint32_t)tile[4 * q + 1][cl] << 16);
      pk.y = (uint32_t)tile[4 * q + 2][cl] | ((uint32_t)tile[4 * q + 3][cl] << 16);
      *reinterpret_cast<uint2*>(&job.tr[(int64_t)c * job.ldt + r]) = pk;
    }
  }
}

// The same transpose for every node of a fold window (blockIdx.z = node).  pad: the columns past a node's rows, up to the
// next multiple of 8, are written as 0.
__global__ __launch_bounds__(256) void transpose_nodes_kernel(NodeList nl, int64_t ldi, int64_t ldo, int C, int pad) {
  __shared__ bf16_t tile[TS][TS + 2];
  const int j = blockIdx.z;
  const int R = nl.rows[j], W = pad ? (R + 7) & ~7 : R;
  const int r0 = blockIdx.y * TS, c0 = blockIdx.x * TS;
  if (r0 >= R) return;
  const bf16_t* __restrict__ in = nl.src[j];
  bf16_t* __restrict__ out = nl.dst[j];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int i = 0; i < TS; i += 8) {
    const int r = r0 + ty + i, c = c0 + tx;
    if (c < C) tile[ty + i][tx] = r < R ? in[(int64_t)r * ldi + c] : (bf16_t)0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TS; i += 8) {
    const int c = c0 + ty + i, r = r0 + tx;
    if (r < W && c < C) out[(int64_t)c * ldo + r] = tile[tx][ty + i];
  }
}

__global__ __launch_bounds__(256) void cast_kernel(const float* __restrict__ in, int64_t ldi,
                                                   bf16_t* __restrict__ out, int64_t ldo, int R, int C) {
  int c = blockIdx.x * 256 + threadIdx.x;
  int r = blockIdx.y;
  if (c < C) out[(int64_t)r * ldo + c] = f32_to_bf16(in[(int64_t)r * ldi + c]);
}

}  // namespace

int launch_transpose_bf16(const bf16_t* in, int64_t ldi, bf16_t* out, int64_t ldo, int R, int C,
                          hipStream_t s) {
  if (R <= 0 || C <= 0) return VF_OK;
  const bool wide = ldi >= ((C + 7) & ~7) && (ldi & 7) == 0 && (ldo & 7) == 0 && ldo >= ((R + 7) & ~7) &&
                    (reinterpret_cast<uintptr_t>(in) & 15) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  if (wide) {
    dim3 grid64((C + 63) / 64, (R + 63) / 64);
    transpose64_kernel<<<grid64, 256, 0, s>>>(in, ldi, out, ldo, R, C);
    VF_LAUNCH_CHECK();
    return VF_OK;
  }
  dim3 grid((C + TS - 1) / TS, (R + TS - 1) / TS);
  transpose_kernel<<<grid, 256, 0, s>>>(in, ldi, out, ldo, R, C);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

int launch_transpose_bf16_jobs(const TransposeJobs& tj, hipStream_t s) {
  if (tj.count < 1 || tj.count > kTransposeJobs || tj.R <= 0 || (tj.ldo & 7) || tj.ldo < ((tj.R + 7) & ~7)) return VF_EINVAL;
  int tiles = 0;
  for (int j = 0; j < tj.count; ++j) {
    if (!tj.in[j] || !tj.out[j] || tj.C[j] <= 0 || (tj.C[j] & 7) || (tj.ldi[j] & 7) || tj.ldi[j] < tj.C[j] ||
        (reinterpret_cast<uintptr_t>(tj.in[j]) & 15) || (reinterpret_cast<uintptr_t>(tj.out[j]) & 15))
      return VF_EINVAL;
    tiles += (tj.C[j] + 63) / 64;
  }
  dim3 grid(tiles, (tj.R + 63) / 64);
  transpose64_jobs_kernel<<<grid, 256, 0, s>>>(tj);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

int launch_transpose_nodes(const NodeList& nl, int64_t ldi, int64_t ldo, int C, hipStream_t s, bool pad) {
  if (nl.count < 1 || nl.count > kFoldMax || C <= 0) return VF_EINVAL;
  int max_rows = 0;
  for (int j = 0; j < nl.count; ++j) {
    if (!nl.src[j] || !nl.dst[j] || nl.rows[j] < 1 || nl.rows[j] > ldo || C > ldi) return VF_EINVAL;
    max_rows = nl.rows[j] > max_rows ? nl.rows[j] : max_rows;
  }
  dim3 grid((C + TS - 1) / TS, (max_rows + TS - 1) / TS, nl.count);
  transpose_nodes_kernel<<<grid, 256, 0, s>>>(nl, ldi, ldo, C, pad);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

template <int MAX>
static int launch_cast_list(CastJobList<MAX>& jobs, hipStream_t s) {
  if (jobs.count < 1 || jobs.count > MAX) return VF_EINVAL;
  int64_t end = 0;
  for (int j = 0; j < jobs.count; ++j) {
    CastJob& g = jobs.job[j];
    if (!g.in || !g.nat || !g.tr || g.R <= 0 || g.C <= 0 || (g.ldn & 3) || (g.ldt & 3) || g.ldn < ((g.C + 3) & ~3) ||
        g.ldt < ((g.R + 3) & ~3) || (reinterpret_cast<uintptr_t>(g.nat) & 7) || (reinterpret_cast<uintptr_t>(g.tr) & 7))
      return VF_EINVAL;
    g.vec = (g.C & 3) == 0 && (reinterpret_cast<uintptr_t>(g.in) & 15) == 0;
    end += (int64_t)((g.R + 63) / 64) * ((g.C + 63) / 64);
    if (end > 0x7fffffff) return VF_EINVAL;
    jobs.end[j] = (int)end;
  }
  for (int j = jobs.count; j < MAX; ++j) jobs.end[j] = 0x7fffffff;
  cast_weight_kernel<MAX><<<(unsigned)end, 256, 0, s>>>(jobs);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

int launch_cast_weights(CastJobs jobs, hipStream_t s) { return launch_cast_list(jobs, s); }

int launch_cast_weight(const float* w, int R, int C, bf16_t* nat, int64_t ldn, bf16_t* tr, int64_t ldt, hipStream_t s) {
  if (R <= 0 || C <= 0) return VF_OK;
  CastJobList<1> jobs{};
  jobs.job[0] = {w, R, C, nat, ldn, tr, ldt, 0};
  jobs.count = 1;
  return launch_cast_list(jobs, s);
}

int launch_cast_bf16(const float* in, int64_t ldi, bf16_t* out, int64_t ldo, int R, int C,
                     hipStream_t s) {
  if (R <= 0 || C <= 0) return VF_OK;
  dim3 grid((C + 255) / 256, R);
  cast_kernel<<<grid, 256, 0, s>>>(in, ldi, out, ldo, R, C);
  VF_LAUNCH_CHECK();
  return VF_OK;
}

}  // namespace vf
