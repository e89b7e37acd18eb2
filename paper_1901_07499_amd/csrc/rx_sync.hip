// rx_sync.hip -- PN-preamble frame synchronisation and slot extraction (gfx950).
//
// The receiver correlates every antenna's stream with the maximum-length PN
// sequence that opens a frame and takes the correlation peak as the start of
// the frame (paper Sec. II-B; Table I: PN length 255):
//   c_a[n] = sum_m p[m] y_a[n+m],   M[n] = sum_a |c_a[n]|^2,
//   offset = the first n with the largest M[n].
// With chips p in {-1, 0, +1} and int16 samples the metric is exact in
// integers (|c| < 2^25 per component, M < 2^64), so the peak decision needs no
// floating point at all.
//
// sync_metric_kernel: workgroup = (1024 candidates, group of antennas).  The
// correlation of 256 candidates n = n0 + 16 row + col is a product of the
// antenna's samples [row][kappa] = y[n0 + 16 row + kappa] and the chips as a
// Toeplitz matrix [kappa][col] = p[kappa - col], kappa < L + 15, on the int8
// matrix cores (v_mfma_i32_16x16x64_i8, exact): a sample's four bytes (upper
// and lower byte of either component, the lower one less 128 to be signed) are
// four operands, and c = 256 C_hi + C_lo + 128 sum p.  The byte planes are
// staged in LDS, where a row of the operand is 16 consecutive bytes at a
// multiple of 16.  The per-group partial metrics are summed by
// sync_reduce_kernel (integer sums: exact in any order, 16 threads per
// candidate), which also reduces each 64 candidates to the best (M, n);
// sync_argmax_kernel reduces those in one workgroup.
// "Best" = larger M, then smaller n: a total order, so the result does not
// depend on the reduction order.
// sync_extract_kernel: copies the slots that follow the preamble into the
// receive path's layout [S][T][A][CP+N] (one complex sample per dword); the
// start index is read from device memory (the detected offset) plus a
// constant, so detection and extraction chain without a host round trip.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rx_launch.h"

namespace rx {
namespace sync {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;       // threads per metric workgroup
constexpr int kTile = 4 * kThreads;  // candidates per metric workgroup
constexpr int kMaxGroups = 64;       // antenna groups (grid.y) at most
constexpr int kTargetGroups = 2048;  // metric workgroups aimed for (8 per CU)
constexpr int kRedCand = 64;         // candidates per reduce workgroup
constexpr int kRedWaves = 16;        // wavefronts per reduce workgroup (threads per candidate)

// K steps of 64 that hold the Toeplitz matrix's L + 15 rows, and the samples
// a workgroup stages.
__host__ __device__ constexpr int k_steps(int L) { return (L + 15 + 63) / 64; }
__host__ __device__ constexpr int staged(int L) { return kTile + 64 * k_steps(L); }
// LDS: four byte planes, the chip operand of every K step (16 bytes per lane),
// and the chips with 16 zeros before and enough behind.
constexpr int kPadChips = 16;
__host__ __device__ constexpr int metric_lds(int L) { return 4 * staged(L) + k_steps(L) * 1024 + kPadChips + 64 * k_steps(L); }

struct Best {
  uint64_t v;
  int64_t i;
};

__device__ __forceinline__ Best better(Best a, Best b) { return (a.v > b.v || (a.v == b.v && a.i < b.i)) ? a : b; }

__device__ __forceinline__ Best shfl_xor(Best x, int o) {
  Best r;
  r.v = ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(x.v >> 32), o, 64) << 32) |
        (uint32_t)__shfl_xor((int)(uint32_t)x.v, o, 64);
  r.i = (int64_t)(((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)((uint64_t)x.i >> 32), o, 64) << 32) |
                  (uint32_t)__shfl_xor((int)(uint32_t)(uint64_t)x.i, o, 64));
  return r;
}

// Best over the workgroup; valid in thread 0.
__device__ __forceinline__ Best block_best(Best b, Best* sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) b = better(b, shfl_xor(b, o));
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[wave] = b;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < nw; w++) b = better(b, sh[w]);
  return b;
}

// Bound: with one antenna per workgroup, staging: 1344 samples for 255 chips,
// then 20 products per wavefront.  17 344 candidates, 64 antennas, 255 chips:
// 7.2 us, where 2-way 16-bit dot products, a sliding window of samples in
// registers, took 21.6 (their instruction rate the bound).
__global__ __launch_bounds__(kThreads) void sync_metric_kernel(const uint32_t* __restrict__ raw, int A, int ag,
                                                               int64_t n_samples, int64_t stride, SyncChips ch,
                                                               int64_t n_search, uint64_t* __restrict__ part) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, L = ch.L, KK = k_steps(L), span = staged(L);
  uint8_t* plane = smem;                                    // [4][span]: re lo, re hi, im lo, im hi
  i32x4* chips = reinterpret_cast<i32x4*>(smem + 4 * span);  // [KK][64]
  int8_t* pad = reinterpret_cast<int8_t*>(chips + KK * 64);  // chip m at kPadChips + m
  const int64_t n0 = (int64_t)blockIdx.x * kTile;
  const int g = blockIdx.y, a0 = g * ag, a1 = min(A, a0 + ag);
  // chips as the second operand: lane (r, q) of step kk holds p[64 kk + 16 q + b - r], b = 0..15
  for (int i = tid; i < kPadChips + 64 * KK; i += kThreads) {
    const int m = i - kPadChips;
    pad[i] = m >= 0 && m < L ? ch.c[m] : (int8_t)0;
  }
  __syncthreads();
  for (int e = tid; e < KK * 64; e += kThreads) {
    const int8_t* p = pad + kPadChips + 64 * (e >> 6) + 16 * ((e >> 4) & 3) - (e & 15);
    i32x4 w;
#pragma unroll
    for (int i = 0; i < 4; i++)
      w[i] = (int)((uint32_t)(uint8_t)p[4 * i] | (uint32_t)(uint8_t)p[4 * i + 1] << 8 |
                   (uint32_t)(uint8_t)p[4 * i + 2] << 16 | (uint32_t)(uint8_t)p[4 * i + 3] << 24);
    chips[e] = w;
  }
  const int wave = tid >> 6, lane = tid & 63, r = lane & 15, q = lane >> 4;
  uint64_t acc[4] = {0, 0, 0, 0};
  for (int a = a0; a < a1; a++) {
    __syncthreads();  // the chips are there; the previous antenna's readers are done
    const uint32_t* ya = raw + (int64_t)a * stride;
    for (int j = 4 * tid; j < span; j += 4 * kThreads) {
      const int64_t i = n0 + j;
      uint32_t y[4];
#pragma unroll
      for (int k = 0; k < 4; k++) y[k] = i + k < n_samples ? ya[i + k] : 0u;
      // 4 x 4 bytes, transposed
      const uint32_t t0 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400u);  // bytes 0, 0', 1, 1'
      const uint32_t t1 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400u);
      const uint32_t t2 = __builtin_amdgcn_perm(y[1], y[0], 0x07030602u);  // bytes 2, 2', 3, 3'
      const uint32_t t3 = __builtin_amdgcn_perm(y[3], y[2], 0x07030602u);
      const uint32_t b[4] = {__builtin_amdgcn_perm(t1, t0, 0x05040100u) ^ 0x80808080u,
                             __builtin_amdgcn_perm(t1, t0, 0x07060302u),
                             __builtin_amdgcn_perm(t3, t2, 0x05040100u) ^ 0x80808080u,
                             __builtin_amdgcn_perm(t3, t2, 0x07060302u)};
#pragma unroll
      for (int k = 0; k < 4; k++) *reinterpret_cast<uint32_t*>(plane + k * span + j) = b[k];
    }
    __syncthreads();
    i32x4 c[4];
#pragma unroll
    for (int k = 0; k < 4; k++) c[k] = i32x4{0, 0, 0, 0};
    const uint8_t* rows = plane + 256 * wave + 16 * (r + q);
    for (int kk = 0; kk < KK; kk++) {
      const i32x4 p = chips[kk * 64 + lane];
#pragma unroll
      for (int k = 0; k < 4; k++)
        c[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const i32x4*>(rows + k * span + 64 * kk), p,
                                                     c[k], 0, 0, 0);
    }
    // lane (r, q), register i: candidate n0 + 256 wave + 16 (4 q + i) + r
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int64_t re = 256 * c[1][i] + c[0][i] + 128 * ch.sum, im = 256 * c[3][i] + c[2][i] + 128 * ch.sum;
      acc[i] += (uint64_t)(re * re) + (uint64_t)(im * im);
    }
  }
  uint64_t* out = part + (int64_t)g * n_search;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int64_t n = n0 + 256 * wave + 16 * (4 * q + i) + r;
    if (n < n_search) out[n] = acc[i];
  }
}

// M[n] = sum over antenna groups (integers: any order is exact), kRedWaves
// threads per candidate (wave w sums groups w, w + kRedWaves, ...: at most
// four loads each, so the partial metrics stream with many loads in flight),
// plus the best (M, n) of each workgroup's kRedCand candidates.
__global__ __launch_bounds__(64 * kRedWaves) void sync_reduce_kernel(const uint64_t* __restrict__ part, int G,
                                                                     int64_t n_search, uint64_t* __restrict__ M,
                                                                     uint64_t* __restrict__ cand_v,
                                                                     int64_t* __restrict__ cand_i) {
  __shared__ uint64_t sums[kRedWaves][kRedCand];
  const int c = threadIdx.x & (kRedCand - 1), w = threadIdx.x / kRedCand;
  const int64_t n = (int64_t)blockIdx.x * kRedCand + c;
  const bool ok = n < n_search;
  uint64_t v = 0;
  if (ok)
    for (int g = w; g < G; g += kRedWaves) v += part[(int64_t)g * n_search + n];
  sums[w][c] = v;
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int k = 1; k < kRedWaves; k++) v += sums[k][c];
    if (ok && M) M[n] = v;
    Best b = {ok ? v : 0ull, ok ? n : INT64_MAX};
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) b = better(b, shfl_xor(b, o));
    if (c == 0) {
      cand_v[blockIdx.x] = b.v;
      cand_i[blockIdx.x] = b.i;
    }
  }
}

__global__ __launch_bounds__(256) void sync_argmax_kernel(const uint64_t* __restrict__ cand_v,
                                                          const int64_t* __restrict__ cand_i, int n_blocks,
                                                          int64_t* __restrict__ offset, uint64_t* __restrict__ peak) {
  __shared__ Best sh[4];
  Best b = {0ull, INT64_MAX};
  for (int k = threadIdx.x; k < n_blocks; k += blockDim.x) b = better(b, Best{cand_v[k], cand_i[k]});
  b = block_best(b, sh);
  if (threadIdx.x == 0) {
    *offset = b.i;
    if (peak) *peak = b.v;
  }
}

// Row r = (s * T + t) * A + a of the output holds symbol t of slot s on
// antenna a: stream samples start + (s * T + t) * sym_len + j, j < sym_len,
// zero outside [0, n_samples).
__global__ __launch_bounds__(256) void sync_extract_kernel(const uint32_t* __restrict__ raw, int A,
                                                           int64_t n_samples, int64_t stride,
                                                           const int64_t* __restrict__ start_dev,
                                                           int64_t start_add, int sym_len, int T, int64_t rows,
                                                           uint32_t* __restrict__ out) {
  const int64_t start = (start_dev ? *start_dev : 0) + start_add;
  for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
    const int a = (int)(r % A);
    const int64_t st = r / A;  // s * T + t
    const int64_t base = start + st * sym_len;
    const uint32_t* ya = raw + (int64_t)a * stride;
    uint32_t* o = out + r * sym_len;
    for (int j = threadIdx.x; j < sym_len; j += blockDim.x) {
      const int64_t i = base + j;
      o[j] = (i >= 0 && i < n_samples) ? ya[i] : 0u;
    }
  }
}

}  // namespace sync

// Antenna groups: enough workgroups to fill the GPU (about kTargetGroups), at
// most one group per antenna.
int sync_groups(int A, int64_t n_search) {
  const int64_t tiles = (n_search + sync::kTile - 1) / sync::kTile;
  int64_t g = (sync::kTargetGroups + tiles - 1) / tiles;
  if (g > A) g = A;
  if (g > sync::kMaxGroups) g = sync::kMaxGroups;
  if (g < 1) g = 1;
  const int ag = (A + (int)g - 1) / (int)g;
  return (A + ag - 1) / ag;
}

size_t sync_workspace(int A, int64_t n_search) {
  const int64_t nb = (n_search + sync::kRedCand - 1) / sync::kRedCand;
  return (size_t)sync_groups(A, n_search) * n_search * 8 + (size_t)nb * 16;
}

hipError_t sync_find(const uint32_t* raw, int A, int64_t n_samples, int64_t stride, const SyncChips& ch,
                     int64_t n_search, uint64_t* M, int64_t* offset, uint64_t* peak, void* workspace,
                     hipStream_t st) {
  const int G = sync_groups(A, n_search);
  const int ag = (A + G - 1) / G;
  const int64_t tiles = (n_search + sync::kTile - 1) / sync::kTile;
  const int64_t nb = (n_search + sync::kRedCand - 1) / sync::kRedCand;
  uint64_t* part = static_cast<uint64_t*>(workspace);
  uint64_t* cv = part + (int64_t)G * n_search;
  int64_t* ci = reinterpret_cast<int64_t*>(cv + nb);
  const size_t lds = (size_t)sync::metric_lds(ch.L);
  hipLaunchKernelGGL(sync::sync_metric_kernel, dim3((unsigned)tiles, (unsigned)G), dim3(sync::kThreads), lds, st,
                     raw, A, ag, n_samples, stride, ch, n_search, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sync::sync_reduce_kernel, dim3((unsigned)nb), dim3(64 * sync::kRedWaves), 0, st,
                     (const uint64_t*)part, G,
                     n_search, M, cv, ci);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(sync::sync_argmax_kernel, dim3(1), dim3(256), 0, st, (const uint64_t*)cv, (const int64_t*)ci,
                     (int)nb, offset, peak);
  return hipGetLastError();
}

hipError_t sync_extract(const uint32_t* raw, int A, int64_t n_samples, int64_t stride, const int64_t* start,
                        int64_t start_add, int sym_len, int T, int64_t S, uint32_t* out, hipStream_t st) {
  const int64_t rows = S * T * A;
  const int64_t grid = rows < 65536 ? rows : 65536;
  hipLaunchKernelGGL(sync::sync_extract_kernel, dim3((unsigned)grid), dim3(256), 0, st, raw, A, n_samples, stride,
                     start, start_add, sym_len, T, rows, out);
  return hipGetLastError();
}

}  // namespace rx
