// Local (one-GPU) data movement of the Ulysses layout switch (Sec. 3.4): a multi-GPU bag goes from
// (partial sequences, full heads) to (full sequences, partial heads) with one all-to-all before
// attention and back with one after it.  The all-to-all moves contiguous buffers, so each GPU
//   before sending   splits its (T_r, H, d) tensor into g slabs (T_r, H/g, d), one per destination,
//   after receiving  puts the chunks of the g received slabs (chunk r of every sequence, from GPU r;
//                    chunks as cut by the second pass of Sec. 3.3) together into whole sequences,
// and runs the inverse of each on the way back.  Both are permutations of (token, head-group) rows of
// (H/g) d elements; the kernels move them in 16-byte units, every unit read once and written once, and
// are bound by HBM bandwidth.  The row permutation of the second step depends only on the bag's sequence
// lengths and is built once per bag (ulysses plan) for q, k, v, the output and every layer.
#include "knap_kernels.h"
#include "knapattn.h"

#include <stdint.h>

namespace knap {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// The copies are bound by HBM; what they ask for is many independent accesses in flight at any time.  One unit per thread and a
// workgroup for every 512 of them: the chip takes a new workgroup whenever one has stored, and its loads are under way while
// others wait for theirs.  (Two units per thread in a grid of 32 workgroups per CU that strides over the tensor has every thread
// wait for its loads before it asks for the next ones.)  Non-temporal loads and stores: +12 % over plain ones.
// Two units in a striding grid -> this, us, buffers rotated out of the Infinity Cache, packing | gathering:
// 150 MB 52.9 -> 49.2 | 51.9 -> 47.7 (6.3 TB/s); 100 MB 34.3 -> 33.6 | 35.4 -> 32.8; 32 MB 12.9 -> 12.4 | 13.6 -> 12.3;
// up to 12 MB the same within 0.4 us.  256 or 1024 threads: the same or up to 4 % slower.
constexpr int kCopyThreads = 512;

__device__ __forceinline__ u32x4_t ld_unit(const u32x4_t* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st_unit(u32x4_t* p, u32x4_t v) { __builtin_nontemporal_store(v, p); }

// y[(r T + t) U + c] = x[(t g + r) U + c]: U units per (token, head-group) row.  Iterates over x's
// linear index, so x is touched in address order and y in runs of U units.
template <bool PACK>
__global__ __launch_bounds__(kCopyThreads) void ulysses_heads_kernel(
    const u32x4_t* __restrict__ src, u32x4_t* __restrict__ dst, uint32_t T, uint32_t U, uint32_t g) {
  const uint32_t GU = g * U;
  const uint32_t xi = blockIdx.x * kCopyThreads + threadIdx.x;
  if (xi >= T * GU) return;
  const uint32_t t = xi / GU;
  const uint32_t w = xi - t * GU;
  const uint32_t r = w / U;
  const uint32_t yi = (r * T + t) * U + (w - r * U);
  st_unit(&dst[PACK ? yi : xi], ld_unit(&src[PACK ? xi : yi]));
}

// gather: z[t] = recv[row_map[t]]; scatter: send[row_map[t]] = z[t]; rows of U units.
template <bool GATHER>
__global__ __launch_bounds__(kCopyThreads) void ulysses_rows_kernel(
    const u32x4_t* __restrict__ src, u32x4_t* __restrict__ dst, const int32_t* __restrict__ row_map,
    uint32_t T, uint32_t U) {
  const uint32_t zi = blockIdx.x * kCopyThreads + threadIdx.x;
  if (zi >= T * U) return;
  const uint32_t t = zi / U;
  const uint32_t mi = (uint32_t)row_map[t] * U + (zi - t * U);
  st_unit(&dst[GATHER ? zi : mi], ld_unit(&src[GATHER ? mi : zi]));
}

constexpr int kPlanThreads = 256;

// row_map[t] for every row t of the (full sequences) layout.  A sequence of L tokens is cut into g chunks of
// base = L / g tokens, the first rem = L mod g one token longer; row t is token j of chunk r of sequence s and lies at
//   (first row of slab r) + (rows of slab r before sequence s) + j.
// Both follow from the sequences' bases and from how many have rem > r, so every workgroup (256 rows) forms them for
// itself in LDS: a scan of the bases, and counts of the remainders over the whole bag and over the sequences before
// the workgroup's first one; the few sequences between that one and s are counted row by row.
// What bounds it is latency, a chain of LDS steps.  A table of the offsets built by a one-workgroup kernel in front of
// this one cost a second launch and a serial walk over the sequences.  Plan alone, before -> now: 5 sequences on 2 GPUs
// 9.6 -> 6.9 us, 200 on 8 19.4 -> 6.6 us, 2000 on 4 150 -> 10.3 us.
__global__ __launch_bounds__(kPlanThreads) void ulysses_row_map_kernel(
    const int32_t* __restrict__ cu, int n_seq, int g, int T, int32_t* __restrict__ row_map) {
  extern __shared__ int32_t s_cu[];                 // n_seq + 1 boundaries
  int32_t* s_base = s_cu + n_seq + 1;               // sum of the bases of the sequences before s
  int32_t* s_rem = s_base + n_seq;
  __shared__ int32_t s_all[KNAP_ULYSSES_MAX_GPUS];      // sequences with each remainder
  __shared__ int32_t s_before[KNAP_ULYSSES_MAX_GPUS];   // those before the workgroup's first sequence
  __shared__ int32_t s_longer[KNAP_ULYSSES_MAX_GPUS];   // sequences whose chunk r is one token longer
  __shared__ int32_t s_first[KNAP_ULYSSES_MAX_GPUS];    // slab r's first row, plus its longer chunks before that sequence
  __shared__ int32_t s_wave[kPlanThreads / 64];
  const int tid = threadIdx.x;
  for (int i = tid; i <= n_seq; i += kPlanThreads) s_cu[i] = cu[i];
  if (tid < KNAP_ULYSSES_MAX_GPUS) s_all[tid] = s_before[tid] = 0;
  __syncthreads();

  // the sequence of row t: largest s with cu[s] <= t among the sequences that have rows
  auto sequence_of = [&](int t) {
    int lo = 0, hi = n_seq - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_cu[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  const int s0 = sequence_of(blockIdx.x * kPlanThreads);
  const int per = (n_seq + kPlanThreads - 1) / kPlanThreads;
  const int lo = min(tid * per, n_seq), hi = min(lo + per, n_seq);
  int local = 0;
  for (int s = lo; s < hi; ++s) {
    const int L = max(s_cu[s + 1] - s_cu[s], 0);
    const int base = L / g, rem = L - base * g;
    s_base[s] = local;
    s_rem[s] = rem;
    local += base;
    if (rem > 0) {
      atomicAdd(&s_all[rem], 1);
      if (s < s0) atomicAdd(&s_before[rem], 1);
    }
  }
  int sum = local;                                  // inclusive over the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(sum, o);
    if ((tid & 63) >= o) sum += x;
  }
  if ((tid & 63) == 63) s_wave[tid >> 6] = sum;
  __syncthreads();
  int before = sum - local, total = 0;
#pragma unroll
  for (int w = 0; w < kPlanThreads / 64; ++w) {
    if (w < tid >> 6) before += s_wave[w];
    total += s_wave[w];
  }
  for (int s = lo; s < hi; ++s) s_base[s] += before;
  int longer_before = 0;
  if (tid < g) {
    int longer = 0;
    for (int m = tid + 1; m < g; ++m) {
      longer += s_all[m];
      longer_before += s_before[m];
    }
    s_longer[tid] = longer;
  }
  __syncthreads();
  if (tid < g) {
    int start = tid * total;
    for (int r = 0; r < tid; ++r) start += s_longer[r];
    s_first[tid] = start + longer_before;
  }
  __syncthreads();

  const int t = blockIdx.x * kPlanThreads + tid;
  if (t >= T) return;
  const int s = sequence_of(t);
  const int L = s_cu[s + 1] - s_cu[s];
  const int i = t - s_cu[s];
  const int base = L / g, rem = L % g;
  // chunks 0 .. rem - 1 hold base + 1 tokens, the others base
  int r, j;
  if (i < rem * (base + 1)) {
    r = i / (base + 1);
    j = i - r * (base + 1);
  } else {
    const int k = i - rem * (base + 1);
    r = rem + k / base;               // base > 0 here: i < L and the longer chunks are used up
    j = k - (r - rem) * base;
  }
  // rows past cu[n_seq] (a total_tokens larger than the lengths add up to) must not index outside the tables
  r = min(max(r, 0), g - 1);
  int row = s_first[r] + s_base[s] + j;
  for (int q = s0; q < s; ++q) row += s_rem[q] > r ? 1 : 0;
  row_map[t] = row;
}

// at most 2^22: the API takes up to 2^31 units
int copy_grid(uint64_t units) { return (int)((units + kCopyThreads - 1) / kCopyThreads); }

}  // namespace

hipError_t launch_ulysses_heads(const void* src, void* dst, uint32_t T, uint32_t U, uint32_t g, bool pack,
                                hipStream_t stream) {
  const int grid = copy_grid((uint64_t)T * g * U);
  if (pack)
    hipLaunchKernelGGL(ulysses_heads_kernel<true>, dim3(grid), dim3(kCopyThreads), 0, stream,
                       (const u32x4_t*)src, (u32x4_t*)dst, T, U, g);
  else
    hipLaunchKernelGGL(ulysses_heads_kernel<false>, dim3(grid), dim3(kCopyThreads), 0, stream,
                       (const u32x4_t*)src, (u32x4_t*)dst, T, U, g);
  return hipGetLastError();
}

hipError_t launch_ulysses_rows(const void* src, void* dst, const int32_t* row_map, uint32_t T, uint32_t U,
                               bool gather, hipStream_t stream) {
  const int grid = copy_grid((uint64_t)T * U);
  if (gather)
    hipLaunchKernelGGL(ulysses_rows_kernel<true>, dim3(grid), dim3(kCopyThreads), 0, stream,
                       (const u32x4_t*)src, (u32x4_t*)dst, row_map, T, U);
  else
    hipLaunchKernelGGL(ulysses_rows_kernel<false>, dim3(grid), dim3(kCopyThreads), 0, stream,
                       (const u32x4_t*)src, (u32x4_t*)dst, row_map, T, U);
  return hipGetLastError();
}

hipError_t launch_ulysses_plan(const int32_t* cu, int n_seq, int g, int T, int32_t* row_map, hipStream_t stream) {
  const size_t dyn = (size_t)(3 * n_seq + 1) * sizeof(int32_t);
  hipLaunchKernelGGL(ulysses_row_map_kernel, dim3((T + kPlanThreads - 1) / kPlanThreads), dim3(kPlanThreads), dyn, stream,
                     cu, n_seq, g, T, row_map);
  return hipGetLastError();
}

}  // namespace knap
