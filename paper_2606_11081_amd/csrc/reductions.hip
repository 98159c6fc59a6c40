// a5 standalone and a6: the consensus error of the stored x over a column
// range, the fixed-order fp64 finalize of workgroup partials, and the
// network average.
#pragma clang fp contract(off)

#include <mutex>
#include <string>

#include "device_common.h"

// Scratch of gasloc_consensus_error_cols_noalloc: the workgroup partials, then
// the finalize's segment sums.  A file-scope device array: every GPU the
// library runs on holds its own copy for the life of the process.  In host
// code `scratch` only names the symbol; its device address on the current GPU
// comes from hipGetSymbolAddress (see noalloc_scratch below).
constexpr int kNoAllocPartials = 1 << 16;
constexpr int kNoAllocSegments = kNoAllocPartials / gasloc::kFinalizeSegment;
static __device__ __align__(256) double scratch[kNoAllocPartials + kNoAllocSegments];

namespace gasloc {
namespace {

// What bounds both reductions is HBM, once the fp64 work (a conversion and
// one or five operations an element) does not: a group of 4 columns per thread
// keeps its sums in few registers, and a step that lies in the range as a whole
// tests nothing per lane, so that the loads of a batch are issued back to back.
// n=16, P=50M bf16: the error 350 -> 267 us (6.0 TB/s), the mean 347 -> 272 us;
// n=16, P=50M fp32: 503 -> 498 (6.4 TB/s), 624 -> 594 us; n=64, P=6M bf16: 175 ->
// 147, 143 -> 136 us.  With 8 bf16 columns per thread the error took 350 us, with
// whole batches split from the last one (more registers) 294, with batches of
// 8 workers the same as with 4.
constexpr int kErrorBatch = 4;  // workers whose loads are in flight at a time

// Columns [lo, hi) of the V-column group at idx (the others read as 0): a
// vector load when the whole group is in range.
template <int DT, int V>
__device__ __forceinline__ void load_cols(const void* base, int64_t idx, int lo, int hi, float (&o)[V]) {
  if (lo == 0 && hi == V) {
    load_params<DT, V>(base, idx, V, o);
    return;
  }
#pragma unroll
  for (int c = 0; c < V; ++c) {
    if (c >= lo && c < hi) {
      if constexpr (DT == GASLOC_BF16)
        o[c] = bf16_to_f32(static_cast<const uint16_t*>(base)[idx + c]);
      else
        o[c] = static_cast<const float*>(base)[idx + c];
    } else {
      o[c] = 0.0f;
    }
  }
}

// One group of a thread: the shifted fp64 sums of its 4 columns of every
// worker, workers in order, with the round kernels' operations (a column's
// error is the same number either way).  EDGE: the group may be cut
// by an end of the range (columns [lo, hi) of it count).
template <int DT, bool EDGE>
__device__ __forceinline__ double group_error(const void* x, int64_t ld, int n, int64_t p, int lo_edge, int hi_edge) {
  constexpr int V = kReduceVec, R = kErrorBatch;
  const int lo = EDGE ? lo_edge : 0, hi = EDGE ? hi_edge : V;
  double shift[V], s[V], q[V];
  {
    float v[V];
    load_cols<DT, V>(x, p, lo, hi, v);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      shift[c] = static_cast<double>(v[c]);
      s[c] = 0.0;
      q[c] = 0.0;
    }
  }
  for (int i0 = 1; i0 < n; i0 += R) {
    float v[R][V];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i0 + r >= n) break;
      load_cols<DT, V>(x, static_cast<int64_t>(i0 + r) * ld + p, lo, hi, v[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i0 + r >= n) break;
#pragma unroll
      for (int c = 0; c < V; ++c) {
        const double d = static_cast<double>(v[r][c]) - shift[c];
        s[c] += d;
        q[c] += d * d;
      }
    }
  }
  const double inv_n = 1.0 / static_cast<double>(n);
  double ce = 0.0;
#pragma unroll
  for (int c = 0; c < V; ++c)
    if (c >= lo && c < hi) ce += q[c] - s[c] * s[c] * inv_n;
  return ce;
}

// A thread takes groups of 4 columns of every worker (groups are aligned so
// every row's vector loads are, and those at the ends of the range are
// masked; a step of the workgroup without such a group tests nothing per lane).
// Workgroup b takes the `per` consecutive steps of blockDim.x groups starting
// at group b * per * blockDim.x (tile order, as the round kernels) and writes
// one partial.
template <int DT>
__global__ __launch_bounds__(reduce_threads(DT)) void k_consensus_error(const void* x, int64_t ld, int n,
                                                                        int64_t p_begin, int64_t p_end, int per,
                                                                        double* partials) {
  constexpr int V = kReduceVec;
  const int64_t base = p_begin - p_begin % V;
  const int64_t groups = (p_end - base + V - 1) / V;
  const int64_t g0 = static_cast<int64_t>(blockIdx.x) * per * blockDim.x;
  const int64_t g_end = groups - g0 < static_cast<int64_t>(per) * blockDim.x ? groups : g0 + per * blockDim.x;
  double ce = 0.0;
  for (int64_t g = g0; g < g_end; g += blockDim.x) {
    const int64_t p = base + (g + threadIdx.x) * V;
    if (base + g * V >= p_begin && base + (g + blockDim.x) * V <= p_end) {
      ce += group_error<DT, false>(x, ld, n, p, 0, V);
    } else if (p < p_end) {
      const int lo = p < p_begin ? static_cast<int>(p_begin - p) : 0;
      const int hi = p_end - p < V ? static_cast<int>(p_end - p) : V;
      ce += group_error<DT, true>(x, ld, n, p, lo, hi);
    }
  }
  const double total = block_sum(ce);
  if (threadIdx.x == 0) partials[blockIdx.x] = total;
}

// Zeros columns [0, P) of n rows (grid: 1024-column tiles, rows).  The row
// padding is the caller's, so a plain fill of the buffer would not do, and the
// runtime's pitched fill runs at 0.5 TB/s: gasloc_init at n=10, P=16.6M with
// padded rows took 5.4 ms with it, 0.58 ms so.
__global__ __launch_bounds__(256) void k_zero_rows(float* x, int64_t ld, int64_t P) {
  constexpr int V = 4;
  const int64_t p = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * V;
  if (p >= P) return;
  const float zero[V] = {};
  store_f32<V>(x + static_cast<int64_t>(blockIdx.y) * ld + p, static_cast<int>(P - p < V ? P - p : V), zero);
}

// The finalize kernels run one workgroup of kFinalizeThreads threads over at
// most kFinalizeSegment partials: each thread's few strided loads are issued
// together, so the kernel is one memory latency long (4096 partials: 5.9 us
// with 256 threads of 16 loads each in turn, 4.3 so).
constexpr int kFinalizeThreads = 1024;
constexpr int kFinalizeLoads = kFinalizeSegment / kFinalizeThreads;

// Sum of thread's partials k, k + kFinalizeThreads, ... of a[0..count), count <= kFinalizeSegment.
__device__ __forceinline__ double strided_sum(const double* a, int count) {
  double v[kFinalizeLoads];
#pragma unroll
  for (int j = 0; j < kFinalizeLoads; ++j) {
    const int k = threadIdx.x + j * kFinalizeThreads;
    v[j] = k < count ? a[k] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kFinalizeLoads; ++j) s += v[j];
  return s;
}

// Fixed-order sum of `count` partials into *out (one workgroup).
__global__ __launch_bounds__(kFinalizeThreads) void k_finalize(const double* partials, int count, double* out) {
  const double total = block_sum(strided_sum(partials, count));
  if (threadIdx.x == 0) *out = total;
}

// The same for the two partial arrays of a round (consensus error, squared
// pseudo-gradients) in one launch: out[0], out[1], each in k_finalize's order.
__global__ __launch_bounds__(kFinalizeThreads) void k_finalize2(const double* a, const double* b, int count,
                                                                double* out) {
  const double va = strided_sum(a, count), vb = strided_sum(b, count);
  double ta, tb;
  block_sum2(va, vb, ta, tb);
  if (threadIdx.x == 0) {
    out[0] = ta;
    out[1] = tb;
  }
}

// First level of the segmented finalize: workgroup s sums the partials
// [s * kFinalizeSegment, (s + 1) * kFinalizeSegment) of `a` (and of `b`
// unless it is NULL; fewer in the last segment) in k_finalize's order, into
// seg[s] (and seg[S + s]).
__global__ __launch_bounds__(kFinalizeThreads) void k_finalize_segments(const double* a, const double* b, int count,
                                                                        double* seg) {
  const int begin = blockIdx.x * kFinalizeSegment;
  const int here = count - begin < kFinalizeSegment ? count - begin : kFinalizeSegment;
  const double va = strided_sum(a + begin, here);
  const double vb = b ? strided_sum(b + begin, here) : 0.0;
  double ta, tb;
  block_sum2(va, vb, ta, tb);
  if (threadIdx.x == 0) {
    seg[blockIdx.x] = ta;
    if (b) seg[gridDim.x + blockIdx.x] = tb;
  }
}

// a / b for a finite b > 0 that is a small whole number, given r = 1 / b
// rounded: the quotient a r corrected twice by its exact remainder is the
// correctly rounded one (Markstein: from a quotient within one unit in the
// last place, which the first correction gives, and a correctly rounded
// reciprocal; compared with the division on 2.56e8 random sums for b = 1 to
// 64), and the fixup restores zeros, infinities and NaN.  Half the instructions
// of the general division.  (The fused multiply-adds are the method's; the
// result is the division's.)
__device__ __forceinline__ double divide_by(double a, double b, double r) {
  double q = a * r;
  q = __builtin_fma(__builtin_fma(-b, q, a), r, q);
  q = __builtin_fma(__builtin_fma(-b, q, a), r, q);
  return __builtin_amdgcn_div_fixup(q, b, a);
}

// The averages of a thread's 4 columns (cnt of them in a ragged last group):
// fp64 sums in worker order, rounded to the param dtype.
template <int DT, bool TAIL>
__device__ __forceinline__ void group_mean(const void* x, int64_t ld, int n, int64_t p, int cnt_tail, void* out) {
  constexpr int V = kReduceVec, R = 8;
  const int cnt = TAIL ? cnt_tail : V;
  double s[V];
#pragma unroll
  for (int c = 0; c < V; ++c) s[c] = 0.0;
  for (int i0 = 0; i0 < n; i0 += R) {
    float v[R][V];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i0 + r >= n) break;
      load_params<DT, V>(x, static_cast<int64_t>(i0 + r) * ld + p, cnt, v[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i0 + r >= n) break;
#pragma unroll
      for (int c = 0; c < V; ++c) s[c] += static_cast<double>(v[r][c]);
    }
  }
  const double b = static_cast<double>(n), r = 1.0 / b;
  float mean[V], kept[V];
#pragma unroll
  for (int c = 0; c < V; ++c) mean[c] = static_cast<float>(divide_by(s[c], b, r));
  store_params<DT, V>(out, p, cnt, mean, kept);
}

// a6: network average; 4 columns per thread, one step per workgroup (with
// more, the next step's loads wait behind this one's store: n=16, P=50M bf16
// 354 us with 8 steps, 318 with one, all else as before).
template <int DT>
__global__ __launch_bounds__(reduce_threads(DT)) void k_replica_mean(const void* x, int64_t ld, int n, int64_t P,
                                                                     void* out) {
  constexpr int V = kReduceVec;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * blockDim.x * V;
  const int64_t p = first + threadIdx.x * V;
  if (first + static_cast<int64_t>(blockDim.x) * V <= P)
    group_mean<DT, false>(x, ld, n, p, V, out);
  else if (p < P)
    group_mean<DT, true>(x, ld, n, p, static_cast<int>(P - p < V ? P - p : V), out);
}

}  // namespace

int consensus_error_blocks(int dtype, int64_t p_begin, int64_t p_end, int per) {
  constexpr int V = kReduceVec;
  const int64_t base = p_begin - p_begin % V;
  const int64_t groups = (p_end - base + V - 1) / V;
  const int64_t span = static_cast<int64_t>(per) * reduce_threads(dtype);
  const int64_t blocks = (groups + span - 1) / span;
  return static_cast<int>(blocks < 1 ? 1 : (blocks > (int64_t(1) << 30) ? (int64_t(1) << 30) : blocks));
}

hipError_t launch_consensus_error(const void* x, int dtype, int64_t ld, int n, int64_t p_begin,
                                  int64_t p_end, int per, double* partials, hipStream_t stream) {
  const int blocks = consensus_error_blocks(dtype, p_begin, p_end, per);
  return launch_kernel(dtype == GASLOC_BF16 ? k_consensus_error<GASLOC_BF16> : k_consensus_error<GASLOC_F32>,
                       dim3(blocks), reduce_threads(dtype), 0, stream, x, ld, n, p_begin, p_end, per, partials);
}

hipError_t launch_finalize_large(const double* a, int count, double* seg, double* out, hipStream_t stream) {
  if (count <= kFinalizeSegment) return launch_finalize(a, count, out, stream);
  const int segments = (count + kFinalizeSegment - 1) / kFinalizeSegment;
  const hipError_t e =
      launch_kernel(k_finalize_segments, dim3(segments), kFinalizeThreads, 0, stream, a, nullptr, count, seg);
  if (e != hipSuccess) return e;
  return launch_finalize(seg, segments, out, stream);
}

hipError_t launch_finalize(const double* partials, int count, double* out, hipStream_t stream) {
  return launch_kernel(k_finalize, dim3(1), kFinalizeThreads, 0, stream, partials, count, out);
}

hipError_t launch_finalize2(const double* a, const double* b, int count, double* out, hipStream_t stream) {
  return launch_kernel(k_finalize2, dim3(1), kFinalizeThreads, 0, stream, a, b, count, out);
}

hipError_t launch_finalize2_large(const double* a, const double* b, int count, double* seg, double* out,
                                  hipStream_t stream) {
  if (count <= kFinalizeSegment) return launch_finalize2(a, b, count, out, stream);
  const int segments = (count + kFinalizeSegment - 1) / kFinalizeSegment;
  const hipError_t e = launch_kernel(k_finalize_segments, dim3(segments), kFinalizeThreads, 0, stream, a, b, count, seg);
  if (e != hipSuccess) return e;
  return launch_finalize2(seg, seg + segments, segments, out, stream);
}

hipError_t launch_zero_rows(float* x, int64_t ld, int n, int64_t P, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>((P + 1023) / 1024), static_cast<unsigned>(n));
  return launch_kernel(k_zero_rows, grid, 256, 0, stream, x, ld, P);
}

hipError_t launch_replica_mean(const void* x, int dtype, int64_t ld, int n, int64_t P, void* out,
                               hipStream_t stream) {
  const int blocks = consensus_error_blocks(dtype, 0, P, 1);
  return launch_kernel(dtype == GASLOC_BF16 ? k_replica_mean<GASLOC_BF16> : k_replica_mean<GASLOC_F32>, dim3(blocks),
                       reduce_threads(dtype), 0, stream, x, ld, n, P, out);
}

}  // namespace gasloc

namespace {

constexpr int kNoAllocPer = 8;  // steps per workgroup, as the context's reduction on long ranges
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch[kMaxDevices] = {};

// Device address of `scratch` on the current GPU, looked up once per device
// with that device current.
hipError_t noalloc_scratch(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = static_cast<double*>(p);
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

gasloc_status noalloc_fail(gasloc_status st, const std::string& msg) {
  gasloc::set_thread_error("consensus_error_cols_noalloc: " + msg);
  return st;
}

}  // namespace

extern "C" gasloc_status gasloc_consensus_error_cols_noalloc(const void* x, int32_t param_dtype, int32_t n,
                                                             int64_t ld, int64_t p_begin, int64_t p_end,
                                                             double* out, void* hip_stream) {
  if (!x || (reinterpret_cast<uintptr_t>(x) & 15u)) return noalloc_fail(GASLOC_EINVAL, "x must be non-NULL and 16-byte aligned");
  if (!out || (reinterpret_cast<uintptr_t>(out) & 7u)) return noalloc_fail(GASLOC_EINVAL, "out must be non-NULL and 8-byte aligned");
  if (param_dtype != GASLOC_F32 && param_dtype != GASLOC_BF16) return noalloc_fail(GASLOC_EINVAL, "param_dtype must be F32 or BF16");
  if (n < 1 || n > gasloc::kMaxReplicas) return noalloc_fail(GASLOC_EINVAL, "n outside [1, 64]");
  const int64_t elem = param_dtype == GASLOC_BF16 ? 2 : 4;
  if (ld < 1 || (ld * elem) % 16 != 0) return noalloc_fail(GASLOC_EINVAL, "ld * sizeof(param) must be a positive multiple of 16 bytes");
  if (p_begin < 0 || p_end < p_begin || p_end > ld || p_end >= (int64_t(1) << 31))
    return noalloc_fail(GASLOC_EINVAL, "need 0 <= p_begin <= p_end <= ld and p_end < 2^31");
  const int blocks = gasloc::consensus_error_blocks(param_dtype, p_begin, p_end, kNoAllocPer);
  if (blocks > kNoAllocPartials) {
    const int64_t most = int64_t(kNoAllocPartials) * kNoAllocPer * gasloc::reduce_step(param_dtype);
    return noalloc_fail(GASLOC_EINVAL, "column range longer than the scratch allows (at most " + std::to_string(most) +
                                           " columns of this dtype per call; split the range and add the results)");
  }
  double* ptr = nullptr;
  hipError_t e = noalloc_scratch(&ptr);
  if (e != hipSuccess) return noalloc_fail(GASLOC_EDEVICE, std::string("scratch address: ") + hipGetErrorString(e));
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  e = gasloc::launch_consensus_error(x, param_dtype, ld, n, p_begin, p_end, kNoAllocPer, ptr, stream);
  if (e == hipSuccess) e = gasloc::launch_finalize_large(ptr, blocks, ptr + kNoAllocPartials, out, stream);
  if (e != hipSuccess) return noalloc_fail(GASLOC_EDEVICE, hipGetErrorString(e));
  return GASLOC_OK;
}
