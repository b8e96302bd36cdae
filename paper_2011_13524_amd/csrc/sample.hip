// Sampling of Z-basis outcomes (section 4.2.2: sampling goes through a
// cumulative distribution built as pre-processing, an extra 2^n-long array).
//
// For a uniform u in [0, 1) the sample is the smallest basis index x with
// C(x) > u * C(N - 1), C the inclusive cumulative sum of |psi|^2 in FP64.
//
// The cumulative distribution is a tree of local scans over chunks of 4096
// entries. Level 0 is the scan of |psi|^2 within each chunk of amplitudes, of
// which only every 16th value is stored (half a byte per amplitude); level l + 1
// holds the scan of the chunk totals of level l, up to a level of one chunk,
// whose last entry is the total. A sample descends the tree with one binary
// search per level, and at level 0 forms the 16 values of the run it lands in
// from the amplitudes, with the same operations.
//
// Within a chunk, thread t of 256 scans its 16 consecutive entries, and the
// thread offsets B_t are chained in order, B_{t+1} = B_t + T_t (T_t the
// thread's sum), by one thread. Every value of the scan is then B_t + run, and the
// first value of a thread equals the last of the previous one plus its own
// entry with the same rounding, so a scan is non-decreasing and rises
// only at entries of nonzero probability: a search never lands on an outcome
// of probability zero. The values stored at level 0 are the B_{t+1}.
#include <algorithm>
#include <vector>

#include "dev_common.h"
#include "qsv_internal.h"

namespace qsv {

constexpr int kScanThreads = 256;
constexpr int kScanChunkBits = 12;
constexpr uint32_t kScanChunk = 1u << kScanChunkBits;
constexpr uint32_t kScanPer = kScanChunk / kScanThreads;  // 16
constexpr int kScanMaxLevels = 4;                          // 4 x 12 bits >= 34 qubits
constexpr int kSampleThreads = 256;

struct ScanTree {
  const double* cdf[kScanMaxLevels];  // level 0: kScanThreads run ends per chunk
  uint64_t count[kScanMaxLevels];
  int levels;
};

// |v|^2 with its rounding spelled out: the table's kernel and the draws have to
// form the same value.
template <typename R>
__device__ __forceinline__ double scan_weight(cx<R> v) {
  return fma(double(v.re), double(v.re), double(v.im) * double(v.im));
}

// A chunk passes through LDS so that global reads and writes stay coalesced;
// entry j sits at j + j / 16 (one pad slot per thread's run of 16) so that the
// per-thread runs fall in different banks.
__device__ __forceinline__ uint32_t scan_slot(uint32_t j) { return j + (j >> 4); }

// base[t] = T_t -> B_t, in order; 16 loads in flight per step. Returns B_256.
__device__ __forceinline__ double scan_chain(double* base) {
  double b = 0.0;
  for (uint32_t t0 = 0; t0 < kScanThreads; t0 += 16) {
    double T[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) T[k] = base[t0 + k];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      base[t0 + k] = b;
      b += T[k];
    }
  }
  return b;
}

// Level 0, one workgroup per chunk (the last may be short): ends[t] = B_{t+1} of
// its runs, sums[blockIdx.x] its total. Bound by the read of the state: 26 qubits
// complex64, 197 us with every value stored, 116 us here (4.6 TB/s; 227 us with
// each thread reading its 16 entries itself).
template <typename R>
__global__ void __launch_bounds__(kScanThreads)
    k_scan_amps(const R* __restrict__ psi, uint64_t count, double* __restrict__ ends, double* __restrict__ sums) {
  __shared__ double p[kScanChunk + kScanChunk / kScanPer];
  __shared__ double base[kScanThreads];
  __shared__ double total;
  const uint64_t first = uint64_t(blockIdx.x) << kScanChunkBits;
  const uint32_t len = uint32_t(min<uint64_t>(kScanChunk, count - first));
  const uint32_t tid = threadIdx.x;
  if (len == kScanChunk) {  // 16-byte vectors, two entries per lane
#pragma unroll
    for (uint32_t i = 0; i < kScanChunk / (2 * kScanThreads); ++i) {
      const uint32_t j = 2 * (tid + i * kScanThreads);
      cx<R> v[2];
      AmpIO<R, 2>::load(psi, first + j, v);
      p[scan_slot(j)] = scan_weight(v[0]);
      p[scan_slot(j + 1)] = scan_weight(v[1]);
    }
  } else {
    for (uint32_t j = tid; j < kScanChunk; j += kScanThreads)
      p[scan_slot(j)] = j < len ? scan_weight(load1(psi, first + j)) : 0.0;
  }
  __syncthreads();
  // thread t's entries 16t .. 16t + 15 (0 past the end)
  double acc = 0.0;
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) acc += p[scan_slot(tid * kScanPer + k)];
  base[tid] = acc;
  __syncthreads();
  if (tid == 0) total = scan_chain(base);
  __syncthreads();
  ends[(uint64_t(blockIdx.x) * kScanThreads) + tid] = tid + 1 < kScanThreads ? base[tid + 1] : total;
  if (tid == 0) sums[blockIdx.x] = total;
}

// A level above: the scan of `count` values, in place, one workgroup per chunk
// (the last may be short); sums[blockIdx.x] = its total (the last scan value).
__global__ void __launch_bounds__(kScanThreads) k_scan_chunks(double* cdf, uint64_t count, double* __restrict__ sums) {
  __shared__ double p[kScanChunk + kScanChunk / kScanPer];
  __shared__ double base[kScanThreads];
  const uint64_t first = uint64_t(blockIdx.x) << kScanChunkBits;
  const uint32_t len = uint32_t(min<uint64_t>(kScanChunk, count - first));
  const uint32_t tid = threadIdx.x;
  for (uint32_t j = tid; j < len; j += kScanThreads) p[scan_slot(j)] = cdf[first + j];
  __syncthreads();
  const uint32_t j0 = tid * kScanPer;
  double run[kScanPer];
  double acc = 0.0;
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) {
    if (j0 + k < len) acc += p[scan_slot(j0 + k)];
    run[k] = acc;
  }
  base[tid] = acc;  // thread total T_t (0 past the end)
  __syncthreads();
  if (tid == 0) scan_chain(base);
  __syncthreads();
  const double b = base[tid];
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k)
    if (j0 + k < len) p[scan_slot(j0 + k)] = b + run[k];
  __syncthreads();
  for (uint32_t j = tid; j < len; j += kScanThreads) cdf[first + j] = p[scan_slot(j)];
  if (tid == 0) sums[blockIdx.x] = p[scan_slot(len - 1)];
}

// Smallest j in [lo, hi) with c[j] > r, given c[hi - 1] > r and c non-decreasing.
__device__ __forceinline__ uint64_t first_above(const double* c, uint64_t lo, uint64_t hi, double r) {
  uint64_t a = lo, b = hi - 1;
  while (a < b) {
    const uint64_t m = (a + b) >> 1;
    if (c[m] > r)
      b = m;
    else
      a = m + 1;
  }
  return a;
}

template <typename R>
__global__ void __launch_bounds__(kSampleThreads)
    k_sample(ScanTree T, const R* __restrict__ psi, const double* __restrict__ sum, const double* __restrict__ u,
             uint64_t count, int64_t* __restrict__ out) {
  const uint64_t i = uint64_t(blockIdx.x) * kSampleThreads + threadIdx.x;
  if (i >= count) return;
  double r = u[i] * sum[0];
  uint64_t seg = 0;
  for (int l = T.levels - 1; l > 0; --l) {
    const double* c = T.cdf[l];
    const uint64_t lo = seg << kScanChunkBits;
    const uint64_t hi = min<uint64_t>(lo + kScanChunk, T.count[l]);
    const double tot = c[hi - 1];  // > 0: the segment was reached through a rise
    if (!(r < tot)) r = nextafter(tot, 0.0);
    const uint64_t a = first_above(c, lo, hi, r);
    if (a > lo) r -= c[a - 1];  // >= 0: c[a - 1] <= r
    seg = a;
  }
  // the chunk: its run, then the entry within the run
  const double* c = T.cdf[0];
  const uint64_t lo = seg * kScanThreads, hi = lo + kScanThreads;
  const double tot = c[hi - 1];
  if (!(r < tot)) r = nextafter(tot, 0.0);
  const uint64_t a = first_above(c, lo, hi, r);
  const double b = a > lo ? c[a - 1] : 0.0;
  const uint64_t x0 = a * kScanPer;
  cx<R> v[kScanPer];
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) v[k] = x0 + k < T.count[0] ? load1(psi, x0 + k) : cx<R>{R(0), R(0)};
  double acc = 0.0;
  uint32_t at = kScanPer - 1;
  bool found = false;
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) {
    acc += scan_weight(v[k]);
    if (!found && b + acc > r) {
      at = k;
      found = true;
    }
  }
  out[i] = int64_t(min<uint64_t>(x0 + at, T.count[0] - 1));
}

namespace {

// Device memory of one sampling call, carved from the state's work buffer
// (kept for the next call; every call synchronises before returning).
struct SampleBuffers {
  char* base = nullptr;
  size_t used = 0, cap = 0;
  template <typename T>
  T* get(size_t n) {
    const size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) / 256 * 256;
    if (used + bytes > cap) return nullptr;
    T* p = reinterpret_cast<T*>(base + used);
    used += bytes;
    return p;
  }
};

template <typename R>
int sample_t(const qsv_state* s, const double* u, int64_t count, int64_t* out) {
  hipStream_t st = s->stream;
  // sizes: level 0 table (one FP64 per 16 amplitudes), the chunk totals of every
  // level, then the uniforms and the outputs
  size_t need = 0;
  auto add = [&need](size_t bytes) { need += (std::max<size_t>(bytes, 1) + 255) / 256 * 256; };
  {
    uint64_t c = dim(s->n);
    add(((c + kScanChunk - 1) >> kScanChunkBits) * kScanThreads * sizeof(double));
    do {
      c = (c + kScanChunk - 1) >> kScanChunkBits;
      add(c * sizeof(double));
    } while (c > 1);
    add(size_t(count) * sizeof(double));
    add(size_t(count) * sizeof(int64_t));
  }
  SampleBuffers buf;
  void* wb = nullptr;
  if (int rc = state_work(s, need, &wb)) return rc;
  buf.base = static_cast<char*>(wb);
  buf.cap = need;
  ScanTree T{};
  uint64_t cnt = dim(s->n);
  // level 0: |psi|^2 chunks of the state; higher levels scan the chunk totals in place
  uint64_t chunks = (cnt + kScanChunk - 1) >> kScanChunkBits;
  double* level_cdf = buf.get<double>(chunks * kScanThreads);
  double* sums = buf.get<double>(chunks);
  if (!level_cdf || !sums) return fail(QSV_ENOMEM, "cumulative table allocation failed");
  hipLaunchKernelGGL((k_scan_amps<R>), dim3(unsigned(chunks)), dim3(kScanThreads), 0, st,
                     static_cast<const R*>(s->ptr), cnt, level_cdf, sums);
  QSV_HIP_CHECK(hipGetLastError());
  T.cdf[0] = level_cdf;
  T.count[0] = cnt;
  T.levels = 1;
  while (chunks > 1) {
    if (T.levels == kScanMaxLevels) return fail(QSV_ERANGE, "state too large for the sampling table");
    cnt = chunks;
    double* in = sums;
    chunks = (cnt + kScanChunk - 1) >> kScanChunkBits;
    sums = buf.get<double>(chunks);
    if (!sums) return fail(QSV_ENOMEM, "cumulative table allocation failed");
    hipLaunchKernelGGL(k_scan_chunks, dim3(unsigned(chunks)), dim3(kScanThreads), 0, st, in, cnt, sums);
    QSV_HIP_CHECK(hipGetLastError());
    T.cdf[T.levels] = in;
    T.count[T.levels] = cnt;
    ++T.levels;
  }
  // the draws are enqueued behind the table (in range whatever it holds), and
  // handed out once its total is known
  int64_t* dout = nullptr;
  if (count > 0) {
    double* du = buf.get<double>(size_t(count));
    dout = buf.get<int64_t>(size_t(count));
    if (!du || !dout) return fail(QSV_ENOMEM, "sample buffer allocation failed");
    QSV_HIP_CHECK(hipMemcpyAsync(du, u, size_t(count) * sizeof(double), hipMemcpyHostToDevice, st));
    const uint64_t blocks = (uint64_t(count) + kSampleThreads - 1) / kSampleThreads;
    hipLaunchKernelGGL((k_sample<R>), dim3(unsigned(blocks)), dim3(kSampleThreads), 0, st, T,
                       static_cast<const R*>(s->ptr), sums, du, uint64_t(count), dout);
    QSV_HIP_CHECK(hipGetLastError());
  }
  double total = 0.0;
  QSV_HIP_CHECK(hipMemcpyAsync(&total, sums, sizeof(double), hipMemcpyDeviceToHost, st));
  QSV_HIP_CHECK(hipStreamSynchronize(st));
  if (!(total > 0.0)) return fail(QSV_EINVAL, "state has zero norm");
  if (count == 0) return QSV_OK;
  QSV_HIP_CHECK(hipMemcpyAsync(out, dout, size_t(count) * sizeof(int64_t), hipMemcpyDeviceToHost, st));
  QSV_HIP_CHECK(hipStreamSynchronize(st));
  return QSV_OK;
}

}  // namespace

}  // namespace qsv

using namespace qsv;

extern "C" {

int qsv_sample(const qsv_state* s, const double* u, int64_t count, int64_t* out) {
  clear_error();
  int rc = check_state(s);
  if (rc) return rc;
  if (count < 0) return fail(QSV_EINVAL, "negative sample count");
  if (count > (int64_t(1) << 31)) return fail(QSV_ERANGE, "at most 2^31 samples per call");
  if (count > 0 && (!u || !out)) return fail(QSV_EINVAL, "null argument");
  bool bad = false;  // (no exit inside: the check runs on vectors)
  for (int64_t i = 0; i < count; ++i) bad |= !(u[i] >= 0.0) | !(u[i] < 1.0);
  for (int64_t i = 0; bad && i < count; ++i)
    if (!(u[i] >= 0.0 && u[i] < 1.0)) return fail(QSV_ERANGE, "uniform %lld outside [0, 1)", (long long)i);
  return s->dtype == QSV_C64 ? sample_t<float>(s, u, count, out) : sample_t<double>(s, u, count, out);
}

}  // extern "C"
