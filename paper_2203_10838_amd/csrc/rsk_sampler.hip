// Row sampler on the device: the index stream tau_k (Sec. 1.1: eta rows per
// step, with replacement, p_i proportional to ||a_i||^2) drawn from the
// counter-based generator Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11)
// and an inverse-CDF search, so long streams need neither host generation
// nor a host-to-device copy.
//
// Index t of step k: Philox4x32-10 of the counter (t, k mod 2^32, k div 2^32, 0)
// under the key (seed mod 2^32, seed div 2^32) gives words w0, w1;
// u = ((w0 >> 5) 2^26 + (w1 >> 6)) 2^-53 in [0, 1); the row is the first i with
// cdf_i > u cdf_{m-1}. Given the same cdf array the stream is bit-for-bit a
// function of (seed, k, t) alone, whatever the launch shape.
//
// The cdf (running sums of the FP64 row norms) is built by a three-pass scan:
// chunk sums, one fixed-order scan of the chunk sums, chunk-local scans.
#include "rsk_device.hpp"
#include "rsk_kernels.hpp"

namespace rsk {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;                       // elements per thread
constexpr int kScanChunk = kScanThreads * kScanPer;

__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

}  // namespace

// One draw: the target of step k0 + e / eta, slot e % eta.
__device__ __forceinline__ double draw_target(int64_t e, int eta, int64_t k0, uint32_t key0, uint32_t key1, double total) {
  const int64_t k = k0 + e / eta;
  uint32_t c[4] = {(uint32_t)(e % eta), (uint32_t)k, (uint32_t)((uint64_t)k >> 32), 0u};
  philox4x32_10(c, key0, key1);
  const uint64_t bits = ((uint64_t)(c[0] >> 5) << 26) | (uint64_t)(c[1] >> 6);
  return (double)bits * (1.0 / 9007199254740992.0) * total;
}

// A draw a thread, every level of its binary search read from the cdf.
__global__ __launch_bounds__(256) void sample_direct_kernel(const double* __restrict__ cdf, int64_t m, uint32_t key0,
                                                            uint32_t key1, int64_t k0, int64_t K, int eta,
                                                            int32_t* __restrict__ out) {
  const double total = cdf[m - 1];
  const int64_t N = K * (int64_t)eta;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < N; e += (int64_t)gridDim.x * blockDim.x) {
    const double target = draw_target(e, eta, k0, key0, key1, total);
    int64_t lo = 0, hi = m;
    while (lo < hi) {
      const int64_t mid = lo + ((hi - lo) >> 1);
      if (cdf[mid] > target) hi = mid;
      else lo = mid + 1;
    }
    out[e] = (int32_t)(lo < m ? lo : m - 1);
  }
}

// Binary search in two levels. kPivots evenly spaced cdf values sit in LDS: the first levels of
// the search read those, and only the last log2(m / kPivots) (a stretch of a few cache lines) read
// the cdf itself; kIlp searches a thread run side by side, so one's loads are in flight under the
// others'. The index is the first i with cdf_i > target, as by any search of a non-decreasing cdf.
// Bound by the gathers (LDS banks for the pivots, one cache line a lane for the rest): 8000 x 1024
// draws from 100000 rows in 213 us (320 us with every level read from the cdf).
constexpr int kPivots = 4096, kSampleThreads = 1024, kIlp = 4;
constexpr int64_t kSampleBlocks = 512;
// Every workgroup fills its pivots from as many cache lines of the cdf, and a long stretch leaves most of a
// search outside them, so the two levels pay for many draws from a cdf of middle length. Measured, us, one
// level / two: 64 draws from 1000, 100000, 10^7 rows 13 / 16, 13 / 20, 13 / 67; 2^18 draws from 100000
// 16 / 23; 2^20 draws from 1000, 8192, 100000, 10^6, 2 10^6, 10^7 17 / 16, 30 / 19, 51 / 38, 76 / 70,
// 100 / 109, 158 / 191; 2^23 draws from 64, 1000, 100000, 10^6, 2 10^6 62 / 60, 84 / 67, 337 / 193, 526 / 444,
// 697 / 771.
constexpr int64_t kTwoLevelDraws = 1 << 20, kTwoLevelMinM = 1000, kTwoLevelMaxM = 1 << 20;

__global__ __launch_bounds__(kSampleThreads) void sample_stream_kernel(const double* __restrict__ cdf, int64_t m,
                                                                       uint32_t key0, uint32_t key1, int64_t k0,
                                                                       int64_t K, int eta,
                                                                       int32_t* __restrict__ out) {
  __shared__ double piv[kPivots];
  // pivot p is the last cdf value of stretch p, rows [p * len, (p + 1) * len)
  const int64_t len = (m + kPivots - 1) / kPivots;
  const int np = (int)((m + len - 1) / len);
  for (int p = threadIdx.x; p < np; p += kSampleThreads) {
    const int64_t e = (int64_t)(p + 1) * len;
    piv[p] = cdf[(e < m ? e : m) - 1];
  }
  const double total = cdf[m - 1];
  __syncthreads();
  const int64_t N = K * (int64_t)eta;
  const int64_t per = (int64_t)kSampleThreads * kIlp;
  for (int64_t base = blockIdx.x * per; base < N; base += gridDim.x * per) {
    double target[kIlp];
    int lo[kIlp], hi[kIlp];
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
      target[u] = draw_target(base + u * kSampleThreads + threadIdx.x, eta, k0, key0, key1, total);
      lo[u] = 0;
      hi[u] = np;
    }
    // first pivot above the target: the stretch that holds the row (np: none, the row is m - 1)
    for (int w = np; w > 0; w >>= 1) {
#pragma unroll
      for (int u = 0; u < kIlp; ++u) {
        const int mid = (lo[u] + hi[u]) >> 1;
        const bool open = lo[u] < hi[u], up = piv[mid < np ? mid : np - 1] > target[u];
        hi[u] = open && up ? mid : hi[u];
        lo[u] = open && !up ? mid + 1 : lo[u];
      }
    }
    int64_t a[kIlp];
    int left[kIlp];
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
      // rows [a, a + left) are still to be searched; the last row of the stretch is known to hold
      a[u] = (int64_t)lo[u] * len;
      const int64_t z = a[u] + len < m ? a[u] + len : m;
      left[u] = lo[u] < np ? (int)(z - a[u]) - 1 : 0;
    }
    for (int64_t w = len; w > 0; w >>= 1) {
#pragma unroll
      for (int u = 0; u < kIlp; ++u) {
        const int half = left[u] >> 1;
        const int64_t mid = a[u] + half;
        const bool open = left[u] > 0, up = cdf[mid < m ? mid : m - 1] > target[u];
        a[u] = open && !up ? mid + 1 : a[u];
        left[u] = open ? (up ? half : left[u] - half - 1) : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
      const int64_t e = base + u * kSampleThreads + threadIdx.x;
      if (e < N) out[e] = (int32_t)(a[u] < m ? a[u] : m - 1);
    }
  }
}

// ||a_i||^2 in double (row i read once, coalesced), divided by row_w[i] when given (the
// sampling weights ||a_i||^2 / w_i of variant v4, Sec. 5).
template <typename T>
__global__ void rownorm2_f64_kernel(const T* __restrict__ A, int64_t m, int64_t n, int64_t ld,
                                    const T* __restrict__ row_w, double* __restrict__ w) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < m; i += nwaves) {
    const double s = row_sq(A + i * ld, n, lane);
    if (lane == 0) w[i] = row_w ? s / (double)row_w[i] : s;
  }
}

// Chunk c covers [c * kScanChunk, (c + 1) * kScanChunk): its sum (thread-sequential, then threads in order).
__global__ __launch_bounds__(kScanThreads) void scan_chunk_sums(const double* __restrict__ w, int64_t m,
                                                                double* __restrict__ csum) {
  __shared__ double part[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j)
    if (base + j < m) s += w[base + j];
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kScanThreads; ++i) t += part[i];
    csum[blockIdx.x] = t;
  }
}

// Exclusive prefix of the chunk sums, in chunk order (one thread).
__global__ void scan_chunk_prefix(double* csum, int64_t nchunks) {
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int64_t c = 0; c < nchunks; ++c) {
    const double v = csum[c];
    csum[c] = s;
    s += v;
  }
}

// Inclusive scan inside each chunk, offset by the chunk's prefix.
__global__ __launch_bounds__(kScanThreads) void scan_chunk_apply(const double* __restrict__ w, int64_t m,
                                                                 const double* __restrict__ cpre,
                                                                 double* __restrict__ cdf) {
  __shared__ double part[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
  double v[kScanPer];
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    v[j] = base + j < m ? w[base + j] : 0.0;
    s += v[j];
  }
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {  // exclusive prefix of the thread sums, in thread order
    double t = 0.0;
    for (int i = 0; i < kScanThreads; ++i) {
      const double x = part[i];
      part[i] = t;
      t += x;
    }
  }
  __syncthreads();
  double r = cpre[blockIdx.x] + part[threadIdx.x];
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    r += v[j];
    if (base + j < m) cdf[base + j] = r;
  }
}

size_t sampling_cdf_ws_bytes(int64_t m) {
  const int64_t nch = (m + kScanChunk - 1) / kScanChunk;
  return ((size_t)m * sizeof(double) + 255) / 256 * 256 + ((size_t)nch * sizeof(double) + 255) / 256 * 256;
}

static void launch_scan(const double* w, int64_t m, double* cdf, double* csum, hipStream_t stream) {
  const int64_t nch = (m + kScanChunk - 1) / kScanChunk;
  hipLaunchKernelGGL(scan_chunk_sums, dim3((unsigned)nch), dim3(kScanThreads), 0, stream, w, m, csum);
  hipLaunchKernelGGL(scan_chunk_prefix, dim3(1), dim3(64), 0, stream, csum, nch);
  hipLaunchKernelGGL(scan_chunk_apply, dim3((unsigned)nch), dim3(kScanThreads), 0, stream, w, m, csum, cdf);
}

template <typename T>
hipError_t launch_sampling_cdf(const T* A, int64_t m, int64_t n, int64_t ld, const T* row_w, double* cdf, void* ws,
                               hipStream_t stream) {
  double* w = (double*)ws;
  double* csum = (double*)((unsigned char*)ws + ((size_t)m * sizeof(double) + 255) / 256 * 256);
  const int64_t waves = m < 65536 ? m : 65536;
  hipLaunchKernelGGL(rownorm2_f64_kernel<T>, dim3((unsigned)((waves * 64 + 255) / 256)), dim3(256), 0, stream, A, m,
                     n, ld, row_w, w);
  launch_scan(w, m, cdf, csum, stream);
  return hipGetLastError();
}

hipError_t launch_sampling_cdf_weights(const double* w, int64_t m, double* cdf, void* ws, hipStream_t stream) {
  double* csum = (double*)((unsigned char*)ws + ((size_t)m * sizeof(double) + 255) / 256 * 256);
  launch_scan(w, m, cdf, csum, stream);
  return hipGetLastError();
}

hipError_t launch_sample_stream(const double* cdf, int64_t m, uint64_t seed, int64_t k0, int64_t K, int eta,
                                int32_t* out, hipStream_t stream) {
  const int64_t N = K * (int64_t)eta;
  if (N == 0) return hipSuccess;
  if (N < kTwoLevelDraws || m < kTwoLevelMinM || m > kTwoLevelMaxM) {
    int64_t blocks = (N + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(sample_direct_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, cdf, m, (uint32_t)seed,
                       (uint32_t)(seed >> 32), k0, K, eta, out);
    return hipGetLastError();
  }
  // two 1024-thread workgroups a CU at most, so that each fills its pivots once for many searches
  int64_t blocks = (N + kSampleThreads * kIlp - 1) / (kSampleThreads * kIlp);
  if (blocks > kSampleBlocks) blocks = kSampleBlocks;
  hipLaunchKernelGGL(sample_stream_kernel, dim3((unsigned)blocks), dim3(kSampleThreads), 0, stream, cdf, m, (uint32_t)seed,
                     (uint32_t)(seed >> 32), k0, K, eta, out);
  return hipGetLastError();
}

template hipError_t launch_sampling_cdf<float>(const float*, int64_t, int64_t, int64_t, const float*, double*,
                                               void*, hipStream_t);
template hipError_t launch_sampling_cdf<double>(const double*, int64_t, int64_t, int64_t, const double*, double*,
                                                void*, hipStream_t);

}  // namespace rsk
