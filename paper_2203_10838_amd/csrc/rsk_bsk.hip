// Block sparse Kaczmarz, eq. (bsk) of Sec. 1.1 (eta <= kBskMaxEta rows a step):
//   x*_{k+1} = x*_k - w A_tau^T (A_tau x_k - b_tau) / ||A_tau||_2^2,  x_{k+1} = S_lambda(x*_{k+1}).
// ||A_tau_k||_2^2 depends on the step's rows only, not on x, so it is computed for every step up
// front: bsk_gram_f32 / bsk_gram_f64 form the Gram matrices A_tau A_tau^T on the matrix cores,
// bsk_lambda_max their largest eigenvalues to rounding (Householder tridiagonalisation in double, Sturm-sequence
// multisection). It writes the per-step relaxation alpha_k = eta w / ||A_tau_k||_2^2, with which the
// RSKA step with unit row norms, (alpha_k / eta) sum_t (<a_t, x> - b_t) a_t, is the block step of
// eq. (bsk); the iteration itself then runs in the persistent RSKA kernels.
#include "rsk_dense_run.hpp"

namespace rsk {

namespace {

constexpr int kE = kBskMaxEta;

}  // namespace

// float32: the Gram matrix of step kbase + (step of the workgroup), NB = ceil(eta / 16) row blocks.
// One wave forms one 16 x 16 block on or below the diagonal, over all n columns in ascending order in
// one accumulator: v_mfma_f32_16x16x4f32 adds its four products as an ascending chain of fused
// multiply-adds, so the entries are those of a plain loop over the columns, to the bit (which a column
// split would not be). The NP = 1 or 2 workgroups of a step (eight apart, on one XCD, whose L2 serves
// the second reading) share the blocks; tiles of kGc columns pass through two LDS buffers, and the
// loads of two tiles ahead are in registers, as a tile's products last less than a load. Bound by the
// matrix cores, 32 cycles a product and a chain of n / 4 of them: 100 steps of 64 rows of 20000
// columns in 230 us (VALU products of one workgroup a step: 1320 us).
constexpr int kGc = 128, kGp = kGc + 4;  // pitch: the 64 lanes of a fragment read hit 64 banks
template <int NB>
struct GramShape {
  static constexpr int blocks = NB * (NB + 1) / 2, parts = NB >= 3 ? 2 : 1, waves = (blocks + parts - 1) / parts;
};
template <int NB>
__global__ __launch_bounds__(64 * GramShape<NB>::waves) void bsk_gram_f32(
    const float* __restrict__ A, int64_t m, int64_t n, int64_t ld, const int* __restrict__ tau0, int eta,
    int64_t kbase, int64_t kcount, double* __restrict__ gram, int* status) {
  using GS = GramShape<NB>;
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float vu __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int NT = 64 * GS::waves, ROWS = 16 * NB, CPR = kGc / 4, PASS = (ROWS * CPR + NT - 1) / NT;
  __shared__ __align__(16) float tile[2][ROWS * kGp];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int64_t id = blockIdx.x, step = GS::parts == 1 ? id : id / 16 * 8 + id % 8;
  const int part = GS::parts == 1 ? 0 : (int)(id / 8 % 2);
  if (step >= kcount) return;
  // this wave's block (bi, bj), bj <= bi, in row-major order of the lower triangle
  const int q = part * GS::waves + wave;
  int bi = 0;
  while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
  const int bj = q - bi * (bi + 1) / 2;
  const bool has = q < GS::blocks;
  // tile element: row tr[u] (of ROWS), columns tc[u] .. tc[u] + 3 of the tile
  const float* rowp[PASS];
  bool ok[PASS];
  int dst[PASS];
#pragma unroll
  for (int u = 0; u < PASS; ++u) {
    const int e = tid + NT * u, tr = e / CPR < ROWS ? e / CPR : ROWS - 1, tc = e % CPR * 4;
    // rows past eta repeat the last one (their products are not used); an index out of range makes a
    // zero row, as it is never read
    const int r = tau0[(kbase + step) * eta + (tr < eta ? tr : eta - 1)];
    ok[u] = r >= 0 && (int64_t)r < m;
    if (!ok[u]) set_status(status, ST_INDEX);
    rowp[u] = A + (int64_t)(ok[u] ? r : 0) * ld + tc;
    dst[u] = tr * kGp + tc;
  }
  auto load = [&](int64_t cb, vu (&v)[PASS]) {
    if (cb + kGc <= n) {
#pragma unroll
      for (int u = 0; u < PASS; ++u) v[u] = *reinterpret_cast<const vu*>(rowp[u] + cb);
    } else {  // the last tile (and past it): element by element, zeros past the row
#pragma unroll
      for (int u = 0; u < PASS; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t c = cb + dst[u] % kGp + e;
          v[u][e] = c < n ? rowp[u][cb + e] : 0.f;
        }
    }
  };
  auto put = [&](const vu (&v)[PASS], int buf) {
    __builtin_amdgcn_sched_barrier(0);  // nothing of a store moves above: it would wait for its loads there
#pragma unroll
    for (int u = 0; u < PASS; ++u) {
      f4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = ok[u] ? v[u][e] : 0.f;
      *reinterpret_cast<f4*>(&tile[buf][dst[u]]) = w;  // (surplus threads of the last pass rewrite the last row)
    }
  };
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  auto products = [&](int buf) {
    if (!has) return;
    const float* ra = &tile[buf][(16 * bi + li) * kGp + lg];
    const float* rb = &tile[buf][(16 * bj + li) * kGp + lg];
#pragma unroll 8
    for (int c = 0; c < kGc; c += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[c], rb[c], acc, 0, 0, 0);
  };
  vu v0[PASS], v1[PASS];
  load(0, v0);
  load(kGc, v1);
  put(v0, 0);
  load(2 * kGc, v0);
  __syncthreads();
  // tile t's products run from LDS buffer t % 2 while tile t + 1 is stored to the other
  for (int64_t cb = 0; cb < n; cb += 2 * kGc) {
    products(0);
    if (cb + kGc >= n) break;
    put(v1, 1);
    load(cb + 3 * kGc, v1);
    __syncthreads();
    products(1);
    put(v0, 0);
    load(cb + 4 * kGc, v0);
    __syncthreads();
  }
  if (!has) return;
  double* G = gram + (size_t)step * kE * kE;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = 16 * bi + 4 * lg + v, j = 16 * bj + li;
    G[i * kE + j] = (double)acc[v];
    if (bi != bj) G[j * kE + i] = (double)acc[v];
  }
}

// float64: partial Gram matrix of step kbase + blockIdx.y over column split blockIdx.x. A lane's 16-byte
// load of V columns of row l % 16 (lane group l / 16 taking the V columns after group l / 16 - 1's)
// feeds V products: the same registers serve as the left and the right operand, and the order of k
// inside a product does not matter as both have it, so no LDS is needed. Only the NB (NB + 1) / 2
// blocks on and below the diagonal are formed. The four waves' sums are added in wave order. Bound by
// the matrix cores.
template <int NB>
__global__ __launch_bounds__(kBskThreads) void bsk_gram_f64(const double* __restrict__ A, int64_t m, int64_t n, int64_t ld,
                                                        const int* __restrict__ tau0, int eta, int64_t kbase,
                                                        int64_t wspan, double* __restrict__ gram, int* status) {
  using T = double;
  typedef double acc_t __attribute__((ext_vector_type(4)));
  constexpr int V = 16 / (int)sizeof(T), CW = 4 * V, NBLK = NB * (NB + 1) / 2;
  typedef T vt __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  __shared__ T part[kBskThreads / 64][NBLK][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int64_t k = kbase + blockIdx.y;
  const T* rowp[NB];
  bool ok[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    // rows past eta repeat the last one (their products are not used); an index out of range makes a
    // zero row, as it is never read
    const int t = 16 * b + li < eta ? 16 * b + li : eta - 1;
    const int r = tau0[k * eta + t];
    ok[b] = r >= 0 && (int64_t)r < m;
    if (!ok[b]) set_status(status, ST_INDEX);
    rowp[b] = A + (int64_t)(ok[b] ? r : 0) * ld;
  }
  const int64_t c0 = (4 * (int64_t)blockIdx.x + wave) * wspan;
  const int64_t c1 = c0 + wspan < n ? c0 + wspan : n;
  auto load = [&](int64_t cb, vt (&v)[NB], int64_t& from) {
    // the lane's V columns from col on; near the row's end its last V, of which those from col on count
    const int64_t col = cb + lg * V;
    const int64_t at = col < n - V ? col : n - V;
    from = col - at;
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = *reinterpret_cast<const vt*>(rowp[b] + at);
  };
  acc_t acc[NBLK];
#pragma unroll
  for (int q = 0; q < NBLK; ++q) acc[q] = acc_t{T(0), T(0), T(0), T(0)};
  auto products = [&](const vt (&v)[NB], int64_t from) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      T x[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) x[b] = ok[b] && e >= from ? v[b][e] : T(0);
      int q = 0;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j, ++q) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], x[j], acc[q], 0, 0, 0);
    }
  };
  if (n >= V) {
    vt v0[NB], v1[NB];
    int64_t f0 = 0, f1 = 0;
    if (c0 < c1) load(c0, v0, f0);
    for (int64_t cb = c0; cb < c1; cb += 2 * CW) {
      load(cb + CW, v1, f1);  // past the span: loaded (the row's last columns at most), not added
      products(v0, f0);
      load(cb + 2 * CW, v0, f0);
      if (cb + CW < c1) products(v1, f1);
    }
  } else if (c0 < c1) {
    vt v[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < V; ++e) v[b][e] = lg == 0 && e < n ? rowp[b][e < n ? e : 0] : T(0);
    products(v, 0);
  }
#pragma unroll
  for (int q = 0; q < NBLK; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][q][(lg + 4 * v) * 16 + li] = acc[q][v];
  __syncthreads();
  double* G = gram + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kE * kE;
  const int i = tid >> 4, j = tid & 15;
  int q = 0;
#pragma unroll
  for (int bi = 0; bi < NB; ++bi)
#pragma unroll
    for (int bj = 0; bj <= bi; ++bj, ++q) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kBskThreads / 64; ++w) s += (double)part[w][q][tid];
      G[(16 * bi + i) * kE + 16 * bj + j] = s;
      if (bi != bj) G[(16 * bj + j) * kE + 16 * bi + i] = s;
    }
}

namespace {

__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}

// LDS words written by some lanes of this wave are read by others after this
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

// Largest eigenvalue of the Gram matrix of step kbase + blockIdx.x (the sum of its column splits in
// order), by one wave: lane i holds row i in registers, which move one column to the left as each
// Householder step uses one up (the shift is part of the rank-two update), so every index is static
// and no barrier is needed. The eigenvalue by multisection: lane l tests shift s_l by the sign
// sequence of the leading minors of s_l I - T, a recurrence of two multiply-adds a row (all positive:
// s_l lies above). A chain of latencies, one wave a step: 126 us for 100 steps (400 us
// with a workgroup and four barriers a Householder step).
template <typename T>
__global__ __launch_bounds__(kBskThreads) void bsk_lambda_max(const double* __restrict__ gram, int splits, int eta,
                                                              int64_t kbase, double w, T* __restrict__ alpha_k,
                                                              double* __restrict__ norm2, int* status) {
  __shared__ double Gm[kE][kE];
  __shared__ double vs[2 * kE], ws[2 * kE], dd[kE], ee[kE];
  const int tid = threadIdx.x;
  const double* g0 = gram + (size_t)blockIdx.x * splits * kE * kE;
  constexpr int kPer = kE * kE / kBskThreads;
  double sum[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) sum[u] = 0.0;
  for (int s = 0; s < splits; ++s)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kBskThreads * u;
      // entries past eta were not formed
      sum[u] += e / kE < eta && e % kE < eta ? g0[(size_t)s * kE * kE + e] : 0.0;
    }
#pragma unroll
  for (int u = 0; u < kPer; ++u) Gm[0][tid + kBskThreads * u] = sum[u];
  if (tid < kE) vs[tid] = vs[tid + kE] = ws[tid] = ws[tid + kE] = dd[tid] = ee[tid] = 0.0;
  __syncthreads();
  if (tid >= 64) return;
  const int i = tid;
  double a[kE];  // a[j]: column k + j of row i
#pragma unroll
  for (int j = 0; j < kE; ++j) a[j] = Gm[j][i];  // symmetric
  for (int k = 0; k + 2 < eta; ++k) {
    const bool own = i > k && i < eta;
    const double xi = own ? a[0] : 0.0;
    const double nx2 = lane_sum(xi * xi, 64);
    const double x0 = __shfl(a[0], k + 1), dk = __shfl(a[0], k);
    double alpha = 0.0, beta = 0.0, vi = 0.0;
    if (nx2 > 0.0) {
      alpha = x0 > 0.0 ? -sqrt(nx2) : sqrt(nx2);
      vi = own ? (i == k + 1 ? xi - alpha : xi) : 0.0;
      beta = 1.0 / (nx2 - alpha * x0);  // 2 / <v, v>
    }
    vs[i] = vi;
    if (i == 0) { dd[k] = dk; ee[k] = alpha; }
    wave_lds_sync();
    double p0 = 0.0, p1 = 0.0;
#pragma unroll
    for (int jb = 0; jb < kE; jb += 16)
      if (k + jb < eta) {
#pragma unroll
        for (int j = jb; j < jb + 16; j += 2) {
          p0 += a[j] * vs[k + j];
          p1 += a[j + 1] * vs[k + j + 1];
        }
      }
    const double pi = own ? beta * (p0 + p1) : 0.0;
    const double pv = lane_sum(pi * vi, 64);
    // (no step where the column has nothing to eliminate or holds a NaN: a NaN row leaves the other rows'
    // eigenvalue as it is, and the solve then reports the row)
    const double wi = nx2 > 0.0 ? pi - 0.5 * beta * pv * vi : 0.0;
    ws[i] = wi;
    wave_lds_sync();
#pragma unroll
    for (int jb = 0; jb < kE; jb += 16)
      if (k + jb < eta) {
#pragma unroll
        for (int j = jb; j < jb + 16; ++j)
          a[j] = j + 1 < kE ? a[j + 1 < kE ? j + 1 : j] - (vi * ws[k + j + 1] + wi * vs[k + j + 1]) : 0.0;
      }
    wave_lds_sync();
  }
  // the last two rows: a[0] is column eta - 2 (or, with eta = 1, column 0)
  const double b0 = __shfl(a[0], eta >= 2 ? eta - 2 : 0), b1 = __shfl(a[0], eta - 1), b2 = __shfl(a[1], eta - 1);
  if (i == 0) {
    if (eta >= 2) {
      dd[eta - 2] = b0;
      ee[eta - 2] = b1;
      dd[eta - 1] = b2;
    } else {
      dd[0] = b0;
    }
  }
  wave_lds_sync();
  const double di = i < eta ? dd[i] : -INFINITY;
  const double ri = i < eta ? fabs(i > 0 ? ee[i - 1] : 0.0) + fabs(i + 1 < eta ? ee[i] : 0.0) : 0.0;
  double lo = wave_max_d(di), hi = wave_max_d(i < eta ? di + ri : -INFINITY);
  if (hi > 0.0 && hi > lo && isfinite(hi)) {
    // T / hi: its eigenvalues lie in [-2, 1] and the minors stay in range with a rescaling every 4 rows
    const double inv = 1.0 / hi;
    const double sd = i < eta ? di * inv : 0.0, se = i + 1 < eta ? (ee[i] * inv) * (ee[i] * inv) : 0.0;
    wave_lds_sync();
    dd[i] = sd;
    ee[i] = se;
    wave_lds_sync();
    double l = lo * inv, h = 1.0;
    constexpr double kParts = 65.0;
    for (int round = 0; round < 10 && h > l; ++round) {
      const double width = h - l, sg = l + width * (double)(i + 1) / kParts;
      double pp = 1.0, pc = sg - dd[0];
      bool above = pc > 0.0;
      for (int tb = 1; tb < eta; tb += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = tb + u < kE ? tb + u : kE - 1;
          const double pn = (sg - dd[t]) * pc - ee[t - 1] * pp;
          if (tb + u < eta) {
            pp = pc;
            pc = pn;
            above = above && pn > 0.0;
          }
        }
        if (pc < 1e-100) {
          pc *= 1e100;
          pp *= 1e100;
        }
      }
      // the shifts at or below the eigenvalue are a prefix of the lanes
      const int nb = (int)__popcll(__ballot(!above));
      const double nl = nb == 0 ? l : l + width * (double)nb / kParts;
      h = nb == 64 ? h : l + width * (double)(nb + 1) / kParts;
      l = nl;
    }
    lo = l * hi;
    hi = h * hi;
  }
  if (i == 0) {
    const int64_t k = kbase + blockIdx.x;
    const double s2 = 0.5 * (lo + hi);
    if (s2 > 0.0 && isfinite(s2)) {
      alpha_k[k] = (T)((double)eta * w / s2);
    } else {
      alpha_k[k] = T(0);
      set_status(status, ST_ZERO_ROW);
    }
    if (norm2) norm2[k] = s2;
  }
}

template <typename T>
__global__ void fill_value(T* p, int64_t count, T v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

template <int NB>
static void launch_gram(const BskArgs<float>& a, int64_t k, int64_t cnt, hipStream_t s) {
  using GS = GramShape<NB>;
  const int64_t wgs = GS::parts == 1 ? cnt : (cnt + 7) / 8 * 16;
  hipLaunchKernelGGL(bsk_gram_f32<NB>, dim3((unsigned)wgs), dim3(64 * GS::waves), 0, s, a.A, a.m, a.n, a.ld, a.tau,
                     a.eta, k, cnt, a.gram, a.status);
}
template <int NB>
static void launch_gram(const BskArgs<double>& a, int64_t k, int64_t cnt, hipStream_t s) {
  hipLaunchKernelGGL(bsk_gram_f64<NB>, dim3((unsigned)a.splits, (unsigned)cnt), dim3(kBskThreads), 0, s, a.A, a.m,
                     a.n, a.ld, a.tau, a.eta, k, a.wspan, a.gram, a.status);
}

template <typename T>
hipError_t launch_bsk_norms(const BskArgs<T>& a, hipStream_t s) {
  const int64_t ib = (a.m + 255) / 256;
  hipLaunchKernelGGL(fill_value<T>, dim3((unsigned)(ib < 1024 ? ib : 1024)), dim3(256), 0, s, a.ones, a.m, T(1));
  const int nb = (a.eta + 15) / 16;
  for (int64_t k = 0; k < a.K; k += a.chunk) {
    const int64_t cnt = a.K - k < a.chunk ? a.K - k : a.chunk;
    switch (nb) {
#define BSK_GRAM(NB) case NB: launch_gram<NB>(a, k, cnt, s); break;
      BSK_GRAM(1) BSK_GRAM(2) BSK_GRAM(3) BSK_GRAM(4)
#undef BSK_GRAM
      default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(bsk_lambda_max<T>, dim3((unsigned)cnt), dim3(kBskThreads), 0, s, a.gram, a.splits, a.eta, k,
                       a.w, a.alpha_k, a.norm2_hist, a.status);
  }
  return hipGetLastError();
}

template hipError_t launch_bsk_norms<float>(const BskArgs<float>&, hipStream_t);
template hipError_t launch_bsk_norms<double>(const BskArgs<double>&, hipStream_t);

}  // namespace rsk

