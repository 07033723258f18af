// Dense RSKA, float32, register-tile step for the batched launch (rska_batched_rt).
//
// The step of the single-system register-tile kernel (rska_dense_rt in rsk_dense_rt_kernel.hpp: same
// lane layout, LDS prefetch of the next step's first slots and exchange protocol), written as a device
// function for a workgroup that solves one system of a batch after another. What differs:
//  * ranks map to column slices in order (the ranks of a system are drawn from a ticket queue,
//    so their XCDs are not known);
//  * only the chunk slots of a lane that hold the system's columns (cplr <= CPL) and the passes
//    that hold rows of the step are loaded and used;
//  * a last float4 of a row that reaches past n (rows padded to a multiple of 4 floats) has its
//    padding masked to zero before the dots and the update;
//  * global memory is read through address-space-1 pointers (the pointers come from a
//    descriptor in memory and would otherwise be FLAT loads, whose count also gates every LDS
//    wait of the step);
//  * the issuing waves wait for their LDS prefetch with the count of HBM slot loads they issued
//    after it, which varies with the system;
//  * rows are reduced by the waves that do not issue the prefetch, and a small system's in one hop, a
//    row a thread.
//
// What bounds it: a step's chain of latencies, 6.4 us for a workgroup's 17 KB of rows and 13 us for
// 160 KB, of which HBM's share is 7 us. 512 systems of up to 8000 x 4000, 100 steps: 22.6 ms with the
// indices fetched at the top of the step that needs them, the tile's bounds in vector registers (each
// of its branches a mask), a prefetch loop that worked out each slot by itself (2.7 us where it had
// next to nothing to load) and two hops for every system of more than 32 rows; 15.0 without these.
#pragma once
#include "rsk_device.hpp"
#include "rsk_kernels.hpp"

namespace rsk {

namespace {

constexpr int kMaxG = 256;  // workgroups the exchange code is unrolled for (4 slots per lane)

__device__ __forceinline__ float dot4(float4 a, float4 b) {
  float s = a.x * b.x;
  s += a.y * b.y;
  s += a.z * b.z;
  s += a.w * b.w;
  return s;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Sum over the 16 lanes of a DPP row; every lane gets it.
__device__ __forceinline__ float row_lanes_sum(float v) {
  v += dpp<0x128>(v);  // row_ror:8
  v += dpp<0x124>(v);  // row_ror:4
  v += dpp<0x122>(v);  // row_ror:2
  v += dpp<0x121>(v);  // row_ror:1
  return v;
}

}  // namespace

// s_waitcnt until at most n vector memory loads of the wave are outstanding (n wave-uniform,
// 0 <= n <= N): the count is an immediate, so uniform branches pick the constant.
template <int N>
__device__ __forceinline__ void wait_vm_at_most(int n) {
  if constexpr (N <= 0) {
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
  } else {
    if (n >= N) __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
    else wait_vm_at_most<N - 1>(n);
  }
}

// One solve on the register tile. g is this workgroup's rank among the a.G that solve the system, its
// columns slice g, cplr the chunk slots of a lane that hold columns of the widest slice.
// PF_BYTES: LDS for the next step's prefetched slots.
template <int NT, int RP, int CPL, int PF_BYTES>
__device__ __forceinline__ void rt_run(const DenseArgs<float>& a, const int g, const int cplr) {
  constexpr int kRtThreads = NT;
  constexpr int kRtWaves = NT / 64;
  constexpr int RL = 16;                          // rows a wave holds per pass
  constexpr int CL = 4;                           // lanes of one row
  constexpr int kRtRowsPerPass = kRtWaves * RL;
  constexpr int SW = 4 * CL * CPL;                // floats of the widest slice
  // the waves that reduce rows (the others issue the LDS prefetch: a wave's loads return in order, so an
  // issuing wave would see the partials it polls only after its share of the prefetch), and rows a wave
  constexpr int kOwners = kRtWaves / 2;
  constexpr int kOwnMax = kRtOwnMax * kRtWaves / kOwners;
  static_assert(64 * kOwners == kBrtOneHopRows, "one hop: a row an owner thread");
  // A form of this step for 256 threads, two workgroups a CU, with the systems' descriptors in scalar registers did not
  // finish a test, and reading it did not show why: another thread count needs that answered first.
  static_assert(NT == 512, "one 512-thread workgroup a CU; a 256-thread form hung for a cause not found");
  static_assert(SW <= NT, "the slice's columns, one a thread");
  __shared__ float4 xs4[CL * CPL];                // x* slice
  __shared__ float4 xv4[CL * CPL];                // x slice
  __shared__ float4 red[kRtWaves][CL * CPL];      // per-wave column sums
  __shared__ float cs[RP * kRtRowsPerPass];        // step coefficients
  __shared__ double mon[2 * kRtWaves + 2];
  __shared__ int orflag[2];  // step-parity flag words of the block OR
  // next-step tile slots prefetched into LDS: (p, r) with s = p * CPL + r < NPF; LDS slot s * NT + tid
  // holds tile[p][r] of thread tid. PL passes hold prefetched slots.
  constexpr int kPfBudget = PF_BYTES / (NT * 16);
  constexpr int NPF = RP * CPL < kPfBudget ? RP * CPL : kPfBudget;
  constexpr int PL = (NPF + CPL - 1) / CPL;
  constexpr int kHbmSlots = RP * CPL - NPF;
  static_assert(kHbmSlots < 64, "vmcnt holds at most 63");
  __shared__ float4 pf[NPF * NT];
  __shared__ int nrow[PL * kRtRowsPerPass];  // rows of the passes holding prefetched slots

  const int G = a.G, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int eta = a.eta;
  const int sl = lane / RL, ri = lane % RL;

  // slice in 4-chunk (64-byte) units
  const int64_t nunits = (a.nchunks + 3) / 4;
  const int64_t u0 = (int64_t)g * nunits / G, u1 = (int64_t)(g + 1) * nunits / G;
  const int64_t q0 = u0 * 4;
  int64_t q1 = u1 * 4;
  if (q1 > a.nchunks) q1 = a.nchunks;
  const int wq = (int)(q1 - q0);
  const int64_t c0 = q0 * 4;
  // last chunk of the row reachable from this slice (clamp target)
  const int qlast = (int)(a.nchunks - 1 - q0);
  // a loaded chunk at or past qlast is the row's last one, whose elements at or past n % 4 are row
  // padding (kept out of the dots and the update)
  const int nrem = (int)(a.n & 3);
  // chunk slots r < cpl of a lane and passes p < np of the wave are loaded and used (both in scalar
  // registers: branches, not masks)
  auto passes_of = [&](int wv) { return (eta - RL * wv + kRtRowsPerPass - 1) / kRtRowsPerPass; };
  int cpl = __builtin_amdgcn_readfirstlane(cplr), np = __builtin_amdgcn_readfirstlane(passes_of(wave));
  auto son = [&](int r) { return r < cpl; };
  auto pon = [&](int p) { return p < np; };
  int nhbm = 0;  // next-step slots this wave loads from HBM (not from the LDS prefetch)
#pragma unroll
  for (int p = 0; p < RP; ++p)
#pragma unroll
    for (int r = 0; r < CPL; ++r)
      if (p * CPL + r >= NPF && son(r) && pon(p)) ++nhbm;
  auto mask_tail = [&](float4& v, int q) {
    if (nrem && q >= qlast) {
      if (nrem < 2) v.y = 0.f;
      if (nrem < 3) v.z = 0.f;
      v.w = 0.f;
    }
  };
  float* xs = reinterpret_cast<float*>(xs4);
  float* xv = reinterpret_cast<float*>(xv4);

  // rows this workgroup reduces: a contiguous block (two hops) or all (one hop)
  const int per = a.two_hop ? (eta + G - 1) / G : eta;
  const int ot0 = a.two_hop ? g * per : 0;
  const int ot1 = (ot0 + per < eta) ? ot0 + per : eta;

  if (tid < 2) orflag[tid] = 0;
  for (int j = tid; j < SW; j += kRtThreads) {
    const int64_t c = c0 + j;
    const float z = (a.warm && j < wq * 4 && c < a.n) ? load_global(a.x_star + c) : 0.f;
    xs[j] = z;
    xv[j] = shrink(z, a.lambda);
  }

  // Prefetched per-step inputs: the lane's rows of the step (tile rows), and
  // for the rows this wave reduces, b and ||a||^2 (over w) of the sampled rows.
  // The row indices load at fixed in-range positions with no branch, all before
  // the first is checked: a load inside a branch is waited for at once, one
  // round trip each.
  int rowi[RP];
  float ob = 0.f, orn = 1.f;  // lane j: those of the wave's row j
  int lerr = 0;
  // raw indices of the lane's rows of step k (the next one's, fetched during the step before it)
  int iraw[RP], oi = 0;
  auto fetch_rows = [&](int64_t k) {
    const int32_t* tk = a.idx + k * (int64_t)eta;
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      const int t = p * kRtRowsPerPass + RL * wave + ri;
      iraw[p] = load_global(tk + (t < eta ? t : 0));
    }
  };
  auto check_rows = [&](int (&ri_out)[RP], int& err) {
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      const int t = p * kRtRowsPerPass + RL * wave + ri;
      int i = iraw[p];
      if (t >= eta) i = -1;
      else if (i < 0 || (int64_t)i >= a.m) { err = ST_INDEX; i = -1; }
      ri_out[p] = i;
    }
  };
  // Two hops: wave w < kOwners reduces rows tw + kOwners * j < ot1, lane j finishing row j. One hop: the
  // owner waves' threads one row each (eta <= 64 kOwners), every slice's partial by the thread itself.
  const int tw = wave < kOwners ? ot0 + wave : ot1;
  int nown = a.two_hop && tw < ot1 ? (ot1 - tw + kOwners - 1) / kOwners : 0;
  if (nown > kOwnMax) nown = kOwnMax;
  const bool omine = a.two_hop ? lane < nown : wave < kOwners && tid < eta;
  const int orow = omine ? (a.two_hop ? tw + kOwners * lane : tid) : 0;
  auto owned_index = [&](int64_t k) { return load_global(a.idx + k * (int64_t)eta + orow); };
  auto owned_inputs = [&](int i, float& b, float& rn) {
    const int ic = i >= 0 && (int64_t)i < a.m ? i : 0;  // (a bad index stops its step before they are used)
    b = load_global(a.b + ic);
    rn = weighted_rn(a.r2, a.row_w, ic);
  };
  if (a.K > 0) {
    fetch_rows(0);
    owned_inputs(owned_index(0), ob, orn);
    check_rows(rowi, lerr);
    const int64_t k1 = a.K > 1 ? 1 : 0;
    fetch_rows(k1);
    oi = owned_index(k1);
  }
  int64_t k_done = 0;
  int stop_code = 0;
  // every workgroup read the same indices, so all skip the loop alike
  if (__syncthreads_or(lerr)) stop_code = ST_INDEX;

  // LDS prefetch of slots s < NPF: the issuing waves (the upper half) load, for consumer wave j,
  // tile slot (p, r) of each of its 64 lanes; lane l of the issuing wave stands for lane l of
  // wave j, so the 64 x 16 B that one global_load_lds writes are the 64 consumers' slots in order.
  auto publish_rows = [&](const int (&rows)[RP]) {
#pragma unroll
    for (int p = 0; p < PL; ++p)
      if (sl == 0) nrow[p * kRtRowsPerPass + RL * wave + ri] = rows[p];
  };
  auto issue_prefetch = [&]() {
    if (wave < kOwners) return;
    // (pass, consumer wave) pairs over the issuing waves
    for (int I = wave - kOwners; I < PL * kRtWaves; I += kRtWaves - kOwners) {
      const int j = I % kRtWaves, p = I / kRtWaves;
      if (p >= passes_of(j)) continue;
      const int row = nrow[p * kRtRowsPerPass + RL * j + ri];
      const float* rp = a.A + (int64_t)(row < 0 ? 0 : row) * a.ld + c0;
      const int rn = NPF - p * CPL < cpl ? NPF - p * CPL : cpl;
      for (int r = 0; r < rn; ++r) {
        const int q = sl + CL * r;
        __builtin_amdgcn_global_load_lds(rp + 4 * (q < qlast ? q : qlast),
                                         (__attribute__((address_space(3))) void*)&pf[(p * CPL + r) * NT + 64 * j], 16,
                                         0, 0);
      }
    }
  };
  if (!stop_code && a.K > 0) {
    publish_rows(rowi);
    __syncthreads();
    issue_prefetch();
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }

  // The step's tile. Slots p * CPL + r < NPF come from the LDS prefetch; the others load from
  // HBM: for step 0 here, for step k + 1 at the end of step k's update (rows past eta read row 0
  // and are never used).
  float4 tile[RP][CPL];
  if (!stop_code && a.K > 0) {
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      if (!pon(p)) continue;
      const float* rowp = a.A + (int64_t)(rowi[p] < 0 ? 0 : rowi[p]) * a.ld + c0;
#pragma unroll
      for (int r = 0; r < CPL; ++r) {
        if (p * CPL + r < NPF || !son(r)) continue;
        const int q = sl + CL * r;  // clamped into the row: past the slice it meets x = 0
        tile[p][r] = load_global_f4(rowp + 4 * (q < qlast ? q : qlast));
      }
    }
  }

  for (int64_t k = 0; k < a.K && !stop_code; ++k) {
    // Re-derive the lane coordinates from an opaque copy of the thread id each
    // step: otherwise the compiler hoists every lane-dependent address out of
    // the loop and keeps it in VGPRs that the register tile needs.
    int tidl = threadIdx.x;
    asm volatile("" : "+v"(tidl));
    const int tid = tidl, lane = tidl & 63, wave = tidl >> 6, sl = lane / RL, ri = lane % RL;
    int cpv = cplr, npv = passes_of(wave);
    asm volatile("" : "+v"(cpv), "+v"(npv));
    cpl = __builtin_amdgcn_readfirstlane(cpv);
    np = __builtin_amdgcn_readfirstlane(npv);
    const unsigned tag = (unsigned)(k + 1);
    u64* xP = a.xP + (size_t)(k & 1) * G * eta;
    const bool has_next = k + 1 < a.K;

#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int r = 0; r < CPL; ++r)
        if (p * CPL + r < NPF && son(r) && pon(p)) tile[p][r] = pf[(p * CPL + r) * NT + tid];
    int rown[RP];
#pragma unroll
    for (int p = 0; p < RP; ++p) rown[p] = -1;
    int nerr = 0;

    // partial dots, published pass by pass
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      if (!pon(p)) continue;
      float acc = 0.f;
#pragma unroll
      for (int r = 0; r < CPL; ++r) {
        if (!son(r)) continue;
        mask_tail(tile[p][r], sl + CL * r);
        acc += dot4(tile[p][r], xv4[sl + CL * r]);
      }
#pragma unroll
      for (int o = RL; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
      const int t = p * kRtRowsPerPass + RL * wave + ri;
      if (sl == 0 && t < eta) put_tagged(&xP[(size_t)g * eta + t], acc, tag);
      __builtin_amdgcn_sched_barrier(0);
    }
    // b and ||a||^2 of the next step's owned rows and the indices of the step after it, under this
    // step's exchange: in one hop before its polls; in two, between the hops, since a wave's polls
    // return after the loads it issued before them, and every workgroup waits for the owners' polls
    // (40 systems of 8000 columns, 300 rows 123 -> 115 us a step; one hop gains nothing by it)
    float obn = 0.f, ornn = 1.f;
    auto fetch_ahead = [&]() {
      if (wave < kOwners) owned_inputs(oi, obn, ornn);
      const int64_t k2 = k + 2 < a.K ? k + 2 : a.K - 1;
      fetch_rows(k2);
      oi = owned_index(k2);
    };
    if (has_next) {
      // every wave has consumed its LDS slots (the dots used them): the next step's may land
      check_rows(rown, nerr);
      publish_rows(rown);
      __syncthreads();
      issue_prefetch();
      if (!a.two_hop) fetch_ahead();
    }
    int bad = 0;
    // reduce the owned rows over the slices; lane j: c_t = (alpha/eta)(r_t - b)/||a||^2 of row j
    float osum = 0.f;
    if (!a.two_hop) {
      if (omine) {
        // four slices a round trip: eight take 16 registers more, and what the two-hop form then spills
        // waits behind the prefetch when it is loaded again (the 40 systems 115 -> 103 us a step)
        constexpr int kN = 4;
        for (int s0 = 0; s0 < G; s0 += kN) {
          float v[kN];
          wait_tagged_batch(&xP[(size_t)s0 * eta + orow], (size_t)eta, G - s0 < kN ? G - s0 : kN, tag, v, lerr);
#pragma unroll
          for (int i = 0; i < kN; ++i) osum += v[i];
        }
      }
    } else if (G <= 64) {
      // one slice a lane: the wave's rows are polled together, one round trip for all of them
      float v[kOwnMax];
      wait_tagged_batch(&xP[(size_t)lane * eta + (nown ? tw : 0)], kOwners, lane < G ? nown : 0, tag, v, lerr);
#pragma unroll
      for (int j = 0; j < kOwnMax; ++j) {
        if (j < nown) {
          const float sum = wave_sum(v[j]);
          if (lane == j) osum = sum;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < kOwnMax; ++j) {
        const int t = tw + kOwners * j;
        if (t < ot1) {
          float v[kMaxG / 64];
          wait_tagged_batch(&xP[(size_t)lane * eta + t], (size_t)64 * eta, (G - lane + 63) / 64, tag, v, lerr);
          float sum = 0.f;
#pragma unroll
          for (int i = 0; i < kMaxG / 64; ++i) sum += v[i];
          sum = wave_sum(sum);
          if (lane == j) osum = sum;
        }
      }
    }
    if (omine) {
      float c;
      if (orn == 0.f) { c = NAN; set_status(a.status, ST_ZERO_ROW); }
      else c = (a.alpha / (float)eta) * (osum - ob) / orn;
      if (a.two_hop) {
        put_tagged(&a.xC[orow], c, tag);
      } else {
        cs[orow] = c;
        bad |= !isfinite(c);
      }
    }
    if (has_next && a.two_hop) fetch_ahead();
    ob = obn;
    orn = ornn;
    if (a.two_hop && tid < kRtRowsPerPass) {
      float v[RP];
      wait_tagged_batch(&a.xC[tid], kRtRowsPerPass, (eta - tid + kRtRowsPerPass - 1) / kRtRowsPerPass, tag,
                        v, lerr);
#pragma unroll
      for (int i = 0; i < RP; ++i)
        if (tid + kRtRowsPerPass * i < eta) {
          cs[tid + kRtRowsPerPass * i] = v[i];
          bad |= !isfinite(v[i]);
        }
    }
    if (lerr) set_status(a.status, lerr);
    // One or-barrier agrees on every condition of the step (an expired wait, a non-finite
    // coefficient, a bad index in the next step), so that the barriers after the update are
    // plain ones, which do not wait for the next step's loads; every workgroup holds the same
    // c_t and the same indices, so all stop at the same step.
    // Block OR in one barrier: the flag word of this step's parity collects the bits, the other
    // word (last read before the previous step's final barrier) is cleared for the next step.
    const int flag = (lerr ? 1 : 0) | (bad ? 2 : 0) | (nerr ? 4 : 0);
    if (flag) atomicOr(&orflag[k & 1], flag);
    __syncthreads();
    const int fl = orflag[k & 1];
    if (tid == 0) orflag[(k + 1) & 1] = 0;
    if (fl & 1) { stop_code = ST_ABORTED; break; }
    if (fl & 2) { stop_code = ST_NONFINITE; break; }
    const int next_bad = fl & 4;

    // transposed update: per chunk slot, sum over own rows, then the 16 lanes
    // holding that chunk, then the waves
    float cp[RP];
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      const int t = p * kRtRowsPerPass + RL * wave + ri;
      cp[p] = t < eta ? cs[t] : 0.f;
    }
    const bool load_next = has_next && !next_bad;
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      if (!son(r)) continue;
      float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int p = 0; p < RP; ++p) {
        if (!pon(p)) continue;
        d.x += cp[p] * tile[p][r].x;
        d.y += cp[p] * tile[p][r].y;
        d.z += cp[p] * tile[p][r].z;
        d.w += cp[p] * tile[p][r].w;
      }
      d.x = row_lanes_sum(d.x);
      d.y = row_lanes_sum(d.y);
      d.z = row_lanes_sum(d.z);
      d.w = row_lanes_sum(d.w);
      if (ri == 0) red[wave][sl + CL * r] = d;
    }
    // the tile is used up: the next step's HBM slots load now, row by row (a row's chunks issued
    // back to back keep the DRAM pages open), and stay in flight across the plain barriers
    if (load_next) {
#pragma unroll
      for (int p = 0; p < RP; ++p) {
        if (!pon(p)) continue;
        const float* rowp = a.A + (int64_t)(rown[p] < 0 ? 0 : rown[p]) * a.ld + c0;
#pragma unroll
        for (int r = 0; r < CPL; ++r) {
          if (p * CPL + r < NPF || !son(r)) continue;
          const int q = sl + CL * r;
          tile[p][r] = load_global_f4(rowp + 4 * (q < qlast ? q : qlast));
        }
      }
    }
    __syncthreads();  // publishes red[]
    if (tid < 4 * wq) {  // chunks past the slice carry clamped data: discarded
      float dsum = 0.f;
#pragma unroll
      for (int w = 0; w < kRtWaves; ++w) dsum += reinterpret_cast<const float*>(red[w])[tid];
      const float z = xs[tid] - dsum;
      xs[tid] = z;
      xv[tid] = shrink(z, a.lambda);
    }
    k_done = k + 1;
    // the LDS prefetch has landed before the barrier: the wave issued at least nhbm loads after it
    // (older ones are done at vmcnt <= nhbm)
    if (wave >= kOwners) {
      if (!load_next) __builtin_amdgcn_s_waitcnt(0);
      else wait_vm_at_most<kHbmSlots>(nhbm);
    }
    __syncthreads();

    if (a.xref && a.check_every > 0 && (k + 1) % a.check_every == 0) {
      const unsigned mtag = (unsigned)((k + 1) / a.check_every);
      double e2 = 0.0, r2s = 0.0;
      for (int j = tid; j < wq * 4; j += kRtThreads) {
        const int64_t c = c0 + j;
        if (c < a.n) {
          const double rf = (double)load_global(a.xref + c);
          const double d = (double)xv[j] - rf;
          e2 += d * d;
          r2s += rf * rf;
        }
      }
      e2 = wave_sum(e2);
      r2s = wave_sum(r2s);
      if (lane == 0) { mon[2 * wave] = e2; mon[2 * wave + 1] = r2s; }
      __syncthreads();
      if (tid == 0) {
        double se = 0.0, sr = 0.0;
        for (int w = 0; w < kRtWaves; ++w) { se += mon[2 * w]; sr += mon[2 * w + 1]; }
        put_tagged(&a.xM[(size_t)g * 4], se, mtag);
        put_tagged(&a.xM[(size_t)g * 4 + 2], sr, mtag);
      }
      __syncthreads();
      if (wave == 0) {
        double se = 0.0, sr = 0.0;
        for (int q = lane; q < G; q += 64) {
          se += wait_tagged<double>(&a.xM[(size_t)q * 4], mtag, lerr);
          sr += wait_tagged<double>(&a.xM[(size_t)q * 4 + 2], mtag, lerr);
        }
        se = wave_sum(se);
        sr = wave_sum(sr);
        if (lane == 0) {
          const double err = sr > 0.0 ? sqrt(se / sr) : sqrt(se);
          if (g == 0 && a.err_hist) a.err_hist[mtag - 1] = err;
          mon[2 * kRtWaves] = err;
        }
      }
      if (lerr) set_status(a.status, lerr);
      if (__syncthreads_or(lerr)) { stop_code = ST_ABORTED; break; }
      if (a.tol > 0.0 && mon[2 * kRtWaves] <= a.tol) break;
    }
    if (next_bad) { stop_code = ST_INDEX; break; }
#pragma unroll
    for (int p = 0; p < RP; ++p) rowi[p] = rown[p];
  }
  if (stop_code && tid == 0) set_status(a.status, stop_code);
  __builtin_amdgcn_s_waitcnt(0);  // no load of a step that will not run stays in flight
  __syncthreads();
  for (int j = tid; j < wq * 4; j += kRtThreads) {
    const int64_t c = c0 + j;
    if (c < a.n) {
      store_global(a.x_star + c, xs[j]);
      store_global(a.x + c, xv[j]);
    }
  }
  if (g == 0 && tid == 0) a.status[1] = (int)k_done;
}

}  // namespace rsk
