// hf_bodies.hpp -- the kernel bodies that horizontal fusion combines.
//
// Each body is written once, as a __device__ function of an interval (Part) and
// a barrier type.  The solo kernel instantiates it with the whole workgroup and
// the native workgroup barrier; the fused kernel instantiates it with one
// wavefront-aligned interval and the interval's LDS barrier (Sec. III-A,
// Generate algorithm: the built-ins threadIdx.x / blockDim.x become the interval
// variables tid_i / size_i, and __syncthreads becomes the interval barrier).
//
// Every body is grid-stride over work units, so it is correct for any grid and
// any interval size; units whose result is floating point are owned by one
// wavefront and reduced in a fixed order, so a fused launch reproduces the solo
// launch bit for bit whatever the split.
#pragma once
#include "hf_device.hpp"

namespace hf {

// ======================================================================= args
// Per-kind kernel arguments, filled on the host from an hf_task.

struct BnArgs {  // per-channel mean / biased variance of NCHW fp32
  const float* x;
  float* mean;
  float* var;
  uint32_t* ctr;   // [C << ctr_shift] unit arrival counters (zero between launches)
  uint32_t* part;  // [C][upc][2] per-unit (mean, M2) as float bits
  uint32_t C, HW, M, CHWm;  // M = N*HW elements per channel, CHWm = (C-1)*HW
  uint32_t upc;             // units per channel
  uint32_t total;           // C * upc
  uint32_t vec;             // float4 path: HW % 4 == 0 and x 16-byte aligned
  uint32_t ctr_shift;       // the counters lie 1 << ctr_shift words apart
  FastDiv div_hw, div_upc;
};

struct MixArgs {  // R rounds of xorshift32 + multiply-add per uint32
  const uint32_t* in;
  uint32_t* out;
  uint32_t n, n4;  // elements, and uint4 vectors in the vector path (0 otherwise)
  int32_t rounds;
};

struct HistArgs {  // 256-bin histogram of bytes
  const uint8_t* in;
  uint32_t* out;
  uint32_t* acc;  // [sums][256] merged counts (zero between launches)
  uint32_t* ctr;  // workgroup arrival counter, then (sums > 1) one per accumulator,
                  // a line apart (zero between launches)
  uint32_t n;
  uint32_t head;        // bytes before the first 16-byte aligned address
  uint32_t n16;         // aligned 16-byte vectors after the head
  uint32_t tail_start;  // head + 16 * n16
  uint32_t sums;        // accumulators: LdsHist::kSums, or 1 in caller scratch
};

struct Im2colArgs {  // patches -> columns, [N][C*kh*kw][Ho*Wo]
  const float* x;
  float* out;
  uint32_t C, H, W, kw, s, p, Ho, Wo, KK;
  uint32_t elems;           // N * C * H * W
  uint32_t items;           // N * C * kh * Ho * (Wo4 or Wo): places of the general path
  uint32_t vec;             // Wo % 4 == 0 and out 16-byte aligned
  FastDiv div_group, div_kh, div_row;  // by Ho * rowlen, kh, and rowlen = Wo4 (vector) or Wo
  uint32_t row3;            // the 3x3 / stride 1 / pad 1 row path (see Im2col)
  uint32_t nch;             // row path: chunks of 64 columns per row, ceil(W / 64)
  uint32_t nq;              // row path: units per channel, ceil(H * nch / 4)
  uint32_t row_units;       // row path: N * C * nq
  FastDiv div_nq, div_nch;
};

struct UpArgs {  // bilinear upsampling by integer factor s, half-pixel centres
  const float* x;
  float* out;
  uint32_t H, W, Ho, Wo;
  float inv_s;
  uint32_t rows;            // N*C*Ho output rows
  uint32_t rows_per_unit;   // rows handled together when rows are short
  uint32_t units;           // ceil(rows / rows_per_unit)
  uint32_t lanes_per_unit;  // rows_per_unit * Wo4 (vector) or * Wo
  uint32_t vec;             // Wo % 4 == 0 and out 16-byte aligned
  FastDiv div_ho, div_row;  // div_row: by Wo4 (vector) or Wo
  uint32_t s;
  uint32_t places;          // the path by places (see Upsample): N * C * H * (Wo4 or Wo), or 0
  FastDiv div_group;        // by H * (Wo4 or Wo)
  uint32_t row2;            // the scale-2 row path (see Upsample)
  uint32_t nch;             // row path: chunks of 32 input columns per row, ceil(W / 32)
  uint32_t nq;              // row path: units per plane, ceil(bands * nch / 4)
  uint32_t row_units;       // row path: N * C * nq
  FastDiv div_nq, div_nch;
};

struct PoolArgs {  // max pooling with the winner's flat index
  const float* x;
  float* out;
  int32_t* idx;  // null: values only
  uint32_t H, W, Ho, Wo, kh, kw, s, p;
  uint32_t total;  // N*C*Ho*Wo outputs
  uint32_t units;  // ceil(total / Maxpool::kUnit)
  FastDiv div_plane, div_wo;  // by Ho*Wo and by Wo
  uint32_t row3;       // the 3x3 / stride 2 / pad 1 row path (see Maxpool)
  uint32_t nch;        // row path: chunks of 128 input columns per row, ceil(W / 128)
  uint32_t nq;         // row path: units per plane, ceil(Ho * nch / 4)
  uint32_t row_units;  // row path: planes * nq
  FastDiv div_nq, div_nch;
};

struct ShaArgs {  // SHA-256d and BLAKE2b over header || nonce
  const uint32_t* hdr;  // 20 words: the 80-byte header
  uint32_t* out;        // [n][8] words: 32-byte digests
  uint32_t nonce0, n;
};

struct EthArgs {  // Ethash-like folds of table rows
  const uint32_t* hdr;  // 20 words: the 80-byte header
  const uint4* table;   // [rows][8] uint4: rows of 128 bytes
  uint32_t* out;        // [n][8] words
  uint32_t nonce0, n;
  FastMod rows;         // rows.d: the table's row count
};

union DevTask {
  BnArgs bn;
  MixArgs mix;
  HistArgs hist;
  Im2colArgs im2col;
  UpArgs up;
  PoolArgs pool;
  ShaArgs sha;
  EthArgs eth;
};

// Agent-scope helpers for partial results exchanged between workgroups.
__device__ __forceinline__ void store_agent(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t load_agent(uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until every vector-memory operation this wave issued has completed
// (s_waitcnt vmcnt(0); expcnt and lgkmcnt left at their maxima, GFX9 encoding).
// For a store or an atomic, completion means the device-coherent level has
// acknowledged it.
__device__ __forceinline__ void wait_vmem() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // keeps prior accesses above
  __builtin_amdgcn_s_waitcnt(0x0F70);
}

// Arrival on a cross-workgroup counter after publishing results.  Everything a
// wave publishes for other workgroups goes through device-coherent accesses
// (agent-scope atomic stores and RMWs, read back with agent-scope atomic loads
// or RMWs), so no L2 writeback or invalidate is needed: it is enough that those
// accesses have completed before the arrival is counted.  An agent-scope
// release would add an L2 writeback, and an acquire an L2 invalidate, to every
// arrival, which on a multi-XCD part stalls every wave of the die.  The wave
// that sees itself as the last arrival reads the published data only with
// agent-scope atomic loads or RMWs issued after its counter RMW returned.
__device__ __forceinline__ uint32_t arrive_after_coherent_stores(uint32_t* ctr, uint32_t n = 1u) {
  wait_vmem();
  return __hip_atomic_fetch_add(ctr, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ================================================================== bn_stats
// Statistics kernel of the normalisation example (Sec. II-C): per-channel mean
// and variance of x[N][C][H][W].
//
// Work decomposition (fixed by the shape, independent of grid and interval):
//   unit = 1024 consecutive elements of one channel's N*H*W sequence.  One
//          wavefront loads it (16 values per lane; the next unit is already in
//          flight in its own register slot), computes the unit's mean and M2
//          by two passes over registers with fixed-order wave sums, and
//          publishes (mean, M2).
//   Each wavefront of the launch owns a contiguous, balanced range of units;
//   at the end of each channel segment of its range it adds the segment's unit
//   count to the channel's arrival counter.  The wavefront that completes a
//   channel merges its units' (count, mean, M2) in double, in unit order, with
//   Chan's pairwise update, and writes mean[c] and var[c] = M2 / M.
// The unit results and their merge order do not depend on which wavefront
// computed a unit, so every grid and split gives the same bits.
//
// What bounds it besides the reads: the arrivals.  Atomics on one line are served
// one after the other, some 13 ns each, so the counters of few channels lie in
// lines of their own where the scratch has room (own_ctr_shift): [76,16,56,56] 49
// us in one line, 10 in sixteen; [54,32,56,112] 51 and 15; [64,256,56,56] 45 and 44.
// The merge asks for four of a lane's unit results at a time.
//
// Short channels are handed out whole: the wavefront keeps the unit results in its
// lanes, as the merge would read them back, and merges at once, so nothing is
// published, counted, waited for or zeroed (each a trip to memory, one after the
// other).  [128,1024,7,7] alone, at block 256, 512 and 1024: 13, 14 and 12 us with
// every unit published, 9.8, 9.3 and 9.2 whole; [32,512,14,14] (seven units): 9.3
// and 7.6.  Fewer or longer channels than that would leave CUs idle ([1,64,56,112],
// seven units: 7.5 us cut, 12 whole).
struct BnStats {
#ifndef HF_BN_VEC
#define HF_BN_VEC 4
#endif
#ifndef HF_BN_DEPTH
#define HF_BN_DEPTH 2
#endif
  static constexpr uint32_t kVec = HF_BN_VEC;      // float4 per lane per unit
  static constexpr uint32_t kVals = 4 * kVec;      // values per lane per unit
  static constexpr uint32_t kUnit = 64 * kVals;    // 1024 elements by default
  static constexpr uint32_t kDepth = HF_BN_DEPTH;  // units in flight per wavefront
  // Channels short enough to be handed out whole (below): a unit or two always,
  // up to eight units where there is a channel for every CU.
  __host__ __device__ static constexpr bool whole_channels(uint32_t upc, uint32_t C) {
    return upc <= 2u || (upc <= 8u && C >= 256u);
  }
  static constexpr uint32_t lds_words(int) { return 0; }

  struct Regs {
    float v[kVals];  // lane-major: every load instruction is coalesced
  };

  // Loads every lane unconditionally (lanes past the channel's end read the
  // channel's first element, which unit_stats masks out), so the loads of a
  // unit are straight-line code and no value is consumed before its reduction.
  template <bool VEC>
  __device__ static __forceinline__ void load_unit(const BnArgs& a, uint32_t c, uint32_t ubase,
                                                   uint32_t lane, Regs& r) {
    const float* xc = a.x + (size_t)c * a.HW;
    if constexpr (VEC) {
#pragma unroll
      for (uint32_t t = 0; t < kVec; ++t) {
        const uint32_t j = ubase + 4u * (lane + 64u * t);
        const bool ok = j < a.M;
        const uint32_t jj = ok ? j : 0u;
        const uint32_t n = fdiv(jj, a.div_hw);
        const float4 q = *reinterpret_cast<const float4*>(xc + ((size_t)jj + (size_t)n * a.CHWm));
        r.v[4 * t + 0] = q.x;
        r.v[4 * t + 1] = q.y;
        r.v[4 * t + 2] = q.z;
        r.v[4 * t + 3] = q.w;
      }
    } else {
#pragma unroll
      for (uint32_t t = 0; t < kVals; ++t) {
        const uint32_t j = ubase + lane + 64u * t;
        const bool ok = j < a.M;
        const uint32_t jj = ok ? j : 0u;
        const uint32_t n = fdiv(jj, a.div_hw);
        r.v[t] = xc[(size_t)jj + (size_t)n * a.CHWm];
      }
    }
  }

  template <bool VEC>
  __device__ static __forceinline__ bool valid(const BnArgs& a, uint32_t ubase, uint32_t lane,
                                               uint32_t t) {
    const uint32_t j = VEC ? ubase + 4u * (lane + 64u * (t >> 2)) + (t & 3u) : ubase + lane + 64u * t;
    return j < a.M;
  }

  // mean and M2 of one unit held in registers: two passes, fixed-order wave
  // sums.  FULL: the unit has kUnit elements (every unit but a channel's last).
  template <bool VEC, bool FULL>
  __device__ static __forceinline__ void unit_stats(const BnArgs& a, const Regs& r, uint32_t ub,
                                                    uint32_t lane, float& mu, float& m2) {
    const uint32_t cnt = FULL ? kUnit : min(kUnit, a.M - ub);
    float s = 0.f, q = 0.f;
    // lanes past the channel's end hold a copy of another element: masked out
#pragma unroll
    for (uint32_t t = 0; t < kVals; ++t) s += (FULL || valid<VEC>(a, ub, lane, t)) ? r.v[t] : 0.f;
    mu = wave_sum(s) / (float)cnt;
#pragma unroll
    for (uint32_t t = 0; t < kVals; ++t) {
      const float d = (FULL || valid<VEC>(a, ub, lane, t)) ? r.v[t] - mu : 0.f;
      q += d * d;
    }
    m2 = wave_sum(q);
  }

  // Reduces the unit held in `r` (unit k of channel c, global unit index u)
  // and publishes its (mean, M2) with one 8-byte store.
  template <bool VEC, bool FULL>
  __device__ static __forceinline__ void consume(const BnArgs& a, const Regs& r, uint32_t u,
                                                 uint32_t k, uint32_t lane) {
    float mu, m2;
    unit_stats<VEC, FULL>(a, r, k * kUnit, lane, mu, m2);
    if (lane == 0) {
      const uint64_t v = (uint64_t)__builtin_bit_cast(uint32_t, mu) |
                         ((uint64_t)__builtin_bit_cast(uint32_t, m2) << 32);
      __hip_atomic_store(reinterpret_cast<uint64_t*>(a.part) + u, v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // Units [k0, k0 + n) of channel c (global index u0 = c * upc + k0).  kDepth
  // register slots; slot s always holds unit i + s of the current stride, so a
  // unit is requested kDepth - 1 reductions before it is reduced.  The steady
  // loop has no branch: every unit in it is full and every reload exists, which
  // keeps the compiler's count of outstanding loads exact.
  template <bool VEC>
  __device__ static __forceinline__ void segment(const BnArgs& a, uint32_t c, uint32_t k0,
                                                 uint32_t u0, uint32_t n, uint32_t lane) {
    Regs buf[kDepth];
    // unconditional, so that the loop is entered with every slot outstanding in
    // slot order (a segment shorter than kDepth loads its last unit again)
#pragma unroll
    for (uint32_t s = 0; s < kDepth; ++s) load_unit<VEC>(a, c, (k0 + min(s, n - 1u)) * kUnit, lane, buf[s]);
    uint32_t i = 0;
    for (; i + 2u * kDepth <= n; i += kDepth) {
#pragma unroll
      for (uint32_t s = 0; s < kDepth; ++s) {
        consume<VEC, true>(a, buf[s], u0 + i + s, k0 + i + s, lane);
        load_unit<VEC>(a, c, (k0 + i + s + kDepth) * kUnit, lane, buf[s]);
      }
    }
#pragma unroll
    for (uint32_t s = 0; s < kDepth; ++s) {
      if (i + s < n) {
        consume<VEC, false>(a, buf[s], u0 + i + s, k0 + i + s, lane);
        if (i + s + kDepth < n) load_unit<VEC>(a, c, (k0 + i + s + kDepth) * kUnit, lane, buf[s]);
      }
    }
#pragma unroll
    for (uint32_t s = 0; s < kDepth; ++s)
      if (i + kDepth + s < n) consume<VEC, false>(a, buf[s], u0 + i + kDepth + s, k0 + i + kDepth + s, lane);
  }

  // The wavefront's contiguous unit range, one channel segment at a time; at
  // the end of each segment it arrives on the channel's counter, and the last
  // arriver merges the channel.
  template <bool VEC>
  __device__ static __forceinline__ void run_range(const BnArgs& a, uint32_t ubeg, uint32_t uend, uint32_t lane) {
    uint32_t c = fdiv(ubeg, a.div_upc);
    uint32_t k0 = ubeg - c * a.upc;
    for (uint32_t u = ubeg; u < uend; ++c, k0 = 0) {
      const uint32_t n = min(uend - u, a.upc - k0);
      segment<VEC>(a, c, k0, u, n, lane);
      uint32_t old = 0;
      if (lane == 0) old = arrive_after_coherent_stores(a.ctr + ((size_t)c << a.ctr_shift), n);
      old = uniform(old);
      if (old + n == a.upc) finish_channel(a, c, lane);
      u += n;
    }
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar&, uint32_t*) {
    const BnArgs& a = dt.bn;
    const uint32_t lane = lane_id();
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t gw = p.wg * p.nwaves + p.wave;
    if (whole_channels(a.upc, a.C)) {
      // a balanced range of neighbours for each workgroup (their planes share
      // lines)
      const uint32_t q = a.C / p.nwg, r = a.C - q * p.nwg;
      const uint32_t cbeg = p.wg * q + min(p.wg, r);
      const uint32_t cend = cbeg + q + (p.wg < r ? 1u : 0u);
      const uint32_t first = cbeg + p.wave;
      if (a.vec)
        for (uint32_t c = first; c < cend; c += p.nwaves) whole<true>(a, c, lane);
      else
        for (uint32_t c = first; c < cend; c += p.nwaves) whole<false>(a, c, lane);
      return;
    }
    const uint32_t q = a.total / nw, r = a.total - q * nw;
    const uint32_t ubeg = gw * q + min(gw, r);
    const uint32_t uend = ubeg + q + (gw < r ? 1u : 0u);
    if (ubeg >= uend) return;
    if (a.vec)
      run_range<true>(a, ubeg, uend, lane);
    else
      run_range<false>(a, ubeg, uend, lane);
  }

  // Channel c, all of whose units (at most 64) this wavefront reduces: unit k's
  // (mean, M2) stays in lane k, where the merge wants it.
  template <bool VEC>
  __device__ static __forceinline__ void whole(const BnArgs& a, uint32_t c, uint32_t lane) {
    // offsets and counts are the same for every channel: kept from the compiler,
    // which would hold the addresses of 16 loads and every division of the merge
    // in registers across the channels (126 VGPRs)
    asm volatile("" : "+v"(lane));
    float mu_k = 0.f, m2_k = 0.f;
    Regs cur, nxt;
    load_unit<VEC>(a, c, 0u, lane, cur);
#pragma unroll 1
    for (uint32_t k = 0; k < a.upc; ++k) {
      // the last unit again past the end, so that the loop has no branch
      load_unit<VEC>(a, c, min(k + 1u, a.upc - 1u) * kUnit, lane, nxt);
      // one by one, the loads leave before this unit is reduced: mixed with it, their
      // 16 addresses live on through it (bound to 64 VGPRs, 12 of them spilled)
      if constexpr (!VEC) __builtin_amdgcn_sched_barrier(0);
      float mu, m2;
      unit_stats<VEC, false>(a, cur, k * kUnit, lane, mu, m2);
      mu_k = lane == k ? mu : mu_k;
      m2_k = lane == k ? m2 : m2_k;
      cur = nxt;
    }
    double n = 0.0, m = 0.0, m2 = 0.0;
    if (lane < a.upc) chan(n, m, m2, (double)min(kUnit, a.M - lane * kUnit), (double)mu_k, (double)m2_k);
    if (a.upc > 1u) butterfly(lane, n, m, m2);  // one unit: itself
    if (lane == 0) {
      a.mean[c] = (float)m;
      a.var[c] = (float)(m2 / (double)a.M);
    }
  }

  // Chan et al. pairwise update of (n, mean, M2) with (nb, mb, m2b), in double.
  __device__ static __forceinline__ void chan(double& n, double& m, double& m2, double nb, double mb,
                                              double m2b) {
    const double nab = n + nb;
    const double d = mb - m;
    m = m + d * (nb / nab);
    m2 = m2 + m2b + d * d * (n * nb / nab);
    n = nab;
  }

  // The 64 lanes' (n, m, m2) merged, the same in every lane.
  __device__ static __forceinline__ void butterfly(uint32_t lane, double& n, double& m, double& m2) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double nb = __shfl_xor(n, off, kWave);
      const double mb = __shfl_xor(m, off, kWave);
      const double m2b = __shfl_xor(m2, off, kWave);
      if (nb > 0.0) {
        if (n > 0.0) {
          // the lower lane of the pair is always the left operand
          if ((lane & (uint32_t)off) == 0u) {
            chan(n, m, m2, nb, mb, m2b);
          } else {
            double nl = nb, ml = mb, m2l = m2b;
            chan(nl, ml, m2l, n, m, m2);
            n = nl;
            m = ml;
            m2 = m2l;
          }
        } else {
          n = nb;
          m = mb;
          m2 = m2b;
        }
      }
    }
  }

  // Merge the units of channel c: each lane merges units lane, lane+64, ... in
  // order, then the 64 lane results are merged by a fixed butterfly.
  __device__ static __forceinline__ void finish_channel(const BnArgs& a, uint32_t c, uint32_t lane) {
    uint64_t* part = reinterpret_cast<uint64_t*>(a.part) + (size_t)c * a.upc;
    double n = 0.0, m = 0.0, m2 = 0.0;
    constexpr uint32_t kReads = 4;  // of a lane's units, requested together
#pragma unroll 1
    for (uint32_t k0 = lane; k0 < a.upc; k0 += 64u * kReads) {
      uint64_t v[kReads];
#pragma unroll
      for (uint32_t t = 0; t < kReads; ++t)
        v[t] = __hip_atomic_load(part + min(k0 + 64u * t, a.upc - 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (uint32_t t = 0; t < kReads; ++t) {
        const uint32_t k = k0 + 64u * t;
        if (k < a.upc)
          chan(n, m, m2, (double)min(kUnit, a.M - k * kUnit), (double)__builtin_bit_cast(float, (uint32_t)v[t]),
               (double)__builtin_bit_cast(float, (uint32_t)(v[t] >> 32)));
      }
    }
    butterfly(lane, n, m, m2);
    // leave the scratch zero-filled, as every kernel of the library does
    for (uint32_t k = lane; k < a.upc; k += 64u)
      __hip_atomic_store(part + k, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane == 0) {
      a.mean[c] = (float)m;
      a.var[c] = (float)(m2 / (double)a.M);
      store_agent(a.ctr + ((size_t)c << a.ctr_shift), 0u);  // leave the counter zero for the next launch
    }
  }
};

// ================================================================== int_mix
// Integer mixing loop standing in for the compute-bound hash kernels: per element
// R rounds of  x ^= x<<13; x ^= x>>17; x ^= x<<5; x = x*2654435761 + r  (mod 2^32).
//
// A lane's grid-stride walk goes in steps of up to four uint4 vectors (sixteen
// independent chains): four while at least four remain, then one step of the
// remaining one to three.  The vector-memory counter retires in order, so the
// wait for a step's loads also waits for the previous step's stores: each step
// exposes one load and one store latency, and four vectors per step divide the
// number of steps, and of exposed latencies, by four without computing any
// vector twice.
//
// Bound by VALU issue.  On gfx950 some instructions issue at twice the rate of
// the others (measured over independent chains, 8 waves per SIMD: and, or, xor,
// 32-bit add, right shift, v_bitop3 and fp32 fma about 2.5 cycles at the nominal
// 2.4 GHz; left shift, 32-bit multiply, v_alignbit and the three-operand adds
// about 4.4; any of them with a scalar register operand 4.4), but only in
// runs: alternating one fast and one slow instruction runs at the slow rate
// throughout.  So a round goes over all words of a step one operation at a time,
// in an order the compiler may not undo, and takes the slow operations three
// instead of four: the multiply and the addition are one 64-bit multiply-add
// whose high half is not used.  2^24 words of 128 rounds: 424 us word by word,
// 378 in runs of the same operation, 366 with the multiply-add.
struct IntMix {
  static constexpr uint32_t lds_words(int) { return 0; }

  __device__ static __forceinline__ uint32_t round1(uint32_t x, uint32_t r) {
    x ^= x << 13;
    x ^= x >> 17;
    x ^= x << 5;
    return x * 2654435761u + r;
  }

  // R rounds on N words, one operation at a time over all of them.
  template <uint32_t N>
  __device__ static __forceinline__ void rounds(uint32_t (&x)[N], uint32_t R) {
    uint32_t t[N], mul = 2654435761u;
    asm("" : "+v"(mul));  // in a vector register: the round index is the one scalar operand
#pragma unroll
    for (uint32_t k = 0; k < N; ++k) t[k] = x[k] << 13;
    for (uint32_t r = 0; r < R; ++r) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) x[k] ^= t[k];
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) x[k] ^= x[k] >> 17;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) t[k] = x[k] << 5;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) x[k] ^= t[k];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) {
        uint64_t d = (uint64_t)x[k] * mul + r;
        asm("" : "+v"(d));  // both halves: one multiply-add instead of a multiply and an add
        x[k] = (uint32_t)d;
      }
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) t[k] = x[k] << 13;
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // vectors i, i + stride, ..., i + (K-1)*stride, all in range
  template <uint32_t K>
  __device__ static __forceinline__ void step(const uint4* in4, uint4* out4, uint32_t i, uint32_t stride,
                                              uint32_t R) {
    uint32_t x[4 * K];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
      const uint4 v = in4[i + k * stride];
      x[4 * k] = v.x;
      x[4 * k + 1] = v.y;
      x[4 * k + 2] = v.z;
      x[4 * k + 3] = v.w;
    }
    rounds(x, R);
#pragma unroll
    for (uint32_t k = 0; k < K; ++k)
      out4[i + k * stride] = make_uint4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar&, uint32_t*) {
    const MixArgs& a = dt.mix;
    const uint32_t gl = 64u * wave_index(p, ((a.n4 ? a.n4 : a.n) + 63u) / 64u) + lane_id();
    const uint32_t stride = p.nwg * p.nlanes;
    const uint32_t R = (uint32_t)a.rounds;
    const uint4* in4 = reinterpret_cast<const uint4*>(a.in);
    uint4* out4 = reinterpret_cast<uint4*>(a.out);
    if (gl < a.n4) {
      // vectors left for this lane, i = gl, gl + stride, ...
      uint32_t left = (a.n4 - gl + stride - 1u) / stride;
      uint32_t i = gl;
      for (; left >= 4u; left -= 4u, i += 4u * stride) step<4>(in4, out4, i, stride, R);
      if (left == 3u) step<3>(in4, out4, i, stride, R);
      else if (left == 2u) step<2>(in4, out4, i, stride, R);
      else if (left == 1u) step<1>(in4, out4, i, stride, R);
    }
    for (uint32_t i = 4u * a.n4 + gl; i < a.n; i += stride) {
      uint32_t x = a.in[i];
      for (uint32_t r = 0; r < R; ++r) x = round1(x, r);
      a.out[i] = x;
    }
  }
};

// ================================================================== lds_hist
// Histogram kernel of Sec. II-C: clear shared-memory bins, count with shared-
// memory atomics, merge the bins into the global counts.  The interval keeps
// kCopies copies of the 256 bins in LDS, interleaved so that bin b of copy k is
// word b*kCopies + k, and lane l counts into copy l % kCopies: lanes of one
// instruction that see the same (frequent) value hit different words in
// different banks instead of serialising on one address.  The interval's
// barriers separate clearing, counting and merging.  Workgroups add their bins
// into one of `sums` agent-scope accumulators (workgroup w into number w % sums);
// the last workgroup to arrive sums those that were used into the output and
// re-zeroes them.  The additions of all dies to one accumulator line are done
// one after the other, about 17 ns per workgroup, which was what bounded the
// kernel while there was one accumulator (2^26 bytes alone: 46, 29 and 21 us at
// 2048, 1024 and 512 workgroups); sixteen of them divide that serial part by
// sixteen.  A caller's scratch holds one (hf_scratch_bytes is part of the
// interface), the library's own has room for all.  A launch of one workgroup (small instances of a batch) has nothing to merge and writes its bins.
#ifndef HF_HIST_COPIES
#define HF_HIST_COPIES 16
#endif
struct LdsHist {
  static constexpr uint32_t kCopies = HF_HIST_COPIES;
  static constexpr uint32_t kSums = 16;
  static constexpr uint32_t kVecs = 2;
  static constexpr uint32_t lds_words(int) { return 256u * kCopies; }

  __device__ static __forceinline__ void count_byte(uint32_t* mine, uint32_t b) {
    __hip_atomic_fetch_add(mine + b * kCopies, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ static __forceinline__ void count_word(uint32_t* mine, uint32_t w) {
    count_byte(mine, w & 0xFFu);
    count_byte(mine, (w >> 8) & 0xFFu);
    count_byte(mine, (w >> 16) & 0xFFu);
    count_byte(mine, w >> 24);
  }
  __device__ static __forceinline__ void count_vec(uint32_t* mine, const uint4& q) {
    count_word(mine, q.x);
    count_word(mine, q.y);
    count_word(mine, q.z);
    count_word(mine, q.w);
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar& bar, uint32_t* lds) {
    const HistArgs& a = dt.hist;
    const uint32_t lane = lane_id();
    for (uint32_t i = p.lane; i < 256u * kCopies; i += p.nlanes) lds[i] = 0u;
    bar.sync();

    uint32_t* mine = lds + (lane % kCopies);
    const uint32_t gl = p.wg * p.nlanes + p.lane;
    const uint32_t stride = p.nwg * p.nlanes;
    const uint4* v16 = reinterpret_cast<const uint4*>(a.in + a.head);
    // kVecs vectors per step, and the next step's requested before this step's
    // atomics, so up to 2 kVecs 16-byte loads per lane are in flight: inside a
    // fused kernel the interval may have only a few wavefronts per CU, and
    // their loads alone must keep the input streaming (four vectors: 19.5 us
    // alone instead of 18.4 on 2^26 bytes, the fused pairs unchanged).  The loop
    // has no stores, so each wait covers only the loads it needs.
    if (gl < a.n16) {
      const uint32_t last = a.n16 - 1u;
      uint4 q[kVecs], nx[kVecs];
#pragma unroll
      for (uint32_t k = 0; k < kVecs; ++k) q[k] = v16[min(gl + k * stride, last)];
      uint32_t i = gl;
      for (; i + (kVecs - 1u) * stride < a.n16; i += kVecs * stride) {
#pragma unroll
        for (uint32_t k = 0; k < kVecs; ++k) nx[k] = v16[min(i + (kVecs + k) * stride, last)];
#pragma unroll
        for (uint32_t k = 0; k < kVecs; ++k) {
          count_vec(mine, q[k]);
          q[k] = nx[k];
        }
      }
#pragma unroll
      for (uint32_t k = 0; k + 1u < kVecs; ++k)  // what a whole step does not cover
        if (i + k * stride < a.n16) count_vec(mine, q[k]);
    }
    if (gl < a.head) count_byte(mine, a.in[gl]);
    for (uint32_t i = a.tail_start + gl; i < a.n; i += stride) count_byte(mine, a.in[i]);
    bar.sync();

    const bool many = a.sums == kSums;
    const uint32_t mine_sum = many ? p.wg % kSums : 0u;
    uint32_t* acc = a.acc + 256u * mine_sum;
    for (uint32_t b = p.lane; b < 256u; b += p.nlanes) {
      uint32_t s = 0;
#pragma unroll
      for (uint32_t k = 0; k < kCopies; ++k) s += lds[b * kCopies + k];
      if (p.nwg == 1u) a.out[b] = s;
      else if (s) __hip_atomic_fetch_add(acc + b, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (p.nwg == 1u) return;
    wait_vmem();  // this wave's merge atomics have completed ...
    bar.sync();   // ... before wave 0 of the interval counts the workgroup in

    if (p.wave == 0 && lane == 0) {
      uint32_t last = 0;
      if (many && p.nwg > 4u * kSums) {
        // the last of each accumulator's workgroups counts the accumulator in
        uint32_t* sub = a.ctr + 32u * (1u + mine_sum);
        const uint32_t of = (p.nwg - mine_sum + kSums - 1u) / kSums;
        if (arrive_after_coherent_stores(sub) == of - 1u) {
          store_agent(sub, 0u);
          last = arrive_after_coherent_stores(a.ctr) == kSums - 1u;
        }
      } else {
        last = arrive_after_coherent_stores(a.ctr) == p.nwg - 1u;
      }
      lds[0] = last;
    }
    bar.sync();
    if (uniform(lds[0]) == 0u) return;
    for (uint32_t b = p.lane; b < 256u; b += p.nlanes) {
      uint32_t* q = a.acc + b;
      uint32_t s = 0;
      if (many) {
        // in fours, up to the last that a workgroup added to (the others are zero, a
        // condition each would be 16 lane masks and addresses in scalar registers);
        // all are requested before the first is used
        uint32_t v[kSums];
#pragma unroll
        for (uint32_t k = 0; k < kSums; ++k) {
          if (k % 4u == 0u && k >= p.nwg) break;
          v[k] = load_agent(q + 256u * k);
        }
#pragma unroll
        for (uint32_t k = 0; k < kSums; ++k) {
          if (k % 4u == 0u && k >= p.nwg) break;
          s += v[k];
          store_agent(q + 256u * k, 0u);
        }
      } else {
        s = load_agent(q);
        store_agent(q, 0u);
      }
      a.out[b] = s;
    }
    if (p.lane == 0) store_agent(a.ctr, 0u);
  }
};

// ================================================================== im2col
// Im2Col (Sec. IV-A): out[n][(c*kh + i)*kw + j][oh*Wo + ow] = x[n][c][oh*s-p+i][ow*s-p+j],
// zero outside the image.
//
// General path: a place is (n, c, kernel row i, output row, four outputs or one);
// the places of a wavefront are 64 consecutive ones, so a plane of any size fills
// its lanes.  A lane reads the input row's span that its outputs need for kJ
// kernel columns at once (3s + kJ elements for 4 kJ outputs) and writes the kJ
// planes.  The span is read whole, in unaligned vector loads, whatever of it lies
// in the padding or in a neighbouring row, and what lies outside the row is
// zeroed afterwards; only a wavefront of which some span would leave the tensor
// reads element by element.  Bound by HBM writes: 7x7 / stride 2 / pad 3 over
// [32,3,224,224], alone: 112, 136 and 181 us at block 256, 512 and 1024 with a
// wavefront per output plane (4704 planes for 8192 wavefronts) and one load per
// output, 44, 46 and 48 us now (236 MB written, 5.9 TB/s).
//
// Row path (3x3 kernel, stride 1, pad 1, W % 4 == 0, 16-byte aligned input and
// output): with stride 1, output plane (i, j) of a channel is the channel
// shifted by i - 1 rows and j - 1 columns with zero fill, so one output row of
// all nine planes is made from three input rows.  Each row is cut into chunks
// of 64 columns; a unit is four consecutive chunks of one channel (four rows
// when W <= 64), one chunk per 16-lane DPP row of the wavefront.  Lane 16q + c
// loads columns 4c..4c+3 of input rows oh-1, oh, oh+1 (one aligned float4 each)
// and writes columns 4c..4c+3 of row oh of all nine planes: a column shift
// takes the neighbouring lane's edge element with a DPP row shift, and the
// first and last lane of a chunk take the element beyond it with one extra
// dword load per row (zero at the image's edge).  Every input element is thus
// loaded by one unit only (plus the rows shared with the neighbouring quads,
// which the same wavefront reads next), instead of once per plane.  All
// accesses go through buffer resources over one plane: rows and columns
// outside the image load zero, which is exactly the zero padding, and lanes
// past the plane's end store nothing, so the loop has no branch around a
// memory access.  Each store instruction writes four chunks of one plane.
// kStep units per step (fewer when a wavefront has fewer): their loads are
// issued together, so the wait for them comes once per kStep units.  Wavefronts
// take steps in turn, so that all of them work on one window of the tensors;
// a contiguous range of units for each keeps 8192 places of DRAM open (with the
// histogram of 2^26 bytes, inputs from HBM: 116 us in ranges, 109 in turn).
struct Im2col {
  static constexpr uint32_t lds_words(int) { return 0; }
  static constexpr uint32_t kStep = 3;

  __device__ static __forceinline__ void run_rows(const Im2colArgs& a, const Part& p, uint32_t lane) {
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t gw = p.wg * p.nwaves + p.wave;
    const uint32_t per = (a.row_units + nw - 1u) / nw;  // units of the busiest wavefront
    const uint32_t st = min(kStep, per);                // taken together
    const uint32_t W = a.W, H = a.H, HW = H * W, pbytes = 4u * HW;
    const uint32_t qrow = lane >> 4, c4 = lane & 15u;
    // The channel and output position of unit u in this lane (shared by both
    // phases; the store phase recomputes it rather than keep registers live).
    auto where = [&](uint32_t u, uint32_t& nc, uint32_t& oh, uint32_t& col) {
      nc = fdiv(u, a.div_nq);
      const uint32_t cid = 4u * (u - nc * a.nq) + qrow;  // chunk of this DPP row
      oh = fdiv(cid, a.div_nch);
      col = 64u * (cid - oh * a.nch) + 4u * c4;
    };
    for (uint32_t u0 = gw * st; u0 < a.row_units; u0 += nw * st) {
      const uint32_t uend = min(u0 + st, a.row_units);
      float4 x[kStep][3];
      float edge[kStep][3];
#pragma unroll
      for (uint32_t k = 0; k < kStep; ++k) {
        uint32_t nc, oh, col;
        where(min(u0 + k, uend - 1u), nc, oh, col);  // a unit past the step repeats the last one
        const __amdgpu_buffer_rsrc_t src = buffer_rsrc(a.x + (size_t)nc * HW, pbytes);
        uint32_t ec = kOutOfRange;  // the column left or right of the lane's four, if another lane's
        if (c4 == 0u && col > 0u) ec = col - 1u;
        if (c4 == 15u && col + 4u < W) ec = col + 4u;
#pragma unroll
        for (uint32_t i = 0; i < 3u; ++i) {
          const uint32_t ih = oh + i - 1u;  // wraps past H above the image
          const bool rowok = oh < H && col < W && ih < H;
          x[k][i] = buffer_load4(src, rowok ? 4u * (ih * W + col) : kOutOfRange);
          edge[k][i] = buffer_load1(src, rowok && ec != kOutOfRange ? 4u * (ih * W + ec) : kOutOfRange);
        }
      }
#pragma unroll
      for (uint32_t k = 0; k < kStep; ++k) {
        uint32_t nc, oh, col;
        where(min(u0 + k, uend - 1u), nc, oh, col);
        const uint32_t at = (oh < H && col < W && u0 + k < uend) ? 4u * (oh * W + col) : kOutOfRange;
#pragma unroll
        for (uint32_t i = 0; i < 3u; ++i) {
          const float4 v = x[k][i];
          // every lane takes part in the shifts (row_shr:1 / row_shl:1)
          const float sl = dpp_f32<0x111>(v.w), sr = dpp_f32<0x101>(v.x);
          const float lft = c4 == 0u ? edge[k][i] : sl;
          const float rgt = c4 == 15u ? edge[k][i] : sr;
          const float* base = a.out + ((size_t)nc * 9u + 3u * i) * HW;  // plane (i, 0) of channel nc
          buffer_store4_nt(buffer_rsrc(base, pbytes), at, lft, v.x, v.y, v.z);
          buffer_store4_nt(buffer_rsrc(base + HW, pbytes), at, v.x, v.y, v.z, v.w);
          buffer_store4_nt(buffer_rsrc(base + 2u * (size_t)HW, pbytes), at, v.y, v.z, v.w, rgt);
        }
      }
    }
  }

  // V outputs per place, S the stride (0: any, read from the arguments), kernel
  // columns in blocks of J.
  template <int V, int S, int J>
  __device__ static __forceinline__ void run_places(const Im2colArgs& a, const Part& p, uint32_t lane) {
    const uint32_t nl = 64u * p.nwg * p.nwaves;
    const uint32_t HW = a.H * a.W, plane = a.Ho * a.Wo;
    const int s = S > 0 ? S : (int)a.s;
    // elements of a lane: E runs of R contiguous ones, s apart
    constexpr int R = S > 0 ? (V - 1) * S + J : J, E = S > 0 ? 1 : V;
    const uint32_t span = (uint32_t)((E - 1) * s + R);
    for (uint32_t t0 = 64u * (p.wg * p.nwaves + p.wave); t0 < a.items; t0 += nl) {
      const uint32_t t = min(t0 + lane, a.items - 1u);  // lanes past the end redo the last place
      const uint32_t g = fdiv(t, a.div_group), pos = t - g * a.div_group.d;
      const uint32_t nc = fdiv(g, a.div_kh), i = g - nc * a.div_kh.d;
      const uint32_t oh = fdiv(pos, a.div_row), col = pos - oh * a.div_row.d;
      const int ih = (int)(oh * a.s + i) - (int)a.p;
      const bool rowok = (uint32_t)ih < a.H;
      const uint32_t row = nc * HW + (rowok ? (uint32_t)ih : 0u) * a.W;
      float* dst = a.out + ((size_t)nc * a.KK + i * a.kw) * plane + oh * a.Wo + (uint32_t)V * col;
      for (uint32_t j0 = 0; j0 < a.kw; j0 += (uint32_t)J) {
        const int iw0 = (int)((uint32_t)V * col * a.s + j0) - (int)a.p;  // column of element 0
        const uint32_t at = row + (uint32_t)iw0;                         // wraps above the tensor's start
        float v[E][R];
        if (__builtin_amdgcn_ballot_w64(at > a.elems || at + span > a.elems) == 0ull) {
          const float* src = a.x + at;
#pragma unroll
          for (int e = 0; e < E; ++e) load_run<R>(src + e * s, v[e]);
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
#pragma unroll
            for (int r = 0; r < R; ++r) v[e][r] = a.x[row + min((uint32_t)max(iw0 + e * s + r, 0), a.W - 1u)];
        }
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
          for (int r = 0; r < R; ++r) v[e][r] = rowok && (uint32_t)(iw0 + e * s + r) < a.W ? v[e][r] : 0.f;
        if (t0 + lane < a.items) {
#pragma unroll
          for (int j = 0; j < J; ++j) {
            if (j0 + (uint32_t)j < a.kw) {
              float* q = dst + (size_t)(j0 + (uint32_t)j) * plane;
              if constexpr (V == 1) __builtin_nontemporal_store(v[0][j], q);
              else if constexpr (S > 0) store_nt4(q, v[0][j], v[0][S + j], v[0][2 * S + j], v[0][3 * S + j]);
              else store_nt4(q, v[0][j], v[1][j], v[2][j], v[3][j]);
            }
          }
        }
      }
    }
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar&, uint32_t*) {
    const Im2colArgs& a = dt.im2col;
    const uint32_t lane = lane_id();
    // the block of kernel columns: about the kernel's width, so that little of
    // the span is read in vain
    if (a.row3) run_rows(a, p, lane);
    else if (!a.vec) a.kw > 1u ? run_places<1, 0, 4>(a, p, lane) : run_places<1, 0, 1>(a, p, lane);
    else if (a.s == 1u) a.kw > 4u ? run_places<4, 1, 8>(a, p, lane)
                        : a.kw > 1u ? run_places<4, 1, 4>(a, p, lane) : run_places<4, 1, 1>(a, p, lane);
    else if (a.s == 2u) a.kw > 4u ? run_places<4, 2, 8>(a, p, lane) : run_places<4, 2, 4>(a, p, lane);
    else run_places<4, 0, 4>(a, p, lane);
  }
};

// ================================================================== upsample
// Bilinear upsampling (Sec. IV-A) by an integer factor s with half-pixel
// centres: t = max(0, (o + 0.5)/s - 0.5), i0 = floor(t), i1 = min(i0+1, L-1),
// l = t - i0; lerp along x on rows y0 and y1, then along y, as a + l*(b - a).
// Units are output rows (several short rows per unit), written front to back.
// For s = 2 the four outputs 4c..4c+3 of a float4 read the four consecutive
// inputs 2c-1..2c+2 (clamped) with weights 0.75, 0.25, 0.75, 0.25, which are
// exactly the values the general formula produces, so both paths give the same
// bits; the fast path just skips the per-output coordinate arithmetic.
struct Upsample {
  static constexpr uint32_t lds_words(int) { return 0; }

  __device__ static __forceinline__ void coord(uint32_t o, float inv_s, uint32_t L, uint32_t& i0,
                                               uint32_t& i1, float& l) {
    const float t = fmaxf(((float)o + 0.5f) * inv_s - 0.5f, 0.f);
    uint32_t a = (uint32_t)t;
    a = min(a, L - 1u);
    i0 = a;
    i1 = min(a + 1u, L - 1u);
    l = t - (float)a;
  }

  __device__ static __forceinline__ float lerp(float a, float b, float l) { return a + l * (b - a); }

  // Row path (scale 2, W even, 8-byte aligned input, 16-byte aligned output).
  // A band of kBand input rows makes 2 kBand output rows and needs one input row
  // more on either side, so a lane reads each row once and keeps its four
  // horizontal interpolations for every output row that uses them.  Bands are
  // cut into chunks that read 32 input columns and write 64 output columns; a
  // unit is four consecutive chunks of one plane (four bands when W <= 32), one
  // chunk per 16-lane DPP row.  Lane 16q + c reads input columns 2c, 2c+1 of its
  // rows (one float2 each) and writes output columns 4c..4c+3 (one float4), so
  // every store instruction covers whole contiguous lines.  Column 2c-1 comes
  // from the lane before and column 2c+2 from the lane after by DPP row shifts,
  // from one extra dword load at a chunk's first and last lane, and from the
  // lane itself at the image's edges (the coordinate clamp).  The four outputs
  // are the general scale-2 path's expressions of the same inputs, so both paths
  // give the same bits.  Buffer accesses keep the loop free of branches around
  // memory instructions.
  //
  // Bound by HBM (one byte read for four written).  [32,64,128,128] with its
  // input in HBM, alone: 190 us with a unit per output row (every input row read
  // by four units) and a contiguous range of units per wavefront; 175 us with
  // the wavefronts taking units in turn, so that all of them work on one window
  // of the tensors instead of keeping 8192 places of DRAM open; 140 us in bands
  // of two input rows, 128 us in bands of four; 111 us with a workgroup for
  // every unit (default_wgs), 6.0 TB/s.
  static constexpr uint32_t kBand = 4;

  struct Rows {
    float2 x[kBand + 2];
    float e[kBand + 2];
  };

  __device__ static __forceinline__ void run_rows(const UpArgs& a, const Part& p, uint32_t lane) {
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t W = a.W, HW = a.H * a.W, OHW = a.Ho * a.Wo;
    const uint32_t qrow = lane >> 4, c4 = lane & 15u;
    auto where = [&](uint32_t u, uint32_t& plane, uint32_t& y0, uint32_t& col) {
      plane = fdiv(u, a.div_nq);
      const uint32_t cid = 4u * (u - plane * a.nq) + qrow;  // chunk of this DPP row
      const uint32_t band = fdiv(cid, a.div_nch);
      y0 = kBand * band;                                // first input row of the band
      col = 32u * (cid - band * a.nch) + 2u * c4;       // first input column of this lane
    };
    auto load = [&](uint32_t u, Rows& r) {
      uint32_t plane, y0, col;
      where(u, plane, y0, col);
      const bool ok = y0 < a.H && col < W;
      const __amdgpu_buffer_rsrc_t src = buffer_rsrc(a.x + (size_t)plane * HW, 4u * HW);
      uint32_t eo = kOutOfRange;  // the column left or right of the lane's two, if another lane's
      if (c4 == 0u && col > 0u) eo = col - 1u;
      if (c4 == 15u && col + 2u < W) eo = col + 2u;
#pragma unroll
      for (uint32_t i = 0; i < kBand + 2u; ++i) {
        const uint32_t y = i == 0u ? (y0 > 0u ? y0 - 1u : 0u) : min(y0 + i - 1u, a.H - 1u);
        r.x[i] = buffer_load2(src, ok ? 4u * (y * W + col) : kOutOfRange);
        r.e[i] = buffer_load1(src, ok && eo != kOutOfRange ? 4u * (y * W + eo) : kOutOfRange);
      }
    };
    auto store = [&](uint32_t u, const Rows& r) {
      uint32_t plane, y0, col;
      where(u, plane, y0, col);
      const bool first = col == 0u, last = col + 2u >= W, top = y0 == 0u;
      const __amdgpu_buffer_rsrc_t dst = buffer_rsrc(a.out + (size_t)plane * OHW, 4u * OHW);
      // the four columns of input row i; every lane takes part in the shifts
      // (row_shr:1 / row_shl:1)
      auto row = [&](uint32_t i, float (&h)[4]) {
        const float sl = dpp_f32<0x111>(r.x[i].y), sr = dpp_f32<0x101>(r.x[i].x);
        const float p0 = first ? r.x[i].x : (c4 == 0u ? r.e[i] : sl), p1 = r.x[i].x, p2 = r.x[i].y;
        const float p3 = last ? r.x[i].y : (c4 == 15u ? r.e[i] : sr);
        h[0] = lerp(p0, p1, 0.75f);
        h[1] = lerp(p1, p2, 0.25f);
        h[2] = lerp(p1, p2, 0.75f);
        h[3] = lerp(p2, p3, 0.25f);
      };
      auto out = [&](uint32_t o, const float (&t)[4], const float (&b)[4], float l) {
        const uint32_t oy = 2u * y0 + o;
        buffer_store4_nt(dst, oy < a.Ho && col < W ? 4u * (oy * a.Wo + 2u * col) : kOutOfRange, lerp(t[0], b[0], l),
                         lerp(t[1], b[1], l), lerp(t[2], b[2], l), lerp(t[3], b[3], l));
      };
      // output row 2y lies between input rows y-1 and y (the image's first row is
      // input row 0 with weight 0 on row 1), output row 2y+1 between y and y+1; of
      // the rows only two are held at a time
      float h[3][4];
      row(0u, h[0]);
      row(1u, h[1]);
#pragma unroll
      for (uint32_t i = 1; i < kBand + 1u; ++i) {
        float(&t)[4] = h[i % 3u], (&b)[4] = h[(i + 1u) % 3u];
        row(i + 1u, b);
        if (i == 1u) {
          float z[4], w[4];
#pragma unroll
          for (uint32_t c = 0; c < 4u; ++c) {
            z[c] = top ? t[c] : h[0][c];
            w[c] = top ? b[c] : t[c];
          }
          out(0u, z, w, top ? 0.f : 0.75f);
        }
        out(2u * i - 1u, t, b, 0.25f);
        if (i < kBand) out(2u * i, t, b, 0.75f);
        // as written: the scheduler, left alone, computes every row before the first
        // store and takes 70 VGPRs for 64, a wavefront per SIMD less
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // the next unit is requested before this one is stored: the vector-memory
    // counter retires in order, so the wait for loads issued after the stores
    // would be a wait for the stores as well
    uint32_t u = p.wg * p.nwaves + p.wave;
    if (u >= a.row_units) return;
    Rows cur, nxt;
    load(u, cur);
    for (; u + nw < a.row_units; u += nw) {
      load(u + nw, nxt);
      store(u, cur);
      cur = nxt;
    }
    store(u, cur);
  }

  // Path by places (any other scale; not float4 stores below scale 3, nor short rows
  // that are no whole lines): a place is
  // a plane, a group of the s output rows s*g .. s*g+s-1, and four adjacent output
  // columns (V = 4) or one.  Its rows lie between three consecutive input rows,
  // its columns between NC consecutive input columns: V = 1 two, V = 4 three from
  // scale 4 on and four at scale 3, where rounding can put the first column
  // left and the last right of an input position.  A lane reads 3 NC inputs for
  // 4 s outputs, interpolates the three rows horizontally once, and combines them
  // for every output row.  Every output keeps its own coordinates (coord) and
  // expressions, so the bits are those of the pointwise path.  x4 over
  // [16,32,65,65], alone: 58 us pointwise (16 reads and eight coordinates per four
  // outputs, and 65 float4 of a row taken in two steps of 64 lanes), 37 us
  // now (147 MB; rows of 1040 bytes leave partial lines); x3 over [16,32,64,64]: 44
  // and 14 us (87 MB, 6.1 TB/s).
  template <int V, int NC>
  __device__ static __forceinline__ void run_places(const UpArgs& a, const Part& p, uint32_t lane) {
    const uint32_t nl = 64u * p.nwg * p.nwaves;
    const uint32_t HW = a.H * a.W, OHW = a.Ho * a.Wo;
    for (uint32_t t0 = 64u * (p.wg * p.nwaves + p.wave); t0 < a.places; t0 += nl) {
      const uint32_t t = min(t0 + lane, a.places - 1u);  // lanes past the end redo the last place
      const uint32_t plane = fdiv(t, a.div_group), pos = t - plane * a.div_group.d;
      const uint32_t g = fdiv(pos, a.div_row), col = (uint32_t)V * (pos - g * a.div_row.d);
      uint32_t x0[V], x1, yb, y1;
      float lx[V], ly;
#pragma unroll
      for (int c = 0; c < V; ++c) coord(col + (uint32_t)c, a.inv_s, a.W, x0[c], x1, lx[c]);
      coord(a.s * g, a.inv_s, a.H, yb, y1, ly);
      const float* img = a.x + (size_t)plane * HW;
      float in[3][NC];
#pragma unroll
      for (uint32_t k = 0; k < 3u; ++k)
#pragma unroll
        for (uint32_t c = 0; c < (uint32_t)NC; ++c)
          in[k][c] = img[min(yb + k, a.H - 1u) * a.W + min(x0[0] + c, a.W - 1u)];
      float h[3][V];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int c = 0; c < V; ++c) {
          const uint32_t d = x0[c] - x0[0];  // 0 .. NC - 2
          float l = in[k][0], r = in[k][1];
#pragma unroll
          for (uint32_t e = 1; e + 1u < (uint32_t)NC; ++e) {
            l = d == e ? in[k][e] : l;
            r = d == e ? in[k][e + 1] : r;
          }
          h[k][c] = lerp(l, r, lx[c]);
        }
      float* dst = a.out + (size_t)plane * OHW + a.s * g * a.Wo + col;
      const bool live = t0 + lane < a.places;
      for (uint32_t r = 0; r < a.s; ++r) {
        uint32_t y0;
        coord(a.s * g + r, a.inv_s, a.H, y0, y1, ly);
        const bool up = y0 != yb;  // then y0 == yb + 1
        float v[V];
#pragma unroll
        for (int c = 0; c < V; ++c) v[c] = lerp(up ? h[1][c] : h[0][c], up ? h[2][c] : h[1][c], ly);
        if (live) {
          if constexpr (V == 4) store_nt4(dst + r * a.Wo, v[0], v[1], v[2], v[3]);
          else __builtin_nontemporal_store(v[0], dst + r * a.Wo);
        }
      }
    }
  }

  __device__ static __forceinline__ float sample(const float* r0, const float* r1, float ly, uint32_t W,
                                                 uint32_t ox, float inv_s) {
    uint32_t x0, x1;
    float lx;
    coord(ox, inv_s, W, x0, x1, lx);
    const float top = lerp(r0[x0], r0[x1], lx);
    const float bot = lerp(r1[x0], r1[x1], lx);
    return lerp(top, bot, ly);
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar&, uint32_t*) {
    const UpArgs& a = dt.up;
    const uint32_t lane = lane_id();
    if (a.row2) {
      run_rows(a, p, lane);
      return;
    }
    if (a.places) {
      if (!a.vec) run_places<1, 2>(a, p, lane);
      else if (a.s == 3u) run_places<4, 4>(a, p, lane);
      else run_places<4, 3>(a, p, lane);
      return;
    }
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t HW = a.H * a.W;
    const bool x2 = a.vec && a.Wo == 2u * a.W;  // scale 2 with float4 stores
    for (uint32_t u = p.wg * p.nwaves + p.wave; u < a.units; u += nw) {
      const uint32_t row0 = u * a.rows_per_unit;
      for (uint32_t t = lane; t < a.lanes_per_unit; t += 64u) {
        const uint32_t rr = fdiv(t, a.div_row);
        const uint32_t col = t - rr * a.div_row.d;
        const uint32_t row = row0 + rr;
        if (row >= a.rows) continue;
        const uint32_t plane = fdiv(row, a.div_ho);
        const uint32_t oy = row - plane * a.Ho;
        uint32_t y0, y1;
        float ly;
        coord(oy, a.inv_s, a.H, y0, y1, ly);
        const float* img = a.x + plane * HW;
        const float* r0 = img + y0 * a.W;
        const float* r1 = img + y1 * a.W;
        float* dst = a.out + row * a.Wo;
        if (x2) {
          const uint32_t xm = col > 0u ? 2u * col - 1u : 0u;
          const uint32_t xp = min(2u * col + 2u, a.W - 1u);
          const float p0 = r0[xm], p1 = r0[2u * col], p2 = r0[2u * col + 1u], p3 = r0[xp];
          const float q0 = r1[xm], q1 = r1[2u * col], q2 = r1[2u * col + 1u], q3 = r1[xp];
          store_nt4(dst + 4u * col, lerp(lerp(p0, p1, 0.75f), lerp(q0, q1, 0.75f), ly),
                    lerp(lerp(p1, p2, 0.25f), lerp(q1, q2, 0.25f), ly),
                    lerp(lerp(p1, p2, 0.75f), lerp(q1, q2, 0.75f), ly),
                    lerp(lerp(p2, p3, 0.25f), lerp(q2, q3, 0.25f), ly));
        } else if (a.vec) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = sample(r0, r1, ly, a.W, 4u * col + e, a.inv_s);
          store_nt4(dst + 4u * col, v[0], v[1], v[2], v[3]);
        } else {
          __builtin_nontemporal_store(sample(r0, r1, ly, a.W, col, a.inv_s), dst + col);
        }
      }
    }
  }
};

// =================================================================== maxpool
// 2-D max pooling (Sec. IV-A "Maxpool").  A unit is kUnit consecutive outputs
// of the flattened [N][C][Ho][Wo] output, kPer per lane (lane l takes outputs
// l, l + 64, ...).  Each wavefront owns a contiguous, balanced range of units,
// so the input rows shared by vertically adjacent windows are re-read from the
// caches of the same CU.
//
// Window coordinates are clamped into the image instead of being skipped: with
// pad < kh, kw a clamped row or column is always inside the window, and it is
// met in the scan before (low side) or after (high side) the real copy of the
// same element, never between two other elements, so under the scan rule (a
// later element wins only if greater or NaN) the winner and its index are
// exactly those of the unclamped scan.  All loads are therefore unconditional.
//
// Row path (3x3 window, stride 2, pad 1, W % 8 == 0, 16-byte aligned
// buffers): each output row is cut into chunks that read 128 input columns
// and write 64 outputs; a unit is four consecutive chunks of one plane (four
// output rows when W <= 128), one per 16-lane DPP row of the wavefront.  Lane
// 16q + c computes outputs 4c..4c+3 of its chunk, whose windows span input
// columns 8c-1 .. 8c+7 (chunk-relative) of three input rows: columns 8c..8c+7
// are two aligned float4 per row, and column 8c-1 is the left neighbour lane's
// last element, taken with a DPP row shift, or, at a chunk's first lane, one
// extra dword load (at the image's first column the column clamps to 0, as in
// the general path).  Rows clamp the same way.  Each window is scanned in the
// general path's order, and values and indices are stored as float4 / int4
// through buffer resources (lanes past the plane's end store nothing), four
// chunks per store instruction.  Wavefronts take units in turn, as in upsample
// ([64,64,112,112] with its input in HBM, alone: 63 us in contiguous ranges, 60
// in turn, 56 with a workgroup for every unit).
struct Maxpool {
  static constexpr int kSoloWaves = 8;  // 45 VGPRs, but 106 SGPRs would allow only 7
  static constexpr uint32_t kPer = 2;
  static constexpr uint32_t kUnit = 64 * kPer;
  static constexpr uint32_t lds_words(int) { return 0; }

  __device__ static __forceinline__ void take(float v, int32_t e, bool first, float& best, int32_t& at) {
    if (first || v > best || __builtin_isnan(v)) {
      best = v;
      at = e;
    }
  }

  __device__ static __forceinline__ void run_rows(const PoolArgs& a, const Part& p, uint32_t lane) {
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t gw = p.wg * p.nwaves + p.wave;
    const uint32_t W = a.W, HW = a.H * a.W, OHW = a.Ho * a.Wo;
    const uint32_t qrow = lane >> 4, c4 = lane & 15u;
    for (uint32_t u = gw; u < a.row_units; u += nw) {
      const uint32_t plane = fdiv(u, a.div_nq);
      const uint32_t cid = 4u * (u - plane * a.nq) + qrow;  // chunk of this DPP row
      const uint32_t oh = fdiv(cid, a.div_nch);
      const uint32_t col = 128u * (cid - oh * a.nch) + 8u * c4;  // first input column of this lane
      const bool ok = oh < a.Ho && col < W;
      const uint32_t ohc = min(oh, a.Ho - 1u);
      const __amdgpu_buffer_rsrc_t src = buffer_rsrc(a.x + (size_t)plane * HW, 4u * HW);
      float4 A[3], B[3];
      float E[3];
#pragma unroll
      for (uint32_t i = 0; i < 3; ++i) {
        const uint32_t h = (uint32_t)clampi((int32_t)(2u * ohc + i) - 1, (int32_t)a.H - 1);
        A[i] = buffer_load4(src, ok ? 4u * (h * W + col) : kOutOfRange);
        B[i] = buffer_load4(src, ok ? 4u * (h * W + col + 4u) : kOutOfRange);
        // column col - 1 of the first lane of a chunk that is not the image's first
        E[i] = buffer_load1(src, ok && c4 == 0u && col > 0u ? 4u * (h * W + col - 1u) : kOutOfRange);
      }
      float best[4];
      int32_t at[4];
#pragma unroll
      for (uint32_t i = 0; i < 3; ++i) {
        const int32_t h = clampi((int32_t)(2u * ohc + i) - 1, (int32_t)a.H - 1);
        const float lft = dpp_f32<0x111>(B[i].w);  // column col - 1 from the lane before
        const int32_t e0 = h * (int32_t)W + (int32_t)col;
        // at the image's first column the window's clamped column is column 0
        const float L = col == 0u ? A[i].x : (c4 == 0u ? E[i] : lft);
        const int32_t eL = col == 0u ? e0 : e0 - 1;
        const bool f = i == 0;
        take(L, eL, f, best[0], at[0]);
        take(A[i].x, e0, false, best[0], at[0]);
        take(A[i].y, e0 + 1, false, best[0], at[0]);
        take(A[i].y, e0 + 1, f, best[1], at[1]);
        take(A[i].z, e0 + 2, false, best[1], at[1]);
        take(A[i].w, e0 + 3, false, best[1], at[1]);
        take(A[i].w, e0 + 3, f, best[2], at[2]);
        take(B[i].x, e0 + 4, false, best[2], at[2]);
        take(B[i].y, e0 + 5, false, best[2], at[2]);
        take(B[i].y, e0 + 5, f, best[3], at[3]);
        take(B[i].z, e0 + 6, false, best[3], at[3]);
        take(B[i].w, e0 + 7, false, best[3], at[3]);
      }
      const uint32_t o = ok ? 4u * (oh * a.Wo + col / 2u) : kOutOfRange;
      buffer_store4_nt(buffer_rsrc(a.out + (size_t)plane * OHW, 4u * OHW), o, best[0], best[1], best[2], best[3]);
      if (a.idx)
        buffer_store4_nt(buffer_rsrc(a.idx + (size_t)plane * OHW, 4u * OHW), o, __builtin_bit_cast(float, at[0]),
                         __builtin_bit_cast(float, at[1]), __builtin_bit_cast(float, at[2]),
                         __builtin_bit_cast(float, at[3]));
    }
  }

  __device__ static __forceinline__ int32_t clampi(int32_t v, int32_t hi) { return min(max(v, 0), hi); }

  // PAD false: no padding, so every window lies in the image and a row of it is
  // one unaligned vector load instead of a clamp and a load per element
  // (3x3 / stride 2 over [32,96,111,111], alone: 72 -> 41 us; 2x2: 48 -> 40).
  template <int KH, int KW, bool PAD>
  __device__ static __forceinline__ void window(const PoolArgs& a, const float* img, int32_t h0, int32_t w0,
                                                uint32_t kh, uint32_t kw, float& best, int32_t& at) {
    const int32_t Hm = (int32_t)a.H - 1, Wm = (int32_t)a.W - 1, W = (int32_t)a.W;
    const uint32_t nh = KH > 0 ? (uint32_t)KH : kh, nw = KW > 0 ? (uint32_t)KW : kw;
    best = 0.f;
    at = -1;
    if constexpr (!PAD) {
      const int32_t e0 = h0 * W + w0;
      float v[KH][KW];
#pragma unroll
      for (int i = 0; i < KH; ++i) load_run<KW>(img + e0 + i * W, v[i]);
#pragma unroll
      for (int i = 0; i < KH; ++i)
#pragma unroll
        for (int j = 0; j < KW; ++j) take(v[i][j], e0 + i * W + j, i == 0 && j == 0, best, at);
      return;
    }
#pragma unroll
    for (uint32_t i = 0; i < nh; ++i) {
      const int32_t h = clampi(h0 + (int32_t)i, Hm);
#pragma unroll
      for (uint32_t j = 0; j < nw; ++j) {
        const int32_t e = h * W + clampi(w0 + (int32_t)j, Wm);
        const float v = img[e];
        if ((i == 0 && j == 0) || v > best || __builtin_isnan(v)) {
          best = v;
          at = e;
        }
      }
    }
  }

  template <int KH, int KW, bool PAD>
  __device__ static __forceinline__ void units(const PoolArgs& a, uint32_t ubeg, uint32_t uend, uint32_t lane) {
    const uint32_t plane_sz = a.H * a.W;
    for (uint32_t u = ubeg; u < uend; ++u) {
#pragma unroll
      for (uint32_t t = 0; t < kPer; ++t) {
        const uint32_t o = u * kUnit + lane + 64u * t;
        const uint32_t oc = min(o, a.total - 1u);  // lanes past the end redo the last output
        const uint32_t plane = fdiv(oc, a.div_plane);
        const uint32_t r = oc - plane * a.div_plane.d;
        const uint32_t oh = fdiv(r, a.div_wo);
        const uint32_t ow = r - oh * a.Wo;
        const float* img = a.x + (size_t)plane * plane_sz;
        float best;
        int32_t at;
        window<KH, KW, PAD>(a, img, (int32_t)(oh * a.s) - (int32_t)a.p, (int32_t)(ow * a.s) - (int32_t)a.p, a.kh,
                       a.kw, best, at);
        if (o < a.total) {
          __builtin_nontemporal_store(best, a.out + o);
          if (a.idx) __builtin_nontemporal_store(at, a.idx + o);
        }
      }
    }
  }

  template <class Bar>
  __device__ static __forceinline__ void run(const DevTask& dt, const Part& p, Bar&, uint32_t*) {
    const PoolArgs& a = dt.pool;
    const uint32_t lane = lane_id();
    if (a.row3) {
      run_rows(a, p, lane);
      return;
    }
    const uint32_t nw = p.nwg * p.nwaves;
    const uint32_t gw = p.wg * p.nwaves + p.wave;
    const uint32_t q = a.units / nw, r = a.units - q * nw;
    const uint32_t ubeg = gw * q + min(gw, r);
    const uint32_t uend = ubeg + q + (gw < r ? 1u : 0u);
    if (ubeg >= uend) return;
    if (a.kh == 3 && a.kw == 3)
      a.p ? units<3, 3, true>(a, ubeg, uend, lane) : units<3, 3, false>(a, ubeg, uend, lane);
    else if (a.kh == 2 && a.kw == 2)
      a.p ? units<2, 2, true>(a, ubeg, uend, lane) : units<2, 2, false>(a, ubeg, uend, lane);
    else
      units<0, 0, true>(a, ubeg, uend, lane);
  }
};

}  // namespace hf

#include "hf_hash.hpp"
