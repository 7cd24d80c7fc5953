// Sampling kernels: section 2.2 standardisation (temperature softmax / argmax),
// inverse-CDF draws from caller-supplied uniforms, and the accept / resample
// part of Algorithm 1: row statistics spread over the chip, then the decisions, the
// draw of the extra token and the commit / roll-back; two launches, small calls and
// argmax sampling one.
//
// Arithmetic of a standardised row z at temperature T > 0:
//   m = max_k z_k,  e_k = exp((z_k - m) / T)  (fp32 hardware exp2 path),
//   S = sum_k e_k (fp64),  prob_k = e_k * (1/S) (fp64).
// Sums and cumulative sums are carried in fp64, so the blocked summation order
// differs from a sequential one only far below the resolution of the uniforms.  (S of a row
// that top-k / nucleus filter: whole numbers where its list is short, else a thread's up to 32 entries in fp32 first.)
// T == 0 uses integer argmax compares (ties to the lowest index).
#pragma once
#include <limits.h>
#include <type_traits>
#include "common.h"
#include "kernels_misc.h"

namespace sd {

constexpr int SAMPLE_THREADS = 1024;
constexpr int SAMPLE_CHUNK = 256;           // vocabulary entries per scan chunk (64 lanes x 4)
constexpr int SAMPLE_MAX_CHUNKS = 1024;     // vocab <= 262144
constexpr int SAMPLE_REG_F4 = 8;            // a row up to 32768 entries is held in registers
constexpr int SAMPLE_MAX_GAMMA = 15;
constexpr int SAMPLE_PARTS = 64;            // parts a logits row is cut into for its statistics, at most
constexpr int SAMPLE_PART = 1024;           // entries a wavefront takes at a time
constexpr int SAMPLE_CHUNKS_WG = 16;        // scan chunks of one workgroup: one per wavefront

struct RowStat {
  float  m;      // max logit
  int    arg;    // lowest index attaining it
  double S;      // sum of e_k over the kept entries
  float  thr;    // entries with a logit below it are dropped (top-k / nucleus); -inf: none
  float  pad;
};

// The statistics of one part of a row.
struct RowPart {
  double S;      // sum of exp((z - m) / T) over its kept entries
  float  m;      // its max logit
  union { int arg; float thr; };   // argmax sampling: lowest index attaining m; filtered rows (one part): the threshold
};

// Working memory of one sequence's accept / resample call or draw; the ticket is zero between calls.
struct SampleScratch {
  unsigned int ticket[SAMPLE_TICKETS];
  double tot[SAMPLE_MAX_CHUNKS];
};
// The same with the statistics of the sequence's rows, for calls on explicit logits.  The layout depends on
// nothing, so calls of any size may follow each other on one allocation.
struct SampleBlock {
  SampleScratch s;
  RowPart part[2 * SAMPLE_MAX_GAMMA + 1][SAMPLE_PARTS];
};

constexpr int SAMPLE_BINS = 2048;           // 11 bits of the order-preserving key
constexpr int SAMPLE_LIST = 2048;

struct SampleSmem {
  float  redf[16];
  double redd[16];
  int    redi[16];
  int    flag;
  int    n;
  int    chunk;          // scan: chunk that holds the threshold
  int    token;
  double before;         // scan: cumulative weight before that chunk
  double total;
  double ctot[SAMPLE_MAX_CHUNKS];
  unsigned long long bins[SAMPLE_BINS];
  unsigned long long wsum[16];
  unsigned int sel;
  unsigned long long above;
  unsigned int list[SAMPLE_LIST];        // keys of the entries a filter still has to look at
  int listed;
};

__device__ __forceinline__ float exp_scaled(float z, float m, float invT, float thr) {
  return (z >= thr) ? __expf((z - m) * invT) : 0.0f;      // padding (-inf) passes the test and gives 0
}

// Order-preserving map of a float onto unsigned integers, and back.
__device__ __forceinline__ unsigned float_key(float z) {
  const unsigned u = __float_as_uint(z);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_float(unsigned k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Entries k .. k + 3 of a row of V entries that starts at any 4-byte boundary (-inf past its end), in two
// steps, so that several loads can leave before any is looked at: a 16-byte load within the row, then
// the entries moved to their places.  Rows of fewer than four entries are read entry by entry.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4_any raw4_row(const float* __restrict__ z, int k, int V) {
  if (__builtin_expect(V >= 4, 1)) return *reinterpret_cast<const f32x4_any*>(z + min(k, V - 4));
  return f32x4_any{z[min(k, V - 1)], z[min(k + 1, V - 1)], z[min(k + 2, V - 1)], z[V - 1]};
}
__device__ __forceinline__ float4 placed4_row(const f32x4_any& t, int k, int V) {
  constexpr float NONE = -INFINITY;
  const int over = (V >= 4) ? k - (V - 4) : 0;       // > 0: the group runs past the row's end
  const float x = over <= 0 ? t[0] : over == 1 ? t[1] : over == 2 ? t[2] : t[3];
  const float y = over <= 0 ? t[1] : over == 1 ? t[2] : t[3];
  const float z = over <= 0 ? t[2] : t[3];
  return make_float4(k < V ? x : NONE, k + 1 < V ? y : NONE, k + 2 < V ? z : NONE, k + 3 < V ? t[3] : NONE);
}
// The same where V >= 4 is known: no branch, whose two sides meeting would make the load be waited for at once.
__device__ __forceinline__ f32x4_any raw4_long_row(const float* __restrict__ z, int k, int V) {
  return *reinterpret_cast<const f32x4_any*>(z + (unsigned)min(k, V - 4));
}
// N groups, the m-th at k + m * step: all loads first.
template <int N> __device__ __forceinline__ void raw4_rows(const float* __restrict__ z, int k, int step, int V, f32x4_any (&t)[N]) {
  if (__builtin_expect(V >= 4, 1)) {
#pragma unroll
    for (int m = 0; m < N; ++m) t[m] = *reinterpret_cast<const f32x4_any*>(z + min(k + m * step, V - 4));
  } else {
#pragma unroll
    for (int m = 0; m < N; ++m) t[m] = raw4_row(z, k + m * step, V);
  }
}
// A sum of exponentials relative to m, brought to the maximum M >= m.  The factor is the weight that every
// other place gives an entry m (a 64-bit factor would not round as the weights do: probabilities would add up
// to 1 less closely, 3.45e-8 instead of 3.35e-8 rms error of beta over temperatures 0.5 .. 1.3 and
// vocabularies 50257 and 131072; 3.33e-8 where the whole row is summed relative to its maximum).
// (Nothing above -inf: no weight; m == M needs no factor, which keeps a row without any finite entry what
// it is, not a number.)
__device__ __forceinline__ double rescaled_sum(double s, float m, float M, float invT) {
  return (m == M) ? s : (m == -INFINITY) ? 0.0 : s * (double)__expf((m - M) * invT);
}

// A row of up to 32768 entries fits the registers of one 1024-thread workgroup:
// thread tid holds float4 number it * 1024 + tid, it = 0 .. NG - 1 (with_sample_groups: as many as the row needs).  In terms of the
// 256-entry scan chunks, v[it] of wavefront w is lane-slice `lane` of chunk it * 16 + w.
template <int NG>
__device__ __forceinline__ void load_row_regs(const float* __restrict__ z, int V, float4 (&v)[NG]) {
  const float4* z4 = reinterpret_cast<const float4*>(z);
  const int n4 = V >> 2, tid = threadIdx.x;
#pragma unroll
  for (int it = 0; it < NG; ++it) {
    const int i = it * SAMPLE_THREADS + tid;
    const float4 t = z4[min(i, n4 - 1)];           // unconditional load, padding by select
    v[it] = (i < n4) ? t : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
  }
}
// The search behind the filters: the largest key tau such that the entries with a key >= tau weigh at
// least `target` together (weights are integers, so the sums do not depend on the order), 11, 11 and 10
// bits at a time.  One step: a histogram of the entries that share the bits found so far, and the bin
// in which the sum from the top reaches the target; `above` is the weight of what lies beyond the
// bins.  each(f) calls f(key, weight) for this thread's entries, weight as a function.  False (in every
// thread): all entries together weigh less.
struct RadixSearch { unsigned tau; unsigned long long above; int step; };
// fill() adds weights to sm.bins and returns the target; then the bin in which the sum from the top, `above` at its beginning,
// reaches it is left in sm.sel and what lies beyond it in sm.above.  False (in every thread): no bin does.
template <typename Fill>
__device__ __forceinline__ bool find_bin(unsigned long long above, SampleSmem& sm, Fill&& fill) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();
  sm.bins[tid] = 0ull; sm.bins[tid + SAMPLE_THREADS] = 0ull;
  if (tid == 0) sm.sel = 0xffffffffu;
  __syncthreads();
  const unsigned long long target = fill();
  __syncthreads();
  // sums from the top: thread tid owns two bins
  const int hi = SAMPLE_BINS - 1 - 2 * tid, lo = hi - 1;
  const unsigned long long bh = sm.bins[hi], bl = sm.bins[lo];
  const unsigned long long inc = wave_scan(bh + bl);
  if (lane == 63) sm.wsum[wave] = inc;
  __syncthreads();
  unsigned long long before = above + inc - (bh + bl);
  for (int w = 0; w < wave; ++w) before += sm.wsum[w];
  if (before < target && before + bh + bl >= target) {              // exactly one thread, if any
    const bool upper = before + bh >= target;
    sm.sel = (unsigned)(upper ? hi : lo);
    sm.above = upper ? before : before + bh;
  }
  __syncthreads();
  return sm.sel != 0xffffffffu;
}
template <typename Each>
__device__ __forceinline__ bool radix_step(RadixSearch& q, unsigned long long target, SampleSmem& sm, Each&& each) {
  const int shift = (q.step == 0) ? 21 : (q.step == 1) ? 10 : 0, bits = (q.step < 2) ? 11 : 10;
  const unsigned mask = (1u << bits) - 1u, top = (q.step == 0) ? 0u : q.tau >> (shift + bits);
  if (!find_bin(q.above, sm, [&] {
        each([&](unsigned k, auto&& weight) {
          if (q.step == 0 || (k >> (shift + bits)) == top) {
            const unsigned long long w = weight();
            if (w != 0ull) atomicAdd(&sm.bins[(k >> shift) & mask], w);
          }
        });
        return target;
      })) return false;
  q.tau |= sm.sel << shift;
  q.above = sm.above;
  ++q.step;
  return true;
}
// Puts the keys of this thread's entries that `want` into the list (order: whatever; the sums are
// integers); the number of them, which may exceed the list's room.
template <int NG, typename Want>
__device__ __forceinline__ int list_entries(const float4 (&v)[NG], int nv4, SampleSmem& sm, Want&& want) {
  const int tid = threadIdx.x;
  __syncthreads();
  if (tid == 0) sm.listed = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NG; ++it) {
    const float z[4] = {v[it].x, v[it].y, v[it].z, v[it].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned k = float_key(z[e]);
      if (it * SAMPLE_THREADS + tid < nv4 && want(k)) {
        const int i = atomicAdd(&sm.listed, 1);
        if (i < SAMPLE_LIST) sm.list[i] = k;
      }
    }
  }
  __syncthreads();
  return sm.listed;
}
// The rest of a search, by one wavefront over a list of keys in LDS: the key bits below `bits`, eight at a
// time, without a barrier.  (A step of the whole workgroup costs 3 us: five barriers of sixteen
// wavefronts.)  False: all listed entries together weigh less than the target.
template <typename W>
__device__ __forceinline__ bool list_search(RadixSearch& q, int bits, unsigned long long target, const unsigned* list, int n, SampleSmem& sm, W&& weight) {
  const int lane = threadIdx.x & 63;
  while (bits > 0) {
    const int take = min(8, bits), shift = bits - take;
    const unsigned mask = (1u << take) - 1u;
    unsigned long long* bins = sm.bins;              // 256 of them: lane owns four
#pragma unroll
    for (int e = 0; e < 4; ++e) bins[lane * 4 + e] = 0ull;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i = lane; i < n; i += WAVE) {
      const unsigned k = list[i];
      if (bits == 32 || (k >> bits) == (q.tau >> bits)) {
        const unsigned long long w = weight(k);
        if (w != 0ull) atomicAdd(&bins[(k >> shift) & mask], w);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    unsigned long long b[4];                         // from the top: bins 255 - 4 lane - e
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = bins[255 - 4 * lane - e];
    const unsigned long long own = b[0] + b[1] + b[2] + b[3];
    const unsigned long long inc = wave_scan(own);
    unsigned long long before = q.above + inc - own;
    const bool here = before < target && before + own >= target;
    const unsigned long long who = __ballot(here);
    if (who == 0ull) return false;
    int bin = 255 - 4 * lane;
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (before + b[e] < target && bin == 255 - 4 * lane - e) { before += b[e]; --bin; }
    const int src = __ffsll((long long)who) - 1;
    q.tau |= (unsigned)__shfl(bin, src, WAVE) << shift;
    q.above = __shfl(before, src, WAVE);
    bits = shift;
  }
  return true;
}
// weight(key): an integer.  nv4: the row's float4 groups (the registers beyond hold padding).
// Most rows are settled on a short list, by one wavefront: filter_fast's (`listed`, on entry: the list holds every entry with a
// key >= tau, whichever tau will be), else the entries that share the first 11 bits of tau.  A row that overflows
// the list (ties) is searched in the registers to the end.
template <int NG, typename W>
__device__ __forceinline__ unsigned filter_threshold(const float4 (&v)[NG], int nv4, unsigned long long target, SampleSmem& sm, bool listed, W&& weight) {
  const int tid = threadIdx.x, wave = tid >> 6;
  auto in_regs = [&](auto&& f) {
#pragma unroll
    for (int it = 0; it < NG; ++it) {
      const float z[4] = {v[it].x, v[it].y, v[it].z, v[it].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned k = float_key(z[e]);
        f(k, [&] { return (it * SAMPLE_THREADS + tid < nv4) ? weight(k) : 0ull; });
      }
    }
  };
  RadixSearch q{0u, 0ull, 0};
  bool ok = true;
  int bits = 32;
  if (!listed) {
    ok = radix_step(q, target, sm, in_regs);
    if (ok) listed = list_entries(v, nv4, sm, [&](unsigned k) { return (k >> 21) == (q.tau >> 21); }) <= SAMPLE_LIST;
    bits = 21;
  }
  if (ok && listed) {
    const int n = sm.listed;
    if (wave == 0) {
      const bool found = list_search(q, bits, target, sm.list, n, sm, weight);
      if (tid == 0) sm.sel = found ? q.tau : 0u;
    }
    __syncthreads();
    q.tau = sm.sel;
  } else {
    while (ok && q.step < 3) ok = radix_step(q, target, sm, in_regs);
    if (!ok) q.tau = 0u;
  }
  __syncthreads();
  return q.tau;
}

// The wavefront's keys (N = 1 or 2 a lane, key i in lane i % 64) in descending order: a bitonic network whose exchanges stay in
// the vector ALU.
template <int OFF> __device__ __forceinline__ unsigned xor_partner(unsigned v, int lane) {
  if (OFF == 4) return (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);     // lane ^ 7, ^ 3
  if (OFF < 16) return dpp_partner<OFF == 4 ? 1 : OFF>(v);
  const u32x2 r = half_swap<OFF < 16 ? 16 : OFF>(v); // {own, partner} in an order that depends on the lane
  return (lane & OFF) ? r.x : r.y;
}
template <int N>
__device__ __forceinline__ void sort_keys(unsigned (&k)[N]) {
  const int lane = threadIdx.x & 63;
  auto exchange = [&](auto off, auto run) {          // runs of `run` keys: the even ones descending, the odd ones ascending
    constexpr int OFF = decltype(off)::value, RUN = decltype(run)::value;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const unsigned o = xor_partner<OFF>(k[r], lane);
      const bool down = ((lane + 64 * r) & RUN) == 0, low = (lane & OFF) == 0;
      k[r] = (down == low) ? max(k[r], o) : min(k[r], o);
    }
  };
  auto merge = [&](auto run) {
    constexpr int RUN = decltype(run)::value;
    if constexpr (RUN == 128) { const unsigned a = max(k[0], k[N - 1]), b = min(k[0], k[N - 1]); k[0] = a; k[N - 1] = b; }
    if constexpr (RUN >= 64) exchange(std::integral_constant<int, 32>(), run);
    if constexpr (RUN >= 32) exchange(std::integral_constant<int, 16>(), run);
    if constexpr (RUN >= 16) exchange(std::integral_constant<int, 8>(), run);
    if constexpr (RUN >= 8) exchange(std::integral_constant<int, 4>(), run);
    if constexpr (RUN >= 4) exchange(std::integral_constant<int, 2>(), run);
    exchange(std::integral_constant<int, 1>(), run);
  };
  merge(std::integral_constant<int, 2>()); merge(std::integral_constant<int, 4>()); merge(std::integral_constant<int, 8>());
  merge(std::integral_constant<int, 16>()); merge(std::integral_constant<int, 32>()); merge(std::integral_constant<int, 64>());
  if constexpr (N == 2) merge(std::integral_constant<int, 128>());
}

// Top-k: the threads' own maxima go into 256 linear bins between the largest and the smallest of
// them; the bin that holds the top_k-th bounds the top_k-th largest entry from below, so few entries are listed
// (top_k to a dozen more).  Where they are no more than two a lane, wavefront 0 settles both filters in its
// registers: it sorts the keys, so that the top_k-th is one lane's and the nucleus one sum in lane order.
// False (in every thread): more are listed than that, and the list is where filter_threshold goes on (`listed`), or more than the
// list has room for (ties), or the maximum is no finite number.
// (16 rows x 11, vocabulary 32000, top_k 50, top_p 0.95: searches over bins of key bits took 22.6 us, eight
// steps of one wavefront each with every key in one or two bins of the first; 13.8 where the top_k-th key was found bit by bit with
// ballots and every lane added up, entry by entry, what is not below its own; now 8.3.  Whole calls: 60 sequences, gamma 7, vocabulary
// 3000, top_k 50 32.6 -> 16.4; one, gamma 4, 32128, top_k 128, some 140 listed: 31.5 when a list too long for registers was thrown away, then 21.4.)
constexpr int SAMPLE_FAST_LIST = 128;
template <int NG>
__device__ __forceinline__ bool filter_fast(const float4 (&v)[NG], int nv4, float best, float m, float invT, int top_k, float top_p,
                                            SampleSmem& sm, RowStat& st, bool& listed) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, real = min(nv4, SAMPLE_THREADS);
  if (tid == 0) sm.listed = 0;
  float bound = -INFINITY;
  if (top_k <= real) {                               // (uniform; else fewer threads with entries: no bound, everything is listed)
    unsigned* bins = reinterpret_cast<unsigned*>(sm.bins);
    if (tid < 256) bins[tid] = 0u;
    // the bins end at the smallest maximum, or where weights are zero anyway: entries that a mask moved down (to -inf, the
    // type's lowest value, -1e9) would leave all others in one bin (and a row of one value has a span all the same)
    const float reach = fmaxf(105.0f * __builtin_amdgcn_rcpf(invT), 1e-4f * fabsf(m));
    const float lo = fmaxf(-block_reduce(tid < real ? -best : -INFINITY, sm.redf, OpMaxF(), -INFINITY), m - reach);
    const float span = fmaxf(m - lo, 1e-6f * fabsf(m) + 1e-30f), c = 255.0f * __builtin_amdgcn_rcpf(span);
    if (!(m - m == 0.0f && span < 1e37f)) return false;                          // (uniform; 1 / span must be a number of its own)
    if (tid < real) atomicAdd(&bins[(int)fminf((m - best) * c, 255.0f)], 1u);
    __syncthreads();
    if (wave == 0) {
      unsigned own[4], sum = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) { own[e] = bins[lane * 4 + e]; sum += own[e]; }
      const unsigned inc = wave_scan(sum);
      unsigned before = inc - sum;
      if (before < (unsigned)top_k && inc >= (unsigned)top_k) {                  // exactly one lane
        int e = 0;
        while (before + own[e] < (unsigned)top_k) before += own[e++];
        sm.sel = (unsigned)(lane * 4 + e);
      }
    }
    __syncthreads();
    // every entry of a bin up to that one is at least this large (rounding of either side is far below the margins)
    bound = m - (float)(sm.sel + 1u) * span * (1.00001f / 255.0f) - 1e-6f * fabsf(m);
  } else {
    if (nv4 * 4 > SAMPLE_LIST) return false;         // (uniform)
    __syncthreads();
  }
#pragma unroll
  for (int it = 0; it < NG; ++it) {
    const bool hit = !(v[it].x < bound) || !(v[it].y < bound) || !(v[it].z < bound) || !(v[it].w < bound);
    if (!__any(hit)) continue;
    const float z[4] = {v[it].x, v[it].y, v[it].z, v[it].w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!(z[e] < bound) && it * SAMPLE_THREADS + tid < nv4) {
        const int i = atomicAdd(&sm.listed, 1);
        if (i < SAMPLE_LIST) sm.list[i] = float_key(z[e]);
      }
  }
  __syncthreads();
  const int n = sm.listed;
  if (n > SAMPLE_FAST_LIST) { listed = n <= SAMPLE_LIST; return false; }       // (uniform)
  if (wave == 0) {
    auto settle = [&](auto words) {                  // one key a lane, or two
      constexpr int N = decltype(words)::value;
      unsigned k[N];
#pragma unroll
      for (int r = 0; r < N; ++r) k[r] = (lane + 64 * r < n) ? sm.list[lane + 64 * r] : 0u;      // (0: no float's key but a NaN's; sorts behind all)
      sort_keys(k);
      // the top_k-th key; fewer listed than top_k: the others weigh nothing
      const unsigned tau = top_k <= n ? (top_k <= 64 ? __builtin_amdgcn_readlane(k[0], (top_k - 1) & 63) : __builtin_amdgcn_readlane(k[N - 1], (top_k - 1) & 63)) : 0u;
      float thr = tau ? key_float(tau) : -INFINITY;
      float e[N];
      // the sum, in whole numbers of 2^-56 (a weight is at most 1, the list holds 128), as the nucleus's are: exact whatever the order
      auto whole = [](float x) {                     // 31 + 25 bits, to nearest
        const float t = x * 0x1p31f;
        const unsigned hi = (unsigned)t;
        return ((unsigned long long)hi << 25) + (unsigned)rintf((t - (float)hi) * 0x1p25f);
      };
      auto total = [&] {
        unsigned long long t = 0ull;
#pragma unroll
        for (int r = 0; r < N; ++r) {
          e[r] = (lane + 64 * r < n) ? exp_scaled(key_float(k[r]), m, invT, thr) : 0.0f;
          t += whole(e[r]);
        }
        return (double)wave_sum(t) * 0x1p-56;
      };
      double S = total();
      if (top_p > 0.0f && top_p < 1.0f) {
        constexpr double UNIT = 17592186044416.0;    // weights in units of 2^-44 of the largest, as 31 + 13 bits
        auto units = [](float x) {
          const float t = x * 2147483648.0f;
          const unsigned hi = (unsigned)t;
          return ((unsigned long long)hi << 13) | (unsigned long long)(unsigned)((t - (float)hi) * 8192.0f);
        };
        const unsigned long long target = (unsigned long long)((double)top_p * S * UNIT);
        // the first key at which the sum from the top reaches the target (equal keys share the threshold, wherever the sum
        // reaches it among them); entries that top-k dropped weigh nothing
        unsigned long long before = 0ull;
        unsigned best_key = 0u;
#pragma unroll
        for (int r = 0; r < N; ++r) {
          const unsigned long long upto = before + wave_scan(units(e[r])), who = __ballot(lane + 64 * r < n && upto >= target);
          if (who != 0ull && best_key == 0u) best_key = __builtin_amdgcn_readlane(k[r], __ffsll((long long)who) - 1);
          before = lane_value(upto, 63);
        }
        thr = fmaxf(best_key ? key_float(best_key) : -INFINITY, thr);
        S = total();
      }
      if (lane == 0) { sm.total = S; sm.sel = __float_as_uint(thr); }
    };
    if (n <= 64) settle(std::integral_constant<int, 1>());
    else settle(std::integral_constant<int, 2>());
  }
  __syncthreads();
  st.S = sm.total;
  st.thr = __uint_as_float(sm.sel);
  __syncthreads();                                   // (the callers use both again)
  return true;
}

// The nucleus of a row that top-k leaves whole: as filter_threshold, but the first bins are linear in the logit, from the maximum to
// where weights are zero (or to the smallest entry, zmin).  Bins of key bits hold a row's bulk in a few dozen of 2048, and
// hundreds of LDS additions to one address wait for one another; in linear bins they spread, and the bin that decides holds a
// few dozen entries, which one wavefront sorts.  The row's sum, which the target hangs on, is taken in the same pass.  units(e): the
// weight as an integer.  The thresholds are the same (exact sums, and the bin of an entry never decreases as the logit falls).
// False (in every thread): left to filter_threshold.
// Whole calls, top_p 0.9: one sequence, gamma 4, vocabulary 32128 36.1 -> 23.4 us; 16, gamma 2, 19424 26.8 -> 21.2; 15, gamma 7,
// 4720 23.9 -> 16.1 (with as many groups a thread as the row needs; eight 19.3); 64, gamma 7, 32128 93.8 -> 75.9.
template <int NG, typename U>
__device__ __forceinline__ bool nucleus_bins(const float4 (&v)[NG], int nv4, float m, float zmin, float invT, double top_p_units,
                                             SampleSmem& sm, unsigned& tau, U&& units) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // (exp(-31) is below one unit of 2^-44, and units() truncates: what lies beyond weighs nothing)
  const float span = fmaxf(fminf(31.0f * __builtin_amdgcn_rcpf(invT), m - zmin), 1e-6f * fabsf(m) + 1e-30f);
  const float c = (float)(SAMPLE_BINS - 1) * __builtin_amdgcn_rcpf(span);
  if (!(m - m == 0.0f && span < 1e34f)) return false;                            // (uniform; 1 / span must be a number of its own)
  auto bin = [&](float z) { return (unsigned)(SAMPLE_BINS - 1 - (int)fminf((m - z) * c, (float)(SAMPLE_BINS - 1))); };
  auto each = [&](auto&& f) {
#pragma unroll
    for (int it = 0; it < NG; ++it) {
      const float z[4] = {v[it].x, v[it].y, v[it].z, v[it].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) f(z[e], it * SAMPLE_THREADS + tid < nv4);
    }
  };
  auto weight = [&](float z) { return exp_scaled(z, m, invT, -INFINITY); };
  unsigned long long target = 0ull;
  if (!find_bin(0ull, sm, [&] {
        float s = 0.0f;                              // (as row_stats_regs adds)
#pragma unroll
        for (int it = 0; it < NG; ++it) {
          const float z[4] = {v[it].x, v[it].y, v[it].z, v[it].w}, e[4] = {weight(z[0]), weight(z[1]), weight(z[2]), weight(z[3])};
          s += (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const unsigned long long w = (it * SAMPLE_THREADS + tid < nv4) ? units(e[i]) : 0ull;
            if (w != 0ull) atomicAdd(&sm.bins[bin(z[i])], w);
          }
        }
        target = (unsigned long long)(top_p_units * block_reduce((double)s, sm.redd, OpSumD(), 0.0));
        return target;
      })) return false;
  const unsigned sel = sm.sel;
  const unsigned long long above = sm.above;
  __syncthreads();
  if (tid == 0) sm.listed = 0;
  __syncthreads();
  each([&](float z, bool ok) {
    if (ok && bin(z) == sel && units(weight(z)) != 0ull) {
      const int i = atomicAdd(&sm.listed, 1);
      if (i < SAMPLE_LIST) sm.list[i] = float_key(z);
    }
  });
  __syncthreads();
  const int n = sm.listed;
  if (n > SAMPLE_LIST) return false;                 // (uniform)
  if (wave == 0) {
    unsigned found = 0u;
    if (n <= SAMPLE_FAST_LIST) {
      unsigned k[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) k[r] = (lane + 64 * r < n) ? sm.list[lane + 64 * r] : 0u;
      sort_keys(k);
      unsigned long long before = above;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const bool ok = lane + 64 * r < n;
        const unsigned long long upto = before + wave_scan(ok ? units(weight(key_float(k[r]))) : 0ull), who = __ballot(ok && upto >= target);
        if (who != 0ull && found == 0u) found = __builtin_amdgcn_readlane(k[r], __ffsll((long long)who) - 1);
        before = lane_value(upto, 63);
      }
    } else {
      RadixSearch q{0u, above, 0};
      if (list_search(q, 32, target, sm.list, n, sm, [&](unsigned k) { return units(weight(key_float(k))); })) found = q.tau;
    }
    if (lane == 0) sm.sel = found;
  }
  __syncthreads();
  tau = sm.sel;
  __syncthreads();
  return true;
}

// top_k > 0 / 0 < top_p < 1 (section 2.2: top-k and nucleus sampling as an adjusted
// distribution): the kept set is {z >= thr}.  Top-k: thr = k-th largest logit.  Nucleus, applied to
// what top-k left: thr = the largest value whose upper set still carries top_p of the mass (in units
// of 2^-44 of the largest entry's).  Ties with the last kept entry are kept.  Argmax sampling
// ignores both.
template <int NG>
__device__ __forceinline__ RowStat row_stats_regs(const float4 (&v)[NG], float invT, bool greedy,
                                                  SampleSmem& sm, int top_k = 0, float top_p = 0.0f, int V = 0) {
  const int tid = threadIdx.x;
  RowStat st; st.arg = 0; st.S = 0.0; st.thr = -INFINITY; st.pad = 0.0f;
  float m = -INFINITY;
#pragma unroll
  for (int it = 0; it < NG; ++it)
    m = fmaxf(m, fmaxf(fmaxf(v[it].x, v[it].y), fmaxf(v[it].z, v[it].w)));
  const float best = m;
  m = block_reduce(m, sm.redf, OpMaxF(), -INFINITY);
  st.m = m;
  if (greedy) {
    int a = INT_MAX;
#pragma unroll
    for (int it = NG - 1; it >= 0; --it) {
      const int k = (it * SAMPLE_THREADS + tid) * 4;
      if (v[it].w == m) a = k + 3;
      if (v[it].z == m) a = k + 2;
      if (v[it].y == m) a = k + 1;
      if (v[it].x == m) a = k;
    }
    st.arg = block_reduce(a, sm.redi, OpMinI(), INT_MAX);
    return st;
  }
  float thr = -INFINITY;
  const int nv4 = V >> 2;
  bool listed = false;
  if (top_k > 0 && top_k < V) {
    if (filter_fast(v, nv4, best, m, invT, top_k, top_p, sm, st, listed)) return st;
    const unsigned tau = filter_threshold(v, nv4, (unsigned long long)top_k, sm, listed, [](unsigned) { return 1ull; });
    thr = tau ? key_float(tau) : -INFINITY;          // (fewer listed than top_k: the others weigh nothing)
  }
  auto mass = [&] {
    float s = 0.0f;
#pragma unroll
    for (int it = 0; it < NG; ++it) {     // exp(-inf) = 0 for the padding
      // (a filtered row keeps few entries: most wavefronts have none in a group of 256)
      if (thr != -INFINITY && !__any(v[it].x >= thr || v[it].y >= thr || v[it].z >= thr || v[it].w >= thr)) continue;
      s += (exp_scaled(v[it].x, m, invT, thr) + exp_scaled(v[it].y, m, invT, thr)) +
           (exp_scaled(v[it].z, m, invT, thr) + exp_scaled(v[it].w, m, invT, thr));
    }
    return block_reduce((double)s, sm.redd, OpSumD(), 0.0);
  };
  const bool nucleus = top_p > 0.0f && top_p < 1.0f;
  unsigned tau = 0u;
  bool settled = false;
  constexpr double UNIT = 17592186044416.0;          // 2^44: 32768 entries of at most 1 stay below 2^60
  auto units = [](float e) {                         // e * 2^44 as 31 + 13 bits
    const float t = e * 2147483648.0f;
    const unsigned hi = (unsigned)t;
    return ((unsigned long long)hi << 13) | (unsigned long long)(unsigned)((t - (float)hi) * 8192.0f);
  };
  if (nucleus && thr == -INFINITY) {                 // (uniform)
    float zmin = m;
#pragma unroll
    for (int it = 0; it < NG; ++it)
      if (it * SAMPLE_THREADS + tid < nv4) zmin = fminf(zmin, fminf(fminf(v[it].x, v[it].y), fminf(v[it].z, v[it].w)));
    zmin = -block_reduce(-zmin, sm.redf, OpMaxF(), -INFINITY);
    settled = nucleus_bins(v, nv4, m, zmin, invT, (double)top_p * UNIT, sm, tau, units);
    if (settled) thr = tau ? key_float(tau) : -INFINITY;
  }
  double S = mass();
  if (nucleus && !settled) {
    const float floor_thr = thr;                     // what top-k dropped stays dropped
    tau = filter_threshold(v, nv4, (unsigned long long)((double)top_p * S * UNIT), sm, listed, [&](unsigned k) {
      return units(exp_scaled(key_float(k), m, invT, floor_thr));
    });
    thr = fmaxf(tau ? key_float(tau) : -INFINITY, floor_thr);
    S = mass();
  }
  st.S = S;
  st.thr = thr;
  return st;
}

// The four weights of entries k..k+3: prob_p, minus prob_q clipped at zero when
// a draft row is given (the unnormalised adjusted distribution of section 2.3).
struct RowPair {
  const float* zp; const float* zq;     // zq == nullptr: plain row
  float mp, mq;
  float tp, tq;                         // drop thresholds of the two rows
  double invSp, invSq;
  float invT;
  int V;
};

struct RawPair { f32x4_any p, q; };
__device__ __forceinline__ RawPair load4(const RowPair& rp, int k) {
  RawPair t;
  t.p = raw4_row(rp.zp, k, rp.V);
  t.q = raw4_row(rp.zq ? rp.zq : rp.zp, k, rp.V);    // (a plain row: the same line again, unused)
  return t;
}

// c: the chunk (uniform) that the wavefront's four entries a lane are of; only the row's last one has entries to move or to leave
// out.  No branch but the uniform ones: a weight behind one each was half of the kernel's instructions.
__device__ __forceinline__ void calc4(const RowPair& rp, int c, const RawPair& t, double (&w)[4]) {
  const int k = c * SAMPLE_CHUNK + (int)(threadIdx.x & 63) * 4;
  const bool whole = (c + 1) * SAMPLE_CHUNK <= rp.V;
  auto weights = [&](const f32x4_any& raw, float m, float thr, double inv, double (&o)[4]) {
    float z[4] = {raw[0], raw[1], raw[2], raw[3]};
    if (!whole) {
      const float4 p = placed4_row(raw, k, rp.V);
      z[0] = p.x; z[1] = p.y; z[2] = p.z; z[3] = p.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (double)exp_scaled(z[e], m, rp.invT, thr) * inv;
  };
  weights(t.p, rp.mp, rp.tp, rp.invSp, w);
  if (rp.zq) {
    double q[4];
    weights(t.q, rp.mq, rp.tq, rp.invSq, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) { w[e] -= q[e]; w[e] = w[e] > 0.0 ? w[e] : 0.0; }
  }
  if (!whole) {
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (k + e < rp.V) ? w[e] : 0.0;
  }
}

__device__ __forceinline__ void weights4(const RowPair& rp, int c, double (&w)[4]) {
  calc4(rp, c, load4(rp, c * SAMPLE_CHUNK + (int)(threadIdx.x & 63) * 4), w);
}

// Wavefront 0: scan the chunk totals (lane l owns chunks [l*cpl, (l+1)*cpl)), find the
// chunk in which the cumulative weight first exceeds u * total, and leave in sm:
// total, chunk (or -1 - last chunk with positive weight when round-off keeps the
// threshold out of reach) and the cumulative weight before that chunk.
__device__ __forceinline__ void scan_chunk_totals(int nchunks, float u, SampleSmem& sm) {
  const int lane = threadIdx.x & 63;
  const int cpl = (nchunks + 63) / 64;
  const int c0 = min(nchunks, lane * cpl), c1 = min(nchunks, c0 + cpl);
  double local = 0.0;
  for (int c = c0; c < c1; ++c) local += sm.ctot[c];
  const double inc = wave_scan(local), total = lane_value(inc, 63);
  const double theta = (double)u * total;
  double cum = inc - local;
  int found = INT_MAX;
  double before = 0.0;
  for (int c = c0; c < c1; ++c) {
    const double nx = cum + sm.ctot[c];
    if (found == INT_MAX && nx > theta) { found = c; before = cum; }
    cum = nx;
  }
  const int first = wave_min(found);
  int lastpos = -1;
  for (int c = c0; c < c1; ++c) if (sm.ctot[c] > 0.0) lastpos = c;
  lastpos = wave_max(lastpos);
  if (found == first && first != INT_MAX) { sm.chunk = first; sm.before = before; }
  if (lane == 0) {
    sm.total = total;
    if (first == INT_MAX) { sm.chunk = -1 - lastpos; sm.before = 0.0; }
  }
}

// One wavefront: entry by entry scan of a 256-entry chunk (lane holds entries k..k+3 with
// weights w).  Returns in every lane the first entry whose cumulative weight exceeds theta,
// or, in fallback mode / if none does, the last entry with positive weight.
__device__ __forceinline__ int pick_in_chunk(const double (&w)[4], int k, int V, bool fallback, double theta,
                                             double before) {
  const int lane = threadIdx.x & 63;
  const double local = (w[0] + w[1]) + (w[2] + w[3]);
  const double inc = wave_scan(local);
  int cand = INT_MAX;
  if (!fallback) {
    double cum = before + (inc - local);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      cum += w[e];
      if (cand == INT_MAX && cum > theta && k + e < V) cand = k + e;
    }
    cand = wave_min(cand);
  }
  if (cand == INT_MAX) {
    int lp = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) if (w[e] > 0.0 && k + e < V) lp = k + e;
    cand = wave_max(lp);
  }
  return cand;
}

// Inverse-CDF draw: smallest k with cumulative weight > u * total weight, in
// vocabulary order.  Chunks of 256 consecutive entries are summed by one
// wavefront each (coalesced 1 KB reads), the chunk totals are scanned, and only
// the chunk that holds the threshold is scanned entry by entry.  Returns -1 in
// every thread if the total weight is not positive (the caller then falls back
// to the unadjusted row).
__device__ __forceinline__ int icdf_row(const float* zp, const RowStat& sp, const float* zq,
                                        const RowStat& sq, float invT, int V, float u,
                                        SampleSmem& sm, double qscale = 1.0) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  RowPair rp;
  rp.zp = zp; rp.zq = zq; rp.mp = sp.m; rp.mq = sq.m; rp.tp = sp.thr; rp.tq = sq.thr;
  rp.invSp = 1.0 / sp.S; rp.invSq = zq ? qscale / sq.S : 0.0;     // q enters the residual as qscale * q
  rp.invT = invT; rp.V = V;
  const int nchunks = (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK;
  __syncthreads();
  constexpr int CB = 2;                          // chunks whose loads a wavefront keeps in flight
  for (int cb = wave; cb < nchunks; cb += nw * CB) {
    RawPair raw[CB];
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = cb + u * nw;
      raw[u] = load4(rp, min(c, nchunks - 1) * SAMPLE_CHUNK + lane * 4);
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = cb + u * nw;
      if (c < nchunks) {
        double w[4];
        calc4(rp, c, raw[u], w);
        const double t = wave_sum((w[0] + w[1]) + (w[2] + w[3]));
        if (lane == 0) sm.ctot[c] = t;
      }
    }
  }
  __syncthreads();
  if (wave == 0) scan_chunk_totals(nchunks, u, sm);
  __syncthreads();
  const double total = sm.total;
  if (!(total > 0.0)) return -1;
  const int chunk = sm.chunk;
  if (wave == 0) {
    const bool fallback = chunk < 0;          // threshold not reached by round-off
    const int c = __builtin_amdgcn_readfirstlane(fallback ? (-1 - chunk) : chunk);
    const int k = c * SAMPLE_CHUNK + lane * 4;
    double w[4];
    weights4(rp, c, w);
    const int tok = pick_in_chunk(w, k, V, fallback, (double)u * total, sm.before);
    if (lane == 0) sm.token = tok;
  }
  __syncthreads();
  return sm.token;
}

// Inverse-CDF draw from rows held in registers (see load_row_regs for the layout):
// same arithmetic and summation order as icdf_row, without touching memory.
__device__ __forceinline__ void weights_of(const float4& zp, const float4& zq, bool with_q, float mp, float mq,
                                           float tp, float tq, double invSp, double invSq, float invT,
                                           double (&w)[4]) {
  const float a[4] = {zp.x, zp.y, zp.z, zp.w}, b[4] = {zq.x, zq.y, zq.z, zq.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double p = (double)exp_scaled(a[e], mp, invT, tp) * invSp;    // padding: exp(-inf) = 0
    if (with_q) {
      p -= (double)exp_scaled(b[e], mq, invT, tq) * invSq;
      p = p > 0.0 ? p : 0.0;
    }
    w[e] = p;
  }
}

template <int NG>
__device__ __forceinline__ int icdf_regs(const float4 (&vp)[NG], const RowStat& sp,
                                         const float4 (&vq)[NG], const RowStat& sq, bool with_q,
                                         float invT, int V, float u, SampleSmem& sm, double qscale = 1.0) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NW = SAMPLE_THREADS / 64;
  const double invSp = 1.0 / sp.S, invSq = with_q ? qscale / sq.S : 0.0;
  const int nchunks = (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NG; ++it) {
    const int c = it * NW + wave;
    double w[4];
    weights_of(vp[it], vq[it], with_q, sp.m, sq.m, sp.thr, sq.thr, invSp, invSq, invT, w);
    const double t = wave_sum((w[0] + w[1]) + (w[2] + w[3]));
    if (lane == 0 && c < nchunks) sm.ctot[c] = t;
  }
  __syncthreads();
  if (wave == 0) scan_chunk_totals(nchunks, u, sm);
  __syncthreads();
  const double total = sm.total;
  if (!(total > 0.0)) return -1;
  const int chunk = sm.chunk;
  const bool fallback = chunk < 0;            // threshold not reached by round-off
  const int c = fallback ? (-1 - chunk) : chunk;
  if (wave == c % NW) {
    double w[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int it = 0; it < NG; ++it)
      if (it == c / NW) weights_of(vp[it], vq[it], with_q, sp.m, sq.m, sp.thr, sq.thr, invSp, invSq, invT, w);
    const int tok = pick_in_chunk(w, c * SAMPLE_CHUNK + lane * 4, V, fallback, (double)u * total, sm.before);
    if (lane == 0) sm.token = tok;
  }
  __syncthreads();
  return sm.token;
}

// ---------------------------------------------------------------------------
// Draw one token from one logits row: x_i ~ q_i of the draft loop, or the
// plain-decoding draw t ~ p.
//   mode 0: store the token as guess number `slot` (st->x[slot])
//   mode 1: commit it (standard decoding): len += 1
// Several sequences: sequence b reads the row at logits + b * seq_stride (floats) and uses
// prm[b], st[b].
// ---------------------------------------------------------------------------
// The draw is spread over the chip: a workgroup finds the row's maximum itself (a cheap pass over the
// whole row), then takes sixteen chunks of 256 entries, one per wavefront.  The chunk totals go to
// memory; the workgroup that arrives last scans them and walks the chunk that holds u * total.
// (One workgroup for the whole row is bound by its own instruction stream: 32 exponentials per thread,
// twice, and the fp64 weights.)  The weights are exp((z - m) / T) without the division by
// their sum: both sides of "cumulative weight > u * total" carry the same factor.
// Argmax: one workgroup holds a row of one pass; of a longer one, each takes the maximum of its own entries
// and the last to arrive the lowest index.
// Rows that top-k / nucleus filter go to sample_row_filter_kernel: one workgroup, the row in registers.
// grid = (sample_workgroups(V), sequences).
__host__ __device__ constexpr int sample_workgroups(int V) {
  return ((V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK + SAMPLE_CHUNKS_WG - 1) / SAMPLE_CHUNKS_WG;
}
// f with the groups of four entries that 1024 threads take of a row of V in one pass (the most they hold: 8),
// as a compile-time number.
template <typename F> void with_sample_groups(int V, F&& f) {
  if (V <= 4 * SAMPLE_THREADS) f(std::integral_constant<int, 1>());
  else if (V <= 8 * SAMPLE_THREADS) f(std::integral_constant<int, 2>());
  else if (V <= 16 * SAMPLE_THREADS) f(std::integral_constant<int, 4>());
  else f(std::integral_constant<int, SAMPLE_REG_F4>());
}

// A finished draw or run of Algorithm 1 into the device's state and, where `host` is given, what the host reads of it into
// pinned host memory, 16 bytes at a time: a copy less behind the launch.
__device__ __forceinline__ void put4(int32_t* p, int a, int b, int c, int d) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  *reinterpret_cast<i32x4*>(p) = i32x4{a, b, c, d};
}
__device__ __forceinline__ void commit_draw(SeqState* st, int mode, int slot, int tok, SeqState* host = nullptr) {
  if (mode == 0) {
    st->x[slot] = tok;
  } else {
    const int len = st->len + 1, last = st->last_tok;
    put4(&st->len, len, tok, last, 0);
    st->out[0] = tok;
    if (host) { put4(&host->len, len, tok, last, 0); host->out[0] = tok; }
  }
}

// One run of Algorithm 1: x_1 .. x_n, t.
__device__ __forceinline__ void commit_run(SeqState* st, int n, int t, int fell_back, SeqState* host) {
  static_assert(offsetof(SeqState, len) == 0 && offsetof(SeqState, last_tok) == 4 && offsetof(SeqState, prev_tok) == 8 &&
                offsetof(SeqState, n) == 12 && offsetof(SeqState, out) % 16 == 0 && sizeof(SeqState) % 16 == 0, "put4");
  int o[16];
  for (int i = 0; i < 16; ++i) o[i] = st->x[i];
  const int len = st->len + n + 1, last = st->last_tok, fallbacks = st->fallbacks + fell_back;
  int prev = last;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    prev = (i == n - 1) ? o[i] : prev;
    o[i] = (i < n) ? o[i] : (i == n ? t : -1);
  }
  auto put = [&](SeqState* s) {
    put4(&s->len, len, t, prev, n);
#pragma unroll
    for (int i = 0; i < 16; i += 4) put4(s->out + i, o[i], o[i + 1], o[i + 2], o[i + 3]);
    s->fallbacks = fallbacks;
  };
  put(st);
  if (host) put(host);
}

// The workgroups' hand-over: each leaves 8-byte results with write-through stores (post) and takes a
// ticket; the last one to arrive sees them all through loads that go past its own caches (collect).  A
// ticket with release / acquire semantics instead writes back and invalidates an L2 per workgroup,
// which costs more than the whole kernel when hundreds of them do it.
__device__ __forceinline__ void post(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double collect(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void post_part(RowPart* p, const RowPart& r) {
  static_assert(sizeof(RowPart) == 16, "two words");
  double w[2];
  __builtin_memcpy(w, &r, 16);
  post(reinterpret_cast<double*>(p), w[0]);
  post(reinterpret_cast<double*>(p) + 1, w[1]);
}
__device__ __forceinline__ RowPart collect_part(const RowPart* p) {
  const double w[2] = {collect(reinterpret_cast<const double*>(p)), collect(reinterpret_cast<const double*>(p) + 1)};
  RowPart r;
  __builtin_memcpy(&r, w, 16);
  return r;
}
__device__ __forceinline__ bool last_to_post(unsigned int* ticket, unsigned int expected, int* lds_flag) {
  if (expected == 1u) { __syncthreads(); return true; }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's posts have reached memory
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = (t == expected - 1u);
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *lds_flag = last;
  }
  __syncthreads();
  return *lds_flag != 0;
}

// Argmax over groups of four entries as raw4_rows loads them, no entry moved to its place: a group past the
// row's end holds the last entries again, under their own indices.  Group `it` starts at k + it * step.
// argmax_groups brings a thread's (m, arg), -inf / INT_MAX at first, up to date; passes go up the row.
template <int NG>
__device__ __forceinline__ void argmax_groups(const f32x4_any (&v)[NG], int k, int step, int V, float& m, int& arg) {
  float mb = -INFINITY;
#pragma unroll
  for (int it = 0; it < NG; ++it) mb = fmaxf(mb, fmaxf(fmaxf(v[it][0], v[it][1]), fmaxf(v[it][2], v[it][3])));
  int ab = INT_MAX;                                  // descending: the lowest index is assigned last
#pragma unroll
  for (int it = NG - 1; it >= 0; --it) {
    const int kk = (V >= 4) ? min(k + it * step, V - 4) : k + it * step;
#pragma unroll
    for (int e = 3; e >= 0; --e) ab = (v[it][e] == mb) ? kk + e : ab;
  }
  arg = (mb > m || arg == INT_MAX) ? ab : arg;       // (equal entries of a later pass have higher indices)
  m = fmaxf(m, mb);
}
// The workgroup's, in wavefront 0 (one barrier); INT_MAX where no entry is a number.
__device__ __forceinline__ void argmax_workgroup(float& m, int& arg, int V, float* wm, int* wa) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (V < 4 && arg != INT_MAX) arg = min(arg, V - 1);                            // (such rows are read entry by entry, the last one repeated)
  const float M = wave_max(m);
  const int A = wave_min(m == M ? arg : INT_MAX);
  if (lane == 0) { wm[wave] = M; wa[wave] = A; }
  __syncthreads();
  if (wave != 0) return;
  const float t = (lane < nw) ? wm[lane & 15] : -INFINITY;
  m = wave_max(t);
  arg = wave_min(lane < nw && t == m ? wa[lane & 15] : INT_MAX);
}

// What follows a draw: the embedding of Mq's next step (e.x given), at position len - 1 + step, its logits for row seq * gamma + step;
// or the committed state's copy for the host.
struct DrawNext {
  EmbedArgs e;
  int step, gamma;
  SeqState* host;        // pinned host memory, [sequences]
};
// Every thread of the workgroup that drew calls; tok: wavefront 0's.
__device__ __forceinline__ void finish_draw(const DrawNext& next, SeqState* st, int mode, int slot, int tok, SampleSmem& sm, int seq) {
  if (threadIdx.x == 0) commit_draw(st, mode, slot, tok, next.host ? next.host + seq : nullptr);
  if (next.e.x == nullptr) return;                   // (uniform)
  if (threadIdx.x == 0) sm.token = tok;
  __syncthreads();
  embed_drawn(next.e, seq, sm.token, st->len - 1 + next.step, seq * next.gamma + next.step, sm.redf);
}

// NG: groups of four entries that a thread takes of the row (with_sample_groups).  The row's first pass and
// this workgroup's own entries are asked for before the step's parameters are waited for: 5.8 -> 5.0 us at
// vocabulary 8192, 6.8 -> 6.6 at 32000; argmax 3.9 -> 2.3 and 4.2 -> 3.7.
template <int NG>
static __global__ __launch_bounds__(SAMPLE_THREADS) void sample_row_split_kernel(
    const float* __restrict__ logits, int V, const StepParams* __restrict__ prm, int uniform_idx,
    SeqState* __restrict__ st, int mode, int slot, size_t seq_stride, SampleScratch* __restrict__ scr, const DrawNext next) {
  __shared__ SampleSmem sm;
  const int w = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  logits += (size_t)blockIdx.y * seq_stride;
  prm += blockIdx.y;
  st += blockIdx.y;
  scr += blockIdx.y;
  const int c = w * SAMPLE_CHUNKS_WG + wave, nchunks = (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK, k_mine = c * SAMPLE_CHUNK + lane * 4;
  f32x4_any v[NG];                                   // (a model's vocabulary is 16 at least)
#pragma unroll
  for (int it = 0; it < NG; ++it) v[it] = raw4_long_row(logits, (it * SAMPLE_THREADS + tid) * 4, V);
  const f32x4_any raw_mine = raw4_long_row(logits, k_mine, V);
  const float T = prm->temperature, u = prm->uniforms[uniform_idx];
  const bool greedy = (T == 0.0f);
  const float invT = greedy ? 1.0f : 1.0f / T;
  int tok = 0;                                       // (wavefront 0's)
  if (greedy) {
    float m = -INFINITY;
    int arg = INT_MAX;
    if (NG < SAMPLE_REG_F4 || V <= 4 * NG * SAMPLE_THREADS) {
      // a row of one pass: one workgroup holds it whole, and needs no hand-over (0.7 us of 3.9 at 8192 entries)
      if (w != 0) return;
      argmax_groups(v, tid * 4, 4 * SAMPLE_THREADS, V, m, arg);
      argmax_workgroup(m, arg, V, sm.redf, sm.redi);
      tok = arg;
    } else {
      // longer: each workgroup its own entries (V >= 4: no index to clamp)
      const f32x4_any one[1] = {raw_mine};
      argmax_groups(one, k_mine, 0, V, m, arg);
      argmax_workgroup(m, arg, V, sm.redf, sm.redi);
      // order of the posted words: larger maximum first (-0 counts as 0), then the lower index
      if (tid == 0)
        post(&scr->tot[w], __longlong_as_double((long long)(((unsigned long long)float_key(m + 0.0f) << 32) | (0xffffffffu - (unsigned)arg))));
      if (!last_to_post(scr->ticket, gridDim.x, &sm.flag)) return;
      if (wave == 0) {
        unsigned long long best = (lane < (int)gridDim.x) ? (unsigned long long)__double_as_longlong(collect(&scr->tot[lane])) : 0ull;
#pragma unroll
        for (int o = 32; o; o >>= 1) {
          const unsigned long long t = __shfl_xor(best, o, WAVE);
          best = t > best ? t : best;
        }
        tok = (int)(0xffffffffu - (unsigned)best);
      }
    }
  } else {
    // The row's maximum.  A group past the row's end reads the row's last entries a second time, which
    // leaves it what it is: no entry is moved or masked (that was 1.0 us of 8.4 at 32128 entries).
    float m = -INFINITY;
    auto take = [&](const f32x4_any (&t)[NG]) {
#pragma unroll
      for (int it = 0; it < NG; ++it) m = fmaxf(m, fmaxf(fmaxf(t[it][0], t[it][1]), fmaxf(t[it][2], t[it][3])));
    };
    take(v);
    for (int k0 = 4 * NG * SAMPLE_THREADS; k0 < V; k0 += 4 * NG * SAMPLE_THREADS) {
#pragma unroll
      for (int it = 0; it < NG; ++it) v[it] = raw4_long_row(logits, k0 + (it * SAMPLE_THREADS + tid) * 4, V);
      take(v);
    }
    m = block_reduce(m, sm.redf, OpMaxF(), -INFINITY);
    const float4 mine = placed4_row(raw_mine, k_mine, V);                        // (past the row: -inf)
    const double t = wave_sum(((double)exp_scaled(mine.x, m, invT, -INFINITY) + (double)exp_scaled(mine.y, m, invT, -INFINITY)) +
                              ((double)exp_scaled(mine.z, m, invT, -INFINITY) + (double)exp_scaled(mine.w, m, invT, -INFINITY)));
    if (lane == 0 && c < nchunks) post(&scr->tot[c], t);
    if (!last_to_post(scr->ticket, gridDim.x, &sm.flag)) return;
    for (int i = tid; i < nchunks; i += SAMPLE_THREADS) sm.ctot[i] = collect(&scr->tot[i]);
    __syncthreads();
    if (wave == 0) {
      scan_chunk_totals(nchunks, u, sm);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const double total = sm.total;
      const int chunk = sm.chunk;
      const bool fallback = chunk < 0;          // threshold not reached by round-off
      const int k = (fallback ? (-1 - chunk) : chunk) * SAMPLE_CHUNK + lane * 4;
      const float4 z = placed4_row(raw4_long_row(logits, k, V), k, V);
      const double wv[4] = {(double)exp_scaled(z.x, m, invT, -INFINITY), (double)exp_scaled(z.y, m, invT, -INFINITY),
                            (double)exp_scaled(z.z, m, invT, -INFINITY), (double)exp_scaled(z.w, m, invT, -INFINITY)};
      tok = pick_in_chunk(wv, k, V, fallback, (double)u * total, sm.before);
    }
  }
  finish_draw(next, st, mode, slot, tok, sm, (int)blockIdx.y);
}

template <int NG>
static __global__ __launch_bounds__(SAMPLE_THREADS) void sample_row_filter_kernel(
    const float* __restrict__ logits, int V, const StepParams* __restrict__ prm, int uniform_idx,
    SeqState* __restrict__ st, int mode, int slot, size_t seq_stride, const DrawNext next) {
  __shared__ SampleSmem sm;
  logits += (size_t)blockIdx.x * seq_stride;
  prm += blockIdx.x;
  st += blockIdx.x;
  const float T = prm->temperature;
  const bool greedy = (T == 0.0f);                   // (ignores the filters)
  const float invT = greedy ? 1.0f : 1.0f / T;
  float4 v[NG];
  load_row_regs(logits, V, v);
  const RowStat rs = row_stats_regs(v, invT, greedy, sm, prm->top_k, prm->top_p, V);
  const int tok = greedy ? rs.arg : icdf_regs(v, rs, v, rs, false, invT, V, prm->uniforms[uniform_idx], sm);
  finish_draw(next, st, mode, slot, tok, sm, (int)blockIdx.x);
}

// ---------------------------------------------------------------------------
// Accept / resample (Algorithm 1, second half), for `rows` independent sequences:
//   row_parts_kernel    statistics of the 2 gamma + 1 logits rows of every sequence (row j <= gamma: p_{j+1};
//                       j > gamma: q_{j-gamma}), a wavefront per 1024 entries; row_filter_kernel
//                       does it for rows that top-k / nucleus filter, a workgroup per row
//   accept_kernel       evaluates r_i <= p_i(x_i)/q_i(x_i) for all i, takes n = index of the first
//                       rejection, draws t from norm(max(0, p_{n+1} - q_{n+1})) (n < gamma) or
//                       p_{gamma+1}, writes n and t, and, when `st` is given, commits the sequence:
//                       out = x_1..x_n, t; len += n+1 (which is the KV roll-back: cache rows
//                       beyond the committed length are dead and get overwritten); further
//                       workgroups compute the acceptance probabilities beta when asked for.
// x, r, s: explicit arrays [rows, gamma] / [rows] or, when prm/st are given,
// taken from the device-resident step parameters and state.
// ---------------------------------------------------------------------------
struct AcceptArgs {
  const float *p, *q;                  // logits [rows][gamma + 1][V], [rows][gamma][V]
  const int* x; const float *r, *s;
  int gamma, V;
  int part_len, nparts;                // entries of one part of a row's statistics (a multiple of SAMPLE_PART), parts per row
  int chunks_wave, draw_wgs;           // accept_kernel: chunks per wavefront; workgroups of a sequence's draw (beta's follow)
  // in-model use: only whether the temperature is 0 and whether the rows are filtered (the values are read from prm)
  float temperature, lenience;
  double log_lenience;
  int top_k; float top_p;
  const StepParams* prm;
  void* scr; size_t scr_stride;        // sequence b's SampleScratch: scr_stride bytes further each
  RowPart* part; size_t part_seq; int part_row;      // statistics of row j of sequence b: part + b * part_seq + j * part_row
  int *out_n, *out_t; float* beta;
  SeqState* st;
  SeqState* host;                      // (with st, optional) pinned host memory for the committed states
};
// Whether row_filter_kernel leaves the statistics (one part a row) instead of row_parts_kernel.
__host__ __device__ inline bool accept_filtered(const AcceptArgs& a) { return a.top_k > 0 || (a.top_p > 0.0f && a.top_p < 1.0f); }
// A row's parts depend on its length only, so its statistics do not depend on the call around it.
__host__ __device__ constexpr int sample_part_len(int V) { return SAMPLE_PART * ((V + SAMPLE_PART * SAMPLE_PARTS - 1) / (SAMPLE_PART * SAMPLE_PARTS)); }
__host__ __device__ constexpr int sample_parts(int V) { return (V + sample_part_len(V) - 1) / sample_part_len(V); }
__device__ __forceinline__ SampleScratch* accept_scratch(const AcceptArgs& a, int b) {
  return reinterpret_cast<SampleScratch*>(static_cast<char*>(a.scr) + (size_t)b * a.scr_stride);
}
__device__ __forceinline__ RowPart* accept_part(const AcceptArgs& a, int b, int j) { return a.part + (size_t)b * a.part_seq + (size_t)j * a.part_row; }
__device__ __forceinline__ const float* accept_row(const AcceptArgs& a, int b, int j) {
  return (j <= a.gamma) ? a.p + ((size_t)b * (a.gamma + 1) + j) * a.V : a.q + ((size_t)b * a.gamma + (j - a.gamma - 1)) * a.V;
}

// A part's first block of entries as it lies in memory, and its statistics.  ANY: rows of fewer than four entries among
// them; else no branch is in the way of the loads, which the compiler would wait for behind it.
typedef f32x4_any PartRaw[SAMPLE_PART / 256];
template <bool ANY>
__device__ __forceinline__ void load_part(const float* z, int k0, int lane, int V, PartRaw& t) {
  if (ANY) raw4_rows(z, k0 + lane * 4, 256, V, t);
  else {
#pragma unroll
    for (int it = 0; it < SAMPLE_PART / 256; ++it) t[it] = raw4_long_row(z, k0 + it * 256 + lane * 4, V);
  }
}
// Every exponential is taken relative to the block's maximum over the whole wavefront (never to a lane's
// own: a lane may hold nothing but padding) and goes into the sum as a double.
// POSTED: another workgroup reads them in the same launch.
template <bool POSTED>
__device__ __forceinline__ void reduce_part(const AcceptArgs& a, int b, int j, int part, int lane, float T, const PartRaw& first) {
  constexpr int NV = SAMPLE_PART / 256;
  const bool greedy = (T == 0.0f);
  if (greedy && j > a.gamma && a.beta == nullptr) return;          // argmax sampling looks at q rows for beta only
  const float invT = greedy ? 1.0f : 1.0f / T;
  float m = -INFINITY;
  double s = 0.0;
  int arg = INT_MAX;
  const int k_end = min(a.V, (part + 1) * a.part_len);
  float4 v[NV];
  auto place = [&](const PartRaw& t, int k0) {
    if (k0 + SAMPLE_PART <= a.V) {                   // (uniform) none to move or to leave out
#pragma unroll
      for (int it = 0; it < NV; ++it) v[it] = make_float4(t[it][0], t[it][1], t[it][2], t[it][3]);
    } else {
#pragma unroll
      for (int it = 0; it < NV; ++it) v[it] = placed4_row(t[it], k0 + it * 256 + lane * 4, a.V);
    }
  };
  place(first, part * a.part_len);
  for (int k0 = part * a.part_len; k0 < k_end; k0 += SAMPLE_PART) {
    if (k0 != part * a.part_len) {                   // (parts longer than a block: more than 65536 entries a row)
      PartRaw t;
      load_part<false>(accept_row(a, b, j), k0, lane, a.V, t);
      place(t, k0);
    }
    float mb = -INFINITY;
#pragma unroll
    for (int it = 0; it < NV; ++it) mb = fmaxf(mb, fmaxf(fmaxf(v[it].x, v[it].y), fmaxf(v[it].z, v[it].w)));
    if (greedy) {
      int ab = INT_MAX;
#pragma unroll
      for (int it = NV - 1; it >= 0; --it) {
        const int k = k0 + it * 256 + lane * 4;
        if (k + 3 < a.V && v[it].w == mb) ab = k + 3;
        if (k + 2 < a.V && v[it].z == mb) ab = k + 2;
        if (k + 1 < a.V && v[it].y == mb) ab = k + 1;
        if (k < a.V && v[it].x == mb) ab = k;
      }
      if (mb > m || (mb == m && ab < arg)) arg = ab;
      m = fmaxf(m, mb);
    } else {
      const float mn = fmaxf(m, wave_max(mb));       // (uniform)
      if (mn != m) s = rescaled_sum(s, m, mn, invT);
      m = mn;
      // (padding and -inf weigh nothing beside any finite maximum; an entry that is not a number never does)
#pragma unroll
      for (int it = 0; it < NV; ++it)
        s += ((double)exp_scaled(v[it].x, m, invT, -INFINITY) + (double)exp_scaled(v[it].y, m, invT, -INFINITY)) +
             ((double)exp_scaled(v[it].z, m, invT, -INFINITY) + (double)exp_scaled(v[it].w, m, invT, -INFINITY));
    }
  }
  RowPart* out = accept_part(a, b, j) + part;
  if (greedy) {
    const float M = wave_max(m);
    arg = wave_min(m == M ? arg : INT_MAX);
    if (lane == 0) { out->S = 0.0; out->m = M; out->arg = arg; }
  } else {
    s = wave_sum(s);
    if (lane == 0) {
      RowPart r;
      r.S = s; r.m = m; r.thr = -INFINITY;
      if (POSTED) post_part(out, r);
      else *out = r;
    }
  }
}

// Bound by the reads.  A wavefront takes every (grid x 4)-th part of the launch (part fastest, then row, then
// sequence) and asks for the next one's 4 KB before it sums this one; no
// barrier, no other wavefront is needed.  No load lies behind a branch and the temperature comes by a scalar load, so the next
// part's stays in flight: 123 MB (64 sequences, gamma 7, vocabulary 32128) 25.2 -> 22.8 us, 5.4 TB/s; 29 MB of unaligned rows
// (16, gamma 4, 50257) 8.2 -> 7.8.  12, 16, 20 and 28 wavefronts a CU: 0.7, 1.0, 0.8 and 0.2 us slower than 24.
// A part's sum is relative to the part's maximum; the parts of a row are brought to the row's by one factor each.
// grid = enough workgroups for one part a wavefront, at most ACCEPT_WAVES_CU wavefronts a CU.
constexpr int ACCEPT_WAVES_CU = 24;
template <bool ANY>
static __global__ __launch_bounds__(256, 6) void row_parts_kernel(const AcceptArgs a, int items, unsigned mag_parts, unsigned mag_rows) {
  const int lane = threadIdx.x & 63, stride = (int)gridDim.x * 4;
  const int nrows = 2 * a.gamma + 1;
  auto locate = [&](int item, int& part, int& j, int& b) {       // (divisions by multiplication: items < 2^32 / 64)
    const int row = (a.nparts == 1) ? item : (int)__umulhi((unsigned)item, mag_parts);
    part = item - row * a.nparts;
    b = (int)__umulhi((unsigned)row, mag_rows); j = row - b * nrows;
  };
  auto load = [&](int item, PartRaw& t) {
    int part, j, b;
    locate(item, part, j, b);
    load_part<ANY>(accept_row(a, b, j), part * a.part_len, lane, a.V, t);
  };
  auto reduce = [&](int item, const PartRaw& t) {
    int part, j, b;
    locate(item, part, j, b);
    const StepParams* prm = a.prm + b;
    const float T = a.prm ? *(const __attribute__((address_space(4))) float*)&prm->temperature : a.temperature;
    reduce_part<false>(a, b, j, part, lane, T, t);
  };
  int item = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (item >= items) return;
  PartRaw t0, t1;
  load(item, t0);
  for (;;) {                                         // (behind the last one: this one's again, from the caches)
    load(item + stride < items ? item + stride : item, t1);
    __builtin_amdgcn_sched_barrier(0);
    reduce(item, t0);
    item += stride;
    if (item >= items) return;
    load(item + stride < items ? item + stride : item, t0);
    __builtin_amdgcn_sched_barrier(0);
    reduce(item, t1);
    item += stride;
    if (item >= items) return;
  }
}

// Top-k / nucleus rows: the search needs the whole row, so one workgroup holds it in registers.
// (Eight groups a thread, vocabularies beyond 16384: the row's 32 registers live through the rare paths too, and 46 registers go to
// 188 bytes a lane of scratch; in sample_row_filter_kernel 48 to 260.  Up to four groups: none.)
// grid = (2 gamma + 1, rows).
template <int NG>
static __global__ __launch_bounds__(SAMPLE_THREADS) void row_filter_kernel(const AcceptArgs a) {
  __shared__ SampleSmem sm;
  const int j = blockIdx.x, b = blockIdx.y;
  const float T = a.prm ? a.prm[b].temperature : a.temperature;
  const bool greedy = (T == 0.0f);                   // (ignores the filters)
  if (greedy && j > a.gamma && a.beta == nullptr) return;
  float4 v[NG];
  load_row_regs(accept_row(a, b, j), a.V, v);
  const RowStat rs = row_stats_regs(v, greedy ? 1.0f : 1.0f / T, greedy, sm, a.prm ? a.prm[b].top_k : a.top_k, a.prm ? a.prm[b].top_p : a.top_p, a.V);
  if (threadIdx.x == 0) {
    RowPart* out = accept_part(a, b, j);
    out->S = rs.S; out->m = rs.m;
    if (greedy) out->arg = rs.arg; else out->thr = rs.thr;
  }
}

// A row's statistics from its parts, by one wavefront (lane = part); every lane gets them.
template <bool POSTED = false>
__device__ __forceinline__ RowStat join_parts(const RowPart* parts, int nparts, bool greedy, float invT) {
  const int i = threadIdx.x & 63;
  const bool ok = i < nparts;
  const RowPart rp = POSTED ? collect_part(parts + min(i, nparts - 1)) : parts[min(i, nparts - 1)];
  RowStat st; st.arg = 0; st.S = 0.0; st.pad = 0.0f;
  st.m = wave_max(ok ? rp.m : -INFINITY);
  st.thr = greedy ? -INFINITY : rp.thr;              // (filtered rows have one part, which every lane read)
  if (greedy) st.arg = wave_min((ok && rp.m == st.m) ? rp.arg : INT_MAX);
  else st.S = wave_sum(ok ? rescaled_sum(rp.S, rp.m, st.m, invT) : 0.0);
  return st;
}

// beta_{i+1} = sum_x min(p(x) / l, q(x)): the probability that guess i+1 is accepted (section 3.1; with
// lenience, appendix A.5).  A wavefront takes SAMPLE_PART entries of both rows at a time.
struct BetaPart { f32x4_any p[SAMPLE_PART / 256], q[SAMPLE_PART / 256]; };
__device__ __forceinline__ void beta_load(BetaPart& t, const float* zp, const float* zq, int k0, int V, int lane) {
  if (k0 + SAMPLE_PART <= V) {                       // (uniform) no entry past the rows
#pragma unroll
    for (int it = 0; it < SAMPLE_PART / 256; ++it) {
      t.p[it] = *reinterpret_cast<const f32x4_any*>(zp + k0 + it * 256 + (unsigned)lane * 4u);
      t.q[it] = *reinterpret_cast<const f32x4_any*>(zq + k0 + it * 256 + (unsigned)lane * 4u);
    }
  } else {
    raw4_rows(zp, k0 + lane * 4, 256, V, t.p);
    raw4_rows(zq, k0 + lane * 4, 256, V, t.q);
  }
}
__device__ __forceinline__ double beta_sum(const BetaPart& t, int k0, int V, int lane, const RowStat& jp, const RowStat& jq, double ip, double iq, float invT) {
  double acc = 0.0;
  auto add = [&](float z, float w) {
    const double pv = (double)exp_scaled(z, jp.m, invT, jp.thr) * ip;
    const double qv = (double)exp_scaled(w, jq.m, invT, jq.thr) * iq;
    acc += pv < qv ? pv : qv;
  };
#pragma unroll
  for (int it = 0; it < SAMPLE_PART / 256; ++it) {
    const int k = k0 + it * 256 + lane * 4;
    if (k0 + SAMPLE_PART <= V) {                     // (uniform) none to move or to leave out
#pragma unroll
      for (int e = 0; e < 4; ++e) add(t.p[it][e], t.q[it][e]);
    } else {
      const float4 p = placed4_row(t.p[it], k, V), q = placed4_row(t.q[it], k, V);
      const float p4[4] = {p.x, p.y, p.z, p.w}, q4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < V) add(p4[e], q4[e]);
    }
  }
  return wave_sum(acc);
}

// One guess's, by a workgroup of NT threads; jr: two entries, ctot: one per SAMPLE_PART entries of the row.
template <int NT>
__device__ __forceinline__ void beta_guess(const AcceptArgs& a, int b, int i, RowStat* jr, double* ctot) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), V = a.V, gamma = a.gamma;
  const StepParams* prm = a.prm ? a.prm + b : nullptr;
  const float T = prm ? prm->temperature : a.temperature;
  const bool greedy = (T == 0.0f);
  const float invT = greedy ? 1.0f : 1.0f / T;
  const double len = (double)(prm ? prm->lenience : a.lenience), log_len = prm ? prm->log_lenience : a.log_lenience;
  const float *zp = accept_row(a, b, i), *zq = accept_row(a, b, gamma + 1 + i);
  BetaPart bp;
  if (!greedy && wave * SAMPLE_PART < V) beta_load(bp, zp, zq, wave * SAMPLE_PART, V, lane);       // arrives while the statistics are joined
  if (wave < 2) {
    const RowStat rs = join_parts(accept_part(a, b, wave ? gamma + 1 + i : i), accept_filtered(a) ? 1 : a.nparts, greedy, invT);
    if (lane == 0) jr[wave] = rs;
  }
  __syncthreads();
  const RowStat jp = jr[0], jq = jr[1];
  double t = 0.0;
  if (greedy) {                                      // one-hot q at its argmax: accepted or not
    const int aq = jq.arg;                           // (INT_MAX: no entry of the draft's row is a number)
    t = ((len < 1.0) ? (aq < V && (double)zp[min(aq, V - 1)] - (double)jp.m >= log_len) : (aq == jp.arg)) ? 1.0 : 0.0;
  } else {
    const double ip = (1.0 / jp.S) / len, iq = 1.0 / jq.S;
    const int nblocks = (V + SAMPLE_PART - 1) / SAMPLE_PART;
    for (int blk = wave; blk < nblocks; blk += NT / WAVE) {
      if (blk != wave) beta_load(bp, zp, zq, blk * SAMPLE_PART, V, lane);
      const double w = beta_sum(bp, blk * SAMPLE_PART, V, lane, jp, jq, ip, iq, invT);
      if (lane == 0) ctot[blk] = w;
    }
    __syncthreads();
    if (wave == 0) {
      for (int blk = lane; blk < nblocks; blk += WAVE) t += ctot[blk];
      t = wave_sum(t);
    }
  }
  if (tid == 0) (a.st ? a.st[b].beta : a.beta + (size_t)b * gamma)[i] = (float)t;
}

// A launch of its own where there are more than two guesses a CU, four in long rows: beyond that the workgroups of
// accept_kernel, two on a CU, would queue (launch_accept, where both sides of the line are measured).  grid = (gamma, rows).
static __global__ __launch_bounds__(256, 6) void beta_kernel(const AcceptArgs a) {
  __shared__ RowStat jr[2];
  __shared__ double ctot[SAMPLE_CHUNK * SAMPLE_MAX_CHUNKS / SAMPLE_PART];
  beta_guess<256>(a, blockIdx.y, blockIdx.x, jr, ctot);
}

// Decisions, draw, commit.  Every workgroup of a sequence joins the statistics and takes the decisions
// itself (a few hundred words), then sums the weights of its chunks of row n (16 chunks_wave of
// them); the last to arrive scans the totals and walks the chunk that holds u * total.
// A small call is this one launch (OWN, launch_accept): a second one would cost it more than its work.
// 64 sequences, gamma 7, vocabulary 32128 (123 MB), both launches, calls back to back: 31.2 us
// (row_parts_kernel 21 - 23: 5.4 TB/s, where a pure read reaches 7); with one 1024-thread workgroup per row and
// then one per sequence it was 42.2.  One sequence, gamma 4: 10.9 us against 16.8.
// OWN_NONE, not ALONE: at most 64 registers, two workgroups a CU, two chunks of row n in flight (60 registers; 33 scalars lie in 36
// bytes a lane of scratch).  ALONE, where every workgroup has a CU of its own: the cap lifted, four chunks in flight, no scratch (65 registers;
// one sequence, gamma 4, 32128 11.2 us -> 10.9; two, gamma 5, 128000 13.6 -> 13.3; with beta,
// two, gamma 6, 40397 13.5 -> 13.1; 16, gamma 5, top-k 50, 32000 15.6 -> 15.4).
enum { OWN_NONE, OWN_SEQUENCE, OWN_ROWS };           // whose the statistics are: row_parts_kernel's; this kernel's, a workgroup per sequence / per logits row
template <int OWN, bool ALONE = OWN != OWN_NONE>
static __global__ __launch_bounds__(SAMPLE_THREADS, ALONE ? 4 : 8) void accept_kernel(const AcceptArgs a) {
  __shared__ SampleSmem sm;
  __shared__ RowStat srow[2 * SAMPLE_MAX_GAMMA + 1];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gamma = a.gamma, V = a.V, nrows = 2 * gamma + 1, nchunks = (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK;
  const StepParams* prm = a.prm ? a.prm + b : nullptr;     // in-model use: per-sequence parameters and state
  SeqState* st = a.st ? a.st + b : nullptr;
  SampleScratch* scr = accept_scratch(a, b);
  const float T = prm ? prm->temperature : a.temperature;
  const bool greedy = (T == 0.0f);
  const float invT = greedy ? 1.0f : 1.0f / T;
  const double len = (double)(prm ? prm->lenience : a.lenience);            // appendix A.5, 1 = exact
  const double log_len = prm ? prm->log_lenience : a.log_lenience;
  const float *P = accept_row(a, b, 0), *Q = accept_row(a, b, gamma + 1);
  const int* x = st ? st->x : a.x + (size_t)b * gamma;
  const float* r = prm ? prm->uniforms + gamma : a.r + (size_t)b * gamma;   // (not read by argmax sampling)
  const float s = greedy ? 0.5f : (prm ? prm->uniforms[2 * gamma] : a.s[b]);
  if (OWN == OWN_NONE && (int)blockIdx.x >= a.draw_wgs) {          // beta of guess i
    beta_guess<SAMPLE_THREADS>(a, b, (int)blockIdx.x - a.draw_wgs, srow, sm.ctot);
    return;
  }
  // what the tests need arrives while the statistics are joined
  int xi = 0;
  float zpx = 0.0f, zqx = 0.0f, ri = 0.5f;
  if (tid < gamma) {
    xi = min(max(x[tid], 0), V - 1);
    zpx = P[(size_t)tid * V + xi];
    if (!greedy) { zqx = Q[(size_t)tid * V + xi]; ri = r[tid]; }
  }
  if (OWN == OWN_SEQUENCE) {
    for (int item = wave; item < nrows * a.nparts; item += SAMPLE_THREADS / 64) {
      PartRaw t;
      load_part<true>(accept_row(a, b, item / a.nparts), item % a.nparts * a.part_len, lane, V, t);
      reduce_part<false>(a, b, item / a.nparts, item % a.nparts, lane, T, t);
    }
    __syncthreads();
  } else if (OWN == OWN_ROWS) {
    for (int part = wave; part < a.nparts; part += SAMPLE_THREADS / 64) {
      PartRaw t;
      load_part<true>(accept_row(a, b, blockIdx.x), part * a.part_len, lane, V, t);
      reduce_part<true>(a, b, blockIdx.x, part, lane, T, t);
    }
    if (!last_to_post(scr->ticket, (unsigned)nrows, &sm.flag)) return;
  }
  for (int row = wave; row < nrows && !(greedy && row > gamma && a.beta == nullptr); row += SAMPLE_THREADS / 64) {
    const RowStat rs = join_parts<OWN == OWN_ROWS>(accept_part(a, b, row), accept_filtered(a) ? 1 : a.nparts, greedy, invT);
    if (lane == 0) srow[row] = rs;
  }
  __syncthreads();
  if (wave == 0) {                        // one lane per guess
    bool reject = false;
    if (tid < gamma) {
      if (greedy) {
        // lenient argmax sampling: keep x when p(x) >= l * max p, p = softmax of the raw logits
        reject = (len < 1.0) ? ((double)zpx - (double)srow[tid].m < log_len) : (srow[tid].arg != xi);
      } else {
        const RowStat sp = srow[tid], sq = srow[gamma + 1 + tid];
        const double p = (double)exp_scaled(zpx, sp.m, invT, sp.thr) * (1.0 / sp.S);
        const double q = (double)exp_scaled(zqx, sq.m, invT, sq.thr) * (1.0 / sq.S);
        const double lq = q * len;
        const double ratio = (lq > 0.0) ? p / lq : INFINITY;
        reject = ((double)ri > ratio);
      }
    }
    const unsigned long long mask = __ballot(reject);
    if (tid == 0) sm.n = mask ? (__ffsll((long long)mask) - 1) : gamma;
  }
  __syncthreads();
  const int n = sm.n;
  int t = 0, fell_back = 0;
  if (greedy) {
    if (OWN == OWN_NONE && blockIdx.x != 0) return;
    t = srow[n].arg;
  } else {
    RowPair rp;
    const bool with_q = n < gamma;
    const RowStat sp = srow[n], sq = srow[gamma + 1 + min(n, gamma - 1)];
    rp.zp = P + (size_t)n * V; rp.zq = with_q ? Q + (size_t)n * V : nullptr;
    rp.mp = sp.m; rp.mq = sq.m; rp.tp = sp.thr; rp.tq = sq.thr; rp.invT = invT; rp.V = V;
    rp.invSp = 1.0 / sp.S; rp.invSq = with_q ? len / sq.S : 0.0;                 // q enters the residual as l * q
    constexpr int CB = ALONE ? 4 : 2;      // chunks whose loads a wavefront keeps in flight
    const int c0 = (OWN ? 0 : (int)blockIdx.x) * SAMPLE_CHUNKS_WG * a.chunks_wave + wave;
    for (int i0 = 0; i0 < a.chunks_wave; i0 += CB) {
      RawPair raw[CB];
#pragma unroll
      for (int i = 0; i < CB; ++i)
        if (i0 + i < a.chunks_wave) raw[i] = load4(rp, min(c0 + (i0 + i) * SAMPLE_CHUNKS_WG, nchunks - 1) * SAMPLE_CHUNK + lane * 4);
#pragma unroll
      for (int i = 0; i < CB; ++i) {
        const int c = c0 + (i0 + i) * SAMPLE_CHUNKS_WG;
        if (i0 + i < a.chunks_wave && c < nchunks) {
          double w[4];
          calc4(rp, c, raw[i], w);
          const double tc = wave_sum((w[0] + w[1]) + (w[2] + w[3]));
          if (lane == 0) post(&scr->tot[c], tc);
        }
      }
    }
    if (!last_to_post(scr->ticket, (unsigned)a.draw_wgs, &sm.flag)) return;
    for (int i = tid; i < nchunks; i += SAMPLE_THREADS) sm.ctot[i] = collect(&scr->tot[i]);
    __syncthreads();
    if (wave == 0) {
      scan_chunk_totals(nchunks, s, sm);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const double total = sm.total;
      if (total > 0.0) {
        const int chunk = sm.chunk;
        const bool fallback = chunk < 0;        // threshold not reached by round-off
        const int c = __builtin_amdgcn_readfirstlane(fallback ? (-1 - chunk) : chunk), k = c * SAMPLE_CHUNK + lane * 4;
        double w[4];
        weights4(rp, c, w);
        const int tok = pick_in_chunk(w, k, V, fallback, (double)s * total, sm.before);
        if (lane == 0) sm.token = tok;
      }
    }
    __syncthreads();
    if (sm.total > 0.0) t = sm.token;
    else if (with_q) { fell_back = 1; t = icdf_row(rp.zp, sp, nullptr, sp, invT, V, s, sm); }     // no residual left: p itself
    else t = -1;
  }
  if (tid == 0) {
    if (a.out_n) a.out_n[b] = n;
    if (a.out_t) a.out_t[b] = t;
    if (st) commit_run(st, n, t, fell_back, a.host ? a.host + b : nullptr);
  }
}

// Argmax sampling without beta: only the target's rows count and nothing is drawn, so
// one launch does it, a workgroup per row; the last of a sequence to arrive decides.  Bound by its chain
// (loads, one barrier, ticket), and with hundreds of sequences by its instructions: hence as many groups of
// four entries a thread and as many threads as the row needs, and everything behind the barrier is one wavefront's.
// Vocabulary 32128, calls back to back in a graph: one sequence, gamma 4: 8.1 -> 4.7 us; 64 sequences: 17.1 -> 10.5.
// grid = (gamma + 1, rows).
template <int NG>
static __global__ __launch_bounds__(SAMPLE_THREADS) void accept_argmax_kernel(const AcceptArgs a) {
  __shared__ float wm[16];
  __shared__ int wa[16];
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, V = a.V, gamma = a.gamma;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = blockDim.x;
  const float* z = accept_row(a, b, j);
  int xi = 0;
  SeqState* st = a.st ? a.st + b : nullptr;
  if (tid < gamma) xi = min(max(st ? st->x[tid] : a.x[(size_t)b * gamma + tid], 0), V - 1);
  float m = -INFINITY;
  int arg = INT_MAX;
  for (int k0 = 0; k0 < V; k0 += 4 * NG * nt) {
    f32x4_any v[NG];
    raw4_rows(z, k0 + tid * 4, 4 * nt, V, v);
    argmax_groups(v, k0 + tid * 4, 4 * nt, V, m, arg);
  }
  argmax_workgroup(m, arg, V, wm, wa);
  if (wave != 0) return;
  SampleScratch* scr = accept_scratch(a, b);
  int last = 0;
  if (lane == 0) {
    post(&scr->tot[j], __longlong_as_double((long long)(((unsigned long long)__float_as_uint(m + 0.0f) << 32) | (unsigned)arg)));     // (-0 counts as 0)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the post has reached memory
    const unsigned t = __hip_atomic_fetch_add(scr->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = t == (unsigned)gamma;
    if (last) __hip_atomic_store(scr->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(last) == 0) return;
  const unsigned long long w = (unsigned long long)__double_as_longlong(collect(&scr->tot[min(lane, gamma)]));
  bool reject = false;
  if (lane < gamma) {
    // lenient argmax sampling: keep x when p(x) >= l * max p, p = softmax of the raw logits
    const float len = a.prm ? a.prm[b].lenience : a.lenience;
    const double log_len = a.prm ? a.prm[b].log_lenience : a.log_lenience;
    reject = ((double)len < 1.0) ? ((double)accept_row(a, b, lane)[xi] - (double)__uint_as_float((unsigned)(w >> 32)) < log_len)
                                : ((int)(unsigned)w != xi);
  }
  const unsigned long long mask = __ballot(reject);
  const int n = mask ? (__ffsll((long long)mask) - 1) : gamma;
  const int t = __shfl((int)(unsigned)w, n, WAVE);
  if (lane == 0) {
    if (a.out_n) a.out_n[b] = n;
    if (a.out_t) a.out_t[b] = t;
    if (st) commit_run(st, n, t, 0, a.host ? a.host + b : nullptr);
  }
}

inline void launch_argmax(hipStream_t stream, const AcceptArgs& a, int rows) {
  with_sample_groups(a.V, [&](auto ng) {
    hipLaunchKernelGGL((accept_argmax_kernel<decltype(ng)::value>), dim3(a.gamma + 1, rows), dim3(min(SAMPLE_THREADS, (a.V + 255) / 256 * WAVE)), 0,
                       stream, a);
  });
}

static __global__ void clear_tickets_kernel(void* scr, size_t stride, int rows, int n) {
  const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (b < rows)
    for (int i = 0; i < n; ++i) reinterpret_cast<SampleScratch*>(static_cast<char*>(scr) + (size_t)b * stride)->ticket[i] = 0u;
}

// The launches of one accept / resample call over `rows` sequences.
inline void launch_accept(hipStream_t stream, AcceptArgs a, int rows, int cus) {
  a.part_len = sample_part_len(a.V); a.nparts = sample_parts(a.V);
  const int nrows = 2 * a.gamma + 1;
  const int wgs = sample_workgroups(a.V);
  if (a.temperature == 0.0f && a.beta == nullptr) {
    launch_argmax(stream, a, rows);
    return;
  }
  // One launch or two: a second one costs the host 2.6 us, a loop of such calls its time.  Us a call, from a host loop /
  // captured, one sequence of gamma 7 unless said:
  //   vocabulary 1000 (15 parts)         OWN_SEQUENCE 9.6 / 9.0
  //   2000 (30)                          OWN_SEQUENCE 12.1 / 11.9   OWN_ROWS 9.8 / 8.6     two 12.5 / 9.4
  //   8000 (120)                                                    OWN_ROWS 11.4 / 11.1   two 12.5 / 11.2
  //   16000, gamma 1 (48)                OWN_SEQUENCE 16.1 / 16.1   OWN_ROWS - / 12.9      two 12.4 / 10.3
  //   50 sequences, gamma 4, 2919 (27)   OWN_SEQUENCE 10.9 / 10.7                          two 12.3 / 10.5
  //   200 sequences, gamma 1, 16384 (48) OWN_SEQUENCE - / 19.6                             two - / 22.9
  const int parts = nrows * a.nparts;
  int own = OWN_NONE;
  if (!accept_filtered(a) && a.beta == nullptr) {
    if (parts <= 16 || (rows * nrows > cus && parts <= 28) || (2 * rows > cus && parts <= 48 && wgs <= 4)) own = OWN_SEQUENCE;
    else if (rows * nrows <= cus && wgs <= 2) own = OWN_ROWS;
  }
  if (accept_filtered(a)) {
    with_sample_groups(a.V, [&](auto ng) {
      hipLaunchKernelGGL((row_filter_kernel<decltype(ng)::value>), dim3(nrows, rows), dim3(SAMPLE_THREADS), 0, stream, a);
    });
  } else if (own == OWN_NONE) {
    const int items = rows * nrows * a.nparts;
    const dim3 parts_grid(min((items + 3) / 4, cus * ACCEPT_WAVES_CU / 4));
    const unsigned mag_parts = (unsigned)((0x100000000ull + a.nparts - 1) / a.nparts), mag_rows = (unsigned)((0x100000000ull + nrows - 1) / nrows);
    if (a.V < 4) hipLaunchKernelGGL((row_parts_kernel<true>), parts_grid, dim3(256), 0, stream, a, items, mag_parts, mag_rows);
    else hipLaunchKernelGGL((row_parts_kernel<false>), parts_grid, dim3(256), 0, stream, a, items, mag_parts, mag_rows);
  }
  // as many workgroups a sequence as fit the CUs in one round, two on each (64 registers; with one on each, 64 sequences of gamma 7
  // 31.9 us a call instead of 31.2, 40 of gamma 3 17.5 instead of 16.2; 128 of gamma 3 33.1 instead of 33.5), but beta's, which are
  // bound by their arithmetic, take one each (16 of gamma 4, vocabulary 50257: 19.5, two on each 26.6); more only repeat the decisions more often
  // (200 sequences, gamma 1, vocabulary 32128: 35.3 us with one, 49.1 with a second that takes the last chunks), beside
  // beta's (16 sequences, gamma 4, vocabulary 50257: 13 and 4 of them a sequence 17.7 us, 7 and 4 13.9), unless
  // those leave less than two of a round (48 sequences, gamma 7, 32128: 45.9 us a call with four, 55.6 with one; 16, gamma
  // 15, 50257: 45.2 with 13, 49.8 with the one that is left; gamma 14: 43.5 with 13, 41.8 with the two)
  // (beta in the launch / apart: 64, gamma 7, 32128 48.0 us / 52.2; 200, gamma 5, 12000 46.9 / 48.6; 40, gamma 10, 4096 12.9 / 16.3;
  //  100, gamma 5, 4096 15.9 / 16.3; but 200, gamma 7, 16384 78.0 / 74.0; 200, gamma 5, 2048 19.7 / 16.5; 200, gamma 3, 1500 17.5 / 15.3;
  //  1000, gamma 1, 8192 52.2 / 50.1)
  const bool beta_apart = a.beta != nullptr && rows * a.gamma > (a.V > 8192 ? 4 : 2) * cus && a.temperature > 0.0f;   // (argmax: no rows to read)
  const int beta_wgs = (a.beta != nullptr && !beta_apart) ? a.gamma : 0;
  const int round = max(1, (beta_wgs ? 1 : 2) * cus / rows), left = round - beta_wgs, most = own ? 1 : min(wgs, left >= 2 ? left : round);
  a.chunks_wave = (wgs + most - 1) / most;
  a.draw_wgs = (wgs + a.chunks_wave - 1) / a.chunks_wave;         // (1 where the statistics are its own work)
  const dim3 grid(own == OWN_ROWS ? nrows : a.draw_wgs + beta_wgs, rows), block(SAMPLE_THREADS);
  if (own == OWN_SEQUENCE) hipLaunchKernelGGL(accept_kernel<OWN_SEQUENCE>, grid, block, 0, stream, a);
  else if (own == OWN_ROWS) hipLaunchKernelGGL(accept_kernel<OWN_ROWS>, grid, block, 0, stream, a);
  else if ((a.draw_wgs + beta_wgs) * rows <= cus) hipLaunchKernelGGL((accept_kernel<OWN_NONE, true>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((accept_kernel<OWN_NONE, false>), grid, block, 0, stream, a);
  if (beta_apart) hipLaunchKernelGGL(beta_kernel, dim3(a.gamma, rows), dim3(256), 0, stream, a);
}

}  // namespace sd
