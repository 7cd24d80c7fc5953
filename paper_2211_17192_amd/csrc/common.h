// Device-side helpers shared by the gfx950 kernels: storage-type traits,
// wavefront (64 lanes) and workgroup reductions, the ticket used by kernels
// whose last-finishing workgroup runs a tail phase.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sd {

constexpr int WAVE = 64;
constexpr int MAX_ROWS = 16;          // rows one forward handles = one MFMA column tile

typedef __bf16 bf16;
typedef float  f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Device-resident decoding state of one sequence (section 2.3 / Algorithm 1:
// the committed prefix is summarised by its length and last two tokens; x
// holds the guesses of the running iteration).
// Slabs of MAX_ROWS rows one batched GEMM launch takes; also the slab count of the fragment-order
// activation buffers ([K/32][GEMM_WIDE_RT][64 lanes][8]) that the producing kernels may write directly.
constexpr int GEMM_WIDE_RT = 6;

struct SeqState {
  int32_t len;                 // committed tokens
  int32_t last_tok;            // token at position len-1
  int32_t prev_tok;            // token at position len-2 (undefined when len < 2)
  int32_t n;                   // accepted guesses of the last iteration
  int32_t x[16];               // guesses x_1..x_gamma of this iteration
  int32_t out[16];             // tokens emitted by the last iteration, -1 padded
  int32_t fallbacks;           // zero-residual fallbacks taken so far
  int32_t pad[3];
  float   beta[16];            // acceptance probabilities beta_1..beta_gamma of the last iteration (when asked for)
};

// Per-call parameters that change between iterations; they live in device
// memory so that a captured graph can be replayed unchanged.
struct StepParams {
  double log_lenience;         // ln(lenience), for the argmax-sampling variant of the lenient test
  float temperature;
  float lenience;              // factor l of the lenient acceptance test, 1 = the exact algorithm
  float uniforms[2 * 15 + 1];  // [0,g) draft draws, [g,2g) accept tests, [2g] final draw
  float top_p;                 // nucleus mass, outside (0,1) = off
  int32_t top_k;               // top-k sampling, 0 = off
  int32_t pad;
};

constexpr int SAMPLE_TICKETS = 64;          // words of a sequence's tickets: the first is the sampling kernels', the others the attention kernel's

// Eight bytes that another workgroup of the same launch reads: written through to memory, read past the caches (their
// order is made by a wait for the stores and a ticket).
__device__ __forceinline__ void post8(float* p, float a, float b) {
  const unsigned long long v = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 collect8(const float* p) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}

// Element (row, k) of the activations of a product over many rows, which lie in MFMA fragment order
// [row / 16][K / 32][64 lanes][8]; KS = K / 32.
__device__ __forceinline__ size_t rows_frag_index(int row, int k, int KS) {
  return (((size_t)(row >> 4) * KS + (k >> 5)) * 64 + (row & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

template <typename T> struct Store;
template <> struct Store<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Store<bf16> {
  static __device__ __forceinline__ float ld(const bf16* p) { return (float)*p; }
  static __device__ __forceinline__ void st(bf16* p, float v) { *p = (bf16)v; }
};

// Round a value the way it would be stored in T and read back.
template <typename T> __device__ __forceinline__ float round_to(float v);
template <> __device__ __forceinline__ float round_to<float>(float v) { return v; }
template <> __device__ __forceinline__ float round_to<bf16>(float v) { return (float)(bf16)v; }

// Load 8 consecutive elements of T (16-byte aligned for bf16, 32 for float) as floats.
template <typename T> __device__ __forceinline__ void load8(const T* p, float (&o)[8]);
template <> __device__ __forceinline__ void load8<float>(const float* p, float (&o)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
template <> __device__ __forceinline__ void load8<bf16>(const bf16* p, float (&o)[8]) {
  const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (float)v[e];
}

// Store 8 consecutive elements of T (aligned as for load8), rounded to T.
template <typename T> __device__ __forceinline__ void store8(T* p, const float (&v)[8]);
template <> __device__ __forceinline__ void store8<float>(float* p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
template <> __device__ __forceinline__ void store8<bf16>(bf16* p, const float (&v)[8]) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
  *reinterpret_cast<bf16x8*>(p) = o;
}

// ---------------------------------------------------------------------------
// Cross-lane combines that stay in the vector ALU: DPP quad permutes and row
// rotations inside a row of 16 lanes, and the gfx950 half-swap instructions
// across rows.  (ds_bpermute-based shuffles go through the LDS pipe, which the
// attention and sampling kernels need for data.)  lane_combine<OFF>(v, op)
// returns op(v, v of the partner lane) in every lane; the partner is lane^OFF
// for OFF in {1, 2, 8, 16, 32} and lane+4 (mod 16, same row) for OFF == 4.
// ---------------------------------------------------------------------------
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <int OFF> __device__ __forceinline__ unsigned dpp_partner(unsigned v) {
  constexpr int ctrl = (OFF == 1) ? 0xB1 : (OFF == 2) ? 0x4E : (OFF == 4) ? 0x124 : 0x128;
  return (unsigned)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xf, 0xf, true);
}
template <int OFF> __device__ __forceinline__ u32x2 half_swap(unsigned v) {
  if (OFF == 16) return __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return __builtin_amdgcn_permlane32_swap(v, v, false, false);
}

template <typename V> struct Words;
template <> struct Words<float> {
  static constexpr int N = 1;
  static __device__ __forceinline__ void split(float v, unsigned (&w)[2]) { w[0] = __float_as_uint(v); w[1] = 0; }
  static __device__ __forceinline__ float join(const unsigned (&w)[2]) { return __uint_as_float(w[0]); }
};
template <> struct Words<int> {
  static constexpr int N = 1;
  static __device__ __forceinline__ void split(int v, unsigned (&w)[2]) { w[0] = (unsigned)v; w[1] = 0; }
  static __device__ __forceinline__ int join(const unsigned (&w)[2]) { return (int)w[0]; }
};
template <> struct Words<unsigned> {
  static constexpr int N = 1;
  static __device__ __forceinline__ void split(unsigned v, unsigned (&w)[2]) { w[0] = v; w[1] = 0; }
  static __device__ __forceinline__ unsigned join(const unsigned (&w)[2]) { return w[0]; }
};
template <> struct Words<double> {
  static constexpr int N = 2;
  static __device__ __forceinline__ void split(double v, unsigned (&w)[2]) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    w[0] = (unsigned)u; w[1] = (unsigned)(u >> 32);
  }
  static __device__ __forceinline__ double join(const unsigned (&w)[2]) {
    return __longlong_as_double((long long)(((unsigned long long)w[1] << 32) | w[0]));
  }
};

template <> struct Words<unsigned long long> {
  static constexpr int N = 2;
  static __device__ __forceinline__ void split(unsigned long long v, unsigned (&w)[2]) { w[0] = (unsigned)v; w[1] = (unsigned)(v >> 32); }
  static __device__ __forceinline__ unsigned long long join(const unsigned (&w)[2]) { return ((unsigned long long)w[1] << 32) | w[0]; }
};

template <int OFF, typename V, typename Op>
__device__ __forceinline__ V lane_combine(V v, Op op) {
  unsigned w[2];
  Words<V>::split(v, w);
  if (OFF < 16) {
    unsigned o[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < Words<V>::N; ++i) o[i] = dpp_partner<OFF>(w[i]);
    return op(v, Words<V>::join(o));
  } else {
    unsigned x[2] = {0, 0}, y[2] = {0, 0};     // {own, partner} in an order that depends on the lane
#pragma unroll
    for (int i = 0; i < Words<V>::N; ++i) { const u32x2 r = half_swap<OFF>(w[i]); x[i] = r.x; y[i] = r.y; }
    return op(Words<V>::join(x), Words<V>::join(y));
  }
}

// The value that lane 0 of this lane's row of 16 holds.  (After the four in-row steps of a sum every
// lane holds a total, but the rotation of the OFF == 4 step gives the quads two different
// association orders; code that must agree bit for bit with code that reads lane 0's total
// takes lane 0's too.)
__device__ __forceinline__ float row_first(float v) {
  const int w = __builtin_bit_cast(int, v);
  const int a = __builtin_amdgcn_readlane(w, 0), b = __builtin_amdgcn_readlane(w, 16);
  const int c = __builtin_amdgcn_readlane(w, 32), d = __builtin_amdgcn_readlane(w, 48);
  const int lane = (int)(threadIdx.x & 63);
  return __builtin_bit_cast(float, lane < 16 ? a : (lane < 32 ? b : (lane < 48 ? c : d)));
}

// All 64 lanes get op over the wavefront (op must be commutative; the
// association order is fixed per lane, so results are run-to-run identical).
template <typename V, typename Op>
__device__ __forceinline__ V wave_allreduce(V v, Op op) {
  v = lane_combine<1>(v, op); v = lane_combine<2>(v, op); v = lane_combine<4>(v, op);
  v = lane_combine<8>(v, op); v = lane_combine<16>(v, op); v = lane_combine<32>(v, op);
  return v;
}

struct OpSumF { __device__ float operator()(float a, float b) const { return a + b; } };
struct OpSumD { __device__ double operator()(double a, double b) const { return a + b; } };
struct OpSumU { __device__ unsigned long long operator()(unsigned long long a, unsigned long long b) const { return a + b; } };
struct OpMaxF { __device__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct OpMinI { __device__ int operator()(int a, int b) const { return min(a, b); } };
struct OpSumI { __device__ int operator()(int a, int b) const { return a + b; } };
struct OpMaxI { __device__ int operator()(int a, int b) const { return max(a, b); } };

__device__ __forceinline__ float wave_sum(float v) { return wave_allreduce(v, OpSumF()); }
__device__ __forceinline__ double wave_sum(double v) { return wave_allreduce(v, OpSumD()); }
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) { return wave_allreduce(v, OpSumU()); }
__device__ __forceinline__ float wave_max(float v) { return wave_allreduce(v, OpMaxF()); }
__device__ __forceinline__ int wave_min(int v) { return wave_allreduce(v, OpMinI()); }
__device__ __forceinline__ int wave_max(int v) { return wave_allreduce(v, OpMaxI()); }

// Inclusive sums over the wavefront in lane order, on the vector ALU too: shifts inside the rows of 16, then the last lane of
// a row into the rows behind it.  (Six steps of ds_bpermute take 0.3 us for a double.)
template <int CTRL, int ROWS, typename V>
__device__ __forceinline__ V dpp_or_zero(V v) {      // (lanes without a source, and rows not in ROWS: zero)
  unsigned w[2], o[2] = {0, 0};
  Words<V>::split(v, w);
#pragma unroll
  for (int i = 0; i < Words<V>::N; ++i) o[i] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w[i], CTRL, ROWS, 0xf, false);
  return Words<V>::join(o);
}
template <typename V> __device__ __forceinline__ V wave_scan(V v) {
  v += dpp_or_zero<0x111, 0xf>(v); v += dpp_or_zero<0x112, 0xf>(v); v += dpp_or_zero<0x114, 0xf>(v); v += dpp_or_zero<0x118, 0xf>(v);
  v += dpp_or_zero<0x142, 0xa>(v);                   // lane 15 of row 0 / 2 into row 1 / 3
  v += dpp_or_zero<0x143, 0xc>(v);                   // lane 31 into rows 2 and 3
  return v;
}
template <typename V> __device__ __forceinline__ V lane_value(V v, int lane) {         // (lane: uniform)
  unsigned w[2], o[2] = {0, 0};
  Words<V>::split(v, w);
#pragma unroll
  for (int i = 0; i < Words<V>::N; ++i) o[i] = (unsigned)__builtin_amdgcn_readlane((int)w[i], lane);
  return Words<V>::join(o);
}

// Workgroup-wide reductions over up to 16 waves.  `red` is LDS scratch of at
// least 16 elements of the value type; every thread gets the result.  The
// combine order is fixed (wave 0..n-1), so results are run-to-run identical.
template <typename V, typename Op>
__device__ __forceinline__ V block_reduce(V v, V* red, Op op, V identity) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_allreduce(v, op);
  __syncthreads();                       // protect `red` from the previous use
  if (lane == 0) red[wave] = v;
  __syncthreads();
  V r = identity;
  if (nw == 16) {                        // (the reads of a loop of unknown length would wait for one another)
#pragma unroll
    for (int w = 0; w < 16; ++w) r = op(r, red[w]);
  } else {
    for (int w = 0; w < nw; ++w) r = op(r, red[w]);
  }
  return r;
}

}  // namespace sd
