// Products over more than one slab of 16 rows (bf16): the prompt of a new sequence, the encoder's
// positions, several sequences decoded together.  Up to 16 rows the weights' way out of memory bounds a
// product (kernels_gemm.h); with hundreds of rows the matrix cores do, and a pass over 16 rows at a time
// reads the weights rows / 16 times.  Here one launch takes all rows of a pass.
//
// Both operands are in MFMA fragment order: the weights as they were re-tiled at load,
// Wt[N/16][K/32][64 lanes][8], and the activations alike, Xf[rows/16][K/32][64 lanes][8], which the
// producing kernels write directly (rows_frag_index).  Every fragment is one contiguous KB: 16-byte
// loads, no swizzle, no LDS bank conflicts.
#pragma once
#include <type_traits>
#include "kernels_gemm.h"

namespace sd {

// Row-major bf16 rows [rows][K] -> fragment order; rows beyond the last repeat it (their results are
// never stored).  grid * 256 threads >= slabs * K/32 * 64.
static __global__ __launch_bounds__(256) void rows_to_slabs_kernel(const bf16* __restrict__ X, bf16* __restrict__ Xf, int rows, int K) {
  const int KS = K >> 5, slabs = (rows + 15) >> 4;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)slabs * KS * 64) return;
  const int lane = (int)(idx & 63);
  const size_t f = idx >> 6;
  const int slab = (int)(f / KS), ks = (int)(f % KS);
  const int row = min(slab * 16 + (lane & 15), rows - 1);
  *reinterpret_cast<bf16x8*>(Xf + idx * 8) = *reinterpret_cast<const bf16x8*>(X + (size_t)row * K + ks * 32 + (lane >> 4) * 8);
}

// LayerNorm of fp32 rows into fragment order: gemm_kernel's statistics (the K-slices of its S
// wavefronts, added in wavefront order) and its normalisation, once per row instead of in every
// workgroup of the product.  grid = slabs, 64 S threads, S = the wavefronts of gemm_kernel.
static __global__ __launch_bounds__(512) void rows_layernorm_kernel(const float* __restrict__ X, const bf16* __restrict__ gain,
                                                                    const bf16* __restrict__ beta, bf16* __restrict__ Xf, int rows, int K,
                                                                    int ksteps_per_wave, float eps) {
  __shared__ float stat[2][8 * 16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, S = blockDim.x >> 6;
  const int j = lane & 15, kq = lane >> 4, KS = K >> 5;
  const int ks0 = min(KS, wave * ksteps_per_wave), ks1 = min(KS, ks0 + ksteps_per_wave);
  const float* x = X + (size_t)min((int)blockIdx.x * 16 + j, rows - 1) * K + kq * 8;
  bf16x8* out = reinterpret_cast<bf16x8*>(Xf) + (size_t)blockIdx.x * KS * 64 + lane;
  // up to HELD k-steps a wavefront (K 1024 with four of them, 2048 with eight) stay in registers over all
  // three passes: one trip to memory instead of three
  constexpr int HELD = 8;
  auto slice_sums = [&](auto&& add) {
    float s = add();
    s = lane_combine<16>(s, OpSumF()); return lane_combine<32>(s, OpSumF());
  };
  auto total = [&](float s, int which) {
    if (kq == 0) stat[which][wave * 16 + j] = s;
    __syncthreads();
    float t = 0.0f;
    for (int w = 0; w < S; ++w) t += stat[which][w * 16 + j];
    return t;
  };
  auto normalise = [&](const float (&xv)[8], int ks, float mu, float rstd, const bf16x8& g, const bf16x8& b) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ln_apply(xv[e], mu, rstd, (float)g[e], (float)b[e]);
    out[ks * 64] = Mma<bf16>::from_floats(v);
  };
  if (ksteps_per_wave <= HELD) {
    float xv[HELD][8];
    bf16x8 g[HELD], b[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const int k = min(ks0 + u, KS - 1) * 32;
      load8<float>(x + k, xv[u]);
      g[u] = Mma<bf16>::load(gain + k + kq * 8);
      b[u] = Mma<bf16>::load(beta + k + kq * 8);
    }
    const float mu = total(slice_sums([&] {
      float s = 0.0f;
#pragma unroll
      for (int u = 0; u < HELD; ++u)
        if (ks0 + u < ks1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) s += xv[u][e];
        }
      return s;
    }), 0) / (float)K;
    const float var = total(slice_sums([&] {
      float s = 0.0f;
#pragma unroll
      for (int u = 0; u < HELD; ++u)
        if (ks0 + u < ks1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) s = add_square(s, xv[u][e] - mu);
        }
      return s;
    }), 1) / (float)K;
    const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
    for (int u = 0; u < HELD; ++u)
      if (ks0 + u < ks1) normalise(xv[u], ks0 + u, mu, rstd, g[u], b[u]);
    return;
  }
  const float mu = total(slice_sums([&] {
    float s = 0.0f;
#pragma unroll 4
    for (int ks = ks0; ks < ks1; ++ks) {
      float v[8]; load8<float>(x + ks * 32, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e];
    }
    return s;
  }), 0) / (float)K;
  const float var = total(slice_sums([&] {
    float s = 0.0f;
#pragma unroll 4
    for (int ks = ks0; ks < ks1; ++ks) {
      float v[8]; load8<float>(x + ks * 32, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s = add_square(s, v[e] - mu);
    }
    return s;
  }), 1) / (float)K;
  const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll 4
  for (int ks = ks0; ks < ks1; ++ks) {
    float v[8]; load8<float>(x + ks * 32, v);
    normalise(v, ks, mu, rstd, Mma<bf16>::load(gain + ks * 32 + kq * 8), Mma<bf16>::load(beta + ks * 32 + kq * 8));
  }
}

struct RowsGemmArgs {
  const bf16* W;          // tiled weights; batch z starts z * w_stride elements further
  const bf16* W2;         // EPI_GATED: the "up" weights
  const bf16* X;          // fragment order
  const bf16* zeros;      // 1 KB of zeros
  // a product behind an RMSNorm: the partial sums of squares of its rows, [slab][n_part][16], slabs
  // ss_stride floats apart (nullptr: no norm, or a LayerNorm that the producer applied)
  const float* ss_in;
  int n_part;
  float eps;
  const bf16* bias;       // [N] or nullptr
  int rows, K, N, kpw, nchunk;   // kpw, nchunk: gemm_kernel's k-steps per wavefront and wavefronts
  int mtiles, ntiles_wg;  // workgroup tiles in either direction
  // EPI_STORE: a batch of products over the same rows, two to a layer: product z takes the weights at
  // W + (z / 2) w_layer + (z % 2) w_which and the output at out + (z / 2) out_layer + (z % 2) out_which
  int batch;
  size_t w_layer, w_which, out_layer, out_which;
  bf16* out;              // EPI_ACT, EPI_GATED: fragment order [rows][N]; EPI_STORE: row-major [rows][N] or
                          // head-major [N / d_head][rows][d_head] (hm != 0)
  int hm, d_head, act;
  // EPI_RESID: x += y; xg = x * gain_next in fragment order and the partial sums of x^2 (both optional)
  float* x;
  bf16* xg;
  const bf16* gain_next;
  float* ss;
  int ss_stride;
  // EPI_QKV
  bf16* q;
  int nq, nkv;
  bf16* kv_pool;
  const int* page_table;
  const int* row_pos;     // < 0: a padding row, nothing goes to the cache
  const int* row_seq;     // several sequences: each row's; its page table starts at page_table + seq * pt_stride
  int pt_stride;
  int page_size, n_kv_heads;
  const float* rope;
  // EPI_LOGITS: row r goes to row out_row[r] of logits (< 0: dropped), times scale
  float* logits;
  const int* out_row;
  float scale;
};

// 1 / rms of the 16 rows of a slab, by one wavefront, into out (LDS): the partial sums in gemm_kernel's
// order.  load() asks for the first 256 of them (d_model <= 4096: all), sums() adds them as they arrive, finish() (lane
// exchanges, division and root) is for behind the main loop, where no multiply waits for it.
struct SlabRms {
  float4 v[16];
  f32x4 q;                                           // rows 4 (lane % 4) .. + 3: the partials lane / 4, lane / 4 + 16, ..
  __device__ __forceinline__ void load(const RowsGemmArgs& a, int slab, int lane) {
    const float* s = a.ss_in + (size_t)slab * a.ss_stride + (lane & 3) * 4;
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = *reinterpret_cast<const float4*>(s + (size_t)min((lane >> 2) + 16 * u, a.n_part - 1) * 16);
  }
  __device__ __forceinline__ void sums(const RowsGemmArgs& a, int slab, int lane) {
    const int f = lane >> 2;
    q = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const bool ok = f + 16 * u < a.n_part;
      q[0] += ok ? v[u].x : 0.0f; q[1] += ok ? v[u].y : 0.0f; q[2] += ok ? v[u].z : 0.0f; q[3] += ok ? v[u].w : 0.0f;
    }
    if (a.n_part > 256) {                            // (uniform)
      const float* s = a.ss_in + (size_t)slab * a.ss_stride + (lane & 3) * 4;
      for (int p = f + 256; p < a.n_part; p += 16) {
        const float4 w = *reinterpret_cast<const float4*>(s + (size_t)p * 16);
        q[0] += w.x; q[1] += w.y; q[2] += w.z; q[3] += w.w;
      }
    }
  }
  static __device__ __forceinline__ void finish(const RowsGemmArgs& a, f32x4 q, int lane, float* out) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      q[e] += __shfl_xor(q[e], 4, 64); q[e] += __shfl_xor(q[e], 8, 64);
      q[e] += __shfl_xor(q[e], 48, 64); q[e] += __shfl_xor(q[e], 16, 64);      // quads 0 + 3, 1 + 2: as the first lane of gemm_kernel's sum
    }
    const int f = lane >> 2;                         // (every lane holds the totals of its four rows: lanes f = 0 .. 3 take one each)
    float t = q[0];
    t = f == 1 ? q[1] : t; t = f == 2 ? q[2] : t; t = f == 3 ? q[3] : t;
    const float r = 1.0f / sqrtf(t / (float)a.K + a.eps);
    if (f < 4) out[(lane & 3) * 4 + f] = r;
  }
};

// What an epilogue needs of a row beside its sums, and of a tile: everything that can be asked for ahead of the main
// loop is, raw, and what depends on a row's position behind the first loads of the stream.  (After the loop, as two or three
// dependent trips to memory, with 1 / rms of the rows ahead of it: 768 features, 128 rows, K-slices, us a launch, LayerNorm
// model: QKV 7.0 -> 6.3, FFN-in 7.3 -> 6.8, FFN-out 7.7 -> 7.4, O 4.9 -> 4.5; 256 features 4.5 -> 3.6; 64 rows of 4096, RMSNorm
// model: QKV 18.7 -> 18.0; of 1024: QKV 6.6 -> 5.7, gated 7.1 -> 6.5; 2000 rows: QKV of 4096 140 -> 133, residual products
// of 1024 27.4 -> 24.7.)
struct RowIn {
  float r1;              // 1 / rms
  int pos;               // EPI_QKV
  unsigned kvrow;        // EPI_QKV: the row of the cache (of d_head elements) that key head 0 goes to
  int orow;              // EPI_LOGITS
};
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
struct TileIn { bf16x4 bias, gain; };

template <int EPI>
struct RowsEpilogue {
  // ---- loads: none behind a branch; what is absent is read from the weights and dropped ----
  static __device__ __forceinline__ int ask_pos(const RowsGemmArgs& a, int rowc) { return EPI == EPI_QKV ? a.row_pos[rowc] : 0; }
  static __device__ __forceinline__ int ask_seq(const RowsGemmArgs& a, int rowc) { return EPI == EPI_QKV ? (a.row_seq != nullptr ? a.row_seq : a.row_pos)[rowc] : 0; }
  static __device__ __forceinline__ int ask_page(const RowsGemmArgs& a, int pos, int seq) {
    return EPI == EPI_QKV ? a.page_table[(a.row_seq != nullptr ? seq * a.pt_stride : 0) + (max(pos, 0) >> (__ffs(a.page_size) - 1))] : 0;
  }
  static __device__ __forceinline__ unsigned cache_row(const RowsGemmArgs& a, int pos, int page) {
    return (unsigned)page * 2u * (unsigned)a.n_kv_heads * (unsigned)a.page_size + (unsigned)(max(pos, 0) & (a.page_size - 1));
  }
  static __device__ __forceinline__ int ask_orow(const RowsGemmArgs& a, int rowc) {
    return EPI == EPI_LOGITS ? (a.out_row != nullptr ? a.out_row : reinterpret_cast<const int*>(a.W))[rowc] : 0;
  }
  static __device__ __forceinline__ TileIn ask_tile(const RowsGemmArgs& a, int n0) {
    TileIn t{};
    if (EPI != EPI_GATED) t.bias = *reinterpret_cast<const bf16x4*>((a.bias != nullptr ? a.bias : a.W) + (unsigned)n0);
    if (EPI == EPI_RESID) t.gain = *reinterpret_cast<const bf16x4*>((a.xg != nullptr ? a.gain_next : a.W) + (unsigned)n0);
    return t;
  }
  // the residual (EPI_RESID), cos and sin of the position (EPI_QKV)
  static __device__ __forceinline__ float4 ask_four(const RowsGemmArgs& a, int rowc, int n0, int pos) {
    if (EPI == EPI_RESID) return *reinterpret_cast<const float4*>(a.x + (size_t)rowc * a.N + n0);
    if (EPI == EPI_QKV) {
      const bool has = a.rope != nullptr;            // (a head's features are whole tiles, q, k and v whole heads: n0 % d_head is the place within the head)
      return *reinterpret_cast<const float4*>((has ? a.rope : reinterpret_cast<const float*>(a.W)) + (has ? (size_t)max(pos, 0) * a.d_head + (n0 & (a.d_head - 1)) : (size_t)0));
    }
    return make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // The finished sums of one 16-feature tile (EPI_GATED: of its gate and up streams): this lane's are the
  // features 16 tile + 4 kq + 0..3 of row 16 slab + j.  gemm_kernel's arithmetic.
  static __device__ __forceinline__ void tile_out(const RowsGemmArgs& a, int slab, int lane, int tile, int bz, const f32x4& s0, const f32x4& s1,
                                                  const RowIn& in, const TileIn& ti, const float4& four) {
    const int j = lane & 15, kq = lane >> 4, row = slab * 16 + j;
    const bool ok = row < a.rows;
    const int n0 = tile * 16 + kq * 4;
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      y[r] = (a.ss_in != nullptr) ? s0[r] * in.r1 : s0[r];
      y[r] += (EPI != EPI_GATED && a.bias != nullptr) ? (float)ti.bias[r] : 0.0f;
    }
    if (EPI == EPI_RESID) {
      float xn[4] = {0.f, 0.f, 0.f, 0.f};
      if (ok) {
        xn[0] = four.x + y[0]; xn[1] = four.y + y[1]; xn[2] = four.z + y[2]; xn[3] = four.w + y[3];
        *reinterpret_cast<float4*>(a.x + (size_t)row * a.N + n0) = make_float4(xn[0], xn[1], xn[2], xn[3]);
      }
      if (a.xg != nullptr) {
        bf16x4 g;
#pragma unroll
        for (int r = 0; r < 4; ++r) g[r] = (bf16)(xn[r] * (float)ti.gain[r]);
        *reinterpret_cast<bf16x4*>(a.xg + rows_frag_index(row, n0, a.N >> 5)) = g;
      }
      if (a.ss != nullptr) {
        // the order of gemm_kernel's 16-lane sum as its first lane sees it: quads 0 + 3, quads 1 + 2
        float q = (square(xn[0]) + square(xn[1])) + (square(xn[2]) + square(xn[3]));
        q += __shfl_xor(q, 48, 64);
        q += __shfl_xor(q, 16, 64);
        if (kq == 0) a.ss[(size_t)slab * a.ss_stride + tile * 16 + j] = q;
      }
    } else if (EPI == EPI_QKV) {
      const bool is_q = n0 < a.nq, is_k = !is_q && n0 < a.nq + a.nkv;          // uniform over the tile
      const int nn = is_q ? n0 : (is_k ? n0 - a.nq : n0 - a.nq - a.nkv);
      const int head = nn >> (__ffs(a.d_head) - 1), d = nn & (a.d_head - 1);
      bf16x4 o;
      if (a.rope != nullptr && (is_q || is_k) && in.pos >= 0) {
        o[0] = (bf16)rope_rotate(y[0], y[1], four.x, four.y, false); o[1] = (bf16)rope_rotate(y[1], y[0], four.x, four.y, true);
        o[2] = (bf16)rope_rotate(y[2], y[3], four.z, four.w, false); o[3] = (bf16)rope_rotate(y[3], y[2], four.z, four.w, true);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (bf16)y[r];
      }
      if (ok) {
        if (is_q) *reinterpret_cast<bf16x4*>(a.q + (size_t)row * a.nq + n0) = o;
        else if (in.pos >= 0) *reinterpret_cast<bf16x4*>(a.kv_pool + ((size_t)in.kvrow + (size_t)((is_k ? 0 : a.n_kv_heads) + head) * a.page_size) * a.d_head + d) = o;
      }
    } else if (EPI == EPI_LOGITS) {
      if (ok && in.orow >= 0)
        *reinterpret_cast<float4*>(a.logits + (size_t)in.orow * a.N + n0) = make_float4(a.scale * y[0], a.scale * y[1], a.scale * y[2], a.scale * y[3]);
    } else {
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = y[r];
        if (EPI == EPI_ACT) v = gelu_tanh(v);
        if (EPI == EPI_GATED) v = ((a.act == ACT_GELU) ? gelu_tanh(v) : silu(v)) * (s1[r] * in.r1);
        o[r] = (bf16)v;
      }
      if (EPI == EPI_STORE) {
        bf16* out = a.out + (size_t)(bz >> 1) * a.out_layer + (size_t)(bz & 1) * a.out_which;
        if (ok) {
          if (a.hm) *reinterpret_cast<bf16x4*>(out + ((size_t)(n0 / a.d_head) * a.rows + row) * a.d_head + n0 % a.d_head) = o;
          else *reinterpret_cast<bf16x4*>(out + (size_t)row * a.N + n0) = o;
        }
      } else {
        *reinterpret_cast<bf16x4*>(a.out + rows_frag_index(row, n0, a.N >> 5)) = o;   // rows past the last: in the padded slab
      }
    }
  }
};

// Workgroups are dealt to the eight XCDs in turn: each XCD gets a contiguous run of tiles with the row
// tiles fastest, so its L2 holds few weight tiles at a time and each is read from memory once.
__device__ __forceinline__ void rows_tile_of_block(const RowsGemmArgs& a, int& bm, int& bn, int& bz) {
  const int total = (int)gridDim.x, b = blockIdx.x, xcd = b & 7, q = total >> 3, r = total & 7;
  const int id = xcd * q + min(xcd, r) + (b >> 3), per = a.mtiles * a.ntiles_wg;
  bz = id / per;
  bm = (id - bz * per) % a.mtiles; bn = (id - bz * per) / a.mtiles;
}

// A weight fragment of the products below.  ONCE: all rows of the launch are one workgroup's, so each weight is read once and need not
// stay in the L2s, where it would drive out the activations that every workgroup reads: non-temporal.  Where several row tiles
// take the same weights, and where they are few (weights_past_l2), they do stay.  64 rows, us a launch, plain / non-temporal: gated 14336 x 4096 49.0 / 42.0, QKV 6144 x 4096 18.4 / 17.7,
// LM head 8192 x 4096 20.5 / 19.4 (a deeper stream without barriers, eight wavefronts with a K-slice each, was as slow as this one with plain
// loads, 49.2); prompts of two row tiles and more (971 to 1314 rows, widths 2048 to 3424) 2 - 10 % slower a call with non-temporal loads.
template <bool ONCE> __device__ __forceinline__ bf16x8 load_weight(const bf16x8* p) {
  if (ONCE) return __builtin_nontemporal_load(p);
  return *p;
}

// A workgroup of NWV (4 or 8) wavefronts takes NT * 16 * NWV features x MT * 16 rows.  A wavefront owns NT
// weight tiles: their fragments go from memory into its registers and nowhere else, while the MT slabs of
// activations pass through LDS and serve all wavefronts.
// Sums are gemm_kernel's, bit for bit: the k-steps of a K-slice accumulate from zero, the slices are
// added in order to a running total.  That doubles the accumulators, so NT * MT is 16 at two wavefronts
// a SIMD (256 registers).  Counters at 1998 rows, gated 14336: matrix cores busy 53 % of the cycles (at the 1.9 GHz
// that the chip holds then), LDS pipe 34 % without a bank conflict, 13 TB/s out of L2 and 2.8 out of memory: none is
// at its limit alone, so it counts what a stall costs: a weight register is reloaded for the next pass of SUB
// k-steps right after its last multiply, the next pass's activations are in flight (registers) while
// this pass is multiplied and reach the other LDS buffer at its end, one barrier per pass.
// Measured with 2000 rows (TFLOP/s; a library product of these sizes reaches 1100 - 1200 on this chip):
//                                     N 4096   N 4096, K 14336   gated 14336   N 6144   (else K 4096)
//   NT 2, MT 8, eight wavefronts        1115        1253             1022        874
//   NT 2, MT 8, four (two workgroups)    938        1066              811        921
//   NT 4, MT 8, four (one a SIMD)        821        1000              725        667
// Eight read the activations once per CU instead of twice, but their workgroups fill the chip in coarser
// rounds (N 6144: 384 workgroups, one round and a half).
template <int EPI, int NT, int MT, int NWV, bool ONCE>
static __global__ __launch_bounds__(64 * NWV, 2) void gemm_rows_kernel(const RowsGemmArgs a) {
  constexpr int SUB = 4, NT_OUT = (EPI == EPI_GATED) ? NT / 2 : NT;
  constexpr int NFRAG = SUB * MT * 64, XPT = NFRAG / (64 * NWV);
  __shared__ __align__(16) bf16x8 xs[2][NFRAG];
  __shared__ float rs_s[MT * 16];
  __shared__ int pos_s[EPI == EPI_QKV ? MT * 16 : 1], row_s[EPI == EPI_QKV || EPI == EPI_LOGITS ? MT * 16 : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KS = a.K >> 5, ntiles = a.N >> 4, slabs = (a.rows + 15) >> 4;
  int bn, bm, bz;
  rows_tile_of_block(a, bm, bn, bz);
  const bf16* wbase[NT];
  int tile0 = (bn * NWV + wave) * NT_OUT;              // first output tile of this wavefront
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int ot = (EPI == EPI_GATED) ? (t >> 1) : t;
    const bf16* w = (EPI == EPI_GATED && (t & 1)) ? a.W2 : a.W + (EPI == EPI_STORE ? (size_t)(bz >> 1) * a.w_layer + (size_t)(bz & 1) * a.w_which : 0);
    wbase[t] = w + (size_t)min(tile0 + ot, ntiles - 1) * KS * 512;
  }

  f32x4 acc[NT][MT], tot[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) { acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f}; tot[t][m] = f32x4{0.f, 0.f, 0.f, 0.f}; }

  bf16x8 wf[NT][SUB], xr[XPT];
  static_assert(SUB == 4 && XPT * NWV == 4 * MT, "wavefront w stages k-step w % 4 of XPT slabs");
  const int kst = wave & 3, slab0 = (wave >> 2) * XPT;
  const bf16x8* xsrc[XPT];                           // uniform
#pragma unroll
  for (int i = 0; i < XPT; ++i) xsrc[i] = reinterpret_cast<const bf16x8*>(a.X) + (size_t)min(bm * MT + slab0 + i, slabs - 1) * KS * 64;
  // k-steps past a slice's end are multiplied with zeros, as gemm_kernel does: they come from a KB of zeros
  auto load_x = [&](int ksb, int len) {
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
      const bf16x8* src = (kst < len) ? xsrc[i] + (size_t)(ksb + kst) * 64 : reinterpret_cast<const bf16x8*>(a.zeros);
      xr[i] = src[(unsigned)lane];
    }
  };
  auto load_w = [&](int u, int ks) {
    const size_t o = (size_t)min(ks, KS - 1) * 512;
#pragma unroll
    for (int t = 0; t < NT; ++t) wf[t][u] = load_weight<ONCE>(reinterpret_cast<const bf16x8*>(wbase[t] + o) + (unsigned)lane);
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XPT; ++i) xs[buf][((slab0 + i) * SUB + kst) * 64 + lane] = xr[i];
  };
  // the order of a pass, which the scheduler would otherwise rearrange so that every load sinks to its
  // end, a few MFMAs ahead of its use: the next k-step's fragments between this one's MFMAs, a
  // weight register's reload behind its last MFMA
  auto order_pass = [&] {
    __builtin_amdgcn_sched_group_barrier(0x100, MT, 0);            // the first k-step's fragments
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);        // MFMAs of one slab
        if (u + 1 < SUB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (u == SUB - 1 && m < XPT) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x020, NT, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x020, XPT, 0);
  };

  // what the epilogue needs of the rows, thread t of row t: asked for ahead of the stream, into LDS behind it
  const int rowc = min(bm * MT * 16 + min((int)threadIdx.x, MT * 16 - 1), a.rows - 1);
  int row_pos = RowsEpilogue<EPI>::ask_pos(a, rowc), row_seq = RowsEpilogue<EPI>::ask_seq(a, rowc);
  const int row_out = RowsEpilogue<EPI>::ask_orow(a, rowc);
  // 1 / rms of the rows: slab w (of four wavefronts: and w + 4) by wavefront w
  SlabRms rms;
  constexpr bool TWO = NWV < MT;
  static_assert(2 * NWV >= MT, "at most two slabs a wavefront");
  f32x4 q2 = {0.f, 0.f, 0.f, 0.f};
  const bool normed = a.ss_in != nullptr;            // (uniform)
  if (normed && wave < MT) rms.load(a, min(bm * MT + wave, slabs - 1), lane);

  // passes of SUB k-steps, never across the end of a K-slice
  int end = min(KS, a.kpw);                          // of the slice being multiplied
  load_x(0, end);
#pragma unroll
  for (int u = 0; u < SUB; ++u) load_w(u, u);
  store_x(0);
  int ksb = 0, next = min(SUB, end);                 // this pass, the next one
  int end_next = (next < end) ? end : min(KS, end + a.kpw);                  // of the slice `next` lies in
  load_x(next, end_next - next);
  if (normed) {
    if (wave < MT) rms.sums(a, min(bm * MT + wave, slabs - 1), lane);
    if (TWO && wave + NWV < MT) {
      SlabRms second;
      second.load(a, min(bm * MT + wave + NWV, slabs - 1), lane);
      second.sums(a, min(bm * MT + wave + NWV, slabs - 1), lane);
      q2 = second.q;
    }
  }
  int row_page = 0;
  if (EPI == EPI_QKV) {
    asm volatile("" : "+v"(row_pos), "+v"(row_seq)); // (no earlier: what is computed of a loaded value waits for it)
    row_page = RowsEpilogue<EPI>::ask_page(a, row_pos, row_seq);
  }
  __syncthreads();
  int buf = 0;
  const int nslices = (KS + a.kpw - 1) / a.kpw;
#pragma unroll 1
  for (int c = 0; c < nslices; ++c) {
#pragma unroll 1
    do {
      const bf16x8* xb = &xs[buf][lane];
      bf16x8 fb[2][MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) fb[0][m] = xb[(m * SUB) * 64];
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t][m] = Mma<bf16>::mma(wf[t][u], fb[u & 1][m], acc[t][m]);
          if (u + 1 < SUB) fb[(u + 1) & 1][m] = xb[(m * SUB + u + 1) * 64];
        }
        load_w(u, next + u);
      }
      store_x(buf ^ 1);
      ksb = next;
      next = min(next + SUB, end_next);
      end_next = (next < end_next) ? end_next : min(KS, end_next + a.kpw);
      load_x(next, end_next - next);
      order_pass();
      __syncthreads();
      buf ^= 1;
    } while (ksb < end);
    end = min(KS, end + a.kpw);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m) { tot[t][m] += acc[t][m]; acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  }
  // slices beyond K are empty in gemm_kernel too: it adds their zeros
  if (nslices < a.nchunk) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m) tot[t][m] += f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- epilogue: all its loads leave together ----
  if (EPI == EPI_QKV && threadIdx.x < MT * 16) {
    pos_s[threadIdx.x % (MT * 16)] = row_pos;
    row_s[threadIdx.x % (MT * 16)] = (int)RowsEpilogue<EPI>::cache_row(a, row_pos, row_page);
  }
  if (EPI == EPI_LOGITS && threadIdx.x < MT * 16) row_s[threadIdx.x % (MT * 16)] = a.out_row != nullptr ? row_out : bm * MT * 16 + (int)threadIdx.x;
  if (normed) {
    if (wave < MT) SlabRms::finish(a, rms.q, lane, rs_s + wave * 16);
    if (TWO && wave + NWV < MT) SlabRms::finish(a, q2, lane, rs_s + (wave + NWV) * 16);
  }
  if (normed || EPI == EPI_QKV || EPI == EPI_LOGITS) __syncthreads();
  const int j = lane & 15, kq = lane >> 4;
  TileIn ti[NT_OUT];
  float4 four[NT_OUT][MT];
#pragma unroll
  for (int t = 0; t < NT_OUT; ++t) {
    const int n0 = min(tile0 + t, ntiles - 1) * 16 + kq * 4;
    ti[t] = RowsEpilogue<EPI>::ask_tile(a, n0);
#pragma unroll
    for (int m = 0; m < MT; ++m)
      four[t][m] = RowsEpilogue<EPI>::ask_four(a, min((bm * MT + m) * 16 + j, a.rows - 1), n0, EPI == EPI_QKV ? pos_s[(m * 16 + j) % (EPI == EPI_QKV ? MT * 16 : 1)] : 0);
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (bm * MT + m >= slabs) break;                 // uniform
    RowIn in{1.0f, 0, 0u, 0};
    if (normed) in.r1 = rs_s[m * 16 + j];
    if (EPI == EPI_QKV) { in.pos = pos_s[(m * 16 + j) % (EPI == EPI_QKV ? MT * 16 : 1)]; in.kvrow = (unsigned)row_s[(m * 16 + j) % (EPI == EPI_QKV ? MT * 16 : 1)]; }
    if (EPI == EPI_LOGITS) in.orow = row_s[(m * 16 + j) % (EPI == EPI_LOGITS ? MT * 16 : 1)];
#pragma unroll
    for (int t = 0; t < NT_OUT; ++t)
      if (tile0 + t < ntiles) {                      // uniform
        if (EPI == EPI_GATED) RowsEpilogue<EPI>::tile_out(a, bm * MT + m, lane, tile0 + t, bz, tot[(2 * t) % NT][m], tot[(2 * t + 1) % NT][m], in, ti[t], four[t][m]);
        else RowsEpilogue<EPI>::tile_out(a, bm * MT + m, lane, tile0 + t, bz, tot[t % NT][m], tot[t % NT][m], in, ti[t], four[t][m]);
      }
  }
}

// The same product where that shape would leave most of the chip idle or walk a long K with few
// wavefronts: a workgroup is gemm_kernel's S wavefronts, each with its K-slice, over NT weight tiles x MT
// slabs.  Nothing is shared inside the workgroup, so both operands go straight into registers, D
// k-steps ahead, and there is no barrier before the slices are added through LDS, in order.  Launches of
// this kind are bound by latency (a few microseconds in all), then by what a CU can pull from L2: NT + MT
// KB for NT * MT MFMAs.
// D: kpw is a multiple of it, or the k-steps past a slice's end are multiplied with zeros.
// dynamic LDS: S * NT * MT KB + MT * 64 bytes.
// The smaller shapes get 128 registers, two workgroups of eight wavefronts a CU, but for three that need 130 and 132 and would keep
// one or two in scratch (us a draft step of 32 rows, 128 / what they need: four layers of 512, LM head of 4096 85.6 / 85.1; of 1024
// 102.3 / 101.9; of 768, 8192 139.0 / 138.5; two layers of 1024, QKV of 2048 over 64 rows 66.8 / 66.0).
template <int EPI, int NT, int MT, int D>
constexpr bool slices_fit_128() {
  if (NT == 1 && MT == 2 && D == 4) return EPI != EPI_QKV && EPI != EPI_LOGITS;
  if (NT + MT == 4 && D == 3) return EPI != EPI_LOGITS;
  return NT + MT <= 3;
}
template <int EPI, int NT, int MT, int D, bool ONCE>
static __global__ __launch_bounds__(512, (slices_fit_128<EPI, NT, MT, D>() ? 4 : 2)) void gemm_slices_kernel(const RowsGemmArgs a) {
  extern __shared__ float lds[];
  f32x4* part = reinterpret_cast<f32x4*>(lds);       // [S][NT][MT][64 lanes]
  constexpr int NT_OUT = (EPI == EPI_GATED) ? NT / 2 : NT;
  const int lane = threadIdx.x & 63, S = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KS = a.K >> 5, ntiles = a.N >> 4, slabs = (a.rows + 15) >> 4;
  int bm, bn, bz;
  rows_tile_of_block(a, bm, bn, bz);
  const int tile0 = bn * NT_OUT;
  const int ks0 = min(KS, wave * a.kpw), ks1 = min(KS, ks0 + a.kpw), ks_last = max(ks1 - 1, 0);
  const bf16x8 *wb[NT], *xb[MT], *zeros = reinterpret_cast<const bf16x8*>(a.zeros);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bf16* w = (EPI == EPI_GATED && (t & 1)) ? a.W2 : a.W + (EPI == EPI_STORE ? (size_t)(bz >> 1) * a.w_layer + (size_t)(bz & 1) * a.w_which : 0);
    wb[t] = reinterpret_cast<const bf16x8*>(w) + (size_t)min(tile0 + ((EPI == EPI_GATED) ? (t >> 1) : t), ntiles - 1) * KS * 64;
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) xb[m] = reinterpret_cast<const bf16x8*>(a.X) + (size_t)min(bm * MT + m, slabs - 1) * KS * 64;
  bf16x8 wf[D][NT], xf[D][MT];
  auto load = [&](int u, int ks) {
    const size_t o = (size_t)min(ks, ks_last) * 64;
#pragma unroll
    for (int t = 0; t < NT; ++t) wf[u][t] = load_weight<ONCE>(wb[t] + o + (unsigned)lane);
#pragma unroll
    for (int m = 0; m < MT; ++m) xf[u][m] = (ks < ks1 ? xb[m] + o : zeros)[(unsigned)lane];
  };
  f32x4 acc[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int u) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t][m] = Mma<bf16>::mma(wf[u][t], xf[u][m], acc[t][m]);
  };
  float* rs_s = lds + (size_t)S * NT * MT * 256;     // [MT][16]
  // what the epilogue reads leaves around the stream's first loads: first the row's position, behind them what depends on it.
  // (tile, slab) pairs, slab fastest, pair i by wavefront i % S: the first of this wavefront's (the others ask for theirs later)
  using Epi = RowsEpilogue<EPI>;
  const int j = lane & 15, kq = lane >> 4;
  const int m1 = wave % MT, t1 = wave / MT, n1 = min(tile0 + min(t1, NT_OUT - 1), ntiles - 1) * 16 + kq * 4;
  const int row1 = (bm * MT + m1) * 16 + j, row1c = min(row1, a.rows - 1);
  int pos1 = Epi::ask_pos(a, row1c), seq1 = Epi::ask_seq(a, row1c);
  const int orow1 = Epi::ask_orow(a, row1c);
  const bool normed = a.ss_in != nullptr;            // (uniform)
  SlabRms rms;
  if (normed && wave < MT) rms.load(a, min(bm * MT + wave, slabs - 1), lane);
#pragma unroll
  for (int u = 0; u < D; ++u) load(u, ks0 + u);
  __builtin_amdgcn_sched_barrier(0);
  if (normed && wave < MT) rms.sums(a, min(bm * MT + wave, slabs - 1), lane);            // (S >= MT)
  if (EPI == EPI_QKV) asm volatile("" : "+v"(pos1), "+v"(seq1));      // (no earlier: what is computed of a loaded value waits for it)
  const int page1 = Epi::ask_page(a, pos1, seq1);
  const TileIn ti1 = Epi::ask_tile(a, n1);
  const float4 four1 = Epi::ask_four(a, row1c, n1, pos1);
  const int blocks = (a.kpw + D - 1) / D;
#pragma unroll 1
  for (int b = 1; b < blocks; ++b) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      multiply(u);
      load(u, ks0 + b * D + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < D; ++u) multiply(u);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) part[((wave * NT + t) * MT + m) * 64 + lane] = acc[t][m];
  if (normed && wave < MT) SlabRms::finish(a, rms.q, lane, rs_s + wave * 16);
  __syncthreads();
  for (int i = wave; i < NT_OUT * MT; i += S) {
    const int t = i / MT, m = i % MT;
    if (bm * MT + m >= slabs || tile0 + t >= ntiles) continue;                 // uniform
    RowIn in{normed ? rs_s[m * 16 + j] : 1.0f, pos1, 0u, a.out_row != nullptr ? orow1 : row1};
    TileIn ti = ti1;
    float4 four = four1;
    int page = page1;
    if (i != wave) {                                 // (uniform)
      const int row = (bm * MT + m) * 16 + j, rowc = min(row, a.rows - 1), n0 = (tile0 + t) * 16 + kq * 4;
      if (m != m1) {
        in.pos = Epi::ask_pos(a, rowc);
        page = Epi::ask_page(a, in.pos, Epi::ask_seq(a, rowc));
        in.orow = a.out_row != nullptr ? Epi::ask_orow(a, rowc) : row;
      }
      ti = Epi::ask_tile(a, n0);
      four = Epi::ask_four(a, rowc, n0, in.pos);
    }
    if (EPI == EPI_QKV) in.kvrow = Epi::cache_row(a, in.pos, page);
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    auto add = [&](auto waves) {                     // (their number at compile time: all reads in flight)
      constexpr int W = decltype(waves)::value;
#pragma unroll
      for (int st = 0; st < ((EPI == EPI_GATED) ? 2 : 1); ++st) {
        const int tt = (EPI == EPI_GATED) ? 2 * t + st : t;
        f32x4 v[W];
#pragma unroll
        for (int w = 0; w < W; ++w) v[w] = part[((w * NT + tt) * MT + m) * 64 + lane];
#pragma unroll
        for (int w = 0; w < W; ++w) s[st] += v[w];
      }
    };
    if (S == 8) add(std::integral_constant<int, 8>());
    else add(std::integral_constant<int, 4>());
    Epi::tile_out(a, bm * MT + m, lane, tile0 + t, bz, s[0], s[1], in, ti, four);
  }
}

}  // namespace sd
