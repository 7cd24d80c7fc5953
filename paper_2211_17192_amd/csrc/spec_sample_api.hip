// C-ABI entry points of the stand-alone accept / resample kernel (the second
// half of Algorithm 1 on explicit logits).  See include/sd.h.
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <string>
#include "../../include/sd.h"
#include "kernels_misc.h"
#include "kernels_sample.h"

extern "C" size_t sd_spec_sample_scratch_bytes(int32_t rows, int32_t gamma) {
  if (rows < 1 || gamma < 1 || gamma > SD_MAX_GAMMA) return 0;
  return (size_t)rows * sizeof(sd::SampleBlock);
}

namespace {
// Argument checks shared by the entry points; fills the resolved options.
struct SampleOpts { float len; double log_len; int top_k; float top_p; };
sd_status check_sample_args(const float* p_logits, const float* q_logits, const int32_t* x, const float* r,
                            const float* s, int32_t rows, int32_t gamma, int32_t vocab, float temperature,
                            const sd_sampling* opt, const int32_t* out_n, const int32_t* out_t, SampleOpts& o) {
  if (!p_logits || !q_logits || !x || !out_n || !out_t) return SD_EINVAL;
  if (rows < 1 || rows > 65535 || gamma < 1 || gamma > SD_MAX_GAMMA || vocab < 1 ||
      vocab > sd::SAMPLE_CHUNK * sd::SAMPLE_MAX_CHUNKS) return SD_EINVAL;
  if (!(temperature >= 0.0f)) return SD_EINVAL;
  if (temperature > 0.0f && (!r || !s)) return SD_EINVAL;
  o.len = opt ? opt->lenience : 1.0f;
  if (!(o.len > 0.0f && o.len <= 1.0f)) return SD_EINVAL;
  o.log_len = std::log((double)o.len);
  o.top_k = opt ? opt->top_k : 0;
  o.top_p = opt ? opt->top_p : 0.0f;
  if (o.top_k < 0 || !(o.top_p >= 0.0f && o.top_p <= 1.0f)) return SD_EINVAL;
  if ((o.top_k > 0 || (o.top_p > 0.0f && o.top_p < 1.0f)) &&
      (vocab > sd::SAMPLE_REG_F4 * 4 * sd::SAMPLE_THREADS || (vocab & 3) ||
       (reinterpret_cast<uintptr_t>(p_logits) & 15) || (reinterpret_cast<uintptr_t>(q_logits) & 15)))
    return SD_EINVAL;                            // the filters run on rows held in registers
  return SD_OK;
}

static_assert(SD_MAX_GAMMA == sd::SAMPLE_MAX_GAMMA, "the sampling kernels' scratch holds SD_MAX_GAMMA guesses");

// The launches of one call; scr: one block per row, its ticket zero before the call and after it.
sd_status launch_spec_sample(const float* p_logits, const float* q_logits, const int32_t* x, const float* r,
                             const float* s, int32_t rows, int32_t gamma, int32_t vocab, float temperature,
                             const SampleOpts& o, int32_t* out_n, int32_t* out_t, float* beta,
                             sd::SampleBlock* scr, hipStream_t s_) {
  sd::AcceptArgs a{};
  a.p = p_logits; a.q = q_logits; a.x = x; a.r = r; a.s = s; a.gamma = gamma; a.V = vocab; a.temperature = temperature;
  a.lenience = o.len; a.log_lenience = o.log_len;
  if (temperature > 0.0f) { a.top_k = o.top_k; a.top_p = o.top_p; }            // (argmax sampling ignores the filters)
  a.scr = scr; a.scr_stride = sizeof(sd::SampleBlock);
  a.part = &scr->part[0][0]; a.part_row = sd::SAMPLE_PARTS; a.part_seq = sizeof(sd::SampleBlock) / sizeof(sd::RowPart);
  a.out_n = out_n; a.out_t = out_t; a.beta = beta;
  sd::launch_accept(s_, a, rows, 256);   // (every gfx950 device has 256 CUs)
  return hipGetLastError() == hipSuccess ? SD_OK : SD_EHIP;
}
}  // namespace

extern "C" sd_status sd_spec_sample_ex(const float* p_logits, const float* q_logits, const int32_t* x,
                                       const float* r, const float* s, int32_t rows, int32_t gamma,
                                       int32_t vocab, float temperature, const sd_sampling* opt,
                                       int32_t* out_n, int32_t* out_t, float* beta, void* scratch, void* stream) {
  if (!scratch) return SD_EINVAL;
  SampleOpts o{};
  const sd_status st = check_sample_args(p_logits, q_logits, x, r, s, rows, gamma, vocab, temperature, opt, out_n, out_t, o);
  if (st != SD_OK) return st;
  return launch_spec_sample(p_logits, q_logits, x, r, s, rows, gamma, vocab, temperature, o, out_n, out_t, beta,
                            static_cast<sd::SampleBlock*>(scratch), static_cast<hipStream_t>(stream));
}

extern "C" sd_status sd_spec_sample(const float* p_logits, const float* q_logits, const int32_t* x,
                                    const float* r, const float* s, int32_t rows, int32_t gamma,
                                    int32_t vocab, float temperature, int32_t* out_n,
                                    int32_t* out_t, void* scratch, void* stream) {
  return sd_spec_sample_ex(p_logits, q_logits, x, r, s, rows, gamma, vocab, temperature, nullptr, out_n, out_t,
                           nullptr, scratch, stream);
}

// ---------------------------------------------------------------------------
// The same call for callers that cannot allocate: its scratch (tickets and row
// statistics) is a fixed array in device memory that belongs to the library.
// Every GPU the library runs on holds its own copy at its own address; host code
// must not hand the array's name to a kernel, it asks the runtime for the address
// once per device and uses that pointer from then on.
// ---------------------------------------------------------------------------
namespace {
constexpr int STATIC_ROWS = SD_SPEC_SAMPLE_STATIC_MAX_ROWS;
static __device__ __align__(256) unsigned char scratch[STATIC_ROWS * sizeof(sd::SampleBlock)];   // 10 MB
static_assert(sizeof(sd::SampleBlock) % sizeof(sd::RowPart) == 0, "the blocks keep their alignment, and a whole number of RowParts lies between two");

constexpr int STATIC_MAX_DEVICES = 64;
void* g_scratch_ptr[STATIC_MAX_DEVICES] = {};    // device address of `scratch` on each device, once known
std::mutex g_scratch_mutex;

// The address of this device's copy of `scratch` (nullptr + *err on failure).
void* static_scratch_address(hipError_t* err) {
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) { *err = hipErrorInvalidDevice; return nullptr; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    *err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (*err != hipSuccess || ptr == nullptr) { if (*err == hipSuccess) *err = hipErrorInvalidSymbol; return nullptr; }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" sd_status sd_spec_sample_static(const float* p_logits, const float* q_logits, const int32_t* x,
                                           const float* r, const float* s, int32_t rows, int32_t gamma,
                                           int32_t vocab, float temperature, const sd_sampling* opt,
                                           int32_t* out_n, int32_t* out_t, float* beta, void* stream) {
  SampleOpts o{};
  const sd_status st = check_sample_args(p_logits, q_logits, x, r, s, rows, gamma, vocab, temperature, opt, out_n, out_t, o);
  if (st != SD_OK) return st;
  if (rows > STATIC_ROWS) {
    g_load_error = "sd_spec_sample_static takes at most " + std::to_string(STATIC_ROWS) + " rows per call (got " +
                   std::to_string(rows) + "): split the call, or use sd_spec_sample_ex with a scratch buffer of your own";
    return SD_ERANGE;
  }
  hipError_t e = hipSuccess;
  void* ptr = static_scratch_address(&e);
  if (ptr == nullptr) {
    g_load_error = std::string("sd_spec_sample_static: address of the scratch array: ") + hipGetErrorString(e);
    return SD_EHIP;
  }
  hipStream_t s_ = static_cast<hipStream_t>(stream);
  // the tickets must start at zero whatever an earlier (possibly failed) call left: a small kernel,
  // not a memset, so that the call can be recorded into a graph
  sd::SampleBlock* scr = static_cast<sd::SampleBlock*>(ptr);
  hipLaunchKernelGGL(sd::clear_tickets_kernel, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, s_, scr, sizeof(sd::SampleBlock), rows, 1);
  return launch_spec_sample(p_logits, q_logits, x, r, s, rows, gamma, vocab, temperature, o, out_n, out_t, beta, scr, s_);
}
