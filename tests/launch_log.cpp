// Drives libsd.so without a GPU: the HIP entry points that the library calls are defined here and write what they are asked for
// to stdout, one line each, instead of doing it.  Reads the pair and the calls from stdin (test_launches.py writes them):
//   model <arch> <layers> <d_model> <heads> <kv_heads> <d_head> <d_ff> <vocab> <max_len> <enc_len> <dtype>   the target, then the draft
//   tensor <name> <rows> <columns or 0>                                                                   of the model above
//   load <batch> <max_gamma> <flags> <caller's stream: 0 / 1> <workspace: 0 = all, 1 = the least that loads>
//   prefill <row> <tokens> | step <gamma> <temperature> | plain <temperature> | measure | time <which> <rows> | filter
//   sample <rows> <gamma> <vocab> <beta: 0 / 1>                                        (needs no pair)
// Lines: "launch <stream> <kernel> <grid x> <y> <z> [notes]", "copy <stream>", "begin" .. "end" (a graph's launches), "graph <stream>",
// "sync <stream>", "record <stream>", "call <line> -> <status>".  Streams: 0 the caller's, 1, 2, .. as they were created.
// Kernels do not run: device memory is never touched, and sd_step finds its states unchanged (SD_EHIP behind its launches).
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>
#include "sd.h"

struct Dim3 { uint32_t x, y, z; };
static std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> m; return m; }
static char streams[16];                             // stream i is &streams[i]
static int made = 0;
static int id(void* s) { return s == nullptr ? -1 : (int)(static_cast<char*>(s) - streams); }
struct Config { Dim3 g, b; size_t lds; void* s; };
static Config config;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels()[host] = name; }
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s) { config = {g, b, lds, s}; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s) { *g = config.g; *b = config.b; *lds = config.lds; *s = config.s; return 0; }
int hipLaunchKernel(const void* f, Dim3 g, Dim3, void** args, size_t, void* s) {
  const std::string& k = kernels()[f];
  printf("launch %d %s %u %u %u", id(s), k.c_str(), g.x, g.y, g.z);
  // embed_kernel's tenth argument: where the step's parameters come from; a draw's DrawNext begins with EmbedArgs, whose fourth
  // word is the x that the next row is embedded into
  if (k.find("embed_kernel") != std::string::npos && *static_cast<void**>(args[9])) printf(" fetches");
  const int next = k.find("sample_row_split_kernel") != std::string::npos ? 9 : k.find("sample_row_filter_kernel") != std::string::npos ? 8 : -1;
  if (next > 0 && static_cast<void**>(args[next])[3]) printf(" embeds");
  printf("\n");
  return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, void* s) { printf("copy %d\n", id(s)); return 0; }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = &streams[++made]; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void* s) { printf("sync %d\n", id(s)); return 0; }
int hipStreamBeginCapture(void*, int) { printf("begin\n"); return 0; }
int hipStreamEndCapture(void*, void** g) { static char graph; *g = &graph; printf("end\n"); return 0; }
int hipGraphInstantiate(void** e, void* g, void*, char*, size_t) { *e = g; return 0; }
int hipGraphLaunch(void*, void* s) { printf("graph %d\n", id(s)); return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipEventCreate(void** e) { static char event; *e = &event; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void* s) { printf("record %d\n", id(s)); return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
}

int main() {
  sd_model_cfg cfg[2] = {};
  std::vector<sd_tensor> tensors[2];
  std::deque<std::string> names;
  int models = 0;
  sd_ctx* c = nullptr;
  std::string line, what;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    in >> what;
    if (what == "model") {
      sd_model_cfg& m = cfg[models++];
      in >> m.arch >> m.n_layers >> m.d_model >> m.n_heads >> m.n_kv_heads >> m.d_head >> m.d_ff >> m.vocab >> m.max_len >> m.enc_len >> m.dtype;
      m.rel_buckets = 32; m.rel_max_dist = 128; m.rope_theta = 10000.0f; m.logit_scale = 1.0f; m.norm_eps = 1e-5f;
      continue;
    }
    if (what == "tensor") {
      std::string name;
      sd_tensor t = {};
      in >> name >> t.shape[0] >> t.shape[1];
      names.push_back(name);
      t.name = names.back().c_str(); t.dev = streams; t.ndim = t.shape[1] ? 2 : 1; t.dtype = cfg[models - 1].dtype;
      tensors[models - 1].push_back(t);
      continue;
    }
    int status = 0, a = 0, b = 0;
    float temperature = 1.0f;
    if (what == "load") {
      sd_runtime_cfg rt = {};
      int own = 0, least = 0;
      in >> rt.batch >> rt.max_gamma >> rt.flags >> own >> least;
      rt.page_size = 16; rt.stream = own ? streams : nullptr;
      rt.workspace = reinterpret_cast<void*>(uintptr_t(1) << 40);      // (an address for arithmetic; nothing reads it)
      rt.workspace_bytes = sd_workspace_bytes(&cfg[0], &cfg[1], &rt);
      auto load = [&] { return (int)sd_load_models(&c, &cfg[0], tensors[0].data(), (int)tensors[0].size(), &cfg[1], tensors[1].data(), (int)tensors[1].size(), &rt); };
      if (least) {
        size_t lo = 0, hi = rt.workspace_bytes;
        while (hi - lo > 256) {
          rt.workspace_bytes = lo + (hi - lo) / 2;
          if (load() == SD_OK) { sd_free(c); hi = rt.workspace_bytes; } else lo = rt.workspace_bytes;
        }
        rt.workspace_bytes = hi;
        made = 0;
      }
      printf("loaded\n");
      status = load();
    } else if (what == "prefill") {
      in >> a >> b;
      std::vector<int32_t> tokens(b, 1);
      static char enc;
      status = sd_prefill(c, a, tokens.data(), b, cfg[0].enc_len ? &enc : nullptr, cfg[1].enc_len ? &enc : nullptr);
    } else if (what == "step") {
      in >> a >> temperature;
      std::vector<float> u(64 * 31, 0.5f);
      std::vector<int32_t> out(64 * 16), n(64);
      status = sd_step(c, nullptr, 0, a, temperature, u.data(), out.data(), n.data());
    } else if (what == "plain") {
      in >> temperature;
      std::vector<float> u(64, 0.5f);
      std::vector<int32_t> out(64);
      status = sd_step_baseline(c, temperature, u.data(), out.data());
    } else if (what == "measure") {
      double q = 0, p = 0;
      status = sd_measure_cost(c, 1, &q, &p);
    } else if (what == "time") {
      double us = 0;
      in >> a >> b;
      status = sd_time_forward(c, a, b, 0, 1, &us);
    } else if (what == "filter") {
      sd_sampling opt = {1.0f, 50, 0.9f};
      status = sd_set_sampling(c, &opt);
    } else if (what == "sample") {
      int vocab = 0, beta = 0;
      in >> a >> b >> vocab >> beta;
      static float f;                                  // (addresses only)
      static int32_t n;
      status = sd_spec_sample_ex(&f, &f, &n, &f, &f, a, b, vocab, 1.0f, nullptr, &n, &n, beta ? &f : nullptr, &f, streams);
    }
    printf("call %s -> %d\n", line.c_str(), status);
    if (status != 0 && what != "step" && what != "plain") { fprintf(stderr, "%s: %s\n", line.c_str(), sd_last_error(c)); return 1; }
  }
  sd_free(c);
  return 0;
}
