// Runs whole passes and operators of the library without a GPU and checks where the slices of split reductions lie.
//
// The HIP calls that the library makes are defined here, so that a launch only reports its kernel and arguments.  Every
// kernel that adds slices up reads exactly what the product in front of it wrote: that range has to lie inside one buffer
// of the handle's workspace (workspace_pieces()).  And every update, which runs over quads, has to start on one.
//
//   scratch_check CASES SEED LAYERS: CASES holds a line of numbers per handle (alexnet_config_t from batch to fc, then
//   precision and flags); LAYERS random layers are checked after them.
#include <cxxabi.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <random>
#include <string>

#define AX_HOST_EMU 1
#include <hip/hip_runtime.h>

#include "../../paper_1412_2302_amd/csrc/kernels.h"

using namespace ax;

namespace ax {
inline void emu_fail(const char* what) {
  fprintf(stderr, "%s\n", what);
  abort();
}
}  // namespace ax

static char* const kBase = reinterpret_cast<char*>(1ull << 40);  // workspace; nothing is ever read there
static std::vector<WorkspacePiece> g_pieces;
static std::string g_what;
static long g_ranges, g_launches, g_bad;

static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}

static void range(const std::string& kernel, const void* p, size_t floats) {
  ++g_ranges;
  const size_t at = (size_t)((const char*)p - kBase), bytes = floats * sizeof(float);
  for (const WorkspacePiece& w : g_pieces)
    if (at >= w.offset && at + bytes <= w.offset + w.bytes) return;
  if (++g_bad > 20) return;
  printf("%s: %s reads %zu bytes of slices at %zu, which lie in no buffer", g_what.c_str(), kernel.c_str(), bytes, at);
  for (const WorkspacePiece& w : g_pieces)
    if (at >= w.offset && at < w.offset + w.bytes) printf(" (%zu left in the one they start in)", w.offset + w.bytes - at);
  printf("\n");
}

// kernels that read and write four floats at a time from these pointers on
static void quads(const std::string& kernel, const void* w, const void* v, const void* g) {
  if (((uintptr_t)w | (uintptr_t)v | (uintptr_t)g) % 16 == 0) return;
  if (++g_bad > 20) return;
  printf("%s: %s takes quads from %p, %p, %p on\n", g_what.c_str(), kernel.c_str(), w, v, g);
}

template <class T>
static T arg(void** args, int i) {
  return *static_cast<T*>(args[i]);
}
static void launched(const std::string& k, void** a) {
  ++g_launches;
  auto is = [&k](const char* name) { return k.compare(0, strlen(name), name) == 0; };
  if (is("ax::slab_finish_kernel("))  // ws, slices, groups, M, N
    range(k, arg<float*>(a, 0), (size_t)arg<int>(a, 1) * arg<int>(a, 2) * arg<long>(a, 3) * arg<int>(a, 4));
  else if (is("ax::fc_fwd_finish_kernel("))  // ws, slices, rows, columns
    range(k, arg<float*>(a, 0), (size_t)arg<int>(a, 1) * arg<int>(a, 2) * arg<int>(a, 3));
  else if (is("ax::fc_bwd_finish_kernel("))  // ws, slices, elements
    range(k, arg<float*>(a, 0), (size_t)arg<int>(a, 1) * arg<size_t>(a, 2));
  else if (is("ax::reduce_slabs_kernel(") || is("ax::reduce_slabs_vec_kernel("))  // ws, slices, slab, groups
    range(k, arg<float*>(a, 0), (size_t)arg<int>(a, 1) * arg<size_t>(a, 2) * arg<int>(a, 3));
  else if (is("ax::reduce_slabs_unpack_kernel("))  // ws, slices, slab
    range(k, arg<float*>(a, 0), (size_t)arg<int>(a, 1) * arg<size_t>(a, 2));
  else if (is("ax::sgd_update_kernel("))
    quads(k, arg<float*>(a, 0), arg<float*>(a, 1), arg<float*>(a, 2));
  else if (is("ax::reduce_slabs_batch_kernel(")) {
    const WgradTail& t = *static_cast<WgradTail*>(a[0]);
    for (int i = 0; i < t.n; ++i)
      if (t.job[i].nsplit > 1) range(k, t.job[i].slices, (size_t)t.job[i].groups36 * t.job[i].nsplit * t.job[i].slab);
  }
  if (is("ax::sgd_colsum_batch_stage2(")) {
    const SgdArgs& u = *static_cast<SgdArgs*>(a[1]);
    quads(k, u.w, u.v, u.g);
  }
  if (k.find("colsum_batch_stage2(") != std::string::npos) {
    const ColsumBatch& b = *static_cast<ColsumBatch*>(a[0]);
    for (int i = 0; i < b.n; ++i) range(k, b.job[i].part, (size_t)b.job[i].nparts * b.job[i].cols);
  }
}

// ---- the HIP calls of the library ----
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
} g_call;
extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int rc = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &rc);
  std::string s = rc == 0 ? d : name;
  if (s.compare(0, 5, "void ") == 0) s = s.substr(5);
  names()[fn] = s;
  free(d);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  g_call = {grid, block, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_call.grid;
  *block = g_call.block;
  *lds = g_call.lds;
  *st = g_call.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void** args, size_t, hipStream_t) {
  launched(names()[fn], args);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(8); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
}

static int fail(const char* call, int rc) {
  printf("%s: %s returned %d (%s)\n", g_what.c_str(), call, rc, alexnet_last_error());
  return 1;
}
#define DO(call)                                   \
  do {                                             \
    const int rc_ = (call);                        \
    if (rc_ != ALEXNET_OK) return fail(#call, rc_); \
  } while (0)

// every pass and operator of a handle; 0 also for a configuration that the library refuses
static int check(const alexnet_config_t& c) {
  size_t n_params = 0, bytes = 0;
  if (alexnet_query(&c, &n_params, &bytes) != ALEXNET_OK) return 0;
  g_pieces.clear();
  DO(workspace_pieces(&c, &g_pieces));
  float* const outside = reinterpret_cast<float*>(1ull << 45);  // the caller's tensors
  float* const p = outside + (1ull << 32);
  alexnet_t* n = nullptr;
  DO(alexnet_create(&c, p, p + (1ull << 32), kBase, bytes, nullptr, &n));
  const int32_t* labels = reinterpret_cast<const int32_t*>(outside);
  DO(alexnet_train_step(n, 0, labels, 1, outside, nullptr));
  DO(alexnet_forward_backward(n, 1, labels, 1, outside, nullptr));
  DO(alexnet_forward(n, outside, outside, nullptr));
  for (int l = 1; l <= 5; ++l) {
    DO(alexnet_conv_forward(n, l, outside, outside, outside, 1, outside, nullptr));
    DO(alexnet_conv_backward_data(n, l, outside, outside, outside, nullptr));
    DO(alexnet_conv_backward_weight(n, l, outside, outside, outside, outside, nullptr));
    DO(alexnet_conv_forward_nhwc(n, l, outside + 1, outside + 1, outside, 0, outside, nullptr));
    DO(alexnet_conv_backward_weight_nhwc(n, l, outside + 1, outside + 1, outside, outside, nullptr));
    DO(alexnet_conv_backward_data_nhwc(n, l, outside + 1, outside + 1, outside + 1, outside, nullptr));
  }
  for (int l = 6; l <= 8; ++l) {
    DO(alexnet_fc_forward(n, l, outside, outside, outside, 1, outside, nullptr));
    DO(alexnet_fc_backward(n, l, outside, outside, outside, outside, outside, outside, nullptr));
  }
  alexnet_destroy(n);
  return 0;
}

static alexnet_config_t defaults() {
  alexnet_config_t c;
  memset(&c, 0, sizeof c);
  c.lrn_n = 5;
  c.lrn_k = 2.f;
  c.lrn_alpha = 1e-4f;
  c.lrn_beta = 0.75f;
  c.dropout_p = 0.5f;
  return c;
}
static void describe(const alexnet_config_t& c) {
  char b[400];
  int k = snprintf(b, sizeof b, "batch %d, %d x %d x %d, precision %d, flags %d:", c.batch, c.in_c, c.crop_h, c.crop_w,
                   c.precision, c.flags);
  for (const alexnet_conv_t& v : c.conv)
    k += snprintf(b + k, sizeof b - k, " (%d,%d,%d,%d,%d,%d,%d)", v.cout, v.k, v.stride, v.pad, v.groups, v.lrn, v.pool);
  snprintf(b + k, sizeof b - k, " %d %d %d", c.fc[0], c.fc[1], c.fc[2]);
  g_what = b;
}

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  long handles = 0;
  FILE* f = fopen(argv[1], "r");
  if (!f) return 2;
  alexnet_config_t c = defaults();
  auto read = [f](int32_t* v) { return fscanf(f, "%d", v) == 1; };
  while (read(&c.batch)) {
    bool ok = read(&c.in_c) && read(&c.crop_h) && read(&c.crop_w) && read(&c.raw_h) && read(&c.raw_w);
    for (alexnet_conv_t& v : c.conv)
      ok = ok && read(&v.cout) && read(&v.k) && read(&v.stride) && read(&v.pad) && read(&v.groups) && read(&v.lrn) && read(&v.pool);
    for (int32_t& v : c.fc) ok = ok && read(&v);
    if (!ok || !read(&c.precision) || !read(&c.flags)) return 2;
    describe(c);
    if (check(c)) return 1;
    ++handles;
  }
  fclose(f);
  // a layer of any kind as the second one, behind a pointwise layer that makes its channels
  std::mt19937 rng((unsigned)atoi(argv[2]));
  auto pick = [&rng](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  for (int i = 0; i < atoi(argv[3]); ++i) {
    c = defaults();
    const int groups = 1 << pick(0, 2), step = pick(0, 2) ? 8 : pick(1, 4);
    const int cin = groups * step * pick(1, 24), side = pick(5, 32), k = pick(1, 7);
    c.batch = 1 << pick(0, 9);
    c.batch += pick(0, c.batch - 1);
    c.in_c = pick(0, 2) ? 3 : 8;
    c.crop_h = c.crop_w = c.raw_h = c.raw_w = side;
    c.conv[0] = {cin, pick(0, 1) ? 1 : 3, 1, 0, 1, 0, 0};
    c.conv[1] = {groups * step * pick(1, 24), k, pick(0, 3) ? 1 : 2, pick(0, k - 1), groups, pick(0, 1), 0};
    for (int j = 2; j < 5; ++j) c.conv[j] = {8, 3, 4, 1, 1, 0, 0};
    c.fc[0] = pick(1, 40) * 8;
    c.fc[1] = pick(1, 300);
    c.fc[2] = pick(1, 40) * 8;
    c.precision = pick(0, 2) ? ALEXNET_PRECISION_BF16 : ALEXNET_PRECISION_FP32;
    describe(c);
    if (check(c)) return 1;
    ++handles;
  }
  printf("%ld handles, %ld launches, %ld ranges, %ld outside\n", handles, g_launches, g_ranges, g_bad);
  return g_bad ? 1 : 0;
}
