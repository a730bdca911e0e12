// The library's host code on a machine without a GPU: the HIP calls it makes are defined here (an executable's symbols
// come before those of the HIP runtime), so that the test sees every allocation and launch and decides what fails.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <tuple>

#include "smart_tree.h"

static int mallocs, frees, launches;
static size_t allocated, refuse_from = (size_t)-1;
static bool capturing;  // of a stream other than the default one
static hipError_t sync_result = hipSuccess, malloc_result = hipErrorOutOfMemory;

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return hipErrorInvalidSymbol; }
hipError_t hipMalloc(void** p, size_t n) {
  ++mallocs;
  if (n >= refuse_from) return malloc_result;
  allocated += n;
  *p = malloc(64);
  return hipSuccess;
}
hipError_t hipFree(void* p) { ++frees; free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return sync_result; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { ++launches; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = dim3(1); *b = dim3(1); *m = 0; *s = nullptr;
  return hipSuccess;
}
}

static char* somewhere() { static char x[4096]; return (char*)(((uintptr_t)x + 255) & ~(uintptr_t)255); }

// One attention call; the launches it made (2: with partial results, 1: the workspace-free form), or its error.
static int call(smart_ctx* ctx, int batch, int nodes, int hq, int hkv, bool interleaved = false) {
  tva_params p;
  memset(&p, 0, sizeof p);
  p.dtype = SMART_BF16;
  p.kv_layout = interleaved ? SMART_KV_INTERLEAVED : SMART_KV_PLAIN;
  p.batch = batch; p.total_nodes = nodes; p.num_q_heads = hq; p.num_kv_heads = hkv; p.head_dim = 128;
  p.block_size = 16; p.max_blocks_per_seq = 1000; p.num_blocks = 1000;
  p.softmax_scale = 0.1f;
  p.cache_token_stride = 128; p.cache_head_stride = 16 * 128; p.cache_block_stride = 16 * 128 * (int64_t)hkv;
  void* x = somewhere();
  p.d_q = p.d_k_tree = p.d_v_tree = p.d_k_cache = p.d_v_cache = x;
  p.d_out = x;
  p.d_block_table = p.d_prefix_len = p.d_cu_nodes = (const int32_t*)x;
  p.d_anc_mask = (const uint64_t*)x;
  launches = 0;
  const int32_t rc = tree_verify_attention(ctx, capturing ? x : nullptr, &p);
  return rc == SMART_OK ? launches : rc;
}

static int failures;
#define EXPECT(x)                                                  \
  do {                                                             \
    if (!(x)) { printf("line %d: %s\n", __LINE__, #x); ++failures; } \
  } while (0)

int main() {
  smart_ctx* ctx = nullptr;
  // a reservation holds for every call inside it, also with head counts that divide otherwise, and holds one buffer
  for (int hq : {1, 3, 30, 32}) for (int hkv : {1, 3, 4}) if (hq % hkv == 0) {
    EXPECT(smart_create(&ctx, 0) == SMART_OK);
    mallocs = 0;
    EXPECT(smart_reserve(ctx, 4, 48, 32, 4) == SMART_OK);
    EXPECT(mallocs == 2);  // partial results, plan
    EXPECT(call(ctx, 4, 48, hq, hkv) == 2);
    EXPECT(call(ctx, 1, 16, hq, hkv) == 2);
    EXPECT(call(ctx, 4, 48, hq, hkv, true) == 2);
    EXPECT(mallocs == 2);
    EXPECT(smart_destroy(ctx) == SMART_OK);
  }
  // 64 sequences of 64 nodes, 64 / 8 heads: no more than the interleaved kernel's own partial results
  EXPECT(smart_create(&ctx, 0) == SMART_OK);
  allocated = 0;
  EXPECT(call(ctx, 64, 4096, 64, 8, true) == 2);
  const size_t interleaved_alone = allocated;
  EXPECT(smart_reserve(ctx, 64, 4096, 64, 8) == SMART_OK);
  EXPECT(allocated == interleaved_alone);
  EXPECT(smart_destroy(ctx) == SMART_OK);
  // no memory: the workspace-free form, asked for once, until a smaller call or a reservation
  EXPECT(smart_create(&ctx, 0) == SMART_OK);
  mallocs = 0;
  refuse_from = 1 << 20;
  for (int i = 0; i < 3; ++i) EXPECT(call(ctx, 4, 48, 32, 4) == 1);
  EXPECT(mallocs == 1);
  EXPECT(call(ctx, 8, 96, 32, 4) == 1);
  EXPECT(mallocs == 1);
  EXPECT(call(ctx, 1, 1, 32, 4) == 1);
  EXPECT(mallocs == 2);
  EXPECT(smart_reserve(ctx, 4, 48, 32, 4) == SMART_ENOMEM);
  refuse_from = (size_t)-1;
  EXPECT(call(ctx, 4, 48, 32, 4) == 2);
  // a failed wait is an error of an earlier call and reported, not a lack of memory
  sync_result = hipErrorLaunchFailure;
  EXPECT(call(ctx, 64, 4096, 32, 4) == SMART_EHIP);
  EXPECT(smart_last_hip_error() == hipErrorLaunchFailure);
  sync_result = hipSuccess;
  EXPECT(call(ctx, 64, 4096, 32, 4) == 2);
  malloc_result = hipErrorUnknown;
  refuse_from = 0;
  EXPECT(call(ctx, 128, 8192, 32, 4) == SMART_EHIP);
  EXPECT(call(ctx, 64, 4096, 32, 4) == 2);
  EXPECT(smart_destroy(ctx) == SMART_OK);
  // more arrival counters, but no larger partial results or plan: what a captured launch of an earlier call holds stays
  refuse_from = (size_t)-1;
  EXPECT(smart_create(&ctx, 0) == SMART_OK);
  EXPECT(call(ctx, 4, 512, 128, 2, true) > 0);
  mallocs = frees = 0;
  for (int hkv = 32; hkv <= 40; hkv += 2) EXPECT(call(ctx, 4, 4, hkv, hkv, true) > 0);
  EXPECT(frees == 0 && mallocs == 1);  // (a block at least twice the last holds the next ones too)
  EXPECT(call(ctx, 4, 512, 128, 2, true) == 2);
  EXPECT(frees == 0 && mallocs == 1);
  EXPECT(smart_destroy(ctx) == SMART_OK);
  EXPECT(frees == 3);  // partial results, plan, counters
  // as many partial results of the two-launch form, more of the finishing form: what a captured launch holds stays
  EXPECT(smart_create(&ctx, 0) == SMART_OK);
  EXPECT(call(ctx, 4, 128, 64, 1, true) > 0);
  frees = 0;
  EXPECT(call(ctx, 4, 448, 12, 3, true) > 0);
  EXPECT(frees == 0);
  EXPECT(smart_destroy(ctx) == SMART_OK);
  // under capture nothing can be allocated: a call that is short of counters only takes two launches, which need none
  // (nodes of the call before it; this call's heads; whether it takes one launch elsewhere)
  for (const auto& [nodes, hkv, one_launch] : {std::tuple{128, 5, false}, {512, 20, true}}) {
    EXPECT(smart_create(&ctx, 0) == SMART_OK);
    EXPECT(call(ctx, 4, nodes, 64, 1, true) > 0);
    mallocs = 0;
    capturing = true;
    sync_result = hipErrorStreamCaptureUnsupported;
    EXPECT(call(ctx, 4, 20, hkv, hkv, true) == 2);
    EXPECT(mallocs == 0);
    capturing = false;
    sync_result = hipSuccess;
    EXPECT(call(ctx, 4, 20, hkv, hkv, true) > 0);
    EXPECT(call(ctx, 4, 20, hkv, hkv, true) == (one_launch ? 1 : 2));
    EXPECT(mallocs == 1);
    EXPECT(smart_destroy(ctx) == SMART_OK);
  }
  // trees of a mean of at most four nodes take two launches under this table, but not if segments are many
  EXPECT(smart_create(&ctx, 0) == SMART_OK);
  EXPECT(smart_reserve(ctx, 17, 64, 64, 64) == SMART_OK);
  EXPECT(call(ctx, 4, 16, 20, 20, true) == 2);
  EXPECT(call(ctx, 4, 17, 20, 20, true) == 1);
  EXPECT(call(ctx, 4, 4, 32, 32, true) == 2);
  EXPECT(call(ctx, 4, 4, 33, 33, true) == 1);
  EXPECT(smart_destroy(ctx) == SMART_OK);
  puts(failures ? "failed" : "workspace driver ok");
  return failures != 0;
}
