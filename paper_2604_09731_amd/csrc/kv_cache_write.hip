// kv_cache_write / tree_commit: scatter token K/V rows into the paged cache.
//
// The interleaved layout groups 8 elements into one matrix-core operand vector
// (K: 8 consecutive head dims of one token; V: 8 consecutive tokens of one head
// dim), so that tree_verify_attention can load operands straight from HBM.
#include "common.h"
#include "fp8.h"

namespace {

template <typename T>
__global__ __launch_bounds__(256) void kv_cache_write_kernel(
    int layout, int n_tokens, int Hkv, int D, int block_size, int num_blocks,
    const T* __restrict__ k_src, const T* __restrict__ v_src,
    const int64_t* __restrict__ slot_mapping, T* __restrict__ k_cache, T* __restrict__ v_cache,
    int64_t block_stride, int64_t head_stride, int64_t token_stride) {
  const int t = blockIdx.x;
  if (t >= n_tokens) return;
  const int64_t slot_id = slot_mapping[t];
  if (slot_id < 0 || slot_id >= (int64_t)num_blocks * block_size) return;
  const int64_t blk = slot_id / block_size;
  const int slot = (int)(slot_id % block_size);
  for (int e = threadIdx.x; e < Hkv * D; e += blockDim.x) {
    const int g = e / D, d = e % D;
    const int64_t page = blk * block_stride + (int64_t)g * head_stride;
    int64_t ko, vo;
    if (layout == SMART_KV_PLAIN) {
      ko = vo = page + (int64_t)slot * token_stride + d;
    } else {
      ko = page + ((int64_t)(d / 8) * block_size + slot) * 8 + d % 8;
      vo = page + ((int64_t)(slot / 8) * D + d) * 8 + slot % 8;
    }
    k_cache[ko] = k_src[(size_t)t * Hkv * D + e];
    v_cache[vo] = v_src[(size_t)t * Hkv * D + e];
  }
}

// The same scatter into an fp8 cache: element = E4M3(source / scale).
__device__ inline float src_to_float(float x) { return x; }
__device__ inline float src_to_float(uint16_t x) { return __uint_as_float(((uint32_t)x) << 16); }

template <typename T>
__global__ __launch_bounds__(256) void kv_cache_write_fp8_kernel(
    int layout, int n_tokens, int Hkv, int D, int block_size, int num_blocks,
    const T* __restrict__ k_src, const T* __restrict__ v_src,
    const int64_t* __restrict__ slot_mapping, uint8_t* __restrict__ k_cache, uint8_t* __restrict__ v_cache,
    int64_t block_stride, int64_t head_stride, int64_t token_stride, float k_scale, float v_scale) {
  const int t = blockIdx.x;
  if (t >= n_tokens) return;
  const int64_t slot_id = slot_mapping[t];
  if (slot_id < 0 || slot_id >= (int64_t)num_blocks * block_size) return;
  const int64_t blk = slot_id / block_size;
  const int slot = (int)(slot_id % block_size);
  for (int e = threadIdx.x; e < Hkv * D; e += blockDim.x) {
    const int g = e / D, d = e % D;
    const int64_t page = blk * block_stride + (int64_t)g * head_stride;
    int64_t ko, vo;
    if (layout == SMART_KV_PLAIN) {
      ko = vo = page + (int64_t)slot * token_stride + d;
    } else {
      ko = page + ((int64_t)(d / 8) * block_size + slot) * 8 + d % 8;
      vo = page + ((int64_t)(slot / 8) * D + d) * 8 + slot % 8;
    }
    k_cache[ko] = smart::float_to_fp8_e4m3(src_to_float(k_src[(size_t)t * Hkv * D + e]) / k_scale);
    v_cache[vo] = smart::float_to_fp8_e4m3(src_to_float(v_src[(size_t)t * Hkv * D + e]) / v_scale);
  }
}

// ---- rows moved in 8-element chunks ------------------------------------------------------------------------------
// Bound by memory: every row is read once and written once.  What the element-wise kernels above spend their time on is
// V's 2-byte stores at a stride of 16 bytes and an integer division per element.  With enough tokens (rows_pay, below) a
// thread moves 8 elements of K at a time (16 bytes of bf16, contiguous in both layouts), and where eight consecutive tokens
// fill a whole slot group
// (slots 8 s .. 8 s + 7 of a block, what every prompt longer than a few tokens consists of) V is transposed in registers:
// a thread reads two head dims of the eight tokens and stores two whole 8-slot vectors.  A workgroup takes eight tokens.
// 8190 tokens of 8 x 128 bf16 (67 MB moved), interleaved: 42.7 -> 17.8 us.
constexpr int kRowsPerWg = 8;
constexpr int kThreads = 256;

template <typename T> struct Elems8 { T v[8]; };
template <typename T> struct alignas(2 * sizeof(T)) Elems2 { T v[2]; };
template <typename T> struct alignas(4 * sizeof(T)) Elems4 { T v[4]; };

template <typename T>
__device__ inline Elems8<T> load8(const T* p) {
  Elems8<T> r;
  if constexpr (sizeof(T) == 2) {
    *reinterpret_cast<uint4*>(r.v) = *reinterpret_cast<const uint4*>(p);
  } else {
    *reinterpret_cast<uint4*>(r.v) = *reinterpret_cast<const uint4*>(p);
    *reinterpret_cast<uint4*>(r.v + 4) = *reinterpret_cast<const uint4*>(p + 4);
  }
  return r;
}
__device__ inline void store8(uint16_t* p, const Elems8<uint16_t>& x) { *reinterpret_cast<uint4*>(p) = *reinterpret_cast<const uint4*>(x.v); }
__device__ inline void store8(uint8_t* p, const Elems8<uint8_t>& x) { *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(x.v); }
__device__ inline void store8(float* p, const Elems8<float>& x) {
  *reinterpret_cast<uint4*>(p) = *reinterpret_cast<const uint4*>(x.v);
  *reinterpret_cast<uint4*>(p + 4) = *reinterpret_cast<const uint4*>(x.v + 4);
}
template <typename C, typename T>
__device__ inline C cache_elem(T x, float scale) {  // C: the cache's element type (T, or uint8_t = E4M3 of source / scale)
  if constexpr (sizeof(C) == 1) return smart::float_to_fp8_e4m3(src_to_float(x) / scale);
  else return x;
}
template <typename C, typename T>
__device__ inline Elems8<C> cache_elems(const Elems8<T>& x, float scale) {
  Elems8<C> r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r.v[i] = cache_elem<C>(x.v[i], scale);
  return r;
}

template <typename T, typename C, bool kInterleaved>
__global__ __launch_bounds__(kThreads) void kv_cache_write_rows_kernel(
    int n_tokens, int Hkv, int D, int block_size, int num_blocks, const T* __restrict__ k_src,
    const T* __restrict__ v_src, const int64_t* __restrict__ slot_mapping, C* __restrict__ k_cache,
    C* __restrict__ v_cache, int64_t block_stride, int64_t head_stride, int64_t token_stride, float k_scale,
    float v_scale) {
  const int t0 = blockIdx.x * kRowsPerWg;
  const int lane = threadIdx.x & 63;
  // Lane i holds the slot of token t0 - 7 + i (lanes 0 .. 21): the eight tokens of this workgroup, seven before (a group
  // they belong to may begin there) and seven after (a group that begins here may end there).  -1: no such token, or
  // one that is skipped.
  const int t = t0 - 7 + lane;
  int64_t slot = -1;
  if (lane < 22 && t >= 0 && t < n_tokens) slot = slot_mapping[t];
  if (slot < 0 || slot >= (int64_t)num_blocks * block_size) slot = -1;
  const int64_t after = __shfl_down(slot, 1);
  const uint64_t next = __ballot(lane < 21 && slot >= 0 && after == slot + 1);  // the next token has the next slot
  uint64_t whole = 0;  // tokens at which a whole group begins (groups are disjoint: each begins at a multiple of 8)
  if (kInterleaved) whole = __ballot(lane < 15 && slot >= 0 && (slot & 7) == 0 && ((next >> lane) & 0x7Full) == 0x7Full);
  uint64_t member = whole;
  member |= member << 1;
  member |= member << 2;
  member |= member << 4;  // a group's eight tokens
  const uint32_t block = slot >= 0 ? (uint32_t)((uint64_t)slot / (uint32_t)block_size) : 0u;
  const int in_block = slot >= 0 ? (int)(slot - (int64_t)block * block_size) : -1;
  // Token i of the eight: its slot and block, from the lane that holds them.  Every lane of the wavefront has to take part
  // (a lane that has left a loop need not keep its registers), so the loops below end for whole wavefronts.
  auto slot_of = [&](int i) { return __builtin_amdgcn_readlane(in_block, 7 + i); };
  auto block_of = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane(block, 7 + i); };
  const int first = threadIdx.x & ~63;
  const int E = Hkv * D, chunks = E / 8;

  // K (and V of plain pages, or of tokens outside whole groups): four tokens of one chunk per thread and turn
  for (int u0 = first; u0 < 2 * chunks; u0 += kThreads) {
    const bool mine = u0 + lane < 2 * chunks;
    const int u = min(u0 + lane, 2 * chunks - 1);  // (loaded again, never stored)
    const int half = u >= chunks ? 1 : 0, c = u - half * chunks;
    const int g = c / (D / 8), d8 = c - g * (D / 8);
    const int64_t head = (int64_t)g * head_stride;
    Elems8<T> kx[4], vx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tok = min(t0 + 4 * half + i, n_tokens - 1);  // (a token past the end is read again, never stored)
      kx[i] = load8(k_src + (int64_t)tok * E + 8 * c);
      if (!kInterleaved) vx[i] = load8(v_src + (int64_t)tok * E + 8 * c);
    }
    int s_of[4];
    uint32_t b_of[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s0 = slot_of(i), s1 = slot_of(4 + i);
      const uint32_t b0 = block_of(i), b1 = block_of(4 + i);
      s_of[i] = half ? s1 : s0;
      b_of[i] = half ? b1 : b0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = s_of[i];
      if (s < 0 || !mine) continue;
      const int64_t page = (int64_t)b_of[i] * block_stride + head;
      if (kInterleaved) {
        store8(k_cache + page + (d8 * block_size + s) * 8, cache_elems<C>(kx[i], k_scale));
      } else {
        const int64_t at = page + (int64_t)s * token_stride + 8 * d8;
        store8(k_cache + at, cache_elems<C>(kx[i], k_scale));
        store8(v_cache + at, cache_elems<C>(vx[i], v_scale));
      }
    }
  }
  if (!kInterleaved) return;

  // V of the whole group that begins in this workgroup's tokens (at most one does)
  const uint64_t mine = (whole >> 7) & 0xFFull;
  if (mine) {
    const int lead = __ffsll((unsigned long long)mine) - 1;
    const int s = __builtin_amdgcn_readlane(in_block, 7 + lead);
    const int64_t page = (int64_t)(uint32_t)__builtin_amdgcn_readlane(block, 7 + lead) * block_stride;
    for (int u = threadIdx.x; u < E / 2; u += kThreads) {
      const int g = u / (D / 2), d = 2 * (u - g * (D / 2));
      Elems2<T> x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        x[i] = *reinterpret_cast<const Elems2<T>*>(v_src + (int64_t)(t0 + lead + i) * E + 2 * u);
      C* dst = v_cache + page + (int64_t)g * head_stride + ((s >> 3) * D + d) * 8;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        Elems8<C> y;
#pragma unroll
        for (int i = 0; i < 8; ++i) y.v[i] = cache_elem<C>(x[i].v[j], v_scale);
        store8(dst + 8 * j, y);
      }
    }
  }
  // V of tokens outside whole groups: a prompt's ragged end, single tokens
  const uint32_t single = (uint32_t)((__ballot(slot >= 0) & ~member) >> 7) & 0xFFu;
  if (single == 0) return;
  for (int e0 = first; e0 < E; e0 += kThreads) {
    const int e = min(e0 + lane, E - 1), g = e / D, d = e - g * D;
    T x[kRowsPerWg];  // (all eight requested at once; a token past the end is read again, never stored)
#pragma unroll
    for (int i = 0; i < kRowsPerWg; ++i) x[i] = v_src[(int64_t)min(t0 + i, n_tokens - 1) * E + e];
#pragma unroll
    for (int i = 0; i < kRowsPerWg; ++i) {
      if (((single >> i) & 1u) == 0) continue;  // (the same for all lanes)
      const int s = slot_of(i);
      const int64_t page = (int64_t)block_of(i) * block_stride;
      if (e0 + lane < E)
        v_cache[page + (int64_t)g * head_stride + ((int64_t)(s >> 3) * D + d) * 8 + (s & 7)] = cache_elem<C>(x[i], v_scale);
    }
  }
}

// Whether every chunk of the call can be moved with one aligned access per side (offsets inside a page are 32-bit there).
static bool rows_in_chunks(bool fp8, int kv_layout, int head_dim, int block_size, const void* k_src, const void* v_src,
                           const void* k_cache, const void* v_cache, int64_t block_stride, int64_t head_stride,
                           int64_t token_stride) {
  const uintptr_t cache_align = fp8 ? 8 : 16;
  auto aligned = [](const void* p, uintptr_t n) { return ((uintptr_t)p & (n - 1)) == 0; };
  return head_dim % 8 == 0 && (int64_t)head_dim * block_size < (1 << 30) && block_stride % 8 == 0 && head_stride % 8 == 0 &&
         (kv_layout == SMART_KV_INTERLEAVED || token_stride % 8 == 0) && aligned(k_src, 16) && aligned(v_src, 16) &&
         aligned(k_cache, cache_align) && aligned(v_cache, cache_align);
}

// Whether the chunk kernel is the faster one (start to end on the device, 6 prompts, chunk kernel against element-wise kernel).
// Its threads do more one after the other, so it needs enough tokens to fill the chip:
//   interleaved, 8 x 128 bf16: 400 tokens 6.7 us against 5.1, 800 6.3 / 6.9, 3200 9.9 / 19.1, 12800 25 / 66 (fp32 9.1 / 6.2,
//   8.5 / 9.4, 17 / 29, 44 / 107); 2 x 64 bf16: 1200 3.6 / 3.5, 1600 3.7 / 3.9, 12800 5.4 / 12.2.
//   Into fp8 the conversions bound both: 8 x 128 3200 17.2-19.2 / 17.4-17.7, 6400 25-27 / 28-31, 12800 32-39 / 50-55; 2 x 64
//   6400 9.5 / 8.3, 12800 10.9 / 12.9.
//   Plain pages need no transposing; 16-byte stores gain only for bf16: 8 x 128 at any size (4 tokens 2.6 / 2.9, 12800 16.8 /
//   23.5), narrower rows from 2^18 elements on (2 x 64: 1600 tokens 2.8 / 2.9, 800 2.7 / 2.6); fp32 34 / 33, fp8 no gain.
static bool rows_pay(bool f32, bool fp8, int kv_layout, int64_t n_tokens, int64_t row) {
  if (kv_layout == SMART_KV_PLAIN) return !f32 && !fp8 && (row >= 1024 || n_tokens * row >= (1 << 18));
  if (fp8) return n_tokens >= (row >= 512 ? 6400 : 12800);
  return n_tokens >= (row >= 512 ? 800 : 1600);
}

template <typename T, typename C, bool kInterleaved>
static void launch_rows(hipStream_t s, int n_tokens, int Hkv, int D, int block_size, int num_blocks, const void* k_src,
                        const void* v_src, const int64_t* slots, void* k_cache, void* v_cache, int64_t block_stride,
                        int64_t head_stride, int64_t token_stride, float k_scale, float v_scale) {
  const dim3 grid((unsigned)(((int64_t)n_tokens + kRowsPerWg - 1) / kRowsPerWg));
  hipLaunchKernelGGL((kv_cache_write_rows_kernel<T, C, kInterleaved>), grid, dim3(kThreads), 0, s, n_tokens, Hkv, D,
                     block_size, num_blocks, (const T*)k_src, (const T*)v_src, slots, (C*)k_cache, (C*)v_cache,
                     block_stride, head_stride, token_stride, k_scale, v_scale);
}

// One workgroup per (path index i, sequence b).  Every wavefront takes the same accept / refuse decision from the same
// inputs (a lane per path entry: two memory round trips per 64 entries); workgroup i = 0 reports it.
// kChunks: rows move in 8-element chunks (V of interleaved pages: four elements read at once, stored one by one); see
// commit_in_chunks.  Four sequences, 8 kv heads of 128, max_depth 8, interleaved bf16: 4.0 us with a serial check of the
// path, 3.6 with this one by element, 3.4 in chunks (start to end on the device).
template <typename T, typename C, bool kChunks>
__global__ __launch_bounds__(256) void tree_commit_kernel(
    int layout, int batch, int max_depth, int Hkv, int D, int block_size, int max_blocks, int num_blocks,
    const int32_t* __restrict__ cu_nodes, const int32_t* __restrict__ accept_len,
    const int32_t* __restrict__ accept_path, const T* __restrict__ k_tree, const T* __restrict__ v_tree,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ prefix_len,
    C* __restrict__ k_cache, C* __restrict__ v_cache, int64_t block_stride, int64_t head_stride,
    int64_t token_stride, int32_t* __restrict__ new_prefix_len, int32_t* __restrict__ status,
    float k_scale, float v_scale) {
  const int i = blockIdx.x, b = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int base = cu_nodes[b];
  const int n = cu_nodes[b + 1] - base;
  const int a = accept_len[b];
  const int start = prefix_len[b];
  const int32_t* path = accept_path + (size_t)b * (max_depth + 1);
  int verdict = SMART_OK, node = 0, block = 0;  // node, block: of path entry i
  if (base < 0 || a < 0 || a > max_depth) {
    verdict = SMART_ETREE;
  } else if (start < 0 || (int64_t)start + a + 1 > (int64_t)max_blocks * block_size) {
    verdict = SMART_ECAP;
  } else {
    for (int k0 = 0; k0 <= a; k0 += 64) {  // at most max_depth + 1 <= 129 entries
      const int k = min(k0 + lane, a);
      const int v = path[k];
      const int blk = block_table[(size_t)b * max_blocks + (start + k) / block_size];
      if (__any(v < 0 || v >= n || blk < 0 || blk >= num_blocks)) verdict = SMART_ETREE;
      if (i >= k0 && i < k0 + 64) {
        node = __builtin_amdgcn_readlane(v, i - k0);
        block = __builtin_amdgcn_readlane(blk, i - k0);
      }
    }
  }
  if (i == 0 && threadIdx.x == 0) {
    status[b] = verdict;
    new_prefix_len[b] = verdict == SMART_OK ? start + a + 1 : start;
  }
  if (verdict != SMART_OK || i > a) return;
  const int slot = (start + i) % block_size;
  const int64_t block_at = (int64_t)block * block_stride;
  const size_t src = (size_t)(base + node) * Hkv * D;
  if (kChunks) {
    const int chunks = Hkv * D / 8;
    const bool plain = layout == SMART_KV_PLAIN;
    // the first `chunks` units move K (and V of plain pages), the rest four elements of an interleaved V each
    for (int u = threadIdx.x; u < (plain ? chunks : 3 * chunks); u += 256) {
      if (u < chunks) {
        const int g = u / (D / 8), d8 = u - g * (D / 8);
        const int64_t page = block_at + (int64_t)g * head_stride;
        const Elems8<T> kx = load8(k_tree + src + 8 * u);
        if (plain) {
          const int64_t at = page + (int64_t)slot * token_stride + 8 * d8;
          const Elems8<T> vx = load8(v_tree + src + 8 * u);
          store8(k_cache + at, cache_elems<C>(kx, k_scale));
          store8(v_cache + at, cache_elems<C>(vx, v_scale));
        } else {
          store8(k_cache + page + ((int64_t)d8 * block_size + slot) * 8, cache_elems<C>(kx, k_scale));
        }
      } else {
        const int e = 4 * (u - chunks), g = e / D, d = e - g * D;
        const Elems4<T> vx = *reinterpret_cast<const Elems4<T>*>(v_tree + src + e);
        C* dst = v_cache + block_at + (int64_t)g * head_stride + ((int64_t)(slot / 8) * D + d) * 8 + slot % 8;
#pragma unroll
        for (int x = 0; x < 4; ++x) dst[8 * x] = cache_elem<C>(vx.v[x], v_scale);
      }
    }
    return;
  }
  for (int e = threadIdx.x; e < Hkv * D; e += blockDim.x) {
    const int g = e / D, d = e % D;
    const int64_t page = block_at + (int64_t)g * head_stride;
    int64_t ko, vo;
    if (layout == SMART_KV_PLAIN) {
      ko = vo = page + (int64_t)slot * token_stride + d;
    } else {
      ko = page + ((int64_t)(d / 8) * block_size + slot) * 8 + d % 8;
      vo = page + ((int64_t)(slot / 8) * D + d) * 8 + slot % 8;
    }
    k_cache[ko] = cache_elem<C>(k_tree[src + e], k_scale);
    v_cache[vo] = cache_elem<C>(v_tree[src + e], v_scale);
  }
}

}  // namespace

// Whether chunks are the faster way (start to end on the device, paths of 5 entries, chunks against elements).
//   Into fp8 a thread converts eight elements in a row, so rows have to occupy the workgroup: 8 x 128, 1 .. 128 sequences,
//   4.2 .. 8.0 us against 4.5 .. 8.3; 4 x 128 plain 4.2 .. 5.4 against 3.5 .. 4.5, interleaved equal; 2 x 64 4.1 .. 5.5 against
//   2.9 .. 3.9.
//   Plain pages: 8 x 128 2.7 .. 4.2 against 3.2 .. 4.7, 4 x 128 2.7 .. 3.7 against 2.8 .. 3.9; 4 x 64 and 2 x 64 2.6 .. 3.7 against
//   2.6 .. 3.6.
//   Interleaved pages: 8 x 128 up to 8 sequences 3.3 .. 3.7 against 3.5 .. 3.8, 16 equal, 32 5.0 .. 5.2 against 4.8 .. 4.9, 128 bf16
//   11.0 against 9.0; 4 x 128 2.9 .. 3.2 against 3.0 .. 3.2, 16 equal, 128 6.1 .. 7.7 against 5.2 .. 7.1; 4 x 64 and 2 x 64
//   2.8 .. 4.9 against 2.7 .. 4.6.
static bool commit_in_chunks(bool fp8, int kv_layout, int64_t batch, int64_t row) {
  if (fp8) return row >= 1024;
  return row >= 512 && (kv_layout == SMART_KV_PLAIN || batch <= 16);
}

static int32_t commit_impl(smart_ctx* ctx, void* stream, int32_t dtype, bool fp8, int32_t kv_layout,
                           int32_t batch, int32_t max_depth, int32_t num_kv_heads, int32_t head_dim,
                           int32_t block_size, int32_t max_blocks_per_seq, int32_t num_blocks,
                           const int32_t* d_cu_nodes, const int32_t* d_accept_len,
                           const int32_t* d_accept_path, const void* d_k_tree, const void* d_v_tree,
                           const int32_t* d_block_table, const int32_t* d_prefix_len,
                           void* d_k_cache, void* d_v_cache, int64_t cache_block_stride,
                           int64_t cache_head_stride, int64_t cache_token_stride,
                           int32_t* d_new_prefix_len, int32_t* d_status, float k_scale, float v_scale) {
  if (!ctx || batch < 0 || max_depth < 0 || max_depth > SMART_MAX_NODES || num_kv_heads <= 0 ||
      head_dim <= 0 || block_size <= 0 || max_blocks_per_seq < 0 || num_blocks < 0)
    return SMART_EINVAL;
  if (dtype != SMART_F32 && dtype != SMART_BF16) return SMART_EINVAL;
  if (kv_layout != SMART_KV_PLAIN && kv_layout != SMART_KV_INTERLEAVED) return SMART_EINVAL;
  if (kv_layout == SMART_KV_INTERLEAVED && (block_size % 8 != 0 || head_dim % 8 != 0))
    return SMART_EINVAL;
  if (fp8 && (!(k_scale > 0.f) || !(k_scale < 3e38f) || !(v_scale > 0.f) || !(v_scale < 3e38f))) return SMART_EINVAL;
  const int64_t page = (int64_t)block_size * head_dim;
  if (kv_layout == SMART_KV_PLAIN && cache_token_stride < head_dim) return SMART_EINVAL;
  if (cache_head_stride < (kv_layout == SMART_KV_PLAIN ? (block_size - 1) * cache_token_stride + head_dim : page))
    return SMART_EINVAL;
  if (cache_block_stride < cache_head_stride) return SMART_EINVAL;
  if (batch == 0) return SMART_OK;
  if (batch > 65535) return SMART_EINVAL;  // grid y
  if (!d_cu_nodes || !d_accept_len || !d_accept_path || !d_k_tree || !d_v_tree || !d_block_table ||
      !d_prefix_len || !d_k_cache || !d_v_cache || !d_new_prefix_len || !d_status ||
      d_new_prefix_len == d_prefix_len)
    return SMART_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid(max_depth + 1, batch);
  const bool chunks = commit_in_chunks(fp8, kv_layout, batch, (int64_t)num_kv_heads * head_dim) &&
                      rows_in_chunks(fp8, kv_layout, head_dim, block_size, d_k_tree, d_v_tree, d_k_cache, d_v_cache,
                                     cache_block_stride, cache_head_stride, cache_token_stride);
#define SMART_LAUNCH_COMMIT_AS(T, C, CHUNKS)                                                                    \
  hipLaunchKernelGGL((tree_commit_kernel<T, C, CHUNKS>), grid, dim3(256), 0, s, kv_layout, batch, max_depth,   \
                     num_kv_heads, head_dim, block_size, max_blocks_per_seq, num_blocks, d_cu_nodes,           \
                     d_accept_len, d_accept_path, (const T*)d_k_tree, (const T*)d_v_tree, d_block_table,       \
                     d_prefix_len, (C*)d_k_cache, (C*)d_v_cache, cache_block_stride, cache_head_stride,        \
                     cache_token_stride, d_new_prefix_len, d_status, k_scale, v_scale)
#define SMART_LAUNCH_COMMIT(T, C)                                                                               \
  do {                                                                                                          \
    if (chunks) SMART_LAUNCH_COMMIT_AS(T, C, true);                                                             \
    else SMART_LAUNCH_COMMIT_AS(T, C, false);                                                                   \
  } while (0)
  if (dtype == SMART_F32) {
    if (fp8) SMART_LAUNCH_COMMIT(float, uint8_t); else SMART_LAUNCH_COMMIT(float, float);
  } else {
    if (fp8) SMART_LAUNCH_COMMIT(uint16_t, uint8_t); else SMART_LAUNCH_COMMIT(uint16_t, uint16_t);
  }
#undef SMART_LAUNCH_COMMIT_AS
#undef SMART_LAUNCH_COMMIT
  SMART_HIP_CHECK(hipGetLastError());
  return SMART_OK;
}

extern "C" int32_t tree_commit(smart_ctx* ctx, void* stream, int32_t dtype, int32_t kv_layout,
                               int32_t batch, int32_t max_depth, int32_t num_kv_heads, int32_t head_dim,
                               int32_t block_size, int32_t max_blocks_per_seq, int32_t num_blocks,
                               const int32_t* d_cu_nodes, const int32_t* d_accept_len,
                               const int32_t* d_accept_path, const void* d_k_tree, const void* d_v_tree,
                               const int32_t* d_block_table, const int32_t* d_prefix_len,
                               void* d_k_cache, void* d_v_cache, int64_t cache_block_stride,
                               int64_t cache_head_stride, int64_t cache_token_stride,
                               int32_t* d_new_prefix_len, int32_t* d_status) {
  return commit_impl(ctx, stream, dtype, false, kv_layout, batch, max_depth, num_kv_heads, head_dim, block_size,
                     max_blocks_per_seq, num_blocks, d_cu_nodes, d_accept_len, d_accept_path, d_k_tree, d_v_tree,
                     d_block_table, d_prefix_len, d_k_cache, d_v_cache, cache_block_stride, cache_head_stride,
                     cache_token_stride, d_new_prefix_len, d_status, 1.f, 1.f);
}

extern "C" int32_t tree_commit_fp8(smart_ctx* ctx, void* stream, int32_t src_dtype, int32_t kv_layout,
                                   int32_t batch, int32_t max_depth, int32_t num_kv_heads, int32_t head_dim,
                                   int32_t block_size, int32_t max_blocks_per_seq, int32_t num_blocks,
                                   const int32_t* d_cu_nodes, const int32_t* d_accept_len,
                                   const int32_t* d_accept_path, const void* d_k_tree, const void* d_v_tree,
                                   const int32_t* d_block_table, const int32_t* d_prefix_len,
                                   void* d_k_cache, void* d_v_cache, int64_t cache_block_stride,
                                   int64_t cache_head_stride, int64_t cache_token_stride,
                                   int32_t* d_new_prefix_len, int32_t* d_status, float k_scale, float v_scale) {
  return commit_impl(ctx, stream, src_dtype, true, kv_layout, batch, max_depth, num_kv_heads, head_dim, block_size,
                     max_blocks_per_seq, num_blocks, d_cu_nodes, d_accept_len, d_accept_path, d_k_tree, d_v_tree,
                     d_block_table, d_prefix_len, d_k_cache, d_v_cache, cache_block_stride, cache_head_stride,
                     cache_token_stride, d_new_prefix_len, d_status, k_scale, v_scale);
}

extern "C" int32_t kv_cache_write(smart_ctx* ctx, void* stream, int32_t dtype, int32_t kv_layout,
                                  int32_t n_tokens, int32_t num_kv_heads, int32_t head_dim,
                                  int32_t block_size, int32_t num_blocks, const void* d_k_src,
                                  const void* d_v_src, const int64_t* d_slot_mapping,
                                  void* d_k_cache, void* d_v_cache, int64_t cache_block_stride,
                                  int64_t cache_head_stride, int64_t cache_token_stride) {
  if (!ctx || n_tokens < 0 || num_kv_heads <= 0 || head_dim <= 0 || block_size <= 0 ||
      num_blocks < 0)
    return SMART_EINVAL;
  if (dtype != SMART_F32 && dtype != SMART_BF16) return SMART_EINVAL;
  if (kv_layout != SMART_KV_PLAIN && kv_layout != SMART_KV_INTERLEAVED) return SMART_EINVAL;
  if (kv_layout == SMART_KV_INTERLEAVED && (block_size % 8 != 0 || head_dim % 8 != 0))
    return SMART_EINVAL;
  const int64_t page = (int64_t)block_size * head_dim;
  if (kv_layout == SMART_KV_PLAIN && cache_token_stride < head_dim) return SMART_EINVAL;
  if (cache_head_stride < (kv_layout == SMART_KV_PLAIN ? (block_size - 1) * cache_token_stride + head_dim : page))
    return SMART_EINVAL;
  if (cache_block_stride < cache_head_stride) return SMART_EINVAL;
  if (n_tokens == 0) return SMART_OK;
  if (!d_k_src || !d_v_src || !d_slot_mapping || !d_k_cache || !d_v_cache) return SMART_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (rows_pay(dtype == SMART_F32, false, kv_layout, n_tokens, (int64_t)num_kv_heads * head_dim) &&
      rows_in_chunks(false, kv_layout, head_dim, block_size, d_k_src, d_v_src, d_k_cache, d_v_cache, cache_block_stride,
                     cache_head_stride, cache_token_stride)) {
    auto launch = kv_layout == SMART_KV_PLAIN ? launch_rows<uint16_t, uint16_t, false>
                  : dtype == SMART_F32        ? launch_rows<float, float, true>
                                              : launch_rows<uint16_t, uint16_t, true>;
    launch(s, n_tokens, num_kv_heads, head_dim, block_size, num_blocks, d_k_src, d_v_src, d_slot_mapping,
           d_k_cache, d_v_cache, cache_block_stride, cache_head_stride, cache_token_stride, 1.f, 1.f);
    SMART_HIP_CHECK(hipGetLastError());
    return SMART_OK;
  }
  if (dtype == SMART_F32)
    hipLaunchKernelGGL(kv_cache_write_kernel<float>, dim3(n_tokens), dim3(256), 0, s, kv_layout,
                       n_tokens, num_kv_heads, head_dim, block_size, num_blocks,
                       (const float*)d_k_src, (const float*)d_v_src, d_slot_mapping,
                       (float*)d_k_cache, (float*)d_v_cache, cache_block_stride,
                       cache_head_stride, cache_token_stride);
  else
    hipLaunchKernelGGL(kv_cache_write_kernel<uint16_t>, dim3(n_tokens), dim3(256), 0, s, kv_layout,
                       n_tokens, num_kv_heads, head_dim, block_size, num_blocks,
                       (const uint16_t*)d_k_src, (const uint16_t*)d_v_src, d_slot_mapping,
                       (uint16_t*)d_k_cache, (uint16_t*)d_v_cache, cache_block_stride,
                       cache_head_stride, cache_token_stride);
  SMART_HIP_CHECK(hipGetLastError());
  return SMART_OK;
}

extern "C" int32_t kv_cache_write_fp8(smart_ctx* ctx, void* stream, int32_t src_dtype, int32_t kv_layout,
                                      int32_t n_tokens, int32_t num_kv_heads, int32_t head_dim,
                                      int32_t block_size, int32_t num_blocks, const void* d_k_src,
                                      const void* d_v_src, const int64_t* d_slot_mapping, void* d_k_cache,
                                      void* d_v_cache, int64_t cache_block_stride, int64_t cache_head_stride,
                                      int64_t cache_token_stride, float k_scale, float v_scale) {
  if (!ctx || n_tokens < 0 || num_kv_heads <= 0 || head_dim <= 0 || block_size <= 0 || num_blocks < 0)
    return SMART_EINVAL;
  if (src_dtype != SMART_F32 && src_dtype != SMART_BF16) return SMART_EINVAL;
  if (kv_layout != SMART_KV_PLAIN && kv_layout != SMART_KV_INTERLEAVED) return SMART_EINVAL;
  if (kv_layout == SMART_KV_INTERLEAVED && (block_size % 8 != 0 || head_dim % 8 != 0)) return SMART_EINVAL;
  if (!(k_scale > 0.f) || !(k_scale < 3e38f) || !(v_scale > 0.f) || !(v_scale < 3e38f)) return SMART_EINVAL;
  const int64_t page = (int64_t)block_size * head_dim;
  if (kv_layout == SMART_KV_PLAIN && cache_token_stride < head_dim) return SMART_EINVAL;
  if (cache_head_stride < (kv_layout == SMART_KV_PLAIN ? (block_size - 1) * cache_token_stride + head_dim : page))
    return SMART_EINVAL;
  if (cache_block_stride < cache_head_stride) return SMART_EINVAL;
  if (n_tokens == 0) return SMART_OK;
  if (!d_k_src || !d_v_src || !d_slot_mapping || !d_k_cache || !d_v_cache) return SMART_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (rows_pay(src_dtype == SMART_F32, true, kv_layout, n_tokens, (int64_t)num_kv_heads * head_dim) &&
      rows_in_chunks(true, kv_layout, head_dim, block_size, d_k_src, d_v_src, d_k_cache, d_v_cache, cache_block_stride,
                     cache_head_stride, cache_token_stride)) {
    auto launch = src_dtype == SMART_F32 ? launch_rows<float, uint8_t, true> : launch_rows<uint16_t, uint8_t, true>;
    launch(s, n_tokens, num_kv_heads, head_dim, block_size, num_blocks, d_k_src, d_v_src, d_slot_mapping,
           d_k_cache, d_v_cache, cache_block_stride, cache_head_stride, cache_token_stride, k_scale, v_scale);
    SMART_HIP_CHECK(hipGetLastError());
    return SMART_OK;
  }
  if (src_dtype == SMART_F32)
    hipLaunchKernelGGL(kv_cache_write_fp8_kernel<float>, dim3(n_tokens), dim3(256), 0, s, kv_layout, n_tokens,
                       num_kv_heads, head_dim, block_size, num_blocks, (const float*)d_k_src, (const float*)d_v_src,
                       d_slot_mapping, (uint8_t*)d_k_cache, (uint8_t*)d_v_cache, cache_block_stride,
                       cache_head_stride, cache_token_stride, k_scale, v_scale);
  else
    hipLaunchKernelGGL(kv_cache_write_fp8_kernel<uint16_t>, dim3(n_tokens), dim3(256), 0, s, kv_layout, n_tokens,
                       num_kv_heads, head_dim, block_size, num_blocks, (const uint16_t*)d_k_src,
                       (const uint16_t*)d_v_src, d_slot_mapping, (uint8_t*)d_k_cache, (uint8_t*)d_v_cache,
                       cache_block_stride, cache_head_stride, cache_token_stride, k_scale, v_scale);
  SMART_HIP_CHECK(hipGetLastError());
  return SMART_OK;
}
