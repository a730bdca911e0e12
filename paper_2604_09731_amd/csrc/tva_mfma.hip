// tree_verify_attention, matrix-core path for bf16, head_dim 128, block_size 16,
// interleaved cache layout (gfx950 / CDNA4).
//
// The work splits in two, following where the bytes are:
//
//  * the cached prefix (thousands of keys per sequence, no mask) is a dense
//    contraction.  A 64-lane wavefront streams 32-key tiles of one
//    (sequence, kv head) and multiplies them against all rows of that kv head
//    at once -- rows = tree nodes x query heads of the GQA group -- so every
//    K/V byte leaves HBM once.  K and V vectors are loaded from HBM directly
//    in v_mfma_f32_32x32x16_bf16 operand layout (that is what the interleaved
//    cache layout is for), scores are kept transposed (keys x rows) so that a
//    row's softmax reduction stays inside a lane, and the probabilities come
//    out of the first product already in the operand layout of the second.
//    The key range of the whole batch is cut into equal shares, one per
//    worker, independent of sequence boundaries, so ragged prefix lengths do
//    not unbalance the machine; each (worker, segment) pair leaves an
//    unnormalised partial (max, sum, O).  Sequences fall in three classes by
//    their rows per kv head (<= 32, <= 64, more); ONE kernel launch serves all
//    three, its workgroups dealt to the classes in proportion to their work:
//    class 0 streams K/V from HBM straight into operand registers (eight
//    wavefronts share a worker's tiles); classes 1 and 2 stage tiles in LDS
//    (HBM -> LDS without passing through registers) for the eight wavefronts
//    of a workgroup: two row tiles x two key groups in class 1, eight row
//    tiles of 32 rows each in class 2.
//
//  * the tree part (a node sees only itself and its ancestors: a handful of
//    keys selected by a 128-bit mask) is sparse and tiny.  In the usual form of
//    the launch (kFinish) the prefix kernel evaluates it as one to four more
//    tiles of masked keys, merges the pieces of a segment and writes the rows:
//    one launch.  Where few segments are cut into many pieces, the prefix
//    kernel leaves its partials and a combine kernel, spread over the whole
//    chip, walks the set bits of each row's mask on the vector ALUs and merges:
//    see finishes().
//
// The paper (Sec. 1) only says that the tree is verified in one forward pass
// of the target model; this file is the attention sub-step of that pass.
#include <hip/hip_ext.h>
#include <math.h>

#include "common.h"
#include "tva_plan.h"
#include "wave.h"

// The timeline build (-DSMART_TVA_TIMELINE, a library of its own: libsmart_tree_timeline.so, read by
// python -m paper_2604_09731_amd.timeline) keeps wall-clock stamps (100 MHz counter) of the LAST launch: per
// workgroup of the prefix kernel its start, end, shader cycles and class; per wavefront of the combine kernel its
// start and end.  Nothing of this is in the ordinary library.
#ifdef SMART_TVA_TIMELINE
namespace timeline {
constexpr int kWorkgroups = 1024, kWaves = 16384;
__device__ unsigned long long wg_stamps[kWorkgroups * 4];  // start, end, shader cycles, class | worker << 8
__device__ unsigned long long wave_stamps[kWaves * 2];     // start, end
}  // namespace timeline
#define SMART_TIMELINE(...) __VA_ARGS__
#else
#define SMART_TIMELINE(...)
#endif

namespace {

using namespace smart::tva;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) float floatx8;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) uint16_t ushortx4;
typedef __attribute__((ext_vector_type(8))) uint16_t ushortx8;

constexpr int kWave = 64;
constexpr int kD = 128;
constexpr int kWgWaves = 8;           // wavefronts per workgroup of the prefix kernel (two per SIMD)
constexpr int kSmallSlot = kSmallRows * kD + 2 * kSmallRows;  // floats: O, then max, then sum
constexpr int kMediumSlot = kMediumRows * kD + 2 * kMediumRows;
constexpr int kLargeSlot = kLargeRows * kD + 2 * kLargeRows;
__host__ __device__ inline int class_rows(int cls) { return cls == 0 ? kSmallRows : (cls == 1 ? kMediumRows : kLargeRows); }
__host__ __device__ inline int class_slot(int cls) { return cls == 0 ? kSmallSlot : (cls == 1 ? kMediumSlot : kLargeSlot); }
// kFinish: every wavefront leaves the row maxima and sums of its row tile beside its part of O.
constexpr int kFinishTail = kWgWaves * 2 * 32;
__host__ __device__ inline int finish_slot(int cls) { return class_rows(cls) * kD + kFinishTail; }
constexpr int kCombineRows = 8;       // rows per combine wavefront (8 lanes per row)
constexpr int kChunkTiles = 64;       // tiles whose block ids one pair of registers holds
constexpr float kLog2e = 1.4426950408889634f;
// Online softmax with a lazy reference: the value m that the exponentials are taken against follows the running
// maximum only when the maximum has moved more than 2^kRescaleStep above it (in the exponent's units), so the
// accumulators are rescaled a few times per segment instead of on most tiles; until then probabilities may reach
// 2^kRescaleStep instead of 1, which binary32 sums and bf16 operands carry at the same relative precision.  The
// partial's (m, l, O) stay consistent with each other, which is all the merges downstream need.
constexpr float kRescaleStep = 8.f;
// Every K/V byte of the cache is read once per call: the loads are marked nontemporal (streaming), which on this
// machine lifts a plain read stream from about 6.1 to 7.0 TB/s.  The same hint as a cache-policy operand (the nt
// bit) for the loads that go straight to LDS.
constexpr int kStreamPolicy = 2;

// ---------------------------------------------------------------------------
// launch plan (device memory; written by tva_plan_kernel, or for batches of at most 64
// sequences by workgroup 0 of the prefix kernel); what it counts: tva_plan.h
// ---------------------------------------------------------------------------
// Segments (partial-result slot groups) per class that the host left room for.
struct SegCaps {
  int64_t segs[kClasses];
};

struct PlanView {
  int64_t* header;               // [2c] units U_c, [2c+1] workers W_c, [6+c] first workgroup of class c
  int64_t* cum_units[kClasses];  // [B+1] per class: units before sequence b
  int32_t* cum_segs[kClasses];   // [B+1] per class: segments before sequence b
  int32_t* cum_chunks;    // [B+1] combine row chunks before sequence b
  SeqInfo* info;          // [B]
};

__host__ __device__ inline size_t plan_bytes_for(int batch) {
  const size_t n = (size_t)batch + 2;
  return sizeof(int64_t) * (16 + kClasses * n) + sizeof(SeqInfo) * (size_t)batch +
         sizeof(int32_t) * (kClasses + 1) * n + 64;
}

__host__ __device__ inline PlanView plan_view(void* base, int batch) {
  PlanView v;
  const size_t n = (size_t)batch + 2;
  char* p = (char*)base;
  v.header = (int64_t*)p;
  p += sizeof(int64_t) * 16;
  for (int c = 0; c < kClasses; ++c) {
    v.cum_units[c] = (int64_t*)p;
    p += sizeof(int64_t) * n;
  }
  v.info = (SeqInfo*)p;
  p += sizeof(SeqInfo) * (size_t)batch;
  for (int c = 0; c < kClasses; ++c) {
    v.cum_segs[c] = (int32_t*)p;
    p += sizeof(int32_t) * n;
  }
  v.cum_chunks = (int32_t*)p;
  return v;
}

using smart::readlane64;
using smart::uniform64;
using smart::wave_excl_scan;

// cu_nodes must be a running sum: 0 <= cu[b] <= cu[b + 1] <= total_nodes for every b.  Otherwise the
// sizes of overlapping ranges could add up to more than total_nodes, the bound every buffer of the
// call was sized by; such a batch is planned as if every tree were empty (no output row is written).
__device__ inline bool offsets_malformed(int base, int next, int total_nodes) {
  return base < 0 || next < base || next > total_nodes;
}

template <bool kOnlySmall, bool kFinish>
__global__ __launch_bounds__(kWave) void tva_plan_kernel(
    void* plan_base, int batch, int total_nodes, int G, int Hkv, int max_blocks, int workgroups,
    SegCaps caps, TreeCost tc, const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ cu_nodes) {
  PlanView pv = plan_view(plan_base, batch);
  const int t = threadIdx.x;
  const int per = (batch + kWave - 1) / kWave;
  const int b0 = min(batch, t * per), b1 = min(batch, b0 + per);
  bool bad = false;
  for (int b = b0; b < b1; ++b) bad = bad || offsets_malformed(cu_nodes[b], cu_nodes[b + 1], total_nodes);
  const bool malformed = __any(bad);
  int64_t units[kClasses] = {0, 0, 0}, segs[kClasses] = {0, 0, 0}, chunks = 0;
  for (int b = b0; b < b1; ++b) {
    SeqInfo si = sequence_info<kOnlySmall>(prefix_len[b], cu_nodes[b], cu_nodes[b + 1], total_nodes, G, max_blocks);
    if (malformed) si.n = si.rg = 0;
    pv.info[b] = si;
    const int rows = si.n * G;
    const int c = plan_class<kOnlySmall>(rows);
    units[c] += sequence_units<kFinish>(si, c, G, Hkv, tc);
    segs[c] += Hkv * si.rg;
    chunks += Hkv * ((rows + kCombineRows - 1) / kCombineRows);
  }
  int64_t tot_u[kClasses], tot_s[kClasses], tot_c, u[kClasses], s[kClasses];
  for (int c = 0; c < kClasses; ++c) {
    u[c] = wave_excl_scan(units[c], t, &tot_u[c]);
    s[c] = wave_excl_scan(segs[c], t, &tot_s[c]);
  }
  int64_t ch = wave_excl_scan(chunks, t, &tot_c);
  // more segments than the host left room for (it sized by a hint that does not hold): nothing runs
  const bool over = tot_s[0] > caps.segs[0] || tot_s[1] > caps.segs[1] || tot_s[2] > caps.segs[2];
  if (over) {
    for (int c = 0; c < kClasses; ++c) tot_u[c] = tot_s[c] = u[c] = s[c] = 0;
    tot_c = ch = 0;
  }
  if (t == 0) {
    int64_t workers[kClasses], first_wg[kClasses + 1];
    apportion<kOnlySmall, kFinish>(tot_u, tot_s, tc, workgroups, workers, first_wg);
    for (int c = 0; c < kClasses; ++c) {
      pv.cum_units[c][batch] = tot_u[c];
      pv.cum_segs[c][batch] = (int32_t)tot_s[c];
      pv.header[2 * c] = tot_u[c];
      pv.header[2 * c + 1] = workers[c];
      pv.header[6 + c] = first_wg[c];
    }
    pv.header[6 + kClasses] = first_wg[kClasses];
    pv.cum_chunks[batch] = (int32_t)tot_c;
  }
  for (int b = b0; b < b1; ++b) {
    SeqInfo si = pv.info[b];
    if (over) {
      si.n = si.rg = 0;
      pv.info[b] = si;
    }
    const int rows = si.n * G;
    const int c = plan_class<kOnlySmall>(rows);
    for (int k = 0; k < kClasses; ++k) {
      pv.cum_units[k][b] = u[k];
      pv.cum_segs[k][b] = (int32_t)s[k];
    }
    pv.cum_chunks[b] = (int32_t)ch;
    u[c] += sequence_units<kFinish>(si, c, G, Hkv, tc);
    s[c] += Hkv * si.rg;
    ch += Hkv * ((rows + kCombineRows - 1) / kCombineRows);
  }
}

// The same plan for a batch of at most 64 sequences, computed by a wavefront for itself: lane
// b holds sequence b (lanes past the batch: an empty sequence, so their prefix sums are the
// totals).  One round trip to memory and a few shuffle scans replace a kernel launch.
struct LanePlan {
  SeqInfo si;                   // per lane
  int32_t cu;                   // cu_nodes[lane]
  int64_t cum_units[kClasses];  // per lane: units before this sequence
  int32_t cum_segs[kClasses];
  int32_t cum_chunks;
  int64_t units[kClasses];      // uniform: totals
  int32_t total_segs[kClasses];
  int64_t workers[kClasses];
  int64_t first_wg[kClasses + 1];
  int32_t chunks;
};

template <bool kOnlySmall, bool kFinish>
__device__ inline void lane_plan(LanePlan& p, const int32_t* prefix_len, const int32_t* cu_nodes, int batch,
                                 int total_nodes, int G, int Hkv, int max_blocks, int workgroups,
                                 const SegCaps& caps, TreeCost tc, int lane) {
  const int b = min(lane, batch - 1);
  const int32_t len = prefix_len[b], base = cu_nodes[min(lane, batch)], next = cu_nodes[b + 1];
  const bool malformed = __any(lane < batch && offsets_malformed(base, next, total_nodes));
  SeqInfo si = sequence_info<kOnlySmall>(len, base, next, total_nodes, G, max_blocks);
  if (lane >= batch) si.len = si.n = si.tiles = si.rg = 0;
  if (malformed) si.n = si.rg = 0;
  p.cu = base;
  // (a second pass only if the first finds more segments than the host left room for: it sized by a
  // hint that does not hold; then nothing runs)
  for (int pass = 0; pass < 2; ++pass) {
    const int rows = si.n * G;
    const int cls = plan_class<kOnlySmall>(rows);
    const int64_t my_units = sequence_units<kFinish>(si, cls, G, Hkv, tc);
    const int64_t my_segs = Hkv * si.rg;
    int64_t tot_s, tot_c;
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      p.cum_units[c] = wave_excl_scan(cls == c ? my_units : 0, lane, &p.units[c]);
      p.cum_segs[c] = (int32_t)wave_excl_scan(cls == c ? my_segs : 0, lane, &tot_s);
      p.total_segs[c] = (int32_t)tot_s;
    }
    p.cum_chunks = (int32_t)wave_excl_scan((int64_t)Hkv * ((rows + kCombineRows - 1) / kCombineRows), lane, &tot_c);
    p.chunks = (int32_t)tot_c;
    if (p.total_segs[0] <= caps.segs[0] && p.total_segs[1] <= caps.segs[1] && p.total_segs[2] <= caps.segs[2]) break;
    si.n = si.rg = 0;
  }
  p.si = si;
  const int64_t total_segs[kClasses] = {p.total_segs[0], p.total_segs[1], p.total_segs[2]};
  apportion<kOnlySmall, kFinish>(p.units, total_segs, tc, workgroups, p.workers, p.first_wg);
}

// ---------------------------------------------------------------------------
// prefix kernels
// ---------------------------------------------------------------------------
// What a kernel that finishes the rows itself needs behind its streaming loops (kFinish): the tree's own rows, the results
// and the arrival counters (one per wavefront and segment; class c's begin at arrive_first[c] segments).
struct FinishArgs {
  const __bf16* q;
  const __bf16* k_tree;
  const __bf16* v_tree;
  const uint32_t* anc_mask;  // four words per node
  __bf16* out;
  float* lse;
  float* ws[3];
  int32_t* arrive;
  int32_t* clear;  // counters of the context's next call, cleared by this one: n_clear, a multiple of 64
  int32_t n_clear;
  int32_t arrive_first[3];
  int32_t Hq, Hkv, G;
  float scale, scale_log2e;  // (without k_scale)
};

struct MainArgs {
  const __bf16* q;
  const __bf16* k_cache;
  const __bf16* v_cache;
  const int32_t* block_table;
  const int32_t* cu_nodes;
  const int32_t* prefix_len;
  void* plan;  // written by the planning kernel; unused for batches of at most 64 sequences
  float* ws[3];  // partial slots per class
  int64_t block_stride, head_stride;
  int32_t batch, total_nodes, Hq, Hkv, G, max_blocks, num_blocks, workgroups;
  SegCaps caps;  // segments per class the partial-result slots have room for
  TreeCost tree_cost;  // kFinish
  float scale_log2e;
  // fp8 cache only: k_cache / v_cache then point at bytes (E4M3), scale_log2e already includes k_scale,
  // a partial's row maxima are multiplied by m_scale (= k_scale) and its O by o_scale (= v_scale)
  float m_scale, o_scale;
  int32_t* status;  // kFinish: of the block-table check
  FinishArgs fin;
};

// Wave-uniform data (block table, plan) is read through the constant address
// space so that the loads are scalar and stay off the vector-memory queue the
// K/V stream uses.  Nothing read this way is written by the same kernel.
typedef const __attribute__((address_space(4))) int32_t* const_i32;
typedef const __attribute__((address_space(4))) int64_t* const_i64;
__device__ inline int32_t sload(const int32_t* p) { return *(const_i32)(uintptr_t)p; }
__device__ inline int64_t sload(const int64_t* p) { return *(const_i64)(uintptr_t)p; }
__device__ inline SeqInfo sload(const SeqInfo* p) {
  SeqInfo si;
  const int32_t* q = (const int32_t*)p;
  si.len = sload(q);
  si.n = sload(q + 1);
  si.tiles = sload(q + 2);
  si.rg = sload(q + 3);
  return si;
}

// Row m of a 16-row half of the score tile holds cache slot sigma(m): swapping
// bits 2 and 3 makes the 8 accumulator registers a lane ends up with (rows
// 4h..4h+3 and 8+4h..8+4h+3 of each half) cover 8 consecutive slots, which is
// one V vector of the interleaved layout.
__device__ inline int sigma(int m) { return (m & 3) | ((m & 4) << 1) | ((m & 8) >> 1); }

// Maximum over the two half-wavefronts (lanes j and j + 32) without touching LDS.
__device__ inline float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float sum_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Addresses of the two cache pages (one per 16-token block) of a 32-key tile.
struct TilePages {
  int64_t page0, page1;  // element offsets of (block, kv head) pages
};

__device__ inline int64_t clamp_block(int64_t blk, int num_blocks) {
  return blk < 0 ? 0 : (blk >= num_blocks ? num_blocks - 1 : blk);
}

__device__ inline TilePages tile_pages(const MainArgs& a, const int32_t* bt_row, int tile,
                                       int n_blocks, int g) {
  const int i0 = 2 * tile;
  const int i1 = min(2 * tile + 1, n_blocks - 1);  // a missing second block is fully masked later
  TilePages tp;
  tp.page0 = clamp_block(sload(bt_row + i0), a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  tp.page1 = clamp_block(sload(bt_row + i1), a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  return tp;
}

// A load of cache contents that this call reads once (kStream: marked nontemporal) or that another wavefront reads
// again (left to the caches).
template <bool kStream, typename T>
__device__ inline T stream_load(const T* p) {
  if (kStream) return __builtin_nontemporal_load(p);
  return *p;
}

// K tile as the A operand of the score product: lane (h, j) holds key row j,
// head dims 16 ks + 8 h .. + 7 for k step ks.
template <bool kStream>
__device__ inline void load_k(bf16x8 (&k)[8], const MainArgs& a, const TilePages& tp, int lane) {
  const int h = lane >> 5, j = lane & 31;
  // rows 0..15 come from the tile's first cache block, rows 16..31 from its second
  // (branch-free select: mask is all ones for the second block)
  const int64_t mask = -(int64_t)(j >> 4);
  const int64_t page = tp.page0 ^ ((tp.page0 ^ tp.page1) & mask);
  const __bf16* kp = a.k_cache + page + (h * 16 + sigma(j & 15)) * 8;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) k[ks] = stream_load<kStream>((const bf16x8*)(kp + ks * 256));
}

// V tile as the A operand of the output product: lane (h, j) holds head dim
// 32 jt + j, tokens 8 h .. 8 h + 7 of cache block kk.
template <bool kStream>
__device__ inline void load_v(bf16x8 (&v)[2][4], const MainArgs& a, const TilePages& tp, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const __bf16* vp0 = a.v_cache + tp.page0 + (h * kD + j) * 8;
  const __bf16* vp1 = a.v_cache + tp.page1 + (h * kD + j) * 8;
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    v[0][jt] = stream_load<kStream>((const bf16x8*)(vp0 + jt * 256));
    v[1][jt] = stream_load<kStream>((const bf16x8*)(vp1 + jt * 256));
  }
}

// The same two tiles out of an fp8 cache: the pages have the same element order, one byte per
// element, so a lane's operand vector is 8 bytes; it becomes bf16 (exactly) just before its MFMA.
typedef __attribute__((ext_vector_type(2))) uint32_t fp8x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Where this lane's vectors of a tile begin (K: 256 bytes from one k step to the next; V: from one d tile to the next).
__device__ inline const uint8_t* k_vectors(const MainArgs& a, const TilePages& tp, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const int64_t mask = -(int64_t)(j >> 4);
  const int64_t page = tp.page0 ^ ((tp.page0 ^ tp.page1) & mask);
  return (const uint8_t*)a.k_cache + page + (h * 16 + sigma(j & 15)) * 8;
}
__device__ inline const uint8_t* v_vectors(const MainArgs& a, int64_t page, int lane) {
  return (const uint8_t*)a.v_cache + page + ((lane >> 5) * kD + (lane & 31)) * 8;
}

template <bool kStream>
__device__ inline void load_k(fp8x8 (&k)[8], const MainArgs& a, const TilePages& tp, int lane) {
  const uint8_t* kp = k_vectors(a, tp, lane);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) k[ks] = stream_load<kStream>((const fp8x8*)(kp + ks * 256));
}

template <bool kStream>
__device__ inline void load_v(fp8x8 (&v)[2][4], const MainArgs& a, const TilePages& tp, int lane) {
  const uint8_t* vp0 = v_vectors(a, tp.page0, lane);
  const uint8_t* vp1 = v_vectors(a, tp.page1, lane);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    v[0][jt] = stream_load<kStream>((const fp8x8*)(vp0 + jt * 256));
    v[1][jt] = stream_load<kStream>((const fp8x8*)(vp1 + jt * 256));
  }
}

__device__ inline bf16x8 operand(const bf16x8& x) { return x; }
__device__ inline bf16x8 operand(const fp8x8& x) {
  const bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[0], 1.0f, false);
  const bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[0], 1.0f, true);
  const bf16x2 c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[1], 1.0f, false);
  const bf16x2 d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[1], 1.0f, true);
  bf16x8 r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
  return r;
}

__device__ inline void zero_token(bf16x8& v, int e) { v[e] = (__bf16)0.f; }
__device__ inline void zero_token(fp8x8& v, int e) { v[e >> 2] &= ~(0xFFu << (8 * (e & 3))); }  // byte 0x00 = +0

// Masks the ragged end of a prefix: scores of tokens >= n_valid become -inf and
// their V entries zero (unused cache slots may hold anything, NaN included).
template <typename Raw>
__device__ inline void mask_tail(floatx16& s, Raw (&v)[2][4], int n_valid, int h) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * h + (r & 3);  // score-tile row of this register
    const int tok = (i & 16) + sigma(i & 15);      // token of the tile it holds
    if (tok >= n_valid) s[r] = -INFINITY;
  }
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (kk * 16 + h * 8 + e >= n_valid) {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) zero_token(v[kk][jt], e);
      }
}

// Online-softmax update of one 32-row tile: scores s (keys x rows, transposed)
// -> bf16 probabilities in the operand layout of the output product.
__device__ inline void softmax_tile(const floatx16& s, float& m, float& l, floatx16 (&o)[4],
                                    bf16x8& pb0, bf16x8& pb1, float c) {
  float mx = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
  mx = max_across_halves(mx);
  const float m_new = fmaxf(m, mx);
  if (__any((m_new - m) * c > kRescaleStep)) {  // the reference follows the maximum in steps: see kRescaleStep
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
    l *= alpha;
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) o[jt] *= alpha;
    m = m_new;
  }
  const float mc = m * c;
  floatx8 p0, p1;
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    p0[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -mc));
    p1[r] = __builtin_amdgcn_exp2f(fmaf(s[r + 8], c, -mc));
    sum += p0[r] + p1[r];
  }
  l += sum;
  pb0 = __builtin_convertvector(p0, bf16x8);
  pb1 = __builtin_convertvector(p1, bf16x8);
}

// The fold of class 1 stores a partial's 16-byte pieces write-through (device scope) instead of leaving them dirty
// in L2: measured on the workload that is mostly class 1 and bound by memory (64 sequences, prefix 16384), the
// prefix kernel takes 692 us instead of 711, three runs each, alternating.  The same policy measured neutral for
// class 0's fold with a bf16 cache and for class 2's partials, and 3 us slower (50 -> 53 us) for the fold of the fp8
// stream, so only class 1 uses it.  The instruction is
// written as assembly (no builtin carries that cache policy for a 16-byte store); the wait states after it are
// what the compiler would insert itself between a store of more than 8 bytes and the next write of its data
// registers.
__device__ inline void store_through(float* dst, floatx4 x) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 3" ::"v"(dst), "v"(x) : "memory");
}

// Writes one 32-row tile of a partial: O as [d / 4][row][4] so that lanes
// write contiguous 16-byte pieces; then the row maxima and sums.
// (fp8 cache: the scores were taken against the raw key bytes and O against the raw value bytes, so the row maxima
// leave multiplied by m_scale = k_scale and O by o_scale = v_scale; both are 1 for a bf16 cache.)
__device__ inline void store_partial(float* slot, int rows_in_slot, int qt, const floatx16 (&o)[4],
                                     float m, float l, int lane, float m_scale = 1.f, float o_scale = 1.f) {
  const int h = lane >> 5, j = lane & 31;
  const float lsum = sum_across_halves(l);
  // One lane-dependent address, formed here, and constant offsets from it: chunk jt * 8 + 2 * r4 + h of the tile
  // lies (jt * 8 + 2 * r4) * 512 bytes behind chunk h.  (Left to itself the compiler kept sixteen 64-bit offsets
  // alive across the whole piece loop, spilled them, and reloaded one before each store -- and a reload waits for
  // every memory operation in flight, the previous store included: 3.7 .. 4.8 us per partial.)
  // (the pointer keeps its global address space through the barrier: a generic one would turn the stores into flat
  // ones, which also count as LDS traffic and would fall among the counted waits of the next piece)
  typedef __attribute__((address_space(1))) float global_float;
  typedef __attribute__((address_space(1))) floatx4 global_floatx4;
  global_float* first = (global_float*)(slot + ((size_t)(qt * 32 + h) * 32 + j) * 4);
  asm volatile("" : "+v"(first));
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      floatx4 x;
      x[0] = o[jt][4 * r4 + 0] * o_scale;
      x[1] = o[jt][4 * r4 + 1] * o_scale;
      x[2] = o[jt][4 * r4 + 2] * o_scale;
      x[3] = o[jt][4 * r4 + 3] * o_scale;
      *(global_floatx4*)(first + (jt * 8 + 2 * r4) * 32 * 4) = x;
    }
  if (h == 0) {
    global_float* ml = (global_float*)(slot + rows_in_slot * kD + qt * 32 + j);
    asm volatile("" : "+v"(ml));
    ml[0] = m * m_scale;  // (-inf stays -inf)
    ml[rows_in_slot] = lsum;
  }
}

// ---- kFinish: the prefix kernel evaluates the tree part and finishes the rows itself -------------------------------
//
// The tree part is one more tile (or up to four) of masked keys behind the last prefix tile, on the matrix cores, and
// belongs to the piece that ends the segment.  A segment that one worker holds alone is finished from registers.  Where
// several workers hold pieces of it, the one that comes last merges them: a wavefront writes its part of the piece through
// to memory, waits for that, and counts itself in (one counter per segment and wavefront, so no wavefront waits for
// another); who finds all others counted takes their parts and writes the rows.  Nobody ever waits for another workgroup.
// Usually a worker's last piece begins a segment that its neighbour ended first thing, so it finds the neighbour counted
// before it has written anything, and merges from registers.  The parts are merged in the order of the workers with the
// same operations whoever does it, so the result does not depend on timing.  The counters return to zero, and a call clears those
// of the context's next one besides (smart::next_counters; 0.0 .. 0.2 us of a call).
// What it costs and saves (stamps; 32 sequences of 4 .. 64 nodes, 8B shapes): the tree part 3.4 .. 5 us and a part's store
// and count 2.2 us per segment, merge and rows at the end 3.2 us, where the combine kernel took 18 us and a launch; the call
// 131 -> 121 us, one sequence of 7 nodes and 517 tokens (a table of at most 1024, see finishes) 18.9 -> 14.5.
struct Finish {
  int pieces, mine;  // pieces of the segment, and which of them this is
  int slot, seg;     // this piece's slot of the class (the pieces of a segment have consecutive ones); segment of the class
  int base, g, rows, row0;  // first node, kv head, rows of the kv head, first row of the row group
};

// The arguments, read again from where the launch put them.  Held in registers across the streaming loops they displace
// what the loops use, which then comes lane by lane from where the compiler put it (fifteen v_readlane per tile).
__device__ inline MainArgs kernel_args() {
  uintptr_t p = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const MainArgs*)(const __attribute__((address_space(4))) MainArgs*)p;
}

// What a stream uses of the arguments, each in registers of its own: as parts of the groups that one load fetched they would
// be kept, or put aside and fetched back, together with the rest of the group.
__device__ inline MainArgs stream_args(MainArgs a) {
  asm volatile("" : "+s"(a.block_stride), "+s"(a.head_stride), "+s"(a.num_blocks), "+s"(a.scale_log2e));
  return a;
}

// This wavefront's counter of segment f.seg.
template <int kCls>
__device__ inline int32_t* counter_of(const FinishArgs& a, const Finish& f, int wv) {
  return a.arrive + ((int64_t)a.arrive_first[kCls] + f.seg) * kWgWaves + wv;
}

// (a lane number that the compiler does not know to be loop-invariant: what follows from it is then computed where it is
// used and does not occupy registers during the stream)
__device__ inline int fresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

__device__ inline Finish finish_of(int64_t ub, int64_t span, int64_t U, int64_t W, int64_t w, int64_t seg, int base, int g,
                                   int rows, int row0) {
  int64_t w_first, w_last;
  segment_workers(ub, span, U, W, w_first, w_last);
  Finish f;
  f.pieces = __builtin_amdgcn_readfirstlane((int)(w_last - w_first) + 1);
  f.mine = __builtin_amdgcn_readfirstlane((int)(w - w_first));
  f.slot = __builtin_amdgcn_readfirstlane((int)(w + seg));
  f.seg = __builtin_amdgcn_readfirstlane((int)seg);
  f.base = base;
  f.g = g;
  f.rows = rows;
  f.row0 = row0;
  return f;
}

// (through a buffer resource: these builtins carry the cache policy that is coherent across the XCDs, sc1)
constexpr int kDevicePolicy = 16;
typedef __attribute__((ext_vector_type(4))) uint32_t uintx4;
__device__ inline __amdgpu_buffer_rsrc_t slot_buffer(float* slot, int floats) {
  return __builtin_amdgcn_make_buffer_rsrc(slot, 0, floats * 4, 0x00027000);
}
__device__ inline floatx4 load_part(__amdgpu_buffer_rsrc_t r, int offset) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, kDevicePolicy));
}
__device__ inline float load_word(__amdgpu_buffer_rsrc_t r, int offset) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, offset, 0, kDevicePolicy));
}

// (one reading for the whole wavefront: others count meanwhile, lanes might read different values, and what follows is decided
// for all of them)
__device__ inline int arrivals(const int32_t* counter) {
  return __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// (x, m, l) and (y, mc, lc) -> (x, m, l); an empty state has maximum -inf and sums of zero.
template <int kQuads>
__device__ inline void merge_part(floatx4 (&x)[kQuads], float& m, float& l, const floatx4 (&y)[kQuads], float mc, float lc,
                                  float c) {
  const float m_new = fmaxf(m, mc);
  const float al = m == m_new ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * c);
  const float wt = mc == m_new ? 1.f : __builtin_amdgcn_exp2f((mc - m_new) * c);
#pragma unroll
  for (int u = 0; u < kQuads; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[u][i] = fmaf(x[u][i], al, wt * y[u][i]);
  l = fmaf(l, al, wt * lc);
  m = m_new;
}

// Rows of this wavefront's row tile, accumulator quads quad0 .. : normalised, rounded and stored.  Lanes (0, j) and (1, j)
// hold halves of each eight head dims of row j; they trade so that each stores 16 bytes.
template <int kQuads>
__device__ inline void write_rows(const FinishArgs& a, const Finish& f, const floatx4 (&x)[kQuads], float m, float l, int quad0,
                                  int rt, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const float inv = l > 0.f ? 1.f / l : 0.f;
  const int rho = f.row0 + rt * 32 + j;
  const bool real = rho < f.rows;
  const int64_t row = (int64_t)(f.base + rho / a.G) * a.Hq + f.g * a.G + rho % a.G;
  __bf16* op = a.out + row * kD + 8 * (quad0 + h);
#pragma unroll
  for (int u = 0; u < kQuads; u += 2) {
    floatx8 y;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y[i] = x[u][i] * inv;
      y[4 + i] = x[u + 1][i] * inv;
    }
    const uintx4 w = __builtin_bit_cast(uintx4, __builtin_convertvector(y, bf16x8));
    const auto lo = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    uintx4 z;
    z[0] = lo[0], z[1] = hi[0], z[2] = lo[1], z[3] = hi[1];
    if (real) *(uintx4*)(op + 8 * u) = z;
  }
  if (a.lse && real && quad0 == 0 && h == 0) a.lse[row] = l > 0.f ? m * a.scale + logf(l) : -INFINITY;
}

// One wavefront's part of a piece, quads quad0 .. of row tile rt (l: of the whole row).
// `early`: the counter as read some time before; it only grows until everyone is counted.
template <int kCls, int kQuads>
__device__ inline void finish_part(const FinishArgs& a, const Finish& f, floatx4 (&x)[kQuads], float m, float l, int quad0,
                                   int rt, int early, int wv, int lane) {
  lane = fresh(lane);
  const int h = lane >> 5, j = lane & 31;
  if (f.pieces > 1) {
    constexpr int kO = (kCls == 0 ? kSmallRows : kCls == 1 ? kMediumRows : kLargeRows) * kD, kSlot = kO + kFinishTail;
    const float c = a.scale_log2e;
    int32_t* const counter = counter_of<kCls>(a, f, wv);
    const int at = ((rt * 32 + 2 * quad0 + h) * 32 + j) * 16, ml = (kO + wv * 64 + j) * 4;
    const bool in_place = early == f.pieces - 1 && (f.mine == 0 || f.pieces == 2);
    if (!in_place) {
      const __amdgpu_buffer_rsrc_t r = slot_buffer(a.ws[kCls] + (size_t)f.slot * kSlot, kSlot);
#pragma unroll
      for (int u = 0; u < kQuads; ++u)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, x[u]), r, at + u * 1024, 0, kDevicePolicy);
      if (h == 0) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m), r, ml, 0, kDevicePolicy);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(l), r, ml + 128, 0, kDevicePolicy);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      int before = 0;
      if (lane == 0) before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_readfirstlane(before) != f.pieces - 1) return;
    }
    asm volatile("" ::: "memory");  // (the parts are requested after the counter said that they are there)
    if (lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float* const first = a.ws[kCls] + (size_t)(f.slot - f.mine) * kSlot;
    int k = 1;
    if (!in_place || f.mine != 0) {
      const __amdgpu_buffer_rsrc_t r = slot_buffer(first, kSlot);
      floatx4 y[kQuads];
#pragma unroll
      for (int u = 0; u < kQuads; ++u) y[u] = load_part(r, at + u * 1024);
      float mc = load_word(r, ml), lc = load_word(r, ml + 128);
      if (in_place) {  // two pieces, this is the second
        merge_part(y, mc, lc, x, m, l, c);
        k = 2;
      }
#pragma unroll
      for (int u = 0; u < kQuads; ++u) x[u] = y[u];
      m = mc;
      l = lc;
    }
    for (; k < f.pieces; ++k) {
      const __amdgpu_buffer_rsrc_t r = slot_buffer(first + (size_t)k * kSlot, kSlot);
      floatx4 y[kQuads];
#pragma unroll
      for (int u = 0; u < kQuads; ++u) y[u] = load_part(r, at + u * 1024);
      const float mc = load_word(r, ml), lc = load_word(r, ml + 128);
      merge_part(x, m, l, y, mc, lc, c);
    }
  }
  write_rows(a, f, x, m, l, quad0, rt, lane);
}

// Ancestor mask of row rho: word tt holds tree keys 32 tt .. 32 tt + 31; bits past the tree are cleared.
__device__ inline uint32_t mask_word(const FinishArgs& a, int base, int rows, int rho, int n, int tt) {
  const int node = base + (rho < rows ? rho : rows - 1) / a.G;
  const uint32_t w = a.anc_mask[4 * (int64_t)node + tt];
  const int left = n - 32 * tt;
  return left >= 32 ? w : (left > 0 ? w & ((1u << left) - 1u) : 0u);
}

// Scores of a tile of tree keys -> probabilities (softmax_tile, for masked keys; the reference follows the maximum at
// once, so that a probability is at most 1 however large the tree's values are).  A row sees few tree keys and often has most of
// its weight on one of them, whose rounding does not average out as that of a prefix's many does: the reference is raised by
// less than a power of two so that the largest probability of the tile is a power of two, which bf16 holds exactly (error
// against 64 bits, 86 sequences of 13 .. 106 tokens, 64 .. 128 nodes: 2.097e-3 without, 2.071e-3 with; 0.0 .. 0.1 us a call.
// Two bf16 parts of each probability, eight more matrix instructions a tile: 2.07e-3, 0.1 .. 0.2 us).
__device__ inline void softmax_tree(floatx16& s, uint32_t word, float& m, float& l, floatx16 (&o)[4], bf16x8& pb0,
                                    bf16x8& pb1, float c, int h) {
  const uint32_t bits = word >> (8 * h);  // register r holds key 16 (r / 8) + 8 h + r % 8: see sigma
  float mx = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r) mx = fmaxf(mx, (bits >> (16 * (r >> 3) + (r & 7))) & 1u ? s[r] : -INFINITY);
  mx = max_across_halves(mx);
  float m_new = fmaxf(m, mx);
  // (infinite, or NaN, if there is no key or an infinite score.  Less than a millionth needs nothing, and a softmax scale whose
  // reciprocal is infinite gives no more)
  const float below = (m_new - mx) * c;
  if (below > 1e-6f && below < 64.f) m_new = fmaf(ceilf(below), __builtin_amdgcn_rcpf(c), mx);
  const float alpha = m_new == m ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * c);
  l *= alpha;
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) o[jt] *= alpha;
  m = m_new;
  const float mc = m * c;
  floatx8 p0, p1;
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    p0[r] = (bits >> r) & 1u ? __builtin_amdgcn_exp2f(fmaf(s[r], c, -mc)) : 0.f;
    p1[r] = (bits >> (16 + r)) & 1u ? __builtin_amdgcn_exp2f(fmaf(s[r + 8], c, -mc)) : 0.f;
    sum += p0[r] + p1[r];
  }
  l += sum;
  pb0 = __builtin_convertvector(p0, bf16x8);
  pb1 = __builtin_convertvector(p1, bf16x8);
}

// Largest magnitude, as bits, of the elements of eight bf16 values seen so far, per half of a dword.
typedef __attribute__((ext_vector_type(2))) uint16_t ushortx2;
typedef __attribute__((ext_vector_type(8))) uint16_t ushort8;
__device__ inline void note_magnitude(ushortx2& top, const ushort8& v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ushortx2 x;
    x[0] = v[2 * i] & 0x7FFF;
    x[1] = v[2 * i + 1] & 0x7FFF;
    top = __builtin_elementwise_max(top, x);
  }
}
__device__ inline bool not_finite(const ushortx2& top) { return top[0] >= 0x7F80 || top[1] >= 0x7F80; }

// The rows of a tree's keys (its first node's row of kv head g on): a uniform base and 32-bit offsets behind it.
struct TreeRows {
  const char *k, *v;
  int pitch, last;  // bytes from node to node; last node
};
__device__ inline TreeRows tree_rows(const FinishArgs& a, int base, int g, int n) {
  const int64_t at = ((int64_t)base * a.Hkv + g) * kD;
  return TreeRows{(const char*)(a.k_tree + at), (const char*)(a.v_tree + at), a.Hkv * kD * 2, n - 1};
}
// A lane's operand vectors of a tile of tree keys.  K: key row j, head dims 16 ks + 8 h ..; V: head dim 32 jt + j, tokens
// 16 kk + 8 h ..: gathered, 64 contiguous bytes per half wavefront and token.  Keys past the tree repeat its last one.
__device__ inline bf16x8 tree_k(const TreeRows& t, int tt, int ks, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const uint32_t at = min(32 * tt + (j & 16) + sigma(j & 15), t.last) * t.pitch + h * 16;
  return *(const bf16x8*)(t.k + at + ks * 32);
}
__device__ inline ushort8 tree_v(const TreeRows& t, int tt, int kk, int jt, int lane) {
  const int h = lane >> 5, j = lane & 31;
  ushort8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t at = min(32 * tt + 16 * kk + 8 * h + e, t.last) * t.pitch + j * 2;
    v[e] = *(const uint16_t*)(t.v + at + jt * 64);
  }
  return v;
}
// Infinite and NaN elements -> 0: on the matrix cores a zero probability times such a value would reach the rows that do
// not see it.
__device__ inline void clear_not_finite(ushort8& v) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (v[e] & 0x7F80) == 0x7F80 ? 0 : v[e];
}
// What clear_not_finite took away of tiles tt .. tt_end - 1, added to the rows that do see it: a positive probability times an
// infinity is that infinity, and NaN stays NaN.  (To the state that carries the tile, whose maximum is no less than the key's
// score: one without the tile may have no weight in the fold, and zero times an infinity is NaN.)
__device__ inline void add_not_finite(floatx16 (&o)[4], const FinishArgs& a, const TreeRows& t, int base, int rows, int rho, int n,
                                      int tt, int tt_end, int lane) {
  // (kept a loop, and what it uses computed here: unrolled and hoisted it cost the kernel 78 spilled registers, a step of four
  // sequences 57 us instead of 50)
  rho = fresh(rho);
  lane = fresh(lane);
  asm volatile("" : "+s"(tt), "+s"(tt_end));
#pragma clang loop unroll(disable)
  for (; tt < tt_end && 32 * tt < n; ++tt) {
    uint32_t bits = mask_word(a, base, rows, rho, n, tt);
    while (__any(bits != 0u)) {
      const uint32_t at = (bits != 0u ? 32 * tt + __ffs(bits) - 1 : 0) * t.pitch + (lane >> 5) * 8;
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint16_t v = *(const uint16_t*)(t.v + at + 64 * jt + 16 * (r >> 2) + 2 * (r & 3));
          if (bits != 0u && (v & 0x7F80) == 0x7F80) o[jt][r] += __uint_as_float((uint32_t)v << 16);
        }
      bits &= bits - 1u;
    }
  }
}

// One tile of tree keys against the 32 rows from `row` on, operands straight from memory (for loops that have no barrier).
__device__ inline void tree_tile(floatx16 (&o)[4], float& m, float& l, const FinishArgs& a, int base, int g, int rows, int row,
                                 int n, int tt, int lane) {
  const float c = a.scale_log2e;
  lane = fresh(lane);
  const int h = lane >> 5, j = lane & 31;
  const TreeRows t = tree_rows(a, base, g, n);
  ushort8 v[2][4];
  bf16x8 k[8], q[8];
  const int rho = row + j < rows ? row + j : rows - 1;
  const __bf16* qp = a.q + ((int64_t)(base + rho / a.G) * a.Hq + g * a.G + rho % a.G) * kD + h * 8;
  const uint32_t word = mask_word(a, base, rows, rho, n, tt);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    k[ks] = tree_k(t, tt, ks, lane);
    q[ks] = *(const bf16x8*)(qp + ks * 16);
  }
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) v[kk][jt] = tree_v(t, tt, kk, jt, lane);
  floatx16 s = (floatx16)(0.f);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[ks], q[ks], s, 0, 0, 0);
  bf16x8 pb0, pb1;
  softmax_tree(s, word, m, l, o, pb0, pb1, c, h);
  ushortx2 top = {0, 0};
#pragma unroll
  for (int i = 0; i < 8; ++i) note_magnitude(top, v[i >> 2][i & 3]);
  const bool mend = __any(not_finite(top));
  if (mend) {
#pragma unroll
    for (int i = 0; i < 8; ++i) clear_not_finite(v[i >> 2][i & 3]);
  }
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v[0][jt]), pb0, o[jt], 0, 0, 0);
    o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v[1][jt]), pb1, o[jt], 0, 0, 0);
  }
  if (mend) add_not_finite(o, a, t, base, rows, rho, n, tt, tt + 1, lane);
}

// The whole workgroup puts up to four tiles of tree keys into LDS stages 0 .. 3 in operand order: wavefront w K step w and
// V vector w of each.  request_tree asks for two tiles; stage_tree, entered after a barrier behind which nobody reads a
// stage and no request for one is in flight, stores them, sees to the rest, and returns after a barrier whether a value is
// infinite or NaN (flags: a word per wavefront).
struct TreePair {
  bf16x8 k[2];
  ushort8 v[2];
};
__device__ inline void request_tree(TreePair& p, const TreeRows& t, int tt, int wv, int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    p.k[i] = tree_k(t, tt + i, wv, lane);
    p.v[i] = tree_v(t, tt + i, wv >> 2, wv & 3, lane);
  }
}
__device__ inline bool stage_tree(TreePair& p, const TreeRows& t, bf16x8* lds, uint32_t* flags, int wv, int lane) {
  ushortx2 top = {0, 0};
  for (int tt = 0;;) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      note_magnitude(top, p.v[i]);
      if (__any(not_finite(top))) clear_not_finite(p.v[i]);
      lds[((tt + i) * 16 + wv) * kWave + lane] = p.k[i];
      lds[((tt + i) * 16 + 8 + wv) * kWave + lane] = __builtin_bit_cast(bf16x8, p.v[i]);
    }
    tt += 2;
    if (32 * tt > t.last) break;
    request_tree(p, t, tt, wv, lane);
  }
  const bool mend = __any(not_finite(top));
  if (lane == 0) flags[wv] = mend ? 1u : 0u;
  __syncthreads();
  uint32_t any = 0u;
#pragma unroll
  for (int i = 0; i < kWgWaves; ++i) any |= flags[i];
  return any != 0u;
}

// Staged tile tt against this wavefront's rows.
__device__ inline void staged_tree_tile(floatx16 (&o)[4], float& m, float& l, const bf16x8 (&q)[8], uint32_t word,
                                        const bf16x8* lds, int tt, float c, int lane) {
  const bf16x8* st = lds + tt * 16 * kWave + lane;
  floatx16 s = (floatx16)(0.f);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st[ks * kWave], q[ks], s, 0, 0, 0);
  bf16x8 pb0, pb1;
  softmax_tree(s, word, m, l, o, pb0, pb1, c, lane >> 5);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st[(8 + jt) * kWave], pb0, o[jt], 0, 0, 0);
    o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st[(12 + jt) * kWave], pb1, o[jt], 0, 0, 0);
  }
}

// Locates the sequence that holds unit u0 in one class's unit space.
__device__ inline int find_sequence(const int64_t* cum_units, int batch, int64_t u0) {
  int lo = 0, hi = batch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sload(cum_units + mid) <= u0) lo = mid; else hi = mid;
  }
  return lo;
}

// ---- class 0: bandwidth-bound kernel, rows <= 32 -----------------------------------------
//
// K and V each have one register buffer.  The loop body is straight-line:
// scores -> request next K -> softmax -> output product -> request next V, so
// each request is in flight during the other half of the iteration and during
// the co-resident wavefront's work (two wavefronts per SIMD).  The last tile
// of a wavefront's share is taken out of the loop and requests nothing (the
// loop body itself has no conditional request, which keeps the hardware wait
// counters exact); within a share longer than 64 tiles, a 64-tile chunk ends on
// a repeated request for its own last tile.
struct SmallState {
  floatx16 o[4];
  float m, l;
};

// Block ids of tiles [tc, tc + 64) of a sequence live in two registers (lane i
// of reg r holds entry 2 tc + 64 r + i); a tile's two ids come out by readlane.
struct BlockIds {
  int32_t lo, hi;
};

__device__ inline TilePages pages_from_ids(const MainArgs& a, const BlockIds& ids, int rel_tile, int g) {
  const int r = 2 * rel_tile;  // even, so both entries sit in the same register
  const int32_t src = r < kWave ? ids.lo : ids.hi;
  const int64_t blk0 = clamp_block(__builtin_amdgcn_readlane(src, r & (kWave - 1)), a.num_blocks);
  const int64_t blk1 = clamp_block(__builtin_amdgcn_readlane(src, (r + 1) & (kWave - 1)), a.num_blocks);
  TilePages tp;
  tp.page0 = blk0 * a.block_stride + (int64_t)g * a.head_stride;
  tp.page1 = blk1 * a.block_stride + (int64_t)g * a.head_stride;
  return tp;
}

// One tile of a share that is not its last: the requests for the next tile go out as soon as the registers they
// refill are free (K after the score product, V after the output product).
template <bool kStream, typename Raw>
__device__ inline void small_tile(SmallState& S, Raw (&k)[8], Raw (&v)[2][4], const bf16x8 (&q)[8],
                                  int lane, float c, const MainArgs& a, const TilePages& next) {
  floatx16 s = (floatx16)(0.f);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(k[ks]), q[ks], s, 0, 0, 0);
  load_k<kStream>(k, a, next, lane);
  bf16x8 pb0, pb1;
  softmax_tile(s, S.m, S.l, S.o, pb0, pb1, c);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    S.o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(v[0][jt]), pb0, S.o[jt], 0, 0, 0);
    S.o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(v[1][jt]), pb1, S.o[jt], 0, 0, 0);
  }
  load_v<kStream>(v, a, next, lane);
}

// The last tile of a share: nothing follows, so nothing is requested (the streamed lines are not kept in L2, a
// repeated request would go to memory again); it is also the only tile that can be ragged (n_valid < 32).
template <typename Raw>
__device__ inline void small_last_tile(SmallState& S, Raw (&k)[8], Raw (&v)[2][4], const bf16x8 (&q)[8],
                                       int lane, float c, int n_valid) {
  floatx16 s = (floatx16)(0.f);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(k[ks]), q[ks], s, 0, 0, 0);
  if (n_valid < kTile) mask_tail(s, v, n_valid, lane >> 5);
  bf16x8 pb0, pb1;
  softmax_tile(s, S.m, S.l, S.o, pb0, pb1, c);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    S.o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(v[0][jt]), pb0, S.o[jt], 0, 0, 0);
    S.o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(v[1][jt]), pb1, S.o[jt], 0, 0, 0);
  }
}

// kStream: no other wavefront reads these tiles (see stream_load).
template <typename Raw = bf16x8, bool kStream = true>
__device__ inline void small_segment(SmallState& S, const MainArgs& a, int b, int g, int base, int t0,
                                     int t1, const SeqInfo si, int lane, int row0 = 0) {
  const int h = lane >> 5, j = lane & 31;
  const int M = si.n * a.G;
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) S.o[jt] = (floatx16)(0.f);
  S.m = -INFINITY;
  S.l = 0.f;
  if (t0 >= t1) return;  // this wavefront has no tile of the piece
  bf16x8 q[8];  // B operand of the score product: query row j, head dims 16 ks + 8 h ..
  {
    const int rho = row0 + j < M ? row0 + j : M - 1;  // padding rows repeat the last real row; never read back
    const int node = base + rho / a.G, head = g * a.G + rho % a.G;
    const __bf16* qp = a.q + ((int64_t)node * a.Hq + head) * kD + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ks] = *(const bf16x8*)(qp + ks * 16);
  }
  const int32_t* bt_row = a.block_table + (int64_t)b * a.max_blocks;
  const int n_blocks = (si.len + kBlock - 1) / kBlock;
  const float c = a.scale_log2e;

  for (int tc = t0; tc < t1; tc += kChunkTiles) {
    const int te = min(t1, tc + kChunkTiles);
    BlockIds ids;
    ids.lo = bt_row[min(2 * tc + lane, n_blocks - 1)];
    ids.hi = bt_row[min(2 * tc + kWave + lane, n_blocks - 1)];
    // Both id registers must have landed before the tile stream starts: inside the loop
    // nothing may wait on them, or the wait would also drain the K/V requests in flight.
    asm volatile("" ::"v"(ids.lo), "v"(ids.hi));
    Raw k[8], v[2][4];
    {
      const TilePages first = pages_from_ids(a, ids, 0, g);
      load_k<kStream>(k, a, first, lane);
      load_v<kStream>(v, a, first, lane);
    }
    // The share's last tile (which the sequence's ragged last tile always is, when the share holds it) is taken
    // out of the loop.  A chunk that is not the share's last ends on a repeated request for its own last tile.
    const bool ends_here = te == t1;
    const int loop_end = ends_here ? te - 1 : te;
    int t = tc;
    for (; t < loop_end; ++t) {
      const TilePages next = pages_from_ids(a, ids, min(t + 1, te - 1) - tc, g);
      small_tile<kStream>(S, k, v, q, lane, c, a, next);
    }
    if (ends_here) small_last_tile(S, k, v, q, lane, c, si.len - t * kTile);
  }
}

// A wavefront's running softmax state in LDS: register by register, lane by lane.
constexpr int kStateFloats = (64 + 2) * kWave;  // 64 accumulator registers + max + sum, per lane

// (four registers of a lane lie together: 16-byte LDS accesses on both sides of the fold)
__device__ inline void state_to_lds(const SmallState& S, float* region, int lane) {
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      floatx4 x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = S.o[jt][4 * r4 + i];
      ((floatx4*)region)[(jt * 4 + r4) * kWave + lane] = x;
    }
  region[64 * kWave + lane] = S.m;
  region[65 * kWave + lane] = S.l;
}
// Accumulator registers 4 quad .. 4 quad + 3 of a lane out of a state in LDS.
__device__ inline floatx4 state_quad(const float* state, int quad, int lane) {
  return ((const floatx4*)state)[quad * kWave + lane];
}


// The eight running states of a piece become ONE partial: every wavefront puts its state in
// LDS, and after one barrier wavefront w merges accumulator registers 8 w .. 8 w + 7 of the
// eight states (always in wavefront order, so the result does not depend on timing) and
// stores that slice of the partial; wavefront 0 also stores the row maxima and sums.
// kScaled (fp8 cache): the partial leaves in true units, row maxima times m_scale, O times o_scale.
// kSlotRows / qt: the slot holds kSlotRows rows and this is its row tile qt.
// kLoadsInFlight: the caller has global loads outstanding that the barriers must not wait for (the next piece's
// first tile); the barriers then only wait for this wavefront's LDS traffic.
// kFinish: the wavefront's slice goes to finish_part instead.
template <bool kScaled = false, int kSlotRows = kSmallRows, bool kLoadsInFlight = false, bool kFinish = false>
__device__ inline void fold_and_store(const SmallState& S, float* lds, float* slot, int wv, int lane, float c,
                                      float m_scale = 1.f, float o_scale = 1.f, int qt = 0,
                                      const FinishArgs* fa = nullptr, const Finish* f = nullptr, int early = 0) {
  const int h = lane >> 5, j = lane & 31;
  state_to_lds(S, lds + wv * kStateFloats, lane);
  if (kLoadsInFlight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else
    __syncthreads();
  float mk[kWgWaves], lk[kWgWaves];
#pragma unroll
  for (int k = 0; k < kWgWaves; ++k) {
    mk[k] = lds[k * kStateFloats + 64 * kWave + lane];
    lk[k] = lds[k * kStateFloats + 65 * kWave + lane];
  }
  floatx4 part[kWgWaves][2];
#pragma unroll
  for (int k = 0; k < kWgWaves; ++k)
#pragma unroll
    for (int u = 0; u < 2; ++u) part[k][u] = state_quad(lds + k * kStateFloats, 2 * wv + u, lane);
  float m_new = mk[0];
#pragma unroll
  for (int k = 1; k < kWgWaves; ++k) m_new = fmaxf(m_new, mk[k]);
  float l_new = 0.f;
  floatx4 x[2] = {(floatx4)(0.f), (floatx4)(0.f)};
#pragma unroll
  for (int k = 0; k < kWgWaves; ++k) {
    // an empty state has max -inf and contributes nothing
    const float sc = mk[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mk[k] - m_new) * c);
    l_new += lk[k] * sc;
    x[0] += part[k][0] * sc;
    x[1] += part[k][1] * sc;
  }
  if (kScaled) {
    x[0] *= o_scale;
    x[1] *= o_scale;
    m_new *= m_scale;  // (-inf stays -inf)
  }
  if (kFinish) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the next piece reuses the LDS regions
    finish_part<kSlotRows == kSmallRows ? 0 : 1, 2>(*fa, *f, x, m_new, sum_across_halves(l_new), 2 * wv, qt, early, wv, lane);
    return;
  }
  // accumulator register 16 jt + 4 r4 + i of lane (h, j) is row j, head dims 4 (8 jt + 2 r4 + h) + i
  const int jt = wv >> 1, r4 = 2 * (wv & 1);
  *(floatx4*)(slot + ((size_t)(qt * 32 + jt * 8 + 2 * r4 + h) * 32 + j) * 4) = x[0];
  *(floatx4*)(slot + ((size_t)(qt * 32 + jt * 8 + 2 * (r4 + 1) + h) * 32 + j) * 4) = x[1];
  if (wv == 0) {
    const float lsum = sum_across_halves(l_new);
    if (h == 0) {
      slot[kSlotRows * kD + qt * 32 + j] = m_new;
      slot[kSlotRows * kD + kSlotRows + qt * 32 + j] = lsum;
    }
  }
  // the next piece reuses the LDS regions
  if (kLoadsInFlight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else
    __syncthreads();
}

// The plan entries of 64 consecutive sequences, one per lane, fetched with one
// round trip; a worker's range rarely leaves the window it starts in.
struct PlanWindow {
  int first;          // sequence held by lane 0
  int64_t cum_units;  // lane i: units before sequence first + i (entry `batch` included)
  int32_t cum_segs;
  int32_t cu_nodes;
  int32_t len, n, tiles, rg;
  int64_t total_units;  // entry 64 of a window that holds a whole batch of 64 (uniform)
};

// Units before the sequence at window index i (0 .. 64).
__device__ inline int64_t window_cum_units(const PlanWindow& w, int i) {
  return i < kWave ? readlane64(w.cum_units, i) : w.total_units;
}

// A workgroup's copy of the plan when its first wavefront derived it (batches of at most 64).
struct PlanShare {
  int64_t cum_units[kClasses][kWave];
  int32_t cum_segs[kClasses][kWave];
  int32_t cu[kWave];
  SeqInfo info[kWave];
  int64_t units[kClasses], workers[kClasses], first_wg[kClasses + 1];
};

__device__ inline void load_window(PlanWindow& w, const PlanView& pv, const int32_t* cu_nodes,
                                   int cls, int batch, int first, int lane) {
  w.first = first;
  const int e = min(first + lane, batch);      // entries 0 .. batch exist
  const int b = min(first + lane, batch - 1);  // per-sequence info exists for 0 .. batch - 1
  w.cum_units = pv.cum_units[cls][e];
  w.cum_segs = pv.cum_segs[cls][e];
  w.cu_nodes = cu_nodes[e];
  const SeqInfo si = pv.info[b];
  w.len = si.len;
  w.n = si.n;
  w.tiles = si.tiles;
  w.rg = si.rg;
  w.total_units = 0;  // never read: such a window is reloaded before its last lane is passed
}

__device__ inline SeqInfo window_info(const PlanWindow& w, int b) {
  const int i = b - w.first;
  SeqInfo si;
  si.len = __builtin_amdgcn_readlane(w.len, i);
  si.n = __builtin_amdgcn_readlane(w.n, i);
  si.tiles = __builtin_amdgcn_readlane(w.tiles, i);
  si.rg = __builtin_amdgcn_readlane(w.rg, i);
  return si;
}

// What a worker needs of the plan: its class's unit and worker counts, and the window (held in
// registers for the whole batch when the wavefront planned for itself, else loaded from the
// plan in memory as the worker moves along).
struct ClassPlan {
  int64_t U, W;
  bool resident;
  PlanWindow win;
};

// Sequence that holds unit u0 of class `cls`, with its plan window loaded.
__device__ inline int locate(ClassPlan& cp, const PlanView& pv, const int32_t* cu_nodes, int cls,
                             int batch, int64_t u0, int lane) {
  if (batch <= kWave) {
    if (!cp.resident) load_window(cp.win, pv, cu_nodes, cls, batch, 0, lane);
    // cum_units is non-decreasing: the lanes with cum <= u0 are a prefix, its last lane is b
    const uint64_t below = __ballot(lane < batch && cp.win.cum_units <= u0);
    return __popcll(below) - 1;
  }
  const int b = find_sequence(pv.cum_units[cls], batch, u0);
  load_window(cp.win, pv, cu_nodes, cls, batch, b, lane);
  return b;
}

// Moves the window along when sequence b is its last lane (a resident window never moves).
__device__ inline void follow(ClassPlan& cp, const PlanView& pv, const int32_t* cu_nodes, int cls, int batch,
                              int b, int lane) {
  if (!cp.resident && b - cp.win.first >= kWave - 1) load_window(cp.win, pv, cu_nodes, cls, batch, b, lane);
}

// One workgroup of eight wavefronts per worker (two per SIMD).  Worker w owns
// units [w U / W, (w+1) U / W) of class 0; every piece of that range (its
// intersection with one (sequence, kv head) segment) is cut into eight
// contiguous sub-ranges, one per wavefront, and the eight running states are
// folded together through LDS after one barrier (fold_and_store), so that a
// piece leaves ONE partial in memory however many wavefronts streamed it.
constexpr int kSmallWaves = kWgWaves;

// A piece: the part of a worker's unit range that lies in one (sequence, kv head) segment.
struct SmallPiece {
  int b, g, base, t0, nt;  // (kFinish: a segment's tree part counts as its tile si.tiles)
  int units;               // of the worker's range that the piece takes up
  int64_t seg, ub;         // segment of the class, its first unit
  SeqInfo si;
  bool valid;
};

// The piece that starts at unit u0 of the worker's range [.., u1) (sequences without units of this class are
// skipped; b moves along).
template <bool kFinish>
__device__ inline SmallPiece small_piece(ClassPlan& cp, const PlanView& pv, const MainArgs& a, int64_t u0, int64_t u1,
                                         int& b, int lane) {
  SmallPiece p;
  p.valid = false;
  PlanWindow& win = cp.win;
  while (u0 < u1 && b < a.batch) {
    follow(cp, pv, a.cu_nodes, 0, a.batch, b, lane);
    const int64_t seq_begin = window_cum_units(win, b - win.first);
    const int64_t seq_end = window_cum_units(win, b + 1 - win.first);
    if (u0 >= seq_end) { ++b; continue; }
    p.si = window_info(win, b);
    // (the divisions run on the vector unit; everything is wavefront-uniform and goes back to scalar registers)
    const int64_t local = u0 - seq_begin;
    const int units = segment_units<kFinish>(p.si, a.tree_cost);
    p.b = __builtin_amdgcn_readfirstlane(b);
    p.g = __builtin_amdgcn_readfirstlane((int)(local / units));
    p.t0 = __builtin_amdgcn_readfirstlane((int)(local % units));
    const int64_t left = u1 - u0;
    p.nt = __builtin_amdgcn_readfirstlane((int)(left < (int64_t)(units - p.t0) ? left : (int64_t)(units - p.t0)));
    p.units = p.nt;
    if (kFinish) {
      p.ub = uniform64(u0 - p.t0);
      const int end = p.t0 + p.nt;
      p.t0 = min(p.t0, p.si.tiles);
      p.nt = min(end, p.si.tiles) - p.t0 + (end == units ? 1 : 0);
    }
    p.seg = uniform64((int64_t)__builtin_amdgcn_readlane(win.cum_segs, b - win.first) + p.g);
    p.base = __builtin_amdgcn_readlane(win.cu_nodes, b - win.first);
    p.valid = true;
    break;
  }
  return p;
}

// Pulls what a wavefront reads first of its share of piece p into the L2 cache: the share's first K/V tile (128
// lines of 128 bytes: lanes 0..31 the first cache block, 32..63 the second), the block ids of its first 64 tiles and
// the query rows.  One dword per lane and line; the values are not used, only kept until the caller has folded the
// current piece, so the requests are in flight during the fold and the share then starts on L2 hits.
__device__ inline void small_touch(uint32_t (&touched)[4], const MainArgs& a, const SmallPiece& p, int s0, int32_t blk0,
                                   int32_t blk1, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const int64_t page = clamp_block(h ? blk1 : blk0, a.num_blocks) * a.block_stride + (int64_t)p.g * a.head_stride;
  touched[0] = *(const uint32_t*)(a.k_cache + page + j * 64);
  touched[1] = *(const uint32_t*)(a.v_cache + page + j * 64);
  const int32_t* bt_row = a.block_table + (int64_t)p.b * a.max_blocks;
  const int n_blocks = (p.si.len + kBlock - 1) / kBlock;
  touched[2] = (uint32_t)bt_row[min(2 * s0 + 2 * lane, n_blocks - 1)];
  const int M = p.si.n * a.G;
  const int rho = j < M ? j : M - 1;
  const int node = p.base + rho / a.G, head = p.g * a.G + rho % a.G;
  touched[3] = *(const uint32_t*)(a.q + ((int64_t)node * a.Hq + head) * kD + h * 64);
}

template <bool kFinish>
__device__ inline void small_worker(const MainArgs& a0, int64_t w, ClassPlan& cp, float* merge_lds /* 132 KB: eight states */) {
  const int64_t U = cp.U, W = cp.W;
  if (w >= W || U <= 0) return;
  int64_t u0 = (w * U) / W;
  const int64_t u1 = ((w + 1) * U) / W;
  if (u0 >= u1) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int b = locate(cp, plan_view(a0.plan, a0.batch), a0.cu_nodes, 0, a0.batch, u0, lane);
  SmallPiece cur = small_piece<kFinish>(cp, plan_view(a0.plan, a0.batch), a0, u0, u1, b, lane);
  while (cur.valid) {
    const MainArgs a = kFinish ? kernel_args() : a0;
    const PlanView pv = plan_view(a.plan, a.batch);
    // The piece after this one is located first: what this wavefront will read first of it is requested before
    // the fold of this piece, so that the stream does not start from memory latency at every piece boundary.
    const SmallPiece nxt = small_piece<kFinish>(cp, pv, a, u0 + cur.units, u1, b, lane);
    // this wavefront's share of the piece, and of the next
    const int s0 = cur.t0 + (int)(((int64_t)cur.nt * wv) / kSmallWaves);
    const int s1 = cur.t0 + (int)(((int64_t)cur.nt * (wv + 1)) / kSmallWaves);
    int n0 = 0, n1 = 0;
    if (nxt.valid) {
      n0 = nxt.t0 + (int)(((int64_t)nxt.nt * wv) / kSmallWaves);
      n1 = nxt.t0 + (int)(((int64_t)nxt.nt * (wv + 1)) / kSmallWaves);
    }
    const bool pre = n0 < (kFinish ? min(n1, nxt.si.tiles) : n1);
    // block ids of the next share's first tile: scalar loads, issued a whole share ahead
    int32_t nb0 = 0, nb1 = 0;
    if (pre) {
      const int32_t* row = a.block_table + (int64_t)nxt.b * a.max_blocks;
      const int nblk = (nxt.si.len + kBlock - 1) / kBlock;
      nb0 = sload(row + min(2 * n0, nblk - 1));
      nb1 = sload(row + min(2 * n0 + 1, nblk - 1));
    }
    Finish fin;
    if (kFinish)
      fin = finish_of(cur.ub, segment_units<true>(cur.si, a.tree_cost), U, W, w, cur.seg, cur.base, cur.g, cur.si.n * a.G, 0);
    SmallState S;
    small_segment(S, a, cur.b, cur.g, cur.base, s0, kFinish ? min(s1, cur.si.tiles) : s1, cur.si, lane);
    uint32_t touched[4] = {0u, 0u, 0u, 0u};
    if (kFinish) {
      const FinishArgs fa = kernel_args().fin;
      const int early = fin.pieces > 1 ? arrivals(counter_of<0>(fa, fin, wv)) : 0;
      if (pre) small_touch(touched, a, nxt, n0, nb0, nb1, lane);
      if (s1 > cur.si.tiles) tree_tile(S.o, S.m, S.l, fa, cur.base, cur.g, fin.rows, 0, cur.si.n, 0, lane);
      fold_and_store<false, kSmallRows, true, true>(S, merge_lds, nullptr, wv, lane, a.scale_log2e, 1.f, 1.f, 0, &fa, &fin, early);
    } else {
      if (pre) small_touch(touched, a, nxt, n0, nb0, nb1, lane);
      fold_and_store<false, kSmallRows, true>(S, merge_lds, a.ws[0] + (size_t)(w + cur.seg) * kSmallSlot, wv, lane,
                                              a.scale_log2e);
    }
    asm volatile("" ::"v"(touched[0]), "v"(touched[1]), "v"(touched[2]), "v"(touched[3]));
    u0 += cur.units;
    cur = nxt;
  }
}

// ---- fp8 cache: trees of up to 64 rows per kv head, streamed into registers ---------------------
//
// The same register-direct stream as class 0, with one or two row tiles per wavefront.

// A row group of two row tiles: every wavefront carries both, so a tile's bytes are loaded and converted once for the
// workgroup (they were streamed by two halves of the workgroup, each of which converted them: 64 sequences of 16384
// tokens, 40 .. 64 rows per kv head, took 626 us, as long as from a bf16 cache of twice the bytes; now 412).  Two states
// leave no registers for the queries: they lie in LDS in operand order (16 KB, read once per tile).

// Puts the 64 query rows of a row group into LDS ([row tile][k step][lane], 16 bytes each); ends with a barrier.
__device__ inline void pair_queries(bf16x8* lds_q, const MainArgs& a, int g, int base, int M, int wv, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const int rho_raw = (wv >> 2) * kSmallRows + j;
  const int rho = rho_raw < M ? rho_raw : M - 1;  // padding rows repeat the last real row; never read back
  const int node = base + rho / a.G, head = g * a.G + rho % a.G;
  const __bf16* qp = a.q + ((int64_t)node * a.Hq + head) * kD + h * 8;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ks = 2 * (wv & 3) + i;
    lds_q[((wv >> 2) * 8 + ks) * kWave + lane] = *(const bf16x8*)(qp + ks * 16);
  }
  __syncthreads();
}

template <bool kMore>
__device__ inline void pair_tile(SmallState (&S)[2], fp8x8 (&k)[8], fp8x8 (&v)[2][4], const bf16x8* lds_q, int lane,
                                 float c, const MainArgs& a, const TilePages& next, int n_valid) {
  floatx16 s[2] = {(floatx16)(0.f), (floatx16)(0.f)};
  // (the scheduling barriers keep the query reads two steps ahead and no further: their registers are not there)
  const uint8_t* kp = kMore ? k_vectors(a, next, lane) : nullptr;
  bf16x8 qx[2][2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) qx[0][rt] = lds_q[rt * 8 * kWave + lane];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    if (ks < 7) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) qx[(ks + 1) & 1][rt] = lds_q[(rt * 8 + ks + 1) * kWave + lane];
    }
    const bf16x8 kx = operand(k[ks]);
    if (kMore) k[ks] = stream_load<true>((const fp8x8*)(kp + ks * 256));
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) s[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx, qx[ks & 1][rt], s[rt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!kMore && n_valid < kTile) {  // only a share's last tile can be ragged
    mask_tail(s[0], v, n_valid, lane >> 5);
    mask_tail(s[1], v, n_valid, lane >> 5);
  }
  bf16x8 pb[2][2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    softmax_tile(s[rt], S[rt].m, S[rt].l, S[rt].o, pb[rt][0], pb[rt][1], c);
    __builtin_amdgcn_sched_barrier(0);
  }
  const uint8_t* vp[2] = {kMore ? v_vectors(a, next.page0, lane) : nullptr, kMore ? v_vectors(a, next.page1, lane) : nullptr};
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const bf16x8 vx = operand(v[kk][jt]);
      if (kMore) v[kk][jt] = stream_load<true>((const fp8x8*)(vp[kk] + jt * 256));
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
        S[rt].o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vx, pb[rt][kk], S[rt].o[jt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
}

// This wavefront's share [t0, t1) of a piece; the registers and requests are those of small_segment.
__device__ inline void pair_segment(SmallState (&S)[2], const bf16x8* lds_q, const MainArgs& a, int b, int g, int t0, int t1,
                                    const SeqInfo si, int lane) {
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) S[rt].o[jt] = (floatx16)(0.f);
    S[rt].m = -INFINITY;
    S[rt].l = 0.f;
  }
  if (t0 >= t1) return;
  const int32_t* bt_row = a.block_table + (int64_t)b * a.max_blocks;
  const int n_blocks = (si.len + kBlock - 1) / kBlock;
  const float c = a.scale_log2e;
  for (int tc = t0; tc < t1; tc += kChunkTiles) {
    const int te = min(t1, tc + kChunkTiles);
    BlockIds ids;
    ids.lo = bt_row[min(2 * tc + lane, n_blocks - 1)];
    ids.hi = bt_row[min(2 * tc + kWave + lane, n_blocks - 1)];
    asm volatile("" ::"v"(ids.lo), "v"(ids.hi));  // landed before the stream starts: see small_segment
    fp8x8 k[8], v[2][4];
    {
      const TilePages first = pages_from_ids(a, ids, 0, g);
      load_k<true>(k, a, first, lane);
      load_v<true>(v, a, first, lane);
    }
    const bool ends_here = te == t1;
    const int loop_end = ends_here ? te - 1 : te;
    int t = tc;
    for (; t < loop_end; ++t) {
      const TilePages next = pages_from_ids(a, ids, min(t + 1, te - 1) - tc, g);
      pair_tile<true>(S, k, v, lds_q, lane, c, a, next, kTile);
    }
    if (ends_here) pair_tile<false>(S, k, v, lds_q, lane, c, a, TilePages{0, 0}, si.len - t * kTile);
  }
}

// The eight states of a row group of two row tiles in LDS, row tile rt's in regions 4 rt .. 4 rt + 3, become one partial:
// wavefront w merges accumulator registers 16 (w % 4) .. + 15 of the four states of row tile w / 4 (always in region
// order) and stores that slice of the 64-row slot.
template <bool kFinish>
__device__ inline void fold_quads_and_store(float* lds, float* slot, int wv, int lane, float c, float m_scale, float o_scale,
                                            const FinishArgs* fa, const Finish* f, int early) {
  const int h = lane >> 5, j = lane & 31;
  const int rt = wv >> 2, part = wv & 3;
  float mk[4], lk[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    mk[k] = lds[(4 * rt + k) * kStateFloats + 64 * kWave + lane];
    lk[k] = lds[(4 * rt + k) * kStateFloats + 65 * kWave + lane];
  }
  const float m_new = fmaxf(fmaxf(mk[0], mk[1]), fmaxf(mk[2], mk[3]));
  float l_new = 0.f;
  floatx4 x[4] = {(floatx4)(0.f), (floatx4)(0.f), (floatx4)(0.f), (floatx4)(0.f)};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    // an empty state has max -inf and contributes nothing
    const float sc = mk[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mk[k] - m_new) * c);
    l_new += lk[k] * sc;
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] += state_quad(lds + (4 * rt + k) * kStateFloats, 4 * part + u, lane) * sc;
  }
  if (kFinish) {
    __syncthreads();  // the next piece reuses the LDS regions
    finish_part<1, 4>(*fa, *f, x, m_new, sum_across_halves(l_new), 4 * part, rt, early, wv, lane);
    return;
  }
  // accumulator register 16 jt + 4 r4 + i of lane (h, j) is row j, head dims 4 (8 jt + 2 r4 + h) + i; here jt = part, r4 = u
#pragma unroll
  for (int u = 0; u < 4; ++u)
    *(floatx4*)(slot + ((size_t)(rt * 32 + part * 8 + 2 * u + h) * 32 + j) * 4) = x[u] * o_scale;
  if (part == 0) {
    const float lsum = sum_across_halves(l_new);
    if (h == 0) {
      slot[kMediumRows * kD + rt * 32 + j] = m_new * m_scale;  // (-inf stays -inf)
      slot[kMediumRows * kD + kMediumRows + rt * 32 + j] = lsum;
    }
  }
  __syncthreads();  // the next piece reuses the LDS regions
}

// LDS holds eight states, not sixteen: wavefronts 4 .. 7 put their pairs there, wavefronts 0 .. 3 merge theirs with them
// and put the result back.
__device__ inline void fold_pairs_and_store(SmallState (&S)[2], float* lds, float* slot, int wv, int lane, float c,
                                            float m_scale, float o_scale) {
  if (wv >= 4) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) state_to_lds(S[rt], lds + (4 * rt + wv - 4) * kStateFloats, lane);
  }
  __syncthreads();
  if (wv < 4) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      float* region = lds + (4 * rt + wv) * kStateFloats;
      const float mk = region[64 * kWave + lane], lk = region[65 * kWave + lane];
      const float m_new = fmaxf(S[rt].m, mk);
      // an empty state has max -inf and contributes nothing
      const float a0 = S[rt].m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((S[rt].m - m_new) * c);
      const float a1 = mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mk - m_new) * c);
#pragma unroll
      for (int quad = 0; quad < 16; ++quad) {
        const floatx4 x = state_quad(region, quad, lane);
        floatx4 y;
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = S[rt].o[quad >> 2][4 * (quad & 3) + i] * a0 + x[i] * a1;
        ((floatx4*)region)[quad * kWave + lane] = y;  // (a lane's own words only)
      }
      region[64 * kWave + lane] = m_new;
      region[65 * kWave + lane] = S[rt].l * a0 + lk * a1;
    }
  }
  __syncthreads();
  fold_quads_and_store<false>(lds, slot, wv, lane, c, m_scale, o_scale, nullptr, nullptr, 0);
}

// (The loop of small_segment is 237 instructions long where the states are handed to the fold by reference as here, 247 with
// the same calls written out in the worker: 40 trees of 48 rows, 1500 tokens, prefix kernel 35.1 us instead of 36.3.)
template <bool kFinish>
__device__ inline void fold_halves_and_store(const SmallState& S, float* lds, float* slot, int wv, int lane, float c,
                                             float m_scale, float o_scale, const FinishArgs* fa, const Finish* f, int early) {
  state_to_lds(S, lds + wv * kStateFloats, lane);
  __syncthreads();
  fold_quads_and_store<kFinish>(lds, slot, wv, lane, c, m_scale, o_scale, fa, f, early);
}

// A worker's pieces.  kPair: two row tiles go to every wavefront; else one to each half of the workgroup (wavefronts 0 .. 3
// carry row tile 0, 4 .. 7 row tile 1, both halves stream the same tiles).
// kFinish: the states take on true units before the tree part (its keys and values have no scales) and the fold; the tree
// part goes to a row tile's last wavefront, or its last two.
__device__ inline void to_true_units(SmallState& S, float m_scale, float o_scale) {
  S.m *= m_scale;  // (-inf stays -inf)
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) S.o[jt] *= o_scale;
}

template <bool kPair, bool kFinish>
__device__ inline void fp8_pieces(const MainArgs& a0, int64_t w, ClassPlan& cp, float* merge_lds, int64_t u0, int64_t u1, int b,
                                  int wv, int lane) {
  PlanWindow& win = cp.win;
  for (;;) {
    const MainArgs a = kFinish ? kernel_args() : a0;
    if (!(u0 < u1 && b < a.batch)) break;
    const PlanView pv = plan_view(a.plan, a.batch);
    follow(cp, pv, a.cu_nodes, 1, a.batch, b, lane);
    const int64_t seq_begin = window_cum_units(win, b - win.first);
    const int64_t seq_end = window_cum_units(win, b + 1 - win.first);
    if (u0 >= seq_end) { ++b; continue; }
    const SeqInfo si = window_info(win, b);
    const int64_t local = u0 - seq_begin;
    const int units = segment_units<kFinish>(si, a.tree_cost);
    const int g = (int)(local / units);  // (one row group: class 1 has at most 64 rows)
    const int begin = (int)(local % units);
    const int64_t left = u1 - u0;
    const int end = begin + (int)(left < (int64_t)(units - begin) ? left : (int64_t)(units - begin));
    // prefix tiles t0 .. t1 of the piece; its tree part counts as one more
    const int t0 = kFinish ? min(begin, si.tiles) : begin, t1 = kFinish ? min(end, si.tiles) : end;
    const bool tree = kFinish && end == units;
    const int nt = t1 - t0 + (tree ? 1 : 0);
    const int64_t seg = (int64_t)__builtin_amdgcn_readlane(win.cum_segs, b - win.first) + g;
    const int base = __builtin_amdgcn_readlane(win.cu_nodes, b - win.first);
    const int M = si.n * a.G;
    float* slot = kFinish ? nullptr : a.ws[1] + (size_t)(w + seg) * kMediumSlot;
    Finish fin;
    if (kFinish) fin = finish_of(u0 - begin, units, cp.U, cp.W, w, seg, base, g, M, 0);
    FinishArgs fa;
    int early = 0;
    float c = a.scale_log2e, m_scale = a.m_scale, o_scale = a.o_scale;
    auto streamed = [&]() {
      if (!kFinish) return;
      const MainArgs z = kernel_args();
      fa = z.fin;
      c = fa.scale_log2e;
      m_scale = z.m_scale;
      o_scale = z.o_scale;
      if (fin.pieces > 1) early = arrivals(counter_of<1>(fa, fin, wv));
    };
    auto cut = [&](int part, int of) {
      const int t = t0 + (int)(((int64_t)nt * part) / of);
      return kFinish ? min(t1, t) : t;
    };
    const int s0 = cut(wv, kWgWaves), s1 = cut(wv + 1, kWgWaves);
    if (M <= kSmallRows) {
      SmallState S;
      small_segment<fp8x8>(S, kFinish ? stream_args(a) : a, b, g, base, s0, s1, si, lane);
      streamed();
      if (kFinish) to_true_units(S, m_scale, o_scale);
      if (tree && wv == kWgWaves - 1) tree_tile(S.o, S.m, S.l, fa, base, g, M, 0, si.n, 0, lane);
      fold_and_store<!kFinish, kMediumRows, false, kFinish>(S, merge_lds, slot, wv, lane, c, m_scale, o_scale, 0, &fa, &fin,
                                                            early);
    } else if (kPair) {
      bf16x8* lds_q = (bf16x8*)merge_lds;  // (the fold's regions: one after the other)
      pair_queries(lds_q, a, g, base, M, wv, lane);
      SmallState P[2];
      pair_segment(P, lds_q, a, b, g, s0, s1, si, lane);
      __syncthreads();  // nobody reads the queries any more
      fold_pairs_and_store(P, merge_lds, slot, wv, lane, c, m_scale, o_scale);
    } else {
      const int rt = wv >> 2, sub = wv & 3;
      const int h0 = cut(sub, 4), h1 = cut(sub + 1, 4);
      SmallState S;
      small_segment<fp8x8, false>(S, kFinish ? stream_args(a) : a, b, g, base, h0, h1, si, lane, rt * kSmallRows);
      streamed();
      if (kFinish) to_true_units(S, m_scale, o_scale);
      if (tree && sub >= 2 && 32 * (3 - sub) < si.n)
        tree_tile(S.o, S.m, S.l, fa, base, g, M, rt * kSmallRows, si.n, 3 - sub, lane);
      fold_halves_and_store<kFinish>(S, merge_lds, slot, wv, lane, c, kFinish ? 1.f : m_scale, kFinish ? 1.f : o_scale, &fa,
                                     &fin, early);
    }
    u0 += end - begin;
  }
}

// A pair costs more to start (queries through LDS) and to fold (two states per wavefront), so it needs long pieces.  Whole
// calls, 64 / 8 heads of 8 nodes, halves against pairs: 32 sequences of 500 tokens 26.9 / 32.9 us, 1500 (47 tiles) 40.0 /
// 44.9, 2500 (79) 58.1 / 57.5, 4000 (125) 82.8 / 74.3, 8000 154 / 118; 2 sequences of 4000 (17 tiles a piece) 32.0 / 37.3.
// A worker whose share or whose first sequence is shorter than this, or whose first tree has one row tile, goes through its
// pieces without them (decided once per worker and in a loop of its own: decided per piece in one loop, spilled registers are
// reloaded in every piece behind the loads in flight: 32 sequences of 1500 tokens 44.5 us, this way 40.9).
constexpr int kPairTiles = 72;
// kPair: of the kernel, which can do both; it runs the other loop a little slower than the kernel that has only that one (60
// trees of one row tile and 4 of class 2, 9000 tokens, 238 us against 237; 20 trees of 48 and 20 of 80 rows, 1500 tokens, 70
// against 67), so a batch that cannot have long pieces runs that: see tva_launch_mfma.
template <bool kPair, bool kFinish>
__device__ inline void fp8_worker(const MainArgs& a, int64_t w, ClassPlan& cp, float* merge_lds /* 132 KB */) {
  const PlanView pv = plan_view(a.plan, a.batch);
  const int64_t U = cp.U, W = cp.W;
  if (w >= W || U <= 0) return;
  const int64_t u0 = (w * U) / W, u1 = ((w + 1) * U) / W;
  if (u0 >= u1) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = locate(cp, pv, a.cu_nodes, 1, a.batch, u0, lane);
  if (kPair && b < a.batch) {
    follow(cp, pv, a.cu_nodes, 1, a.batch, b, lane);
    const SeqInfo first = window_info(cp.win, b - cp.win.first);
    if (u1 - u0 >= kPairTiles && first.tiles >= kPairTiles && first.n * a.G > kSmallRows) {
      fp8_pieces<true, false>(a, w, cp, merge_lds, u0, u1, b, wv, lane);
      return;
    }
  }
  fp8_pieces<false, kFinish>(a, w, cp, merge_lds, u0, u1, b, wv, lane);
}

// ---- classes 1 and 2: K/V tiles staged in LDS, shared by the eight wavefronts of a workgroup --
//
// A workgroup of eight wavefronts (two per SIMD) is the worker.  A tile (16 KB: 8 K + 8 V
// operand vectors per lane) is fetched from HBM once per workgroup, each wavefront requesting
// an eighth of it, straight into LDS in operand order -- the vector a lane will feed to the
// MFMA sits at [instruction][lane], so reads are 16 bytes per lane at consecutive addresses,
// free of bank conflicts.
//   class 2 (more than 64 rows): row groups of up to 256 rows, wavefront w carries rows
//     32 w .. 32 w + 31; one tile per iteration and barrier; the score product of the next
//     tile is woven into the softmax of the current one (staged_segment).
//   class 1 (33 .. 64 rows): row tile = w / 2 (tiles 0 and 1 have rows), key group = w % 2;
//     two tiles per iteration, one per key group; the two states of a row tile are folded
//     through LDS at the end of the segment (grouped_segment).
// K/V tiles travel HBM -> LDS without passing through registers (global_load_lds, 16 bytes a
// lane).  A stage holds one 32-key tile in operand order: eight K vectors (k steps) then
// eight V vectors (cache block kk, d tile jt at 4 kk + jt), 64 lanes x 16 bytes each;
// wavefront w fetches vectors 2 w and 2 w + 1 of every tile.  kStages tiles are in flight.
constexpr int kStages = 8;
constexpr int kStageVecs = 16 * kWave;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_void;

__device__ inline uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_void*)p; }

// What a lane fetches of every tile: fixed offset inside a page, and which of the tile's two
// pages (mask all ones: the second).
struct FetchLane {
  const __bf16* base;
  int64_t second_page;
};

__device__ inline FetchLane fetch_lane(const MainArgs& a, int wv, int lane) {
  const int h = lane >> 5, j = lane & 31;
  FetchLane f;
  if (wv < 4) {  // K vectors of k steps 2 wv, 2 wv + 1: key row j, head dims 16 ks + 8 h ..
    f.base = a.k_cache + (h * 16 + sigma(j & 15)) * 8 + wv * 2 * 256;
    f.second_page = -(int64_t)(j >> 4);
  } else {  // V vectors of cache block (wv - 4) / 2, d tiles 2 ((wv - 4) % 2) + {0, 1}
    f.base = a.v_cache + (h * kD + j) * 8 + 2 * ((wv - 4) & 1) * 256;
    f.second_page = -(int64_t)((wv - 4) >> 1);
  }
  return f;
}

// `again`: the tile is requested more than once -- a request past the end of a segment repeats the segment's last
// tile so that every iteration issues the same number of requests (it is never consumed), and a tree with several row
// groups streams the prefix once per group.  Such requests are left cacheable, so that the repeats can hit in L2 or
// the last-level cache instead of going to memory like the read-once stream does.
__device__ inline void request_tile(const MainArgs& a, const FetchLane& f, int32_t blk0, int32_t blk1, int g,
                                    bf16x8* stage, int wv, bool again) {
  const int64_t page0 = clamp_block(blk0, a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  const int64_t page1 = clamp_block(blk1, a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  const __bf16* src = f.base + (page0 ^ ((page0 ^ page1) & f.second_page));
  bf16x8* dst = stage + 2 * wv * kWave;
  if (again) {
    __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)dst, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 256), (lds_void*)(dst + kWave), 16, 0, 0);
  } else {
    __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)dst, 16, 0, kStreamPolicy);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 256), (lds_void*)(dst + kWave), 16, 0, kStreamPolicy);
  }
}

// The same tile out of an fp8 cache.  The pages have the same element order with one byte per element, so the two
// operand vectors a lane is responsible for are 8 bytes each, 256 bytes apart.  They travel HBM -> LDS as four
// dwords per lane (the LDS-direct load takes 4 or 16 bytes a lane) into this wavefront's 1 KB of a raw slot:
// plane p of 64 dwords holds dword p of every lane (vector 0 low, vector 0 high, vector 1 low, vector 1 high).
// convert_tile_fp8 then turns them into the two bf16 operand vectors of the stage, exactly (E4M3 -> bf16).
__device__ inline FetchLane fetch_lane_fp8(const MainArgs& a, int wv, int lane) {
  const int h = lane >> 5, j = lane & 31;
  const uint8_t* kb = (const uint8_t*)a.k_cache;
  const uint8_t* vb = (const uint8_t*)a.v_cache;
  FetchLane f;
  if (wv < 4) {
    f.base = (const __bf16*)(kb + (h * 16 + sigma(j & 15)) * 8 + wv * 2 * 256);
    f.second_page = -(int64_t)(j >> 4);
  } else {
    f.base = (const __bf16*)(vb + (h * kD + j) * 8 + 2 * ((wv - 4) & 1) * 256);
    f.second_page = -(int64_t)((wv - 4) >> 1);
  }
  return f;
}

__device__ inline void request_tile_fp8(const MainArgs& a, const FetchLane& f, int32_t blk0, int32_t blk1, int g,
                                        uint32_t* raw /* this wavefront's 4 x 64 dwords of the slot */, bool again) {
  const int64_t page0 = clamp_block(blk0, a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  const int64_t page1 = clamp_block(blk1, a.num_blocks) * a.block_stride + (int64_t)g * a.head_stride;
  const uint8_t* src = (const uint8_t*)f.base + (page0 ^ ((page0 ^ page1) & f.second_page));
  if (again) {
    __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)raw, 4, 0, 0);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 4), (lds_void*)(raw + kWave), 4, 0, 0);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 256), (lds_void*)(raw + 2 * kWave), 4, 0, 0);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 260), (lds_void*)(raw + 3 * kWave), 4, 0, 0);
  } else {
    __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)raw, 4, 0, kStreamPolicy);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 4), (lds_void*)(raw + kWave), 4, 0, kStreamPolicy);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 256), (lds_void*)(raw + 2 * kWave), 4, 0, kStreamPolicy);
    __builtin_amdgcn_global_load_lds((global_void*)(src + 260), (lds_void*)(raw + 3 * kWave), 4, 0, kStreamPolicy);
  }
}

// raw_addr: LDS byte address of this lane's dword in plane 0 of the raw slot; dst_addr: that of its first operand
// vector in the stage (the second is 64 vectors further).  Written as assembly like the operand reads: an LDS access
// the compiler can see makes it wait for every LDS-direct load in flight.  Ends with the writes done.
__device__ inline void convert_tile_fp8(uint32_t raw_addr, uint32_t dst_addr) {
  uint32_t d0, d1, d2, d3;
  asm volatile(
      "ds_read_b32 %0, %4\n\t"
      "ds_read_b32 %1, %4 offset:256\n\t"
      "ds_read_b32 %2, %4 offset:512\n\t"
      "ds_read_b32 %3, %4 offset:768\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3)
      : "v"(raw_addr)
      : "memory");
  fp8x8 r0, r1;
  r0[0] = d0, r0[1] = d1, r1[0] = d2, r1[1] = d3;
  const bf16x8 b0 = operand(r0), b1 = operand(r1);
  asm volatile(
      "ds_write_b128 %0, %1\n\t"
      "ds_write_b128 %0, %2 offset:1024\n\t"
      "s_waitcnt lgkmcnt(0)"
      :
      : "v"(dst_addr), "v"(b0), "v"(b1)
      : "memory");
}

// LDS reads of the staged tiles are written as assembly: the compiler would otherwise wait
// for every outstanding global_load_lds before each read it can see.  The counter waits
// below carry the registers they release as operands, so that no use can move above them.
#define SMART_LDS_READ(dst, addr, OFFSET) \
  asm volatile("ds_read_b128 %0, %1 offset:" #OFFSET : "=v"(dst) : "v"(addr) : "memory")
#define SMART_LDS_WAIT(reg, N) asm volatile("s_waitcnt lgkmcnt(" #N ")" : "+v"(reg) : : "memory")

__device__ inline void lds_read_half(bf16x8 (&r)[8], uint32_t addr, int half) {
  if (half == 0) {
    SMART_LDS_READ(r[0], addr, 0);
    SMART_LDS_READ(r[1], addr, 1024);
    SMART_LDS_READ(r[2], addr, 2048);
    SMART_LDS_READ(r[3], addr, 3072);
  } else {
    SMART_LDS_READ(r[4], addr, 4096);
    SMART_LDS_READ(r[5], addr, 5120);
    SMART_LDS_READ(r[6], addr, 6144);
    SMART_LDS_READ(r[7], addr, 7168);
  }
}

// The V fetchers clear the entries of tokens >= n_valid in their two vectors of a landed
// stage (ragged end of a prefix; unowned slots may hold NaN).
__device__ inline void zero_invalid_v_lds(bf16x8* stage, int wv, int lane, int n_valid) {
  if (wv < 4) return;
  const int h = lane >> 5, kk = (wv - 4) >> 1;
  const uint32_t addr = lds_address(stage + 2 * wv * kWave + lane);
  bf16x8 v0, v1;
  SMART_LDS_READ(v0, addr, 0);
  SMART_LDS_READ(v1, addr, 1024);
  SMART_LDS_WAIT(v0, 0);
  SMART_LDS_WAIT(v1, 0);
#pragma unroll
  for (int x = 0; x < 8; ++x)
    if (kk * 16 + h * 8 + x >= n_valid) {
      v0[x] = (__bf16)0.f;
      v1[x] = (__bf16)0.f;
    }
  asm volatile("ds_write_b128 %0, %1\n\tds_write_b128 %0, %2 offset:1024\n\ts_waitcnt lgkmcnt(0)"
               :
               : "v"(addr), "v"(v0), "v"(v1)
               : "memory");
}

__device__ inline void mask_scores(floatx16& s, int n_valid, int h) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * h + (r & 3);
    const int tok = (i & 16) + sigma(i & 15);
    if (tok >= n_valid) s[r] = -INFINITY;
  }
}

// Scores of one staged tile (used for the first tile of a segment only).
__device__ inline void score_tile(floatx16& s, uint32_t k_addr, const bf16x8 (&q)[8]) {
  bf16x8 kop[8];
  lds_read_half(kop, k_addr, 0);
  lds_read_half(kop, k_addr, 1);
  SMART_LDS_WAIT(kop[0], 0);
  s = (floatx16)(0.f);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    if (ks > 0) SMART_LDS_WAIT(kop[ks], 0);
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[ks], q[ks], s, 0, 0, 0);
  }
}

// One iteration of a wavefront with rows: softmax and output product of tile t (scores
// s_in, V at v_addr) with the score product of tile t + 1 (K at k_addr, result s_out) woven
// in, so that the matrix cores run in the shadow of the exponentials:
//   8 x { score MFMA k step i | exp of first-half probability i }
//   4 x { output MFMA (first cache block, d tile jt) | exp of second-half probabilities 2 jt, 2 jt + 1 }
//   4 x   output MFMA (second cache block)
// The scheduling barriers keep that order.  `between` runs after the first LDS reads are
// issued (the caller's fetch requests go there, in the shadow of the LDS latency).  The
// counts of the LDS waits follow the order in which the 16 reads are issued: K 0..7 and
// V 0..3 up front, V 4..7 after the fourth score step.
template <typename Between>
__device__ inline void woven_tile(const floatx16& s, floatx16& s_next, floatx16 (&o)[4], float& m, float& l,
                                  const bf16x8 (&q)[8], uint32_t k_addr, uint32_t v_addr, float c,
                                  Between between) {
  bf16x8 kop[8], vop[8];
  lds_read_half(kop, k_addr, 0);
  lds_read_half(kop, k_addr, 1);
  lds_read_half(vop, v_addr, 0);
  between();
  float mx = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
  mx = max_across_halves(mx);
  const float m_new = fmaxf(m, mx);
  if (__any((m_new - m) * c > kRescaleStep)) {  // the reference follows the maximum in steps: see kRescaleStep
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
    l *= alpha;
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) o[jt] *= alpha;
    m = m_new;
  }
  const float mc = m * c;
  s_next = (floatx16)(0.f);
  floatx8 p0, p1;
  float sum = 0.f;
  __builtin_amdgcn_sched_barrier(0);
#define SMART_SCORE_STEP(I, N)                                                        \
  SMART_LDS_WAIT(kop[I], N);                                                          \
  s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[I], q[I], s_next, 0, 0, 0);    \
  p0[I] = __builtin_amdgcn_exp2f(fmaf(s[I], c, -mc));                                 \
  sum += p0[I];                                                                       \
  __builtin_amdgcn_sched_barrier(0);
  SMART_SCORE_STEP(0, 11)
  SMART_SCORE_STEP(1, 10)
  SMART_SCORE_STEP(2, 9)
  SMART_SCORE_STEP(3, 8)
  lds_read_half(vop, v_addr, 1);  // outstanding: K 4..7, V 0..7
  SMART_SCORE_STEP(4, 11)
  SMART_SCORE_STEP(5, 10)
  SMART_SCORE_STEP(6, 9)
  SMART_SCORE_STEP(7, 8)
#undef SMART_SCORE_STEP
  const bf16x8 pb0 = __builtin_convertvector(p0, bf16x8);
  __builtin_amdgcn_sched_barrier(0);
#define SMART_OUTPUT_STEP(JT, N)                                                      \
  SMART_LDS_WAIT(vop[JT], N);                                                         \
  o[JT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[JT], pb0, o[JT], 0, 0, 0);      \
  p1[2 * JT] = __builtin_amdgcn_exp2f(fmaf(s[8 + 2 * JT], c, -mc));                   \
  p1[2 * JT + 1] = __builtin_amdgcn_exp2f(fmaf(s[9 + 2 * JT], c, -mc));               \
  sum += p1[2 * JT] + p1[2 * JT + 1];                                                 \
  __builtin_amdgcn_sched_barrier(0);
  SMART_OUTPUT_STEP(0, 7)
  SMART_OUTPUT_STEP(1, 6)
  SMART_OUTPUT_STEP(2, 5)
  SMART_OUTPUT_STEP(3, 4)
#undef SMART_OUTPUT_STEP
  l += sum;
  const bf16x8 pb1 = __builtin_convertvector(p1, bf16x8);
  SMART_LDS_WAIT(vop[4], 3);
  o[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[4], pb1, o[0], 0, 0, 0);
  SMART_LDS_WAIT(vop[5], 2);
  o[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[5], pb1, o[1], 0, 0, 0);
  SMART_LDS_WAIT(vop[6], 1);
  o[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[6], pb1, o[2], 0, 0, 0);
  SMART_LDS_WAIT(vop[7], 0);
  o[3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[7], pb1, o[3], 0, 0, 0);
}

// All eight wavefronts of the workgroup run this together (it contains barriers);
// kRows = false marks a wavefront without rows in this row group: it only helps to fetch.
// kFp8: the cache holds E4M3 bytes.  LDS then holds four bf16 stages (a tile is used during two iterations) and,
// behind them, kStages raw slots of 8 KB; a wavefront converts its own share of tile t + 1 as soon as it has
// landed (nobody else touches those bytes), before the barrier that publishes the stage.
// kFinish: tiles t0 .. t1 may be none, `tree`: the segment's tree part belongs to this piece; the rows go to finish_part.
template <bool kRows, bool kFp8 = false, bool kFinish = false>
__device__ inline void staged_segment(const MainArgs& a, int b, int g, int base, int row0, int t0, int t1,
                                      const SeqInfo si, float* slot, int wv, int lane, bf16x8* lds, bool tree = false,
                                      const Finish* fin = nullptr) {
  constexpr int kRing = kFp8 ? 4 : kStages;  // bf16 stages
  constexpr int kLoads = kFp8 ? 4 : 2;       // vector-memory loads per tile and wavefront
  const int h = lane >> 5, j = lane & 31;
  const int M = si.n * a.G;
  floatx16 o[4];
  bf16x8 q[8];
  float m = -INFINITY, l = 0.f;
  if (kRows) {
    int rho = row0 + j;
    rho = rho < M ? rho : M - 1;  // padding rows repeat the last real row; never read back
    const int node = base + rho / a.G, head = g * a.G + rho % a.G;
    const __bf16* qp = a.q + ((int64_t)node * a.Hq + head) * kD + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ks] = *(const bf16x8*)(qp + ks * 16);
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) o[jt] = (floatx16)(0.f);
    // (not waited for here: the tile requests below are younger loads, so the wait for the first tile covers these)
  }
  const int32_t* bt_row = a.block_table + (int64_t)b * a.max_blocks;
  const int n_blocks = (si.len + kBlock - 1) / kBlock;
  const float c = a.scale_log2e;
  const FetchLane f = kFp8 ? fetch_lane_fp8(a, wv, lane) : fetch_lane(a, wv, lane);
  const uint32_t rd = lds_address(lds + lane);  // this lane's slice of vector 0 of stage 0
  const int last = t1 - 1;
  auto stage_of = [&](int t) { return lds + (t & (kRing - 1)) * kStageVecs; };
  // fp8: this wavefront's 4 x 64 dwords of tile t's raw slot, and the conversion of its share of tile t
  uint32_t* const raw_base = (uint32_t*)(lds + kRing * kStageVecs) + wv * (4 * kWave);
  auto raw_of = [&](int t) { return raw_base + (t & (kStages - 1)) * (kWgWaves * 4 * kWave); };
  auto request = [&](int32_t blk0, int32_t blk1, int t, bool again) {
    if (kFp8) request_tile_fp8(a, f, blk0, blk1, g, raw_of(t), again);
    else request_tile(a, f, blk0, blk1, g, stage_of(t), wv, again);
  };
  auto convert = [&](int t) {
    if (kFp8)
      convert_tile_fp8(lds_address(raw_of(t) + lane),
                       rd + ((t & (kRing - 1)) * kStageVecs + 2 * wv * kWave) * 16);
  };
  auto block_id = [&](int t, int which) { return sload(bt_row + min(2 * min(t, last) + which, n_blocks - 1)); };
  auto land = [&](int t) {  // after this wavefront's share of tile t arrived: mend a ragged tile
    const int n_valid = si.len - t * kTile;
    if (t <= last && n_valid < kTile) zero_invalid_v_lds(stage_of(t), wv, lane, n_valid);
  };

  __builtin_amdgcn_s_barrier();  // the previous segment is done with every stage
  if (!kFinish || t0 < t1) {
#pragma unroll
    for (int i = 0; i < kStages - 1; ++i)  // tiles t0 .. t0 + kStages - 2; past the end: the last tile again (L2 hits)
      request(block_id(t0 + i, 0), block_id(t0 + i, 1), t0 + i, t0 + i > last || si.rg > 1);
    int32_t nb0 = block_id(t0 + kStages - 1, 0), nb1 = block_id(t0 + kStages - 1, 1);
    asm volatile("" ::"s"(nb0), "s"(nb1));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads * (kStages - 2)) : "memory");  // tile t0 is in
    convert(t0);
    land(t0);
    __builtin_amdgcn_s_barrier();
    floatx16 s;
    if (kRows) {
      score_tile(s, rd + (t0 & (kRing - 1)) * (kStageVecs * 16), q);
      if (si.len - t0 * kTile < kTile) mask_scores(s, si.len - t0 * kTile, h);
    }
    // iteration t: s_in holds the scores of tile t, s_out receives those of tile t + 1.  Only a sequence's last tile
    // can be ragged, so the iterations that land and mask a full tile (kChecked = false) carry no test for it.
    auto iter = [&](auto checked, int t, const floatx16& s_in, floatx16& s_out) {
      constexpr bool kChecked = decltype(checked)::value;
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads * (kStages - 3)) : "memory");  // tile t + 1 is in
      convert(t + 1);
      if (kChecked) land(t + 1);
      // every share of tile t + 1 is visible, and everyone is done with tile t - 1
      __builtin_amdgcn_s_barrier();
      auto fetch = [&]() {
        request(nb0, nb1, t + kStages - 1, t + kStages - 1 > last || si.rg > 1);
        nb0 = block_id(t + kStages, 0);
        nb1 = block_id(t + kStages, 1);
      };
      if (kRows) {
        const uint32_t k_addr = rd + ((t + 1) & (kRing - 1)) * (kStageVecs * 16);
        const uint32_t v_addr = rd + (t & (kRing - 1)) * (kStageVecs * 16) + 8 * kWave * 16;
        woven_tile(s_in, s_out, o, m, l, q, k_addr, v_addr, c, fetch);
        if (kChecked) {
          const int nv_next = si.len - (t + 1) * kTile;
          if (nv_next < kTile) mask_scores(s_out, nv_next, h);
        }
      } else {
        fetch();
      }
      // the block ids are in before the next iteration issues its LDS reads (no wait among them)
      asm volatile("" ::"s"(nb0), "s"(nb1));
    };
    // tile t + 1 is full for every t < len / kTile - 1
    const int t_plain = min(t1, si.len / kTile - 1);
    floatx16 s2;
    int t = t0;
    for (; t + 2 <= t_plain; t += 2) {
      iter(std::false_type{}, t, s, s2);
      iter(std::false_type{}, t + 1, s2, s);
    }
    for (; t < t1; ++t) {
      iter(std::true_type{}, t, s, s2);
      s = s2;
    }
  }
  if (!kFinish) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no fetch of this segment may land later
    if (kRows) store_partial(slot, kLargeRows, wv, o, m, l, lane, a.m_scale, a.o_scale);
    return;
  }
  if (kFp8 && kRows) {  // (true units: see fp8_pieces)
    m *= a.m_scale;
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) o[jt] *= a.o_scale;
  }
  const FinishArgs fa = kernel_args().fin;
  int early = 0;
  if (kRows && fin->pieces > 1) early = arrivals(counter_of<2>(fa, *fin, wv));
  if (!tree) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    const int ln = fresh(lane);
    const TreeRows t = tree_rows(fa, base, g, si.n);
    TreePair pair;
    request_tree(pair, t, 0, wv, ln);
    uint32_t word[4];
    if (kRows)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) word[tt] = mask_word(fa, base, M, row0 + (ln & 31), si.n, tt);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    const bool mend = stage_tree(pair, t, lds, (uint32_t*)(lds + kStages * kStageVecs), wv, ln);
    if (kRows) {
      for (int tt = 0; 32 * tt < si.n; ++tt)
        staged_tree_tile(o, m, l, q, tt == 0 ? word[0] : tt == 1 ? word[1] : tt == 2 ? word[2] : word[3], lds, tt,
                         fa.scale_log2e, ln);
      if (mend) add_not_finite(o, fa, t, base, M, row0 + (ln & 31), si.n, 0, 4, ln);
    }
  }
  if (kRows) {
    floatx4 x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[u][i] = o[u >> 2][4 * (u & 3) + i];
    finish_part<2, 16>(fa, *fin, x, m, sum_across_halves(l), 0, wv, early, wv, lane);
  }
}

// One staged tile against this wavefront's 32 rows, nothing woven in: all 16 operand reads
// are issued up front, the counts of the waits follow that order.
__device__ inline void plain_tile(floatx16 (&o)[4], float& m, float& l, const bf16x8 (&q)[8], uint32_t k_addr,
                                  uint32_t v_addr, float c, int n_valid, int h) {
  bf16x8 kop[8], vop[8];
  lds_read_half(kop, k_addr, 0);
  lds_read_half(kop, k_addr, 1);
  lds_read_half(vop, v_addr, 0);
  lds_read_half(vop, v_addr, 1);
  floatx16 s = (floatx16)(0.f);
#define SMART_SCORE_STEP(I, N) \
  SMART_LDS_WAIT(kop[I], N);   \
  s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[I], q[I], s, 0, 0, 0);
  SMART_SCORE_STEP(0, 15)
  SMART_SCORE_STEP(1, 14)
  SMART_SCORE_STEP(2, 13)
  SMART_SCORE_STEP(3, 12)
  SMART_SCORE_STEP(4, 11)
  SMART_SCORE_STEP(5, 10)
  SMART_SCORE_STEP(6, 9)
  SMART_SCORE_STEP(7, 8)
#undef SMART_SCORE_STEP
  if (n_valid < kTile) mask_scores(s, n_valid, h);
  bf16x8 pb0, pb1;
  softmax_tile(s, m, l, o, pb0, pb1, c);
#define SMART_OUTPUT_STEP(I, N, PB) \
  SMART_LDS_WAIT(vop[I], N);        \
  o[I & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[I], PB, o[I & 3], 0, 0, 0);
  SMART_OUTPUT_STEP(0, 7, pb0)
  SMART_OUTPUT_STEP(1, 6, pb0)
  SMART_OUTPUT_STEP(2, 5, pb0)
  SMART_OUTPUT_STEP(3, 4, pb0)
  SMART_OUTPUT_STEP(4, 3, pb1)
  SMART_OUTPUT_STEP(5, 2, pb1)
  SMART_OUTPUT_STEP(6, 1, pb1)
  SMART_OUTPUT_STEP(7, 0, pb1)
#undef SMART_OUTPUT_STEP
}

// The states of a grouped segment (R row tiles x K = 8 / R key groups, wavefront = row tile *
// K + key group) become one partial: all eight states go to LDS, and after one barrier
// wavefront w merges, for row tile w / K, accumulator registers [(w % K) 64 / K, ...) of
// that row tile's K states (always in key-group order) and stores that slice.
template <int R, bool kFinish = false>
__device__ inline void fold_groups(const SmallState& S, float* lds, float* slot, int rows_in_slot, int wv, int lane,
                                   float c, const FinishArgs* fa = nullptr, const Finish* f = nullptr, int early = 0) {
  constexpr int K = kWgWaves / R, kRegs = 64 / K;
  const int h = lane >> 5, j = lane & 31;
  state_to_lds(S, lds + wv * kStateFloats, lane);
  __syncthreads();
  const int rt = wv / K, part_index = wv % K;
  float mk[K], lk[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float* src = lds + (rt * K + k) * kStateFloats;
    mk[k] = src[64 * kWave + lane];
    lk[k] = src[65 * kWave + lane];
  }
  floatx4 part[K][kRegs / 4];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int u = 0; u < kRegs / 4; ++u)
      part[k][u] = state_quad(lds + (rt * K + k) * kStateFloats, part_index * (kRegs / 4) + u, lane);
  float m_new = mk[0];
#pragma unroll
  for (int k = 1; k < K; ++k) m_new = fmaxf(m_new, mk[k]);
  float l_new = 0.f;
  floatx4 x[kRegs / 4];
#pragma unroll
  for (int u = 0; u < kRegs / 4; ++u) x[u] = (floatx4)(0.f);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    // an empty state has max -inf and contributes nothing
    const float sc = mk[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mk[k] - m_new) * c);
    l_new += lk[k] * sc;
#pragma unroll
    for (int u = 0; u < kRegs / 4; ++u) x[u] += part[k][u] * sc;
  }
  if (kFinish) {
    __syncthreads();  // the next segment reuses the LDS
    if (rt * 32 < f->rows)
      finish_part<1, kRegs / 4>(*fa, *f, x, m_new, sum_across_halves(l_new), part_index * (kRegs / 4), rt, early,
                                               wv, lane);
    return;
  }
  // accumulator register 16 jt + 4 r4 + i of lane (h, j) is row j, head dims 4 (8 jt + 2 r4 + h) + i
  const bool in_slot = rt * 32 < rows_in_slot;  // a 64-row slot has no room for row tiles 2 and 3 (they hold no rows)
#pragma unroll
  for (int u = 0; u < kRegs / 4; ++u) {
    const int reg = part_index * kRegs + 4 * u, jt = reg >> 4, r4 = (reg & 15) >> 2;
    if (in_slot) store_through(slot + ((size_t)(rt * 32 + jt * 8 + 2 * r4 + h) * 32 + j) * 4, x[u]);
  }
  if (part_index == 0) {
    const float lsum = sum_across_halves(l_new);
    if (h == 0 && in_slot) {
      slot[rows_in_slot * kD + rt * 32 + j] = m_new;
      slot[rows_in_slot * kD + rows_in_slot + rt * 32 + j] = lsum;
    }
  }
  __syncthreads();  // the next segment reuses the LDS
}

// Segments of at most 32 R rows (R = 2 or 4): the eight wavefronts are R row tiles x K = 8 / R
// key groups, and an iteration consumes K tiles at once (key group kg takes tile kg of the
// iteration), so that the stream, not the per-tile arithmetic of one wavefront, sets the pace.
// Tiles are staged as in staged_segment (every wavefront fetches an eighth of every tile); the
// iterations 8 / K - 1 ahead of the one being consumed are in flight.
template <int R, bool kFinish = false>
__device__ inline void grouped_segment(const MainArgs& a, int b, int g, int base, int t0, int t1, const SeqInfo si,
                                       float* slot, int rows_in_slot, int wv, int lane, bf16x8* lds, bool tree = false,
                                       const Finish* fin = nullptr) {
  constexpr int K = kWgWaves / R;
  constexpr int kAhead = kStages / K - 1;
  // (row tile = wv / K: when only the first row tiles hold rows, the busy wavefronts sit on different SIMDs)
  const int rt = wv / K, kg = wv % K;
  const int h = lane >> 5, j = lane & 31;
  const int M = si.n * a.G;
  const bool has_rows = rt * 32 < M;
  SmallState S;
  bf16x8 q[8];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) S.o[jt] = (floatx16)(0.f);
  S.m = -INFINITY;
  S.l = 0.f;
  if (has_rows) {
    int rho = rt * 32 + j;
    rho = rho < M ? rho : M - 1;  // padding rows repeat the last real row; never read back
    const int node = base + rho / a.G, head = g * a.G + rho % a.G;
    const __bf16* qp = a.q + ((int64_t)node * a.Hq + head) * kD + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ks] = *(const bf16x8*)(qp + ks * 16);
    asm volatile("" ::"v"(q[0]), "v"(q[7]));  // landed: the counted waits below see tile fetches only
  }
  const int32_t* bt_row = a.block_table + (int64_t)b * a.max_blocks;
  const int n_blocks = (si.len + kBlock - 1) / kBlock;
  const float c = a.scale_log2e;
  const FetchLane f = fetch_lane(a, wv, lane);
  const uint32_t rd = lds_address(lds + lane);
  const int last = t1 - 1;
  auto stage_of = [&](int t) { return lds + (t & (kStages - 1)) * kStageVecs; };
  auto block_id = [&](int t, int which) { return sload(bt_row + min(2 * min(t, last) + which, n_blocks - 1)); };
  auto land = [&](int t) {
    const int n_valid = si.len - t * kTile;
    if (t <= last && n_valid < kTile) zero_invalid_v_lds(stage_of(t), wv, lane, n_valid);
  };

  __builtin_amdgcn_s_barrier();  // the previous segment is done with the LDS
  if (!kFinish || t0 < t1) {
#pragma unroll
    for (int i = 0; i < kAhead * K; ++i)  // past the end: the last tile again (L2 hits), never consumed
      request_tile(a, f, block_id(t0 + i, 0), block_id(t0 + i, 1), g, stage_of(t0 + i), wv, t0 + i > last || si.rg > 1);
    int32_t nb[K][2];
#pragma unroll
    for (int x = 0; x < K; ++x) {
      nb[x][0] = block_id(t0 + kAhead * K + x, 0);
      nb[x][1] = block_id(t0 + kAhead * K + x, 1);
    }
    for (int tb = t0; tb < t1; tb += K) {
#pragma unroll
      for (int x = 0; x < K; ++x) asm volatile("" ::"s"(nb[x][0]), "s"(nb[x][1]));  // ids are in (no wait among LDS reads)
      // this wavefront's share of the K tiles of this iteration has landed: what may still be
      // outstanding are the kAhead - 1 iterations after it, 2 K fetches each
      if (K == 4) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
#pragma unroll
      for (int x = 0; x < K; ++x) land(tb + x);
      // every share of this iteration's tiles is visible, and everyone is done with the previous iteration's
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int x = 0; x < K; ++x)
        request_tile(a, f, nb[x][0], nb[x][1], g, stage_of(tb + kAhead * K + x), wv, tb + kAhead * K + x > last || si.rg > 1);
#pragma unroll
      for (int x = 0; x < K; ++x) {
        nb[x][0] = block_id(tb + (kAhead + 1) * K + x, 0);
        nb[x][1] = block_id(tb + (kAhead + 1) * K + x, 1);
      }
      const int t = tb + kg;
      if (has_rows && t < t1) {
        const uint32_t stage = rd + (t & (kStages - 1)) * (kStageVecs * 16);
        plain_tile(S.o, S.m, S.l, q, stage, stage + 8 * kWave * 16, c, si.len - t * kTile, h);
      }
    }
  }
  FinishArgs fa;
  int early = 0;
  if (kFinish) {
    fa = kernel_args().fin;
    if (fin->pieces > 1) early = arrivals(counter_of<1>(fa, *fin, wv));
  }
  TreePair pair;
  uint32_t word = 0u;
  TreeRows t;
  const int ln = fresh(lane);
  if (kFinish && tree) {  // at most 64 nodes: two tiles of tree keys, one per key group
    t = tree_rows(fa, base, g, si.n);
    request_tree(pair, t, 0, wv, ln);
    word = mask_word(fa, base, M, rt * 32 + (ln & 31), si.n, kg);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no fetch of this segment may land later
  __builtin_amdgcn_s_barrier();                      // and nobody still reads a stage: the fold reuses the LDS
  if (kFinish && tree) {
    const bool mend = stage_tree(pair, t, lds, (uint32_t*)(lds + kStages * kStageVecs), wv, ln);
    if (has_rows) {
      if (32 * kg < si.n) staged_tree_tile(S.o, S.m, S.l, q, word, lds, kg, c, ln);
      if (mend) add_not_finite(S.o, fa, t, base, M, rt * 32 + (ln & 31), si.n, kg, kg + 1, ln);
    }
    __syncthreads();
  }
  if (kFinish) fold_groups<R, true>(S, (float*)lds, nullptr, rows_in_slot, wv, lane, c, &fa, fin, early);
  else fold_groups<R>(S, (float*)lds, slot, rows_in_slot, wv, lane, c);
}

// Worker of classes 1 and 2 (kCls): a workgroup walks the pieces of its share of the class's units.
template <int kCls, bool kFp8 = false, bool kFinish = false>
__device__ inline void staged_worker(const MainArgs& a0, int64_t w, ClassPlan& cp, bf16x8* lds /* 132 KB: kStages tiles, or eight states */) {
  const int64_t U = cp.U, W = cp.W;
  PlanWindow& win = cp.win;
  if (w >= W || U <= 0) return;
  int64_t u0 = share_begin(w, U, W);
  const int64_t u1 = share_begin(w + 1, U, W);
  if (u0 >= u1) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int b = locate(cp, plan_view(a0.plan, a0.batch), a0.cu_nodes, kCls, a0.batch, u0, lane);
  while (u0 < u1 && b < a0.batch) {
    const MainArgs a = kFinish ? kernel_args() : a0;
    const PlanView pv = plan_view(a.plan, a.batch);
    follow(cp, pv, a.cu_nodes, kCls, a.batch, b, lane);
    const int64_t seq_begin = window_cum_units(win, b - win.first);
    const int64_t seq_end = window_cum_units(win, b + 1 - win.first);
    if (u0 >= seq_end) { ++b; continue; }
    const SeqInfo si = window_info(win, b);
    const int64_t local = u0 - seq_begin;
    const int base = __builtin_amdgcn_readlane(win.cu_nodes, b - win.first);
    if (kCls == 1) {
      const int units = segment_units<kFinish>(si, a.tree_cost);
      const int seg_local = (int)(local / units);
      const int t0 = (int)(local % units);
      const int g = seg_local;
      const int64_t left = u1 - u0;
      const int nt = (int)(left < (int64_t)(units - t0) ? left : (int64_t)(units - t0));
      const int64_t seg = (int64_t)__builtin_amdgcn_readlane(win.cum_segs, b - win.first) + seg_local;
      // At most 64 rows: row tiles 0 and 1 of four, times two key groups.  (Two row tiles x four
      // key groups would keep every wavefront busy but leaves only one iteration of fetches in
      // flight; measured slower.)
      if (kFinish) {
        const Finish f = finish_of(u0 - t0, units, U, W, w, seg, base, g, si.n * a.G, 0);
        grouped_segment<4, true>(a, b, g, base, min(t0, si.tiles), min(t0 + nt, si.tiles), si, nullptr, kMediumRows, wv, lane, lds,
                                 t0 + nt == units, &f);
      } else
      grouped_segment<4>(a, b, g, base, t0, t0 + nt, si, a.ws[1] + (size_t)(w + seg) * kMediumSlot, kMediumRows, wv,
                         lane, lds);
      u0 += nt;
    } else {
      // the unit space of class 2 is a cost: see large_spans and large_tile_at
      const LargeSpans ls = large_spans<kFinish>(si, a.G, a.tree_cost);
      const int g = (int)(local / ls.span_head);
      const int64_t in_head = local - (int64_t)g * ls.span_head;
      int rgi = (int)(in_head / ls.span_full);
      rgi = rgi < si.rg - 1 ? rgi : si.rg - 1;
      const int64_t off = in_head - (int64_t)rgi * ls.span_full;
      const int cost = rgi < si.rg - 1 ? kLargeTileCost[kLargeRows / 32] : ls.cost_last;
      const int64_t span = rgi < si.rg - 1 ? ls.span_full : ls.span_last;
      const int seg_local = g * si.rg + rgi;
      const int64_t seg_end = u0 - off + span;
      const int64_t stop = u1 < seg_end ? u1 : seg_end;
      const int t0 = large_tile_at(off, cost, si.tiles);
      const int t1 = stop == seg_end ? si.tiles : large_tile_at(off + (stop - u0), cost, si.tiles);
      const int64_t ub = u0 - off;
      u0 = stop;
      const int64_t seg = (int64_t)__builtin_amdgcn_readlane(win.cum_segs, b - win.first) + seg_local;
      // rows of the group are dealt to the eight wavefronts in 32-row tiles
      const int row0 = rgi * kLargeRows + wv * 32;
      if (kFinish) {
        const Finish f = finish_of(ub, span, U, W, w, seg, base, g, si.n * a.G, rgi * kLargeRows);
        // (a share that covers less than a tile of the segment counts its empty state in)
        if (row0 < f.rows)
          staged_segment<true, kFp8, true>(a, b, g, base, row0, t0, t1, si, nullptr, wv, lane, lds, stop == seg_end, &f);
        else
          staged_segment<false, kFp8, true>(a, b, g, base, row0, t0, t1, si, nullptr, wv, lane, lds, stop == seg_end, &f);
        continue;
      }
      float* slot = a.ws[2] + (size_t)(w + seg) * kLargeSlot;
      if (t1 <= t0) {
        // The share covers less than a tile of this segment (rare).  The combine step
        // merges the partial of every worker whose share touches the segment, so this one leaves a partial that adds
        // nothing: row maxima of -inf (weight exp2(-inf) = 0), sums and O of zero.
        for (int i = threadIdx.x; i < kLargeSlot; i += kWgWaves * kWave)
          slot[i] = i >= kLargeRows * kD && i < kLargeRows * kD + kLargeRows ? -INFINITY : 0.f;
        continue;
      }
      if (row0 < si.n * a.G) staged_segment<true, kFp8>(a, b, g, base, row0, t0, t1, si, slot, wv, lane, lds);
      else staged_segment<false, kFp8>(a, b, g, base, row0, t0, t1, si, slot, wv, lane, lds);
    }
  }
}

// ---- the prefix kernel: one launch, workgroups apportioned to the classes by the plan ------
// kFp8: the cache holds E4M3 bytes; trees of up to 64 rows are class 1 and streamed into registers by
// fp8_worker, larger ones are class 2 and go through the staged loop after conversion to bf16 in LDS.
template <bool kFp8, bool kPair, bool kFinish>
__global__ __launch_bounds__(kWgWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tva_prefix_kernel(MainArgs a) {
  __shared__ float4 lds_raw[8448];  // 132 KB, carved up per class (class 0: eight states of 16.5 KB)
  SMART_TIMELINE(const unsigned long long tl_start = wall_clock64(); const unsigned long long tl_cycles = clock64();)
  // Workgroups are dealt to the eight XCDs round robin; consecutive WORKERS (consecutive unit ranges: the row groups
  // of one segment, the two ends of a segment) are put on one XCD so that what they read in common meets in its L2.
  // (The grid's size from the arguments: gridDim lies behind them, a line of host memory further; 0.15 .. 0.35 us of a call.  From
  // an fp8 cache in two launches that gains nothing, and the kernel that holds a.workgroups takes longer, compiled: 2 sequences
  // of 2048 tokens and 44 nodes 42.7 us, this way 42.3, of 8000 and 60 51.1 and 50.7.)
  const unsigned grid = kFp8 && !kFinish ? gridDim.x : (a.workgroups > kClasses ? a.workgroups : kClasses);
  const int64_t wg = grid % 8 == 0 ? (int64_t)(blockIdx.x % 8) * (grid / 8) + blockIdx.x / 8 : (int64_t)blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ClassPlan cp;
  int64_t first1, first2, end;
  if (kFinish && a.status && (wv > 0 || a.batch > kWave)) {  // the block-table check, while wavefront 0 plans
    for (int64_t b = blockIdx.x + (int64_t)grid * (wv - (a.batch <= kWave ? 1 : 0)); b < a.batch;
         b += (int64_t)grid * (a.batch <= kWave ? kWgWaves - 1 : kWgWaves))
      smart::tva_validate_block_table((int)b, a.block_table, a.prefix_len, a.max_blocks, kBlock, a.num_blocks, a.status, lane);
  }
  if (a.batch <= kWave) {
    // No planning kernel ran: wavefront 0 derives the plan and hands it to the others through
    // LDS; workgroup 0 also writes it to memory for the combine kernel.
    __shared__ PlanShare share;
    if (wv == 0) {
      LanePlan lp;
      lane_plan<kFp8, kFinish>(lp, a.prefix_len, a.cu_nodes, a.batch, a.total_nodes, a.G, a.Hkv, a.max_blocks, a.workgroups, a.caps,
                               a.tree_cost, lane);
#pragma unroll
      for (int c = 0; c < kClasses; ++c) {
        share.cum_units[c][lane] = lp.cum_units[c];
        share.cum_segs[c][lane] = lp.cum_segs[c];
      }
      share.cu[lane] = lp.cu;
      share.info[lane] = lp.si;
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kClasses; ++c) {
          share.units[c] = lp.units[c];
          share.workers[c] = lp.workers[c];
          share.first_wg[c] = lp.first_wg[c];
        }
        share.first_wg[kClasses] = lp.first_wg[kClasses];
      }
      if (!kFinish && wg == 0) {
        const PlanView pv = plan_view(a.plan, a.batch);
        if (lane <= a.batch) {
#pragma unroll
          for (int c = 0; c < kClasses; ++c) {
            pv.cum_units[c][lane] = lp.cum_units[c];
            pv.cum_segs[c][lane] = lp.cum_segs[c];
          }
          pv.cum_chunks[lane] = lp.cum_chunks;
        }
        if (a.batch == kWave && lane == 0) {  // entry 64 has no lane: the totals
#pragma unroll
          for (int c = 0; c < kClasses; ++c) {
            pv.cum_units[c][kWave] = lp.units[c];
            pv.cum_segs[c][kWave] = lp.total_segs[c];
          }
          pv.cum_chunks[kWave] = lp.chunks;
        }
        if (lane < a.batch) pv.info[lane] = lp.si;
        if (lane == 0) {
#pragma unroll
          for (int c = 0; c < kClasses; ++c) {
            pv.header[2 * c] = lp.units[c];
            pv.header[2 * c + 1] = lp.workers[c];
            pv.header[6 + c] = lp.first_wg[c];
          }
          pv.header[6 + kClasses] = lp.first_wg[kClasses];
        }
      }
    }
    __syncthreads();
    first1 = uniform64(share.first_wg[1]), first2 = uniform64(share.first_wg[2]), end = uniform64(share.first_wg[3]);
    const int cls = wg < first1 ? 0 : (wg < first2 ? 1 : 2);
    cp.U = uniform64(share.units[cls]);
    cp.W = uniform64(share.workers[cls]);
    cp.resident = true;
    cp.win.first = 0;
    cp.win.cum_units = share.cum_units[cls][lane];
    cp.win.cum_segs = share.cum_segs[cls][lane];
    cp.win.cu_nodes = share.cu[lane];
    const SeqInfo si = share.info[lane];
    cp.win.len = si.len;
    cp.win.n = si.n;
    cp.win.tiles = si.tiles;
    cp.win.rg = si.rg;
    cp.win.total_units = cp.U;
  } else {
    const PlanView pv = plan_view(a.plan, a.batch);
    first1 = sload(pv.header + 7), first2 = sload(pv.header + 8), end = sload(pv.header + 9);
    const int cls = wg < first1 ? 0 : (wg < first2 ? 1 : 2);
    cp.U = sload(pv.header + 2 * cls);
    cp.W = sload(pv.header + 2 * cls + 1);
    cp.resident = false;
  }
  // (by every workgroup, before those without a worker leave)
  if (kFinish)
    for (int i = (int)(blockIdx.x * kWgWaves + wv) * kWave; i < a.fin.n_clear; i += (int)grid * kWgWaves * kWave)
      a.fin.clear[i + (int)(threadIdx.x & (kWave - 1))] = 0;
  if (wg >= end) return;
  SMART_TIMELINE(auto tl_end = [&]() {
    __syncthreads();  // the workgroup's end is its last wavefront's
    if (threadIdx.x == 0 && blockIdx.x < timeline::kWorkgroups) {
      unsigned long long* d = timeline::wg_stamps + 4 * blockIdx.x;
      d[0] = tl_start;
      d[1] = wall_clock64();
      d[2] = clock64() - tl_cycles;
      d[3] = (unsigned long long)(wg < first1 ? 0 : (wg < first2 ? 1 : 2)) | ((unsigned long long)wg << 8) | (1ull << 63);
    }
  };)
  if (kFp8) {
    if (wg >= first1 && wg < first2) fp8_worker<kPair, kFinish>(a, wg - first1, cp, (float*)lds_raw);
    else if (wg >= first2) staged_worker<2, true, kFinish>(a, wg - first2, cp, (bf16x8*)lds_raw);
    SMART_TIMELINE(tl_end();)
    return;
  }
  if (wg < first1) {
    small_worker<kFinish>(a, wg, cp, (float*)lds_raw);
  } else if (wg < first2) {
    staged_worker<1, false, kFinish>(a, wg - first1, cp, (bf16x8*)lds_raw);
  } else {
    staged_worker<2, false, kFinish>(a, wg - first2, cp, (bf16x8*)lds_raw);
  }
  SMART_TIMELINE(tl_end();)
}

// ---------------------------------------------------------------------------
// combine kernel: tree part on the vector ALUs + merge of the prefix partials
// ---------------------------------------------------------------------------
struct CombineArgs {
  const uint16_t* q;
  const uint16_t* k_tree;
  const uint16_t* v_tree;
  const int32_t* cu_nodes;
  const uint64_t* anc_mask;
  void* plan;
  const float* ws[kClasses];
  uint16_t* out;
  float* lse;
  int32_t batch, Hq, Hkv, G;
  float scale, scale_log2e;
  int32_t only_small;  // fp8 cache: the classes are those of plan_class<true>
  // block-table check (status may be null: no check)
  const int32_t* block_table;
  const int32_t* prefix_len;
  int32_t* status;
  int32_t max_blocks, num_blocks;
};

__device__ inline float bf16_to_f32(uint16_t x) { return __uint_as_float(((uint32_t)x) << 16); }
typedef __attribute__((ext_vector_type(2))) uint32_t uintx2;
typedef __attribute__((ext_vector_type(2))) float floatx2;
// A dword as a pair of bf16 values.  (The dword goes through a register of its own first: a bit cast applied
// directly to an element of a two-dword vector has been seen to read the vector's first element for both.)
__device__ inline bf16x2 bf16_pair(uint32_t w) {
  asm volatile("" : "+v"(w));
  return __builtin_bit_cast(bf16x2, w);
}
__device__ inline uint16_t f32_to_bf16(float v) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// 8 lanes per query row; lane e of a row owns d = 4c .. 4c+3 for c = e, e+8, e+16, e+24.
// With one wavefront per SIMD (small batches of small trees) memory round trips are the cost here, so independent
// loads are issued together: the plan entries, the K and V rows of a step's tree keys, all of a partial's pieces.
// With several wavefronts per SIMD (large trees) the vector instructions of the tree part are, so it works on
// packed bf16 pairs (below), which also leaves room for five resident wavefronts per SIMD.
constexpr int kKeyPairs = 1;  // pairs of tree keys per step (2 and 4 measured slower: their registers cost resident wavefronts)

__global__ __launch_bounds__(kWave) void tva_combine_kernel(CombineArgs a) {
  const int wc = blockIdx.x;
  const int lane = threadIdx.x;
  SMART_TIMELINE(const unsigned long long tl_start = wall_clock64();)
  // the first `batch` wavefronts also check one sequence's block-table entries each (the grid has at least that many)
  if (a.status && wc < a.batch)
    smart::tva_validate_block_table(wc, a.block_table, a.prefix_len, a.max_blocks, kBlock, a.num_blocks, a.status, lane);
  const PlanView pv = plan_view(a.plan, a.batch);
  int b;
  if (a.batch <= kWave) {
    // cum_chunks is non-decreasing: lanes with cum <= wc are a prefix whose last lane is b
    const int32_t cum = pv.cum_chunks[min(lane, a.batch - 1)];
    const int32_t total = sload(pv.cum_chunks + a.batch);
    if (wc >= total) return;
    const uint64_t below = __ballot(lane < a.batch && cum <= wc);
    b = __popcll(below) - 1;
  } else {
    if (wc >= sload(pv.cum_chunks + a.batch)) return;
    int lo = 0, hi = a.batch;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (sload(pv.cum_chunks + mid) <= wc) lo = mid; else hi = mid;
    }
    b = lo;
  }
  const SeqInfo si = sload(pv.info + b);
  const int cls = a.only_small ? plan_class<true>(si.n * a.G) : seq_class(si.n * a.G);
  const int chunk_base = sload(pv.cum_chunks + b);
  const int base = sload(a.cu_nodes + b);
  const int64_t U = sload(pv.header + 2 * cls), W = sload(pv.header + 2 * cls + 1);
  // (selected with compares: indexing the pointer arrays with a run-time class would push the plan view to scratch)
  const int32_t* segs_c = cls == 0 ? pv.cum_segs[0] : (cls == 1 ? pv.cum_segs[1] : pv.cum_segs[2]);
  const int64_t* units_c = cls == 0 ? pv.cum_units[0] : (cls == 1 ? pv.cum_units[1] : pv.cum_units[2]);
  const int64_t seg_base = sload(segs_c + b);
  const int64_t unit_base = sload(units_c + b);
  const int M = si.n * a.G;
  const int per_g = (M + kCombineRows - 1) / kCombineRows;
  const int local = wc - chunk_base;
  const int g = local / per_g, chunk = local % per_g;
  const int e = lane & 7;
  const int rho_raw = chunk * kCombineRows + (lane >> 3);
  const bool active = rho_raw < M;
  const int rho = active ? rho_raw : M - 1;
  const int node = base + rho / a.G, head = g * a.G + rho % a.G;
  const float c = a.scale_log2e;

  // tree keys: the set bits of this row's ancestor mask, lowest first
  uint64_t mlo = active ? a.anc_mask[2 * (size_t)node] : 0ull;
  uint64_t mhi = active ? a.anc_mask[2 * (size_t)node + 1] : 0ull;
  uint32_t qw[8];  // the lane's 16 query elements as 8 bf16 pairs (dims 4 (e + 8 k) + 2 w, + 1)
  {
    const uint16_t* qp = a.q + ((int64_t)node * a.Hq + head) * kD;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uintx2 x = *(const uintx2*)(qp + 4 * (e + 8 * k));
      qw[2 * k] = x[0];
      qw[2 * k + 1] = x[1];
    }
  }
  if (si.n < 64) mlo &= (1ull << si.n) - 1ull, mhi = 0ull;           // never index past the tree
  else if (si.n < 128) mhi &= (1ull << (si.n - 64)) - 1ull;

  float m = -INFINITY, l = 0.f, acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;

  // Two keys per step, on the packed bf16 dot product: the score is q . k over bf16 pairs (products exact, sums in
  // binary32, as before); the two probabilities are rounded to bf16 like those of the matrix-core path, and one
  // instruction adds p0 v0[d] + p1 v1[d] to an output element (the V elements of the two keys paired by a byte
  // permute).  With several wavefronts per SIMD this loop is bound by its vector instructions, not by its loads.
  while (__any((mlo | mhi) != 0ull)) {
    int jn[2 * kKeyPairs];
    bool have[2 * kKeyPairs];
#pragma unroll
    for (int u = 0; u < 2 * kKeyPairs; ++u) {
      have[u] = (mlo | mhi) != 0ull;
      jn[u] = 0;
      if (mlo) { jn[u] = __ffsll((unsigned long long)mlo) - 1; mlo &= mlo - 1; }
      else if (mhi) { jn[u] = 64 + __ffsll((unsigned long long)mhi) - 1; mhi &= mhi - 1; }
    }
    uint32_t kw[2 * kKeyPairs][8], vw[2 * kKeyPairs][8];
#pragma unroll
    for (int u = 0; u < 2 * kKeyPairs; ++u) {
      const uint16_t* kp = a.k_tree + ((int64_t)(base + jn[u]) * a.Hkv + g) * kD;
      const uint16_t* vp = a.v_tree + ((int64_t)(base + jn[u]) * a.Hkv + g) * kD;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uintx2 x = *(const uintx2*)(kp + 4 * (e + 8 * k));
        const uintx2 y = *(const uintx2*)(vp + 4 * (e + 8 * k));
        kw[u][2 * k] = x[0];
        kw[u][2 * k + 1] = x[1];
        vw[u][2 * k] = y[0];
        vw[u][2 * k + 1] = y[1];
      }
    }
#pragma unroll
    for (int pr = 0; pr < kKeyPairs; ++pr) {
      float dot[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float d0 = 0.f, d1 = 0.f;  // two chains
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          d0 = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(qw[i]), bf16_pair(kw[2 * pr + u][i]), d0, false);
          d1 = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(qw[i + 1]), bf16_pair(kw[2 * pr + u][i + 1]), d1, false);
        }
        float d = d0 + d1;
        d += __shfl_xor(d, 1);
        d += __shfl_xor(d, 2);
        d += __shfl_xor(d, 4);
        dot[u] = have[2 * pr + u] ? d : -INFINITY;
      }
      const float m_new = fmaxf(m, fmaxf(dot[0], dot[1]));
      const float al = m_new == m ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * c);  // (also when both are -inf)
      floatx2 p;
      p[0] = have[2 * pr] ? __builtin_amdgcn_exp2f((dot[0] - m_new) * c) : 0.f;
      p[1] = have[2 * pr + 1] ? __builtin_amdgcn_exp2f((dot[1] - m_new) * c) : 0.f;
      l = l * al + (p[0] + p[1]);
      m = m_new;
      const bf16x2 pp = __builtin_convertvector(p, bf16x2);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t lo = __builtin_amdgcn_perm(vw[2 * pr + 1][i], vw[2 * pr][i], 0x05040100u);  // (v0[d], v1[d])
        const uint32_t hi = __builtin_amdgcn_perm(vw[2 * pr + 1][i], vw[2 * pr][i], 0x07060302u);  // (v0[d + 1], v1[d + 1])
        acc[2 * i] = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(lo), pp, acc[2 * i] * al, false);
        acc[2 * i + 1] = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(hi), pp, acc[2 * i + 1] * al, false);
      }
    }
  }

  // prefix partials of this row's segment: workers w_first .. w_last of its class
  if (si.tiles > 0 && active) {
    const int rows_per_group = class_rows(cls);
    const int slot_floats = class_slot(cls);
    const float* ws = cls == 0 ? a.ws[0] : (cls == 1 ? a.ws[1] : a.ws[2]);
    const int rgi = rho / rows_per_group;
    const int seg_local = g * si.rg + rgi;
    const int64_t seg = seg_base + seg_local;
    const LargeSpans ls = large_spans<false>(si, a.G, TreeCost{0, 0});
    const bool last_group = rgi == si.rg - 1;
    const int64_t span = cls < 2 ? si.tiles : (last_group ? ls.span_last : ls.span_full);
    const int64_t ub = unit_base + (cls < 2 ? (int64_t)seg_local * si.tiles : g * ls.span_head + rgi * ls.span_full);
    int64_t w_first, w_last;
    segment_workers(ub, span, U, W, w_first, w_last);
    const int row = rho % rows_per_group;  // = qt * 32 + j
    const int qt = row >> 5, j = row & 31;
    for (int64_t w = w_first; w <= w_last; ++w) {
      const float* slot = ws + (size_t)(w + seg) * slot_floats;
      const float mc = slot[rows_per_group * kD + row];
      const float lc = slot[rows_per_group * kD + rows_per_group + row];
      floatx4 x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        x[k] = *(const floatx4*)(slot + ((size_t)(qt * 32 + e + 8 * k) * 32 + j) * 4);
      const float m_new = fmaxf(m, mc);
      const float al = __builtin_amdgcn_exp2f((m - m_new) * c);
      const float wt = __builtin_amdgcn_exp2f((mc - m_new) * c);
      l = l * al + lc * wt;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[4 * k + i] = acc[4 * k + i] * al + wt * x[k][i];
      m = m_new;
    }
  }
  if (!active) return;
  const float inv = l > 0.f ? 1.f / l : 0.f;
  uint16_t* op = a.out + ((int64_t)node * a.Hq + head) * kD;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ushortx4 y;
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = f32_to_bf16(acc[4 * k + i] * inv);
    *(ushortx4*)(op + 4 * (e + 8 * k)) = y;
  }
  if (a.lse && e == 0)
    a.lse[(int64_t)node * a.Hq + head] = l > 0.f ? m * a.scale + logf(l) : -INFINITY;
  SMART_TIMELINE(if (lane == 0 && wc < timeline::kWaves) {  // (lane 0's row always exists)
    timeline::wave_stamps[2 * wc] = tl_start;
    timeline::wave_stamps[2 * wc + 1] = wall_clock64();
  })
}

}  // namespace

namespace smart {

// Workgroups of the prefix kernel: one per compute unit (eight wavefronts, two per SIMD).  The
// plan deals them to the classes; a class never gets more workers than this bound.
static int32_t prefix_workgroups(const smart_ctx* ctx) {
  if (ctx->opt_workers > 0) return (int32_t)ctx->opt_workers;
  return ctx->num_cus > 0 ? ctx->num_cus : 256;
}
static int32_t class_workers(const smart_ctx* ctx, int cls) {
  const int32_t asked = prefix_workgroups(ctx);
  const int32_t wg = asked > kClasses ? asked : kClasses;
  (void)cls;
  return wg;  // a worker is a workgroup in every class
}
int32_t tva_mfma_default_workers(const smart_ctx* ctx) { return prefix_workgroups(ctx); }

// Segments per class a call can have at most when only the totals are known (every tree's size may be
// anything that adds up to total_nodes): one row group per sequence in classes 0 and 1; with an fp8
// cache every sequence is class 1, in row groups of 64 rows.
static void segment_bounds(int32_t batch, int32_t total_nodes, int32_t num_q_heads, int32_t num_kv_heads,
                           int64_t (&segs)[kClasses]) {
  const int64_t G = num_q_heads / num_kv_heads;
  segs[0] = (int64_t)num_kv_heads * batch;
  segs[1] = (int64_t)num_kv_heads * batch;
  segs[2] = (int64_t)num_kv_heads * (((int64_t)total_nodes * G + kLargeRows - 1) / kLargeRows + batch);
}

// The same from the trees' sizes (host copy of the offsets): exactly the segments the plan will count.
// False if the offsets are not a running sum inside [0, total_nodes].
static bool segment_counts(const int32_t* h_cu_nodes, int32_t batch, int32_t total_nodes, int32_t num_q_heads,
                           int32_t num_kv_heads, bool fp8, int64_t (&segs)[kClasses]) {
  const int G = num_q_heads / num_kv_heads;
  for (int c = 0; c < kClasses; ++c) segs[c] = 0;
  for (int32_t b = 0; b < batch; ++b) {
    const int64_t base = h_cu_nodes[b], next = h_cu_nodes[b + 1];
    if (base < 0 || next < base || next > total_nodes) return false;
    int64_t n = next - base;
    n = n > SMART_MAX_NODES ? SMART_MAX_NODES : n;
    const int rows = (int)n * G;
    if (rows == 0) continue;
    const int cls = fp8 ? plan_class<true>(rows) : seq_class(rows);
    if (cls < 2) segs[cls] += num_kv_heads;
    else segs[2] += (int64_t)num_kv_heads * ((rows + kLargeRows - 1) / kLargeRows);
  }
  return true;
}

// Slots of a class: worker w's piece of segment s goes to slot w + s.
static size_t class_slots(const smart_ctx* ctx, int cls, int64_t segs) {
  if (segs == 0) return 0;  // no sequence of this class: the plan gives it no worker
  return (size_t)class_workers(ctx, cls) + (size_t)segs + 1;
}

// Partial-result slots and arrival counters of a call with these segments.
struct Slots {
  size_t count[kClasses], floats, counters;
};
static Slots slots_for(const smart_ctx* ctx, const int64_t (&segs)[kClasses], bool finish) {
  Slots s;
  s.floats = s.counters = 0;
  for (int c = 0; c < kClasses; ++c) {
    s.count[c] = class_slots(ctx, c, segs[c]);
    s.floats += s.count[c] * (finish ? finish_slot(c) : class_slot(c));
    s.counters += (size_t)segs[c] * kWgWaves;
  }
  return s;
}

void tva_mfma_workspace(const smart_ctx* ctx, int32_t batch, int32_t total_nodes, int32_t num_q_heads,
                        int32_t num_kv_heads, size_t* ws_bytes, size_t* plan_bytes, size_t* counters) {
  int64_t segs[kClasses];
  segment_bounds(batch, total_nodes, num_q_heads, num_kv_heads, segs);
  const Slots s = slots_for(ctx, segs, false);
  // Room for both forms.  The finishing form's slots are larger, class 0's by the most; every class's are counted that much
  // larger here, so that a call whose two-launch form fits a buffer fits it in either form: it must not replace a buffer that a
  // captured launch of another call still holds.
  *ws_bytes = (s.floats * finish_slot(0) / class_slot(0) + 1) * sizeof(float);
  *plan_bytes = plan_bytes_for(batch);
  *counters = s.counters;
}

bool tva_mfma_supported(const tva_params& p) {
  auto aligned16 = [](const void* x) { return ((uintptr_t)x & 15u) == 0; };
  return p.dtype == SMART_BF16 && p.kv_layout == SMART_KV_INTERLEAVED && p.head_dim == kD &&
         p.block_size == kBlock && p.cache_block_stride % 8 == 0 && p.cache_head_stride % 8 == 0 &&
         aligned16(p.d_q) && aligned16(p.d_k_cache) && aligned16(p.d_v_cache) &&
         aligned16(p.d_k_tree) && aligned16(p.d_v_tree) && aligned16(p.d_out) && p.num_blocks > 0;
}

// Tiles of the longest prefix that the block table has room for.
static int64_t longest_prefix(const tva_params& p) {
  return ((int64_t)p.max_blocks_per_seq * kBlock + kTile - 1) / kTile;
}

// fp8 cache: the host knows the trees' mean size and what the block table can hold.  A batch of trees of one row tile has
// a mean of at most 32 rows, and a table that holds fewer than kPairTiles tiles a sequence, or too few in all for such
// shares, has no long pieces: those run the kernel that has no pairs.  With a larger mean and longer tables trees of two
// row tiles are the usual ones and gain most (64 sequences of 16384 tokens, 4 .. 10 nodes of 8 rows, 712 -> 503 us); the
// rest is decided by each worker (fp8_worker).
static bool pairs(const tva_params& p, int32_t workgroups) {
  const int64_t G = p.num_q_heads / p.num_kv_heads, longest = longest_prefix(p);
  return p.total_nodes * G > (int64_t)kSmallRows * p.batch && longest >= kPairTiles &&
         longest * p.batch * p.num_kv_heads >= (int64_t)kPairTiles * workgroups;
}

// Whether the prefix kernel finishes the rows itself.  The last of a segment's pieces is merged by one workgroup, about
// 0.85 us for each other piece of 256 rows; the combine kernel spreads that over the chip and costs a launch.  So it is left
// to the combine kernel where few segments may be long: one sequence, 8 kv heads, 60 nodes: 1000 tokens 34.5 us (combine
// 34.2), 2000 45.4 (39.0), 16384 80 (58); 16 segments of 4000 tokens 49.9 (44.8); but 32 segments of 2048 33.5 (38.5), of
// 16384 102.8 (106.9).  And pairs of row tiles from an fp8 cache have no registers left for it: 64 sequences of 3600 tokens,
// 9 .. 16 nodes 138 .. 153 us (128); by halves, and finished, they win only while prefixes are shorter: 64 sequences of 2400
// tokens 80 us (107), 32 of 4000 76 (74).
// Nor do trees of a node or a few gain where segments of long prefixes are cut into many pieces: their rows take the combine
// kernel one round trip each, and the last piece is as long as the others.  One launch / two: 8 sequences of 1 node, 8 kv heads,
// 2000 tokens 26.4 / 23.8 us, 4000 35.1 / 31.7, of 4 nodes about 6 % more, of 5 and 8 nodes 0 .. 4, but a mean of 1 .. 4 and 256
// segments 0.97 .. 1.00, 1000 tokens 0.94 .. 1.06; fp8 cache, 16 of 1 node, 4000 tokens 34.2 / 31.0, 1500 0.93 .. 1.04.  And one
// or two sequences whose trees fill several row groups leave all of them to few workgroups, with a part of 256 rows from each
// piece: one of 128 nodes, 8 kv heads, 700 tokens 40.5 / 33.5, 500 37.5 / 34.0, but 200 1.01; 16 segments 0.84 .. 1.05.
constexpr int kFewTiles = 32, kFewPieces = 8, kLongPairTiles = 120;
static bool finishes(const tva_params& p, int32_t workgroups, bool pairs_pay) {
  const int64_t longest = longest_prefix(p), segs = (int64_t)p.batch * p.num_kv_heads;
  const int64_t rows = (int64_t)p.total_nodes * (p.num_q_heads / p.num_kv_heads);
  if (pairs_pay && longest >= kLongPairTiles) return false;
  if (p.total_nodes <= 4 * (int64_t)p.batch && longest > (p.kv_cache_dtype == SMART_FP8_E4M3 ? 60 : 40) && 2 * segs <= workgroups)
    return false;
  if (rows > (int64_t)kLargeRows * p.batch && longest > 10 && 32 * segs <= workgroups) return false;
  return longest <= kFewTiles || segs * kFewPieces >= workgroups;
}

// With many segments a worker holds several, and each costs a start, a fold and a tree part beside its tiles; where every
// worker has a part of one segment, all have a start and an end, and only the tree part sets the last one apart.  (The lengths
// are not known here; the line is at a third of a segment per workgroup.)  Calls with ragged prefixes, no cost / these: 96
// sequences of 100 .. 2000 tokens, 4 .. 7 nodes 108 / 89 us, 24 .. 48 nodes 184 / 145; 64 of 100 .. 4096, 1 .. 64 nodes
// 186 / 163.  4 sequences of 2048, 4 .. 7 nodes (4, 60) 18.7, (12, 160) 21.2 us; 24 of 500, 40 nodes 33.7 and 32.2.  From an
// fp8 cache a unit of class 1 is less than half as long.
static TreeCost tree_cost(const tva_params& p, int32_t workgroups) {
  const bool fp8 = p.kv_cache_dtype == SMART_FP8_E4M3;
  if ((int64_t)p.batch * p.num_kv_heads * 3 < workgroups) return fp8 ? TreeCost{8, 60} : TreeCost{4, 60};
  return fp8 ? TreeCost{40, 160} : TreeCost{12, 160};
}

int32_t tva_launch_mfma(smart_ctx* ctx, hipStream_t stream, const tva_params& p, const TvaWorkspace* fixed) {
  if (p.batch == 0 || p.total_nodes == 0) return SMART_OK;
  const int G = p.num_q_heads / p.num_kv_heads;
  const int32_t workgroups = prefix_workgroups(ctx);
  const bool fp8 = p.kv_cache_dtype == SMART_FP8_E4M3;
  // Room for partial results: by the totals alone (the context's own workspace, grown when needed), or, in a
  // caller-provided buffer of fixed size, by the trees' sizes when the host copy of the offsets is there.  The
  // plan counts the segments again on the device and runs nothing if they do not fit.
  SegCaps caps;
  if (!fixed || !p.h_cu_nodes) {
    segment_bounds(p.batch, p.total_nodes, p.num_q_heads, p.num_kv_heads, caps.segs);
  } else if (!segment_counts(p.h_cu_nodes, p.batch, p.total_nodes, p.num_q_heads, p.num_kv_heads, fp8, caps.segs)) {
    return SMART_EINVAL;
  }
  void* ws_base;
  void* plan_base;
  int32_t *arrive = nullptr, *clear = nullptr;
  const bool pairs_pay = fp8 && pairs(p, workgroups);
  bool finish = finishes(p, workgroups, pairs_pay);
  const TreeCost tc = tree_cost(p, workgroups);
  Slots slots = slots_for(ctx, caps.segs, finish);
  const size_t plan_bytes = plan_bytes_for(p.batch);
  if (fixed) {
    if (finish && slots.floats * sizeof(float) + slots.counters * sizeof(int32_t) > fixed->ws_bytes) {
      finish = false;  // (it needs the larger slots, and counters)
      slots = slots_for(ctx, caps.segs, false);
    }
    if (slots.floats * sizeof(float) > fixed->ws_bytes || plan_bytes > fixed->plan_bytes) return SMART_ECAP;
    ws_base = fixed->ws;
    plan_base = fixed->plan;
    if (finish) {  // (nothing in this buffer is known to hold zeros)
      arrive = (int32_t*)((float*)fixed->ws + slots.floats);
      int32_t rc = zero_counters(stream, arrive, slots.counters);
      if (rc != SMART_OK) return rc;
    }
  } else {
    size_t ws_most, plan_most, counters;
    tva_mfma_workspace(ctx, p.batch, p.total_nodes, p.num_q_heads, p.num_kv_heads, &ws_most, &plan_most, &counters);
    // a launch that is being captured cannot allocate: where it is only the counters that are too few, it takes the form that
    // has none
    if (counters > ctx->counters && stream != nullptr) {
      hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();
      if (capture != hipStreamCaptureStatusNone) {
        finish = false;
        slots = slots_for(ctx, caps.segs, false);
        counters = 0;
      }
    }
    int32_t rc = ensure_workspace(ctx, stream, ws_most, plan_most, counters);
    if (rc != SMART_OK) return rc;
    ws_base = ctx->ws;
    plan_base = ctx->plan;
    if (finish) next_counters(ctx, &arrive, &clear);
  }
  float* ws[kClasses];
  ws[0] = (float*)ws_base;
  for (int c = 1; c < kClasses; ++c)
    ws[c] = ws[c - 1] + slots.count[c - 1] * (finish ? finish_slot(c - 1) : class_slot(c - 1));

  if (p.batch > kWave) {  // smaller batches: the prefix kernel derives the plan itself
    auto plan = fp8 ? (finish ? tva_plan_kernel<true, true> : tva_plan_kernel<true, false>)
                    : (finish ? tva_plan_kernel<false, true> : tva_plan_kernel<false, false>);
    hipLaunchKernelGGL(plan, dim3(1), dim3(kWave), 0, stream, plan_base, p.batch, p.total_nodes, G, p.num_kv_heads,
                       p.max_blocks_per_seq, workgroups, caps, tc, p.d_prefix_len, p.d_cu_nodes);
    SMART_HIP_CHECK(hipGetLastError());
  }

  MainArgs ma;
  ma.q = (const __bf16*)p.d_q;
  ma.k_cache = (const __bf16*)p.d_k_cache;
  ma.v_cache = (const __bf16*)p.d_v_cache;
  ma.block_table = p.d_block_table;
  ma.cu_nodes = p.d_cu_nodes;
  ma.prefix_len = p.d_prefix_len;
  ma.total_nodes = p.total_nodes;
  ma.workgroups = workgroups;
  ma.plan = plan_base;
  ma.caps = caps;
  ma.tree_cost = tc;
  for (int c = 0; c < kClasses; ++c) ma.ws[c] = ws[c];
  ma.block_stride = p.cache_block_stride;
  ma.head_stride = p.cache_head_stride;
  ma.batch = p.batch;
  ma.Hq = p.num_q_heads;
  ma.Hkv = p.num_kv_heads;
  ma.G = G;
  ma.max_blocks = p.max_blocks_per_seq;
  ma.num_blocks = p.num_blocks;
  ma.scale_log2e = p.softmax_scale * kLog2e * (fp8 ? p.k_scale : 1.f);
  ma.m_scale = fp8 ? p.k_scale : 1.f;
  ma.o_scale = fp8 ? p.v_scale : 1.f;
  ma.status = p.d_status;
  ma.fin.q = ma.q;
  ma.fin.k_tree = (const __bf16*)p.d_k_tree;
  ma.fin.v_tree = (const __bf16*)p.d_v_tree;
  ma.fin.anc_mask = (const uint32_t*)p.d_anc_mask;
  ma.fin.out = (__bf16*)p.d_out;
  ma.fin.lse = p.d_lse;
  ma.fin.arrive = arrive;
  ma.fin.clear = clear;
  ma.fin.n_clear = clear ? (int32_t)ctx->counters : 0;
  for (int c = 0, first = 0; c < kClasses; first += (int)caps.segs[c++]) {
    ma.fin.ws[c] = ws[c];
    ma.fin.arrive_first[c] = first;
  }
  ma.fin.Hq = p.num_q_heads;
  ma.fin.Hkv = p.num_kv_heads;
  ma.fin.G = G;
  ma.fin.scale = p.softmax_scale;
  ma.fin.scale_log2e = p.softmax_scale * kLog2e;
  // (every class with work needs a workgroup, however few were asked for)
  const dim3 grid(workgroups > kClasses ? workgroups : kClasses);
  hipEvent_t ev_start = nullptr, ev_stop = nullptr;
  // (no events: an ordinary launch; else the events ride on the dispatch and hold the kernel's own start and end)
  const bool recorded = profile_events(ctx, &ev_start, &ev_stop);
  auto launch = [&](void (*kernel)(MainArgs)) {
    if (recorded) hipExtLaunchKernelGGL(kernel, grid, dim3(kWgWaves * kWave), 0, stream, ev_start, ev_stop, 0, ma);
    else hipLaunchKernelGGL(kernel, grid, dim3(kWgWaves * kWave), 0, stream, ma);
  };
  if (pairs_pay && !finish) launch(tva_prefix_kernel<true, true, false>);
  else if (fp8) launch(finish ? tva_prefix_kernel<true, false, true> : tva_prefix_kernel<true, false, false>);
  else launch(finish ? tva_prefix_kernel<false, false, true> : tva_prefix_kernel<false, false, false>);
  SMART_HIP_CHECK(hipGetLastError());
  if (recorded) profile_launched(ctx);
  if (finish) return SMART_OK;

  CombineArgs ca;
  ca.q = (const uint16_t*)p.d_q;
  ca.k_tree = (const uint16_t*)p.d_k_tree;
  ca.v_tree = (const uint16_t*)p.d_v_tree;
  ca.cu_nodes = p.d_cu_nodes;
  ca.anc_mask = p.d_anc_mask;
  ca.plan = plan_base;
  for (int c = 0; c < kClasses; ++c) ca.ws[c] = ws[c];
  ca.out = (uint16_t*)p.d_out;
  ca.lse = p.d_lse;
  ca.batch = p.batch;
  ca.Hq = p.num_q_heads;
  ca.Hkv = p.num_kv_heads;
  ca.G = G;
  ca.scale = p.softmax_scale;
  ca.scale_log2e = p.softmax_scale * kLog2e;
  ca.only_small = fp8 ? 1 : 0;
  ca.block_table = p.d_block_table;
  ca.prefix_len = p.d_prefix_len;
  ca.status = p.d_status;
  ca.max_blocks = p.max_blocks_per_seq;
  ca.num_blocks = p.num_blocks;
  const int64_t max_chunks =
      (int64_t)p.num_kv_heads * (((int64_t)p.total_nodes * G + kCombineRows - 1) / kCombineRows + p.batch);
  if (max_chunks > 0x7FFFFFFF) return SMART_EINVAL;
  hipLaunchKernelGGL(tva_combine_kernel, dim3((unsigned)max_chunks), dim3(kWave), 0, stream, ca);
  SMART_HIP_CHECK(hipGetLastError());
  return SMART_OK;
}

}  // namespace smart

#ifdef SMART_TVA_TIMELINE
// Stamps of the last launch on the current device into host arrays of 4 x 1024 and 2 x 16384 words (unused entries
// are zero after smart_timeline_clear); both calls synchronize the device.
extern "C" int32_t smart_timeline_read(uint64_t* h_workgroups, uint64_t* h_waves) {
  if (!h_workgroups || !h_waves) return SMART_EINVAL;
  SMART_HIP_CHECK(hipDeviceSynchronize());
  SMART_HIP_CHECK(hipMemcpyFromSymbol(h_workgroups, HIP_SYMBOL(timeline::wg_stamps), sizeof(timeline::wg_stamps)));
  SMART_HIP_CHECK(hipMemcpyFromSymbol(h_waves, HIP_SYMBOL(timeline::wave_stamps), sizeof(timeline::wave_stamps)));
  return SMART_OK;
}
extern "C" int32_t smart_timeline_clear() {
  SMART_HIP_CHECK(hipDeviceSynchronize());
  void* p = nullptr;
  SMART_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(timeline::wg_stamps)));
  SMART_HIP_CHECK(hipMemset(p, 0, sizeof(timeline::wg_stamps)));
  SMART_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(timeline::wave_stamps)));
  SMART_HIP_CHECK(hipMemset(p, 0, sizeof(timeline::wave_stamps)));
  return SMART_OK;
}
#endif
