// tree_verify_attention, tiled matrix-core path for what the interleaved-cache bf16 path does not cover: fp32 and
// bf16, both cache layouts, head dims 64 and 128, any block size, fp8 caches.
//
// The prefix is a dense contraction of all rows of a kv head (tree nodes x query heads of the group) with the cached
// keys, so a workgroup takes a row group of up to 128 rows and streams the keys past it: every K/V byte leaves HBM once
// per row group, instead of once per (node, head) as in the general kernel, and the products run on the matrix cores.
//
//   * A step is four tiles of 32 keys (bf16) or 16 keys (fp32): 64 KB of K and V at head dim 128.  The 512 threads of a
//     workgroup load a step with 16-byte loads into registers while the step before is being computed, and put it into
//     the other of two LDS stages; one barrier per step.  (Eight wavefronts and not twice four: half the staging
//     registers per thread.  With four the compiler spilled, and reloading a spill waits for every load in flight:
//     the prefix kernel of the first workload below took 152 us instead of 98.)
//   * Eight wavefronts, two per SIMD.  With up to 32 rows four of them take one tile of the step each, with up to 64 rows
//     four wavefronts share a row tile, with more two do.  The states that share a row tile are folded through LDS
//     at the end of a piece, in a fixed order.
//   * Scores are kept transposed (keys x rows): a row's softmax stays inside a lane (and its partner lanes), and the
//     probabilities come out in the operand layout of the second product.
//   * Plain pages are staged row by row with their 16-byte chunks permuted by row, so that the score product's reads
//     (one row per lane) and the output product's reads (transposing LDS reads, ds_read_b64_tr_b16, for bf16) are both
//     free of bank conflicts.  Interleaved pages are staged in operand order.
//   * Nothing is rounded below what the general kernel holds: bf16 products are exact in binary32, a probability goes
//     into the second product as the sum of three bf16 values, which is its binary32 value exactly (three MFMAs per
//     tile instead of one; the loop is bound by its loads up to about 100 rows), and fp32 uses the fp32 MFMAs.
//   * The same range, too.  A probability's smaller parts are often zero or negative and make NaN of an infinite value,
//     and probabilities above 1 (kRescaleStep) can take the product with a very large one past binary32.  So a row that
//     comes out infinite or NaN is evaluated once more, key by key (Finish::walk).  Looking at the finished rows takes the
//     first workload below from 99.2 us to 99.7 and the workspace-free form from 10.6 .. 47.0 us to 10.9 .. 47.7; a look at
//     every staged value took it to 102, smaller parts kept off the infinities inside the loop to 105, a loop that
//     can go over a piece again to 104 (its offsets spill).
//
// Two forms.  Split: the units (steps of all segments = (sequence, kv head, row group)) are cut into equal shares, one
// per workgroup, every piece leaves a partial (max, sum, O) in slot workgroup + segment, and a second kernel merges
// them with the tree part.  Direct: one workgroup per segment, which also does the tree part; needs no workspace.
//
// The tree part (a node sees only itself and its ancestors, a handful of keys chosen by a 128-bit mask) is evaluated
// on the vector ALUs in fp32 by walking the set bits, so what other nodes hold never enters a row.
//
// Measured against the general kernel (whole call): bf16 plain pages, batch 16, 32 / 8 heads of 128, prefixes of
// 1024 .. 4096, trees of 4 .. 64 nodes 12.9 ms -> 96 us (prefix kernel 86, of which 62 are the MFMAs of its fullest
// workgroups; finishing kernel 18); fp32 plain pages, batch 8, 8 / 2 heads of 64, prefixes of 128 .. 1536, 15-node trees
// 778 -> 19 us, and its error against binary64 falls from 5.6e-7 to 3.1e-7 (shorter sums).
//
// The paper (Sec. 1) has the target model verify the tree in one forward pass; this is the attention sub-step.
#include <math.h>

#include "common.h"
#include "wave.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short shortx4;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(8))) float floatx8;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) uint32_t uintx4;
typedef __attribute__((ext_vector_type(2))) uint32_t uintx2;
typedef __attribute__((ext_vector_type(2))) float floatx2;

constexpr int kWave = 64;
constexpr int kWaves = 8;
constexpr int kThreads = kWave * kWaves;
constexpr int kRowTile = 32;
constexpr int kGroupRows = 128;      // rows of a row group: four row tiles
constexpr int kTilesPerStep = 4;
constexpr int kCombineLanes = 8;     // lanes per row in the finishing step
constexpr float kLog2e = 1.4426950408889634f;
// The value the exponentials are taken against follows the running maximum only when that has moved more than
// 2^kRescaleStep above it (in the exponent's units): a partial's max, sum and O stay consistent with each other.
constexpr float kRescaleStep = 8.f;

template <typename T> struct TileKeys;
template <> struct TileKeys<__bf16> { static constexpr int value = 32; };
template <> struct TileKeys<float> { static constexpr int value = 16; };
template <typename T> constexpr int step_keys() { return kTilesPerStep * TileKeys<T>::value; }

__host__ __device__ constexpr int slot_floats(int D) { return kGroupRows * (D + 2); }

struct TiledArgs {
  const void* q;
  const void* k_tree;
  const void* v_tree;
  const void* k_cache;
  const void* v_cache;
  const int32_t* block_table;
  const int32_t* prefix_len;
  const int32_t* cu_nodes;
  const uint64_t* anc_mask;
  void* out;
  float* lse;
  int32_t* status;
  float* ws;       // split form: partial slots
  int64_t* plan;   // split form: units, workers, then per sequence the units and the segments before it
  int64_t block_stride, head_stride, token_stride;
  int32_t batch, total_nodes, Hq, Hkv, G, block_size, max_blocks, num_blocks;
  int32_t segment_cost;   // units of a segment beside its steps
  bool fp8, plain;        // the cache's element type and layout, where they are no template arguments
  uint32_t block8_magic;  // token / 8 / (block_size / 8) by multiplication
  float scale;
  float c;         // softmax scale in powers of two (log2 e folded in)
  float c_stored;  // the same against stored key values: c k_scale
  float m_scale;   // = k_scale: row maxima leave the prefix kernel in true units
  float o_scale;   // = v_scale
};

// The unit the split form cuts into shares is a cost: a step of a row group with r row tiles counts StepCost, a segment
// beside its steps segment_cost (behind them; a share that begins there leaves no partial).  The two wavefronts of a SIMD
// have one tile of a step between them with one row tile, two with two, four with three or four (the third's SIMD partner
// idles).  Stamps, bf16, the first workload above: 2.06 us a step with one row tile, 2.75 with two, 4.35 with three, 4.42 with
// four (with 4, 4, 7 units the call took 104 us, with these 101); the fp32 products always set the pace.
template <typename T> struct StepCost;
template <> struct StepCost<__bf16> { static constexpr int one = 4, two = 5, four = 8; };
template <> struct StepCost<float> { static constexpr int one = 4, two = 7, four = 14; };

// What a call uses of one sequence: lengths and sizes clamped to what the arrays hold.  A range that leaves the arrays
// has no rows (nothing of it is read).
struct Shape {
  int len, base, n, rows, groups, steps;
  int cost_last;       // of a step of the last row group (the others: StepCost::four)
  int64_t full, head;  // units of a full row group, of a kv head
};

template <typename T>
__device__ inline Shape shape_of(const TiledArgs& a, int len, int base, int next) {
  Shape s;
  const int cap = a.max_blocks * a.block_size;
  s.len = len < 0 ? 0 : (len > cap ? cap : len);
  int64_t n = (int64_t)next - base;
  n = n < 0 ? 0 : (n > SMART_MAX_NODES ? SMART_MAX_NODES : n);
  if (base < 0 || base + n > a.total_nodes) n = 0;
  s.base = base;
  s.n = (int)n;
  s.rows = s.n * a.G;
  s.groups = (s.rows + kGroupRows - 1) / kGroupRows;
  s.steps = s.groups > 0 ? (s.len + step_keys<T>() - 1) / step_keys<T>() : 0;
  const int last = s.rows - (s.groups - 1) * kGroupRows;
  s.cost_last = last <= kRowTile ? StepCost<T>::one : (last <= 2 * kRowTile ? StepCost<T>::two : StepCost<T>::four);
  const int extra = s.steps > 0 ? a.segment_cost : 0;
  s.full = (int64_t)s.steps * StepCost<T>::four + extra;
  s.head = s.groups > 0 ? (s.groups - 1) * s.full + (int64_t)s.steps * s.cost_last + extra : 0;
  return s;
}

// Where a unit (or, in the direct form, a segment) lies: its sequence and what comes before that.
struct Place {
  int b;
  int64_t units_before, segs_before;
};

// What lies before a place in the batch, or in all of it.  Ascending offsets make the sequences' ranges disjoint, which is
// what the segments and slots of a call were counted by; a call whose offsets are not ascending has no segments at all and
// its rows are evaluated one by one (Finish::walk), each for the sequence that owner_of finds, like the general kernel's.
struct Sums {
  int64_t units, segs, steps;
  int flags;
};
constexpr int kDescending = 1;  // an offset is smaller than the one before it
constexpr int kIrregular = 2;   // a range leaves the arrays or holds more nodes than a tree can have

// One wavefront goes through chunks c0 .. c1 - 1 of 64 sequences: visit(first sequence, lane has one, its units and segments,
// units and segments before it); `sums` moves from before the chunks to behind them.
template <typename T, typename Visit>
__device__ inline void scan_batch(const TiledArgs& a, int lane, int c0, int c1, Sums* sums, Visit visit) {
  for (int b0 = c0 * kWave; b0 < min(c1 * kWave, a.batch); b0 += kWave) {
    const int b = min(b0 + lane, a.batch - 1);
    const int base = a.cu_nodes[b], next = a.cu_nodes[b + 1];
    const Shape s = shape_of<T>(a, a.prefix_len[b], base, next);
    const bool there = b0 + lane < a.batch;
    if (__any(next < base)) sums->flags |= kDescending;
    if (__any(s.n != (int64_t)next - base)) sums->flags |= kIrregular;
    const int64_t segs = there ? (int64_t)s.groups * a.Hkv : 0;
    const int64_t units = there ? s.head * a.Hkv : 0;
    int64_t tu, ts, tt;
    smart::wave_excl_scan(segs * s.steps, lane, &tt);
    const int64_t eu = smart::wave_excl_scan(units, lane, &tu) + sums->units;
    const int64_t es = smart::wave_excl_scan(segs, lane, &ts) + sums->segs;
    visit(b0, there, units, segs, eu, es);
    sums->units += tu;
    sums->segs += ts;
    sums->steps += tt;
  }
}

__device__ inline int clamp_block(int b, int num_blocks) { return b < 0 ? 0 : (b >= num_blocks ? num_blocks - 1 : b); }

// Row m of a 16-row half of the score tile holds key sigma(m) when the values are staged as vectors of 8 consecutive
// keys: swapping bits 2 and 3 makes the eight registers a lane ends up with eight consecutive keys.
__device__ inline int sigma(int m) { return (m & 3) | ((m & 4) << 1) | ((m & 8) >> 1); }

__device__ inline float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float max_rows16(float x) {  // over the lanes with the same lane % 16
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float sum_rows16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return sum_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// exp2((x - m) c) with an empty reference (m = -inf: no key so far scored above -inf) giving 0 for x = -inf.
__device__ inline float weight(float x, float m, float c) {
  return __builtin_amdgcn_exp2f((x - (m == -INFINITY ? 0.f : m)) * c);
}

// ---- staging: global memory -> registers -> LDS --------------------------------------------------------------------
// A chunk is 16 bytes of T in LDS: 8 bf16 or 4 fp32 elements, which come from as many bytes / 2 or / 4 of an fp8 cache.
template <typename T, bool kFp8> struct RawChunk;
template <> struct RawChunk<__bf16, false> { typedef uintx4 type; };
template <> struct RawChunk<float, false> { typedef uintx4 type; };
template <> struct RawChunk<__bf16, true> { typedef uintx2 type; };
template <> struct RawChunk<float, true> { typedef uint32_t type; };

__device__ inline uintx4 staged(uintx4 x, float) { return x; }
__device__ inline uintx4 staged(uintx4 x, __bf16) { return x; }
__device__ inline uintx4 staged(uintx2 x, __bf16) {  // eight E4M3 bytes -> bf16, exactly
  const bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[0], 1.0f, false);
  const bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[0], 1.0f, true);
  const bf16x2 c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[1], 1.0f, false);
  const bf16x2 d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[1], 1.0f, true);
  bf16x8 r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
  return __builtin_bit_cast(uintx4, r);
}
__device__ inline uintx4 staged(uint32_t x, float) {  // four E4M3 bytes -> fp32, exactly
  floatx4 r;
  r[0] = __builtin_amdgcn_cvt_f32_fp8(x, 0);
  r[1] = __builtin_amdgcn_cvt_f32_fp8(x, 1);
  r[2] = __builtin_amdgcn_cvt_f32_fp8(x, 2);
  r[3] = __builtin_amdgcn_cvt_f32_fp8(x, 3);
  return __builtin_bit_cast(uintx4, r);
}

// The permutation of a plain row's chunks in LDS: chunk c of row `key` lies at position c ^ swizzle(key).  Sixteen
// consecutive rows put the same chunk at sixteen positions of a 256-byte line (the score product reads one row per
// lane), and four consecutive rows put a pair of chunks at four different pairs (the transposing reads).
template <typename T, int D>
__device__ inline int swizzle(int key) {
  if (sizeof(T) == 4) return key & 15;
  if (D == 128) return ((key & 7) << 1) | ((key >> 3) & 1);
  return (((key >> 1) & 3) << 1) | ((key >> 3) & 1);
}

template <typename T, bool kFp8, bool kPlain, int D>
struct Stager {
  typedef typename RawChunk<T, kFp8>::type Raw;
  static constexpr int kE = 16 / (int)sizeof(T);          // elements per chunk
  static constexpr int kTileChunks = 4 * D;               // chunks of a tile's K (or V)
  static constexpr int kStepChunks = kTilesPerStep * kTileChunks;
  static constexpr int kPer = kStepChunks / kThreads;     // chunks a thread moves per step, of K and of V
  static constexpr int kKeys = TileKeys<T>::value;
  static constexpr int kStepKeys = step_keys<T>();

  int32_t idk[kPer], idv[kPlain ? 1 : kPer];
  Raw k[kPer], v[kPer];

  // Key of the step that chunk p of K / of V starts at, and the chunk's element offset in its page given the slot.
  __device__ static int key_of_k(int p) {
    if (kPlain) return p / (D / kE);
    const int x = p % kTileChunks, tile = p / kTileChunks;
    return tile * kKeys + (sizeof(T) == 2 ? x & 31 : (x >> 1) & 15);
  }
  __device__ static int key_of_v(int p) {
    if (kPlain) return key_of_k(p);
    const int x = p % kTileChunks, tile = p / kTileChunks;
    return tile * kKeys + 8 * (sizeof(T) == 2 ? x / D : (x >> 1) / D);
  }
  __device__ static int64_t offset_k(const TiledArgs& a, int p, int slot) {
    if (kPlain) {
      const int key = p / (D / kE);
      return (int64_t)slot * a.token_stride + ((p % (D / kE)) ^ swizzle<T, D>(key)) * kE;
    }
    const int x = p % kTileChunks;
    if (sizeof(T) == 2) return ((x >> 5) * a.block_size + slot) * 8;
    return ((x >> 5) * a.block_size + slot) * 8 + 4 * (x & 1);
  }
  __device__ static int64_t offset_v(const TiledArgs& a, int p, int slot) {
    if (kPlain) return offset_k(a, p, slot);
    const int x = p % kTileChunks;
    if (sizeof(T) == 2) return ((slot >> 3) * D + x % D) * 8;
    return ((slot >> 3) * D + (x >> 1) % D) * 8 + 4 * (x & 1);
  }
  // Token of a key of the step, kept inside the prefix (what lies past it is masked later): a V vector of an
  // interleaved page starts at a multiple of 8.
  __device__ static int token_k(int step, int key, int len) { return min(step * kStepKeys + key, len - 1); }
  __device__ static int token_v(int step, int key, int len) {
    return kPlain ? token_k(step, key, len) : min(step * kStepKeys + key, (len - 1) & ~7);
  }
  __device__ static int block_of(const TiledArgs& a, int token) {
    return (int)__umulhi(((uint32_t)token >> 3) << 1, a.block8_magic);
  }

  __device__ void load_ids(const TiledArgs& a, const int32_t* row, int step, int len, int tid) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      idk[i] = row[block_of(a, token_k(step, key_of_k(i * kThreads + tid), len))];
      if (!kPlain) idv[i] = row[block_of(a, token_v(step, key_of_v(i * kThreads + tid), len))];
    }
  }
  __device__ void load(const TiledArgs& a, int step, int len, int g, int tid) {
    constexpr int kB = kFp8 ? 1 : (int)sizeof(T);  // bytes of a cache element
    const char* kc = (const char*)a.k_cache + (int64_t)g * a.head_stride * kB;
    const char* vc = (const char*)a.v_cache + (int64_t)g * a.head_stride * kB;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int p = i * kThreads + tid;
      const int tk = token_k(step, key_of_k(p), len);
      const int64_t at = clamp_block(idk[i], a.num_blocks) * a.block_stride +
                         offset_k(a, p, tk - block_of(a, tk) * a.block_size);
      k[i] = *(const Raw*)(kc + at * kB);
      if (kPlain) v[i] = *(const Raw*)(vc + at * kB);
    }
    if (!kPlain) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int p = i * kThreads + tid;
        const int tv = token_v(step, key_of_v(p), len);
        const int64_t at = clamp_block(idv[i], a.num_blocks) * a.block_stride +
                           offset_v(a, p, tv - block_of(a, tv) * a.block_size);
        v[i] = *(const Raw*)(vc + at * kB);
      }
    }
  }
  // `n_valid`: keys of this step inside the prefix.  Values past it become zero (their slots may hold anything, NaN
  // included, and they are multiplied by probabilities of zero); their scores are masked.
  __device__ void store(uintx4* lds, int tid, int n_valid) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      lds[i * kThreads + tid] = staged(k[i], T());
      lds[kStepChunks + i * kThreads + tid] = staged(v[i], T());
    }
    if (n_valid >= kStepKeys) return;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int p = i * kThreads + tid;
      uintx4& x = lds[kStepChunks + p];
      if (kPlain) {
        if (key_of_v(p) >= n_valid) x = (uintx4)(0u);
      } else if (sizeof(T) == 2) {  // eight keys of one head dim
        const int keep = n_valid - key_of_v(p);
        uintx4 y = x;
#pragma unroll
        for (int w = 0; w < 4; ++w) y[w] = keep >= 2 * w + 2 ? y[w] : (keep == 2 * w + 1 ? y[w] & 0xFFFFu : 0u);
        x = y;
      } else {  // four keys of one head dim
        const int keep = n_valid - key_of_v(p) - 4 * (p & 1);
        uintx4 y = x;
#pragma unroll
        for (int w = 0; w < 4; ++w) y[w] = w < keep ? y[w] : 0u;
        x = y;
      }
    }
  }
};

// Eight bf16 widened.  kInPlace: out of the four registers that hold them, a shift or a mask each.  Converted with the vector
// type's own conversion the compiler rounds every element a second time to have it in the upper half of a register: 32 of
// a tile's 200 vector instructions, which take their SIMD's issue beside the matrix ones.  The bits are the same.  Plain bf16,
// batch of 16: 97.7 -> 95.6 us, 16 sequences of 100 .. 800 tokens, 64 / 8 heads of 64 55.8 -> 53.8, of 500 .. 4000 with 64 .. 128
// nodes 166.2 -> 163.3.  Not from an fp8 cache, whose conversions fill the same places (16 of 500 .. 2000 48.4 -> 49.0).
template <bool kInPlace>
__device__ inline floatx8 unpacked(bf16x8 x) {
  if (!kInPlace) return __builtin_convertvector(x, floatx8);
  const uintx4 w = __builtin_bit_cast(uintx4, x);
  floatx8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float even, odd;  // (in assembly, or the compiler looks through the packing)
    asm("v_lshlrev_b32 %0, 16, %1" : "=v"(even) : "v"(w[i]));
    asm("v_and_b32 %0, 0xffff0000, %1" : "=v"(odd) : "v"(w[i]));
    r[2 * i] = even;
    r[2 * i + 1] = odd;
  }
  return r;
}

// ---- one wavefront's 32 rows against one staged tile ------------------------------------------------------------------
template <typename T, bool kPlain, int D> struct Rows;

typedef __attribute__((address_space(3))) shortx4 lds_shortx4;

template <bool kPlain, int D>
struct Rows<__bf16, kPlain, D> {
  static constexpr int kRowChunks = D / 8;
  bf16x8 q[D / 16];
  floatx16 o[D / 32];
  float m, l;  // of row lane % 32; l: this half-wavefront's keys

  __device__ void begin(const TiledArgs& a, int base, int g, int row0, int rows, int lane) {
    const int h = lane >> 5, j = lane & 31;
    const int rho = min(row0 + j, rows - 1);  // padding rows repeat the last real row; never read back
    const int node = base + rho / a.G, head = g * a.G + rho % a.G;
    const __bf16* qp = (const __bf16*)a.q + ((int64_t)node * a.Hq + head) * D + h * 8;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) q[ks] = *(const bf16x8*)(qp + ks * 16);
    reset();
  }
  __device__ void reset() {
#pragma unroll
    for (int jt = 0; jt < D / 32; ++jt) o[jt] = (floatx16)(0.f);
    m = -INFINITY;
    l = 0.f;
  }
  __device__ static int key_of_row(int i) { return kPlain ? i : (i & 16) + sigma(i & 15); }

  template <bool kInPlace>
  __device__ void tile(const uintx4* kt, const uintx4* vt, int n_valid, float c, int lane) {
    const int h = lane >> 5, j = lane & 31;
    const int key = key_of_row(j);
    bf16x8 kx[D / 16];  // all operands of a product are requested before its first MFMA
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const int chunk = 2 * ks + h;
      kx[ks] = __builtin_bit_cast(bf16x8, kt[kPlain ? key * kRowChunks + (chunk ^ swizzle<__bf16, D>(key)) : chunk * 32 + key]);
    }
    floatx16 s = (floatx16)(0.f);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx[ks], q[ks], s, 0, 0, 0);
    bf16x8 v[2][D / 32];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int jt = 0; jt < D / 32; ++jt) v[kk][jt] = value_operand(vt, jt, kk, lane);
    if (n_valid < 32) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key_of_row(8 * (r >> 2) + 4 * h + (r & 3)) >= n_valid) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = max_halves(mx);
    const float m_new = fmaxf(m, mx);
    if (__any((m_new - m) * c > kRescaleStep)) {
      const float alpha = weight(m, m_new, c);
      l *= alpha;
#pragma unroll
      for (int jt = 0; jt < D / 32; ++jt) o[jt] *= alpha;
      m = m_new;
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      floatx8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = weight(s[8 * kk + e], m, c);
      l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      // p = hi + mid + lo exactly: three bf16 values hold the 24 bits of a binary32
      const bf16x8 hi = __builtin_convertvector(p, bf16x8);
      const floatx8 r1 = p - unpacked<kInPlace>(hi);
      const bf16x8 mid = __builtin_convertvector(r1, bf16x8);
      const bf16x8 lo = __builtin_convertvector(r1 - unpacked<kInPlace>(mid), bf16x8);
#pragma unroll
      for (int jt = 0; jt < D / 32; ++jt) o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[kk][jt], hi, o[jt], 0, 0, 0);
#pragma unroll
      for (int jt = 0; jt < D / 32; ++jt) o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[kk][jt], mid, o[jt], 0, 0, 0);
#pragma unroll
      for (int jt = 0; jt < D / 32; ++jt) o[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[kk][jt], lo, o[jt], 0, 0, 0);
    }
  }
  // Lane (h, j): head dim 32 jt + j of the eight keys whose probabilities the lane's half holds in registers 8 kk ...
  __device__ static bf16x8 value_operand(const uintx4* vt, int jt, int kk, int lane) {
    const int h = lane >> 5, j = lane & 31;
    if (!kPlain) return __builtin_bit_cast(bf16x8, vt[(2 * kk + h) * D + 32 * jt + j]);
    // transposing read: sixteen lanes fetch four rows of sixteen elements, lane i receives column i
    const int li = lane & 15, jh = (lane >> 4) & 1;
    shortx4 part[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int token = 16 * kk + 8 * half + 4 * h + (li >> 2);
      const int chunk = 4 * jt + 2 * jh + ((li & 3) >> 1);
      const char* at = (const char*)(vt + token * kRowChunks + (chunk ^ swizzle<__bf16, D>(token))) + 8 * (li & 1);
      part[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)at);
    }
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
  }
  // The state in LDS: O as [d / 4][32 rows][4], the row maxima, the row sums.
  __device__ void put(float* region, int lane) {
    const int h = lane >> 5, j = lane & 31;
#pragma unroll
    for (int jt = 0; jt < D / 32; ++jt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        floatx4 x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = o[jt][4 * r4 + i];
        ((floatx4*)region)[(8 * jt + 2 * r4 + h) * kRowTile + j] = x;
      }
    const float sum = sum_halves(l);
    if (h == 0) {
      region[kRowTile * D + j] = m;
      region[kRowTile * D + kRowTile + j] = sum;
    }
  }
};

template <bool kPlain, int D>
struct Rows<float, kPlain, D> {
  static constexpr int kRowChunks = D / 4;
  floatx4 q[2][D / 16];
  floatx4 o[2][D / 16];
  float m[2], l[2];  // of rows lane % 16 and lane % 16 + 16; l: this quarter-wavefront's keys

  __device__ void begin(const TiledArgs& a, int base, int g, int row0, int rows, int lane) {
    const int quarter = lane >> 4, j = lane & 15;
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
      const int rho = min(row0 + 16 * nh + j, rows - 1);
      const int node = base + rho / a.G, head = g * a.G + rho % a.G;
      const float* qp = (const float*)a.q + ((int64_t)node * a.Hq + head) * D + 4 * quarter;
#pragma unroll
      for (int s = 0; s < D / 16; ++s) q[nh][s] = *(const floatx4*)(qp + 16 * s);
    }
    reset();
  }
  __device__ void reset() {
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
#pragma unroll
      for (int t = 0; t < D / 16; ++t) o[nh][t] = (floatx4)(0.f);
      m[nh] = -INFINITY;
      l[nh] = 0.f;
    }
  }
  template <bool kInPlace>
  __device__ void tile(const uintx4* kt, const uintx4* vt, int n_valid, float c, int lane) {
    const int quarter = lane >> 4, i = lane & 15;
    floatx4 s[2] = {(floatx4)(0.f), (floatx4)(0.f)};
    // contraction step (t, e): the four quarters hold head dims 16 t + 4 quarter + e
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      const int chunk = 4 * t + quarter;
      const int at = kPlain ? i * kRowChunks + (chunk ^ swizzle<float, D>(i)) : ((chunk >> 1) * 16 + i) * 2 + (chunk & 1);
      const floatx4 k = __builtin_bit_cast(floatx4, kt[at]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int nh = 0; nh < 2; ++nh) s[nh] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[e], q[nh][t][e], s[nh], 0, 0, 0);
    }
    // register r of a lane: key 4 quarter + r
    const bool ragged = n_valid < 16;
    floatx4 p[2];
    float m_new[2];
    bool move = false;
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
      if (ragged) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * quarter + r >= n_valid) s[nh][r] = -INFINITY;
      }
      const float mx = max_rows16(fmaxf(fmaxf(s[nh][0], s[nh][1]), fmaxf(s[nh][2], s[nh][3])));
      m_new[nh] = fmaxf(m[nh], mx);
      move = move || (m_new[nh] - m[nh]) * c > kRescaleStep;
    }
    if (__any(move)) {
#pragma unroll
      for (int nh = 0; nh < 2; ++nh) {
        const float alpha = weight(m[nh], m_new[nh], c);
        l[nh] *= alpha;
#pragma unroll
        for (int t = 0; t < D / 16; ++t) o[nh][t] *= alpha;
        m[nh] = m_new[nh];
      }
    }
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
#pragma unroll
      for (int r = 0; r < 4; ++r) p[nh][r] = weight(s[nh][r], m[nh], c);
      l[nh] += (p[nh][0] + p[nh][1]) + (p[nh][2] + p[nh][3]);
    }
    if (kPlain) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int token = 4 * quarter + r;
#pragma unroll
        for (int u = 0; u < D / 64; ++u) {  // lane i: head dims 64 u + 4 i + e
          const floatx4 v = __builtin_bit_cast(floatx4, vt[token * kRowChunks + ((16 * u + i) ^ swizzle<float, D>(token))]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nh = 0; nh < 2; ++nh)
              o[nh][4 * u + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], p[nh][r], o[nh][4 * u + e], 0, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < D / 16; ++t) {  // lane i: head dim 16 t + i of the quarter's four keys
        const floatx4 v = __builtin_bit_cast(floatx4, vt[((quarter >> 1) * D + 16 * t + i) * 2 + (quarter & 1)]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int nh = 0; nh < 2; ++nh)
            o[nh][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r], p[nh][r], o[nh][t], 0, 0, 0);
      }
    }
  }
  __device__ void put(float* region, int lane) {
    const int quarter = lane >> 4, j = lane & 15;
    floatx4* dst = (floatx4*)region;
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
      const int row = 16 * nh + j;
      if (kPlain) {  // register r of accumulator 4 u + e: head dim 64 u + 16 quarter + 4 r + e
#pragma unroll
        for (int u = 0; u < D / 64; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            floatx4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = o[nh][4 * u + e][r];
            dst[(16 * u + 4 * quarter + r) * kRowTile + row] = x;
          }
      } else {  // register r of accumulator t: head dim 16 t + 4 quarter + r
#pragma unroll
        for (int t = 0; t < D / 16; ++t) dst[(4 * t + quarter) * kRowTile + row] = o[nh][t];
      }
      const float sum = sum_rows16(l[nh]);
      if (quarter == 0) {
        region[kRowTile * D + row] = m[nh];
        region[kRowTile * D + kRowTile + row] = sum;
      }
    }
  }
};

constexpr int region_floats(int D) { return kRowTile * (D + 2); }

// ---- finishing a row: the tree part, then the prefix partials ------------------------------------------------------
// Four elements as they lie in memory (converted where they are used: half the registers for bf16).
template <typename T> struct Four { typedef floatx4 type; };
template <> struct Four<__bf16> { typedef bf16x4 type; };
__device__ inline floatx4 widen(floatx4 x) { return x; }
__device__ inline floatx4 widen(bf16x4 x) { return __builtin_convertvector(x, floatx4); }
__device__ inline void store4(float* p, floatx4 x) { *(floatx4*)p = x; }
__device__ inline void store4(__bf16* p, floatx4 x) { *(bf16x4*)p = __builtin_convertvector(x, bf16x4); }

// Last sequence b with cu_nodes[b] <= node (0 if there is none).
__device__ inline int owner_of(const TiledArgs& a, int node) {
  int lo = 0, hi = a.batch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.cu_nodes[mid] <= node) lo = mid; else hi = mid;
  }
  return lo;
}

// Eight lanes per row; lane e of a row owns head dims 4 (e + 8 k) + 0 .. 3.  A row is a chain of memory round trips, so
// what does not depend on each other is requested together: the mask and the query while the plan is looked up, the
// next two tree keys while the last two are used, two partials at a time.  All lanes of a wavefront go through this
// together (rows that are not `active` have no keys and are not written).
template <typename T, int D>
struct Finish {
  static constexpr int K4 = D / 32;
  typedef typename Four<T>::type Raw;
  uint64_t mlo, mhi;
  Raw q[K4];
  floatx4 acc[K4];
  float m = -INFINITY, l = 0.f;

  __device__ void clear() {
#pragma unroll
    for (int k = 0; k < K4; ++k) acc[k] = (floatx4)(0.f);
  }
  __device__ void request(const TiledArgs& a, int node, int head, bool active, int e) {
    mlo = active ? a.anc_mask[2 * (size_t)node] : 0ull;
    mhi = active ? a.anc_mask[2 * (size_t)node + 1] : 0ull;
    const T* qp = (const T*)a.q + ((int64_t)node * a.Hq + head) * D;
#pragma unroll
    for (int k = 0; k < K4; ++k) q[k] = active ? *(const Raw*)(qp + 4 * (e + 8 * k)) : Raw();
    clear();
  }

  struct Keys {
    Raw k[2][K4], v[2][K4];
    bool have[2];
  };
  __device__ Keys next_keys(const T* kt, const T* vt, int64_t node_stride, int e) {
    Keys x;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      x.have[u] = (mlo | mhi) != 0ull;
      int j = 0;
      if (mlo) { j = __ffsll((unsigned long long)mlo) - 1; mlo &= mlo - 1; }
      else if (mhi) { j = 64 + __ffsll((unsigned long long)mhi) - 1; mhi &= mhi - 1; }
#pragma unroll
      for (int k = 0; k < K4; ++k) {
        x.k[u][k] = x.have[u] ? *(const Raw*)(kt + j * node_stride + 4 * (e + 8 * k)) : Raw();
        x.v[u][k] = x.have[u] ? *(const Raw*)(vt + j * node_stride + 4 * (e + 8 * k)) : Raw();
      }
    }
    return x;
  }
  // The tree part: the set bits of the row's ancestor mask, lowest first, of a tree of n nodes.
  __device__ void tree(const TiledArgs& a, int g, int base, int n, int e) {
    if (n < 64) mlo &= (1ull << n) - 1ull, mhi = 0ull;  // never index past the tree
    else if (n < 128) mhi &= (1ull << (n - 64)) - 1ull;
    const T* kt = (const T*)a.k_tree + ((int64_t)base * a.Hkv + g) * D;
    const T* vt = (const T*)a.v_tree + ((int64_t)base * a.Hkv + g) * D;
    const int64_t node_stride = (int64_t)a.Hkv * D;
    Keys cur = next_keys(kt, vt, node_stride, e);
    while (__any(cur.have[0])) {
      const Keys nxt = next_keys(kt, vt, node_stride, e);
      float dot[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        floatx4 d = widen(q[0]) * widen(cur.k[u][0]);
#pragma unroll
        for (int k = 1; k < K4; ++k) d += widen(q[k]) * widen(cur.k[u][k]);
        float x = (d[0] + d[1]) + (d[2] + d[3]);
        x += __shfl_xor(x, 1);
        x += __shfl_xor(x, 2);
        x += __shfl_xor(x, 4);
        dot[u] = cur.have[u] ? x : -INFINITY;
      }
      const float m_new = fmaxf(m, fmaxf(dot[0], dot[1]));
      const float al = weight(m, m_new, a.c);
      const float p0 = cur.have[0] ? weight(dot[0], m_new, a.c) : 0.f, p1 = cur.have[1] ? weight(dot[1], m_new, a.c) : 0.f;
      l = l * al + (p0 + p1);
      m = m_new;
#pragma unroll
      for (int k = 0; k < K4; ++k) acc[k] = acc[k] * al + (p0 * widen(cur.v[0][k]) + p1 * widen(cur.v[1][k]));
      cur = nxt;
    }
  }
  // One partial: its max, sum and the row's O, which lies in groups of four elements `stride` floats apart.
  struct Partial {
    float m, l;
    floatx4 o[K4];
  };
  __device__ static Partial fetch(float mc, float lc, const float* o, int stride, int e) {
    Partial p;
    p.m = mc;
    p.l = lc;
#pragma unroll
    for (int k = 0; k < K4; ++k) p.o[k] = *(const floatx4*)(o + (e + 8 * k) * stride);
    return p;
  }
  __device__ void merge(const Partial& p, float c) {
    const float m_new = fmaxf(m, p.m);
    const float al = weight(m, m_new, c), wt = weight(p.m, m_new, c);
    l = l * al + p.l * wt;
#pragma unroll
    for (int k = 0; k < K4; ++k) acc[k] = acc[k] * al + wt * p.o[k];
    m = m_new;
  }
  __device__ void write(const TiledArgs& a, int node, int head, int e) const {
    const int64_t row = (int64_t)node * a.Hq + head;
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int k = 0; k < K4; ++k) store4((T*)a.out + row * D + 4 * (e + 8 * k), acc[k] * inv);
    if (a.lse && e == 0) a.lse[row] = l > 0.f ? m * a.scale + logf(l) : -INFINITY;
  }
  // Whether one of the eight lanes of this row holds an infinity or NaN that does not come from NaN scores (those stay NaN
  // whichever way they are summed).  All lanes of the wavefront take part.
  __device__ bool row_overflowed(int lane) const {
    float x = 0.f;
#pragma unroll
    for (int k = 0; k < K4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) x = fmaf(acc[k][i], 0.f, x);
    return ((__ballot(x != 0.f) >> (lane & ~(kCombineLanes - 1))) & ((1u << kCombineLanes) - 1u)) != 0 && l < INFINITY;
  }
  // The whole row again, key by key: the prefix, then the tree part, in binary32 products with probabilities of at most 1.
  // For rows that are hardly ever seen, so it is small and not fast: 2 us a key (one sequence of 16384 tokens whose values
  // hold an infinity 33 ms, the general kernel 13.4).
  __device__ static void walk(const TiledArgs& a, int64_t row, bool active, int e) {
    asm volatile("" : "+v"(row));  // everything is derived anew, so that nothing lives in registers until here
    const int node = (int)(row / a.Hq), head = (int)(row % a.Hq), g = head / a.G;
    const int b = owner_of(a, node);
    const Shape sh = shape_of<T>(a, a.prefix_len[b], a.cu_nodes[b], a.cu_nodes[b + 1]);
    Finish f;
    f.request(a, node, head, active, e);
    const int len = active ? sh.len : 0;
    constexpr int kAtOnce = 2;  // keys whose loads are in flight together (the last one again past the end)
    for (int t0 = 0; __any(t0 < len); t0 += kAtOnce) {
      floatx4 k4[kAtOnce][K4], v4[kAtOnce][K4];
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const int t = max(0, min(t0 + u, len - 1)), block = t / a.block_size, slot = t - block * a.block_size;
        const int64_t page = clamp_block(a.block_table[(int64_t)b * a.max_blocks + block], a.num_blocks) * a.block_stride +
                             g * a.head_stride;
#pragma unroll
        for (int k = 0; k < K4; ++k) {
          const int d = 4 * (e + 8 * k);  // four head dims of K, and of V in plain pages, lie together
          const int64_t row_at = page + slot * a.token_stride + d;
          k4[u][k] = cached4(a, a.k_cache, a.plain ? row_at : page + ((d >> 3) * a.block_size + slot) * 8 + (d & 7), false);
          v4[u][k] = cached4(a, a.v_cache, a.plain ? row_at : page + ((slot >> 3) * D + d) * 8 + (slot & 7), !a.plain);
        }
      }
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) f.add_key(k4[u], v4[u], t0 + u < len, a.m_scale, a.o_scale, a.c);
    }
    const T* kt = (const T*)a.k_tree + ((int64_t)sh.base * a.Hkv + g) * D;
    const T* vt = (const T*)a.v_tree + ((int64_t)sh.base * a.Hkv + g) * D;
    for (int j = 0; __any(active && j < sh.n); ++j) {
      const bool have = active && j < sh.n && (((j < 64 ? f.mlo >> j : f.mhi >> (j - 64)) & 1ull) != 0);
      floatx4 k4[K4], v4[K4];
#pragma unroll
      for (int k = 0; k < K4; ++k)
        if (have) {
          const int64_t at = j * (int64_t)a.Hkv * D + 4 * (e + 8 * k);
          k4[k] = widen(*(const Raw*)(kt + at));
          v4[k] = widen(*(const Raw*)(vt + at));
        }
      f.add_key(k4, v4, have, 1.f, 1.f, a.c);
    }
    if (active) f.write(a, node, head, e);
  }
  // Four elements of the cache: together (and aligned as such, like all chunks of this path), or eight elements apart.
  __device__ static floatx4 cached4(const TiledArgs& a, const void* p, int64_t at, bool apart) {
    floatx4 r;
    if (a.fp8) {
      const uint8_t* x = (const uint8_t*)p + at;
      const uint32_t w = apart ? x[0] | x[8] << 8 | x[16] << 16 | (uint32_t)x[24] << 24 : *(const uint32_t*)x;
      r[0] = __builtin_amdgcn_cvt_f32_fp8(w, 0);
      r[1] = __builtin_amdgcn_cvt_f32_fp8(w, 1);
      r[2] = __builtin_amdgcn_cvt_f32_fp8(w, 2);
      r[3] = __builtin_amdgcn_cvt_f32_fp8(w, 3);
      return r;
    }
    const T* x = (const T*)p + at;
    if (!apart) return widen(*(const Raw*)x);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (float)x[8 * i];
    return r;
  }
  __device__ void add_key(const floatx4 (&k4)[K4], const floatx4 (&v4)[K4], bool have, float k_scale, float v_scale, float c) {
    float x = 0.f;
    if (have) {
#pragma unroll
      for (int k = 0; k < K4; ++k) {
        const floatx4 d = widen(q[k]) * k4[k];
        x += (d[0] + d[1]) + (d[2] + d[3]);
      }
    }
    x += __shfl_xor(x, 1);
    x += __shfl_xor(x, 2);
    x += __shfl_xor(x, 4);
    x *= k_scale;
    if (!have || x == -INFINITY) return;
    const float m_new = fmaxf(m, x), p = exp2f((x - m_new) * c), al = m_new == m ? 1.f : exp2f((m - m_new) * c);
    l = l * al + p;
    m = m_new;
#pragma unroll
    for (int k = 0; k < K4; ++k) acc[k] = acc[k] * al + p * (v_scale * v4[k]);
  }
};

// Rows of no sequence (offsets that leave the arrays, rows past the trees): defined output.
template <typename T, int D>
__device__ inline void zero_row(const TiledArgs& a, int64_t row, int e) {
#pragma unroll
  for (int k = 0; k < D / 32; ++k) store4((T*)a.out + row * D + 4 * (e + 8 * k), (floatx4)(0.f));
  if (a.lse && e == 0) a.lse[row] = -INFINITY;
}

// ---- the prefix kernel ----------------------------------------------------------------------------------------------------
template <typename T, bool kFp8, bool kPlain, int D, bool kDirect>
__global__ __launch_bounds__(kThreads, 2) void tva_tiled_kernel(TiledArgs a) {
  typedef Stager<T, kFp8, kPlain, D> Stage;
  constexpr int kStepKeys = step_keys<T>();
  constexpr int kRegion = region_floats(D);
  constexpr int kStageBytes = 2 * 2 * Stage::kStepChunks * 16, kFoldBytes = kWaves * kRegion * 4;
  __shared__ uintx4 lds[(kStageBytes > kFoldBytes ? kStageBytes : kFoldBytes) / 16];
  __shared__ float s_ml[2][kGroupRows];
  __shared__ Sums s_part[kWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workers (the row groups of a segment, the two ends of one) sit behind one L2
  const int64_t wg = gridDim.x % 8 == 0 ? (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8 : (int64_t)blockIdx.x;

  if (kDirect && a.status)
    for (int b = (int)(wg * kWaves + wv); b < a.batch; b += gridDim.x * kWaves)
      smart::tva_validate_block_table(b, a.block_table, a.prefix_len, a.max_blocks, a.block_size, a.num_blocks, a.status,
                                      lane);

  // Every wavefront plans for itself: what comes out is uniform over the workgroup.  Batches of more than 512 sequences are
  // summed by the eight wavefronts together (an eighth each) and searched in the eighth that holds what is looked for: a
  // chunk is a memory round trip, and this runs once per workgroup.  (Workspace-free form, 4096 sequences of 33 tokens, one
  // node, 8 kv heads of 128, bf16: 4378 us with every wavefront going through all of it, 2389 now; 1024 sequences 508 and
  // 354; split 904 and 841, 231 and 215.)
  Place at{-1, 0, 0};
  int64_t u0 = 0, u1 = 1;
  Sums all{};
  const int chunks = (a.batch + kWave - 1) / kWave;
  const bool divided = chunks > kWaves;
  auto first_chunk = [&](int w) { return (int)((int64_t)chunks * w / kWaves); };
  auto find = [&](int64_t want, bool by_segment) {
    Sums before{};
    int c0 = 0, c1 = chunks;
    for (int k = 0; divided && k < kWaves; ++k) {
      c0 = first_chunk(k);
      c1 = first_chunk(k + 1);
      if (want < (by_segment ? before.segs + s_part[k].segs : before.units + s_part[k].units)) break;
      before.units += s_part[k].units;
      before.segs += s_part[k].segs;
    }
    scan_batch<T>(a, lane, c0, c1, &before, [&](int b0, bool, int64_t units, int64_t segs, int64_t eu, int64_t es) {
      const int64_t first = by_segment ? es : eu, count = by_segment ? segs : units;
      const uint64_t hit = __ballot(want >= first && want < first + count);
      if (hit) {
        const int i = __ffsll((unsigned long long)hit) - 1;
        at.b = b0 + i;
        at.units_before = smart::readlane64(eu, i);
        at.segs_before = smart::readlane64(es, i);
      }
    });
    return before.flags;
  };
  auto keep_plan = [&](int b0, bool there, int64_t, int64_t, int64_t eu, int64_t es) {
    if (wg == 0 && (divided || wv == 0) && there) {
      a.plan[2 + b0 + lane] = eu;
      a.plan[2 + a.batch + b0 + lane] = es;
    }
  };
  if (divided) {
    Sums mine{};
    scan_batch<T>(a, lane, first_chunk(wv), first_chunk(wv + 1), &mine, [](int, bool, int64_t, int64_t, int64_t, int64_t) {});
    if (lane == 0) s_part[wv] = mine;
    __syncthreads();
    Sums before{};
    for (int k = 0; k < kWaves; ++k) {
      if (k == wv) before = all;
      all.units += s_part[k].units;
      all.segs += s_part[k].segs;
      all.steps += s_part[k].steps;
      all.flags |= s_part[k].flags;
    }
    if (!kDirect && wg == 0) scan_batch<T>(a, lane, first_chunk(wv), first_chunk(wv + 1), &before, keep_plan);
  } else if (!kDirect) {
    scan_batch<T>(a, lane, 0, chunks, &all, keep_plan);
  }
  if (kDirect) {
    const int flags = find(wg, true);
    if (!divided) all.flags = flags;
    if (all.flags & kDescending) at.b = -1;
  } else {
    const int64_t U = all.flags & kDescending ? -1 : all.units;
    const int64_t W = U <= 0 ? 0 : (all.steps < (int64_t)gridDim.x ? all.steps : (int64_t)gridDim.x);
    if (wg == 0 && tid == 0) {
      a.plan[0] = U;
      a.plan[1] = W;
    }
    if (wg >= W) return;
    u0 = (wg * U) / W;
    u1 = ((wg + 1) * U) / W;
    find(u0, false);
  }

  if (at.b >= 0) {
    int b = at.b;
    Shape sh = shape_of<T>(a, a.prefix_len[b], a.cu_nodes[b], a.cu_nodes[b + 1]);
    while (u0 < u1) {
      // on to the next sequence with units
      while (!kDirect && u0 >= at.units_before + a.Hkv * sh.head) {
        at.units_before += a.Hkv * sh.head;
        at.segs_before += (int64_t)a.Hkv * sh.groups;
        ++b;
        if (b >= a.batch) return;
        sh = shape_of<T>(a, a.prefix_len[b], a.cu_nodes[b], a.cu_nodes[b + 1]);
      }
      int g, group, t0, t1;
      if (kDirect) {
        const int local = (int)(wg - at.segs_before);
        g = local / sh.groups;
        group = local % sh.groups;
        t0 = 0;
        t1 = sh.steps;
      } else {
        // (a share boundary inside a step goes down to the step's beginning)
        const int64_t local = u0 - at.units_before;
        g = (int)(local / sh.head);
        const int64_t in_head = local - g * sh.head;
        group = (int)min(in_head / sh.full, (int64_t)sh.groups - 1);
        const int64_t off = in_head - group * sh.full;
        const int cost = group < sh.groups - 1 ? StepCost<T>::four : sh.cost_last;
        const int64_t left = (int64_t)sh.steps * cost - off;  // units to the end of the segment's steps
        const int64_t share = u1 - u0;
        u0 = min(u1, u0 + left + a.segment_cost);
        if (left <= 0) continue;  // (the finishing step does not count this worker)
        t0 = (int)(off / cost);
        t1 = share >= left ? sh.steps : (int)((off + share) / cost);
        // (a share that ends inside the segment's first step has none of its steps and is not counted either: to begin and fold
        // a piece takes 4 .. 5 us also where it is empty.  2 sequences of 35 and 47 nodes, 119 and 115 tokens, 32 / 8 heads of
        // 128, plain bf16 34.1 -> 30.2 us)
        if (t1 == 0) continue;
      }
      b = __builtin_amdgcn_readfirstlane(b);
      g = __builtin_amdgcn_readfirstlane(g);
      group = __builtin_amdgcn_readfirstlane(group);
      t0 = __builtin_amdgcn_readfirstlane(t0);
      t1 = __builtin_amdgcn_readfirstlane(t1);
      const int len = __builtin_amdgcn_readfirstlane(sh.len), rows = __builtin_amdgcn_readfirstlane(sh.rows);
      const int row0 = group * kGroupRows;
      const int group_rows = min(kGroupRows, rows - row0);
      const int r = (group_rows + kRowTile - 1) / kRowTile;
      // row tile, first tile of a step and stride between tiles of this wavefront; wavefronts rt, rt + apart, ... share one
      const int apart = r >= 3 ? 4 : r;
      const int shared = r >= 3 ? 2 : 4;  // wavefronts per row tile
      const int rt = wv & (apart - 1), first = r == 1 ? wv : (r == 2 ? wv >> 1 : wv >> 2);
      const bool busy = rt < r && first < kTilesPerStep;

      Rows<T, kPlain, D> rowset;
      rowset.begin(a, sh.base, g, row0 + (busy ? rt * kRowTile : 0), rows, lane);
      const int32_t* table = a.block_table + (int64_t)b * a.max_blocks;
      Stage st;
      if (t0 < t1) {
        st.load_ids(a, table, t0, len, tid);
        st.load(a, t0, len, g, tid);
        if (t0 + 1 < t1) st.load_ids(a, table, t0 + 1, len, tid);
      }
      __syncthreads();  // the piece before is done with the LDS
      for (int t = t0; t < t1; ++t) {
        uintx4* stage = lds + (t & 1) * (2 * Stage::kStepChunks);
        st.store(stage, tid, len - t * kStepKeys);
        if (t + 1 < t1) {
          st.load(a, t + 1, len, g, tid);
          if (t + 2 < t1) st.load_ids(a, table, t + 2, len, tid);
        }
        __syncthreads();  // the stage is full, and everyone is done with the other one
        if (busy)
          for (int x = first; x < kTilesPerStep; x += shared) {
            const int n_valid = len - t * kStepKeys - x * Stage::kKeys;
            if (n_valid <= 0) break;
            rowset.template tile<!kFp8>(stage + x * Stage::kTileChunks, stage + Stage::kStepChunks + x * Stage::kTileChunks, n_valid,
                                        a.c_stored, lane);
          }
      }
      // fold: the states that share a row tile, in wavefront order
      __syncthreads();
      float* regions = (float*)lds;
      rowset.put(regions + wv * kRegion, lane);
      __syncthreads();
      float* slot = kDirect ? nullptr : a.ws + (wg + at.segs_before + (int64_t)g * sh.groups + group) * slot_floats(D);
      if (tid < r * kRowTile) {
        const float* ml = regions + (tid >> 5) * kRegion + kRowTile * D + (tid & 31);
        float m = ml[0], l = ml[kRowTile];
        for (int k = 1; k < shared; ++k) {
          const float mk = ml[k * apart * kRegion], lk = ml[k * apart * kRegion + kRowTile];
          const float m_new = fmaxf(m, mk);
          l = l * weight(m, m_new, a.c_stored) + lk * weight(mk, m_new, a.c_stored);
          m = m_new;
        }
        s_ml[0][tid] = m;
        s_ml[1][tid] = l;
        if (slot) {
          slot[kGroupRows * D + tid] = m * a.m_scale;  // (-inf stays -inf)
          slot[kGroupRows * D + kGroupRows + tid] = l;
        }
      }
      __syncthreads();
      for (int i = tid; i < r * (D / 4) * kRowTile; i += kThreads) {
        const int tile = i / (D / 4 * kRowTile), x = i % (D / 4 * kRowTile), row = x % kRowTile;
        float* src = regions + tile * kRegion;
        floatx4 o = ((const floatx4*)src)[x];
        const float m = s_ml[0][tile * kRowTile + row];
        o *= weight(src[kRowTile * D + row], m, a.c_stored);
        for (int k = 1; k < shared; ++k)
          o += ((const floatx4*)(src + k * apart * kRegion))[x] * weight(src[k * apart * kRegion + kRowTile * D + row], m, a.c_stored);
        o *= a.o_scale;
        if (slot) ((floatx4*)slot)[(x / kRowTile) * kGroupRows + tile * kRowTile + row] = o;
        else ((floatx4*)src)[x] = o;  // (only this thread reads what it overwrites)
      }
      if (kDirect) {
        __syncthreads();
        const int e = tid & (kCombineLanes - 1);
        for (int i0 = 0; i0 < group_rows; i0 += kThreads / kCombineLanes) {
          const int i = i0 + tid / kCombineLanes;
          const bool active = i < group_rows;
          const int rho = row0 + (active ? i : 0);
          const int node = sh.base + rho / a.G, head = g * a.G + rho % a.G;
          Finish<T, D> f;
          f.request(a, node, head, active, e);
          f.tree(a, g, sh.base, sh.n, e);
          if (active && t0 < t1)
            f.merge(f.fetch(s_ml[0][i] * a.m_scale, s_ml[1][i], regions + (i >> 5) * kRegion + (i & 31) * 4, kRowTile * 4, e),
                    a.c);
          if (active) f.write(a, node, head, e);
          const bool again = f.row_overflowed(lane) && active;
          if (__any(again)) f.walk(a, (int64_t)node * a.Hq + head, again, e);
        }
        break;
      }
    }
  }

  // rows nobody owns (regular offsets: only before the first and behind the last); all rows of a call without segments
  if (kDirect) {
    const int first_node = a.cu_nodes[0], end_node = a.cu_nodes[a.batch];
    const bool ascending = (all.flags & kDescending) == 0;
    for (int64_t node = wg; node < a.total_nodes; node += gridDim.x) {
      if (all.flags == 0 && node >= first_node && node < end_node) continue;
      const int b = owner_of(a, (int)node);
      const Shape sh = shape_of<T>(a, a.prefix_len[b], a.cu_nodes[b], a.cu_nodes[b + 1]);
      const bool owned = node >= sh.base && node - sh.base < sh.n;
      if (owned && ascending) continue;
      const int e = tid & (kCombineLanes - 1);
      for (int h0 = 0; h0 < a.Hq; h0 += kThreads / kCombineLanes) {
        const int h = h0 + tid / kCombineLanes;
        if (owned) Finish<T, D>::walk(a, node * a.Hq + min(h, a.Hq - 1), h < a.Hq, e);
        else if (h < a.Hq) zero_row<T, D>(a, node * a.Hq + h, e);
      }
    }
  }
}

// ---- split form: merging the partials, with the tree part ----------------------------------------------------------
// A row is two chains of memory round trips, the tree part (mask, keys two at a time) and the partials (plan, then two at a
// time).  kParts > 0: a workgroup per eight (node, head) rows, one wavefront for the tree part and kParts that share the
// partials, merged by the first in a fixed order; for launches that leave wavefront slots idle (see finish_parts).
// kParts = 0: a wavefront per eight rows goes through both.
constexpr int finish_waves(int parts) { return parts > 0 ? 1 + parts : 4; }
template <typename T, int D, int kParts>
__global__ __launch_bounds__(finish_waves(kParts) * kWave, kParts == 0 ? 2 : 1) void tva_tiled_finish_kernel(TiledArgs a) {
  constexpr int kRows = kWave / kCombineLanes, K4 = D / 32;
  constexpr int kStates = kParts > 0 ? kParts : 1;
  __shared__ floatx4 s_acc[kStates][K4][kWave];
  __shared__ float s_m[kStates][kRows], s_l[kStates][kRows];
  const int lane = threadIdx.x & (kWave - 1), e = lane & (kCombineLanes - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int part = kParts > 0 ? wv - 1 : -1;  // -1: the tree part
  const int64_t wave = (int64_t)blockIdx.x * finish_waves(kParts) + wv;
  if (a.status)
    for (int64_t b = wave; b < a.batch; b += (int64_t)gridDim.x * finish_waves(kParts))
      smart::tva_validate_block_table((int)b, a.block_table, a.prefix_len, a.max_blocks, a.block_size, a.num_blocks,
                                      a.status, lane);
  const int64_t n_rows = (int64_t)a.total_nodes * a.Hq, first = (kParts > 0 ? (int64_t)blockIdx.x : wave) * kRows;
  if (first >= n_rows) return;
  const int64_t row_raw = first + lane / kCombineLanes;
  const bool there = row_raw < n_rows;
  const int64_t row = there ? row_raw : n_rows - 1;
  const int node = (int)(row / a.Hq), head = (int)(row % a.Hq), g = head / a.G;
  Finish<T, D> f;
  if (part < 0) f.request(a, node, head, there, e);
  else f.clear();
  const int64_t U = a.plan[0], W = a.plan[1];
  int b;
  if (a.batch <= kWave) {
    // the offsets of the whole batch, one per lane; the wavefront's rows lie in a few consecutive nodes
    const int cu = a.cu_nodes[min(lane, a.batch - 1)];
    b = 0;
    const int n0 = __builtin_amdgcn_readfirstlane(node), n1 = __builtin_amdgcn_readlane(node, kWave - 1);
    for (int x = n0; x <= n1; ++x) {
      const uint64_t below = __ballot(lane < a.batch && cu <= x);
      if (node == x && below) b = 63 - __clzll((unsigned long long)below);
    }
  } else {
    b = owner_of(a, node);
  }
  if (U < 0) b = owner_of(a, node);  // offsets that are not ascending
  const Shape sh = shape_of<T>(a, a.prefix_len[b], a.cu_nodes[b], a.cu_nodes[b + 1]);
  const bool owned = there && node >= sh.base && (int64_t)node - sh.base < sh.n;
  const int64_t units_before = a.plan[2 + b], segs_before = a.plan[2 + a.batch + b];
  if (part < 0) f.tree(a, g, sh.base, owned ? sh.n : 0, e);
  if ((kParts == 0 || part >= 0) && owned && sh.steps > 0 && U > 0) {
    const int rho = (node - sh.base) * a.G + head % a.G;
    const int group = rho / kGroupRows, r = rho % kGroupRows, local = g * sh.groups + group;
    // (a step belongs to the worker that holds its last unit)
    const int64_t ub = units_before + g * sh.head + group * sh.full;
    const int cost = group < sh.groups - 1 ? StepCost<T>::four : sh.cost_last;
    const int64_t w_first = ((ub + cost) * W - 1) / U, w_last = ((ub + (int64_t)sh.steps * cost) * W - 1) / U;
    auto partial = [&](int64_t w) {
      const float* slot = a.ws + (w + segs_before + local) * slot_floats(D);
      return f.fetch(slot[kGroupRows * D + r], slot[kGroupRows * D + kGroupRows + r], slot + r * 4, kGroupRows * 4, e);
    };
    for (int64_t w = w_first + (kParts > 0 ? part : 0); w <= w_last; w += 2 * kStates) {
      const auto p0 = partial(w);
      auto p1 = partial(min(w + kStates, w_last));  // (no branch around it: both are requested before the first is used)
      if (w + kStates > w_last) p1.m = -INFINITY;
      f.merge(p0, a.c);
      f.merge(p1, a.c);
    }
  }
  if (kParts > 0) {
    if (part >= 0) {
#pragma unroll
      for (int k = 0; k < K4; ++k) s_acc[part][k][lane] = f.acc[k];
      if (e == 0) {
        s_m[part][lane / kCombineLanes] = f.m;
        s_l[part][lane / kCombineLanes] = f.l;
      }
    }
    __syncthreads();
    if (part >= 0) return;
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      typename Finish<T, D>::Partial x;
      x.m = s_m[p][lane / kCombineLanes];
      x.l = s_l[p][lane / kCombineLanes];
#pragma unroll
      for (int k = 0; k < K4; ++k) x.o[k] = s_acc[p][k][lane];
      f.merge(x, a.c);
    }
  }
  if (owned) f.write(a, node, head, e);
  const bool again = (f.row_overflowed(lane) || U < 0) && owned;
  if (__any(again)) f.walk(a, (int64_t)node * a.Hq + head, again, e);
  if (there && !owned) zero_row<T, D>(a, row, e);
}

}  // namespace

namespace smart {

// Workers of the split form: one workgroup per compute unit.
static int32_t tiled_workgroups(const smart_ctx* ctx) {
  if (ctx->opt_workers > 0) return (int32_t)ctx->opt_workers;
  return ctx->num_cus > 0 ? ctx->num_cus : 256;
}

static int64_t tiled_segments(int32_t batch, int32_t total_nodes, int32_t num_q_heads, int32_t num_kv_heads) {
  const int64_t G = num_q_heads / num_kv_heads;
  return (int64_t)num_kv_heads * (((int64_t)total_nodes * G + kGroupRows - 1) / kGroupRows + batch);
}

static size_t partials_bytes(const smart_ctx* ctx, int64_t segs, int32_t head_dim) {
  return ((size_t)(tiled_workgroups(ctx) + segs + 1) * slot_floats(head_dim) * sizeof(float) + 255) & ~(size_t)255;
}
static size_t plan_bytes(int32_t batch) { return sizeof(int64_t) * (2 + 2 * (size_t)batch); }

// (no smaller head counts have more segments: Hkv ceil(N G / 128) < N Hq / 128 + Hkv)
size_t tva_tiled_reserve(const smart_ctx* ctx, int32_t batch, int32_t total_nodes, int32_t num_q_heads,
                         int32_t num_kv_heads) {
  const int64_t segs = ((int64_t)total_nodes * num_q_heads + kGroupRows - 1) / kGroupRows + (int64_t)num_kv_heads * (batch + 1);
  return partials_bytes(ctx, segs, 128) + plan_bytes(batch);
}

// Every 16-byte chunk of a staged row, every query row and every tree row must be addressable with one load.
bool tva_tiled_supported(const tva_params& p) {
  const bool fp8 = p.kv_cache_dtype == SMART_FP8_E4M3;
  const int chunk = p.dtype == SMART_F32 ? 4 : 8;                            // elements
  const uintptr_t cache_align = fp8 ? (uintptr_t)chunk : 16;                 // bytes
  auto aligned = [](const void* x, uintptr_t n) { return ((uintptr_t)x & (n - 1)) == 0; };
  if (p.max_blocks_per_seq <= 0 || p.num_blocks <= 0) return false;
  if (p.cache_block_stride % chunk || p.cache_head_stride % chunk) return false;
  if (p.kv_layout == SMART_KV_PLAIN && p.cache_token_stride % chunk) return false;
  return aligned(p.d_k_cache, cache_align) && aligned(p.d_v_cache, cache_align) && aligned(p.d_q, 16) &&
         aligned(p.d_k_tree, 16) && aligned(p.d_v_tree, 16) && aligned(p.d_out, 16);
}

// A piece takes 3 us to start and 4 to fold, which a worker that holds the ends of two segments pays twice: counted like two
// steps of one row tile (bf16), it leaves such a worker fewer steps.  Without / with, us: the bf16 workload above 95 / 84.6,
// 16 sequences of 60 .. 500 tokens, 4 .. 64 nodes 45.6 / 37.3, of 100 .. 800, 30 .. 66 nodes, 64 / 8 heads of 64 65.8 / 49.4,
// fp32, 10 of 200 .. 1600 41.3 / 36.0; 4 and 12 in its place 86.6 and 84.9, 37.8 and 36.9, 52.5 and 50.3, 37.3 and 38.2.
// Few segments are cut into many pieces of a step or two each, and where they are equally long the cuts fall on whole steps
// without it: 4 sequences of 1000, 8 kv heads 30.4 / 33.3, 16 of 2000, 2 kv heads 33.1 / 36.2, but 5 of 1000, 8 kv heads
// 38.6 / 33.6.
static int32_t segment_cost(const tva_params& p, int32_t workgroups) {
  return (int64_t)p.batch * p.num_kv_heads * 8 > workgroups ? 8 : 0;
}

// `rows8`: groups of eight rows.  Whole calls, one wavefront for both chains / a second for the partials / seven for them:
// 28 groups, one sequence of 4000 tokens, plain bf16 36.1 / 26.4 / 22.7 us; 120 groups, the fp32 workload above (up to 24
// partials a row) 23.1 / 20.8 / 19.0; 480 groups, 4 sequences of 1000 33.7 / 30.4 / 36.2; 576 37.1 / 34.2; from there on either way
// (720 53.5 / 51.0, 756 27.0 / 28.3, 832 44.0 / 42.5); 1500, 16 sequences of 60 .. 128 nodes, 31.9 / 34.6 / 42.7; 2016 42.2 /
// 47.7 / 70.6; the bf16 workload above (2176) 95.2 / 97.1 / 117.6.
static int finish_parts(int64_t rows8) { return rows8 <= 128 ? 7 : (rows8 <= 640 ? 1 : 0); }
template <typename T, int D>
static void launch_finish(const TiledArgs& a, int64_t rows8, hipStream_t stream) {
  const int parts = finish_parts(rows8), waves = finish_waves(parts);
  const dim3 grid((unsigned)(parts > 0 ? rows8 : (rows8 + waves - 1) / waves)), block(waves * kWave);
  if (parts == 7) hipLaunchKernelGGL((tva_tiled_finish_kernel<T, D, 7>), grid, block, 0, stream, a);
  else if (parts == 1) hipLaunchKernelGGL((tva_tiled_finish_kernel<T, D, 1>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((tva_tiled_finish_kernel<T, D, 0>), grid, block, 0, stream, a);
}

template <typename T, bool kFp8, bool kPlain, int D>
static hipError_t launch_tiled(const TiledArgs& a, bool direct, unsigned grid, hipStream_t stream) {
  if (direct)
    hipLaunchKernelGGL((tva_tiled_kernel<T, kFp8, kPlain, D, true>), dim3(grid), dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((tva_tiled_kernel<T, kFp8, kPlain, D, false>), dim3(grid), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

int32_t tva_launch_tiled(smart_ctx* ctx, hipStream_t stream, const tva_params& p, const TvaWorkspace* fixed) {
  const int G = p.num_q_heads / p.num_kv_heads;
  const bool fp8 = p.kv_cache_dtype == SMART_FP8_E4M3, f32 = p.dtype == SMART_F32;
  const int64_t segs = tiled_segments(p.batch, p.total_nodes, p.num_q_heads, p.num_kv_heads);
  const int64_t rows8 = ((int64_t)p.total_nodes * p.num_q_heads + kWave / kCombineLanes - 1) / (kWave / kCombineLanes);
  if (segs > 0x7FFFFFFF) return SMART_EINVAL;
  // The workspace-free form: for callers that cannot allocate, for launches that are being captured (a graph must not
  // hold a workspace that a later, larger call replaces), and when no memory is left.  It is also the faster one, by the
  // second launch, where a segment is a few steps, its rows fit one pass of the finishing step (64) and every segment has
  // a compute unit: 15-node trees of 60 rows, batch 8, bf16 20.9 us against 15.8 at 33 tokens, 27.7 against 24.8 at 513,
  // 29.9 against 33.8 at 1025; fp32 (a step is half as long and takes twice as long) 18.1 against 15.2 at 33 tokens,
  // 19.0 against 19.4 at 129; batch 32, 376 segments, 27.2 against 30.7.  Larger trees too where a segment is a single step
  // (the tree part of a deep tree takes most of the time then, and here all rows of a workgroup read the same tree): 33
  // tokens, one sequence of 48 nodes, 32 / 8 heads of 128, bf16 28.7 us against 21.3 (general kernel 36.7), 8 / 2 of 64, fp32
  // 24.8 against 17.7 (22.1), 66 nodes 22.8 against 18.2 (25.6), up to a mean of 384 rows (64 / 8 heads, 48 nodes, 19.1 against
  // 17.9); 512 rows 18.7 against 19.9.
  // Where it runs for its other reasons it can leave compute units idle: 8 kv heads, 4 heads each, one bf16 sequence of
  // 16384 tokens, one node, 200 us (128 steps in a row on 8 of them; split 39, general kernel 13340), 64 nodes 454 (64,
  // 18089); four such sequences 204 .. 465; fp32, 2 x 4 heads of 64, 397 .. 1218 (46 .. 54, 8165 .. 8500).
  // Lengths are on the device, so a wide table with hardly anything in it runs split: 4096 tokens wide, prefixes of one
  // token, 16-node trees, 14.7 .. 15.5 us in fp32 where the general kernel takes 12.8 .. 13.8; from 8 tokens on it is behind.
  const int64_t longest = (int64_t)p.max_blocks_per_seq * p.block_size;
  const int64_t step = f32 ? step_keys<float>() : step_keys<__bf16>(), rows = (int64_t)p.total_nodes * G;
  const bool few_steps = (longest <= step && rows <= 384 * (int64_t)p.batch) ||
                         (!f32 && longest <= 4 * step && rows <= 64 * (int64_t)p.batch);
  bool direct = fixed != nullptr || (few_steps && segs <= (ctx->num_cus > 0 ? ctx->num_cus : 256));
  if (!direct) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (stream != nullptr && hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();
    direct = capture != hipStreamCaptureStatusNone;
  }
  void* ws = nullptr;
  const size_t partials = partials_bytes(ctx, segs, p.head_dim);  // then the plan
  if (!direct) {
    const int32_t rc = tiled_workspace(ctx, stream, partials + plan_bytes(p.batch), &ws);
    if (rc == SMART_EHIP) return rc;
    direct = rc != SMART_OK;
  }
  TiledArgs a;
  a.q = p.d_q;
  a.k_tree = p.d_k_tree;
  a.v_tree = p.d_v_tree;
  a.k_cache = p.d_k_cache;
  a.v_cache = p.d_v_cache;
  a.block_table = p.d_block_table;
  a.prefix_len = p.d_prefix_len;
  a.cu_nodes = p.d_cu_nodes;
  a.anc_mask = p.d_anc_mask;
  a.out = p.d_out;
  a.lse = p.d_lse;
  a.status = p.d_status;
  a.ws = direct ? nullptr : (float*)ws;
  a.plan = direct ? nullptr : (int64_t*)((char*)ws + partials);
  a.block_stride = p.cache_block_stride;
  a.head_stride = p.cache_head_stride;
  a.token_stride = p.cache_token_stride;
  a.batch = p.batch;
  a.total_nodes = p.total_nodes;
  a.Hq = p.num_q_heads;
  a.Hkv = p.num_kv_heads;
  a.G = G;
  a.block_size = p.block_size;
  a.max_blocks = p.max_blocks_per_seq;
  a.num_blocks = p.num_blocks;
  a.segment_cost = segment_cost(p, tiled_workgroups(ctx));
  a.fp8 = fp8;
  a.plain = p.kv_layout == SMART_KV_PLAIN;
  // t8 / d as the high word of 2 t8 * (floor(2^31 / d) + 1): exact for t8 < 2^28 and d <= 8
  a.block8_magic = (uint32_t)((1ull << 31) / ((uint32_t)p.block_size / 8)) + 1u;
  a.scale = p.softmax_scale;
  a.c = p.softmax_scale * kLog2e;
  a.c_stored = a.c * (fp8 ? p.k_scale : 1.f);
  a.m_scale = fp8 ? p.k_scale : 1.f;
  a.o_scale = fp8 ? p.v_scale : 1.f;

  int32_t rc = profile_begin(ctx, stream);
  if (rc != SMART_OK) return rc;
  const unsigned grid = direct ? (unsigned)segs : (unsigned)tiled_workgroups(ctx);
  const bool plain = a.plain;
  hipError_t err = hipErrorInvalidValue;
#define SMART_TILED(T, FP8, PLAIN) \
  err = p.head_dim == 128 ? launch_tiled<T, FP8, PLAIN, 128>(a, direct, grid, stream) : launch_tiled<T, FP8, PLAIN, 64>(a, direct, grid, stream)
  if (f32) {
    if (fp8) { if (plain) SMART_TILED(float, true, true); else SMART_TILED(float, true, false); }
    else { if (plain) SMART_TILED(float, false, true); else SMART_TILED(float, false, false); }
  } else {
    if (fp8) { if (plain) SMART_TILED(__bf16, true, true); else SMART_TILED(__bf16, true, false); }
    else { if (plain) SMART_TILED(__bf16, false, true); else SMART_TILED(__bf16, false, false); }
  }
#undef SMART_TILED
  SMART_HIP_CHECK(err);
  rc = profile_end(ctx, stream);
  if (rc != SMART_OK || direct) return rc;
  if (f32) {
    if (p.head_dim == 128) launch_finish<float, 128>(a, rows8, stream);
    else launch_finish<float, 64>(a, rows8, stream);
  } else {
    if (p.head_dim == 128) launch_finish<__bf16, 128>(a, rows8, stream);
    else launch_finish<__bf16, 64>(a, rows8, stream);
  }
  SMART_HIP_CHECK(hipGetLastError());
  return SMART_OK;
}

}  // namespace smart
