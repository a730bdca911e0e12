// tree_accept_sample: temperature-1 (sampling) verification of a draft tree whose nodes'
// children are deterministic proposals (the draft model's top-k tokens).
//
// The paper evaluates at temperatures 0 and 1 and relies on verification being lossless (Sec. 4,
// evaluation paragraph).  For deterministic proposals the lossless rule is: at the current node,
// with target distribution p, visit the children in node order; a child proposing token x is
// accepted with probability p(x) / (mass not yet rejected at this node); a rejected token's
// mass is removed; when no child is accepted the bonus token is drawn from what is left of p.
// The emitted token is then distributed exactly as p.
//
// Every decision is taken on integers so that it cannot depend on a summation order:
// w(x) = floor(p(x) 2^32), a 64-bit draw r, remaining weight R; mulhi(r, R) is uniform on
// [0, R); accept iff mulhi(r, R) < w(x); the bonus token is the first index whose running weight
// sum exceeds mulhi(r, R).  Draws are Philox-4x32-10 (Salmon et al., SC 2011) with counter
// (draw index, step low, step high, sequence) and key (seed low, seed high).
//
// Two launches.  A single compute unit pulls only a few tens of GB/s by itself, so the rows of
// the target distribution are not streamed by the workgroup that walks a sequence: first
// every row of the batch is summed by many small workgroups at once (64 contiguous ranges per
// row, the weight sum of each kept in the context's workspace: 512 bytes a row); then one
// wavefront per sequence walks its tree.  The walk is a chain of memory round trips, so what it may need is
// requested before it is known to be needed: the weight of every node's token in its parent's row, and the range
// sums of the first nodes' rows (one range per lane).  The bonus token is found by a lane scan over the range sums
// followed by a rescan of the single range (1/64 of a row) that holds the target weight.
// Batch 32, trees of 4 .. 7 nodes, 32000 tokens (24 MB): row sums 10.8 -> 6.5 us, walk 17.4 -> 6.8 us.
#include "common.h"

namespace {

constexpr int kWave = 64;
constexpr int kRanges = 64;  // ranges a row is cut into: one per lane of the walking wavefront

// floor(p 2^32): p 2^32 is exact in binary32 (an exponent shift), so below 1 the conversion's truncation is the floor
// and the result fits 32 bits.  NaN, zero and negatives count 0, values from 1 on 2^32.
__device__ inline uint64_t weight_of(float p) {
  const bool one = p >= 1.f;
  const float x = p > 0.f && !one ? p * 4294967296.f : 0.f;
  return (uint64_t)(uint32_t)x + ((uint64_t)(one ? 1u : 0u) << 32);
}

__device__ inline void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

__device__ inline uint64_t rand64(uint64_t seed, uint64_t step, uint32_t seq, uint32_t draw) {
  uint32_t c[4] = {draw, (uint32_t)step, (uint32_t)(step >> 32), seq};
  philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
  return (uint64_t)c[0] | ((uint64_t)c[1] << 32);
}

__device__ inline uint64_t wave_sum(uint64_t v) {
  for (int sh = 32; sh >= 1; sh >>= 1) v += __shfl_xor(v, sh);
  return v;
}

__device__ inline uint64_t wave_incl_scan(uint64_t v, int lane) {
  for (int sh = 1; sh < kWave; sh <<= 1) {
    const uint64_t up = __shfl_up(v, sh);
    if (lane >= sh) v += up;
  }
  return v;
}

// Tokens per range: a 64th of the vocabulary, rounded up to whole 16-byte vectors.
__host__ __device__ inline int range_of(int V) { return ((V + kRanges - 1) / kRanges + 3) / 4 * 4; }

// Weight sums of the 64 ranges of every row.  A wavefront takes kPer consecutive ranges, two vectors per lane and range
// in flight at once; workgroup (row, y): four wavefronts.
template <int kPer>
__global__ __launch_bounds__(4 * kWave) void range_sums_kernel(int total_nodes, int V, int64_t stride,
                                                               const float* __restrict__ prob,
                                                               uint64_t* __restrict__ sums) {
  const int node = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  if (node >= total_nodes) return;
  const int range = range_of(V);
  const bool vec = (stride % 4 == 0) && (((uintptr_t)prob & 15u) == 0);
  const float* row = prob + (size_t)node * stride;
  const int first = (blockIdx.y * 4 + wv) * kPer;
  uint64_t acc[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) acc[r] = 0;
  if (vec) {
    constexpr int kInFlight = kPer >= 4 ? 2 : 8;
    for (int v0 = 4 * lane; v0 < range; v0 += 4 * kWave * kInFlight) {
      float4 x[kPer][kInFlight];
#pragma unroll
      for (int r = 0; r < kPer; ++r)
#pragma unroll
        for (int i = 0; i < kInFlight; ++i) {
          const int in_range = v0 + i * 4 * kWave, v = (first + r) * range + in_range;
          x[r][i] = in_range < range && v + 3 < V ? *reinterpret_cast<const float4*>(row + v) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
      for (int r = 0; r < kPer; ++r)
#pragma unroll
        for (int i = 0; i < kInFlight; ++i) {
          const int in_range = v0 + i * 4 * kWave, v = (first + r) * range + in_range;
          acc[r] += (weight_of(x[r][i].x) + weight_of(x[r][i].y)) + (weight_of(x[r][i].z) + weight_of(x[r][i].w));
          if (in_range < range && v < V && v + 3 >= V)  // the ragged end of the vocabulary
            for (int e = 0; v + e < V; ++e) acc[r] += weight_of(row[v + e]);
        }
    }
  } else {
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int v_begin = (first + r) * range, v_end = v_begin + range < V ? v_begin + range : V;
#pragma unroll 8
      for (int v = v_begin + lane; v < v_end; v += kWave) acc[r] += weight_of(row[v]);
    }
  }
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    acc[r] = wave_sum(acc[r]);
    if (lane == 0) sums[(size_t)node * kRanges + first + r] = acc[r];
  }
}

__device__ inline uint64_t readlane64(uint64_t v, int lane) {  // lane is wave-uniform
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// The token of a range at which the running weight sum (rejected tokens left out) exceeds T, which lies below the range's
// sum.  The range is gone through in pieces of 64 x kRun tokens: a lane takes kRun consecutive tokens (all of its loads in
// flight at once) and sums them, a lane scan finds the lane whose run holds the target, and that lane goes through its
// run once more, out of registers.  `rejected(i)`: the i-th rejected token.
template <int kRun, typename Rejected>
__device__ inline int find_in_range(const float* row, int v_begin, int v_end, uint64_t T, int nrej, Rejected rejected, int lane) {
  for (int vb = v_begin; vb < v_end; vb += kWave * kRun) {
    const int my_begin = vb + lane * kRun;
    float x[kRun];
#pragma unroll
    for (int k = 0; k < kRun; ++k) x[k] = my_begin + k < v_end ? row[my_begin + k] : 0.f;
    for (int i = 0; i < nrej; ++i) {
      const int gone = rejected(i) - my_begin;
#pragma unroll
      for (int k = 0; k < kRun; ++k) x[k] = gone == k ? 0.f : x[k];
    }
    uint64_t w[kRun], run_sum = 0;
#pragma unroll
    for (int k = 0; k < kRun; ++k) {
      w[k] = weight_of(x[k]);
      run_sum += w[k];
    }
    const uint64_t run_incl = wave_incl_scan(run_sum, lane);
    const uint64_t piece = readlane64(run_incl, kWave - 1);
    if (piece <= T) {  // the target lies further on
      T -= piece;
      continue;
    }
    const int owner = __ffsll((unsigned long long)__ballot(run_incl > T)) - 1;
    const uint64_t t_run = T - readlane64(run_incl - run_sum, owner);
    uint64_t acc = 0;
    int before = 0;  // tokens of the run the target lies behind (only the owner's is meaningful)
#pragma unroll
    for (int k = 0; k < kRun; ++k) {
      acc += w[k];
      before += acc <= t_run ? 1 : 0;
    }
    return __builtin_amdgcn_readlane(my_begin + before, owner);
  }
  return -1;
}

// The walk: one wavefront per sequence, lane l owns range l of the current row.
constexpr int kRowsAhead = 8;  // nodes whose range sums are fetched before the walk
__global__ __launch_bounds__(kWave) void tree_accept_sample_kernel(
    int batch, int total_nodes, int max_depth, int V, int64_t stride, const int32_t* __restrict__ cu_nodes,
    const int32_t* __restrict__ parent, const int32_t* __restrict__ token, const float* __restrict__ prob,
    const uint64_t* __restrict__ sums, uint64_t seed, uint64_t step, int32_t* __restrict__ accept_len,
    int32_t* __restrict__ accept_path, int32_t* __restrict__ bonus_token) {
  __shared__ int32_t sRej[SMART_MAX_NODES];
  __shared__ uint64_t sSums[kRowsAhead][kRanges];
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  if (b >= batch) return;
  const int base = cu_nodes[b];
  const int n = cu_nodes[b + 1] - base;
  int32_t* path = accept_path + (size_t)b * (max_depth + 1);
  for (int d = lane; d <= max_depth; d += kWave) path[d] = d == 0 ? 0 : -1;
  if (base < 0 || n < 1 || n > SMART_MAX_NODES || base + n > total_nodes) {
    if (lane == 0) {
      path[0] = -1;
      accept_len[b] = -1;
      bonus_token[b] = -1;
    }
    return;
  }
  // this lane's two nodes
  const int c0 = lane, c1 = lane + kWave;
  const int p0 = c0 < n ? parent[base + c0] : -2, x0 = c0 < n ? token[base + c0] : -1;
  const int p1 = c1 < n ? parent[base + c1] : -2, x1 = c1 < n ? token[base + c1] : -1;
  uint64_t ahead[kRowsAhead];
#pragma unroll
  for (int i = 0; i < kRowsAhead; ++i) ahead[i] = sums[(size_t)(base + (i < n ? i : 0)) * kRanges + lane];
  // Draws 0 .. 127 of this step, two per lane (a walk takes one per visited child and one for the bonus token).
  const uint64_t r0 = rand64(seed, step, (uint32_t)b, lane), r1 = rand64(seed, step, (uint32_t)b, lane + kWave);
  uint32_t draw = 0;
  auto next_draw = [&]() {  // draw stays wave-uniform
    const uint32_t d = draw++;
    if (d >= 2 * kWave) return rand64(seed, step, (uint32_t)b, d);
    const int l = __builtin_amdgcn_readfirstlane((int)(d & (kWave - 1)));
    return d < kWave ? readlane64(r0, l) : readlane64(r1, l);
  };
  // a node can be a child only of an older node, and only with a token of the vocabulary; its weight in its parent's row
  const bool child0 = p0 >= 0 && p0 < c0 && x0 >= 0 && x0 < V, child1 = p1 >= 0 && p1 < c1 && x1 >= 0 && x1 < V;
  const uint64_t w0 = child0 ? weight_of(prob[(size_t)(base + p0) * stride + x0]) : 0;
  const uint64_t w1 = child1 ? weight_of(prob[(size_t)(base + p1) * stride + x1]) : 0;
#pragma unroll
  for (int i = 0; i < kRowsAhead; ++i) sSums[i][lane] = ahead[i];  // (read back by the lane that wrote it)
  const int range = range_of(V);
  int cur = 0, len = 0, nrej = 0;
  uint64_t mine, R;  // this lane's range sum (less what was rejected in it), and the row's remaining weight
  for (;;) {
    mine = cur < kRowsAhead ? sSums[cur][lane] : sums[(size_t)(base + cur) * kRanges + lane];
    const uint64_t m0 = __ballot(child0 && p0 == cur && len < max_depth), m1 = __ballot(child1 && p1 == cur && len < max_depth);
    R = wave_sum(mine);
    nrej = 0;
    int nxt = -1;
    uint64_t rejected0 = 0, rejected1 = 0;  // rejected children, one bit per lane
    for (int half = 0; half < 2 && nxt < 0; ++half) {
      uint64_t m = half ? m1 : m0;
      while (m) {  // children in node order; everything in here is wave-uniform
        const int l = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)m) - 1);
        m &= m - 1;
        const int xc = half ? __builtin_amdgcn_readlane(x1, l) : __builtin_amdgcn_readlane(x0, l);
        const uint64_t wc = half ? readlane64(w1, l) : readlane64(w0, l);
        // an earlier sibling proposed the same token and was rejected
        if ((__ballot(x0 == xc) & rejected0) | (__ballot(x1 == xc) & rejected1)) continue;
        const uint64_t r = next_draw();
        if (R > 0 && __umul64hi(r, R) < wc) {
          nxt = l + kWave * half;
          break;
        }
        R -= wc;
        if (lane == xc / range) mine -= wc;
        if (half) rejected1 |= 1ull << l; else rejected0 |= 1ull << l;
        if (lane == 0) sRej[nrej] = xc;
        ++nrej;
      }
    }
    if (nxt < 0) break;
    cur = nxt;
    ++len;
    if (lane == 0) path[len] = cur;
  }
  if (lane == 0) accept_len[b] = len;
  if (R == 0) {
    if (lane == 0) bonus_token[b] = -1;
    return;
  }
  // bonus: first token whose running weight sum (rejected tokens left out) exceeds the target
  uint64_t T = __umul64hi(next_draw(), R);
  const uint64_t incl = wave_incl_scan(mine, lane);
  const uint64_t hit = __ballot(incl > T);  // never empty: T < R = the last lane's inclusive sum
  const int rg = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)hit) - 1);
  T -= readlane64(incl - mine, rg);  // the target inside range rg
  const float* row = prob + (size_t)(base + cur) * stride;
  const int v_begin = rg * range, v_end = (rg + 1) * range < V ? (rg + 1) * range : V;
  __syncthreads();  // (the rejected tokens are in LDS)
  auto rejected = [&](int i) { return sRej[i]; };
  // Up to 512 tokens (a vocabulary of 32768) eight tokens per lane are the whole range; beyond, 32 keep a 128k
  // vocabulary's range to one piece as well.
  const int found = range <= 8 * kWave ? find_in_range<8>(row, v_begin, v_end, T, nrej, rejected, lane)
                                       : find_in_range<32>(row, v_begin, v_end, T, nrej, rejected, lane);
  if (lane == 0) bonus_token[b] = found;
}

}  // namespace

extern "C" int32_t tree_accept_sample(smart_ctx* ctx, void* stream, int32_t batch, int32_t total_nodes,
                                      int32_t max_depth, int32_t vocab, const int32_t* d_cu_nodes,
                                      const int32_t* d_parent, const int32_t* d_token, const float* d_target_prob,
                                      int64_t prob_row_stride, uint64_t seed, uint64_t step, int32_t* d_accept_len,
                                      int32_t* d_accept_path, int32_t* d_bonus_token) {
  if (!ctx || batch < 0 || total_nodes < 0 || max_depth < 0 || max_depth > SMART_MAX_NODES) return SMART_EINVAL;
  if (vocab < 1 || prob_row_stride < vocab) return SMART_EINVAL;
  if (!d_cu_nodes || !d_parent || !d_token || !d_target_prob || !d_accept_len || !d_accept_path || !d_bonus_token)
    return SMART_EINVAL;
  if (batch == 0) return SMART_OK;
  int prev = 0;
  SMART_HIP_CHECK(hipGetDevice(&prev));
  if (prev != ctx->device) SMART_HIP_CHECK(hipSetDevice(ctx->device));
  const size_t need = (size_t)(total_nodes > 0 ? total_nodes : 1) * kRanges * sizeof(uint64_t);
  int32_t rc = smart::ensure_workspace(ctx, (hipStream_t)stream, need, 0, 0);
  if (rc == SMART_OK) {
    uint64_t* sums = (uint64_t*)ctx->ws;
    // Four ranges per wavefront (eight vectors in flight per lane) once that still leaves every compute unit two
    // workgroups; fewer rows are spread over four times as many wavefronts.
    if (total_nodes >= 128)
      hipLaunchKernelGGL(range_sums_kernel<4>, dim3(total_nodes, kRanges / 16), dim3(4 * kWave), 0, (hipStream_t)stream,
                         total_nodes, vocab, prob_row_stride, d_target_prob, sums);
    else if (total_nodes > 0)
      hipLaunchKernelGGL(range_sums_kernel<1>, dim3(total_nodes, kRanges / 4), dim3(4 * kWave), 0, (hipStream_t)stream,
                         total_nodes, vocab, prob_row_stride, d_target_prob, sums);
    hipLaunchKernelGGL(tree_accept_sample_kernel, dim3(batch), dim3(kWave), 0, (hipStream_t)stream, batch, total_nodes,
                       max_depth, vocab, prob_row_stride, d_cu_nodes, d_parent, d_token, d_target_prob, sums, seed,
                       step, d_accept_len, d_accept_path, d_bonus_token);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
      smart::set_last_hip_error(e);
      rc = SMART_EHIP;
    }
  }
  if (prev != ctx->device) (void)hipSetDevice(prev);
  return rc;
}
