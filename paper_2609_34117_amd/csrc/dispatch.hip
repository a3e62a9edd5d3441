// Dispatch plan of a decode step on gfx950 (Section 2.1: the step reads the
// union of the experts selected across the batch): the histogram of the
// selected expert ids, its exclusive scan, the active-expert list and the
// stable permutation that groups pairs by expert.
//
// Up to kSingleBlockPairs pairs, one block builds everything, two pairs a
// thread (1024 threads, or 512 for at most 1024 pairs over at most 512
// experts).
// Larger batches (prefill) split the pairs into 1024-pair chunks, one block
// each, in two launches:
//   1. per-chunk histograms (and id validation);
//   2. every chunk's block adds the histograms up per expert, scans the
//      totals (block 0 writes counts / offsets / active from them), and
//      scatters its pairs in pair order from offsets[e] plus the counts of e
//      in the earlier chunks.
// The result is identical to the single block's: chunk c's pairs of expert e
// land after those of chunks 0 .. c-1, each chunk in pair order.
#include "dispatch_block.h"
#include "sw_launch.h"

namespace sw {
namespace {

constexpr int kDispatchThreads = 1024;
constexpr int kDispatchWaves = kDispatchThreads / kWave;
constexpr int kMaxPool = 1024;
constexpr int kSingleBlockPairs = 2048;  // two pairs a thread of the largest block

__global__ __launch_bounds__(kDispatchThreads) void dispatch_kernel(
    const int* __restrict__ ids, int n_pairs, int m, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ perm, int* __restrict__ active,
    int* __restrict__ n_active) {
  __shared__ int cursor[kMaxPool];
  __shared__ int wave_base[kDispatchWaves * kMaxPool];
  __shared__ uint8_t wave_cnt[kDispatchWaves * kMaxPool];
  __shared__ uint32_t scan_scratch[34];
  __shared__ int bad;
  const DispatchLds lds{cursor, wave_base, wave_cnt, scan_scratch, &bad};
  dispatch_block(ids, n_pairs, m, lds, counts, offsets, perm, active, n_active);
}

// The plan of at most 2 * NT pairs over at most NT experts, in one block of NT
// threads.  Pair p belongs to run p / 64 (the pairs of one wave); within a
// run, ballots match equal ids (a pair's rank among them, the run's count of
// each id); thread e then adds expert e's counts over the runs, leaving each
// run its start within the expert, and one block scan of the totals gives the
// offsets and the active list; a pair's place is its expert's offset, plus its
// run's start, plus its rank.  Four barriers and no atomics, whatever the
// pairs: latency bounds it.  Over logits and top-k it adds 3.3 us at 512 pairs
// over 256 experts (3.7 us with dispatch_block's LDS-atomic histogram and one
// barriered scatter a chunk) and 5.0 us at 2048 (7.1 us).
template <int NT>
__global__ __launch_bounds__(NT) void dispatch_runs_kernel(
    const int* __restrict__ ids, int n_pairs, int m, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ perm, int* __restrict__ active,
    int* __restrict__ n_active) {
  constexpr int kWaves = NT / kWave, kRuns = 2 * kWaves;
  __shared__ uint32_t run_cnt_words[kRuns * NT / 4];  // [run][m] bytes
  __shared__ uint16_t run_start[kRuns * NT];          // [run][m]
  __shared__ int offset_s[NT];
  __shared__ uint32_t wave_sum[2][kWaves];
  __shared__ int bad;
  uint8_t* run_cnt = reinterpret_cast<uint8_t*>(run_cnt_words);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int id[2], rank[2];
  bool valid[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = tid + i * NT;
    valid[i] = p < n_pairs;
    id[i] = valid[i] ? ids[p] : 0;
  }
  const int runs = (n_pairs + kWave - 1) / kWave;
  for (int i = tid; i < (runs * m + 3) / 4; i += NT) run_cnt_words[i] = 0u;
  if (tid == 0) bad = 0;
  __syncthreads();

  const int nbits = id_bits(m);
  const uint64_t lt_mask = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool ok = valid[i] && id[i] >= 0 && id[i] < m;
    if (valid[i] && !ok) bad = 1;
    valid[i] = ok;
    const uint64_t peers = match_peers(ok ? id[i] : 0, ok, nbits);
    rank[i] = __popcll(peers & lt_mask);
    if (ok && rank[i] == 0)
      run_cnt[(i * kWaves + wave) * m + id[i]] = static_cast<uint8_t>(__popcll(peers));
  }
  __syncthreads();

  if (bad) {  // an id outside [0, m): the flagged plan
    for (int e = tid; e <= m; e += NT) {
      if (e < m) counts[e] = 0;
      offsets[e] = 0;
    }
    for (int p = tid; p < n_pairs; p += NT) perm[p] = p;
    if (tid == 0) *n_active = -1;
    return;
  }
  uint32_t c = 0;
  if (tid < m) {
    for (int r = 0; r < runs; ++r) {
      run_start[r * m + tid] = static_cast<uint16_t>(c);
      c += run_cnt[r * m + tid];
    }
  }
  const uint32_t a = c > 0 ? 1u : 0u;
  const uint32_t ic = wave_inclusive_scan_u32(c), ia = wave_inclusive_scan_u32(a);
  if (lane == 63) {
    wave_sum[0][wave] = ic;
    wave_sum[1][wave] = ia;
  }
  __syncthreads();
  uint32_t bc = 0, ba = 0, tc = 0, ta = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t sc = wave_sum[0][w], sa = wave_sum[1][w];
    bc += w < wave ? sc : 0u;
    ba += w < wave ? sa : 0u;
    tc += sc;
    ta += sa;
  }
  if (tid < m) {
    const int off = (int)(bc + ic - c);
    offset_s[tid] = off;
    counts[tid] = (int)c;
    offsets[tid] = off;
    if (a) active[ba + ia - 1] = tid;
  }
  if (tid == 0) {
    offsets[m] = (int)tc;
    *n_active = (int)ta;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (valid[i])
      perm[offset_s[id[i]] + run_start[(i * kWaves + wave) * m + id[i]] + rank[i]] = tid + i * NT;
}

// Scratch of the chunked dispatch (inside the caller's workspace).
struct ChunkScratch {
  int* hist;  // [n_chunks][m] per-chunk histograms
  int* bad;   // [n_chunks] invalid id seen in the chunk
};

int n_chunks_of(int n_pairs) { return (n_pairs + kDispatchThreads - 1) / kDispatchThreads; }

ChunkScratch carve_chunks(void* ws, int n_pairs, int m) {
  char* p = static_cast<char*>(ws);
  ChunkScratch s;
  s.hist = reinterpret_cast<int*>(p);
  p += align_up((size_t)n_chunks_of(n_pairs) * m * 4, 256);
  s.bad = reinterpret_cast<int*>(p);
  return s;
}

__global__ __launch_bounds__(kDispatchThreads) void dispatch_count_kernel(
    const int* __restrict__ ids, int n_pairs, int m, int* __restrict__ hist_out,
    int* __restrict__ bad_out) {
  __shared__ int hist[kMaxPool];
  __shared__ int bad;
  const int tid = threadIdx.x;
  if (tid == 0) bad = 0;
  for (int e = tid; e < m; e += kDispatchThreads) hist[e] = 0;
  __syncthreads();
  const int p = blockIdx.x * kDispatchThreads + tid;
  if (p < n_pairs) {
    const int e = ids[p];
    if (e < 0 || e >= m)
      atomicOr(&bad, 1);
    else
      atomicAdd(&hist[e], 1);
  }
  __syncthreads();
  for (int e = tid; e < m; e += kDispatchThreads) hist_out[(size_t)blockIdx.x * m + e] = hist[e];
  if (tid == 0) bad_out[blockIdx.x] = bad;
}

// Chunk b = blockIdx.x: expert e's total over all chunks and over the chunks
// before b (thread e, eight loads in flight at a time), the block scan of
// the totals, and the stable scatter of the chunk from offsets[e] plus the
// earlier chunks' count.  Block 0 also writes counts, offsets, active and
// n_active.
__global__ __launch_bounds__(kDispatchThreads) void dispatch_scatter_kernel(
    const int* __restrict__ ids, int n_pairs, int m, int n_chunks, const int* __restrict__ hist,
    const int* __restrict__ bad_in, int* __restrict__ counts, int* __restrict__ offsets,
    int* __restrict__ perm, int* __restrict__ active, int* __restrict__ n_active) {
  __shared__ int cursor[kMaxPool];
  __shared__ int wave_base[kDispatchWaves * kMaxPool];
  __shared__ uint8_t wave_cnt[kDispatchWaves * kMaxPool];
  __shared__ uint32_t scan_scratch[34];
  const int tid = threadIdx.x, b = blockIdx.x, c0 = b * kDispatchThreads;
  int any_bad = 0;
  for (int c = tid; c < n_chunks; c += kDispatchThreads) any_bad |= bad_in[c];
  if (__syncthreads_or(any_bad)) {  // an invalid id: perm is the identity
    if (c0 + tid < n_pairs) perm[c0 + tid] = c0 + tid;
    if (b == 0) {
      for (int e = tid; e <= m; e += kDispatchThreads) {
        if (e < m) counts[e] = 0;
        offsets[e] = 0;
      }
      if (tid == 0) *n_active = -1;
    }
    return;
  }
  uint32_t total = 0, before = 0;
  if (tid < m) {
    const int* col = hist + tid;
    int ch = 0;
    for (; ch + 8 <= n_chunks; ch += 8) {
      int v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = col[(size_t)(ch + j) * m];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        total += (uint32_t)v[j];
        before += ch + j < b ? (uint32_t)v[j] : 0u;
      }
    }
    for (; ch < n_chunks; ++ch) {
      const uint32_t v = (uint32_t)col[(size_t)ch * m];
      total += v;
      before += ch < b ? v : 0u;
    }
  }
  uint32_t off, apos, sum, n_act;
  block_exclusive_scan2(total, total > 0 ? 1u : 0u, scan_scratch, &off, &apos, &sum, &n_act);
  if (tid < m) cursor[tid] = (int)(off + before);
  for (int i = tid; i < kDispatchWaves * m; i += kDispatchThreads) wave_cnt[i] = 0;
  if (b == 0) {
    if (tid < m) {
      counts[tid] = (int)total;
      offsets[tid] = (int)off;
      if (total > 0) active[apos] = tid;
    }
    if (tid == 0) {
      offsets[m] = (int)sum;
      *n_active = (int)n_act;
    }
  }
  __syncthreads();
  const DispatchLds lds{cursor, wave_base, wave_cnt, nullptr, nullptr};
  scatter_chunk(ids, c0, n_pairs, m, id_bits(m), lds, perm);
}

}  // namespace

size_t dispatch_workspace_bytes(int n_pairs, int m) {
  if (n_pairs <= kSingleBlockPairs) return 0;
  const int nc = n_chunks_of(n_pairs);
  return align_up((size_t)nc * m * 4, 256) + align_up((size_t)nc * 4, 256);
}

hipError_t launch_dispatch(const int* topk_ids, int n_pairs, int m, int* counts, int* offsets,
                           int* perm, int* active, int* n_active, hipStream_t stream,
                           void* workspace) {
  if (n_pairs <= kSingleBlockPairs) {
    if (n_pairs <= 1024 && m <= 512)
      dispatch_runs_kernel<512><<<1, 512, 0, stream>>>(topk_ids, n_pairs, m, counts, offsets,
                                                       perm, active, n_active);
    else
      dispatch_runs_kernel<1024><<<1, 1024, 0, stream>>>(topk_ids, n_pairs, m, counts, offsets,
                                                         perm, active, n_active);
    return hipGetLastError();
  }
  if (workspace == nullptr) {  // one block, chunk by chunk
    dispatch_kernel<<<1, kDispatchThreads, 0, stream>>>(topk_ids, n_pairs, m, counts, offsets, perm,
                                                        active, n_active);
    return hipGetLastError();
  }
  const int nc = n_chunks_of(n_pairs);
  const ChunkScratch s = carve_chunks(workspace, n_pairs, m);
  dispatch_count_kernel<<<nc, kDispatchThreads, 0, stream>>>(topk_ids, n_pairs, m, s.hist, s.bad);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  dispatch_scatter_kernel<<<nc, kDispatchThreads, 0, stream>>>(
      topk_ids, n_pairs, m, nc, s.hist, s.bad, counts, offsets, perm, active, n_active);
  return hipGetLastError();
}

}  // namespace sw
