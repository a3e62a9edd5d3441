// Router of the MoE layer on gfx950: fp32 logits, masked top-k selection and
// renormalised gates (Section 3.1, Eq. 2 and the renormalisation after it),
// and the fused route + dispatch of small (decode-sized) batches.
#include <algorithm>

#include "dispatch_block.h"
#include "sw_launch.h"

namespace sw {
namespace {

// fp32 w = hi + mid + lo exactly, each piece a bf16 (truncating split: hi
// keeps the top 8 significand bits, mid the next 8, lo the last 8), for
// eight weights at once; returns the three packed bf16x8 operands.
__device__ __forceinline__ void split3_bf16x8(const float4& a, const float4& b, u32x4& hi,
                                              u32x4& mid, u32x4& lo) {
  const float w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t h[8], md[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t u = __float_as_uint(w[i]);
    h[i] = u & 0xffff0000u;
    const float r1 = w[i] - __uint_as_float(h[i]);
    md[i] = __float_as_uint(r1) & 0xffff0000u;
    l[i] = __float_as_uint(r1 - __uint_as_float(md[i]));
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    hi[q] = (h[2 * q] >> 16) | h[2 * q + 1];
    mid[q] = (md[2 * q] >> 16) | md[2 * q + 1];
    lo[q] = (l[2 * q] >> 16) | (l[2 * q + 1] & 0xffff0000u);
  }
}

// Partial logits part[ks][t][e] = sum over the ks-th slice of H of
// x[t, h] * wr[e, h], fp32.  Grid (token tiles, expert tiles, KS); a block
// is KW waves that split its slice; tile = 16 experts x 16 tokens.  The
// router row is split exactly into three bf16 pieces, so each 32-wide K step
// is three bf16 MFMAs whose products are exact in fp32.  Spreading H over KS
// blocks lets a decode-sized batch (few tiles) use many compute units.
template <int KW>
__global__ __launch_bounds__(64 * KW) void route_logits_kernel(const uint16_t* __restrict__ x,
                                                              const float* __restrict__ wr,
                                                              float* __restrict__ part, int T,
                                                              int H, int m) {
  constexpr int kChunk = 4;  // K steps whose loads are issued together
  __shared__ f32x4 red[KW][kWave];
  const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 16, ks = blockIdx.z, KS = gridDim.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const auto w_rsrc = make_rsrc(wr, 4u * (uint32_t)m * (uint32_t)H);
  const auto x_rsrc = make_rsrc(x, 2u * (uint32_t)T * (uint32_t)H);
  const bool e_ok = e0 + r < m, t_ok = t0 + r < T;
  const uint32_t w_row = (uint32_t)(e0 + r) * H * 4u, x_row = (uint32_t)(t0 + r) * H * 2u;
  const int nsteps = (H + 31) >> 5;
  const int b_lo = (ks * nsteps) / KS, b_hi = ((ks + 1) * nsteps) / KS;
  const int s_lo = b_lo + (wave * (b_hi - b_lo)) / KW;
  const int s_hi = b_lo + ((wave + 1) * (b_hi - b_lo)) / KW;

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int sb = s_lo; sb < s_hi; sb += kChunk) {
    u32x4 wa[kChunk], wb[kChunk], xb[kChunk];
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      const int col = (sb + c) * 32 + kg * 8;
      const bool ok = sb + c < s_hi && col < H;
      const uint32_t wo = (ok && e_ok) ? w_row + (uint32_t)col * 4u : kOutOfRange;
      wa[c] = buf_ld128(w_rsrc, wo);
      wb[c] = buf_ld128(w_rsrc, wo + 16u);
      xb[c] = buf_ld128(x_rsrc, (ok && t_ok) ? x_row + (uint32_t)col * 2u : kOutOfRange);
    }
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      u32x4 hi, mid, lo;
      split3_bf16x8(__builtin_bit_cast(float4, wa[c]), __builtin_bit_cast(float4, wb[c]), hi, mid, lo);
      acc = mfma_16x16x32(hi, xb[c], acc);
      acc = mfma_16x16x32(mid, xb[c], acc);
      acc = mfma_16x16x32(lo, xb[c], acc);
    }
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    f32x4 c = red[0][lane];
#pragma unroll
    for (int w = 1; w < KW; ++w) c += red[w][lane];
    // c[i] = partial z of expert e0 + 4*kg + i, token t0 + r
    const int t = t0 + r;
    if (t < T) {
      float* dst = part + ((size_t)ks * T + t) * m;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = e0 + 4 * kg + i;
        if (e < m) dst[e] = c[i];
      }
    }
  }
}

// Router logits of prefill-sized batches: a block of 8 waves computes 32 TF
// tokens x 64 experts over slice blockIdx.z of H (KS = gridDim.z slices of
// whole 128-column units); wave w takes experts e0 + 16 (w % 4) .. + 15 of the
// token half w / 4.  Same exact three-piece products as route_logits_kernel,
// accumulated over H in ascending order.
//
// The matrix cores need 5 us of 3 bf16 MFMAs a product at 4096 tokens x 256
// experts; what bounds the loop is how the operands arrive.  An MFMA operand
// wants consecutive lanes in different rows, and a load like that costs the
// compute unit's address path one cycle per lane (64 a load, against 8 to 16
// where consecutive lanes share a line: 52K of the 70K cycles of the former
// kernel, which read the router so).  So both operands go straight into LDS,
// 8 or 16 consecutive lanes a row (buffer loads with the LDS bit), three
// 64-column chunks ahead in a four-slot ring, and the operand reads pick
// their rows there.  A router fragment is split into its three pieces once
// for TF token blocks.  At 4096 tokens x 256 experts, H 2048, kernel trace:
// 27 us with the router read into registers (64-token tiles of 4 waves),
// 29 us so with the x ring and 128-token tiles, 19 us with both rings; with
// 64-token tiles and both rings (the router read twice as often) 27 us.
constexpr int kWideE = 64, kWideKc = 128;    // experts a block, columns of a slice's unit
constexpr int kWideWaves = 8, kWideAhead = 3, kWideSlots = kWideAhead + 1;
constexpr int kWideCols = 64;                // columns of a chunk
constexpr int kWideSteps = kWideCols / 32;   // MFMA steps a chunk

// The 16-byte pieces of a staged row sit in XOR-swizzled places, so that the
// operand reads hit distinct banks: 8 pieces a 128-byte x row, 16 a 256-byte
// router row.  (A 16-lane phase of a 128-bit LDS read covers rows 0-3 and 12-15
// of one piece and rows 4-11 of the next k-group's: a swizzle that also mixes in
// row / 8 counted one conflict cycle for every two reads, this one none.)
__device__ __forceinline__ int wide_x_place(int row, int piece) {
  return piece ^ (row & 7);
}
__device__ __forceinline__ int wide_w_place(int row, int piece) { return piece ^ (row & 15); }

template <int TF>
__global__ __launch_bounds__(64 * kWideWaves) void route_logits_wide_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ wr, float* __restrict__ part, int T,
    int H, int m) {
  constexpr int kTok = 32 * TF;                 // tokens a block
  constexpr int kXSegs = kTok / 8 / kWideWaves;   // 1 KiB x loads (8 rows) a wave and chunk
  constexpr int kWSegs = kWideE / 4 / kWideWaves;  // 1 KiB router loads (4 rows)
  static_assert(kTok % (8 * kWideWaves) == 0 && kWideE % (4 * kWideWaves) == 0,
                "whole rounds of segments");
  constexpr int kX = kTok * kWideCols, kSlot = kX + 2 * kWideE * kWideCols;  // in 16-bit words
  __shared__ __attribute__((aligned(1024))) uint16_t ring0[kSlot];
  __shared__ __attribute__((aligned(1024))) uint16_t ring1[kSlot];
  __shared__ __attribute__((aligned(1024))) uint16_t ring2[kSlot];
  __shared__ __attribute__((aligned(1024))) uint16_t ring3[kSlot];
  const int t0 = blockIdx.x * kTok, e0 = blockIdx.y * kWideE;
  const int ks = blockIdx.z, KS = gridDim.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const u32x4 w_rsrc = rsrc_words(wr, 4u * (uint32_t)m * (uint32_t)H);
  const u32x4 x_rsrc = rsrc_words(x, 2u * (uint32_t)T * (uint32_t)H);
  const int eg = (wave & 3) * 16, half = wave >> 2;
  const int all = H / kWideKc;
  const int c_lo = ((ks * all) / KS) * (kWideKc / kWideCols);
  const int n = (((ks + 1) * all) / KS) * (kWideKc / kWideCols) - c_lo;  // chunks, an even number
  // source offsets of this lane's piece of each segment; a row past the batch
  // or the pool reads out of range in every chunk (less than a row's bytes are
  // added to 2^31, still past the resource)
  uint32_t x_off[kXSegs], w_off[kWSegs];
#pragma unroll
  for (int j = 0; j < kXSegs; ++j) {
    const int row = (wave + j * kWideWaves) * 8 + (lane >> 3);
    const int piece = wide_x_place(row, lane & 7);
    x_off[j] = t0 + row < T
                   ? ((uint32_t)(t0 + row) * H + (uint32_t)(c_lo * kWideCols + piece * 8)) * 2u
                   : kOutOfRange;
  }
#pragma unroll
  for (int j = 0; j < kWSegs; ++j) {
    const int row = (wave + j * kWideWaves) * 4 + (lane >> 4);
    const int piece = wide_w_place(row, lane & 15);
    w_off[j] = e0 + row < m
                   ? ((uint32_t)(e0 + row) * H + (uint32_t)(c_lo * kWideCols + piece * 4)) * 4u
                   : kOutOfRange;
  }
  auto slot = [&](int k) { return k == 0 ? ring0 : k == 1 ? ring1 : k == 2 ? ring2 : ring3; };
  // chunk c into ring slot k = c % kWideSlots
  // (past the slice's end its last chunk again: load_lds16's `add` stays below
  // the resource, which a router of one expert is only a row long)
  auto stage = [&](int c, int k) {
    c = min(c, n - 1);
    const uint32_t at = lds_address(slot(k)) + (uint32_t)wave * 1024u;
    for_each_index<kXSegs>([&](auto j) {
      load_lds16<decltype(j)::value * kWideWaves * 1024>(x_rsrc, x_off[decltype(j)::value],
                                                         (uint32_t)(c * kWideCols * 2), at);
    });
    for_each_index<kWSegs>([&](auto j) {
      load_lds16<kX * 2 + decltype(j)::value * kWideWaves * 1024>(
          w_rsrc, w_off[decltype(j)::value], (uint32_t)(c * kWideCols * 4), at);
    });
  };
  // this lane's operand places (in 16-bit words), per step
  int b_place[kWideSteps], w_place[kWideSteps][2];
#pragma unroll
  for (int st = 0; st < kWideSteps; ++st) {
    b_place[st] = (half * 16 * TF + r) * kWideCols + wide_x_place(r, st * 4 + kg) * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      w_place[st][i] = kX + (eg + r) * 2 * kWideCols + wide_w_place(r, st * 8 + kg * 2 + i) * 8;
  }

  f32x4 acc[TF];
#pragma unroll
  for (int nb = 0; nb < TF; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kWideAhead; ++c) stage(c, c);
  // Loads issued after chunk c's when chunk c is about to be read: the next
  // kWideAhead - 1 chunks'.  Past the slice's end the last chunk is staged like
  // any other (into slots never read again), so the count holds to the end.
  constexpr int kAfter = (kWideAhead - 1) * (kXSegs + kWSegs);
  for (int c0 = 0; c0 < n; c0 += kWideSlots) {
#pragma unroll
    for (int d = 0; d < kWideSlots; ++d) {
      if (d == 2 && c0 + 2 >= n) break;  // n is even
      // this wave's part of chunk c0 + d landed and its reads of the chunk
      // before are done; then so are every wave's, and that slot is free
      __builtin_amdgcn_s_waitcnt(vmcnt_at_most_lds_done(kAfter));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");  // (no LDS read moves above it)
      stage(c0 + d + kWideAhead, (d + kWideAhead) % kWideSlots);
      const uint16_t* buf = slot(d);
      // every operand read of the chunk goes out before the splits, and the
      // MFMAs run piece by piece over TF independent accumulators
      u32x4 w[kWideSteps][2], b[kWideSteps][TF];
#pragma unroll
      for (int st = 0; st < kWideSteps; ++st) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          w[st][i] = *reinterpret_cast<const u32x4*>(buf + w_place[st][i]);
#pragma unroll
        for (int nb = 0; nb < TF; ++nb)
          b[st][nb] = *reinterpret_cast<const u32x4*>(buf + b_place[st] + nb * 16 * kWideCols);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < kWideSteps; ++st) {
        u32x4 w3[3];
        split3_bf16x8(__builtin_bit_cast(float4, w[st][0]), __builtin_bit_cast(float4, w[st][1]),
                      w3[0], w3[1], w3[2]);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int nb = 0; nb < TF; ++nb) acc[nb] = mfma_16x16x32(w3[p], b[st][nb], acc[nb]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));  // the loads past the end landed in LDS
  // acc[nb][i]: expert e0 + eg + 4 kg + i, token t0 + 16 (half TF + nb) + r
  const int e = e0 + eg + 4 * kg;
#pragma unroll
  for (int nb = 0; nb < TF; ++nb) {
    const int t = t0 + (half * TF + nb) * 16 + r;
    if (t < T) {
      float* dst = part + ((size_t)ks * T + t) * m + e;
      if ((m & 3) == 0) {  // whole 16-byte groups of experts
        if (e < m) *reinterpret_cast<f32x4*>(dst) = acc[nb];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (e + i < m) dst[i] = acc[nb][i];
      }
    }
  }
}

constexpr int kMaxSplit = 4;  // slices of H per logit tile

// Columns of a routing call: the m experts the top-k selects from, whose
// partial logits sit in rows of ld >= m columns (ld = m + 1 when the last
// column is the shared expert's gate logit), the k routed slots and the S
// slots of the shared expert's parts after them (ids m .. m + S - 1).
struct Cols {
  int m, ld, k, S;
  int R;  // token groups of the shared parts: the pool holds R copies of the S parts
  __device__ __host__ int plan_m() const { return m + R * S; }
};

// Token t's group of shared-part copies: R contiguous runs of the batch.
__device__ __forceinline__ int token_group(const Cols& c, int t, int T) {
  return c.R > 1 ? (int)((long long)t * c.R / T) : 0;
}

// The partial logits of one token for this lane's KPL experts, and what the
// lane knows of those experts whatever the token: their biases and whether
// they may be selected.  Every load is unconditional, at a clamped index, and
// nothing is computed between the loads: with a branch around each expert's
// loads the compiler waits for them one expert at a time, a memory round trip
// each (three with a mask and a bias): logits and top-k of 64 tokens over 256
// experts took 9.2 us that way and take 7.7 us this way.
template <int KPL>
struct LogitParts {
  float z[kMaxSplit][KPL];
  float gate[kMaxSplit];  // of the shared expert's gate column, with one
};

template <int KPL>
struct LaneExperts {
  float bias[KPL];
  bool ok[KPL];
};

template <int KPL>
__device__ __forceinline__ LogitParts<KPL> load_logits(const float* __restrict__ part, int KS,
                                                       int T, const Cols& c, int t,
                                                       const int (&eid)[KPL]) {
  LogitParts<KPL> l;
  const float* p = part + (size_t)min(t, T - 1) * c.ld;
  const size_t plane = (size_t)T * c.ld;
#pragma unroll
  for (int ks = 0; ks < kMaxSplit; ++ks) {
#pragma unroll
    for (int q = 0; q < KPL; ++q) l.z[ks][q] = 0.f;
    if (ks < KS) {  // uniform
#pragma unroll
      for (int q = 0; q < KPL; ++q) l.z[ks][q] = p[ks * plane + min(eid[q], c.m - 1)];
    }
    l.gate[ks] = ks < KS && c.S > 0 ? p[ks * plane + c.m] : 0.f;  // uniform
  }
  return l;
}

template <int KPL>
__device__ __forceinline__ LaneExperts<KPL> load_experts(const Cols& c, const int (&eid)[KPL],
                                                         const float* __restrict__ bias,
                                                         const uint8_t* __restrict__ keep_mask) {
  LaneExperts<KPL> x;
  uint8_t keep[KPL];
#pragma unroll
  for (int q = 0; q < KPL; ++q) {
    x.bias[q] = 0.f;
    keep[q] = 1;
  }
  if (bias != nullptr) {
#pragma unroll
    for (int q = 0; q < KPL; ++q) x.bias[q] = bias[min(eid[q], c.m - 1)];
  }
  if (keep_mask != nullptr) {
#pragma unroll
    for (int q = 0; q < KPL; ++q) keep[q] = keep_mask[min(eid[q], c.m - 1)];
  }
#pragma unroll
  for (int q = 0; q < KPL; ++q) x.ok[q] = eid[q] < c.m && keep[q] != 0;
  return x;
}

// Order keys of a token's logits: z = sum of the KS partials in slice order,
// plus the bias; 0 marks an ineligible expert (the one logit whose key is 0,
// a NaN, is nudged to 1).
template <int KPL>
__device__ __forceinline__ void logit_keys(const LogitParts<KPL>& l, const LaneExperts<KPL>& x,
                                           int KS, bool biased, uint32_t (&key)[KPL]) {
#pragma unroll
  for (int q = 0; q < KPL; ++q) {
    float z = l.z[0][q];
#pragma unroll
    for (int ks = 1; ks < kMaxSplit; ++ks)
      if (ks < KS) z += l.z[ks][q];
    if (biased) z += x.bias[q];
    key[q] = x.ok[q] ? max(f32_order_key(z), 1u) : 0u;
  }
}

// Gate of the shared expert (Section 3.3): the sigmoid of its gate logit, the
// partials of column m summed in slice order like every other logit.
__device__ __forceinline__ float shared_gate(const float (&zp)[kMaxSplit], int KS) {
  float z = zp[0];
#pragma unroll
  for (int ks = 1; ks < kMaxSplit; ++ks)
    if (ks < KS) z += zp[ks];
  return 1.0f / (1.0f + expf(-z));
}

// Result of one token's selection, held by the lanes of its wave: lane j < k
// holds slot j.
struct Selection {
  int id;        // expert id of this lane's slot, -1 if none
  float z;       // its logit
  float gate;    // renormalised gate (0 without an expert)
  float gap;     // z_(k) - z_(k+1); +inf if only k eligible; NaN if fewer
};

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// The k + 1 selection rounds and the softmax over the k selected logits of a
// wave that holds one token's keys, lane l those of experts q * 64 + l.  Each
// round takes the largest remaining order key (a wave max) and the smallest
// expert id holding it: the first set bit of the first non-empty ballot
// (scalar work, in place of a second cross-lane reduction).  The (k+1)-th
// round only reads the runner-up for the gap.
template <int KPL>
__device__ __forceinline__ Selection select_topk(uint32_t (&key)[KPL], const int (&eid)[KPL],
                                                 int k, int lane) {
  Selection s{-1, 0.f, 0.f, 0.f};
  float z_first = 0.f, zk = 0.f, zk1 = 0.f;
  bool complete = true, have_next = false;
  for (int j = 0; j <= k; ++j) {
    uint32_t lm = key[0];
#pragma unroll
    for (int q = 1; q < KPL; ++q) lm = umax(lm, key[q]);
    const uint32_t best = wave_max_u32(lm);
    const bool found = best != 0;  // uniform
    const float ze = f32_from_order_key(best);
    if (j == k) {
      if (found) {
        zk1 = ze;
        have_next = true;
      }
      break;
    }
    if (!found) complete = false;
    int e = 0;
#pragma unroll
    for (int q = KPL - 1; q >= 0; --q) {
      const uint64_t holds = __ballot(key[q] == best);
      if (holds != 0) e = q * 64 + __builtin_ctzll(holds);
    }
    if (found) {
      if (j == 0) z_first = ze;
      if (lane == j) {
        s.id = e;
        s.z = ze;
      }
      if (j == k - 1) zk = ze;
#pragma unroll
      for (int q = 0; q < KPL; ++q)
        if (eid[q] == e) key[q] = 0u;
    }
  }
  const float ex = (lane < k && s.id >= 0) ? expf(s.z - z_first) : 0.f;
  const float sum = wave_sum_f32(ex);
  s.gate = s.id >= 0 ? ex / sum : 0.f;
  s.gap = !complete ? __builtin_nanf("") : (have_next ? zk - zk1 : __builtin_inff());
  return s;
}

// A token's selection and its shared gate (0 without a shared expert).
struct Routed {
  Selection s;
  float sgate;
};

template <int KPL>
__device__ __forceinline__ void wave_experts(int lane, int (&eid)[KPL]) {
#pragma unroll
  for (int q = 0; q < KPL; ++q) eid[q] = q * 64 + lane;
}

// Top-k of one token per wave, from its loaded logits.
template <int KPL>
__device__ __forceinline__ Routed select_wave(const LogitParts<KPL>& l, const LaneExperts<KPL>& x,
                                              const int (&eid)[KPL], int KS, const Cols& c,
                                              bool biased) {
  uint32_t key[KPL];
  Routed o;
  o.sgate = c.S > 0 ? shared_gate(l.gate, KS) : 0.f;
  logit_keys<KPL>(l, x, KS, biased, key);
  o.s = select_topk<KPL>(key, eid, c.k, threadIdx.x & 63);
  return o;
}

// Slot `slot` of token t: a routed slot (slot < k) takes the selection,
// a shared slot k + s the shared expert's part m + s with the shared gate.
__device__ __forceinline__ int slot_id(const Selection& s, const Cols& c, int slot, int t, int T) {
  return slot < c.k ? s.id : c.m + token_group(c, t, T) * c.S + slot - c.k;
}

__device__ __forceinline__ void store_selection(const Routed& o, int t, int T, const Cols& c,
                                                int slot, int* __restrict__ topk_ids,
                                                float* __restrict__ topk_w,
                                                float* __restrict__ gap) {
  const int kout = c.k + c.S;
  if (slot < kout) {
    topk_ids[(size_t)t * kout + slot] = slot_id(o.s, c, slot, t, T);
    topk_w[(size_t)t * kout + slot] = slot < c.k ? o.s.gate : o.sgate;
  }
  if (gap != nullptr && slot == 0) gap[t] = o.s.gap;
}

// One token per wave, four per block.  (Four tokens a wave, one per row of 16
// lanes, holds 16 experts a lane where this holds 4, and the rounds' work per
// lane counts more than the waves saved: logits and top-k of 8 tokens over
// 256 experts took 9.9 us that way and take 7.4 us this way, of 37 tokens over
// 128 experts 8.7 and 7.2 us, of 20 tokens over 32 experts 6.6 and 6.1 us.)
template <int KPL>
__global__ __launch_bounds__(256) void route_topk_kernel(const float* __restrict__ part, int KS,
                                                        const float* __restrict__ bias,
                                                        const uint8_t* __restrict__ keep_mask,
                                                        int T, Cols c,
                                                        int* __restrict__ topk_ids,
                                                        float* __restrict__ topk_w,
                                                        float* __restrict__ gap) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;  // wave-uniform
  int eid[KPL];
  wave_experts<KPL>(threadIdx.x & 63, eid);
  const LogitParts<KPL> l = load_logits<KPL>(part, KS, T, c, t, eid);
  const LaneExperts<KPL> x = load_experts<KPL>(c, eid, bias, keep_mask);
  const Routed o = select_wave<KPL>(l, x, eid, KS, c, bias != nullptr);
  store_selection(o, t, T, c, threadIdx.x & 63, topk_ids, topk_w, gap);
}

// Route + dispatch of a small batch in one block: wave t selects token t, the
// ids go to LDS as well as to memory, and the first wave then builds the
// dispatch plan from them.  Up to 16 tokens and 64 pairs, what a block of one
// wave a token and a plan of one pair a lane hold: 9.0 us with the logits for
// one token over 256 experts and 9.7 us for 8, against 10.4 us for the top-k
// and dispatch kernels at 8.  Beyond, one block would serialise selections and
// plan (two tokens a wave and a block-wide plan took 9.5 against 8.8 us at 20
// tokens over 32 experts, and 12.8 against 10.8 us over 256); over small pools
// the row form below takes such batches.
constexpr int kFusedMaxPool = 256;
constexpr int kFusedMaxTokens = 16;
constexpr int kFusedMaxPairs = 64;

// The plan of at most 64 pairs over at most 256 experts, by one wave with
// ballots and wave scans, without a barrier; lane q < n_pairs holds pair q's
// id in e.  Expert i's count and offset live on lane i % 64, slot i / 64, and
// go between the pairs' lanes and the experts' through `lds` (kFusedMaxPool
// words of this wave's own).  The plan is the one dispatch_block builds, value
// for value.
__device__ __forceinline__ void wave_plan(int e, int n_pairs, int m, volatile int* lds,
                                          int* __restrict__ counts, int* __restrict__ offsets,
                                          int* __restrict__ perm, int* __restrict__ active,
                                          int* __restrict__ n_active) {
  const int lane = threadIdx.x & 63;
  const bool valid = lane < n_pairs;
  if (__ballot(valid && (e < 0 || e >= m)) != 0) {  // the flagged plan
    for (int i = lane; i <= m; i += 64) {
      if (i < m) counts[i] = 0;
      offsets[i] = 0;
    }
    if (valid) perm[lane] = lane;
    if (lane == 0) *n_active = -1;
    return;
  }
  // the lanes of equal ids: the first of them posts their number
  const uint64_t peers = match_peers(e, valid, id_bits(m));
  const int rank = __popcll(peers & ((1ull << lane) - 1ull));
#pragma unroll
  for (int j = 0; j < 4; ++j) lds[j * 64 + lane] = 0;
  __builtin_amdgcn_wave_barrier();
  if (valid && rank == 0) lds[e] = __popcll(peers);
  __builtin_amdgcn_wave_barrier();
  int cnt[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cnt[j] = lds[j * 64 + lane];
  __builtin_amdgcn_wave_barrier();
  // offsets = exclusive scan of the counts, active = the experts with pairs,
  // both in expert order (slot-major)
  uint32_t run_off = 0, run_act = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (j * 64 >= m) break;  // uniform
    const int i = j * 64 + lane;
    const uint32_t c = i < m ? (uint32_t)cnt[j] : 0u, a = c > 0 ? 1u : 0u;
    const uint32_t ic = wave_inclusive_scan_u32(c), ia = wave_inclusive_scan_u32(a);
    const int off = (int)(run_off + ic - c);
    lds[i] = off;
    if (i < m) {
      counts[i] = (int)c;
      offsets[i] = off;
      if (c > 0) active[run_act + ia - a] = i;
    }
    run_off += __builtin_amdgcn_readlane(ic, 63);
    run_act += __builtin_amdgcn_readlane(ia, 63);
  }
  if (lane == 0) {
    offsets[m] = (int)run_off;
    *n_active = (int)run_act;
  }
  // stable scatter: pair q goes after the earlier pairs of its expert
  __builtin_amdgcn_wave_barrier();
  if (valid) perm[lds[e] + rank] = lane;
}

template <int KPL>
__global__ __launch_bounds__(64 * kFusedMaxTokens) void route_select_dispatch_kernel(
    const float* __restrict__ part, int KS, const float* __restrict__ bias,
    const uint8_t* __restrict__ keep_mask, int T, Cols c, int* __restrict__ topk_ids,
    float* __restrict__ topk_w, float* __restrict__ gap, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ perm, int* __restrict__ active,
    int* __restrict__ n_active) {
  __shared__ int ids_s[kFusedMaxPairs];
  __shared__ int plan_s[kFusedMaxPool];
  const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;  // one wave per token
  const int kout = c.k + c.S, n_pairs = T * kout;
  int eid[KPL];
  wave_experts<KPL>(lane, eid);
  const LogitParts<KPL> l = load_logits<KPL>(part, KS, T, c, t, eid);
  const LaneExperts<KPL> x = load_experts<KPL>(c, eid, bias, keep_mask);
  const Routed o = select_wave<KPL>(l, x, eid, KS, c, bias != nullptr);
  store_selection(o, t, T, c, lane, topk_ids, topk_w, gap);
  if (lane < kout) ids_s[t * kout + lane] = slot_id(o.s, c, lane, t, T);
  __syncthreads();
  if (t == 0)
    wave_plan(lane < n_pairs ? ids_s[lane] : 0, n_pairs, c.plan_m(), plan_s, counts, offsets,
              perm, active, n_active);
}

// The same for up to 32 tokens over a small pool, beyond the 64 pairs of one
// plan wave: a row of 16 lanes selects a token (four tokens a wave, 512 threads)
// and the block then builds the plan.  A lane holds four times the experts of
// the wave form's, so this pays while they are few (with logits, against the
// top-k and dispatch kernels): 32 tokens, top-4 over 32 experts 8.0 and 8.7 us,
// over 64 8.5 and 8.9 us, top-8 over 64 9.6 and 9.7 us; over 128 the separate
// kernels are ahead (9.3 against 10.8 us, top-4).
constexpr int kRowFusedMaxPool = 64;  // of the experts selected from
constexpr int kRowFusedTokens = 32, kRowFusedMaxK = 16;
constexpr int kRowFusedThreads = 16 * kRowFusedTokens;

// Reductions inside one 16-lane row (quad swaps, then the half-row and row
// mirrors): every lane of the row ends with the row's result.
template <typename Op>
__device__ __forceinline__ uint32_t row_reduce_u32(uint32_t v, uint32_t identity, Op op) {
  v = op(v, dpp_mov<dpp::kXor1>(identity, v));
  v = op(v, dpp_mov<dpp::kXor2>(identity, v));
  v = op(v, dpp_mov<dpp::kHalfMirror>(identity, v));
  return op(v, dpp_mov<dpp::kMirror>(identity, v));
}

// select_topk for one token a row, lane r of it holding the keys of experts
// q * 16 + r.  The largest key is a row maximum, the smallest expert holding
// it a row minimum.  The softmax sum pairs the row's lanes as the first four
// steps of the wave's sum do (whose others only add +0), so the gates are the
// same bits.
template <int KPL>
__device__ __forceinline__ Selection select_row(uint32_t (&key)[KPL], const int (&eid)[KPL], int k,
                                                int r) {
  Selection s{-1, 0.f, 0.f, 0.f};
  float z_first = 0.f, zk = 0.f, zk1 = 0.f;
  bool complete = true, have_next = false;
  for (int j = 0; j <= k; ++j) {
    uint32_t lm = key[0];
#pragma unroll
    for (int q = 1; q < KPL; ++q) lm = umax(lm, key[q]);
    const uint32_t best = row_reduce_u32(lm, 0u, umax);
    const bool found = best != 0;  // uniform over the row
    const float ze = f32_from_order_key(best);
    if (j == k) {
      zk1 = ze;
      have_next = found;
      break;
    }
    uint32_t cand = 0xffffffffu;
#pragma unroll
    for (int q = KPL - 1; q >= 0; --q) cand = key[q] == best ? (uint32_t)eid[q] : cand;
    const int e = (int)row_reduce_u32(cand, 0xffffffffu,
                                      [](uint32_t a, uint32_t b) { return a < b ? a : b; });
    if (!found) complete = false;
    if (found) {
      if (j == 0) z_first = ze;
      if (r == j) {
        s.id = e;
        s.z = ze;
      }
      if (j == k - 1) zk = ze;
#pragma unroll
      for (int q = 0; q < KPL; ++q)
        if (eid[q] == e) key[q] = 0u;
    }
  }
  const float ex = r < k && s.id >= 0 ? expf(s.z - z_first) : 0.f;
  const float sum = __uint_as_float(row_reduce_u32(
      __float_as_uint(ex), 0u, [](uint32_t a, uint32_t b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
      }));
  s.gate = s.id >= 0 ? ex / sum : 0.f;
  s.gap = !complete ? __builtin_nanf("") : (have_next ? zk - zk1 : __builtin_inff());
  return s;
}

template <int KPL>
__global__ __launch_bounds__(kRowFusedThreads) void route_select_dispatch_rows_kernel(
    const float* __restrict__ part, int KS, const float* __restrict__ bias,
    const uint8_t* __restrict__ keep_mask, int T, Cols c, int* __restrict__ topk_ids,
    float* __restrict__ topk_w, float* __restrict__ gap, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ perm, int* __restrict__ active,
    int* __restrict__ n_active) {
  constexpr int kWaves = kRowFusedThreads / kWave;
  __shared__ int ids_s[kRowFusedTokens * kRowFusedMaxK];
  __shared__ int cursor[kFusedMaxPool];
  __shared__ int wave_base[kWaves * kFusedMaxPool];
  __shared__ uint8_t wave_cnt[kWaves * kFusedMaxPool];
  __shared__ uint32_t scan_scratch[34];
  __shared__ int bad;
  const int t = threadIdx.x >> 4, r = threadIdx.x & 15;
  const int kout = c.k + c.S;
  if ((threadIdx.x >> 6) * 4 < T) {  // wave-uniform
    int eid[KPL];
#pragma unroll
    for (int q = 0; q < KPL; ++q) eid[q] = q * 16 + r;
    const LogitParts<KPL> l = load_logits<KPL>(part, KS, T, c, t, eid);
    const LaneExperts<KPL> x = load_experts<KPL>(c, eid, bias, keep_mask);
    uint32_t key[KPL];
    Routed o;
    o.sgate = c.S > 0 ? shared_gate(l.gate, KS) : 0.f;
    logit_keys<KPL>(l, x, KS, bias != nullptr, key);
    o.s = select_row<KPL>(key, eid, c.k, r);
    if (t < T) {
      store_selection(o, t, T, c, r, topk_ids, topk_w, gap);
      if (r < kout) ids_s[t * kout + r] = slot_id(o.s, c, r, t, T);
    }
  }
  __syncthreads();
  const DispatchLds lds{cursor, wave_base, wave_cnt, scan_scratch, &bad};
  dispatch_block(ids_s, T * kout, c.plan_m(), lds, counts, offsets, perm, active, n_active);
}

// Split of the router contraction for T tokens and m experts: KW waves per
// block, KS slices of H (blocks per output tile).  Few tiles (decode): 4
// waves and up to 4 slices of H, so that about 256 blocks share the router
// bytes; many tiles (prefill): route_logits_wide_kernel's tiles of 128 tokens x
// 64 experts over slices of at least 8 units of 128 columns (2 slices at H =
// 2048), or, when H is not a whole number of units, 2-wave 16 x 16 tiles and no
// split.  At 1024 tiles the wide form fills a quarter of the chip (64 blocks at
// 1024 tokens x 256 experts, H 2048) and is ahead all the same: logits and top-k
// 18.6 us, 22.2 with the 64-token register tiles it replaced, and it stayed ahead
// of those at every size measured up to 32,768 tokens, but for pools of at most
// 24 experts right past 16,384 tokens, where two slices leave a last wave of two
// blocks (33.9 against 32.6 us at 8 experts).
struct LogitsSplit {
  int kw, ks;
  bool wide;  // route_logits_wide_kernel
};

LogitsSplit logits_split(int T, int H, int m) {
  const long tiles = (long)((T + 15) / 16) * ((m + 15) / 16);
  if (tiles >= 1024) {
    if (H % kWideKc != 0) return {2, 1, false};
    // slices of at least 8 units: at 4096 tokens over 256 experts that is one
    // block a compute unit (and fewer slices are fewer partials to re-read)
    return {4, std::min(kMaxSplit, std::max(1, H / kWideKc / 8)), true};
  }
  const int nsteps = (H + 31) / 32;
  const int max_ks = std::min(kMaxSplit, std::max(1, nsteps / 16));  // waves keep >= 4 K steps
  const long want = (256 + tiles - 1) / tiles;
  return {4, (int)std::max<long>(1, std::min<long>(want, max_ks)), false};
}

hipError_t launch_logits(const uint16_t* x, int T, const float* wr, int H, int m, float* part,
                         const LogitsSplit& sp, hipStream_t stream) {
  if (sp.wide) {
    const dim3 wgrid((T + 127) / 128, (m + kWideE - 1) / kWideE, sp.ks);
    route_logits_wide_kernel<4><<<wgrid, 64 * kWideWaves, 0, stream>>>(x, wr, part, T, H, m);
    return hipGetLastError();
  }
  const dim3 grid((T + 15) / 16, (m + 15) / 16, sp.ks);
  if (sp.kw == 4)
    route_logits_kernel<4><<<grid, 256, 0, stream>>>(x, wr, part, T, H, m);
  else
    route_logits_kernel<2><<<grid, 128, 0, stream>>>(x, wr, part, T, H, m);
  return hipGetLastError();
}

void launch_topk(const float* part, int KS, const float* bias, const uint8_t* keep_mask, int T,
                 const Cols& c, int* topk_ids, float* topk_w, float* gap, hipStream_t stream) {
  const int blocks = (T + 3) / 4, kpl = (c.m + 63) / 64;
#define SW_TK(KPL)                                                                             \
  route_topk_kernel<KPL><<<blocks, 256, 0, stream>>>(part, KS, bias, keep_mask, T, c, topk_ids, \
                                                     topk_w, gap)
  if (kpl <= 1)
    SW_TK(1);
  else if (kpl <= 2)
    SW_TK(2);
  else if (kpl <= 4)
    SW_TK(4);
  else if (kpl <= 8)
    SW_TK(8);
  else
    SW_TK(16);
#undef SW_TK
}

// ---------------------------------------------------------------------------
// Routing-mass statistics (Section 2.3: an importance criterion aggregating
// the router's gate probabilities over calibration tokens).
//
// Two kernels after the logits.  The first gives every wave a contiguous run
// of tokens: the wave holds one token's logits (lane l experts q * 64 + l),
// selects its top k as the router does, and adds its softmax and its gates
// to per-expert sums in registers; a block adds its waves' sums in wave
// order and writes one row of partial sums.  The second adds the rows, in an
// order that depends on nothing but the shape.  (One thread per expert
// walking all tokens, as this was, is one chain of T dependent exponentials
// on 256 threads of the chip: 1672 us of a 1681 us call at 4096 tokens over
// 256 experts, H 2048.  Now the whole call takes 37 us, 19 of them the logits,
// and needs no dispatch plan.)

constexpr int kMassWaves = 8;        // waves per block of the first kernel
constexpr int kMassTokens = 2;       // tokens a wave takes while blocks are left to give
constexpr int kMassMaxBlocks = 512;  // two per compute unit
constexpr int kMassSumRows = 16;     // row groups of the second kernel

template <int KPL>
__global__ __launch_bounds__(64 * kMassWaves) void mass_partial_kernel(
    const float* __restrict__ part, int KS, const float* __restrict__ bias,
    const uint8_t* __restrict__ keep_mask, int T, int m, int k, bool want_topk,
    float* __restrict__ rows) {
  __shared__ float red[kMassWaves][2][64 * KPL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long n_waves = (long long)gridDim.x * kMassWaves;
  const long long w = (long long)blockIdx.x * kMassWaves + wave;
  const int t_lo = (int)(w * T / n_waves), t_hi = (int)((w + 1) * T / n_waves);
  const Cols c{m, m, k, 0, 1};
  int eid[KPL];
  float soft[KPL], top[KPL];
  wave_experts<KPL>(lane, eid);
#pragma unroll
  for (int q = 0; q < KPL; ++q) soft[q] = top[q] = 0.f;
  const LaneExperts<KPL> x = load_experts<KPL>(c, eid, bias, keep_mask);
  LogitParts<KPL> next = load_logits<KPL>(part, KS, T, c, t_lo, eid);
  for (int t = t_lo; t < t_hi; ++t) {
    const LogitParts<KPL> now = next;
    next = load_logits<KPL>(part, KS, T, c, t + 1, eid);  // read a token ahead
    uint32_t key[KPL], best = 0u;  // order keys (0: ineligible)
    float ex[KPL], sum = 0.f;
    logit_keys<KPL>(now, x, KS, bias != nullptr, key);
#pragma unroll
    for (int q = 0; q < KPL; ++q) best = umax(best, key[q]);
    const float zm = f32_from_order_key(wave_max_u32(best));
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
      ex[q] = key[q] != 0u ? expf(f32_from_order_key(key[q]) - zm) : 0.f;
      sum += ex[q];
    }
    const float denom = wave_sum_f32(sum);
#pragma unroll
    for (int q = 0; q < KPL; ++q)
      if (key[q] != 0u) soft[q] += ex[q] / denom;
    if (want_topk) {  // uniform
      const Selection s = select_topk<KPL>(key, eid, k, lane);
      for (int j = 0; j < k; ++j) {
        const int id = __builtin_amdgcn_readlane(s.id, j);
        const float g =
            __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s.gate), j));
#pragma unroll
        for (int q = 0; q < KPL; ++q) top[q] += eid[q] == id ? g : 0.f;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < KPL; ++q) {
    red[wave][0][eid[q]] = soft[q];
    red[wave][1][eid[q]] = top[q];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * m; i += 64 * kMassWaves) {
    const int which = i >= m ? 1 : 0, e = i - which * m;
    float v = red[0][which][e];
#pragma unroll
    for (int u = 1; u < kMassWaves; ++u) v += red[u][which][e];
    rows[(size_t)blockIdx.x * 2 * m + i] = v;
  }
}

// Adds the partial rows to the masses: first + blockIdx.y 0 the softmax mass, 1
// the top-k mass.  Thread (r, lane) sums rows r, r + kMassSumRows, ... of expert
// blockIdx.x * 64 + lane; the row groups are then added in order.  The top-k
// mass is left alone when fewer than k experts are eligible (every token's
// selection then lacks a slot).
__global__ __launch_bounds__(64 * kMassSumRows) void mass_sum_kernel(
    const float* __restrict__ rows, int n_rows, const uint8_t* __restrict__ keep_mask, int m,
    int k, int first, float* mass_softmax, float* mass_topk) {
  __shared__ float red[kMassSumRows][64];
  const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane, which = first + (int)blockIdx.y;
  float* mass = which == 0 ? mass_softmax : mass_topk;
  if (mass == nullptr) return;  // block-uniform
  int missing = 0;              // pruned experts (of those this thread counts)
  if (keep_mask != nullptr)
    for (int i = threadIdx.x; i < m; i += 64 * kMassSumRows) missing += keep_mask[i] == 0 ? 1 : 0;
  float v = 0.f;
  if (e < m)
    for (int i = r; i < n_rows; i += kMassSumRows)
      v += rows[(size_t)i * 2 * m + (size_t)which * m + e];
  red[r][lane] = v;
  // m <= 64 * kMassSumRows: a thread counts at most one expert
  const int eligible = m - __syncthreads_count(missing);
  if (r != 0 || e >= m || (which == 1 && eligible < k)) return;
  float s = red[0][lane];
#pragma unroll
  for (int u = 1; u < kMassSumRows; ++u) s += red[u][lane];
  if (keep_mask == nullptr || keep_mask[e] != 0) mass[e] += s;
}

}  // namespace

size_t routing_mass_workspace_bytes(int T, int H, int m, int k) {
  if (T <= 0) return 0;
  const size_t P = (size_t)T * k;
  return route_workspace_bytes(T, H, m, k) + 3 * align_up(P * 4, 256) +
         3 * align_up((size_t)(m + 1) * 4, 256) + 256 + 2 * align_up((size_t)T * 4, 256);
}

// Blocks of mass_partial_kernel: kMassTokens tokens a wave until two blocks a
// compute unit, as far as the workspace behind the logits holds their rows
// (at least one: it holds 3 (m + 1) words).
static int mass_blocks(int T, int m, size_t row_bytes) {
  const long want = ((long)T + kMassWaves * kMassTokens - 1) / (kMassWaves * kMassTokens);
  const long fit = (long)(row_bytes / ((size_t)2 * m * sizeof(float)));
  return (int)std::max(1L, std::min({want, fit, (long)kMassMaxBlocks}));
}

hipError_t launch_routing_mass(const uint16_t* x, int T, const float* wr, const float* bias,
                               const uint8_t* keep_mask, int H, int m, int k, float* mass_softmax,
                               float* mass_topk, void* workspace, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  float* part = static_cast<float*>(workspace);
  const size_t logit_bytes = route_workspace_bytes(T, H, m, k);
  float* rows = reinterpret_cast<float*>(static_cast<char*>(workspace) + logit_bytes);
  const int n_rows = mass_blocks(T, m, routing_mass_workspace_bytes(T, H, m, k) - logit_bytes);
  const LogitsSplit sp = logits_split(T, H, m);
  hipError_t err = launch_logits(x, T, wr, H, m, part, sp, stream);
  if (err != hipSuccess) return err;
#define SW_MP(KPL)                                                                             \
  mass_partial_kernel<KPL><<<n_rows, 64 * kMassWaves, 0, stream>>>(                               \
      part, sp.ks, bias, keep_mask, T, m, k, mass_topk != nullptr, rows)
  if (m <= 64)
    SW_MP(1);
  else if (m <= 128)
    SW_MP(2);
  else if (m <= 256)
    SW_MP(4);
  else if (m <= 512)
    SW_MP(8);
  else
    SW_MP(16);
#undef SW_MP
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  // one launch for both masses, unless they are the same array: a block adds to
  // it what it read
  const int both = mass_softmax == mass_topk ? 1 : 2;
  for (int first = 0; first < 2; first += both)
    mass_sum_kernel<<<dim3((m + 63) / 64, both), 64 * kMassSumRows, 0, stream>>>(
        rows, n_rows, keep_mask, m, k, first, mass_softmax, mass_topk);
  return hipGetLastError();
}

// Logit partials, then the chunked dispatch's scratch (used once the
// partials have been read).
static size_t part_bytes(int T, int H, int m) {
  return align_up((size_t)logits_split(T, H, m).ks * T * m * sizeof(float), 256);
}

size_t route_workspace_bytes(int T, int H, int m, int k) {
  if (T <= 0) return 0;
  return part_bytes(T, H, m) + dispatch_workspace_bytes(T * k, m);
}

size_t route_shared_workspace_bytes(int T, int H, int m, int k, int S, int R) {
  if (T <= 0) return 0;
  return part_bytes(T, H, m + 1) + dispatch_workspace_bytes(T * (k + S), m + R * S);
}

namespace {

// Logits of the c.ld router rows, then the top-k over the first c.m.
hipError_t route_cols(const uint16_t* x, int T, const float* wr, const float* bias,
                      const uint8_t* keep_mask, int H, const Cols& c, int* topk_ids,
                      float* topk_w, float* gap, void* workspace, hipStream_t stream) {
  float* part = static_cast<float*>(workspace);
  const LogitsSplit sp = logits_split(T, H, c.ld);
  hipError_t err = launch_logits(x, T, wr, H, c.ld, part, sp, stream);
  if (err != hipSuccess) return err;
  launch_topk(part, sp.ks, bias, keep_mask, T, c, topk_ids, topk_w, gap, stream);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_route(const uint16_t* x, int T, const float* wr, const float* bias,
                        const uint8_t* keep_mask, int H, int m, int k, int* topk_ids,
                        float* topk_w, float* gap, void* workspace, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  return route_cols(x, T, wr, bias, keep_mask, H, Cols{m, m, k, 0, 1}, topk_ids, topk_w, gap,
                    workspace, stream);
}

hipError_t launch_route_select(const uint16_t* x, int T, const float* wr, const float* bias,
                               const uint8_t* keep_mask, int H, int m, int k, int* topk_ids,
                               float* topk_w, float* gap, void* workspace, hipStream_t stream,
                               int n_shared, int n_groups) {
  if (T == 0) return hipSuccess;
  const Cols c{m, n_shared > 0 ? m + 1 : m, k, n_shared, n_shared > 0 ? n_groups : 1};
  return route_cols(x, T, wr, bias, keep_mask, H, c, topk_ids, topk_w, gap, workspace, stream);
}

// Which one-block selection + plan a batch takes: one wave a token, a row of 16
// lanes a token, or none.
enum class Fused { kNone, kWaves, kRows };

static Fused fused_route_dispatch(int T, int m, int k, int S, int R) {
  if (T <= 0 || m + R * S > kFusedMaxPool) return Fused::kNone;
  if (T <= kFusedMaxTokens && T * (k + S) <= kFusedMaxPairs) return Fused::kWaves;
  return T <= kRowFusedTokens && k + S <= kRowFusedMaxK && m <= kRowFusedMaxPool ? Fused::kRows
                                                                                 : Fused::kNone;
}

hipError_t launch_route_dispatch(const uint16_t* x, int T, const float* wr, const float* bias,
                                 const uint8_t* keep_mask, int H, int m, int k, int* topk_ids,
                                 float* topk_w, float* gap, int* counts, int* offsets, int* perm,
                                 int* active, int* n_active, void* workspace, hipStream_t stream,
                                 int n_shared, int n_groups) {
  const Cols c{m, n_shared > 0 ? m + 1 : m, k, n_shared, n_shared > 0 ? n_groups : 1};
  const int kout = k + n_shared, m_plan = c.plan_m();
  const Fused fused = fused_route_dispatch(T, m, k, n_shared, c.R);
  if (fused == Fused::kNone) {
    if (T > 0) {
      hipError_t err = route_cols(x, T, wr, bias, keep_mask, H, c, topk_ids, topk_w, gap,
                                  workspace, stream);
      if (err != hipSuccess) return err;
    }
    return launch_dispatch(topk_ids, T * kout, m_plan, counts, offsets, perm, active, n_active,
                           stream, static_cast<char*>(workspace) + part_bytes(T, H, c.ld));
  }
  float* part = static_cast<float*>(workspace);
  const LogitsSplit sp = logits_split(T, H, c.ld);
  hipError_t err = launch_logits(x, T, wr, H, c.ld, part, sp, stream);
  if (err != hipSuccess) return err;
#define SW_FR(KPL)                                                                             \
  route_select_dispatch_rows_kernel<KPL><<<1, kRowFusedThreads, 0, stream>>>(                    \
      part, sp.ks, bias, keep_mask, T, c, topk_ids, topk_w, gap, counts, offsets, perm, active,   \
      n_active)
  if (fused == Fused::kRows) {
    if (m <= 16)
      SW_FR(1);
    else if (m <= 32)
      SW_FR(2);
    else
      SW_FR(4);
    return hipGetLastError();
  }
#undef SW_FR
  const int kpl = (m + 63) / 64;
#define SW_FD(KPL)                                                                             \
  route_select_dispatch_kernel<KPL><<<1, 64 * T, 0, stream>>>(                                    \
      part, sp.ks, bias, keep_mask, T, c, topk_ids, topk_w, gap, counts, offsets, perm, active,   \
      n_active)
  if (kpl <= 1)
    SW_FD(1);
  else if (kpl <= 2)
    SW_FD(2);
  else
    SW_FD(4);
#undef SW_FD
  return hipGetLastError();
}

}  // namespace sw
