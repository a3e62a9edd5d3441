// Expert FFN kernels for prefill-sized batches on gfx950 (Section 2.1: with
// many tokens per expert the layer reuses each weight across those tokens,
// so the step turns from weight streaming toward MFMA work).
//
// The decode kernels keep an expert's tokens in LDS over the whole
// contraction and stream each 16-row tile once per 32-token pass; with
// ~128 tokens per expert that would re-stream every weight four times.
// Here the loop order is inverted:
//   - a unit is (active expert, group of 16 row tiles); a persistent grid of
//     one 8-wave block per compute unit walks the units, each XCD taking a
//     contiguous run of every round's units (an expert's units then share one
//     L2 for its gathered activations);
//   - a pass covers up to 160 of the expert's tokens (10 MFMA column
//     blocks), so a unit streams its weights once per pass, normally once.
//     Wave w computes row tiles 4 (w % 4) .. + 3 for half of the pass's column
//     blocks (w / 4), so an operand read from LDS feeds 4 or 5 MFMAs;
//   - the contraction runs in chunks of 32 or 64 columns.  Weights and
//     activations both go straight from memory into an LDS ring (buffer loads
//     with the LDS bit) that runs some chunks ahead of the one computed.  Such
//     a load holds no register and no wait of the compiler's, so the ring runs
//     on across the end of a pass: the last chunks of one
//     pass are computed, and its results stored, while the first chunks of
//     the next (its expert, pairs and rows looked up a few chunks earlier)
//     are already on their way.
// (The down projection of long tiled rows is a kernel of another form, below.)
// Each output accumulates over K in the same order as the decode kernels,
// except where the rows of a row-major w13 are a multiple of 4 KiB apart.
//
// What bounds it (4096 tokens, 256 experts, H 2048, I 512, top-8: 137 GFLOP of
// gate/up products, 137 of down's over two planes, 1.07 and 0.54 GB of weights):
// memory.  With the MFMAs and operand reads left out gate/up takes 210 of its
// 228 us (1.28 GB at 6.1 TB/s) and down 198 of its 204 (0.61 GB read, 0.27
// written); with the loads left out 134 and 101.  1531 row-major tokens over 128
// experts of I 768: 167 of 170 and 128 of 129.
// Before, the weights came through registers one 64-column chunk ahead, two
// row tiles a wave (an LDS operand fed two MFMAs), each pass began with an
// empty pipeline and results were stored a token per lane.  Before -> now, kernel
// traces at 4096 tokens: gate/up 234 -> 225 us, down 208 -> 200, the reduction
// that reads its results 52 -> 48 (whole lines written: down wrote 297 MB for
// 268).  1531 row-major tokens: gate/up 206 -> 170, down 137 -> 129.
#include <type_traits>

#include "sw_device.h"
#include "sw_launch.h"

namespace sw {
namespace {

constexpr int kWv = 8;                    // waves per block
constexpr int kBlk = 64 * kWv;            // threads per block
constexpr int kTpw = 4;                   // 16-row tiles per wave
constexpr int kRowGroups = 4;             // waves w % 4: row tiles
constexpr int kColGroups = kWv / kRowGroups;  // waves w / 4: column blocks
constexpr int kTpu = kTpw * kRowGroups;   // tiles per unit
constexpr int kMaxNb = 5;                 // 16-token column blocks of a wave
constexpr int kNT = 16 * kMaxNb * kColGroups;  // tokens per pass
constexpr int kFrag = 512;                // 16-bit words of a fragment: 16 rows x 32 columns
static_assert(kTpu % kWv == 0, "whole rounds of weight loads");

// A staged fragment holds 16 rows of 64 bytes (one 1 KiB load of a wave, four
// consecutive lanes a row); the four 16-byte pieces of a row sit in swizzled
// places, so that a 16-lane phase of a 128-bit LDS read (rows 0-3 and 12-15 of
// one piece, rows 4-11 of the next k-group's) hits distinct banks.  The
// swizzle is its own inverse.
__device__ __forceinline__ int place(int row, int piece) { return piece ^ (((row >> 3) & 1) * 3); }

// One pass of a unit: (expert, 16 row tiles) x (up to kNT of its pairs).
struct Pass {
  int e, grp, base, cnt, p0;
  int nb;  // column blocks a wave computes: the pass's tokens, split over the column groups
};

// The passes of one block, in order.  The plan is read in three steps that
// the caller spreads over chunks: each is one round trip to memory.
struct PassWalk {
  const int *active, *counts, *offsets;
  int m, n_pairs, n_units, gpe, step;
  int u;     // unit of `next`
  Pass next;
  bool more;  // `next` is a pass of this block

  __device__ __forceinline__ void set_blocks() {
    const int n = min(kNT, next.cnt - next.p0);
    next.nb = (n + 16 * kColGroups - 1) / (16 * kColGroups);
  }
  // 1: the following pass of the unit, or the next unit's expert
  __device__ __forceinline__ void expert_of(const Pass& cur, bool first) {
    next = cur;
    more = true;
    if (!first && cur.p0 + kNT < cur.cnt) {
      next.p0 = cur.p0 + kNT;
      return;
    }
    if (!first) u += step;
    next.p0 = 0;
    next.cnt = 0;
    more = u < n_units;
    if (!more) return;
    const int a = u / gpe;
    next.grp = u - a * gpe;
    next.e = active[a];
  }
  // 2: its pairs
  __device__ __forceinline__ void pairs_of() {
    if (!more || next.p0 > 0) return;
    const bool ok = next.e >= 0 && next.e < m;
    next.cnt = ok ? counts[next.e] : 0;
    next.base = ok ? offsets[next.e] : 0;
  }
  // 3: checked against the plan's bounds; units without valid pairs are
  // skipped (here without spreading: a plan of the dispatch has none)
  __device__ __forceinline__ void check() {
    if (!more) return;
    while (next.p0 == 0 &&
           !(next.cnt > 0 && next.base >= 0 && next.cnt <= n_pairs - next.base)) {
      u += step;
      if (u >= n_units) {
        more = false;
        return;
      }
      const int a = u / gpe;
      next.grp = u - a * gpe;
      next.e = active[a];
      pairs_of();
    }
    set_blocks();
  }
};

// Slot of block b in each round of gridDim.x units.  Blocks are dispatched
// round-robin over the eight XCDs (block b runs on XCD b % 8); giving each
// XCD a contiguous run of the round's units puts the units of one expert
// (consecutive in the list) on one XCD at the same time, so they share that
// XCD's L2 for the expert's gathered activations.
__device__ __forceinline__ int unit_slot() {
  const int b = blockIdx.x, g = gridDim.x;
  return (g & 7) ? b : (b & 7) * (g >> 3) + (b >> 3);
}

// Waits until at most n of this wave's vector-memory operations are
// outstanding and its LDS accesses are done.  The instruction takes a
// constant: n is one of a few values, tried in turn.
template <int N>
__device__ __forceinline__ void wait_exactly() {
  static_assert(N >= 0 && N < 64, "six bits of vmcnt");
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most_lds_done(N));
}

// n = lo .. lo + kCount - 1 in steps of kStep (uniform; above: as the last).
template <int kLo, int kStep, int kCount>
__device__ __forceinline__ void wait_one_of(int n) {
  if constexpr (kCount == 1) {
    wait_exactly<kLo>();
  } else {
    if (n <= kLo)
      wait_exactly<kLo>();
    else
      wait_one_of<kLo + kStep, kStep, kCount - 1>(n);
  }
}

// Pair ids of walk.next's tokens, straight into LDS (one load of a few waves).
constexpr int kPidWords = (kNT + 63) / 64 * 64;
__device__ __forceinline__ void load_pids(u32x4 perm, const PassWalk& walk, int wave, int lane,
                                          int* dst) {
  if (wave * 64 < kNT) {  // wave-uniform
    const int i = wave * 64 + lane, s = walk.next.p0 + i;
    load_lds4(perm,
              i < kNT && s < walk.next.cnt ? (uint32_t)(walk.next.base + s) * 4u : kOutOfRange,
              lds_address(dst + wave * 64));
  }
}

// This wave's LDS accesses are done; past the barrier so are every wave's.
__device__ __forceinline__ void pass_barrier() {
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most_lds_done(63));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");  // (no LDS read moves above it)
}

__device__ __forceinline__ void landed_barrier() {
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));
  pass_barrier();
}

// The chunk's MFMAs, in the K order of every output.
template <int NB>
__device__ __forceinline__ void chunk_mfmas(const u32x4 (&a)[kTpw], const u32x4 (&b)[NB],
                                            f32x4 (&acc)[kTpw][NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int t = 0; t < kTpw; ++t) acc[t][nb] = mfma_16x16x32(a[t], b[nb], acc[t][nb]);
}

// A wave's operands of one MFMA step: 4 row tiles, NB column blocks.
template <int NB>
struct Operands {
  u32x4 a[kTpw], b[NB];
};

// gate/up's activations of a chunk are 4 loads of 1 KiB for every column block
// of a wave, dealt out over the 8 waves in rounds; an odd number of blocks leaves
// half a round, which the other half repeats, so that every wave issues the
// same number.
__host__ __device__ constexpr int act_loads(int nb) { return (4 * nb + kWv - 1) / kWv; }
constexpr int kMaxActLoads = act_loads(kMaxNb);
__device__ __forceinline__ int act_load(int nb, int wave, int j) {
  const int f = wave + j * kWv;
  return f < 4 * nb ? f : f - 4;
}

template <typename F>
__device__ __forceinline__ void with_blocks(int nb, F&& f) {
  switch (nb) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 5>{}); break;
  }
}

// ---------------------------------------------------------------------------
// gate/up + SwiGLU
//
// A chunk is 64 columns (two MFMA steps), the ring three slots.  The one
// barrier of a chunk sits between its two steps: by then every wave has read
// the chunk's operands, so its slot takes the chunk three ahead, and the next
// chunk, which has landed, gives its first step's operands during the MFMAs of
// the second.  (One step a chunk and barrier, in a ring of four: 249 us at 4096
// tokens.  With the waits for loads chosen inside one loop over the chunks, and
// the first step's MFMAs waiting for the second's LDS reads too: 265.)  The
// number of loads a wave issues for a chunk is the same for every wave and a
// constant of the pass, so the loop over the chunks has one wait and no branch.

constexpr int kGuCols = 64, kGuSteps = kGuCols / 32, kGuSlots = 3;
constexpr int kGuTile = 16 * kGuCols;                       // words of a tile's chunk
constexpr int kGuX = kTpu * kGuTile;                        // the slot's x rows start here
constexpr int kGuSlot = kGuX + kNT * kGuCols;               // words
constexpr int kGuW = kTpu * kGuSteps / kWv;                 // weight loads a wave and chunk
constexpr int kGuOverlap = 8;  // chunks from which a pass looks up and stages the next one
static_assert(kWv * 2 * kFrag <= kGuSlot, "a slot holds the waves' result transpositions");

template <bool kTiled>
__global__ __launch_bounds__(kBlk, 1) void gate_up_prefill_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w13,
    const int* __restrict__ counts, const int* __restrict__ offsets,
    const int* __restrict__ perm, const int* __restrict__ active,
    const int* __restrict__ n_active, uint16_t* __restrict__ h_hi, uint16_t* __restrict__ h_lo,
    int H, int I, int m, int k, int n_pairs) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kGuSlots * kGuSlot];
  __shared__ int pids_s[2][kPidWords];  // pair ids of the pass and the next
  const int n_act = *n_active;
  if (n_act <= 0 || n_act > m) return;
  const int lane_id = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int tpe = I / 8;                           // tiles per expert: 8 gate and 8 up rows each
  const int n = H / kGuCols;                       // chunks, at least 2
  const uint32_t w_bytes = 4u * (uint32_t)I * (uint32_t)H;
  const u32x4 x_r = rsrc_words(x, 2u * (uint32_t)(n_pairs / k) * (uint32_t)H);
  const u32x4 perm_r = rsrc_words(perm, 4u * (uint32_t)n_pairs);
  PassWalk walk{active, counts, offsets, m, n_pairs, n_act * ((tpe + kTpu - 1) / kTpu),
                (tpe + kTpu - 1) / kTpu, (int)gridDim.x, unit_slot(), {}, false};

  // What is staged: the pass's weights, and source offsets at chunk 0 (out of
  // range stays out of range for every chunk: at most a row is added to 2^31).
  // Staged rows have 128 bytes, their 16-byte pieces in places row_place;
  // tiled weights keep their fragments.
  auto row_place = [](int row, int piece) { return piece ^ (row & 7); };
  u32x4 w_r;
  // Row-major rows of a multiple of 4 KiB have a column of every row in the
  // same few memory and L2 channels, and blocks in step read the same column:
  // there the unit's contraction starts grp / gpe into the row and wraps, so
  // that the units of an expert read different channels.  (H 2048: 1531 tokens
  // over 128 experts, I 768, 202 -> 170 us; 4096 over 256, I 512, 294 -> 262.
  // H 1920 as before 159, against 153 tiled; H 1024 no faster with it.)
  const bool wrap = !kTiled && H % 2048 == 0;
  int first = 0;  // the chunk of the row that the pass takes first
  uint32_t w_off[kGuW], x_off[kMaxActLoads];
  auto stage_from = [&](const Pass& s, const int* pids) {
    int lane = lane_id;
    asm volatile("" : "+v"(lane));  // (nothing of this is kept across passes)
    const int l_row = lane >> 3, l_piece = row_place(l_row, lane & 7);
    w_r = rsrc_words(w13 + (size_t)s.e * 2 * I * H, w_bytes);
    first = wrap ? s.grp * n / walk.gpe : 0;
#pragma unroll
    for (int j = 0; j < kGuW; ++j) {
      // load f = wave + 8 j: half f % 2 of tile f / 2 -- a fragment, or rows
      const int f = wave + j * kWv, tile = s.grp * kTpu + f / 2;
      if (kTiled)
        w_off[j] = (uint32_t)tile * 32u * (uint32_t)H + (uint32_t)(f % 2) * 1024u +
                   (uint32_t)lane * 16u;
      else  // the 8 gate rows, the 8 up rows
        w_off[j] = ((uint32_t)((f % 2) * I + tile * 8 + l_row) * (uint32_t)H +
                    (uint32_t)l_piece * 8u) * 2u;
      if (tile >= tpe) w_off[j] = kOutOfRange;
    }
#pragma unroll
    for (int j = 0; j < kMaxActLoads; ++j) {
      const int row = act_load(s.nb, wave, j) * 8 + l_row, sl = s.p0 + row;
      const int q = row < kNT ? pids[row] : -1;
      x_off[j] = row < kNT && sl < s.cnt && q >= 0 && q < n_pairs
                     ? ((uint32_t)(q / k) * (uint32_t)H + (uint32_t)l_piece * 8u) * 2u
                     : kOutOfRange;
    }
  };
  const uint32_t ring_at = lds_address(ring);
  constexpr uint32_t kSlotBytes = kGuSlot * 2;
  auto next_slot = [](uint32_t q) {
    return q + kSlotBytes == kGuSlots * kSlotBytes ? 0u : q + kSlotBytes;
  };
  // chunk c of a pass with nb column blocks into the slot at byte q
  auto stage = [&](auto nbc, int c, uint32_t q) {
    constexpr int NB = decltype(nbc)::value;
    const uint32_t at = ring_at + q + (uint32_t)wave * 1024u;
    if (!kTiled) {
      c += first;
      if (c >= n) c -= n;
    }
    const uint32_t wc = (uint32_t)c * (kTiled ? 2048u : 128u), xc = (uint32_t)c * 128u;
    for_each_index<kGuW>([&](auto j) {
      load_lds16<decltype(j)::value * kWv * 1024, kTiled>(w_r, w_off[decltype(j)::value], wc, at);
    });
    // (the last round of an odd number of blocks repeats its first half)
    for_each_index<act_loads(NB)>([&](auto j) {
      constexpr int J = decltype(j)::value;
      constexpr bool kRepeat = (J + 1) * kWv > 4 * NB;
      const uint32_t back = kRepeat ? (uint32_t)(wave & 4) * 1024u : 0u;
      load_lds16<kGuX * 2 + J * kWv * 1024>(x_r, x_off[J], xc, at - back);
    });
  };
  auto stage_next = [&](int c, uint32_t q) {
    with_blocks(walk.next.nb, [&](auto nbc) { stage(nbc, c, q); });
  };

  Pass cur{0, 0, 0, 0, 0, 0};
  int half = 0;        // the pass's half of pids_s
  uint32_t q = 0;      // slot of the chunk being computed, in bytes
  int stored = 0;      // result stores of the last pass, by this wave (0: all waited for)
  const bool overlap = n >= kGuOverlap;
  // from an empty pipeline: the first pass, and every one of a short K
  auto fill = [&]() {
    landed_barrier();
    stored = 0;
    stage_from(walk.next, pids_s[half]);
    stage_next(0, q);
    stage_next(1, next_slot(q));
  };
  walk.expert_of(cur, true);
  walk.pairs_of();
  walk.check();
  if (!walk.more) return;
  load_pids(perm_r, walk, wave, lane_id, pids_s[half]);
  fill();
  cur = walk.next;

  auto run_pass = [&](auto nbc) {
    constexpr int NB = decltype(nbc)::value;
    constexpr int kLoads = kGuW + act_loads(NB);  // a wave's loads of a chunk
    int lane = lane_id;
    asm volatile("" : "+v"(lane));  // (the addresses of the five widths are not kept)
    const int r = lane & 15, kg = lane >> 4;
    f32x4 acc[kTpw][NB];
#pragma unroll
    for (int t = 0; t < kTpw; ++t)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    int w_at[kGuSteps], x_at[kGuSteps];  // operand places in a slot (bytes), per step
#pragma unroll
    for (int st = 0; st < kGuSteps; ++st) {
      const int pl = row_place(r, st * 4 + kg) * 8;
      w_at[st] = 2 * ((wave % kRowGroups) * kTpw * kGuTile +
                      (kTiled ? st * kFrag + lane * 8 : r * kGuCols + pl));
      x_at[st] = 2 * (kGuX + ((wave / kRowGroups) * NB * 16 + r) * kGuCols + pl);
    }
    auto read = [&](Operands<NB>& o, uint32_t slot, auto stc) {
      constexpr int st = decltype(stc)::value;
      const char* wb = reinterpret_cast<const char*>(ring) + (slot + (uint32_t)w_at[st]);
      const char* xb = reinterpret_cast<const char*>(ring) + (slot + (uint32_t)x_at[st]);
#pragma unroll
      for (int t = 0; t < kTpw; ++t)
        o.a[t] = *reinterpret_cast<const u32x4*>(wb + t * kGuTile * 2);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        o.b[nb] = *reinterpret_cast<const u32x4*>(xb + nb * 16 * kGuCols * 2);
      __builtin_amdgcn_sched_barrier(0);  // on their way during the MFMAs that follow
    };
    // waits until only one chunk's loads, and the last pass's result stores,
    // are outstanding
    auto wait_past_stores = [&]() {
      wait_one_of<kLoads, 2, kMaxNb + 1>(kLoads + stored);
    };

    // Chunk 0 landed: after its loads came chunk 1's and the last pass's
    // stores.  Past the barrier no wave reads the last pass's results from
    // the slot that chunk 2 takes.
    wait_past_stores();
    pass_barrier();
    if (2 < n) stage(nbc, 2, next_slot(next_slot(q)));
    Operands<NB> o0, o1;
    read(o0, q, std::integral_constant<int, 0>{});
    // One chunk: the MFMAs of its two steps, `between` (the wait for the next
    // chunk, the barrier after which every wave has this chunk's operands, and
    // what is staged into its slot) between them.
    auto chunk = [&](auto last, auto&& between) {
      constexpr bool kLast = decltype(last)::value;
      // step 0's operands have arrived (during the previous MFMAs); said here,
      // so that their MFMAs do not wait for step 1's
      __builtin_amdgcn_s_waitcnt(vmcnt_at_most_lds_done(63));
      read(o1, q, std::integral_constant<int, 1>{});
      chunk_mfmas<NB>(o0.a, o0.b, acc);
      between();
      if constexpr (!kLast) {
        const uint32_t nq = next_slot(q);
        read(o0, nq, std::integral_constant<int, 0>{});
        q = nq;
      }
      chunk_mfmas<NB>(o1.a, o1.b, acc);
    };
    using No = std::false_type;
    using Yes = std::true_type;
    if (overlap) {
      // The next pass is looked up in two steps; its pair ids land before
      // chunk 4, so before they are used at the earliest (chunk n - 3).  Chunk
      // c + 1 has landed when only chunk c + 2's loads (for c = 0 also the
      // stores before them) are outstanding.
      chunk(No{}, [&]() {
        wait_past_stores();
        pass_barrier();
        walk.expert_of(cur, false);
        stage(nbc, 3, q);
      });
      chunk(No{}, [&]() {
        wait_exactly<kLoads>();
        pass_barrier();
        walk.pairs_of();
        walk.check();
        if (walk.more) load_pids(perm_r, walk, wave, lane_id, pids_s[half ^ 1]);
        stage(nbc, 4, q);
      });
      for (int c = 2; c + 3 < n; ++c)
        chunk(No{}, [&]() {
          wait_exactly<kLoads>();
          pass_barrier();
          stage(nbc, c + 3, q);
        });
      chunk(No{}, [&]() {
        wait_exactly<kLoads>();
        pass_barrier();
        if (walk.more) {
          stage_from(walk.next, pids_s[half ^ 1]);
          stage_next(0, q);
        }
      });
      chunk(No{}, [&]() {
        if (walk.more)
          wait_one_of<kGuW + 1, 1, kMaxActLoads>(kGuW + act_loads(walk.next.nb));
        else
          wait_exactly<0>();
        pass_barrier();
        if (walk.more) stage_next(1, q);
      });
    } else {
      for (int c = 0; c + 1 < n; ++c)
        chunk(No{}, [&]() {
          if (c + 2 < n)
            wait_exactly<kLoads>();
          else
            wait_exactly<0>();
          pass_barrier();
          if (c == 0) walk.expert_of(cur, false);
          if (c + 3 < n) stage(nbc, c + 3, q);
        });
    }
    // (the last chunk's slot carries the results; the next pass's chunk 2
    // follows them)
    chunk(Yes{}, [&]() {
      pass_barrier();
      if (!overlap) {
        walk.pairs_of();
        walk.check();
        if (walk.more) load_pids(perm_r, walk, wave, lane_id, pids_s[half ^ 1]);
      }
    });

    // SwiGLU of two tiles at a time, so that every lane finishes an output:
    // lanes 0-31 hold tile a's gates and lanes 32-63 its ups (likewise for
    // tile b); one exchange across the halves hands lanes 0-31 a's ups and
    // lanes 32-63 b's gates.  The 32 outputs of a token then pass through the
    // wave's part of the free slot, so that four consecutive lanes store 64
    // consecutive bytes of it (a store with a token per lane costs the address
    // path a cycle a lane).
    uint16_t* trans = ring + q / 2 + wave * 2 * kFrag;
    const int tile0 = cur.grp * kTpu + (wave % kRowGroups) * kTpw;
    const int blk0 = (wave / kRowGroups) * NB;
    const uint32_t hbytes = 2u * (uint32_t)cur.cnt * (uint32_t)I;
    const auto hh = make_rsrc(h_hi + (size_t)cur.base * I, hbytes);
    const auto hl = make_rsrc(h_lo + (size_t)cur.base * I, hbytes);
    const int up = lane >> 5, kgx = kg & 1;
    const int l_row = lane >> 2, l_piece = place(l_row, lane & 3);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int t = 0; t < kTpw; t += 2) {
        f32x4 g4, u4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = acc[t][nb][i], b = acc[t + 1][nb][i];
          const float z = __shfl_xor(up ? a : b, 32);  // lanes < 32: a's up; else b's gate
          g4[i] = up ? z : a;
          u4[i] = up ? b : z;
        }
        float hv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) hv[i] = swiglu(g4[i], u4[i]);
        u32x2 hw, lw;
        split_bf16x4(hv, hw, lw);
        uint16_t* at = trans + (r * 4 + place(r, t + up)) * 8 + kgx * 4;
        *reinterpret_cast<u32x2*>(at) = hw;
        *reinterpret_cast<u32x2*>(at + kFrag) = lw;
      }
      const u32x4 vh = *reinterpret_cast<const u32x4*>(trans + lane * 8);
      const u32x4 vl = *reinterpret_cast<const u32x4*>(trans + kFrag + lane * 8);
      const int sl = cur.p0 + (blk0 + nb) * 16 + l_row, tile = tile0 + l_piece;
      const uint32_t off =
          sl < cur.cnt && tile < tpe ? ((uint32_t)sl * I + (uint32_t)tile * 8u) * 2u : kOutOfRange;
      __builtin_amdgcn_raw_buffer_store_b128(vh, hh, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(vl, hl, off, 0, 0);
    }
    stored = 2 * NB;
    q = next_slot(q);
  };
  for (;;) {
    with_blocks(cur.nb, run_pass);
    if (!walk.more) break;
    half ^= 1;
    if (!overlap) fill();  // (past its barrier every wave is done with the results' slot)
    cur = walk.next;
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));
}

// ---------------------------------------------------------------------------
// down projection
//
// A chunk is one MFMA step (32 columns) of the weights and of both h planes,
// the ring four slots.  A chunk's weight and hi operands are in registers
// before its turn; the lo plane is read in its turn, during the hi plane's
// MFMAs (both planes a chunk ahead take more registers than there are).  As in
// gate/up a wave issues the same number of loads for every chunk of a pass:
// waves 0-3 stage the hi plane and waves 4-7 the lo plane.  (With the fragments
// dealt over all waves and the waits chosen at run time, 4 to 9% slower for 150
// and more row-major tokens an expert.  With 64 columns a chunk in two slots:
// 0 to 9% faster from 128 tokens an expert on, but up to 12% slower at 48 and
// fewer, where a chunk's loads have nothing in flight behind them.)

constexpr int kDnSlots = 4, kDnAhead = kDnSlots - 1;
constexpr int kDnPlane = kNT * 32;                          // words of a staged plane
constexpr int kDnSlot = kTpu * kFrag + 2 * kDnPlane;
constexpr int kDnW = kTpu / kWv;                            // weight loads a wave and chunk

// A plane's 1 KiB fragments (two for every column block of a wave), dealt out
// over the plane's 4 waves; an odd number of blocks repeats half a round.
constexpr int kPlaneWaves = kWv / 2;
__host__ __device__ constexpr int plane_loads(int nb) {
  return (kColGroups * nb + kPlaneWaves - 1) / kPlaneWaves;
}
constexpr int kMaxPlaneLoads = plane_loads(kMaxNb);
static_assert(kColGroups == 2 && kPlaneWaves == 4, "half a round is two fragments");

template <bool kTiled>
__global__ __launch_bounds__(kBlk, 1) void down_prefill_kernel(
    const uint16_t* __restrict__ h_hi, const uint16_t* __restrict__ h_lo,
    const uint16_t* __restrict__ w2, const int* __restrict__ counts,
    const int* __restrict__ offsets, const int* __restrict__ perm,
    const int* __restrict__ active, const int* __restrict__ n_active, float* __restrict__ y, int H,
    int I, int m, int n_pairs) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kDnSlots * kDnSlot];
  __shared__ __attribute__((aligned(1024))) uint16_t trans_s[kWv * kFrag];
  __shared__ int pids_s[2][kPidWords];  // pair ids of the pass and the next
  const int n_act = *n_active;
  if (n_act <= 0 || n_act > m) return;
  const int lane_id = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int plane = wave / kPlaneWaves, plane_wave = wave % kPlaneWaves;
  const int tpe = H / 16;                          // tiles per expert: 16 output rows each
  const int n = I / 32;                            // chunks, a multiple of kDnSlots
  const uint32_t w_bytes = 2u * (uint32_t)H * (uint32_t)I;
  const u32x4 h_r = rsrc_words(plane ? h_lo : h_hi, 2u * (uint32_t)n_pairs * (uint32_t)I);
  const u32x4 perm_r = rsrc_words(perm, 4u * (uint32_t)n_pairs);
  uint16_t* trans = trans_s + wave * kFrag;
  PassWalk walk{active, counts, offsets, m, n_pairs, n_act * ((tpe + kTpu - 1) / kTpu),
                (tpe + kTpu - 1) / kTpu, (int)gridDim.x, unit_slot(), {}, false};

  // what is staged (as for gate/up); the h rows are the expert's dispatch
  // slots, so they need no pair ids
  u32x4 w_r;
  uint32_t w_off[kDnW], h_off[kMaxPlaneLoads];
  auto stage_from = [&](const Pass& s) {
    int lane = lane_id;
    asm volatile("" : "+v"(lane));
    const int l_row = lane >> 2, l_piece = place(l_row, lane & 3);
    w_r = rsrc_words(w2 + (size_t)s.e * H * I, w_bytes);
#pragma unroll
    for (int j = 0; j < kDnW; ++j) {
      const int tile = s.grp * kTpu + wave + j * kWv;
      w_off[j] = kTiled ? (uint32_t)tile * 32u * (uint32_t)I + (uint32_t)lane * 16u
                        : ((uint32_t)(tile * 16 + l_row) * (uint32_t)I + (uint32_t)l_piece * 8u) * 2u;
      if (tile >= tpe) w_off[j] = kOutOfRange;
    }
#pragma unroll
    for (int j = 0; j < kMaxPlaneLoads; ++j) {
      const int f = plane_wave + j * kPlaneWaves, blocks = kColGroups * s.nb;
      const int sl = s.p0 + (f < blocks ? f : f - 2) * 16 + l_row;
      h_off[j] = sl < s.cnt
                     ? ((uint32_t)(s.base + sl) * (uint32_t)I + (uint32_t)l_piece * 8u) * 2u
                     : kOutOfRange;
    }
  };
  const uint32_t ring_at = lds_address(ring);
  constexpr uint32_t kSlotBytes = kDnSlot * 2;
  auto next_slot = [](uint32_t q) {
    return q + kSlotBytes == kDnSlots * kSlotBytes ? 0u : q + kSlotBytes;
  };
  auto slot_before = [](uint32_t q) {
    return q == 0 ? (kDnSlots - 1) * kSlotBytes : q - kSlotBytes;
  };
  // chunk c of a pass with nb column blocks into the slot at byte q
  auto stage = [&](auto nbc, int c, uint32_t q) {
    constexpr int NB = decltype(nbc)::value;
    const uint32_t at = ring_at + q;
    const uint32_t wc = (uint32_t)c * (kTiled ? 1024u : 64u), hc = (uint32_t)c * 64u;
    const uint32_t h_at = at + (uint32_t)(plane * kDnPlane * 2 + plane_wave * 1024);
    for_each_index<plane_loads(NB)>([&](auto j) {
      constexpr int J = decltype(j)::value;
      constexpr bool kRepeat = (J + 1) * kPlaneWaves > kColGroups * NB;
      const uint32_t back = kRepeat ? (uint32_t)(plane_wave & 2) * 1024u : 0u;
      load_lds16<kTpu * kFrag * 2 + J * kPlaneWaves * 1024>(h_r, h_off[J], hc, h_at - back);
    });
    for_each_index<kDnW>([&](auto j) {
      load_lds16<decltype(j)::value * kWv * 1024, kTiled>(w_r, w_off[decltype(j)::value], wc,
                                                          at + (uint32_t)wave * 1024u);
    });
  };
  auto stage_next = [&](int c, uint32_t q) {
    with_blocks(walk.next.nb, [&](auto nbc) { stage(nbc, c, q); });
  };

  Pass cur{0, 0, 0, 0, 0, 0};
  walk.expert_of(cur, true);
  walk.pairs_of();
  walk.check();
  if (!walk.more) return;
  int half = 0;    // the pass's half of pids_s
  int stored = 0;  // result stores of the last pass, by this wave
  load_pids(perm_r, walk, wave, lane_id, pids_s[0]);
  landed_barrier();
  cur = walk.next;
  stage_from(cur);
#pragma unroll
  for (int c = 0; c < kDnAhead; ++c) stage_next(c, (uint32_t)c * kSlotBytes);

  auto run_pass = [&](auto nbc) {
    constexpr int NB = decltype(nbc)::value;
    constexpr int kLoads = kDnW + plane_loads(NB);  // a wave's loads of a chunk
    int lane = lane_id;
    asm volatile("" : "+v"(lane));  // (the addresses of the five widths are not kept)
    const int r = lane & 15, kg = lane >> 4;
    f32x4 acc[kTpw][NB];
#pragma unroll
    for (int t = 0; t < kTpw; ++t)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int at = (r * 4 + place(r, kg)) * 16;  // operand places in a slot (bytes)
    const int w_at = (wave % kRowGroups) * kTpw * kFrag * 2 + (kTiled ? lane * 16 : at);
    const int h_at = (kTpu + (wave / kRowGroups) * NB) * kFrag * 2 + at;
    auto read = [&](Operands<NB>& o, uint32_t slot) {
      const char* wb = reinterpret_cast<const char*>(ring) + (slot + (uint32_t)w_at);
      const char* hb = reinterpret_cast<const char*>(ring) + (slot + (uint32_t)h_at);
#pragma unroll
      for (int t = 0; t < kTpw; ++t) o.a[t] = *reinterpret_cast<const u32x4*>(wb + t * kFrag * 2);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        o.b[nb] = *reinterpret_cast<const u32x4*>(hb + nb * kFrag * 2);
    };
    uint32_t q = 0;  // slot of the chunk being computed, in bytes
    // One chunk: `before` ends with the barrier past which the next chunk has
    // landed and the slot before this one is free, and stages into that slot.
    auto chunk = [&](const Operands<NB>& o, Operands<NB>& ahead, auto last, auto&& before) {
      before();
      u32x4 lo[NB];
      const char* lb = reinterpret_cast<const char*>(ring) + (q + (uint32_t)h_at + kDnPlane * 2);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) lo[nb] = *reinterpret_cast<const u32x4*>(lb + nb * kFrag * 2);
      q = next_slot(q);
      if constexpr (!decltype(last)::value) read(ahead, q);
      __builtin_amdgcn_sched_barrier(0);  // on their way during the MFMAs
      chunk_mfmas<NB>(o.a, o.b, acc);
      chunk_mfmas<NB>(o.a, lo, acc);
    };
    using No = std::false_type;
    using Yes = std::true_type;
    Operands<NB> o0, o1;
    // Chunk 0 landed: after its loads came those of two more chunks, then the
    // last pass's stores.
    wait_one_of<2 * kLoads, kTpw, kMaxNb + 1>(2 * kLoads + stored);
    pass_barrier();
    read(o0, q);
    // Chunk c + 1 has landed when only chunk c + 2's loads (for c < 2 also the
    // stores before or between them) are outstanding.  The next pass is looked
    // up in chunks 0 and 1, or at once in a pass of four chunks, whose chunk 1
    // already stages the next pass's first; its pair ids are used in its own
    // epilogue, many chunks later.
    const bool short_pass = n == kDnSlots;
    auto look_up = [&]() {
      walk.pairs_of();
      walk.check();
      if (walk.more) load_pids(perm_r, walk, wave, lane_id, pids_s[half ^ 1]);
    };
    auto turn_over = [&]() {  // three chunks before the end
      if (walk.more) {
        stage_from(walk.next);
        stage_next(0, slot_before(q));
      }
    };
    chunk(o0, o1, No{}, [&]() {
      wait_one_of<kLoads, kTpw, kMaxNb + 1>(kLoads + stored);
      pass_barrier();
      walk.expert_of(cur, false);
      if (short_pass) look_up();
      stage(nbc, 3, slot_before(q));
    });
    chunk(o1, o0, No{}, [&]() {
      wait_one_of<kLoads, kTpw, kMaxNb + 1>(kLoads + stored);
      pass_barrier();
      if (short_pass) {
        turn_over();
      } else {
        look_up();
        stage(nbc, 4, slot_before(q));
      }
    });
    if (!short_pass) {
      auto middle = [&](int c) {
        wait_exactly<kLoads>();
        pass_barrier();
        stage(nbc, c + 3, slot_before(q));
      };
      for (int c = 2; c + 4 < n; c += 2) {
        chunk(o0, o1, No{}, [&]() { middle(c); });
        chunk(o1, o0, No{}, [&]() { middle(c + 1); });
      }
      chunk(o0, o1, No{}, [&]() { middle(n - 4); });
      chunk(o1, o0, No{}, [&]() {
        wait_exactly<kLoads>();
        pass_barrier();
        turn_over();
      });
    }
    chunk(o0, o1, No{}, [&]() {
      if (walk.more)
        wait_one_of<kDnW + 1, 1, kMaxPlaneLoads>(kDnW + plane_loads(walk.next.nb));
      else
        wait_exactly<0>();
      pass_barrier();
      if (walk.more) stage_next(1, slot_before(q));
    });
    chunk(o1, o0, Yes{}, [&]() {
      pass_barrier();
      if (walk.more) stage_next(2, slot_before(q));
    });

    // y: lane (r, kg) holds rows 4 kg .. + 3 of a tile for token r of a column
    // block; they pass through the wave's own LDS as gate/up's results do
    const auto yr = make_rsrc(y, 4u * (uint32_t)n_pairs * (uint32_t)H);
    const int l_row = lane >> 2, l_piece = place(l_row, lane & 3);
    const int tile0 = cur.grp * kTpu + (wave % kRowGroups) * kTpw;
    const int blk0 = (wave / kRowGroups) * NB;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int sl = cur.p0 + (blk0 + nb) * 16 + l_row;
      const int p = pids_s[half][(blk0 + nb) * 16 + l_row];
      const bool ok = sl < cur.cnt && p >= 0 && p < n_pairs;
#pragma unroll
      for (int t = 0; t < kTpw; ++t) {
        *reinterpret_cast<u32x4*>(trans + (r * 4 + place(r, kg)) * 8) =
            __builtin_bit_cast(u32x4, acc[t][nb]);
        const u32x4 v = *reinterpret_cast<const u32x4*>(trans + lane * 8);
        const uint32_t off =
            ok && tile0 + t < tpe
                ? ((uint32_t)p * (uint32_t)H + (uint32_t)((tile0 + t) * 16 + l_piece * 4)) * 4u
                : kOutOfRange;
        __builtin_amdgcn_raw_buffer_store_b128(v, yr, off, 0, 0);
      }
    }
    stored = kTpw * NB;
  };
  for (;;) {
    with_blocks(cur.nb, run_pass);
    if (!walk.more) break;
    cur = walk.next;
    half ^= 1;
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));
}

// ---------------------------------------------------------------------------
// down projection of tiled weights with long rows: weights through registers
//
// A wave owns two row tiles and computes every column block of a pass; its
// weights go from memory into its registers, 2 KiB of a tile a chunk of 64
// columns, one chunk ahead, so no wave waits for another's; only h goes through
// LDS, two chunks of both planes.  A pass begins with an empty pipeline, which a
// pass of the ring above does not: the fewer chunks a pass has, the more that
// counts.  Against the ring, H 2048, 4 slots a token: I 512, 256 experts, 48 /
// 96 / 150 tokens each: 122 / 160 / 267 us here, 120 / 151 / 244 there; I 768,
// 128 experts: 90 / 117 / 160 here, 96 / 121 / 178 there; I 1024, 60 experts:
// 55 / 70 / 108 here, 53 / 77 / 113 there.  Row-major weights, whose 64-byte
// pieces cost the address path four times as much on the way into registers,
// take the ring at every I (I 768: 110 / 138 / 192 us so, 108 / 130 / 184 there).

constexpr int kRingDownMaxI = 512;              // tiled rows up to which the ring is used
constexpr int kRgTpw = 2;                       // row tiles a wave
constexpr int kRgCols = 64, kRgSteps = kRgCols / 32;
constexpr int kRgRows = 8;                      // staged rows per 1 KiB load of a wave
static_assert(kWv * kRgTpw == kTpu, "one unit size");

// A pass of NBK column blocks (those past the pass's tokens multiply zero
// rows).  The ring slots are distinct restrict pointers: the compiler then
// knows that the loads into one do not write the one being read.
template <int NBK>
__device__ __forceinline__ void down_regs_pass(__amdgpu_buffer_rsrc_t w,
                                               __amdgpu_buffer_rsrc_t hi_r,
                                               __amdgpu_buffer_rsrc_t lo_r, int tile0, int tpe,
                                               const int* __restrict__ perm, int n_pairs,
                                               uint16_t* __restrict__ slot0,
                                               uint16_t* __restrict__ slot1,
                                               __amdgpu_buffer_rsrc_t yr, int base, int p0,
                                               int cnt, int H, int I, int lane, int wave) {
  constexpr int kHalf = NBK * 16 / kRgRows;     // a plane's loads a chunk, over the waves
  static_assert(2 * kHalf % kWv == 0, "whole rounds of loads");
  constexpr int kLoads = 2 * kHalf / kWv, kWLoads = kRgTpw * kRgSteps;
  const int r = lane & 15, kg = lane >> 4, n = I / kRgCols;  // n chunks, an even number
  auto swizzle = [](int row) { return (row & 7) ^ ((row >> 3) & 1); };
  // the y row of each of this lane's output columns; loaded now, before the
  // staging loads that the waits count
  int pid[NBK];
#pragma unroll
  for (int nb = 0; nb < NBK; ++nb) {
    const int sl = p0 + nb * 16 + r;
    const int p = sl < cnt ? perm[base + sl] : -1;
    pid[nb] = p >= 0 && p < n_pairs ? p : -1;
  }
  uint32_t off[kLoads];  // this lane's piece of each load in chunk 0
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const int f = wave + j * kWv, row = (f < kHalf ? f : f - kHalf) * kRgRows + (lane >> 3);
    const int piece = (lane & 7) ^ swizzle(row);
    off[j] = p0 + row < cnt ? ((uint32_t)(base + p0 + row) * I + (uint32_t)piece * 8u) * 2u
                            : kOutOfRange;
  }
  auto stage = [&](int c, uint16_t* buf) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int f = wave + j * kWv;  // hi rows, then lo rows
      const bool lo = f >= kHalf;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          lo ? lo_r : hi_r,
          (__attribute__((address_space(3))) void*)(buf + ((lo ? kNT : 0) +
                                                           (lo ? f - kHalf : f) * kRgRows) * kRgCols),
          16, off[j] + (uint32_t)c * kRgCols * 2u, 0, 0, 0);
    }
  };
  auto issue = [&](int c, u32x4 (&A)[kRgTpw][kRgSteps]) {
#pragma unroll
    for (int t = 0; t < kRgTpw; ++t) {
      const uint32_t at = (uint32_t)(tile0 + t) * 32u * I + (uint32_t)lane * 16u;
      const bool ok = c < n && tile0 + t < tpe;
#pragma unroll
      for (int st = 0; st < kRgSteps; ++st)
        A[t][st] = buf_ld128_stream(w, ok ? at + (uint32_t)(c * kRgSteps + st) * 1024u : kOutOfRange);
    }
  };
  int h_at[kRgSteps];
#pragma unroll
  for (int st = 0; st < kRgSteps; ++st) h_at[st] = ((st * 4 + kg) ^ swizzle(r)) * 8;

  stage(0, slot0);
  __builtin_amdgcn_sched_barrier(0);  // the load order the waits below count on
  u32x4 A[2][kRgTpw][kRgSteps];
  issue(0, A[0]);
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc[kRgTpw][NBK];
#pragma unroll
  for (int t = 0; t < kRgTpw; ++t)
#pragma unroll
    for (int nb = 0; nb < NBK; ++nb) acc[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < n; c0 += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      // chunk c0 + d of h landed (its weights, issued after it, need not have),
      // and every wave is done with the other slot
      __builtin_amdgcn_s_waitcnt(vmcnt_at_most_lds_done(kWLoads));
      __builtin_amdgcn_s_barrier();
      stage(c0 + d + 1, d ? slot0 : slot1);  // (past the end: rows that nothing reads)
      __builtin_amdgcn_sched_barrier(0);
      issue(c0 + d + 1, A[d ^ 1]);
      __builtin_amdgcn_sched_barrier(0);  // loads ahead of the chunk's MFMAs
      const uint16_t* buf = d ? slot1 : slot0;
#pragma unroll
      for (int st = 0; st < kRgSteps; ++st) {
#pragma unroll
        for (int nb = 0; nb < NBK; ++nb) {
          const uint16_t* row = buf + (nb * 16 + r) * kRgCols + h_at[st];
          const u32x4 bh = *reinterpret_cast<const u32x4*>(row);
          const u32x4 bl = *reinterpret_cast<const u32x4*>(row + kNT * kRgCols);
#pragma unroll
          for (int t = 0; t < kRgTpw; ++t) {
            acc[t][nb] = mfma_16x16x32(A[d][t][st], bh, acc[t][nb]);
            acc[t][nb] = mfma_16x16x32(A[d][t][st], bl, acc[t][nb]);
          }
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));  // the loads past the end landed

  // lane (r, kg) holds output rows tile * 16 + 4 kg .. + 3 of pair pid[nb]
#pragma unroll
  for (int t = 0; t < kRgTpw; ++t) {
#pragma unroll
    for (int nb = 0; nb < NBK; ++nb) {
      const uint32_t at = tile0 + t < tpe && pid[nb] >= 0
                              ? ((uint32_t)pid[nb] * H + (uint32_t)((tile0 + t) * 16 + kg * 4)) * 4u
                              : kOutOfRange;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[t][nb]), yr, at, 0, 0);
    }
  }
}

__global__ __launch_bounds__(kBlk, 1) void down_prefill_regs_kernel(
    const uint16_t* __restrict__ h_hi, const uint16_t* __restrict__ h_lo,
    const uint16_t* __restrict__ w2, const int* __restrict__ counts,
    const int* __restrict__ offsets, const int* __restrict__ perm,
    const int* __restrict__ active, const int* __restrict__ n_active, float* __restrict__ y, int H,
    int I, int m, int n_pairs) {
  __shared__ __attribute__((aligned(1024))) uint16_t slot0[2 * kNT * kRgCols];
  __shared__ __attribute__((aligned(1024))) uint16_t slot1[2 * kNT * kRgCols];
  const int n_act = *n_active;
  if (n_act <= 0 || n_act > m) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int tpe = H / 16, gpe = (tpe + kTpu - 1) / kTpu;
  const uint32_t h_bytes = 2u * (uint32_t)n_pairs * (uint32_t)I;
  const auto hi_r = make_rsrc(h_hi, h_bytes), lo_r = make_rsrc(h_lo, h_bytes);
  const auto yr = make_rsrc(y, 4u * (uint32_t)n_pairs * (uint32_t)H);
  for (int u = unit_slot(); u < n_act * gpe; u += gridDim.x) {
    const int a = u / gpe, e = active[a];
    if (e < 0 || e >= m) continue;
    const int cnt = counts[e], base = offsets[e];
    if (cnt <= 0 || base < 0 || cnt > n_pairs - base) continue;
    const auto w = make_rsrc(w2 + (size_t)e * H * I, 2u * (uint32_t)H * (uint32_t)I);
    const int tile0 = (u - a * gpe) * kTpu + wave * kRgTpw;
    for (int p0 = 0; p0 < cnt; p0 += kNT) {
      const int blocks = (min(kNT, cnt - p0) + 15) >> 4;
      __syncthreads();  // the previous pass's reads of the ring are done
      auto pass = [&](auto nbk) {
        down_regs_pass<decltype(nbk)::value>(w, hi_r, lo_r, tile0, tpe, perm, n_pairs, slot0,
                                             slot1, yr, base, p0, cnt, H, I, lane, wave);
      };
      if (blocks <= 4)
        pass(std::integral_constant<int, 4>{});
      else if (blocks <= 8)
        pass(std::integral_constant<int, 8>{});
      else
        pass(std::integral_constant<int, kNT / 16>{});
    }
  }
}

int prefill_grid() {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  return cus;
}

}  // namespace

bool prefill_supported(int T, int H, int I, int m, int k) {
  // 16 or more pairs per expert on average over a pool large enough to
  // spread its units over the chip, K in whole rounds of the pipelines (H
  // and I multiples of 128), and 32-bit offsets.  From 16 pairs an expert
  // on, its 160-token passes beat the decode kernels' 32-token ones
  // (measured on the 256-expert layer at H 2048, I 512: batch 256 over 64
  // kept experts 146 -> 100 us a step, gate/up at 5.5 instead of 3.1 TB/s;
  // batch 128 over 64 and batch 256 over 128, 4-6 us faster); at 8 a
  // decode step is faster on the decode kernels.
  return m >= 16 && (int64_t)T * k >= (int64_t)16 * m && H % (2 * kGuCols) == 0 &&
         I % (32 * kDnSlots) == 0 &&
         H <= 32768 && 4 * (int64_t)T * k * H < ((int64_t)1 << 31);
}

hipError_t launch_gate_up_prefill(const uint16_t* x, int T, const uint16_t* w13, bool tiled,
                                  const int* counts, const int* offsets, const int* perm,
                                  const int* active, const int* n_active, int H, int I, int m,
                                  int k, uint16_t* h_hi, uint16_t* h_lo, hipStream_t stream) {
  if (tiled)
    gate_up_prefill_kernel<true><<<prefill_grid(), kBlk, 0, stream>>>(
        x, w13, counts, offsets, perm, active, n_active, h_hi, h_lo, H, I, m, k, T * k);
  else
    gate_up_prefill_kernel<false><<<prefill_grid(), kBlk, 0, stream>>>(
        x, w13, counts, offsets, perm, active, n_active, h_hi, h_lo, H, I, m, k, T * k);
  return hipGetLastError();
}

hipError_t launch_down_prefill(int T, const uint16_t* w2, bool tiled, const int* counts,
                               const int* offsets, const int* perm, const int* active,
                               const int* n_active, int H, int I, int m, int k,
                               const uint16_t* h_hi, const uint16_t* h_lo, float* y,
                               hipStream_t stream) {
  if (tiled && I > kRingDownMaxI)
    down_prefill_regs_kernel<<<prefill_grid(), kBlk, 0, stream>>>(
        h_hi, h_lo, w2, counts, offsets, perm, active, n_active, y, H, I, m, T * k);
  else if (tiled)
    down_prefill_kernel<true><<<prefill_grid(), kBlk, 0, stream>>>(
        h_hi, h_lo, w2, counts, offsets, perm, active, n_active, y, H, I, m, T * k);
  else
    down_prefill_kernel<false><<<prefill_grid(), kBlk, 0, stream>>>(
        h_hi, h_lo, w2, counts, offsets, perm, active, n_active, y, H, I, m, T * k);
  return hipGetLastError();
}

}  // namespace sw
