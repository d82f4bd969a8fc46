// plan.cpp -- argument validation and the split-KV work decomposition.
// Pure host arithmetic: no HIP call is made here, so every error path can be
// exercised on a machine without a GPU.
#include <limits.h>
#include <stdlib.h>

#include <algorithm>

#include "internal.h"

namespace md {

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Largest visible range of any unit, in tokens.  Verify: the whole cache.
// Draft: sinks plus the union of the L queries' windows, which is
// [S - L - W + 1, S) -- or the whole prefix when that reaches the sinks.
int64_t visible_bound(int64_t max_kv_len, int L, int mode, int64_t n_sink, int64_t window) {
  if (mode == MD_MODE_VERIFY) return max_kv_len;
  if (mode == MD_MODE_DRAFT_INDEXED) return window + L;  // list capacity + speculated tokens
  int64_t lo = max_kv_len - L - window + 1;
  if (lo <= n_sink) return max_kv_len;
  return n_sink + (max_kv_len - lo);
}

}  // namespace

// Sizes that are malformed in themselves.
static int check_attn_shape(const md_attn_args* a) {
  if (a->num_seqs < 0) return MD_ERR_INVALID_ARG;
  if (a->q_len < 1 || a->q_len > 16) return MD_ERR_INVALID_ARG;
  if (a->num_q_heads < 1 || a->num_kv_heads < 1) return MD_ERR_INVALID_ARG;
  if (a->num_q_heads % a->num_kv_heads != 0) return MD_ERR_INVALID_ARG;
  if (a->head_dim < 1) return MD_ERR_INVALID_ARG;
  if (a->max_kv_len < a->q_len) return MD_ERR_INVALID_ARG;
  return MD_OK;
}

int env_knob(const char* name, int lo, int hi) {
  const char* e = getenv(name);
  const int v = e ? atoi(e) : 0;
  return (v >= lo && v <= hi) ? v : 0;
}

int check_attn_sizes(const md_attn_args* a) {
  const int shape = check_attn_shape(a);
  if (shape != MD_OK) return shape;
  if (a->head_dim != 64 && a->head_dim != 128) return MD_ERR_UNSUPPORTED;
  if (static_cast<int64_t>(a->num_q_heads / a->num_kv_heads) * a->q_len > kMaxRows)
    return MD_ERR_UNSUPPORTED;
  if (a->kv_stride_tok > kMaxTokStride) return MD_ERR_UNSUPPORTED;
  if (a->max_kv_len > kMaxPosition) return MD_ERR_UNSUPPORTED;
  // Units (workgroups) and query rows (merge workgroups of four rows) in 32 bits.
  if (static_cast<int64_t>(a->num_seqs) * a->num_kv_heads > INT32_MAX) return MD_ERR_UNSUPPORTED;
  const int64_t rows_per_seq = static_cast<int64_t>(a->q_len) * a->num_q_heads;
  if (a->num_seqs > 4 * static_cast<int64_t>(INT32_MAX) / rows_per_seq) return MD_ERR_UNSUPPORTED;
  return MD_OK;
}

int validate_attn(const md_attn_args* a, int mode, int n_sink, int window, Plan* plan) {
  if (!a) return MD_ERR_INVALID_ARG;
  if (mode != MD_MODE_VERIFY && mode != MD_MODE_DRAFT && mode != MD_MODE_DRAFT_INDEXED)
    return MD_ERR_INVALID_ARG;
  if (mode == MD_MODE_DRAFT && (n_sink < 0 || window < 1)) return MD_ERR_INVALID_ARG;
  if (mode == MD_MODE_DRAFT_INDEXED && window < 1) return MD_ERR_INVALID_ARG;
  const int shape = check_attn_shape(a);
  if (shape != MD_OK) return shape;
  if (a->dtype != MD_F32 && a->dtype != MD_BF16) return MD_ERR_INVALID_ARG;
  const bool paged = a->page_size != 0;
  if (a->page_size < 0) return MD_ERR_INVALID_ARG;
  if (paged) {
    if (!is_pow2(a->page_size) || a->max_pages_per_seq < 1 || a->num_pages < 1)
      return MD_ERR_INVALID_ARG;
    if (ceil_div(a->max_kv_len, a->page_size) > a->max_pages_per_seq) return MD_ERR_INVALID_ARG;
    if (a->num_pages > INT32_MAX) return MD_ERR_INVALID_ARG;  // page ids are int32
  }
  if (a->kv_stride_blk < 0 || a->kv_stride_tok < 0 || a->kv_stride_head < 0)
    return MD_ERR_INVALID_ARG;
  // Every malformed argument above is reported before a limit below.
  if (mode != MD_MODE_VERIFY && window > kMaxPosition) return MD_ERR_UNSUPPORTED;
  const int sizes = check_attn_sizes(a);
  if (sizes != MD_OK) return sizes;
  if (a->num_seqs == 0) return MD_OK;  // nothing will be read or written
  const int num_cus = device_cu_count();
  const Plan p = plan_call(a, mode, n_sink, window, num_cus);
  if (plan) *plan = p;
  if (p.n_chunks > kMaxChunks) return MD_ERR_UNSUPPORTED;  // unreachable below ~16k compute units

  if (!a->q || !a->k || !a->v || !a->o || !a->kv_lens) return MD_ERR_INVALID_ARG;
  if (paged != (a->page_table != nullptr)) return MD_ERR_INVALID_ARG;
  if (!aligned16(a->q) || !aligned16(a->k) || !aligned16(a->v) || !aligned16(a->o))
    return MD_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(a->kv_lens) & 3u) ||
      (a->lse && (reinterpret_cast<uintptr_t>(a->lse) & 3u)) ||
      (paged && (reinterpret_cast<uintptr_t>(a->page_table) & 3u)) ||
      (reinterpret_cast<uintptr_t>(a->err_word) & 3u))
    return MD_ERR_INVALID_ARG;
  // Every token row must start on a 16-byte boundary for the 128-bit loads.
  const int64_t per16 = a->dtype == MD_BF16 ? 8 : 4;
  if (a->kv_stride_blk % per16 || a->kv_stride_tok % per16 || a->kv_stride_head % per16)
    return MD_ERR_INVALID_ARG;
  // A token row must not overlap the next head's row.
  if (a->num_kv_heads > 1 && a->kv_stride_head < a->head_dim) return MD_ERR_INVALID_ARG;

  if (p.workspace_bytes) {
    if (!a->workspace || a->workspace_bytes < p.workspace_bytes) return MD_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(a->workspace) & 255u) return MD_ERR_WORKSPACE;
  }
  return MD_OK;
}

// What a launch of `wgs` workgroups of `bytes` K/V bytes each costs, in
// microseconds, as measured on MI355X: `start` per round of resident
// workgroups (first tile, epilogue), the stream at most at `wg_rate` bytes/us
// per workgroup, kCuRate per compute unit and kChipRate altogether.
// Workgroups past the resident ones wait for a whole round.
struct StreamCost {
  double start;      // us
  double wg_rate;    // bytes/us of one workgroup
  int resident;      // workgroups a compute unit holds
};
constexpr double kChipUs = 1.0 / 7.0e6, kCuUs = 1.0 / 34.0e3;  // us per byte
static double launch_us(const StreamCost& c, int32_t wgs, double bytes, int32_t cus) {
  const int32_t round = cus * c.resident;
  const double slowest = 1.0 / c.wg_rate;
  double us = 0.0;
  for (int32_t left = wgs; left > 0; left -= round) {
    const int32_t w = std::min(left, round);
    const int32_t per_cu = w <= cus ? 1 : (w + cus - 1) / cus;
    // Later rounds start as workgroups of the round before finish.
    us += c.start + bytes * std::max(slowest, std::max(per_cu * kCuUs, w * kChipUs));
  }
  return us;
}

// The range split for n_groups workgroups' worth of units of U tokens.  The
// plain rule gives a group one chunk when the groups alone cover every compute
// unit, else just as many as cover them, never below `min_chunk` tokens
// per chunk (kMinChunkTokens, a tile for each wave: a 5-token verify of one
// 4001-token sequence takes 27.7 us in 1024-token chunks, 16.2 in 256 and 15.0
// in 128); a range of at most `whole` tokens is not cut.  That leaves a second round of few
// workgroups wherever the groups do not divide the compute units (40 sequences
// of 8 heads and 3000 tokens: 64 of 320 workgroups run alone), so any other
// count that the launch cost above puts at 5% less is taken instead.
static void split_units(int64_t U, int64_t n_groups, int64_t slots, int64_t whole,
                        int64_t min_chunk, const StreamCost* cost, int64_t group_rows,
                        int64_t tok_bytes, int d, int64_t* n_chunks_out,
                        int64_t* chunk_len_out) {
  int64_t n_chunks = 1;
  const int64_t cap = U <= whole ? 1 : ceil_div(U, min_chunk);
  if (n_groups > 0 && n_groups < slots) n_chunks = std::min(ceil_div(slots, n_groups), cap);
  if (cost && n_groups > 0 && cap > 1 && n_groups < 2 * slots) {
    // In tiles and 32 bits: a division of 64 would cost as much as the rest.
    const uint32_t tiles = static_cast<uint32_t>(ceil_div(U, kTile));
    const int32_t g = static_cast<int32_t>(n_groups), cus = static_cast<int32_t>(slots);
    const double tile_bytes = static_cast<double>(kTile * tok_bytes);
    const double part_bytes = static_cast<double>(n_groups * group_rows * (d + 1) * 4);
    auto us = [&](uint32_t n, uint32_t len) {
      return launch_us(*cost, static_cast<int32_t>(n) * g, len * tile_bytes, cus) +
             (n > 1 ? kMergeUs + n * part_bytes * (2.0 / 6.0e6) : 0.0);
    };
    const uint32_t first = static_cast<uint32_t>(n_chunks);
    double best = us(first, (tiles + first - 1) / first) * 0.95;
    const uint32_t last = static_cast<uint32_t>(std::min(
        std::min(cap, 4 * slots / n_groups),
        std::max<int64_t>(1, static_cast<int64_t>(kSplitMaxPartials / part_bytes))));
    const uint32_t half = static_cast<uint32_t>(cus / (2 * g));
    for (uint32_t n = 1; n <= last;) {
      const uint32_t len = (tiles + n - 1) / n;
      const double t = us(n, len);
      if (t < best) {
        best = t;
        n_chunks = n;
      }
      if (len <= 1) break;
      // The next count that shortens the chunk (those between cost no less),
      // from a split over half of the compute units on.
      n = std::max((tiles + len - 2) / (len - 1), half);
    }
  }
  int64_t chunk_len = ceil_div(ceil_div(U, n_chunks), kTile) * kTile;
  if (chunk_len < kTile) chunk_len = kTile;
  n_chunks = ceil_div(U, chunk_len);
  if (n_chunks < 1) n_chunks = 1;
  *n_chunks_out = n_chunks;
  *chunk_len_out = chunk_len;
}

// The launch cost of an attention instance.  Starts: 6.7 us measured with one
// row tile, ~10 with two, 16 with four.  A workgroup streams 34 KB/us with up to
// two row tiles (1.9 us per tile of its four waves), 24-28 with more; rows of
// 64 channels halve the bytes of a tile, not its work.  Two workgroups fit a
// compute unit's registers and LDS with up to two row tiles of bf16 or with 64
// channels, else one.
static StreamCost stream_cost(int NT, int d, bool bf16) {
  StreamCost c;
  c.start = 4.0 + 3.0 * NT;
  if (bf16)
    c.wg_rate = d == 128 ? (NT <= 2 ? 34.0e3 : (NT == 3 ? 28.0e3 : 24.0e3))
                         : (NT <= 2 ? 27.0e3 : 22.0e3);
  else
    c.wg_rate = NT == 1 ? 27.0e3 : 27.0e3 / NT;
  c.resident = (bf16 && NT <= 2) || (d == 64 && (bf16 || NT <= 2)) ? 2 : 1;
  return c;
}

// The balanced verify of groups that do not cover the compute units: all of them
// stream, and every workgroup cuts a group and merges it.  Measured over its
// stream, uniform lengths: 31 us with one row tile, 53 with two, 68 with three.
// Balancing every such group instead: 53 sequences of 8 KV heads and 5264 tokens,
// two row tiles, 229 us against 192 whole; none: 43 x 8, 7652, three, 272 against
// 234.  Over 436 such random shapes this choice is 11% faster than balancing all.
static double balanced_us(const StreamCost& c, int NT, double bytes, int64_t cus) {
  return 10.0 + 20.0 * NT +
         bytes * std::max(1.0 / (static_cast<double>(cus) * c.wg_rate), kChipUs);
}

// Kv heads per workgroup.  In the token-major cache the kv heads of a token
// are adjacent, so a workgroup that serves two heads of a sequence (two waves
// each) reads 2 x 256 B runs of every token row (bf16, d = 128) side by side
// instead of one: on MI355X a load-only model of the verify stream read the
// B = 64, S = 32768 cache at 7.03 TB/s this way against 6.62 TB/s with one
// head per workgroup.  Pairs halve the workgroups, though, so a range that
// must be split to fill the device is cut into twice as many chunks, each
// paying a pipeline fill and its share of the merge.  Measured over verify
// and draft calls of B = 1 .. 64 and S = 2048 .. 131072 (Llama-3.1-8B heads):
// pairs gain 5-13% where they alone fill the device and 2-3% where their
// chunks stay at 4096 tokens or more, and lose up to a third on short split
// ranges (one-token verify at B = 1, S = 4096: 35 us against 26).  So pairs
// are taken in those two cases only.  A listed draft reads a different list
// per head -- no adjacent rows -- and keeps one head per workgroup.
// MD_HEADS_PER_WG (1 or 2) overrides, for measurement.
static int heads_per_workgroup(const md_attn_args* a, int mode, int64_t U, int64_t slots,
                               int64_t whole, int64_t min_chunk, const StreamCost* cost,
                               int64_t rows, int64_t tok_bytes) {
  const int forced = env_knob("MD_HEADS_PER_WG", 1, 2);
  if (a->num_kv_heads % 2) return 1;
  if (forced) return forced;
  if (mode == MD_MODE_DRAFT_INDEXED) return 1;
  const int64_t pairs = static_cast<int64_t>(a->num_seqs) * a->num_kv_heads / 2;
  if (pairs >= slots) return 2;
  // No chunk is as long, or such chunks use less than half of the device.
  if (U <= kPairMinChunkTokens - kTile ||
      ceil_div(U, kPairMinChunkTokens - kTile) * pairs < slots / 2)
    return 1;
  int64_t n_chunks, chunk_len;
  split_units(U, pairs, slots, whole, min_chunk, cost, 2 * rows, 2 * tok_bytes, a->head_dim,
              &n_chunks, &chunk_len);
  return chunk_len >= kPairMinChunkTokens ? 2 : 1;
}

Plan make_plan(const md_attn_args* a, int mode, int n_sink, int window, int num_cus,
               bool plain) {
  Plan p;
  const int L = a->q_len;
  p.G = a->num_q_heads / a->num_kv_heads;
  p.R = p.G * L;
  p.NT = (p.R + 15) / 16;
  const int64_t U = visible_bound(a->max_kv_len, L, mode, n_sink, window);
  p.U_max = static_cast<int32_t>(U);
  p.n_rows = static_cast<int64_t>(a->num_seqs) * L * a->num_q_heads;
  p.n_units = static_cast<int64_t>(a->num_seqs) * a->num_kv_heads;

  // One workgroup of kWaves waves (one per SIMD) per compute unit is enough
  // to stream at full rate.  When the workgroups alone cover every compute
  // unit, one chunk per unit avoids the merge pass; else each unit's range is
  // split just until they do (split_units).  (Every
  // chunk pays a pipeline fill, a cross-wave merge and a partial write:
  // measured on MI355X, splitting further -- two or four workgroups per
  // compute unit -- was 5-15% slower on long caches and slower still on
  // short draft ranges.)
  // MD_SLOTS_SCALE = 2..4 plans for that many workgroups per compute unit
  // (measurement only).
  const int64_t slots = (num_cus > 0 ? num_cus : 256) * std::max(1, env_knob("MD_SLOTS_SCALE", 2, 4));
  // Up to kWholeTokens one pass does: 256 tokens in one chunk take 8.9-10.2 us
  // and in two 9.4-11.0; at 430-512 the kernels gain 3 us of 13 but a caller
  // issuing call after call loses 5 us of host time to the second launch (82
  // units of 427 tokens through the binding: 17.4 us whole, 17.9 split).  Listed
  // drafts cost the host more, so one pass does for longer: whole / split through
  // the binding, one sequence of 8 KV heads, one token, 520 entries 16.5 / 21.1
  // us, 768 18.7 / 21.0, 1020 21.0 / 21.0; five tokens, 1020 entries 27.9 / 20.8.
  // (Replayed from a graph, which has no host time, splits win from 520 entries
  // on: 14.9 / 10.2, 20.8 / 10.5 at 1020.)
  const int64_t min_chunk = plain ? kPlainChunkTokens : kMinChunkTokens;
  const bool listed = mode == MD_MODE_DRAFT_INDEXED;
  const int64_t whole =
      plain ? std::max<int64_t>(kPlainChunkTokens, listed ? kBareList + L : 0)
            : (listed ? kWholeList : kWholeTokens);
  const bool bf16 = a->dtype == MD_BF16;
  const StreamCost sc = stream_cost(p.NT, a->head_dim, bf16);
  const StreamCost* cost = plain || env_knob("MD_SLOTS_SCALE", 2, 4) ? nullptr : &sc;
  const int64_t tok_bytes = int64_t{2} * a->head_dim * (bf16 ? 2 : 4);
  p.hp = heads_per_workgroup(a, mode, U, slots, whole, min_chunk, cost, p.R, tok_bytes);
  p.n_groups = p.n_units / p.hp;
  int64_t n_chunks, chunk_len;
  // Long ranges of groups that cover the device are the balanced verify's (or
  // longest-first's): one chunk.
  const int bal_min = bf16 ? kBalMinLen : kLptMinLen;
  if (p.n_groups >= slots && U >= bal_min) cost = nullptr;
  split_units(U, p.n_groups, slots, whole, min_chunk, cost, p.hp * p.R, p.hp * tok_bytes,
              a->head_dim, &n_chunks, &chunk_len);
  p.n_chunks = static_cast<int32_t>(n_chunks);
  p.chunk_len = static_cast<int32_t>(chunk_len);
  // Balanced verify: where the units alone fill the device and lengths may
  // differ (the cases longest-first dispatch serves), every workgroup takes
  // an equal share of all head groups' tiles, in pairs of adjacent kv heads
  // when the head count is even.  Only with at most two head groups per
  // compute unit: there the longest sequence sets the makespan of one group
  // per workgroup, while with more groups per unit the hardware dispatcher
  // already evens the load out and the extra pieces only add prologues.  Groups
  // that leave compute units idle are streamed whole unless balancing them is
  // put at less (balanced_us).
  // MD_BALANCED = 1 / 2 turns it off / on wherever allowed (measurement).
  const int bal_knob = env_knob("MD_BALANCED", 1, 2);
  const int bal_hp =
      (a->num_kv_heads % 2 == 0 && env_knob("MD_HEADS_PER_WG", 1, 2) != 1) ? 2 : 1;
  const int64_t cus = num_cus > 0 ? num_cus : 256;
  if (mode == MD_MODE_VERIFY && p.n_chunks == 1 && a->num_seqs >= 2 &&
      a->num_seqs <= kLptMaxSeqs && bal_knob != 1 && p.NT <= kBalMaxNT(a->dtype == MD_BF16) &&
      (bal_knob == 2 ||
       (a->max_kv_len >= bal_min && p.n_units / bal_hp <= 2 * cus &&
        (p.n_groups >= slots ||
         balanced_us(sc, p.NT, static_cast<double>(p.n_units * tok_bytes * U), cus) <
             launch_us(sc, static_cast<int32_t>(p.n_groups),
                       static_cast<double>(p.hp * tok_bytes * p.chunk_len),
                       static_cast<int32_t>(cus)))))) {
    const int hp = bal_hp;
    const int64_t groups = p.n_units / hp;
    // One workgroup per compute unit: every range then streams at once.
    // MD_BAL_WG_PER_CU = 2 doubles them, MD_BAL_NW sets their number
    // (measurement).
    const int64_t wpc = std::max(1, env_knob("MD_BAL_WG_PER_CU", 1, 2));
    const int64_t nw_forced = env_knob("MD_BAL_NW", 1, 4096);
    const int64_t nw = nw_forced ? nw_forced : cus * wpc;
    const int64_t tiles = ceil_div(a->max_kv_len, kTile) * (a->num_kv_heads / hp);
    const size_t slots = static_cast<size_t>(2 * nw);  // a first and a last piece per workgroup
    const size_t ctr = align_up(static_cast<size_t>(groups) * 8, 256);
    const size_t po = align_up(slots * hp * p.R * a->head_dim * 4, 256);
    const size_t pl = align_up(slots * hp * p.R * 4, 256);
    if (tiles * a->num_seqs < (int64_t{1} << 30) && ctr + po + pl <= kBalMaxWorkspace) {
      p.bal = true;
      p.hp = hp;
      p.n_groups = groups;
      p.bal_nw = static_cast<int32_t>(nw);
      p.counter_bytes = ctr;
      p.part_o_bytes = po;
      p.part_lse_bytes = pl;
      p.workspace_bytes = ctr + po + pl;
      return p;
    }
  }
  if (p.n_chunks > 1) {
    p.counter_bytes = align_up(static_cast<size_t>(p.n_groups) * 8, 256);
    p.part_o_bytes = align_up(static_cast<size_t>(n_chunks) * p.n_rows * a->head_dim * 4, 256);
    p.part_lse_bytes = align_up(static_cast<size_t>(n_chunks) * p.n_rows * 4, 256);
    p.workspace_bytes = p.counter_bytes + p.part_o_bytes + p.part_lse_bytes;
  }
  return p;
}

Plan plan_call(const md_attn_args* a, int mode, int n_sink, int window, int num_cus) {
  const Plan p = make_plan(a, mode, n_sink, window, num_cus);
  const size_t have = a->workspace && !(reinterpret_cast<uintptr_t>(a->workspace) & 255u)
                          ? a->workspace_bytes : 0;
  if (have >= p.workspace_bytes) return p;
  const Plan q = make_plan(a, mode, n_sink, window, num_cus, true);
  return have >= q.workspace_bytes ? q : p;
}

size_t workspace_need(const md_attn_args* a, int mode, int n_sink, int window, int num_cus) {
  const size_t need = make_plan(a, mode, n_sink, window, num_cus).workspace_bytes;
  if (!need) return 0;
  return std::max(need, make_plan(a, mode, n_sink, window, num_cus, true).workspace_bytes);
}

namespace {

// What one SnapKV pass over chunks of `keys` keys costs in `wgs` workgroups, in
// microseconds, as measured on MI355X: a compute unit takes key_us per key when
// at least `busy` workgroups share it (its workgroups then take turns: the most
// loaded unit sets the time), every round of `resident` ones start_us, and
// unequal speeds waste some of the last workgroup of each unit.
struct PassCost {
  double key_us, start_us;
  int busy, resident;
};
double pass_us(const PassCost& c, int64_t wgs, int64_t keys, int64_t cus) {
  constexpr double uneven = 0.15;
  const int64_t per_cu = std::max<int64_t>(ceil_div(wgs, cus), c.busy);
  const double stream = static_cast<double>(keys) * c.key_us * static_cast<double>(per_cu);
  return stream * (1.0 + uneven * static_cast<double>(cus) / static_cast<double>(wgs)) +
         c.start_us * static_cast<double>(ceil_div(wgs, cus * c.resident));
}

// Chunks of a range of U keys over n_units units: the fewest within 1% of the
// least pass_us, down to kSnapkvMinChunk keys a chunk (one prompt of 4000
// tokens, 8 heads of 128 rows: 49 us at 1024 keys a chunk, 19.4 at 256, 15.2 at
// 128, 16.2 at 64) and up to sixteen workgroups per compute unit (64 prompts of
// 32768: 1700 us with eight chunks a unit, 1764 with two).
void split_range(int64_t U, int64_t n_units, const PassCost& cost, int64_t cus,
                 int32_t* n_chunks_out, int32_t* chunk_len_out) {
  const int64_t whole = ceil_div(U > 0 ? U : 1, kTile) * kTile;
  int64_t chunk_len = whole;
  if (n_units > 0) {
    double best = pass_us(cost, n_units, whole, cus);
    for (int64_t n = 2; n * n_units <= 16 * cus;) {
      const int64_t len = ceil_div(ceil_div(U, n), kTile) * kTile;
      if (len < kSnapkvMinChunk) break;
      const int64_t n_len = ceil_div(U, len);
      const double t = pass_us(cost, n_len * n_units, len, cus);
      if (t < 0.99 * best) {
        best = t;
        chunk_len = len;
      }
      // The next shorter length, in steps of a sixteenth.
      n = std::max(n_len + 1, ceil_div(U, std::max<int64_t>(kTile, len - std::max<int64_t>(
                                                 kTile, len / 16 / kTile * kTile))));
    }
  }
  *n_chunks_out = static_cast<int32_t>(ceil_div(U > 0 ? U : 1, chunk_len));
  *chunk_len_out = static_cast<int32_t>(chunk_len);
}

// The chunks of a plain plan: enough for wg_per_cu workgroups per compute unit
// twice over, of at least kPlainChunkTokens keys.
void split_range_plain(int64_t U, int64_t n_units, int64_t wgs, int32_t* n_chunks_out,
                       int32_t* chunk_len_out) {
  int64_t n = 1;
  if (n_units > 0 && n_units < 2 * wgs)
    n = std::max<int64_t>(1, std::min(ceil_div(2 * wgs, n_units), ceil_div(U, kPlainChunkTokens)));
  const int64_t chunk_len = ceil_div(ceil_div(U > 0 ? U : 1, n), kTile) * kTile;
  *n_chunks_out = static_cast<int32_t>(ceil_div(U > 0 ? U : 1, chunk_len));
  *chunk_len_out = static_cast<int32_t>(chunk_len);
}

// key_us: the scores of a key (0.013 us at 128 rows in bf16, 0.107 in fp32,
// d = 128) or its bytes, whichever takes longer.  start_us grows with the rows
// of Q a workgroup loads: 50 fp32 units of 256 rows take 258 us in 250
// workgroups, one round, and 322 in 1000.  Residency as the registers and LDS of
// the pass instances allow.  At 33-64 rows of bf16 the counts chosen take no more
// than 3% over the best of a sweep of counts (one to 128 prompts of 2000 to 32768
// tokens, both head dims, paged and contiguous: 44 shapes), 5% at one.
PassCost pass_cost(int R, int d, bool f32) {
  const double rows = R / 128.0, wide = d / 128.0;
  PassCost c;
  if (f32) {
    c.key_us = 0.107 * std::max(rows, 0.125) * wide;
    c.start_us = 4.0 + 15.0 * rows * wide;
    c.resident = R <= 128 ? (d == 64 ? 4 : 2) : (d == 64 ? 2 : 1);
    c.busy = R <= 64 && d == 64 ? 2 : 1;
  } else {
    c.key_us = std::max(0.0094 * wide, 0.013 * rows);
    c.start_us = 3.0 + 4.0 * rows;
    c.resident = R <= 32 ? 4 : (R <= 64 ? 6 : (R <= 128 ? 4 : 2));
    c.busy = R <= 64 ? 4 : (R <= 128 ? 3 : 2);
  }
  return c;
}

}  // namespace

int validate_snapkv(const md_snapkv_args* a) {
  if (!a) return MD_ERR_INVALID_ARG;
  if (a->num_seqs < 0 || a->n_obs < 1 || a->num_q_heads < 1 || a->num_kv_heads < 1)
    return MD_ERR_INVALID_ARG;
  if (a->num_q_heads % a->num_kv_heads) return MD_ERR_INVALID_ARG;
  if (a->dtype != MD_F32 && a->dtype != MD_BF16) return MD_ERR_INVALID_ARG;
  if (a->max_prompt_len < a->n_obs) return MD_ERR_INVALID_ARG;
  if (a->votes_stride < 1 || a->votes_stride < a->max_prompt_len - a->n_obs)
    return MD_ERR_INVALID_ARG;
  const bool paged = a->page_size != 0;
  if (a->page_size < 0) return MD_ERR_INVALID_ARG;
  if (paged) {
    if (!is_pow2(a->page_size) || a->max_pages_per_seq < 1 || a->num_pages < 1 ||
        a->num_pages > INT32_MAX)
      return MD_ERR_INVALID_ARG;
    if (ceil_div(a->max_prompt_len, a->page_size) > a->max_pages_per_seq) return MD_ERR_INVALID_ARG;
  }
  if (a->kv_stride_blk < 0 || a->kv_stride_tok < 0 || a->kv_stride_head < 0)
    return MD_ERR_INVALID_ARG;
  if (a->head_dim != 64 && a->head_dim != 128) return MD_ERR_UNSUPPORTED;
  if (static_cast<int64_t>(a->num_q_heads / a->num_kv_heads) * a->n_obs > kSnapkvMaxRows)
    return MD_ERR_UNSUPPORTED;
  if (static_cast<int64_t>(a->num_seqs) * a->num_kv_heads > INT32_MAX) return MD_ERR_UNSUPPORTED;
  if (a->num_seqs == 0) return MD_OK;
  if (!a->q_obs || !a->k || !a->prompt_lens || !a->votes) return MD_ERR_INVALID_ARG;
  if (paged != (a->page_table != nullptr)) return MD_ERR_INVALID_ARG;
  if (!aligned16(a->q_obs) || !aligned16(a->k) || (reinterpret_cast<uintptr_t>(a->votes) & 3u) ||
      (reinterpret_cast<uintptr_t>(a->prompt_lens) & 3u))
    return MD_ERR_INVALID_ARG;
  const int64_t per16 = a->dtype == MD_BF16 ? 8 : 4;
  if (a->kv_stride_blk % per16 || a->kv_stride_tok % per16 || a->kv_stride_head % per16)
    return MD_ERR_INVALID_ARG;
  if (a->num_kv_heads > 1 && a->kv_stride_head < a->head_dim) return MD_ERR_INVALID_ARG;
  const SnapkvPlan pl = snapkv_plan_call(a, device_cu_count());
  if (!a->workspace || a->workspace_bytes < pl.workspace_bytes ||
      (reinterpret_cast<uintptr_t>(a->workspace) & 255u))
    return MD_ERR_WORKSPACE;
  return MD_OK;
}

SnapkvPlan make_snapkv_plan(const md_snapkv_args* a, int num_cus, bool plain) {
  SnapkvPlan p;
  p.G = a->num_q_heads / a->num_kv_heads;
  p.R = p.G * a->n_obs;
  p.TW = p.R <= 64 ? 1 : (p.R <= 128 ? 2 : 4);
  p.n_units = a->num_seqs * a->num_kv_heads;
  const int64_t cus = num_cus > 0 ? num_cus : 256;
  const int64_t U = a->max_prompt_len, U_votes = U - a->n_obs;
  if (plain) {
    const int64_t wgs = cus * (p.TW == 1 ? 2 : 8);
    split_range_plain(U, p.n_units, wgs, &p.n_chunks_stats, &p.chunk_len_stats);
    split_range_plain(U_votes, p.n_units, wgs, &p.n_chunks_votes, &p.chunk_len_votes);
  } else {
    const PassCost cost = pass_cost(p.R, a->head_dim, a->dtype == MD_F32);
    split_range(U, p.n_units, cost, cus, &p.n_chunks_stats, &p.chunk_len_stats);
    split_range(U_votes, p.n_units, cost, cus, &p.n_chunks_votes, &p.chunk_len_votes);
  }
  p.part_bytes = align_up(static_cast<size_t>(p.n_units) * p.n_chunks_stats * p.R * 4, 256);
  p.lse_bytes = align_up(static_cast<size_t>(p.n_units) * p.R * 4, 256);
  p.workspace_bytes = 2 * p.part_bytes + p.lse_bytes;
  return p;
}

SnapkvPlan snapkv_plan_call(const md_snapkv_args* a, int num_cus) {
  const SnapkvPlan p = make_snapkv_plan(a, num_cus);
  if (a->workspace_bytes >= p.workspace_bytes) return p;
  const SnapkvPlan q = make_snapkv_plan(a, num_cus, true);
  return a->workspace_bytes >= q.workspace_bytes ? q : p;
}

size_t snapkv_workspace_need(const md_snapkv_args* a, int num_cus) {
  return std::max(make_snapkv_plan(a, num_cus).workspace_bytes,
                  make_snapkv_plan(a, num_cus, true).workspace_bytes);
}

int validate_accept(int32_t num_seqs, int32_t n_draft, int32_t vocab, int32_t dtype) {
  // vocab <= 2^30: a chunk's length, rounded up to 8 elements, stays an int32.
  if (num_seqs < 0 || n_draft < 0 || n_draft + 1 > kAcceptMaxRowsPerSeq || vocab < 1 ||
      vocab > (1 << 30))
    return MD_ERR_INVALID_ARG;
  if (dtype != MD_F32 && dtype != MD_BF16) return MD_ERR_INVALID_ARG;
  const int64_t rows = static_cast<int64_t>(num_seqs) * (n_draft + 1);
  if (rows * 64 > INT32_MAX) return MD_ERR_INVALID_ARG;  // grid bound at the largest split
  return MD_OK;
}

AcceptPlan make_accept_plan(int32_t num_seqs, int32_t n_draft, int32_t vocab, int num_cus) {
  AcceptPlan pl;
  const int64_t rows = static_cast<int64_t>(num_seqs) * (n_draft + 1);
  if (rows <= 0 || vocab < 1) return pl;
  constexpr int64_t kMinChunk = 2048;
  const int64_t L = n_draft + 1;
  int64_t n = (8 * static_cast<int64_t>(num_cus) + rows - 1) / rows;
  n = std::min<int64_t>(n, (vocab + kMinChunk - 1) / kMinChunk);
  n = std::min<int64_t>(n, kAcceptMaxPartialsPerSeq / L);  // the accept pass stages L * n in LDS
  n = std::max<int64_t>(1, std::min<int64_t>(n, 64));
  int64_t len = (vocab + n - 1) / n;
  len = (len + 7) / 8 * 8;
  pl.chunk_len = static_cast<int32_t>(len);
  pl.n_chunks = static_cast<int32_t>((vocab + len - 1) / len);
  pl.part_bytes = align_up(static_cast<size_t>(rows) * pl.n_chunks * 4, 256);
  pl.workspace_bytes = 2 * pl.part_bytes;
  return pl;
}

int validate_kv_cache(const md_kv_cache* c, int32_t n_new) {
  if (!c || n_new < 0) return MD_ERR_INVALID_ARG;
  if (c->num_seqs < 0 || c->num_kv_heads < 1 || c->head_dim < 1) return MD_ERR_INVALID_ARG;
  if (c->dtype != MD_F32 && c->dtype != MD_BF16) return MD_ERR_INVALID_ARG;
  const int64_t es = c->dtype == MD_BF16 ? 2 : 4;
  if ((c->head_dim * es) % 16) return MD_ERR_INVALID_ARG;
  if (c->kv_stride_blk < 0 || c->kv_stride_tok < 0 || c->kv_stride_head < 0 ||
      (c->kv_stride_blk * es) % 16 || (c->kv_stride_tok * es) % 16 || (c->kv_stride_head * es) % 16)
    return MD_ERR_INVALID_ARG;
  if (c->page_size != 0) {
    if (c->page_size < 0 || (c->page_size & (c->page_size - 1)) || !c->page_table ||
        c->max_pages_per_seq < 1 || c->num_pages < 1)
      return MD_ERR_INVALID_ARG;
  } else {
    if (c->page_table || c->capacity < 1) return MD_ERR_INVALID_ARG;
  }
  return MD_OK;
}

}  // namespace md
