// Host-side launch planning of libpic's attention kernels: how many workgroups split a key
// range, and the workspace their partial results need.  Plain C++ (no device code), so the
// sanitizer build of the host library compiles this file as it is.
#include "pic_internal.h"

namespace pic {

namespace {

int64_t prefill_m_tiles(const AttnShape& s, int32_t n_suffix) {
  const int64_t M = (int64_t)n_suffix * (s.n_q_heads / s.n_kv_heads);
  return (M + kPrefillRowsPerWG - 1) / kPrefillRowsPerWG;
}
int64_t prefill_rows(const AttnShape& s, int32_t n_suffix) {
  return (int64_t)s.n_layers * s.batch * n_suffix * s.n_q_heads;
}
int prefill_tiles(int32_t n_suffix, int32_t max_ctx) {
  return (int)(((int64_t)max_ctx + n_suffix + kPrefillKeys - 1) / kPrefillKeys);
}

int64_t prefill_units(const AttnShape& s, int32_t n_suffix) {
  return prefill_m_tiles(s, n_suffix) * s.batch * s.n_kv_heads * s.n_layers;
}

// A launch whose units fill half the compute units or whose key ranges would be shorter than 8
// tiles needs no workspace: it can run whole, its sums in float32 from end to end (and keeps them
// so, with float32 partials, where the plan below splits it).  Any other brings bf16 partials for
// this count, which covers the compute units in whole rounds at the least rounds * tiles, one tile
// for the combine launch and the partial traffic counted in (ties within 3% go to fewer).
int prefill_bf16_splits_held(const AttnShape& s, int32_t n_suffix, int32_t max_ctx) {
  const int64_t base = prefill_units(s, n_suffix);
  if (base >= 128) return 1;
  const double rows = (double)prefill_rows(s, n_suffix);
  const int tiles = prefill_tiles(n_suffix, max_ctx);
  int best = 1;
  double best_cost = 1e30;
  for (int sp = 1; sp <= kPrefillMaxSplits; ++sp) {
    const int tps = (tiles + sp - 1) / sp;
    if (sp > 1 && tps < 8) break;
    const int64_t rounds = (base * sp + 255) / 256;
    const double partials = sp > 1 ? 1.0 + sp * rows * 2.0 * (double)prefill_partial_bytes(s.head_dim, false) / 4e12 / 2e-6 : 0.0;
    const double cost = (double)rounds * tps + partials;
    if (cost < best_cost * 0.97) {
      best_cost = cost;
      best = sp;
    }
  }
  return best;
}

}  // namespace

// Key-range splits of the prefill, by estimated time in us.  Under load the chip sits at its power
// limit, where a busy compute unit runs slower the more of them are busy: a workgroup's 64-key
// tile takes t_few with up to half of them busy and t_full with all (measured: 16 to 128
// workgroups 1.35 us, 192 1.65, 256 2.0; up to 128 rows the loads bound it, 1.15 to 1.2 us in short
// ranges, 1.55 where all are busy for long; at head_dim 64 1.0 and 1.2 us).  A split run adds the
// combine launch (5 us, a little more for each split) and the partials, written and read at ~5
// TB/s; the split that ends in the suffix has dearer tiles (rows addressed one by one, masked,
// perhaps turned) and is better one that is not full.  Ties go to fewer splits.
//  * Below 128 units up to the held count: 4 requests of 32K, 28/4 heads x 256 tokens (112 units) 434 us
//    in 9 splits / 420 in 2.
//  * From 128 to 192, where the plan's full workspace is there and the estimate promises 2.5 %, else
//    whole.  Whole / split, us: 8 requests of 10K x 128 tokens (128 units) 222 / 173, 16 of 4K x 32
//    76 / 61, 10 of 10K x 128 (160 units) 245 / 227, 12 of 32K x 128 (192) 828 / 772; contexts down to
//    half as long: 225 / 160, 64 / 50, 230 / 209.
//  * Beyond, none: up to 256 there is little to gain (28 requests of 32K x 32 tokens, 224 units: 701 us
//    whole, 772 in 8), and past a full round, where long equal contexts would gain (264 units over 32K
//    1.2 to 1.4 times), rounds are not in lockstep: uneven contexts fill the last one by themselves (40
//    requests of 2K to 4K keys, 28/4 heads x 73 tokens, 320 units: 165 us whole, 196 in 2; 48 of 5K to
//    10K x 32 tokens, 384 units: 345 / 379), and inline layouts, which plan alike, by their dispatch
//    order (10 of 16K x 252 inline tokens, 320 units: 439 / 591).
SplitPlan plan_prefill_splits(const AttnShape& s, int32_t n_suffix, int32_t max_ctx, size_t ws_bytes) {
  SplitPlan p;
  const int held = prefill_bf16_splits_held(s, n_suffix, max_ctx);
  const int64_t base = prefill_units(s, n_suffix);
  const bool may_whole = prefill_bf16_may_run_whole(s, n_suffix);
  p.m_tiles = (int)prefill_m_tiles(s, n_suffix);
  p.f32_partials = held == 1;
  const double split_bytes = (double)prefill_rows(s, n_suffix) * (double)prefill_partial_bytes(s.head_dim, p.f32_partials);
  const int tiles = prefill_tiles(n_suffix, max_ctx);
  const bool narrow = (int64_t)n_suffix * (s.n_q_heads / s.n_kv_heads) <= 128;
  const double t_few = s.head_dim == 64 ? 1.0 : (narrow ? 1.15 : 1.36);
  const double t_full = s.head_dim == 64 ? 1.2 : (narrow ? (may_whole ? 1.55 : 1.2) : 2.0);
  auto tile_us = [&](int64_t active) { return active <= 128 ? t_few : t_few + (t_full - t_few) * (double)(active - 128) / 128.0; };
  auto range = [&](int sp) { return (tiles + sp - 1) / sp; };
  auto cost = [&](int sp) {
    const int64_t wgs = base * sp;
    const double us = range(sp) * ((double)(wgs / 256) * t_full + (wgs % 256 ? tile_us(wgs % 256) : 0.0));
    return sp == 1 ? us : us + 5.0 + 0.3 * sp + 2.0 * sp * split_bytes / 5e6 + (sp * range(sp) == tiles ? 1.0 : 0.0);
  };
  const int most = !may_whole ? held : (base <= 192 ? kPrefillMaxSplits : 1);
  int best = 1;
  double best_us = cost(1);
  for (int sp = 2; sp <= most; ++sp) {
    if ((tiles + range(sp) - 1) / range(sp) < sp) continue;   // (the same ranges as fewer splits)
    if (cost(sp) < best_us * 0.99) {
      best = sp;
      best_us = cost(sp);
    }
  }
  if (may_whole && (best_us > cost(1) * 0.975 || best * split_bytes > (double)ws_bytes)) best = 1;
  // (short launches: what the estimate cannot tell apart, machines of other clocks do)
  if (held > 1 && best_us < 100.0 && cost(held) < best_us + 2.0) best = held;
  p.n_splits = best;
  p.tiles_per_split = range(best);
  return p;
}

// What the query call says.  Below 128 units that is room for the held count, whatever smaller count
// the plan takes: a caller sizes one workspace for its largest call, and planned room can be less
// there than for a smaller one (64 query heads over 8, 8 tokens over 49K keys: 6 requests run in 5
// ranges of 0.8 MB, one request in 31 of 0.135 MB).
size_t prefill_bf16_workspace(const AttnShape& s, int32_t n_suffix, int32_t max_ctx) {
  const int held = prefill_bf16_splits_held(s, n_suffix, max_ctx);
  const SplitPlan p = plan_prefill_splits(s, n_suffix, max_ctx, SIZE_MAX);
  const int n = held > 1 ? held : p.n_splits;
  return n == 1 ? 0 : (size_t)n * prefill_rows(s, n_suffix) * prefill_partial_bytes(s.head_dim, p.f32_partials);
}

bool prefill_bf16_may_run_whole(const AttnShape& s, int32_t n_suffix) { return prefill_units(s, n_suffix) >= 128; }

int32_t slot_map_tiles(int32_t map_cap) { return (int32_t)(((int64_t)map_cap + kPrefillKeys - 1) / kPrefillKeys); }

namespace {

int64_t decode_pairs(const AttnShape& s) { return (int64_t)s.batch * s.n_kv_heads * s.n_layers * decode_head_groups(s); }

// A split count, so that every wave keeps at least kDecodeMinWaveKeys keys.
int32_t decode_cap_splits(int64_t splits, int32_t max_len) {
  const int64_t per_split = (int64_t)kDecodeWaves * kDecodeMinWaveKeys;
  return (int32_t)std::max<int64_t>(1, std::min(splits, ((int64_t)max_len + per_split - 1) / per_split));
}

}  // namespace

// Key ranges per (request, kv head, group of 16 query heads), each wave keeping at least
// kDecodeMinWaveKeys keys.  Head_dim 128: one workgroup alone on a compute unit streams about 36
// GB/s, so some 200 of the 256 reach the HBM's rate and what counts is that no compute unit gets one
// workgroup more than the others:
//  * up to 128 pairs, as many ranges as leave at most one workgroup per compute unit (a second one on
//    a few units costs as much as on all; rounded down / up, 16K keys: 72 pairs 88 / 124 us, 104 135 /
//    174, 136 207 / 251, 192 238 / 268, 248 305 / 309; 2K keys: 19 / 21, 25 / 30, 36 / 39, 36 / 41, 47 / 49);
//  * from 129 to 256, none;
//  * from 257 to 384, 4 of long enough ranges, equal contexts or not (whole / in 4, 10K keys, and 10K
//    of uneven length: 264 pairs 306 / 229 us and 235 / 191, 320 313 / 254 and 274 / 205, 384 325 / 304
//    and 286 / 245; of 4K keys 264 129 / 101 and 97 / 98, 384 139 / 135 and 127 / 134, hence the later line);
//  * beyond, none: uneven contexts even out by themselves (400 pairs of 4K keys 139 / 144, 520 205 / 185
//    but uneven 138 / 166, 776 281 / 267 but uneven 209 / 238).
// Head_dim 64 keeps up to four workgroups on a compute unit, which evens that out by itself (384
// pairs: 120 us whole, 137 us in 4), and each has half the bytes in flight: there the count is rounded
// up where rounding down leaves under 200 workgroups or one range (down / up, 4K keys, and 16K keys
// half as long at the shortest: 88 pairs 24.7 / 23.6 and 72 / 69 us, 136 41.9 / 35.1 and 131 / 101, 192
// 41.1 / 39.7 and 131 / 111, 224 45.2 / 43.3 and 134 / 122), and down elsewhere (72 pairs 18.6 / 19.4
// and 51 / 56, 104 27.0 / 26.6 and 74 / 74, 120 27.5 / 28.0 and 76 / 78).
int32_t decode_bf16_auto_splits(const AttnShape& s, int32_t max_len) {
  const int64_t pairs = decode_pairs(s);
  if (pairs > 256) {
    return s.head_dim == 128 && pairs <= 384 && max_len >= (pairs <= 352 ? 4096 : 6144) ? 4 : 1;
  }
  int64_t splits = pairs > 0 ? 256 / pairs : 1;
  if (s.head_dim == 64 && pairs > 0 && pairs < 256 && (splits == 1 || splits * pairs < 200)) ++splits;
  return decode_cap_splits(splits, max_len);
}

// Launches that fill the GPU unsplit: with no split count asked for they run without a workspace.
bool decode_bf16_may_run_whole(const AttnShape& s) {
  return decode_pairs(s) >= 256;
}

// Bytes for a call that leaves the split count to the library: at least what that count needs, and up
// to 256 pairs those of the rounded-up count.  A caller sizes one workspace for its largest batch,
// and counts rounded down leave too little there for a smaller one (88 pairs in 2 ranges need the
// room of 176, 64 pairs in 4 that of 256).
size_t decode_bf16_auto_workspace(const AttnShape& s, int32_t max_len) {
  int32_t splits = decode_bf16_auto_splits(s, max_len);
  const int64_t pairs = decode_pairs(s);
  if (pairs > 0 && pairs <= 256) splits = std::max(splits, decode_cap_splits((256 + pairs - 1) / pairs, max_len));
  return decode_bf16_workspace(s, max_len, splits);
}

size_t decode_bf16_workspace(const AttnShape& s, int32_t, int32_t n_splits) {
  if (n_splits <= 1) return 0;
  const size_t rows = (size_t)s.n_layers * s.batch * s.n_q_heads * n_splits;
  return rows * (s.head_dim + 2) * sizeof(float);
}

}  // namespace pic
