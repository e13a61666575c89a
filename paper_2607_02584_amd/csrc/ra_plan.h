// ra_plan.h -- how the query tiles of an attention call are divided between
// kernels (plain C++ on sizes, so it is also checked without a GPU).  `units` is
// the number of compute units of the device: 256 on a whole chip, where the
// figures below were measured, a fraction of it on a partition of one.
#pragma once

namespace ra {

// Tiles of 256 queries, in the order of the list (head by head): `whole` on
// 8-wave workgroups, then `halves` as two 4-wave workgroups each, then
// `quarters` as four key-split workgroups each.  Or, with tiles128, that many
// tiles of 128 queries, all on 4-wave workgroups.
struct TilePlan {
  int whole, halves, quarters, tiles128;
};

// The 16-bit fallback.  Whole rounds of 256-query workgroups, one per compute
// unit, on the 8-wave kernel; a last round of up to half the units on 128-query
// workgroups of 4 waves (one wave per SIMD), of up to a quarter on the key-split
// kernel.  The attention alone, 8 waves / 4 waves / key-split, at kv_block 64: 1024
// tokens, 64 tiles 29.3 / 22.4 / 18.8 us, 72 tiles 29.2 / 22.5 / 24.9, 128 tiles
// 29.9 / 23.4 / 26.8; 30720 tokens, 40 tiles after five rounds 5227 / 4902 / 4747.
// At kv_block 128: 64 tiles 29.0 / 24.7 / 19.9 us, 72 tiles 29.1 / 24.9 / 37.5, 128
// tiles 29.6 / 25.7 / 37.8; 40 tiles after five rounds 5159 / 5009 / 4743.  From 129
// tiles on two smaller workgroups would share a unit (168 tiles of 1560 tokens, the
// whole forward, kv_block 64: 62 / 64 / 82 us).
// Heads of an odd number of 128-query tiles leave half of their last 256-query
// tile empty.  Where that starts one round more than the 128-query tiles alone
// take (two workgroups a unit at kv_block 64; at 128 the tiles of one workgroup
// fill the LDS), all run on 4 waves.  Measured, the attention alone, divided
// tiles / all on 4 waves: 64 tokens, 640 heads 22.7 / 14.2 us; 384 tokens, 129
// heads 28.2 / 17.7; 1560 tokens, 37 heads 80 / 55; 4224 tokens, 31 heads 323 /
// 270.  Where both take the same rounds the 8 waves are the faster from about 1000
// tokens on (1024 tokens, 65 heads 56.6 / 58.8 us); below, 4 waves take up to 13 %
// less (256 tokens, 340 heads 26.8 / 23.3), which this rule leaves.
inline TilePlan plan_fallback(int npad, int bh, int kv_block, int units) {
  const int total = (npad + 255) / 256 * bh, total128 = npad / 128 * bh;
  TilePlan p{0, 0, 0, 0};
  if (kv_block == 64 && (total128 + 2 * units - 1) / (2 * units) < (total + units - 1) / units) {
    p.tiles128 = total128;
    return p;
  }
  const int rest = total % units;
  if (4 * rest <= units) p.quarters = rest;
  else if (2 * rest <= units) p.halves = rest;
  p.whole = total - p.quarters - p.halves;
  return p;
}

// The FP6 kernels of the E2M3 container.  Whole rounds of 256-query tiles, one
// workgroup per compute unit, run on the 8-wave kernel.  A last round of at most
// half the units would leave the others idle: its tiles run in smaller workgroups,
// in four on the key-split kernel (kv_block 128) while that is at most one
// workgroup a unit, in two of 4 waves above that (one wave per SIMD).  The
// attention alone, 8 waves / halves / quarters, at kv_block 128: 1024 tokens, 64
// tiles 24.8 / 21.2 / 17.5 us, 72 tiles 24.9 / 21.1 / 21.2; 7680 tokens, 120 tiles
// 125 / 101 / 105; 30720 tokens, 104 tiles after a round 898 / 820 / 831, with Q
// smoothing 1019 / 942 / 987, with per-token K scales 1162 / 1060 / 1050, so those
// stay on quarters.  At kv_block 64 (no key-split kernel): 1024 tokens, 8 tiles
// 29.4 / 25.8, 128 tiles 30.8 / 27.2; 30720 tokens, 104 tiles after a round 1183 /
// 1097.  Above half the units both lose (186 tiles of 7800 tokens, the whole
// forward: 161 / - / 224 us).
inline TilePlan plan_e2m3(int npad, int bh, int kv_block, bool k_per_token, int units) {
  const int total = (npad + 255) / 256 * bh, rest = total % units;
  const int split_max = kv_block != 128 ? 0 : (k_per_token ? units / 2 : units / 4);
  TilePlan p{0, 0, 0, 0};
  if (rest <= split_max) p.quarters = rest;
  else if (rest <= units / 2) p.halves = rest;
  p.whole = total - p.quarters - p.halves;
  return p;
}

}  // namespace ra
