// ra_plan.h -- how the query tiles of an attention call are divided between
// kernels (plain C++ on sizes, so it is also checked without a GPU).
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
// kernel.  Measured, kv_block 64, 8 waves / 4 waves / key-split: 7 tiles (1560
// tokens, 1 head) 49 / 39 / 33 us; 42 tiles 54 / 44 / 38; 84 tiles 58 / 48 / 52;
// 126 tiles 61 / 51 / 55; 168 tiles 62 / 64 / 82; 320 tiles (20280 tokens, 4
// heads) 1043 / 1001 / 862 us.
// Heads of an odd number of 128-query tiles leave half of their last 256-query
// tile empty.  Where that starts one round more than the 128-query tiles alone
// take (two workgroups a unit at kv_block 64; at 128 the tiles of one workgroup
// fill the LDS), all run on 4 waves.  Measured, the attention alone, divided
// tiles / all on 4 waves: 64 tokens, 640 heads 22.7 / 14.2 us; 384 tokens, 129
// heads 28.2 / 17.7; 1560 tokens, 37 heads 80 / 55; 4224 tokens, 31 heads 323 /
// 270.  Where both take the same rounds the two are alike below 1000 tokens and
// the 8 waves faster above (4224 tokens, 48 heads 457 / 471 us).
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

}  // namespace ra
