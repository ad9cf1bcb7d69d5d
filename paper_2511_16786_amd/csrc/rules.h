// Choices by size alone, for host and device (constexpr functions serve both) and without HIP, so that they can be
// compiled and checked by themselves.
#ifndef FC_RULES_H_
#define FC_RULES_H_

namespace fc {

// Half turns of the residual kernel's workgroups in a round of `units` units: two for each of an XCD's 32 compute units take
// its items, `windows` for each four units, one after the other.  The last turn of no more than 32 workgroups has a compute unit for
// each and is over in half the time.  Rounds of 36, 40, ... 76 units of 32768 tokens, M = 3072 (22 windows for an XCD):
// 158, 163, 187, 202, 207, 233, 246, 250, 279, 292, 318 us, 22.4 to 23.4 for each half turn.  An even number of them costs a
// little more, since the last ones share compute units: 33 against 32.
constexpr long long residual_cost(int units, int windows) {
  const long long halves = ((units + 3) / 4 * (long long)windows + 31) / 32;
  return halves * (halves % 2 ? 32 : 33);
}

// Units of a round of scoring, of at most `most`, `windows` as above: as few rounds as whole sets of four units (the
// residual kernel's waves) allow, alike or, where that makes the residual's turns fewer or their ends shorter, the last one
// shorter than the others.  Scoring, us by units of a round, equal ones first, the rule's choice marked:
//   112 units of 32768, M = 3072: 56 1074, *60 1051, 64 1049, 72 1054, 76 1092    128 of 24000, M = 3072: *64 960, 68 975, 72 977, 80 980
//   224 units of 16384, M = 3072: 76 1366, *80 1348           256 of 16384, M = 3072: *64 1536, 68 1573, 72 1557, 76 1585, 80 1573
//   100 units of  8000, M = 4096: *36 664, 40 671, 48 685      96 of 32768, M = 6144: *32 1170, 36 1194, 40 1204
// Units that fill up what whole sets leave of `most` are not worth a set begun: 30 units of 32768 tokens with 256 columns,
// M = 16384, most 6: eight rounds of 4 1510 us, five of 6 1588.
constexpr int round_units(int units, int most, int windows) {
  if (units <= most) return units;
  if (most < 4) return most;
  const int cap = most / 4 * 4, rounds = (units + cap - 1) / cap, equal = (units + 4 * rounds - 1) / (4 * rounds) * 4;
  int best = equal;
  long long least = 0;
  for (int c = equal; c <= cap && c < equal + 64; c += 4) {
    const int full = (units - 1) / c;                      // (rounds before the last: no more than as many as there have to be)
    const long long cost = full * residual_cost(c, windows) + residual_cost(units - full * c, windows);
    if (c == equal || cost < least) { best = c; least = cost; }
  }
  return best;
}

// The row kernels' work are rectangles, tiles or windows along one side and groups of units along the other.  Each of the 8 XCDs takes a
// rectangle of its own: neighbours along the first side share rows, weights and lines of the grid, which its L2 then holds.  The first
// side is cut for 2^xcds_along XCDs, all 8 if it can be, fewer where that makes the two kernels' largest rectangles smaller by
// more than a sixteenth: a short sequence has fewer tiles or windows than XCDs, or a few more.  The cut is the same for both, so that
// an XCD's L2 has the second kernel's rows where they fit (4 layers of 4096 tokens, cut for 8 and for 4: 43 us, both for 8 42).
// Scoring, us, cut for 8 always / now: 720 units of 1024 tokens, 64 columns 215 / 145, 128 of 512, 128 columns 51 / 40, 112 of 4096 205 /
// 184, 248 of 1938 219 / 204.  Where the second kernel's items, cut along the tokens, are all under way at once (at_once of an XCD), so they are
// as cut: a rectangle a few items larger costs it a second turn (41 units of 4869 tokens, 63 and 66 items where an XCD holds 64: 67.3 and 76.9 us, 82
// of 2731, 8 columns 36.4 and 43.3).
struct Sides { int first, second; };
constexpr int xcd_items(int along, Sides r) {               // of the largest rectangle
  return ((r.first + (1 << along) - 1) >> along) * ((r.second + (8 >> along) - 1) >> (3 - along));
}
constexpr int xcds_along(Sides a, Sides b, int at_once) {
  const long long all_a = (long long)a.first * a.second, all_b = (long long)b.first * b.second;
  int best = 3;
  long long least = xcd_items(3, a) * all_b + xcd_items(3, b) * all_a;
  const bool one_turn = xcd_items(3, b) <= at_once;
  for (int along = 2; along >= 0; --along) {
    if (one_turn && xcd_items(along, b) > at_once) continue;
    const long long cost = xcd_items(along, a) * all_b + xcd_items(along, b) * all_a;
    if (16 * cost < 15 * least) { best = along; least = cost; }
  }
  return best;
}
struct Span { int from, count; };
constexpr Span xcd_first(int xcd, int along, int first) {
  const int a = xcd & ((1 << along) - 1), from = first * a >> along;
  return {from, (first * (a + 1) >> along) - from};
}
constexpr Span xcd_second(int xcd, int along, int second) {
  const int b = xcd >> along, from = second * b >> (3 - along);
  return {from, (second * (b + 1) >> (3 - along)) - from};
}

// The slots (16-byte pieces of K and V rows) of a unit are dealt out to waves, 16 to each of its parts: as many waves as have one.  A
// lane past the last slot loads that one again, whose lines its wave takes anyway.  (When it loaded the first, which is K's, and waves
// came in powers of two, such widths read K twice and had waves without a slot.  fp32 scoring, us, before / after: 419 units of 7087 tokens, 40
// columns 834 / 715, 154 of 12032, 72 columns 869 / 733, 112 of 8192, 96 columns 452 / 400, 112 of 1024, 136 columns 123 / 94.)
constexpr int slot_waves(int slots) { return (slots + 15) / 16; }
constexpr int lane_slot(int part, int lane, int slots) { return part * 16 + lane < slots ? part * 16 + lane : slots - 1; }

// Tiles of the grid for a decimation wave: four, two or one.  Fewer of them read the rows under the seams again (1.75 times the rows with one);
// more make a wave's walk through the tokens longer, by half for two tiles where the tokens are many for a grid point, and workgroups
// fewer.  So it depends on what a launch waits for: its rows, or the longest walk, which weighs the less the more workgroups there
// are beside one another: 75 MB with 160 workgroups, 32 with 384 (fp32 86 with 256, 57 with 384).  Waves with empty lanes walk as long for fewer
// bytes, which count the less; sequences of less than 16 groups of tiles have most of their rows under seams.
// Workgroups' weights are to fit a compute unit's 160 KB of LDS twice (10 steps for four tiles, N/M up to 11; two tiles there:
// 519 instead of 473 us at 32768 tokens, M = 3072).
// Decimation alone, us, more tiles less fewer, mean of launches drawn at random (and the extremes), by workgroups of the more:
//   bf16, four or two: rows below 55 MB, 224 to 255 +2.2 (+0.3 .. 7.8), 256 to 383 +0.5 (-2.6 .. 5.2), 384 to 511 -1.6 (-4.5 .. 0.3); above, 224
//   to 255 0.0 (-2.0 .. 2.6), 256 to 383 -3.8 (-10.2 .. -0.1), 384 to 511 -4.8 (-8.4 .. -2.1).
//   bf16, two or one: below, 256 to 383 +1.1 (-0.2 .. 4.2), 384 to 511 0.0 (-4.1 .. 3.3); above, 128 to 159 +0.1 (-1.7 .. 3.1), 160 to 223 -1.3
//   (-4.1 .. 1.4), 224 to 255 -2.2 (-3.9 .. -1.2), 256 to 383 -2.7 (-5.5 .. 2.5), 384 to 511 -7.3 (-13.8 .. -3.2).
//   fp32, four or two: below, 384 to 511 +1.2 (-2.0 .. 3.4), 512 on +1.9 (-1.0 .. 6.2); above, 256 to 383 +4.5 (-0.5 .. 9.5), 384 to 511 -3.7 (-9.2
//   .. 2.1), 112 units of 8192 tokens 230 / 270.  Two or one: below, 256 to 511 +1.0 (-3.4 .. 3.6), 640 on -0.5 (-2.0 .. 1.2); above, 256 to 383
//   -1.3 (-4.4 .. 2.9), 384 to 511 -6.1 (-13.9 .. 1.8).
constexpr int decimate_tiles(int m, int groups, int steps, bool bf16, int slots, long long row_bytes) {
  const int lanes = 16 * slot_waves(slots);
  const long long carried = row_bytes / lanes * slots;
  for (int gt = 4; gt > 1; gt /= 2) {
    const int supers = m / 16 / gt;
    const long long workgroups = (long long)supers * groups;
    const bool rows_bound = carried * workgroups >= (bf16 ? 12000000000 : 22000000000) || (slots == lanes && supers < 16 && row_bytes >= 20000000);
    const int least = gt == 4 ? (bf16 ? (rows_bound ? 256 : 384) : (rows_bound ? 384 : 1 << 30))
                              : (bf16 ? (rows_bound ? 160 : 512) : (rows_bound ? 256 : 640));
    if (gt * steps * 2048 <= 80 * 1024 && workgroups >= least) return gt;
  }
  return 1;
}

// A window's tiles are cut in blocks, with a wave each, in launches that leave room for it.
constexpr int window_blocks(int tpw) { return tpw > 8 ? 4 : (tpw > 4 ? 2 : 1); }
constexpr int window_block(int tpw) { return (tpw + window_blocks(tpw) - 1) / window_blocks(tpw); }

// Waves of the residual kernel for a compute unit.  bf16 rows: eight, what it holds.  A wave of fp32 rows has half the columns and so half the
// registers: 16 are under way in launches of one segment for each (ONCE); others have nine, in whole workgroups, though it holds twelve.  Scoring, us, by
// workgroups of an XCD: of three waves, 64 and 96, 150 units of 9000 tokens, 72 columns 493 / 473; of four, 32, 64 and 96, 112 of 8192 555 / 507 /
// 513, 300 of 8192, 64 columns 727 / 672 / 679, 400 of 8192, 32 columns 496 / 465 / 473 (80 and 112, which compute units share
// unevenly, 5 % more); of five, 32, 64 and 96, 80 of 8192, 136 columns 467 / 469 / 474; of six, 50 of 8192, 192 columns 366 / 367 / 370.
// Where a fifth of the lanes of a unit's waves has no slot, workgroups of four are three: so much less is under way.  Two / three: 205 of
// 3840, 40 columns 293 / 283, 145 of 4096 203 / 197, 600 of 8192, 8 columns 423 / 393, 280, 48 columns 551 / 543; random launches,
// three over two, mean and extremes: 8 columns (12 of 16 lanes idle) 0.937 (0.89 .. 1.00), 40 (12 of 32) 0.984 (0.94 .. 1.02), 24 and 48 (a quarter)
// 0.993 (0.95 .. 1.02), but 104 (12 of 64) 1.002 (0.97 .. 1.04), 56 and 112 (an eighth) 1.002 (0.95 .. 1.03), 120 1.007 (0.96 .. 1.03).
// (Of three waves, three and four, 150 of 8192, 80 columns 469 / 507.)
constexpr int residual_waves(bool bf16, bool once, bool full) { return bf16 ? 8 : (once ? 16 : (full ? 9 : 12)); }
constexpr int residual_groups(bool bf16, bool once, int waves, int slots) {
  return 32 * (residual_waves(bf16, once, waves != 4 || 64 * slot_waves(slots) < 5 * slots) / (once && waves < 4 ? 4 : waves));
}

// Work of a residual launch: windows (wins, of tpw tiles) along one side, units abreast in a workgroup along the other; a unit has slots, and
// as many parts as slot_waves.  Workgroups of four waves take a unit each and its parts in turn, or (split) a unit's parts side by side, of five to
// eight waves where a unit has that many.
// Split is what leaves an XCD's compute units two workgroups each where four units for one do not.  fp32 rows are split in others too, in
// turn / side by side: 112 units of 8192 tokens 526 / 510 us, 154 of 12032, 72 columns 587 / 562, 50 of 9000, 256 columns 533 / 486, 36 of 16384,
// 64 columns 184 / 171, one of 55808 85 / 62 (three of four waves had no unit).  Not so where a window is a single tile, for each of which
// the waves would wait for one another: 50 of 8192, r = 3400 507 / 514, of 192 columns 760 / 847, 275 of 507, r = 163 164 / 178.
// In launches that leave room for it each block of a window's tiles, of each part, has a wave of its own: all of them resident at
// once (eight waves a compute unit), as workgroups of four to eight.  Scoring, us, a wave for a window / for a block: 8 units of 1381 tokens,
// 64 columns (13 tiles) 30.4 / 23.1, 16 of 3697 38.7 / 28.4, 20 of 2304 38.5 / 33.3, 8 of 1024 27.3 / 24.8, 2 of 512 in fp32
// (6 tiles) 21.3 / 20.0; windows of three tiles cut in two 26.7 / 27.4, so four are left whole.
struct ResidualPlan {
  int waves, abreast, blocks;         // of a workgroup; units side by side; of a window's tiles (1: a wave takes them all)
  bool split, once;                   // parts side by side; no more than one segment for each wave
  int along, workgroups;              // the XCDs' cut; of an XCD
};
constexpr ResidualPlan residual_plan(int wins, int tpw, int slots, int units, Sides dec, bool bf16) {
  const int parts = slot_waves(slots), blocks = window_blocks(tpw), unit_waves = parts * blocks, block_waves = unit_waves > 4 ? unit_waves : 4;
  const int block_units = block_waves / unit_waves > 1 ? block_waves / unit_waves : 1;
  const Sides small{wins, (units + block_units - 1) / block_units}, fours{wins, (units + 3) / 4};
  if (blocks > 1 && unit_waves <= 8) {
    const int at_once = 32 * (8 / block_waves), along = xcds_along(dec, small, at_once), items = xcd_items(along, small);
    if (items <= at_once) return {block_waves, block_units, blocks, parts > 1, true, along, items};
  }
  const bool many = xcd_items(xcds_along(dec, fours, 64), fours) >= 64, idle = 16 * fours.second > 5 * units;    // (a fifth of the waves)
  const bool split = parts > 1 && !(many && (bf16 || (tpw == 1 && !idle)));
  const int abreast = split ? (parts < 4 ? 4 / parts : 1) : 4, waves = split ? abreast * parts : 4;
  const Sides all{wins, (units + abreast - 1) / abreast};
  const int held = residual_groups(bf16, false, waves, slots), held_once = residual_groups(bf16, true, waves, slots);
  const int along = xcds_along(dec, all, split || parts == 1 ? held_once : held), items = xcd_items(along, all);
  const bool once = (split || parts == 1) && items <= held_once;
  return {waves, abreast, 1, split, once, along, once || items < held ? items : held};
}

// Whether the row kernels read a round's rows with a claim on the last-level cache.  Rows that fit it are found there on their second
// reading; of others it is left to the grid.  Scoring, us, kept / not kept: 246 MB of rows 168 / 182, 268 MB 234 / 232, 470 MB 413 /
// 377, 738 MB 516 / 457; 34 MB 50 / 60.  fp32: 940 MB 575 / 558, 560 MB 1093 / 1040 (in rounds), 34 MB 114 / 126, 7 MB 38 / 44.
// Rows that are not whole lines of 128 bytes are kept whatever their size: a line is asked for by the rows or waves that share it, and read
// past the cache it is often gone by then.  fp32 rows of 8192 tokens, r = 820, kept / not kept: 8 columns 577 / 607, 24 396 / 436, 40 521 / 559, 248 295 /
// 314, but 32 504 / 477, 96 370 / 358, 160 395 / 383, 224 430 / 415; bf16: 8 columns 658 / 677, 24 448 / 481, 72 634 / 689, 136 571 / 604.
constexpr bool round_keeps_rows(long long round_bytes, int row_bytes) { return row_bytes % 128 != 0 || round_bytes <= 256 * 1000 * 1000; }

// Workgroups of a selection that copies the rows as well, 0: the copying is a launch of its own.  Those with an index set in common all make
// the selection, so that there must be compute units to spare, and their own share of rows has to be short, since a workgroup copies it
// alone, a 16-byte vector of K and of V a thread and turn: four turns at most, two and a half where each first looks a page up, and
// 112 KB read and written.  The heads' scores of a shared set are read by each of its workgroups, 40 MB of them at most.
// Two launches / one, us, with the bytes that a workgroup copies: 2 sets of 512 tokens (6 KB) 8.3 / 5.8, 16 of 4096 (52) 10.2 /
// 8.5, 16 of 1280 (28) 8.7 / 6.5, 64 of 2048 (52) 9.6 / 7.8, 4 of 16384 (105) 11.6 / 11.0, 32 of 8192 (105) 13.2 / 12.4; 4 of 4096, heads'
// rows alike (209) 10.8 / 13.1, 8 of 16384 (315) 17.3 / 19.3; 128 of 512 (92) 11.3 / 12.3.  One less two, launches drawn at random, up to 112 KB,
// mean and extremes by turns: packed, 2 to 3 -1.0 (-1.6 .. -0.2), 3 to 4 -0.8 (-2.1 .. -0.1), 4 to 5 -0.3 (-0.7 .. 0.3), 5 to 7 +0.4 (-0.5 .. 0.8);
// paged, 1.5 to 2 -1.2 (-3.0 .. 0.1), 2 to 2.5 -0.7 (-1.2 .. -0.1), 2.5 to 3 -0.2 (-1.9 .. 0.8), 3 to 5 +0.5 (-1.2 .. 1.5), 5 to 7 +2.6 (1.3 .. 3.9);
// by the scores read: 20 to 30 MB -1.1 (-1.9 .. -0.5), 30 to 40 -0.6 (-1.6 .. 0.1), 40 to 50 +0.2 (-1.0 .. 2.2), more +1.7 (0.2 .. 4.0).
constexpr int select_threads(int n) { return n <= 1024 ? 256 : (n <= 4096 ? 512 : 1024); }    // (of its workgroups, up to 32768 tokens)
constexpr int copy_groups(int lists, int layers, int n, int heads, long long rows, int vec_per_row, bool paged) {
  if (n > 16384 || lists > 64) return 0;
  const int of_list = 256 / lists < 16 ? 256 / lists : 16, groups = lists * of_list, sharing = layers == 1 ? groups : groups - lists;
  const long long vectors = rows * vec_per_row, a_turn = (long long)sharing * select_threads(n);
  if (64 * vectors > (long long)sharing * (112 << 10) || 2 * vectors > (paged ? 5 : 8) * a_turn) return 0;
  return heads > 1 && 4LL * groups * heads * n > 40000000 ? 0 : groups;
}

// The grid transforms' LDS has a free place after each `group` of points, point i is at i + i / group.  Whether the points of a butterfly, t R + q after the
// first pass (done = 1) and t / done * done R + t % done + q done after others, are at the place of the first and that of q, or q done, alone:
// their sum must not reach into a group's next one.
constexpr bool pads_apart(int radix, int done, int group) {
  return done == 1 ? group % radix == 0 || radix % group == 0 : done % group == 0;
}

// Where the grid begins in its region of a workspace, both at multiples of 256 bytes: an odd multiple, whatever the
// workspace's own address is.  A grid at a multiple of 512 costs the residual kernel a tenth where M is a power of two (28 layers of
// 4096 tokens, M = 4096: 182 us at 128, 256, 768, 1280 and 2304 bytes past a multiple of 4096, 204 at 0 and 512).
constexpr unsigned long long kGridSlack = 256;
constexpr unsigned long long grid_start(unsigned long long at) { return at | kGridSlack; }

// Decode: whether a sequence's layers are worked on by falling budget, `rows` being the sum of their budgets.  Worth its
// while where pieces are long, of K rows of 72 KiB and more by the mean budget; with shorter ones the ranking is what
// counts.  By number / by budget, us, and a piece's rows: 28 layers of 4 heads, bf16, 128 columns, one sequence, 728 rows
// 70.6 / 67.4, through tables 80.7 / 71.5, 349 rows 35.1 / 34.6, 194 rows 23.0 / 24.7; eight sequences, through tables, 819
// rows 147 / 137, 354 rows 68.8 / 66.1, 150 rows 38.8 / 41.2, packed, 326 rows 59.5 / 56.6, 300 rows 49.6 / 50.9, 279 rows
// 45.6 / 47.8; 64 columns, 697 rows 37.7 / 34.1, 598 rows 49.1 / 47.5, 523 rows 43.5 / 42.6, 480 rows 39.9 / 40.2, 387 rows
// 23.1 / 24.1; fp32, 163 rows 58.5 / 56.1, 130 rows 45.7 / 45.8, 120 rows 42.3 / 45.4.
constexpr bool ranks_by_budget(long long rows, int layers, int splits, int row_bytes) {
  return rows * row_bytes >= (72LL << 10) * layers * splits;
}

// Decode: whether a launch's rows, of K and as many of V, fit the last-level cache (256 MB) from one step to the next and claim it;
// else they are read past it.  Kept / not kept, us: 1.5 GB of fp32 280 / 252, 0.75 GB 158 / 143, 0.38 GB of bf16 78 / 74; 26 MB from
// step to step 16.1 / 17.6.
constexpr bool keeps_rows(long long rows, int row_bytes) { return 2 * rows * row_bytes <= 256000000; }

}  // namespace fc
#endif
