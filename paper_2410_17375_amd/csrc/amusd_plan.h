// Choices between forms of a stage that follow from sizes alone.  Host code, no GPU needed.
#pragma once

namespace amusd {

// Attention of a prompt's rows: a workgroup per row tile and kv head that walks all keys (whole), or the keys split into
// stretches and the chunks' partials merged.
//
// The whole form takes, per 1000 keys, `alone` us while each of its workgroups has a compute unit for itself (the last tile's
// walk is its time), and `two` where some share one (a middling tile's; the longest begin first).  The split form fills the
// chip whatever the number of tiles: `split` us per 1000 keys and workgroup of the whole form per compute unit, the partials
// (stored and read back at 7.5 TB/s) on top, and a stretch and 2 us for its ends.  A key block at the end of an odd run takes
// 0.75 of a step of two.  From 1.9 workgroups a compute unit on the whole form is the faster one for any number of keys.
// Measured (MI355X, 1521 prompts of 17 to 2000 rows behind 0 to 14000 keys, 1 to 32 kv heads, the eight forms, contexts of 1000
// to 16384): the choice is 0.4 % from the better form on average, 20 % and more in six.  whole / split us: heads of 64 in fours,
// 8 kv heads, 768 rows behind 8000 keys 185 / 152, float32 622 / 465; in eights, 4 kv heads, 192 / 233; heads of 128 in fours, 250
// rows behind 1500 43 / 32, 600 rows behind none 22 / 55.
inline bool pf_attention_walks_whole_rows(bool bf16, int head_dim, int group, int kv_heads, int rows, int keys, int cus, int chunk, int run_blocks,
                                          int stretch) {
    struct Rates { double alone, two, split; };
    static const Rates rates[2][2][2] = {{{{48, 72, 30}, {76, 136, 70}}, {{81, 136, 69}, {137, 274, 158}}},      // float32: heads of 64, 128,
                                         {{{15, 20, 7}, {17, 38, 18}}, {{19, 28, 14}, {26, 56, 33}}}};           // in fours, eights
    if (group != 4 && group != 8) return false;
    const Rates& r = rates[bf16][head_dim == 128][group == 8];
    const int wgs = (rows + 15) / 16 * kv_heads;
    const double per_cu = (double)wgs / cus;
    if (per_cu >= 1.9) return true;
    const bool pairs = run_blocks == 1 && group == 4 && head_dim == 64;       // a chunk's two runs in one step
    const double odd = run_blocks % 2 && !pairs ? (run_blocks - 1 + 2 * 0.75) / run_blocks : 1.;
    const double partials = 1000. / chunk * 16 * group * wgs * (head_dim + 4) * 8 / 7.5e6;
    const double whole = per_cu <= 1 ? keys * r.alone * odd : (keys - 0.4 * rows) * r.two * odd;    // ns
    const double split = keys * (per_cu * r.split * odd + partials);
    return whole <= split + r.alone * stretch + 2000;
}

// Attention of a verify pass, groups of 4 or 8 heads: tiles of (row, head) pairs (true) or a tile per head, whose units are one
// (kv head, chunk) each.  units: of the latter; tiles: of pairs, per chunk on average; run_blocks: key blocks of a wave's run.
//
// A tile per head is a workgroup a compute unit, round after round, over blocks that are staged once for all heads.  Pairs need
// fewer products while rows are few, and their workgroups share a compute unit; with many rows each tile fetches the keys for
// itself.  So pairs
//   where there is more than one round (168 sizes of the eight forms: all faster, by 0.2 to 154 us a layer.  Many rows to a unit do
//     not occur there, as it takes three sequences and a pass has 16 rows: at most 0.47 tiles a head);
//   up to half as many tiles as heads (float32 heads of 128, twice the registers a block: fewer);
//   and for 16-bit heads of 64 in runs of up to 7 blocks whatever the rows: both of a unit's forms are then mostly its beginning and
//     end (40 sizes, 0.8 us a layer less in the mean, 0.8 more at most; with 8 and more blocks and every compute unit taken
//     1.2 more: 16 rows behind 16360 keys 18.8 / 20.0).
// The line holds for full contexts, whose units are about the compute units.  With fewer than 200 of 256 pairs were faster for any number
// of rows (191 sizes that this takes a tile per head for, 0.2 us a layer slower at worst, 1 to 10 faster in the mean of a form): not made use of.
// Measured (MI355X): the attention's and the O-projection's kernels over 990 sizes, 1 to 8 sequences of 1 to 16 rows behind 100 to 16360
// keys; where the rule says pairs they are 1 us a layer slower at worst.  Whole passes of 2 layers, us, tile per head / pairs: 8B, 8 rows
// behind 2000 keys 211 / 208, behind 12000 224 / 219, 16 rows 238 / 241; 8 sequences of one row to 4000 260 / 235; heads in eights, 12 rows
// behind 7000 234 / 238; float32, 8 rows behind 2000 359 / 365, 2 rows behind 7000 391 / 375; 1B (4 layers), 16 rows behind 4000 236 / 229.
inline bool attention_packs_rows(bool bf16, int head_dim, int group, int units, double tiles, int run_blocks, int cus) {
    if (units > cus) return true;
    if (tiles <= group * (head_dim == 128 && !bf16 ? 0.375 : 0.5)) return true;
    return bf16 && head_dim == 64 && run_blocks < 8;
}

}  // namespace amusd
