// Whether a prompt's attention walks whole rows, against measured times of both forms (us, MI355X; 256 compute units): sizes where one
// is at least 1.3 times as fast.  No GPU, no HIP.
#include <cstdio>

#include "../../paper_2410_17375_amd/csrc/amusd_plan.h"

struct Point {
    bool bf16;
    int head_dim, group, kv_heads, rows, keys, chunk, run_blocks, stretch;
    double whole, split;
};
static const Point points[] = {
    {false, 64, 4, 2, 1500, 1500, 64, 2, 256, 82, 54},
    {false, 64, 4, 2, 900, 900, 64, 2, 256, 51, 35},
    {false, 64, 4, 8, 2000, 2000, 512, 16, 512, 170, 250},
    {false, 64, 4, 8, 250, 250, 32, 1, 256, 19, 34},
    {false, 64, 4, 2, 1500, 3000, 64, 2, 256, 161, 109},
    {false, 64, 4, 8, 17, 817, 32, 1, 256, 51, 28},
    {false, 64, 8, 4, 250, 750, 256, 16, 256, 63, 34},
    {false, 64, 8, 4, 250, 750, 16, 1, 256, 79, 58},
    {false, 64, 8, 4, 500, 600, 16, 1, 256, 64, 99},
    {false, 64, 8, 4, 250, 250, 16, 1, 256, 29, 44},
    {false, 64, 8, 4, 61, 861, 16, 1, 256, 87, 47},
    {false, 64, 8, 4, 600, 4600, 256, 16, 256, 369, 239},
    {false, 128, 4, 8, 128, 378, 160, 5, 160, 37, 26},
    {false, 128, 4, 8, 350, 1350, 160, 5, 160, 120, 90},
    {false, 128, 4, 4, 180, 180, 32, 1, 256, 24, 34},
    {false, 128, 4, 4, 500, 600, 32, 1, 256, 68, 91},
    {false, 128, 4, 4, 350, 1350, 32, 1, 256, 147, 81},
    {false, 128, 4, 4, 40, 540, 32, 1, 256, 60, 40},
    {false, 128, 8, 4, 2000, 3500, 256, 16, 256, 704, 1039},
    {false, 128, 8, 4, 600, 600, 256, 16, 256, 88, 145},
    {false, 128, 8, 4, 400, 1900, 256, 16, 256, 265, 181},
    {false, 128, 8, 4, 61, 14061, 256, 16, 256, 1918, 172},
    {true, 64, 4, 8, 900, 900, 192, 3, 192, 24, 43},
    {true, 64, 4, 8, 500, 750, 64, 1, 256, 22, 34},
    {true, 64, 4, 2, 17, 4017, 128, 2, 256, 75, 12},
    {true, 64, 4, 8, 61, 1561, 512, 8, 512, 29, 18},
    {true, 64, 8, 4, 1000, 2500, 256, 8, 256, 61, 114},
    {true, 64, 8, 4, 1000, 9000, 256, 8, 256, 204, 309},
    {true, 64, 8, 4, 1500, 1500, 256, 8, 256, 39, 109},
    {true, 64, 8, 4, 2000, 2500, 96, 3, 192, 90, 190},
    {true, 64, 8, 4, 61, 1561, 256, 8, 256, 35, 15},
    {true, 64, 8, 4, 250, 14250, 256, 8, 256, 286, 128},
    {true, 128, 4, 8, 2000, 4000, 192, 3, 192, 224, 387},
    {true, 128, 4, 32, 128, 1128, 576, 9, 576, 33, 43},
    {true, 128, 4, 8, 61, 1561, 192, 3, 192, 44, 19},
    {true, 128, 4, 8, 180, 1680, 64, 1, 256, 64, 47},
    {true, 128, 8, 1, 1000, 1500, 64, 2, 256, 52, 74},
    {true, 128, 8, 1, 900, 1400, 64, 2, 256, 48, 72},
    {true, 128, 8, 8, 128, 228, 32, 1, 256, 17, 30},
    {true, 128, 8, 8, 250, 500, 32, 1, 256, 29, 67},
    {true, 128, 8, 1, 350, 4350, 64, 2, 256, 136, 54},
    {true, 128, 8, 1, 128, 1628, 64, 2, 256, 54, 24},
};

// Whether a verify pass's attention is tiles of (row, head) pairs or a tile per head, against measured times of a pass of two layers (us; of four below):
// sizes that differ by 1 % and more.
struct Pass {
    bool bf16;
    int head_dim, group, units;
    double tiles;
    int run_blocks;
    double pairs, heads;
};
static const Pass passes[] = {
    {true, 64, 4, 16, 1, 1, 194.4, 199.8},       {true, 64, 4, 256, 2, 8, 122.1, 124.2},      {true, 64, 4, 224, 4, 4, 131.7, 135.1},
    {true, 64, 4, 808, 1, 4, 231.7, 268.6},      {true, 64, 4, 280, 1.5, 16, 142.6, 165.0},   {true, 64, 8, 256, 6, 16, 154.6, 152.3},
    {true, 64, 8, 220, 8, 4, 141.2, 143.8},      {true, 128, 4, 128, 2, 2, 207.9, 211.0},     {true, 128, 4, 256, 2, 6, 219.4, 224.8},
    {true, 128, 4, 256, 4, 6, 241.6, 238.1},     {true, 128, 4, 280, 1.5, 16, 259.9, 300.8},  {true, 128, 4, 1552, 1, 4, 298.8, 343.8},
    {true, 128, 8, 220, 1, 4, 201.9, 207.5},     {true, 128, 8, 252, 4, 8, 219.0, 222.8},     {true, 128, 8, 220, 6, 4, 237.6, 233.5},
    {true, 128, 8, 252, 8, 8, 252.8, 246.9},     {false, 64, 4, 256, 1, 7, 155.9, 163.3},     {false, 64, 4, 256, 4, 16, 202.2, 196.6},
    {false, 64, 8, 252, 4, 16, 175.0, 188.9},    {false, 64, 8, 252, 8, 16, 211.0, 202.5},    {false, 128, 4, 168, 2, 3, 363.9, 357.6},
    {false, 128, 4, 232, 1.45, 5, 372.6, 382.0}, {false, 128, 4, 256, 3, 16, 439.7, 430.8},   {false, 128, 4, 656, 1, 5, 387.7, 431.7},
    // more units than compute units, and the most rows a unit then has: a window of 13 rows and three of one
    {true, 64, 4, 464, 1.83, 4, 248.7, 262.6},   {true, 64, 8, 448, 2.71, 1, 234.8, 246.8},   {true, 128, 4, 456, 1.84, 1, 229.9, 233.2},
    {true, 128, 8, 448, 2.71, 1, 229.6, 234.8},  {false, 64, 4, 456, 1.84, 2, 130.1, 136.7},  {false, 64, 8, 448, 2.71, 2, 132.8, 142.1},
    {false, 128, 4, 456, 1.84, 4, 164.5, 176.2}, {false, 128, 8, 448, 2.71, 2, 219.7, 235.2},
    // 16-bit heads of 64 in short runs, many rows
    {true, 64, 4, 104, 4, 2, 210.8, 214.6},      {true, 64, 4, 32, 4, 2, 205.0, 212.9},       {true, 64, 8, 104, 8, 2, 217.0, 223.2},
    {true, 64, 8, 128, 8, 1, 226.2, 234.4},      {true, 64, 8, 244, 4.67, 1, 233.4, 240.8},   {true, 64, 4, 248, 2.55, 4, 235.7, 241.1},
};

extern "C" int whole_rows(int bf16, int head_dim, int group, int kv_heads, int rows, int keys, int cus, int chunk, int run_blocks, int stretch) {
    return amusd::pf_attention_walks_whole_rows(bf16, head_dim, group, kv_heads, rows, keys, cus, chunk, run_blocks, stretch);
}

int main() {
    int wrong = 0;
    for (const Point& p : points) {
        const bool whole = amusd::pf_attention_walks_whole_rows(p.bf16, p.head_dim, p.group, p.kv_heads, p.rows, p.keys, 256, p.chunk, p.run_blocks, p.stretch);
        if (whole == (p.whole < p.split)) continue;
        std::printf("%s, heads of %d in groups of %d, %d kv heads, %d rows, %d keys: %.0f us, the other form %.0f\n", p.bf16 ? "bf16" : "float32", p.head_dim,
                    p.group, p.kv_heads, p.rows, p.keys, whole ? p.whole : p.split, whole ? p.split : p.whole);
        ++wrong;
    }
    for (const Pass& p : passes) {
        const bool pairs = amusd::attention_packs_rows(p.bf16, p.head_dim, p.group, p.units, p.tiles, p.run_blocks, 256);
        if (pairs == (p.pairs < p.heads)) continue;
        std::printf("verify pass, %s, heads of %d in groups of %d, %d units, %.2f tiles, %d blocks: pairs %.1f us, heads %.1f\n", p.bf16 ? "bf16" : "float32",
                    p.head_dim, p.group, p.units, p.tiles, p.run_blocks, p.pairs, p.heads);
        ++wrong;
    }
    // groups of 1 and 2 have no such kernel
    for (int group = 1; group <= 2; ++group) wrong += amusd::pf_attention_walks_whole_rows(true, 64, group, 8, 2000, 2000, 256, 64, 1, 256);
    std::printf(wrong ? "WRONG\n" : "OK\n");
    return wrong != 0;
}
