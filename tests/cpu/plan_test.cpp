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
    // groups of 1 and 2 have no such kernel
    for (int group = 1; group <= 2; ++group) wrong += amusd::pf_attention_walks_whole_rows(true, 64, group, 8, 2000, 2000, 256, 64, 1, 256);
    std::printf(wrong ? "WRONG\n" : "OK\n");
    return wrong != 0;
}
