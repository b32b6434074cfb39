// Prefill pass for gfx950: up to kPfMaxRows prompt tokens of one sequence through the decoder at once.
//
// The verify pass serves 16 rows and is bound by streaming the weights; a prompt that goes through it 8 rows at a time
// streams all weights n/8 times (8B shape: 3.07 ms per 8 tokens).  Here a weight fragment that has been fetched is used
// for 64 rows of a wave, and the pass is bound by the matrix cores.
//
// A row gets the same bits as in the verify pass, whatever the number of rows: an output element is, as there, eight
// chains of 16x16 matrix instructions over the same K slices in the same order (k_slice), each for the hi and the lo
// halves of the activations, W.hi + W.lo added per slice, slices added in wave order.  What eight waves do there side by
// side a wave does here one after the other, with the slice's two sums and the total in registers.  The order inside a
// slice depends on the tile (its workgroup there), so a workgroup here takes tiles whose walks start alike: tile lists
// ordered by that start are made once per model.
#include <algorithm>
#include <array>
#include <utility>
#include <vector>

#include "amusd_attention.h"
#include "amusd_plan.h"

namespace amusd {

// ---------------------------------------------------------------- operand layout of the pass's activations
// [128-row block][K block][16-row tile of the block][hi, lo][64 lanes][EPL]: what a workgroup stages per K block is
// contiguous.
template <class DT>
struct PfAct {
    static constexpr int AF = DT::HAS_LO ? 2 : 1;
    static constexpr int kBlockTiles = kPfBlockRows / 16;
    // 16-byte fragment index of lane 0 of (row tile, K block, part)
    static __device__ __forceinline__ size_t frag(int kblocks, int rt, int kb, int part) {
        return ((((size_t)(rt / kBlockTiles) * kblocks + kb) * kBlockTiles + rt % kBlockTiles) * AF + part) * 64;
    }
    // two neighbouring columns (col even) of one row
    static __device__ __forceinline__ void store2(void* buf, int kblocks, int row, int col, float x0, float x1) {
        const int kb = col / DT::KB, g = (col % DT::KB) / DT::EPL, e = col % DT::EPL;
        const size_t at = (frag(kblocks, row >> 4, kb, 0) + g * 16 + (row & 15)) * DT::EPL + e;
        if constexpr (DT::HAS_LO) {
            const uint32_t h0 = bf16_rne(x0), h1 = bf16_rne(x1);
            const uint32_t l0 = bf16_rne(x0 - bf16_to_f32(h0)), l1 = bf16_rne(x1 - bf16_to_f32(h1));
            uint16_t* b = reinterpret_cast<uint16_t*>(buf);
            *reinterpret_cast<uint32_t*>(b + at) = h0 | (h1 << 16);
            *reinterpret_cast<uint32_t*>(b + at + 64 * DT::EPL) = l0 | (l1 << 16);
        } else {
            *reinterpret_cast<float2*>(reinterpret_cast<float*>(buf) + at) = float2{x0, x1};
        }
    }
    // four neighbouring columns (col a multiple of 4) of one row
    static __device__ __forceinline__ void store4(void* buf, int kblocks, int row, int col, v4f x) {
        const int kb = col / DT::KB, g = (col % DT::KB) / DT::EPL, e = col % DT::EPL;
        const size_t at = (frag(kblocks, row >> 4, kb, 0) + g * 16 + (row & 15)) * DT::EPL + e;
        if constexpr (DT::HAS_LO) {
            uint32_t h[4], l[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = bf16_rne(x[i]);
                l[i] = bf16_rne(x[i] - bf16_to_f32(h[i]));
            }
            uint16_t* b = reinterpret_cast<uint16_t*>(buf);
            *reinterpret_cast<uint2*>(b + at) = uint2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
            *reinterpret_cast<uint2*>(b + at + 64 * DT::EPL) = uint2{l[0] | (l[1] << 16), l[2] | (l[3] << 16)};
        } else {
            *reinterpret_cast<v4f*>(reinterpret_cast<float*>(buf) + at) = x;
        }
    }
    static __device__ __forceinline__ void store1(void* buf, int kblocks, int row, int col, float x) {
        const int kb = col / DT::KB, g = (col % DT::KB) / DT::EPL, e = col % DT::EPL;
        const size_t at = (frag(kblocks, row >> 4, kb, 0) + g * 16 + (row & 15)) * DT::EPL + e;
        if constexpr (DT::HAS_LO) {
            const uint32_t h = bf16_rne(x), l = bf16_rne(x - bf16_to_f32(h));
            reinterpret_cast<uint16_t*>(buf)[at] = (uint16_t)h;
            reinterpret_cast<uint16_t*>(buf)[at + 64 * DT::EPL] = (uint16_t)l;
        } else {
            reinterpret_cast<float*>(buf)[at] = x;
        }
    }
};

// ---------------------------------------------------------------- contraction
template <int STAGE>
struct PfWalk;
template <> struct PfWalk<kPfQKV> { using T = KWalkQKV; };
template <> struct PfWalk<kPfOproj> { using T = KWalkOproj; };
template <> struct PfWalk<kPfGateUp> { using T = KWalkWide; };
template <> struct PfWalk<kPfDown> { using T = KWalkDown; };
template <> struct PfWalk<kPfLMHead> { using T = KWalkWide; };
// A split stage of the verify pass walks by the index of its workgroup in the pair's K ranges, not by its tile's as here:
// the two are the same walk only while the workgroup does not shift it.
static_assert(KWalkDown::kRotWg == 0, "the prefill pass would start the down projection's slices elsewhere than the verify pass");

// Slices first .. last - 1 of a contraction, block by block: slice s is that of wave s mod 8 of the verify pass, in K range
// s / 8 of those that pairs of its workgroups share (kh blocks each).  Kept as straight stretches, so that the step to the
// next block, which every block's loads wait for, is an addition.
template <class Walk>
struct KSequence {
    int kh, wg, s, last, kb = 0, run = 1, stride = 0, rest = 0, kb0 = 0;   // run: blocks to the end of this straight stretch
    __device__ __forceinline__ KSequence(int kh_, int wg_, int first, int last_) : kh(kh_), wg(wg_), s(first - 1), last(last_) { stretch(); }
    // the slice's blocks from its start to its end, then those before its start
    __device__ __forceinline__ void stretch() {
        if (rest > 0) {
            kb = kb0;
            run = rest;
            rest = 0;
            return;
        }
#pragma unroll 1
        for (;;) {
            if (s + 1 >= last) {         // past the end the last block again
                run = 1 << 30;
                stride = 0;
                return;
            }
            ++s;
            const KSlice ks = k_slice_of<Walk>(kh, wg, s % kWaves);
            if (ks.S <= 0) continue;
            kb0 = s / kWaves * kh + ks.kb0;
            stride = ks.stride;
            kb = kb0 + ks.rot * stride;
            run = ks.S - ks.rot;
            rest = ks.rot;
            return;
        }
    }
    __device__ __forceinline__ int take() {
        const int at = kb;
        if (--run == 0) stretch();
        else kb += stride;
        return at;
    }
};

// A workgroup of WN x WM waves computes WN*A column tiles x WM*B row tiles, a wave A x B of them.  Weight and activation
// fragments of SLOTS K blocks go through a ring in LDS, filled by loads that deliver straight into it (SLOTS - 1 blocks
// ahead; the loop has no other vector-memory instruction, so its waits can count them), and each fragment is read from
// there by the waves of its row or column.
//   4 x 2 waves of 4 x 4 tiles (256 columns x 128 rows, 32 KiB per K block): per K block 1024 clocks of matrix instructions
//       on each SIMD, 96 KiB of LDS reads (768 clocks) and 32 KiB of loads.  A slice's two sums and the total fill 192 of a
//       wave's 256 registers.  8B shape, 2048 rows: gate/up 782 us -> 742, down 393 -> 369, O-projection 149 -> 120 (loads all
//       behind the barrier -> spread over the block).  With data that is all zero gate/up takes 600: the rest is the power that
//       random data costs, and a bare loop of these instructions reaches 1.78 PFLOP/s with it (2.37 with zeros).  One sum for
//       the hi and the lo products (gate/up 727, down 350) rounds the lo products to the hi sum's last place: not taken.
//   smaller ones where that shape leaves compute units without a tile.  They are bound by what a compute unit can have under
//       way, about 64 KiB whatever the ring's depth: 58 GB/s from HBM, 110 from L2, i.e. 0.28 us per K block of 16 KiB.
//       (Touching the lines of later blocks, so that the loads find them in L2, was 3 to 20 % slower.)
template <int WN_, int WM_, int A_, int B_, int SLOTS_>
struct PfShape {
    static constexpr int WN = WN_, WM = WM_, A = A_, B = B_, SLOTS = SLOTS_;
    static constexpr int kTiles = WN * A, kRowTiles = WM * B, kThreads = WN * WM * 64;
    // accumulators in vector registers proper: with fewer waves the compiler keeps them in accumulation registers and
    // copies them back and forth around every slice
    static constexpr int kMinWaves = A * B >= 8 ? 2 : 4;
};
template <class DT, int STAGE, class Sh>
struct PfGemm {
    static constexpr int WN = Sh::WN, WM = Sh::WM, A = Sh::A, B = Sh::B, SLOTS = Sh::SLOTS;
    using Shape = Sh;
    static constexpr int AF = PfAct<DT>::AF;
    static constexpr int NF = WN * A + WM * B * AF;    // fragments per K block
    static constexpr int NPW = NF / (WN * WM);         // loads per wave and K block
    static_assert(NF % (WN * WM) == 0 && SLOTS >= 3, "");
    static constexpr int kSlotBytes = NF * 1024;
    static constexpr int kLdsBytes = SLOTS * kSlotBytes;
    using Walk = typename PfWalk<STAGE>::T;

    // Weight fragments are read WD ahead of their use, the next block's activation fragments as this one's are used up.
    static constexpr int WR = A >= 4 ? 4 : 2, WD = WR / 2;
    static constexpr int MID = A / 2;
    static_assert(A % WR == 0 && MID + WD <= A, "");
    v4f tot[A][B], acc[A][B][AF];
    uint4 wf[WR], af[B][AF];

    __device__ __forceinline__ uint4 lds_frag(const char* slot, int f, int lane) const {
        return *reinterpret_cast<const uint4*>(slot + f * 1024 + lane * 16);
    }

    // The slice's sums go to the total, and the next slice's start at zero.
    __device__ __forceinline__ void fold(int i, int j) {
        if constexpr (AF == 2) tot[i][j] += acc[i][j][0] + acc[i][j][1];
        else tot[i][j] += acc[i][j][0];
#pragma unroll
        for (int f = 0; f < AF; ++f) acc[i][j][f] = v4f{0.f, 0.f, 0.f, 0.f};
    }

    // One K block from slot `cur`; the following one is in `nxt` after the barrier in the middle, where the loads of the block
    // SLOTS - 1 ahead begin (into the slot of the block before this one: every wave is past it).  They are issued a few per
    // step, up to the middle of the next block: all at once they hold the wave up, and with it its matrix instructions.  FIRST,
    // at the first block of a slice: the sums of the slice before are added to the total, tile by tile between the matrix
    // instructions, and the new ones start at zero.
    template <bool FIRST, class Issue>
    __device__ __forceinline__ void block(const char* cur, const char* nxt, int wn, int wm, int lane, Issue&& issue) {
#pragma unroll
        for (int i = 0; i < A; ++i) {
            if (i == MID) {
                wait_vm<(SLOTS - 3) * NPW>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                issue(-1);
            }
            {
                const int k = (i - MID + A) % A;
#pragma unroll
                for (int q = k * NPW / A; q < (k + 1) * NPW / A; ++q) issue(q);
            }
            if (i + WD < A) wf[(i + WD) % WR] = lds_frag(cur, wn * A + i + WD, lane);
            else wf[(i + WD) % WR] = lds_frag(nxt, wn * A + i + WD - A, lane);
            if constexpr (FIRST) {
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    fold(i, j);
                    asm volatile("" : "+v"(tot[i][j]));
                }
            }
#pragma unroll
            for (int f = 0; f < AF; ++f)
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    acc[i][j][f] = DT::mfma(wf[i % WR], af[j][f], acc[i][j][f]);
                    if (i == A - 1) {
                        __builtin_amdgcn_sched_barrier(0);
                        af[j][f] = lds_frag(nxt, WN * A + (wm * B + j) * AF + f, lane);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // The first K range is done: its total waits in memory, and this thread reads it back at the end.
    __device__ __forceinline__ void spill_total(float* spill) {
        float* hp = spill + threadIdx.x * 4;
        asm volatile("" : "+v"(hp));                    // its addresses are not to be kept in registers from the start
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) {
                fold(i, j);
                *reinterpret_cast<v4f*>(hp + (i * B + j) * (Sh::kThreads * 4)) = tot[i][j];
                tot[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
            }
    }

    template <class Issue>
    __device__ __forceinline__ void run_blocks(int kh, int wg, int first, int last, int wn, int wm, int lane, float* spill, char* smem,
                                               Issue&& issue) {
        wait_vm<(SLOTS - 3) * NPW + NPW * (A - MID) / A>();
        // no scalar load may be pending at the loop's entry: the compiler would then wait for all LDS reads at once in it
        __builtin_amdgcn_s_waitcnt(0xC07F);             // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < WD; ++i) wf[i] = lds_frag(smem, wn * A + i, lane);
#pragma unroll
        for (int x = 0; x < B * AF; ++x) af[x / AF][x % AF] = lds_frag(smem, WN * A + wm * (B * AF) + x, lane);
        int cslot = 0;
        auto one = [&](auto begin) {
            const char* cur = smem + cslot * kSlotBytes;
            cslot = cslot + 1 == SLOTS ? 0 : cslot + 1;
            const char* nxt = smem + cslot * kSlotBytes;
            block<decltype(begin)::value>(cur, nxt, wn, wm, lane, issue);
        };
#pragma unroll 1
        for (int s = first; s < last; ++s) {
            if (spill && s == kWaves) spill_total(spill);
            const int S = __builtin_amdgcn_readfirstlane(k_slice_of<Walk>(kh, wg, s % kWaves).S);
            if (S <= 0) continue;
            one(std::true_type());
#pragma unroll 1
            for (int i = 1; i < S; ++i) one(std::false_type());
        }
    }

    // Slices first .. last - 1.  spill: where the total over the first K range waits while the second is summed (null:
    // there is only one range in first .. last).  begun(): called when the first blocks are under way.
    template <class Begun>
    __device__ __forceinline__ void contract(const uint4* __restrict__ W, const uint4* __restrict__ act, const int* tiles, int rt0,
                                             int kblocks, int kh, int wgs, int first, int last, float* spill, char* smem, Begun&& begun) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int wn = wave % Sh::WN, wm = wave / Sh::WN;
        const int t0 = __builtin_amdgcn_readfirstlane(tiles[0]);   // all of the workgroup's tiles walk K alike
        const char* src[NPW];
#pragma unroll
        for (int q = 0; q < NPW; ++q) {
            const int f = wave * NPW + q;
            if (f < WN * A) {
                const int t = __builtin_amdgcn_readfirstlane(tiles[f]);
                src[q] = reinterpret_cast<const char*>(W + (size_t)(t < 0 ? t0 : t) * kblocks * 64);
            } else {
                const int x = f - WN * A;
                src[q] = reinterpret_cast<const char*>(act + PfAct<DT>::frag(kblocks, rt0 + x / AF, 0, x % AF));
            }
        }
        KSequence<Walk> ahead(kh, t0 % wgs, first, last);
        int islot = 0;
        const unsigned lane16 = lane * 16;
        const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
        unsigned dst = 0, ow = 0, oa = 0;
        auto issue = [&](int q) {
            if (q < 0) {
                const int kb = ahead.take();
                dst = lds0 + islot * kSlotBytes + wave * (NPW * 1024);
                // byte offsets of the block in a weight tile and in the activations (below 4 GiB: K up to 8 million)
                ow = (unsigned)kb * 1024u + lane16;
                oa = (unsigned)kb * (unsigned)(PfAct<DT>::kBlockTiles * AF * 1024) + lane16;
                islot = islot + 1 == SLOTS ? 0 : islot + 1;
            } else {
                load_to_lds(src[q], wave * NPW + q < WN * A ? ow : oa, dst + q * 1024);
            }
        };
#pragma unroll 1
        for (int s = 0; s < SLOTS - 1; ++s) {
            issue(-1);
#pragma unroll
            for (int q = 0; q < NPW * (A - MID) / A; ++q) issue(q);
            if (s < SLOTS - 2)
#pragma unroll
                for (int q = NPW * (A - MID) / A; q < NPW; ++q) issue(q);
        }
        begun();
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) {
                tot[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < AF; ++f) acc[i][j][f] = v4f{0.f, 0.f, 0.f, 0.f};
            }
        run_blocks(kh, t0 % wgs, first, last, wn, wm, lane, spill, smem, issue);
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) fold(i, j);
        if (spill) {
            const float* hp = spill + threadIdx.x * 4;
            asm volatile("" : "+v"(hp));
#pragma unroll
            for (int i = 0; i < A; ++i)
#pragma unroll
                for (int j = 0; j < B; ++j) tot[i][j] = *reinterpret_cast<const v4f*>(hp + (i * B + j) * (Sh::kThreads * 4)) + tot[i][j];
        }
        wait_vm<0>();                                   // the blocks loaded past the end
        __syncthreads();
    }
};

// Adds the sums that `shares` workgroups have of the same tiles, one per K range: each writes its own to device memory and counts
// itself; the one that counts last adds all of them in the order of the ranges and goes on (returns true).  Nobody waits for
// anybody.  Relaxed device-scope accesses, counted after every wave has seen its stores acknowledged, as in the verify pass's
// down projection.
template <class G>
__device__ __forceinline__ bool combine_shares(G& acc, float* xch, int* ticket, int share, int shares, char* smem) {
    using Sh = typename G::Shape;
    constexpr int N = Sh::A * Sh::B, kFloats = Sh::kThreads * N * 4, XB = N % 2 == 0 ? 2 : 1;
    auto at = [&](int sh, int x) { return reinterpret_cast<uint64_t*>(xch + (size_t)sh * kFloats + x * (Sh::kThreads * 4) + threadIdx.x * 4); };
#pragma unroll
    for (int x = 0; x < N; ++x) {
        const v4f v = acc.tot[x / Sh::B][x % Sh::B];
        uint64_t* p = at(share, x);
        __hip_atomic_store(p, (uint64_t)__float_as_uint(v.x) | (uint64_t)__float_as_uint(v.y) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 1, (uint64_t)__float_as_uint(v.z) | (uint64_t)__float_as_uint(v.w) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* flag = reinterpret_cast<int*>(smem);
    if (threadIdx.x == 0) {
        const int seen = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (seen == shares - 1) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next stage
        *flag = seen == shares - 1;
    }
    __syncthreads();
    if (!*flag) return false;
#pragma unroll
    for (int x0 = 0; x0 < N; x0 += XB) {                 // all loads of a range and two fragments first, then the additions
        for (int r = 0; r < shares; ++r) {
            uint64_t raw[XB][2];
#pragma unroll
            for (int x = 0; x < XB; ++x)
#pragma unroll
                for (int h = 0; h < 2; ++h) raw[x][h] = __hip_atomic_load(at(r, x0 + x) + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int x = 0; x < XB; ++x) {
                const v4f v = v4f{__uint_as_float((uint32_t)raw[x][0]), __uint_as_float((uint32_t)(raw[x][0] >> 32)),
                                  __uint_as_float((uint32_t)raw[x][1]), __uint_as_float((uint32_t)(raw[x][1] >> 32))};
                v4f& t = acc.tot[(x0 + x) / Sh::B][(x0 + x) % Sh::B];
                t = r ? t + v : v;
            }
        }
    }
    return true;
}

// Position of a workgroup in the grid of (column group, row group).  Workgroups are dealt to the eight XCDs in turn; an
// XCD takes a contiguous stretch of the column-major list, so the ones that run at a time on it share weight tiles and
// activation rows in its L2.
__device__ __forceinline__ int xcd_contiguous(int wg, int total) {
    const int x = wg & 7, s = wg >> 3, per = total >> 3, rem = total & 7;
    return x * per + (x < rem ? x : rem) + s;
}

// idx-th (column group, row group) in patches of kPatchCols x kPatchRows, so that the workgroups an XCD runs at a time
// (32 of them) read few different weight tiles and rows per K block.
constexpr int kPatchCols = 4, kPatchRows = 8;
__device__ __forceinline__ void patch_order(int idx, int cols, int rows, int& cg, int& rg) {
    const int cb = idx / (kPatchCols * rows), x = idx - cb * kPatchCols * rows;
    const int nc = cols - cb * kPatchCols < kPatchCols ? cols - cb * kPatchCols : kPatchCols;
    const int rb = x / (kPatchRows * nc), y = x - rb * kPatchRows * nc;
    const int nr = rows - rb * kPatchRows < kPatchRows ? rows - rb * kPatchRows : kPatchRows;
    cg = cb * kPatchCols + y / nr;
    rg = rb * kPatchRows + y % nr;
}

// Weights, activations, contraction length and K ranges of a stage.
template <int STAGE>
__device__ __forceinline__ void pf_inputs(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const uint4*& W, const void*& act,
                                          int& K, int& ways) {
    if constexpr (STAGE == kPfQKV) { W = Ly.wqkv; act = T.A; K = M.d; }
    else if constexpr (STAGE == kPfOproj) { W = Ly.wo; act = T.O; K = M.qdim; }
    else if constexpr (STAGE == kPfGateUp) { W = Ly.wgu; act = T.A; K = M.d; }
    else if constexpr (STAGE == kPfDown) { W = Ly.wd; act = T.H; K = M.F; }
    else { W = M.wlm; act = T.A; K = M.d; }
    ways = STAGE == kPfDown && M.split_down ? 2 : 1;
}

// A 16 x 16 fragment's lane (m = row, g) has columns 4g .. 4g+3 of it.  After a swap between the half-waves it has columns
// r0, r0 + 1 and their partners r0 + 8, r0 + 9, the pairs that the verify pass's epilogues work on.
struct PfPairs {
    float u0, u1, w0, w1;        // columns r0, r0 + 1, r0 + 8, r0 + 9
    __device__ __forceinline__ explicit PfPairs(v4f c) {
        const auto pa = __builtin_amdgcn_permlane32_swap(__float_as_uint(c.x), __float_as_uint(c.z), false, false);
        const auto pb = __builtin_amdgcn_permlane32_swap(__float_as_uint(c.y), __float_as_uint(c.w), false, false);
        u0 = __uint_as_float(pa[0]); u1 = __uint_as_float(pb[0]);
        w0 = __uint_as_float(pa[1]); w1 = __uint_as_float(pb[1]);
    }
    static __device__ __forceinline__ int r0() { return 4 * ((threadIdx.x >> 4) & 1) + 2 * ((threadIdx.x & 63) >> 5); }
};

// The residual stream, fragment by fragment in the order of a wave's result registers: [row tile][column tile][64 lanes][4].
__device__ __forceinline__ v4f* pf_x_frag(const DevModel& M, const PrefillBufs& T, int tile, int rt) {
    return reinterpret_cast<v4f*>(T.X) + ((size_t)rt * (M.d / 16) + tile) * 64 + (threadIdx.x & 63);
}
// A fragment of the stream's new value: stored, times the next norm's gain as the next contraction's input, and its sum of
// squares per row.  All lanes of a wave call it.
template <class DT>
__device__ __forceinline__ void pf_residual(const DevModel& M, const PrefillBufs& T, const PrefillArgs& P, int tile, int rt, v4f x, v4f gain) {
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int row = rt * 16 + m;
    const bool on = row < P.n;
    if (on) {
        *pf_x_frag(M, T, tile, rt) = x;
        PfAct<DT>::store4(T.A, M.d / DT::KB, row, tile * 16 + 4 * g, x * gain);
    }
    const PfPairs p(x);
    float sq = square_pair(p.u0, p.w0) + square_pair(p.u1, p.w1);
    sq = wave_xor_add<32>(sq);
    sq = wave_xor_add<16>(sq);
    if (on && g == 0) T.ssq[(size_t)tile * T.cap + row] = sq;
}

// 1 / rms of a workgroup's rows.  32 sums per row, of tiles s, s + 32, .., and then of each other, in the verify pass's order: a
// thread takes a row and PER of the sums, the workgroup's waves have the rest.  load() before the contraction's first loads,
// so that they are under way together; sum() is a thread's part; of() adds a row's parts, which all threads have put into LDS.
// The contraction takes 0.3 (streaming form) to 2.4 us longer with it and a launch of 4.6 to 4.8 us in front of it goes, two a
// layer: prompt of 61 rows, 4 layers of 8B shape 726 us -> 707, 509 rows of the 1B shape 3030 -> 2950, 333 rows of a small fp32
// model 173 -> 161.
template <int ROWS, int THREADS>
struct PfScales {
    static constexpr int Q = THREADS / ROWS, PER = 32 / Q, AHEAD = 4;
    static_assert(Q >= 1 && Q <= 16 && (Q & (Q - 1)) == 0, "");
    float raw[2][AHEAD][PER];
    const float* at;
    size_t step;                 // from a tile to the next
    int ntp, q;
    __device__ __forceinline__ void load(float (&v)[AHEAD][PER], int t0) {
#pragma unroll
        for (int t = 0; t < AHEAD; ++t)
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int i = q + Q * p + 32 * (t0 + t);
                v[t][p] = at[(i < ntp ? i : ntp - 1) * step];
            }
    }
    __device__ __forceinline__ void load(const DevModel& M, const PrefillBufs& T, const PrefillArgs& P, int rt0) {
        const int row = rt0 * 16 + (int)threadIdx.x % ROWS;
        q = threadIdx.x / ROWS;
        ntp = M.d / 16;
        step = T.cap;
        at = T.ssq + (row < P.n ? row : P.n - 1);
        load(raw[0], 0);
        if (ntp > 32 * AHEAD) load(raw[1], AHEAD);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ float sum() {
        float a[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) a[p] = 0.f;
        auto add = [&](const float (&v)[AHEAD][PER], int t0) {
#pragma unroll
            for (int t = 0; t < AHEAD; ++t)
#pragma unroll
                for (int p = 0; p < PER; ++p) a[p] += q + Q * p + 32 * (t0 + t) < ntp ? v[t][p] : 0.f;
        };
        add(raw[0], 0);
        if (ntp > 32 * AHEAD) add(raw[1], AHEAD);
        for (int t0 = 2 * AHEAD; 32 * t0 < ntp; t0 += AHEAD) {
            load(raw[0], t0);
            add(raw[0], t0);
        }
#pragma unroll
        for (int h = PER / 2; h > 0; h /= 2)
#pragma unroll
            for (int p = 0; p < h; ++p) a[p] += a[p + h];
        return a[0];
    }
    static __device__ __forceinline__ float of(const DevModel& M, const float* lds, int row) {
        float a[Q];
#pragma unroll
        for (int p = 0; p < Q; ++p) a[p] = lds[p * ROWS + row];
#pragma unroll
        for (int h = Q / 2; h > 0; h /= 2)
#pragma unroll
            for (int p = 0; p < h; ++p) a[p] += a[p + h];
        return 1.0f / sqrtf(a[0] / (float)M.d + M.eps);
    }
};
template <int STAGE>
constexpr bool kPfScaled = STAGE == kPfQKV || STAGE == kPfGateUp || STAGE == kPfLMHead;

// What a stage does with a finished fragment (column tile `tile`, row tile rt).  fetch() asks for what finish() needs from
// memory: a wave fetches for all of its fragments before it finishes the first, because the compiler moves no load in front
// of another fragment's stores and the wave then waits for memory once per fragment (16 of them, 8B shape, 2048 rows: 26 us
// of the O-projection's 142, 9 us of each round of gate/up's).  fetch() stays inside the buffers for fillers and for rows past
// the last one.  LM head: the lane's best of the columns it has seen so far goes to best_v, best_i.
template <class DT, int STAGE>
struct PfEpilogue {
    v4f x, gain;                 // O-projection, down projection
    float sc;                    // the others: the row's 1 / rms, set by the kernel
    float2 cs, sn;               // QKV: the rotation
    __device__ __forceinline__ void fetch(const DevModel& M, const PrefillBufs& T, const PrefillArgs& P, const float* gain_next, int tile, int rt) {
        const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
        const int row = rt * 16 + m;
        if (tile < 0) tile = 0;
        if constexpr (STAGE == kPfOproj || STAGE == kPfDown) {
            x = *pf_x_frag(M, T, tile, rt);
            gain = *reinterpret_cast<const v4f*>(gain_next + tile * 16 + 4 * g);
        }
        if constexpr (STAGE == kPfQKV) {
            const int hd = M.hd, tph = hd / 16;
            if (tile < (M.qdim + M.kvdim) / 16) {
                const size_t ro = (size_t)(P.L0 + (row < P.n ? row : 0)) * (hd / 2) + (tile % tph) * 8 + PfPairs::r0();
                cs = *reinterpret_cast<const float2*>(M.rope_cos + ro);
                sn = *reinterpret_cast<const float2*>(M.rope_sin + ro);
            }
        }
    }
    __device__ __forceinline__ void finish(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, int tile, int rt,
                                           v4f c, float& best_v, int& best_i) const {
        if constexpr (STAGE == kPfOproj || STAGE == kPfDown) pf_residual<DT>(M, T, P, tile, rt, x + c, gain);
        else finish_scaled(M, Ly, T, P, tile, rt, c, best_v, best_i);
    }
    __device__ __forceinline__ void finish_scaled(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, int tile,
                                                  int rt, v4f c, float& best_v, int& best_i) const {
        const int lane = threadIdx.x & 63, m = lane & 15;
        const int row = rt * 16 + m, r0 = PfPairs::r0();
        if constexpr (STAGE == kPfLMHead) {        // logits of the rows that are kept, arg-max per row
            if (row >= P.n) return;
            const int c0 = tile * 16 + 4 * (lane >> 4);
            const v4f z = c * sc;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (better(z[e], c0 + e, best_v, best_i)) { best_v = z[e]; best_i = c0 + e; }
            if (row >= P.keep0) *reinterpret_cast<v4f*>(M.logits + (size_t)(row - P.keep0) * M.V + c0) = z;
            return;
        }
        const PfPairs p(c);
        if (row >= P.n) return;
        const float a0 = p.u0 * sc, a1 = p.u1 * sc, b0 = p.w0 * sc, b1 = p.w1 * sc;
        if constexpr (STAGE == kPfGateUp) {
            PfAct<DT>::store2(T.H, M.F / DT::KB, row, tile * 8 + r0, swiglu(a0, b0), swiglu(a1, b1));
        } else if constexpr (STAGE == kPfQKV) {
            const int hd = M.hd, tph = hd / 16, qt = M.qdim / 16, kt = M.kvdim / 16, pos = P.L0 + row;
            const size_t slot_base = (size_t)P.slot * M.Hkv * M.ctx_pad * hd;
            if (tile < qt + kt) {
                const bool isq = tile < qt;
                const int tt = isq ? tile : tile - qt;
                const int head = tt / tph, c1 = (tt % tph) * 8 + r0;
                float x0, x1, y0, y1;
                rotate_pair(a0, b0, cs.x, sn.x, x0, y0);
                rotate_pair(a1, b1, cs.y, sn.y, x1, y1);
                if (isq) {
                    const size_t o = (size_t)row * M.qdim + head * hd + c1;
                    if constexpr (DT::HAS_LO) {
                        auto put = [&](size_t at, float v, float w) {
                            const uint32_t h0 = DT::att_bits(v), h1 = DT::att_bits(w);
                            const uint32_t l0 = DT::att_bits(v - DT::att_float(h0)), l1 = DT::att_bits(w - DT::att_float(h1));
                            *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(T.Q_hi) + at) = h0 | (h1 << 16);
                            *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(T.Q_lo) + at) = l0 | (l1 << 16);
                        };
                        put(o, x0, x1);
                        put(o + hd / 2, y0, y1);
                    } else {
                        *reinterpret_cast<float2*>(reinterpret_cast<float*>(T.Q_hi) + o) = float2{x0, x1};
                        *reinterpret_cast<float2*>(reinterpret_cast<float*>(T.Q_hi) + o + hd / 2) = float2{y0, y1};
                    }
                } else {
                    const size_t hb = slot_base + (size_t)head * M.ctx_pad * hd;
                    auto put = [&](int col, float v, float w) {      // neighbouring columns are neighbours in the cache
                        const size_t at = hb + kcache_index<DT>(hd, pos, col);
                        if constexpr (DT::HAS_LO)
                            *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(Ly.kcache) + at) = DT::att_bits(v) | (DT::att_bits(w) << 16);
                        else
                            *reinterpret_cast<float2*>(reinterpret_cast<float*>(Ly.kcache) + at) = float2{v, w};
                    };
                    put(c1, x0, x1);
                    put(c1 + hd / 2, y0, y1);
                }
            } else {
                const int tt = tile - qt - kt;
                const int head = tt / tph, c1 = (tt % tph) * 16 + r0;
                const size_t hb = slot_base + (size_t)head * M.ctx_pad * hd;
                auto put = [&](int col, float v) {
                    const size_t at = hb + vcache_index<DT>(hd, pos, col);
                    if constexpr (DT::HAS_LO) reinterpret_cast<uint16_t*>(Ly.vcache)[at] = (uint16_t)DT::att_bits(v);
                    else reinterpret_cast<float*>(Ly.vcache)[at] = v;
                };
                put(c1, a0);
                put(c1 + 1, a1);
                put(c1 + 8, b0);
                put(c1 + 9, b1);
            }
        }
    }
};

template <class DT, int STAGE, class Sh>
__global__ void __launch_bounds__(Sh::kThreads, Sh::kMinWaves) k_pf_gemm(DevModel M, DevLayer Ly, PrefillBufs T, PfTiles L, PrefillArgs P,
                                                                          const float* gain_next, int shares, bool own_scales) {
    extern __shared__ char pf_smem[];
    using G = PfGemm<DT, STAGE, Sh>;
    constexpr int A = Sh::A, B = Sh::B;
    const int row_groups = (P.n + Sh::kRowTiles * 16 - 1) / (Sh::kRowTiles * 16);
    const int tiles_wg = gridDim.x / shares;              // (column group, row group) pairs
    const int share = blockIdx.x / tiles_wg;
    const int idx = xcd_contiguous(blockIdx.x % tiles_wg, tiles_wg);
    int cg, rg;
    patch_order(idx, L.n / Sh::kTiles, row_groups, cg, rg);
    const int* tiles = L.order + cg * Sh::kTiles;
    const uint4* W;
    const void* act;
    int K, ways;
    pf_inputs<STAGE>(M, Ly, T, W, act, K, ways);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % Sh::WN, wm = wave / Sh::WN;
    const int rt0 = rg * Sh::kRowTiles;
    const int kblocks = K / DT::KB, slices = ways * kWaves, per = slices / shares;   // shares: 1, `ways` or `slices`
    float* xch = T.xch + (size_t)idx * shares * (Sh::kThreads * A * B * 4);
    using Scales = PfScales<Sh::kRowTiles * 16, Sh::kThreads>;
    Scales scales;
    float scale_part = 0.f;                             // in a register: the ring of PfMid leaves no LDS for a second workgroup's
    if constexpr (kPfScaled<STAGE>)
        if (own_scales) scales.load(M, T, P, rt0);
    G acc;
    acc.contract(W, reinterpret_cast<const uint4*>(act), tiles, rt0, kblocks, kblocks / ways, L.wgs, share * per, share * per + per,
                 per > kWaves ? xch : nullptr, pf_smem, [&] {
                     if constexpr (kPfScaled<STAGE>)
                         if (own_scales) scale_part = scales.sum();
                 });
    if (shares > 1) {                                    // k_pf_add goes on
        v4f* out = reinterpret_cast<v4f*>(xch + (size_t)share * (Sh::kThreads * A * B * 4)) + threadIdx.x;
#pragma unroll
        for (int x = 0; x < A * B; ++x) out[x * Sh::kThreads] = acc.tot[x / B][x % B];
        return;
    }
    float* scale_sums = reinterpret_cast<float*>(pf_smem);
    if constexpr (kPfScaled<STAGE>)
        if (own_scales) {
            scale_sums[threadIdx.x] = scale_part;
            __syncthreads();
        }

    float best_v[B];
    int best_i[B];
#pragma unroll
    for (int j = 0; j < B; ++j) { best_v[j] = -INFINITY; best_i[j] = 0x7fffffff; }
    PfEpilogue<DT, STAGE> epi[A][B];
#pragma unroll
    for (int i = 0; i < A; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j) epi[i][j].fetch(M, T, P, gain_next, tiles[wn * A + i], rt0 + wm * B + j);
    if constexpr (kPfScaled<STAGE>)
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int row = (wm * B + j) * 16 + (lane & 15);
            const float sc = own_scales ? Scales::of(M, scale_sums, row) : T.rstd[rt0 * 16 + row];
#pragma unroll
            for (int i = 0; i < A; ++i) epi[i][j].sc = sc;
        }
    wait_vm<0>();                                       // fillers and rows past the last use nothing of it
#pragma unroll
    for (int i = 0; i < A; ++i) {
        const int tile = __builtin_amdgcn_readfirstlane(tiles[wn * A + i]);
        if (tile < 0) continue;
#pragma unroll
        for (int j = 0; j < B; ++j) epi[i][j].finish(M, Ly, T, P, tile, rt0 + wm * B + j, acc.tot[i][j], best_v[j], best_i[j]);
    }
    const int m = lane & 15, g = lane >> 4;
    if constexpr (STAGE == kPfLMHead) {
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int row = (rt0 + wm * B + j) * 16 + m;
            keep_better_xor<16>(best_v[j], best_i[j]);
            keep_better_xor<32>(best_v[j], best_i[j]);
            if (g == 0 && row < P.n) {
                T.best_val[(size_t)(cg * Sh::WN + wn) * P.n + row] = best_v[j];
                T.best_idx[(size_t)(cg * Sh::WN + wn) * P.n + row] = best_i[j];
            }
        }
    }
}

// The rest of a stage whose tiles `shares` workgroups of k_pf_gemm share: a wave adds a fragment's sums up in the order of the slices
// and finishes it (LM head: the A fragments of a wave there, one after the other, for its best column).  All of a fragment's
// sums are under way at once.  61 rows of the 8B shape's down projection, 16 slices on 512 workgroups and this: 40 us (43 in the
// streaming form; 52 where the last workgroup of a tile added them all).
template <class DT, int STAGE, class Sh>
__global__ void __launch_bounds__(256) k_pf_add(DevModel M, DevLayer Ly, PrefillBufs T, PfTiles L, PrefillArgs P, const float* gain_next, int shares,
                                                int total) {
    constexpr int A = Sh::A, B = Sh::B, WAVES = Sh::WN * Sh::WM, FR = STAGE == kPfLMHead ? A : 1;     // fragments of a wave here
    constexpr int kPlaces = WAVES * (A / FR) * B;
    const int x = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    const int idx = x / kPlaces, place = x % kPlaces;
    if (idx >= total) return;
    const int lane = threadIdx.x & 63, m = lane & 15;
    const int row_groups = (P.n + Sh::kRowTiles * 16 - 1) / (Sh::kRowTiles * 16);
    int cg, rg;
    patch_order(idx, L.n / Sh::kTiles, row_groups, cg, rg);
    const int wave = place / ((A / FR) * B), i0 = place % ((A / FR) * B) / B * FR, j = place % B;
    const int wn = wave % Sh::WN, wm = wave / Sh::WN, rt = rg * Sh::kRowTiles + wm * B + j;
    const int* tiles = L.order + cg * Sh::kTiles + wn * A;
    constexpr size_t kFrags = (size_t)Sh::kThreads * A * B;
    const v4f* in = reinterpret_cast<const v4f*>(T.xch) + (size_t)idx * shares * kFrags + wave * 64 + lane;
    const int per = shares >= kWaves ? kWaves : 1;         // sums per K range
    float best_v = -INFINITY;
    int best_i = 0x7fffffff;
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        const int tile = __builtin_amdgcn_readfirstlane(tiles[i0 + f]);
        PfEpilogue<DT, STAGE> epi;
        epi.fetch(M, T, P, gain_next, tile, rt);
        if constexpr (kPfScaled<STAGE>) epi.sc = T.rstd[rt * 16 + m];
        const v4f* at = in + (size_t)((i0 + f) * B + j) * Sh::kThreads;
        v4f raw[2 * kWaves];
#pragma unroll
        for (int s = 0; s < 2 * kWaves; ++s) raw[s] = at[(size_t)(s < shares ? s : shares - 1) * kFrags];
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        if (per == 1) {
            sum = raw[0];
            if (shares == 2) sum = sum + raw[1];
        } else {
#pragma unroll
            for (int s = 0; s < kWaves; ++s) sum += raw[s];
            if (shares == 2 * kWaves) {
                v4f second = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < kWaves; ++s) second += raw[kWaves + s];
                sum = sum + second;
            }
        }
        wait_vm<0>();                                      // fillers and rows past the last use nothing of it
        if (tile >= 0) epi.finish(M, Ly, T, P, tile, rt, sum, best_v, best_i);
    }
    if constexpr (STAGE == kPfLMHead) {
        const int row = rt * 16 + m;
        keep_better_xor<16>(best_v, best_i);
        keep_better_xor<32>(best_v, best_i);
        if (lane < 16 && row < P.n) {
            T.best_val[(size_t)(cg * Sh::WN + wn) * P.n + row] = best_v;
            T.best_idx[(size_t)(cg * Sh::WN + wn) * P.n + row] = best_i;
        }
    }
}

// Few tiles: bound by streaming the weights, as the verify pass is, and built like its stages.  A workgroup owns NT column
// tiles x RT row tiles; its eight waves contract over the eight K slices side by side, fetching weight and activation
// fragments straight into registers D blocks ahead, and the slices' sums meet in LDS in wave order.  `shares` > 1: one
// workgroup per K range.  Against the form above: no barrier per K block, eight streams per workgroup, and every compute
// unit has weights to stream where that form has a few dozen tiles.
template <int F>
struct PfSums {                  // what combine_shares works on: F fragments per thread of eight waves
    using Shape = PfShape<kWaves, 1, 1, F, 3>;
    v4f tot[1][F];
};
template <class DT, int STAGE, int NT, int RT, int D>
__global__ void __launch_bounds__(kThreads, 2) k_pf_stream(DevModel M, DevLayer Ly, PrefillBufs T, PfTiles L, PrefillArgs P,
                                                            const float* gain_next, int shares) {
    extern __shared__ char pf_smem[];
    constexpr int AF = PfAct<DT>::AF, F = (NT * RT + kWaves - 1) / kWaves;   // fragments a wave finishes
    PfSums<F> sum;
    using Walk = typename PfWalk<STAGE>::T;
    const int row_groups = (P.n + RT * 16 - 1) / (RT * 16);
    const int groups = gridDim.x / shares;
    const int share = blockIdx.x / groups, idx = xcd_contiguous(blockIdx.x % groups, groups);
    int cg, rg;
    patch_order(idx, L.n / NT, row_groups, cg, rg);
    const int* tiles = L.order + cg * NT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = __builtin_amdgcn_readfirstlane(tiles[0]);
    const int rt0 = rg * RT;
    static_assert(STAGE != kPfLMHead, "");
    float best_v = 0.f;       // (the LM head's)
    int best_i = 0;
    using Scales = PfScales<RT * 16, kThreads>;
    __shared__ float scale_sums[kPfScaled<STAGE> ? kThreads : 1];
    // A form whose sums take half of a wave's registers adds its scales up before it fetches its first blocks: nothing of them
    // is then held beside the fragments (held across the fetches they go to scratch: 24 rows of the 8B shape, gate/up 58 us
    // against 47, 128 rows QKV 40 against 32).
    constexpr bool kScalesFirst = NT * RT * AF >= 32;
    Scales scales;
    if constexpr (kPfScaled<STAGE>) {
        scales.load(M, T, P, rt0);
        if constexpr (kScalesFirst) scale_sums[threadIdx.x] = scales.sum();
    }
    const uint4* W;
    const void* act;
    int K, ways;
    pf_inputs<STAGE>(M, Ly, T, W, act, K, ways);
    const int kblocks = K / DT::KB, kh = kblocks / ways;
    v4f acc[NT][RT][AF];
    // K ranges of this workgroup: all of them one after the other, or its own
    for (int range = share; range < ways; range += shares) {
        const KSlice ks = k_slice_of<Walk>(kh, t0 % L.wgs, wave);
        const int S = ks.S;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < RT; ++j)
#pragma unroll
                for (int f = 0; f < AF; ++f) acc[i][j][f] = v4f{0.f, 0.f, 0.f, 0.f};
        if (S > 0) {
            const uint4* wp[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int t = __builtin_amdgcn_readfirstlane(tiles[i]);
                wp[i] = W + ((size_t)(t < 0 ? t0 : t) * kblocks + range * kh + ks.kb0) * 64;
            }
            const uint4* ap = reinterpret_cast<const uint4*>(act) + PfAct<DT>::frag(kblocks, rt0, range * kh + ks.kb0, 0);
            uint4 wb[D][NT], ab[D][RT][AF];
            const int last = S - 1;
            const unsigned ln = lane;
            auto fetch = [&](int st, int to) {
                const int x = st + ks.rot;
                const int s = (x >= S ? x - S : x) * ks.stride;
#pragma unroll
                for (int i = 0; i < NT; ++i) wb[to][i] = load_stream(wp[i] + (size_t)s * 64 + ln);
#pragma unroll
                for (int j = 0; j < RT; ++j)
#pragma unroll
                    for (int f = 0; f < AF; ++f) ab[to][j][f] = (ap + (size_t)s * (PfAct<DT>::kBlockTiles * AF * 64) + (j * AF + f) * 64)[ln];
                __builtin_amdgcn_sched_barrier(0);      // the loads stay in this order, and behind the products before them
            };
            auto multiply = [&](int from) {
#pragma unroll
                for (int f = 0; f < AF; ++f)
#pragma unroll
                    for (int i = 0; i < NT; ++i)
#pragma unroll
                        for (int j = 0; j < RT; ++j) acc[i][j][f] = DT::mfma(wb[from][i], ab[from][j][f], acc[i][j][f]);
            };
#pragma unroll
            for (int d = 0; d < D; ++d) fetch(d < last ? d : last, d);
            if constexpr (kPfScaled<STAGE> && !kScalesFirst) scale_sums[threadIdx.x] = scales.sum();    // (these stages have one K range)
            int s0 = 0;
            for (; s0 + D < S; s0 += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    multiply(d);
                    fetch(s0 + d + D < last ? s0 + d + D : last, d);
                }
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (s0 + d < S) multiply(d);
        } else if constexpr (kPfScaled<STAGE> && !kScalesFirst) {
            scale_sums[threadIdx.x] = scales.sum();
        }
        if (range != share) __syncthreads();        // the sums of the range before have been read
        v4f* lds = reinterpret_cast<v4f*>(pf_smem);   // [wave][fragment][lane]
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                v4f v = acc[i][j][0];
                if constexpr (AF == 2) v += acc[i][j][1];
                lds[(wave * (NT * RT) + i * RT + j) * 64 + lane] = v;
            }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < F; ++x) {
            const int f = wave + x * kWaves;
            v4f v = v4f{0.f, 0.f, 0.f, 0.f};
            if (f < NT * RT)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v += lds[(w * (NT * RT) + f) * 64 + lane];
            sum.tot[0][x] = range == share ? v : sum.tot[0][x] + v;
        }
    }
    // The last fetches are repeats of the last block that nothing multiplies, so nothing has waited for them, and a
    // wave without a fragment to finish would end with them under way.
    wait_vm<0>();
    if (shares > 1) {
        __syncthreads();
        float* xch = T.xch + (size_t)idx * shares * (kThreads * F * 4);
        if (!combine_shares<PfSums<F>>(sum, xch, T.ticket + idx, share, shares, pf_smem)) return;
    }
    PfEpilogue<DT, STAGE> epi[F];
#pragma unroll
    for (int x = 0; x < F; ++x) {
        const int f = wave + x * kWaves < NT * RT ? wave + x * kWaves : 0;
        epi[x].fetch(M, T, P, gain_next, tiles[f / RT], rt0 + f % RT);
        if constexpr (kPfScaled<STAGE>) epi[x].sc = Scales::of(M, scale_sums, f % RT * 16 + (lane & 15));
    }
    wait_vm<0>();
#pragma unroll
    for (int x = 0; x < F; ++x) {
        const int f = wave + x * kWaves;
        const int tile = f < NT * RT ? __builtin_amdgcn_readfirstlane(tiles[f / RT]) : -1;
        if (tile >= 0) epi[x].finish(M, Ly, T, P, tile, rt0 + f % RT, sum.tot[0][x], best_v, best_i);
    }
}

// ---------------------------------------------------------------- the stages around the contractions
// Embedding rows -> residual stream, first norm input, sums of squares.  A wave takes TILES column tiles of one row tile: many,
// so that a row's token (host memory) is read a few times and not once per tile, where there are waves enough all the same.
template <class DT, int TILES>
__global__ void __launch_bounds__(256) k_pf_embed(DevModel M, PrefillBufs T, PrefillArgs P, const float* gain) {
    const int ntiles = M.d / 16;
    // counts of the stages whose tiles several workgroups share: each returns to 0 by itself; a pass still starts clean
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < kPfTickets; i += 256) __hip_atomic_store(T.ticket + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int per = (ntiles + 4 * TILES - 1) / (4 * TILES);       // workgroups of a row tile
    const int rt = blockIdx.x / per, first = (blockIdx.x % per * 4 + (threadIdx.x >> 6)) * TILES;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int row = rt * 16 + m;
    const size_t at = (size_t)T.tokens[row < P.n ? row : P.n - 1] * M.d + 4 * g;
    v4f x[TILES], gn[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int tile = first + t < ntiles ? first + t : ntiles - 1;
        if constexpr (DT::HAS_LO) {
            const uint2 v = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(M.embed) + at + tile * 16);
            x[t] = v4f{bf16_to_f32(v.x & 0xFFFFu), bf16_to_f32(v.x >> 16), bf16_to_f32(v.y & 0xFFFFu), bf16_to_f32(v.y >> 16)};
        } else {
            x[t] = *reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(M.embed) + at + tile * 16);
        }
        gn[t] = *reinterpret_cast<const v4f*>(gain + tile * 16 + 4 * g);
    }
    wait_vm<0>();                                         // a wave past the last tile uses nothing of it
#pragma unroll
    for (int t = 0; t < TILES; ++t)
        if (first + t < ntiles) pf_residual<DT>(M, T, P, first + t, rt, x[t], gn[t]);
}

// 1 / rms of each row, for the contractions that don't take it themselves: a workgroup has 16 rows.
__global__ void __launch_bounds__(256) k_pf_rstd(DevModel M, PrefillBufs T, PrefillArgs P) {
    using Scales = PfScales<16, 256>;
    __shared__ float sums[256];
    Scales scales;
    scales.load(M, T, P, blockIdx.x);
    sums[threadIdx.x] = scales.sum();
    __syncthreads();
    const int row = blockIdx.x * 16 + threadIdx.x;
    if (threadIdx.x < 16 && row < P.n) T.rstd[row] = Scales::of(M, sums, threadIdx.x);
}

// Attention of row tiles rt0 .. rt0 + nrt - 1 (16 rows each, at positions L0 + 16 rt ..) against all keys before them.
// General form: one unit of the verify pass per workgroup -> (row tile, chunk, kv head).
template <class DT, int HD>
__global__ void __launch_bounds__(kThreads) k_pf_attention_unit(DevModel M, DevLayer Ly, PrefillBufs T, PrefillArgs P, int rt0, int nch) {
    extern __shared__ float att_smem[];
    const int kvh = blockIdx.x % M.Hkv, rest = blockIdx.x / M.Hkv;
    const int c = rest % nch, t = rest / nch, rt = rt0 + t;
    const int L = P.L0 + 16 * rt;
    const int k = P.n - 16 * rt < 16 ? P.n - 16 * rt : 16;
    if (c * M.chunk >= L + k) return;
    const size_t q0 = (size_t)rt * 16 * M.qdim * DT::ESZ;
    const size_t slot_frags = (size_t)P.slot * M.Hkv * M.ctx_pad * HD / DT::EPL;
    attention_unit<DT, HD>(M, Ly, reinterpret_cast<const char*>(T.Q_hi) + q0, reinterpret_cast<const char*>(T.Q_lo) + q0, slot_frags,
                           kvh, c, L, k, 0, PartialOut<HD>{T.att_part + (((size_t)t * M.Hkv + kvh) * nch + c) * M.G * kRows * (HD + kPartRow)}, att_smem);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // a wave must not end while its look-ahead fetch is in flight
}

// Form for groups of 4 or 8 query heads (a chunk is two runs or one).  In the unit above every wave fetches the cache
// blocks of its run for itself and a workgroup ends with its chunk.  Here the G waves of a workgroup (the heads of one kv
// head) walk the blocks of `span` chunks together for one row tile, two blocks a step; a block is staged once, by loads
// that deliver straight into an LDS ring, and read from there by all of them.  A wave does the runs of a chunk one after
// the other and merges the two in registers, with the unit's operations in the unit's order.  8B heads, one layer: 2000 rows
// behind 14288 keys 1560 us -> 1020-1190, 2048 rows 229 -> 105, 509 rows 44 -> 26; 1B heads, 509 rows 36 -> 16.  Matrix cores busy
// for 36 % of the time, vector instructions for 32: the registers allow two waves per SIMD, and each is a chain of products,
// softmax, products.  Measured slower: two heads or two row tiles per wave (no registers for either), eight waves on two row
// tiles (26 %), fragments read a group ahead of their products (4 %), chunks before row tiles in the grid (9 %: the XCD's
// workgroups then read different keys).
template <class DT, int HD, int G, bool WHOLE = false>
struct PfAtt {
    static constexpr int FR = HD / 4 / DT::EPL, HT = HD / 16, TPB = DT::TPB;
    static constexpr int NF = TPB * FR + HT;             // fragments of a key block: keys, then values
    static constexpr int NPW = NF / G;
    // Three sets of numerators of 128 columns, queries and fragments do not fit 256 registers: half of the totals, which are
    // touched once a chunk, takes a ring slot's place in LDS (two workgroups per compute unit, 80 KiB each).
    static constexpr int TL = WHOLE && DT::HAS_LO && HD == 128 && G == 4 ? HT / 2 : 0;     // tiles of the totals in LDS
    static constexpr int SLOTS = TL ? 4 : 5;
    static constexpr int kSlotBytes = NF * 1024, kTotalsAt = SLOTS * kSlotBytes, kLdsBytes = kTotalsAt + G * TL * 1024;
    static_assert(NF % G == 0 && (G == 4 || G == 8), "");
};
// Totals of a row tile's chunks, the denominators in 64 bits (merge_chunks).  TL > 0: the last TL numerator tiles stand at
// `rest` in LDS (the wave's own).
template <int HD, int TL>
struct PfTotals {
    static constexpr int HT = HD / 16, TR = HT - TL;
    float m = -INFINITY;
    double l = 0.;
    v4f o[TR];
    v4f* rest;
    __device__ __forceinline__ explicit PfTotals(v4f* rest_) : rest(rest_) {
#pragma unroll
        for (int j = 0; j < TR; ++j) o[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = TR; j < HT; ++j) rest[(j - TR) * 64] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ v4f get(int j) const { return j < TR ? o[j < TR ? j : 0] : rest[(j - TR) * 64]; }
    __device__ __forceinline__ void add(const AttState<HD>& s) {
        const bool up = att_outgrown(s.m, m), any = __builtin_amdgcn_ballot_w64(up) != 0;
        const float a = up ? exp2_fast(m - s.m) : 1.f;
        m = up ? s.m : m;
        const float w = s.m == -INFINITY ? 0.f : exp2_fast(s.m - m);
        if (any) {
            l *= (double)a;
#pragma unroll
            for (int j = 0; j < TR; ++j) o[j] = o[j] * a;
        }
        l = fma((double)w, (double)s.l, l);
#pragma unroll
        for (int j = 0; j < TR; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[j][e] = fmaf(w, s.o[j][e], o[j][e]);
#pragma unroll
        for (int j = TR; j < HT; ++j) {
            v4f x = rest[(j - TR) * 64];
            if (any) x = x * a;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = fmaf(w, s.o[j][e], x[e]);
            rest[(j - TR) * 64] = x;
        }
    }
};
// WHOLE: a workgroup walks all keys of its row tile and keeps the rows' totals over the chunks in registers, which the merge
// kernel would otherwise add up from the chunks' partials in memory; the row tiles with most keys begin first.
template <class DT, int HD, int G, bool WHOLE>
__device__ __forceinline__ void pf_attention(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, int rt0,
                                             int nrt, int nch, int span, char* smem) {
    using C = PfAtt<DT, HD, G, WHOLE>;
    constexpr int FR = C::FR, HT = C::HT, BK = DT::BLOCK_KEYS, NPW = C::NPW, SLOTS = C::SLOTS;
    constexpr int PARTS = kWaves / G;
    constexpr bool kPairs = WHOLE && PARTS == 2 && HD == 64;
    const int lane = threadIdx.x & 63, hq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    // row tiles fastest: the workgroups that run together on an XCD (its kv head's, with 8 of them) walk the same keys
    const int kvh = blockIdx.x % M.Hkv, rest = blockIdx.x / M.Hkv;
    const int t = WHOLE ? nrt - 1 - rest : rest % nrt, sp = WHOLE ? 0 : rest / nrt;   // row tile, from rt0; stretch of chunks
    const int row0 = 16 * (rt0 + t);
    const int L = P.L0 + row0, k = P.n - row0 < 16 ? P.n - row0 : 16;
    const int key0 = sp * span * M.chunk;
    if (!WHOLE && key0 >= L + k) return;
    const int key1 = !WHOLE && key0 + span * M.chunk < L + k ? key0 + span * M.chunk : L + k;
    const int b0 = key0 / BK, nb = (key1 - key0 + BK - 1) / BK;   // blocks with visible keys
    const int lim = m < k ? L + m : -1;

    const size_t slot_bytes = (size_t)P.slot * M.Hkv * M.ctx_pad * HD * DT::ESZ, head_bytes = (size_t)M.ctx_pad * HD * DT::ESZ;
    const char* kc = reinterpret_cast<const char*>(Ly.kcache) + slot_bytes + kvh * head_bytes;
    const char* vc = reinterpret_cast<const char*>(Ly.vcache) + slot_bytes + kvh * head_bytes;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    int next = 0, nslot = 0;
    auto issue = [&]() {                                  // block b0 + next
        const int b = b0 + next;
        const unsigned dst = lds0 + nslot * C::kSlotBytes;
#pragma unroll
        for (int q = 0; q < NPW; ++q) {
            const int f = hq * NPW + q;
            const char* src = f < C::TPB * FR ? kc + (size_t)b * (C::TPB * FR * 1024) + f * 1024
                                              : vc + (size_t)b * (HT * 1024) + (f - C::TPB * FR) * 1024;
            load_to_lds(src, lane * 16, dst + f * 1024);
        }
        ++next;
        nslot = nslot + 1 == SLOTS ? 0 : nslot + 1;
    };
    uint4 qh[FR], ql[FR];
    const size_t q0 = (size_t)(row0 + (m < k ? m : 0)) * M.qdim + (kvh * G + hq) * HD + g * (HD / 4);
#pragma unroll
    for (int i = 0; i < FR; ++i) {
        qh[i] = load_frag<DT>(T.Q_hi, q0 + i * DT::EPL);
        ql[i] = uint4{0, 0, 0, 0};
        if constexpr (DT::HAS_LO) ql[i] = load_frag<DT>(T.Q_lo, q0 + i * DT::EPL);
    }
    // the loop's waits count its own loads: everything else arrives before it
    wait_vm<0>();
#pragma unroll
    for (int i = 0; i < FR; ++i)
        asm volatile("" : "+v"(qh[i].x), "+v"(qh[i].y), "+v"(qh[i].z), "+v"(qh[i].w), "+v"(ql[i].x), "+v"(ql[i].y), "+v"(ql[i].z), "+v"(ql[i].w));
    for (int s = 0; s < SLOTS && s < nb; ++s) issue();

    AttState<HD> s, s0;                                   // the run at hand; the chunk's first run once it is done
    s.clear();
    s0.clear();
    PfTotals<HD, C::TL> all(reinterpret_cast<v4f*>(smem + C::kTotalsAt) + hq * C::TL * 64 + lane);
    int run = 0, part = 0, c = sp * span, cslot = 0;     // run: blocks of it that are done
    // A chunk's result leaves in kStores stores.  They are younger than the loads that are under way, and the waits for
    // those must not include them (a store takes as long as a load).  The compiler must make exactly these stores of what
    // is written below, and no other access to memory in the loop: tests/test_device_code.py reads that off its assembly.
    constexpr int kStores = HT + 1;
    int older = 0;                                        // blocks under way whose loads are older than the last stores
    auto wait_blocks = [&](int newer, bool slack) {       // at most `newer` blocks (and the stores) are still under way
        if (slack) {
            if (newer >= 4) wait_vm<4 * NPW + kStores>();
            else if (newer == 3) wait_vm<3 * NPW + kStores>();
            else if (newer == 2) wait_vm<2 * NPW + kStores>();
            else if (newer == 1) wait_vm<NPW + kStores>();
            else wait_vm<kStores>();
        } else {
            if (newer >= 4) wait_vm<4 * NPW>();
            else if (newer == 3) wait_vm<3 * NPW>();
            else if (newer == 2) wait_vm<2 * NPW>();
            else if (newer == 1) wait_vm<NPW>();
            else wait_vm<0>();
        }
    };
    int freed = 0;                                        // ring slots whose blocks the step before used
    for (int ib = 0; ib < nb;) {
        const bool pair = kPairs && M.bpw == 1 && ib + 1 < nb;   // a chunk's two runs of one block each, in one step
        const int two = pair || (run + 1 < M.bpw && ib + 1 < nb) ? 2 : 1;   // blocks of this step
        __builtin_amdgcn_s_waitcnt(0xC07F);               // no LDS read of the step before is pending
        wait_blocks(next - ib - two, !WHOLE && older >= two);
        older -= two;
        __builtin_amdgcn_s_barrier();                     // .. of all waves; and all are done with the step before
        asm volatile("" ::: "memory");
        for (int x = 0; x < freed && next < nb; ++x) issue();
        freed = two;
        const char* slot0 = smem + cslot * C::kSlotBytes + lane * 16;
        cslot = cslot + 1 == SLOTS ? 0 : cslot + 1;
        const char* slot1 = smem + cslot * C::kSlotBytes + lane * 16;
        auto kf = [&](int bb, int tt, int i) { return *reinterpret_cast<const uint4*>((bb ? slot1 : slot0) + (tt * FR + i) * 1024); };
        auto vf = [&](int bb, int j) { return *reinterpret_cast<const uint4*>((bb ? slot1 : slot0) + (C::TPB * FR + j) * 1024); };
        const int p0 = (b0 + ib) * BK;
        if (kPairs && pair) {
            cslot = cslot + 1 == SLOTS ? 0 : cslot + 1;
            auto kf1 = [&](int, int tt, int i) { return kf(1, tt, i); };
            auto vf1 = [&](int, int j) { return vf(1, j); };
            s0.clear();
            attention_step<DT, HD, 1, true>(s0, qh, ql, kf, vf, p0, lim, g, M.att_scale, true);
            attention_step<DT, HD, 1, true>(s, qh, ql, kf1, vf1, p0 + BK, lim, g, M.att_scale, true);
            s0.close();
            part = 1;
        } else if (two == 2) {
            cslot = cslot + 1 == SLOTS ? 0 : cslot + 1;
            if (p0 + 2 * BK - 1 > L) attention_step<DT, HD, 2, true>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, run == 0);
            else attention_step<DT, HD, 2, false>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, run == 0);
        } else {
            attention_step<DT, HD, 1, true>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, run == 0);
        }
        ib += two;
        run += two;
        if (run >= M.bpw || ib >= nb) {
            run = 0;
            s.close();
            if (PARTS == 2 && part == 0 && ib < nb) {     // the chunk's second run follows
                s0 = s;
                s.clear();
                part = 1;
                continue;
            }
            // a chunk that ends with its first run: the second, without keys, counts for nothing
            if constexpr (WHOLE) {                        // (added to nothing, the first chunk stays what it is)
                if (PARTS == 2 && part == 1) {
                    s0.add(s);
                    all.add(s0);
                } else {
                    all.add(s);
                }
            } else {
                if (PARTS == 2 && part == 1) {
                    s0.add(s);
                    s = s0;
                }
                // rows past the tile's last one are written too (their places are there and nobody reads them), so that every
                // wave issues all its stores
                float* out = T.att_part + ((((size_t)t * M.Hkv + kvh) * nch + c) * G + hq) * (kRows * (HD + kPartRow)) + m * (HD + kPartRow);
#pragma unroll
                for (int j = 0; j < HT; ++j) *reinterpret_cast<v4f*>(out + j * 16 + g * 4) = s.o[j];
                if (g == 0) *reinterpret_cast<float2*>(out + HD) = float2{s.m, s.l};
            }
            s.clear();
            if constexpr (!WHOLE) older = next - ib;
            part = 0;
            ++c;
        }
    }
    wait_vm<0>();
    if constexpr (WHOLE) {
        const float inv = 1.0f / (float)all.l;
        if (m < k)
#pragma unroll
            for (int j = 0; j < HT; ++j) PfAct<DT>::store4(T.O, M.qdim / DT::KB, row0 + m, (kvh * G + hq) * HD + j * 16 + g * 4, all.get(j) * inv);
    }
}
template <class DT, int HD, int G>
__global__ void __launch_bounds__(64 * G, 2) k_pf_attention(DevModel M, DevLayer Ly, PrefillBufs T, PrefillArgs P, int rt0, int nrt,
                                                             int nch, int span) {
    extern __shared__ float att_smem[];
    pf_attention<DT, HD, G, false>(M, Ly, T, P, rt0, nrt, nch, span, reinterpret_cast<char*>(att_smem));
}
template <class DT, int HD, int G>
__global__ void __launch_bounds__(64 * G, 2) k_pf_attention_rows(DevModel M, DevLayer Ly, PrefillBufs T, PrefillArgs P) {
    extern __shared__ float att_smem[];
    pf_attention<DT, HD, G, true>(M, Ly, T, P, 0, (P.n + 15) / 16, 0, 0, reinterpret_cast<char*>(att_smem));
}

constexpr int kPfSpanKeys = 256;     // keys a workgroup walks at least (whole chunks)
static int pf_span(const DevModel& M) { return kPfSpanKeys > M.chunk ? kPfSpanKeys / M.chunk : 1; }   // chunks of a stretch

// One wave per (row, query head).
template <class DT, int HD>
__global__ void __launch_bounds__(256) k_pf_merge(DevModel M, PrefillBufs T, PrefillArgs P, int rt0, int rows, int nch) {
    constexpr int ROW = HD + kPartRow, PER = HD / 64;
    const int lane = threadIdx.x & 63;
    const int x = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (x >= rows * M.Hq) return;
    // head fastest by kv head, so that with 8 of them a head's partials are merged where they were written
    const int kvh = x % M.Hkv, y = x / M.Hkv, hq = y % M.G, rr = y / M.G;
    const int row = rt0 * 16 + rr, t = rr >> 4, mm = rr & 15;
    const int n = (P.L0 + row) / M.chunk + 1;
    const float* base = T.att_part + ((((size_t)t * M.Hkv + kvh) * nch * M.G + hq) * kRows + mm) * ROW;
    float num[PER];
    merge_chunks<HD>(base, (size_t)M.G * kRows * ROW, n, lane, num);
#pragma unroll
    for (int i = 0; i < PER; ++i)
        PfAct<DT>::store1(T.O, M.qdim / DT::KB, row, (kvh * M.G + hq) * HD + lane + 64 * i, num[i]);
}

// Arg-max of each row over the workgroups' partials.  A workgroup takes 16 rows, so that a load's lanes share lines, in 32 walks
// over the partials with eight loads under way each (a wave per row, one partial a lane: 5.3 us at 61 rows and 500 partials,
// 14.5 at 2048).
__global__ void __launch_bounds__(512) k_pf_greedy(DevModel M, PrefillBufs T, PrefillArgs P, int parts) {
    const int own = (P.n + 15) / 16;
    if ((int)blockIdx.x >= own) {
        export_logits(M, P.export_bytes, blockIdx.x - own);
        return;
    }
    __shared__ float vals[8][16];
    __shared__ int idxs[8][16];
    constexpr int AHEAD = 8;
    const int r = threadIdx.x & 15, row = blockIdx.x * 16 + r, at = row < P.n ? row : P.n - 1;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int w0 = threadIdx.x >> 4; w0 < parts; w0 += 32 * AHEAD) {
        float v[AHEAD];
        int i[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int w = w0 + 32 * u;
            const size_t from = (size_t)(w < parts ? w : parts - 1) * P.n + at;     // the last one again changes nothing
            v[u] = T.best_val[from];
            i[u] = T.best_idx[from];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (better(v[u], i[u], bv, bi)) { bv = v[u]; bi = i[u]; }
    }
    keep_better_xor<16>(bv, bi);
    keep_better_xor<32>(bv, bi);
    if ((threadIdx.x & 63) < 16) {
        vals[threadIdx.x >> 6][r] = bv;
        idxs[threadIdx.x >> 6][r] = bi;
    }
    __syncthreads();
    if (threadIdx.x >= 16 || row >= P.n) return;
#pragma unroll
    for (int w = 1; w < 8; ++w)
        if (better(vals[w][r], idxs[w][r], bv, bi)) { bv = vals[w][r]; bi = idxs[w][r]; }
    T.greedy[row] = bi;
}

// ---------------------------------------------------------------- host side
template <class Walk>
static void order_tiles(int n_tiles, int kblocks, int wgs, std::vector<int>& orders, PfTileSet& set) {
    // tiles by where their eight walks start, which is the same for tiles of one workgroup of the verify pass
    std::vector<std::pair<std::array<int, kWaves>, int>> key(wgs);
    for (int g = 0; g < wgs; ++g) {
        key[g].second = g;
        for (int w = 0; w < kWaves; ++w) key[g].first[w] = k_slice_of<Walk>(kblocks, g, w).rot;
    }
    std::sort(key.begin(), key.end());
    std::vector<int> tiles, ends;                  // the starts' tiles one after the other, and where each start's end
    for (int a = 0, b; a < wgs; a = b) {
        for (b = a; b < wgs && key[b].first == key[a].first; ++b) {}
        for (int t0 = 0; t0 < n_tiles; t0 += wgs)
            for (int g = a; g < b; ++g)
                if (t0 + key[g].second < n_tiles) tiles.push_back(t0 + key[g].second);
        ends.push_back((int)tiles.size());
    }
    // Each start's are filled up with -1 to whole groups, for every size of group by itself: a filler is read and multiplied
    // like a tile.  Where slices are of unequal length there are many starts: d = 3200 has 156, and filled to 16 the
    // O-projection's 200 tiles took 2496 places, also in groups of one.
    for (int g = kPfGroups - 1, n = -1; g >= 0; --g) {
        const int size = 1 << g;
        int filled = 0;
        for (size_t c = 0, first = 0; c < ends.size(); first = ends[c++]) filled += (ends[c] - (int)first + size - 1) / size * size;
        PfTiles& t = set.groups[g];
        if (filled == n) {                         // no fewer than for the larger group: the same list
            t = set.groups[g + 1];
            continue;
        }
        t = PfTiles{reinterpret_cast<const int*>(orders.size() * sizeof(int)), n = filled, wgs};
        for (size_t c = 0, first = 0; c < ends.size(); first = ends[c++]) {
            orders.insert(orders.end(), tiles.begin() + first, tiles.begin() + ends[c]);
            orders.insert(orders.end(), (size - (ends[c] - first) % size) % size, -1);
        }
    }
}

void prefill_tile_orders(const DevModel& M, int stage, int nwg, std::vector<int>& orders, PfTileSet& set) {
    const int kb = M.dtype ? BF16::KB : FP32::KB;
    const int tiles = stage == kPfQKV ? M.nqkv / 16 : stage == kPfGateUp ? 2 * M.F / 16 : stage == kPfLMHead ? M.V / 16 : M.d / 16;
    const int K = stage == kPfOproj ? M.qdim : stage == kPfDown ? M.F : M.d;
    const int wgs = tiles < nwg ? tiles : nwg;
    switch (stage) {
        case kPfQKV: order_tiles<KWalkQKV>(tiles, K / kb, wgs, orders, set); break;
        case kPfOproj: order_tiles<KWalkOproj>(tiles, K / kb, wgs, orders, set); break;
        case kPfDown: order_tiles<KWalkDown>(tiles, K / kb / (M.split_down ? 2 : 1), wgs, orders, set); break;
        default: order_tiles<KWalkWide>(tiles, K / kb, wgs, orders, set); break;
    }
}

static const PfTiles& group_tiles(const PfTileSet& set, int size) { return set.groups[__builtin_ctz(size)]; }

// What workgroups that share tiles write of their sums, `fragments` each (T.xch holds T.xch_bytes).  Who chooses to share looks at it
// first; a launch that would go past the buffer is refused all the same.
static size_t shared_bytes(size_t workgroups, size_t fragments) { return workgroups * fragments * 1024; }
// .. a workgroup of the streaming form: a slice's sums are spread over its waves
static constexpr size_t stream_fragments(int nt, int rt) { return (size_t)(nt * rt + kWaves - 1) / kWaves * kWaves; }

template <class DT, int STAGE, class Sh>
static hipError_t launch_pf_gemm_v(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                                   const float* gain, hipStream_t s, int* parts, int shares) {
    const int lds = PfGemm<DT, STAGE, Sh>::kLdsBytes;
    static const hipError_t set = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pf_gemm<DT, STAGE, Sh>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (set != hipSuccess) return set;
    const PfTiles& L = group_tiles(tiles[STAGE], Sh::kTiles);
    const int groups = L.n / Sh::kTiles;
    const int grid = groups * ((P.n + Sh::kRowTiles * 16 - 1) / (Sh::kRowTiles * 16)) * shares;
    if (shares > 1 && shared_bytes(grid, Sh::kTiles * Sh::kRowTiles) > T.xch_bytes) return hipErrorInvalidValue;
    if (parts) *parts = groups * Sh::WN;
    // Its workgroups take 1 / rms of their rows themselves while they read less than this of the sums of squares per compute
    // unit.  us more for the contraction (k_pf_rstd and its launch take 4.8): 8B shape 61 rows gate/up 64 KiB 2.3, LM head 2.4,
    // 2048 rows QKV 384 KiB 5.3, gate/up 900 KiB 18, LM head 4 MiB 25; 1B shape 509 rows gate/up 64 KiB 1.3, QKV 24 KiB 1.3.
    constexpr double kOwnScaleBytes = 320 << 10;
    const bool own_scales = shares == 1 && (double)grid / T.cus * Sh::kRowTiles * M.d * 4 <= kOwnScaleBytes;
    if (kPfScaled<STAGE> && !own_scales) hipLaunchKernelGGL(k_pf_rstd, dim3((P.n + 15) / 16), dim3(256), 0, s, M, T, P);
    hipLaunchKernelGGL((k_pf_gemm<DT, STAGE, Sh>), dim3(grid), dim3(Sh::kThreads), lds, s, M, Ly, T, L, P, gain, shares, own_scales);
    if (shares > 1) {
        const int total = grid / shares, waves = total * Sh::WN * Sh::WM * Sh::B * (STAGE == kPfLMHead ? 1 : Sh::A);
        hipLaunchKernelGGL((k_pf_add<DT, STAGE, Sh>), dim3((waves + 3) / 4), dim3(256), 0, s, M, Ly, T, L, P, gain, shares, total);
    }
    return hipSuccess;
}

template <class DT, int STAGE, int NT, int RT, int D>
static hipError_t launch_pf_stream_v(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                                     const float* gain, hipStream_t s, int shares) {
    constexpr int lds = kWaves * NT * RT * 1024;
    static const hipError_t set = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pf_stream<DT, STAGE, NT, RT, D>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (set != hipSuccess) return set;
    const PfTiles& L = group_tiles(tiles[STAGE], NT);
    const int wgs = L.n / NT * ((P.n + RT * 16 - 1) / (RT * 16));
    if (shares > 1 && (wgs > kPfTickets || shared_bytes((size_t)wgs * shares, stream_fragments(NT, RT)) > T.xch_bytes)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_pf_stream<DT, STAGE, NT, RT, D>), dim3(wgs * shares), dim3(kThreads), lds, s, M, Ly, T, L, P, gain, shares);
    return hipSuccess;
}

// The streaming form where one round of workgroups does the stage: with the fewest column tiles (1, 2, 4) x 2 row tiles that
// does it, else 8 x 2 for prompts of at most 32 rows, else 4 x 4.  More work per workgroup means fewer bytes, less means more
// compute units that load.  us a layer that the best plan of the other form, sharing included, takes more (minus: less).  8B shape: 17
// rows QKV 9, O 4, gate/up 10, down 4; 61 rows 5, 0, (gate/up does not fit a round), -4 (launch_pf_gemm); 120 rows 4, 2, -, -1; 250 rows
// O 3.  1B shape: 17 rows 6, 5, 9, 2; 61 rows 6, 2, 4, -2; 250 rows 4, 5, -, 3; 509 rows O 4.  Width 1024: 17 rows 5, 2, 6, 3; 250 rows
// 7, 3, -, 4.  The down projection of widths whose K range is one would gain from 8 slices here as well and has no such rule: width 3072 at 61
// rows -8, 5120 at 61 rows -13, at 120 -30.
// Between its own forms, 61 rows of the 8B shape: O with 1, 2, 4 column tiles 26, 20, 23, down 57, 57 (2), 41 (4) (6 of timing in each).
template <class DT, int STAGE>
static bool launch_pf_stream(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                             const float* gain, hipStream_t s, hipError_t& e) {
    int shares = STAGE == kPfDown && M.split_down ? 2 : 1;
    auto wgs = [&](int nt, int rt) { return group_tiles(tiles[STAGE], nt).n / nt * ((P.n + rt * 16 - 1) / (rt * 16)); };
    auto round = [&](int nt, int rt) { return wgs(nt, rt) * shares <= T.cus; };
    const int nt = round(1, 2) ? 1 : round(2, 2) ? 2 : round(4, 2) ? 4 : P.n <= 32 && round(8, 2) ? 8 : 4;
    const int rt = round(nt, 2) ? 2 : 4;
    if (!round(nt, rt)) return false;
    if (wgs(nt, rt) > kPfTickets || shared_bytes((size_t)wgs(nt, rt) * shares, stream_fragments(nt, rt)) > T.xch_bytes) shares = 1;
    e = nt == 1 ? launch_pf_stream_v<DT, STAGE, 1, 2, 8>(M, Ly, T, tiles, P, gain, s, shares)
      : nt == 2 ? launch_pf_stream_v<DT, STAGE, 2, 2, 6>(M, Ly, T, tiles, P, gain, s, shares)
      : nt == 8 ? launch_pf_stream_v<DT, STAGE, 8, 2, 2>(M, Ly, T, tiles, P, gain, s, shares)
      : rt == 2 ? launch_pf_stream_v<DT, STAGE, 4, 2, 4>(M, Ly, T, tiles, P, gain, s, shares)
                : launch_pf_stream_v<DT, STAGE, 4, 4, 2>(M, Ly, T, tiles, P, gain, s, shares);
    return true;
}

// Workgroup shapes; the two smaller ones run two to a compute unit.
using PfLarge = PfShape<4, 2, 4, 4, 4>;   // 256 columns x 128 rows
using PfMid = PfShape<2, 2, 4, 2, 5>;     // 128 x 64
using PfSmall = PfShape<2, 2, 2, 2, 6>;   // 64 x 64

// Which shape a stage takes, and over how many workgroups the K slices of a tile are shared: the smallest estimate of
// rounds x (K blocks x time of a block + a workgroup's beginning and end), plus what the sharing costs.  The times were fitted
// to measurements of all choices on the 8B and 1B shapes at 17 to 2048 rows: 0.82 us per K block of a large tile; 0.30 and
// 0.20 us of the smaller ones, 0.50 and 0.35 when two share a compute unit; 12, 7.5 and 6 us at the ends, 4 more for the large
// tile's rotations.  For instance at 250 rows of the 8B shape gate/up takes 114 us on 224 large tiles and 150 on 896 of the middle
// ones, at 128 rows 97 and 86.
//
// Sharing costs k_pf_add and its launch, less the epilogues that the tiles' own workgroups then do without: 3 us, 0.3 per workgroup of a
// tile and the sums' bytes, written and read, at 13 TB/s; and k_pf_rstd, where those workgroups might have taken 1 / rms themselves.  us per
// prompt, with the estimate's choice / another: down of a model 1024 wide (8 layers), 600 rows, over 2 workgroups 911, over 1 961;
// 3072 wide (4 layers), 350 rows, 8 / 1 1041 / 1105; the 8B shape (4 layers), 160 rows, 2 / 16 1119 / 1128, 1370 rows 2 / 1 5445 / 5536.
//
// All choices of a stage were measured at 18 lengths from 17 to 2048 rows, where the forms above do not come first.  8B and 1B shapes: the
// choice takes up to 2 % of the prompt's time more than the best at 122 of 124, 3.1 % at worst; widths 1024 to 8192: at 236 of 242, 5.9 %
// at worst (gate/up of width 5120, 160 rows).  The rates are those of 16-bit models: float32, 66 of 82, 7.1 % at worst.
struct PfPlan { int shape, shares; };
static PfPlan plan_pf_gemm(const DevModel& M, const PrefillBufs& T, const PfTileSet* sets, int n, int stage) {
    struct Shape { int tiles, rows, per_cu; double alone, full, ends; };
    static const Shape shapes[3] = {{PfLarge::kTiles, PfLarge::kRowTiles * 16, 1, 0.82, 0.82, 12.},
                                    {PfMid::kTiles, PfMid::kRowTiles * 16, 2, 0.30, 0.50, 7.5},
                                    {PfSmall::kTiles, PfSmall::kRowTiles * 16, 2, 0.20, 0.35, 6.}};
    const int K = stage == kPfOproj ? M.qdim : stage == kPfDown ? M.F : M.d;
    const int kblocks = K / (M.dtype ? BF16::KB : FP32::KB), ways = stage == kPfDown && M.split_down ? 2 : 1;
    const bool scaled = stage == kPfQKV || stage == kPfGateUp || stage == kPfLMHead;
    PfPlan best{0, 1};
    double least = 0;
    for (int s = 0; s < 3; ++s)
        for (int shares : {1, ways, ways * kWaves}) {
            const Shape& h = shapes[s];
            const size_t tiles = (size_t)group_tiles(sets[stage], h.tiles).n / h.tiles * ((n + h.rows - 1) / h.rows);
            const size_t sum_bytes = shared_bytes(tiles * shares, h.tiles * h.rows / 16);
            if (shares > 1 && sum_bytes > T.xch_bytes) continue;
            const size_t wgs = tiles * shares, round = (size_t)T.cus * h.per_cu, rest = wgs % round;
            const double ends = h.ends + (s == 0 && stage == kPfQKV ? 4. : 0.), blocks = (double)kblocks / shares;
            const double full = blocks * h.full + ends, alone = blocks * h.alone + ends;
            const double us = wgs / round * full + (rest > (size_t)T.cus ? full : rest ? alone : 0.) +
                              (shares > 1 ? 3. + 0.3 * shares + 1.5e-7 * sum_bytes + (scaled ? 4.8 : 0.) : 0.);
            if (least == 0 || us < least) {
                least = us;
                best = PfPlan{s, shares};
            }
        }
    return best;
}

template <class DT, int STAGE>
static hipError_t launch_pf_gemm(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                                 const float* gain, hipStream_t s, int* parts = nullptr) {
    // The down projection of one row group in all its 16 slices, where those are a workgroup a compute unit and no more than one round:
    // each workgroup then loads a few hundred KB, where the streaming form's 1.8 MB are what its time is.  us per prompt of 4 layers,
    // streaming / so: 8B shape 40 rows 678 / 654, 61 rows 659 / 647, 120 rows (256 x 128 tiles) 925 / 890 (17 rows: 4.7 a layer more);
    // 16 layers of 1B, 35 rows 1108 / 1064, 61 rows 1134 / 1072 (120 rows: 128 workgroups, 1 a layer more).
    if constexpr (STAGE == kPfDown)
        if (M.split_down) {
            auto one_round = [&](auto shape, int per_cu) {
                using Sh = decltype(shape);
                const size_t wgs = (size_t)group_tiles(tiles[STAGE], Sh::kTiles).n / Sh::kTiles * 2 * kWaves;
                return P.n <= Sh::kRowTiles * 16 && wgs >= (size_t)T.cus && wgs <= (size_t)T.cus * per_cu &&
                       shared_bytes(wgs, Sh::kTiles * Sh::kRowTiles) <= T.xch_bytes;
            };
            if (P.n > 32 && one_round(PfMid(), 2)) return launch_pf_gemm_v<DT, STAGE, PfMid>(M, Ly, T, tiles, P, gain, s, parts, 2 * kWaves);
            if (P.n > 64 && one_round(PfLarge(), 1)) return launch_pf_gemm_v<DT, STAGE, PfLarge>(M, Ly, T, tiles, P, gain, s, parts, 2 * kWaves);
        }
    if constexpr (STAGE != kPfLMHead) {      // (its partial maxima would outgrow best_val, and it gains nothing)
        hipError_t e;
        if (launch_pf_stream<DT, STAGE>(M, Ly, T, tiles, P, gain, s, e)) return e;
    }
    const PfPlan p = plan_pf_gemm(M, T, tiles, P.n, STAGE);
    switch (p.shape) {
        case 0: return launch_pf_gemm_v<DT, STAGE, PfLarge>(M, Ly, T, tiles, P, gain, s, parts, p.shares);
        case 1: return launch_pf_gemm_v<DT, STAGE, PfMid>(M, Ly, T, tiles, P, gain, s, parts, p.shares);
        default: return launch_pf_gemm_v<DT, STAGE, PfSmall>(M, Ly, T, tiles, P, gain, s, parts, p.shares);
    }
}

template <class DT, int HD, int G>
static hipError_t launch_pf_attention_g(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, int rt0, int nrt,
                                        int nch, hipStream_t s) {
    constexpr int lds = PfAtt<DT, HD, G>::kLdsBytes;
    static const hipError_t set = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pf_attention<DT, HD, G>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (set != hipSuccess) return set;
    const int span = pf_span(M);
    hipLaunchKernelGGL((k_pf_attention<DT, HD, G>), dim3(nrt * ((nch + span - 1) / span) * M.Hkv), dim3(64 * G), lds, s, M, Ly, T, P, rt0,
                       nrt, nch, span);
    return hipSuccess;
}

template <class DT, int HD, int G>
static hipError_t launch_pf_attention_rows(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, hipStream_t s) {
    constexpr int lds = PfAtt<DT, HD, G, true>::kLdsBytes;
    static const hipError_t set = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pf_attention_rows<DT, HD, G>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (set != hipSuccess) return set;
    hipLaunchKernelGGL((k_pf_attention_rows<DT, HD, G>), dim3((P.n + 15) / 16 * M.Hkv), dim3(64 * G), lds, s, M, Ly, T, P);
    return hipSuccess;
}

template <class DT, int HD>
static hipError_t launch_pf_attention(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, int rt0, int nrt,
                                      int nch, hipStream_t s) {
    if (M.G == 4) return launch_pf_attention_g<DT, HD, 4>(M, Ly, T, P, rt0, nrt, nch, s);
    if (M.G == 8) return launch_pf_attention_g<DT, HD, 8>(M, Ly, T, P, rt0, nrt, nch, s);
    constexpr int lds = (kWaves * kRows * (HD + kAttPad) + kWaves * kRows * 2) * 4;
    static const hipError_t set = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pf_attention_unit<DT, HD>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (set != hipSuccess) return set;
    hipLaunchKernelGGL((k_pf_attention_unit<DT, HD>), dim3(nrt * nch * M.Hkv), dim3(kThreads), lds, s, M, Ly, T, P, rt0, nch);
    return hipSuccess;
}

// A layer's attention: whole rows, or stretches of keys and a merge.
template <class DT, int HD>
static hipError_t pf_attention_all(const DevModel& M, const DevLayer& Ly, const PrefillBufs& T, const PrefillArgs& P, hipStream_t s) {
    const int rts = (P.n + 15) / 16;
    if (pf_attention_walks_whole_rows(DT::HAS_LO, HD, M.G, M.Hkv, P.n, P.L0 + P.n, T.cus, M.chunk, M.bpw, pf_span(M) * M.chunk))
        return M.G == 4 ? launch_pf_attention_rows<DT, HD, 4>(M, Ly, T, P, s) : launch_pf_attention_rows<DT, HD, 8>(M, Ly, T, P, s);
    for (int rt = 0; rt < rts; rt += T.att_tiles) {
        const int nrt = rts - rt < T.att_tiles ? rts - rt : T.att_tiles;
        const int last = P.n < (rt + nrt) * 16 ? P.n : (rt + nrt) * 16;     // rows below this one
        const int nch = (P.L0 + last + M.chunk - 1) / M.chunk;
        const hipError_t e = launch_pf_attention<DT, HD>(M, Ly, T, P, rt, nrt, nch, s);
        if (e != hipSuccess) return e;
        const int rows = last - rt * 16;
        hipLaunchKernelGGL((k_pf_merge<DT, HD>), dim3((rows * M.Hq + 3) / 4), dim3(256), 0, s, M, T, P, rt, rows, nch);
    }
    return hipSuccess;
}

template <class DT, int HD>
static hipError_t launch_prefill_t(const DevModel& M, const DevLayer* Ls, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                                   hipStream_t s) {
    const int rts = (P.n + 15) / 16;
    hipError_t e;
    // One tile a wave up to four workgroups a compute unit, else eight (us, one / eight: 61 rows of the 8B shape 5.4 / 7.7, 509 rows of
    // the 1B shape 6.8 / 9.2, 2048 rows of the 8B shape 37 / 23).
    const int one = (M.d / 16 + 3) / 4 * rts, eight = (M.d / 16 + 31) / 32 * rts;
    if (one <= 4 * T.cus) hipLaunchKernelGGL((k_pf_embed<DT, 1>), dim3(one), dim3(256), 0, s, M, T, P, Ls[0].g_attn);
    else hipLaunchKernelGGL((k_pf_embed<DT, 8>), dim3(eight), dim3(256), 0, s, M, T, P, Ls[0].g_attn);
    for (int l = 0; l < M.n_layers; ++l) {
        const float* gain_next = l + 1 < M.n_layers ? Ls[l + 1].g_attn : M.g_final;
        if ((e = launch_pf_gemm<DT, kPfQKV>(M, Ls[l], T, tiles, P, nullptr, s)) != hipSuccess) return e;
        if ((e = pf_attention_all<DT, HD>(M, Ls[l], T, P, s)) != hipSuccess) return e;
        if ((e = launch_pf_gemm<DT, kPfOproj>(M, Ls[l], T, tiles, P, Ls[l].g_mlp, s)) != hipSuccess) return e;
        if ((e = launch_pf_gemm<DT, kPfGateUp>(M, Ls[l], T, tiles, P, nullptr, s)) != hipSuccess) return e;
        if ((e = launch_pf_gemm<DT, kPfDown>(M, Ls[l], T, tiles, P, gain_next, s)) != hipSuccess) return e;
    }
    int parts = 0;
    if ((e = launch_pf_gemm<DT, kPfLMHead>(M, Ls[0], T, tiles, P, nullptr, s, &parts)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_pf_greedy, dim3((P.n + 15) / 16 + export_wgs(P.export_bytes, 512)), dim3(512), 0, s, M, T, P, parts);
    return hipGetLastError();
}

hipError_t launch_prefill(const DevModel& M, const DevLayer* Ls, const PrefillBufs& T, const PfTileSet* tiles, const PrefillArgs& P,
                          hipStream_t stream) {
    if (M.dtype)
        return M.hd == 128 ? launch_prefill_t<BF16, 128>(M, Ls, T, tiles, P, stream) : launch_prefill_t<BF16, 64>(M, Ls, T, tiles, P, stream);
    return M.hd == 128 ? launch_prefill_t<FP32, 128>(M, Ls, T, tiles, P, stream) : launch_prefill_t<FP32, 64>(M, Ls, T, tiles, P, stream);
}

}  // namespace amusd
