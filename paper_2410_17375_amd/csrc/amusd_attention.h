// The attention work unit and the merge of chunk partials, shared by the verify pass and the prefill pass: a row's
// scores, softmax and sums are computed by the same code at the same absolute key boundaries in both, so its bits do
// not depend on which of them it went through.
#pragma once
#include "amusd_math.h"

namespace amusd {

constexpr int kAttPad = 4;    // row padding of the attention partials (spreads LDS banks)
constexpr int kPartRow = 4;   // floats appended to a partial's numerator: reference, denominator, 2 pad (keeps 16-byte alignment)

// Scores, maxima and weights are in units of log2: the score scale carries the factor log2(e), and every exponential is
// the hardware's power of two.
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Exponentials are taken against a reference that a row's maximum may exceed by up to 2^kAttSlack: sums are rescaled only
// when it grows beyond.  (The true maximum grows in most steps of a run, for one of a wave's 16 rows or another.)  Numerators
// stay far inside the half range, whose hi + lo pairs are as precise at 256 as at 1.
constexpr float kAttSlack = 8.f;
static_assert(kAttSlack < 15.f, "weights are converted to half unclamped");   // (and a reference is off by 2^-4 at most, kAttFar)
__device__ __forceinline__ bool att_outgrown(float m, float ref) { return m > ref + kAttSlack; }   // false for -inf against -inf

// The scale of a score is taken into the subtraction of the reference where that is exact enough: a reference is a rounded
// product, off by up to half its last place (at 2^28 by 16: weights would be 2^16 times too large or too small).  From
// kAttFar on the product is rounded first, as the reference was.  A row's own reference decides, so that its bits do not
// depend on its neighbours; references that large are rare, and a wave without one does nothing more than ask.
constexpr float kAttFar = 1 << 20;

// Running softmax of one wave: 16 rows of one query head, a run of key blocks.
template <int HD>
struct AttState {
    float m, l;              // reference and denominator of row lane & 15; l: this lane's part of it until close()
    v4f o[HD / 16];          // numerator: o[j][e] is head_dim column 16 j + 4 (lane >> 4) + e
    __device__ __forceinline__ void clear() {
        m = -INFINITY;
        l = 0.f;
#pragma unroll
        for (int j = 0; j < HD / 16; ++j) o[j] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void rescale(bool up, float to) {
        const float a = up ? exp2_fast(m - to) : 1.f;
        m = up ? to : m;
        l *= a;
        // scaled where they stand, ahead of all products: left alone the compiler scales each into a temporary right
        // before its product and waits for the temporary to be free again after every one
#pragma unroll
        for (int j = 0; j < HD / 16; ++j) o[j] = o[j] * a;
    }
    // the end of a run: the denominator from the four lanes that share the row
    __device__ __forceinline__ void close() {
        l = wave_xor_add<16>(l);
        l = wave_xor_add<32>(l);
    }
    // adds a later (closed) run or chunk of the same rows; the first is copied
    __device__ __forceinline__ void add(const AttState& s) {
        const bool up = att_outgrown(s.m, m);
        if (__builtin_amdgcn_ballot_w64(up)) rescale(up, s.m);
        const float w = s.m == -INFINITY ? 0.f : exp2_fast(s.m - m);
        l = fmaf(w, s.l, l);
#pragma unroll
        for (int j = 0; j < HD / 16; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[j][e] = fmaf(w, s.o[j][e], o[j][e]);
    }
};

// One step of a run: NB (two, or one at the end of a run of odd length) key blocks, keys p0 ...  Scores are computed
// transposed (keys x rows), so that the result registers are, after the softmax numerator, the operand of the P.V product.
// kf(b, t, i), vf(b, j): the blocks' fragments.  MASKED: the blocks may hold keys that some row does not see (lim: the row's
// last visible key, -1 for a row that is not the sequence's); the other form gives the same values for rows that see all of
// them.  first: the run's first step (the numerators are zero).
// Two blocks per step: a block's 8 scores per lane cost two exchanges across lanes, and its products are short chains; two
// share the former and fill the gaps of the latter.  Groups of 4 and 8 heads take
// two (always the same two of a run), groups of 1 and 2 one.  A second block without a visible key is left out: it would add
// zeros, but what rolled-back rows have left in it may be no number, and zero times that is none either.
// scored: called when the keys have been used.
struct AttNothing {
    __device__ __forceinline__ void operator()() const {}
};
template <class DT, int HD, int NB, bool MASKED, class KF, class VF, class Scored = AttNothing>
__device__ __forceinline__ void attention_step(AttState<HD>& s, const uint4* qh, const uint4* ql, KF&& kf, VF&& vf, int p0, int lim,
                                               int g, float scale, bool first, Scored&& scored = Scored()) {
    constexpr int FR = HD / 4 / DT::EPL, HT = HD / 16, TPB = DT::TPB, NTL = NB * TPB;
    // Products are issued so that those of one accumulator are not neighbours; its own order stays (hi, lo, next fragment).
    v4f sc[NTL];
#pragma unroll
    for (int i = 0; i < FR; ++i) {
        uint4 k[NTL];
#pragma unroll
        for (int t = 0; t < NTL; ++t) k[t] = kf(t / TPB, t % TPB, i);
#pragma unroll
        for (int t = 0; t < NTL; ++t) sc[t] = DT::mfma_att(k[t], qh[i], i ? sc[t] : v4f{0.f, 0.f, 0.f, 0.f});
        if constexpr (DT::HAS_LO)
#pragma unroll
            for (int t = 0; t < NTL; ++t) sc[t] = DT::mfma_att(k[t], ql[i], sc[t]);
    }
    scored();
    __builtin_amdgcn_sched_barrier(0);
    // maxima and sums by tile: a chain over all of a lane's scores is as long as the products
    float mt[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (MASKED && p0 + t * 16 + g * 4 + e > lim) sc[t][e] = -INFINITY;
        mt[t] = fmaxf(fmaxf(sc[t].x, sc[t].y), fmaxf(sc[t].z, sc[t].w));
    }
    float mx = mt[0];
#pragma unroll
    for (int t = 1; t < NTL; ++t) mx = fmaxf(mx, mt[t]);
    mx = fmaxf(mx, lane_xor<16>(mx));
    mx = fmaxf(mx, lane_xor<32>(mx));
    const float top = mx * scale;
    if (first) {
        s.m = top;
    } else {
        const bool up = att_outgrown(top, s.m);
        if (__builtin_amdgcn_ballot_w64(up)) s.rescale(up, top);
    }
    const float mref = s.m == -INFINITY ? 0.f : s.m;
    const bool far = fabsf(mref) >= kAttFar;
    if (__builtin_amdgcn_ballot_w64(far)) {
        const float by = far ? scale : 1.f;
#pragma unroll
        for (int t = 0; t < NTL; ++t) sc[t] = sc[t] * by;
        scale = far ? 1.f : scale;
    }
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[t][e] = exp2_fast(fmaf(sc[t][e], scale, -mref));
#pragma unroll
    for (int t = 0; t < NTL; ++t) s.l += (sc[t].x + sc[t].y) + (sc[t].z + sc[t].w);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        uint4 ph, pl = uint4{0, 0, 0, 0};
        const v4f a0 = sc[b * TPB], a1 = sc[b * TPB + TPB - 1];
        if constexpr (DT::HAS_LO) {
            DT::att_split2(a0.x, a0.y, ph.x, pl.x);
            DT::att_split2(a0.z, a0.w, ph.y, pl.y);
            DT::att_split2(a1.x, a1.y, ph.z, pl.z);
            DT::att_split2(a1.z, a1.w, ph.w, pl.w);
        } else {
            ph = uint4{__float_as_uint(a0.x), __float_as_uint(a0.y), __float_as_uint(a0.z), __float_as_uint(a0.w)};
        }
        constexpr int JG = 4;
#pragma unroll
        for (int j0 = 0; j0 < HT; j0 += JG) {
            uint4 v[JG];
#pragma unroll
            for (int j = 0; j < JG; ++j) v[j] = vf(b, j0 + j);
#pragma unroll
            for (int j = 0; j < JG; ++j) s.o[j0 + j] = DT::mfma_att(v[j], ph, s.o[j0 + j]);
            if constexpr (DT::HAS_LO)
#pragma unroll
                for (int j = 0; j < JG; ++j) s.o[j0 + j] = DT::mfma_att(v[j], pl, s.o[j0 + j]);
        }
    }
}

// The runs of a unit's heads, one per wave, through LDS to one partial per (head, row): out(head, row, column, four numerators,
// reference, denominator).  smem: kWaves * kRows * (HD + kAttPad + 2) floats, free to be written.
template <int HD, class Out>
__device__ __forceinline__ void merge_runs(AttState<HD>& s, int G, int parts, int hq, int part, int row0, int k, Out&& out, float* smem) {
    constexpr int HT = HD / 16, HDP = HD + kAttPad;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    float* partO = smem;                               // [hq][part][16][HD + pad]
    float* partML = smem + kWaves * kRows * HDP;       // [hq][part][16][2]
    // run partial to LDS: o[j][e] is head_dim index 16j + 4g + e of row m
    const int slot = hq * parts + part;
    s.close();
#pragma unroll
    for (int j = 0; j < HT; ++j)
        *reinterpret_cast<v4f*>(partO + ((size_t)(slot * kRows + m) * HDP + j * 16 + g * 4)) = s.o[j];
    if (g == 0) {
        partML[(slot * kRows + m) * 2 + 0] = s.m;
        partML[(slot * kRows + m) * 2 + 1] = s.l;
    }
    __syncthreads();
    // merge the runs of each head in run order; item = (head, row, 4 consecutive head_dim entries)
    for (int it = tid; it < G * kRows * (HD / 4); it += kThreads) {
        const int c4 = it % (HD / 4), mm = (it / (HD / 4)) % kRows, hh = it / (kRows * (HD / 4));
        if (mm < row0 || mm >= row0 + k) continue;
        float Mx = partML[(hh * parts * kRows + mm) * 2], den = partML[(hh * parts * kRows + mm) * 2 + 1];
        v4f num = *reinterpret_cast<const v4f*>(partO + ((size_t)(hh * parts * kRows + mm) * HDP + c4 * 4));
        for (int pp = 1; pp < parts; ++pp) {           // AttState::add
            const int sl = hh * parts + pp;
            const float mw = partML[(sl * kRows + mm) * 2];
            if (att_outgrown(mw, Mx)) {
                const float a = exp2_fast(Mx - mw);
                Mx = mw;
                den *= a;
                num = num * a;
            }
            const float wt = mw == -INFINITY ? 0.f : exp2_fast(mw - Mx);
            den = fmaf(wt, partML[(sl * kRows + mm) * 2 + 1], den);
            const v4f x = *reinterpret_cast<const v4f*>(partO + ((size_t)(sl * kRows + mm) * HDP + c4 * 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) num[e] = fmaf(wt, x[e], num[e]);
        }
        out(hh, mm, c4 * 4, num, Mx, den);
    }
    __syncthreads();
}

// .. to memory, for the merge of the chunks: [head][row][HD numerators, reference, denominator, pad]
template <int HD>
struct PartialOut {
    float* part_out;
    __device__ __forceinline__ void operator()(int hh, int mm, int col, v4f num, float ref, float den) const {
        float* out = part_out + ((size_t)hh * kRows + mm) * (HD + kPartRow);
        *reinterpret_cast<v4f*>(out + col) = num;
        if (col == 0) { out[HD] = ref; out[HD + 1] = den; }
    }
};

// One unit: chunk c of kv head kvh (the 8/G runs of bpw key blocks that the waves of a workgroup walk) against the tile
// rows row0 .. row0+k-1, which stand at positions L .. L+k-1.  q_hi / q_lo: the tile's query rows, row-major.
// slot_frags: start of the sequence's cache, in 16-byte fragments.  out: as in merge_runs, heads
// counted in the group.  smem: kWaves * kRows * (HD + kAttPad + 2) floats.
template <class DT, int HD, class Out>
__device__ __forceinline__ void attention_unit(const DevModel& M, const DevLayer& Ly, const void* q_hi, const void* q_lo,
                                               size_t slot_frags, int kvh, int c, int L, int k, int row0, Out&& out, float* smem) {
    constexpr int FR = HD / 4 / DT::EPL;     // 16-byte fragments per lane along head_dim
    constexpr int HT = HD / 16;              // 16-wide head_dim tiles
    constexpr int BK = DT::BLOCK_KEYS, TPB = DT::TPB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int G = M.G, bpw = M.bpw;
    const int lg = __builtin_ctz((unsigned)G);         // G is 1, 2, 4 or 8 (checked at model creation): shifts, no divisions
    const int parts = kWaves >> lg, hq = wave & (G - 1), part = wave >> lg;
    const int nblk = M.ctx_pad / BK;
    const uint4 zero4 = uint4{0, 0, 0, 0};
    const int T = L + k;
    const bool mine = m >= row0 && m < row0 + k;     // tile row m belongs to this sequence
    const int head = kvh * G + hq;
    const int b0 = (c * parts + part) * bpw;       // first block of this wave's run
    uint4 qh[FR], ql[FR];
    {
        const int mq = mine ? m : row0;            // other rows mirror row0; fully masked, never written out
        const size_t q0 = (size_t)mq * M.qdim + head * HD + g * (HD / 4);
#pragma unroll
        for (int i = 0; i < FR; ++i) {
            qh[i] = load_frag<DT>(q_hi, q0 + i * DT::EPL);
            ql[i] = zero4;
            if constexpr (DT::HAS_LO) ql[i] = load_frag<DT>(q_lo, q0 + i * DT::EPL);
        }
    }
    uint4 kf[TPB][FR], vf[HT];
    auto load_block = [&](int b, uint4 (&kd)[TPB][FR], uint4 (&vd)[HT]) {
        const int bb = b < nblk ? b : nblk - 1;    // stay inside the cache allocation
        const uint4* kb = reinterpret_cast<const uint4*>(Ly.kcache) + slot_frags +
                          ((size_t)kvh * (M.ctx_pad / 16) + (size_t)bb * TPB) * FR * 64 + lane;
#pragma unroll
        for (int t = 0; t < TPB; ++t)
#pragma unroll
            for (int i = 0; i < FR; ++i) kd[t][i] = kb[(t * FR + i) * 64];
        const uint4* vb = reinterpret_cast<const uint4*>(Ly.vcache) + slot_frags +
                          (((size_t)kvh * nblk + bb) * HT) * 64 + lane;
#pragma unroll
        for (int j = 0; j < HT; ++j) vd[j] = vb[j * 64];
    };
    load_block(b0, kf, vf);
    AttState<HD> s;
    s.clear();
    const int lim = mine ? L + m - row0 : -1;          // causal: the sequence's j-th row (tile row row0 + j) sees keys 0 .. L + j
    auto kfrag = [&](int, int t, int i) { return kf[t][i]; };
    auto vfrag = [&](int, int j) { return vf[j]; };
    for (int ib = 0; ib < bpw; ++ib) {
        const int p0 = (b0 + ib) * BK;
        if (p0 >= T) break;                         // wave-uniform: later blocks of the run hold no visible key
        uint4 kn[TPB][FR], vn[HT];
        // next block of the run, fetched while this one is used; at the run's last useful block, that block
        // again (a cache hit) rather than a block the neighbouring run owns: the fetch stays unconditional, so
        // it is issued ahead of the matrix instructions, but nothing waits for the last one before the end
        const bool more = ib + 1 < bpw && p0 + BK < T;
        load_block(more ? b0 + ib + 1 : b0 + ib, kn, vn);
        if (p0 + BK - 1 > L) attention_step<DT, HD, 1, true>(s, qh, ql, kfrag, vfrag, p0, lim, g, M.att_scale, ib == 0);
        else attention_step<DT, HD, 1, false>(s, qh, ql, kfrag, vfrag, p0, lim, g, M.att_scale, ib == 0);
        if (!more) break;     // wave-uniform; the look-ahead fetch is retired at the end of the stage
#pragma unroll
        for (int t = 0; t < TPB; ++t)
#pragma unroll
            for (int i = 0; i < FR; ++i) kf[t][i] = kn[t][i];
#pragma unroll
        for (int j = 0; j < HT; ++j) vf[j] = vn[j];
    }
    merge_runs<HD>(s, G, parts, hq, part, row0, k, out, smem);
}

// The same unit for groups of 4 or 8 heads: the blocks of a run are needed by all G waves that walk it, so they are staged
// in LDS once, two blocks of every run per step, by loads that deliver straight into it; a step's successor is under way
// while it is used.  (Fetched by each wave for itself a unit pulls G times the bytes through its compute unit's load path,
// and a lane holds 128 registers of them.)  smem: at least kStagedBytes and merge_runs' area.
template <class DT, int HD, int G>
struct AttStaged {
    static constexpr int FR = HD / 4 / DT::EPL, HT = HD / 16, TPB = DT::TPB;
    static constexpr int PARTS = kWaves / G;
    static constexpr int NF = TPB * FR + HT;             // fragments of a key block: keys, then values
    static constexpr int NPW = PARTS * 2 * NF / kWaves;  // loads per wave and step of two blocks
    static constexpr int kStepBytes = PARTS * 2 * NF * 1024, kStagedBytes = 2 * kStepBytes;
    static_assert(PARTS * NF % kWaves == 0 && (G == 4 || G == 8), "");
};
template <class DT, int HD, int G>
__device__ __forceinline__ void attention_unit_staged(const DevModel& M, const DevLayer& Ly, const void* q_hi, const void* q_lo,
                                                      size_t slot_frags, int kvh, int c, int L, int k, int row0, float* part_out,
                                                      float* smem) {
    using C = AttStaged<DT, HD, G>;
    constexpr int FR = C::FR, BK = DT::BLOCK_KEYS, PARTS = C::PARTS, NF = C::NF, NPW = C::NPW;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int hq = wave % G, part = wave / G, bpw = M.bpw;
    const bool mine = m >= row0 && m < row0 + k;         // tile row m belongs to this sequence
    const int T = L + k;
    const int head = kvh * G + hq;
    const int first = c * PARTS * bpw;                   // first block of the unit
    const int b0 = first + part * bpw;                   // first block of this wave's run
    uint4 qh[FR], ql[FR];
    {
        const int mq = mine ? m : row0;                  // other rows mirror row0; never written out
        const size_t q0 = (size_t)mq * M.qdim + head * HD + g * (HD / 4);
#pragma unroll
        for (int i = 0; i < FR; ++i) {
            qh[i] = load_frag<DT>(q_hi, q0 + i * DT::EPL);
            ql[i] = uint4{0, 0, 0, 0};
            if constexpr (DT::HAS_LO) ql[i] = load_frag<DT>(q_lo, q0 + i * DT::EPL);
        }
    }
    const char* kc = reinterpret_cast<const char*>(Ly.kcache) + slot_frags * 16 + (size_t)kvh * M.ctx_pad * HD * DT::ESZ;
    const char* vc = reinterpret_cast<const char*>(Ly.vcache) + slot_frags * 16 + (size_t)kvh * M.ctx_pad * HD * DT::ESZ;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    const int steps_all = (bpw + 1) / 2;
    int steps = (T - first * BK + 2 * BK - 1) / (2 * BK);    // the first run's steps with visible keys: it has the most
    if (steps > steps_all) steps = steps_all;
    auto fetch = [&](int b, int place, int f) {          // fragment f of block b to place (in fragments) of the ring
        const char* src = f < C::TPB * FR ? kc + (size_t)b * (C::TPB * FR * 1024) + f * 1024
                                          : vc + (size_t)b * (C::HT * 1024) + (f - C::TPB * FR) * 1024;
        load_to_lds(src, lane * 16, lds0 + place * 1024);
    };
    // step s: [run][block of the step][fragment]; an odd run's last step has one block per run
    auto issue = [&](int s) {
        const int base = (s & 1) * (PARTS * 2 * NF);
        if (2 * s + 1 < bpw) {
#pragma unroll
            for (int q = 0; q < NPW; ++q) {
                const int x = wave * NPW + q;
                fetch(first + x / (2 * NF) * bpw + 2 * s + x / NF % 2, base + x, x % NF);
            }
        } else {
#pragma unroll
            for (int q = 0; q < NPW / 2; ++q) {
                const int x = wave * (NPW / 2) + q;
                fetch(first + x / NF * bpw + 2 * s, base + x / NF * (2 * NF) + x % NF, x % NF);
            }
        }
    };
    issue(0);
    // the queries are used from here on as far as the compiler can tell: its wait for them is the first step's as well
#pragma unroll
    for (int i = 0; i < FR; ++i)
        asm volatile("" : "+v"(qh[i].x), "+v"(qh[i].y), "+v"(qh[i].z), "+v"(qh[i].w), "+v"(ql[i].x), "+v"(ql[i].y), "+v"(ql[i].z), "+v"(ql[i].w));
    wait_vm<0>();
    AttState<HD> s;
    s.clear();
    const int lim = mine ? L + m - row0 : -1;            // causal: the sequence's j-th row (tile row row0 + j) sees keys 0 .. L + j
    for (int st = 0; st < steps; ++st) {
        // The loads of this step are the only ones under way.  Behind the barrier they are there for all waves, and all
        // waves are done with the step before, whose place the next one takes.
        if (st) {
            __builtin_amdgcn_s_waitcnt(0xC07F);          // no LDS read is pending
            wait_vm<0>();
        }
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (st + 1 < steps) issue(st + 1);
        const char* at = reinterpret_cast<const char*>(smem) + ((st & 1) * PARTS + part) * (2 * NF * 1024) + lane * 16;
        auto kf = [&](int b, int t, int i) { return *reinterpret_cast<const uint4*>(at + (b * NF + t * FR + i) * 1024); };
        auto vf = [&](int b, int j) { return *reinterpret_cast<const uint4*>(at + (b * NF + C::TPB * FR + j) * 1024); };
        const int p0 = (b0 + 2 * st) * BK;
        if (p0 < T) {                                    // wave-uniform
            if (2 * st + 1 >= bpw || p0 + BK >= T) attention_step<DT, HD, 1, true>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, st == 0);
            else if (p0 + 2 * BK - 1 > L) attention_step<DT, HD, 2, true>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, st == 0);
            else attention_step<DT, HD, 2, false>(s, qh, ql, kf, vf, p0, lim, g, M.att_scale, st == 0);
        }
    }
    __syncthreads();                                     // the runs' sums take the place of the blocks
    merge_runs<HD>(s, G, PARTS, hq, part, row0, k, PartialOut<HD>{part_out}, smem);
}

// The same unit for a sequence with few rows: its rows times the group's heads fill fewer 16-row tiles than a tile
// per head, of which a decoding step has one row each.  A unit is one such tile: lane m has the pair 16 t + m = row * G + head.
// A run is a wave's, as its blocks are no one else's, and comes straight into registers: no block is waited for by more than
// the wave that uses it, and several workgroups (of PARTS waves) share a compute unit.  smem: kLdsFloats.
template <class DT, int HD, int G>
struct AttPacked {
    static constexpr int PARTS = kWaves / G, kThreads = PARTS * 64;
    static constexpr int FR = HD / 4 / DT::EPL, HT = HD / 16, BK = DT::BLOCK_KEYS, TPB = DT::TPB;
    static constexpr int kRunFloats = (HD / 4 + 2) * 64;         // a run's sums in LDS: numerators, references, denominators
    static constexpr int kLdsFloats = PARTS > 1 ? kRunFloats : 1;
    AttState<HD> s;                                              // sums of the run that walk() walked
    uint4 qh[FR], ql[FR], kb[2][TPB][FR], vb[2][HT];
    const uint4* kc;                                             // the kv head's keys and values, this lane's of each fragment
    const uint4* vc;
    int lane, g, row, hq, lim, T, bpw, L;                        // row: of the sequence; lim: its last visible key, -1 if it has no such row
    float scale;
    __device__ __forceinline__ AttPacked(const DevModel& M, const DevLayer& Ly, size_t slot_frags, int kvh, int t, int L_, int k) {
        lane = threadIdx.x & 63;
        g = lane >> 4;
        row = (16 * t + (lane & 15)) / G;
        hq = (16 * t + (lane & 15)) % G;
        L = L_;
        T = L + k;
        lim = row < k ? L + row : -1;
        bpw = M.bpw;
        scale = M.att_scale;
        kc = reinterpret_cast<const uint4*>(Ly.kcache) + slot_frags + (size_t)kvh * (M.ctx_pad / BK) * (TPB * FR * 64) + lane;
        vc = reinterpret_cast<const uint4*>(Ly.vcache) + slot_frags + (size_t)kvh * (M.ctx_pad / BK) * (HT * 64) + lane;
    }
    __device__ __forceinline__ void load_queries(const DevModel& M, const void* q_hi, const void* q_lo, int kvh, int row0) {
        const size_t q0 = (size_t)(row0 + (lim >= 0 ? row : 0)) * M.qdim + (kvh * G + hq) * HD + g * (HD / 4);
#pragma unroll
        for (int i = 0; i < FR; ++i) {
            qh[i] = load_frag<DT>(q_hi, q0 + i * DT::EPL);
            ql[i] = uint4{0, 0, 0, 0};
            if constexpr (DT::HAS_LO) ql[i] = load_frag<DT>(q_lo, q0 + i * DT::EPL);
        }
    }
    // steps of the run from block b0 on with visible keys
    __device__ __forceinline__ int steps(int b0) const {
        const int n = (T - b0 * BK + 2 * BK - 1) / (2 * BK);
        return n < (bpw + 1) / 2 ? n : (bpw + 1) / 2;
    }
    // whether step st of that run has a second block with visible keys
    __device__ __forceinline__ bool two(int b0, int st) const { return 2 * st + 1 < bpw && (b0 + 2 * st + 1) * BK < T; }
    __device__ __forceinline__ void load_keys(int b0, int st) {
        const uint4* p = kc + (size_t)(b0 + 2 * st) * (TPB * FR * 64);
#pragma unroll
        for (int x = 0; x < TPB * FR; ++x) kb[0][x / FR][x % FR] = p[x * 64];
        if (two(b0, st))
#pragma unroll
            for (int x = 0; x < TPB * FR; ++x) kb[1][x / FR][x % FR] = p[(TPB * FR + x) * 64];
    }
    // (values of no visible block count as zero, with weights of zero: what is there may be no number)
    __device__ __forceinline__ void load_values(int b0, int st) {
        const uint4* p = vc + (size_t)(b0 + 2 * st) * (HT * 64);
#pragma unroll
        for (int j = 0; j < HT; ++j) vb[0][j] = p[j * 64];
        if (two(b0, st))
#pragma unroll
            for (int j = 0; j < HT; ++j) vb[1][j] = p[(HT + j) * 64];
        else
#pragma unroll
            for (int j = 0; j < HT; ++j) vb[1][j] = uint4{0, 0, 0, 0};
    }
    // Step st of the run from block b0 on.  next_keys: asks for the step to come; its values follow behind.
    template <class Next>
    __device__ __forceinline__ void step(int b0, int st, Next&& next_keys) {
        const int p0 = (b0 + 2 * st) * BK, end = two(b0, st) ? lim : p0 + BK - 1;
        auto kf = [&](int b, int tt, int i) { return kb[b][tt][i]; };
        auto vf = [&](int b, int j) { return vb[b][j]; };
        attention_step<DT, HD, 2, true>(s, qh, ql, kf, vf, p0, lim < end ? lim : end, g, scale, st == 0, next_keys);
    }
    // The run from block b0 on, to its end.
    __device__ __forceinline__ void walk(const DevModel& M, const void* q_hi, const void* q_lo, int kvh, int row0, int b0) {
        const int n = steps(b0);
        s.clear();
        if (n > 0) {
            load_queries(M, q_hi, q_lo, kvh, row0);
            load_keys(b0, 0);
            load_values(b0, 0);
        }
#pragma unroll 1
        for (int st = 0; st < n; ++st) {
            step(b0, st, [&] {
                if (st + 1 < n) load_keys(b0, st + 1);
            });
            if (st + 1 < n) load_values(b0, st + 1);
        }
        wait_vm<0>();                                            // (nothing is under way: the last step asks for no other)
        s.close();
    }
    __device__ __forceinline__ void put(float* lds) const {
#pragma unroll
        for (int j = 0; j < HT; ++j) reinterpret_cast<v4f*>(lds)[j * 64 + lane] = s.o[j];
        lds[HT * 256 + lane] = s.m;
        lds[HT * 256 + 64 + lane] = s.l;
    }
};
template <class DT, int HD, int G>
__device__ __forceinline__ void attention_unit_packed(const DevModel& M, const DevLayer& Ly, const void* q_hi, const void* q_lo,
                                                      size_t slot_frags, int kvh, int c, int t, int L, int k, int row0, float* part_out,
                                                      float* smem) {
    using A = AttPacked<DT, HD, G>;
    constexpr int HT = A::HT, PARTS = A::PARTS;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    A at(M, Ly, slot_frags, kvh, t, L, k);
    at.walk(M, q_hi, q_lo, kvh, row0, (c * PARTS + part) * at.bpw);
    AttState<HD>& s = at.s;
    if constexpr (PARTS == 2) {                          // the second run is added to the first, as merge_runs does
        if (part == 1) at.put(smem);
        __syncthreads();
        if (part == 1) return;
        AttState<HD> s1;
#pragma unroll
        for (int j = 0; j < HT; ++j) s1.o[j] = reinterpret_cast<v4f*>(smem)[j * 64 + at.lane];
        s1.m = smem[HT * 256 + at.lane];
        s1.l = smem[HT * 256 + 64 + at.lane];
        s.add(s1);
    }
    if (at.lim < 0) return;
    float* out = part_out + ((size_t)at.hq * kRows + row0 + at.row) * (HD + kPartRow);
#pragma unroll
    for (int j = 0; j < HT; ++j) *reinterpret_cast<v4f*>(out + j * 16 + at.g * 4) = s.o[j];
    if (at.g == 0) *reinterpret_cast<float2*>(out + HD) = float2{s.m, s.l};
}

// The same for a sequence whose keys are few (at most kWaves runs): a workgroup of eight waves walks all of a (kv head, tile of
// pairs) and adds the runs and chunks up in LDS, in their order and with the operations of merge_runs and merge_chunks: no
// partials, no launch to merge them.  smem: kRunFloats per run.
template <class DT, int HD, int G>
__device__ __forceinline__ void attention_whole_packed(const DevModel& M, const DevLayer& Ly, const void* q_hi, const void* q_lo,
                                                       size_t slot_frags, int kvh, int t, int L, int k, int row0, int k_rows, float* smem) {
    using A = AttPacked<DT, HD, G>;
    constexpr int HT = A::HT, PARTS = A::PARTS;
    const int run = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    A at(M, Ly, slot_frags, kvh, t, L, k);
    const int bpw = at.bpw, runs = (at.T + bpw * A::BK - 1) / (bpw * A::BK), b0 = run * bpw;
    if (run < runs) {
        at.walk(M, q_hi, q_lo, kvh, row0, b0);
        at.put(smem + run * A::kRunFloats);
    }
    __syncthreads();
    const int j = threadIdx.x >> 6;                      // 16 columns of a pair: a lane has four of them
    if (j >= HT || at.lim < 0) return;
    auto part = [&](int r, float& m, float& l) {
        const float* p = smem + r * A::kRunFloats;
        m = p[HT * 256 + at.lane];
        l = p[HT * 256 + 64 + at.lane];
        return reinterpret_cast<const v4f*>(p)[j * 64 + at.lane];
    };
    float ref = 0.f;
    double den = 0.;
    v4f num;
    const int chunks = at.lim / (PARTS * bpw * A::BK) + 1;                // with keys that the row sees
    for (int c = 0; c < chunks; ++c) {
        float m, l;
        v4f o = part(c * PARTS, m, l);
        if (PARTS == 2 && c * PARTS + 1 < runs) {        // AttState::add
            float m1, l1;
            const v4f o1 = part(c * PARTS + 1, m1, l1);
            const bool up = att_outgrown(m1, m);
            const float a = up ? exp2_fast(m - m1) : 1.f;
            m = up ? m1 : m;
            const float w = m1 == -INFINITY ? 0.f : exp2_fast(m1 - m);
            l = fmaf(w, l1, l * a);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(w, o1[e], o[e] * a);
        }
        if (c == 0) {
            ref = m;
            den = l;
            num = o;
            continue;
        }
        if (att_outgrown(m, ref)) {
            const float a = exp2_fast(ref - m);
            ref = m;
            den *= a;
            num = num * a;
        }
        const float w = m == -INFINITY ? 0.f : exp2_fast(m - ref);
        den = fma((double)w, (double)l, den);
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] = fmaf(w, o[e], num[e]);
    }
    store_gemm_in4<DT>(M.O, k_rows, row0 + at.row, (kvh * G + at.hq) * HD + j * 16 + at.g * 4, num * (1.0f / (float)den));
}

// Merge of the chunk partials of one (head, row) in chunk order by one wave, with the prefill pass's operations (PfTotals::add)
// in its order: lanes first hold one chunk each (reference, weight, denominator), then one slice of head_dim each.  The
// denominators, one after the other and hundreds of them in a long context, are added in 64 bits.  base: the row's partial of
// chunk 0; cstride: floats from chunk to chunk.  num[i]: normalised output of head_dim column lane + 64 i.
template <int HD>
__device__ __forceinline__ void merge_chunks(const float* base, size_t cstride, int nch, int lane, float (&num)[HD / 64]) {
    constexpr int PER = HD / 64;
    float ref = 0.f;
    double den = 0.;
    // numerators of the first chunks are fetched together with the references: one memory round trip
    constexpr int CPRE = 24;
    float pre[CPRE][PER];
#pragma unroll
    for (int j = 0; j < CPRE; ++j) {
        const float* pj = base + (size_t)(j < nch ? j : nch - 1) * cstride;
#pragma unroll
        for (int i = 0; i < PER; ++i) pre[j][i] = pj[lane + 64 * i];
    }
    for (int c0 = 0; c0 < nch; c0 += 64) {        // groups of 64 chunks, in order
        const int cc = c0 + lane;
        const bool on = cc < nch;
        const float* p = base + (size_t)(on ? cc : c0) * cstride;
        const float mc = on ? p[HD] : -INFINITY;
        const float dc = on ? p[HD + 1] : 0.f;
        const int ng = nch - c0 < 64 ? nch - c0 : 64;
        int j0 = 0;
        if (c0 == 0) {                            // the first chunk is copied
            ref = lane_value(mc, 0);
            den = lane_value(dc, 0);
#pragma unroll
            for (int i = 0; i < PER; ++i) num[i] = pre[0][i];
            j0 = 1;
        }
        if (__builtin_amdgcn_ballot_w64(att_outgrown(mc, ref)) == 0) {      // the usual case: all against one reference
            const float wt = mc == -INFINITY ? 0.f : exp2_fast(mc - ref);
            const double wd = (double)wt * (double)dc;                     // exact
            // (lanes past the last chunk hold weight and denominator 0, and what is fetched there is the last chunk's)
            if (c0 == 0) {
#pragma unroll
                for (int j = 1; j < CPRE; ++j) {
                    const float wj = lane_value(wt, j);
                    den += lane_value(wd, j);
#pragma unroll
                    for (int i = 0; i < PER; ++i) num[i] = fmaf(wj, pre[j][i], num[i]);
                }
                j0 = CPRE;
            }
            constexpr int CB = 8;                  // the others, CB at a time
            for (int j = j0; j < ng; j += CB) {
                float x[CB][PER];
#pragma unroll
                for (int u = 0; u < CB; ++u) {
                    const float* pj = base + (size_t)(c0 + (j + u < ng ? j + u : ng - 1)) * cstride;
#pragma unroll
                    for (int i = 0; i < PER; ++i) x[u][i] = pj[lane + 64 * i];
                }
#pragma unroll
                for (int u = 0; u < CB; ++u) {
                    const float wj = lane_value(wt, j + u);
                    den += lane_value(wd, j + u);
#pragma unroll
                    for (int i = 0; i < PER; ++i) num[i] = fmaf(wj, x[u][i], num[i]);
                }
            }
        } else {
            for (int j = j0; j < ng; ++j) {
                const float mj = lane_value(mc, j);
                const float* pj = base + (size_t)(c0 + j) * cstride;
                if (att_outgrown(mj, ref)) {
                    const float a = exp2_fast(ref - mj);
                    ref = mj;
                    den *= a;
#pragma unroll
                    for (int i = 0; i < PER; ++i) num[i] *= a;
                }
                const float wj = mj == -INFINITY ? 0.f : exp2_fast(mj - ref);
                den = fma((double)wj, (double)lane_value(dc, j), den);
#pragma unroll
                for (int i = 0; i < PER; ++i) num[i] = fmaf(wj, pj[lane + 64 * i], num[i]);
            }
        }
    }
    const float inv = 1.0f / (float)den;
#pragma unroll
    for (int i = 0; i < PER; ++i) num[i] *= inv;
}

}  // namespace amusd
