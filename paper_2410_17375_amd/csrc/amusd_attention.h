// The attention work unit and the merge of chunk partials, shared by the verify pass and the prefill pass: a row's
// scores, softmax and sums are computed by the same code at the same absolute key boundaries in both, so its bits do
// not depend on which of them it went through.
#pragma once
#include "amusd_math.h"

namespace amusd {

constexpr int kAttPad = 4;    // row padding of the attention partials (spreads LDS banks)
constexpr int kPartRow = 4;   // floats appended to a partial's numerator: max, denominator, 2 pad (keeps 16-byte alignment)

// One unit: chunk c of kv head kvh (the 8/G runs of bpw key blocks that the waves of a workgroup walk) against the tile
// rows row0 .. row0+k-1, which stand at positions L .. L+k-1.  q_hi / q_lo: the tile's query rows, row-major.
// slot_frags: start of the sequence's cache, in 16-byte fragments.  Writes [head of the group][row][HD numerators, max,
// denominator, pad] to part_out.  smem: kWaves * kRows * (HD + kAttPad + 2) floats.
template <class DT, int HD>
__device__ __forceinline__ void attention_unit(const DevModel& M, const DevLayer& Ly, const void* q_hi, const void* q_lo,
                                               size_t slot_frags, int kvh, int c, int L, int k, int row0, float* part_out,
                                               float* smem) {
    constexpr int FR = HD / 4 / DT::EPL;     // 16-byte fragments per lane along head_dim
    constexpr int HT = HD / 16;              // 16-wide head_dim tiles
    constexpr int BK = DT::BLOCK_KEYS, TPB = DT::TPB;
    constexpr int HDP = HD + kAttPad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int G = M.G, bpw = M.bpw;
    const int lg = __builtin_ctz((unsigned)G);         // G is 1, 2, 4 or 8 (checked at model creation): shifts, no divisions
    const int parts = kWaves >> lg, hq = wave & (G - 1), part = wave >> lg;
    float* partO = smem;                               // [hq][part][16][HD + pad]
    float* partML = smem + kWaves * kRows * HDP;       // [hq][part][16][2]
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
    float mrun = -INFINITY, lrun = 0.f;
    v4f o[HT];
#pragma unroll
    for (int j = 0; j < HT; ++j) o[j] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int ib = 0; ib < bpw; ++ib) {
        const int p0 = (b0 + ib) * BK;
        if (p0 >= T) break;                         // wave-uniform: later blocks of the run hold no visible key
        uint4 kn[TPB][FR], vn[HT];
        // next block of the run, fetched while this one is used; at the run's last useful block, that block
        // again (a cache hit) rather than a block the neighbouring run owns: the fetch stays unconditional, so
        // it is issued ahead of the matrix instructions, but nothing waits for the last one before the end
        const bool more = ib + 1 < bpw && p0 + BK < T;
        load_block(more ? b0 + ib + 1 : b0 + ib, kn, vn);
        float sv[TPB][4];
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < TPB; ++t) {
            v4f sc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < FR; ++i) {
                sc = DT::mfma_att(kf[t][i], qh[i], sc);
                if constexpr (DT::HAS_LO) sc = DT::mfma_att(kf[t][i], ql[i], sc);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = p0 + t * 16 + g * 4 + e;
                // causal: the sequence's j-th row (tile row row0+j) sees keys 0..L+j
                sv[t][e] = mine && key <= L + m - row0 ? sc[e] * M.att_scale : -INFINITY;
                mx = fmaxf(mx, sv[t][e]);
            }
        }
        mx = fmaxf(mx, lane_xor<16>(mx));
        mx = fmaxf(mx, lane_xor<32>(mx));
        const float mnew = fmaxf(mrun, mx);
        const float mref = mnew == -INFINITY ? 0.f : mnew;
        const float alpha = __expf(mrun - mref);     // 0 for the first visible block
        float pv[TPB][4], lsum = 0.f;
#pragma unroll
        for (int t = 0; t < TPB; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                pv[t][e] = __expf(sv[t][e] - mref);
                lsum += pv[t][e];
            }
        lsum = wave_xor_add<16>(lsum);
        lsum = wave_xor_add<32>(lsum);
        lrun = fmaf(lrun, alpha, lsum);
        mrun = mnew;
        uint4 ph, pl = zero4;
        if constexpr (DT::HAS_LO) {
            uint32_t h[8], l[8];
#pragma unroll
            for (int t = 0; t < TPB; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    h[t * 4 + e] = DT::att_bits(pv[t][e]);
                    l[t * 4 + e] = DT::att_bits(pv[t][e] - DT::att_float(h[t * 4 + e]));
                }
            ph = uint4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
            pl = uint4{l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16)};
        } else {
            ph = uint4{__float_as_uint(pv[0][0]), __float_as_uint(pv[0][1]), __float_as_uint(pv[0][2]), __float_as_uint(pv[0][3])};
        }
#pragma unroll
        for (int j = 0; j < HT; ++j) {
            o[j] = o[j] * alpha;
            o[j] = DT::mfma_att(vf[j], ph, o[j]);
            if constexpr (DT::HAS_LO) o[j] = DT::mfma_att(vf[j], pl, o[j]);
        }
        if (!more) break;     // wave-uniform; the look-ahead fetch is retired at the end of the stage
#pragma unroll
        for (int t = 0; t < TPB; ++t)
#pragma unroll
            for (int i = 0; i < FR; ++i) kf[t][i] = kn[t][i];
#pragma unroll
        for (int j = 0; j < HT; ++j) vf[j] = vn[j];
    }
    // run partial to LDS: o[j][e] is head_dim index 16j + 4g + e of row m
    const int slot = hq * parts + part;
#pragma unroll
    for (int j = 0; j < HT; ++j)
        *reinterpret_cast<v4f*>(partO + ((size_t)(slot * kRows + m) * HDP + j * 16 + g * 4)) = o[j];
    if (g == 0) {
        partML[(slot * kRows + m) * 2 + 0] = mrun;
        partML[(slot * kRows + m) * 2 + 1] = lrun;
    }
    __syncthreads();
    // merge the runs of each head in run order; item = (head, row, 4 consecutive head_dim entries)
    for (int it = tid; it < G * kRows * (HD / 4); it += kThreads) {
        const int c4 = it % (HD / 4), mm = (it / (HD / 4)) % kRows, hh = it / (kRows * (HD / 4));
        if (mm < row0 || mm >= row0 + k) continue;
        float Mx = -INFINITY;
        for (int pp = 0; pp < parts; ++pp) Mx = fmaxf(Mx, partML[((hh * parts + pp) * kRows + mm) * 2]);
        float den = 0.f;
        v4f num = v4f{0.f, 0.f, 0.f, 0.f};
        for (int pp = 0; pp < parts; ++pp) {
            const int sl = hh * parts + pp;
            const float mw = partML[(sl * kRows + mm) * 2];
            const float wt = mw == -INFINITY ? 0.f : __expf(mw - Mx);
            den = fmaf(wt, partML[(sl * kRows + mm) * 2 + 1], den);
            const v4f x = *reinterpret_cast<const v4f*>(partO + ((size_t)(sl * kRows + mm) * HDP + c4 * 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) num[e] = fmaf(wt, x[e], num[e]);
        }
        float* out = part_out + ((size_t)hh * kRows + mm) * (HD + kPartRow);
        *reinterpret_cast<v4f*>(out + c4 * 4) = num;
        if (c4 == 0) { out[HD] = Mx; out[HD + 1] = den; }
    }
    __syncthreads();
}

// Merge of the chunk partials of one (head, row) in chunk order by one wave: lanes first hold one chunk each (max,
// weight, denominator), then one slice of head_dim each.  base: the row's partial of chunk 0; cstride: floats from chunk
// to chunk.  num[i]: normalised output of head_dim column lane + 64 i.
template <int HD>
__device__ __forceinline__ void merge_chunks(const float* base, size_t cstride, int nch, int lane, float (&num)[HD / 64]) {
    constexpr int PER = HD / 64;
    float Mrun = -INFINITY, den = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) num[i] = 0.f;
    // numerators of the first chunks are fetched together with the maxima: one memory round trip
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
        float Mg = mc;
        Mg = wave_max_all(Mg);
        const float Mnew = fmaxf(Mrun, Mg);       // finite: chunk 0 always holds key 0
        const float scale_old = __expf(Mrun - Mnew);
        const float wt = mc == -INFINITY ? 0.f : __expf(mc - Mnew);
        float dsum = wt * dc;
        dsum = wave_sum_all(dsum);
        den = fmaf(den, scale_old, dsum);
#pragma unroll
        for (int i = 0; i < PER; ++i) num[i] *= scale_old;
        const int ng = nch - c0 < 64 ? nch - c0 : 64;
        if (c0 == 0) {
#pragma unroll
            for (int j = 0; j < CPRE; ++j) {
                const float wj = j < ng ? lane_value(wt, j) : 0.f;
#pragma unroll
                for (int i = 0; i < PER; ++i) num[i] = fmaf(wj, pre[j][i], num[i]);
            }
        }
        for (int j = c0 == 0 ? CPRE : 0; j < ng; ++j) {
            const float wj = lane_value(wt, j);
            const float* pj = base + (size_t)(c0 + j) * cstride;
#pragma unroll
            for (int i = 0; i < PER; ++i) num[i] = fmaf(wj, pj[lane + 64 * i], num[i]);
        }
        Mrun = Mnew;
    }
    const float inv = 1.0f / den;
#pragma unroll
    for (int i = 0; i < PER; ++i) num[i] *= inv;
}

}  // namespace amusd
