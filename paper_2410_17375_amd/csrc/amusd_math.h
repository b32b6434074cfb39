// Device helpers shared by the kernels of the verify pass (amusd_kernels.hip) and of the prefill pass
// (amusd_prefill.hip): element types, matrix-core operand layouts, lane exchanges, the K walk of a contraction.
// A token row must get the same bits from both, so what a row's value depends on is written once, here, and every
// multiply-add that is to be one operation says so (the compiler fuses nothing by itself).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>

#include <type_traits>

#include "amusd_launch.h"

#pragma clang fp contract(off)

namespace amusd {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- dtype traits
struct BF16 {
    static constexpr int EPL = 8;         // elements in a lane's 16-byte fragment
    static constexpr int KB = 32;         // contraction elements per fragment (4 lane groups x EPL)
    static constexpr int ESZ = 2;
    static constexpr int TPB = 2;         // 16-key score tiles per value block
    static constexpr int BLOCK_KEYS = 32;
    static constexpr bool HAS_LO = true;
    static __device__ __forceinline__ v4f mfma(uint4 a, uint4 b, v4f c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    }
    // Attention operands (cache, queries, softmax weights) are IEEE half: the same 2 bytes per element as
    // bf16 with three more mantissa bits; their magnitudes (keys, values, queries O(1), weights up to
    // 2^kAttSlack) sit well inside the half range, and stores of the cache and the queries clamp to it.
    static __device__ __forceinline__ v4f mfma_att(uint4 a, uint4 b, v4f c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t att_bits(float x) {
        const float c = fminf(fmaxf(x, -65504.f), 65504.f);
        return (uint32_t)__half_as_ushort(__float2half_rn(c));
    }
    static __device__ __forceinline__ float att_float(uint32_t b) { return __half2float(__ushort_as_half((unsigned short)b)); }
    // hi and lo halves of two softmax weights (at most 2^kAttSlack: nothing to clamp), packed.  The subtraction of a half from its
    // float is one mixed-precision instruction (an exact fused multiply-add by one; the compiler converts and subtracts).
    static __device__ __forceinline__ void att_split2(float a, float b, uint32_t& hi, uint32_t& lo) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        typedef float f2 __attribute__((ext_vector_type(2)));
        hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, h2));
        f2 r;
        asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r.x) : "v"(hi), "v"(a));
        asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r.y) : "v"(hi), "v"(b));
        lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, h2));
    }
};
struct FP32 {
    static constexpr int EPL = 4;
    static constexpr int KB = 16;
    static constexpr int ESZ = 4;
    static constexpr int TPB = 1;
    static constexpr int BLOCK_KEYS = 16;
    static constexpr bool HAS_LO = false;
    static __device__ __forceinline__ v4f mfma(uint4 a, uint4 b, v4f c) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ v4f mfma_att(uint4 a, uint4 b, v4f c) { return mfma(a, b, c); }
    static __device__ __forceinline__ uint32_t att_bits(float x) { return __float_as_uint(x); }
    static __device__ __forceinline__ float att_float(uint32_t b) { return __uint_as_float(b); }
};

__device__ __forceinline__ uint32_t bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// store a query element: fp32 as is; 16-bit models as hi + lo halves of the attention element type
template <class DT>
__device__ __forceinline__ void store_act(void* hi, void* lo, size_t idx, float x) {
    if constexpr (DT::HAS_LO) {
        uint32_t h = DT::att_bits(x);
        uint32_t l = DT::att_bits(x - DT::att_float(h));
        reinterpret_cast<uint16_t*>(hi)[idx] = (uint16_t)h;
        reinterpret_cast<uint16_t*>(lo)[idx] = (uint16_t)l;
    } else {
        reinterpret_cast<float*>(hi)[idx] = x;
    }
}

// GEMM inputs are kept in matrix-core operand order, so that a wave fetches the
// 16 rows x one K block it needs with ONE contiguous 1 KiB load, exactly like
// a weight fragment: buf[kb][part][lane = g*16 + slot][EPL elements], where g
// selects the lane group's EPL columns of the K block.
//   fp32        : one part, slot = row.
//   bf16, k <= 8: one part; slots 0-7 hold the hi halves of rows 0-7 and slots
//                 8-15 their lo halves (x = hi + lo), so one MFMA yields W.hi in
//                 result columns 0-7 and W.lo in columns 8-15;
//   bf16, k > 8 : two parts (hi, lo), slot = row.
// In both bf16 forms a wave adds its W.hi and W.lo sums before the cross-wave
// reduction, so a row's value does not depend on which form carried it.
template <class DT>
__device__ __forceinline__ void store_gemm_in(void* buf, int k_rows, int m, int col, float x) {
    const int kb = col / DT::KB, g = (col % DT::KB) / DT::EPL, e = col % DT::EPL;
    if constexpr (DT::HAS_LO) {
        const uint32_t h = bf16_rne(x);
        const uint32_t l = bf16_rne(x - bf16_to_f32(h));
        uint16_t* b = reinterpret_cast<uint16_t*>(buf);
        if (k_rows <= 8) {
            const size_t base = ((size_t)kb * 64 + g * 16 + m) * 8 + e;
            b[base] = (uint16_t)h;
            b[base + 8 * 8] = (uint16_t)l;                 // slot m + 8
        } else {
            const size_t base = ((size_t)kb * 128 + g * 16 + m) * 8 + e;
            b[base] = (uint16_t)h;
            b[base + 64 * 8] = (uint16_t)l;                // part 1
        }
    } else {
        reinterpret_cast<float*>(buf)[((size_t)kb * 64 + g * 16 + m) * 4 + e] = x;
    }
}

// four neighbouring columns (col a multiple of 4) of one row
template <class DT>
__device__ __forceinline__ void store_gemm_in4(void* buf, int k_rows, int m, int col, v4f x) {
    const int kb = col / DT::KB, g = (col % DT::KB) / DT::EPL, e = col % DT::EPL;
    if constexpr (DT::HAS_LO) {
        uint32_t h[4], l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = bf16_rne(x[i]);
            l[i] = bf16_rne(x[i] - bf16_to_f32(h[i]));
        }
        uint16_t* b = reinterpret_cast<uint16_t*>(buf) + ((size_t)kb * (k_rows <= 8 ? 64 : 128) + g * 16 + m) * 8 + e;
        *reinterpret_cast<uint2*>(b) = uint2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
        *reinterpret_cast<uint2*>(b + (k_rows <= 8 ? 8 : 64) * 8) = uint2{l[0] | (l[1] << 16), l[2] | (l[3] << 16)};
    } else {
        *reinterpret_cast<v4f*>(reinterpret_cast<float*>(buf) + ((size_t)kb * 64 + g * 16 + m) * 4 + e) = x;
    }
}

// Element index of key `pos`, head_dim column `c` in a kv head's key cache.  Keys are kept in the operand
// order of the score product: [16-key tile][fragment i][lane = g*16 + key%16][EPL], where lane group g owns
// columns g*hd/4 .. (g+1)*hd/4 and fragment i its i-th run of EPL columns, so a wave fetches one
// (tile, fragment) with a single contiguous 1 KiB load.
template <class DT>
__device__ __forceinline__ size_t kcache_index(int hd, int pos, int c) {
    const int q = hd / 4, g = c / q, w = c % q;
    return ((((size_t)(pos >> 4) * (q / DT::EPL) + w / DT::EPL) * 64) + g * 16 + (pos & 15)) * DT::EPL + w % DT::EPL;
}

// Weights are read once per pass: a non-temporal load keeps them from evicting
// the (re-read) activations from L2.
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const u4 v = __builtin_nontemporal_load(reinterpret_cast<const u4*>(p));
    return uint4{v.x, v.y, v.z, v.w};
}

template <class DT>
__device__ __forceinline__ uint4 load_frag(const void* base, size_t elem_index) {
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(base) + elem_index * DT::ESZ);
}

// Forces a (wave-uniform) kernel argument into a scalar register at this point of the program.  Left to itself
// the compiler loads an argument where it is first used, often behind a branch; a stage that starts by asking
// for everything it needs waits for argument memory once instead of several times in a row.
template <class T>
__device__ __forceinline__ void pin_scalar(const T& x) { asm volatile("" ::"s"(x)); }

// The value that lane (l ^ OFF) holds, without going through the LDS crossbar (`__shfl_xor` compiles to
// ds_bpermute, 50-100 clocks each, and these exchanges sit in chains on the critical path of every stage's end):
// data-parallel-primitive modifiers inside a row of 16 lanes, the gfx950 row and half-wave swaps across rows.
template <int OFF>
__device__ __forceinline__ uint32_t lane_xor_u(uint32_t v) {
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "one bit of the lane index");
    const int x = (int)v;
    if constexpr (OFF == 1) {
        return (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false);        // quad_perm:[1,0,3,2]
    } else if constexpr (OFF == 2) {
        return (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false);        // quad_perm:[2,3,0,1]
    } else if constexpr (OFF == 4) {
        const int t = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xf, 0x5, false);          // row_shl:4 into lanes 0-3, 8-11
        return (uint32_t)__builtin_amdgcn_update_dpp(t, x, 0x114, 0xf, 0xa, false);       // row_shr:4 into lanes 4-7, 12-15
    } else if constexpr (OFF == 8) {
        return (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x128, 0xf, 0xf, false);       // row_ror:8
    } else if constexpr (OFF == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // p[0]: rows 0,0,2,2   p[1]: rows 1,1,3,3
        return (threadIdx.x & 16) ? p[0] : p[1];
    } else {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // p[0]: lanes 0-31 twice   p[1]: lanes 32-63 twice
        return (threadIdx.x & 32) ? p[0] : p[1];
    }
}
template <int OFF>
__device__ __forceinline__ float lane_xor(float v) { return __uint_as_float(lane_xor_u<OFF>(__float_as_uint(v))); }
template <int OFF>
__device__ __forceinline__ int lane_xor(int v) { return (int)lane_xor_u<OFF>((uint32_t)v); }
template <int OFF>
__device__ __forceinline__ float wave_xor_add(float v) { return v + lane_xor<OFF>(v); }
// lane j's value in every lane (j the same in all lanes)
__device__ __forceinline__ float lane_value(float v, int j) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), j));
}
__device__ __forceinline__ double lane_value(double v, int j) {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, j), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), j);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// ---------------------------------------------------------------- loads that deliver into LDS
// 16 bytes per lane from base + offset to LDS bytes dst + 16 lane.  In assembly, because the compiler takes the builtin
// for an access to all of LDS and then waits for every LDS read at once (lgkmcnt(0)) throughout the loop; it has no result
// registers, and every wait for it is written out (wait_vm).  m0 is named as overwritten: the compiler keeps it from one
// of its own loads of this kind to the next, and a kernel may hold both.  (It warns that m0 is a reserved register; that
// is why nothing of its own can be kept in it across the statement.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(const char* base, unsigned offset, unsigned dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(dst) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ---------------------------------------------------------------- K walk of a contraction
// A wave's share of the K blocks of a GEMM stage, and where in it the wave starts its walk: blocks
// kb0 + stride * ((i + rot) mod S), i = 0 .. S-1.
// K split: SIMD s hosts waves s and s+4; they share the K quarter of their SIMD, the first of them taking
// old_share sixteenths (the first wave of a SIMD wins the issue arbitration and streams faster, but which split is
// fastest was measured per stage, and it also shifts where the second wave's stream starts).
// Interleaved form: the waves take every eighth block instead (the two waves of a SIMD neighbouring ones), so that a
// workgroup's eight streams move through the tile as one window of 8 KiB.
struct KSlice {
    int kb0, S, rot, stride;
};
__host__ __device__ __forceinline__ KSlice k_slice(int kblocks, int wg, int wave, bool stagger, int rot_wg, int rot_wave,
                                          bool interleave, int old_share) {
    const int simd = wave & 3, young = wave >> 2;
    const int q0 = (kblocks * simd) / 4, q1 = (kblocks * (simd + 1)) / 4;
    const int cut = q0 + ((q1 - q0) * old_share + 8) / 16;
    KSlice k;
    k.kb0 = young ? cut : q0;
    k.S = (young ? q1 : cut) - k.kb0;
    k.stride = 1;
    if (interleave) {
        k.kb0 = simd * 2 + young;
        k.S = (kblocks - k.kb0 + kWaves - 1) / kWaves;
        k.stride = kWaves;
    }
    k.rot = stagger && k.S > 0 ? (int)(((unsigned)wg * (unsigned)rot_wg + (unsigned)wave * (unsigned)rot_wave) % (unsigned)k.S) : 0;
    return k;
}

// How each projection stage splits its K blocks over the waves and where they start (k_slice), swept per stage on the
// chip.  They fix the order in which a row's products are added, for passes of every size.
struct KWalkQKV {      // no shift (short slices, two tile counts: measured slower with one); the first wave of a SIMD takes
                       // 12 of 32 blocks: 0.4 us per launch faster than an even split (10 likewise; 4, 12, odd values not)
    static constexpr bool kStagger = false, kInterleave = false;
    static constexpr int kRotWg = 0, kRotWave = 0, kOldShare = 6;
};
struct KWalkOproj {    // fastest when nobody is shifted by its wave
    static constexpr bool kStagger = true, kInterleave = false;
    static constexpr int kRotWg = 5, kRotWave = 0, kOldShare = 8;
};
struct KWalkWide {     // gate/up and LM head: an even wave coefficient costs 0.3-6 us per launch
    static constexpr bool kStagger = true, kInterleave = false;
    static constexpr int kRotWg = 5, kRotWave = 11, kOldShare = 8;
};
struct KWalkDown {     // fastest when all workgroups start alike and only the waves differ; interleaved 0.4 us per launch faster
    static constexpr bool kStagger = true, kInterleave = true;
    static constexpr int kRotWg = 0, kRotWave = 5, kOldShare = 8;
};
template <class W>
__host__ __device__ __forceinline__ KSlice k_slice_of(int kblocks, int wg, int wave) {
    return k_slice(kblocks, wg, wave, W::kStagger, W::kRotWg, W::kRotWave, W::kInterleave, W::kOldShare);
}

// ---------------------------------------------------------------- a row's arithmetic between the contractions
__device__ __forceinline__ float square_pair(float x1, float x2) { return fmaf(x2, x2, x1 * x1); }
__device__ __forceinline__ void rotate_pair(float x1, float x2, float c, float s, float& y1, float& y2) {
    y1 = fmaf(x1, c, -(x2 * s));
    y2 = fmaf(x1, s, x2 * c);
}
__device__ __forceinline__ float swiglu(float gate, float up) { return gate / (1.0f + __expf(-gate)) * up; }
// value-cache element of (position, feature column c) inside a kv head's cache: [key block][16-feature tile][64 lanes][EPL]
template <class DT>
__device__ __forceinline__ size_t vcache_index(int hd, int pos, int c) {
    constexpr int BK = DT::BLOCK_KEYS;
    const int b = pos / BK, q = pos % BK;
    const int e = (q / 16) * 4 + (q % 4), g = (q % 16) / 4;
    return (((size_t)b * (hd / 16) + c / 16) * 64 + g * 16 + c % 16) * DT::EPL + e;
}
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }
// keeps the better of this lane's (value, index) and lane (l ^ OFF)'s
template <int OFF>
__device__ __forceinline__ void keep_better_xor(float& bv, int& bi) {
    const float ov = lane_xor<OFF>(bv);
    const int oi = lane_xor<OFF>(bi);
    if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
}


// Workgroup `wg` of those behind a pass's last kernel's own: its part of the logits to pinned host memory, a thread 16 bytes, while
// the others finish the pass.  Fetching them afterwards takes a launch or a copy: 16 KB 17 us by hipMemcpy, 7.5 by k_export.
__device__ __forceinline__ void export_logits(const DevModel& M, int bytes, int wg) {
    const int at = (wg * (int)blockDim.x + (int)threadIdx.x) * 16;
    if (at < bytes) *reinterpret_cast<uint4*>(M.export_host + at) = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(M.logits) + at);
}
// .. how many
inline int export_wgs(int bytes, int threads) { return (bytes + threads * 16 - 1) / (threads * 16); }

}  // namespace amusd
