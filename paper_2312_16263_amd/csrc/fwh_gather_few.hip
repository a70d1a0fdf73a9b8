// Forward gather for a few observers on a small surface (gfx950).
//
// The streaming gather (gather_stream_kernel) gives a panel split to one block that computes every
// sample of at most 8 observers, 128 panels one after the other.  With few splits most of the chip
// is idle and the launch lasts as long as one block's chain of 128 copies (0.8 us each): 107 us for
// a 2048-panel, 512-frame surface and 8 observers.  Here a wave owns one observer and one row of 61
// samples of one split, so the same splits run on 7 x 8 times as many waves, and loads its
// coefficients itself, kFewAhead panels ahead, from L2 (every observer's windows again: the reason not
// to use it where the coefficients outgrow the caches).  The splits, and the order of every sum, are the streaming
// gather's: the two give the same results bit for bit.  28 us for that surface.
#include <type_traits>

#include "fwh_internal.h"

namespace fwh {
namespace {

typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kFewAhead = 4;     // panels per batch of loads
constexpr int kFewChunk = 256;   // panels summed in FP32 before adding into the partial signal

__device__ __forceinline__ float next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130 /* wave_shl:1 */, 0xF, 0xF, true));
}

// One panel of one row, FP32: g = sum_c K_c coef_c, then the four taps into one accumulator.  rec: dword
// lane % 16 of the pair's record in every row of 16 lanes (K_0 .. K_7, w_0 .. w_3, n0w, n0), read as the
// broadcast DPP source of each FMA.  A DPP read needs two wait states after a VALU write of its source
// (s_nop: rec may come from a register copy, g and its shifts are written here).
__device__ __forceinline__ void few_panel(float &acc, float rec, uintx4 a, uintx4 b) {
    float g, t;
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %1, %3, %4 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %5 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %6 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %7 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %8 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %9 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %10 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %3, %11 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %3, %1 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_mov_b32_dpp %2, %1 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %0, %3, %2 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_mov_b32_dpp %1, %2 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %0, %3, %1 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_mov_b32_dpp %2, %1 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %0, %3, %2 row_newbcast:11 row_mask:0xf bank_mask:0xf"
        : "+v"(acc), "=&v"(g), "=&v"(t)
        : "v"(rec), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]));
}

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

template <typename TS>
__global__ __launch_bounds__(256) void gather_few_kernel(GatherArgs a, int64_t rows) {
    constexpr bool kBf = std::is_same<TS, uint16_t>::value;
    constexpr int EB = 4 * (int)sizeof(TS);
    constexpr int NT = kBf ? 4 : 1;  // accumulators, as in the streaming gather
    const int64_t P = a.P, nt_max = a.nt_max;
    const int O = (int)a.O;  // at most kLdsWaves, one tile
    const int lane = threadIdx.x & 63;
    // wave -> (split, row, observer), observers fastest: neighbouring waves read the same panels at nearly
    // the same indices
    const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= rows * O * a.splits) return;
    const int o = (int)(wave % O);
    const int64_t rest = wave / O, r = rest % rows, z = rest / rows;
    const int64_t pb = z * a.p_chunk, pe = pb + a.p_chunk < P ? pb + a.p_chunk : P;
    const int64_t k = r * kLdsLanesOut + lane;
    float *row = a.partial + (z * O + o) * nt_max;
    const bool out = lane < kLdsLanesOut && k < nt_max;
    const int ntw = a.nt[o];
    if (r * kLdsLanesOut >= ntw) {
        if (out) row[k] = 0.f;
        return;
    }
    const int rowb = (int)a.NS * EB;
    const uint32_t *rp = rec_block(a.rec, 0, 0, P, O) + rec_dword(lane & 15, o, O);
    const uint32_t *bp = kBf ? rbf_block(a.rbf, 0, 0, P, O) + 8 * o + (lane & 7) : nullptr;
    using Q = typename std::conditional<kBf, uintx2, uintx4>::type;
    struct Batch {
        uint32_t rec[kFewAhead], bf[kFewAhead];
        Q x0[kFewAhead], x1[kFewAhead];
    };
    // records of the batch from panel ps (panels past the split repeat its last one)
    auto load_rec = [&](int64_t ps, Batch &b) {
#pragma unroll
        for (int i = 0; i < kFewAhead; ++i) {
            const int64_t p = ps + i < pe ? ps + i : pe - 1;
            b.rec[i] = rp[p * 16 * O];
            if constexpr (kBf) b.bf[i] = bp[p * 8 * O];
        }
    };
    auto load_coef = [&](int64_t ps, Batch &b) {
#pragma unroll
        for (int i = 0; i < kFewAhead; ++i) {
            const int64_t p = ps + i < pe ? ps + i : pe - 1;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<unsigned char *>(static_cast<const unsigned char *>(a.coef)) + (size_t)p * 2 * (size_t)rowb,
                0, 2 * rowb, 0x00020000);
            const int soff = (__builtin_amdgcn_readlane((int)b.rec[i], kRecN0) + (int)r * kLdsLanesOut) * EB;
            if constexpr (kBf) {
                b.x0[i] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane * EB, soff, 0);
                b.x1[i] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane * EB, soff + rowb, 0);
            } else {
                b.x0[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * EB, soff, 0);
                b.x1[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * EB, soff + rowb, 0);
            }
        }
    };
    float acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = 0.f;
    bool flushed = false;
    auto flush = [&](bool final_sums) {
        float sum = acc[0];
        if constexpr (NT == 4) {
            float s3 = acc[3];
            s3 = acc[2] + next_lane(s3);
            s3 = acc[1] + next_lane(s3);
            sum = acc[0] + next_lane(s3);
        }
        if (out) {
            const float v = (flushed ? row[k] : 0.f) + sum;
            row[k] = !final_sums || k < ntw ? v : 0.f;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = 0.f;
        flushed = true;
    };
    // the batch's first n panels (kFewAhead of them unless `part`)
    auto compute = [&](const Batch &b, auto part, int n) {
#pragma unroll
        for (int i = 0; i < kFewAhead; ++i) {
            if (!decltype(part)::value || i < n) {
                if constexpr (kBf) {
                    uint32_t Kw[8];
#pragma unroll
                    for (int f = 0; f < 8; ++f) Kw[f] = __builtin_amdgcn_readlane((int)b.bf[i], f);
                    float w[4];
#pragma unroll
                    for (int f = 0; f < 4; ++f)
                        w[f] = __int_as_float(__builtin_amdgcn_readlane((int)b.rec[i], kRecW + f));
                    float g = 0.f;
#pragma unroll
                    for (int h = 0; h < 8; h += 4) {
                        g = dot2_bf16(Kw[h], b.x0[i].x, g);
                        g = dot2_bf16(Kw[h + 1], b.x0[i].y, g);
                        g = dot2_bf16(Kw[h + 2], b.x1[i].x, g);
                        g = dot2_bf16(Kw[h + 3], b.x1[i].y, g);
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[t] = fmaf(w[t], g, acc[t]);
                } else {
                    few_panel(acc[0], __uint_as_float(b.rec[i]), b.x0[i], b.x1[i]);
                }
            }
        }
    };
    // chunks of kFewChunk panels (two batches at a time: coefficients of the next batch and records of the one
    // after it in flight)
    static_assert(kFewChunk % (2 * kFewAhead) == 0, "whole batches per chunk");
    Batch A, B;
    if (pb < pe) {
        load_rec(pb, A);
        load_coef(pb, A);
        load_rec(pb + kFewAhead, B);
    }
    for (int64_t pc = pb; pc < pe; pc += kFewChunk) {
        const int64_t pce = pc + kFewChunk < pe ? pc + kFewChunk : pe;
        int64_t p = pc;
        for (; p + 2 * kFewAhead <= pce; p += 2 * kFewAhead) {
            load_coef(p + kFewAhead, B);
            compute(A, std::false_type{}, 0);
            load_rec(p + 2 * kFewAhead, A);
            load_coef(p + 2 * kFewAhead, A);
            compute(B, std::false_type{}, 0);
            load_rec(p + 3 * kFewAhead, B);
        }
        if (p < pce) {  // the split's last panels
            load_coef(p + kFewAhead, B);
            compute(A, std::true_type{}, (int)(pce - p));
            compute(B, std::true_type{}, (int)(pce - p) - kFewAhead);
        }
        if (pce < pe) flush(false);
    }
    flush(true);
}

}  // namespace

hipError_t launch_gather_few(int coef_type, const PairRec *rec, const PairBf *rbf, const int32_t *nt, const void *coef,
                             int64_t P, int64_t O, int64_t NS, int64_t nt_max, int splits, float *partial,
                             hipStream_t stream) {
    if (O > kLdsWaves) return hipErrorInvalidValue;
    const int64_t p_chunk = (P + splits - 1) / splits, rows = (nt_max + kLdsLanesOut - 1) / kLdsLanesOut;
    const GatherArgs a{rec, rbf, nullptr, nt, coef, P, O, NS, nt_max, p_chunk, 0, 0, splits, partial, 0};
    const dim3 grid((unsigned)((rows * O * splits + 3) / 4));
    if (coef_type == 1) gather_few_kernel<float><<<grid, dim3(256), 0, stream>>>(a, rows);
    else gather_few_kernel<uint16_t><<<grid, dim3(256), 0, stream>>>(a, rows);
    return hipGetLastError();
}

}  // namespace fwh
