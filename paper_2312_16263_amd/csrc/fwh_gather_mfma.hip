// Forward gather with the channel combine on the matrix cores (gfx950).
//
// The surface sum of Sec. III C after the change of frame is, per observer o
// and sample k,
//   p'(o, k) = sum_p sum_jj w_jj(o,p) Y_p(o, n0(o,p) + k + jj),
//   Y_p(o, i) = sum_c K_c(o,p) coef_c(p, i),
// with fixed taps w, weights K and delay index n0 per (observer, panel) pair.
// For one panel and a tile of 16 observers, Y_p over a window of coefficient
// indices is a small dense product (window x 8 channels) x (8 channels x 16
// observers), which runs as matrix-core instructions, 16 indices x 16 observers
// per unit (v_mfma_f32_16x16x4f32, twice, in FP32 storage;
// v_mfma_f32_16x16x16bf16_1k with the weights split into bfloat16 high and low
// parts, once, in BF16 storage: products of bfloat16 values are exact in FP32,
// so both forms accumulate exact products in FP32).  Y goes through LDS; each
// observer then reads it at its own delay index and applies the four taps on the
// vector ALU.
//
// Block = kYWaves waves, observer tile t (16 observers), samples k0 ..
// k0 + 61 * rows - 1, panels [z*p_chunk, ...).  Per panel:
//   1. matrix units of the panel's window [lo + k0, lo + k0 + need), lo = min n0 over the tile,
//      `need` from the panel's own spread of n0, in blocks of 64 indices over the waves; the
//      16 x 16 results go to Y[observer][index] in LDS (one 16-byte write per lane); coefficients
//      and weights were loaded a panel ahead;
//   2. barrier;
//   3. taps: each wave for its observers of the tile, lane l of row m reads
//      Y[j][n0_j - lo + 61 m + l];
//   4. barrier (Y is rewritten by the next panel).
// Bound by instruction issue: FP32 matrix and vector instructions do not overlap (together 78 % of the
// slots; 240000 panels x 72 observers x 4096 frames 75 %, there with the data-return path 87 % busy), and in launches
// of few blocks by the chain of the four steps, about 1.2 us a panel.  The
// combine is done once per tile and index instead of once per observer and sample.  32768 panels x 360
// observers x 2048 frames: 7.8 ms (62 TFLOP/s of the sum's 24 flop per term) against 10.2 ms
// LDS-staged, BF16 storage 5.3 against 10.0; 240000 panels x 72 observers 32.4 against 36.8 ms.
#include <type_traits>

#include "fwh_internal.h"

namespace fwh {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) const uint32_t *const_u32_t;  // uniform loads stay scalar

constexpr int kYChunk = 256;  // panels summed in FP32 before adding into the partial signal
constexpr int kYBlk = 64;     // coefficient indices of one operand load

// Barrier for LDS data only: the waves' LDS accesses are complete and visible after it;
// outstanding global loads (the next panel's operands) stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Value of lane l+1 (wavefront shift by one lane; lane 63 receives 0).
__device__ __forceinline__ float next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130 /* wave_shl:1 */, 0xF, 0xF, true));
}

// Taps 1 and 3 of NSUB rows: a += w1 g', b += w3 g' with g' the next lane's g (a DPP source of the FMA:
// the shift costs no instruction).  A DPP read needs two wait states after a VALU write of its
// source: g comes from LDS, and the s_nop covers a register copy in between.
template <int NSUB>
__device__ __forceinline__ void taps_next(float (&acc)[NSUB][2], const float (&g)[NSUB], float w1, float w3) {
    if constexpr (NSUB == 4) {
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %8, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %8, %13 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %2, %9, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %3, %9, %13 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %4, %10, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %5, %10, %13 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %6, %11, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %7, %11, %13 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[1][0]), "+v"(acc[1][1]), "+v"(acc[2][0]), "+v"(acc[2][1]),
              "+v"(acc[3][0]), "+v"(acc[3][1])
            : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(w1), "v"(w3));
    } else {
#pragma unroll
        for (int m = 0; m < NSUB; ++m)
            asm("s_nop 1\n\t"
                "v_fmac_f32_dpp %0, %2, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_fmac_f32_dpp %1, %2, %4 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
                : "+v"(acc[m][0]), "+v"(acc[m][1])
                : "v"(g[m]), "v"(w1), "v"(w3));
    }
}

// Coefficients of kYBlk indices (four matrix units of 16) of both channel groups.  The loads go
// through a buffer descriptor of the panel's two rows (indices past them read zero), consecutive
// lanes reading consecutive memory; unit(t) turns unit t into the A operand by row swaps.  (Loading
// the operand lanes directly, channel lane / 16 of index lane % 16, made every 16 lanes touch 256
// bytes for 64 bytes of data and held the kernel at the texture addresser: 15.1 ms against 10.2 ms
// for the LDS-staged gather on the 32768-panel, 360-observer sphere.)
template <typename TS>
struct YBlock;
template <>
struct YBlock<float> {
    uintx4 x0, x1;  // lane l: the 4 channels of group 0, 1 at index l
    static __device__ __forceinline__ int lane_offset(int lane, int) { return lane * 16; }
    static __device__ __forceinline__ int lane_index(int lane) { return lane; }  // lowest index the lane loads
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff, int rowb) {
        x0 = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
        x1 = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff + rowb, 0);
    }
    // 4 x 4 transposes of (register = channel, row of 16 lanes = unit): then register t holds, in row
    // q, channel q of unit t
    static __device__ __forceinline__ void transpose(uintx4 &x) {
        const auto a = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
        const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
        const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
        x = uintx4{c[0], c[1], d[0], d[1]};
    }
    __device__ __forceinline__ void prepare() {
        transpose(x0);
        transpose(x1);
    }
    template <int T>
    __device__ __forceinline__ floatx4 unit(uintx2 b) const {
        floatx4 d = {0.f, 0.f, 0.f, 0.f};
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x0[T]), __uint_as_float(b.x), d, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x1[T]), __uint_as_float(b.y), d, 0, 0, 0);
    }
};
template <>
struct YBlock<uint16_t> {
    // x[h]: lane (row q, li): the 4 channels of group q & 1 at index 32 h + 16 (q >> 1) + li
    uintx2 x[2];
    static __device__ __forceinline__ int lane_offset(int lane, int rowb) {
        return (lane & 15) * 8 + (lane >> 5) * 128 + ((lane >> 4) & 1) * rowb;
    }
    static __device__ __forceinline__ int lane_index(int lane) { return (lane & 15) + (lane >> 5) * 16; }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff, int) {
        x[0] = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
        x[1] = __builtin_amdgcn_raw_buffer_load_b64(r, voff + 256, soff, 0);
    }
    __device__ __forceinline__ void prepare() {}
    // unit T: its two rows (groups 0 and 1) against the high parts of the weights, and again against
    // the low parts
    template <int T>
    __device__ __forceinline__ floatx4 unit(uintx2 b) const {
        const uintx2 v = x[T >> 1];
        const auto p = __builtin_amdgcn_permlane32_swap(v.x, v.x, false, false);
        const auto q = __builtin_amdgcn_permlane32_swap(v.y, v.y, false, false);
        const uintx2 a = {p[T & 1], q[T & 1]};
        const floatx4 d = {0.f, 0.f, 0.f, 0.f};
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(shortx4, a), __builtin_bit_cast(shortx4, b),
                                                         d, 0, 0, 0);
    }
};

template <int I, int N, typename F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<I + 1, N>(f);
    }
}

// One (tile, k block, split): NSUB rows of 61 samples have an output inside some window of the
// tile; FULL: all kYTile observers exist.
template <typename TS, int NSUB, bool FULL, int AHEAD>
__device__ __forceinline__ void gather_y_panels(const GatherArgs &a, int64_t t, int nobs, int64_t k0, int64_t z,
                                                float *__restrict__ Y) {
    constexpr bool kBf = std::is_same<TS, uint16_t>::value;
    constexpr int EB = 4 * (int)sizeof(TS);                 // bytes of one index of one channel group
    constexpr int OPW = kYTile / kYWaves;                   // observers per wave (at most)
    // operand blocks per wave that every panel needs; with a single one (NSUB = 1) every wave loads it, and
    // any further one, and does one of its four units
    constexpr bool kShare = NSUB == 1;
    static_assert(kYWaves == 4, "a block of 64 indices is four units");
    constexpr int MW = (NSUB + kYWaves - 1) / kYWaves;
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t P = a.P, O = a.O, nt_max = a.nt_max, tbase = t * kYTile;
    const int64_t pb = z * a.p_chunk, pe = pb + a.p_chunk < P ? pb + a.p_chunk : P;
    const int YR = a.NW;
    const int rowb = (int)a.NS * EB;
    // lane li of each row of 16 lanes is observer slot li: its column of the matrix product (slots past
    // the last observer repeat it), its row of Y; the wave's own observers are slots own0 + j
    const int slot = FULL ? li : (li < nobs ? li : nobs - 1);
    const int per_wave = FULL ? OPW : (nobs + kYWaves - 1) / kYWaves;
    const int own0 = wv * per_wave;
    const int nown = FULL ? OPW : (nobs - own0 < per_wave ? (nobs > own0 ? nobs - own0 : 0) : per_wave);

    float acc[OPW][NSUB][2];
#pragma unroll
    for (int j = 0; j < OPW; ++j)
#pragma unroll
        for (int m = 0; m < NSUB; ++m) acc[j][m][0] = acc[j][m][1] = 0.f;

    // window start (n0 - d16) and width of panel p, lane q: panel ps + q
    int wlo = 0, wwd = 0;
    auto load_win = [&](int64_t ps) {
        const int64_t q = ps + lane < pe ? ps + lane : pe - 1;
        const uint32_t *blk = rec_block(a.rec, t, q, P, nobs);
        wlo = (int)(blk[kRecN0 * nobs] - blk[kRecD16 * nobs]);
        wwd = (int)blk[kRecW16 * nobs];
    };
    const int voff = YBlock<TS>::lane_offset(lane, rowb);
    const uint32_t *kp = (kBf ? rbf_block(a.rbf, t, pb, P, nobs) : rec_block(a.rec, t, pb, P, nobs)) + 8 * slot + 2 * lq;
    // Taps and window offsets of the wave's own observers, wave-uniform.  AHEAD = 1: scalar loads at the
    // panel's start.  Else (few waves to hide their latency behind) one vector load with the operands,
    // lane 4 j + q: w_q of own observer j, lane 4 OPW + j: its offset, moved to scalars when used.
    struct Taps {
        float w[OPW][4];
        int d[OPW];
    };
    static_assert(5 * OPW <= 64, "taps of a wave in one load");
    const int tap_j = lane < 4 * OPW ? lane >> 2 : (lane < 5 * OPW ? lane - 4 * OPW : 0);
    const int tap_s = own0 + tap_j < nobs ? own0 + tap_j : nobs - 1;
    const uint32_t *tp = rec_block(a.rec, t, pb, P, nobs) +
                         (lane < 4 * OPW ? kRecW * nobs + 4 * tap_s + (lane & 3) : kRecD16 * nobs + tap_s);
    auto load_taps = [&](int64_t p, Taps &x) {
        const_u32_t blk = (const_u32_t)rec_block(a.rec, t, p, P, nobs);
#pragma unroll
        for (int j = 0; j < OPW; ++j)
            if (FULL || j < nown) {
#pragma unroll
                for (int q = 0; q < 4; ++q) x.w[j][q] = __uint_as_float(blk[kRecW * nobs + 4 * (own0 + j) + q]);
                x.d[j] = (int)blk[kRecD16 * nobs + own0 + j];
            }
    };
    auto unpack_taps = [&](uint32_t v, Taps &x) {
#pragma unroll
        for (int j = 0; j < OPW; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) x.w[j][q] = __int_as_float(__builtin_amdgcn_readlane((int)v, 4 * j + q));
            x.d[j] = __builtin_amdgcn_readlane((int)v, 4 * OPW + j);
        }
    };
    // operands of one panel: the blocks every panel needs, and one block past them per wave, in turn
    struct Operands {
        YBlock<TS> A[MW], T;
        uintx2 Bk;
        uint32_t taps;  // AHEAD > 1
        int need, soff, tb;
        __amdgpu_buffer_rsrc_t rsrc;
    };
    // panel p (its window in lane p - pb & 63 of wlo, wwd)
    auto load_panel = [&](int64_t p, Operands &X) {
        const int q = (int)((p - pb) & 63);
        if (q == 0) load_win(p);
        const int lo = __builtin_amdgcn_readlane(wlo, q), wd = __builtin_amdgcn_readlane(wwd, q);
        X.need = wd + kLdsLanesOut * NSUB + kLdsHalo;
        X.soff = (lo + (int)k0) * EB;
        X.rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(static_cast<const unsigned char *>(a.coef)) + (size_t)p * 2 * (size_t)rowb, 0,
            2 * rowb, 0x00020000);
        X.Bk = *reinterpret_cast<const uintx2 *>(kp);
        kp += nobs * (kBf ? 8 : 16);
        if constexpr (AHEAD > 1) {
            X.taps = *tp;
            tp += nobs * 16;
        }
#pragma unroll
        for (int i = 0; i < MW; ++i)
            if (kShare || (i + 1) * kYWaves <= NSUB || wv + i * kYWaves < NSUB)
                X.A[i].load(X.rsrc, voff, X.soff + (kShare ? 0 : wv + i * kYWaves) * kYBlk * EB, rowb);
        X.tb = kShare ? 1 : NSUB + ((wv + (int)p) & (kYWaves - 1));
        if (YBlock<TS>::lane_index(lane) < X.need - X.tb * kYBlk)
            X.T.load(X.rsrc, voff, X.soff + X.tb * kYBlk * EB, rowb);
    };
    // the units of block b (indices 64 b ..) into Y, those below `need` if `part`
    float *const ybase = Y + li * YR + 4 * lq;
    auto units = [&](YBlock<TS> &B, const Operands &X, int b, auto part) {
        B.prepare();
        unroll<0, 4>([&](auto tc) {
            constexpr int U = decltype(tc)::value;
            if ((!kShare || U == wv) && (!decltype(part)::value || b * kYBlk + U * 16 < X.need))
                *reinterpret_cast<floatx4 *>(ybase + b * kYBlk + U * 16) = B.template unit<U>(X.Bk);
        });
    };
    auto multiply = [&](Operands &X) {
#pragma unroll
        for (int i = 0; i < MW; ++i)
            if (kShare || (i + 1) * kYWaves <= NSUB || wv + i * kYWaves < NSUB)
                units(X.A[i], X, kShare ? 0 : wv + i * kYWaves, std::false_type{});
        if (X.tb * kYBlk < X.need) units(X.T, X, X.tb, std::true_type{});
        // wide windows: blocks beyond those loaded ahead
        for (int b = kShare ? 2 : NSUB + kYWaves + wv; b * kYBlk < X.need; b += kShare ? 1 : kYWaves) {
            YBlock<TS> B;
            B.load(X.rsrc, voff, X.soff + b * kYBlk * EB, rowb);
            units(B, X, b, std::true_type{});
        }
    };
    const float *const yown = Y + own0 * YR + lane;
    auto flush = [&](bool add, bool last) {
#pragma unroll
        for (int j = 0; j < OPW; ++j) {
            if (FULL || j < nown) {
                const int64_t o = tbase + own0 + j;
                float *row = a.partial + (z * O + o) * nt_max;
                const int ntl = last ? a.nt[o] : 0;
#pragma unroll
                for (int m = 0; m < NSUB; ++m) {
                    const float v = acc[j][m][0] + next_lane(next_lane(acc[j][m][1]));
                    const int64_t k = k0 + m * kLdsLanesOut + lane;
                    if (lane < kLdsLanesOut && k < nt_max) {
                        const float s = (add ? row[k] : 0.f) + v;
                        row[k] = !last || k < ntl ? s : 0.f;
                    }
                    acc[j][m][0] = acc[j][m][1] = 0.f;
                }
            }
        }
    };

    int cnt = 0;
    bool flushed = false;
    Taps now;
    Operands X[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (pb + i < pe) load_panel(pb + i, X[i]);
    for (int64_t ps = pb; ps < pe; ps += AHEAD) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int64_t p = ps + i;
            if (p >= pe) break;
            if constexpr (AHEAD > 1) unpack_taps(X[i].taps, now);
            else load_taps(p, now);
            lds_barrier();  // every wave has read the previous panel's Y (and, first time round, another item's)
            multiply(X[i]);
            if (p + AHEAD < pe) load_panel(p + AHEAD, X[i]);
            lds_barrier();
#pragma unroll
            for (int j = 0; j < OPW; ++j) {
                if (FULL || j < nown) {
                    const float *y = yown + j * YR + now.d[j];
                    float g[NSUB];
#pragma unroll
                    for (int m = 0; m < NSUB; ++m) g[m] = y[m * kLdsLanesOut];
#pragma unroll
                    for (int m = 0; m < NSUB; ++m) {
                        acc[j][m][0] = fmaf(now.w[j][0], g[m], acc[j][m][0]);
                        acc[j][m][1] = fmaf(now.w[j][2], g[m], acc[j][m][1]);
                    }
                    taps_next<NSUB>(acc[j], g, now.w[j][1], now.w[j][3]);
                }
            }
            if (++cnt == kYChunk) {
                flush(flushed, false);
                flushed = true;
                cnt = 0;
            }
        }
    }
    flush(flushed, true);
}

template <typename TS, int AHEAD>
__device__ __forceinline__ void gather_y_body(const GatherArgs &a, int64_t t, int64_t kb, int64_t z,
                                              float *__restrict__ Y) {
    const int64_t tbase = t * kYTile, k0 = kb * kLdsLanesOut * a.rows;
    const int nobs = (int)(a.O - tbase < kYTile ? a.O - tbase : kYTile);
    int nt_tile = 0;
    for (int j = 0; j < nobs; ++j) {
        const int n = a.nt[tbase + j];
        nt_tile = n > nt_tile ? n : nt_tile;
    }
    int nsub = (int)((nt_tile - k0 + kLdsLanesOut - 1) / kLdsLanesOut);
    nsub = __builtin_amdgcn_readfirstlane(nsub < 0 ? 0 : (nsub > a.rows ? a.rows : nsub));
    // rows past the tile's windows, of the block's `rows` rows, are zero
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int m = nsub; m < a.rows; ++m)
        for (int j = wv; j < nobs; j += kYWaves) {
            const int64_t k = k0 + m * kLdsLanesOut + lane;
            if (lane < kLdsLanesOut && k < a.nt_max) a.partial[(z * a.O + tbase + j) * a.nt_max + k] = 0.f;
        }
    if (nobs == kYTile) {
        switch (nsub) {
            case 0: break;
            case 1: gather_y_panels<TS, 1, true, AHEAD>(a, t, nobs, k0, z, Y); break;
            case 2: gather_y_panels<TS, 2, true, AHEAD>(a, t, nobs, k0, z, Y); break;
            case 3: gather_y_panels<TS, 3, true, AHEAD>(a, t, nobs, k0, z, Y); break;
            default: gather_y_panels<TS, 4, true, AHEAD>(a, t, nobs, k0, z, Y); break;
        }
    } else {
        switch (nsub) {
            case 0: break;
            case 1: gather_y_panels<TS, 1, false, AHEAD>(a, t, nobs, k0, z, Y); break;
            case 2: gather_y_panels<TS, 2, false, AHEAD>(a, t, nobs, k0, z, Y); break;
            case 3: gather_y_panels<TS, 3, false, AHEAD>(a, t, nobs, k0, z, Y); break;
            default: gather_y_panels<TS, 4, false, AHEAD>(a, t, nobs, k0, z, Y); break;
        }
    }
}

// Waves per SIMD the registers are held to, for operands loaded AHEAD panels ahead.
template <typename TS, int AHEAD>
constexpr int y_waves_per_eu() {
    constexpr bool f32 = std::is_same<TS, float>::value;
    return AHEAD == 1 ? (f32 ? 5 : 6) : AHEAD == 2 ? (f32 ? 4 : 5) : (f32 ? 3 : 4);
}
template <typename TS, int AHEAD>
__global__ __launch_bounds__(kYWaves * 64) __attribute__((amdgpu_waves_per_eu(y_waves_per_eu<TS, AHEAD>())))
void gather_y_kernel(GatherArgs a, int64_t tiles, int64_t kblocks) {
    extern __shared__ __align__(16) float ysm[];
    // 1-D grid, block order (tile fastest, k block, split) regrouped per XCD
    const int64_t L = xcd_block(blockIdx.x, gridDim.x);
    const int64_t t = L % tiles, rest = L / tiles;
    gather_y_body<TS, AHEAD>(a, t, rest % kblocks, rest / kblocks, ysm);
}

// Persistent batched form: blocks pull work items (case, tile, k block, split) in
// list order (longest first) through an atomic counter until the list is
// exhausted; each item runs the body above on its case's arguments.  The Y tile
// is reused from item to item (the loop-top barrier orders the last reads of one
// item before the first writes of the next).
template <typename TS, int AHEAD>
__global__ __launch_bounds__(kYWaves * 64) __attribute__((amdgpu_waves_per_eu(y_waves_per_eu<TS, AHEAD>())))
void gather_y_persistent(const BatchCase *__restrict__ cases, const int4 *__restrict__ items, int n_items,
                         int *__restrict__ counter) {
    extern __shared__ __align__(16) float ysm[];
    __shared__ int cur;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) cur = atomicAdd(counter, 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(cur);
        if (it >= n_items) break;
        const int4 w = items[it];
        const int c = __builtin_amdgcn_readfirstlane(w.x);
        gather_y_body<TS, AHEAD>(cases[c].gat, __builtin_amdgcn_readfirstlane(w.y), __builtin_amdgcn_readfirstlane(w.z),
                                 __builtin_amdgcn_readfirstlane(w.w), ysm);
    }
}

constexpr int kYAheadFull = 1, kYAheadFew = 4, kYAheadBatch = 2;

}  // namespace

template <typename TS, int AHEAD>
static int y_blocks_per_cu(size_t shmem) {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, reinterpret_cast<const void *>(&gather_y_kernel<TS, AHEAD>), kYWaves * 64, shmem);
    return e == hipSuccess && n > 0 ? n : 0;
}

int gather_mfma_blocks_per_cu(int coef_type, int w16, bool few) {
    const size_t shmem = gather_mfma_shmem(w16);
    if (shmem > kYShmemMax) return 0;
    if (few)
        return coef_type == 1 ? y_blocks_per_cu<float, kYAheadFew>(shmem) : y_blocks_per_cu<uint16_t, kYAheadFew>(shmem);
    return coef_type == 1 ? y_blocks_per_cu<float, kYAheadFull>(shmem) : y_blocks_per_cu<uint16_t, kYAheadFull>(shmem);
}

hipError_t launch_gather_mfma(int coef_type, const PairRec *rec_op, const PairBf *rbf, const int32_t *nt,
                              const void *coef, int64_t P, int64_t O, int64_t NS, int64_t nt_max, int splits, int w16,
                              int64_t few_blocks, float *partial, hipStream_t stream) {
    const int64_t p_chunk = (P + splits - 1) / splits, tiles = (O + kYTile - 1) / kYTile;
    // rows of 61 samples per block: 4, fewer where all blocks still fit the device at once (a short launch
    // lasts as long as one block's chain of panels, and a panel's product and taps are shorter with fewer rows)
    int rows = kLdsSub;
    auto blocks = [&](int r) { return tiles * ((nt_max + kLdsLanesOut * r - 1) / (kLdsLanesOut * r)) * splits; };
    while (rows > 1 && blocks(rows / 2) <= few_blocks) rows /= 2;
    const int64_t kblocks = (nt_max + kLdsLanesOut * rows - 1) / (kLdsLanesOut * rows);
    const GatherArgs a{rec_op, rbf, nullptr, nt, coef, P, O, NS, nt_max, p_chunk, gather_mfma_y_row(w16), 0, splits,
                       partial, rows};
    const dim3 n1((unsigned)(tiles * kblocks * splits)), blk(kYWaves * 64);
    const size_t shmem = gather_mfma_shmem(w16);
    const bool few = blocks(rows) <= few_blocks;
    if (coef_type == 1) {
        if (few) gather_y_kernel<float, kYAheadFew><<<n1, blk, shmem, stream>>>(a, tiles, kblocks);
        else gather_y_kernel<float, kYAheadFull><<<n1, blk, shmem, stream>>>(a, tiles, kblocks);
    } else {
        if (few) gather_y_kernel<uint16_t, kYAheadFew><<<n1, blk, shmem, stream>>>(a, tiles, kblocks);
        else gather_y_kernel<uint16_t, kYAheadFull><<<n1, blk, shmem, stream>>>(a, tiles, kblocks);
    }
    return hipGetLastError();
}

hipError_t launch_gather_mfma_persistent(int coef_type, const BatchCase *cases, const int4 *items, int n_items,
                                         int *counter, int grid, size_t shmem, hipStream_t stream) {
    const dim3 g((unsigned)grid), blk(kYWaves * 64);
    if (coef_type == 1)
        gather_y_persistent<float, kYAheadBatch><<<g, blk, shmem, stream>>>(cases, items, n_items, counter);
    else gather_y_persistent<uint16_t, kYAheadBatch><<<g, blk, shmem, stream>>>(cases, items, n_items, counter);
    return hipGetLastError();
}

}  // namespace fwh
