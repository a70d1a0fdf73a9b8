// Transposed gather of the adjoint (gfx950, FP32/BF16 forms): the coefficient adjoints
//   cbar_c(p, i) = sum_o K_c(o, p) sum_j w_j(o, p) gbar(o, i - n0(o, p) - j),
// a contraction over observers for every (panel, index): it runs on the matrix cores.  Bound by
// matrix and vector issue (76 % of the slots) and by the data return of 16-byte loads at dword
// alignment (82 % busy).  Two forms, the same sums bit for bit: products of one observer each (4x4x1), and of
// four (16x16x4) for short records and small surfaces.  32768 panels x 360 observers x 2048 frames: 8.25 ms
// against 10.1 in the second form; 240000 panels x 72 observers x 4096 frames: 24.8 against 31.4.
#include <type_traits>

#include "fwh_internal.h"

namespace fwh {
namespace {

// Zero-padded copy of dJ/dp': gpad[o][k + padlo] = gbar[o][k] for 0 <= k < N_t(o), 0 elsewhere.
__device__ __forceinline__ void pad_grad_body(const PadArgs &a, int64_t i) {
    if (i >= a.O * a.LR) return;
    const int64_t o = i / a.LR;
    const int64_t k = i - o * a.LR - a.padlo;
    a.gpad[i] = (k >= 0 && k < a.nt[o]) ? a.gbar[o * a.nt_max + k] : 0.f;
}

__global__ __launch_bounds__(256) void pad_grad_kernel(PadArgs a) {
    pad_grad_body(a, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

__global__ __launch_bounds__(256) void pad_grad_batched(const BatchCase *__restrict__ cases,
                                                        const int64_t *__restrict__ start, int n) {
    const int c = find_case(start, n, blockIdx.x);
    pad_grad_body(cases[c].pad, ((int64_t)blockIdx.x - start[c]) * 256 + threadIdx.x);
}

// Transposed gather on the matrix cores.  For panel p and coefficient index i,
//   cbar_c(p, i) = sum_o K_c(o, p) H(o, i),  H(o, i) = sum_j w_j(o, p) gbar(o, i - n0(o, p) - j),
// an outer product of 4 channels and 64 indices per observer and v_mfma_f32_4x4x1f32 (16 independent
// 4 x 4 products): B = H (lane l: one index), A = the 4 weights of a channel group, taken from block s
// of a register that holds the weights of 16 observers (lane 4 s + n: K_n of slot s; the
// instruction's CBSZ/ABID broadcast), D (lane l, register r) accumulates channel r at lane l's index
// over all observers.  Every one of its multiply-adds is used, where a 16x16x4 product over 4
// observers had 8 of its 16 columns empty.
//
// Lane l holds the indices 4 l + t - 4 (t = 0..3) of its wave's block of kAdjIdx: one 16-byte load of
// gbar at the observer's shift, the 3 positions below from lane l - 1 (a wavefront shift; lane 0's
// products are not stored), 16 FMA with the taps from scalar registers (one observer at a time for
// the whole wave), 8 products.
//
// A wave owns panel p and kAdjMW blocks.  Waves go in tiles of kAdjPT panels x all index blocks,
// panels fastest: the 4 waves of a block (and neighbouring blocks on one XCD) read the same
// observers' gbar windows a few samples apart and adjacent pair tables, and a tile's tables stay in
// L2 for all its index blocks.
typedef float floatx4_t __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) AdjF4 {
    float x, y, z, w;
};
typedef __attribute__((address_space(4))) const uint32_t *const_u32_t;  // uniform loads stay scalar

// lane l receives lane l - 1's x (lane 0: 0)
__device__ __forceinline__ float from_prev_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138 /* wave_shr:1 */, 0xF, 0xF, true));
}

constexpr int kAdjG = 2;  // observers per group of loads

// One group of kAdjG observers: taps and gbar windows.
template <int NB>
struct AdjGroup {
    float w[kAdjG][4];
    AdjF4 x[kAdjG][NB];
    bool on;  // some observer of the group reaches the wave's indices
};

template <int NB>  // index blocks of the wave (1 or 2)
__device__ __forceinline__ void adj_gather_body(const AdjArgs &a, int64_t p, int64_t ib) {
    const int64_t P = a.P, O = a.O, LR = a.LR;
    const int lane = threadIdx.x & 63;
    const bool check = ib < a.edge_lo || ib + kAdjIdx * NB - 1 > a.edge_hi;  // wave-uniform
    floatx4_t acc[NB][4][2];
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[u][t][0] = acc[u][t][1] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    const int64_t tiles = (O + kYTile - 1) / kYTile;
    const float *gw = a.gpad + a.padlo + ib - 4;
    // loads of the observers t*16 + s0 .. + kAdjG - 1 (those that exist)
    auto load = [&](int64_t t, int s0, AdjGroup<NB> &b) {
        const int64_t o = t * kYTile + s0;
        b.on = o < O;
        if (!b.on) return;
        const int c = rec_tile_obs(t, O);
        const_u32_t blk = (const_u32_t)rec_block(a.rec, t, p, P, c);
        int n0[kAdjG];
#pragma unroll
        for (int j = 0; j < kAdjG; ++j) n0[j] = (int)blk[kRecN0 * c + min(s0 + j, c - 1)];
        if (check) {
            // observer o + j adds to the indices [n0, n0 + N_t + 2] only
            bool on = false;
#pragma unroll
            for (int j = 0; j < kAdjG; ++j)
                on |= n0[j] < (int)ib + kAdjIdx * NB &&
                      n0[j] + ((const_u32_t)a.nt)[min(o + j, O - 1)] + 2 >= (unsigned)ib;
            b.on = on;
            if (!on) return;
        }
#pragma unroll
        for (int j = 0; j < kAdjG; ++j) {
            const int s = min(s0 + j, c - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) b.w[j][q] = __uint_as_float(blk[kRecW * c + 4 * s + q]);
            const float *g = gw + (t * kYTile + s) * LR - n0[j];
#pragma unroll
            for (int u = 0; u < NB; ++u) b.x[j][u] = *reinterpret_cast<const AdjF4 *>(g + u * kAdjIdx + 4 * lane);
        }
    };
    // weights of a tile: lane 4 s + n holds K_n (group 0) and K_{4+n} (group 1) of slot s, 0 past the
    // last observer
    auto load_k = [&](int64_t t, float &k0, float &k1) {
        k0 = k1 = 0.f;
        const int c = rec_tile_obs(t, O);
        if ((lane >> 2) < c) {
            const uint2 k = *reinterpret_cast<const uint2 *>(rec_block(a.rec, t, p, P, c) + 2 * lane);
            k0 = __uint_as_float(k.x);
            k1 = __uint_as_float(k.y);
        }
    };
    auto compute = [&](auto sc, const AdjGroup<NB> &b, float k0, float k1) {
        constexpr int S0 = decltype(sc)::value;
        if (!b.on) return;
        auto one = [&](auto jc) {
            constexpr int J = decltype(jc)::value;
            const float w0 = b.w[J][0], w1 = b.w[J][1], w2 = b.w[J][2], w3 = b.w[J][3];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const AdjF4 x = b.x[J][u];
                const float m1 = from_prev_lane(x.w), m2 = from_prev_lane(x.z), m3 = from_prev_lane(x.y);
                float h[4];
                h[0] = fmaf(w3, m3, fmaf(w2, m2, fmaf(w1, m1, w0 * x.x)));
                h[1] = fmaf(w3, m2, fmaf(w2, m1, fmaf(w1, x.x, w0 * x.y)));
                h[2] = fmaf(w3, m1, fmaf(w2, x.x, fmaf(w1, x.y, w0 * x.z)));
                h[3] = fmaf(w3, x.x, fmaf(w2, x.y, fmaf(w1, x.z, w0 * x.w)));
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    acc[u][t][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(k0, h[t], acc[u][t][0], 4, S0 + J, 0);
                    acc[u][t][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(k1, h[t], acc[u][t][1], 4, S0 + J, 0);
                }
            }
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
    };
    static_assert(kAdjG == 2, "compute handles two observers");
    AdjGroup<NB> A, B;
    float k0, k1, kn0, kn1;
    load_k(0, k0, k1);
    load(0, 0, A);
    // groups alternate between A and B; the next group's loads (and the next tile's weights) are in
    // flight while one is computed
#pragma unroll 1
    for (int64_t t = 0; t < tiles; ++t) {
        kn0 = kn1 = 0.f;
        if (t + 1 < tiles) load_k(t + 1, kn0, kn1);
#define FWH_ADJ_STEP(S, CUR, NXT)                                      \
    if ((S) + kAdjG < kYTile) load(t, (S) + kAdjG, NXT);               \
    else load(t + 1, 0, NXT);                                          \
    compute(std::integral_constant<int, S>{}, CUR, k0, k1);
        FWH_ADJ_STEP(0, A, B)
        FWH_ADJ_STEP(2, B, A)
        FWH_ADJ_STEP(4, A, B)
        FWH_ADJ_STEP(6, B, A)
        FWH_ADJ_STEP(8, A, B)
        FWH_ADJ_STEP(10, B, A)
        FWH_ADJ_STEP(12, A, B)
        FWH_ADJ_STEP(14, B, A)
#undef FWH_ADJ_STEP
        k0 = kn0;
        k1 = kn1;
    }
    // lane l > 0: indices e .. e + 3, e = ib + 252 u + 4 (l - 1), of all 8 channels; the indices past the
    // record (row padding) are written too where they lie inside the row
    const int64_t NS = a.NS;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int64_t e = ib + u * kAdjIdx + 4 * (lane - 1);
        if (lane > 0 && e < NS) {
#pragma unroll
            for (int ch = 0; ch < 8; ++ch)
                *reinterpret_cast<float4 *>(a.cbar + ((int64_t)ch * P + p) * NS + e) =
                    make_float4(acc[u][0][ch >> 2][ch & 3], acc[u][1][ch >> 2][ch & 3], acc[u][2][ch >> 2][ch & 3],
                                acc[u][3][ch >> 2][ch & 3]);
        }
    }
}

__device__ __forceinline__ void adj_gather_wave(const AdjArgs &a, int64_t wave_id) {
    const int64_t P = a.P, nib = a.nib;
    if (wave_id >= P * nib) return;
    // tile of kAdjPT panels (the last one narrower) x nib index blocks, panels fastest
    const int64_t tile = wave_id / (kAdjPT * nib);
    const int64_t r = wave_id - tile * (kAdjPT * nib);
    const int64_t tw = min<int64_t>(kAdjPT, P - tile * kAdjPT);
    const int64_t bi = r / tw;
    const int64_t p = tile * kAdjPT + (r - bi * tw);
    const int64_t ib = bi * (kAdjIdx * kAdjMW);
    if (ib + kAdjIdx < a.N + 2) adj_gather_body<2>(a, p, ib);
    else adj_gather_body<1>(a, p, ib);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void adj_gather_mfma_kernel(AdjArgs a) {
    // consecutive blocks (neighbouring index blocks and panels) regrouped per XCD
    adj_gather_wave(a, xcd_block(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// The form for short records and small surfaces: one v_mfma_f32_16x16x4f32 per 4 observers and 16
// indices, A[m][k] = H(observer o + k, index m), B[k][n] = K_n(o + k, p) (zero for n >= 8), D[m][n] = the
// contribution of channel n at index m.  Lane (q, s) of the wave (q = lane / 16, s = lane % 16) owns
// observer o + q and the 4 indices ib + 4 s + t (t = 0..3): it loads gbar at the 4 shifted positions with
// one 16-byte load and takes the 3 positions below from lane s - 1 of its row (a row shift; lane s = 0
// from lane 15's load of the previous block of 64, by a row rotation, and by a load of its own for the first
// block).  Product t takes rows m = s as index ib + 4 m + t, so lane (q', n) of its output holds channel
// n at indices ib + 16 q' + 4 r + t (r = 0..3).  A row fetches its pair's tables with one dword per lane
// (lane s: field s) and takes the taps and n0 from lanes 8 .. 11 and 13 by row broadcasts.  Half of a
// product's columns are empty, but four observers advance at once and an index block is 64 wide.
__device__ __forceinline__ float adj_row_rot(float x) {
    // lane s of each row of 16 receives lane s - 1 (mod 16); every lane has a source
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x121 /* row_ror:1 */, 0xF, 0xF, false));
}
__device__ __forceinline__ float adj_row_prev(float x, float old) {
    // lane s of each row of 16 receives lane s - 1's x; lane 0 keeps `old`
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x111 /* row_shr:1 */,
                                                      0xF, 0xF, false));
}
template <int LANE>
__device__ __forceinline__ float adj_row_bcast(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + LANE /* row_newbcast */, 0xF, 0xF, false));
}

// One group of 4 observers (one per row of the wave): the rows' pair tables and gbar windows.
template <int NB>
struct Adj16Group {
    float rv;     // field s of the pair (o + q, p)
    AdjF4 x[NB];  // gbar at e .. e + 3, e = ib + 64 u + 4 s - n0
    AdjF4 pv;     // gbar at e - 4 .. e - 1 of block u = 0 (lane s = 0 only)
};

template <int NB>  // index blocks of the wave (1 .. kAdj16MW)
__device__ __forceinline__ void adj_gather16_body(const AdjArgs &a, int64_t p, int64_t ib) {
    const int64_t P = a.P, O = a.O, NS = a.NS, LR = a.LR;
    const int lane = threadIdx.x & 63, q = lane >> 4, s = lane & 15;
    const float *g = a.gpad + a.padlo + ib + 4 * s;
    floatx4_t acc[NB][4];
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[u][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    // Loads run ahead of the arithmetic: while group o is computed, the gbar windows of group o + 4 and the
    // pair tables of group o + 8 are in flight.  Observers past O are clamped to O - 1 for the loads and get K = 0.
    // field s of slot j in a block of c observers (rec_dword): fj j + fc c + f0; lanes 12 .. 15 all load n0
    const int fj = s < kRecW ? 8 : s < kRecN0w ? 4 : 1, fc = s < kRecW ? 0 : s < kRecN0w ? kRecW : kRecN0,
              f0 = s < kRecW ? 2 * (s & 3) + (s >> 2) : s < kRecN0w ? s - kRecW : 0;
    auto tile_rec = [&](int64_t t) {
        const int c = rec_tile_obs(t, O);
        return rec_block(a.rec, t, p, P, c) + (fc * c + f0);
    };
    // tables of group g of a tile (rt its tile_rec, slots past `lim` repeat it)
    auto load_rec = [&](const uint32_t *rt, int g, int lim) {
        return __uint_as_float(rt[fj * min(4 * g + q, lim)]);
    };
    auto load_x = [&](int64_t o, Adj16Group<NB> &b) {
        const int n0 = __float_as_int(adj_row_bcast<kRecN0>(b.rv));
        const float *go = g + min(o + q, O - 1) * LR - n0;
#pragma unroll
        for (int u = 0; u < NB; ++u) b.x[u] = *reinterpret_cast<const AdjF4 *>(go + 64 * u);
        // only lane 0 of each row uses pv; every lane loads it (in bounds: the row's lead pad holds
        // N + 4 floats and n0 <= N), so the register is not merged with its old value
        b.pv = *reinterpret_cast<const AdjF4 *>(go - 4);
    };
    // Waves near either end of the index range (check): 64-index blocks u_lo .. u_hi, those that some observer of
    // the group reaches (observer o + q adds to the indices [n0, n0 + N_t + 2] only, N_t bounded by the longest
    // window); the others would get exact zeros.
    const bool check = ib < a.edge_lo || ib + 64 * NB - 1 > a.edge_hi;  // wave-uniform
    auto compute = [&](int64_t o, const Adj16Group<NB> &b) {
        const float kb = (o + q < O && s < 8) ? b.rv : 0.f;
        const float w0 = adj_row_bcast<kRecW>(b.rv), w1 = adj_row_bcast<kRecW + 1>(b.rv),
                    w2 = adj_row_bcast<kRecW + 2>(b.rv), w3 = adj_row_bcast<kRecW + 3>(b.rv);
        int u_lo = 0, u_hi = NB - 1;
        if (check) {
            int n0lo = __builtin_amdgcn_readlane(__float_as_int(b.rv), kRecN0), n0hi = n0lo;
#pragma unroll
            for (int r4 = 1; r4 < 4; ++r4) {
                const int v = __builtin_amdgcn_readlane(__float_as_int(b.rv), 16 * r4 + kRecN0);
                n0lo = min(n0lo, v);
                n0hi = max(n0hi, v);
            }
            const int ibi = (int)ib;
            u_lo = max(0, (n0lo - ibi) >> 6);
            u_hi = min(NB - 1, (n0hi + (int)a.nt_max + 2 - ibi) >> 6);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if (u >= u_lo && u <= u_hi) {
                const AdjF4 xv = b.x[u];
                // lane 0's values below e: its own load (u = 0) or lane 15's of block u - 1
                const AdjF4 &xp = b.x[u > 0 ? u - 1 : 0];
                const float o1 = u == 0 ? b.pv.w : adj_row_rot(xp.w);
                const float o2 = u == 0 ? b.pv.z : adj_row_rot(xp.z);
                const float o3 = u == 0 ? b.pv.y : adj_row_rot(xp.y);
                const float m1 = adj_row_prev(xv.w, o1);  // gbar at e - 1
                const float m2 = adj_row_prev(xv.z, o2);  // e - 2
                const float m3 = adj_row_prev(xv.y, o3);  // e - 3
                const float h0 = fmaf(w3, m3, fmaf(w2, m2, fmaf(w1, m1, w0 * xv.x)));
                const float h1 = fmaf(w3, m2, fmaf(w2, m1, fmaf(w1, xv.x, w0 * xv.y)));
                const float h2 = fmaf(w3, m1, fmaf(w2, xv.x, fmaf(w1, xv.y, w0 * xv.z)));
                const float h3 = fmaf(w3, xv.x, fmaf(w2, xv.y, fmaf(w1, xv.z, w0 * xv.w)));
                acc[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(h0, kb, acc[u][0], 0, 0, 0);
                acc[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(h1, kb, acc[u][1], 0, 0, 0);
                acc[u][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(h2, kb, acc[u][2], 0, 0, 0);
                acc[u][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(h3, kb, acc[u][3], 0, 0, 0);
            }
        }
    };
    // before step(o, ..): cur holds the tables and windows of group o, nxt the tables of group o + 4.  Loads
    // complete in issue order, so the tables of o + 8 go first: the next step waits for them without waiting
    // for the windows issued after them.
    auto step = [&](int64_t o, Adj16Group<NB> &cur, Adj16Group<NB> &nxt, const uint32_t *rt, int g, int lim) {
        const float rnew = load_rec(rt, g, lim);
        load_x(o + 4, nxt);
        compute(o, cur);
        cur.rv = rnew;
    };
    const int64_t tiles = (O + kYTile - 1) / kYTile;
    const uint32_t *rt = tile_rec(0);
    int lim = rec_tile_obs(0, O) - 1;
    Adj16Group<NB> A, B;
    A.pv = B.pv = AdjF4{0.f, 0.f, 0.f, 0.f};
    A.rv = load_rec(rt, 0, lim);
    B.rv = load_rec(rt, 1, lim);
    load_x(0, A);
#pragma unroll 1
    for (int64_t t = 0; t < tiles; ++t) {
        const int64_t o = t * kYTile, tn = min(t + 1, tiles - 1);
        const uint32_t *const rn = tile_rec(tn);
        const int limn = rec_tile_obs(tn, O) - 1;
        step(o, A, B, rt, 2, lim);
        if (o + 4 >= O) break;
        step(o + 4, B, A, rt, 3, lim);
        if (o + 8 >= O) break;
        step(o + 8, A, B, rn, 0, limn);
        if (o + 12 >= O) break;
        step(o + 12, B, A, rn, 1, limn);
        rt = rn;
        lim = limn;
    }
    if (s < 8) {
        float *out = a.cbar + ((int64_t)s * P + p) * NS + ib + 16 * q;
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                *reinterpret_cast<float4 *>(out + 64 * u + 4 * rr) =
                    make_float4(acc[u][0][rr], acc[u][1][rr], acc[u][2][rr], acc[u][3][rr]);
    }
}

__device__ __forceinline__ void adj_gather16_wave(const AdjArgs &a, int64_t wave_id) {
    const int64_t P = a.P, nib = a.nib;
    if (wave_id >= P * nib) return;
    // tiles of kAdjPT panels x nib index blocks, panels fastest, as above
    const int64_t tile = wave_id / (kAdjPT * nib);
    const int64_t r = wave_id - tile * (kAdjPT * nib);
    const int64_t tw = min<int64_t>(kAdjPT, P - tile * kAdjPT);
    const int64_t bi = r / tw;
    const int64_t p = tile * kAdjPT + (r - bi * tw);
    const int64_t ib = bi * (64 * kAdj16MW);
    switch ((a.NS - ib) >> 6) {  // NS is a multiple of 64
        case 1: adj_gather16_body<1>(a, p, ib); break;
        case 2: adj_gather16_body<2>(a, p, ib); break;
        case 3: adj_gather16_body<3>(a, p, ib); break;
        case 4: adj_gather16_body<4>(a, p, ib); break;
        default: adj_gather16_body<kAdj16MW>(a, p, ib); break;
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void adj_gather16_kernel(AdjArgs a) {
    adj_gather16_wave(a, xcd_block(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// Batched transposed gather over a longest-first work list: block b runs item b,
// (case c, group g) = the waves 4 g .. 4 g + 3 of case c, wave w being (panel
// w / nib, index block w % nib); waves past the case's P * nib return at once.
// The items are sorted by their work (the paper's greedy partition by size) and
// blocks are dispatched in order, so every compute unit takes the longest item
// left when one of its blocks ends.  (A persistent form pulling items through a
// counter keeps the case arguments live across items: it needs more registers per
// lane than the waves per SIMD this launch runs with allow.)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void adj_gather_listed(const BatchCase *__restrict__ cases,
                                                         const int2 *__restrict__ items) {
    const int2 w = items[blockIdx.x];
    const int c = __builtin_amdgcn_readfirstlane(w.x);
    const int64_t g = __builtin_amdgcn_readfirstlane(w.y);
    adj_gather_wave(cases[c].adj, g * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void adj_gather16_listed(
    const BatchCase *__restrict__ cases, const int2 *__restrict__ items) {
    const int2 w = items[blockIdx.x];
    const int c = __builtin_amdgcn_readfirstlane(w.x);
    const int64_t g = __builtin_amdgcn_readfirstlane(w.y);
    adj_gather16_wave(cases[c].adj, g * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

}  // namespace

hipError_t launch_adj_gather(const PairRec *rec_op, const int32_t *nt, const float *gbar, int64_t P, int64_t O,
                                 int64_t N, int64_t NS, int64_t nt_min, int64_t nt_max, float *gpad, float *cbar,
                                 hipStream_t stream) {
    const int64_t edge_lo = N - nt_min, edge_hi = nt_min + 2;
    const int64_t LR = adj_pad_row(N, NS), padlo = adj_pad_lo(N);
    const PadArgs pa{gbar, nt, O, nt_max, LR, padlo, gpad};
    pad_grad_kernel<<<dim3((unsigned)((O * LR + 255) / 256)), dim3(256), 0, stream>>>(pa);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool narrow = adj_takes_16(O, NS, P * adj_blocks(N));
    const int64_t nib = narrow ? adj16_blocks(NS) : adj_blocks(N);
    const AdjArgs aa{rec_op, nt, gpad, P, O, N, NS, LR, padlo, nib, nt_max, cbar, edge_lo, edge_hi};
    const dim3 grid((unsigned)((P * nib + 3) / 4));
    if (narrow) adj_gather16_kernel<<<grid, dim3(256), 0, stream>>>(aa);
    else adj_gather_mfma_kernel<<<grid, dim3(256), 0, stream>>>(aa);
    return hipGetLastError();
}

hipError_t launch_batch_adjoint(int in_dtype, const BatchCase *cases, BatchIndex idx, int64_t blocks_pad,
                                const int2 *adj_items, int n_adj_items, int n_adj16, int64_t blocks_sadj, int64_t blocks_sadjg,
                                hipStream_t stream) {
    pad_grad_batched<<<dim3((unsigned)blocks_pad), dim3(256), 0, stream>>>(cases, idx.pad, idx.n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n_adj16 > 0) {
        adj_gather16_listed<<<dim3((unsigned)n_adj16), dim3(256), 0, stream>>>(cases, adj_items);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (n_adj_items > n_adj16) {
        adj_gather_listed<<<dim3((unsigned)(n_adj_items - n_adj16)), dim3(256), 0, stream>>>(cases, adj_items + n_adj16);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return launch_batch_source_adjoint(in_dtype, cases, idx.sadj, idx.sadjg, idx.n, blocks_sadj, blocks_sadjg, stream);
}

}  // namespace fwh
