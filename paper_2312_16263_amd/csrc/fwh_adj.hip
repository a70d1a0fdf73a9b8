// Transposed gather of the adjoint (gfx950, FP32/BF16 forms): the coefficient adjoints
//   cbar_c(p, i) = sum_o K_c(o, p) sum_j w_j(o, p) gbar(o, i - n0(o, p) - j),
// a contraction over observers for every (panel, index): it runs on the matrix cores.  Bound by
// matrix and vector issue (80 % of the slots) and by the data return of 16-byte loads at dword
// alignment (84 % busy).  32768 panels x 360 observers x 2048 frames: 8.25 ms against 10.1 as 16x16x4
// products; 240000 panels x 72 observers x 4096 frames: 24.8 against 31.4.
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
    const int64_t nib = adj_blocks(N);
    const AdjArgs aa{rec_op, nt, gpad, P, O, N, NS, LR, padlo, nib, cbar, edge_lo, edge_hi};
    adj_gather_mfma_kernel<<<dim3((unsigned)((P * nib + 3) / 4)), dim3(256), 0, stream>>>(aa);
    return hipGetLastError();
}

hipError_t launch_batch_adjoint(int in_dtype, const BatchCase *cases, BatchIndex idx, int64_t blocks_pad,
                                const int2 *adj_items, int n_adj_items, int64_t blocks_sadj, int64_t blocks_sadjg,
                                hipStream_t stream) {
    pad_grad_batched<<<dim3((unsigned)blocks_pad), dim3(256), 0, stream>>>(cases, idx.pad, idx.n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    adj_gather_listed<<<dim3((unsigned)n_adj_items), dim3(256), 0, stream>>>(cases, adj_items);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_batch_source_adjoint(in_dtype, cases, idx.sadj, idx.sadjg, idx.n, blocks_sadj, blocks_sadjg, stream);
}

}  // namespace fwh
