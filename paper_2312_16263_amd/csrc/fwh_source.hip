// Source stage (gfx950): per panel and source frame, the source terms of
// Eqs. (Qn_New_nd), (Li_New_nd); their 2nd-order source-time derivatives
// (one-sided at the first and last frame, central elsewhere; Sec. III B); and the
// B-spline coefficients of the natural cubic spline through each of the 8
// resulting series (the observer-independent half of the "interp pressure
// signal" step).  Plus the exact transpose of this stage for the adjoint.
//
// The natural cubic spline through f_0..f_{N-1} is sum_n c_n B((tau - tau_n)/dtau)
// with B the uniform cubic B-spline; natural end conditions give c_0 = f_0,
// c_{N-1} = f_{N-1}, c_{-1} = 2c_0 - c_1, c_N = 2c_{N-1} - c_{N-2} and, inside,
// (c_{n-1} + 4 c_n + c_{n+1})/6 = f_n, a constant tridiagonal system solved by
// the Thomas algorithm with the precomputed pivots cp[r] (cp[1] = 1/4,
// cp[r] = 1/(4 - cp[r-1])).
//
// FP32 and BF16 coefficient storage (the plain FP64 form is in fwh_f64.hip): chunks of the record,
// coefficients out panel-major with the 4 channels of a group interleaved, coef[P][2][NS][4] (one
// 4-channel quad per time index).  All arithmetic FP64.
#include "fwh_internal.h"

namespace fwh {
namespace {

struct bf16s {
    uint16_t bits;
};

// ------------------------------------------------------- chunked source stage
// Geometry in fwh_internal.h: a block owns 32 panels
// and 64 coefficient indices; wave w handles base quantity w (Q, L_1, L_2, L_3)
// with lanes 0-31 on its derivative channel and lanes 32-63 on the channel
// itself, so the source terms are wave-uniform.  Each thread runs the forward
// elimination over the rows [R0, R0 + kSrcW) (pivots from the exact table, so a
// window that reaches row 1 is exact) and back-substitutes from the top of the
// window (exact when it reaches row N-2).  Starting elsewhere from zero moves
// the chunk's coefficients by about (2 - sqrt 3)^kSrcH = 7e-10 of their local
// scale, below the FP32/BF16 storage rounding.  No workspace buffer: the
// coefficients leave through an LDS tile [kSrcTC / 4][257], a quarter of the
// chunk at a time, as 16-byte (8-byte for BF16) quads of the interleaved layout.
constexpr int kSrcRS = 257;  // LDS row: 8 channels x 32 panels + 1

// Per-thread source-term form X = a p' + rho (b u_i - g) u.n - d, which covers
// Q (a = 0, b = 0, g = -1, d = U0.n) and L_i (a = n_i, b = 1, g = U0_i, d = 0).
template <typename TIn>
struct SrcLane {
    const TIn *rho, *u, *pp;
    int64_t NP;
    double nx, ny, nz, al, b, gm, dl;
    int uw;               // the base quantity's component of u (0..2; Q: any, times zero)
    double s_der, s_val;  // f = s_der (X+ - X-) + s_val X
    int ch;               // channel index (0..7)
    __device__ __forceinline__ SrcLane(const SrcFwdArgs &a, int64_t pc) {
        rho = static_cast<const TIn *>(a.rho) + pc;
        u = static_cast<const TIn *>(a.u) + pc;
        pp = static_cast<const TIn *>(a.pp) + pc;
        NP = a.N * a.P;
        const int w = threadIdx.x >> 6;
        const bool der = (threadIdx.x & 32) == 0;
        ch = w == 0 ? (der ? 0 : 1) : (der ? 1 + w : 4 + w);
        nx = a.normal[3 * pc];
        ny = a.normal[3 * pc + 1];
        nz = a.normal[3 * pc + 2];
        const double Ux = a.f.ca, Uy = a.f.sa;
        al = w == 1 ? nx : (w == 2 ? ny : (w == 3 ? nz : 0.0));
        b = w == 0 ? 0.0 : 1.0;
        uw = __builtin_amdgcn_readfirstlane(w == 0 ? 0 : w - 1);
        gm = w == 0 ? -1.0 : (w == 1 ? Ux : (w == 2 ? Uy : 0.0));
        dl = w == 0 ? Ux * nx + Uy * ny : 0.0;
        s_der = der ? 1.0 / (2.0 * a.f.dtau) : 0.0;
        s_val = der ? 0.0 : 1.0;
    }
    // the five inputs at a time row, and component uw of u again (read from LDS: fewer instructions than
    // its selection from the three)
    struct Raw {
        TIn r, u1, u2, u3, p, uw;
    };
    __device__ __forceinline__ double X(const Raw &v) const {
        const double r = (double)v.r;
        const double u1 = (double)v.u1, u2 = (double)v.u2, u3 = (double)v.u3;
        const double un = u1 * nx + u2 * ny + u3 * nz;
        const double bu = b * (double)v.uw - gm;
        return al * (double)v.p + r * bu * un - dl;
    }
};

__device__ __forceinline__ uint16_t bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ void store_quad(float *dst, const float *v) {
    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store_quad(bf16s *dst, const float *v) {
    uint2 w;
    w.x = (uint32_t)bf16_rne(v[0]) | ((uint32_t)bf16_rne(v[1]) << 16);
    w.y = (uint32_t)bf16_rne(v[2]) | ((uint32_t)bf16_rne(v[3]) << 16);
    *reinterpret_cast<uint2 *>(dst) = w;
}

// tile[q * kSrcRS + c * 32 + pl] (q < TC) -> coef quads; a wave writes TC
// consecutive indices of one panel and channel group (64 / TC groups per wave).
template <typename TOut, int TC = kSrcTC>
__device__ __forceinline__ void src_flush(const float *tile, TOut *coef, int64_t pbase, int64_t P, int64_t NS,
                                          int64_t i0) {
    for (int e = threadIdx.x; e < kSrcPanels * 2 * TC; e += 256) {
        const int pl = e / (2 * TC);
        const int g = (e / TC) & 1;
        const int q = e & (TC - 1);
        const int64_t p = pbase + pl;
        if (p < P) {
            float v[4];
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) v[cc] = tile[q * kSrcRS + (4 * g + cc) * 32 + pl];
            store_quad(coef + ((p * 2 + g) * NS + i0 + q) * 4, v);
        }
    }
}

// Chunk of kSrcTC coefficient indices i0 .. i0 + 63 for 32 panels: the
// Thomas forward elimination over the kSrcW rows [R0, R0 + kSrcW), R0 = i0 - 17,
// and the back substitution from the top of that window, reduced right-hand
// sides in registers, overwritten by the coefficients.  The block's inputs (5
// variables x 32 panels per source-term row, rows R0 - 3 .. R0 + kSrcW + 2) are
// loaded once, cooperatively, in groups of G = kSrcG rows by direct global -> LDS
// copies into three buffers: groups m + 1 and m + 2 are in flight while group m
// is used, one barrier per group.  The four waves (four base quantities) read
// their inputs from LDS (both half-waves read the same panel's row: a broadcast).
// Bound by the data-return path (90 % busy: 4 bytes a lane), in FP32 data also by vector
// issue (60 % of the cycles; 38 % in FP64), with three blocks of 150 registers per CU: 18252
// panels x 6535 frames, FP32 data, 1.61 ms (6.3 GB, 3.9 TB/s), 1.77 ms with one group in flight and
// per-lane copy addresses; 32768 x 2048, FP64 data, 1.22 ms (4.9 GB) against 1.44.
//
// GEN = false: interior chunk (every row in [kSrcPivotRows, N - 3]): central
// differences, constant pivot, no end rows, no branches.  GEN = true: a chunk
// with a record end in reach: zero source terms outside the record, one-sided
// differences at the first and last frame, exact pivots, the end rows'
// right-hand-side corrections and the end coefficients c_{-1}, c_0, c_{N-1},
// c_N, zero padding past c_N.  Row positions are compile-time (unrolled) and
// the end rules block-uniform predicates, so both kinds keep the right-hand
// sides in registers.  The coefficients leave through a [kSrcTC / 4][kSrcRS]
// LDS tile in four quarters.
// rows per staged group: three buffers of a group, the LDS tile and the end values leave room for three
// blocks per CU
template <typename TIn>
constexpr int kSrcG = sizeof(TIn) == 8 ? 8 : 12;
constexpr int kSrcNX = kSrcW + 6;               // source-term rows R0 - 3 .. R0 + kSrcW + 2
template <typename TIn>
constexpr int kSrcNG = (kSrcNX + kSrcG<TIn> - 1) / kSrcG<TIn>;
template <typename TIn>
constexpr int kSrcGV = kSrcG<TIn> * 5 * kSrcPanels;  // values per group

typedef __attribute__((address_space(3))) void *src_lds_ptr_t;

// Direct global -> LDS copies of the staged groups.  Group m goes to
// dst[var][r][panel]: variables [rho, u1, u2, u3, p'], source-term rows k =
// m*G + r (record row R0 - 3 + k, clamped to [0, N-1]), panels pbase ..
// pbase + 31.  A piece of 64 dwords (4 bytes per lane) is one (variable, row) in
// FP64 and two rows of a variable in FP32; the lane's panel (clamped to P - 1),
// dword half and row within the piece are fixed.  Wave wv issues the pieces wv,
// wv + 4, ...; one whose first row lies past the staged rows takes the last of them instead, since the waits
// count the pieces issued.
template <typename TIn>
struct SrcDma {
    static constexpr int DW = (int)sizeof(TIn) / 4;  // dwords per value
    static constexpr int RPP = 2 / DW;               // rows per piece
    static constexpr int G = kSrcG<TIn>;
    static constexpr int PPV = G / RPP;          // pieces per variable
    static constexpr int NPIECE = 5 * PPV;
    static constexpr int NI = (NPIECE + 3) / 4;      // pieces per wave (at most)
    const unsigned char *vbase[NI];                  // variable base of piece i (uniform)
    int r[NI];                                       // its first row in the group
    int64_t rowb;                                    // bytes per record row (P values)

    __device__ __forceinline__ SrcDma(const SrcFwdArgs &a, int wv) {
        rowb = a.P * (int64_t)sizeof(TIn);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            int pc = wv + 4 * i;
            pc = pc < NPIECE ? pc : NPIECE - 1;
            const int var = pc / PPV;
            r[i] = (pc - var * PPV) * RPP;
            vbase[i] = var == 0 ? static_cast<const unsigned char *>(a.rho)
                                : (var == 4 ? static_cast<const unsigned char *>(a.pp)
                                            : static_cast<const unsigned char *>(a.u) + (int64_t)(var - 1) * a.N * rowb);
        }
    }

    // lane_row: row of this lane within a piece (0, or lane >> 5 in FP32);
    // lane_off: byte offset of the lane's panel and dword half within a row.
    // CLAMP: rows outside the record are clamped, lane by lane.  Otherwise (interior chunks, all of whose
    // rows are in the record) a piece is a uniform address and the lane's constant offset, no vector
    // arithmetic (in FP32 that was a quarter of the kernel's); a piece of two rows of which the second is
    // past the staged rows reads the first one twice.
    template <bool CLAMP>
    __device__ __forceinline__ void issue(int m, TIn *dst, int wv, int lane_row, uint32_t lane_off, int64_t R0,
                                          int64_t N) const {
        const uint32_t piece_off = (uint32_t)lane_row * (uint32_t)rowb + lane_off;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int pc = wv + 4 * i;
            const int k0 = min(m * G + r[i], kSrcNX - 1);
            const bool go = NPIECE % 4 == 0 || i + 1 < NI || pc < NPIECE;
            if (go) {
                const unsigned char *src;
                if constexpr (CLAMP) {
                    int64_t row = R0 - 3 + k0 + lane_row;
                    row = row < 0 ? 0 : (row > N - 1 ? N - 1 : row);
                    src = vbase[i] + row * rowb + lane_off;
                } else {
                    src = vbase[i] + (R0 - 3 + k0) * rowb + ((m + 1) * G <= kSrcNX || k0 + RPP <= kSrcNX ? piece_off : lane_off);
                }
                __builtin_amdgcn_global_load_lds((const void *)src, (src_lds_ptr_t)((unsigned char *)dst + pc * 256), 4,
                                                 0, 0);
            }
        }
    }
};

// ENDS (GEN): which record ends the chunk's rows can reach, bit 0 the first frame (R0 <= 3), bit 1
// the last (R0 + kSrcW >= N - 1); the rules of an end out of reach are compiled out (they would be
// false at run time).
template <typename TIn, typename TOut, bool GEN, int ENDS = 3>
__device__ __forceinline__ void src_chunk(const SrcFwdArgs &a, int64_t pbk, int64_t i0, TIn *ring0, TIn *ring1, TIn *ring2,
                                          float *tile, double *endv) {
    constexpr bool kStart = (ENDS & 1) != 0, kEnd = (ENDS & 2) != 0;
    const int64_t P = a.P, N = a.N;
    const int pl = threadIdx.x & 31;
    const int half = (threadIdx.x >> 5) & 1;  // row of a pair this half-wave computes X for
    const int64_t pbase = pbk * kSrcPanels;
    const int64_t pc = min(pbase + pl, P - 1);
    const SrcLane<TIn> L(a, pc);
    using Raw = typename SrcLane<TIn>::Raw;
    const double cpi = 2.0 - sqrt(3.0);
    // interior: the right-hand side's 6 and the pivot are in the scales of f
    const double s_der = GEN ? L.s_der : 6.0 * cpi * L.s_der, s_val = GEN ? L.s_val : 6.0 * cpi * L.s_val;
    const int64_t R0 = i0 - 1 - kSrcH;
    // Exact Thomas pivots of tridiag(1, 4, 1) (GEN): c'_1 = 1/4, c'_n = 1/(4 - c'_{n-1}), from the
    // plan's table a.cp (a uniform load; equal to cpi to double precision past n = 30, so rows from
    // 64 on take cpi)
    const double *__restrict__ cpt = a.cp;
    auto pivot = [&](int rr) { return rr < 64 ? cpt[rr] : cpi; };
    // 32-bit copies for the block-uniform end rules (records are far below 2^31 frames)
    const int R0i = (int)R0, Ni = (int)N;
    // three buffers of [rho, u1, u2, u3, p'] x G rows x 32 panels; group m in buffer m % 3
    constexpr int G = kSrcG<TIn>, NG = kSrcNG<TIn>, VS = G * kSrcPanels;  // VS: variable stride
    const int own = half * kSrcPanels + pl, own_uw = own + (1 + L.uw) * VS;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int lane_row;
    uint32_t lane_off;
    if constexpr (sizeof(TIn) == 8) {
        lane_row = 0;
        lane_off = (uint32_t)(min(pbase + (lane >> 1), P - 1) * 8 + (lane & 1) * 4);
    } else {
        lane_row = lane >> 5;
        lane_off = (uint32_t)(min(pbase + (lane & 31), P - 1) * 4);
    }
    const SrcDma<TIn> dma(a, wv);
    dma.template issue<GEN>(0, ring0, wv, lane_row, lane_off, R0, N);
    dma.template issue<GEN>(1, ring1, wv, lane_row, lane_off, R0, N);
    // reduced right-hand sides, then coefficients, of window rows s, in registers
    const int col = L.ch * 32 + pl;
    float dvr[kSrcW];
    auto DV = [&](int s_) -> float & { return dvr[s_]; };
    // Forward sweep over source-term rows k (record row R0 - 3 + k).  Step it (it = 0 .. kSrcW + 1,
    // right-hand side of frame n = R0 - 1 + it) takes X of frames n - 2 .. n + 2 = rows it .. it + 4.
    double Xa = 0.0, Xb = 0.0, Xc = 0.0, Xd = 0.0, Xe = 0.0;
    double fprev = 0.0, dprev = 0.0, f0 = 0.0;
#pragma unroll
    for (int m = 0; m < NG; ++m) {
        // this wave's copies of group m have landed (those of group m + 1 may be in flight); the barrier
        // makes every wave's visible and frees the buffer of group m - 1, which receives group m + 2
        constexpr int kAhead = SrcDma<TIn>::NPIECE / 4;  // copies of a group, of the wave with the fewest
        if (m + 1 < NG) __builtin_amdgcn_s_waitcnt((kAhead & 15) | 0x70 | (kAhead >> 4) << 14);
        else __builtin_amdgcn_s_waitcnt(0x70);
        // (no __syncthreads: it waits for every copy in flight)
        asm volatile("s_barrier" ::: "memory");
        if (m + 2 < NG)
            dma.template issue<GEN>(m + 2, (m + 2) % 3 == 0 ? ring0 : ((m + 2) % 3 == 1 ? ring1 : ring2), wv, lane_row,
                                    lane_off, R0, N);
        const TIn *buf = m % 3 == 0 ? ring0 : (m % 3 == 1 ? ring1 : ring2);
        // Rows go in pairs: lanes 0-31 compute X of row k, lanes 32-63 (the same panel and base
        // quantity) X of row k + 1, and one swap of the halves (v_permlane32_swap, per dword) gives
        // every lane both, so each source term is computed once instead of once per half.
        auto row_step = [&](const int k, const double Xn) __attribute__((always_inline)) {
            Xa = Xb;
            Xb = Xc;
            Xc = Xd;
            Xd = Xe;
            Xe = Xn;
            if (k >= 4) {
                const int it = k - 4;
                const int n = R0i - 1 + it;
                double fn;
                if constexpr (!GEN) {
                    fn = s_der * (Xd - Xb) + s_val * Xc;
                } else {
                    fn = 0.0;
                    if ((unsigned)n < (unsigned)Ni) {
                        const double dx = (kStart && n == 0) ? -3.0 * Xc + 4.0 * Xd - Xe
                                          : ((kEnd && n == Ni - 1) ? 3.0 * Xc - 4.0 * Xb + Xa : Xd - Xb);
                        fn = s_der * dx + s_val * Xc;
                    }
                    if (kStart && n == 0) f0 = fn;
                    // f_{N-1} and (below) d_{N-2} wait in LDS for the end coefficients: held in
                    // registers across the back substitution they cost it about 110 registers
                    if (kEnd && n == Ni - 1) endv[col] = fn;
                }
                if (it >= 2) {
                    float dvs;
                    if constexpr (!GEN) {
                        const double d = fma(-cpi, dprev, fprev);
                        dprev = d;
                        dvs = (float)d;
                    } else {
                        const int rr = n - 1;  // system row
                        dvs = 0.f;
                        if ((unsigned)(rr - 1) < (unsigned)(Ni - 2)) {
                            double rhs = 6.0 * fprev;
                            if (kStart && rr == 1) rhs -= f0;
                            if (kEnd && rr == Ni - 2) rhs -= fn;
                            const double piv = pivot(rr);
                            const double d = (rhs - dprev) * piv;
                            dprev = d;
                            dvs = (float)d;
                            if (kEnd && rr == Ni - 2) endv[256 + col] = d;
                        }
                    }
                    dvr[it - 2] = dvs;
                    // computed here, not sunk to the back substitution (which would keep every
                    // row's inputs live)
                    asm volatile("" : "+v"(dvr[it - 2]));
                }
                fprev = fn;
            }
        };
#pragma unroll
        for (int r = 0; r < G; r += 2) {
            const int k = m * G + r;
            if (k < kSrcNX) {
                // (one integer offset from the buffer: through a longer chain of pointers the compiler no
                // longer sees that the copies in flight go to other buffers, and waits for them here)
                const int at = own + r * kSrcPanels, at_uw = own_uw + r * kSrcPanels;
                const Raw v{buf[at], buf[at + VS], buf[at + 2 * VS], buf[at + 3 * VS], buf[at + 4 * VS], buf[at_uw]};
                double Xm = L.X(v);
                if constexpr (GEN) {
                    const int mrow = R0i - 3 + k + half;
                    if ((unsigned)mrow >= (unsigned)Ni) Xm = 0.0;
                }
                const unsigned xl = (unsigned)__double2loint(Xm), xh = (unsigned)__double2hiint(Xm);
                const auto sl = __builtin_amdgcn_permlane32_swap(xl, xl, false, false);
                const auto sh = __builtin_amdgcn_permlane32_swap(xh, xh, false, false);
                row_step(k, __hiloint2double((int)sh[0], (int)sl[0]));  // row k (lanes 0-31's value)
                if (k + 1 < kSrcNX) row_step(k + 1, __hiloint2double((int)sh[1], (int)sl[1]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // back substitution from the top of the window; window row s holds coefficient index i = R0 + s + 1
    double x = 0.0;
#pragma unroll
    for (int s = kSrcW - 1; s >= 0; --s) {
        if constexpr (!GEN) {
            x = (double)dvr[s] - cpi * x;
            dvr[s] = (float)x;
        } else {
            const int rr = R0i + s;
            if ((unsigned)(rr - 1) < (unsigned)(Ni - 2)) x = (double)DV(s) - pivot(rr) * x;
            if (s >= kSrcH && s < kSrcH + kSrcTC) {
                const int i = rr + 1;
                double v;
                if (kStart && i == 0) v = 2.0 * f0 - x;
                else if (kStart && i == 1) v = f0;
                else if (i < Ni) v = x;
                else v = 0.0;  // c_N and c_{N+1} are set as the coefficients leave (below)
                DV(s) = (float)v;
            }
        }
    }
    TOut *coef = static_cast<TOut *>(a.coef);
    constexpr int QT = kSrcTC / 4;
#pragma unroll
    for (int qt = 0; qt < 4; ++qt) {
        __syncthreads();  // the previous quarter's tile has been read
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            float c = dvr[kSrcH + qt * QT + q];
            if constexpr (GEN && kEnd) {
                // the last frame's end coefficients c_N = f_{N-1}, c_{N+1} = 2 f_{N-1} - d_{N-2} (both
                // rows lie in the window of a chunk that holds index N or N + 1)
                const int i = (int)i0 + qt * QT + q;
                if (i == Ni) c = (float)endv[col];
                else if (i == Ni + 1) c = (float)(2.0 * endv[col] - endv[256 + col]);
            }
            tile[q * kSrcRS + col] = c;
        }
        __syncthreads();
        src_flush<TOut, QT>(tile, coef, pbase, P, a.NS, i0 + qt * QT);
    }
}

// Chunk k of panel block pbk, with the end rules it can reach.  One set of LDS arrays for all forms:
// separate arrays of the instantiations inlined into one kernel would add up.
template <typename TIn, typename TOut>
__device__ __forceinline__ void src_chunk_block(const SrcFwdArgs &a, int64_t pbk, int64_t k, bool interior) {
    __shared__ TIn ring0[kSrcGV<TIn>], ring1[kSrcGV<TIn>], ring2[kSrcGV<TIn>];
    __shared__ float tile[(kSrcTC / 4) * kSrcRS];
    __shared__ double endv[2 * 256];  // f_{N-1}, d_{N-2} per thread
    const int64_t i0 = k * kSrcTC, R0 = i0 - 1 - kSrcH;
    if (interior) {
        src_chunk<TIn, TOut, false>(a, pbk, i0, ring0, ring1, ring2, tile, endv);
    } else {
        const bool s_in = R0 <= 3, e_in = R0 + kSrcW >= a.N - 1;
        if (s_in && e_in) src_chunk<TIn, TOut, true, 3>(a, pbk, i0, ring0, ring1, ring2, tile, endv);
        else if (e_in) src_chunk<TIn, TOut, true, 2>(a, pbk, i0, ring0, ring1, ring2, tile, endv);
        else src_chunk<TIn, TOut, true, 1>(a, pbk, i0, ring0, ring1, ring2, tile, endv);
    }
}

// ------------------------------------------------ chunked source adjoint stage
// FP32/BF16 modes: the exact transpose of the chunked source stage, fused with
// the derivative transpose and the chain rule (geometry in fwh_internal.h).
// With a_k the adjoint of coefficient c_k (storage index k + 1):
//   chat_r = a_r - [r = 1] a_{-1} - [r = N-2] a_N   (r = 1 .. N-2),  z = A^{-1} chat,
//   fbar_j = 6 z_j (1 <= j <= N-2),  fbar_0 = a_0 + 2 a_{-1} - z_1,
//   fbar_{N-1} = a_{N-1} + 2 a_N - z_{N-2}
// (A = tridiag(1, 4, 1) is symmetric, so its transpose solve is the same Thomas
// sweep); then Xbar = fbar (value channels) or D^T fbar (derivative channels)
// and the chain rule through the source terms at every frame of the chunk.
// Wave w, lanes 0-31 / 32-63: base w, derivative / value channel (as forward).

// Xbar of 8 channels at (frame m, panel) from tile[(m - m0) * kSrcRS + c * 32 + pl];
// chain rule; gradients out time-major (32 consecutive panels per frame).
template <typename TIn, int TC = kSrcTC>
__device__ __forceinline__ void src_adj_chain_out(const float *tile, const SrcAdjArgs &a, int64_t pbase, int64_t m0) {
    const int64_t P = a.P, N = a.N, NP = N * P;
    const TIn *__restrict__ rho = static_cast<const TIn *>(a.rho);
    const TIn *__restrict__ u = static_cast<const TIn *>(a.u);
    TIn *__restrict__ g_rho = static_cast<TIn *>(a.g_rho);
    TIn *__restrict__ g_u = static_cast<TIn *>(a.g_u);
    TIn *__restrict__ g_p = static_cast<TIn *>(a.g_p);
    const int pl = threadIdx.x & 31;
    const int64_t p = pbase + pl;
    if (p >= P) return;
    const double nx = a.normal[3 * p], ny = a.normal[3 * p + 1], nz = a.normal[3 * p + 2];
    const double Ux = a.f.ca, Uy = a.f.sa;
    // all of this thread's frames are loaded before any gradient is stored
    constexpr int NF = TC / 8;
    TIn vr[NF], v1[NF], v2[NF], v3[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int64_t m = m0 + (threadIdx.x >> 5) + 8 * f;
        const int64_t idx = (m < N ? m : N - 1) * P + p;
        vr[f] = rho[idx];
        v1[f] = u[idx];
        v2[f] = u[NP + idx];
        v3[f] = u[2 * NP + idx];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int ml = (threadIdx.x >> 5) + 8 * f;
        const int64_t m = m0 + ml;
        if (m < N) {
            const float *t = tile + ml * kSrcRS + pl;
            const double Qb = (double)t[0] + (double)t[32];
            const double L1 = (double)t[2 * 32] + (double)t[5 * 32];
            const double L2 = (double)t[3 * 32] + (double)t[6 * 32];
            const double L3 = (double)t[4 * 32] + (double)t[7 * 32];
            const int64_t idx = m * P + p;
            const double r = (double)vr[f];
            const double u1 = (double)v1[f], u2 = (double)v2[f], u3 = (double)v3[f];
            const double un = u1 * nx + u2 * ny + u3 * nz;
            const double w1 = u1 - Ux, w2 = u2 - Uy, w3 = u3;
            const double S = Qb + L1 * w1 + L2 * w2 + L3 * w3;
            g_rho[idx] = (TIn)(un * S);
            g_u[idx] = (TIn)(r * nx * S + r * un * L1);
            g_u[NP + idx] = (TIn)(r * ny * S + r * un * L2);
            g_u[2 * NP + idx] = (TIn)(r * nz * S + r * un * L3);
            g_p[idx] = (TIn)(L1 * nx + L2 * ny + L3 * nz);
        }
    }
}

struct AdjLane {
    double s_der, s_val;
    int ch;
    __device__ __forceinline__ explicit AdjLane(double dtau) {
        const int w = threadIdx.x >> 6;
        const bool der = (threadIdx.x & 32) == 0;
        ch = w == 0 ? (der ? 0 : 1) : (der ? 1 + w : 4 + w);
        s_der = der ? 1.0 / (2.0 * dtau) : 0.0;
        s_val = der ? 0.0 : 1.0;
    }
};

constexpr int kAdjSlab = 32;            // storage indices per staged slab
constexpr int kAdjSlabRS = kAdjSlab + 1;

// One chunk of kSrcTC frames m0 .. m0 + 63 for 32 panels: window rows s = 0 .. kAdjW - 1 are
// system rows r = m0 - kAdjLo + s (storage index r + 1).  The coefficient adjoints come in
// through LDS slabs of 32 indices x 256 rows (8 lanes per 128-byte row segment); the reduced
// right-hand sides, then z, then Xbar stay in registers (the window loops are unrolled, so every
// row position is a compile-time index).
// GEN = false (interior chunk, every row in [kSrcPivotRows, N - 3]): constant pivot, no end rows.
// GEN = true (either record end in reach, or a short record): the exact pivots cp[r], the end
// rows' right-hand-side corrections, fbar_0 and fbar_{N-1}, one-sided differences at the first
// and last frames, as block-uniform predicates on the row; slab indices outside the row are
// clamped into it (those rows are never used).
template <typename TIn, bool GEN>
__device__ __forceinline__ void src_adj_chunk(const SrcAdjArgs &a, int64_t pbk, int64_t k, float *lds) {
    const int64_t P = a.P, NS = a.NS;
    const int pl = threadIdx.x & 31;
    const int64_t pbase = pbk * kSrcPanels;
    const AdjLane L(a.f.dtau);
    const double cpi = 2.0 - sqrt(3.0);
    const int64_t m0 = k * kSrcTC;
    const int64_t i_lo = m0 - kAdjLo + 1;  // storage index of window row 0
    // cooperative slab loads: float4 e = tid + 256 j -> row e / 8 (channel-major rows c*32 + pl), quad e % 8
    auto slab_load = [&](int t, float4 *v) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = threadIdx.x + 256 * j;
            const int row = e >> 3, qd = e & 7;
            const int64_t pr = min(pbase + (row & 31), P - 1);
            int64_t idx = i_lo + t * kAdjSlab + 4 * qd;  // a multiple of 4, as NS is
            if constexpr (GEN) idx = idx < 0 ? 0 : (idx > NS - 4 ? NS - 4 : idx);
            const float *src = a.cbar + ((int64_t)(row >> 5) * P + pr) * NS + idx;
            v[j] = *reinterpret_cast<const float4 *>(src);
        }
    };
    auto slab_store = [&](const float4 *v) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = threadIdx.x + 256 * j;
            float *dst = lds + (e >> 3) * kAdjSlabRS + 4 * (e & 7);
            dst[0] = v[j].x;
            dst[1] = v[j].y;
            dst[2] = v[j].z;
            dst[3] = v[j].w;
        }
    };
    const int myrow = L.ch * 32 + pl;
    // GEN: end data of this thread's row (a_{-1}, a_0, a_{N-1}, a_N) and 32-bit row positions
    const int Ni = (int)a.N, R0i = (int)(m0 - kAdjLo);
    const double *__restrict__ cp = a.cp;
    double am1 = 0.0, a0 = 0.0, aN1 = 0.0, aN = 0.0;
    if constexpr (GEN) {
        const float *row = a.cbar + ((int64_t)L.ch * P + min(pbase + pl, P - 1)) * NS;
        am1 = row[0];
        a0 = row[1];
        aN1 = row[Ni];
        aN = row[Ni + 1];
    }
    auto inside = [&](int r) { return (unsigned)(r - 1) < (unsigned)(Ni - 2); };  // 1 <= r <= N - 2
    auto pivot = [&](int r) { return r < 64 ? cp[r] : cpi; };
    float dv[kAdjW];
    double dprev = 0.0;
    float4 cur[8], nxt[8];
    slab_load(0, cur);
#pragma unroll
    for (int t = 0; t < kAdjW / kAdjSlab; ++t) {
        if (t + 1 < kAdjW / kAdjSlab) slab_load(t + 1, nxt);
        __syncthreads();
        slab_store(cur);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kAdjSlab; ++q) {
            const double c = (double)lds[myrow * kAdjSlabRS + q];
            if constexpr (!GEN) {
                const double d = (c - dprev) * cpi;
                dprev = d;
                dv[t * kAdjSlab + q] = (float)d;
            } else {
                const int r = R0i + t * kAdjSlab + q;
                float v = 0.f;
                if (inside(r)) {
                    double cc = c;
                    if (r == 1) cc -= am1;
                    if (r == Ni - 2) cc -= aN;
                    const double d = (cc - dprev) * pivot(r);
                    dprev = d;
                    v = (float)d;
                }
                dv[t * kAdjSlab + q] = v;
            }
        }
        if (t + 1 < kAdjW / kAdjSlab) {
#pragma unroll
            for (int j = 0; j < 8; ++j) cur[j] = nxt[j];
        }
    }
    if constexpr (!GEN) {
        // back substitution; Xbar_m once fbar_{m-1} is known (window row s = m - m0 + kAdjLo - 1),
        // kept in place of the consumed right-hand side dv[s]
        double z = 0.0, fp1 = 0.0, fc = 0.0;
#pragma unroll
        for (int s = kAdjW - 1; s >= 0; --s) {
            z = (double)dv[s] - cpi * z;
            const double fm1 = 6.0 * z;
            const int ml = s - kAdjLo + 1;  // frame m = m0 + ml has fbar_{m-1} = fm1
            if (ml >= 0 && ml < kSrcTC) dv[s] = (float)(L.s_val * fc + L.s_der * (fm1 - fp1));
            fp1 = fc;
            fc = fm1;
        }
    } else {
        // back substitution (z rounded to FP32 in place), then fbar and Xbar_m, which overwrites
        // the row of fbar_{m-1} (no later frame needs it)
        double z = 0.0, z1 = 0.0, zN2 = 0.0;
#pragma unroll
        for (int s = kAdjW - 1; s >= 0; --s) {
            const int r = R0i + s;
            if (inside(r)) {
                z = (double)dv[s] - pivot(r) * z;
                dv[s] = (float)z;
                if (r == 1) z1 = z;
                if (r == Ni - 2) zN2 = z;
            }
        }
        const double fb0 = a0 + 2.0 * am1 - z1, fbN1 = aN1 + 2.0 * aN - zN2;
        // fbar_j of window row s = j - (m0 - kAdjLo)
        auto fbar = [&](int j, int s_) -> double {
            if (j == 0) return fb0;
            if (j == Ni - 1) return fbN1;
            if (inside(j)) return 6.0 * (double)dv[s_];
            return 0.0;
        };
        const double sd = L.s_der;
#pragma unroll
        for (int ml = 0; ml < kSrcTC; ++ml) {
            const int m = R0i + kAdjLo + ml;
            double xb = 0.0;
            if (m < Ni) {
                const double fm = fbar(m, ml + kAdjLo);
                double dx = 0.0;
                if (inside(m - 1)) dx += fbar(m - 1, ml + kAdjLo - 1);
                if (inside(m + 1)) dx -= fbar(m + 1, ml + kAdjLo + 1);
                if (m == 0) dx -= 3.0 * fb0;
                if (m == 1) dx += 4.0 * fb0;
                if (m == 2) dx -= fb0;
                if (m == Ni - 1) dx += 3.0 * fbN1;
                if (m == Ni - 2) dx -= 4.0 * fbN1;
                if (m == Ni - 3) dx += fbN1;
                xb = L.s_val * fm + sd * dx;
            }
            dv[ml + kAdjLo - 1] = (float)xb;
        }
    }
    // chain rule in two halves of kSrcTC / 2 frames through a [kSrcTC / 2][kSrcRS] tile
    constexpr int HT = kSrcTC / 2;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __syncthreads();  // the slabs (first half) or the previous half's tile have been read
#pragma unroll
        for (int q = 0; q < HT; ++q) lds[q * kSrcRS + myrow] = dv[half * HT + q + kAdjLo - 1];
        __syncthreads();
        src_adj_chain_out<TIn, HT>(lds, a, pbase, m0 + half * HT);
    }
}

// slabs [256][kAdjSlabRS], then the Xbar tile [kSrcTC / 2][kSrcRS]
constexpr int kAdjWords = 256 * kAdjSlabRS > (kSrcTC / 2) * kSrcRS ? 256 * kAdjSlabRS : (kSrcTC / 2) * kSrcRS;
template <typename TIn>
__device__ __forceinline__ void src_adj_block(const SrcAdjArgs &a, int64_t pbk, int64_t k, bool interior) {
    __shared__ float lds[kAdjWords];
    if (interior) src_adj_chunk<TIn, false>(a, pbk, k, lds);
    else src_adj_chunk<TIn, true>(a, pbk, k, lds);
}

// One launch for all chunks: the boundary chunks' blocks first (ngen chunks of every panel block,
// padded to a multiple of kXcds blocks), then the interior ones, so that the boundary chunks do not run
// as a launch of their own with most of the chip idle at its end (source adjoint of a 2048-panel,
// 512-frame surface: 46 us in two launches).
// Interior: (panel block, chunk) pairs, chunks fastest, renumbered per XCD: the chunks of
// one panel block run together on one XCD, so the coefficient-adjoint rows that neighbouring chunks
// both read (the recurrences' overlap) come from that XCD's L2 rather than from HBM twice.
// INT: there are interior chunks (records without any run the boundary form alone, a smaller kernel: 8281 panels x 76
// frames 38 us, 46 with both).
template <typename TIn, bool INT>
__global__ __launch_bounds__(256) void src_adj_kernel(SrcAdjArgs a, int64_t pb, int64_t ngen, int64_t nint,
                                                      int64_t gen_blocks) {
    const int64_t h = blockIdx.x;
    if (!INT || h < gen_blocks) {
        if (h < pb * ngen) src_adj_block<TIn>(a, h % pb, src_general_chunk(h / pb, nint), false);
    } else {
        const int64_t L = xcd_block(h - gen_blocks, gridDim.x - gen_blocks), pbk = L / nint;
        src_adj_block<TIn>(a, pbk, 1 + L - pbk * nint, true);
    }
}
// batched: the boundary chunks of all cases, then the interior ones
template <typename TIn, bool INT>
__global__ __launch_bounds__(256) void src_adj_batched(const BatchCase *__restrict__ cases,
                                                       const int64_t *__restrict__ start,
                                                       const int64_t *__restrict__ startg, int n, int64_t gen_blocks) {
    const int64_t g = blockIdx.x;
    if (!INT || g < gen_blocks) {
        if (g >= startg[n]) return;
        const int c = find_case(startg, n, g);
        const int64_t local = g - startg[c], N = cases[c].sadj.N;
        const int64_t nint = adj_interior_chunks(N), ng = adj_chunks(N) - nint, pbk = local / ng;
        src_adj_block<TIn>(cases[c].sadj, pbk, src_general_chunk(local - pbk * ng, nint), false);
    } else {
        const int64_t h = xcd_block(g - gen_blocks, gridDim.x - gen_blocks);
        const int c = find_case(start, n, h);
        const int64_t local = h - start[c];
        const int64_t nk = adj_interior_chunks(cases[c].sadj.N), pbk = local / nk;
        src_adj_block<TIn>(cases[c].sadj, pbk, 1 + local - pbk * nk, true);
    }
}

constexpr int64_t round_xcd(int64_t blocks) { return (blocks + kXcds - 1) / kXcds * kXcds; }

template <typename TIn>
hipError_t src_adj_chunk_launch_t(const SrcAdjArgs &a, hipStream_t stream) {
    const int64_t pb = (a.P + kSrcPanels - 1) / kSrcPanels;
    const int64_t nint = adj_interior_chunks(a.N), ngen = adj_chunks(a.N) - nint, gb = round_xcd(pb * ngen);
    const dim3 grid((unsigned)(gb + pb * nint));
    if (nint > 0) src_adj_kernel<TIn, true><<<grid, dim3(256), 0, stream>>>(a, pb, ngen, nint, gb);
    else src_adj_kernel<TIn, false><<<grid, dim3(256), 0, stream>>>(a, pb, ngen, nint, gb);
    return hipGetLastError();
}

// grid (panel blocks, chunks): the ngen boundary chunks first, then the interior ones k = 1 .. nint, all in
// one launch (a launch per boundary chunk ran 1024 blocks each on the 32768-panel sphere, 100 us apiece,
// 0.25 ms of its 1.30 ms).  (Chunks of one panel block on one XCD, as the source adjoint runs them, did
// not cut this stage's HBM reads: a chunk reads the rows it shares with the next one last, the next
// chunk reads them first.)
template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void src_kernel(SrcFwdArgs a, int64_t ngen,
                                                                                         int64_t nint) {
    const int64_t g = blockIdx.y;
    src_chunk_block<TIn, TOut>(a, blockIdx.x, g < ngen ? src_general_chunk(g, nint) : 1 + g - ngen, g >= ngen);
}
// batched: the boundary chunks of all cases, then the interior ones; blocks of case c are [start[c],
// start[c+1]) of each, panel block major
template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void src_batched(
    const BatchCase *__restrict__ cases, const int64_t *__restrict__ start, const int64_t *__restrict__ startg, int n) {
    const int64_t gen_blocks = startg[n], g = blockIdx.x;
    const bool interior = g >= gen_blocks;
    const int64_t h = interior ? g - gen_blocks : g;
    const int64_t *st = interior ? start : startg;
    const int c = find_case(st, n, h);
    const int64_t local = h - st[c], nint = src_interior_chunks(cases[c].src.N);
    const int64_t nk = interior ? nint : cases[c].src.NS / kSrcTC - nint, pbk = local / nk, j = local - pbk * nk;
    src_chunk_block<TIn, TOut>(cases[c].src, pbk, interior ? 1 + j : src_general_chunk(j, nint), interior);
}

template <typename TIn, typename TOut>
hipError_t source_chunk_launch_t(const SrcFwdArgs &a, hipStream_t stream) {
    const int64_t nint = src_interior_chunks(a.N), nk = a.NS / kSrcTC;
    src_kernel<TIn, TOut><<<dim3((unsigned)((a.P + kSrcPanels - 1) / kSrcPanels), (unsigned)nk), dim3(256), 0, stream>>>(
        a, nk - nint, nint);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_source(int in_dtype, int coef_type, const void *rho, const void *u, const void *pp,
                         const double *normal, int64_t P, int64_t N, int64_t NS, Flow f, const double *cp, void *coef,
                         hipStream_t stream) {
    const SrcFwdArgs a{rho, u, pp, normal, P, N, NS, f, cp, nullptr, coef};
    if (in_dtype == 0)
        return coef_type == 1 ? source_chunk_launch_t<double, float>(a, stream)
                              : source_chunk_launch_t<double, bf16s>(a, stream);
    return coef_type == 1 ? source_chunk_launch_t<float, float>(a, stream)
                          : source_chunk_launch_t<float, bf16s>(a, stream);
}

hipError_t launch_source_adjoint(int in_dtype, const void *cbar, const void *rho, const void *u, const double *normal,
                                 int64_t P, int64_t N, int64_t NS, Flow f, const double *cp, void *g_rho, void *g_u,
                                 void *g_p, hipStream_t stream) {
    const SrcAdjArgs sa{static_cast<const float *>(cbar), rho, u, normal, P, N, NS, f, cp, g_rho, g_u, g_p};
    if (in_dtype == 0) return src_adj_chunk_launch_t<double>(sa, stream);
    return src_adj_chunk_launch_t<float>(sa, stream);
}

// Batched source stages.
hipError_t launch_batch_source(int in_dtype, int coef_type, const BatchCase *cases, const int64_t *start_int,
                               const int64_t *start_gen, int n, int64_t blocks_int, int64_t blocks_gen,
                               hipStream_t stream) {
    const dim3 g((unsigned)(blocks_int + blocks_gen)), b(256);
    if (in_dtype == 0) {
        if (coef_type == 1) src_batched<double, float><<<g, b, 0, stream>>>(cases, start_int, start_gen, n);
        else src_batched<double, bf16s><<<g, b, 0, stream>>>(cases, start_int, start_gen, n);
    } else {
        if (coef_type == 1) src_batched<float, float><<<g, b, 0, stream>>>(cases, start_int, start_gen, n);
        else src_batched<float, bf16s><<<g, b, 0, stream>>>(cases, start_int, start_gen, n);
    }
    return hipGetLastError();
}

hipError_t launch_batch_source_adjoint(int in_dtype, const BatchCase *cases, const int64_t *start_int,
                                       const int64_t *start_gen, int n, int64_t blocks_int, int64_t blocks_gen,
                                       hipStream_t stream) {
    const int64_t gb = round_xcd(blocks_gen);
    const dim3 g((unsigned)(blocks_int + gb)), b(256);
    if (in_dtype == 0) {
        if (blocks_int > 0) src_adj_batched<double, true><<<g, b, 0, stream>>>(cases, start_int, start_gen, n, gb);
        else src_adj_batched<double, false><<<g, b, 0, stream>>>(cases, start_int, start_gen, n, gb);
    } else {
        if (blocks_int > 0) src_adj_batched<float, true><<<g, b, 0, stream>>>(cases, start_int, start_gen, n, gb);
        else src_adj_batched<float, false><<<g, b, 0, stream>>>(cases, start_int, start_gen, n, gb);
    }
    return hipGetLastError();
}

}  // namespace fwh
