// Setup kernels: per-pair delay, per-observer delay extremes, and the per-pair
// tables of the fixed fractional-delay gather (gfx950).
//
// Geometry follows Sec. II C: Garrick distance with the AoA rotation,
// Eqs. (R_New), (R_s_New), (M1), (M2); radiation direction Eqs. (d1_prime)..(R2_New);
// surface Mach vector M = -M0 U0hat (the surface moves against the mean flow in
// the frame where the medium is at rest), M_R = M . Rhat; delay R/c0 = M0 R,
// Eq. (tau2) with c0 = 1/M0 (Sec. II D).  Everything here is FP64.
#include "fwh_internal.h"

namespace fwh {
namespace {

constexpr double kPi = 3.14159265358979323846;

// FP64 pair geometry, evaluated without contraction so that the delay is the
// correctly rounded result of each printed operation in order.
__device__ __forceinline__ void pair_geometry(const double *x, const double *y, const Flow &f, double &R, double Rh[3],
                                              double &MR) {
#pragma clang fp contract(off)
    const double M1 = f.M0 * f.ca, M2 = f.M0 * f.sa;
    const double d1 = x[0] - y[0], d2 = x[1] - y[1], d3 = x[2] - y[2];
    const double md = M1 * d1 + M2 * d2;
    const double Rs = sqrt(md * md + f.beta2 * (d1 * d1 + d2 * d2 + d3 * d3));
    R = (-M1 * d1 - M2 * d2 + Rs) / f.beta2;
    const double d1p = d1 * f.ca + d2 * f.sa;
    const double d2p = -d1 * f.sa + d2 * f.ca;
    const double R1p = (-f.M0 * Rs + d1p) / (f.beta2 * R);
    const double R2p = d2p / R;
    Rh[0] = R1p * f.ca - R2p * f.sa;
    Rh[1] = R1p * f.sa + R2p * f.ca;
    Rh[2] = d3 / R;
    MR = (-f.M0 * f.ca) * Rh[0] + (-f.M0 * f.sa) * Rh[1];
}

__global__ __launch_bounds__(256) void delay_kernel(const double *__restrict__ y, const double *__restrict__ x_obs,
                                                    int64_t P, int64_t O, Flow f, double *__restrict__ D,
                                                    int *__restrict__ zeroed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0 && zeroed) *zeroed = 0;
    if (i >= P * O) return;
    const int64_t o = i / P, p = i - o * P;
    double R, Rh[3], MR;
    pair_geometry(x_obs + 3 * o, y + 3 * p, f, R, Rh, MR);
    D[i] = f.M0 * R;
}

// Per observer: max and min delay over panels (the paper's per-observer R_max,
// R_min of Eqs. (t_start), (t_end)).
__global__ __launch_bounds__(256) void minmax_kernel(const double *__restrict__ D, int64_t P,
                                                     double *__restrict__ dmm) {
    const int64_t o = blockIdx.x;
    double mx = -HUGE_VAL, mn = HUGE_VAL;
    for (int64_t p = threadIdx.x; p < P; p += blockDim.x) {
        const double d = D[o * P + p];
        mx = fmax(mx, d);
        mn = fmin(mn, d);
    }
    __shared__ double smx[256], smn[256];
    smx[threadIdx.x] = mx;
    smn[threadIdx.x] = mn;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            smx[threadIdx.x] = fmax(smx[threadIdx.x], smx[threadIdx.x + s]);
            smn[threadIdx.x] = fmin(smn[threadIdx.x], smn[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        dmm[2 * o] = smx[0];
        dmm[2 * o + 1] = smn[0];
    }
}

// Fractional delay index s0 >= 0 of a pair and its integer part, kept below N - nt so that the window's last
// sample stays in the record (holds by construction)
__device__ __forceinline__ double delay_index(double ts, double D, const Flow &f, double n_max, double &s0) {
    s0 = (ts - D - f.tau0) / f.dtau;
    if (!(s0 > 0.0)) s0 = 0.0;
    const double nf = floor(s0);
    return nf > n_max ? n_max : nf;
}

// Widest spread of n0 over the observers of a 16-observer tile (any panel) -> *width (zero before), from
// the delays and their extremes alone, so that the host reads it with the extremes and the tables are
// written while it goes on.  Thread = a panel, block = 256 panels of a tile: the 16 loads of a thread are in
// flight together, and one atomic per block (they all go to one word and queue).  8192 panels x 72
// observers 4.9 us; a pair per thread, 16 panels per block, 19.7 us.
__global__ __launch_bounds__(256) void spread_kernel(const double *__restrict__ D, const double *__restrict__ dmm,
                                                     int64_t P, int64_t O, int64_t N, Flow f, int64_t pblocks,
                                                     int *__restrict__ width) {
    __shared__ double start[kYTile], n_max[kYTile];
    __shared__ int sw[4];
    const int tid = threadIdx.x;
    const int64_t t = blockIdx.x / pblocks, p = (blockIdx.x - t * pblocks) * 256 + tid;
    const int c = rec_tile_obs(t, O);
    const double *Dt = D + t * kYTile * P + (p < P ? p : P - 1);
    double d[kYTile];
#pragma unroll
    for (int s = 0; s < kYTile; ++s) d[s] = Dt[(s < c ? s : c - 1) * P];
    if (tid < kYTile) {
        const int64_t o = t * kYTile + (tid < c ? tid : c - 1);
        double ts, te;
        n_max[tid] = (double)N - obs_window(dmm[2 * o], dmm[2 * o + 1], f.tau0, f.dtau, N, ts, te);
        start[tid] = ts;
    }
    __syncthreads();
    double lo = HUGE_VAL, hi = -HUGE_VAL, s0;
#pragma unroll
    for (int s = 0; s < kYTile; ++s) {
        const double n0 = delay_index(start[s], d[s], f, n_max[s], s0);
        lo = fmin(lo, n0);
        hi = fmax(hi, n0);
    }
    int w = (int)fmin(hi - lo, (double)N);  // (beyond N: an empty window, which the host refuses)
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) w = max(w, __shfl_xor(w, m));
    if ((tid & 63) == 0) sw[tid >> 6] = w;
    __syncthreads();
    if (tid == 0) atomicMax(width, max(max(sw[0], sw[1]), max(sw[2], sw[3])));
}

// Per pair: fractional delay index s0 = (t_start - delay - tau0)/dtau of observer
// sample k = 0 (sample k sits at s0 + k), its integer part n0 and the uniform
// cubic B-spline taps of frac = s0 - n0 acting on coefficients c[n0-1..n0+2];
// and the weights of the 8 source channels in the integrand of
// Eqs. (pT_WT_nd) + (pL_WT_nd), dS/(4 pi) included:
//   Qdot:   1/(R om^2)                 Q:   (M_R - M0^2)/(M0 R^2 om^3)
//   Ldot_i: M0 Rhat_i/(R om^2)         L_i: (Rhat_i - M_i)/(R^2 om^2) + Rhat_i (M_R - M0^2)/(R^2 om^3)
// with om = 1 - M_R (the L_M term is L . M, Eq. (LM)).  With rbf (BF16 mode)
// the weights are also stored split into bfloat16 high and low parts.
struct PairTab {
    double K[8], w[4];
    int32_t n0;
};

__device__ __forceinline__ PairTab pair_tables(const double *__restrict__ y, const double *__restrict__ dS,
                                               const double *__restrict__ x_obs, const double *__restrict__ t_start,
                                               const int32_t *__restrict__ nt, int64_t N, const Flow &f, int64_t o,
                                               int64_t p) {
    PairTab pt;
    double R, Rh[3], MR;
    pair_geometry(x_obs + 3 * o, y + 3 * p, f, R, Rh, MR);
    double D;
    {
#pragma clang fp contract(off)
        D = f.M0 * R;
    }
    double s0;
    const double nf = delay_index(t_start[o], D, f, (double)(N - nt[o]), s0);
    double t = s0 - nf;
    if (t > 1.0) t = 1.0;
    pt.n0 = (int32_t)nf;
    const double u = 1.0 - t;
    pt.w[0] = u * u * u / 6.0;
    pt.w[1] = (3.0 * t * t * t - 6.0 * t * t + 4.0) / 6.0;
    pt.w[2] = (-3.0 * t * t * t + 3.0 * t * t + 3.0 * t + 1.0) / 6.0;
    pt.w[3] = t * t * t / 6.0;

    const double M0 = f.M0, M2 = f.M0 * f.M0;
    const double Mv[3] = {-M0 * f.ca, -M0 * f.sa, 0.0};
    const double om = 1.0 - MR, om2 = om * om, om3 = om2 * om;
    const double ws = dS[p] / (4.0 * kPi);
    pt.K[0] = ws / (R * om2);
    pt.K[1] = ws * (MR - M2) / (M0 * R * R * om3);
    for (int c = 0; c < 3; ++c) {
        pt.K[2 + c] = ws * M0 * Rh[c] / (R * om2);
        pt.K[5 + c] = ws * ((Rh[c] - Mv[c]) / (R * R * om2) + Rh[c] * (MR - M2) / (R * R * om3));
    }
    return pt;
}

// plain FP64 form: the tables as FP64 arrays in tiles of kYTile observers (layout in fwh_f64.hip), a pair per
// thread, observer slots fastest; written through LDS, so that the stores of a wave are consecutive
__global__ __launch_bounds__(256) void tables_f64_kernel(const double *__restrict__ y, const double *__restrict__ dS,
                                                         const double *__restrict__ x_obs,
                                                         const double *__restrict__ t_start,
                                                         const int32_t *__restrict__ nt, int64_t P, int64_t O,
                                                         int64_t N, Flow f, double *__restrict__ K64,
                                                         double *__restrict__ W64, int32_t *__restrict__ N0,
                                                         int *__restrict__ spoiled) {
    __shared__ double sk[256 * 9], sw[256 * 5];
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + threadIdx.x;  // pair index: tile, panel, slot
    if (i == 0) *spoiled = 0;
    if (i < P * O) {
        const int64_t t = i / (kYTile * P);
        const int c = rec_tile_obs(t, O);
        const int64_t e = i - t * kYTile * P, p = e / c;
        const int s = (int)(e - p * c);
        const PairTab pt = pair_tables(y, dS, x_obs, t_start, nt, N, f, t * kYTile + s, p);
        for (int f8 = 0; f8 < 8; ++f8) sk[threadIdx.x * 9 + f8] = pt.K[f8];
        for (int j = 0; j < 4; ++j) sw[threadIdx.x * 5 + j] = pt.w[j];
        N0[i] = pt.n0;
    }
    __syncthreads();
    const int np = (int)min<int64_t>(256, P * O - i0);
    for (int q = threadIdx.x; q < np * 8; q += 256) K64[i0 * 8 + q] = sk[(q >> 3) * 9 + (q & 7)];
    for (int q = threadIdx.x; q < np * 4; q += 256) W64[i0 * 4 + q] = sw[(q >> 2) * 5 + (q & 3)];
}

// FP32/BF16 forms: block = two observer tiles (kObsTile = 2 kYTile observers) x kTabPanels panels; thread
// (observer slot j, panel q) computes the pair's tables.  Their FP64 arithmetic is what bounds it, so
// the pairs of the slots that exist are packed into the first waves: 1 and 8 observers x 32768 panels 14 us,
// 22 with 32 lanes to a panel whatever the number of slots.  The block reduces n0 over the observers
// per panel: tw[t][p] = (lo, hi) = (min n0, max n0), and wblk[block] = the widest window of the
// block's panels over the 32 observers, and over its 16-observer tiles in the high 16 bits (blocks
// t * bpt .. t * bpt + bpt - 1 belong to 32-observer tile t, bpt = ceil(P / kTabPanels)).  The pair
// tables leave through LDS: a tile's blocks of the kTabPanels panels are one contiguous piece of
// memory (16 c dwords per panel), written by consecutive lanes.
constexpr int kTabPanels = 256 / kObsTile;
static_assert(kObsTile == 2 * kYTile, "the table kernel handles two 16-observer tiles");
__global__ __launch_bounds__(256) void tables_tile_kernel(const double *__restrict__ y, const double *__restrict__ dS,
                                                          const double *__restrict__ x_obs,
                                                          const double *__restrict__ t_start,
                                                          const int32_t *__restrict__ nt, int64_t P, int64_t O,
                                                          int64_t N, Flow f, int64_t bpt, PairRec *__restrict__ rec,
                                                          PairBf *__restrict__ rbf, int2 *__restrict__ tw,
                                                          int32_t *__restrict__ wblk) {
    const int64_t t = blockIdx.x / bpt;
    const int64_t nobs = O - t * kObsTile < kObsTile ? O - t * kObsTile : kObsTile;
    const int q = (int)(threadIdx.x / (unsigned)nobs), j = (int)threadIdx.x - q * (int)nobs;
    const int64_t p0 = (blockIdx.x - t * bpt) * kTabPanels;
    const int64_t o = t * kObsTile + j, p = p0 + q;
    const int h = j / kYTile, s = j % kYTile;  // 16-observer tile 2 t + h, slot s
    __shared__ int sn0[kTabPanels][kObsTile + 1];
    __shared__ int slo[kTabPanels], slo16[2][kTabPanels], sw16[2][kTabPanels];
    __shared__ int sw[kTabPanels];
    __shared__ uint32_t out[2][kTabPanels * kYTile * 16];
    const int np = (int)(P - p0 < kTabPanels ? P - p0 : kTabPanels);
    const int c0 = (int)(nobs < kYTile ? nobs : kYTile), c1 = (int)nobs - c0;
    const int c = h == 0 ? c0 : c1;
    const bool valid = q < kTabPanels && p < P;
    PairTab pt;
    if (valid) pt = pair_tables(y, dS, x_obs, t_start, nt, N, f, o, p);
    if (valid) sn0[q][j] = pt.n0;
    __syncthreads();
    if (threadIdx.x < kTabPanels) {
        const int qq = threadIdx.x;
        int lo = INT_MAX, hi = INT_MIN, w16 = 0;
        for (int hh = 0; hh < 2; ++hh) {
            int l = INT_MAX, u = INT_MIN;
            for (int jj = hh * kYTile; jj < (hh + 1) * kYTile && jj < nobs; ++jj) {
                l = sn0[qq][jj] < l ? sn0[qq][jj] : l;
                u = sn0[qq][jj] > u ? sn0[qq][jj] : u;
            }
            const int w = l <= u ? u - l : 0;
            slo16[hh][qq] = l;
            sw16[hh][qq] = w;
            w16 = w > w16 ? w : w16;
            lo = l < lo ? l : lo;
            hi = u > hi ? u : hi;
        }
        int width = 0;
        if (p0 + qq < P) {
            tw[t * P + p0 + qq] = make_int2(lo, hi);
            width = (hi - lo) | (w16 << 16);
        }
        sw[qq] = width;
        slo[qq] = lo;
    }
    __syncthreads();
    if (valid) {
        uint32_t *blk = out[h] + q * 16 * c;
        for (int cc = 0; cc < 8; ++cc) blk[rec_dword(cc, s, c)] = __float_as_uint((float)pt.K[cc]);
        for (int jj = 0; jj < 4; ++jj) blk[kRecW * c + 4 * s + jj] = __float_as_uint((float)pt.w[jj]);
        blk[kRecN0 * c + s] = (uint32_t)pt.n0;
        blk[kRecN0w * c + s] = (uint32_t)((pt.n0 - slo[q]) * (rbf ? 8 : 16));
        blk[kRecD16 * c + s] = (uint32_t)(pt.n0 - slo16[h][q]);
        blk[kRecW16 * c + s] = (uint32_t)sw16[h][q];
    }
    __syncthreads();
    for (int hh = 0; hh < 2; ++hh) {
        const int cc = hh == 0 ? c0 : c1;
        const int n16 = np * cc * 4;  // 16-byte pieces
        uint4 *dst = reinterpret_cast<uint4 *>(rec + (2 * t + hh) * kYTile * P + p0 * cc);
        for (int u = threadIdx.x; u < n16; u += 256) dst[u] = reinterpret_cast<const uint4 *>(out[hh])[u];
    }
    if (rbf) {
        __syncthreads();
        if (valid) {
            // bfloat16 by round-to-nearest-even of the FP32 value (weights are finite)
            auto bf16 = [](double v) {
                const uint32_t b = __float_as_uint((float)v);
                return (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;
            };
            uint32_t *blk = out[h] + q * 8 * c;
            for (int cc = 0; cc < 4; ++cc) {
                uint32_t hb[2], lb[2];
                for (int e = 0; e < 2; ++e) {
                    hb[e] = bf16(pt.K[2 * cc + e]);
                    lb[e] = bf16(pt.K[2 * cc + e] - (double)__uint_as_float(hb[e] << 16));
                }
                blk[8 * s + cc] = hb[0] | (hb[1] << 16);
                blk[8 * s + 4 + cc] = lb[0] | (lb[1] << 16);
            }
        }
        __syncthreads();
        for (int hh = 0; hh < 2; ++hh) {
            const int cc = hh == 0 ? c0 : c1;
            const int n16 = np * cc * 2;
            uint4 *dst = reinterpret_cast<uint4 *>(rbf + (2 * t + hh) * kYTile * P + p0 * cc);
            for (int u = threadIdx.x; u < n16; u += 256) dst[u] = reinterpret_cast<const uint4 *>(out[hh])[u];
        }
    }
    if (threadIdx.x == 0) {
        unsigned m = 0, m16 = 0;
        for (int qq = 0; qq < kTabPanels; ++qq) {
            const unsigned w = (unsigned)sw[qq];
            m = (w & 0xffffu) > m ? w & 0xffffu : m;
            m16 = (w >> 16) > m16 ? w >> 16 : m16;
        }
        wblk[blockIdx.x] = (int32_t)(m | (m16 << 16));
    }
}

}  // namespace

hipError_t launch_delay(const double *y, const double *x_obs, int64_t P, int64_t O, Flow f, double *D, int *zeroed,
                        hipStream_t stream) {
    const int64_t n = P * O;
    delay_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(y, x_obs, P, O, f, D, zeroed);
    return hipGetLastError();
}

hipError_t launch_spread(const double *D, const double *dmm, int64_t P, int64_t O, int64_t N, Flow f, int *width,
                         hipStream_t stream) {
    const int64_t tiles = (O + kYTile - 1) / kYTile, pblocks = (P + 255) / 256;
    spread_kernel<<<dim3((unsigned)(tiles * pblocks)), dim3(256), 0, stream>>>(D, dmm, P, O, N, f, pblocks, width);
    return hipGetLastError();
}

hipError_t launch_minmax(const double *D, int64_t P, int64_t O, double *dmm, hipStream_t stream) {
    minmax_kernel<<<dim3((unsigned)O), dim3(256), 0, stream>>>(D, P, dmm);
    return hipGetLastError();
}

hipError_t launch_tables(int mode, const double *y, const double *dS, const double *x_obs, const double *t_start,
                         const int32_t *nt, int64_t P, int64_t O, int64_t N, Flow f, double *K64, double *W64,
                         int32_t *N0, int *spoiled, PairRec *rec_op, PairBf *rbf, int2 *tw, int32_t *wblk, hipStream_t stream) {
    if (mode == 0) {
        const int64_t n = P * O;
        tables_f64_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(y, dS, x_obs, t_start, nt, P,
                                                                                        O, N, f, K64, W64, N0,
                                                                                        spoiled);
    } else {
        tables_tile_kernel<<<dim3((unsigned)tile_window_blocks(P, O)), dim3(256), 0, stream>>>(
            y, dS, x_obs, t_start, nt, P, O, N, f, (P + kTabPanels - 1) / kTabPanels, rec_op, rbf, tw, wblk);
    }
    return hipGetLastError();
}

}  // namespace fwh
