// Plain FP64 form (gfx950): FP64 tables, coefficients, gathers and accumulation throughout.
//
// Source stage: the recurrences of the spline prefilter (forward elimination, back substitution, and
// their transposes) run in chunks of the record, one thread per (panel, channel, chunk).  A
// recurrence started kF64H rows outside its chunk with zero is off by (2 - sqrt 3)^kF64H = 7e-18 of
// the local values at the chunk's edge, below FP64 rounding; a chunk within kF64H rows of a record
// end starts at the end and is exact.  (One thread per whole record left a 2048-panel, 512-frame
// surface with 256 waves and a serial chain of 512 rows: 420 us forward.)  A value that is not finite stays
// in a recurrence to its end, and so in every coefficient of its (panel, channel): a sweep whose
// last row is not finite sets *spoiled, and the back substitutions, only when it is set, look at the last row
// of every chunk.  The last launch of the call clears it again.
//
// Gathers: the forward one as in fwh_gather_mfma.hip (channel combine by v_mfma_f64_16x16x4f64 for a
// tile of 16 observers, taps on the vector ALU after a pass through LDS), or a thread per output for small
// surfaces; the transposed one with the observers' taps and weights from scalar registers, four indices
// per lane, no matrix product.  FP64 step, 8192 panels x 72 observers x 1024 frames: gather 7.8 -> 0.68 ms (data
// return 80 % busy, issue 47 %, half of it the products), transposed 1.6 -> 0.55 (FP64 issue 63 %, data return 71 %),
// source stage 1.5 -> 0.74 and its adjoint 1.25 -> 0.86 (data return 90 % busy; 2.7 and 3.6 GB of HBM traffic,
// most of it through the time-major scratch).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "fwh_internal.h"

namespace fwh {
namespace {

constexpr int kF64H = 30;  // warm-up rows of a chunk's recurrences

// Channel c: base quantity (0 = Q, 1..3 = L_i) and whether it is the derivative.
__device__ __forceinline__ int channel_base(int c) { return c <= 1 ? 0 : (c <= 4 ? c - 1 : c - 4); }
__device__ __forceinline__ bool channel_deriv(int c) { return c == 0 || (c >= 2 && c <= 4); }

// Source term of the given base at time-major index idx (Eqs. (Qn_New_nd), (Li_New_nd)):
//   Q = rho u.n - U0.n,  L_i = p' n_i + rho (u_i - U0_i) u.n
template <typename TIn>
struct SrcTerm {
    const TIn *rho, *u, *pp;
    int64_t P, NP;
    int base;
    double nx, ny, nz, U0n, ca, sa;
    __device__ __forceinline__ SrcTerm(const SrcFwdArgs &a, int64_t p, int b)
        : rho(static_cast<const TIn *>(a.rho) + p), u(static_cast<const TIn *>(a.u) + p),
          pp(static_cast<const TIn *>(a.pp) + p), P(a.P), NP(a.N * a.P), base(b), nx(a.normal[3 * p]),
          ny(a.normal[3 * p + 1]), nz(a.normal[3 * p + 2]), U0n(a.f.ca * nx + a.f.sa * ny), ca(a.f.ca), sa(a.f.sa) {}
    __device__ __forceinline__ double operator()(int64_t n) const {
        const int64_t i = n * P;
        const double r = (double)rho[i];
        const double u1 = (double)u[i], u2 = (double)u[NP + i], u3 = (double)u[2 * NP + i];
        const double un = u1 * nx + u2 * ny + u3 * nz;
        if (base == 0) return r * un - U0n;
        const double pv = (double)pp[i];
        if (base == 1) return pv * nx + r * (u1 - ca) * un;
        if (base == 2) return pv * ny + r * (u2 - sa) * un;
        return pv * nz + r * u3 * un;
    }
    // channel value at the first / last frame (one-sided differences for a derivative channel)
    __device__ __forceinline__ double first(bool deriv, double i2h) const {
        return deriv ? (-3.0 * (*this)(0) + 4.0 * (*this)(1) - (*this)(2)) * i2h : (*this)(0);
    }
    __device__ __forceinline__ double last(int64_t N, bool deriv, double i2h) const {
        return deriv ? (3.0 * (*this)(N - 1) - 4.0 * (*this)(N - 2) + (*this)(N - 3)) * i2h : (*this)(N - 1);
    }
};

// Block = the 4 channels of one group (a wave each) for 64 panels, rows [r0, r0 + T) of the system rows
// 1 .. N-2, r0 = 1 + z T: reduced right-hand sides d_r -> scr[channel][r][p] (time-major); returns the last
// and, of the record ends that the rows reach, the channel's values there.
template <typename TIn, int PF = 8>  // PF: rows loaded ahead
__device__ __forceinline__ double src64_sweep(const SrcFwdArgs &a, int T, int64_t z, double &f0, double &fN1) {
    const int64_t P = a.P, N = a.N;
    const int lane = threadIdx.x & 63, ch = (int)blockIdx.y * 4 + (int)(threadIdx.x >> 6);
    const bool deriv = channel_deriv(ch);
    const int64_t p = (int64_t)blockIdx.x * 64 + lane;
    const bool active = p < P;
    const SrcTerm<TIn> X(a, active ? p : P - 1, channel_base(ch));
    const double i2h = 1.0 / (2.0 * a.f.dtau);
    const int64_t r0 = 1 + z * T, r1 = min<int64_t>(N - 2, r0 + T - 1);
    const int64_t rs = max<int64_t>(1, r0 - kF64H);
    f0 = rs == 1 ? X.first(deriv, i2h) : 0.0;
    fN1 = r1 == N - 2 ? X.last(N, deriv, i2h) : 0.0;
    const double *__restrict__ cp = a.cp;
    double *scr = static_cast<double *>(a.scr) + (int64_t)ch * N * P + p;
    double Xm = X(rs - 1), Xc = X(rs), dprev = 0.0;
    for (int64_t rb = rs; rb <= r1; rb += PF) {
        double Xf[PF], pv[PF];
#pragma unroll
        for (int i = 0; i < PF; ++i) pv[i] = cp[min<int64_t>(rb + i, N - 2)];
#pragma unroll
        for (int i = 0; i < PF; ++i) Xf[i] = X(min<int64_t>(rb + i + 1, N - 1));
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const int64_t r = rb + i;
            if (r <= r1) {
                double rhs = 6.0 * (deriv ? (Xf[i] - Xm) * i2h : Xc);
                if (r == 1) rhs -= f0;
                if (r == N - 2) rhs -= fN1;
                const double d = (rhs - dprev) * pv[i];
                if (r >= r0 && active) scr[r * P] = d;
                dprev = d;
                Xm = Xc;
                Xc = Xf[i];
            }
        }
    }
    return dprev;
}

// Whether the forward sweep of some chunk of T rows met a value that is not finite (scr: the channel's
// reduced right-hand sides of one panel, [N][P])
__device__ __forceinline__ bool record_spoiled(const double *scr, int64_t P, int64_t N, int T) {
    bool bad = false;
    for (int64_t r = T; r < N - 2; r += T) bad |= !__builtin_isfinite(scr[r * P]);
    return bad | !__builtin_isfinite(scr[(N - 2) * P]);
}

// Back substitution of the storage indices [i0, i0 + T), i0 = z T (index i: coefficient c_{i-1}; past N + 1:
// zero), coefficients out panel-major with the 4 channels of a group interleaved, through LDS.  f0, fN1: the
// channel's end values, xN2: its reduced row N - 2 (where the indices reach them); x_above: 0, or NaN where the
// panel's record is spoiled.
constexpr int kB64CH = 16, kB64RS = kB64CH * 4 + 1;
__device__ __forceinline__ void src64_back(const SrcFwdArgs &a, int T, int64_t z, double f0, double fN1, double xN2,
                                           double x_above, double *stage) {
    constexpr int CH = kB64CH, RS = kB64RS;
    const int64_t P = a.P, N = a.N, NS = a.NS;
    const int lane = threadIdx.x & 63, cc = threadIdx.x >> 6, by = blockIdx.y, ch = by * 4 + cc;
    const int64_t pbase = (int64_t)blockIdx.x * 64, p = pbase + lane, pc = p < P ? p : P - 1;
    const int64_t i0 = z * T, i1 = min<int64_t>(NS, i0 + T);
    const double *__restrict__ cp = a.cp;
    const double *scr = static_cast<const double *>(a.scr) + (int64_t)ch * N * P + pc;
    double *coef = static_cast<double *>(a.coef);
    // x_r = d_r - cp_r x_{r+1} (x_{N-1} = 0) from kF64H rows above the chunk
    double x = x_above;
    constexpr int PF = 8;
    const int64_t above = i1 - 1;  // first row past the chunk's
    for (int64_t rb = min<int64_t>(N - 2, above + kF64H - 1); rb >= above; rb -= PF) {
        double d[PF], pv[PF];
#pragma unroll
        for (int q = 0; q < PF; ++q) pv[q] = cp[max<int64_t>(1, rb - q)];
#pragma unroll
        for (int q = 0; q < PF; ++q) d[q] = scr[max<int64_t>(1, rb - q) * P];
#pragma unroll
        for (int q = 0; q < PF; ++q)
            if (rb - q >= above) x = d[q] - pv[q] * x;
    }
    double d[CH], dn[CH];  // rows of this pass and of the next
    auto load = [&](int64_t ib, double (&v)[CH]) {
#pragma unroll
        for (int q = 0; q < CH; ++q) v[q] = scr[min<int64_t>(max<int64_t>(1, ib + q - 1), N - 2) * P];
    };
    if (i1 - CH <= N) load(i1 - CH, dn);
    for (int64_t ib = i1 - CH; ib >= i0; ib -= CH) {
#pragma unroll
        for (int q = 0; q < CH; ++q) d[q] = dn[q];
        if (ib > i0 && ib - CH <= N) load(ib - CH, dn);  // (indices past N + 1 have no row)
        double pv[CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) pv[q] = cp[min<int64_t>(max<int64_t>(1, ib + q - 1), N - 2)];
#pragma unroll
        for (int q = CH - 1; q >= 0; --q) {
            const int64_t i = ib + q;
            double v;
            if (i >= N + 2) v = 0.0;
            else if (i == N + 1) v = 2.0 * fN1 - xN2;
            else if (i == N) v = fN1;
            else if (i >= 2) {
                x = d[q] - pv[q] * x;
                v = x;
            } else if (i == 1) v = f0;
            else v = 2.0 * f0 - x;
            stage[lane * RS + q * 4 + cc] = v;
        }
        __syncthreads();
        for (int t = threadIdx.x; t < 64 * CH; t += 256) {
            const int r = t / CH, col = t - r * CH;
            if (pbase + r < P) {
                double *dst = coef + (((pbase + r) * 2 + by) * NS + ib + col) * 4;
                const double *src = stage + r * RS + col * 4;
                *reinterpret_cast<double2 *>(dst) = make_double2(src[0], src[1]);
                *reinterpret_cast<double2 *>(dst + 2) = make_double2(src[2], src[3]);
            }
        }
        __syncthreads();
    }
}

template <typename TIn>
__global__ __launch_bounds__(256) void src64_sweep_kernel(SrcFwdArgs a, int T, int *spoiled) {
    double f0, fN1;
    if (!__builtin_isfinite(src64_sweep<TIn>(a, T, blockIdx.z, f0, fN1))) *spoiled = 1;
}
template <typename TIn>
__global__ __launch_bounds__(256) void src64_back_kernel(SrcFwdArgs a, int T, const int *__restrict__ spoiled) {
    __shared__ double stage[64 * kB64RS];
    const int64_t P = a.P, N = a.N, i0 = (int64_t)blockIdx.z * T, i1 = min(a.NS, i0 + T);
    const int ch = (int)(blockIdx.y * 4 + (threadIdx.x >> 6));
    const int64_t p = min((int64_t)blockIdx.x * 64 + (threadIdx.x & 63), P - 1);
    const double *scr = static_cast<const double *>(a.scr) + (int64_t)ch * N * P + p;
    const double x_above = *spoiled && record_spoiled(scr, P, N, T) ? __builtin_nan("") : 0.0;
    double f0 = 0.0, fN1 = 0.0, xN2 = 0.0;
    if (i0 == 0 || i1 > N) {
        const SrcTerm<TIn> X(a, p, channel_base(ch));
        const bool deriv = channel_deriv(ch);
        const double i2h = 1.0 / (2.0 * a.f.dtau);
        if (i0 == 0) f0 = X.first(deriv, i2h);
        if (i1 > N) {
            fN1 = X.last(N, deriv, i2h);
            xN2 = scr[(N - 2) * P] + x_above;
        }
    }
    src64_back(a, T, blockIdx.z, f0, fN1, xN2, x_above, stage);
}
// Records of one chunk of 64 indices: a thread reads back the scratch that it wrote itself, one launch instead of two
// (30 panels x 35 frames 38 -> 32 us), four rows ahead rather than eight: such a call is as long as the
// fetch of its instructions (sixteen: 35 us).  With the pivots read ahead, out of the chain: 28 us.
template <typename TIn>
__global__ __launch_bounds__(256) void src64_short_kernel(SrcFwdArgs a, int T) {
    __shared__ double stage[64 * kB64RS];
    double f0, fN1;
    const double d = src64_sweep<TIn, 4>(a, T, 0, f0, fN1);
    src64_back(a, T, 0, f0, fN1, d, __builtin_isfinite(d) ? 0.0 : __builtin_nan(""), stage);
}

// ------------------------------------------------------------------ source adjoint
// Transpose of the prefilter for one (panel, channel): coefficient adjoints a_{-1..N} (storage indices
// 0 .. N+1) -> adjoints of the channel values f_0 .. f_{N-1}:
//   z = A^{-1} chat, chat_r = a_r - [r = 1] a_{-1} - [r = N-2] a_N (A = tridiag(1, 4, 1), symmetric);
//   fbar_r = 6 z_r (r = 1 .. N-2), fbar_0 = a_0 + 2 a_{-1} - z_1, fbar_{N-1} = a_{N-1} + 2 a_N - z_{N-2}.
// Forward sweep of rows [r0, r0 + T) into scr [8][N][P]; rows 0 and N-1 of scr take the end terms
// a_0 + 2 a_{-1} and a_{N-1} + 2 a_N.
__global__ __launch_bounds__(256) void adj64_sweep_kernel(PreAdjArgs a, int T, int *spoiled) {
    constexpr int CH = 16;
    __shared__ double stage[4][64][CH + 1];
    const int64_t P = a.P, N = a.N, NS = a.NS;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, ch = (int)blockIdx.y * 4 + wv;
    const int64_t pbase = (int64_t)blockIdx.x * 64, p = pbase + lane;
    const bool active = p < P;
    const double *cb = static_cast<const double *>(a.cbar) + (int64_t)ch * P * NS;
    const double *row = cb + (active ? p : P - 1) * NS;
    double *scr = static_cast<double *>(a.scr) + (int64_t)ch * N * P + p;
    const double *__restrict__ cp = a.cp;
    const int64_t r0 = 1 + (int64_t)blockIdx.z * T, r1 = min<int64_t>(N - 2, r0 + T - 1);
    const int64_t rs = max<int64_t>(1, r0 - kF64H);
    const double am1 = rs == 1 ? row[0] : 0.0, aN = r1 == N - 2 ? row[N + 1] : 0.0;
    if (r0 == 1 && active) scr[0] = row[1] + 2.0 * am1;
    if (r1 == N - 2 && active) scr[(N - 1) * P] = row[N] + 2.0 * aN;
    double dprev = 0.0;
    for (int64_t ib = (rs + 1) / CH * CH; ib <= r1 + 1; ib += CH) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int e = lane + 64 * j, r = e / CH, col = e % CH;
            stage[wv][r][col] = pbase + r < P && ib + col < NS ? cb[(pbase + r) * NS + ib + col] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int64_t r = ib + q - 1;
            if (r >= rs && r <= r1) {
                double c = stage[wv][lane][q];
                if (r == 1) c -= am1;
                if (r == N - 2) c -= aN;
                const double d = (c - dprev) * cp[r];
                if (r >= r0 && active) scr[r * P] = d;
                dprev = d;
            }
        }
    }
    if (!__builtin_isfinite(dprev)) *spoiled = 1;
}

// Back substitution of rows [r0, r0 + T): fbar time-major into out [8][N][P].
__global__ __launch_bounds__(256) void adj64_back_kernel(const double *__restrict__ scr_all, const double *__restrict__ cp,
                                                         int64_t P, int64_t N, int T, const int *__restrict__ spoiled,
                                                         double *__restrict__ out_all) {
    const int64_t p = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    if (p >= P) return;
    const int64_t ch = (int64_t)blockIdx.y * 4 + (threadIdx.x >> 6);
    const double *scr = scr_all + ch * N * P + p;
    double *out = out_all + ch * N * P + p;
    const int64_t r0 = 1 + (int64_t)blockIdx.z * T, r1 = min<int64_t>(N - 2, r0 + T - 1);
    double z = *spoiled && record_spoiled(scr, P, N, T) ? __builtin_nan("") : 0.0;
    constexpr int PF = 8;
    for (int64_t rb = min<int64_t>(N - 2, r1 + kF64H); rb >= r0; rb -= PF) {
        double d[PF];
#pragma unroll
        for (int q = 0; q < PF; ++q) d[q] = scr[max<int64_t>(1, rb - q) * P];
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const int64_t r = rb - q;
            if (r >= r0) {
                z = d[q] - cp[r] * z;
                if (r <= r1) out[r * P] = 6.0 * z;
                if (r == N - 2) out[(N - 1) * P] = scr[(N - 1) * P] - z;
            }
        }
    }
    if (r0 == 1) out[0] = scr[0] - z;
}

// Per (frame n, panel p): source-term adjoints
//   Qbar = fbar_Q + D^T fbar_Qdot,  Lbar_i = fbar_Li + D^T fbar_Ldot_i
// (D the derivative matrix: central rows 1..N-2, one-sided rows 0 and N-1), then the
// chain rule through Q = rho u.n - U0.n and L_i = p' n_i + rho (u_i - U0_i) u.n:
//   drho = u.n (Qbar + Lbar.w),  du = rho n (Qbar + Lbar.w) + rho u.n Lbar,
//   dp' = Lbar.n,  with w = u - U0.
template <typename TIn>
__global__ __launch_bounds__(256) void source_adj_chain_kernel(ChainArgs a, int *spoiled) {
    const int64_t bx = blockIdx.x, n = blockIdx.y;
    if (bx == 0 && n == 0 && threadIdx.x == 0) *spoiled = 0;
    const double *__restrict__ scr = static_cast<const double *>(a.scr);
    const TIn *__restrict__ rho = static_cast<const TIn *>(a.rho);
    const TIn *__restrict__ u = static_cast<const TIn *>(a.u);
    const double *__restrict__ normal = a.normal;
    const int64_t P = a.P, N = a.N;
    const Flow f = a.f;
    TIn *__restrict__ g_rho = static_cast<TIn *>(a.g_rho);
    TIn *__restrict__ g_u = static_cast<TIn *>(a.g_u);
    TIn *__restrict__ g_p = static_cast<TIn *>(a.g_p);
    const int64_t p = bx * 256 + threadIdx.x;
    if (p >= P) return;
    const int64_t NP = N * P;
    const double i2h = 1.0 / (2.0 * f.dtau);
    auto S = [&](int c, int64_t m) { return scr[(int64_t)c * NP + m * P + p]; };
    auto DT = [&](int c) {  // (D^T v)_n for channel c
        double s = 0.0;
        if (n - 1 >= 1 && n - 1 <= N - 2) s += S(c, n - 1);
        if (n + 1 >= 1 && n + 1 <= N - 2) s -= S(c, n + 1);
        if (n <= 2) s += (n == 0 ? -3.0 : (n == 1 ? 4.0 : -1.0)) * S(c, 0);
        if (n >= N - 3) s += (n == N - 1 ? 3.0 : (n == N - 2 ? -4.0 : 1.0)) * S(c, N - 1);
        return s * i2h;
    };
    const double Qb = S(1, n) + DT(0);
    double Lb[3];
    for (int i = 0; i < 3; ++i) Lb[i] = S(5 + i, n) + DT(2 + i);
    const double nx = normal[3 * p], ny = normal[3 * p + 1], nz = normal[3 * p + 2];
    const int64_t idx = n * P + p;
    const double r = (double)rho[idx];
    const double u1 = (double)u[idx], u2 = (double)u[NP + idx], u3 = (double)u[2 * NP + idx];
    const double un = u1 * nx + u2 * ny + u3 * nz;
    const double Lw = Lb[0] * (u1 - f.ca) + Lb[1] * (u2 - f.sa) + Lb[2] * u3;
    const double q = Qb + Lw;
    g_rho[idx] = (TIn)(un * q);
    g_u[idx] = (TIn)(r * nx * q + r * un * Lb[0]);
    g_u[NP + idx] = (TIn)(r * ny * q + r * un * Lb[1]);
    g_u[2 * NP + idx] = (TIn)(r * nz * q + r * un * Lb[2]);
    g_p[idx] = (TIn)(Lb[0] * nx + Lb[1] * ny + Lb[2] * nz);
}

// ------------------------------------------------------------------ forward gather
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) const double *const_f64_t;  // uniform loads stay scalar
typedef __attribute__((address_space(4))) const int32_t *const_i32_t;

constexpr int kY64Waves = 4;
constexpr int kY64Obs = kYTile / kY64Waves;  // observers per wave

__device__ __forceinline__ double next_lane64(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x130, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double prev_lane64(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x138, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int I, int N, typename F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<I + 1, N>(f);
    }
}

// Pair tables of the FP64 form, in tiles of kYTile observers like the FP32 ones: pair index of (tile
// t with c observers, panel p, slot s) = (t 16 P + p c + s); K64[8 pair + f], W64[4 pair + j],
// N0[pair].
__device__ __forceinline__ int64_t pair64(int64_t t, int64_t p, int64_t P, int c) { return t * kYTile * P + p * c; }

struct Gather64Args {
    const double *K64, *W64;
    const int32_t *N0, *nt;
    const double *coef;
    int64_t P, O, NS, nt_max, p_chunk;
    int YR, splits;
    double *partial;  // [splits][O][nt_max]; the output itself when splits == 1
    int *spoiled;     // the source stage's mark, cleared here
};

// 64 coefficient indices of both channel groups; lane l = 16 r + i: index 16 r + 4 (i & 3) + (i >> 2),
// which makes the four results of a lane (rows 4 j + lane / 16 of the product) consecutive indices.
struct Y64Block {
    uintx4 x[2][2];  // [group][channels 0-1, 2-3]
    static __device__ __forceinline__ int lane_offset(int lane) {
        return ((lane & 48) + 4 * (lane & 3) + ((lane >> 2) & 3)) * 32;
    }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff, int rowb) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) x[g][h] = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 16 * h, soff + g * rowb, 0);
    }
    // (register = channel, row of 16 lanes = unit) -> (register = unit, row = channel), per dword
    static __device__ __forceinline__ void transpose(unsigned &x0, unsigned &x1, unsigned &x2, unsigned &x3) {
        const auto a = __builtin_amdgcn_permlane32_swap(x0, x2, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(x1, x3, false, false);
        const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
        const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
        x0 = c[0];
        x1 = c[1];
        x2 = d[0];
        x3 = d[1];
    }
    __device__ __forceinline__ void prepare() {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                unsigned a = x[g][0][e], b = x[g][0][2 + e], c = x[g][1][e], d = x[g][1][2 + e];
                transpose(a, b, c, d);
                x[g][0][e] = a;
                x[g][0][2 + e] = b;
                x[g][1][e] = c;
                x[g][1][2 + e] = d;
            }
    }
    template <int T>
    __device__ __forceinline__ doublex4 unit(double b0, double b1) const {
        doublex4 d = {0.0, 0.0, 0.0, 0.0};
        constexpr int h = T >> 1, e = 2 * (T & 1);
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(__hiloint2double((int)x[0][h][e + 1], (int)x[0][h][e]), b0, d, 0, 0, 0);
        return __builtin_amdgcn_mfma_f64_16x16x4f64(__hiloint2double((int)x[1][h][e + 1], (int)x[1][h][e]), b1, d, 0, 0,
                                                    0);
    }
};

// As gather_y_panels of fwh_gather_mfma.hip, with kY64Waves waves of 4 observers: block b = wave of
// the four (NSUB) operand blocks every panel needs, then one further block per wave in turn.
template <int NSUB>
__device__ __forceinline__ void gather64_panels(const Gather64Args &a, int64_t t, int nobs, int64_t k0, int64_t z,
                                                double *__restrict__ Y) {
    constexpr int EB = 32;
    const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t P = a.P, O = a.O, nt_max = a.nt_max, tbase = t * kYTile;
    const int64_t pb = z * a.p_chunk, pe = pb + a.p_chunk < P ? pb + a.p_chunk : P;
    const int YR = a.YR, rowb = (int)a.NS * EB;
    const int slot = li < nobs ? li : nobs - 1;
    const int per_wave = (nobs + kY64Waves - 1) / kY64Waves, own0 = wv * per_wave;
    const int nown = max(0, min(per_wave, nobs - own0));
    double acc[kY64Obs][NSUB][2];
#pragma unroll
    for (int j = 0; j < kY64Obs; ++j)
#pragma unroll
        for (int m = 0; m < NSUB; ++m) acc[j][m][0] = acc[j][m][1] = 0.0;
    int wlo = 0, wwd = 0;  // window start and width of panel ps + lane
    auto load_win = [&](int64_t ps) {
        const int32_t *n = a.N0 + pair64(t, ps + lane < pe ? ps + lane : pe - 1, P, nobs);
        int lo = INT_MAX, hi = INT_MIN;
        for (int s = 0; s < nobs; ++s) {
            const int v = n[s];
            lo = min(lo, v);
            hi = max(hi, v);
        }
        wlo = lo;
        wwd = hi - lo;
    };
    const int voff = Y64Block::lane_offset(lane);
    const double *kp = a.K64 + (pair64(t, pb, P, nobs) + slot) * 8 + lq;
    Y64Block A, T;
    double b0 = 0.0, b1 = 0.0;
    int need = 0, soff = 0, tb = 0, lo = 0;
    __amdgpu_buffer_rsrc_t rsrc;
    auto load_panel = [&](int64_t p) {
        const int q = (int)((p - pb) & 63);
        lo = __builtin_amdgcn_readlane(wlo, q);
        need = __builtin_amdgcn_readlane(wwd, q) + kLdsLanesOut * NSUB + kLdsHalo;
        soff = (lo + (int)k0) * EB;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(reinterpret_cast<const unsigned char *>(a.coef)) + (size_t)p * 2 * (size_t)rowb,
            0, 2 * rowb, 0x00020000);
        b0 = kp[0];
        b1 = kp[4];
        kp += nobs * 8;
        if (wv < NSUB) A.load(rsrc, voff, soff + wv * 64 * EB, rowb);
        tb = NSUB + ((wv + (int)p) & (kY64Waves - 1));
        if (tb * 64 < need) T.load(rsrc, voff, soff + tb * 64 * EB, rowb);
    };
    double *ybase = Y + li * YR + 4 * lq;
    const double *yown = Y + own0 * YR + lane;
    auto units = [&](Y64Block &X, int b) {
        X.prepare();
        unroll<0, 4>([&](auto tc) {
            constexpr int U = decltype(tc)::value;
            if (b * 64 + U * 16 < need) {
                const doublex4 d = X.template unit<U>(b0, b1);
                double2 *y = reinterpret_cast<double2 *>(ybase + b * 64 + U * 16);
                y[0] = make_double2(d[0], d[1]);
                y[1] = make_double2(d[2], d[3]);
            }
        });
    };
    if (pb < pe) {
        load_win(pb);
        load_panel(pb);
    }
    for (int64_t p = pb; p < pe; ++p) {
        const int64_t pr = pair64(t, p, P, nobs) + own0;
        const const_f64_t W = (const_f64_t)(a.W64 + pr * 4);
        const const_i32_t n0 = (const_i32_t)(a.N0 + pr);
        double w[kY64Obs][4];
        int d[kY64Obs];
#pragma unroll
        for (int j = 0; j < kY64Obs; ++j)
            if (j < nown) {
#pragma unroll
                for (int q = 0; q < 4; ++q) w[j][q] = W[4 * j + q];
                d[j] = n0[j] - lo;
            }
        lds_barrier();  // every wave has read the previous panel's Y
        if (wv < NSUB) units(A, wv);
        if (tb * 64 < need) units(T, tb);
        for (int b = NSUB + kY64Waves + wv; b * 64 < need; b += kY64Waves) {
            Y64Block X;
            X.load(rsrc, voff, soff + b * 64 * EB, rowb);
            units(X, b);
        }
        if (p + 1 < pe) {
            if (((p + 1 - pb) & 63) == 0) load_win(p + 1);
            load_panel(p + 1);
        }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < kY64Obs; ++j)
            if (j < nown) {
                const double *y = yown + j * YR + d[j];
                double g[NSUB];
#pragma unroll
                for (int m = 0; m < NSUB; ++m) g[m] = y[m * kLdsLanesOut];
#pragma unroll
                for (int m = 0; m < NSUB; ++m) {
                    const double gn = next_lane64(g[m]);
                    acc[j][m][0] = fma(w[j][0], g[m], acc[j][m][0]);
                    acc[j][m][1] = fma(w[j][2], g[m], acc[j][m][1]);
                    acc[j][m][0] = fma(w[j][1], gn, acc[j][m][0]);
                    acc[j][m][1] = fma(w[j][3], gn, acc[j][m][1]);
                }
            }
    }
#pragma unroll
    for (int j = 0; j < kY64Obs; ++j)
        if (j < nown) {
            const int64_t o = tbase + own0 + j;
            double *row = a.partial + (z * O + o) * nt_max;
            const int ntl = a.nt[o];
#pragma unroll
            for (int m = 0; m < NSUB; ++m) {
                const double v = acc[j][m][0] + next_lane64(next_lane64(acc[j][m][1]));
                const int64_t k = k0 + m * kLdsLanesOut + lane;
                if (lane < kLdsLanesOut && k < nt_max) row[k] = k < ntl ? v : 0.0;
            }
        }
}

__global__ __launch_bounds__(kY64Waves * 64) __attribute__((amdgpu_waves_per_eu(3))) void gather64_kernel(
    Gather64Args a, int64_t tiles, int64_t kblocks) {
    extern __shared__ __align__(16) double ysm64[];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.spoiled = 0;
    const int64_t L = xcd_block(blockIdx.x, gridDim.x);
    const int64_t t = L % tiles, rest = L / tiles;
    const int64_t k0 = rest % kblocks * kLdsK, z = rest / kblocks, tbase = t * kYTile;
    const int nobs = rec_tile_obs(t, a.O);
    int nt_tile = 0;
    for (int j = 0; j < nobs; ++j) nt_tile = max(nt_tile, a.nt[tbase + j]);
    int nsub = (int)((nt_tile - k0 + kLdsLanesOut - 1) / kLdsLanesOut);
    nsub = __builtin_amdgcn_readfirstlane(nsub < 0 ? 0 : (nsub > kLdsSub ? kLdsSub : nsub));
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int m = nsub; m < kLdsSub; ++m)  // rows past the tile's windows
        for (int j = wv; j < nobs; j += kY64Waves) {
            const int64_t k = k0 + m * kLdsLanesOut + lane;
            if (lane < kLdsLanesOut && k < a.nt_max) a.partial[(z * a.O + tbase + j) * a.nt_max + k] = 0.0;
        }
    switch (nsub) {
        case 0: break;
        case 1: gather64_panels<1>(a, t, nobs, k0, z, ysm64); break;
        case 2: gather64_panels<2>(a, t, nobs, k0, z, ysm64); break;
        case 3: gather64_panels<3>(a, t, nobs, k0, z, ysm64); break;
        default: gather64_panels<4>(a, t, nobs, k0, z, ysm64); break;
    }
}

__global__ __launch_bounds__(256) void reduce64_kernel(const double *__restrict__ part, int splits, int64_t n,
                                                       double *__restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    double s = 0.0;
    int z = 0;
    for (; z + 8 <= splits; z += 8) {  // eight reads in flight, added in order
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = part[(int64_t)(z + j) * n + e];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; z < splits; ++z) s += part[(int64_t)z * n + e];
    out[e] = s;
}

// Windows too wide for the LDS tile, and small surfaces: one thread per (observer, sample), loop over panels.
__global__ __launch_bounds__(256) void gather64_wide_kernel(Gather64Args a, int64_t kblocks) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.spoiled = 0;
    const int64_t o = blockIdx.x / kblocks;
    const int64_t k = (blockIdx.x - o * kblocks) * blockDim.x + threadIdx.x;
    if (k >= a.nt_max) return;
    double acc = 0.0;
    if (k < a.nt[o]) {
        const int64_t t = o / kYTile;
        const int s = (int)(o - t * kYTile), nc = rec_tile_obs(t, a.O);
        // (uniform tables by scalar loads, the delay index a panel ahead: the chain per panel is one read of
        // its coefficients)
        const const_i32_t N0 = (const_i32_t)a.N0;
        int n0 = N0[pair64(t, 0, a.P, nc) + s];
        for (int64_t p = 0; p < a.P; ++p) {
            const int64_t b = pair64(t, p, a.P, nc) + s;
            const const_f64_t K = (const_f64_t)(a.K64 + b * 8), W = (const_f64_t)(a.W64 + b * 4);
            const int64_t base = (int64_t)n0 + k;
            n0 = N0[p + 1 < a.P ? b + nc : b];
            double v = 0.0;
            for (int jj = 0; jj < 4; ++jj) {
                double g = 0.0;
                for (int c = 0; c < 8; ++c) g += K[c] * a.coef[((p * 2 + (c >> 2)) * a.NS + base + jj) * 4 + (c & 3)];
                v += W[jj] * g;
            }
            acc += v;
        }
    }
    a.partial[o * a.nt_max + k] = acc;
}

// ------------------------------------------------------------------ transposed gather
//   cbar_c(p, i) = sum_o K_c(o,p) sum_j w_j(o,p) gbar(o, i - n0(o,p) - j)
struct AdjGather64Args {
    const double *K64, *W64;
    const int32_t *N0, *nt;
    const double *g;  // zero-padded copy of gbar [O][LR], sample 0 at padlo (null: gbar itself [O][nt_max])
    int64_t P, O, N, NS, LR, padlo, nib;
    double *cbar;     // [8][P][NS]
};

__global__ __launch_bounds__(256) void pad64_kernel(const double *__restrict__ gbar, const int32_t *__restrict__ nt,
                                                    int64_t O, int64_t nt_max, int64_t LR, int64_t padlo,
                                                    double *__restrict__ g) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < O * LR; i += (int64_t)gridDim.x * 256) {
        const int64_t o = i / LR, k = i - o * LR - padlo;
        g[i] = k >= 0 && k < nt[o] ? gbar[o * nt_max + k] : 0.0;
    }
}

// A wave owns panel p and kAdjIdx indices: lane l the indices ib + 4 (l - 1) .. + 3 (lane 0 only supplies
// the values below lane 1's); per observer one load of 4 shifted samples per lane, 16 FMA for the taps
// and 32 for the channels, taps and weights from scalar registers.  Consecutive waves take
// consecutive panels at the same indices (nearly the same samples).
struct __attribute__((packed, aligned(8))) F64x4 {
    double x, y, z, w;
};
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void adj_gather64_kernel(AdjGather64Args a) {
    const int64_t wave = xcd_block(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t P = a.P, O = a.O;
    if (wave >= P * a.nib) return;
    const int64_t bi = wave / P, p = wave - bi * P, ib = bi * kAdjIdx;
    const int lane = threadIdx.x & 63;
    const double *gw = a.g + a.padlo + ib - 4 + 4 * lane;
    double acc[8][4];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[c][e] = 0.0;
    const int64_t tiles = (O + kYTile - 1) / kYTile;
    for (int64_t t = 0; t < tiles; ++t) {
        const int c = rec_tile_obs(t, O);
        const int64_t b = pair64(t, p, P, c);
        const const_i32_t n0 = (const_i32_t)(a.N0 + b);
        const const_f64_t W = (const_f64_t)(a.W64 + b * 4), K = (const_f64_t)(a.K64 + b * 8);
        auto load = [&](int s) { return *reinterpret_cast<const F64x4 *>(gw + (t * kYTile + s) * a.LR - n0[s]); };
        F64x4 nx = load(0);
        for (int s = 0; s < c; ++s) {
            const F64x4 x = nx;
            if (s + 1 < c) nx = load(s + 1);
            const double w0 = W[4 * s], w1 = W[4 * s + 1], w2 = W[4 * s + 2], w3 = W[4 * s + 3];
            const double m1 = prev_lane64(x.w), m2 = prev_lane64(x.z), m3 = prev_lane64(x.y);
            double h[4];
            h[0] = fma(w3, m3, fma(w2, m2, fma(w1, m1, w0 * x.x)));
            h[1] = fma(w3, m2, fma(w2, m1, fma(w1, x.x, w0 * x.y)));
            h[2] = fma(w3, m1, fma(w2, x.x, fma(w1, x.y, w0 * x.z)));
            h[3] = fma(w3, x.x, fma(w2, x.y, fma(w1, x.z, w0 * x.w)));
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const double k = K[8 * s + ch];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[ch][e] = fma(k, h[e], acc[ch][e]);
            }
        }
    }
    const int64_t e = ib + 4 * (lane - 1);
    if (lane > 0 && e < a.NS) {
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) {
            double2 *dst = reinterpret_cast<double2 *>(a.cbar + ((int64_t)ch * P + p) * a.NS + e);
            dst[0] = make_double2(acc[ch][0], acc[ch][1]);
            dst[1] = make_double2(acc[ch][2], acc[ch][3]);
        }
    }
}

// Without room for the padded copy: one thread per (panel, index), loop over observers.
__global__ __launch_bounds__(256) void adj_gather64_plain_kernel(AdjGather64Args a, int64_t nt_max, int64_t iblocks) {
    const int64_t p = blockIdx.x / iblocks;
    const int64_t i = (blockIdx.x - p * iblocks) * blockDim.x + threadIdx.x;
    if (i >= a.NS) return;
    double acc[8];
    for (int c = 0; c < 8; ++c) acc[c] = 0.0;
    for (int64_t o = 0; o < a.O; ++o) {
        const int64_t t = o / kYTile;
        const int s = (int)(o - t * kYTile), nc = rec_tile_obs(t, a.O);
        const int64_t b = pair64(t, p, a.P, nc);
        const int64_t kb = i - (int64_t)a.N0[b + s], ntl = a.nt[o];
        double h = 0.0;
        for (int jj = 0; jj < 4; ++jj) {
            const int64_t k = kb - jj;
            if (k >= 0 && k < ntl) h += a.W64[(b + s) * 4 + jj] * a.g[o * nt_max + k];
        }
        for (int c = 0; c < 8; ++c) acc[c] += a.K64[(b + s) * 8 + c] * h;
    }
    for (int c = 0; c < 8; ++c) a.cbar[((int64_t)c * a.P + p) * a.NS + i] = acc[c];
}

// frames per chunk of the recurrences: shorter chunks (more of them, more warm-up) where longer
// ones would leave the chip idle (2 channel groups x P / 64 blocks of 4 waves per chunk)
int chunk_frames(int64_t P, int64_t N) {
    int T = 64;
    for (int t = 128; t <= 1024; t *= 2)
        if ((P + 63) / 64 * 2 * ((N + t - 1) / t) >= (t == 128 ? 1024 : 1900)) T = t;
    return T;
}

}  // namespace

// Whether the tiled gather, in `splits` panel ranges of `blocks` blocks each (`resident` fit the device at once), is
// the faster one.  Times in us as measured: the plain form's loop takes 0.6 per panel (windows below 128
// samples, else 0.8), or 0.6 ns per wave of 64 samples where these fill the device; a range of the
// tiled one 1.3 per panel, and 8 to start, 4 more to add the ranges.  Forward gather, us, plain / tiled: 24
// panels x 8 observers x 250 frames 21 / 41, 64 x 30 x 20 29 / 30, 140 x 8 x 250 104 / 35, 384 x 2000 x 20 390 /
// 602, 384 x 2000 x 100 786 / 659.
bool gather64_tiles_better(int64_t P, int64_t O, int64_t nt_max, int64_t blocks, int64_t splits, int64_t resident) {
    const double waves = (double)O * (double)((nt_max + 63) / 64), fill = (double)(blocks * splits) / (double)resident;
    const double plain = (double)P * std::max(nt_max < 128 ? 0.6 : 0.8, 6e-4 * waves);
    const double tiled = 8.0 + (splits > 1 ? 4.0 : 0.0) + 1.3 * (double)((P + splits - 1) / splits) * std::max(1.0, fill);
    return tiled < plain;
}

int gather64_y_row(int w16) { return ((w16 + kLdsK + kLdsHalo + 15) / 16) * 16 + 4; }
bool gather64_tiled(int w16) { return (size_t)kYTile * gather64_y_row(w16) * sizeof(double) <= kYShmemMax; }

int gather64_blocks_per_cu(int w16) {
    if (!gather64_tiled(w16)) return 0;
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, reinterpret_cast<const void *>(&gather64_kernel), kY64Waves * 64,
        (size_t)kYTile * gather64_y_row(w16) * sizeof(double));
    return e == hipSuccess && n > 0 ? n : 1;
}

hipError_t launch_source64(int in_dtype, const void *rho, const void *u, const void *pp, const double *normal, int64_t P,
                           int64_t N, int64_t NS, Flow f, const double *cp, void *scratch, int *spoiled, void *coef,
                           hipStream_t stream) {
    const SrcFwdArgs a{rho, u, pp, normal, P, N, NS, f, cp, scratch, coef};
    const int T = chunk_frames(P, N);
    const unsigned pb = (unsigned)((P + 63) / 64);
    const dim3 g1(pb, 2, (unsigned)((N - 2 + T - 1) / T)), g2(pb, 2, (unsigned)((NS + T - 1) / T)), b(256);
    if (NS <= 64) {
        if (in_dtype == 0) src64_short_kernel<double><<<dim3(pb, 2), b, 0, stream>>>(a, T);
        else src64_short_kernel<float><<<dim3(pb, 2), b, 0, stream>>>(a, T);
        return hipGetLastError();
    }
    if (in_dtype == 0) src64_sweep_kernel<double><<<g1, b, 0, stream>>>(a, T, spoiled);
    else src64_sweep_kernel<float><<<g1, b, 0, stream>>>(a, T, spoiled);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (in_dtype == 0) src64_back_kernel<double><<<g2, b, 0, stream>>>(a, T, spoiled);
    else src64_back_kernel<float><<<g2, b, 0, stream>>>(a, T, spoiled);
    return hipGetLastError();
}

hipError_t launch_source_adjoint64(int in_dtype, void *cbar, const void *rho, const void *u, const double *normal,
                                   int64_t P, int64_t N, int64_t NS, Flow f, const double *cp, void *scratch, int *spoiled,
                                   void *g_rho, void *g_u, void *g_p, hipStream_t stream) {
    const PreAdjArgs pa{cbar, P, N, NS, cp, scratch};
    const int T = chunk_frames(P, N);
    const dim3 g((unsigned)((P + 63) / 64), 2, (unsigned)((N - 2 + T - 1) / T)), b(256);
    adj64_sweep_kernel<<<g, b, 0, stream>>>(pa, T, spoiled);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // fbar [8][N][P] takes the place of the coefficient adjoints (NS >= N), which the sweep has read
    adj64_back_kernel<<<g, b, 0, stream>>>(static_cast<const double *>(scratch), cp, P, N, T, spoiled,
                                          static_cast<double *>(cbar));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const ChainArgs ca{cbar, rho, u, normal, P, N, f, g_rho, g_u, g_p};
    const dim3 gc((unsigned)((P + 255) / 256), (unsigned)N);
    if (in_dtype == 0) source_adj_chain_kernel<double><<<gc, b, 0, stream>>>(ca, spoiled);
    else source_adj_chain_kernel<float><<<gc, b, 0, stream>>>(ca, spoiled);
    return hipGetLastError();
}

hipError_t launch_gather64(const double *K64, const double *W64, const int32_t *N0, const int32_t *nt,
                           const double *coef, int64_t P, int64_t O, int64_t NS, int64_t nt_max, bool tiled, int w16,
                           int splits, double *partial, int *spoiled, double *out, hipStream_t stream) {
    if (!tiled) splits = 1;
    const int64_t p_chunk = (P + splits - 1) / splits;
    const Gather64Args a{K64, W64, N0, nt, coef, P, O, NS, nt_max, p_chunk, gather64_y_row(w16), splits,
                         splits == 1 ? out : partial, spoiled};
    if (!tiled) {
        const int64_t kb = (nt_max + 255) / 256;
        gather64_wide_kernel<<<dim3((unsigned)(kb * O)), dim3(256), 0, stream>>>(a, kb);
        return hipGetLastError();
    }
    const int64_t tiles = (O + kYTile - 1) / kYTile, kblocks = (nt_max + kLdsK - 1) / kLdsK;
    gather64_kernel<<<dim3((unsigned)(tiles * kblocks * splits)), dim3(kY64Waves * 64),
                      (size_t)kYTile * a.YR * sizeof(double), stream>>>(a, tiles, kblocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    const int64_t n = O * nt_max;
    reduce64_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(partial, splits, n, out);
    return hipGetLastError();
}

hipError_t launch_adj_gather64(const double *K64, const double *W64, const int32_t *N0, const int32_t *nt,
                               const double *gbar, int64_t P, int64_t O, int64_t N, int64_t NS, int64_t nt_max,
                               double *pad, size_t pad_bytes, double *cbar, hipStream_t stream) {
    const int64_t LR = adj_pad_row(N, NS), padlo = adj_pad_lo(N), nib = (N + 2 + kAdjIdx - 1) / kAdjIdx;
    if ((size_t)O * LR * sizeof(double) > pad_bytes) {
        const AdjGather64Args a{K64, W64, N0, nt, gbar, P, O, N, NS, LR, padlo, nib, cbar};
        const int64_t ibl = (NS + 255) / 256;
        adj_gather64_plain_kernel<<<dim3((unsigned)(ibl * P)), dim3(256), 0, stream>>>(a, nt_max, ibl);
        return hipGetLastError();
    }
    // (a launch holds fewer than 2^32 threads, a copy of 34 GB or more has as many elements)
    const unsigned pad_blocks = (unsigned)std::min<int64_t>((O * LR + 255) / 256, (int64_t)1 << 23);
    pad64_kernel<<<dim3(pad_blocks), dim3(256), 0, stream>>>(gbar, nt, O, nt_max, LR, padlo, pad);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const AdjGather64Args a{K64, W64, N0, nt, pad, P, O, N, NS, LR, padlo, nib, cbar};
    adj_gather64_kernel<<<dim3((unsigned)((P * nib + 3) / 4)), dim3(256), 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace fwh
