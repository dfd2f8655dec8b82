// Initial data, status reset, diagnostics and mode projection kernels for the
// AdS4 scalar-collapse library (Liebling & Khanna, arXiv:1706.07413, Sec. II).
#include <math.h>

#include <algorithm>

#include "stage.h"

namespace adscl {
namespace {

// Pi(x,0) = (2 eps/pi) exp(-4 tan^2 x/(pi^2 sigma^2)), Phi(x,0) = 0 (Sec. II:
// data Phi, Pi given at t = 0); Pi = 0 at x = pi/2 (Eq. (10)).
__global__ void init_gaussian_kernel(int n_inst, const InstConst* ic, const double* eps, const double* sigma,
                                     double* Phi, double* Pi)
{
    const int b = blockIdx.y;
    if (b >= n_inst) return;
    const InstConst c = ic[b];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < c.N; i += gridDim.x * blockDim.x) {
        const double x = (double)i * c.h;
        const double t = tan(x);
        const double s = sigma[b];
        double v = (2.0 * eps[b] / kPi) * exp(-4.0 * t * t / (kPi * kPi * s * s));
        if (i == c.N - 1) v = 0.0;
        Phi[c.off + i] = 0.0;
        Pi[c.off + i] = v;
    }
}

// Pi(x,0) = eps sum_{j<Jc} c_j e_j(x), Phi(x,0) = 0.
__global__ void init_modes_kernel(int n_inst, const InstConst* ic, const double* eps, const double* c, int Jc,
                                  const double* const* emode, double* Phi, double* Pi)
{
    const int b = blockIdx.y;
    if (b >= n_inst) return;
    const InstConst k = ic[b];
    const double* e = emode[b];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k.N; i += gridDim.x * blockDim.x) {
        double sum = 0.0;
        for (int j = 0; j < Jc; ++j) sum += c[(size_t)b * Jc + j] * e[(size_t)j * k.N + i];
        Phi[k.off + i] = 0.0;
        Pi[k.off + i] = (i == k.N - 1) ? 0.0 : eps[b] * sum;
    }
}

// Phi(0) = 0, Phi(pi/2) = Pi(pi/2) = 0 (Eqs. (7), (9), (10)).
__global__ void pins_kernel(int n_inst, const InstConst* ic, double* Phi, double* Pi)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst) return;
    const InstConst c = ic[b];
    Phi[c.off] = 0.0;
    Phi[c.off + c.N - 1] = 0.0;
    Pi[c.off + c.N - 1] = 0.0;
}

__global__ void reset_status_kernel(int n_inst, InstStatus* st)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst) return;
    InstStatus o;
    o.steps = 0;
    o.target = 0;
    o.t_c = -1.0;
    o.minA = 1.0;
    o.mass = 0.0;
    o.state = ST_RUNNING;
    o.pad = 0;
    st[b] = o;
}

__global__ void set_targets_kernel(int n_inst, const InstConst* ic, InstStatus* st, int64_t max_steps)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst) return;
    InstStatus o = st[b];
    int64_t t = o.steps + max_steps;
    if (t > ic[b].n_final) t = ic[b].n_final;
    if (t < o.steps) t = o.steps;
    o.target = t;
    st[b] = o;
}

// Block-wide exclusive prefix sum of one value per thread (up to 1024 threads) and
// its total; contains one barrier.  `sh`: 16 doubles that no wavefront still reads
// from an earlier call (callers alternate between two).
__device__ __forceinline__ double block_scan(double v, double* sh, double& total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const double x = wave_incl_scan(v);
    if (lane == 63) sh[wv] = x;
    __syncthreads();
    double w = (lane < nw) ? sh[lane < nw ? lane : 0] : 0.0;
    w += dpp_d<0x111, 0xf>(w);  // at most 16 wavefronts: a prefix over one row of lanes
    w += dpp_d<0x112, 0xf>(w);
    w += dpp_d<0x114, 0xf>(w);
    w += dpp_d<0x118, 0xf>(w);
    total = readlane_d(w, 15);
    const int u = __builtin_amdgcn_readfirstlane(wv);
    // the lanes before: the left lane's sum, not this one's less v, which would lose
    // the small sums near x = 0 next to a far larger v
    return (u > 0 ? readlane_d(w, u > 0 ? u - 1 : 0) : 0.0) + dpp_d<0x138, 0xf>(x);
}

struct FinArgs {
    const InstConst* ic;
    InstStatus* st;
    const double* const* nat;  // tables in grid order per instance (kNat*)
    double* state5;
    int64_t total;
    double a_collapse;
    double* snaps;
    int32_t snap_every;
    int32_t n_slots;
    int32_t gauge;
    int32_t frozen;
    int32_t final_;
    int32_t a_reint;  // > 0: A is evolved; the state's A is kept unless steps % a_reint == 0
};

constexpr int kFinK = 4;  // consecutive points per thread

// Constraint solve of the packed state of one instance per block (Sec. II,
// Eqs. (5)-(6), the same discretisation as the evolution kernel: 4-point cell rule
// in prefix-sum form, m = (1 - A) sin x / cos^3 x), written out as (Phi, Pi, A,
// delta, m); then min A, the mass m(pi/2) and, at the end of a call, the collapse /
// non-finite test of the final state.  With A evolved (a_reint > 0) the state's A
// is kept (and tested) except at steps that are a multiple of a_reint, where the
// solve's A replaces it as the evolution would.
//
// The interior points 1 .. N-2 go in tiles of four consecutive ones per thread; the
// running sums carry over the tiles.  The first pass takes the total of p (the
// boundary gauge's shift enters every exponential), the second the two prefix sums
// side by side.  A thread forms p and sigma at its neighbours' adjacent points
// itself (two more exponentials for its four) instead of exchanging them, so that
// two scans are a tile's only barriers; the coefficients come from tables in grid
// order.  The order of every sum is that of threads of four points, whatever the
// block's size (which follows the batch's largest grid), so that an instance's
// results do not hang on the batch it is in.
// Bound by the latency of those scans and of the loads: one instance of 513, 1025,
// 16385 and 32769 points 9.1, 9.9, 54 and 92 us, against 18, 28, 342 and 608 with
// 256 threads, a run of N/256 points each, and sin, cos, tan and three exponentials
// per point; 64 instances of 4097 points 19 against 90, a batch of 1024 (1025 to
// 4097 points) 62 against 457.
__global__ void __launch_bounds__(1024) finalize_kernel(FinArgs f)
{
    __shared__ double sh[3][16];
    __shared__ int ish[16];
    const int b = blockIdx.x;
    const InstStatus st = f.st[b];
    const InstConst c = f.ic[b];
    const bool snap = f.snaps && f.snap_every > 0 && (st.steps % f.snap_every) == 0 &&
                      (st.steps / f.snap_every) < f.n_slots;
    if (!snap && !f.final_) return;
    constexpr int K = kFinK;
    const int N = c.N, tid = threadIdx.x, tile = blockDim.x * K;
    const double h24 = c.h24;
    const ADSCL_GLOBAL double* const Phi = gmem(f.state5 + c.off);
    const ADSCL_GLOBAL double* const Pi = gmem(f.state5 + f.total + c.off);
    const ADSCL_GLOBAL double* const Arow = gmem(f.state5 + 2 * f.total + c.off);
    const ADSCL_GLOBAL double* const nat = gmem(f.nat[b]);
    double* const dst[2] = {f.final_ ? f.state5 + c.off : nullptr,
                            snap ? f.snaps + (size_t)(st.steps / f.snap_every) * 5 * (size_t)f.total + c.off : nullptr};
    auto put = [&](int row, int i, double v) {
        if (dst[0]) dst[0][row * f.total + i] = v;
        if (dst[1]) dst[1][row * f.total + i] = v;
    };
    const bool keepA = f.a_reint > 0 && (st.steps % f.a_reint) != 0;
    double mn = 1.0, chk = 0.0, dN = 0.0, tot2 = 0.0;
    int col = 0;

    if (!f.frozen) {
        // q and p = sin x cos x q (0 at both ends and past them)
        auto q_at = [&](int i) -> double { return Phi[i] * Phi[i] + Pi[i] * Pi[i]; };
        double tot = 0.0;
        {
            double s = 0.0;
            for (int t0 = 1; t0 <= N - 2; t0 += tile)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int i = t0 + tid * K + k;
                    if (i <= N - 2) s += nat[kNatSC * N + i] * q_at(i);
                }
            block_scan(s, sh[2], tot);
        }
        const double p1 = nat[kNatSC * N + 1] * q_at(1), pN2 = nat[kNatSC * N + N - 2] * q_at(N - 2);
        dN = -h24 * (24.0 * tot + 2.0 * pN2 + 2.0 * p1);
        const double shift = (f.gauge == 0) ? dN : 0.0;
        double carry = 0.0, carry2 = 0.0;  // sums over the tiles before
        for (int t0 = 1; t0 <= N - 2; t0 += tile) {
            const int i0 = t0 + tid * K;
            // p and q at i0 - 2 .. i0 + K + 1, index i - i0 + 2
            double p[K + 4], q[K + 4], ps = 0.0;
#pragma unroll
            for (int k = 0; k < K + 4; ++k) {
                const int i = i0 - 2 + k;
                const bool in = i >= 1 && i <= N - 2;
                q[k] = in ? q_at(i) : 0.0;
                p[k] = in ? nat[kNatSC * N + i] * q[k] : 0.0;
                if (k >= 2 && k < K + 2) ps += p[k];
            }
            double tt;
            const double R0 = carry + block_scan(ps, sh[0], tt);  // sum of p before i0
            carry += tt;
            // delta~, e^-delta and sigma = tan^2 x q e^-delta at i0 - 1 .. i0 + K, index i - i0 + 1
            double dl[K + 2], E[K + 2], sg[K + 2], ss = 0.0, R = R0 - p[1];
#pragma unroll
            for (int k = 0; k < K + 2; ++k) {
                const int i = i0 - 1 + k;
                const bool in = i >= 1 && i <= N - 2;
                R += p[k + 1];
                dl[k] = -h24 * (24.0 * R - 12.0 * p[k + 1] + p[k] - p[k + 2] + 2.0 * p1) - shift;
                E[k] = exp(-dl[k]);
                sg[k] = in ? nat[kNatT2 * N + i] * q[k + 1] * E[k] : 0.0;
                if (k >= 1 && k < K + 1) ss += sg[k];
            }
            double R2 = carry2 + block_scan(ss, sh[1], tt);
            carry2 += tt;
#pragma unroll
            for (int k = 1; k < K + 1; ++k) {
                const int i = i0 - 1 + k;
                if (i > N - 2) break;
                R2 += sg[k];
                const double S = h24 * (24.0 * R2 - 12.0 * sg[k] + sg[k - 1] - sg[k + 1]);
                const double m = S / E[k], c3s = nat[kNatC3S * N + i];
                double A;
                if (keepA) {
                    A = Arow[i];
                    if (A < f.a_collapse) col = 1;
                } else {
                    A = 1.0 - c3s * m;
                    if (E[k] - c3s * S < f.a_collapse * E[k]) col = 1;
                }
                mn = fmin(mn, A);
                chk = fma(q[k + 1], 0.0, chk);
                chk = fma(A, 0.0, chk);
                chk = fma(dl[k], 0.0, chk);
                put(2, i, A);
                put(3, i, dl[k]);
                put(4, i, m);
            }
        }
        tot2 = carry2;
        if (tid < 2) {  // the ends: A = 1, delta~ = 0 at x = 0 and dN at pi/2, S = 0 and h sum sigma
            const int i = tid == 0 ? 0 : N - 1;
            const double dt = tid == 0 ? 0.0 : dN, d = dt - shift;
            const double A = keepA ? Arow[i] : 1.0;
            if (keepA && A < f.a_collapse) col = 1;
            mn = fmin(mn, A);
            chk = fma(q_at(i), 0.0, chk);
            chk = fma(A, 0.0, chk);
            chk = fma(d, 0.0, chk);
            put(2, i, A);
            put(3, i, d);
            put(4, i, tid == 0 ? 0.0 : 24.0 * h24 * tot2 / exp(-d));
        }
    } else {
        for (int i = tid; i < N; i += blockDim.x) {
            chk = fma(Phi[i] * Phi[i] + Pi[i] * Pi[i], 0.0, chk);
            put(2, i, 1.0);
            put(3, i, 0.0);
            put(4, i, 0.0);
        }
    }
    if (dst[1])
        for (int i = tid; i < N; i += blockDim.x) {
            dst[1][i] = Phi[i];
            dst[1][f.total + i] = Pi[i];
        }
    if (!isfinite(chk) || !isfinite(dN)) col |= 2;
    if (1.0 < f.a_collapse) col |= 1;
    // block reductions of min A and the flags
    for (int d = 32; d >= 1; d >>= 1) mn = fmin(mn, __shfl_xor(mn, d, 64));
    const int wcol = __any(col & 1) ? 1 : 0;
    const int wnf = __any(col & 2) ? 2 : 0;
    if ((tid & 63) == 0) {
        sh[2][tid >> 6] = mn;  // (last read before the tiles' barriers; with the metric frozen never)
        ish[tid >> 6] = wcol | wnf;
    }
    __syncthreads();
    if (tid == 0) {
        double mA = 1.0;
        int fl = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            mA = fmin(mA, sh[2][w]);
            fl |= ish[w];
        }
        if (f.final_) {
            InstStatus o = st;
            o.minA = mA;
            o.mass = f.frozen ? 0.0 : c.h * tot2 / ((f.gauge == 0) ? 1.0 : exp(-dN));
            if (o.state == ST_RUNNING || o.state == ST_DONE) {
                if (fl & 2) {
                    o.state = ST_NONFINITE;
                    o.t_c = (double)o.steps * c.dt;
                } else if (fl & 1) {
                    o.state = ST_COLLAPSED;
                    o.t_c = (double)o.steps * c.dt;
                } else {
                    o.state = (o.steps >= c.n_final) ? ST_DONE : ST_RUNNING;
                }
            }
            f.st[b] = o;
        }
    }
}

// Maximum of non-negative values over the block (up to 16 wavefronts), on thread 0.
// nan: a NaN among them is kept (else it is passed over).
__device__ double block_max(double v, bool nan, double* sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    auto worse = [&](double a, double o) -> double { return (nan && !(o == o)) ? o : (nan && !(a == a)) ? a : fmax(a, o); };
    for (int d = 32; d >= 1; d >>= 1) v = worse(v, __shfl_xor(v, d, 64));
    __syncthreads();
    if (lane == 0) sh[wv] = v;
    __syncthreads();
    double r = sh[0];
    for (int w = 1; w < nw; ++w) r = worse(r, sh[w]);
    return r;
}

// Diagnostics of the packed state (Phi, Pi, A, delta, m) of the current step, whose
// metric is the constraint solve of (Phi, Pi), into out [n_inst][5]: the residuals
// of Eqs. (5)-(6) at interior points (columns 0, 1), of Eq. (4) (2), the mass
// m(pi/2) (3) and the mass integral of Sec. II (4).
//
// Residual of Eq. (4), A_t = -2 sin x cos x A^2 e^-delta Phi Pi, which the
// evolution never imposes (Sec. II monitors the residuals of its equations):
// A_t is the time derivative of the discrete A of the constraint solve along
// the semi-discrete flow, the derivative of A(Phi, Pi) in the direction of the
// right-hand sides (Phi_t, Pi_t) of Eqs. (2)-(3), taken through each step of
// the solve (q = Phi^2 + Pi^2, p = sin x cos x q, delta~ = -prefix cell rule of
// p, E = e^-delta, sigma = tan^2 x q E, S = prefix cell rule of sigma,
// m = S / E, A = 1 - cos^3 x / sin x m):
//   q_t = 2 (Phi Phi_t + Pi Pi_t),  p_t = sin x cos x q_t,
//   delta~_t = -prefix cell rule of p_t,  E_t = -E delta~_t,
//   sigma_t = tan^2 x (q_t E + q E_t),  S_t = prefix cell rule of sigma_t,
//   m_t = (S_t - m E_t) / E,  A_t = -cos^3 x / sin x m_t.
// E is e^-delta of the gauge-shifted delta: m_t is homogeneous of degree 0 in
// a constant factor of E, S and their derivatives, so the shift drops out.
// Column 2 is max over interior points of |A_t + 2 sin x cos x A^2 e^-delta Phi
// Pi|; NaN with the metric frozen (A is then held, not solved).
//
// One block per instance; the interior points go in tiles of kDiagTile, kDiagK
// consecutive ones per thread.  First loop: the fluxes of a tile and two points on
// each side into LDS (one exponential per point), the right-hand sides, and q_t, p_t
// into `scr` (two doubles per packed point).  Second loop: both prefix sums side by
// side, their sums carried over the tiles; a thread forms sigma_t at its
// neighbours' adjacent points itself.  The mass integral's 4-point rule sums to
// h sum tan^2 x A q (the integrand is even and 0 at both ends).
// Bound by the latency of the loads and scans of a tile: one instance of 1025
// points 16 us, the 1024-instance batch (1025 to 4097) 124, against 61 and 1085 in
// two kernels with 256 threads, a run of N/256 points each and about eight tangents
// and thirteen exponentials per point.
constexpr int kDiagK = 4, kDiagThreads = 512, kDiagTile = kDiagK * kDiagThreads;

__global__ void __launch_bounds__(kDiagThreads) diagnostics_kernel(const InstConst* ic, const double* const* nats,
                                                                   const double* state5, int64_t total, int frozen,
                                                                   double ko, double* scr, double* out)
{
    __shared__ double sf[kDiagTile + 4], sgx[kDiagTile + 4];  // f1 and g of points t0 - 2 ..
    __shared__ double sh[3][16];
    constexpr int K = kDiagK;
    const int b = blockIdx.x, tid = threadIdx.x;
    const InstConst c = ic[b];
    const int N = c.N;
    const double h24 = c.h24, i12h = c.i12h, kof = ko / (64.0 * c.h);
    const ADSCL_GLOBAL double* const Ph = gmem(state5 + c.off);
    const ADSCL_GLOBAL double* const Pq = gmem(state5 + total + c.off);
    const ADSCL_GLOBAL double* const Aa = gmem(state5 + 2 * total + c.off);
    const ADSCL_GLOBAL double* const dd = gmem(state5 + 3 * total + c.off);
    const ADSCL_GLOBAL double* const mm = gmem(state5 + 4 * total + c.off);
    const ADSCL_GLOBAL double* const nat = gmem(nats[b]);
    ADSCL_GLOBAL double* const X = gmem(scr + c.off);          // p_t
    ADSCL_GLOBAL double* const Y = gmem(scr + total + c.off);  // q_t
    // the point a ghost mirrors; sl, sr: the sign it takes left of x = 0, right of pi/2
    auto mir = [&](int i, double sl, double sr, double& sg) -> int {
        sg = i < 0 ? sl : (i > N - 1 ? sr : 1.0);
        return i < 0 ? -i : (i > N - 1 ? 2 * (N - 1) - i : i);
    };
    // Phi odd about 0, even about pi/2; Pi even about 0, odd about pi/2
    auto phg = [&](int i) -> double { double sg; const int j = mir(i, -1.0, 1.0, sg); return sg * Ph[j]; };
    auto pig = [&](int i) -> double { double sg; const int j = mir(i, 1.0, -1.0, sg); return sg * Pq[j]; };
    // A even about 0, A - 1 odd about pi/2; delta even about both ends
    auto Ag = [&](int i) -> double { double sg; const int j = mir(i, 1.0, -1.0, sg); return sg > 0.0 ? Aa[j] : 2.0 - Aa[j]; };
    auto dg = [&](int i) -> double { double sg; return dd[mir(i, 1.0, 1.0, sg)]; };
    auto w_at = [&](int i) -> double { return Aa[i] * exp(-dd[i]); };
    auto g_in = [&](int i) -> double { return nat[kNatT2 * N + i] * (w_at(i) * Ph[i]); };
    auto ko7 = [&](auto&& u, int i) -> double {
        return kof * (u(i - 3) - 6.0 * u(i - 2) + 15.0 * u(i - 1) - 20.0 * u(i) + 15.0 * u(i + 1) - 6.0 * u(i + 2)
                      + u(i + 3));
    };
    auto d5 = [&](auto&& u, int i) -> double { return (u(i - 2) - 8.0 * u(i - 1) + 8.0 * u(i + 1) - u(i + 2)) * i12h; };

    double rA = 0.0, rd = 0.0, rt = 0.0, T = 0.0;
    for (int t0 = 1; t0 <= N - 2; t0 += kDiagTile) {
        if (!frozen) {
            __syncthreads();  // the last tile's readers are done
            for (int k = tid; k < kDiagTile + 4; k += kDiagThreads) {
                const int i = t0 - 2 + k;
                if (i > N) break;
                // f1 = w Pi: even about 0, odd about pi/2; g = tan^2 x w Phi up to N - 2,
                // the even 6th-order extrapolation at N - 1: odd about 0, even about pi/2
                double sg1, sg2;
                const int j = mir(i, 1.0, -1.0, sg1);
                mir(i, -1.0, 1.0, sg2);
                const double w = w_at(j);
                sf[k] = sg1 * (w * Pq[j]);
                sgx[k] = j == N - 1 ? (15.0 * g_in(N - 2) - 6.0 * g_in(N - 3) + g_in(N - 4)) / 10.0
                                    : sg2 * (nat[kNatT2 * N + j] * (w * Ph[j]));
            }
            __syncthreads();
        }
        for (int k = tid; k < kDiagTile; k += kDiagThreads) {
            const int i = t0 + k;
            if (i > N - 2) break;
            const double sc = nat[kNatSC * N + i], q = Ph[i] * Ph[i] + Pq[i] * Pq[i];
            T += nat[kNatT2 * N + i] * Aa[i] * q;
            rA = fmax(rA, fabs(d5(Ag, i) - (nat[kNatRA * N + i] * (1.0 - Aa[i]) - sc * Aa[i] * q)));
            rd = fmax(rd, fabs(d5(dg, i) + sc * q));
            if (!frozen) {
                const double rPh = d5([&](int j) -> double { return sf[j - t0 + 2]; }, i) + ko7(phg, i);
                const double rPi = nat[kNatCT2 * N + i] * d5([&](int j) -> double { return sgx[j - t0 + 2]; }, i) +
                                   ko7(pig, i);
                const double qt = 2.0 * (Ph[i] * rPh + Pq[i] * rPi);
                X[i] = sc * qt;
                Y[i] = qt;
            }
        }
    }
    double tot;
    block_scan(T, sh[2], tot);
    __syncthreads();
    if (!frozen) {
        // X past the ends is never needed: sigma_t is 0 there
        auto in = [&](int i) -> bool { return i >= 1 && i <= N - 2; };
        const double p1 = X[1];
        double carry = 0.0, carry2 = 0.0;
        for (int t0 = 1; t0 <= N - 2; t0 += kDiagTile) {
            const int i0 = t0 + tid * K;
            double x[K + 4], ps = 0.0;  // i0 - 2 .. i0 + K + 1
#pragma unroll
            for (int k = 0; k < K + 4; ++k) {
                x[k] = in(i0 - 2 + k) ? X[i0 - 2 + k] : 0.0;
                if (k >= 2 && k < K + 2) ps += x[k];
            }
            double tt;
            double R = carry + block_scan(ps, sh[0], tt) - x[1];
            carry += tt;
            double E[K + 2], Et[K + 2], sg[K + 2], ss = 0.0;  // i0 - 1 .. i0 + K
#pragma unroll
            for (int k = 0; k < K + 2; ++k) {
                const int i = i0 - 1 + k;
                R += x[k + 1];
                E[k] = Et[k] = sg[k] = 0.0;
                if (in(i)) {
                    E[k] = exp(-dd[i]);
                    Et[k] = E[k] * (h24 * (24.0 * R - 12.0 * x[k + 1] + x[k] - x[k + 2] + 2.0 * p1));
                    sg[k] = nat[kNatT2 * N + i] * (Y[i] * E[k] + (Ph[i] * Ph[i] + Pq[i] * Pq[i]) * Et[k]);
                }
                if (k >= 1 && k < K + 1) ss += sg[k];
            }
            double R2 = carry2 + block_scan(ss, sh[1], tt);
            carry2 += tt;
#pragma unroll
            for (int k = 1; k < K + 1; ++k) {
                const int i = i0 - 1 + k;
                if (i > N - 2) break;
                R2 += sg[k];
                const double St = h24 * (24.0 * R2 - 12.0 * sg[k] + sg[k - 1] - sg[k + 1]);
                const double mt = (St - mm[i] * Et[k]) / E[k];
                const double r = -nat[kNatC3S * N + i] * mt +
                                 2.0 * nat[kNatSC * N + i] * Aa[i] * Aa[i] * E[k] * Ph[i] * Pq[i];
                rt = (r == r) ? fmax(rt, fabs(r)) : r;  // keep a NaN
            }
        }
    }
    rA = block_max(rA, false, sh[2]);
    rd = block_max(rd, false, sh[2]);
    rt = frozen ? __builtin_nan("") : block_max(rt, true, sh[2]);
    if (tid == 0) {
        out[b * 5 + 0] = rA;
        out[b * 5 + 1] = rd;
        out[b * 5 + 2] = rt;
        out[b * 5 + 3] = mm[N - 1];
        out[b * 5 + 4] = c.h * tot;
    }
}

}  // namespace

hipError_t launch_init_gaussian(int n_inst, const InstConst* ic, const double* eps, const double* sigma,
                                double* Phi, double* Pi, int64_t max_N, hipStream_t s)
{
    const int gx = (int)((max_N + 255) / 256);
    init_gaussian_kernel<<<dim3(gx, n_inst), dim3(256), 0, s>>>(n_inst, ic, eps, sigma, Phi, Pi);
    return hipGetLastError();
}

hipError_t launch_init_modes(int n_inst, const InstConst* ic, const double* eps, const double* c, int Jc,
                             const double* const* emode, double* Phi, double* Pi, int64_t max_N, hipStream_t s)
{
    const int gx = (int)((max_N + 255) / 256);
    init_modes_kernel<<<dim3(gx, n_inst), dim3(256), 0, s>>>(n_inst, ic, eps, c, Jc, emode, Phi, Pi);
    return hipGetLastError();
}

hipError_t launch_pins(int n_inst, const InstConst* ic, double* Phi, double* Pi, hipStream_t s)
{
    pins_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, ic, Phi, Pi);
    return hipGetLastError();
}

hipError_t launch_reset_status(int n_inst, InstStatus* st, hipStream_t s)
{
    reset_status_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, st);
    return hipGetLastError();
}

hipError_t launch_set_targets(int n_inst, const InstConst* ic, InstStatus* st, int64_t max_steps, hipStream_t s)
{
    set_targets_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, ic, st, max_steps);
    return hipGetLastError();
}

hipError_t launch_finalize(int n_inst, int64_t max_N, const InstConst* ic, InstStatus* st, const double* const* nat,
                           double* state5, int64_t total, int gauge, int frozen, double a_collapse, bool final,
                           int32_t snap_every, int32_t n_slots, double* snaps, hipStream_t s, int32_t a_reint)
{
    FinArgs f;
    f.ic = ic;
    f.st = st;
    f.nat = nat;
    f.state5 = state5;
    f.total = total;
    f.a_collapse = a_collapse;
    f.snaps = snaps;
    f.snap_every = snap_every;
    f.n_slots = n_slots;
    f.gauge = gauge;
    f.frozen = frozen;
    f.final_ = final ? 1 : 0;
    f.a_reint = a_reint;
    // one tile for the largest grid where 1024 threads hold it
    const int waves = (int)std::min<int64_t>(16, (max_N - 2 + 64 * kFinK - 1) / (64 * kFinK));
    finalize_kernel<<<dim3(n_inst), dim3(64 * waves), 0, s>>>(f);
    return hipGetLastError();
}

hipError_t launch_diagnostics(int n_inst, const InstConst* ic, const double* const* nat, const double* state5,
                              int64_t total, int frozen, double ko, double* scr, double* out, hipStream_t s)
{
    diagnostics_kernel<<<dim3(n_inst), dim3(kDiagThreads), 0, s>>>(ic, nat, state5, total, frozen, ko, scr, out);
    return hipGetLastError();
}

}  // namespace adscl
