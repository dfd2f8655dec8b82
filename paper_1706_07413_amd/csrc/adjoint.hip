// Discrete adjoint (reverse-mode derivative) of the batched AdS4 evolution
// (Liebling & Khanna, arXiv:1706.07413, Sec. II), gfx950.
//
// The derivative is that of the computation the forward kernels perform: the
// constraint solve of Eqs. (5)-(6) by two prefix sums, the right-hand sides of
// Eqs. (2)-(3) with their parity ghosts and end extrapolation, the
// Kreiss-Oliger terms and the four stages of classical RK4.  Transposed, the
// prefix sums become suffix sums (total minus exclusive prefix), each stencil
// becomes its mirror image, and a ghost entry's weight goes back to the point
// it mirrors with the parity sign.
//
// Layout and launch shape are those of the forward kernel (stage.h): one
// workgroup per instance, lane l owns points l*P .. l*P+P-1 in registers.  For
// each step t (in reverse) the kernel takes the four stage
// inputs V_s with their e^-delta and w from the stage record that the forward
// recompute of the segment kept (the forward kernel's own arithmetic, its
// tables in LDS), or, where the records would not fit, recomputes them from
// the stored U^t into a per-instance scratch (REC false); both are
// lane-interleaved, so each lane reads back only what it (or its forward
// counterpart) wrote.  Then it runs the four stage adjoints in reverse.
//
// A reverse stage is bound by latency: three barriers, the scans between them and,
// with one workgroup on a compute unit, the way of its record from HBM (128 KB per stage
// at N = 4097).  So the record is read once, in pairs that a wavefront takes as whole
// lines, each pair as soon as the registers of the stage before fall free (e^-delta
// and w between the two scans, Phi and Pi at the stage's end), and nothing that a
// stage waits for at once is asked for after them, since vector loads return in order.
// The adjoint state sits in LDS (128 KB at N = 4097, which leaves the registers to the
// record in flight) with the rows of tan^2 x that fit beside it; the other tables come
// from L2, asked for a scan or a set of stencils ahead.
// Measured per step, one instance of 4097 points: 22.6 us against 45 with the record's
// fields loaded where they are used and the tables re-read there; 121 instances of 4097
// beside 135 of 2049: 34 us against 57.  What a stage holds must fit the 256 registers
// a lane has at 4097 points: with the running adjoint in registers instead (76 spilled)
// a step took 37 and 63 us.  Ragged grids take the same path: N = 3001 66 -> 24 us.
#include <math.h>

#include "stage.h"

namespace adscl {
namespace {

// The per-instance stage scratch of the kernel that recomputes the stages: one step's
// stage record, 16 fields of [P][64 W] doubles (four stages of Phi, Pi, e^-delta and w).
constexpr int kFields = 16;

// Sum of the wavefront totals r[0..W) over the wavefronts after this one
// (`after`), the outermost first, and over all (`all`).  Lanes v < W hold r[v] and
// a DPP suffix runs over them (W <= 16: within the first row of 16 lanes), so
// that, as in wave_incl_suffix, no total is ever subtracted.  `rest`: r[W].
template <int W>
__device__ __forceinline__ void wave_suffixes(const double* r, int lane, int wv, double& after, double& all, double& rest)
{
    const double y = (lane <= W) ? r[lane <= W ? lane : 0] : 0.0;
    rest = readlane_d(y, W);
    double x = (lane < W) ? y : 0.0;
    if constexpr (W > 1) x += dpp_d<0x101, 0xf>(x);  // row_shl:1
    if constexpr (W > 2) x += dpp_d<0x102, 0xf>(x);  // row_shl:2
    if constexpr (W > 4) x += dpp_d<0x104, 0xf>(x);  // row_shl:4
    if constexpr (W > 8) x += dpp_d<0x108, 0xf>(x);  // row_shl:8
    all = readlane_d(x, 0);
    const int w = __builtin_amdgcn_readfirstlane(wv);
    after = (w < W - 1) ? readlane_d(x, w < W - 1 ? w + 1 : 0) : 0.0;
}

// A wavefront-uniform value in scalar registers.
__device__ __forceinline__ double uni(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ ADSCL_GLOBAL double* uni(ADSCL_GLOBAL double* p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (ADSCL_GLOBAL double*)(((uint64_t)hi << 32) | lo);
}

template <int P, int W, bool FULL>
struct Rev {
    static constexpr int NL = 64 * W;
    using S_t = Stage<P, W, FULL>;

    // Adds to (vb0, vb1) the adjoint, through the constraint solve of the state
    // (v0, v1) with e^-delta E, of the cotangents Eb (of e^-delta, gauge applied) and
    // Sb (of S).
    //   S_k = h/24 (24 R_k - 12 s_k + s_{k-1} - s_{k+1}), R_k = sum_{i<=k} s_i,
    //   s = tan^2 x q e^-delta  ->  sbar_j = h/24 (24 sum_{k>=j} Sb_k - 12 Sb_j + Sb_{j+1} - Sb_{j-1});
    //   e^-delta = exp(-(dt_k - shift)), shift = dt_{N-1} (boundary gauge) or 0;
    //   dt_k = -h/24 (24 R_k - 12 p_k + p_{k-1} - p_{k+1} + 2 p_1), p = sin x cos x q.
    // At points past N - 2 v0, v1, Eb, Sb and the tables are 0 and e^-delta finite, so
    // all that is formed there is 0.  lt(f, k) gives sin x cos x
    // (f = 0) and tan^2 x (1) of the lane's point k.
    // Contains two barriers.  `mid` runs between the scans, when E is no longer needed.
    template <class LT, class M>
    static __device__ __forceinline__ void constraint_reverse(S_t& sg, const double* v0, const double* v1,
                                                              const double* E, const double* Eb, const double* Sb,
                                                              double* vb0, double* vb1, LT&& lt, M&& mid)
    {
        const int tid = sg.tid, lane = sg.lane, wv = __builtin_amdgcn_readfirstlane(sg.wv);
        const double h24 = sg.h24, a24 = uni(24.0 * h24), a12 = uni(12.0 * h24);
        double* red = sg.red;

        // suffix sums of Sb, accumulated from the outer end: the lane's points
        // from P-1 down, the lanes to its right by doubling steps, the
        // wavefronts to its right from the last one in (never a total minus a
        // prefix, which would lose the small suffixes away from the origin)
        double tot1 = 0.0;
#pragma unroll
        for (int k = P - 1; k >= 0; --k) tot1 += Sb[k];
        const double sinc = wave_incl_suffix(tot1);
        if (lane == 0) {
            red[W + wv] = sinc;
            sg.RSb[2 * (wv + 1)] = Sb[0];
        }
        if (lane == 63) sg.RSb[2 * (wv + 1) + 1] = Sb[P - 1];
        __syncthreads();
        double d[P], qb[P], t0[P];
        double d0 = 0.0;
        {
            double after, all, rest;
            wave_suffixes<W>(red + W, lane, wv, after, all, rest);
            double run = S_t::from_right(sinc) + after;  // the lanes right of this one, and the wavefronts
            const double sl = dpp_old<0x138>(sg.RSb[2 * wv + 1], Sb[P - 1]);
            const double sr = dpp_old<0x130>(sg.RSb[2 * (wv + 2)], Sb[0]);
#pragma unroll
            for (int k = P - 1; k >= 0; --k) {
                run += Sb[k];
                const double sm = (k == 0) ? sl : Sb[k - 1];
                const double sp = (k == P - 1) ? sr : Sb[k + 1];
                const double sb = fma(a24, run, fma(-a12, Sb[k], h24 * (sp - sm)));
                const double ts = lt(1, k) * sb;
                qb[k] = E[k] * ts;
                const double q = fma(v0[k], v0[k], v1[k] * v1[k]);
                d[k] = -E[k] * fma(q, ts, Eb[k]);  // cotangent of dt_k
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) t0[k] = lt(0, k);
        mid();
        if (tid == 0) {  // dt_0 is identically 0, its share goes to the shift only
            d0 = d[0];
            d[0] = 0.0;
        }
        // suffix sums of d, the same way
        double tot = 0.0;
#pragma unroll
        for (int k = P - 1; k >= 0; --k) tot += d[k];
        const double sinc2 = wave_incl_suffix(tot);
        if (lane == 0) {
            red[2 * W + wv] = sinc2;
            red[3 * W + wv] = d0;
            sg.RDt[2 * (wv + 1)] = d[0];
        }
        if (lane == 63) sg.RDt[2 * (wv + 1) + 1] = d[P - 1];
        __syncthreads();
        double after2, tot2, dt0;  // dt0: d0 of the first wavefront
        wave_suffixes<W>(red + 2 * W, lane, wv, after2, tot2, dt0);
        double run = S_t::from_right(sinc2) + after2;
        const double dl = dpp_old<0x138>(sg.RDt[2 * wv + 1], d[P - 1]);
        const double dr = dpp_old<0x130>(sg.RDt[2 * (wv + 2)], d[0]);
        // boundary gauge: shift = dt_{N-1} = -h/24 (24 sum p + 2 p_{N-2} + 2 p_1)
        const double shb = sg.bgauge ? -(tot2 + dt0) : 0.0;
        const double cs = -a24 * shb;
        double x1 = 0.0, xe = 0.0;  // what p_1 and p_{N-2} get besides
        if (tid == 0) x1 = -2.0 * h24 * (tot2 + shb);
        if (sg.has_nm2) xe = -2.0 * h24 * shb;
        const int e = FULL ? P - 1 : sg.end_here() - 1;
#pragma unroll
        for (int k = P - 1; k >= 0; --k) {
            run += d[k];
            const double dm = (k == 0) ? dl : d[k - 1];
            const double dp = (k == P - 1) ? dr : d[k + 1];
            double pb = fma(-a24, run, fma(a12, d[k], fma(-h24, dp - dm, cs)));
            if (k == 1) pb += x1;
            if (FULL) {
                if (k == P - 1) pb += xe;
            } else {
                pb += (k == e) ? xe : 0.0;
            }
            const double q2 = 2.0 * fma(t0[k], pb, qb[k]);  // table is 0 off 1..N-2
            vb0[k] = fma(v0[k], q2, vb0[k]);
            vb1[k] = fma(v1[k], q2, vb1[k]);
        }
    }

    // Adjoint of one stage map V -> k = (Phi_t, Pi_t)(V): given the cotangents
    // (kb0, kb1) of k at the own points (0 elsewhere), returns (vb0, vb1) = J^T kb.
    // v0, v1, E, w: the stage's input, e^-delta and A e^-delta.  ct2: cot^2 x of the
    // lane's points; lt(f, k): sin x cos x (f = 0), tan^2 x (1) and cot^2 x (2) of its
    // point k.
    // The edge and reduction slots are free to be written: their last reads lie before
    // the barrier before last (or, of the recomputed stages' slots, before the last).
    // TK: the points from k = TK on whose tan^2 x is held here, not asked for again.
    template <int TK, class LT, class M>
    static __device__ __forceinline__ void stage_reverse(S_t& sg, const double* v0, const double* v1, const double* E,
                                                         const double* w, const double* kb0, const double* kb1,
                                                         const double* ct2, double* vb0, double* vb1, LT&& lt, M&& mid)
    {
        const int tid = sg.tid, lane = sg.lane, wv = __builtin_amdgcn_readfirstlane(sg.wv);
        const double i12h = sg.i12h, kof = sg.kof;
        double f1b[P], gb[P], t0[P], t1[P], t2[P];
        {
            // row cotangents in registers: ya (Phi_t rows 1..N-2), yb = kb1 (Pi_t
            // rows 0..N-2), yg = cot^2 x yb (rows of D g); the neighbours' by DPP,
            // the adjacent wavefronts' through RU / RF; ghosts carry zero
            double ya[P], yg[P];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                ya[k] = (k == 0 && tid == 0) ? 0.0 : kb0[k];
                yg[k] = ct2[k] * kb1[k];
            }
            {
                double2* ru = sg.RU + (wv + 1) * 6;
                double* rf = sg.RF + (wv + 1) * 4;
                if (lane == 0) {
#pragma unroll
                    for (int r = 0; r < 3; ++r) ru[r] = make_double2(ya[r], kb1[r]);
                    rf[0] = yg[0];
                    rf[1] = yg[1];
                }
                if (lane == 63) {
#pragma unroll
                    for (int r = 0; r < 3; ++r) ru[3 + r] = make_double2(ya[P - 1 - r], kb1[P - 1 - r]);
                    rf[2] = yg[P - 1];
                    rf[3] = yg[P - 2];
                }
            }
            // RAG: the rows of the two lanes that hold N - 4 .. N - 2, in the halves of GU
            // and GF that the last recomputed stage did not use
            double2 *gu = nullptr, *gf = nullptr;
            if constexpr (S_t::RAG) {
                gu = sg.GU + (sg.buf ^ 1) * 2 * P;
                gf = sg.GF + (sg.buf ^ 1) * 2 * P;
                if (sg.near_end) {
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        gu[sg.i0 - sg.jb + k] = make_double2(ya[k], kb1[k]);
                        gf[sg.i0 - sg.jb + k].x = yg[k];
                    }
                }
            }
            __syncthreads();
            // points i0-3 .. i0+P+2 of the rows; lanes 0 / 63 take the neighbouring
            // wavefront's (or the ghost) slot
            const double2* xl = sg.RU + wv * 6;
            const double2* xr = sg.RU + (wv + 2) * 6;
            {
                double w[P + 6];
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    w[r] = dpp_old<0x138>(xl[5 - r].x, ya[P - 3 + r]);
                    w[P + 3 + r] = dpp_old<0x130>(xr[r].x, ya[r]);
                }
#pragma unroll
                for (int k = 0; k < P; ++k) w[3 + k] = ya[k];
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    // the Kreiss-Oliger stencil is symmetric: its transpose is itself
                    vb0[k] = kof * (w[k] - 6.0 * w[k + 1] + 15.0 * w[k + 2] - 20.0 * w[k + 3]
                                    + 15.0 * w[k + 4] - 6.0 * w[k + 5] + w[k + 6]);
                    // D is antisymmetric: its transpose is -D
                    f1b[k] = (w[k + 5] - 8.0 * w[k + 4] + 8.0 * w[k + 2] - w[k + 1]) * i12h;
                }
            }
            {
                double w[P + 6];
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    w[r] = dpp_old<0x138>(xl[5 - r].y, kb1[P - 3 + r]);
                    w[P + 3 + r] = dpp_old<0x130>(xr[r].y, kb1[r]);
                }
#pragma unroll
                for (int k = 0; k < P; ++k) w[3 + k] = kb1[k];
#pragma unroll
                for (int k = 0; k < P; ++k)
                    vb1[k] = kof * (w[k] - 6.0 * w[k + 1] + 15.0 * w[k + 2] - 20.0 * w[k + 3]
                                    + 15.0 * w[k + 4] - 6.0 * w[k + 5] + w[k + 6]);
            }
            {
                const double* fl = sg.RF + wv * 4;
                const double* fr = sg.RF + (wv + 2) * 4;
                double fw[P + 4];  // points i0-2 .. i0+P+1
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    fw[r] = dpp_old<0x138>(fl[3 - r], yg[P - 2 + r]);
                    fw[P + 2 + r] = dpp_old<0x130>(fr[r], yg[r]);
                }
#pragma unroll
                for (int k = 0; k < P; ++k) fw[2 + k] = yg[k];
#pragma unroll
                for (int k = 0; k < P; ++k) gb[k] = (fw[k + 4] - 8.0 * fw[k + 3] + 8.0 * fw[k + 1] - fw[k]) * i12h;
            }
            // the tables for what follows, on their way during the corrections
#pragma unroll
            for (int k = 0; k < P; ++k) {
                t0[k] = lt(0, k);
                t1[k] = lt(1, k);
                t2[k] = lt(2, k);
            }
            // rows whose stencils reach past pi/2 (Phi even, Pi odd, f1 odd, g even)
            // and g_{N-1} = (15 g_{N-2} - 6 g_{N-3} + g_{N-4}) / 10
            if constexpr (FULL) {
                if (sg.near_end) {  // the last lane
                    const double gN1 = (8.0 * yg[P - 1] - yg[P - 2]) * i12h;
                    vb0[P - 1] += kof * (-6.0 * kb0[P - 1] + kb0[P - 2]);
                    vb1[P - 1] -= kof * (-6.0 * kb1[P - 1] + kb1[P - 2]);
                    f1b[P - 1] += kb0[P - 1] * i12h;
                    gb[P - 1] += -yg[P - 1] * i12h + 1.5 * gN1;
                    vb0[P - 2] += kof * kb0[P - 1];
                    vb1[P - 2] -= kof * kb1[P - 1];
                    gb[P - 2] += -0.6 * gN1;
                    gb[P - 3] += 0.1 * gN1;
                }
            } else {
                if (sg.near_end) {
                    const int n2 = sg.N - 2 - sg.jb, e = sg.end_here() - 1;
                    const double2 u2 = gu[n2], u3 = gu[n2 - 1];
                    const double yg2 = gf[n2].x, yg3 = gf[n2 - 1].x;
                    const double gN1 = (8.0 * yg2 - yg3) * i12h;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        if (k == e) {
                            vb0[k] += kof * (-6.0 * u2.x + u3.x);
                            vb1[k] -= kof * (-6.0 * u2.y + u3.y);
                            f1b[k] += u2.x * i12h;
                            gb[k] += -yg2 * i12h + 1.5 * gN1;
                        }
                        if (k == e - 1) {
                            vb0[k] += kof * u2.x;
                            vb1[k] -= kof * u2.y;
                            gb[k] += -0.6 * gN1;
                        }
                        if (k == e - 2) gb[k] += 0.1 * gN1;
                    }
                }
                if (sg.at_end) {  // the points past N - 2 stay 0
                    const int e = sg.end_here();
#pragma unroll
                    for (int k = 0; k < P; ++k)
                        if (k >= e) vb0[k] = vb1[k] = f1b[k] = gb[k] = 0.0;
                }
            }
        }
        // rows whose stencils reach the ghosts left of x = 0 (Phi odd, Pi even,
        // f1 even, g odd) and the origin row Pi_t(0) = 3 D f2(0) + KO Pi
        double ob = 0.0;
        if (tid == 0) {
            const double ya1 = kb0[1], ya2 = kb0[2];
            const double yb0 = kb1[0], yb1 = kb1[1], yb2 = kb1[2];
            const double yg1 = ct2[1] * kb1[1];
            vb0[1] -= kof * (-6.0 * ya1 + ya2);
            vb0[2] -= kof * ya1;
            vb1[1] += kof * (15.0 * yb0 - 6.0 * yb1 + yb2);
            vb1[2] += kof * (-6.0 * yb0 + yb1);
            vb1[3] += kof * yb0;
            f1b[1] += ya1 * i12h;
            gb[1] -= yg1 * i12h;
            ob = 3.0 * yb0 * i12h;
        }

        double Eb[P], Sb[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            double f2b = t1[k] * gb[k];
            if (k == 1) f2b += 16.0 * ob;
            if (k == 2) f2b -= 2.0 * ob;
            vb0[k] = fma(w[k], f2b, vb0[k]);
            vb1[k] = fma(w[k], f1b[k], vb1[k]);
            Eb[k] = fma(v1[k], f1b[k], v0[k] * f2b);
            Sb[k] = -(t2[k] * t0[k]) * Eb[k];  // cos^3 x/sin x
        }
        constraint_reverse(sg, v0, v1, E, Eb, Sb, vb0, vb1,
                           [&](int f, int k) -> double { return (f == 1 && k >= TK) ? t1[k] : lt(f, k); }, mid);
        if (tid == 0) vb0[0] = 0.0;  // Phi_0 is pinned
    }
};

// Rows of tan^2 x and cot^2 x ([P] each) that the reverse kernel keeps in LDS beside the
// stage's and four fields of adjoint state: what is left of 160 KB (at N = 4097, where
// the state takes 128 KB, 6 of the 8 rows of tan^2 x), or of 80 KB where two workgroups
// share a compute unit; the rest is read from L2.
template <int P, int W, bool FULL>
constexpr int adj_table_rows()
{
    constexpr size_t base = Stage<P, W, FULL>::lds_doubles + (size_t)4 * P * 64 * W;
    constexpr size_t cap = (base * 8 <= 80 * 1024 ? 80 : 160) * 1024 / 8;
    constexpr size_t rows = (cap - base) / (64 * W);
    return (int)(rows < 2 * P ? rows : 2 * P);
}

// LDS of the reverse kernel.
template <int P, int W, bool FULL>
constexpr size_t adj_lds_bytes()
{
    return (Stage<P, W, FULL>::lds_doubles + (size_t)(4 * P + adj_table_rows<P, W, FULL>()) * 64 * W) * sizeof(double);
}

// Rows of [64 W] doubles in LDS from byte `at` on, of which a lane uses its own entries:
// one 64 KB window's base per register, so that an access is a base and an immediate
// offset.  fresh() keeps the compiler from forming the accesses' addresses ahead of a
// loop and holding (or spilling) each of them.
template <int NL, size_t AT>
struct LaneLds {
    char* base;
    unsigned o[3];
    __device__ __forceinline__ LaneLds(double* lds, int lane_id) : base((char*)lds)
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) o[i] = (unsigned)lane_id * 8u + (unsigned)i * 65536u;
        fresh();
    }
    __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2])); }
    __device__ __forceinline__ double& at(int row) const
    {
        const unsigned c = (unsigned)AT + (unsigned)row * (NL * 8);
        return *(double*)(base + (o[c >> 16] + (c & 65535u)));
    }
};

// REC: the segment's stage record was kept (AdjointArgs::keep).
template <int P, int W, bool FULL, bool REC>
__global__ void __launch_bounds__(64 * W) adjoint_kernel(AdjointArgs a)
{
    constexpr int NL = 64 * W;
    using R = Rev<P, W, FULL>;
    extern __shared__ double lds[];
    const int b = a.order[blockIdx.x];
    const AdjSeg sq = a.sg[b];
    if (!sq.active) return;
    const InstConst ic = a.ic[b];
    using S_t = Stage<P, W, FULL>;
    S_t sg;
    sg.setup(lds, ic, a.tab[b], a.gauge, 0.0);
    const int N = sg.N, i0 = sg.i0, tid = sg.tid;
    const double dt = sg.dt, dt2 = uni(0.5 * dt), dt6 = uni(dt / 6.0);
    // In the LDS past the stage's, each lane its own entries only: the step's incoming
    // adjoint state, dt/6 U-bar' (fields 0, 1), the running one (2, 3), and then as many rows
    // of tan^2 x and cot^2 x as fit.
    LaneLds<NL, S_t::lds_doubles * 8> own(lds, tid);
    constexpr int TR = adj_table_rows<P, W, FULL>();
    auto lt = [&](int f, int k) -> double {
        const int r = (f - 1) * P + k;
        if (f > 0 && r < TR) return own.at(4 * P + r);
        return sg.tab(sg.tables(), f, k);
    };
#pragma unroll
    for (int r = 0; r < TR; ++r) own.at(4 * P + r) = sg.tab0[(P + r) * NL + tid];
    auto ub = [&](int f, int k) -> double& { return own.at(f * P + k); };
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const bool o = sg.own(k);
        ub(2, k) = o ? a.Ubar[ic.off + i0 + k] : 0.0;
        ub(3, k) = o ? a.Ubar[a.total + ic.off + i0 + k] : 0.0;
    }

    // The stage at hand, V_s with e^-delta and w, and cot^2 x.
    constexpr size_t kStage = (size_t)4 * P * NL, kRec = 4 * kStage;
    double v0[P], v1[P], E[P], w[P], ct2[P];
    auto load_v = [&](ADSCL_GLOBAL double* stage) {
        const auto r = stage_rec<P, NL>(stage, tid);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const pair_t x = r.ld(0, k);
            v0[k] = x[0];
            v1[k] = x[1];
        }
    };
    auto load_e = [&](ADSCL_GLOBAL double* stage) {
        const auto r = stage_rec<P, NL>(stage, tid);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const pair_t x = r.ld(1, k);
            E[k] = x[0];
            w[k] = x[1];
        }
    };
    // (a segment is at most 2^31 - 1 steps; 32-bit counters keep the record's address scalar)
    const int n_seg = (int)(sq.n1 - sq.n0);
    ADSCL_GLOBAL double* st = REC ? gmem(a.keep[b]) + (size_t)(n_seg - 1) * kRec : gmem(a.stg[b]);
#pragma unroll
    for (int k = 0; k < P; ++k) ct2[k] = lt(2, k);
    if (REC) {
        load_e(uni(st + 3 * kStage));
        load_v(uni(st + 3 * kStage));
    }
    for (int t = n_seg - 1; t >= 0; --t) {
        // the stage inputs V_s of step t and their e^-delta and w: read from the
        // record, or recomputed from U^t into the scratch
        if constexpr (!REC) {
            const ADSCL_GLOBAL double* u = gmem(a.seg[b]) + (size_t)t * 2 * (size_t)N;
            double un0[P], un1[P];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const bool o = sg.own(k);
                un0[k] = o ? u[i0 + k] : 0.0;
                un1[k] = o ? u[N + i0 + k] : 0.0;
            }
            // the reverse sweep's last readers of the LDS edges are done
            __syncthreads();
            sg.publish(un0, un1);
            double cv0[P], cv1[P];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                cv0[k] = un0[k];
                cv1[k] = un1[k];
            }
#pragma unroll 1
            for (int s = 0; s < 4; ++s) {
                double r0[P], r1[P];
                // stores V_s, e^-delta and w as stage s of the scratch's record
                sg.template rhs<true>(false, false, cv0, cv1, r0, r1, uni(st), s);
                if (s < 3) {
                    const double c_next = (s == 2) ? dt : 0.5 * dt;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        cv0[k] = un0[k] + c_next * r0[k];
                        cv1[k] = un1[k] + c_next * r1[k];
                    }
                    sg.publish(cv0, cv1);
                }
            }
            load_e(uni(st + 3 * kStage));
            load_v(uni(st + 3 * kStage));
        }
        // reverse of U' = U + dt sum_s b_s k_s with stage inputs V_s = U + c_s dt k_{s-1}:
        // kbar_s = dt b_s U-bar' + c_{s+1} dt Vbar_{s+1}, U-bar = U-bar' + sum_s Vbar_s
        double kb0[P], kb1[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double u0 = ub(2, k), u1 = ub(3, k);
            kb0[k] = dt6 * u0;
            kb1[k] = dt6 * u1;
            ub(0, k) = kb0[k];
            ub(1, k) = kb1[k];
        }
        // the step before this one (at the segment's start: any record, its values unused)
        ADSCL_GLOBAL double* const before = (REC && t > 0) ? st - kRec : st;
#pragma unroll 1
        for (int s = 3; s >= 0; --s) {
            ADSCL_GLOBAL double* const next = uni((s > 0) ? st + (size_t)(s - 1) * kStage : before + 3 * kStage);
            own.fresh();
            double vb0[P], vb1[P];
            R::template stage_reverse<(TR < P ? TR : P)>(sg, v0, v1, E, w, kb0, kb1, ct2, vb0, vb1, lt, [&]() {
                // vector loads return in order: first what the next stage needs first
#pragma unroll
                for (int k = 0; k < P; ++k) ct2[k] = lt(2, k);
                load_e(next);
            });
            load_v(next);
            const double cs = (s == 3) ? dt : dt2;
            const double bp = (s == 1) ? 1.0 : 2.0;  // b_{s-1}, in sixths
#pragma unroll
            for (int k = 0; k < P; ++k) {
                ub(2, k) += vb0[k];
                ub(3, k) += vb1[k];
                kb0[k] = fma(cs, vb0[k], bp * ub(0, k));
                kb1[k] = fma(cs, vb1[k], bp * ub(1, k));
            }
        }
        st = before;
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if (sg.own(k)) {
            a.Ubar[ic.off + i0 + k] = ub(2, k);
            a.Ubar[a.total + ic.off + i0 + k] = ub(3, k);
        }
    }
}

// Adjoint at an end point: E_j = Pihat_j^2 + Phihat_j^2 with Pihat_j =
// sum_i wPi_ji sqrt(A_i) Pi_i, Phihat_j = sum_i wPhi_ji sqrt(A_i) Phi_i, then
// A = 1 - cos^3 x / sin x S / e^-delta through the constraint solve.
template <int P, int W, bool FULL>
__global__ void __launch_bounds__(64 * W) endpoint_kernel(EndArgs a)
{
    using R = Rev<P, W, FULL>;
    extern __shared__ double lds[];
    const int b = a.order[blockIdx.x];
    if (a.status[b].state != ST_DONE) return;
    const InstConst ic = a.ic[b];
    Stage<P, W, FULL> sg;
    sg.setup(lds, ic, a.tab[b], a.gauge, 0.0);
    const int N = sg.N, i0 = sg.i0, tid = sg.tid;
    const auto tb = sg.tables();

    double v0[P], v1[P], q[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const bool o = sg.own(k);
        v0[k] = o ? a.Phi[ic.off + i0 + k] : 0.0;
        v1[k] = o ? a.Pi[ic.off + i0 + k] : 0.0;
        q[k] = o ? fma(v0[k], v0[k], v1[k] * v1[k]) : 0.0;
    }
    double dl[P], E[P], S[P], dN, tot2;
    sg.constraints(q, dl, E, S, dN, tot2);

    double sp[P], sf[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        sp[k] = 0.0;
        sf[k] = 0.0;
    }
    const ADSCL_GLOBAL double* wp = gmem(a.wPi[b]);
    const ADSCL_GLOBAL double* wf = gmem(a.wPhi[b]);
    for (int m = 0; m < a.J; ++m) {
        const size_t bj = (size_t)b * a.J + m;
        const double eb = 2.0 * a.sgn * (a.ET[bj] - a.E0[bj]);
        const double ab = 2.0 * a.Pihat[bj] * eb;
        const double bb = 2.0 * a.Phihat[bj] * eb;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (sg.own(k)) {
                sp[k] += ab * wp[(size_t)m * N + i0 + k];
                sf[k] += bb * wf[(size_t)m * N + i0 + k];
            }
        }
    }
    double vb0[P], vb1[P], Eb[P], Sb[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const double c3s = sg.tab(tb, 2, k) * sg.tab(tb, 0, k);
        const double Ak = 1.0 - c3s * (S[k] / E[k]);
        const double sA = sqrt(Ak);
        const bool o = sg.own(k);
        vb0[k] = o ? sA * sf[k] : 0.0;
        vb1[k] = o ? sA * sp[k] : 0.0;
        const double Ab = o ? (sp[k] * v1[k] + sf[k] * v0[k]) / (2.0 * sA) : 0.0;
        // A = 1 - c3s S / E
        Eb[k] = o ? c3s * S[k] * Ab / (E[k] * E[k]) : 0.0;
        Sb[k] = o ? -c3s * Ab / E[k] : 0.0;
    }
    __syncthreads();  // the solve's readers of the edge and reduction slots are done
    R::constraint_reverse(
        sg, v0, v1, E, Eb, Sb, vb0, vb1, [&](int f, int k) -> double { return sg.tab(tb, f, k); }, [] {});
    if (tid == 0) vb0[0] = 0.0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if (sg.own(k)) {
            a.Ubar[ic.off + i0 + k] += vb0[k];
            a.Ubar[a.total + ic.off + i0 + k] += vb1[k];
        }
    }
}

__global__ void adj_prepare_kernel(int n_inst, const InstConst* ic, const InstStatus* st, int64_t K, int64_t r,
                                   InstStatus* rst, AdjSeg* sg)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst) return;
    const int64_t nf = ic[b].n_final;
    const int64_t n1 = nf - r * K;
    const bool act = st[b].state == ST_DONE && n1 > 0;
    AdjSeg g;
    g.n0 = act && n1 > K ? n1 - K : 0;
    g.n1 = act ? n1 : 0;
    g.active = act ? 1 : 0;
    g.pad = 0;
    sg[b] = g;
    InstStatus o;
    o.steps = g.n0;
    o.target = g.n1;
    o.t_c = -1.0;
    o.minA = 1.0;
    o.mass = 0.0;
    o.state = act ? ST_RUNNING : ST_COLLAPSED;
    o.pad = 0;
    rst[b] = o;
}

// One 256-thread block per instance.
__global__ void __launch_bounds__(256) adj_finish_kernel(int n_inst, const InstConst* ic, const InstStatus* st,
                                                         const double* Ubar, int64_t total,
                                                         const double* const* emode, const double* eps, int Jc,
                                                         const double* E0, const double* ET, int J, double* L,
                                                         double* dLdc, int32_t* valid)
{
    __shared__ double sh[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const InstConst c = ic[b];
    const bool ok = st[b].state == ST_DONE;
    const double* pib = Ubar + total + c.off;
    for (int k = 0; k < Jc; ++k) {
        const double* e = emode[b] + (size_t)k * c.N;
        double s = 0.0;
        for (int i = tid; i <= c.N - 2; i += 256) s += pib[i] * e[i];
        for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
        if ((tid & 63) == 0) sh[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) dLdc[(size_t)b * Jc + k] = ok ? eps[b] * ((sh[0] + sh[1]) + (sh[2] + sh[3])) : 0.0;
        __syncthreads();
    }
    if (tid == 0) {
        double l = 0.0;
        for (int j = 0; j < J; ++j) {
            const double d = ET[(size_t)b * J + j] - E0[(size_t)b * J + j];
            l += d * d;
        }
        L[b] = l;
        valid[b] = ok ? 1 : 0;
    }
}

// Device fill (used instead of a memset so that the enqueue sequence can be
// captured into a graph).
__global__ void fill_kernel(double* p, int64_t n, double v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void mask_kernel(int n_inst, InstStatus* st, const int32_t* active)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst || active[b]) return;
    InstStatus o = st[b];
    o.state = ST_COLLAPSED;
    st[b] = o;
}

__global__ void gd_init_kernel(int n_inst, double step0, GdState g)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b == 0) g.iter[0] = 0;
    if (b >= n_inst) return;
    g.s[b] = step0;
    g.Lprev[b] = INFINITY;
    g.active[b] = 1;
}

// One thread per instance: the descent step of iteration g.iter[0].
__global__ void gd_update_kernel(int n_inst, int Jc, double* c, const double* grad, const double* L,
                                 const int32_t* valid, GdState g, double* L_hist)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_inst) return;
    const int it = g.iter[0];
    double* lh = L_hist + (size_t)it * n_inst + b;
    if (!g.active[b]) {
        *lh = NAN;
        return;
    }
    const double l = L[b];
    *lh = l;
    if (!valid[b]) {
        g.active[b] = 0;
        return;
    }
    double s = g.s[b];
    if (l > g.Lprev[b]) s *= 0.5;
    g.s[b] = s;
    g.Lprev[b] = l;
    double* cb = c + (size_t)b * Jc;
    const double* gb = grad + (size_t)b * Jc;
    double cn = 0.0, gn = 0.0;
    for (int k = 0; k < Jc; ++k) {
        cn += cb[k] * cb[k];
        gn += gb[k] * gb[k];
    }
    if (gn > 0.0) {
        const double f = s * sqrt(cn) / sqrt(gn);
        for (int k = 0; k < Jc; ++k) cb[k] -= f * gb[k];
    }
}

__global__ void gd_tick_kernel(GdState g)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) g.iter[0] += 1;
}

template <int P, int W, bool FULL>
constexpr size_t end_lds_bytes()
{
    return Stage<P, W, FULL>::lds_doubles * sizeof(double);
}

template <int P, int W, bool FULL>
void launch_adj_f(int n_blocks, const AdjointArgs& a, hipStream_t s)
{
    const dim3 g(n_blocks), t(64 * W);
    if (a.keep) adjoint_kernel<P, W, FULL, true><<<g, t, adj_lds_bytes<P, W, FULL>(), s>>>(a);
    else adjoint_kernel<P, W, FULL, false><<<g, t, adj_lds_bytes<P, W, FULL>(), s>>>(a);
}

template <int P, int W>
hipError_t launch_adj_t(bool full, int n_blocks, const AdjointArgs& a, hipStream_t s)
{
    if (full) launch_adj_f<P, W, true>(n_blocks, a, s);
    else launch_adj_f<P, W, false>(n_blocks, a, s);
    return hipGetLastError();
}

template <int P, int W>
hipError_t launch_end_t(bool full, int n_blocks, const EndArgs& a, hipStream_t s)
{
    if (full)
        endpoint_kernel<P, W, true><<<dim3(n_blocks), dim3(64 * W), end_lds_bytes<P, W, true>(), s>>>(a);
    else
        endpoint_kernel<P, W, false><<<dim3(n_blocks), dim3(64 * W), end_lds_bytes<P, W, false>(), s>>>(a);
    return hipGetLastError();
}

template <int P, int W>
hipError_t prepare_adj_t(size_t max_lds)
{
    const void* fns[] = {(const void*)adjoint_kernel<P, W, true, true>,   (const void*)adjoint_kernel<P, W, true, false>,
                         (const void*)adjoint_kernel<P, W, false, true>,  (const void*)adjoint_kernel<P, W, false, false>,
                         (const void*)endpoint_kernel<P, W, true>,        (const void*)endpoint_kernel<P, W, false>};
    const size_t af = adj_lds_bytes<P, W, true>(), ar = adj_lds_bytes<P, W, false>();
    const size_t need[] = {af, af, ar, ar, end_lds_bytes<P, W, true>(), end_lds_bytes<P, W, false>()};
    for (int i = 0; i < 6; ++i) {
        if (need[i] > max_lds) return hipErrorInvalidValue;
        hipError_t e = hipFuncSetAttribute(fns[i], hipFuncAttributeMaxDynamicSharedMemorySize, (int)need[i]);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

#define ADSCL_ADJ_CLASSES(X) \
    X(4, 1)                  \
    X(4, 2)                  \
    X(4, 4)                  \
    X(4, 8)                  \
    X(4, 16)                 \
    X(8, 1)                  \
    X(8, 2)                  \
    X(8, 4)                  \
    X(8, 8)                  \
    X(16, 1)                 \
    X(16, 2)                 \
    X(16, 4)

size_t adjoint_scratch_len(ClassCfg c) { return (size_t)kFields * c.P * 64 * c.W; }
size_t stage_record_len(ClassCfg c) { return (size_t)16 * c.P * 64 * c.W; }

hipError_t prepare_adjoint(ClassCfg c, size_t max_lds)
{
#define X(p, w) \
    if (c.P == p && c.W == w) return prepare_adj_t<p, w>(max_lds);
    ADSCL_ADJ_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint(ClassCfg c, bool full, int n_blocks, const AdjointArgs& a, hipStream_t s)
{
#define X(p, w) \
    if (c.P == p && c.W == w) return launch_adj_t<p, w>(full, n_blocks, a, s);
    ADSCL_ADJ_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_endpoint(ClassCfg c, bool full, int n_blocks, const EndArgs& a, hipStream_t s)
{
#define X(p, w) \
    if (c.P == p && c.W == w) return launch_end_t<p, w>(full, n_blocks, a, s);
    ADSCL_ADJ_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_adj_prepare(int n_inst, const InstConst* ic, const InstStatus* st, int64_t K, int64_t r,
                              InstStatus* rst, AdjSeg* sg, hipStream_t s)
{
    adj_prepare_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, ic, st, K, r, rst, sg);
    return hipGetLastError();
}

hipError_t launch_fill(double* p, int64_t n, double v, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    fill_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_mask(int n_inst, InstStatus* st, const int32_t* active, hipStream_t s)
{
    mask_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, st, active);
    return hipGetLastError();
}

hipError_t launch_gd_init(int n_inst, double step0, const GdState& g, hipStream_t s)
{
    gd_init_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, step0, g);
    return hipGetLastError();
}

hipError_t launch_gd_update(int n_inst, int Jc, double* c, const double* grad, const double* L, const int32_t* valid,
                            const GdState& g, double* L_hist, hipStream_t s)
{
    gd_update_kernel<<<dim3((n_inst + 255) / 256), dim3(256), 0, s>>>(n_inst, Jc, c, grad, L, valid, g, L_hist);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    gd_tick_kernel<<<dim3(1), dim3(64), 0, s>>>(g);
    return hipGetLastError();
}

hipError_t launch_adj_finish(int n_inst, const InstConst* ic, const InstStatus* st, const double* Ubar,
                             int64_t total, const double* const* emode, const double* eps, int Jc,
                             const double* E0, const double* ET, int J, double* L, double* dLdc,
                             int32_t* valid, hipStream_t s)
{
    adj_finish_kernel<<<dim3(n_inst), dim3(256), 0, s>>>(n_inst, ic, st, Ubar, total, emode, eps, Jc, E0, ET, J, L,
                                                        dLdc, valid);
    return hipGetLastError();
}

}  // namespace adscl
