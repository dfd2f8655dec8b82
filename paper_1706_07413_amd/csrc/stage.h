// One workgroup's view of one instance during an RK4 stage of the AdS4
// Einstein-Klein-Gordon evolution (Liebling & Khanna, arXiv:1706.07413,
// Sec. II), shared by the forward evolution kernel and the reverse (adjoint)
// kernel, which recomputes forward stages.
//
// Lane l of the workgroup owns the P consecutive grid points l*P .. l*P+P-1 and
// keeps them in registers; neighbours' edge points cross lanes by DPP, and
// wavefronts through small LDS slots.
//
// Prefix-sum form of the cell rule: with C_i = h(-u_{i-1}+13u_i+13u_{i+1}-u_{i+2})/24
// and R_k = sum_{j<=k} u_j,
//   sum_{i<k} C_i = h/24 (24 R_k - 12 u_k + u_{k-1} - u_{k+1} - u_{-1} - 12 u_0 + u_1),
// the same sum of cells regrouped; for p (odd about 0, p_0 = 0) the last three
// terms are 2 p_1, for sigma (even, sigma_0 = 0) they vanish.
// The gauge shift is applied before the exponential: e^{-delta} with delta =
// delta~ - delta~_{N-1} (boundary time, Eq. (12)) or delta = delta~ (origin
// time); S, e^{-delta} and so A e^{-delta} scale consistently, and m = S/e^{-delta}
// does not depend on the shift, so one exponential per point suffices.
#pragma once

#include <math.h>

#include "internal.h"

namespace adscl {

// Global-memory (address space 1) view of a device pointer.  A pointer read
// from a per-instance pointer array is generic to the compiler, which then
// emits flat memory instructions (64-bit VGPR addresses per access, counted
// against the LDS wait counter as well); through this cast it emits global ones.
#define ADSCL_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ ADSCL_GLOBAL T* gmem(T* p)
{
    return (ADSCL_GLOBAL T*)p;
}

// DPP move of a double: both 32-bit halves through the same data-parallel
// primitive (lanes without a source read 0).  With every row enabled the
// zero comes from the bound control, so no destination has to be cleared
// first; a partial row mask keeps the old value (0) in the masked rows.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double v)
{
    constexpr bool bc = ROW_MASK == 0xf;
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, bc);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, bc);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// DPP move of a double where lanes without a source lane keep `old`.
template <int CTRL>
__device__ __forceinline__ double dpp_old(double old, double v)
{
    const long long o = __double_as_longlong(old), b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)(o & 0xffffffffll), (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// e^x by Tang's table-driven method (P. T. P. Tang, ACM Trans. Math. Softw. 15
// (1989) 144-157): x = (64 m + j) ln 2/64 + r with |r| <= ln 2/128, so that
// e^x = 2^m 2^(j/64) e^r.  r is formed against a two-part ln 2/64 (the second
// part holds the bits the first drops), e^r - 1 is its degree-5 Taylor
// polynomial (truncation below r^6/720 < 4e-17), and the 64 values 2^(j/64)
// come from a table (t64, in LDS).  Arguments below -746 are raised to -746
// (e^x is 0 in double there), and so is a NaN (the constraint solve tests q,
// e^-delta and delta~_{N-1} for finiteness itself); up to x = 2.3e7 it is
// e^x within about 2 ulp (1.3 ulp over [-700, 700] with correctly rounded table
// entries; the table's own exp2 adds at most its error), overflowing to +inf
// through the exponent m, and past that it is not finite.
__device__ __forceinline__ double exp_tab(double x, const double* t64)
{
    x = __builtin_fmax(x, -746.0);
    const double n = __builtin_rint(x * 0x1.71547652b82fep+6);  // 64/ln 2
    double r = __builtin_fma(-n, 0x1.62e42fefa39efp-7, x);       // ln 2/64, leading part
    r = __builtin_fma(-n, 0x1.abc9e3b39803fp-62, r);             // and the rest
    const int ni = (int)n;
    double e = __builtin_fma(r, 1.0 / 120.0, 1.0 / 24.0);
    e = __builtin_fma(r, e, 1.0 / 6.0);
    e = __builtin_fma(r, e, 0.5);
    e = __builtin_fma(r, e, 1.0);
    e *= r;  // e^r - 1
    const double t = t64[ni & 63];
    return __builtin_ldexp(__builtin_fma(t, e, t), ni >> 6);
}

// Double of lane `l` (wavefront-uniform) broadcast to every lane.
__device__ __forceinline__ double readlane_d(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Inclusive prefix sum over the 64 lanes of a wavefront: shifts by 1, 2, 4, 8
// within rows of 16 lanes, then the row totals through the row broadcasts of
// lanes 15 and 31 (gfx9 DPP row_shr / row_bcast).
__device__ __forceinline__ double wave_incl_scan(double v)
{
    v += dpp_d<0x111, 0xf>(v);  // row_shr:1
    v += dpp_d<0x112, 0xf>(v);  // row_shr:2
    v += dpp_d<0x114, 0xf>(v);  // row_shr:4
    v += dpp_d<0x118, 0xf>(v);  // row_shr:8
    v += dpp_d<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_d<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Inclusive suffix sum over the 64 lanes of a wavefront (lane l: the sum over
// lanes l..63): shifts from higher lanes by 1, 2, 4, 8 within rows of 16 lanes
// (DPP row_shl; lanes past a row's end read 0), then the totals of the rows to
// the right, the outermost first, read from each row's first lane.  Every
// partial result is a sum over a run of lanes to the right, so no total is ever
// subtracted: a suffix keeps its own precision even when the terms left of it
// are far larger (the adjoint of the constraint solve meets cotangents of order
// 1/e^-delta at the origin of strong fields).
__device__ __forceinline__ double wave_incl_suffix(double v)
{
    v += dpp_d<0x101, 0xf>(v);  // row_shl:1
    v += dpp_d<0x102, 0xf>(v);  // row_shl:2
    v += dpp_d<0x104, 0xf>(v);  // row_shl:4
    v += dpp_d<0x108, 0xf>(v);  // row_shl:8
    const int row = (threadIdx.x & 63) >> 4;
    const double t3 = readlane_d(v, 48), t2 = readlane_d(v, 32), t1 = readlane_d(v, 16);
    double right = (row < 3) ? t3 : 0.0;
    if (row < 2) right += t2;
    if (row < 1) right += t1;
    return v + right;
}

// Sums of the wavefront totals r[0..W): over the wavefronts before this one
// (`before`) and over all (`all`).  Lanes v < W hold r[v], a DPP prefix
// runs over them (W <= 16: within the first row of 16 lanes), and two
// wavefront-uniform lane reads broadcast the results, instead of every lane
// adding all W totals under a mask.
template <int W>
__device__ __forceinline__ void wave_totals(const double* r, int lane, int wv, double& before, double& all)
{
    double x = (lane < W) ? r[lane < W ? lane : 0] : 0.0;
    if constexpr (W > 1) x += dpp_d<0x111, 0xf>(x);  // row_shr:1
    if constexpr (W > 2) x += dpp_d<0x112, 0xf>(x);  // row_shr:2
    if constexpr (W > 4) x += dpp_d<0x114, 0xf>(x);  // row_shr:4
    if constexpr (W > 8) x += dpp_d<0x118, 0xf>(x);  // row_shr:8
    all = readlane_d(x, W - 1);
    const int w = __builtin_amdgcn_readfirstlane(wv);
    before = (w > 0) ? readlane_d(x, w > 0 ? w - 1 : 0) : 0.0;
}

// A lane-interleaved global array of doubles, [field][P][64 W]: entry (f, k) of
// lane l at ((f P + k) 64 W + l).  Held as a uniform base and the lane's byte
// offset, the latter opaque to the compiler, so that each access is a scalar
// base plus a 32-bit vector offset formed where it is used (rather than a
// 64-bit address per entry computed once and kept, or spilled, for the whole
// kernel).  Make a fresh view per phase with lane_arr().
template <int P, int NL>
struct LaneArr {
    ADSCL_GLOBAL char* base;
    unsigned o;
    __device__ __forceinline__ ADSCL_GLOBAL double* at(int f, int k) const
    {
        return (ADSCL_GLOBAL double*)(base + (o + (unsigned)((f * P + k) * NL * 8)));
    }
    __device__ __forceinline__ double ld(int f, int k) const { return *at(f, k); }
    __device__ __forceinline__ void st(int f, int k, double v) const { *at(f, k) = v; }
};

template <int P, int NL>
__device__ __forceinline__ LaneArr<P, NL> lane_arr(ADSCL_GLOBAL double* base, int lane_id)
{
    unsigned o = (unsigned)lane_id * 8u;
    asm volatile("" : "+v"(o));
    return LaneArr<P, NL>{(ADSCL_GLOBAL char*)base, o};
}

// One step's stage record for the adjoint: for RK stage s (0..3) and point k of
// lane l, the stage input (Phi, Pi) in plane 0 and (e^-delta, w = A e^-delta) in plane 1,
// [s][plane][P][64 W] pairs of doubles, so that a wavefront's access to either
// pair of a point is 1 KB of whole lines and each plane can be loaded when its
// registers fall free.  The same opaque lane offset as LaneArr, on a base that
// is uniform for each (plane, k).
typedef double pair_t __attribute__((ext_vector_type(2)));
template <int P, int NL>
struct StageRec {
    ADSCL_GLOBAL char* base;
    unsigned o;
    __device__ __forceinline__ ADSCL_GLOBAL pair_t* at(int plane, int k) const
    {
        ADSCL_GLOBAL char* p = base + (unsigned)((plane * P + k) * NL * 16);
        asm("" : "+s"(p));  // a scalar address, not one more vector add
        return (ADSCL_GLOBAL pair_t*)(p + o);
    }
    __device__ __forceinline__ pair_t ld(int plane, int k) const { return *at(plane, k); }
    __device__ __forceinline__ void st(int k, double v0, double v1, double e, double w) const
    {
        *at(0, k) = pair_t{v0, v1};
        *at(1, k) = pair_t{e, w};
    }
};

// The stage's part of a record, at the uniform address `stage`, as seen by a lane.
template <int P, int NL>
__device__ __forceinline__ StageRec<P, NL> stage_rec(ADSCL_GLOBAL double* stage, int lane_id)
{
    unsigned o = (unsigned)lane_id * 16u;
    asm volatile("" : "+v"(o));
    return StageRec<P, NL>{(ADSCL_GLOBAL char*)stage, o};
}

template <int P, int W, bool FULL, bool FWD = false>
struct Stage {
    static constexpr int NL = 64 * W;
    static_assert(P >= 4, "lane 0 must own grid points 0..3");

    // Lanes keep their own points in registers and take
    // their neighbours' edge values (the last / first three stage-input points,
    // p and sigma, the last / first two fluxes) across lanes with DPP wavefront
    // shifts; only lanes 0 and 63 go through small LDS slots (X*, and R* for the
    // adjoint's transposed stencils and reverse scans) to reach the adjacent
    // wavefront.
    // The forward kernels (FWD) keep the coefficient tables in LDS; the
    // adjoint reads them from global memory and keeps its own state in LDS.
    // On grids that do not fill the lanes (RAG) points past
    // N - 2 stay 0, and what their images past pi/2 would have added to the stencils of
    // the last points is added to the right-hand sides afterwards (end_terms): the
    // place of the end within a lane is not known at compile time, and choosing
    // registers by it costs more instructions than the whole correction.
    // Measured, one instance of 3001 / 2001 / 1001 / 201 points: 17.9, 12.3, 9.1 and
    // 8.1 us per step, against 28.6, 19.2, 10.5 and 9.1 with whole rows in LDS, a fourth
    // barrier per stage and the tables in L2 (full lanes: 15.6 at 4097, 8.2 at 1025).
    static constexpr bool RAG = !FULL;
    static constexpr size_t lds_doubles = (size_t)44 * (W + 2) + (FWD ? 0 : 20 * (W + 2)) + (RAG ? 20 * P : 0)
                                          + (FWD ? (size_t)3 * P * NL : 0) + 4 * W + 8 + 64;

    // Edge slots, one per wavefront (slot wv + 1) plus two ghost slots: slot 0
    // holds the parity images left of x = 0 as if a wavefront -1 had written
    // them, slot W + 1 the end point and its images past pi/2, so that every
    // wavefront reads its two neighbours' slots the same way
    double2* XU;    // [2 buffers][W+2][6] points 0..2 of lane 0, then P-1..P-3 of lane 63
    double* XP;     // [W+2][2] p of the first point of lane 0, of the last point of lane 63
    double* XS;     // [W+2][2] the same for sigma
    double2* XF;    // [2 buffers][W+2][4] fluxes of points 0, 1 of lane 0 and P-1, P-2 of lane 63;
                    // the buffer follows XU's, since with the metric frozen B3 is the only
                    // barrier of a stage and a wavefront may write its next stage's fluxes
                    // while its neighbour still reads this stage's
    // the adjoint's slots, laid out the same way, their ghosts 0 throughout:
    double2* RU;    // [W+2][6] row cotangents (Phi_t, Pi_t) of points 0..2 of lane 0, P-1..P-3 of lane 63
    double* RF;     // [W+2][4] cotangents of the D g rows, points 0, 1 of lane 0, P-1, P-2 of lane 63
    double* RSb;    // [W+2][2] S-bar of the first point of lane 0, of the last point of lane 63
    double* RDt;    // [W+2][2] the same for the delta~ cotangents
    // RAG: the points of the two lanes from jb on that hold N - 4 .. N - 2
    double2* GU;    // [2 buffers][2 P] their stage input
    double2* GF;    // [2 buffers][2 P] their fluxes
    double2* GR;    // [2 P] what end_terms adds to their right-hand sides
    double* T;      // FWD: the coefficient tables, [3][P][64 W] as in global memory
    double* red;    // [0,W) delta~ totals, [W,2W) S totals, [2W,3W) flags (the adjoint: cotangent totals),
                    // [3W,4W) the adjoint's origin cotangent, 4W: p_1, 4W+1: p_{N-2}
    double* X64;    // 2^(j/64), j = 0..63, the table of exp_tab
    int tid, lane, wv, i0, N;
    int buf;        // XU buffer of the last publish
    bool has_nm2, near_end, bgauge;
    int jb;         // RAG: see GU
    bool at_end;    // RAG: this lane holds points past N - 2 that a stencil from the last points reaches
    double h, dt, h24, i12h, kof, thr;
    const ADSCL_GLOBAL double* tab0;

    __device__ __forceinline__ void setup(double* lds, const InstConst& ic, const double* tab, int gauge,
                                          double a_collapse)
    {
        setup(lds, ic, tab, gauge, a_collapse, (int)threadIdx.x);
    }

    // t: the thread's index within the 64 W threads that run the instance (the
    // workgroup's own index unless the workgroup runs several instances).
    __device__ __forceinline__ void setup(double* lds, const InstConst& ic, const double* tab, int gauge,
                                          double a_collapse, int t)
    {
        double* p = lds;
        XU = reinterpret_cast<double2*>(p);
        p += 24 * (W + 2);
        XP = p;
        p += 2 * (W + 2);
        XS = p;
        p += 2 * (W + 2);
        XF = reinterpret_cast<double2*>(p);
        p += 16 * (W + 2);
        RU = GU = GF = GR = nullptr;
        RF = RSb = RDt = T = nullptr;
        if constexpr (!FWD) {
            RU = reinterpret_cast<double2*>(p);
            p += 12 * (W + 2);
            RF = p;
            p += 4 * (W + 2);
            RSb = p;
            p += 2 * (W + 2);
            RDt = p;
            p += 2 * (W + 2);
        }
        if (RAG) {
            GU = reinterpret_cast<double2*>(p);
            GF = GU + 4 * P;
            GR = GF + 4 * P;
            p += 20 * P;
        }
        if (FWD) {
            T = p;
            p += 3 * P * NL;
        }
        red = p;
        X64 = red + 4 * W + 8;
        buf = 0;
        tid = t;
        // read only after the barrier of the first constraint solve
        if (tid < 64) X64[tid] = exp2((double)tid * (1.0 / 64.0));
        lane = tid & 63;
        wv = tid >> 6;
        N = ic.N;
        h = ic.h;
        dt = ic.dt;
        h24 = ic.h24;
        i12h = ic.i12h;
        kof = ic.kof;
        thr = a_collapse;
        bgauge = gauge == 0;
        i0 = tid * P;
        // FULL: N - 1 == 64 W P, so every lane owns P evolved points and the
        // last lane owns N-4..N-2; otherwise lanes past N-2 idle and the end moves.
        has_nm2 = FULL ? (tid == NL - 1) : ((i0 <= N - 2) && (N - 2 < i0 + P));
        near_end = FULL ? (tid == NL - 1) : ((i0 + P + 2 >= N - 4) && (i0 <= N - 2));
        at_end = false;
        jb = 0;
        if constexpr (RAG) {
            jb = ((N - 2) / P - 1) * P;
            near_end = i0 >= jb && i0 <= N - 2;  // the two lanes
            at_end = i0 + P > N - 1 && i0 <= N + 1;
            // past the last lane: zeros, as in every lane past the end
            if (tid == 0) XP[2 * (W + 1)] = XS[2 * (W + 1)] = 0.0;
            if (tid < 12) XU[(tid / 6 * (W + 2) + W + 1) * 6 + tid % 6] = make_double2(0.0, 0.0);
            if (tid < 8) XF[(tid / 4 * (W + 2) + W + 1) * 4 + tid % 4] = make_double2(0.0, 0.0);
            if (tid < 2 * P) GR[tid] = make_double2(0.0, 0.0);
        }
        if constexpr (!FWD) {  // the ghost slots, read after a later barrier
            if (tid < 12) RU[tid / 6 * (W + 1) * 6 + tid % 6] = make_double2(0.0, 0.0);
            if (tid < 8) RF[tid / 4 * (W + 1) * 4 + tid % 4] = 0.0;
            if (tid < 4) RSb[tid / 2 * (W + 1) * 2 + tid % 2] = RDt[tid / 2 * (W + 1) * 2 + tid % 2] = 0.0;
        }
        tab0 = gmem(tab);
        if constexpr (FWD) {
            // each lane copies exactly the entries it reads later, so no barrier
#pragma unroll
            for (int t = 0; t < 3 * P; ++t) T[t * NL + tid] = tab0[t * NL + tid];
        }
    }

    // Value of v at the lane to the left (tid - 1) / right (tid + 1) within the
    // wavefront (DPP wave_shr:1 / wave_shl:1); lanes 0 / 63 get 0.  All lanes
    // must be active.
    static __device__ __forceinline__ double from_left(double v) { return dpp_d<0x138, 0xf>(v); }
    static __device__ __forceinline__ double from_right(double v) { return dpp_d<0x130, 0xf>(v); }

    __device__ __forceinline__ bool own(int k) const { return FULL || (i0 + k <= N - 2); }

    // The place of pi/2 relative to the lane's first point, opaque to the compiler:
    // conditions on single points are then formed where they are used, by the
    // wavefronts that meet them, instead of being kept as lane masks for the
    // whole kernel (which spills scalar registers).
    __device__ __forceinline__ int end_here() const
    {
        int e = N - 1 - i0;
        asm volatile("" : "+v"(e));
        return e;
    }

    // RAG: the points past N - 2 back to 0, and the terms of the images past pi/2
    // (Phi even, Pi odd, f1 odd, g even about it; Phi = Pi = f1 = 0 there, g the even
    // 6th-order extrapolation) in the stencils of N - 2 and N - 3.
    __device__ __forceinline__ void end_terms(double* r0, double* r1) const
    {
        if (at_end) {
            const int e = end_here();
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k >= e) r0[k] = r1[k] = 0.0;
        }
        if (near_end) {
            const int e = N - 2 - jb;
            const double2 *gu = GU + buf * 2 * P + e, *gf = GF + buf * 2 * P + e;
            const double2 v2 = gu[0], v3 = gu[-1], f2 = gf[0], f3 = gf[-1], f4 = gf[-2];
            const int l2 = (N - 2) / P, l3 = (N - 3) / P;
            const int e2 = (2 * P + (N - 2) - l2 * P) * NL + l2, e3 = (2 * P + (N - 3) - l3 * P) * NL + l3;
            const double c2 = FWD ? T[e2] : tab0[e2], c3 = FWD ? T[e3] : tab0[e3];
            const double gext = (fma(15.0, f2.y, -6.0 * f3.y) + f4.y) / 10.0;
            // both lanes write the same; each then reads its own points
            GR[e] = make_double2(fma(kof, fma(-6.0, v2.x, v3.x), i12h * f2.x),
                                 fma(kof, fma(6.0, v2.y, -v3.y), c2 * (i12h * fma(8.0, gext, -f2.y))));
            GR[e - 1] = make_double2(kof * v2.x, fma(-kof, v2.y, c3 * (-i12h * gext)));
            const double2* const gr = GR + (i0 - jb);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double2 g = gr[k];
                r0[k] += g.x;
                r1[k] += g.y;
            }
        }
    }

    // Per-stage view of the coefficient tables: a uniform base and the lane's
    // byte offset, opaque to the compiler so that table loads are issued again
    // in each stage (L2 hits) instead of being held in registers across the
    // time loop, and take the scalar-base plus 32-bit vector-offset form.
    struct TabView {
        const ADSCL_GLOBAL char* base;
        unsigned o;
    };
    __device__ __forceinline__ TabView tables() const
    {
        unsigned o = (unsigned)tid * 8u;
        asm volatile("" : "+v"(o));
        return TabView{(const ADSCL_GLOBAL char*)tab0, o};
    }

    // Table t (0 sin x cos x, 1 tan^2 x, 2 cot^2 x) at the lane's point k.
    __device__ __forceinline__ double tab(const TabView& v, int t, int k) const
    {
        if constexpr (FWD) return T[(t * P + k) * NL + tid];
        return *(const ADSCL_GLOBAL double*)(v.base + (v.o + (unsigned)((t * P + k) * NL * 8)));
    }

    // Publish (v0, v1) = (Phi, Pi) of the own points with parity ghosts:
    // Phi odd / Pi even about x = 0, Phi even / Pi odd about pi/2, Phi = Pi = 0 at pi/2.
    __device__ __forceinline__ void publish(const double* v0, const double* v1)
    {
        // neighbours within the wavefront read the registers; lanes 0 and 63
        // leave their edge points for the adjacent wavefronts
        buf ^= 1;
        double2* xu = XU + (buf * (W + 2) + wv + 1) * 6;
        if (lane == 0) {
#pragma unroll
            for (int r = 0; r < 3; ++r) xu[r] = make_double2(v0[r], v1[r]);
        }
        if (lane == 63) {
#pragma unroll
            for (int r = 0; r < 3; ++r) xu[3 + r] = make_double2(v0[P - 1 - r], v1[P - 1 - r]);
        }
        if (tid == 0) {  // Phi odd, Pi even about x = 0: points -1, -2, -3
            double2* g = XU + buf * (W + 2) * 6;
#pragma unroll
            for (int r = 0; r < 3; ++r) g[3 + r] = make_double2(-v0[1 + r], v1[1 + r]);
        }
        if (FULL && tid == NL - 1) {  // Phi = Pi = 0 at pi/2; Phi even, Pi odd about it; points N-1, N, N+1
            double2* g = XU + (buf * (W + 2) + W + 1) * 6;
            g[0] = make_double2(0.0, 0.0);
            g[1] = make_double2(v0[P - 1], -v1[P - 1]);
            g[2] = make_double2(v0[P - 2], -v1[P - 2]);
        }
        if constexpr (RAG) {
            if (near_end) {
#pragma unroll
                for (int k = 0; k < P; ++k) GU[buf * 2 * P + i0 - jb + k] = make_double2(v0[k], v1[k]);
            }
        }
    }

    __device__ __forceinline__ void wave_totals(const double* r, double& before, double& all) const
    {
        adscl::wave_totals<W>(r, lane, wv, before, all);
    }

    // Constraint solve of the published state given q = Phi^2 + Pi^2 of the own
    // points (Eqs. (5)-(6)): delta (gauge applied), e^{-delta} and S at own
    // points, the delta~ end value dN and the S total tot2.  Contains barriers
    // B1 and B2.
    __device__ __forceinline__ void constraints(const double* q, double* dl, double* E, double* S, double& dN,
                                                double& tot2)
    {
        const auto tb = tables();
        double p[P];
        double ptot = 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            p[k] = tab(tb, 0, k) * q[k];  // table is 0 off 1..N-2
            ptot += p[k];
        }
        const double incl = wave_incl_scan(ptot);
        if (lane == 63) red[wv] = incl;
        if (lane == 0) XP[2 * (wv + 1)] = p[0];
        if (lane == 63) XP[2 * (wv + 1) + 1] = p[P - 1];
        if (tid == 0) XP[1] = -p[1];                // p_{-1} = -p_1
        if (FULL && tid == NL - 1) XP[2 * (W + 1)] = 0.0;  // p_{N-1} = 0
        if (tid == 0) red[4 * W] = p[1];
        if (FULL) {
            if (tid == NL - 1) red[4 * W + 1] = p[P - 1];
        } else if (has_nm2) {
            const int e = end_here() - 1;
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k == e) red[4 * W + 1] = p[k];
        }
        __syncthreads();  // B1
        double carry, tot;
        wave_totals(red, carry, tot);
        carry += incl - ptot;
        const double p1 = red[4 * W], pN2 = red[4 * W + 1];
        double pl, pr;
        // lanes 0 / 63 take the neighbouring wavefront's (or the ghost) slot
        pl = dpp_old<0x138>(XP[2 * wv + 1], p[P - 1]);
        pr = dpp_old<0x130>(XP[2 * (wv + 2)], p[0]);
        dN = -h24 * fma(24.0, tot, 2.0 * pN2 + 2.0 * p1);        // delta~_{N-1}
        const double shift = bgauge ? dN : 0.0;
        // -delta = h24 (24 R - 12 p + p_m - p_p + 2 p_1) + shift, with h24
        // distributed over the terms: one add and three FMAs per point
        const double a24 = 24.0 * h24, a12 = -12.0 * h24, c0 = fma(2.0 * h24, p1, shift);

        double sg[P];
        double R = carry, stot = 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            R += p[k];
            const double pm = (k == 0) ? pl : p[k - 1];
            const double pp = (k == P - 1) ? pr : p[k + 1];
            const double nd = fma(a24, R, fma(a12, p[k], fma(h24, pm - pp, c0)));
            dl[k] = -nd;
            E[k] = exp_tab(nd, X64);
            sg[k] = tab(tb, 1, k) * q[k] * E[k];  // table is 0 off 1..N-2
            stot += sg[k];
        }
        const double incl2 = wave_incl_scan(stot);
        if (lane == 63) red[W + wv] = incl2;
        if (lane == 0) XS[2 * (wv + 1)] = sg[0];
        if (lane == 63) XS[2 * (wv + 1) + 1] = sg[P - 1];
        if (tid == 0) XS[1] = sg[1];                // sigma_{-1} = sigma_1
        if (FULL && tid == NL - 1) XS[2 * (W + 1)] = 0.0;  // sigma_{N-1} = 0
        __syncthreads();  // B2
        double carry2;
        wave_totals(red + W, carry2, tot2);
        carry2 += incl2 - stot;
        double sl, sr;
        sl = dpp_old<0x138>(XS[2 * wv + 1], sg[P - 1]);
        sr = dpp_old<0x130>(XS[2 * (wv + 2)], sg[0]);
        double R2 = carry2;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            R2 += sg[k];
            const double sm = (k == 0) ? sl : sg[k - 1];
            const double sp = (k == P - 1) ? sr : sg[k + 1];
            // h24 (24 R2 - 12 sigma + sigma_m - sigma_p), h24 distributed
            S[k] = fma(a24, R2, fma(a12, sg[k], h24 * (sm - sp)));
        }
    }

    // The first prefix sum of the constraint solve alone (Eq. (6)): delta (gauge
    // applied) and e^{-delta} at own points and the delta~ end value dN, for
    // stages whose A is evolved with Eq. (4) instead of solved from Eq. (5).
    // Contains barrier B1.
    __device__ __forceinline__ void delta_scan(const double* q, double* dl, double* E, double& dN)
    {
        const auto tb = tables();
        double p[P];
        double ptot = 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            p[k] = tab(tb, 0, k) * q[k];  // table is 0 off 1..N-2
            ptot += p[k];
        }
        const double incl = wave_incl_scan(ptot);
        if (lane == 63) red[wv] = incl;
        if (lane == 0) XP[2 * (wv + 1)] = p[0];
        if (lane == 63) XP[2 * (wv + 1) + 1] = p[P - 1];
        if (tid == 0) XP[1] = -p[1];                // p_{-1} = -p_1
        if (FULL && tid == NL - 1) XP[2 * (W + 1)] = 0.0;  // p_{N-1} = 0
        if (tid == 0) red[4 * W] = p[1];
        if (FULL) {
            if (tid == NL - 1) red[4 * W + 1] = p[P - 1];
        } else if (has_nm2) {
            const int e = end_here() - 1;
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k == e) red[4 * W + 1] = p[k];
        }
        __syncthreads();  // B1
        double carry, tot;
        wave_totals(red, carry, tot);
        carry += incl - ptot;
        const double p1 = red[4 * W], pN2 = red[4 * W + 1];
        double pl, pr;
        pl = dpp_old<0x138>(XP[2 * wv + 1], p[P - 1]);
        pr = dpp_old<0x130>(XP[2 * (wv + 2)], p[0]);
        dN = -h24 * fma(24.0, tot, 2.0 * pN2 + 2.0 * p1);
        const double shift = bgauge ? dN : 0.0;
        const double a24 = 24.0 * h24, a12 = -12.0 * h24, c0 = fma(2.0 * h24, p1, shift);
        double R = carry;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            R += p[k];
            const double pm = (k == 0) ? pl : p[k - 1];
            const double pp = (k == P - 1) ? pr : p[k + 1];
            const double nd = fma(a24, R, fma(a12, p[k], fma(h24, pm - pp, c0)));  // -delta, as in constraints
            dl[k] = -nd;
            E[k] = exp_tab(nd, X64);
        }
    }

    // Barriers one call of rhs passes (EVA off): B1, B2 and B3, or B3 alone with the
    // metric frozen.
    static __device__ __forceinline__ int rhs_barriers(bool frozen) { return frozen ? 1 : 3; }

    // Right-hand sides of Eqs. (2)-(3) at the published stage input (v0, v1): q, the
    // constraint solve (B1, B2), the fluxes f1 = A e^-delta Pi, g = tan^2 x A
    // e^-delta Phi with parity ghosts (B3), the Kreiss-Oliger terms and the centred
    // D stencil.  With `check`, the division-free test
    // e^-delta - cos^3 x/sin x S < thr e^-delta (A < thr) and a finiteness test
    // run before B3 and the function returns their workgroup-wide bits
    // (1 collapsed, 2 non-finite) without computing r when any is set.
    // r0, r1: Phi_t, Pi_t of the own points (0 at pinned points).  KEEP: also
    // stores the stage input (v0, v1), e^-delta and w = A e^-delta of the lane's points as
    // stage ks of the stage record ES (StageRec).
    // EVA (A evolved by Eq. (4), the paper's alternative to solving Eq. (5) at
    // every stage): the stage's A of the own points is `av`; only the first
    // prefix sum runs (delta from Eq. (6)), the fluxes take w = av e^-delta, the
    // collapse test is av < thr; with `reint` the full solve runs instead and
    // its A, 1 - cos^3 x/sin x S/e^-delta, replaces `av` (re-integration from
    // Eq. (5)).  `wout` receives w = A e^-delta of the own points.
    // Sums of two products are written with fma, so that the kernels that share this
    // code (the recompute of a segment for the adjoint among them) round alike.
    // No barrier before the scans: the stage input is in
    // registers and its edges were published before the first scan barrier.
    // The stage-input and flux slots (XU, XF) are double-buffered by stage, so
    // their last readers (after B3) never meet the next stage's writers even
    // with the metric frozen, when B3 is a stage's only barrier; the scan slots
    // (XP, XS) are written before B1 / B2 and read after them, with B3 between
    // a stage's reads and the next stage's writes.
    template <bool KEEP = false, bool EVA = false>
    __device__ __forceinline__ int rhs(bool check, bool frozen, const double* v0, const double* v1, double* r0,
                                       double* r1, ADSCL_GLOBAL double* ES = nullptr, int ks = 0,
                                       double* av = nullptr, double* wout = nullptr, bool reint = false)
    {
        const auto tb = tables();
        double q[P];
#pragma unroll
        for (int k = 0; k < P; ++k) q[k] = fma(v0[k], v0[k], v1[k] * v1[k]);
        double dl[P], E[P], S[P];
        double dN = 0.0, tot2 = 0.0;
        if (!frozen) {
            if (EVA && !reint) {
                delta_scan(q, dl, E, dN);
#pragma unroll
                for (int k = 0; k < P; ++k) S[k] = 0.0;
            } else {
                constraints(q, dl, E, S, dN, tot2);
            }
        } else {
#pragma unroll
            for (int k = 0; k < P; ++k) { dl[k] = 0.0; E[k] = 1.0; S[k] = 0.0; }
        }
        double wr[KEEP ? P : 1];  // w for the record
        double ff[P], fg[P], chk = 0.0, f2_1 = 0.0, f2_2 = 0.0;
        int cl = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double c3s = tab(tb, 2, k) * tab(tb, 0, k);
            double wk;
            if constexpr (EVA) {
                if (reint) av[k] = 1.0 - c3s * (S[k] / E[k]);
                wk = av[k] * E[k];
                wout[k] = wk;
            } else {
                wk = E[k] - c3s * S[k];
            }
            if constexpr (KEEP) wr[k] = wk;
            const double f2 = wk * v0[k];
            ff[k] = wk * v1[k];
            fg[k] = tab(tb, 1, k) * f2;
            if (k == 1) f2_1 = f2;
            if (k == 2) f2_2 = f2;
            if (check) {
                if (wk < thr * E[k]) cl = 1;
                chk = fma(q[k], 0.0, chk);
                chk = fma(wk, 0.0, chk);
                chk = fma(E[k], 0.0, chk);
            }
        }
        double2* const XFb = XF + buf * (W + 2) * 4;  // this stage's flux slots
        {
            double2* xf = XFb + (wv + 1) * 4;
            if (lane == 0) {
                xf[0] = make_double2(ff[0], fg[0]);
                xf[1] = make_double2(ff[1], fg[1]);
            }
            if (lane == 63) {
                xf[2] = make_double2(ff[P - 1], fg[P - 1]);
                xf[3] = make_double2(ff[P - 2], fg[P - 2]);
            }
            if (tid == 0) {  // f1 even, g odd about x = 0: points -1, -2
                XFb[2] = make_double2(ff[1], -fg[1]);
                XFb[3] = make_double2(ff[2], -fg[2]);
            }
            if (FULL && tid == NL - 1) {
                // f1_{N-1} = 0, g_{N-1} the even 6th-order extrapolation; ghost N
                XFb[(W + 1) * 4] = make_double2(0.0, (fma(15.0, fg[P - 1], -6.0 * fg[P - 2]) + fg[P - 3]) / 10.0);
                XFb[(W + 1) * 4 + 1] = make_double2(-ff[P - 1], fg[P - 1]);
            }
            if constexpr (RAG) {
                if (near_end) {
#pragma unroll
                    for (int k = 0; k < P; ++k) GF[buf * 2 * P + i0 - jb + k] = make_double2(ff[k], fg[k]);
                }
            }
        }
        if (check) {
            if (1.0 < thr) cl = 1;
            if (!isfinite(dN) || !isfinite(chk)) cl |= 2;
            const int wcol = __any(cl & 1) ? 1 : 0;
            const int wnf = __any(cl & 2) ? 2 : 0;
            if (lane == 0) red[2 * W + wv] = (double)(wcol | wnf);
        }
        if constexpr (KEEP) {
            // after the flux loop, so that its table loads do not wait for
            // these stores (vector loads and stores retire in issue order)
            const auto es = stage_rec<P, NL>(ES + (size_t)ks * 4 * P * NL, tid);
#pragma unroll
            for (int k = 0; k < P; ++k) es.st(k, v0[k], v1[k], E[k], wr[k]);
        }
        __syncthreads();  // B3
        if (check) {
            int fl_ = 0;
#pragma unroll
            for (int v = 0; v < W; ++v) fl_ |= (int)red[2 * W + v];
            if (fl_) return fl_;
        }
        double ko0[P], ko1[P];
        {
            double2 w[P + 6];  // points i0-3 .. i0+P+2
            {
                // lanes 0 / 63 take the neighbouring wavefront's (or the ghost) slot
                const double2* xl = XU + (buf * (W + 2) + wv) * 6;
                const double2* xr = XU + (buf * (W + 2) + wv + 2) * 6;
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const double2 gl = xl[5 - r], gr = xr[r];
                    w[r] = make_double2(dpp_old<0x138>(gl.x, v0[P - 3 + r]), dpp_old<0x138>(gl.y, v1[P - 3 + r]));
                    w[P + 3 + r] = make_double2(dpp_old<0x130>(gr.x, v0[r]), dpp_old<0x130>(gr.y, v1[r]));
                }
            }
#pragma unroll
            for (int k = 0; k < P; ++k) w[3 + k] = make_double2(v0[k], v1[k]);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                ko0[k] = kof * (w[k].x - 6.0 * w[k + 1].x + 15.0 * w[k + 2].x - 20.0 * w[k + 3].x
                                + 15.0 * w[k + 4].x - 6.0 * w[k + 5].x + w[k + 6].x);
                ko1[k] = kof * (w[k].y - 6.0 * w[k + 1].y + 15.0 * w[k + 2].y - 20.0 * w[k + 3].y
                                + 15.0 * w[k + 4].y - 6.0 * w[k + 5].y + w[k + 6].y);
            }
        }
        double2 fw[P + 4];  // points i0-2 .. i0+P+1
        {
            const double2* xl = XFb + wv * 4;
            const double2* xr = XFb + (wv + 2) * 4;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const double2 gl = xl[3 - r], gr = xr[r];
                fw[r] = make_double2(dpp_old<0x138>(gl.x, ff[P - 2 + r]), dpp_old<0x138>(gl.y, fg[P - 2 + r]));
                fw[P + 2 + r] = make_double2(dpp_old<0x130>(gr.x, ff[r]), dpp_old<0x130>(gr.y, fg[r]));
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) fw[2 + k] = make_double2(ff[k], fg[k]);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double Df1 = fw[k].x - 8.0 * fw[k + 1].x + 8.0 * fw[k + 3].x - fw[k + 4].x;
            const double Dg = (fw[k].y - 8.0 * fw[k + 1].y + 8.0 * fw[k + 3].y - fw[k + 4].y) * i12h;
            r0[k] = fma(Df1, i12h, ko0[k]);
            r1[k] = fma(tab(tb, 2, k), Dg, ko1[k]);
        }
        if (tid == 0) {
            // Phi_0 = 0; lim tan^-2 (tan^2 f2)' = 3 f2'(0) with f2 odd about x = 0
            r0[0] = 0.0;
            r1[0] = fma(3.0, (16.0 * f2_1 - 2.0 * f2_2) * i12h, ko1[0]);
        }
        if constexpr (RAG) end_terms(r0, r1);
        return 0;
    }
};

}  // namespace adscl
