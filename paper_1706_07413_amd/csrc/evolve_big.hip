// RK4 evolution of one large instance (N above what one workgroup holds) over
// several workgroups, gfx950 (Liebling & Khanna, arXiv:1706.07413, Sec. II).
//
// The instance's evolved points are cut into G chunks of C = 64 W P points; the
// workgroup of chunk g keeps its points in registers as the single-workgroup
// kernel does (lane l owns P consecutive points, neighbours' values by DPP, small
// LDS slots between wavefronts) and exchanges with the other workgroups through a
// small global record per chunk.  Per stage:
//   U  stage input: each chunk's first and last four points, published when the
//      stage input is formed and read by the two neighbours.
//   B  the constraint scans.  Within a chunk both prefix sums are taken
//      locally, the first without its carry: with R'_k the local prefix of
//      p = sin x cos x q, delta~'_k = -h/24 (24 R'_k - 12 p_k + p_{k-1} - p_{k+1})
//      and E'_k = exp(-delta~'_k), the true weight is e^{-(delta~_k - shift)} =
//      E'_k F_g with one factor per chunk, F_g = exp(24 h/24 C_g + 2 h/24 p_1 +
//      shift), C_g the p total of the chunks before g.  So the totals of p and of
//      sigma' = tan^2 x q E'_k are all a chunk publishes, and every chunk then
//      finishes its own points:
//      S_k = h/24 (24 (D_g + F_g R2'_k) - 12 s_k + s_{k-1} - s_{k+1}), s = F sigma',
//      D_g = sum_{h<g} F_h (sigma' total of h).
// The fluxes need no exchange: with the four published points past its end, and
// the same factorisation, a chunk forms e^-delta, S and the flux at the two points
// past the end itself (R and R2 there are the chunk's own totals continued by a
// few terms) while B's words travel.
//
// A workgroup has W main wavefronts, which hold the chunk, and a helper, which
// polls and publishes the words and does the work past the ends, so that the main
// wavefronts' instruction streams stay as short as the single-workgroup kernel's:
// with one wavefront per SIMD every instruction of a stage is on its critical path.
//
// What bounds a stage is latency.  Of about 7600 cycles at N = 16385, publishing
// the sums to having everyone's takes 3100, of which about 2200 are the fabric's
// (the same all-gather alone, nothing else running); the dependent scans,
// exponentials and five workgroup barriers are the rest.  The chunks' places on
// the eight XCDs (an instance's chunks on one, or dealt over all) change a step by
// 1 to 4 %, either way, and are left to the dispatcher.
// Measured, us per step: N = 16385 13.2, N = 32769 13.8, eight of 16385 13.8, 64
// third-order instances of 8193 points 14.0, N = 65537 with the metric frozen 8.0;
// with three barriers over an arrival counter per stage, whole LDS rows and no
// helper 36.4, 36.2, 38.7, 51.4 and 25.6.
//
// Exchange words.  A word is one 64-bit value written by one lane with a
// device-scope relaxed store and read with device-scope relaxed loads (which go
// past the non-coherent per-XCD caches), so a word carries its own arrival: the
// reader polls until it is no longer kEmpty, a signalling-NaN pattern that
// arithmetic never produces (put() replaces it, should data hold it).  No counter,
// no release or acquire of other memory.  Words live in four slots taken in turn
// by the stages, and each stage's words are set back to kEmpty by their chunk one
// stage later, when every reader is known to be past them (it has published the
// next stage's words), three stages before they are written again.  Those stores
// have arrived before the chunk publishes the words of the stage after that (the
// helper waits for later loads of its own in between), and a reader polls the slot
// again only once it has those.
// A poll is bounded; one that runs out sets the instance's error flag, every
// wavefront leaves and the host reports it.  The launch is cooperative, so all
// chunks are resident together.  Several large instances share one launch (as
// many as the device holds at once) and never wait for each other.
#include <math.h>

#include <algorithm>

#include "stage.h"

namespace adscl {
namespace {

typedef unsigned long long u64;

// Exchange words of one chunk and slot.
enum : int {
    XW_P = 0,    // p total of the chunk
    XW_S = 1,    // sigma' total of the chunk
    XW_PF = 2,   // p at the first point (chunk 0: p_1)
    XW_PL = 3,   // p at the last point (last chunk: p_{N-2})
    XW_SF = 4,   // sigma' at the first point
    XW_SL = 5,   // sigma' at the last point
    XW_NB = 6,   // words of exchange B
    XW_L = 16,   // (Phi, Pi) of points a .. a+3, then A of a, a+1
    XW_R = 32,   // (Phi, Pi) of points a+C-1 .. a+C-4, then A of a+C-1, a+C-2
    XW_N = 48    // (B, L and R in 128-byte lines of their own: they have different readers)
};
constexpr int kSlots = 4;
constexpr int XW_BITS = kSlots * XW_N;  // then, slot by step, the chunk's collapse / non-finite bits
static_assert(kBigRecWords == XW_BITS + 16, "record size");

constexpr u64 kEmpty = 0x7ff4c0de5eedface;

// How long a wait has gone on: it gives up after 2^31 ticks of the 100 MHz wall clock
// (21 s), looked at every 256th poll, whatever a poll takes.  Legitimate waits are
// microseconds, save for workgroups of the launch that have yet to start, since another
// stream's kernel may hold their compute units for seconds.
struct Wait {
    unsigned polls = 0;
    u64 since = 0;
    __device__ __forceinline__ bool look() { return (++polls & 255) == 0; }
    __device__ __forceinline__ bool over(u64 now)
    {
        if (polls == 256) since = now;
        return now - since > 1ull << 31;
    }
};

// The word that carries v, never kEmpty: a signalling NaN (data could hold that pattern)
// becomes a quiet one.
__device__ __forceinline__ u64 word_of(double v) { return (u64)__double_as_longlong(__builtin_canonicalize(v)); }

__device__ __forceinline__ void put(ADSCL_GLOBAL u64* w, double v)
{
    __hip_atomic_store(w, word_of(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void clear(ADSCL_GLOBAL u64* w)
{
    __hip_atomic_store(w, kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS of a chunk: as the edge path of Stage, a slot per main wavefront (slot wv + 1)
// and the two next to them, which hold what lies past the chunk's ends (parity
// images at x = 0 and pi/2, or the helper's halo).
template <int P, int W>
struct Lds {
    double2* XU;   // [2 buffers][W+2][6] stage input: points 0..2 of lane 0, then P-1..P-3 of lane 63
    double2* XF;   // [2 buffers][W+2][4] fluxes: points 0, 1 of lane 0, then P-1, P-2 of lane 63
    double2* GU;   // [2 buffers][2] last chunk, end inside a wavefront: stage input at N-2, N-3
    double2* GF;   // [2 buffers][3] the same: fluxes at N-2, N-3, N-4
    double* XP;    // [W+2][2] p of the first point of lane 0, of the last point of lane 63; XP[0] p_1, the last p_{N-2}
    double* XS;    // [W+2][2] the same for sigma' (of the next to last point, in the last chunk, nothing)
    double* red;   // [0,W) p totals, [W,2W) sigma' totals, [2W,3W) check bits
    double* CT;    // CT_*: what the helper made of the other chunks' words
    double* X64;   // 2^(j/64), j = 0..63, the table of exp_tab
    double* T;     // this chunk's coefficient tables, [3][P][64 W] (where they are not in registers)
    double* ACC;   // the RK4 accumulator, [2][P][64 W], each lane its own entries (two
                   // of a lane's accesses per point and stage; in registers it costs
                   // the third workgroup of a compute unit)
    static constexpr bool RT = W <= 4;
    // CT_STOP: [2 buffers] what ends the evolution at this stage: 0, the check bits, or -1 (a wait ran out)
    enum { CT_F, CT_D, CT_DN, CT_CL, CT_CR, CT_DL, CT_STOP, CT_SIZE = CT_STOP + 2 };
    static constexpr size_t doubles = (size_t)2 * (W + 2) * 12 + 2 * (W + 2) * 8 + 2 * 4 + 2 * 6 + 4 * (W + 2) + 3 * W +
                                      (W & 1) + CT_SIZE + 64 + (RT ? 0 : 3 * (size_t)P * 64 * W) + 2 * (size_t)P * 64 * W;

    __device__ __forceinline__ explicit Lds(double* l)
    {
        XU = reinterpret_cast<double2*>(l);
        XF = XU + 2 * (W + 2) * 6;
        GU = XF + 2 * (W + 2) * 4;
        GF = GU + 4;
        XP = reinterpret_cast<double*>(GF + 6);
        XS = XP + 2 * (W + 2);
        red = XS + 2 * (W + 2);
        CT = red + 3 * W + (W & 1);
        X64 = CT + CT_SIZE;
        T = X64 + 64;
        ACC = T + (RT ? 0 : 3 * P * 64 * W);
    }
    __device__ __forceinline__ double2* xu(int buf, int s) const { return XU + (buf * (W + 2) + s) * 6; }
    __device__ __forceinline__ double2* xf(int buf, int s) const { return XF + (buf * (W + 2) + s) * 4; }
};

// What both kinds of wavefront know of the chunk.
struct ChunkInfo {
    int g, G, a, N;
    bool first, last, bgauge, frozen;
    double h24, i12h, kof, thr;
    ADSCL_GLOBAL u64* xg;  // exchange records [G][kBigRecWords]
    ADSCL_GLOBAL int* err;
    __device__ __forceinline__ ADSCL_GLOBAL u64* rec(int c, int sl) const
    {
        return xg + (size_t)c * kBigRecWords + sl * XW_N;
    }
};

__device__ __forceinline__ int next_slot(int s) { return s == kSlots - 1 ? 0 : s + 1; }
__device__ __forceinline__ int prev_slot(int s) { return s == 0 ? kSlots - 1 : s - 1; }

// The wavefront that talks to the other chunks.  Per stage it passes the main
// wavefronts' barriers; between them it reads the neighbours' published edges,
// continues the chunk's own sums past its ends (lane i < 4: point a - 1 - i, lane
// 8 + i: point a + C + i, side by side), publishes the chunk's totals, waits for
// everyone's and forms the carries.
template <int P, int W, bool EVA>
struct Helper {
    static constexpr int C = P * 64 * W;
    using L = Lds<P, W>;
    const L& m;
    const ChunkInfo& c;
    int lane, i, slot, buf;
    bool left, right, on;  // on: this lane serves a point past an end that another chunk owns
    double sc, t2, c3s;    // tables at that point
    const double* word;    // where the main wavefronts leave this lane's word of B (lanes XW_PF .. XW_SL)

    __device__ __forceinline__ Helper(const L& m_, const ChunkInfo& c_, const ADSCL_GLOBAL double* tabI) : m(m_), c(c_)
    {
        lane = threadIdx.x & 63;
        i = lane & 7;
        left = lane < 4 && !c.first;
        right = lane >= 8 && lane < 12 && !c.last;
        on = left || right;
        slot = 0;
        buf = 1;
        sc = t2 = c3s = 0.0;
        word = m.red;
        if (lane == XW_PF) word = m.XP + (c.first ? 0 : 2);
        if (lane == XW_PL) word = m.XP + (c.last ? 2 * (W + 1) + 1 : 2 * W + 1);
        if (lane == XW_SF) word = m.XS + 2;
        if (lane == XW_SL) word = m.XS + 2 * W + 1;
        if (on) {
            const int j = left ? c.a - 1 - i : c.a + C + i;
            const int gg = j / C, jl = j - gg * C, l = jl / P, k = jl - l * P;
            const ADSCL_GLOBAL double* const tj = tabI + (size_t)gg * 3 * C + (size_t)k * 64 * W + l;
            sc = tj[0];
            t2 = tj[C];
            c3s = tj[2 * C] * sc;
        }
    }

    // Polls NW consecutive words at `p` (per lane; lanes with `act` only) until
    // none is kEmpty.  False when the wait ran out here or elsewhere.
    template <int NW>
    __device__ __forceinline__ bool get(const ADSCL_GLOBAL u64* p, bool act, double (&v)[NW]) const
    {
        u64 w[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = 0;
        bool ok = true;
        for (Wait wait;;) {
            bool miss = false;
            if (act) {
#pragma unroll
                for (int k = 0; k < NW; ++k) w[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < NW; ++k) miss |= w[k] == kEmpty;
            }
            if (!__any(miss)) break;
            if (wait.look() &&
                (wait.over(wall_clock64()) || __hip_atomic_load(c.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                __hip_atomic_store(c.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = false;
                break;
            }
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) v[k] = __longlong_as_double((long long)w[k]);
        return ok;
    }

    // Prefix sums over the lanes of a side, the nearest point first.
    static __device__ __forceinline__ double side_scan(double v)
    {
        v += dpp_d<0x111, 0xf>(v);  // row_shr:1
        v += dpp_d<0x112, 0xf>(v);  // row_shr:2
        return v;
    }

    // The terms of the cell rule next to a point past the end: value at the
    // neighbour left of it minus value at the one right of it; `edge`: at the
    // chunk's own end, next to the nearest point.
    __device__ __forceinline__ double around(double v, double edge) const
    {
        const double nearer = dpp_d<0x111, 0xf>(v), out = dpp_d<0x101, 0xf>(v);  // (by every lane)
        const double in = i == 0 ? edge : nearer;
        return left ? out - in : in - out;
    }

    // All chunks' check bits of the step (-1: the wait ran out); the words of the
    // step before are then read by everyone.
    __device__ __forceinline__ int bits(int bslot) const
    {
        double w[1];
        const bool ok = get(c.rec(lane < c.G ? lane : 0, 0) + XW_BITS + bslot, lane < c.G, w);
        if (lane == 0) clear(c.rec(c.g, 0) + XW_BITS + prev_slot(bslot));
        const int bl = (lane < c.G) ? (int)w[0] : 0;
        return ok ? (__any(bl & 1) ? 1 : 0) | (__any(bl & 2) ? 2 : 0) : -1;
    }

    // One stage; true when the evolution ends at this stage (bits set, or a wait ran
    // out): the main wavefronts find it in CT_STOP.
    __device__ __forceinline__ bool stage(bool check, bool gather, int bslot, bool solveS)
    {
        bool ok = true;
        int stop = 0;
        const double h24 = c.h24, a24 = 24.0 * h24;
        double tot = 0.0, tot2 = 0.0;
        if (!c.frozen) {
            double none;
            __syncthreads();  // B1
            wave_totals<W>(m.red, lane, 0, none, tot);
            if (solveS) {
                __syncthreads();  // B2
                wave_totals<W>(m.red + W, lane, 0, none, tot2);
            }
            double v = *word;  // lanes XW_PF .. XW_SL: from the slots the main wavefronts left
            if (!solveS && lane >= XW_SF) v = 0.0;
            if (lane == XW_P) v = tot;
            if (lane == XW_S) v = tot2;
            if (lane < XW_NB) put(c.rec(c.g, slot) + lane, v);
        }
        // While those words travel: the neighbours' edges (here by now), (Phi, Pi)
        // of this lane's point and, EVA, its A.
        double u[2], A[1] = {1.0};
        const ADSCL_GLOBAL u64* r = left ? c.rec(c.g - 1, slot) + XW_R : c.rec(right ? c.g + 1 : c.g, slot) + XW_L;
        ok &= get(r + (on ? 2 * i : 0), on, u);
        if constexpr (EVA) ok &= get(r + (on && i < 2 ? 8 + i : 8), on && i < 2, A);
        // (what the last stage set back to kEmpty has arrived: a wavefront's memory
        // operations end in order, and these loads are back)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        double w = 1.0;  // A e^-delta at the lane's point
        if (on && i < 3) m.xu(buf, left ? 0 : W + 1)[left ? 3 + i : i] = make_double2(u[0], u[1]);
        if (c.frozen) {
            if (gather) stop = bits(bslot);
        } else {
            const double q = u[0] * u[0] + u[1] * u[1];
            const double p = on ? sc * q : 0.0;
            const double ps = side_scan(p);
            const double pown = left ? m.XP[2] : m.XP[2 * W + 1];
            // e^-delta / F_g: R is 0 left of the chunk and its total right of it,
            // continued over the points in between
            const double R = left ? p - ps : tot + ps;
            const double e = exp_tab(fma(a24, R, fma(-12.0 * h24, p, h24 * around(p, pown))), m.X64);
            const double sg = (solveS && on) ? t2 * q * e : 0.0;
            const double ss = side_scan(sg);
            if (on && i == 0) m.XS[left ? 1 : 2 * (W + 1)] = sg;
            __syncthreads();  // BH
            // lane h (< G <= 64): chunk h's words, factor F_h and sigma carry D_h
            double b[XW_NB];
            ok &= get(c.rec(lane < c.G ? lane : 0, slot), lane < c.G, b);
            if (gather) stop = bits(bslot);
            const double cL = exp_tab(h24 * dpp_d<0x138, 0xf>(b[XW_PL]), m.X64);   // 1 in chunk 0
            const double cR = exp_tab(-h24 * dpp_d<0x130, 0xf>(b[XW_PF]), m.X64);  // 1 in chunk G - 1
            const double dL = b[XW_SF] * (cL - 1.0), dR = b[XW_SL] * (cR - 1.0);
            const int gl = __builtin_amdgcn_readfirstlane(c.G - 1), gu = __builtin_amdgcn_readfirstlane(c.g);
            const double p1 = readlane_d(b[XW_PF], 0), pN2 = readlane_d(b[XW_PL], gl);
            const double inc = wave_incl_scan(b[XW_P]);
            const double dN = -h24 * (24.0 * readlane_d(inc, 63) + 2.0 * pN2 + 2.0 * p1);
            const double Fh = exp_tab(fma(a24, inc - b[XW_P], fma(2.0 * h24, p1, c.bgauge ? dN : 0.0)), m.X64);
            const double fs = (lane < c.G) ? Fh * (b[XW_S] + (dL + dR)) : 0.0;
            const double Dh = wave_incl_scan(fs) - fs;
            if (lane == c.g) {
                m.CT[L::CT_F] = Fh;
                m.CT[L::CT_D] = Dh;
                m.CT[L::CT_DN] = dN;
                m.CT[L::CT_CL] = cL;
                m.CT[L::CT_CR] = cR;
                m.CT[L::CT_DL] = dL;
            }
            __syncthreads();  // BC
            const double Fg = readlane_d(Fh, gu), Dg = readlane_d(Dh, gu);
            const double sown = left ? m.XS[2] * readlane_d(cL, gu) : m.XS[2 * W + 1] * readlane_d(cR, gu);
            // R2 in units of F_g past the carry D_g, as R above
            const double R2 = left ? sg - ss : tot2 + readlane_d(dL, gu) + readlane_d(dR, gu) + ss;
            const double S = fma(a24, fma(Fg, R2, Dg), h24 * Fg * fma(-12.0, sg, around(sg, sown)));
            const double E = e * Fg;
            if constexpr (EVA) w = (solveS ? 1.0 - c3s * (S / E) : A[0]) * E;
            else w = E - c3s * S;
        }
        if (on && i < 2) m.xf(buf, left ? 0 : W + 1)[left ? 2 + i : i] = make_double2(w * u[1], t2 * (w * u[0]));
        if (!ok) stop = -1;
        if (lane == 0) m.CT[L::CT_STOP + buf] = (double)stop;
        __syncthreads();  // B3
        // everyone has published this stage's words: those of the stage before are
        // read (they are written again three stages on)
        if (!c.frozen && lane < XW_NB) clear(c.rec(c.g, prev_slot(slot)) + lane);
        if (on) {  // and so has this neighbour its edge
            ADSCL_GLOBAL u64* wr = c.rec(c.g, prev_slot(slot)) + (left ? XW_L : XW_R);
            clear(wr + 2 * i);
            clear(wr + 2 * i + 1);
            if (EVA && i < 2) clear(wr + 8 + i);
        }
        if (check && lane == 0) {
            int b = 0;
            for (int v = 0; v < W; ++v) b |= (int)m.red[2 * W + v];
            put(c.rec(c.g, 0) + XW_BITS + bslot, (double)b);
        }
        slot = next_slot(slot);
        buf ^= 1;
        return stop != 0;
    }
};

// A main wavefront's part of the chunk: lane l owns the P consecutive points
// a + l P .. of the instance, l counted over the chunk.
template <int P, int W, bool EVA>
struct Chunk {
    static constexpr int NL = 64 * W;
    static constexpr int C = P * NL;
    static_assert(P >= 4, "a lane must own at least 4 points");
    using L = Lds<P, W>;
    const L& m;
    const ChunkInfo& c;
    int tid, lane, wv, i0;
    int buf;    // XU / XF / GU / GF buffer of the current stage input
    int slot;   // exchange slot of the current stage
    bool has_nm2, near_end, wave_end, all_own;
    // the coefficient tables at the lane's points, up to four main wavefronts in
    // registers, more in LDS
    static constexpr bool RT = L::RT;
    double rt[RT ? 3 : 1][P];

    __device__ __forceinline__ Chunk(const L& m_, const ChunkInfo& c_) : m(m_), c(c_)
    {
        tid = threadIdx.x;
        lane = tid & 63;
        wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        i0 = c.a + tid * P;
        buf = 0;
        slot = kSlots - 1;  // the first publish takes slot 0
        const int N = c.N, wend = c.a + (wv + 1) * 64 * P;  // first point past the wavefront's
        has_nm2 = c.last && (i0 <= N - 2) && (N - 2 < i0 + P);
        // x = pi/2 just past the wavefront's last lane (any power of two of intervals), or elsewhere
        wave_end = c.last && wend == N - 1 && lane == 63;
        near_end = c.last && (N - 1 - c.a) % (64 * P) != 0 && (i0 + P + 2 >= N - 1) && (i0 <= N - 2);
        all_own = wend - 1 <= N - 2;
    }

    __device__ __forceinline__ bool own(int k) const { return i0 + k <= c.N - 2; }
    __device__ __forceinline__ double tab(int t, int k) const
    {
        if constexpr (RT) return rt[t][k];
        return m.T[(t * P + k) * NL + tid];
    }
    __device__ __forceinline__ double c3s(int k) const { return tab(2, k) * tab(0, k); }
    __device__ __forceinline__ void load_tables(const ADSCL_GLOBAL double* tab0)
    {
        // each lane copies exactly the table entries it reads later
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double v = tab0[(t * P + k) * NL + tid];
                if constexpr (RT) rt[t][k] = v;
                else m.T[(t * P + k) * NL + tid] = v;
            }
    }

    // Position of pi/2 relative to the lane's first point, opaque to the compiler:
    // conditions on single points of the last chunk are then formed where they are
    // used (by the wavefronts that meet them) instead of being kept as lane masks
    // for the whole kernel, which spills scalar registers.
    __device__ __forceinline__ int end_here() const
    {
        int e = c.N - 1 - i0;
        asm volatile("" : "+v"(e));
        return e;
    }

    // The next stage's input (own points; EVA: its A): the edges between
    // wavefronts and the parity ghosts into LDS, the chunk's edges into the
    // exchange words of the next slot.
    __device__ __forceinline__ void publish(const double* v0, const double* v1, const double* av)
    {
        buf ^= 1;
        slot = next_slot(slot);
        double2* xu = m.xu(buf, wv + 1);
        if (lane == 0 && own(0)) {
#pragma unroll
            for (int r = 0; r < 3; ++r) xu[r] = make_double2(v0[r], v1[r]);
            if (wv == 0) {
                if (c.first) {  // Phi odd, Pi even about x = 0: points -1, -2, -3
#pragma unroll
                    for (int r = 0; r < 3; ++r) m.xu(buf, 0)[3 + r] = make_double2(-v0[1 + r], v1[1 + r]);
                } else {
                    ADSCL_GLOBAL u64* r = c.rec(c.g, slot) + XW_L;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        put(r + 2 * k, v0[k]);
                        put(r + 2 * k + 1, v1[k]);
                    }
                    if (EVA) {
                        put(r + 8, av[0]);
                        put(r + 9, av[1]);
                    }
                }
            }
        }
        if (lane == 63) {
#pragma unroll
            for (int r = 0; r < 3; ++r) xu[3 + r] = make_double2(v0[P - 1 - r], v1[P - 1 - r]);
            if (wv == W - 1 && !c.last) {
                ADSCL_GLOBAL u64* r = c.rec(c.g, slot) + XW_R;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    put(r + 2 * k, v0[P - 1 - k]);
                    put(r + 2 * k + 1, v1[P - 1 - k]);
                }
                if (EVA) {
                    put(r + 8, av[P - 1]);
                    put(r + 9, av[P - 2]);
                }
            }
            if (wave_end) {  // Phi = Pi = 0 at pi/2; Phi even, Pi odd about it
                double2* gh = m.xu(buf, wv + 2);
                gh[0] = make_double2(0.0, 0.0);
                gh[1] = make_double2(v0[P - 1], -v1[P - 1]);
                gh[2] = make_double2(v0[P - 2], -v1[P - 2]);
            }
        }
        if (near_end) {
            const int e = end_here() - 1;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const int r = e - k;
                if (r == 0 || r == 1) m.GU[buf * 2 + r] = make_double2(v0[k], v1[k]);
            }
        }
    }

    // Right-hand sides at the published stage input (v0, v1).  check: the test of
    // a step's first stage; its bits are gathered during the next stage, before U
    // is advanced.  Returns what ends the evolution here (CT_STOP), or 0.
    // EVA (A evolved by Eq. (4)): the stage's A of the own points is `av`; only
    // delta's prefix sum runs, the fluxes take w = av e^-delta and the collapse
    // test is av < thr; with `reint` the full solve runs and its A,
    // 1 - cos^3 x/sin x S/e^-delta, replaces `av`.  `wout` receives w = A e^-delta
    // of the own points (EVA).
    __device__ __forceinline__ int rhs(bool check, const double* v0, const double* v1, double* r0, double* r1,
                                       double* av, double* wout, bool reint)
    {
        const bool solveS = !EVA || reint;
        const double h24 = c.h24, i12h = c.i12h, thr = c.thr;
        double q[P];
#pragma unroll
        for (int k = 0; k < P; ++k) q[k] = v0[k] * v0[k] + v1[k] * v1[k];
        double E[P], S[P], ko0[P], ko1[P];
        double dN = 0.0;
        if (c.frozen) {
#pragma unroll
            for (int k = 0; k < P; ++k) {
                E[k] = 1.0;
                S[k] = 0.0;
            }
        } else {
            // Local prefix sums of p and sigma'.  The points past the chunk's ends
            // are not waited for here: p there is taken as 0, which leaves the
            // factors c_L = exp(h/24 p_{a-1}) of E' at the first and c_R =
            // exp(-h/24 p_{a+C}) at the last point to be applied after B (to E',
            // sigma' and the sums they enter).
            double p[P];
            double ptot = 0.0;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                p[k] = tab(0, k) * q[k];  // table is 0 off 1..N-2
                ptot += p[k];
            }
            const double incl = wave_incl_scan(ptot);
            if (lane == 0) {
                m.XP[2 * (wv + 1)] = p[0];
                if (c.first && wv == 0) {
                    m.XP[0] = p[1];
                    m.XP[1] = -p[1];  // p_{-1} = -p_1
                }
            }
            if (lane == 63) {
                m.red[wv] = incl;
                m.XP[2 * (wv + 1) + 1] = p[P - 1];
            }
            if (has_nm2) {
                const int e = end_here() - 1;
#pragma unroll
                for (int k = 0; k < P; ++k)
                    if (k == e) m.XP[2 * (W + 1) + 1] = p[k];
            }
            __syncthreads();  // B1
            double carry, tot;
            wave_totals<W>(m.red, lane, wv, carry, tot);
            carry += incl - ptot;
            const double pl = dpp_old<0x138>(m.XP[2 * wv + 1], p[P - 1]);
            const double pr = dpp_old<0x130>(m.XP[2 * (wv + 2)], p[0]);
            double sg[P];
            double R = carry, stot = 0.0;
            const double a24 = 24.0 * h24, a12 = -12.0 * h24;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                R += p[k];
                const double pm = (k == 0) ? pl : p[k - 1];
                const double pp = (k == P - 1) ? pr : p[k + 1];
                // minus the chunk-local delta~': h24 (24 R - 12 p + p_m - p_p), h24 distributed
                E[k] = exp_tab(fma(a24, R, fma(a12, p[k], h24 * (pm - pp))), m.X64);
                sg[k] = solveS ? tab(1, k) * q[k] * E[k] : 0.0;
                stot += sg[k];
            }
            double carry2 = 0.0;
            if (solveS) {  // uniform: the sigma' prefix sums only where S is needed
                const double incl2 = wave_incl_scan(stot);
                if (lane == 0) {
                    m.XS[2 * (wv + 1)] = sg[0];
                    if (c.first && wv == 0) m.XS[1] = sg[1];  // sigma_{-1} = sigma_1
                }
                if (lane == 63) {
                    m.red[W + wv] = incl2;
                    m.XS[2 * (wv + 1) + 1] = sg[P - 1];
                }
                __syncthreads();  // B2
                double tot2;
                wave_totals<W>(m.red + W, lane, wv, carry2, tot2);
                carry2 += incl2 - stot;
            }
            __syncthreads();  // BH: the points past the chunk's ends are in
            kreiss_oliger(v0, v1, ko0, ko1);  // while B's words travel
#pragma unroll
            for (int k = 0; k < P; ++k) asm volatile("" : "+v"(ko0[k]), "+v"(ko1[k]));  // (not sunk past the barrier)
            __syncthreads();  // BC
            const double Fg = m.CT[L::CT_F], aD = a24 * m.CT[L::CT_D];
            dN = m.CT[L::CT_DN];
            double R2 = carry2 + m.CT[L::CT_DL];
            if (tid == 0) {
                const double cL = m.CT[L::CT_CL];
                E[0] *= cL;
                sg[0] *= cL;
                R2 = carry2;
            }
            if (tid == NL - 1) {
                const double cR = m.CT[L::CT_CR];
                E[P - 1] *= cR;
                sg[P - 1] *= cR;
            }
            if (solveS) {
                const double sm0 = dpp_old<0x138>(m.XS[2 * wv + 1], sg[P - 1]);
                const double sp0 = dpp_old<0x130>(m.XS[2 * (wv + 2)], sg[0]);
                const double aF = a24 * Fg, hF = h24 * Fg;
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    R2 += sg[k];
                    const double sm = (k == 0) ? sm0 : sg[k - 1];
                    const double sp = (k == P - 1) ? sp0 : sg[k + 1];
                    // h24 (24 (Dg + Fg R2) + Fg (-12 sigma + sigma_m - sigma_p)), h24 and Fg distributed
                    S[k] = fma(aF, R2, fma(hF, fma(-12.0, sg[k], sm - sp), aD));
                }
            }
#pragma unroll
            for (int k = 0; k < P; ++k) E[k] *= Fg;
        }

        // fluxes; c3s and tan^2 x are 0 at x = 0 in the tables, so w_0 = E_0, g_0 = 0
        double ff[P], fg[P], f2_1 = 0.0, f2_2 = 0.0, chk = 0.0;
        int cl = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            double wk;
            if constexpr (EVA) {
                if (reint) av[k] = 1.0 - c3s(k) * (S[k] / E[k]);
                wk = av[k] * E[k];
                wout[k] = wk;
            } else {
                wk = E[k] - c3s(k) * S[k];
            }
            const double f2 = wk * v0[k];
            ff[k] = wk * v1[k];
            fg[k] = tab(1, k) * f2;
            if (k == 1) f2_1 = f2;
            if (k == 2) f2_2 = f2;
            if (check) {  // (past N-2: c3s = 0, so w = E, and q = 0)
                if (wk < thr * E[k]) cl = 1;
                chk = fma(q[k], 0.0, chk);
                chk = fma(wk, 0.0, chk);
                chk = fma(E[k], 0.0, chk);
            }
        }
        if (lane == 0 && own(0)) {
            double2* xf = m.xf(buf, wv + 1);
            xf[0] = make_double2(ff[0], fg[0]);
            xf[1] = make_double2(ff[1], fg[1]);
            if (c.first && wv == 0) {  // f1 even, g odd about x = 0: points -1, -2
                double2* gh = m.xf(buf, 0);
                gh[2] = make_double2(ff[1], -fg[1]);
                gh[3] = make_double2(ff[2], -fg[2]);
            }
        }
        if (lane == 63) {
            double2* xf = m.xf(buf, wv + 1);
            xf[2] = make_double2(ff[P - 1], fg[P - 1]);
            xf[3] = make_double2(ff[P - 2], fg[P - 2]);
            if (wave_end) {
                // f1_{N-1} = 0, g_{N-1} the even 6th-order extrapolation; N the image of N-2
                double2* gh = m.xf(buf, wv + 2);
                gh[0] = make_double2(0.0, (15.0 * fg[P - 1] - 6.0 * fg[P - 2] + fg[P - 3]) / 10.0);
                gh[1] = make_double2(-ff[P - 1], fg[P - 1]);
            }
        }
        if (near_end) {
            const int e = end_here() - 1;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const int r = e - k;
                if (r >= 0 && r <= 2) m.GF[buf * 3 + r] = make_double2(ff[k], fg[k]);
            }
        }
        if (check) {
            if (1.0 < thr) cl = 1;
            if (!isfinite(dN) || !isfinite(chk)) cl |= 2;
            const int wcol = __any(cl & 1) ? 1 : 0;
            const int wnf = __any(cl & 2) ? 2 : 0;
            if (lane == 0) m.red[2 * W + wv] = (double)(wcol | wnf);
        }
        __syncthreads();  // B3
        const double stop = m.CT[L::CT_STOP + buf];
        if (c.frozen) kreiss_oliger(v0, v1, ko0, ko1);
        double2 fw[P + 4];  // points i0-2 .. i0+P+1
        {
            const double2 *xl = m.xf(buf, wv), *xr = m.xf(buf, wv + 2);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const double2 gl = xl[3 - r], gr = xr[r];
                fw[r] = make_double2(dpp_old<0x138>(gl.x, ff[P - 2 + r]), dpp_old<0x138>(gl.y, fg[P - 2 + r]));
                fw[P + 2 + r] = make_double2(dpp_old<0x130>(gr.x, ff[r]), dpp_old<0x130>(gr.y, fg[r]));
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) fw[2 + k] = make_double2(ff[k], fg[k]);
        if (near_end) {
            const double2 e2 = m.GF[buf * 3], e3 = m.GF[buf * 3 + 1], e4 = m.GF[buf * 3 + 2];
            const double gext = (15.0 * e2.y - 6.0 * e3.y + e4.y) / 10.0;
            const int e = end_here() + 2;
#pragma unroll
            for (int t = 0; t < P + 4; ++t) {
                if (t == e) fw[t] = make_double2(0.0, gext);
                if (t == e + 1) fw[t] = make_double2(-e2.x, e2.y);
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double Df1 = (fw[k].x - 8.0 * fw[k + 1].x + 8.0 * fw[k + 3].x - fw[k + 4].x) * i12h;
            const double Dg = (fw[k].y - 8.0 * fw[k + 1].y + 8.0 * fw[k + 3].y - fw[k + 4].y) * i12h;
            r0[k] = Df1 + ko0[k];
            r1[k] = tab(2, k) * Dg + ko1[k];
        }
        if (c.first && tid == 0) {
            // Phi_0 = 0; lim tan^-2 (tan^2 f2)' = 3 f2'(0) with f2 odd about x = 0
            r0[0] = 0.0;
            r1[0] = 3.0 * ((16.0 * f2_1 - 2.0 * f2_2) * i12h) + ko1[0];
        }
        if (!all_own) {
            const int e = end_here();
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k >= e) r0[k] = r1[k] = 0.0;
        }
        return (int)stop;
    }

    // Kreiss-Oliger terms of the own points from the +-3 window of the stage input.
    __device__ __forceinline__ void kreiss_oliger(const double* v0, const double* v1, double* ko0, double* ko1) const
    {
        const double kof = c.kof;
        double2 w[P + 6];  // points i0-3 .. i0+P+2
        const double2 *xl = m.xu(buf, wv), *xr = m.xu(buf, wv + 2);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const double2 gl = xl[5 - r], gr = xr[r];
            w[r] = make_double2(dpp_old<0x138>(gl.x, v0[P - 3 + r]), dpp_old<0x138>(gl.y, v1[P - 3 + r]));
            w[P + 3 + r] = make_double2(dpp_old<0x130>(gr.x, v0[r]), dpp_old<0x130>(gr.y, v1[r]));
        }
#pragma unroll
        for (int k = 0; k < P; ++k) w[3 + k] = make_double2(v0[k], v1[k]);
        if (near_end) {
            // Phi = Pi = 0 at pi/2; Phi even, Pi odd about it
            const double2 e2 = m.GU[buf * 2], e3 = m.GU[buf * 2 + 1];
            const int e = end_here() + 3;
#pragma unroll
            for (int t = 0; t < P + 6; ++t) {
                if (t == e) w[t] = make_double2(0.0, 0.0);
                if (t == e + 1) w[t] = make_double2(e2.x, -e2.y);
                if (t == e + 2) w[t] = make_double2(e3.x, -e3.y);
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            ko0[k] = kof * (w[k].x - 6.0 * w[k + 1].x + 15.0 * w[k + 2].x - 20.0 * w[k + 3].x + 15.0 * w[k + 4].x
                            - 6.0 * w[k + 5].x + w[k + 6].x);
            ko1[k] = kof * (w[k].y - 6.0 * w[k + 1].y + 15.0 * w[k + 2].y - 20.0 * w[k + 3].y + 15.0 * w[k + 4].y
                            - 6.0 * w[k + 5].y + w[k + 6].y);
        }
    }
};

// RK: Runge-Kutta order (4 classical; 3 and 2 the Shu-Osher methods, as the
// one-workgroup scheme kernel); EVA: A evolved by Eq. (4) and re-integrated
// from Eq. (5) at steps that are multiples of a.a_reint (its A row of the
// packed state holds the evolved A between calls).
template <int P, int W, int RK, bool EVA>
__global__ void __launch_bounds__(64 * (W + 1), W == 3 && !EVA ? 3 : 1) evolve_big_kernel(EvolveArgs a, BigArgs x)
{
    extern __shared__ double lds[];
    constexpr int NL = 64 * W, C = P * NL;
    const BigBlock blk = x.block[blockIdx.x];  // this workgroup's instance in the launch, and its chunk
    const int d = blk.desc;
    const BigDesc bd = x.desc[d];
    const int b = bd.inst;
    const InstStatus st0 = a.status[b];
    if (st0.state == ST_COLLAPSED || st0.state == ST_NONFINITE) return;
    const InstConst ic = a.ic[b];
    const Lds<P, W> m(lds);
    ChunkInfo c;
    c.g = blk.chunk;
    c.G = bd.chunks;
    c.a = c.g * C;
    c.N = ic.N;
    c.first = c.g == 0;
    c.last = c.g == c.G - 1;
    c.bgauge = a.gauge == 0;
    c.frozen = a.frozen != 0;
    c.h24 = ic.h24;
    c.i12h = ic.i12h;
    c.kof = ic.kof;
    c.thr = a.a_collapse;
    c.xg = reinterpret_cast<ADSCL_GLOBAL u64*>(gmem(x.xch)) + (size_t)bd.first * kBigRecWords;
    c.err = gmem(x.err) + d;
    const ADSCL_GLOBAL double* const tabI = gmem(a.tab[b]);  // tables of the whole instance, [g][3][P][NL]
    const int64_t K = a.a_reint;
    int64_t n = st0.steps;
    int64_t seg_end = st0.target;
    if (a.snap_every > 0) {
        const int64_t nb = (n / a.snap_every + 1) * a.snap_every;
        if (nb < seg_end) seg_end = nb;
    }
    int bslot = 0;  // exchange slot of this step's check bits
    if (threadIdx.x < 64) m.X64[threadIdx.x] = exp2((double)threadIdx.x * (1.0 / 64.0));

    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) == W) {
        if (threadIdx.x == NL) {
            // p past the chunk's ends (chunk 0 writes its own), sigma past pi/2
            m.XP[1] = m.XP[2 * (W + 1)] = m.XS[2 * (W + 1)] = 0.0;
        }
        Helper<P, W, EVA> h(m, c, tabI);
        __syncthreads();  // the LDS tables
        for (; n < seg_end; ++n, bslot = next_slot(bslot))
#pragma unroll 1
            for (int s = 0; s < RK; ++s)
                if (h.stage(s == 0, s == 1, bslot, !EVA || (s == 0 && (n % K) == 0))) return;
        return;
    }

    Chunk<P, W, EVA> cs(m, c);
    const int i0 = cs.i0;
    const double dt = ic.dt;
    cs.load_tables(tabI + (size_t)c.g * 3 * C);
    // u: U^n; cv: the current stage input
    double un0[P], un1[P], unA[P], cv0[P], cv1[P], cvA[P], accA[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const bool o = cs.own(k);
        un0[k] = o ? a.Phi[ic.off + i0 + k] : 0.0;
        un1[k] = o ? a.Pi[ic.off + i0 + k] : 0.0;
        unA[k] = (EVA && o) ? a.A[ic.off + i0 + k] : 1.0;
        cv0[k] = un0[k];
        cv1[k] = un1[k];
        cvA[k] = unA[k];
        accA[k] = 0.0;
    }
    int stop_bits = 0;
    cs.publish(un0, un1, unA);
    __syncthreads();  // the LDS tables
    while (n < seg_end && !stop_bits) {
#pragma unroll 1
        for (int s = 0; s < RK; ++s) {
            double r0[P], r1[P], w[P], rA[P];
            const bool reint = EVA && s == 0 && (n % K) == 0;
            stop_bits = cs.rhs(s == 0, cv0, cv1, r0, r1, cvA, w, reint);
            if (stop_bits) break;
            if (reint) {
#pragma unroll
                for (int k = 0; k < P; ++k) unA[k] = cvA[k];
            }
            if constexpr (EVA) {
#pragma unroll
                for (int k = 0; k < P; ++k) rA[k] = -2.0 * cs.tab(0, k) * cvA[k] * w[k] * cv0[k] * cv1[k];
            }
            // one uniform branch per stage; with EVA, A is a third field
            double* const acc = m.ACC + cs.tid;
            auto each = [&](auto&& f) {
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    f(un0[k], cv0[k], r0[k], acc[k * NL]);
                    f(un1[k], cv1[k], r1[k], acc[(P + k) * NL]);
                    if constexpr (EVA) f(unA[k], cvA[k], rA[k], accA[k]);
                }
            };
            if constexpr (RK == 4) {
                const double c_next = (s == 2) ? dt : 0.5 * dt;
                if (s == 0) each([&](double& u, double& v, double r, double& ac) { ac = r; v = u + c_next * r; });
                else if (s < 3) each([&](double& u, double& v, double r, double& ac) { ac = ac + 2.0 * r; v = u + c_next * r; });
                else each([&](double& u, double& v, double r, double& ac) { v = u = u + (dt / 6.0) * (ac + r); });
            } else if constexpr (RK == 3) {
                if (s == 0) each([&](double& u, double& v, double r, double&) { v = u + dt * r; });
                else if (s == 1) each([&](double& u, double& v, double r, double&) { v = 0.75 * u + 0.25 * (v + dt * r); });
                else each([&](double& u, double& v, double r, double&) { v = u = u / 3.0 + (2.0 / 3.0) * (v + dt * r); });
            } else {
                if (s == 0) each([&](double& u, double& v, double r, double&) { v = u + dt * r; });
                else each([&](double& u, double& v, double r, double&) { v = u = 0.5 * u + 0.5 * (v + dt * r); });
            }
            cs.publish(cv0, cv1, cvA);
        }
        if (stop_bits) break;
        ++n;
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if (cs.own(k)) {
            a.Phi[ic.off + i0 + k] = un0[k];
            a.Pi[ic.off + i0 + k] = un1[k];
            if (EVA) a.A[ic.off + i0 + k] = unA[k];
        }
    }
    if (c.first && cs.tid == 0) {
        InstStatus o = st0;
        o.steps = n;
        if (stop_bits < 0) {
            o.state = ST_NONFINITE;
            o.t_c = -2.0;
        } else if (stop_bits) {
            o.state = (stop_bits & 2) ? ST_NONFINITE : ST_COLLAPSED;
            o.t_c = (double)n * dt;
        }
        a.status[b] = o;
    }
}

// All exchange words of the launch to kEmpty, its instances' error flags to zero.
__global__ void __launch_bounds__(256) big_reset_kernel(BigArgs x, int words)
{
    u64* const w = reinterpret_cast<u64*>(x.xch);
    const int t = blockIdx.x * 256 + threadIdx.x;
    for (int i = t; i < words; i += gridDim.x * 256) w[i] = kEmpty;
    for (int i = t; i < x.n_desc; i += gridDim.x * 256) x.err[i] = 0;
}

template <int P, int W>
constexpr size_t big_lds_bytes_for()
{
    return Lds<P, W>::doubles * sizeof(double);
}

template <int P, int W, int RK, bool EVA>
hipError_t launch_big_t(int blocks, const EvolveArgs& a, const BigArgs& x, hipStream_t s)
{
    if (x.n_desc < 1 || x.n_desc > 1024) return hipErrorInvalidValue;
    const int words = blocks * kBigRecWords;
    big_reset_kernel<<<dim3(std::min(64, (words + 255) / 256)), dim3(256), 0, s>>>(x, words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = big_lds_bytes_for<P, W>();
    EvolveArgs ea = a;
    BigArgs xa = x;
    void* args[] = {(void*)&ea, (void*)&xa};
    return hipLaunchCooperativeKernel((const void*)evolve_big_kernel<P, W, RK, EVA>, dim3(blocks), dim3(64 * (W + 1)), args,
                                      lds, s);
}

template <int P, int W, int RK, bool EVA>
hipError_t capacity_t(int device, int* blocks)
{
    int cus = 0, per_cu = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)evolve_big_kernel<P, W, RK, EVA>, 64 * (W + 1),
                                                     big_lds_bytes_for<P, W>());
    if (e != hipSuccess) return e;
    *blocks = per_cu * cus;
    return hipSuccess;
}

template <int P, int W, int RK, bool EVA>
hipError_t prepare_big_t(size_t max_lds)
{
    const size_t need = big_lds_bytes_for<P, W>();
    if (need > max_lds) return hipErrorInvalidValue;
    return hipFuncSetAttribute((const void*)evolve_big_kernel<P, W, RK, EVA>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)need);
}

// The kernel variant of a scheme: RK order 2, 3 or 4, A solved or evolved.
#define ADSCL_BIG_SCHEME(FN, p, w, ...)                                               \
    do {                                                                              \
        if (rk == 4 && !eva) return FN<p, w, 4, false>(__VA_ARGS__);                 \
        if (rk == 4 && eva) return FN<p, w, 4, true>(__VA_ARGS__);                   \
        if (rk == 3 && !eva) return FN<p, w, 3, false>(__VA_ARGS__);                 \
        if (rk == 3 && eva) return FN<p, w, 3, true>(__VA_ARGS__);                   \
        if (rk == 2 && !eva) return FN<p, w, 2, false>(__VA_ARGS__);                 \
        if (rk == 2 && eva) return FN<p, w, 2, true>(__VA_ARGS__);                   \
        return hipErrorInvalidValue;                                                  \
    } while (0)

}  // namespace

#define ADSCL_BIG_CLASSES(X) \
    X(4, 3)                  \
    X(4, 4)                  \
    X(4, 8)

bool big_class_supported(ClassCfg c)
{
#define X(p, w) \
    if (c.P == p && c.W == w) return true;
    ADSCL_BIG_CLASSES(X)
#undef X
    return false;
}

size_t big_lds_bytes(ClassCfg c)
{
#define X(p, w) \
    if (c.P == p && c.W == w) return big_lds_bytes_for<p, w>();
    ADSCL_BIG_CLASSES(X)
#undef X
    return 0;
}

hipError_t prepare_evolve_big(ClassCfg c, int rk, bool eva, size_t max_lds)
{
#define X(p, w) \
    if (c.P == p && c.W == w) ADSCL_BIG_SCHEME(prepare_big_t, p, w, max_lds);
    ADSCL_BIG_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_evolve_big(ClassCfg c, int rk, bool eva, int blocks, const EvolveArgs& a, const BigArgs& x,
                             hipStream_t s)
{
#define X(p, w) \
    if (c.P == p && c.W == w) ADSCL_BIG_SCHEME(launch_big_t, p, w, blocks, a, x, s);
    ADSCL_BIG_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t big_capacity(ClassCfg c, int rk, bool eva, int device, int* blocks)
{
#define X(p, w) \
    if (c.P == p && c.W == w) ADSCL_BIG_SCHEME(capacity_t, p, w, device, blocks);
    ADSCL_BIG_CLASSES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace adscl
