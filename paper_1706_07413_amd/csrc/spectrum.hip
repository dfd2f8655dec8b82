// Projection of states on the linear AdS4 eigenmodes (Liebling & Khanna,
// arXiv:1706.07413, Sec. II: decomposition into normal modes), as FP64 matrix
// products on the MFMA units.
//
//   Pihat_rj = sum_i sqrt(A_ri) Pi_ri wPi[j][i],   Phihat_rj = sum_i sqrt(A_ri) Phi_ri wPhi[j][i],
//   E_rj = Pihat_rj^2 + Phihat_rj^2,
// with wPi = h tan^2 x e_j(x), wPhi = h tan^2 x e_j'(x)/omega_j (zero at both
// ends).  A row r is one state of one instance (an instance of the current
// batch, or an instance in one snapshot slot); rows of one grid size N form a
// (rows x N) . (N x J) product, evaluated in 16 x 16 output tiles with
// v_mfma_f64_16x16x4_f64: lane l supplies A[l % 16][l / 16] of the 16 x 4 block
// and B[l / 16][l % 16] of the 4 x 16 block, and holds accumulators
// D[l / 16 + 4 q][l % 16], q = 0..3.
#include <math.h>

#include "stage.h"

namespace adscl {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16;

// One workgroup per (16-row tile, 16-mode tile), all tiles of all grid sizes in one
// launch.  Its wavefronts take the contraction in turns of 16 points; lane l
// supplies points 4 (l / 16) + t of a turn for the t-th of four products (the
// order of the points is free as long as both operands agree), so that its loads of
// a row are 32 consecutive bytes and four lanes' a whole line.  The partial
// tiles are summed through LDS in a fixed order.
// Bound by the latency of those loads, which is why sixteen wavefronts share a tile:
// the contraction of one 16385-point state with 64 modes has only four tiles.
// Measured: the 1024-instance batch (three grid sizes, 32 modes) 72 us against 364
// with one launch per grid size and four wavefronts per tile that took turns of 4
// points; 16 modes of one 4097-point state 40 against 143; 64 modes of five
// 16385-point states 178 against 823.
__global__ void __launch_bounds__(64 * kWaves) spectrum_mfma_kernel(const double* base, const SpecRow* rows,
                                                                    const SpecTile* tiles, int J, double* E,
                                                                    double* Pihat, double* Phihat)
{
    __shared__ double part[kWaves][8][64];
    const SpecTile T = tiles[blockIdx.x];
    const int N = T.N;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = lane & 15, kk = lane >> 4;
    const int j = blockIdx.y * 16 + i;  // mode of the B operand this lane supplies
    const bool vr = i < T.rows, vj = j < J;
    const SpecRow R = rows[T.first + (vr ? i : 0)];  // row of the A operand this lane supplies
    const ADSCL_GLOBAL double* const a = gmem(base + R.a + 4 * kk);
    const ADSCL_GLOBAL double* const pi = gmem(base + R.pi + 4 * kk);
    const ADSCL_GLOBAL double* const phi = gmem(base + R.phi + 4 * kk);
    const ADSCL_GLOBAL double* const wp = gmem(T.wPi + (size_t)(vj ? j : 0) * N + 4 * kk);
    const ADSCL_GLOBAL double* const wf = gmem(T.wPhi + (size_t)(vj ? j : 0) * N + 4 * kk);
    v4d cp = {0.0, 0.0, 0.0, 0.0}, cf = {0.0, 0.0, 0.0, 0.0};
    auto turn = [&](int k0, auto&& in) {
        double va[4], vp[4], vf[4], bp[4], bf[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = in(t) ? k0 + t : 0;  // (a point past N - 1 loads another one's and is masked below)
            va[t] = a[k];
            vp[t] = pi[k];
            vf[t] = phi[k];
            bp[t] = wp[k];
            bf[t] = wf[k];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool o = vr && in(t);
            const double sA = sqrt(va[t]);
            const double ap = o ? sA * vp[t] : 0.0, af = o ? sA * vf[t] : 0.0;
            const double wp_ = vj && in(t) ? bp[t] : 0.0, wf_ = vj && in(t) ? bf[t] : 0.0;
            cp = __builtin_amdgcn_mfma_f64_16x16x4f64(ap, wp_, cp, 0, 0, 0);
            cf = __builtin_amdgcn_mfma_f64_16x16x4f64(af, wf_, cf, 0, 0, 0);
        }
    };
    int k0 = 16 * wv;
#pragma unroll 2
    for (; k0 + 16 <= N; k0 += 16 * kWaves) turn(k0, [](int) { return true; });
    if (k0 < N) turn(k0, [&](int t) { return k0 + 4 * kk + t < N; });
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        part[wv][q][lane] = cp[q];
        part[wv][4 + q][lane] = cf[q];
    }
    __syncthreads();
    // wavefront q finishes accumulator q: accumulator q of lane l is output row
    // l / 16 + 4 q, column l % 16
    if (wv >= 4) return;
    double sp = 0.0, sf = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        sp += part[w][wv][lane];
        sf += part[w][4 + wv][lane];
    }
    const int row = (lane >> 4) + 4 * wv, col = blockIdx.y * 16 + (lane & 15);
    if (row < T.rows && col < J) {
        const size_t o = (size_t)rows[T.first + row].out * J + col;
        if (Pihat) Pihat[o] = sp;
        if (Phihat) Phihat[o] = sf;
        if (E) E[o] = sp * sp + sf * sf;
    }
}

}  // namespace

hipError_t launch_spectrum(const double* base, const SpecRow* rows, const SpecTile* tiles, int n_tiles, int J, double* E,
                           double* Pihat, double* Phihat, hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    spectrum_mfma_kernel<<<dim3(n_tiles, (J + 15) / 16), dim3(64 * kWaves), 0, s>>>(base, rows, tiles, J, E, Pihat,
                                                                                   Phihat);
    return hipGetLastError();
}

}  // namespace adscl
