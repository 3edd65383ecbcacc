// LIM stages (eq. LIM, eq. LIM_last) on 1D grids, up to 48 per launch.
//
// A wave owns a segment of 256 cells, four adjacent cells per lane, in
// registers and runs all K stages of the launch on it: x-neighbours are the
// lane's own cells or come from the adjacent lanes (DPP).  The K cells at each
// end of the segment go stale and belong to the neighbouring segments, so
// waves never exchange anything: no LDS, no barrier.
//
// What bounds it: a launch's latency.  The 23 stages of a 1024-cell step took
// 23 launches of 3.5 us (one stage each); here they are one launch of 6.9 us.
//
// The operations and their order are those of the one-stage kernels (k_stage64,
// k_final64, k_stage32), so the bits are too: S = (w mean)_left (v_a - v_left)
// + (w mean)_right (v_a - v_right), out = c_m (G + tau b_m v_a - (tau rC) S).
#include <hip/hip_runtime.h>

#include "tlim_device.h"
#include "tlim_sweep.h"

namespace tlim {

namespace {

using tb::fold;
using tb::from_left;
using tb::from_right;

constexpr int kLineK = 48;  // stages per launch (one per lane for their parameters, and a segment's halo)
constexpr int kCells = 4;   // cells per lane
constexpr int kSegment = 64 * kCells;

template <typename R>
struct LineArgs {
    const R* v;
    const R* G;
    const R* Lam;
    const R* rC;
    R* out;
    const double* lam;  // accumulator row of lambda_max (NULL: tb given)
    double tau, w;
    double tb[kLineK], chat[kLineK];
    const double* Tit;  // FP64, launch with the final stage: the pass reductions go to ps
    PassSlots ps;
    int n, per, K, face, ox;
};

template <typename R>
__global__ void __launch_bounds__(64) k_line(LineArgs<R> a) {
    constexpr int C = kCells;
    const int lane = threadIdx.x & 63, K = a.K, n = a.n;
    const int x0 = (int)blockIdx.x * a.ox - K + C * lane;
    double lamr[kSlots / 64] = {};
    if (a.lam) {
#pragma unroll
        for (int k = 0; k < kSlots / 64; ++k) lamr[k] = a.lam[lane + 64 * k];
    }
    R v[C], G[C], L[C], t[C];
    int xi[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
        xi[j] = fold(x0 + j, n, a.per);
        v[j] = a.v[xi[j]];
        G[j] = a.G[xi[j]];
        L[j] = a.Lam[xi[j]];
        t[j] = a.rC[xi[j]];
    }
    // stage s's tau b and c in lane s
    double lamv = 0.0;
    if (a.lam) {
#pragma unroll
        for (int k = 0; k < kSlots / 64; ++k) lamv = fmax(lamv, lamr[k]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lamv = fmax(lamv, __shfl_xor(lamv, o, 64));
    }
    double ptb = 0.0, pcm = 1.0;
    if (lane < K) {
        ptb = a.lam ? a.tau * lamv * a.chat[lane] : a.tb[lane];
        pcm = 1.0 / (1.0 + ptb);
    }
    R kL[C], kR[C];  // w mean(Lambda), 0 at a wall
    {
        // (neighbours with every lane active)
        const R Lr = from_right(L[0]);
        R M[C];
#pragma unroll
        for (int j = 0; j < C; ++j) M[j] = (R)a.w * tb::fmean<R>(L[j], j < C - 1 ? L[j < C - 1 ? j + 1 : j] : Lr, a.face);
        const R Ml = from_left(M[C - 1]);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int x = x0 + j;
            const bool in = x >= 0 && x < n;
            const bool fL = a.per ? n > 1 : (in && x > 0), fR = a.per ? n > 1 : (in && x < n - 1);
            kL[j] = fL ? (j > 0 ? M[j > 0 ? j - 1 : 0] : Ml) : R(0);
            kR[j] = fR ? M[j] : R(0);
            t[j] *= (R)a.tau;
        }
    }
    for (int s = 0; s < K; ++s) {
        const R tb = (R)tb::lane_value(ptb, s), cm = (R)tb::lane_value(pcm, s);
        R d[C];  // v_j - v_(j+1): minus the right neighbour's difference to its left
        const R vr = from_right(v[0]);
#pragma unroll
        for (int j = 0; j < C; ++j) d[j] = v[j] - (j < C - 1 ? v[j < C - 1 ? j + 1 : j] : vr);
        const R dl = from_left(d[C - 1]);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const R S = fma(kR[j], d[j], kL[j] * -(j > 0 ? d[j > 0 ? j - 1 : 0] : dl));
            v[j] = cm * fma(-t[j], S, fma(tb, v[j], G[j]));
        }
    }
    double dmax = 0.0, tmax = 0.0, bad = 0.0;
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int c = C * lane + j, x = x0 + j;
        if (c >= K && c < K + a.ox && x < n) {
            a.out[x] = v[j];
            if (a.Tit) {
                const double tn = (double)v[j];
                if (a.ps.dmax) dmax = fmax(dmax, fabs(tn - a.Tit[x]));
                tmax = fmax(tmax, fabs(tn));
                if (!(tn > 0.0) || isinf(tn)) bad += 1.0;
            }
        }
    }
    if (a.Tit) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
            tmax = fmax(tmax, __shfl_xor(tmax, o, 64));
            bad += __shfl_xor(bad, o, 64);
        }
        if (lane == 0) {
            const int sl = (int)(blockIdx.x % kSlots);
            if (a.ps.dmax)
                atomicMax((unsigned long long*)(a.ps.dmax + sl), (unsigned long long)__double_as_longlong(dmax + 0.0));
            atomicMax((unsigned long long*)(a.ps.tmax + sl), (unsigned long long)__double_as_longlong(tmax + 0.0));
            if (bad != 0.0) atomicAdd(a.ps.bad + sl, bad);
        }
    }
}

}  // namespace

bool use_line(const DevGrid& g) { return g.ny == 1 && g.nz == 1; }

int line_stages(int count) {
    const int launches = (count + kLineK - 1) / kLineK;
    return (count + launches - 1) / launches;
}

template <typename R>
void launch_line(hipStream_t s, const DevGrid& g, int face, const R* v, const R* G, const R* Lam, const R* rC, R* out,
                 Stages st, int K, double tau, const double* Tit, PassSlots ps) {
    LineArgs<R> a{};
    a.v = v;
    a.G = G;
    a.Lam = Lam;
    a.rC = rC;
    a.out = out;
    a.lam = st.lam;
    a.tau = tau;
    a.w = g.w[0];
    for (int k = 0; k < K; ++k) {
        if (st.lam) a.chat[k] = st.chat[k];
        else a.tb[k] = st.tb[k];
    }
    a.Tit = Tit;
    a.ps = ps;
    a.n = g.nx;
    a.per = g.per[0];
    a.K = K;
    a.face = face;
    a.ox = kSegment - 2 * K;
    hipLaunchKernelGGL(k_line<R>, dim3((unsigned)((g.nx + a.ox - 1) / a.ox)), dim3(64), 0, s, a);
}

template void launch_line<double>(hipStream_t, const DevGrid&, int, const double*, const double*, const double*,
                                  const double*, double*, Stages, int, double, const double*, PassSlots);
template void launch_line<float>(hipStream_t, const DevGrid&, int, const float*, const float*, const float*,
                                 const float*, float*, Stages, int, double, const double*, PassSlots);

}  // namespace tlim
