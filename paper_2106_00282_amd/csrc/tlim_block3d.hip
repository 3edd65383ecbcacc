// Several LIM stages (eq. LIM, the last of them eq. LIM_last when it is the
// final one) per launch on 3D grids: temporal blocking along the z-march.
//
// One stage per launch reads v, G, Lambda and 1/C and writes v for every
// stage, 20 B (float) or 40 B (double) per cell, and runs at the memory's
// rate.  Here a workgroup owns a column of 64 x cells (one per lane) by
// WAVES*ROWS y rows and walks a chunk of z planes; while plane z arrives,
// stage s of the launch advances plane z - s, so K stages read and write
// their words once.  A stage needs the plane above from the stage before it
// in the lane's own registers only (the 7-point stencil has no corner), and
// its x- and y-neighbours on its own plane, which the step before finished:
//   - x-neighbours by DPP wave shifts,
//   - y-neighbours in the lane's registers, at the seams between waves
//     through LDS (all K stages publish their seam rows together, so there is
//     one barrier per plane, not one per stage),
//   - z-neighbours in registers; the flux through the face between two
//     planes is formed once and kept for the upper plane.
// Planes z - 1 .. z - K of Lambda, 1/C and G wait in registers for the later
// stages, and plane z + 1 is being loaded while plane z is used.  The K
// cells at the column's x and y edges go stale (they are written by the
// neighbouring columns), and a chunk starts K planes early and ends K late.
//
// What bounds it: at 512^3 in float a launch of 3 stages takes 726 us, 4.5 TB/s
// over the 23.5 B per cell it moves with the column halos (64 x 64 cells for
// 58 x 58 results); one stage per launch took 549 us.  Per stage 549 -> 242 us
// there, 77 -> 41 us at 256^3, in double 22 -> 13.5 us at 128^3 and 28 -> 11.7 us
// at 150 x 131 x 97.  The registers of K stages set the rows per wave: 8 waves
// (two per SIMD, 256 VGPRs each) of 8 float rows, or of 3 (K = 3) or 4 (K = 2)
// double rows; one row more spills (K = 3: 726 -> 1352 us with 4 rows on 16
// waves of 128 VGPRs, 40 -> 61 us at 128^3 in double with 4 rows).
//
// Arithmetic of a stage: with F_f = mean(Lambda_a, Lambda_b) (v_b - v_a) formed
// once per face and shared by its two cells,
//   out = c_m (G + tau b_m v + rC sum_d tau w_d (F_up - F_low)).
#include <hip/hip_runtime.h>

#include "tlim_device.h"
#include "tlim_sweep.h"

namespace tlim {

namespace {

using tb::fold;
using tb::from_left;
using tb::from_right;

constexpr int KMAX3 = 3;
constexpr int kCUs = 256;

template <typename R>
struct B3Args {
    const R* v;  // NULL: the input is the stage before the first from w = 0, c_in G
    const R* G;
    const R* Lam;
    const R* rC;
    R* out;
    R* stages;  // nullable: the result of stage s < K also goes to stages + s*sstride
    int64_t sstride;
    const double* lam;  // accumulator row of lambda_max (NULL: tb given)
    double tau;
    double tb[KMAX3], chat[KMAX3];
    double tb_in, chat_in;  // stage parameter of the input stage (v == NULL)
    const double* Tit;      // FP64, launch with the final stage: the pass reductions go to ps
    PassSlots ps;
    int nx, ny, nz, perx, pery, perz;
    R wx, wy, wz;  // tau * w_d, times 1/2 for arithmetic face means
    int tiles_x, tiles_y, zc;
};

// Face value of the conductivities, up to the factor 1/2 of the arithmetic
// mean (in the weights).
template <typename R, bool kHarm>
__device__ __forceinline__ R face_of(R a, R b) {
    const R s = a + b;
    if constexpr (kHarm) return s > R(0) ? R(2) * (a * b) / s : R(0);
    else return s;
}

template <typename R, int K, int ROWS, int WAVES, bool kHarm>
__global__ void __launch_bounds__(64 * WAVES) k_b3d(B3Args<R> a) {
    constexpr int RW = ROWS + 2;
    constexpr int OX = 64 - 2 * K, EXT_Y = WAVES * ROWS, OY = EXT_Y - 2 * K;
    // seam rows of the K stage inputs: [buffer][stage][wave][first / last row]
    __shared__ R sh[2][K][WAVES][2][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    // stage parameters (every wave folds the bound's row)
    double lamv = 0.0;
    if (a.lam) {
#pragma unroll
        for (int k = 0; k < kSlots / 64; ++k) lamv = fmax(lamv, a.lam[lane + 64 * k]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lamv = fmax(lamv, __shfl_xor(lamv, o, 64));
        lamv = tb::lane_value(lamv, 0);
    }
    R tbk[K], cmk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double t = a.lam ? a.tau * lamv * a.chat[k] : a.tb[k];
        tbk[k] = (R)t;
        cmk[k] = (R)(1.0 / (1.0 + t));
    }
    const bool from_g = a.v == nullptr;
    const R vs = from_g ? (R)(1.0 / (1.0 + (a.lam ? a.tau * lamv * a.chat_in : a.tb_in))) : R(1);
    const R* __restrict__ vin_p = from_g ? a.G : a.v;

    const int tile = tb::xcd_block();
    const int tx = tile % a.tiles_x, rest = tile / a.tiles_x;
    const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
    const int xg = tx * OX - K + lane;
    const unsigned xi = (unsigned)fold(xg, nx, a.perx);
    const int y0 = ty * OY - K + wv * ROWS;  // first own row
    const int z0 = tz * a.zc;
    const int z1 = z0 + a.zc < nz ? z0 + a.zc : nz;
    const bool xout = lane >= K && lane < 64 - K && xg < nx;

    // weights of the faces: zero where the grid has none (walls)
    const R wxr = (a.perx ? nx > 1 : (xg >= 0 && xg < nx - 1)) ? a.wx : R(0);
    R wyf[ROWS + 1];  // between rows r - 1 and r
#pragma unroll
    for (int r = 0; r <= ROWS; ++r) {
        const int y = y0 + r - 1;
        wyf[r] = (a.pery ? ny > 1 : (y >= 0 && y < ny - 1)) ? a.wy : R(0);
    }
    const int64_t plane = (int64_t)nx * ny;
    int rowoff[RW];  // wave-uniform offsets of rows -1 .. ROWS within a plane
#pragma unroll
    for (int r = 0; r < RW; ++r) rowoff[r] = fold(y0 - 1 + r, ny, a.pery) * nx;

    R vc[K][ROWS];     // input of stage q + 1 on plane z - 1 - q
    R fz[K][ROWS];     // its weighted flux through the face below that plane
    R Lq[K + 1][RW];   // Lambda on planes z .. z - K
    R rc[K][ROWS], Gq[K][ROWS];  // 1/C and G on planes z - 1 .. z - K
    R nv[ROWS], nL[RW], nrc[ROWS], nG[ROWS];  // in flight: v, Lambda of plane z, 1/C and G of plane z - 1
    auto load_vL = [&](int z) {
        const int64_t pz = fold(z, nz, a.perz) * plane;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) nv[r] = (vin_p + (pz + rowoff[r + 1]))[xi];
#pragma unroll
        for (int r = 0; r < RW; ++r) nL[r] = (a.Lam + (pz + rowoff[r]))[xi];
    };
    auto load_cG = [&](int z) {
        const int64_t pz = fold(z, nz, a.perz) * plane;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            nrc[r] = (a.rC + (pz + rowoff[r + 1]))[xi];
            nG[r] = (a.G + (pz + rowoff[r + 1]))[xi];
        }
    };
    const int zs = z0 - K;  // first plane
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) vc[q][r] = fz[q][r] = rc[q][r] = Gq[q][r] = R(0);
#pragma unroll
    for (int q = 0; q <= K; ++q)
#pragma unroll
        for (int r = 0; r < RW; ++r) Lq[q][r] = R(0);
    load_vL(zs);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) vc[0][r] = vs * nv[r];
#pragma unroll
    for (int r = 0; r < RW; ++r) Lq[0][r] = nL[r];
    load_vL(zs + 1);
    load_cG(zs);
    const int wdn = wv > 0 ? wv - 1 : 0, wup = wv < WAVES - 1 ? wv + 1 : wv;
    auto publish = [&](int buf) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            sh[buf][q][wv][0][lane] = vc[q][0];
            sh[buf][q][wv][1][lane] = vc[q][ROWS - 1];
        }
    };
    publish(0);
    double dmax = 0.0, tmax = 0.0, bad = 0.0;
    int buf = 0;
    for (int z = zs + 1; z < z1 + K; ++z) {
        // plane z has arrived: shift the waiting planes and start the next loads
        R vin[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) vin[r] = vs * nv[r];
#pragma unroll
        for (int q = K; q > 0; --q)
#pragma unroll
            for (int r = 0; r < RW; ++r) Lq[q][r] = Lq[q - 1][r];
#pragma unroll
        for (int r = 0; r < RW; ++r) Lq[0][r] = nL[r];
#pragma unroll
        for (int q = K - 1; q > 0; --q)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                rc[q][r] = rc[q - 1][r];
                Gq[q][r] = Gq[q - 1][r];
            }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            rc[0][r] = nrc[r];
            Gq[0][r] = nG[r];
        }
        load_vL(z + 1);
        load_cG(z);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        R nxt[ROWS];  // the stage's input on the plane above
#pragma unroll
        for (int r = 0; r < ROWS; ++r) nxt[r] = vin[r];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int p = z - 1 - q;  // this stage's plane
            const R wzf = (a.perz ? nz > 1 : (p >= 0 && p < nz - 1)) ? a.wz : R(0);
            const R vlo = sh[buf][q][wdn][1][lane], vhi = sh[buf][q][wup][0][lane];
            R fy = wyf[0] * face_of<R, kHarm>(Lq[q + 1][0], Lq[q + 1][1]) * (vc[q][0] - vlo);
            R res[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const R c = vc[q][r], La = Lq[q + 1][r + 1];
                const R up = r < ROWS - 1 ? vc[q][r < ROWS - 1 ? r + 1 : r] : vhi;
                const R fx = wxr * face_of<R, kHarm>(La, from_right(La)) * (from_right(c) - c);
                const R fyu = wyf[r + 1] * face_of<R, kHarm>(La, Lq[q + 1][r + 2]) * (up - c);
                const R fzu = wzf * face_of<R, kHarm>(La, Lq[q][r + 1]) * (nxt[r] - c);
                const R acc = (fx - from_left(fx)) + (fyu - fy) + (fzu - fz[q][r]);
                fy = fyu;
                fz[q][r] = fzu;
                res[r] = cmk[q] * (Gq[q][r] + tbk[q] * c + rc[q][r] * acc);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                vc[q][r] = nxt[r];  // next step's centre
                nxt[r] = res[r];
            }
            if (q < K - 1 ? a.stages != nullptr : true) {
                if (p >= z0 && p < z1) {  // uniform
                    R* dst = (q < K - 1 ? a.stages + (int64_t)(q + 1) * a.sstride : a.out) + p * plane;
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        const int row = wv * ROWS + r, y = y0 + r;
                        if (row >= K && row < EXT_Y - K && y < ny && xout) {
                            (dst + (int64_t)y * nx)[(unsigned)xg] = res[r];
                            if (sizeof(R) == 8 && q == K - 1 && a.Tit) {
                                const double tn = (double)res[r];
                                if (a.ps.dmax)
                                    dmax = fmax(dmax, fabs(tn - (a.Tit + (p * plane + (int64_t)y * nx))[(unsigned)xg]));
                                tmax = fmax(tmax, fabs(tn));
                                if (!(tn > 0.0) || isinf(tn)) bad += 1.0;
                            }
                        }
                    }
                }
            }
        }
        buf ^= 1;
        publish(buf);
    }
    if (sizeof(R) == 8 && a.Tit) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
            tmax = fmax(tmax, __shfl_xor(tmax, o, 64));
            bad += __shfl_xor(bad, o, 64);
        }
        if (lane == 0) {
            const int sl = (int)(((int64_t)blockIdx.x * WAVES + wv) % kSlots);
            if (a.ps.dmax)
                atomicMax((unsigned long long*)(a.ps.dmax + sl), (unsigned long long)__double_as_longlong(dmax + 0.0));
            atomicMax((unsigned long long*)(a.ps.tmax + sl), (unsigned long long)__double_as_longlong(tmax + 0.0));
            if (bad != 0.0) atomicAdd(a.ps.bad + sl, bad);
        }
    }
}

// y rows per wave: what K stages' planes leave room for in the 256 VGPRs of
// two waves per SIMD (one row more spills)
template <typename R, int K>
constexpr int b3_rows() {
    return sizeof(R) == 4 ? 8 : (K == 3 ? 3 : 4);
}

template <typename R, int K>
void launch_b3d_k(hipStream_t s, const DevGrid& g, int face, B3Args<R>& a) {
    constexpr int rows = b3_rows<R, K>(), waves = 8;
    constexpr int OX = 64 - 2 * K, OY = rows * waves - 2 * K;
    a.tiles_x = (g.nx + OX - 1) / OX;
    a.tiles_y = (g.ny + OY - 1) / OY;
    // z chunks: one workgroup per CU at a time, each walking its chunk and
    // 2K planes more; the count with the fewest planes walked in turn
    const int64_t cols = (int64_t)a.tiles_x * a.tiles_y;
    int64_t best = 0;
    int zc = g.nz;
    for (int n = 1; n <= g.nz && n <= 4 * kCUs; ++n) {
        const int c = (g.nz + n - 1) / n;
        const int64_t wg = cols * ((g.nz + c - 1) / c);
        const int64_t cost = (wg + kCUs - 1) / kCUs * (c + 2 * K + 1);
        if (n == 1 || cost < best) {
            best = cost;
            zc = c;
        }
    }
    a.zc = zc;
    const dim3 grid((unsigned)(cols * ((g.nz + zc - 1) / zc))), block(64 * waves);
    if (face == 1) hipLaunchKernelGGL((k_b3d<R, K, rows, waves, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_b3d<R, K, rows, waves, false>), grid, block, 0, s, a);
}

}  // namespace

int b3d_stages(const DevGrid& g, int count) {
    if (!use_z3d(g)) return 1;
    const int launches = (count + KMAX3 - 1) / KMAX3;
    return (count + launches - 1) / launches;
}

template <typename R>
void launch_b3d(hipStream_t s, const DevGrid& g, int face, const R* v, const R* G, const R* Lam, const R* rC, R* out,
                Stages st, int K, double tau, const double* Tit, PassSlots ps, R* stages, int64_t sstride,
                StageParam sp_in) {
    B3Args<R> a{};
    a.v = v;
    a.G = G;
    a.Lam = Lam;
    a.rC = rC;
    a.out = out;
    a.stages = stages;
    a.sstride = sstride;
    a.lam = st.lam;
    a.tau = tau;
    for (int k = 0; k < K; ++k) {
        if (st.lam) a.chat[k] = st.chat[k];
        else a.tb[k] = st.tb[k];
    }
    a.tb_in = sp_in.tb;
    a.chat_in = sp_in.chat;
    a.Tit = Tit;
    a.ps = ps;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.perx = g.per[0];
    a.pery = g.per[1];
    a.perz = g.per[2];
    const double half = face == 1 ? 1.0 : 0.5;
    a.wx = (R)(half * tau * g.w[0]);
    a.wy = (R)(half * tau * g.w[1]);
    a.wz = (R)(half * tau * g.w[2]);
    if (K == 3) launch_b3d_k<R, 3>(s, g, face, a);
    else launch_b3d_k<R, 2>(s, g, face, a);
}

template void launch_b3d<double>(hipStream_t, const DevGrid&, int, const double*, const double*, const double*,
                                 const double*, double*, Stages, int, double, const double*, PassSlots, double*,
                                 int64_t, StageParam);
template void launch_b3d<float>(hipStream_t, const DevGrid&, int, const float*, const float*, const float*,
                                const float*, float*, Stages, int, double, const double*, PassSlots, float*, int64_t,
                                StageParam);

}  // namespace tlim
