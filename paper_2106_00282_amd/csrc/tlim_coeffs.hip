// Coefficients of a Picard pass and the Gershgorin bound on grids whose heat
// step has no source term (Sec. 3.4.2, eq. qk_dis; bound of eq. LIM).
//
// Per cell: Lambda = sum_k alpha_k lambda_k(T^(it)) and, where it changes,
// 1/C_eff; per cell the bound 2 rC sum_f w_f mean(Lambda_a, Lambda_b), folded
// into a max.  Without sources g = T^n, so no right-hand side is written (the
// stages read T^n), and with p_inf,1 = p_inf,2 the capacity depends on the
// partial densities only, which the parabolic step does not change: 1/C is
// then built by the first pass of a step and read by the others.
//
// The first pass of a step can also take the temperature relaxation
// (Sec. 3.4.1) that precedes it: every strip then relaxes its cells (halo
// rows included) from (alpha2, T1, T2, m1, m2) before building the
// coefficients at the relaxed state, and writes T^n and the relaxed alpha2
// of its own cells to separate arrays (alpha2 is not updated in place, as
// neighbouring strips still read the unrelaxed values of their halo).
//
// One wave owns a strip of 64 columns (62 output columns plus one halo
// column on each side) by kRows rows and marches down it, keeping the
// conductivities of three consecutive rows in registers; the x-neighbours
// come from the adjacent lanes (DPP).  Loads of T and alpha2 are coalesced
// 512 B rows; halo overhead is (kRows+2)/kRows x 64/62.  No LDS, no barrier:
// waves are independent.  Strips of 4 rows: more waves in flight hide the
// memory latency better than the smaller halo of 8 rows saves (the fused
// relaxation kernel measured 23.6 us against 30.2 us at 1024^2).
#include <hip/hip_runtime.h>

#include "tlim_device.h"
#include "tlim_internal.h"

namespace tlim {

namespace {

using phys::cell_conductivity;
using phys::inv_heat_capacity;
using tb::fmean;
using tb::fold;
using tb::from_left;
using tb::from_right;

constexpr int kRows = 4;
constexpr int kOut = 62;
constexpr int kWaves = 4;

struct Coef2DArgs {
    DevPhases ph;
    const double* T;      // T^(it); with relaxation: T1
    const double* T2;     // with relaxation
    double* Tn_out;       // with relaxation: the relaxed T
    double* a2_out;       // with relaxation or the update: the new alpha2
    const double* Tit;    // with the update: the iterate before T
    const double* a2n;    // with the update: the relaxed alpha2 (alpha2 at T^n)
    const double* alpha2;
    const double* m1;
    const double* m2;
    const double* g;      // T^n (read for the FP32 correction source only)
    const double* rC_in;  // 1/C of the step when it is not rebuilt
    double* Lam;          // nullable
    double* rC;           // written when rebuilt
    float* Lam32;         // FP32 contexts
    float* rC32;
    float* q32;
    float* w0;
    double* lam;          // accumulator row of the bound
    int nx, ny, perx, pery;
    double wx, wy, tau, eps;
    int face, rebuild, tiles_x, strips;
    // 3D grids
    int nz, perz, tiles_y, zc, waves;
    double wz;
};

// With kUpdate (unequal p_inf) the pass before this one ends here: alpha2 of the
// interface cells follows the new T, d alpha2 = -B1/(T^2 W) dT from the step's start
// with the coefficient at (T^(it), alpha2^(it)), on every row of the strip, and
// goes to an array of its own.  As a kernel of its own (15.4 us at 1024^2, then
// 16.0 for this one) the update reads T, T^(it), T^n, both alpha2 and m1, m2, most of
// which the coefficients need again; together 21.6 us.
template <bool kRelax, bool kSH, bool kUpdate = false>
__global__ void __launch_bounds__(64 * kWaves) k_coeffs2d(Coef2DArgs a) {
    const int lane = threadIdx.x & 63;
    const int strip = tb::xcd_block() * kWaves + (threadIdx.x >> 6);  // strips in XCD order
    if (strip >= a.strips) return;  // wave-uniform
    const int tx = strip % a.tiles_x, ty = strip / a.tiles_x;
    const int xg = tx * kOut - 1 + lane;
    const int xi = fold(xg, a.nx, a.perx);
    const bool out_lane = lane >= 1 && lane <= kOut && xg < a.nx;
    const bool fL = a.perx ? a.nx > 1 : xg > 0;
    const bool fR = a.perx ? a.nx > 1 : xg < a.nx - 1;
    const int y0 = ty * kRows;
    const bool q = a.q32 != nullptr;

    auto at = [&](int y) { return (int64_t)fold(y, a.ny, a.pery) * a.nx + xi; };
    // rows y0-1 .. y0+kRows: T, alpha2 -> Lambda (and g in FP32 contexts).
    // Every word the kernel reads is in flight before the first law
    // evaluation (one round trip to memory, not one per row): m1, m2 for the
    // relaxation, the Spitzer-Harm law and 1/C, and 1/C itself when kept.
    double Lw[kRows + 2], tw[kRows + 2], aw[kRows + 2], gw[kRows + 2];
    double m1w[kRows + 2], m2w[kRows + 2], rcw[kRows + 2];
    const bool need_m = kRelax || kSH || kUpdate || a.rebuild;
    {
        double t2w[kRows + 2], tiw[kRows + 2], anw[kRows + 2];
#pragma unroll
        for (int r = 0; r < kRows + 2; ++r) {
            const int64_t idx = at(y0 - 1 + r);
            tw[r] = a.T[idx];
            aw[r] = a.alpha2[idx];
            if constexpr (kRelax) t2w[r] = a.T2[idx];
            else gw[r] = kUpdate || q ? a.g[idx] : 0.0;
            if constexpr (kUpdate) {
                tiw[r] = a.Tit[idx];
                anw[r] = a.a2n[idx];
            }
            m1w[r] = need_m ? a.m1[idx] : 0.0;
            m2w[r] = need_m ? a.m2[idx] : 0.0;
            rcw[r] = a.rebuild ? 0.0 : a.rC_in[idx];
        }
        if constexpr (kRelax) {
#pragma unroll
            for (int r = 0; r < kRows + 2; ++r) {
                phys::relax_cell(a.ph, a.eps, aw[r], tw[r], t2w[r], m1w[r], m2w[r], tw[r], aw[r]);
                gw[r] = tw[r];  // g = T^n, the relaxed T
            }
        }
        if constexpr (kUpdate) {
            const double B1 = a.ph.pinf[0] - a.ph.pinf[1];
#pragma unroll
            for (int r = 0; r < kRows + 2; ++r)
                if (phys::is_mixed(anw[r], a.eps))
                    aw[r] = phys::updated_alpha2(a.ph, B1, anw[r], aw[r], tw[r], tiw[r], gw[r], m1w[r], m2w[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < kRows + 2; ++r) {
        if constexpr (kSH) Lw[r] = phys::cell_conductivity(a.ph, tw[r], aw[r], m1w[r] + m2w[r]);
        else Lw[r] = phys::cell_conductivity_pow(a.ph, tw[r], aw[r]);
    }

    double bound = 0.0;
#pragma unroll
    for (int r = 1; r <= kRows; ++r) {
        const int y = y0 + r - 1;
        const double L = Lw[r], Lm = Lw[r - 1], Lp = Lw[r + 1];
        const double Ll = from_left(L), Lr = from_right(L);
        const float Lf = (float)L;
        const float Llf = from_left(Lf), Lrf = from_right(Lf);
        const double gl = from_left(gw[r]), gr = from_right(gw[r]);
        if (out_lane && y < a.ny) {
            const int64_t o = (int64_t)y * a.nx + xg;
            const bool fD = a.pery ? a.ny > 1 : y > 0;
            const bool fU = a.pery ? a.ny > 1 : y < a.ny - 1;
            if constexpr (kRelax) a.Tn_out[o] = tw[r];
            if constexpr (kRelax || kUpdate) a.a2_out[o] = aw[r];
            double rc;
            if (a.rebuild) {
                rc = inv_heat_capacity(a.ph, a.eps, tw[r], aw[r], m1w[r], m2w[r]);
                a.rC[o] = rc;
                if (a.rC32) a.rC32[o] = (float)rc;
            } else {
                rc = rcw[r];
            }
            if (a.Lam) a.Lam[o] = L;
            if (a.Lam32) a.Lam32[o] = Lf;
            // faces in the order -x, +x, -y, +y
            double d = 0.0;
            if (fL) d += a.wx * fmean<double>(L, Ll, a.face);
            if (fR) d += a.wx * fmean<double>(L, Lr, a.face);
            if (fD) d += a.wy * fmean<double>(L, Lm, a.face);
            if (fU) d += a.wy * fmean<double>(L, Lp, a.face);
            bound = fmax(bound, 2.0 * d * rc);
            if (q) {
                // q = -tau rC' D' g from the float-rounded Lambda' and rC'
                const double La = (double)Lf, rf = (double)(float)rc, ga = gw[r];
                double S = 0.0;
                if (fL) S += a.wx * fmean<double>(La, (double)Llf, a.face) * (ga - gl);
                if (fR) S += a.wx * fmean<double>(La, (double)Lrf, a.face) * (ga - gr);
                if (fD) S += a.wy * fmean<double>(La, (double)(float)Lm, a.face) * (ga - gw[r - 1]);
                if (fU) S += a.wy * fmean<double>(La, (double)(float)Lp, a.face) * (ga - gw[r + 1]);
                a.q32[o] = (float)(-a.tau * rf * S);
                if (a.w0) a.w0[o] = 0.0f;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, __shfl_xor(bound, o, 64));
    if (lane == 0) {
        const int sl = strip % kSlots;
        atomicMax((unsigned long long*)(a.lam + sl), (unsigned long long)__double_as_longlong(bound + 0.0));
    }
}

// 3D grids: the same per-cell work.  A workgroup of four waves (fewer on grids of
// up to six rows) owns 62 columns by 4 kRows3 rows and marches through a chunk of z planes, each wave keeping the
// conductivities (and g) of its kRows3 rows in the previous, current and next
// plane in registers.  Rows next to another wave's come through LDS (one
// barrier a plane, two buffers); the rows beyond the workgroup's are built by
// its first and last wave.
//
// What bounds it: memory, at 512^3 (FP32 form, 5.4 GB a pass: 4.1 TB/s); on
// smaller grids latency.  With independent waves the law and the relaxation ran
// on 4 rows to write 2, and that arithmetic was the bound: 1743 us against 1322
// at 512^3, 327 against 220 at 256^3, 37 against 29 at 128^3; with the
// relaxation 3242 against 2636, 448 against 364 and 57 against 46.  Four rows a
// wave need half again the registers and are slower (1450 us at 512^3).  Waves
// past the last row would evaluate the laws all the same: at 1000 x 1 x 1000 four
// took 56 us (92 with the relaxation) and one takes 24 (40); at 1000 x 4 x 1000 73
// (116), and two take 46 (86).
constexpr int kRows3 = 2;

template <bool kRelax, bool kSH>
__global__ void __launch_bounds__(64 * kWaves) k_coeffs3d(Coef2DArgs a) {
    constexpr int kRO = kRows3;
    __shared__ double sL[2][kWaves][2][64], sg[2][kWaves][2][64];  // [plane parity][wave][first, last row]
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = a.waves;
    const int wid = blockIdx.x;  // launch order: XCD order measured up to 20% slower
    const int tx = wid % a.tiles_x, rest = wid / a.tiles_x;
    const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int xg = tx * kOut - 1 + lane;
    const int xi = fold(xg, nx, a.perx);
    const bool out_lane = lane >= 1 && lane <= kOut && xg < nx;
    const bool fL = a.perx ? nx > 1 : xg > 0;
    const bool fR = a.perx ? nx > 1 : xg < nx - 1;
    const int y0 = (ty * nw + w) * kRO, z0 = tz * a.zc;
    const int z1 = z0 + a.zc < nz ? z0 + a.zc : nz;
    const bool q = a.q32 != nullptr;
    // this wave builds the row before or after its own as well (a single wave has
    // no other rows: two periodic rows are each other's neighbours)
    const bool halo = nw > 1 && (w == 0 || w == nw - 1);

    // 32-bit element offsets (the launcher requires N < 2^32); row kRO: the halo row
    unsigned rowoff[kRO + 1];
#pragma unroll
    for (int r = 0; r < kRO; ++r) rowoff[r] = (unsigned)fold(y0 + r, ny, a.pery) * (unsigned)nx;
    rowoff[kRO] = (unsigned)fold(w == 0 ? y0 - 1 : y0 + kRO, ny, a.pery) * (unsigned)nx;
    const unsigned plane = (unsigned)nx * (unsigned)ny;
    // T, alpha2 (relaxed when kRelax), 1/C, Lambda and g of the rows of plane z
    auto load_plane = [&](int z, double* tw, double* aw, double* rw, double* Lw, double* gw, bool h) {
        const unsigned pz = (unsigned)fold(z, nz, a.perz) * plane;
        // all rows' words in flight before the first law evaluation
        double t2w[kRO + 1], m1w[kRO + 1], m2w[kRO + 1];
#pragma unroll
        for (int r = 0; r <= kRO; ++r) {
            if (r == kRO && !h) continue;
            const unsigned idx = pz + rowoff[r] + (unsigned)xi;
            tw[r] = a.T[idx];
            aw[r] = a.alpha2[idx];
            if constexpr (kRelax) t2w[r] = a.T2[idx];
            else gw[r] = q ? a.g[idx] : 0.0;
            if (kRelax || kSH || (r < kRO && a.rebuild)) {
                m1w[r] = a.m1[idx];
                m2w[r] = a.m2[idx];
            }
            if (!kRelax && r < kRO && !a.rebuild) rw[r] = a.rC_in[idx];
        }
#pragma unroll
        for (int r = 0; r <= kRO; ++r) {
            if (r == kRO && !h) continue;
            if constexpr (kRelax) {
                phys::relax_cell(a.ph, a.eps, aw[r], tw[r], t2w[r], m1w[r], m2w[r], tw[r], aw[r]);
                gw[r] = tw[r];
            }
            if constexpr (kSH) Lw[r] = phys::cell_conductivity(a.ph, tw[r], aw[r], m1w[r] + m2w[r]);
            else Lw[r] = phys::cell_conductivity_pow(a.ph, tw[r], aw[r]);
            if (r < kRO && (kRelax || a.rebuild)) rw[r] = inv_heat_capacity(a.ph, a.eps, tw[r], aw[r], m1w[r], m2w[r]);
        }
    };
    auto share = [&](int b, const double* Lw, const double* gw) {
        sL[b][w][0][lane] = Lw[0];
        sL[b][w][1][lane] = Lw[kRO - 1];
        if (q) {
            sg[b][w][0][lane] = gw[0];
            sg[b][w][1][lane] = gw[kRO - 1];
        }
    };
    // window: Lambda and g of planes z-1, z, z+1; T, alpha2 and 1/C of z and z+1
    double Lm[kRO + 1], gm[kRO + 1], tc[kRO + 1], ac[kRO + 1], rc[kRO + 1], Lc[kRO + 1], gc[kRO + 1];
    double tp[kRO + 1], ap[kRO + 1], rp[kRO + 1], Lp[kRO + 1], gp[kRO + 1];
    load_plane(z0 - 1, tp, ap, rp, Lm, gm, false);
    load_plane(z0, tc, ac, rc, Lc, gc, halo);
    share(0, Lc, gc);
    __syncthreads();
    double bound = 0.0;
    int b = 0;
    for (int z = z0; z < z1; ++z) {
        load_plane(z + 1, tp, ap, rp, Lp, gp, halo);
        const bool fB = a.perz ? nz > 1 : z > 0;
        const bool fF = a.perz ? nz > 1 : z < nz - 1;
        // the rows before and after this wave's own
        const int wdn = w > 0 ? w - 1 : nw - 1, wup = w < nw - 1 ? w + 1 : 0;
        const double Ldn = w == 0 && nw > 1 ? Lc[kRO] : sL[b][wdn][1][lane];
        const double Lup = w == nw - 1 && nw > 1 ? Lc[kRO] : sL[b][wup][0][lane];
        double gdn = 0.0, gup = 0.0;
        if (q) {
            gdn = w == 0 && nw > 1 ? gc[kRO] : sg[b][wdn][1][lane];
            gup = w == nw - 1 && nw > 1 ? gc[kRO] : sg[b][wup][0][lane];
        }
#pragma unroll
        for (int r = 0; r < kRO; ++r) {
            const int y = y0 + r;
            const double L = Lc[r];
            const double Ll = from_left(L), Lr = from_right(L);
            const double Ld = r > 0 ? Lc[r > 0 ? r - 1 : 0] : Ldn, Lu = r < kRO - 1 ? Lc[r + 1] : Lup;
            const float Lf = (float)L;
            const float Llf = from_left(Lf), Lrf = from_right(Lf);
            const double gl = from_left(gc[r]), gr = from_right(gc[r]);
            if (out_lane && y < ny) {
                const unsigned o = (unsigned)z * plane + (unsigned)y * (unsigned)nx + (unsigned)xg;
                const bool fD = a.pery ? ny > 1 : y > 0;
                const bool fU = a.pery ? ny > 1 : y < ny - 1;
                if constexpr (kRelax) {
                    a.Tn_out[o] = tc[r];
                    a.a2_out[o] = ac[r];
                }
                if (kRelax || a.rebuild) {
                    a.rC[o] = rc[r];
                    if (a.rC32) a.rC32[o] = (float)rc[r];
                }
                if (a.Lam) a.Lam[o] = L;
                if (a.Lam32) a.Lam32[o] = Lf;
                // faces in the order -x, +x, -y, +y, -z, +z
                double d = 0.0;
                if (fL) d += a.wx * fmean<double>(L, Ll, a.face);
                if (fR) d += a.wx * fmean<double>(L, Lr, a.face);
                if (fD) d += a.wy * fmean<double>(L, Ld, a.face);
                if (fU) d += a.wy * fmean<double>(L, Lu, a.face);
                if (fB) d += a.wz * fmean<double>(L, Lm[r], a.face);
                if (fF) d += a.wz * fmean<double>(L, Lp[r], a.face);
                bound = fmax(bound, 2.0 * d * rc[r]);
                if (q) {
                    const double La = (double)Lf, rf = (double)(float)rc[r], ga = gc[r];
                    const double gd = r > 0 ? gc[r > 0 ? r - 1 : 0] : gdn, gu = r < kRO - 1 ? gc[r + 1] : gup;
                    double S = 0.0;
                    if (fL) S += a.wx * fmean<double>(La, (double)Llf, a.face) * (ga - gl);
                    if (fR) S += a.wx * fmean<double>(La, (double)Lrf, a.face) * (ga - gr);
                    if (fD) S += a.wy * fmean<double>(La, (double)(float)Ld, a.face) * (ga - gd);
                    if (fU) S += a.wy * fmean<double>(La, (double)(float)Lu, a.face) * (ga - gu);
                    if (fB) S += a.wz * fmean<double>(La, (double)(float)Lm[r], a.face) * (ga - gm[r]);
                    if (fF) S += a.wz * fmean<double>(La, (double)(float)Lp[r], a.face) * (ga - gp[r]);
                    a.q32[o] = (float)(-a.tau * rf * S);
                    if (a.w0) a.w0[o] = 0.0f;
                }
            }
        }
        // the other buffer was last read before the last barrier
        b ^= 1;
        share(b, Lp, gp);
        __syncthreads();
#pragma unroll
        for (int r = 0; r <= kRO; ++r) {
            Lm[r] = Lc[r];
            gm[r] = gc[r];
            tc[r] = tp[r];
            ac[r] = ap[r];
            rc[r] = rp[r];
            Lc[r] = Lp[r];
            gc[r] = gp[r];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, __shfl_xor(bound, o, 64));
    if (lane == 0) {
        const int sl = (int)(((int64_t)wid * nw + w) % kSlots);
        atomicMax((unsigned long long*)(a.lam + sl), (unsigned long long)__double_as_longlong(bound + 0.0));
    }
}

// The viscous part's coefficients and sources: a wave owns 62 columns by
// kRowsV rows and marches a chunk of z planes with the neighbours in registers
// (loads of the rows beside its own hit the caches), any grid.
constexpr int kRowsV = 4;

struct StripArgs {
    // coefficients: mu = (1 - alpha2) mu_1 + alpha2 mu_2, 1/rho, bounds
    const double* alpha2;
    const double* m1;
    const double* m2;
    double* Lam;
    double* rC;
    float* Lam32;
    float* rC32;
    double* rows;  // the components' accumulator rows
    double mu0, mu1, wc[3][3];
    int mask;
    // correction source
    const double* g;
    const double* v0;
    const float* L32;
    const float* r32;
    float* q;
    float* w0;
    double tau, w[3];
    int nx, ny, nz, perx, pery, perz, face, tiles_x, tiles_y, zc, strips;
};

struct Strip {
    int xg, y0, z0, z1;
    bool out_lane, fL, fR;
    int64_t plane, rowoff[kRowsV + 2];
    __device__ __forceinline__ Strip(const StripArgs& a, int wid, int lane) {
        const int tx = wid % a.tiles_x, rest = wid / a.tiles_x;
        const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
        xg = tx * kOut - 1 + lane;
        out_lane = lane >= 1 && lane <= kOut && xg < a.nx;
        fL = a.perx ? a.nx > 1 : xg > 0;
        fR = a.perx ? a.nx > 1 : xg < a.nx - 1;
        y0 = ty * kRowsV;
        z0 = tz * a.zc;
        z1 = z0 + a.zc < a.nz ? z0 + a.zc : a.nz;
        const int xi = fold(xg, a.nx, a.perx);
        plane = (int64_t)a.nx * a.ny;
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) rowoff[r] = (int64_t)fold(y0 - 1 + r, a.ny, a.pery) * a.nx + xi;
    }
    __device__ __forceinline__ int64_t base(const StripArgs& a, int z) const { return fold(z, a.nz, a.perz) * plane; }
};

// mu, 1/rho and the Gershgorin bounds 2 rC sum_f w_f mean(mu_a, mu_b) of the
// three velocity components.  Bound by memory: 3 arrays read, 4 written, each
// once.  As two kernels, the second reading mu and 1/rho back per face without
// reuse, the bounds took 219 us more at 256^3.
__global__ void __launch_bounds__(64 * kWaves) k_visc_coeffs(StripArgs a) {
    const int lane = threadIdx.x & 63, wid = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (wid >= a.strips) return;  // wave-uniform
    const Strip t(a, wid, lane);
    auto load = [&](int z, double* L) {
        const double* p = a.alpha2 + t.base(a, z);
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) L[r] = p[t.rowoff[r]];
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) L[r] = (1.0 - L[r]) * a.mu0 + L[r] * a.mu1;
    };
    double Lm[kRowsV + 2], Lc[kRowsV + 2], Lp[kRowsV + 2], mx[3] = {0.0, 0.0, 0.0};
    load(t.z0, Lc);
#pragma unroll
    for (int r = 0; r < kRowsV + 2; ++r) Lm[r] = Lp[r] = 0.0;
    if (a.nz > 1) load(t.z0 - 1, Lm);
    for (int z = t.z0; z < t.z1; ++z) {
        double rho[kRowsV];
        {
            const int64_t b = t.base(a, z);
            double x1[kRowsV], x2[kRowsV];
#pragma unroll
            for (int r = 0; r < kRowsV; ++r) {
                x1[r] = a.m1[b + t.rowoff[r + 1]];
                x2[r] = a.m2[b + t.rowoff[r + 1]];
            }
            if (a.nz > 1) load(z + 1, Lp);
#pragma unroll
            for (int r = 0; r < kRowsV; ++r) rho[r] = x1[r] + x2[r];
        }
        const bool fB = a.perz ? a.nz > 1 : z > 0;
        const bool fF = a.perz ? a.nz > 1 : z < a.nz - 1;
#pragma unroll
        for (int r = 1; r <= kRowsV; ++r) {
            const int y = t.y0 + r - 1;
            const double L = Lc[r];
            const double Ll = from_left(L), Lr = from_right(L);
            if (t.out_lane && y < a.ny) {
                const int64_t o = z * t.plane + t.rowoff[r];
                const double rc = 1.0 / rho[r - 1];
                a.Lam[o] = L;
                a.rC[o] = rc;
                if (a.Lam32) {
                    a.Lam32[o] = (float)L;
                    a.rC32[o] = (float)rc;
                }
                const bool fD = a.pery ? a.ny > 1 : y > 0;
                const bool fU = a.pery ? a.ny > 1 : y < a.ny - 1;
                // faces in the order -x, +x, -y, +y, -z, +z
                const double m[6] = {t.fL ? fmean<double>(L, Ll, a.face) : 0.0,
                                     t.fR ? fmean<double>(L, Lr, a.face) : 0.0,
                                     fD ? fmean<double>(L, Lc[r - 1], a.face) : 0.0,
                                     fU ? fmean<double>(L, Lc[r + 1], a.face) : 0.0,
                                     fB ? fmean<double>(L, Lm[r], a.face) : 0.0,
                                     fF ? fmean<double>(L, Lp[r], a.face) : 0.0};
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double d = 0.0;
#pragma unroll
                    for (int f = 0; f < 6; ++f) d += a.wc[c][f >> 1] * m[f];
                    mx[c] = fmax(mx[c], 2.0 * d * rc);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) {
            Lm[r] = Lc[r];
            Lc[r] = Lp[r];
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (!((a.mask >> c) & 1)) continue;  // uniform
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx[c] = fmax(mx[c], __shfl_xor(mx[c], o, 64));
        if (lane == 0)
            atomicMax((unsigned long long*)(a.rows + (size_t)c * kSlots + wid % kSlots),
                      (unsigned long long)__double_as_longlong(mx[c] + 0.0));
    }
}

// q = -tau rC' D' g of a pass whose coefficients are already in place, from the
// float-rounded Lambda' and rC'; w0 = v0 - g where it is not zero.  Bound by
// memory: 3 arrays read, 1 written (20 B a cell).  One thread per cell with
// its neighbours from memory took 213 us at 256^3.
__global__ void __launch_bounds__(64 * kWaves) k_q32(StripArgs a) {
    const int lane = threadIdx.x & 63, wid = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (wid >= a.strips) return;  // wave-uniform
    const Strip t(a, wid, lane);
    auto load = [&](int z, double* g, float* L) {
        const int64_t b = t.base(a, z);
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) {
            g[r] = a.g[b + t.rowoff[r]];
            L[r] = a.L32[b + t.rowoff[r]];
        }
    };
    double gm[kRowsV + 2], gc[kRowsV + 2], gp[kRowsV + 2];
    float Lm[kRowsV + 2], Lc[kRowsV + 2], Lp[kRowsV + 2];
    load(t.z0, gc, Lc);
#pragma unroll
    for (int r = 0; r < kRowsV + 2; ++r) {
        gm[r] = gp[r] = 0.0;
        Lm[r] = Lp[r] = 0.0f;
    }
    if (a.nz > 1) load(t.z0 - 1, gm, Lm);
    for (int z = t.z0; z < t.z1; ++z) {
        float rc[kRowsV];
        double v0[kRowsV];
        {
            const int64_t b = t.base(a, z);
#pragma unroll
            for (int r = 0; r < kRowsV; ++r) {
                rc[r] = a.r32[b + t.rowoff[r + 1]];
                v0[r] = a.w0 ? a.v0[b + t.rowoff[r + 1]] : 0.0;
            }
            if (a.nz > 1) load(z + 1, gp, Lp);
        }
        const bool fB = a.perz ? a.nz > 1 : z > 0;
        const bool fF = a.perz ? a.nz > 1 : z < a.nz - 1;
#pragma unroll
        for (int r = 1; r <= kRowsV; ++r) {
            const int y = t.y0 + r - 1;
            const double ga = gc[r], La = (double)Lc[r];
            const double gl = from_left(ga), gr = from_right(ga);
            const float Ll = from_left(Lc[r]), Lr = from_right(Lc[r]);
            if (t.out_lane && y < a.ny) {
                const int64_t o = z * t.plane + t.rowoff[r];
                const bool fD = a.pery ? a.ny > 1 : y > 0;
                const bool fU = a.pery ? a.ny > 1 : y < a.ny - 1;
                double S = 0.0;
                if (t.fL) S += a.w[0] * fmean<double>(La, (double)Ll, a.face) * (ga - gl);
                if (t.fR) S += a.w[0] * fmean<double>(La, (double)Lr, a.face) * (ga - gr);
                if (fD) S += a.w[1] * fmean<double>(La, (double)Lc[r - 1], a.face) * (ga - gc[r - 1]);
                if (fU) S += a.w[1] * fmean<double>(La, (double)Lc[r + 1], a.face) * (ga - gc[r + 1]);
                if (fB) S += a.w[2] * fmean<double>(La, (double)Lm[r], a.face) * (ga - gm[r]);
                if (fF) S += a.w[2] * fmean<double>(La, (double)Lp[r], a.face) * (ga - gp[r]);
                a.q[o] = (float)(-a.tau * (double)rc[r - 1] * S);
                if (a.w0) a.w0[o] = (float)(v0[r - 1] - ga);
            }
        }
#pragma unroll
        for (int r = 0; r < kRowsV + 2; ++r) {
            gm[r] = gc[r];
            gc[r] = gp[r];
            Lm[r] = Lc[r];
            Lc[r] = Lp[r];
        }
    }
}

// Grid of a strip kernel: z chunks for about 8192 waves, 4 to 16 planes each.
dim3 strip_grid(const DevGrid& g, int face, StripArgs& a) {
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.perx = g.per[0];
    a.pery = g.per[1];
    a.perz = g.per[2];
    a.face = face;
    a.tiles_x = (g.nx + kOut - 1) / kOut;
    a.tiles_y = (g.ny + kRowsV - 1) / kRowsV;
    const int64_t cols = (int64_t)a.tiles_x * a.tiles_y;
    int64_t zc = (int64_t)g.nz * cols / 8192;
    zc = zc < 4 ? 4 : (zc > 16 ? 16 : zc);
    a.zc = (int)zc;
    a.strips = (int)(cols * ((g.nz + a.zc - 1) / a.zc));
    return dim3((unsigned)((a.strips + kWaves - 1) / kWaves));
}

}  // namespace

bool coeffs2d_applies(const DevGrid& g) { return g.nz == 1 || g.N < ((int64_t)1 << 32); }

void launch_coeffs2d(hipStream_t s, const DevGrid& g, const DevPhases& ph, double eps, double tau, int face,
                     const double* T, const double* alpha2, const double* m1, const double* m2, const double* Tn,
                     int rebuild, double* Lam, double* rC, float* Lam32, float* rC32, float* q32, float* w0,
                     double* lam, const double* T2_relax, double* Tn_out, double* a2_out, const double* Tit,
                     const double* a2n) {
    Coef2DArgs a{};
    a.Tit = Tit;
    a.a2n = a2n;
    a.ph = ph;
    a.T = T;
    a.T2 = T2_relax;
    a.Tn_out = Tn_out;
    a.a2_out = a2_out;
    a.alpha2 = alpha2;
    a.m1 = m1;
    a.m2 = m2;
    a.g = Tn;
    a.rC_in = rC;
    a.Lam = Lam;
    a.rC = rC;
    a.Lam32 = Lam32;
    a.rC32 = rC32;
    a.q32 = q32;
    a.w0 = w0;
    a.lam = lam;
    a.nx = g.nx;
    a.ny = g.ny;
    a.perx = g.per[0];
    a.pery = g.per[1];
    a.wx = g.w[0];
    a.wy = g.w[1];
    a.tau = tau;
    a.eps = eps;
    a.face = face;
    a.rebuild = rebuild;
    a.tiles_x = (g.nx + kOut - 1) / kOut;
    if (T2_relax) a.rebuild = 1;
    if (g.nz == 1) {
        a.strips = a.tiles_x * ((g.ny + kRows - 1) / kRows);
        const int blocks = (a.strips + kWaves - 1) / kWaves;
        if (Tit) {
            if (ph.spitzer) hipLaunchKernelGGL((k_coeffs2d<false, true, true>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
            else hipLaunchKernelGGL((k_coeffs2d<false, false, true>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
        } else if (ph.spitzer) {
            if (T2_relax) hipLaunchKernelGGL((k_coeffs2d<true, true>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
            else hipLaunchKernelGGL((k_coeffs2d<false, true>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
        } else {
            if (T2_relax) hipLaunchKernelGGL((k_coeffs2d<true, false>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
            else hipLaunchKernelGGL((k_coeffs2d<false, false>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, a);
        }
        return;
    }
    a.nz = g.nz;
    a.perz = g.per[2];
    a.wz = g.w[2];
    a.waves = (g.ny + kRows3 - 1) / kRows3;
    if (a.waves > kWaves) a.waves = kWaves;
    a.tiles_y = (g.ny + a.waves * kRows3 - 1) / (a.waves * kRows3);
    // z chunks sized for about 4096 waves, at least 4 planes each and at most
    // 16: the workgroups in flight then work on neighbouring planes.  With the
    // relaxation's ten streams 8 are better (512^3: 2636 us against 2755 with 16
    // and 3560 with 64; without it 1382, 1322 and 1350).
    const int64_t cols = (int64_t)a.tiles_x * a.tiles_y;
    const int64_t cap = T2_relax ? 8 : 16;
    int64_t zc = (int64_t)g.nz * cols * a.waves / 4096;
    zc = zc < 4 ? 4 : (zc > cap ? cap : zc);
    a.zc = (int)zc;
    const unsigned blocks = (unsigned)(cols * ((g.nz + a.zc - 1) / a.zc));
    if (ph.spitzer) {
        if (T2_relax) hipLaunchKernelGGL((k_coeffs3d<true, true>), dim3(blocks), dim3(64 * a.waves), 0, s, a);
        else hipLaunchKernelGGL((k_coeffs3d<false, true>), dim3(blocks), dim3(64 * a.waves), 0, s, a);
    } else {
        if (T2_relax) hipLaunchKernelGGL((k_coeffs3d<true, false>), dim3(blocks), dim3(64 * a.waves), 0, s, a);
        else hipLaunchKernelGGL((k_coeffs3d<false, false>), dim3(blocks), dim3(64 * a.waves), 0, s, a);
    }
}

void launch_visc_coeffs(hipStream_t s, const DevGrid& g, const DevPhases& ph, int face, const double* alpha2,
                        const double* m1, const double* m2, double* Lam, double* rC, float* Lam32, float* rC32,
                        const double wc[3][3], int mask, double* rows) {
    StripArgs a{};
    a.alpha2 = alpha2;
    a.m1 = m1;
    a.m2 = m2;
    a.Lam = Lam;
    a.rC = rC;
    a.Lam32 = Lam32;
    a.rC32 = rC32;
    a.rows = rows;
    a.mu0 = ph.mu[0];
    a.mu1 = ph.mu[1];
    for (int c = 0; c < 3; ++c)
        for (int d = 0; d < 3; ++d) a.wc[c][d] = wc[c][d];
    a.mask = mask;
    const dim3 grid = strip_grid(g, face, a);
    hipLaunchKernelGGL(k_visc_coeffs, grid, dim3(64 * kWaves), 0, s, a);
}

void launch_q32(hipStream_t s, const DevGrid& g, int face, const double* rhs, const double* v0,
                const float* Lam32, const float* rC32, double tau, float* q, float* w0) {
    StripArgs a{};
    a.g = rhs;
    a.v0 = v0;
    a.L32 = Lam32;
    a.r32 = rC32;
    a.q = q;
    a.w0 = w0;
    a.tau = tau;
    for (int d = 0; d < 3; ++d) a.w[d] = g.w[d];
    const dim3 grid = strip_grid(g, face, a);
    hipLaunchKernelGGL(k_q32, grid, dim3(64 * kWaves), 0, s, a);
}

}  // namespace tlim
