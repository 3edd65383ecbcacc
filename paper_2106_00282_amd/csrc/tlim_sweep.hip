// Inner LIM stages (eq. LIM) with temporal blocking for 2D grids.
//
// One stage of eq. LIM is a 5-point explicit update,
//   v^(m)_a = c_m (G_a + tau b_m v^(m-1)_a - sum_f kappa_af (v^(m-1)_a - v^(m-1)_f)),
//   kappa_af = tau / C_a * w_f * Lambda_f,
// with G = g = T^n + tau f (FP64 form) or G = -tau A' g (FP32 correction form,
// where v is the correction w = v - g).  The final stage (b = 0) of the FP64
// form is the same update with c = 1.
//
// k_tb2d advances K stages per launch.  A workgroup of 16 wave64s loads an
// extended tile once (v, G, Lambda, 1/C; every row's loads in flight before
// the first is used), builds the four kappa of every cell in registers, and
// then runs the K stages out of registers:
//   - each lane owns C adjacent cells of a row (C = 1 or 2) in RW consecutive
//     rows: x-neighbours come from the lane's own cells or from the adjacent
//     lanes through DPP wave shifts;
//   - y-neighbours are the lane's own registers, except at the seams between
//     waves, which go through a double-buffered LDS row (one barrier per
//     stage).
// Cells within K of the extended tile's edge go stale one ring per stage;
// the inner (64C-2K) x (16RW-2K) cells are exact and written out.
//
// What bounds it: one workgroup per CU, so a launch is its start (2 us), its
// load phase, its stages and its epilogue in turn.  The stage loop runs at
// about the VALU issue rate (per cell and stage in double: 8 operations, and
// 2 (C = 2) or 4 (C = 1) DPP moves).  On the 1024^2 grid a double launch of 8
// stages takes 17.5 us on 128 x 64 tiles (20.5 us on 64 x 128 tiles with the
// rows loaded one round trip after the other, the factor c_m applied per
// stage and one cell per lane), 25 us with the next pass's coefficients
// built in its epilogue (33 us), 31 us with the next step's start (39 us).  Smaller grids
// leave CUs idle on such tiles and take smaller ones (Shape below).
// Bytes per launch: 4 words read per extended cell + 1 word written per
// output cell, for K stages.
#include <hip/hip_runtime.h>

#include "tlim_device.h"
#include "tlim_sweep.h"

namespace tlim {

namespace {

using tb::row_index;
using tb::lane_value;

constexpr int KMAX_TB = 16;  // stages per launch
constexpr int NWAVES = 16;   // waves per workgroup
constexpr int kCUs = 256;

// Tiles of a workgroup: C cells per lane in x by RW rows per wave in y.  A
// launch of K stages takes about 2 us plus, for each round of one workgroup
// per CU, base + fill * (share of the CUs with a tile) + K * stage, in us
// (double, float; fitted to 96^2 .. 2048^2 grids at K = 2 .. 15).  Grids that
// leave CUs idle on large tiles run on smaller ones: 512 x 300 in double at
// K = 8 takes 12.7 us on 128 x 64 tiles, 15.5 on 64 x 128, 9.4 on 64 x 64 and
// 7.2 on 64 x 32; 1024^2 takes 17.8, 19.3, 19.6 and 25.1.
struct Shape {
    int c, rw;
    double base[2], fill[2], stage[2];
    int ext_x() const { return 64 * c; }
    int ext_y() const { return NWAVES * rw; }
};
enum { S_WIDE, S_TALL, S_SQUARE, S_FLAT, kShapes };
constexpr Shape kShapeTab[kShapes] = {{2, 4, {5.1, 3.7}, {3.6, 0.9}, {0.76, 0.55}},
                                      {1, 8, {7.1, 3.9}, {2.6, 0.9}, {0.81, 0.57}},
                                      {1, 4, {4.0, 2.2}, {1.2, 1.0}, {0.41, 0.38}},
                                      {1, 2, {2.6, 1.6}, {1.4, 1.4}, {0.32, 0.34}}};

// Cost of a launch of K stages (halo H) on tiles of shape i; 0 where the
// tile does not apply.
double launch_cost(const DevGrid& g, int i, int K, int H, bool f32) {
    const Shape& t = kShapeTab[i];
    // two cells per lane: a lane's pair must not straddle a periodic wrap
    if (t.c == 2 && (g.nx < 2 || (g.per[0] && g.nx % 2))) return 0.0;
    const int hx = t.c == 2 ? (H + 1) & ~1 : H;
    const int ox = t.ext_x() - 2 * hx, oy = t.ext_y() - 2 * H;
    if (ox < 4 || oy < 4) return 0.0;
    const int64_t tiles = (int64_t)((g.nx + ox - 1) / ox) * ((g.ny + oy - 1) / oy);
    const int64_t rounds = (tiles + kCUs - 1) / kCUs;
    const double share = tiles < kCUs ? (double)tiles / kCUs : 1.0;
    return 2.0 + (double)rounds * (t.base[f32] + t.fill[f32] * share + K * t.stage[f32]);
}

// The shape with the least cost for K stages and halo H.
int best_shape(const DevGrid& g, int K, int H, bool f32, double* cost = nullptr) {
    int best = -1;
    double low = 0.0;
    for (int i = 0; i < kShapes; ++i) {
        const double c = launch_cost(g, i, K, H, f32);
        if (c > 0.0 && (best < 0 || c < low)) {
            best = i;
            low = c;
        }
    }
    if (cost) *cost = low;
    return best;
}
using tb::from_left;
using tb::from_right;
using tb::fmean;
using tb::fold;

template <typename R>
struct TBArgs {
    const R* v;
    const R* G;
    const R* Lam;
    const R* rC;
    R* out;
    const double* lam;       // accumulator row of lambda_max (NULL: use tb)
    const double* Tit;       // previous iterate: accumulate the pass reductions (last launch, FP64)
    PassSlots ps;
    R* stages;               // non-NULL: the result of stage s < K-1 also goes to stages + (s+1)*sstride
    int64_t sstride;
    // FP32 correction form: with g64 != NULL the launch's last stage is the
    // final one, evaluated in double from g64 + w with rC64, into out64
    const double* g64;
    const double* rC64;
    double* out64;
    double g64w[2];          // face weights in double for that stage
    // Launch with the final stage: with lam_next != NULL also the next
    // Picard pass's conductivities (Lam_next) and Gershgorin bound (max into
    // the row lam_next) from the new iterate; the output ring is then one
    // cell narrower (halo H = K + 1) so that the new iterate is known on the
    // neighbours of every output cell.
    double* lam_next;
    const double* alpha2;
    double* Lam_next;        // FP64
    float* Lam32_next;       // FP32 correction form: float conductivities and
    float* q32_next;         // the correction source -tau rC' D' g of the next pass
    // partial densities (rho = m1 + m2 of the Spitzer-Harm law, and the
    // relaxation); next_step: the next step's relaxation and first
    // coefficients instead of the next pass's (relaxed T and alpha2 to
    // Tn_next/a2_next; 1/C is unchanged with equal p_inf)
    const double* m1;
    const double* m2;
    int next_step;
    double* Tn_next;
    double* a2_next;
    double eps;
    DevPhases ph;
    int nx, ny, perx, pery;
    R wx, wy, tau;
    R fx, fy;  // wx, wy, halved for arithmetic face means
    int K, H, hx, tiles_x, ox, oy;
    int vzero;  // float stages: v is the all-zero start w0 = 0 (not read)
    double taud;
    double tb[KMAX_TB], chat[KMAX_TB];
};

// kSH: the conductivities built in the epilogue follow the Spitzer-Harm law
// in some phase (its logarithms would otherwise take registers from the
// power-law kernels).  C: cells per lane along x (1: 64-wide tiles of 8, 4 or 2
// rows per wave; 2: 128-wide tiles of 4 rows per wave, lane l owning cells 2l and
// 2l + 1, so that one of each cell's x-neighbours is in the lane itself).
template <typename R, int NW, int RW, int C, bool kKeep, bool kSH, bool kHarm>
__global__ void __launch_bounds__(64 * NW, 4) k_tb2d(TBArgs<R> a) {
    constexpr int WAVES = NW;
    constexpr int EXT_X = 64 * C;
    constexpr int EXT_Y = NW * RW;
    __shared__ R sh_lo[2][WAVES][C][64];  // row 0 of each wave (the "up" row of the wave below)
    __shared__ R sh_hi[2][WAVES][C][64];  // row RW-1 of each wave (the "down" row of the wave above)
    constexpr int face = kHarm ? 1 : 0;
    const int lane = threadIdx.x & 63;
    // the wave's number in a scalar register: rows, their addresses and their
    // wall tests are then scalar work
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Lambda of a cell in the epilogues (rho = m1 + m2 used only under the
    // Spitzer-Harm law)
    auto law = [&](double t, double a2, double m1, double m2) -> double {
        if constexpr (kSH) return phys::cell_conductivity(a.ph, t, a2, m1 + m2);
        else return phys::cell_conductivity_pow(a.ph, t, a2);
    };
    // x-neighbours of cell j of this lane, from the lane's own cells or the
    // adjacent lanes (j is a compile-time index in the unrolled loops)
    auto left_of = [&](const auto (&x)[C], int j) { return j > 0 ? x[j - 1] : from_left(x[C - 1]); };
    auto right_of = [&](const auto (&x)[C], int j) { return j < C - 1 ? x[j + 1] : from_right(x[0]); };
    const int K = a.K, H = a.H;
    // the x ring: H, or with two cells per lane H rounded up to even, so that
    // the tile starts at an even column and a lane's two cells are adjacent
    // in memory (periodic x with an even width, or clamped walls)
    const int HX = a.hx;
    // tiles in XCD order: x-neighbours, whose extended tiles overlap by 2H
    // columns, mostly share an L2
    const int tile = tb::xcd_block();
    const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
    const int yg0 = ty * a.oy - H + wv * RW;
    int xg[C], xi[C];
    bool fL[C], fR[C];
    // output column: cell j of this lane is at least HX in from the tile's x edges
    bool xo[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int xl = C * lane + j;
        xg[j] = tx * a.ox - HX + xl;
        xi[j] = tb::fold_tile(xg[j], a.nx, a.perx);
        const bool inx = xg[j] >= 0 && xg[j] < a.nx;
        fL[j] = a.perx ? a.nx > 1 : (inx && xg[j] > 0);
        fR[j] = a.perx ? a.nx > 1 : (inx && xg[j] < a.nx - 1);
        xo[j] = xl >= HX && xl < EXT_X - HX && xg[j] < a.nx;
    }
    // Two cells per lane come in one load of two words at column sx: the
    // pair (xi0, xi0 + 1) away from the walls, the clamped copies (both the
    // wall cell) beyond them; sel_j tells which word is cell j.
    const unsigned sx = (unsigned)(C == 2 ? min(xi[0], a.nx - 2) : xi[0]);
    bool sel[C];
#pragma unroll
    for (int j = 0; j < C; ++j) sel[j] = xi[j] == (int)sx;
    // first word of each row in a field (scalar: every field's load of the
    // row takes it as its base, with the lane's column as the offset)
    int yr[RW];
    const int yi0 = fold(yg0, a.ny, a.pery);
#pragma unroll
    for (int r = 0; r < RW; ++r) yr[r] = row_index(yi0, yg0, r, a.ny, a.pery);
    auto row = [&](auto* f, int r) { return f + (int64_t)yr[r] * a.nx; };
    auto ld = [&](const auto* f, int r, auto (&out)[C]) {
        if constexpr (C == 1) {
            out[0] = row(f, r)[sx];
        } else {
            using T = std::remove_cv_t<std::remove_reference_t<decltype(f[0])>>;
            struct alignas(sizeof(T)) Pair { T x, y; } pr;
            __builtin_memcpy(&pr, row(f, r) + sx, sizeof(Pair));
#pragma unroll
            for (int j = 0; j < C; ++j) out[j] = sel[j] ? pr.x : pr.y;
        }
    };
    // this lane's output cells of row r (C = 2: both in one store; the second
    // is past the grid only at the right end of an odd width)
    auto put = [&](auto* f, int r, const auto (&x)[C]) {
        if constexpr (C == 1) {
            if (xo[0]) row(f, r)[(unsigned)xg[0]] = x[0];
        } else {
            using T = std::remove_reference_t<decltype(f[0])>;
            struct alignas(sizeof(T)) Pair { T x, y; } pr{x[0], x[1]};
            if (xo[1]) __builtin_memcpy(row(f, r) + (unsigned)xg[0], &pr, sizeof(Pair));
            else if (xo[0]) row(f, r)[(unsigned)xg[0]] = x[0];
        }
    };
    // wave-uniform: the face between rows y and y + 1 exists (the grids blocked
    // here have more than one row)
    const int ylo = a.pery ? -(1 << 30) : 0, yhi = a.pery ? 1 << 30 : a.ny - 1;
    auto face_above = [&](int y) { return (int)(y >= ylo) & (int)(y < yhi); };
    auto yout = [&](int r) { const int row = wv * RW + r; return row >= H && row < EXT_Y - H && yg0 + r < a.ny; };
    // Output rows and the rows next to them: the others need no conductivity of
    // the next pass.  With Spitzer-Harm laws its evaluation is half of a
    // launch's time (517 x 301: 13 of 24 us), so rows that need none skip it,
    // and with them whole waves (4 of 16 at H = 9 on 64 rows, one per SIMD:
    // 22.5 us); under the power law the tests cost what they save.
    auto near_out = [&](int r) {
        const int row = wv * RW + r;
        return !kSH || (row >= H - 1 && row <= EXT_Y - H && yg0 + r <= a.ny);
    };
    const bool near_wave = !kSH || (wv * RW + RW >= H && wv * RW <= EXT_Y - H && yg0 <= a.ny);

    constexpr bool kFloat = sizeof(R) == 4;
    const bool fin = kFloat && a.g64 != nullptr;
    // A float pass's first launch starts from w0 = 0, where its first stage
    // gives c_0 G exactly: v is then not read, and that stage is c_0 G.
    const bool vz = kFloat && !kKeep && a.vzero && a.v != a.G && (fin ? K - 1 : K) >= 1;
    // In double the source G lives in LDS (read once per cell and stage):
    // with 8 cells per lane the four kappa and v already take 80 of the 128
    // VGPRs that four waves per SIMD leave, and G in registers spills.
    constexpr bool kGinLds = !kFloat && RW * C == 8;
    __shared__ R sG[kGinLds ? EXT_Y : 1][C][64];
    R v[RW][C], G[RW][C], kL[RW][C], kR[RW][C], kD[RW][C], kU[RW][C];
    const bool same = a.v == a.G;
    R Lk[RW][C];     // cell conductivities, kept for a fused FP64 final stage
    R Ldk[C], Luk[C];
    double lamr[kSlots / 64] = {};  // lambda_G of the pass: its accumulator row (every wave folds it)
    {
        // Every row's words are in flight before the first is used.  Waiting
        // row by row (as the compiler does when the first use of a row's word
        // comes before the next row's loads) costs one memory round trip per
        // row: the load phase of a 64 x 128 tile took 11 us that way.
        R L[RW][C], t[RW][C];
        if (a.lam) {
#pragma unroll
            for (int k = 0; k < kSlots / 64; ++k) lamr[k] = a.lam[lane + 64 * k];
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            ld(a.Lam, r, L[r]);
            ld(a.rC, r, t[r]);
            ld(a.G, r, G[r]);
        }
        // the first launch of a pass starts from v^(0) = T^n = g
        if (!same && !vz) {
#pragma unroll
            for (int r = 0; r < RW; ++r) ld(a.v, r, v[r]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            sh_lo[0][wv][j][lane] = L[0][j];
            sh_hi[0][wv][j][lane] = L[RW - 1][j];
        }
        if constexpr (kGinLds) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) sG[wv * RW + r][j][lane] = G[r][j];
        }
        __syncthreads();
        R Ldn[C], Lup[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            Ldn[j] = wv > 0 ? sh_hi[0][wv > 0 ? wv - 1 : 0][j][lane] : L[0][j];
            Lup[j] = wv < WAVES - 1 ? sh_lo[0][wv < WAVES - 1 ? wv + 1 : wv][j][lane] : L[RW - 1][j];
        }
        // arithmetic means: the sum of a face's two cells is formed once (its
        // half goes into the weight, which is exact)
        auto mean = [&](R x, R y) { return kHarm ? fmean<R>(x, y, 1) : x + y; };
        R Mdn[C];
#pragma unroll
        for (int j = 0; j < C; ++j) Mdn[j] = mean(L[0][j], Ldn[j]);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const R wD = face_above(yg0 + r - 1) ? a.fy : R(0), wU = face_above(yg0 + r) ? a.fy : R(0);
            R Mrt[C];
#pragma unroll
            for (int j = 0; j < C; ++j) Mrt[j] = mean(L[r][j], right_of(L[r], j));
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const R tr = a.tau * t[r][j];
                const R Mup = mean(L[r][j], r < RW - 1 ? L[r < RW - 1 ? r + 1 : r][j] : Lup[j]);
                const R Mlf = left_of(Mrt, j);  // (every lane takes part)
                kL[r][j] = tr * (fL[j] ? a.fx : R(0)) * Mlf;
                kR[r][j] = tr * (fR[j] ? a.fx : R(0)) * Mrt[j];
                kD[r][j] = tr * wD * Mdn[j];
                kU[r][j] = tr * wU * Mup;
                Mdn[j] = Mup;
            }
            // (row by row: interleaved over all rows, this spills)
            __builtin_amdgcn_sched_barrier(0);
        }
        if (same || vz) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    if constexpr (kGinLds) v[r][j] = sG[wv * RW + r][j][lane];
                    else v[r][j] = vz ? R(0) : G[r][j];
                }
        }
        if constexpr (kFloat) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) Lk[r][j] = L[r][j];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                Ldk[j] = Ldn[j];
                Luk[j] = Lup[j];
            }
        }
    }
    double lamv = 0.0;
    if (a.lam) {
#pragma unroll
        for (int k = 0; k < kSlots / 64; ++k) lamv = fmax(lamv, lamr[k]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lamv = fmax(lamv, __shfl_xor(lamv, o, 64));
    }
    // Stage parameters: lane s holds tau*b_s and c_s = 1/(1 + tau*b_s) of
    // stage s; the stage loop reads them with readlane.
    double ptb = 0.0, pcm = 1.0;
    if (lane < K) {
        ptb = a.lam ? a.taud * lamv * a.chat[lane] : a.tb[lane];
        pcm = 1.0 / (1.0 + ptb);
    }
    // In double the stages before the launch's last run on V^(s) = Q_s v^(s),
    // Q_s = prod_{k<s} (1 + tau b_k):
    //   V^(s+1) = Q_s G + tau b_s V^(s) - sum_f kappa_f (V_a - V_f)^(s),
    // one product per cell and stage less than with the factor c_s.  Lane s
    // holds Q_s and 1/Q_(s+1).  The last stage takes the scale off the
    // differences, not off the result,
    //   v^(K) = c (G + (tau b V - sum_f kappa_f (V_a - V_f)) / Q),
    // so that the final one (b = 0) is G minus differences as in every other
    // kernel.  G Q / Q left all cells off by one factor (up to 1e-16 per step,
    // which nothing wears off: 6e-16 of T after 5 steps at 768^2, and a gradient
    // through them 6.0e-15 from 64-bit arithmetic instead of 3.1e-15), and
    // a uniform T was no equilibrium.
    double pQ = 1.0, piQ = 1.0;
    if constexpr (!kFloat) {
        double hi = 1.0 + ptb;  // inclusive product over the lanes up to this one
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const double up = __shfl_up(hi, o, 64);
            if (lane >= o) hi *= up;
        }
        const double below = __shfl_up(hi, 1, 64);
        pQ = lane == 0 ? 1.0 : below;
        piQ = 1.0 / hi;
    }
    // Stage s exchanges the seam rows through LDS buffer (s+1)&1; buffer 0
    // held the Lambda seams, whose reads all precede the first barrier below.
    // The end waves read a row of their own: their outer rows go stale anyway.
    const int Kin = fin ? K - 1 : K;
    const int wdn = wv > 0 ? wv - 1 : 0, wup = wv < WAVES - 1 ? wv + 1 : wv;
    // from w0 = 0 the first stage is c_0 G (the same number the stage below
    // gives with every difference zero)
    int s0 = 0;
    if (vz) {
        const R cm0 = (R)lane_value(pcm, 0);
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int j = 0; j < C; ++j) v[r][j] = cm0 * G[r][j];
        s0 = 1;
    }
    auto stage = [&](int s, auto scale) {  // scale: the last stage of a double launch
        constexpr bool kScale = decltype(scale)::value;
        // the first stage run writes buffer 1 (buffer 0 held the Lambda seams)
        const int buf = (s - s0 + 1) & 1;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            sh_lo[buf][wv][j][lane] = v[0][j];
            sh_hi[buf][wv][j][lane] = v[RW - 1][j];
        }
        __syncthreads();
        R vup[C], vdn[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            vdn[j] = sh_hi[buf][wdn][j][lane];
            vup[j] = sh_lo[buf][wup][j][lane];
        }
        const double tbd = lane_value(ptb, s);
        const R cm = (R)lane_value(kFloat || kScale ? pcm : pQ, s), tb = (R)tbd;
        const R iQ = kScale && s > 0 ? (R)lane_value(piQ, s > 0 ? s - 1 : 0) : R(1);
        // Each face difference is formed once and shared by the face's two
        // cells: c - c_left is minus the left neighbour's c - c_right, and
        // c - c_below minus the row below's c - c_above (exact in floating
        // point, so S is the same number as with four differences per cell).
        // The rows run from the second one up and the first one comes last,
        // so the seam rows are on their way from LDS meanwhile.
        R d0[C], ddn[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            d0[j] = v[0][j] - v[1][j];
            ddn[j] = -d0[j];
        }
#pragma unroll
        for (int q = 1; q <= RW; ++q) {
            const int r = q == RW ? 0 : q;
            R drt[C];
#pragma unroll
            for (int j = 0; j < C; ++j) drt[j] = v[r][j] - right_of(v[r], j);
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const R c = v[r][j];
                const R dlf = -left_of(drt, j);
                const R dup = r == 0 ? d0[j] : c - (r < RW - 1 ? v[r < RW - 1 ? r + 1 : r][j] : vup[j]);
                const R dd = r == 0 ? c - vdn[j] : ddn[j];
                const R S = kL[r][j] * dlf + kR[r][j] * drt[j] + kD[r][j] * dd + kU[r][j] * dup;
                R Gr;
                if constexpr (kGinLds) Gr = sG[wv * RW + r][j][lane];
                else Gr = G[r][j];
                if constexpr (kFloat) v[r][j] = cm * (Gr + tb * c - S);
                else if constexpr (kScale) v[r][j] = cm * fma(tb * c - S, iQ, Gr);
                else v[r][j] = cm * Gr + (tb * c - S);
                ddn[j] = -dup;
            }
        }
        // the output cells are exact after every stage: keep the intermediate
        // stages when asked (the adjoint's recomputation; without the test of
        // the pointer, and with the rows' stores interleaved, this spills)
        if (kKeep && !kScale && a.stages != nullptr) {
            const R iq = (R)lane_value(piQ, s);
            R* dst = a.stages + (int64_t)(s + 1) * a.sstride;
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                R x[C];
#pragma unroll
                for (int j = 0; j < C; ++j) x[j] = v[r][j] * iq;
                if (yout(r)) put(dst, r, x);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    for (int s = s0; s < (kFloat ? Kin : K - 1); ++s) stage(s, std::false_type{});
    if constexpr (!kFloat) stage(K - 1, std::true_type{});
    // Final stage (b = 0) of the FP32 correction form, in double on v = g + w:
    // T = g - tau rC64 sum_f w_f mean(Lambda'_a, Lambda'_b) (v_a - v_b), with
    // Lambda' the float conductivities, into Tfin (every cell of the tile:
    // exact K - 1 in from the edge); gfin holds g, rcfin rC64.
    double Tfin[RW][C], gfin[RW][C], rcfin[RW][C];
    if constexpr (kFloat) {
        if (fin) {
            __shared__ double dsh_lo[WAVES][C][64], dsh_hi[WAVES][C][64];
            double vf[RW][C];
#pragma unroll
            for (int r = 0; r < RW; ++r) ld(a.g64, r, gfin[r]);
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) vf[r][j] = gfin[r][j] + (double)v[r][j];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                dsh_lo[wv][j][lane] = vf[0][j];
                dsh_hi[wv][j][lane] = vf[RW - 1][j];
            }
            __syncthreads();
            double vup[C], prev[C];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                prev[j] = wv > 0 ? dsh_hi[wv - 1][j][lane] : vf[0][j];
                vup[j] = wv < WAVES - 1 ? dsh_lo[wv + 1][j][lane] : vf[RW - 1][j];
            }
            const double wxd = a.g64w[0], wyd = a.g64w[1];
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const int y = yg0 + r;
                const bool iny = y >= 0 && y < a.ny;
                const bool fD = a.pery ? a.ny > 1 : (iny && y > 0);
                const bool fU = a.pery ? a.ny > 1 : (iny && y < a.ny - 1);
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    const double c = vf[r][j];
                    const double up = r < RW - 1 ? vf[r + 1][j] : vup[j];
                    const double La = (double)Lk[r][j];
                    const double Ll = (double)left_of(Lk[r], j), Lr = (double)right_of(Lk[r], j);
                    const double Ld = (double)(r > 0 ? Lk[r - 1][j] : Ldk[j]);
                    const double Lu = (double)(r < RW - 1 ? Lk[r + 1][j] : Luk[j]);
                    const double lf = left_of(vf[r], j), rt = right_of(vf[r], j);
                    double S = 0.0;
                    if (fL[j]) S += wxd * fmean<double>(La, Ll, face) * (c - lf);
                    if (fR[j]) S += wxd * fmean<double>(La, Lr, face) * (c - rt);
                    if (fD) S += wyd * fmean<double>(La, Ld, face) * (c - prev[j]);
                    if (fU) S += wyd * fmean<double>(La, Lu, face) * (c - up);
                    prev[j] = c;
                    Tfin[r][j] = S;
                }
            }
#pragma unroll
            for (int r = 0; r < RW; ++r) ld(a.rC64, r, rcfin[r]);
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) Tfin[r][j] = gfin[r][j] - a.taud * rcfin[r][j] * Tfin[r][j];
            if (a.lam_next) {
                // Coefficients of the next Picard pass at the new iterate T
                // (valid K cells in from the edge; g = T^n): the conductivity
                // in double for the bound, its float rounding and the source
                // q = -tau rC' D' g from the float-rounded Lambda' and rC', at
                // the output cells (K+1 in), faces in the order -x, +x, -y, +y.
                double Ln[RW][C], a2v[RW][C], m1v[RW][C], m2v[RW][C];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    ld(a.alpha2, r, a2v[r]);
                    if constexpr (kSH) {
                        ld(a.m1, r, m1v[r]);
                        ld(a.m2, r, m2v[r]);
                    } else {
#pragma unroll
                        for (int j = 0; j < C; ++j) m1v[r][j] = m2v[r][j] = 0.0;
                    }
                }
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const double tn = Tfin[r][j];
                        if constexpr (kSH) Ln[r][j] = near_out(r) ? law(tn, a2v[r][j], m1v[r][j], m2v[r][j]) : 0.0;
                        else Ln[r][j] = law(tn, a2v[r][j], m1v[r][j], m2v[r][j]);
                    }
                __shared__ double esh[4][WAVES][C][64];  // seams of Lambda and g
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    esh[0][wv][j][lane] = Ln[0][j];
                    esh[1][wv][j][lane] = Ln[RW - 1][j];
                    esh[2][wv][j][lane] = gfin[0][j];
                    esh[3][wv][j][lane] = gfin[RW - 1][j];
                }
                __syncthreads();
                double Ldn[C], Lup[C], gdn[C], gup[C];
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    Ldn[j] = wv > 0 ? esh[1][wv - 1][j][lane] : Ln[0][j];
                    Lup[j] = wv < WAVES - 1 ? esh[0][wv + 1][j][lane] : Ln[RW - 1][j];
                    gdn[j] = wv > 0 ? esh[3][wv - 1][j][lane] : gfin[0][j];
                    gup[j] = wv < WAVES - 1 ? esh[2][wv + 1][j][lane] : gfin[RW - 1][j];
                }
                double bound = 0.0;
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    float Lf[C];
#pragma unroll
                    for (int j = 0; j < C; ++j) Lf[j] = (float)Ln[r][j];
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const double L = Ln[r][j];
                        const double Ll = left_of(Ln[r], j), Lr = right_of(Ln[r], j);
                        const float Llf = left_of(Lf, j), Lrf = right_of(Lf, j);
                        const double gl = left_of(gfin[r], j), gr = right_of(gfin[r], j);
                        const double Ld = r > 0 ? Ln[r - 1][j] : Ldn[j], Lu = r < RW - 1 ? Ln[r + 1][j] : Lup[j];
                        const double gd = r > 0 ? gfin[r - 1][j] : gdn[j], gu = r < RW - 1 ? gfin[r + 1][j] : gup[j];
                        const int y = yg0 + r;
                        if (xo[j] && yout(r)) {
                            const bool fD = a.pery ? a.ny > 1 : y > 0;
                            const bool fU = a.pery ? a.ny > 1 : y < a.ny - 1;
                            const int64_t o = (int64_t)y * a.nx + xg[j];
                            double d = 0.0;
                            if (fL[j]) d += wxd * fmean<double>(L, Ll, face);
                            if (fR[j]) d += wxd * fmean<double>(L, Lr, face);
                            if (fD) d += wyd * fmean<double>(L, Ld, face);
                            if (fU) d += wyd * fmean<double>(L, Lu, face);
                            bound = fmax(bound, 2.0 * d * rcfin[r][j]);
                            const double La = (double)Lf[j], rf = (double)(float)rcfin[r][j], ga = gfin[r][j];
                            double Sq = 0.0;
                            if (fL[j]) Sq += wxd * fmean<double>(La, (double)Llf, face) * (ga - gl);
                            if (fR[j]) Sq += wxd * fmean<double>(La, (double)Lrf, face) * (ga - gr);
                            if (fD) Sq += wyd * fmean<double>(La, (double)(float)Ld, face) * (ga - gd);
                            if (fU) Sq += wyd * fmean<double>(La, (double)(float)Lu, face) * (ga - gu);
                            a.Lam32_next[o] = Lf[j];
                            a.q32_next[o] = (float)(-a.taud * rf * Sq);
                        }
                    }
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, __shfl_xor(bound, o, 64));
                if (lane == 0) {
                    const int sl = (int)(((int64_t)blockIdx.x * WAVES + wv) % kSlots);
                    atomicMax((unsigned long long*)(a.lam_next + sl),
                              (unsigned long long)__double_as_longlong(bound + 0.0));
                }
            }
        }
    }
    double dmax = 0.0, tmax = 0.0, bad = 0.0;
    // the first pass's previous iterate is T^n = g, already on chip
    const bool tit_is_g = kFloat ? (fin && a.Tit == a.g64) : (const void*)a.Tit == (const void*)a.G;
    // Words of the epilogue are read for every row before the first is used.
    // Output cells: rows yo (scalar), columns xo; lanes beyond them read the
    // row's first word and discard it.
    bool yo[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) yo[r] = yout(r);
    unsigned xs[C];
#pragma unroll
    for (int j = 0; j < C; ++j) xs[j] = xo[j] ? (unsigned)xg[j] : 0u;
    if (a.Tit) {
        if (a.ps.dmax) {  // the Picard change only where asked for
            double titv[RW][C];
            if (!tit_is_g) {
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int j = 0; j < C; ++j) titv[r][j] = row(a.Tit, r)[xs[j]];
            } else {
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        if constexpr (kFloat) titv[r][j] = gfin[r][j];
                        else if constexpr (kGinLds) titv[r][j] = (double)sG[wv * RW + r][j][lane];
                        else titv[r][j] = (double)G[r][j];
                    }
            }
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    const double tn = fin ? Tfin[r][j] : (double)v[r][j];
                    dmax = fmax(dmax, yo[r] && xo[j] ? fabs(tn - titv[r][j]) : 0.0);
                }
        }
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const double tn = fin ? Tfin[r][j] : (double)v[r][j];
                const bool o = yo[r] && xo[j];
                tmax = fmax(tmax, o ? fabs(tn) : 0.0);
                bad += o && (!(tn > 0.0) || isinf(tn)) ? 1.0 : 0.0;
            }
    }
    if (fin) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (yo[r]) put(a.out64, r, Tfin[r]);
    } else {
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (yo[r]) put(a.out, r, v[r]);
    }
    if (a.Tit) {
        // wave-level fold, then lane 0 of every wave adds to a slot of the rows
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
    if constexpr (!kFloat) {
        if (a.lam_next) {
            // Coefficients of the next Picard pass at the new iterate v (valid
            // K cells in from the edge): Lambda = sum_k alpha_k lambda_k(v),
            // and at the output cells (K+1 in) the bound 2 rC sum_f w_f
            // mean(Lambda_a, Lambda_b), faces in the order -x, +x, -y, +y.
            // With next_step the next step's instead: every cell relaxed from
            // (alpha2, v, v, m1, m2) first, Lambda at the relaxed state.
            const bool next_step = a.next_step != 0;
            // The partial densities enter only the relaxation of interface
            // cells (pure cells keep their T and alpha2) and the Spitzer-Harm
            // law; 1/C, which they also fix, is the step's own (equal p_inf),
            // so under the power law they are read in interface cells only
            // (the other lanes read the row's first word).
            double Ln[RW][C], a2v[RW][C], m1v[RW][C], m2v[RW][C];
            if constexpr (kSH) {
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int j = 0; j < C; ++j) Ln[r][j] = a2v[r][j] = 0.0;
            }
            if (near_wave) {
#pragma unroll
                for (int r = 0; r < RW; ++r) ld(a.alpha2, r, a2v[r]);
                if constexpr (kSH) {
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        ld(a.m1, r, m1v[r]);
                        ld(a.m2, r, m2v[r]);
                    }
                } else if (next_step) {
#pragma unroll
                    for (int r = 0; r < RW; ++r)
#pragma unroll
                        for (int j = 0; j < C; ++j) {
                            const bool mx = phys::is_mixed(a2v[r][j], a.eps);
                            const unsigned xm = mx ? sx + (sel[j] ? 0u : 1u) : 0u;
                            m1v[r][j] = row(a.m1, r)[xm];
                            m2v[r][j] = row(a.m2, r)[xm];
                        }
                }
                if (next_step) {
#pragma unroll
                    for (int r = 0; r < RW; ++r)
#pragma unroll
                        for (int j = 0; j < C; ++j)
                            if (phys::is_mixed(a2v[r][j], a.eps))
                                phys::relax_equal_pinf(a.ph, v[r][j], m1v[r][j], m2v[r][j], v[r][j], a2v[r][j]);
                }
                if constexpr (kSH) {
#pragma unroll
                    for (int r = 0; r < RW; ++r)
#pragma unroll
                        for (int j = 0; j < C; ++j)
                            if (near_out(r)) Ln[r][j] = law(v[r][j], a2v[r][j], m1v[r][j], m2v[r][j]);
                } else {
                    phys::lambda_rows(a.ph, v, a2v, Ln);
                }
            }
            // the seam buffer not used by the last stage: its reads all
            // precede that stage's barrier
            const int b2 = (K + 1) & 1;
#pragma unroll
            for (int j = 0; j < C; ++j) {
                sh_lo[b2][wv][j][lane] = Ln[0][j];
                sh_hi[b2][wv][j][lane] = Ln[RW - 1][j];
            }
            double rcv[RW][C];
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int j = 0; j < C; ++j) rcv[r][j] = row(a.rC, r)[xs[j]];
            __syncthreads();
            double Ldn[C], Lup[C];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                Ldn[j] = wv > 0 ? sh_hi[b2][wv > 0 ? wv - 1 : 0][j][lane] : Ln[0][j];
                Lup[j] = wv < WAVES - 1 ? sh_lo[b2][wv < WAVES - 1 ? wv + 1 : wv][j][lane] : Ln[RW - 1][j];
            }
            double bound = 0.0;
            if (near_wave) {
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const double Ll = left_of(Ln[r], j), Lr = right_of(Ln[r], j);
                        const double Ld = r > 0 ? Ln[r - 1][j] : Ldn[j];
                        const double Lu = r < RW - 1 ? Ln[r + 1][j] : Lup[j];
                        const int y = yg0 + r;
                        const bool fD = a.pery ? a.ny > 1 : y > 0;
                        const bool fU = a.pery ? a.ny > 1 : y < a.ny - 1;
                        double d = 0.0;
                        if (fL[j]) d += a.wx * fmean<double>(Ln[r][j], Ll, face);
                        if (fR[j]) d += a.wx * fmean<double>(Ln[r][j], Lr, face);
                        if (fD) d += a.wy * fmean<double>(Ln[r][j], Ld, face);
                        if (fU) d += a.wy * fmean<double>(Ln[r][j], Lu, face);
                        bound = fmax(bound, yo[r] && xo[j] ? 2.0 * d * rcv[r][j] : 0.0);
                    }
            }
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (yo[r]) {
                    put(a.Lam_next, r, Ln[r]);
                    if (next_step) {
                        put(a.Tn_next, r, v[r]);
                        put(a.a2_next, r, a2v[r]);
                    }
                }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, __shfl_xor(bound, o, 64));
            if (lane == 0) {
                const int sl = (int)(((int64_t)blockIdx.x * WAVES + wv) % kSlots);
                atomicMax((unsigned long long*)(a.lam_next + sl), (unsigned long long)__double_as_longlong(bound + 0.0));
            }
        }
    }
}

template <typename R>
int launch_tb2d(hipStream_t s, const DevGrid& g, int face, const R* v, const R* G, const R* Lam, const R* rC,
                R* out, Stages st, int count, double tau, const double* Tit, PassSlots ps, R* stages = nullptr,
                int64_t sstride = 0, const double* g64 = nullptr, const double* rC64 = nullptr,
                double* out64 = nullptr, const NextCoef* nc = nullptr, int vzero = 0) {
    TBArgs<R> a{};
    a.vzero = vzero;
    if (nc) {
        a.lam_next = nc->lam;
        a.alpha2 = nc->alpha2;
        a.Lam_next = nc->Lam;
        a.Lam32_next = nc->Lam32;
        a.q32_next = nc->q32;
        a.ph = nc->ph;
        a.m1 = nc->m1;
        a.m2 = nc->m2;
        a.next_step = nc->next_step;
        a.Tn_next = nc->Tn;
        a.a2_next = nc->a2;
        a.eps = nc->eps;
    }
    a.g64 = g64;
    a.rC64 = rC64;
    a.out64 = out64;
    a.g64w[0] = g.w[0];
    a.g64w[1] = g.w[1];
    a.stages = stages;
    a.sstride = sstride;
    const int K = count < KMAX_TB ? count : KMAX_TB;
    const int shape = best_shape(g, K, nc ? K + 1 : K, sizeof(R) == 4);
    const Shape& t = kShapeTab[shape];
    a.v = v;
    a.G = G;
    a.Lam = Lam;
    a.rC = rC;
    a.out = out;
    a.lam = st.lam;
    a.Tit = Tit;
    a.ps = ps;
    a.nx = g.nx;
    a.ny = g.ny;
    a.perx = g.per[0];
    a.pery = g.per[1];
    a.wx = (R)g.w[0];
    a.wy = (R)g.w[1];
    a.fx = (R)(face == 1 ? g.w[0] : 0.5 * g.w[0]);
    a.fy = (R)(face == 1 ? g.w[1] : 0.5 * g.w[1]);
    a.tau = (R)tau;
    a.taud = tau;
    a.K = K;
    a.H = nc ? K + 1 : K;
    a.hx = t.c == 2 ? (a.H + 1) & ~1 : a.H;
    a.ox = t.ext_x() - 2 * a.hx;
    a.oy = t.ext_y() - 2 * a.H;
    a.tiles_x = (g.nx + a.ox - 1) / a.ox;
    int tiles_y = (g.ny + a.oy - 1) / a.oy;
    for (int k = 0; k < K; ++k) {
        if (st.lam) a.chat[k] = st.chat[k];
        else a.tb[k] = st.tb[k];
    }
    const dim3 grid((unsigned)(a.tiles_x * tiles_y));
    const bool sh = nc && nc->ph.spitzer;
    auto go = [&](auto harm, auto keep, auto spitzer) {
        constexpr bool kHarm = decltype(harm)::value, kKeep = decltype(keep)::value, kSH = decltype(spitzer)::value;
        auto run = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(64 * NWAVES), 0, s, a); };
        switch (shape) {
            case S_WIDE: run(k_tb2d<R, NWAVES, 4, 2, kKeep, kSH, kHarm>); break;
            case S_TALL: run(k_tb2d<R, NWAVES, 8, 1, kKeep, kSH, kHarm>); break;
            case S_SQUARE: run(k_tb2d<R, NWAVES, 4, 1, kKeep, kSH, kHarm>); break;
            default: run(k_tb2d<R, NWAVES, 2, 1, kKeep, kSH, kHarm>); break;
        }
    };
    auto laws = [&](auto harm) {
        if constexpr (sizeof(R) == 8) {  // kept stages (the adjoint's recompute): FP64, no epilogue
            if (stages) return go(harm, std::true_type{}, std::false_type{});
        }
        if (sh) go(harm, std::false_type{}, std::true_type{});
        else go(harm, std::false_type{}, std::false_type{});
    };
    if (face == 1) laws(std::true_type{});
    else laws(std::false_type{});
    return K;
}

bool use_tb2d(const DevGrid& g, int count) {
    return g.nz == 1 && g.ny >= 32 && count >= 2;
}

StageParam one_stage(const Stages& st) {
    StageParam sp;
    sp.lam = st.lam;
    sp.tb = st.lam ? 0.0 : st.tb[0];
    sp.chat = st.lam ? st.chat[0] : 0.0;
    return sp;
}

}  // namespace

int launch_sweeps64_keep(hipStream_t s, const DevGrid& g, int face, const double* v, const double* rhs,
                         const double* Lam, const double* rC, double* out, Stages st, int count, double tau,
                         double* stages, int64_t sstride) {
    if (use_tb2d(g, count))
        return launch_tb2d<double>(s, g, face, v, rhs, Lam, rC, out, st, count, tau, nullptr, PassSlots{}, stages,
                                   sstride);
    const int k = b3d_stages(g, face, count, false);
    if (k > 1) {
        launch_b3d<double>(s, g, face, v, rhs, Lam, rC, out, st, k, tau, nullptr, PassSlots{},
                           StageParam{nullptr, 0.0, 0.0}, true, stages, sstride);
        return k;
    }
    return -1;
}

bool final32_apart(const DevGrid& g) { return use_z3d(g) || use_line(g); }

int sweeps_per_launch(const DevGrid& g, int face, int count, bool f32) {
    if (use_line(g)) return line_stages(count);
    if (!use_tb2d(g, count)) return b3d_stages(g, face, count, f32);
    // equal launches (a launch of K stages recomputes a ring of width K, so
    // even launches waste least), as many as cost least
    int best = 0;
    double low = 0.0;
    for (int n = (count + KMAX_TB - 1) / KMAX_TB; n <= count && (best == 0 || n <= best + 4); ++n) {
        const int k = (count + n - 1) / n;
        double cost;
        if (best_shape(g, k, k + 1, f32, &cost) < 0) continue;
        if (best == 0 || n * cost < low) {
            best = n;
            low = n * cost;
        }
    }
    return (count + best - 1) / best;
}

StagePlan stage_plan(const DevGrid& g, int face, int count, bool f32, bool coeffs) {
    const int k = sweeps_per_launch(g, face, count, f32);
    if (use_tb2d(g, k)) {
        const Shape& t = kShapeTab[best_shape(g, k, coeffs ? k + 1 : k, f32)];
        return StagePlan{PLAN_TILES, k, t.ext_x(), t.ext_y()};
    }
    if (use_line(g)) return StagePlan{PLAN_LINE, k, 256, 1};
    if (k > 1) return StagePlan{PLAN_BLOCKED_MARCH, k, 64, b3d_rows(face, k, f32)};
    if (use_z3d(g)) return StagePlan{PLAN_MARCH, 1, 64, z3d_rows(f32)};
    return StagePlan{PLAN_GENERAL, 1, 0, 0};
}

int reverse_plan(const DevGrid& g, int face) {
    if (use_adj_tb2d(g, face)) return PLAN_TILES;
    if (use_adj_b3d(g, face)) return PLAN_BLOCKED_MARCH;
    return use_adj_z3d(g, face) ? PLAN_MARCH : PLAN_GENERAL;
}

bool big_tiles2d(const DevGrid& g) {
    if (!use_tb2d(g, 8)) return false;
    const int shape = best_shape(g, 8, 9, false);
    return shape == S_WIDE || shape == S_TALL;
}

int launch_sweeps64(hipStream_t s, const DevGrid& g, int face, const double* v, const double* rhs,
                    const double* Lam, const double* rC, double* out, Stages st, int count, bool last, double tau,
                    const double* Tit, PassSlots ps, const NextCoef* nc, bool* nc_done) {
    if (nc_done) *nc_done = false;
    if (use_tb2d(g, count)) {
        const bool with_nc = last && nc != nullptr;
        if (nc_done) *nc_done = with_nc;
        return launch_tb2d<double>(s, g, face, v, rhs, Lam, rC, out, st, count, tau, last ? Tit : nullptr, ps,
                                   nullptr, 0, nullptr, nullptr, nullptr, with_nc ? nc : nullptr);
    }
    if (use_line(g)) {
        const int k = line_stages(count);
        launch_line<double>(s, g, face, v, rhs, Lam, rC, out, st, k, tau, last ? Tit : nullptr, ps);
        return k;
    }
    if (const int k = b3d_stages(g, face, count, false); k > 1) {
        launch_b3d<double>(s, g, face, v, rhs, Lam, rC, out, st, k, tau, last ? Tit : nullptr, ps);
        return k;
    }
    if (use_z3d(g)) {
        if (last) launch_z3d<double>(s, g, face, v, rhs, Lam, rC, out, StageParam{nullptr, 0.0, 0.0}, tau, Tit, ps);
        else launch_z3d<double>(s, g, face, v, rhs, Lam, rC, out, one_stage(st), tau, nullptr, PassSlots{});
        return 1;
    }
    if (last) {
        // the final stage, b = 0, in flux form
        launch_final64(s, g, face, v, rhs, Lam, rC, out, tau, Tit, ps);
    } else {
        launch_stage64(s, g, face, v, rhs, Lam, rC, out, one_stage(st), tau);
    }
    return 1;
}

int launch_sweeps32(hipStream_t s, const DevGrid& g, int face, const float* w, const float* qn,
                    const float* Lam32, const float* rC32, float* out, Stages st, int count, bool last, double tau,
                    const double* rhs, const double* rC, double* out64, const double* Tit, PassSlots ps,
                    const NextCoef* nc, bool* nc_done, bool w_zero) {
    if (nc_done) *nc_done = false;
    if (use_tb2d(g, count)) {
        if (last) {
            if (nc_done) *nc_done = nc != nullptr;
            return launch_tb2d<float>(s, g, face, w, qn, Lam32, rC32, nullptr, st, count, tau, Tit, ps, nullptr, 0,
                                      rhs, rC, out64, nc, w_zero ? 1 : 0);
        }
        return launch_tb2d<float>(s, g, face, w, qn, Lam32, rC32, out, st, count, tau, nullptr, PassSlots{}, nullptr,
                                  0, nullptr, nullptr, nullptr, nullptr, w_zero ? 1 : 0);
    }
    if (last) {
        if (use_z3d(g)) launch_z3d_final32(s, g, face, w, rhs, Lam32, rC, out64, tau, Tit, ps);
        else launch_final32(s, g, face, w, rhs, Lam32, rC, out64, tau, Tit, ps);
    } else if (use_line(g)) {
        const int k = line_stages(count);
        launch_line<float>(s, g, face, w, qn, Lam32, rC32, out, st, k, tau, nullptr, PassSlots{});
        return k;
    } else if (const int k = b3d_stages(g, face, count, true); k > 1) {
        launch_b3d<float>(s, g, face, w, qn, Lam32, rC32, out, st, k, tau, nullptr, PassSlots{});
        return k;
    } else if (use_z3d(g)) {
        launch_z3d<float>(s, g, face, w, qn, Lam32, rC32, out, one_stage(st), tau, nullptr, PassSlots{});
    } else {
        launch_stage32(s, g, face, w, qn, Lam32, rC32, out, one_stage(st), tau);
    }
    return 1;
}

}  // namespace tlim
