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
// What bounds it: a plane step's instructions and, on grids beyond the
// caches, memory.  At 512^3 in float a launch of 4 stages takes 780 us (195 us
// per stage; 549 us one stage per launch), at 256^3 108 us (27 against 77), and
// a launch of 3 at 512^3 moves 3.9 GB at 5.6 TB/s (64 x 48 cells read for 58 x 42
// results, in rows that do not start on a cache line).  In double a launch of
// 3 stages takes 31 us at 128^3 (10.5 us per stage against 22) and 27 us at
// 150 x 131 x 97 (9.1 against 28).  The registers of K stages set the rows per
// wave: 8 waves of two per SIMD, 256 VGPRs each; one row more spills (4 stages
// at 256^3: 108 -> 153 us).
//
// Arithmetic of a stage: with F_f = mean(Lambda_a, Lambda_b) (v_b - v_a) formed
// once per face and shared by its two cells,
//   out = c_m (G + tau b_m v + rC sum_d tau w_d (F_up - F_low)).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "tlim_device.h"
#include "tlim_sweep.h"

namespace tlim {

namespace {

using tb::fold;
using tb::from_left;
using tb::from_right;

constexpr int KMAX3 = 4;
constexpr int kWaves3 = 8;  // waves per workgroup
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

// A plane of a field as a buffer (wave-uniform: four scalar registers): its
// words are addressed by the lane's 32-bit byte offset alone, where a pointer
// takes a register pair and an addition per access.  Offsets past the plane
// read 0 and write nothing.
template <typename T>
struct Plane {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Plane(T* f, int64_t pz, int bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(
              const_cast<char*>(reinterpret_cast<const char*>(f) + pz), 0, bytes, 0x00027000)) {}
    __device__ __forceinline__ T get(unsigned o) const {
        if constexpr (sizeof(T) == 8) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
            return __builtin_bit_cast(std::remove_const_t<T>, x);
        } else {
            const auto x = __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
            return __builtin_bit_cast(std::remove_const_t<T>, x);
        }
    }
    __device__ __forceinline__ void put(unsigned o, T x) const {
        if constexpr (sizeof(T) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), x), r, o, 0, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, o, 0, 0);
    }
};

// Byte offset of cell (xg, y) within a plane (xi: xg folded into the grid).
// Cells that no result of a K-stage launch depends on -- beyond a wall, or more
// than K past the end of a periodic axis, where the last column of a grid
// reaches -- get an offset past the plane: they are not read (128^3 with 60 of
// 64 x cells per column: 140 instead of 192 x cells read per row).
template <int K>
__device__ __forceinline__ unsigned word_offset(int xg, int y, int xi, int nx, int ny, int perx, int pery,
                                                unsigned size) {
    const bool needed = (perx ? xg < nx + K : (xg >= 0) & (xg < nx)) && (pery ? y < ny + K : (y >= 0) & (y < ny));
    return needed ? (unsigned)(fold(y, ny, pery) * nx + xi) * size : 0x80000000u;
}

// f(0), f(1), ... with compile-time arguments.
template <typename F, int... J>
__device__ __forceinline__ void unroll(F&& f, std::integer_sequence<int, J...>) {
    (f(std::integral_constant<int, J>{}), ...);
}

// step(slot, z) for z = zb .. ze - 1, the first in slot 1 of a ring of U: whole
// periods without a test between the steps (one would pin every register of
// the rings and cost a move for each of them per step), then what is left.
template <int U, typename F>
__device__ __forceinline__ void run_steps(int zb, int ze, F&& step) {
    int z = zb;
    for (; z + U <= ze; z += U)
        unroll([&](auto J) { step(std::integral_constant<int, (1 + decltype(J)::value) % U>{}, z + decltype(J)::value); },
               std::make_integer_sequence<int, U>{});
    unroll(
        [&](auto J) {
            if (z + decltype(J)::value < ze)
                step(std::integral_constant<int, (1 + decltype(J)::value) % U>{}, z + decltype(J)::value);
        },
        std::make_integer_sequence<int, U - 1>{});
}

// What a launch does beside the stages themselves.
enum B3Mode {
    B3_PLAIN,
    B3_FROM_G,  // the input is c_in G (v is not read)
    B3_KEEP,    // every stage's result is kept (stages set), or the same arithmetic without
    B3_REDUCE   // the pass reductions of the last stage's result
};

// A plane step executes a fixed number of instructions per wave, and with two
// waves per SIMD these set its time as soon as the loads are ahead (the first
// form of this kernel ran 1850 of them in 4 us; the arithmetic of 24 cell
// stages is 540), so: words are addressed through plane buffers, planes wrap by
// a counter, and Lambda, 1/C and G of the waiting planes sit in rings of K + 1
// registers that the loads fill in place, indexed at compile time in a plane
// loop unrolled K + 1 times, instead of being moved along (22 instructions per
// cell and stage, 16 of them arithmetic).
template <typename R, int K, int ROWS, int WAVES, bool kHarm, B3Mode kMode>
__global__ void __launch_bounds__(64 * WAVES) k_b3d(B3Args<R> a) {
    constexpr int RW = ROWS + 2, U = K + 1;
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
    const R vs = kMode == B3_FROM_G ? (R)(1.0 / (1.0 + (a.lam ? a.tau * lamv * a.chat_in : a.tb_in))) : R(1);

    const int tile = tb::xcd_block();
    const int tx = tile % a.tiles_x, rest = tile / a.tiles_x;
    const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
    const int xg = tx * OX - K + lane;
    const int xi = fold(xg, nx, a.perx);
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
    const int zlo = a.perz ? -(1 << 30) : 0, zhi = a.perz ? (nz > 1 ? 1 << 30 : -(1 << 30)) : nz - 1;
    unsigned rows_out = 0;  // output rows of this wave
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int row = wv * ROWS + r;
        rows_out |= (unsigned)((row >= K) & (row < EXT_Y - K) & (y0 + r < ny)) << r;
    }
    // byte offsets of the lane's cells of rows -1 .. ROWS within a plane
    const int64_t plane = (int64_t)nx * ny * (int64_t)sizeof(R);
    unsigned off[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) off[r] = word_offset<K>(xg, y0 - 1 + r, xi, nx, ny, a.perx, a.pery, sizeof(R));
    R vc[K][ROWS];            // input of stage q + 1 on plane z - 1 - q
    R fz[K][ROWS];            // its weighted flux through the face below that plane
    R Lr[U][RW], nL[RW];      // Lambda: ring of planes z .. z - K, and plane z + 1 in flight
    R rc[U][ROWS], Gq[U][ROWS];  // 1/C and G: ring of planes z (in flight) .. z - K
    R nv[ROWS];               // v: plane z + 1 in flight
    int zi = fold(z0 - K, nz, a.perz);  // folded index of the plane zv that was loaded last
    int zv = z0 - K;
    auto load_vL = [&](R (&vv)[ROWS], R (&LL)[RW]) {
        const int64_t pz = (int64_t)zi * plane;
        const Plane<const R> fv(kMode == B3_FROM_G ? a.G : a.v, pz, (int)plane);
        const Plane<const R> fL(a.Lam, pz, (int)plane);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) vv[r] = fv.get(off[r + 1]);
#pragma unroll
        for (int r = 0; r < RW; ++r) LL[r] = fL.get(off[r]);
    };
    auto load_cG = [&](R (&cc)[ROWS], R (&GG)[ROWS]) {
        const int64_t pz = (int64_t)zi * plane;
        const Plane<const R> fc(a.rC, pz, (int)plane);
        const Plane<const R> fG(a.G, pz, (int)plane);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            cc[r] = fc.get(off[r + 1]);
            GG[r] = fG.get(off[r + 1]);
        }
    };
    auto next_plane = [&]() {  // wraps on a periodic axis, stays within the grid at walls
        ++zv;
        if (a.perz) zi = zi + 1 == nz ? 0 : zi + 1;
        else zi = zv < 0 ? 0 : (zv < nz ? zv : nz - 1);
    };
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) vc[q][r] = fz[q][r] = R(0);
#pragma unroll
    for (int q = 0; q < U; ++q) {
#pragma unroll
        for (int r = 0; r < RW; ++r) Lr[q][r] = R(0);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) rc[q][r] = Gq[q][r] = R(0);
    }
    // ring slot of plane zs + j: j % U.  Plane zs (slot 0) is the first input;
    // plane zs + 1 is in flight when the loop begins.
    load_vL(vc[0], Lr[0]);
    load_cG(rc[0], Gq[0]);
    next_plane();
    load_vL(nv, nL);
    if constexpr (kMode == B3_FROM_G) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) vc[0][r] *= vs;
    }
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
    const int ze = z1 + K;  // planes zs + 1 .. ze - 1 arrive in turn
    // one plane step: plane z = zs + j has arrived (ring slot S = j % U)
    auto step = [&](auto S_, int z) {
        constexpr int S = decltype(S_)::value;
        R nxt[ROWS];  // the stage's input on the plane above
#pragma unroll
        for (int r = 0; r < ROWS; ++r) nxt[r] = kMode == B3_FROM_G ? vs * nv[r] : nv[r];
#pragma unroll
        for (int r = 0; r < RW; ++r) Lr[S][r] = nL[r];
        load_cG(rc[S], Gq[S]);  // plane z
        next_plane();
        load_vL(nv, nL);  // plane z + 1
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int p = z - 1 - q;  // this stage's plane, in slot P; the plane above in slot N
            constexpr int UU = U;
            const int P = (S + 2 * UU - 1 - q) % UU, N = (S + 2 * UU - q) % UU;
            const R wzf = ((p >= zlo) & (p < zhi)) ? a.wz : R(0);
            const R vlo = sh[buf][q][wdn][1][lane], vhi = sh[buf][q][wup][0][lane];
            R fy = wyf[0] * face_of<R, kHarm>(Lr[P][0], Lr[P][1]) * (vc[q][0] - vlo);
            R res[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const R c = vc[q][r], La = Lr[P][r + 1];
                const R up = r < ROWS - 1 ? vc[q][r < ROWS - 1 ? r + 1 : r] : vhi;
                const R fx = wxr * face_of<R, kHarm>(La, from_right(La)) * (from_right(c) - c);
                const R fyu = wyf[r + 1] * face_of<R, kHarm>(La, Lr[P][r + 2]) * (up - c);
                const R fzu = wzf * face_of<R, kHarm>(La, Lr[N][r + 1]) * (nxt[r] - c);
                const R acc = (fx - from_left(fx)) + (fyu - fy) + (fzu - fz[q][r]);
                fy = fyu;
                fz[q][r] = fzu;
                res[r] = cmk[q] * (Gq[P][r] + tbk[q] * c + rc[P][r] * acc);
                // (the divisions of several rows interleaved would spill)
                if constexpr (kHarm) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                vc[q][r] = nxt[r];  // next step's centre
                nxt[r] = res[r];
            }
            if ((q == K - 1 || (kMode == B3_KEEP && a.stages)) && p >= z0 && p < z1) {  // uniform
                const Plane<R> dst(q < K - 1 ? a.stages + (int64_t)(q + 1) * a.sstride : a.out, p * plane, (int)plane);
                if (xout) {
#pragma unroll
                    for (int r = 0; r < ROWS; ++r)
                        if (rows_out >> r & 1u) dst.put(off[r + 1], res[r]);
                }
                if constexpr (kMode == B3_REDUCE) {
                    if (a.ps.dmax) {
                        const Plane<const double> tit(a.Tit, p * plane, (int)plane);
                        double t[ROWS];
#pragma unroll
                        for (int r = 0; r < ROWS; ++r) t[r] = tit.get(off[r + 1]);
#pragma unroll
                        for (int r = 0; r < ROWS; ++r)
                            dmax = fmax(dmax, xout && (rows_out >> r & 1u) ? fabs((double)res[r] - t[r]) : 0.0);
                    }
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        const double tn = (double)res[r];
                        const bool o = xout && (rows_out >> r & 1u);
                        tmax = fmax(tmax, o ? fabs(tn) : 0.0);
                        bad += o && (!(tn > 0.0) || isinf(tn)) ? 1.0 : 0.0;
                    }
                }
            }
        }
        buf ^= 1;
        publish(buf);
    };
    // steps j = 1, 2, ...: slot j % U
    run_steps<U>(z0 - K + 1, ze, step);
    if constexpr (kMode == B3_REDUCE) {
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
// two waves per SIMD (harmonic means take a few more registers)
template <typename R, int K, bool kHarm>
constexpr int b3_rows() {
    if (sizeof(R) == 8) return (K == 3 ? 3 : 4) - (kHarm ? 1 : 0);
    return (K == 4 ? 5 : K == 3 ? 6 : 8) - (kHarm ? (K >= 3 ? 2 : 1) : 0);
}

// stages per launch
template <typename R>
constexpr int b3_kmax() {
    return sizeof(R) == 8 ? 3 : 4;
}

// Columns of ox x oy results and the z chunks of a launch of K stages: one
// workgroup per CU at a time, each walking its chunk and 2K planes more; the
// count of chunks with the fewest planes walked in turn (planes).
struct Columns {
    int tiles_x, tiles_y, zc;
    int64_t planes;
};
Columns z_chunks(const DevGrid& g, int ox, int oy, int K) {
    Columns w{(g.nx + ox - 1) / ox, (g.ny + oy - 1) / oy, g.nz, 0};
    const int64_t cols = (int64_t)w.tiles_x * w.tiles_y, over = 2 * K + 1;
    // for each number of rounds the shortest chunks that fill it
    for (int64_t r = (cols + kCUs - 1) / kCUs; w.planes == 0 || r * (1 + over) < w.planes; ++r) {
        const int64_t n = r * kCUs / cols;  // chunks per column
        const int c = (int)((g.nz + n - 1) / n);
        if (w.planes == 0 || r * (c + over) < w.planes) {
            w.planes = r * (c + over);
            w.zc = c;
        }
        if (c == 1) break;
    }
    return w;
}

// (a plane's byte offsets fit 31 bits)
bool b3d_applies(const DevGrid& g) { return use_z3d(g) && (int64_t)g.nx * g.ny < ((int64_t)1 << 28); }

template <typename R, int K, bool kHarm>
Columns b3d_columns(const DevGrid& g) {
    return z_chunks(g, 64 - 2 * K, b3_rows<R, K, kHarm>() * kWaves3 - 2 * K, K);
}

// Whether launches of K stages beat one stage a launch.  A column of a
// workgroup is 10 to 32 rows of results whatever the grid has, so on grids of few
// y rows (and with harmonic means, whose columns are narrowest, on some more)
// they compute rows that are no cells: 1000 x 1 x 1000 in double takes 37 us a
// stage in launches of 3 and 23 one by one, x 4 rows 37.7 and 38.5, x 5 rows 39
// and 57; 64 x 1 x 20000 77 and 28.  Where a launch is mostly its start they pay
// on any grid (256 x 1 x 256: 6.5 and 9.1).  A launch takes 1.7 us and `step` us
// for each plane walked in turn, or the memory's rate.
template <typename R, int K, bool kHarm>
bool b3d_pays(const DevGrid& g, double step) {
    const double walk = 1.7 + step * (double)b3d_columns<R, K, kHarm>(g).planes;
    const double mem = (double)g.N * (sizeof(R) * 5 / 4.5e6);
    return (walk > mem ? walk : mem) <= K * z3d_cost(g, kHarm ? 1 : 0, sizeof(R) == 4);
}

template <typename R, int K, bool kHarm>
void launch_b3d_k(hipStream_t s, const DevGrid& g, B3Args<R>& a, bool keep) {
    constexpr int rows = b3_rows<R, K, kHarm>(), waves = kWaves3;
    const Columns w = b3d_columns<R, K, kHarm>(g);
    a.tiles_x = w.tiles_x;
    a.tiles_y = w.tiles_y;
    a.zc = w.zc;
    const int64_t wg = (int64_t)a.tiles_x * a.tiles_y * ((g.nz + a.zc - 1) / a.zc);
    const dim3 grid((unsigned)wg), block(64 * waves);
    auto go = [&](auto mode) {
        hipLaunchKernelGGL((k_b3d<R, K, rows, waves, kHarm, decltype(mode)::value>), grid, block, 0, s, a);
    };
    if constexpr (sizeof(R) == 8) {
        if (keep) go(std::integral_constant<B3Mode, B3_KEEP>{});
        else if (a.Tit) go(std::integral_constant<B3Mode, B3_REDUCE>{});
        else go(std::integral_constant<B3Mode, B3_PLAIN>{});
    } else {
        if (!a.v) go(std::integral_constant<B3Mode, B3_FROM_G>{});
        else go(std::integral_constant<B3Mode, B3_PLAIN>{});
    }
}

}  // namespace

int b3d_rows(int face, int K, bool f32) {
    auto rows = [&](auto harm) {
        constexpr bool h = decltype(harm)::value;
        if (f32) return K == 4 ? b3_rows<float, 4, h>() : K == 3 ? b3_rows<float, 3, h>() : b3_rows<float, 2, h>();
        return K == 3 ? b3_rows<double, 3, h>() : b3_rows<double, 2, h>();
    };
    return kWaves3 * (face == 1 ? rows(std::true_type{}) : rows(std::false_type{}));
}

int b3d_stages(const DevGrid& g, int face, int count, bool f32) {
    if (!b3d_applies(g)) return 1;
    const bool pays = f32 ? (face == 1 ? b3d_pays<float, 4, true>(g, 2.5) : b3d_pays<float, 4, false>(g, 1.52))
                          : (face == 1 ? b3d_pays<double, 3, true>(g, 1.9) : b3d_pays<double, 3, false>(g, 1.4));
    if (!pays) return 1;
    const int kmax = f32 ? b3_kmax<float>() : b3_kmax<double>();
    const int launches = (count + kmax - 1) / kmax;
    return (count + launches - 1) / launches;
}

template <typename R>
void launch_b3d(hipStream_t s, const DevGrid& g, int face, const R* v, const R* G, const R* Lam, const R* rC, R* out,
                Stages st, int K, double tau, const double* Tit, PassSlots ps, StageParam sp_in, bool keep, R* stages,
                int64_t sstride) {
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
    auto run = [&](auto harm) {
        constexpr bool h = decltype(harm)::value;
        if (K == 2) return launch_b3d_k<R, 2, h>(s, g, a, keep);
        if constexpr (b3_kmax<R>() >= 4) {
            if (K == 4) return launch_b3d_k<R, 4, h>(s, g, a, keep);
        }
        launch_b3d_k<R, 3, h>(s, g, a, keep);
    };
    if (face == 1) run(std::true_type{});
    else run(std::false_type{});
}

template void launch_b3d<double>(hipStream_t, const DevGrid&, int, const double*, const double*, const double*,
                                 const double*, double*, Stages, int, double, const double*, PassSlots, StageParam,
                                 bool, double*, int64_t);
template void launch_b3d<float>(hipStream_t, const DevGrid&, int, const float*, const float*, const float*,
                                const float*, float*, Stages, int, double, const double*, PassSlots, StageParam,
                                bool, float*, int64_t);

}  // namespace tlim

// ------------------------------------------------------------------ adjoint

namespace tlim {

namespace {

// Reverse stages of the LIM adjoint on 3D grids in psi = C^-1 lambda form
// (arithmetic face means), K = 1 or 2 per launch, along the same z-march:
//   psi^(m-1) = c_m (tau b_m psi^(m) - tau rC sum_f w_f Lambda_f (psi_a - psi_b)),
//   dgpsi += c_m psi^(m)_a,
//   gLam  += c_m sum_f (tau w_f / 2) (v_b - v_a)^(m-1) (psi_a - psi_b)^(m).
// With e_f = (tau w_f / 2)(psi_b - psi_a) formed once per face, both sums of a
// face follow from it: (Lambda_a + Lambda_b) e_f for psi and (v_b - v_a) e_f for
// gLam, shared by the face's two cells.  The sums dgpsi and gLam of a plane
// wait in registers from one stage to the next.
// Per cell two stages read psi, Lambda, 1/C, both sums and two stored iterates
// and write psi and both sums: 80 B against 144 B for two launches of one
// stage.  At 128^3 a launch of two stages takes 53 us (one stage per launch by
// waves of two rows, each with its own windows: 37 us), and waits for issue and
// for memory in about equal parts; registers hold two rows per wave for K = 2
// (three spill).
struct A3Args {
    const double* psi;
    const double* v[2];  // v^(m-1) of the launch's stages, in the order they are reversed
    const double* Lam;
    const double* rC;
    double* psi_out;
    double* dgpsi;
    double* gLam;
    double cm[2], tb[2];
    int nx, ny, nz, perx, pery, perz;
    double hx, hy, hz;  // tau w / 2
    int tiles_x, tiles_y, zc;
};

template <int K, int ROWS, bool kAcc>
__global__ void __launch_bounds__(512) k_adj_b3d(A3Args a) {
    constexpr int WAVES = kWaves3, RW = ROWS + 2, U = K + 1;
    constexpr int OX = 64 - 2 * K, EXT_Y = WAVES * ROWS, OY = EXT_Y - 2 * K;
    // seam rows of the stages' psi and v: [buffer][stage][psi, v][wave][first / last row]
    __shared__ double sh[2][K][2][WAVES][2][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int tile = tb::xcd_block();
    const int tx = tile % a.tiles_x, rest = tile / a.tiles_x;
    const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
    const int xg = tx * OX - K + lane;
    const int xi = fold(xg, nx, a.perx);
    const int y0 = ty * OY - K + wv * ROWS;
    const int z0 = tz * a.zc;
    const int z1 = z0 + a.zc < nz ? z0 + a.zc : nz;
    const bool xout = lane >= K && lane < 64 - K && xg < nx;
    const double hxr = (a.perx ? nx > 1 : (xg >= 0 && xg < nx - 1)) ? a.hx : 0.0;
    double hyf[ROWS + 1];
#pragma unroll
    for (int r = 0; r <= ROWS; ++r) {
        const int y = y0 + r - 1;
        hyf[r] = (a.pery ? ny > 1 : (y >= 0 && y < ny - 1)) ? a.hy : 0.0;
    }
    const int zlo = a.perz ? -(1 << 30) : 0, zhi = a.perz ? (nz > 1 ? 1 << 30 : -(1 << 30)) : nz - 1;
    unsigned rows_out = 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int row = wv * ROWS + r;
        rows_out |= (unsigned)((row >= K) & (row < EXT_Y - K) & (y0 + r < ny)) << r;
    }
    const int64_t plane = (int64_t)nx * ny * 8;
    unsigned off[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) off[r] = word_offset<K>(xg, y0 - 1 + r, xi, nx, ny, a.perx, a.pery, 8);

    double pc[K][ROWS], fz[K][ROWS], gz[K][ROWS];  // stage q + 1 on plane z - 1 - q: psi, face sums below
    double va[K][ROWS], vb[K][ROWS], nv[K][ROWS];  // its v on that plane, the one above, and the next in flight
    double Lr[U][RW], nL[RW];                      // Lambda: planes z .. z - K, and z + 1 in flight
    double rc[U][ROWS];                            // 1/C: planes z (in flight) .. z - K
    double np[ROWS], nd[ROWS], ng[ROWS];           // in flight: psi of z + 1, the sums of z
    double ds[K][ROWS], gs[K][ROWS];               // the sums before stage q + 1 on its plane
    int zi = fold(z0 - K, nz, a.perz), zv = z0 - K;  // plane zv (folded zi) was loaded last
    auto load_a = [&]() {  // plane zv: psi, Lambda, v of the first stage
        const int64_t pz = (int64_t)zi * plane;
        const Plane<const double> fp(a.psi, pz, (int)plane), fv(a.v[0], pz, (int)plane), fL(a.Lam, pz, (int)plane);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            np[r] = fp.get(off[r + 1]);
            nv[0][r] = fv.get(off[r + 1]);
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) nL[r] = fL.get(off[r]);
    };
    auto load_b = [&](double (&cc)[ROWS]) {  // plane zv: 1/C, the sums, v of the second stage
        const int64_t pz = (int64_t)zi * plane;
        const Plane<const double> fc(a.rC, pz, (int)plane);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) cc[r] = fc.get(off[r + 1]);
        if constexpr (K == 2) {
            const Plane<const double> fv(a.v[1], pz, (int)plane);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) nv[1][r] = fv.get(off[r + 1]);
        }
        if constexpr (kAcc) {
            const Plane<const double> fd(a.dgpsi, pz, (int)plane), fg(a.gLam, pz, (int)plane);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                nd[r] = fd.get(off[r + 1]);
                ng[r] = fg.get(off[r + 1]);
            }
        }
    };
    auto next_plane = [&]() {
        ++zv;
        if (a.perz) zi = zi + 1 == nz ? 0 : zi + 1;
        else zi = zv < 0 ? 0 : (zv < nz ? zv : nz - 1);
    };
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            pc[q][r] = fz[q][r] = gz[q][r] = va[q][r] = vb[q][r] = nv[q][r] = ds[q][r] = gs[q][r] = nd[r] = ng[r] = 0.0;
#pragma unroll
    for (int q = 0; q < U; ++q) {
#pragma unroll
        for (int r = 0; r < RW; ++r) Lr[q][r] = 0.0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) rc[q][r] = 0.0;
    }
    load_a();
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        pc[0][r] = np[r];
        va[0][r] = nv[0][r];
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) Lr[0][r] = nL[r];
    load_b(rc[0]);
    next_plane();
    load_a();
    const int wdn = wv > 0 ? wv - 1 : 0, wup = wv < WAVES - 1 ? wv + 1 : wv;
    auto publish = [&](int buf) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            sh[buf][q][0][wv][0][lane] = pc[q][0];
            sh[buf][q][0][wv][1][lane] = pc[q][ROWS - 1];
            sh[buf][q][1][wv][0][lane] = va[q][0];
            sh[buf][q][1][wv][1][lane] = va[q][ROWS - 1];
        }
    };
    publish(0);
    int buf = 0;
    const int ze = z1 + K;
    auto step = [&](auto S_, int z) {
        constexpr int S = decltype(S_)::value;
        // plane z has arrived (psi, Lambda and the first stage's v), and plane
        // z - 1 of the rest
        double nxt[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            nxt[r] = np[r];
            ds[0][r] = nd[r];
            gs[0][r] = ng[r];
        }
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) vb[q][r] = nv[q][r];
#pragma unroll
        for (int r = 0; r < RW; ++r) Lr[S][r] = nL[r];
        load_b(rc[S]);
        next_plane();
        load_a();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        double dn[K][ROWS], gn[K][ROWS];  // the sums after each stage
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int p = z - 1 - q;
            constexpr int UU = U;
            const int P = (S + 2 * UU - 1 - q) % UU, N = (S + 2 * UU - q) % UU;
            const double hzf = ((p >= zlo) & (p < zhi)) ? a.hz : 0.0;
            const double plo = sh[buf][q][0][wdn][1][lane], phi = sh[buf][q][0][wup][0][lane];
            const double vlo = sh[buf][q][1][wdn][1][lane], vhi = sh[buf][q][1][wup][0][lane];
            double ed = hyf[0] * (pc[q][0] - plo);
            double fy = (Lr[P][0] + Lr[P][1]) * ed, gy = (va[q][0] - vlo) * ed;
            double res[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const double c = pc[q][r], v = va[q][r], La = Lr[P][r + 1];
                const double up = r < ROWS - 1 ? pc[q][r < ROWS - 1 ? r + 1 : r] : phi;
                const double vu = r < ROWS - 1 ? va[q][r < ROWS - 1 ? r + 1 : r] : vhi;
                const double ex = hxr * (from_right(c) - c);
                const double fx = (La + from_right(La)) * ex, gx = (from_right(v) - v) * ex;
                const double ey = hyf[r + 1] * (up - c);
                const double fyu = (La + Lr[P][r + 2]) * ey, gyu = (vu - v) * ey;
                const double ez = hzf * (nxt[r] - c);
                const double fzu = (La + Lr[N][r + 1]) * ez, gzu = (vb[q][r] - v) * ez;
                const double acc = (fx - from_left(fx)) + (fyu - fy) + (fzu - fz[q][r]);
                const double g = (gx + from_left(gx)) + (gyu + gy) + (gzu + gz[q][r]);
                fy = fyu;
                gy = gyu;
                fz[q][r] = fzu;
                gz[q][r] = gzu;
                dn[q][r] = ds[q][r] + a.cm[q] * c;
                gn[q][r] = gs[q][r] - a.cm[q] * g;
                res[r] = a.cm[q] * (a.tb[q] * c + rc[P][r] * acc);
                __builtin_amdgcn_sched_barrier(0);  // (rows interleaved would spill)
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                pc[q][r] = nxt[r];
                nxt[r] = res[r];
                va[q][r] = vb[q][r];
            }
            if (q == K - 1 && p >= z0 && p < z1) {  // uniform
                const Plane<double> op(a.psi_out, p * plane, (int)plane), od(a.dgpsi, p * plane, (int)plane),
                    og(a.gLam, p * plane, (int)plane);
                if (xout) {
#pragma unroll
                    for (int r = 0; r < ROWS; ++r)
                        if (rows_out >> r & 1u) {
                            op.put(off[r + 1], res[r]);
                            od.put(off[r + 1], dn[q][r]);
                            og.put(off[r + 1], gn[q][r]);
                        }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // the sums of a plane wait for the next stage's step
#pragma unroll
        for (int q = 1; q < K; ++q)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                ds[q][r] = dn[q - 1][r];
                gs[q][r] = gn[q - 1][r];
            }
        buf ^= 1;
        publish(buf);
    };
    run_steps<U>(z0 - K + 1, ze, step);
}

constexpr int adj_rows(int K) { return K == 2 ? 2 : 4; }
Columns adj_columns(const DevGrid& g, int K) { return z_chunks(g, 64 - 2 * K, adj_rows(K) * kWaves3 - 2 * K, K); }

template <int K>
void launch_adj_b3d_k(hipStream_t s, const DevGrid& g, A3Args& a, bool accumulate) {
    constexpr int rows = adj_rows(K), waves = kWaves3;
    const Columns w = adj_columns(g, K);
    a.tiles_x = w.tiles_x;
    a.tiles_y = w.tiles_y;
    a.zc = w.zc;
    const int64_t wg = (int64_t)a.tiles_x * a.tiles_y * ((g.nz + a.zc - 1) / a.zc);
    if (accumulate) hipLaunchKernelGGL((k_adj_b3d<K, rows, true>), dim3((unsigned)wg), dim3(64 * waves), 0, s, a);
    else hipLaunchKernelGGL((k_adj_b3d<K, rows, false>), dim3((unsigned)wg), dim3(64 * waves), 0, s, a);
}

__global__ void __launch_bounds__(256) k_scale_rc(int64_t n, const double* __restrict__ x, const double* __restrict__ rC,
                                                  double* __restrict__ y) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = x[i] * rC[i];
}

}  // namespace

// As b3d_pays: on grids of one to four y rows most of a column's 12 rows are no
// cells (gradient of one step of two passes, two stages per launch and one:
// 1000 x 1 x 1000 3.7 and 2.7 ms, x 3 rows 4.1 and 4.5; 64 x 1 x 20000 7.8 and
// 4.6 ms; 256 x 1 x 256 0.67 and 0.74).
bool use_adj_b3d(const DevGrid& g, int face) {
    return face == 0 && b3d_applies(g) && 1.7 + 1.6 * (double)adj_columns(g, 2).planes <= 2.0 * adj_z3d_cost(g);
}

void launch_psi_from_lambda(hipStream_t s, int64_t n, const double* lam, const double* rC, double* psi) {
    const int64_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_scale_rc, dim3((unsigned)(b < 8192 ? b : 8192)), dim3(256), 0, s, n, lam, rC, psi);
}

void launch_adj_b3d(hipStream_t s, const DevGrid& g, int K, const double* psi, const double* const v[2],
                    const double* Lam, const double* rC, double* psi_out, double* dgpsi, double* gLam,
                    const double cm[2], const double tb[2], double tau, int accumulate) {
    A3Args a{};
    a.psi = psi;
    a.Lam = Lam;
    a.rC = rC;
    a.psi_out = psi_out;
    a.dgpsi = dgpsi;
    a.gLam = gLam;
    for (int k = 0; k < K; ++k) {
        a.v[k] = v[k];
        a.cm[k] = cm[k];
        a.tb[k] = tb[k];
    }
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.perx = g.per[0];
    a.pery = g.per[1];
    a.perz = g.per[2];
    a.hx = 0.5 * tau * g.w[0];
    a.hy = 0.5 * tau * g.w[1];
    a.hz = 0.5 * tau * g.w[2];
    if (K == 2) launch_adj_b3d_k<2>(s, g, a, accumulate != 0);
    else launch_adj_b3d_k<1>(s, g, a, accumulate != 0);
}

}  // namespace tlim
