// P2G: spreading of the 3-vector forces onto the uniform grid, eq. (p2g):
//   phi(g_l) = sum_j sum_p w(g_l - y_j + p) f_j,  w separable, P points per axis.
//
// Atomic-free, owner-computes design for MI355X.  One wavefront covers an 8 x 8 patch of grid
// lines along x (lane (ly, lz) owns line (y0+ly, z0+lz)).  A particle in cell-x c adds
// w_x[k] * w_y * w_z * f to the points x = c - P/2 + 1 + k of every line of its footprint.  The
// particles of a slab (cell-x constant) that can reach the patch, a (8+P-1)^2 window of cells,
// are contiguous runs of the cell-sorted arrays.  Every grid point is written once, as a sum in
// a fixed order: deterministic, no atomics, no zero-fill.  The x direction is exact (no wasted
// work); in y and z a lane whose line is outside a particle's footprint multiplies by zero.
#include <algorithm>
#include <climits>

#include "window.h"

namespace ewald {

namespace {

constexpr int kPatch = 8;     // lines per patch edge (8 x 8 = 64 lanes)
constexpr int kWaves = 4;     // waves per block, all owning the block's lines
constexpr int kSlabs = 4;     // slabs of a pass, and points merged after it
constexpr int kWindow = kWaves * kSlabs;  // most slabs whose runs are tabulated at a time
constexpr int kBatch = 16;    // particles staged per wave and round, four lanes each
constexpr int kMaxRuns = 320; // runs per slab (window rows x z-tile segments)
constexpr int kTable = 1536;  // entries of the run table (a window has fewer slabs where runs are many)
static_assert(kTable >= (kMaxRuns + 1) * kSlabs, "the runs of kSlabs slabs must fit the table");
static_assert(kSlabs == kWaves, "a merge gives each wave one point");

// acc[k][c] += w_x[k] g_c for all k: lane i of every row of 16 lanes holds w_x[i], and the DPP
// row_newbcast of v_fmac_f64 broadcasts w_x[k] from it, so that a particle's x weights take one LDS
// read instead of P.  The s_nop covers the two wait states between a VALU write of w (a register copy)
// and its use as a DPP operand.
#define EWALD_FMAC3(a0, a1, a2, k)                                                               \
    "v_fmac_f64_dpp %" #a0 ", %[w], %[g0] row_newbcast:%c[" #k "] row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f64_dpp %" #a1 ", %[w], %[g1] row_newbcast:%c[" #k "] row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f64_dpp %" #a2 ", %[w], %[g2] row_newbcast:%c[" #k "] row_mask:0xf bank_mask:0xf\n\t"
#define EWALD_ACC3(k) "+v"(a[k][0]), "+v"(a[k][1]), "+v"(a[k][2])
template <int K0, int P>
__device__ inline void spread(double (*acc)[3], double w, double g0, double g1, double g2)
{
    double(*a)[3] = acc + K0;
    if constexpr (K0 + 4 <= P) {
        asm("s_nop 1\n\t" EWALD_FMAC3(0, 1, 2, k0) EWALD_FMAC3(3, 4, 5, k1) EWALD_FMAC3(6, 7, 8, k2)
                EWALD_FMAC3(9, 10, 11, k3)
            : EWALD_ACC3(0), EWALD_ACC3(1), EWALD_ACC3(2), EWALD_ACC3(3)
            : [w] "v"(w), [g0] "v"(g0), [g1] "v"(g1), [g2] "v"(g2), [k0] "n"(K0), [k1] "n"(K0 + 1),
              [k2] "n"(K0 + 2), [k3] "n"(K0 + 3));
    } else {
        asm("s_nop 1\n\t" EWALD_FMAC3(0, 1, 2, k0) EWALD_FMAC3(3, 4, 5, k1)
            : EWALD_ACC3(0), EWALD_ACC3(1)
            : [w] "v"(w), [g0] "v"(g0), [g1] "v"(g1), [g2] "v"(g2), [k0] "n"(K0), [k1] "n"(K0 + 1));
    }
    if constexpr (K0 + 4 < P) spread<K0 + 4, P>(acc, w, g0, g1, g2);
}
#undef EWALD_FMAC3
#undef EWALD_ACC3

// the value of another lane of this lane's four
template <int kPerm>
__device__ inline int quad_lane(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, kPerm, 0xf, 0xf, true);
}

// A block of kWaves waves owns one patch and the x-segment [x0, x0 + seg).  It takes the segment in
// windows of up to kWindow slabs (their run table in LDS) and a window in passes of kSlabs slabs.  A wave
// spreads a quarter of each slab's particles into its own register window of kSlabs + P - 1 points; after
// a pass the waves' sums of the kSlabs points that no later slab reaches are added through LDS in a
// fixed order and written, and the other P - 1 points stay in the waves' registers.  A point's four sums
// run over the slabs' quarters in the order of the sort, whatever the lengths of passes and windows, so
// that its value does not depend on them.  The first and last P - 1 points of a segment also receive from
// the neighbouring segments: they go, as partial sums, to halo planes (head[s][k] and tail[s][k] hold
// the points x0 - P/2 + 1 + k and x1 - P/2 + 1 + k), and the first FFT pass adds them as it reads (k_p2g_halo_sum into the grid, with stresslet sources or
// where the grid itself is asked for).  Fold (M1
// = 8 < P: one segment, shorter than the stencil): the points are added modulo M1 instead, each wave
// keeping its two of the eight.
//
// What bounds it: FP64 FMAs at the patches' lane efficiency where particles are dense (c2: 3P FMAs of
// 3P + 7 instructions per particle and patch, two waves per SIMD by the 6 (kSlabs + P - 1) accumulator
// registers); latency of the tables, the staging and the barriers where they are sparse, and the halo
// planes' traffic (24 systems of 5e3 on 64^3: segments of 16 points, about 0.1 ms).  One pass per slab,
// staged and merged by itself, spent 14 thousand cycles a slab on 30 particles; four slabs of its own
// per wave and one merge per window took 0.05 ms less for the 24 systems and 0.03 for 1e6 on 256^3 with P = 8, but
// added a point's contributions in another order.  P2G ms with a pass per slab and with four
// (and the halo planes added by the FFT, 0.03 ms of it for the 24 systems): 1e6 uniform on 256^3, P = 16 3.01 ->
// 1.56, P = 8 (FP32) 2.17 -> 0.56; 24 systems of 5e3 0.85 -> 0.27; 1.5e5 on 128 x 128 x 256 0.71 -> 0.31; 1e3 on 32^3
// 0.083 -> 0.028; dense grids: c2 1.46 -> 1.32, H 0.91 -> 0.73, c4 4.38 -> 4.09, c3 8.8 -> 8.0; one loss: 2e4 in two
// clusters of five cells 0.46 -> 0.53 (few patches hold everything, and a lone wave per SIMD, which issues an FP64
// instruction every eight cycles, pays the staging's latency), 0.48 since the search tries the last round's runs
// first (locate; spread as a whole, with the sort, 0.64 -> 0.56; 24 systems 0.27 -> 0.25, H 0.73 -> 0.72, c2 1.32 -> 1.34).
//
// Staging: 16 particles at a time, four lanes each (two halves of the x weights, the y weights of the
// patch's lines, and their z weights times f, zero off the footprint), every lane by one recurrence of
// at most eight steps; the next particles' records are fetched while these are spread, across passes.
template <typename TG, int P, bool Fold>
__global__ __launch_bounds__(kWaves * 64, P <= 14 ? 3 : 2) void k_p2g_sweep(const Rec64* __restrict__ rec,
                                                           const int* __restrict__ start, Geometry g,
                                                           WinArgs<double> wa, int seg, int npy, int npz,
                                                           const double* __restrict__ sv, int sv_off,
                                                           TG* __restrict__ grid, double* __restrict__ halo,
                                                           int64_t grid_stride, int64_t halo_stride)
{
    constexpr int W = kPatch + P - 1;
    constexpr int kPts = kSlabs + P - 1;  // points of a wave's register window
    // staged particle: P x weights, 8 y weights, 8 z weights times each component of f (an odd row
    // length: the rows of consecutive particles start in different banks)
    constexpr int kRow = P + 4 * kPatch + 1;
    constexpr int kOut = kSlabs * 3 * kWave;  // sums of a wave's finished points
    constexpr int kMine = kBatch * kRow > kOut ? kBatch * kRow : kOut;
    __shared__ double smem[kWaves * kMine];
    __shared__ int run_start[kTable], run_pre[kTable];
    __shared__ int slab_n[kWindow];
    __shared__ int slab_end[kWaves][kWindow], slab_at[kWaves][kWindow];

    // system blockIdx.y of a batch: its cell list, grid and halo planes
    start += (int64_t)blockIdx.y * g.ncells;
    grid += (int64_t)blockIdx.y * grid_stride;
    halo += (int64_t)blockIdx.y * halo_stride;

    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int item = blockIdx.x;
    const int pz = item % npz, py = (item / npz) % npy, sx = item / (npz * npy);
    const int M1 = g.M[0], M2 = g.M[1], M3 = g.M[2];
    const int x0 = sx * seg;
    const int y0 = py * kPatch, z0 = pz * kPatch;
    const int ly = lane >> 3, lz = lane & 7;
    const int B = g.B;

    const int zlo = z0 - P / 2, zhi = z0 + kPatch - 1 + P / 2 - 1;
    const int zt0 = floor_div(zlo, B), zt1 = floor_div(zhi, B);
    const int nzs = zt1 - zt0 + 1;
    const int R = W * nzs;
    const int nzs_inv = 65536 / nzs + 1;  // r / nzs = (r nzs_inv) >> 16 for r < kMaxRuns
    int wn = min(kWindow, seg);
    while (wn * (R + 1) > kTable) wn >>= 1;

    // this lane's part of a staged particle (see above)
    const int role = lane & 3, axis = role < 2 ? 0 : role - 1;
    const double h = g.h[axis];
    const double e2 = exp(-2.0 * wa.beta);  // ratio of consecutive Gaussian recurrence factors
    double* const row0 = smem + wid * kMine;
    double* const mine = row0 + (lane >> 2) * kRow;

    const int64_t nc = g.ncells;
    const int64_t m23 = (int64_t)M2 * M3;
    const unsigned line = (unsigned)((y0 + ly) * M3 + (z0 + lz));
    const int hk = P - 1;
    double* const head = halo + (int64_t)sx * hk * 3 * m23;
    double* const tail = halo + ((int64_t)gridDim.x / (npy * npz) + sx) * hk * 3 * m23;

    double acc[kPts][3];
#pragma unroll
    for (int k = 0; k < kPts; ++k) acc[k][0] = acc[k][1] = acc[k][2] = 0.0;
    double folded[2][3] = {};  // Fold: points wid and wid + 4 modulo 8

    // The waves' first kSlabs points are added in wave order, point wid by this wave, and the windows move
    // on by kSlabs points.
    double v[3];
    auto merge = [&]() {
#pragma unroll
        for (int k = 0; k < kSlabs; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) row0[(k * 3 + c) * kWave + lane] = acc[k][c];
        __syncthreads();
        double a[kWaves][3];
#pragma unroll
        for (int q = 0; q < kWaves; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) a[q][c] = smem[q * kMine + (wid * 3 + c) * kWave + lane];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = a[0][c];
#pragma unroll
            for (int q = 1; q < kWaves; ++q) v[c] += a[q][c];
        }
#pragma unroll
        for (int k = 0; k < kPts; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[k][c] = k + kSlabs < kPts ? acc[k + kSlabs < kPts ? k + kSlabs : 0][c] : 0.0;
        __syncthreads();
    };

    for (int sb = 0; sb < seg; sb += wn) {
        // run table of the window's slabs: one run per (window row, z-tile segment); entry r of slab s
        // holds the run's first particle and the number of the slab's particles before it, entry R ends
        // the slab's search
        // (a wave's slabs, every fourth of the window, side by side: their loads and scans overlap)
        constexpr int kSide = kWindow / kWaves;
        int before[kSide] = {};
        for (int r0 = 0; r0 < R; r0 += kWave) {
            const int r = r0 + lane;
            const int iy = (r * nzs_inv) >> 16, zs = r - iy * nzs;
            const int cy = wrapi(y0 - P / 2 + iy, M2);
            const int zt = zt0 + zs;
            const int au = max(zlo, zt * B), bu = min(zhi, zt * B + B - 1);
            const int cz = wrapi(au, M3);
            int st[kSide], len[kSide];
#pragma unroll
            for (int j = 0; j < kSide; ++j) {
                const int s = wid + kWaves * j;
                st[j] = len[j] = 0;
                if (s < wn && r < R) {
                    const int k0 = cell_key(wrapi(x0 + sb + s, M1), cy, cz, g);
                    st[j] = start[k0];
                    len[j] = start[k0 + (bu - au) + 1];
                }
            }
#pragma unroll
            for (int j = 0; j < kSide; ++j) {
                const int s = wid + kWaves * j;
                if (s >= wn) break;
                const int n = len[j] - st[j];
                const int inc = wave_scan(n);
                if (r < R) {
                    run_start[s * (R + 1) + r] = st[j];
                    run_pre[s * (R + 1) + r] = before[j] + inc - n;
                }
                before[j] += __builtin_amdgcn_readlane(inc, kWave - 1);
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < kSide; ++j) {
                const int s = wid + kWaves * j;
                if (s >= wn) break;
                slab_n[s] = before[j];
                run_pre[s * (R + 1) + R] = INT_MAX;
            }
        }
        __syncthreads();

        const int in_slab = lane < wn ? slab_n[lane < wn ? lane : 0] : 0;
        // this wave's quarter of the slab: particles [qa, qa + qn)
        const int quarter = (in_slab + kWaves - 1) / kWaves;
        const int qa = min(in_slab, wid * quarter), qn = min(in_slab, qa + quarter) - qa;
        const int ends = wave_scan(qn);  // of the wave's quarters one after the other
        if (lane < kWindow) {
            slab_end[wid][lane] = ends;
            slab_at[wid][lane] = qa + qn - ends;
        }
        wave_lds_sync();
        const int all = __builtin_amdgcn_readlane(ends, kWindow - 1);

        // A particle of the wave's share, from its place in the order of the slabs' run tables
        // (places past the last repeat it): its index, and the stencil offset of this lane's first
        // weight (for z without the cell's offset in its tile).  The four lanes of a particle search
        // its run together, four ways a step; where the last round's particles lay in one run or two
        // (dense columns), the four runs from its first particle's on are tried before.
        int idx = 0, off = 0;
        int slab0 = 0, run0 = -1;  // the last round's first particle's; -1: not to be tried
        auto locate = [&](int base) {
            const int flat = min(base + (lane >> 2), all - 1);
            int k = 0, lo = 0, tb = 0, t = 0;
            auto among4 = [](bool is) {  // how many of this lane's four
                int below = is ? 1 : 0;
                below += quad_lane<0xb1>(below);  // lane ^ 1
                below += quad_lane<0x4e>(below);  // lane ^ 2
                return below;
            };
            bool found = false;
            if (run0 >= 0 && min(base + kBatch, all) <= __builtin_amdgcn_readlane(ends, slab0)) {
                k = slab0;
                tb = k * (R + 1);
                t = flat + slab_at[wid][slab0];
                lo = among4(run_pre[tb + min(run0 + role + 1, R)] <= t);
                found = __builtin_amdgcn_readlane(lo, kWave - 1) < 4;
                lo += run0;
            }
            if (!found) {
                // its slab: the number of slabs that end at or before it, four ways a step
                k = 0;
                auto slab_step = [&](int s) {
                    k += s * among4(slab_end[wid][min(k + s * (role + 1), kWindow) - 1] <= flat);
                };
                slab_step(4);
                slab_step(1);
                tb = k * (R + 1);
                t = flat + slab_at[wid][k];
                lo = 0;
                auto step = [&](int s) { lo += s * among4(run_pre[tb + min(lo + s * (role + 1), R)] <= t); };
                if (R > 256) step(256);
                step(64);
                step(16);
                step(4);
                step(1);
            }
            slab0 = __builtin_amdgcn_readlane(k, 0);
            run0 = __builtin_amdgcn_readlane(lo, 0);
            if (__builtin_amdgcn_readlane(tb + lo, kWave - 1) - (slab0 * (R + 1) + run0) > 1) run0 = -1;
            idx = run_start[tb + lo] + (t - run_pre[tb + lo]);
            const int iy = (lo * nzs_inv) >> 16, zs = lo - iy * nzs;
            off = role < 2 ? role * (P / 2) : role == 2 ? P - 1 - iy : z0 + P / 2 - 1 - (zt0 + zs) * B;
        };
        struct Part {  // what this lane reads of a particle
            double x, f0, f1, f2;
            int c, off;
        } p;
        auto fetch = [&]() {
            const Rec64& q = rec[idx];
            p.x = q.x[axis];
            p.c = q.c[axis];
            p.off = off;
            p.f0 = 1.0;
            if (role == 3) {
                const double* f = sv ? sv + 6 * (int64_t)idx + sv_off : q.f;
                p.f0 = f[0];
                p.f1 = f[1];
                p.f2 = f[2];
            }
        };
        auto stage = [&]() {
            const double t = p.x / h - (double)p.c;
            const int j0 = p.off - (role == 3 ? (p.c & (B - 1)) : 0);
            const unsigned support = t == 0.0 ? P - 1 : P;  // open: no weight at distance P/2
            double* const to = mine + (role < 2 ? role * (P / 2) : P + (role - 2) * kPatch);
            auto put = [&](int l, double w) {
                if (l < P / 2 || role >= 2) to[l] = w * p.f0;  // (times 1 for the x and y weights)
                if (role == 3) {
                    to[kPatch + l] = w * p.f1;
                    to[2 * kPatch + l] = w * p.f2;
                }
            };
            if (!wa.kb) {
                // w(u + 1) = w(u) exp(-beta (2u + 1)) from u0, the distance of offset j0
                const double u0 = (double)(j0 - (P / 2 - 1)) - t;
                double w = exp(-wa.beta * u0 * u0);
                double r = exp(-wa.beta * (2.0 * u0 + 1.0));
#pragma unroll
                for (int l = 0; l < kPatch; ++l) {
                    put(l, (unsigned)(j0 + l) < support ? w : 0.0);
                    w *= r;
                    r *= e2;
                }
            } else {
#pragma unroll
                for (int l = 0; l < kPatch; ++l) {
                    const int j = j0 + l;
                    if (l < P / 2 || role >= 2)
                        put(l, (unsigned)j < support ? window_weight_one<double, P>(j, t, wa) : 0.0);
                }
            }
        };

        if (all > 0) {
            locate(0);
            fetch();
        }
        int base = 0;
        for (int sa = 0; sa < wn; sa += kSlabs) {
            int end[kSlabs];
#pragma unroll
            for (int k = 0; k < kSlabs; ++k) end[k] = __builtin_amdgcn_readlane(ends, sa + k);
            while (base < end[kSlabs - 1]) {
                const int cnt = min(kBatch, end[kSlabs - 1] - base);
                locate(base + cnt);
                stage();
                wave_lds_sync();
                fetch();
                // single-value LDS loads (a paired load occupies the LDS pipeline twice as long), those of
                // particle q + 1 ahead of the sums of particle q
                const double* r = row0;
                double nx = ld1(r[lane & 15]), ny = ld1(r[P + ly]);
                double n0 = ld1(r[P + kPatch + lz]), n1 = ld1(r[P + 2 * kPatch + lz]), n2 = ld1(r[P + 3 * kPatch + lz]);
                int q = 0;
#pragma unroll
                for (int k = 0; k < kSlabs; ++k)
                    for (const int qe = min(cnt, end[k] - base); q < qe; ++q) {
                        const double w = nx;
                        const double g0 = ny * n0, g1 = ny * n1, g2 = ny * n2;
                        r = row0 + min(q + 1, kBatch - 1) * kRow;
                        nx = ld1(r[lane & 15]);
                        ny = ld1(r[P + ly]);
                        n0 = ld1(r[P + kPatch + lz]);
                        n1 = ld1(r[P + 2 * kPatch + lz]);
                        n2 = ld1(r[P + 3 * kPatch + lz]);
                        spread<0, P>(acc + k, w, g0, g1, g2);
                    }
                base += cnt;
                wave_lds_sync();
            }
            merge();
            const int at = sb + sa + wid;  // point of the segment
            if constexpr (Fold) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if (at & kWaves) folded[1][c] += v[c];
                    else folded[0][c] += v[c];
                }
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if (at < hk) (head + ((int64_t)at * 3 + c) * m23)[line] = v[c];
                    else (grid + (c * nc + (int64_t)(x0 - P / 2 + 1 + at) * m23))[line] = (TG)v[c];
                }
            }
        }
    }
    // the points past the segment's slabs
#pragma unroll
    for (int i = 0; i * kSlabs < P - 1; ++i) {
        merge();
        const int p = i * kSlabs + wid;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if constexpr (Fold) folded[i & 1][c] += v[c];  // (point 8 + p)
            else if (p < hk) (tail + ((int64_t)p * 3 + c) * m23)[line] = v[c];
        }
    }
    if constexpr (Fold) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int x = wrapi(wid + kWaves * i - P / 2 + 1, M1);
                (grid + (c * nc + (int64_t)x * m23))[line] = (TG)folded[i][c];
            }
    }
}

// The points next to the segment boundaries: grid(x0(s) - P/2 + 1 + k) = head[s][k] + tail[s-1][k]
// (periodic in s), for k < P - 1, every line and component; head and tail planes are laid out
// [segment][k][component][line].
template <typename TG>
__global__ __launch_bounds__(256) void k_p2g_halo_sum(const double* __restrict__ halo, int nseg, int seg, int P,
                                                      Geometry g, TG* __restrict__ grid, int64_t grid_stride,
                                                      int64_t halo_stride)
{
    halo += (int64_t)blockIdx.y * halo_stride;
    grid += (int64_t)blockIdx.y * grid_stride;
    const int64_t m23 = (int64_t)g.M[1] * g.M[2];
    const int64_t planes = (int64_t)nseg * (P - 1) * 3;
    const int64_t total = planes * m23;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t yz = i % m23, pl = i / m23;
        const int c = (int)(pl % 3), sk = (int)(pl / 3);
        const int k = sk % (P - 1), sg = sk / (P - 1);
        const int sp = (sg + nseg - 1) % nseg;
        const double v = halo[i] + halo[total + ((int64_t)(sp * (P - 1) + k) * 3 + c) * m23 + yz];
        const int x = wrapi(sg * seg - P / 2 + 1 + k, g.M[0]);
        grid[(int64_t)c * g.ncells + (int64_t)x * m23 + yz] = (TG)v;
    }
}


template <typename TG, int P>
hipError_t launch_p2g_t(const Plan& pl, const Work& w, hipStream_t s, bool st, int nsys, bool open)
{
    const Geometry& g = pl.g;
    const int npy = g.M[1] / kPatch, npz = g.M[2] / kPatch;
    const int seg = p2g_segment_length(g.M, P);
    const int nseg = g.M[0] / seg;
    const int blocks = nseg * npy * npz;
    // with halo planes every boundary point lies in exactly two segments; without (M1 = 8 < P, one
    // segment) the sweep folds its points
    double* halo = seg >= P ? w.p2g_halo : nullptr;
    const int64_t halo_n = (int64_t)nseg * (P - 1) * 3 * g.M[1] * g.M[2];
    const int fix_blocks = (int)std::min<int64_t>((halo_n + 255) / 256, 4096);
    // force (3 components); with stresslet sources also the 6 tensor components, three per sweep
    const int passes = st ? 3 : 1;
    const int64_t gstride = (int64_t)(st ? 9 : 3) * g.ncells, hstride = p2g_halo_elems(pl);
    for (int ps = 0; ps < passes; ++ps) {
        TG* grid = (TG*)w.grid + (int64_t)3 * ps * g.ncells;
        const double* sv = ps == 0 ? nullptr : w.srec;
        auto sweep = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(blocks, nsys), dim3(kWaves * kWave), 0, s, (const Rec64*)w.rec, w.start,
                               g, make_win_args<double>(pl), seg, npy, npz, sv, 3 * (ps - 1), grid, halo, gstride,
                               hstride);
        };
        if (halo) {
            sweep(k_p2g_sweep<TG, P, false>);
            if (open) continue;  // the first FFT pass adds them (the stresslet sweeps share one buffer)
            hipLaunchKernelGGL((k_p2g_halo_sum<TG>), dim3(fix_blocks, nsys), dim3(256), 0, s, (const double*)halo,
                               nseg, seg, P, g, grid, gstride, hstride);
        } else if constexpr (P > 8) {
            sweep(k_p2g_sweep<TG, P, true>);
        } else {
            return hipErrorInvalidValue;  // grids have at least 8 points: seg >= P
        }
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_p2g_p(const Plan& pl, const Work& w, hipStream_t s, bool st, int nsys, bool open)
{
    switch (pl.P) {
    case 4: return launch_p2g_t<T, 4>(pl, w, s, st, nsys, open);
    case 6: return launch_p2g_t<T, 6>(pl, w, s, st, nsys, open);
    case 8: return launch_p2g_t<T, 8>(pl, w, s, st, nsys, open);
    case 10: return launch_p2g_t<T, 10>(pl, w, s, st, nsys, open);
    case 12: return launch_p2g_t<T, 12>(pl, w, s, st, nsys, open);
    case 14: return launch_p2g_t<T, 14>(pl, w, s, st, nsys, open);
    case 16: return launch_p2g_t<T, 16>(pl, w, s, st, nsys, open);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int p2g_max_runs() { return kMaxRuns; }

// x-segment length of the sweep: halved while segments stay longer than 2P (the halo planes
// are then a small share of a segment's points) and the launch has fewer than 2048 blocks
// (measured: c3 P2G 10.3 -> 9.8 ms, c4 4.89 -> 4.76 ms against 4P and 1024 blocks)
int p2g_segment_length(const int M[3], int P)
{
    const int npy = M[1] / kPatch, npz = M[2] / kPatch;
    int seg = M[0];
    while (seg > 2 * P && (int64_t)(M[0] / seg) * npy * npz < 2048) seg >>= 1;
    return seg;
}

int64_t p2g_halo_elems(const Plan& pl)
{
    const int seg = p2g_segment_length(pl.g.M, pl.P);
    if (seg < pl.P) return 0;
    return 2 * (int64_t)(pl.g.M[0] / seg) * (pl.P - 1) * 3 * pl.g.M[1] * pl.g.M[2];
}

hipError_t launch_p2g(const Plan& pl, const Work& w, int n, hipStream_t s, bool st, int nsys, bool open)
{
    (void)n;
    if (pl.grid64) return launch_p2g_p<double>(pl, w, s, st, nsys, open);
    return launch_p2g_p<float>(pl, w, s, st, nsys, open);
}

}  // namespace ewald
