// Bin / sort stage: counting sort of the particles by grid cell (tile-major key), the
// cell list every other kernel reads (Sec. 3: cell lists of the near and far field; here
// one compact CSR list keyed by grid cell serves both, since P2P cells are unions of grid
// cells).  Integer atomics touch only the per-cell counters; the order inside a cell is
// made deterministic by sorting it by original index.
#include <algorithm>
#include <climits>

#include "internal.h"

namespace ewald {

namespace {

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;                          // consecutive elements per thread: 16-byte accesses
constexpr int kScanChunk = kScanThreads * kScanItems;  // elements per block
constexpr int kScanDirect = 4096;   // up to so many block sums every block adds those before it itself
constexpr int kTilesDirect = 32768; // up to so many tiles one block scans the P2P work list

__global__ void k_fill_i32(int* __restrict__ p, int64_t count, int value)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = i; k < count; k += stride) p[k] = value;
}

// count[0..ncells) = 0, and the lengths of the sort's two lists
__global__ void k_clear(int* __restrict__ count, int ncells, int* __restrict__ lists)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    for (int k = i; k < ncells / 4; k += stride) reinterpret_cast<int4*>(count)[k] = int4{0, 0, 0, 0};
    if (i < 2) lists[i] = 0;
}

// Periodic wrap into [0, L) and grid cell / fraction along one axis: c = floor(y/h),
// t = y/h - c.  The same function is used wherever a particle's cell is needed.
__device__ inline void cell_of(double x, double L, double h, int M, int& c, double& t, double& w)
{
    w = x - L * floor(x / L);
    if (w >= L) w -= L;
    if (w < 0.0) w = 0.0;
    const double s = w / h;
    int ci = (int)floor(s);
    if (ci >= M) ci = M - 1;
    if (ci < 0) ci = 0;
    c = ci;
    t = s - (double)ci;
}

// key = system * ncells + cell key: the systems of a batch occupy consecutive key ranges.  rank: the
// particle's (arbitrary) place among those of its cell, so that the scatter needs no second counter.
__global__ void k_bin(int n, const double* __restrict__ x, Geometry g, int* __restrict__ key,
                      int* __restrict__ rank, int* __restrict__ count, Batch b)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int c[3];
    double t, wx;
#pragma unroll
    for (int d = 0; d < 3; ++d) cell_of(x[(int64_t)d * n + i], g.L[d], g.h[d], g.M[d], c[d], t, wx);
    const int k = batch_system(b, i) * g.ncells + cell_key(c[0], c[1], c[2], g);
    key[i] = k;
    rank[i] = atomicAdd(&count[k], 1);
}

__global__ void k_scatter(int n, const int* __restrict__ key, const int* __restrict__ rank,
                          const int* __restrict__ start, int* __restrict__ perm, double* __restrict__ u_near)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    perm[start[key[i]] + rank[i]] = i;
    // the near field that the symmetric P2P adds to
    u_near[i] = 0.0;
    u_near[(int64_t)n + i] = 0.0;
    u_near[2 * (int64_t)n + i] = 0.0;
}

// The order inside a cell is by original index, so that the sorted order (and every sum taken in it)
// does not depend on the order of the scatter's atomics.  In cells of up to kCellSerial particles the
// gather counts the smaller indices of each particle's cell; larger cells are appended to one of two
// lists by the scan (`lists[0]`, `lists[1]` hold their lengths) and their indices sorted, by one
// wavefront per cell up to kCellMid particles, by one block per cell above.  The lists' order varies,
// but each cell's result does not.
constexpr int kCellSerial = 16;
constexpr int kCellMid = 256;
constexpr int kBigThreads = 256;
constexpr int kBigRun = 4096;  // ints sorted in LDS at once (two buffers of 16 KB)

__host__ __device__ inline int64_t mid_list_cap(int64_t n) { return n / (kCellSerial + 1) + 1; }
__host__ __device__ inline int64_t big_list_cap(int64_t n) { return n / (kCellMid + 1) + 1; }

// One wavefront per listed cell (kCellSerial < size <= kCellMid): every lane holds up to
// four of the cell's (distinct) indices, counts how many of the cell's indices are smaller
// (a broadcast read of each from LDS) and writes its index at that rank.
__device__ void sort_mid_cells(const int* __restrict__ start, int* __restrict__ perm,
                               const int* __restrict__ lists, int* sh, int block, int blocks)
{
    constexpr int kPer = kCellMid / kWave;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    int* s = sh + wv * kCellMid;
    const int nmid = lists[0];
    const int waves = blocks * (blockDim.x / kWave);
    for (int q = block * (blockDim.x / kWave) + wv; q < nmid; q += waves) {
        const int c = lists[2 + q];
        const int a = start[c], m = start[c + 1] - a;
        int v[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = lane + k * kWave;
            v[k] = i < m ? perm[a + i] : 0;
            s[i] = i < m ? v[k] : INT_MAX;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int rank[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) rank[k] = 0;
        for (int t = 0; t < m; t += 8) {
            const int4 o = *reinterpret_cast<const int4*>(s + t), p = *reinterpret_cast<const int4*>(s + t + 4);
#pragma unroll
            for (int k = 0; k < kPer; ++k)
                rank[k] += (o.x < v[k]) + (o.y < v[k]) + (o.z < v[k]) + (o.w < v[k]) + (p.x < v[k]) + (p.y < v[k]) +
                           (p.z < v[k]) + (p.w < v[k]);
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (lane + k * kWave < m) perm[a + rank[k]] = v[k];
        // the next cell overwrites this wave's LDS row
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// number of entries of the ascending, distinct a[0..len) below v
__device__ inline int count_below(const int* __restrict__ a, int len, int v)
{
    int lo = 0, hi = len;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One pass of a merge sort in LDS: src[0, len) holds ascending runs of w (distinct values), dst gets runs
// of 2 w.  Each value goes to its offset in its own run plus the number of smaller values in the other,
// found by halving steps; a thread searches for eight values at a time, whose reads overlap.
__device__ inline void merge_runs(const int* src, int* dst, int len, int w)
{
    constexpr int kSide = 8;
    for (int i0 = threadIdx.x; i0 < len; i0 += kSide * kBigThreads) {
        int val[kSide], at[kSide], other[kSide], n[kSide], pos[kSide];
#pragma unroll
        for (int q = 0; q < kSide; ++q) {
            const int i = min(i0 + q * kBigThreads, len - 1);
            const int lo = i & ~(2 * w - 1), mid = min(lo + w, len), hi = min(lo + 2 * w, len);
            val[q] = src[i];
            at[q] = i < mid ? i : lo + i - mid;  // plus pos: its place
            other[q] = i < mid ? mid : lo;
            n[q] = i < mid ? hi - mid : mid - lo;
            pos[q] = 0;
        }
        for (int step = w; step >= 1; step >>= 1) {
#pragma unroll
            for (int q = 0; q < kSide; ++q) {
                const int to = pos[q] + step;
                const int o = src[min(other[q] + to, len) - 1];
                pos[q] = (to <= n[q]) & (o < val[q]) ? to : pos[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kSide; ++q)
            if (i0 + q * kBigThreads < len) dst[at[q] + pos[q]] = val[q];
    }
    __syncthreads();
}

// One block per listed cell (size > kCellMid): runs of kBigRun indices are sorted in LDS (runs of 64
// by counting, one per wave and turn, then merged pairwise: 2e4 particles in two clusters, cells of up to
// 1.8e3, 64 us by a bitonic network and 23 us so), then merged pairwise, each index placed at
// its rank in the merged run (its offset in its own run plus the count of smaller indices
// in the other, by binary search), ping-ponging between the cell's range of `perm` and
// the same range of `scratch`.
__device__ void sort_big_cells(const int* __restrict__ start, int* __restrict__ perm, int* __restrict__ scratch,
                               const int* __restrict__ lists, int64_t mid_cap, int* s, int block, int blocks)
{
    const int nbig = lists[1];
    const int tid = threadIdx.x;
    for (int q = blocks - 1 - block; q < nbig; q += blocks) {  // from the last block on: the first have the others
        const int c = lists[2 + mid_cap + q];
        const int a = start[c], m = start[c + 1] - a;
        int* v = perm + a;
        for (int r0 = 0; r0 < m; r0 += kBigRun) {
            const int len = min(kBigRun, m - r0);
            for (int i = tid; i < len; i += kBigThreads) s[i] = v[r0 + i];
            __syncthreads();
            const int lane = tid & (kWave - 1);
            for (int b = tid - lane; b < len; b += kBigThreads) {
                const int val = b + lane < len ? s[b + lane] : INT_MAX;
                int below = 0;
#pragma unroll
                for (int k = 0; k < kWave; ++k) below += __builtin_amdgcn_readlane(val, k) < val ? 1 : 0;
                wave_lds_sync();
                if (b + lane < len) s[b + below] = val;
            }
            __syncthreads();
            int *from = s, *to = s + kBigRun;
            for (int w = kWave; w < len; w *= 2) {
                merge_runs(from, to, len, w);
                int* t = from;
                from = to;
                to = t;
            }
            for (int i = tid; i < len; i += kBigThreads) v[r0 + i] = from[i];
            __syncthreads();
        }
        int* src = v;
        int* dst = scratch + a;
        for (int w = kBigRun; w < m; w *= 2) {
            for (int i = tid; i < m; i += kBigThreads) {
                const int lo = (i / (2 * w)) * (2 * w);
                const int mid = min(lo + w, m), hi = min(lo + 2 * w, m);
                const int val = src[i];
                const int pos = (i < mid) ? (i - lo) + count_below(src + mid, hi - mid, val)
                                          : (i - mid) + count_below(src + lo, mid - lo, val);
                dst[lo + pos] = val;
            }
            __syncthreads();
            int* t = src;
            src = dst;
            dst = t;
        }
        if (src != v) {
            for (int i = tid; i < m; i += kBigThreads) v[i] = src[i];
        }
        __syncthreads();
    }
}

// Records in sorted order.  The sorted position of particle i is its cell's start plus the number of
// smaller indices in the cell (counted where cells are small, by binary search where they have been
// sorted); key[i] takes it, for k_gather_st.  The caller's (3, N) arrays are read in their own order
// (coalesced) and each whole record is written to its sorted position; gathering through perm instead
// reads six arrays at random positions, which costs a full memory segment per 8-byte value (15 times
// the bytes used at 1e6 uniform particles).
__global__ void k_gather64(int n, const double* __restrict__ x, const double* __restrict__ f,
                           const int* __restrict__ start, const int* __restrict__ perm, int* __restrict__ key,
                           Geometry g, Rec64* __restrict__ rec)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Rec64 r;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double t;
        cell_of(x[(int64_t)d * n + i], g.L[d], g.h[d], g.M[d], r.c[d], t, r.x[d]);
        r.f[d] = f[(int64_t)d * n + i];
    }
    r.orig = i;
    const int k = key[i], a = start[k], m = start[k + 1] - a;
    int pos = a;
    if (m > kCellSerial) {
        pos += count_below(perm + a, m, i);
    } else if (m > 1) {
        for (int j = 0; j < m; ++j) pos += perm[a + j] < i ? 1 : 0;
    }
    key[i] = pos;
    rec[pos] = r;
}

// Symmetric part of each stresslet source tensor q n^T, in sorted order: the stresslet
// kernel is symmetric in all three indices, so only (q n^T + n q^T)/2 contributes.
__global__ void k_gather_st(int n, const double* __restrict__ q, const double* __restrict__ nrm,
                            const int* __restrict__ inv, double* __restrict__ srec)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double q0 = q[i], q1 = q[(int64_t)n + i], q2 = q[2 * (int64_t)n + i];
    const double n0 = nrm[i], n1 = nrm[(int64_t)n + i], n2 = nrm[2 * (int64_t)n + i];
    double* o = srec + 6 * (int64_t)inv[i];
    o[0] = q0 * n0;
    o[1] = q1 * n1;
    o[2] = q2 * n2;
    o[3] = 0.5 * (q0 * n1 + q1 * n0);
    o[4] = 0.5 * (q0 * n2 + q2 * n0);
    o[5] = 0.5 * (q1 * n2 + q2 * n1);
}

// ---- exclusive scan (block sums, scan of sums where there are many, block scans) ----

__device__ inline int block_exclusive_scan(int v, int* sh, int& total)
{
    // inclusive scan within each wave
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    const int inc = wave_scan(v);
    if (lane == kWave - 1) sh[wid] = inc;
    __syncthreads();
    const int nw = blockDim.x / kWave;
    int off = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        const int s = sh[k];
        if (k < wid) off += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return off + inc - v;
}

// a thread's kScanItems consecutive elements (0 past the end); the arrays are 256-byte aligned
__device__ inline int4 scan_load(const int* __restrict__ in, int i, int count)
{
    if (i + 3 < count) return *reinterpret_cast<const int4*>(in + i);
    int4 v = {0, 0, 0, 0};
    if (i < count) v.x = in[i];
    if (i + 1 < count) v.y = in[i + 1];
    if (i + 2 < count) v.z = in[i + 2];
    return v;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(const int* __restrict__ in, int count,
                                                              int* __restrict__ part)
{
    __shared__ int sh[kScanThreads / kWave];
    const int4 v = scan_load(in, blockIdx.x * kScanChunk + threadIdx.x * kScanItems, count);
    int total;
    block_exclusive_scan(v.x + v.y + v.z + v.w, sh, total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Single block: exclusive scan of part[0..nb) in place; part[nb] = grand total.
__global__ void k_scan_parts(int* __restrict__ part, int nb)
{
    __shared__ int sh[1024 / kWave];
    const int per = (nb + blockDim.x - 1) / blockDim.x;
    const int a = threadIdx.x * per;
    int s = 0;
    for (int k = 0; k < per; ++k)
        if (a + k < nb) s += part[a + k];
    int total;
    int off = block_exclusive_scan(s, sh, total);
    for (int k = 0; k < per; ++k)
        if (a + k < nb) {
            const int v = part[a + k];
            part[a + k] = off;
            off += v;
        }
    if (threadIdx.x == 0) part[nb] = total;
}

// Direct: part holds the block sums themselves, and every block adds those before it (a launch less);
// otherwise their exclusive scan.  lists (or null): the cells of more than kCellSerial elements are
// appended to the sort's lists.
template <bool Direct>
__global__ void __launch_bounds__(kScanThreads) k_scan_final(const int* __restrict__ in, int count,
                                                             const int* __restrict__ part, int* __restrict__ out,
                                                             int* __restrict__ lists, int64_t mid_cap)
{
    __shared__ int sh[kScanThreads / kWave];
    const int base = blockIdx.x * kScanChunk + threadIdx.x * kScanItems;
    const int4 v = scan_load(in, base, count);
    int before = 0;
    if (Direct) {
        int s = 0;
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += kScanThreads) s += part[k];
        block_exclusive_scan(s, sh, before);
    } else {
        before = part[blockIdx.x];
    }
    int total;
    const int off = block_exclusive_scan(v.x + v.y + v.z + v.w, sh, total) + before;
    const int4 o = {off, off + v.x, off + v.x + v.y, off + v.x + v.y + v.z};
    if (base + 3 < count) {
        *reinterpret_cast<int4*>(out + base) = o;
    } else {
        if (base < count) out[base] = o.x;
        if (base + 1 < count) out[base + 1] = o.y;
        if (base + 2 < count) out[base + 2] = o.z;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[count] = before + total;
    if (lists && max(max(v.x, v.y), max(v.z, v.w)) > kCellSerial) {
        const int m[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (m[k] > kCellMid) lists[2 + mid_cap + atomicAdd(&lists[1], 1)] = base + k;
            else if (m[k] > kCellSerial) lists[2 + atomicAdd(&lists[0], 1)] = base + k;
        }
    }
}

// Number of 64-target chunks of a P2P tile (the tiles of all systems).
__device__ inline int tile_chunks(const Geometry& g, const int* __restrict__ start, int t)
{
    const int per = 1 << (3 * g.log2B);
    return (start[(t + 1) * per] - start[t * per] + kWave - 1) / kWave;
}

__global__ void k_tile_chunks(Geometry g, const int* __restrict__ start, int* __restrict__ chunks)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < g.ntiles * g.nsys) chunks[t] = tile_chunks(g, start, t);
}

// Index order of the listed cells, and in block 0 the P2P work list (chunk_off: the exclusive scan of
// the tiles' chunks; null where other kernels make it): one launch for what only waits for the
// scatter.  `scratch` is the merge buffer of the largest cells.
__global__ void __launch_bounds__(kBigThreads) k_order_cells(const int* __restrict__ start, int* __restrict__ perm,
                                                             int* __restrict__ scratch, const int* __restrict__ lists,
                                                             int64_t mid_cap, Geometry g, int* __restrict__ chunk_off)
{
    __shared__ __align__(16) int s[2 * kBigRun];
    static_assert(kBigRun >= kBigThreads / kWave * kCellMid, "one LDS row per wave");
    if (blockIdx.x == 0) {
        if (!chunk_off) return;
        const int nt = g.ntiles * g.nsys;
        int before = 0;
        for (int t0 = 0; t0 < nt; t0 += 4 * kBigThreads) {
            const int t = t0 + 4 * threadIdx.x;
            int v[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = t + k < nt ? tile_chunks(g, start, t + k) : 0;
                sum += v[k];
            }
            int total;
            int off = before + block_exclusive_scan(sum, s, total);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (t + k < nt) chunk_off[t + k] = off;
                off += v[k];
            }
            before += total;
        }
        if (threadIdx.x == 0) chunk_off[nt] = before;
        return;
    }
    const int block = blockIdx.x - 1, blocks = gridDim.x - 1;
    sort_mid_cells(start, perm, lists, s, block, blocks);
    __syncthreads();
    sort_big_cells(start, perm, scratch, lists, mid_cap, s, block, blocks);
}

inline int blocks_for(int64_t n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

int scan_part_elems(int count) { return (count + kScanChunk - 1) / kScanChunk + 1; }

int64_t cell_list_elems(int64_t n) { return 2 + mid_list_cap(n) + big_list_cap(n); }

hipError_t launch_fill_i32(int* p, int64_t count, int value, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    int blocks = (int)((count + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, s, p, count, value);
    return hipGetLastError();
}

namespace {

__global__ void k_count_nonfinite(const double* __restrict__ a, int64_t count, int* __restrict__ out)
{
    int bad = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
        bad += isfinite(a[i]) ? 0 : 1;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) bad += __shfl_xor(bad, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0 && bad) atomicAdd(out, bad);
}

}  // namespace

hipError_t launch_count_nonfinite(const double* a, int64_t count, int* out, hipStream_t s, bool reset)
{
    if (reset) {
        hipError_t e = launch_fill_i32(out, 1, 0, s);
        if (e != hipSuccess) return e;
    }
    const int blocks = (int)std::min<int64_t>(1024, std::max<int64_t>(1, (count + 255) / 256));
    hipLaunchKernelGGL(k_count_nonfinite, dim3(blocks), dim3(256), 0, s, a, count, out);
    return hipGetLastError();
}

// Exclusive scan of in[0..count) into out[0..count] (out[count] = total); see k_scan_final
static void launch_scan(const int* in, int* out, int count, int* part, int* lists, int64_t mid_cap, hipStream_t s)
{
    const int nb = (count + kScanChunk - 1) / kScanChunk;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanThreads), 0, s, in, count, part);
    if (nb <= kScanDirect) {
        hipLaunchKernelGGL((k_scan_final<true>), dim3(nb), dim3(kScanThreads), 0, s, in, count, part, out, lists,
                           mid_cap);
    } else {
        hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(1024), 0, s, part, nb);
        hipLaunchKernelGGL((k_scan_final<false>), dim3(nb), dim3(kScanThreads), 0, s, in, count, part, out, lists,
                           mid_cap);
    }
}

// Seven launches: clear, bin, two for the scan, scatter, order (with the P2P work list), gather.  Small
// evaluations are bound by launches (about 4.5 us each behind one another).
hipError_t launch_sort(const Plan& pl, const Work& w, int n, const double* x, const double* f,
                       const Batch& b, hipStream_t s)
{
    Geometry g = pl.g;
    g.nsys = b.count;
    const int ncells = g.ncells * g.nsys, ntiles = g.ntiles * g.nsys;  // over all systems
    int* rank = (int*)w.rec;  // the records come last
    const int64_t mid_cap = mid_list_cap(n);
    const int clear_blocks = (int)std::min<int64_t>(65536, blocks_for(ncells, 1024));
    hipLaunchKernelGGL(k_clear, dim3(clear_blocks), dim3(256), 0, s, w.count, ncells, w.cell_lists);
    hipLaunchKernelGGL(k_bin, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, x, g, w.key, rank, w.count, b);
    launch_scan(w.count, w.start, ncells, w.part, w.cell_lists, mid_cap, s);
    hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, w.key, rank, w.start, w.perm,
                       w.u_near);
    // the rank array is free after the scatter and serves as the merge buffer of the largest cells
    const bool direct = ntiles <= kTilesDirect;
    const int order_blocks = 1 + (int)std::min<int64_t>(2048, std::max<int64_t>(1, mid_list_cap(n) / 4));
    hipLaunchKernelGGL(k_order_cells, dim3(order_blocks), dim3(kBigThreads), 0, s, w.start, w.perm, rank,
                       w.cell_lists, mid_cap, g, direct ? w.chunk_off : nullptr);
    hipLaunchKernelGGL(k_gather64, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, x, f, w.start, w.perm, w.key, g,
                       (Rec64*)w.rec);
    if (!direct) {
        hipLaunchKernelGGL(k_tile_chunks, dim3(blocks_for(ntiles, 256)), dim3(256), 0, s, g, w.start, w.count);
        launch_scan(w.count, w.chunk_off, ntiles, w.part, nullptr, 0, s);
    }
    return hipGetLastError();
}

hipError_t launch_gather_st(const Plan& pl, const Work& w, int n, const double* q, const double* nrm,
                            hipStream_t s)
{
    (void)pl;
    hipLaunchKernelGGL(k_gather_st, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, q, nrm, w.key, w.srec);
    return hipGetLastError();
}

}  // namespace ewald
