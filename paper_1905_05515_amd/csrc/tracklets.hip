// Kalman-filter tracklet construction, one lane per chain start (the
// arithmetic is in tracklet_dev.hpp).
#include "block_dev.hpp"
#include "tracklet_dev.hpp"

#include <atomic>

namespace tpc {

// Lanes of a wave that take a start, for `count` starts and `slots` waves
// (two per compute unit, half the SIMDs).  A wave's step runs every path
// that one of its lanes takes (the window search above all), so fewer starts
// to a wave end sooner while SIMDs are free; events in flight on other
// streams want those SIMDs too.  Alone, 1,976 starts took 482 / 462 / 410 us
// over 256 / 1024 / 2048 waves, a central event's 37,203 starts 612 us with
// 64 to a wave, 593 us with 37, 654 us with 19; three such events in flight
// took 228 / 214 / 269 us each with 256 / 512 / 2048 slots, and three
// central events 471 / 471 / 512 us with 256 / 512 / 1024.
__device__ __forceinline__ int wave_starts(int64_t count, int64_t slots)
{
    const int64_t per = (count + slots - 1) / slots;
    return per < kWave ? (int)per : kWave;
}

// One wave per group of consecutive starts, the waves dealt to the XCDs in
// contiguous ranges, so that the starts of one sector, and the grid rows
// they search, share an L2; waves that start together also walk the rows
// together.  What bounds it: few starts, the serial chain of the longest
// tracklet (a wave issues one VALU instruction per 4.3 cycles, ~355 per row
// of a lone chain lane, ~520 where lanes search, and waits a third of its
// time for the search's two dependent loads); many starts, VALU issue (on a
// 64-collision time frame, 3.0M starts, the SIMDs issue VALU 98% of the
// time; its sectors' starts are ordered, see below).  Walking the rows of a
// wave in step took 180,000 starts of 512 sector instances from 1386 to 930 us
// and the time frame's 23.1 to 12.6 ms (each lane at its own row fetched
// 5.2 GB past the L2s on the former); a form with the hit lists in LDS, a
// fifth of the waves in flight, was no faster on small events any more, nor
// was a queue form that refills idle lanes (27.4 ms on the time frame).
// 128 VGPRs hold four waves a SIMD (137, and three waves: 13.9 ms).
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void k_tracklets(
    const tpc_sector* __restrict__ sec, int n_rows, const float* __restrict__ row_x,
    tpc_params prm, const int32_t* __restrict__ bin_start, const float* __restrict__ yg,
    const float* __restrict__ zg, const int32_t* __restrict__ idg,
    const int32_t* __restrict__ gsr, const int32_t* __restrict__ up,
    const int32_t* __restrict__ starts, tpc_status* __restrict__ status,
    const int64_t* __restrict__ t_lo, const int64_t* __restrict__ t_hi, int64_t count_cap,
    int64_t cap, int64_t slots, const int32_t* __restrict__ ord, int32_t* __restrict__ t_start,
    int32_t* __restrict__ t_hits, int32_t* __restrict__ t_nhits, int32_t* __restrict__ t_rin, float* __restrict__ t_par,
    float* __restrict__ t_cov, float* __restrict__ t_chi2)
{
    __shared__ float4 keep[kKeepVec];
    extern __shared__ float xs[];          // n_rows row positions
    const int64_t lo = *t_lo < count_cap ? *t_lo : count_cap;
    const int64_t m = *t_hi < count_cap ? *t_hi : count_cap;
    if (m <= lo) return;
    const int L = wave_starts(m - lo, slots);
    const int64_t nb = (m - lo + L - 1) / L;
    if ((int64_t)blockIdx.x >= nb) return;
    for (int i = threadIdx.x; i < n_rows; i += blockDim.x) xs[i] = row_x[i];
    __syncthreads();
    int n_prop = 0, n_upd = 0, n_cand = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += gridDim.x) {
        const int64_t chunk = nb - b0 < (int64_t)gridDim.x ? nb - b0 : (int64_t)gridDim.x;
        if ((int64_t)blockIdx.x >= chunk) break;
        const int64_t q = lo + (b0 + xcd_remap(blockIdx.x, (int)chunk)) * L + threadIdx.x;
        build_tracklets((uint32_t)q, ord, (int)threadIdx.x < L && q < m, sec, n_rows, xs, prm,
                        bin_start, yg, zg, idg, gsr, up, starts, t_hits, cap,
                        keep + threadIdx.x, t_start, t_nhits, t_rin, t_par, t_cov, t_chi2,
                        n_prop, n_upd, n_cand);
    }
    add_work(status, n_prop, n_upd, n_cand);
}

// ---- processing order ---------------------------------------------------------
// The starts of big sectors are processed by z slab and start row: the lanes
// of a wave join and leave the walk together, and the waves in flight read
// one part of the sector's grid.  One block orders a group of at most
// kSortMax starts (a sector's starts in equal groups): a start's row and its
// quantile in the row's positions, which the grid orders by z, follow from
// its grid position and the sector's row boundaries alone; a counting sort
// over (slab, row) in LDS.  The order inside a bin is that of the atomics:
// nothing but the time depends on it.  ord[q]: the tracklet processed at slot
// q; inv[t]: the slot of tracklet t in its group.
//
// The tracklet kernel writes hit lists in processing order (its lanes' words
// of a row are one line; at their own columns they are scattered words: 17 ms
// for 12.6 on the time frame), and k_hits_unsort puts the rows of a
// group back in the order of the starts, whole in LDS as 16-bit offsets from
// the row's first position: sectors with a row of 65535 positions or more
// keep the order of the starts.
//
// Time frame, 3.0M starts of 36 sectors: 12.8 ms in the order of the starts;
// 8.65 + 0.10 to sort + 1.06 to put the lists back.  What bounds the kernel is
// VALU issue still (75,000 instructions a wave for 104,000), and 12.8 GB
// fetched for 38.5.  8192, 32768 starts a group: 9.9, 8.1 ms where whole
// sectors take 7.2 (columns in processing order throughout); 16, 32, 64
// slabs: 8.9, 8.65, 8.7.  A sector order with columns by group: 8.35, but
// 0.32 to sort.
constexpr int kSortMax = 65536;
constexpr int kSortSlabs = 32;
constexpr int kSortBlock = 1024;

// start range of group j of sector si (empty if there is none)
struct SortGroup {
    int64_t lo, hi;
};
__device__ __forceinline__ SortGroup sort_group(const int64_t* __restrict__ sec_start, int si,
                                                int j, int64_t count_cap)
{
    int64_t lo = sec_start[si], hi = sec_start[si + 1];
    if (hi > count_cap) hi = count_cap;
    if (lo > hi) lo = hi;
    const int64_t n = hi - lo, ng = (n + kSortMax - 1) / kSortMax;
    if (j >= ng) return {hi, hi};
    const int64_t len = (n + ng - 1) / ng;
    lo += j * len;
    return {lo, lo + len < hi ? lo + len : hi};
}

// Is the sector sorted?  (host and device; the rows' sizes on the device.)
// The line lies where the order pays for its two launches: a time frame of 4,
// 6, 8, 12 and 24 collisions (78,000 to 466,000 clusters a sector) takes
// 1.53, 2.96, 4.17, 6.78 and 13.3 ms without, 1.60, 2.93, 4.16, 6.53 and 12.6
// with it.
constexpr int64_t kSortClusters = int64_t(1) << 17;
__host__ __device__ inline bool sort_sector(const tpc_sector& s)
{
    return s.end - s.begin >= kSortClusters;
}

// rows[0..n_rows]: first grid position of every row; true if each fits
__device__ __forceinline__ bool sector_rows(const tpc_sector& s, int n_rows,
                                            const int32_t* __restrict__ bin_start, int* rows)
{
    const int per_row = s.nbz * s.nby;
    for (int r = threadIdx.x; r <= n_rows; r += blockDim.x)
        rows[r] = bin_start[s.bin_base + r * per_row];
    __syncthreads();
    bool fits = true;
    for (int r = threadIdx.x; r < n_rows; r += blockDim.x) fits &= rows[r + 1] - rows[r] < 65535;
    return __syncthreads_and(fits);
}

__global__ __launch_bounds__(kSortBlock) void k_start_sort(
    const tpc_sector* __restrict__ sec, int sec_lo, int groups, int n_rows,
    const int32_t* __restrict__ bin_start, const int32_t* __restrict__ starts,
    const int64_t* __restrict__ sec_start, int64_t count_cap, int32_t* __restrict__ ord,
    uint16_t* __restrict__ inv)
{
    __shared__ int rows[256 + 1];
    __shared__ int cnt[kSortSlabs * 256];
    __shared__ int part[kSortBlock / kWave];
    const int si = sec_lo + (int)(blockIdx.x / groups);
    const SortGroup g = sort_group(sec_start, si, (int)(blockIdx.x % groups), count_cap);
    if (g.lo >= g.hi) return;
    const tpc_sector s = sec[si];
    const bool sorted = sort_sector(s) && sector_rows(s, n_rows, bin_start, rows);
    if (!sorted) {
        for (int64_t t = g.lo + threadIdx.x; t < g.hi; t += blockDim.x) ord[t] = (int32_t)t;
        return;
    }
    const int nbin = kSortSlabs * n_rows;
    for (int k = threadIdx.x; k < nbin; k += blockDim.x) cnt[k] = 0;
    __syncthreads();
    // bin of a start: its row by bisection, its slab by its place in the row
    auto bin = [&](int h) {
        int lo = 0, hi = n_rows - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rows[mid] <= h) lo = mid; else hi = mid - 1;
        }
        const int slab = (h - rows[lo]) * kSortSlabs / (rows[lo + 1] - rows[lo]);
        return slab * n_rows + lo;
    };
    for (int64_t t = g.lo + threadIdx.x; t < g.hi; t += blockDim.x)
        atomicAdd(&cnt[bin(starts[t])], 1);
    __syncthreads();
    // exclusive scan of the counts: kPer consecutive bins a thread
    constexpr int kPer = kSortSlabs * 256 / kSortBlock;
    int v[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int b = (int)threadIdx.x * kPer + k;
        v[k] = b < nbin ? cnt[b] : 0;
        sum += v[k];
    }
    const int x = wave_incl_scan(sum);
    const int wid = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) part[wid] = x;
    __syncthreads();
    int at = x - sum;
    for (int w = 0; w < wid; ++w) at += part[w];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int b = (int)threadIdx.x * kPer + k;
        if (b < nbin) cnt[b] = at;
        at += v[k];
    }
    __syncthreads();
    for (int64_t t = g.lo + threadIdx.x; t < g.hi; t += blockDim.x) {
        const int slot = atomicAdd(&cnt[bin(starts[t])], 1);
        ord[g.lo + slot] = (int32_t)t;
        inv[t] = (uint16_t)slot;
    }
}

// Each item a (group, row): the row's entries of the group's tracklets, in
// processing order on entry, in the order of the starts on exit.  The groups
// are counted on the device (a sector has up to a third of its clusters in
// starts, and a fifth of that number is usual), and blocks take items in turn.
__global__ __launch_bounds__(kSortBlock) void k_hits_unsort(
    const tpc_sector* __restrict__ sec, int sec_lo, int n_sec, int n_rows,
    const int32_t* __restrict__ bin_start, const int64_t* __restrict__ sec_start,
    int64_t count_cap, const uint16_t* __restrict__ inv, int32_t* t_hits, int64_t cap)
{
    __shared__ uint16_t off[kSortMax];
    __shared__ int rows[256 + 1];
    __shared__ int groups;
    if (threadIdx.x == 0) groups = 0;
    __syncthreads();
    for (int k = threadIdx.x; k < n_sec; k += blockDim.x) {
        const int64_t n = sec_start[sec_lo + k + 1] - sec_start[sec_lo + k];
        if (n > 0 && sort_sector(sec[sec_lo + k]))
            atomicMax(&groups, (int)((n + kSortMax - 1) / kSortMax));
    }
    __syncthreads();
    const int64_t items = (int64_t)groups * n_sec * n_rows;
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int r = (int)(it % n_rows);
        const int si = sec_lo + (int)(it / n_rows % n_sec);
        const SortGroup g = sort_group(sec_start, si, (int)(it / n_rows / n_sec), count_cap);
        if (g.lo >= g.hi) continue;
        const tpc_sector s = sec[si];
        if (!sort_sector(s) || !sector_rows(s, n_rows, bin_start, rows)) continue;
        const int n = (int)(g.hi - g.lo), p0 = rows[r];
        int32_t* row = t_hits + r * cap + g.lo;
        constexpr int kU = 8;
        for (int i0 = threadIdx.x; i0 < n; i0 += kU * kSortBlock) {
            int h[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u)
                h[u] = i0 + u * kSortBlock < n ? row[i0 + u * kSortBlock] : -1;
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (i0 + u * kSortBlock < n)
                    off[i0 + u * kSortBlock] = h[u] < 0 ? 0xFFFFu : (uint16_t)(h[u] - p0);
        }
        __syncthreads();
        for (int i0 = threadIdx.x; i0 < n; i0 += kU * kSortBlock) {
            int k[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u)
                k[u] = i0 + u * kSortBlock < n ? inv[g.lo + i0 + u * kSortBlock] : 0;
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int o = off[k[u]];
                if (i0 + u * kSortBlock < n)
                    row[i0 + u * kSortBlock] = o == 0xFFFF ? -1 : p0 + o;
            }
        }
        __syncthreads();   // off and rows are the next item's
    }
}

// waves the starts of a small event are dealt to: two per compute unit of
// the current device (kept per device: the query is not free and the
// per-sector form asks once per sector)
static int64_t tracklet_slots()
{
    constexpr int kDevs = 16;
    static std::atomic<int64_t> cache[kDevs];
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 512;
    if (dev >= 0 && dev < kDevs && cache[dev].load() > 0) return cache[dev].load();
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 512;
    const int64_t v = (int64_t)n_cu * 2;
    if (dev >= 0 && dev < kDevs) cache[dev].store(v);
    return v;
}

// Tracklets of the starts of sectors [sec_lo, sec_hi) (the start range that
// run_find_neighbours recorded for them).
int run_construct_tracklets(const tpc_problem* p, int sec_lo, int sec_hi, tpc_grid grid_,
                            tpc_links links, tpc_starts starts, tpc_tracklets trl,
                            const Workspace& ws, hipStream_t st)
{
    // tracklets processed: bounded by both capacities; the hit array's row
    // stride is the tracklet capacity
    const int64_t count_cap = starts.capacity < trl.capacity ? starts.capacity : trl.capacity;
    const int64_t bound = (p->h_sectors[sec_hi - 1].end - p->h_sectors[sec_lo].begin) / 3 + 1;
    const int64_t n_launch = bound < count_cap ? bound : count_cap;
    // the most waves any count up to the bound is dealt to, capped: empty
    // waves cost their launch (65,536 of them 15 us)
    const int64_t slots = tracklet_slots();
    const int64_t few = n_launch < slots ? n_launch : slots;
    int64_t g = ceil_div(n_launch, kWave);
    g = g < few ? few : g;
    g = g < 1 ? 1 : g > 65536 ? 65536 : g;
    // the processing order, where big sectors hold half of the clusters (the
    // sort and the way back visit every sector); the arrays of the
    // selection's lengths hold it meanwhile
    int64_t big = 0, in_big = 0;
    for (int i = sec_lo; i < sec_hi; ++i) {
        const tpc_sector& s = p->h_sectors[i];
        if (!sort_sector(s)) continue;
        in_big += s.end - s.begin;
        if (s.end - s.begin > big) big = s.end - s.begin;
    }
    if (in_big * 2 < p->h_sectors[sec_hi - 1].end - p->h_sectors[sec_lo].begin) big = 0;
    const int groups = (int)ceil_div(big / 3 + 1, kSortMax);
    int32_t* ord = big ? reinterpret_cast<int32_t*>(ws.tlen) : nullptr;
    uint16_t* inv = reinterpret_cast<uint16_t*>(ws.toff);
    const int64_t n_groups = (int64_t)(sec_hi - sec_lo) * groups;
    if (ord)
        TPC_LAUNCH(k_start_sort, dim3((unsigned)n_groups), dim3(kSortBlock), 0, st, p->d_sectors,
                   sec_lo, groups, p->n_rows, (const int32_t*)grid_.bin_start,
                   (const int32_t*)starts.pos, (const int64_t*)ws.sec_start, count_cap, ord, inv);
    TPC_LAUNCH(k_tracklets, dim3((unsigned)g), dim3(kWave), sizeof(float) * p->n_rows, st,
               p->d_sectors, p->n_rows, p->d_row_x, p->params, (const int32_t*)grid_.bin_start,
               (const float*)grid_.y, (const float*)grid_.z, (const int32_t*)grid_.id,
               (const int32_t*)ws.gsr, (const int32_t*)links.up, (const int32_t*)starts.pos,
               ws.status, (const int64_t*)(ws.sec_start + sec_lo),
               (const int64_t*)(ws.sec_start + sec_hi), count_cap, trl.capacity, slots,
               (const int32_t*)ord, trl.start, trl.hits, trl.nhits, trl.row_inner, trl.par,
               trl.cov, trl.chi2);
    if (ord)
        TPC_LAUNCH(k_hits_unsort, dim3(grid_for_block(n_groups * p->n_rows, 1, 1024)),
                   dim3(kSortBlock), 0, st, p->d_sectors, sec_lo, sec_hi - sec_lo, p->n_rows, (const int32_t*)grid_.bin_start,
                   (const int64_t*)ws.sec_start, count_cap, (const uint16_t*)inv, trl.hits,
                   trl.capacity);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}

}  // namespace tpc
