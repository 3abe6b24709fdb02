// Kalman-filter tracklet construction, one lane per chain start (the
// arithmetic is in tracklet_dev.hpp).
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
// time).  Walking the rows of a wave in step took 180,000 starts of
// 512 sector instances from 1386 to 930 us and the time frame's 23.1 to 12.6 ms
// (each lane at its own row fetched 5.2 GB past the L2s on the former); a form
// with the hit lists in LDS, a fifth of the waves in flight, was no faster
// on small events any more, nor was a queue form that refills idle lanes
// (27.4 ms on the time frame).  Starts sorted by z or by row inside tiles
// made the hit list stores scattered words: 17 ms on the time frame.
// 128 VGPRs hold four waves a SIMD (137, and three waves: 13.9 ms).
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void k_tracklets(
    const tpc_sector* __restrict__ sec, int n_rows, const float* __restrict__ row_x,
    tpc_params prm, const int32_t* __restrict__ bin_start, const float* __restrict__ yg,
    const float* __restrict__ zg, const int32_t* __restrict__ idg,
    const int32_t* __restrict__ gsr, const int32_t* __restrict__ up,
    const int32_t* __restrict__ starts, tpc_status* __restrict__ status,
    const int64_t* __restrict__ t_lo, const int64_t* __restrict__ t_hi, int64_t count_cap,
    int64_t cap, int64_t slots, int32_t* __restrict__ t_start, int32_t* __restrict__ t_hits,
    int32_t* __restrict__ t_nhits, int32_t* __restrict__ t_rin, float* __restrict__ t_par,
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
        const int64_t t = lo + (b0 + xcd_remap(blockIdx.x, (int)chunk)) * L + threadIdx.x;
        build_tracklets((uint32_t)t, (int)threadIdx.x < L && t < m, sec, n_rows, xs, prm,
                        bin_start, yg, zg, idg, gsr, up, starts, t_hits, cap,
                        keep + threadIdx.x, t_start, t_nhits, t_rin, t_par, t_cov, t_chi2,
                        n_prop, n_upd, n_cand);
    }
    add_work(status, n_prop, n_upd, n_cand);
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
    TPC_LAUNCH(k_tracklets, dim3((unsigned)g), dim3(kWave), sizeof(float) * p->n_rows, st,
               p->d_sectors, p->n_rows, p->d_row_x, p->params, (const int32_t*)grid_.bin_start,
               (const float*)grid_.y, (const float*)grid_.z, (const int32_t*)grid_.id,
               (const int32_t*)ws.gsr, (const int32_t*)links.up, (const int32_t*)starts.pos,
               ws.status, (const int64_t*)(ws.sec_start + sec_lo),
               (const int64_t*)(ws.sec_start + sec_hi), count_cap, trl.capacity, slots,
               trl.start, trl.hits, trl.nhits, trl.row_inner, trl.par, trl.cov, trl.chi2);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}

}  // namespace tpc
