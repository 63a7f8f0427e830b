// Monte Carlo response matrix and MLEM (paper Sec. 5.1, Eq. IMC and Eq. MLEM).
//
// Response matrix.  Each tally contribution of the forward call is an event
// (projection bin j, phantom voxel of emission, weight: 1 for an analog
// arrival, the score of a forced-detection copy).  With i the image voxel of
// the emission (phantom voxel / image_factor per axis),
//     T_ij = c_ij / n_i(j),   n_i(j) = N_view(j) * A_i / A,
// c_ij the summed weight of the events (i, j), N_view(j) the histories of bin j's view,
// A_i the activity in image voxel i and A the total: the estimated probability
// that a photon emitted in image voxel i is counted in bin j.  Bins merge the
// primary and scatter classes (the camera cannot tell them apart): j =
// (view * nv + iv) * nu + iu.  The projection P_j = sum_i c_ij is the same
// run's counts, so P = T n exactly.
//
// Both orientations are built as CSR (bins x voxels and voxels x bins): the
// events are radix-sorted by (bin, voxel) and runs of equal keys merged, the
// weights summed as Q31.32 integers, so the result does not depend on the
// order of the event list; the merged entries are then stably sorted by voxel,
// which gives the other orientation with the same values.
//
// MLEM.  S_i <- S_i / sens_i * sum_j T_ij P_j / y_j, y = T S, sens_i =
// sum_j T_ij; FP32 matrix values, FP64 accumulation; bins with y_j = 0 add
// nothing; voxels with sens_i = 0 stay 0.  Only the non-empty rows are swept,
// listed once per matrix, by groups of 1 to 64 lanes sized to their length;
// of a large dense matrix the rows are streamed instead, a tile of entries at
// a time, where that is the faster (mlem_forward_lanes, mlem_update_lanes).
#include <algorithm>

#include "mc_internal.h"

namespace mcs {
namespace {

constexpr int T256 = 256;
constexpr int SCAN_PER = 16;                     // items per thread in the block scan
constexpr int SCAN_BLOCK = T256 * SCAN_PER;      // items per scan block

int grid_for(uint64_t n, int threads, int cap) {
    uint64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    if (g > (uint64_t)cap) g = cap;
    return (int)g;
}

__device__ inline uint64_t wave_sum64(uint64_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ---- generic exclusive scan: uint32 counts -> uint64 offsets [n + 1] ----

__global__ __launch_bounds__(T256) void k_sum_blocks(const uint32_t* __restrict__ in, uint64_t n,
                                                     uint64_t* __restrict__ bsum) {
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_BLOCK;
    uint64_t s = 0;
    for (int j = threadIdx.x; j < SCAN_BLOCK; j += T256) {
        const uint64_t i = base + j;
        if (i < n) s += in[i];
    }
    s = wave_sum64(s);
    __shared__ uint64_t part[T256 / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int w = 0; w < T256 / 64; ++w) t += part[w];
        bsum[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(1024) void k_scan_blocks(uint64_t* bsum, int nb) {
    __shared__ uint64_t tot[1024];
    const int per = (nb + 1023) / 1024;
    const int b0 = threadIdx.x * per;
    uint64_t s = 0;
    for (int j = 0; j < per; ++j) if (b0 + j < nb) s += bsum[b0 + j];
    tot[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t v = threadIdx.x >= (unsigned)off ? tot[threadIdx.x - off] : 0;
        __syncthreads();
        tot[threadIdx.x] += v;
        __syncthreads();
    }
    uint64_t run = tot[threadIdx.x] - s;
    for (int j = 0; j < per; ++j) {
        if (b0 + j < nb) {
            const uint64_t v = bsum[b0 + j];
            bsum[b0 + j] = run;
            run += v;
        }
    }
}

// out[i] = sum_{k<i} in[k] for i in [0, n]; out[n] = total.
__global__ __launch_bounds__(T256) void k_scan_write(const uint32_t* __restrict__ in, uint64_t n,
                                                     const uint64_t* __restrict__ bsum,
                                                     uint64_t* __restrict__ out) {
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_BLOCK + (uint64_t)threadIdx.x * SCAN_PER;
    uint32_t v[SCAN_PER];
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < SCAN_PER; ++j) {
        const uint64_t i = base + j;
        v[j] = i < n ? in[i] : 0u;
        s += v[j];
    }
    __shared__ uint64_t tot[T256];
    tot[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < T256; off <<= 1) {
        const uint64_t t = threadIdx.x >= (unsigned)off ? tot[threadIdx.x - off] : 0;
        __syncthreads();
        tot[threadIdx.x] += t;
        __syncthreads();
    }
    uint64_t run = bsum[blockIdx.x] + tot[threadIdx.x] - s;
#pragma unroll
    for (int j = 0; j < SCAN_PER; ++j) {
        const uint64_t i = base + j;
        if (i <= n) out[i] = run;   // i == n: the total
        run += v[j];
    }
}

// out[i] = sum_{k<i} in[k] for i in [0, n].
hipError_t exclusive_scan(const uint32_t* in, uint64_t n, uint64_t* out, uint64_t* bsum, hipStream_t s) {
    // one extra item so the block holding index n writes the total
    const int nb = (int)((n + 1 + SCAN_BLOCK - 1) / SCAN_BLOCK);
    k_sum_blocks<<<nb, T256, 0, s>>>(in, n, bsum);
    k_scan_blocks<<<1, 1024, 0, s>>>(bsum, nb);
    k_scan_write<<<nb, T256, 0, s>>>(in, n, bsum, out);
    return hipGetLastError();
}

// ---- response matrix ----

struct SysArgs {
    const mc_event* events;
    const uint64_t* n_events;
    uint64_t capacity;
    uint32_t class_mask;     // bit 0: primary events, bit 1: scattered events
    uint32_t nv_nu;          // bins per view and class
    uint32_t nx, ny, f, mx, my;
    uint64_t q_per_view, r_extra;
};

// Items of a list whose count is on the device (it may exceed the capacity).
__device__ inline uint64_t items_of(const uint64_t* n_p, uint64_t capacity) {
    const uint64_t n = *n_p;
    return n < capacity ? n : capacity;
}

// projection bin (classes merged) and image voxel of event e; false if the
// event's class is filtered out
__device__ inline bool event_rc(const SysArgs& a, const mc_event& ev, uint32_t& bin, uint32_t& img) {
    const uint32_t per_view = 2u * a.nv_nu;
    const uint32_t cls = (ev.bin / a.nv_nu) & 1u;
    if (!((a.class_mask >> cls) & 1u)) return false;
    const uint32_t view = ev.bin / per_view;
    bin = view * a.nv_nu + (ev.bin % a.nv_nu);
    const uint32_t v = ev.emit_voxel;
    const uint32_t ix = v % a.nx, iy = (v / a.nx) % a.ny, iz = v / (a.nx * a.ny);
    img = (ix / a.f) + a.mx * ((iy / a.f) + a.my * (iz / a.f));
    return true;
}

__global__ __launch_bounds__(T256) void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * T256 + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * T256) p[i] = v;
}

// Activity per image voxel (a_img, zeroed before), and the total in
// TOTAL_SLOTS partial sums.  A workgroup takes an image row (x) and a share of
// the f x f phantom rows behind it: a thread adds up its columns, LDS adds the f columns of an image voxel.  Bound by the read of
// the activity: 256^3, f = 4: 376 us with an atomic per voxel, 28 us now.
constexpr uint32_t TOTAL_SLOTS = 64;

__global__ __launch_bounds__(T256) void k_image_activity(const uint32_t* __restrict__ act,
                                                         uint32_t nx, uint32_t ny, uint32_t f, uint32_t mx,
                                                         uint32_t my, uint32_t shares,
                                                         unsigned long long* __restrict__ a_img,
                                                         unsigned long long* __restrict__ total) {
    __shared__ unsigned long long acc[T256];
    __shared__ unsigned long long part[T256 / 64];
    const uint32_t share = blockIdx.x % shares, row = blockIdx.x / shares, jy = row % my, jz = row / my;
    const uint32_t r0 = (uint32_t)((uint64_t)f * f * share / shares);
    const uint32_t r1 = (uint32_t)((uint64_t)f * f * (share + 1) / shares);
    unsigned long long* out = a_img + (uint64_t)mx * (jy + (uint64_t)my * jz);
    // columns c0 .. c0 + w - 1 at a time: whole image voxels, or part of one
    const uint32_t w = f >= T256 ? T256 : T256 / f * f;
    uint64_t sum = 0;
    for (uint32_t c0 = 0; c0 < nx; c0 += w) {
        const uint32_t x = c0 + threadIdx.x, first = c0 / f;
        acc[threadIdx.x] = 0;
        __syncthreads();
        uint64_t t = 0;
        if (threadIdx.x < w && x < nx)
            for (uint32_t r = r0; r < r1; ++r)
                t += act[x + (uint64_t)nx * (jy * f + r % f + (uint64_t)ny * (jz * f + r / f))];
        if (t) atomicAdd(&acc[x / f - first], (unsigned long long)t);
        sum += t;
        __syncthreads();
        const unsigned long long v = acc[threadIdx.x];
        if (v) atomicAdd(out + first + threadIdx.x, v);
        __syncthreads();
    }
    sum = wave_sum64(sum);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long t = (part[0] + part[1]) + (part[2] + part[3]);
        if (t) atomicAdd(total + blockIdx.x % TOTAL_SLOTS, t);
    }
}

// ---- response matrix rows by LSD radix sort ----
//
// The events are sorted by the key (bin << col_bits) | voxel, and the merged
// entries by voxel, with a least-significant-digit radix sort (digits of up to
// 8 bits, stable), so a row's items end up together, ordered by column, with
// duplicates adjacent.  A pass is three launches: per-tile digit histograms
// (LDS counters; of the first pass, together with the keys), for each digit
// an exclusive scan over the tiles, and a stable scatter: within a tile, items
// are ranked round by round (256 consecutive items), inside a wavefront by
// matching digits with eight ballots and across the four wavefronts through
// LDS counts.  No global atomics: the per-event atomics of a counting sort
// contend on the rows that collect many events.  The item count is read on
// the device, so nothing waits on the host; tiles past it do no work.
// Events of a filtered class take row n_rows and sort last.
//
// Sorting the merged entries by voxel alone, instead of the events a second
// time by (voxel, bin), takes 3 passes over 12-byte items for 5 over 16-byte
// ones (1.16e7 events, 2.0e6 bins x 2.6e5 voxels: the whole build 3.2 ms as two
// sorts of the events with scans over all digit counts, 1.2 ms now).

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;              // digits per pass (= T256)
constexpr int RADIX_ITEMS = 16;                     // items per thread and tile
constexpr uint64_t RADIX_TILE = (uint64_t)T256 * RADIX_ITEMS;
static_assert(RADIX == T256, "one digit counter per thread");

int bit_width(uint64_t v) {
    int b = 0;
    while (v) { ++b; v >>= 1; }
    return b;
}

// Tile of workgroup b.  Workgroups are dealt to the 8 XCDs in turn; the
// tiles that hold items (the first `used`) are remapped so that each XCD
// takes a contiguous run of them, so neighbouring tiles share one L2 (their
// histogram and offset lines, and the adjacent digit runs they write).
// Empty tiles keep their own index.
__device__ inline uint32_t tile_of(uint32_t b, uint64_t n) {
    const uint32_t used = (uint32_t)((n + RADIX_TILE - 1) / RADIX_TILE);
    if (b >= used) return b;
    const uint32_t per = used / 8, rem = used % 8, x = b % 8, q = b / 8;
    return x * per + (x < rem ? x : rem) + q;
}

// Keys and weights of the events, with the first pass's histogram (as
// k_radix_hist).
__global__ __launch_bounds__(T256) void k_make_keys(SysArgs a, uint64_t n_rows, int col_bits, uint32_t mask,
                                                    uint32_t n_tiles, uint64_t* __restrict__ keys,
                                                    int64_t* __restrict__ vals, uint32_t* __restrict__ hist) {
    __shared__ uint32_t cnt[RADIX];
    const uint64_t n = items_of(a.n_events, a.capacity);
    const uint32_t tile = tile_of(blockIdx.x, n);
    const uint64_t base = (uint64_t)tile * RADIX_TILE;
    if (base >= n) return;       // an empty tile (the whole workgroup leaves)
    cnt[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll 4
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint64_t e = base + (uint64_t)j * T256 + threadIdx.x;
        if (e >= n) break;
        uint32_t bin, img;
        const mc_event ev = a.events[e];
        uint64_t k = n_rows << col_bits;
        int64_t v = 0;
        if (event_rc(a, ev, bin, img)) {
            k = ((uint64_t)bin << col_bits) | img;
            v = ev.weight;
        }
        keys[e] = k;
        vals[e] = v;
        atomicAdd(&cnt[(uint32_t)k & mask], 1u);
    }
    __syncthreads();
    hist[(uint64_t)threadIdx.x * n_tiles + tile] = cnt[threadIdx.x];
}

// hist[d * n_tiles + t]: items of tile t (one workgroup per tile) with digit d
template <class Key>
__global__ __launch_bounds__(T256) void k_radix_hist(const Key* __restrict__ keys, const uint64_t* __restrict__ n_p,
                                                     uint64_t capacity, int shift, uint32_t mask,
                                                     uint32_t n_tiles, uint32_t* __restrict__ hist) {
    __shared__ uint32_t cnt[RADIX];
    const uint64_t n = items_of(n_p, capacity);
    const uint32_t tile = tile_of(blockIdx.x, n);
    const uint64_t base = (uint64_t)tile * RADIX_TILE;
    if (base >= n) return;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    Key k[RADIX_ITEMS];
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint64_t i = base + (uint64_t)j * T256 + threadIdx.x;
        k[j] = keys[i < n ? i : n - 1];
    }
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint64_t i = base + (uint64_t)j * T256 + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(uint32_t)(k[j] >> shift) & mask], 1u);
    }
    __syncthreads();
    hist[(uint64_t)threadIdx.x * n_tiles + tile] = cnt[threadIdx.x];
}

// Exclusive scan of digit blockIdx.x's counts over the tiles that hold items,
// in place, and the digit's total.  (A scan over all digits and tiles of the
// list's capacity was three launches and 39 us for 3e7 slots; 5 us now.)
__global__ __launch_bounds__(1024) void k_digit_scan(const uint64_t* __restrict__ n_p, uint64_t capacity,
                                                     uint32_t n_tiles, uint32_t* __restrict__ hist,
                                                     uint32_t* __restrict__ tot) {
    __shared__ uint32_t part[16];
    const uint64_t n = items_of(n_p, capacity);
    const uint32_t used = (uint32_t)((n + RADIX_TILE - 1) / RADIX_TILE);
    uint32_t* __restrict__ h = hist + (uint64_t)blockIdx.x * n_tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t run = 0;
    for (uint32_t t0 = 0; t0 < used; t0 += 1024) {
        const uint32_t t = t0 + threadIdx.x, c = t < used ? h[t] : 0u;
        uint32_t x = c;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) part[wave] = x;
        __syncthreads();
        uint32_t before = run, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) before += part[w];
            all += part[w];
        }
        if (t < used) h[t] = before + x - c;
        run += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) tot[blockIdx.x] = run;
}

// Stable scatter of tile t's items to the digit's first slot + the scan of its
// counts at t + their rank among the tile's items of the digit.  Each wavefront
// takes a quarter of the tile (1024 consecutive items, 16 per lane, loaded at
// once) and ranks it on its own, 64 items per round: lanes with equal digits
// found with eight ballots, and a running count per digit kept in the
// wavefront's row of LDS.  After one barrier, the earlier wavefronts' counts
// place each item in a digit-ordered copy of the tile in LDS (keys, then
// values through the same 32 KB), which is written out so that each digit's
// run from this tile (16 items on average) goes to consecutive addresses.
// Bound by reading and writing the items.  col (nullable): the last pass of the
// entries' sort writes the two halves of a value to col and val.
constexpr uint32_t RADIX_WAVE_ITEMS = (uint32_t)(RADIX_TILE / (T256 / 64));

template <class Key>
__global__ __launch_bounds__(T256) void k_radix_scatter(const Key* __restrict__ kin,
                                                        const uint64_t* __restrict__ vin,
                                                        Key* __restrict__ kout, uint64_t* __restrict__ vout,
                                                        int32_t* __restrict__ col, float* __restrict__ val,
                                                        const uint64_t* __restrict__ n_p, uint64_t capacity,
                                                        int shift, uint32_t mask, uint32_t n_tiles,
                                                        const uint32_t* __restrict__ hist,
                                                        const uint32_t* __restrict__ tot) {
    __shared__ uint64_t stage[RADIX_TILE];         // the tile's keys, then values, in digit order
    __shared__ uint32_t gbase[RADIX];              // global slot of each digit's first item, less its tile slot
    __shared__ uint32_t lstart[RADIX];             // tile slot of each digit's first item
    __shared__ uint32_t wcnt[T256 / 64][RADIX];    // items of each digit per wavefront
    __shared__ uint2 wsum[T256 / 64];
    const uint64_t n = items_of(n_p, capacity);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lane_lt = (1ull << lane) - 1ull;
    const uint32_t tile = tile_of(blockIdx.x, n);
    const uint64_t base = (uint64_t)tile * RADIX_TILE;
    if (base >= n) return;       // an empty tile (the whole workgroup leaves)
    const uint64_t wbase = base + (uint64_t)wave * RADIX_WAVE_ITEMS;

    Key k[RADIX_ITEMS];
    uint64_t v[RADIX_ITEMS];
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint64_t i = wbase + (uint64_t)j * 64 + lane;
        k[j] = i < n ? kin[i] : 0;
        v[j] = i < n ? vin[i] : 0;
    }
    // this thread's digit: its items in the tile, in earlier tiles, and in all;
    // exclusive scans of the first (tile slots) and the last (global slots)
    const uint32_t* h = hist + (uint64_t)threadIdx.x * n_tiles + tile;
    const uint32_t all = tot[threadIdx.x], before_t = h[0];
    const uint32_t c = (base + RADIX_TILE < n ? h[1] : all) - before_t;
#pragma unroll
    for (int w = 0; w < T256 / 64; ++w) wcnt[w][threadIdx.x] = 0;
    uint32_t x = c, g = all;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64), z = __shfl_up(g, o, 64);
        if (lane >= o) { x += y; g += z; }
    }
    if (lane == 63) wsum[wave] = uint2{x, g};
    __syncthreads();
    x -= c;
    g -= all;
    for (int w = 0; w < wave; ++w) { x += wsum[w].x; g += wsum[w].y; }
    lstart[threadIdx.x] = x;
    gbase[threadIdx.x] = g + before_t - x;

    // rank within this wavefront: items of the same digit in earlier rounds
    // (the running count) plus lower lanes of this round
    uint32_t rk[RADIX_ITEMS];
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const bool ok = wbase + (uint64_t)j * 64 + lane < n;
        const uint32_t d = ok ? (uint32_t)(k[j] >> shift) & mask : 0;
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int b = 0; b < RADIX_BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lane_lt);
        const uint32_t before = ok ? wcnt[wave][d] : 0;
        rk[j] = before + rank;
        if (ok && rank == 0) wcnt[wave][d] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // tile slots of this lane's items (kept for the second staging)
    Key* const kstage = (Key*)stage;
    uint32_t slot[RADIX_ITEMS];
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        slot[j] = RADIX_TILE;
        if (wbase + (uint64_t)j * 64 + lane >= n) continue;
        const uint32_t d = (uint32_t)(k[j] >> shift) & mask;
        uint32_t sl = lstart[d] + rk[j];
        for (int w = 0; w < wave; ++w) sl += wcnt[w][d];
        slot[j] = sl;
        if (sl < RADIX_TILE) kstage[sl] = k[j];
    }
    __syncthreads();
    // global slots of the tile slots this thread writes out
    const uint32_t in_tile = (uint32_t)(n - base < RADIX_TILE ? n - base : RADIX_TILE);
    uint32_t pos[RADIX_ITEMS];
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint32_t t = (uint32_t)j * T256 + threadIdx.x;
        pos[j] = UINT32_MAX;
        if (t < in_tile) {
            const Key key = kstage[t];
            const uint32_t p = gbase[(uint32_t)(key >> shift) & mask] + t;
            if (p < capacity) {
                pos[j] = p;
                kout[p] = key;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j)
        if (slot[j] < RADIX_TILE) stage[slot[j]] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RADIX_ITEMS; ++j) {
        const uint32_t t = (uint32_t)j * T256 + threadIdx.x;
        if (pos[j] == UINT32_MAX) continue;
        const uint64_t x = stage[t];
        if (col) {
            col[pos[j]] = (int32_t)(uint32_t)x;
            val[pos[j]] = __uint_as_float((uint32_t)(x >> 32));
        } else {
            vout[pos[j]] = x;
        }
    }
}

// Merging of the sorted events, a tile of RUN_TILE per workgroup.
constexpr int RUN_ITEMS = 8;
constexpr int RUN_TILE = T256 * RUN_ITEMS;

// cnt[t]: runs of equal keys that start in tile t, of the unfiltered events
// (0 for tiles past the count)
__global__ __launch_bounds__(T256) void k_count_runs(const uint64_t* __restrict__ keys, SysArgs a,
                                                     uint64_t n_rows, int col_bits, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t part[T256 / 64];
    const uint64_t n = items_of(a.n_events, a.capacity), end = n_rows << col_bits;
    const uint64_t base = (uint64_t)blockIdx.x * RUN_TILE;
    uint32_t c = 0;
    if (base < n) {
#pragma unroll
        for (int u = 0; u < RUN_ITEMS; ++u) {
            const uint64_t i = base + (uint64_t)u * T256 + threadIdx.x, j = i < n ? i : n - 1;
            const uint64_t k = keys[j], p = keys[j ? j - 1 : 0];
            c += (uint32_t)__popcll(__ballot(i < n && k < end && (i == 0 || k != p)));
        }
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

// The runs that start in a tile (one distinct (bin, voxel) each) become the
// entries first[tile], ...: the column and T = c / n_i(j), with c the run's
// summed weight, and pair = bin | value << 32 for the other orientation.
// acc[bin] (nullable, zeroed before) collects the weights of a bin.  A thread
// takes eight consecutive events from LDS; scans over the tile number its runs
// and add up the weights, so a run's or a bin's sum is a difference of two
// prefix sums (modulo 2^64, exact), and runs and bins are then taken one per
// thread, with coalesced writes.  A run that goes on past the tile is summed to
// its end by the whole workgroup, and bins cut by the tile's ends are added
// atomically.  Bound by the read of the events and the write of the entries.
// (Flags, a scan over them, a thread per run and one per bin, each reading its
// own events: 270 us for 1.16e7 events; 156 us now with k_count_runs.)
__global__ __launch_bounds__(T256) void k_emit_runs(SysArgs a, const uint64_t* __restrict__ keys,
                                                    const int64_t* __restrict__ w,
                                                    const uint64_t* __restrict__ first, uint64_t n_rows,
                                                    int col_bits, int32_t* __restrict__ col,
                                                    float* __restrict__ val, uint64_t* __restrict__ pair,
                                                    unsigned long long* __restrict__ acc,
                                                    const unsigned long long* __restrict__ a_img,
                                                    const unsigned long long* __restrict__ total_p) {
    // one slot of padding per thread's eight: its reads spread over the banks
    constexpr int PAD = RUN_TILE + RUN_TILE / RUN_ITEMS + 1;
    __shared__ uint64_t key_s[PAD];
    __shared__ uint64_t sum_s[PAD];                // weights, then their exclusive prefix sums
    __shared__ uint16_t run_at[RUN_TILE + 1];      // the tile's runs, and bins, by their first event
    __shared__ uint16_t bin_at[RUN_TILE + 1];
    __shared__ uint32_t part_n[T256 / 64];
    __shared__ uint64_t part_w[T256 / 64];
    const auto at = [](int i) { return i + i / RUN_ITEMS; };
    const uint64_t n = items_of(a.n_events, a.capacity), end = n_rows << col_bits;
    const uint64_t base = (uint64_t)blockIdx.x * RUN_TILE;
    if (base >= n) return;
    const int m = (int)(n - base < RUN_TILE ? n - base : RUN_TILE);
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // a list that lost events (count above the capacity) gives no matrix
    const bool lost = *a.n_events > a.capacity;
    const double total = (double)wave_sum64(total_p[lane]);
    static_assert(TOTAL_SLOTS == 64, "a lane per partial sum");
    const uint64_t before = base ? keys[base - 1] : ~0ull;
#pragma unroll
    for (int u = 0; u < RUN_ITEMS; ++u) {
        const int i = u * T256 + tid;
        if (i < m) {
            key_s[at(i)] = keys[base + i];
            sum_s[at(i)] = (uint64_t)w[base + i];
        }
    }
    __syncthreads();
    // low half: runs, high half: bins
    uint32_t flags[RUN_ITEMS], mine = 0;
    uint64_t pre[RUN_ITEMS], sum = 0;
    uint64_t prev = tid == 0 ? before : key_s[at(tid * RUN_ITEMS - 1)];
#pragma unroll
    for (int u = 0; u < RUN_ITEMS; ++u) {
        const int i = tid * RUN_ITEMS + u;
        const bool in = i < m;
        const uint64_t k = in ? key_s[at(i)] : prev;
        flags[u] = (k != prev ? 1u : 0u) | (in && (i == 0 || k >> col_bits != prev >> col_bits) ? 0x10000u : 0u);
        pre[u] = sum;
        sum += in ? sum_s[at(i)] : 0;
        mine += flags[u];
        prev = k;
    }
    uint32_t x = mine;
    uint64_t y = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t p = __shfl_up(x, o, 64);
        const uint64_t q = __shfl_up(y, o, 64);
        if (lane >= o) { x += p; y += q; }
    }
    if (lane == 63) {
        part_n[wave] = x;
        part_w[wave] = y;
    }
    __syncthreads();
    x -= mine;
    y -= sum;
    uint32_t tot_n = 0;
    uint64_t tot_w = 0;
    for (int v = 0; v < T256 / 64; ++v) {
        if (v < wave) { x += part_n[v]; y += part_w[v]; }
        tot_n += part_n[v];
        tot_w += part_w[v];
    }
    const int n_run = (int)(tot_n & 0xFFFFu), n_bin = (int)(tot_n >> 16);
#pragma unroll
    for (int u = 0; u < RUN_ITEMS; ++u) {
        const int i = tid * RUN_ITEMS + u;
        if (flags[u] & 1u) run_at[x & 0xFFFFu] = (uint16_t)i;
        if (flags[u] >> 16) bin_at[x >> 16] = (uint16_t)i;
        x += flags[u];
        if (i < m) sum_s[at(i)] = y + pre[u];
    }
    if (tid == 0) {
        run_at[n_run] = (uint16_t)m;
        bin_at[n_bin] = (uint16_t)m;
        sum_s[at(m)] = tot_w;
    }
    __syncthreads();
    // the rest of the last run, past the tile
    uint64_t extra = 0;
    const uint64_t last = key_s[at(m - 1)];
    if (n_run > 0 && last < end && base + RUN_TILE < n && keys[base + RUN_TILE] == last) {
        for (uint64_t p = base + RUN_TILE; p < n; p += T256) {
            const bool same = p + tid < n && keys[p + tid] == last;
            if (same) extra += (uint64_t)w[p + tid];
            if (!__syncthreads_and(same)) break;
        }
        extra = wave_sum64(extra);
        if (lane == 0) part_w[wave] = extra;
        __syncthreads();
        extra = (part_w[0] + part_w[1]) + (part_w[2] + part_w[3]);
    }
    const uint64_t o0 = first[blockIdx.x], mask = (1ull << col_bits) - 1ull;
    for (int q = tid; q < n_run; q += T256) {
        const int i = run_at[q], j = run_at[q + 1];
        const uint64_t k = key_s[at(i)];
        if (k >= end) break;
        const long long cw = (long long)(sum_s[at(j)] - sum_s[at(i)] + (q == n_run - 1 ? extra : 0));
        const uint32_t bin = (uint32_t)(k >> col_bits), img = (uint32_t)(k & mask);
        const uint32_t view = bin / a.nv_nu;
        const double n_view = (double)(a.q_per_view + (view < a.r_extra ? 1u : 0u));
        const double n_i = n_view * (double)a_img[img] / total;
        const float t = lost ? __builtin_nanf("") : (float)((double)cw * 0x1p-32 / n_i);
        col[o0 + q] = (int32_t)img;
        val[o0 + q] = t;
        pair[o0 + q] = bin | (uint64_t)__float_as_uint(t) << 32;
    }
    if (!acc) return;
    for (int q = tid; q < n_bin; q += T256) {
        const int i = bin_at[q], j = bin_at[q + 1];
        const uint64_t bin = key_s[at(i)] >> col_bits;
        if (bin >= n_rows) break;
        const unsigned long long c = sum_s[at(j)] - sum_s[at(i)];
        if (q > 0 && q < n_bin - 1) acc[bin] = c;
        else if (c) atomicAdd(acc + bin, c);
    }
}

// rowptr[r] (r = 0..n_rows): first of the nnz entries, sorted by row, whose row
// is >= r (a binary search: non-decreasing and within [0, nnz] whatever the
// rows hold).  With proj: P_r = the summed weight of bin r's events; NaN when
// the list lost events.
template <class Row>
__global__ __launch_bounds__(T256) void k_row_ptr(const Row* __restrict__ rows, const uint64_t* __restrict__ nnz,
                                                  uint64_t capacity, uint64_t n_rows,
                                                  int64_t* __restrict__ rowptr, const int64_t* __restrict__ acc,
                                                  const uint64_t* __restrict__ n_events,
                                                  float* __restrict__ proj) {
    const uint64_t n = items_of(nnz, capacity);
    const bool lost = proj && *n_events > capacity;
    for (uint64_t r = (uint64_t)blockIdx.x * T256 + threadIdx.x; r <= n_rows;
         r += (uint64_t)gridDim.x * T256) {
        uint32_t lo = 0, hi = (uint32_t)n;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if ((uint32_t)rows[mid] < r) lo = mid + 1; else hi = mid;
        }
        rowptr[r] = (int64_t)lo;
        if (proj && r < n_rows) proj[r] = lost ? __builtin_nanf("") : (float)((double)acc[r] * 0x1p-32);
    }
}

// ---- MLEM ----
//
__device__ inline double wave_sum_f64(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// MLEM state in the workspace (device uint32 [ST_WORDS]), written by the
// set-up of a matrix and kept for every later call on it: the lengths of the
// two row lists; a flag set when the entry count the caller gave is not the
// matrix's own; a flag set by each call when it does not match the set-up
// (its sizes differ from the fingerprint); for the compact layout, per
// matrix and per (group, length class) key (2 x 32), the rows counted, their
// first list position and an append cursor; the fingerprint (n_bins, n_vox,
// nnz).  With either flag set the iterations sweep nothing and the image is
// NaN.
enum {
    ST_BINS = 0, ST_VOXS = 1, ST_BAD = 2, ST_CALL_BAD = 3, ST_HIST = 4, ST_OFF = 68, ST_CUR = 132,
    ST_FP = 196, ST_WORDS = 200
};

// Set-up: the state zeroed, the entry count checked against both row-pointer
// arrays, the fingerprint stored (one workgroup).
__device__ inline void mlem_setup(int64_t n_bins, int64_t n_vox, int64_t nnz, const int64_t* __restrict__ T_rp,
                                  const int64_t* __restrict__ Tt_rp, uint32_t* __restrict__ st) {
    const uint32_t t = threadIdx.x;
    if (t >= ST_WORDS) return;
    uint32_t v = 0;
    if (t == ST_BAD) v = (T_rp[n_bins] != nnz || Tt_rp[n_vox] != nnz) ? 1u : 0u;
    else if (t == ST_FP) v = (uint32_t)n_bins;
    else if (t == ST_FP + 1) v = (uint32_t)n_vox;
    else if (t == ST_FP + 2) v = (uint32_t)(uint64_t)nnz;
    else if (t == ST_FP + 3) v = (uint32_t)((uint64_t)nnz >> 32);
    st[t] = v;
}

__global__ __launch_bounds__(T256) void k_mlem_setup(int64_t n_bins, int64_t n_vox, int64_t nnz,
                                                     const int64_t* __restrict__ T_rp,
                                                     const int64_t* __restrict__ Tt_rp,
                                                     uint32_t* __restrict__ st) {
    mlem_setup(n_bins, n_vox, nnz, T_rp, Tt_rp, st);
}

// A call's sizes against the set-up's fingerprint (and its entry-count flag).
__device__ inline bool mlem_call_bad(const uint32_t* __restrict__ st, int64_t n_bins, int64_t n_vox,
                                     int64_t nnz) {
    return st[ST_BAD] != 0 || st[ST_FP] != (uint32_t)n_bins || st[ST_FP + 1] != (uint32_t)n_vox ||
           st[ST_FP + 2] != (uint32_t)(uint64_t)nnz || st[ST_FP + 3] != (uint32_t)((uint64_t)nnz >> 32);
}

// Rows a workgroup takes at a time in the set-up of the compact layout.
constexpr int ROWS_PER_THREAD = 16;
constexpr int ROW_CHUNK = T256 * ROWS_PER_THREAD;

// The rows a group of GS lanes visits: row g, g + n_groups, ... (g: the
// group's index among n_groups); every lane of a group sees the same rows.
template <int GS>
struct RowGroups {
    int64_t first, step;
    int sub;
    __device__ RowGroups(int64_t block, int64_t n_blocks) {
        const int64_t t = block * T256 + threadIdx.x;
        first = t / GS;
        step = n_blocks * T256 / GS;
        sub = (int)(threadIdx.x & (GS - 1));
    }
};

// Sum over k in [k0, k1) of term(k, valid) by a group of GS lanes (sub: the
// lane's index in the group).  Indices past the end are clamped to k1 - 1 so
// every load is in bounds and issued unconditionally; term() zeroes them.
// Each lane adds its four terms in order, then a butterfly over the group:
// the summation order depends only on the row and GS.
template <int GS, class Term>
__device__ inline double group_row_sum(int64_t k0, int64_t k1, int sub, Term term) {
    double acc = 0.0;
    for (int64_t k = k0 + sub; k < k1; k += 4 * GS) {
        double t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t kk = k + (int64_t)u * GS;
            t[u] = term(kk < k1 ? kk : k1 - 1, kk < k1);
        }
        acc += t[0];
        acc += t[1];
        acc += t[2];
        acc += t[3];
    }
#pragma unroll
    for (int o = GS / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, GS);
    return acc;
}

// ---- row order.  Tiles of a large dense matrix: a workgroup takes consecutive
// rows, whose entries are consecutive too, and streams them a tile of LOADS
// entries per thread at a time: coalesced loads of columns and values, LOADS gathers in
// flight per thread, the products in LDS in FP64, then each row summed from
// there by a power-of-two number of lanes.  The order of a sum depends only on
// the matrix.  Bound by the stream of entries (8 bytes each) and the gathers'
// traffic from L2 to L1, a line per entry.  On a forced-detection matrix of 4.6e7
// entries, 1.97 M bins and 2.6e5 voxels, 156 us per forward sweep, against 233 us
// by a lane group per listed row, four rows per pass.  Each XCD works on
// neighbouring rows (sweep_chunk), so a sweep's gathers fall in what its L2
// holds.  (Where columns are random, which no camera gives, a backprojection in
// slices of the bins, one per XCD, which was here before, is the better: 2^20
// bins x 2^17 voxels, 3e7 entries: 437 us per iteration against 471 now.)

// Rows per workgroup, of mean entries each: three quarters of a tile on
// average, so that most need one.
inline int sweep_per(int loads, int64_t mean) {
    const int64_t per = loads * T256 * 3 / 4 / std::max<int64_t>(1, mean);
    return (int)std::min<int64_t>(T256, std::max<int64_t>(1, per));
}

// Workgroups for n chunks of rows, and the chunk of this workgroup.  Workgroups
// are dealt to the 8 XCDs in turn: each XCD takes runs of consecutive chunks,
// one run in eight, 16 runs per XCD, so neighbouring rows meet in one L2 and
// dense and empty regions are spread over the XCDs (with one contiguous eighth
// each, the CUs were busy 70 % of a backprojection).
constexpr int SWEEP_RUNS = 16;
inline unsigned sweep_grid(int64_t n_chunks) {
    const int64_t run = (n_chunks + 8 * SWEEP_RUNS - 1) / (8 * SWEEP_RUNS);
    return (unsigned)(8 * SWEEP_RUNS * run);
}
__device__ __forceinline__ int64_t sweep_chunk() {
    const uint32_t run = gridDim.x / (8 * SWEEP_RUNS), j = blockIdx.x / 8;
    return (int64_t)((j / run * 8 + blockIdx.x % 8) * run + j % run);
}

__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Sum over each row r in [r0, r0 + n) (n <= T256) of its entries' terms,
// done(r, sum) by one lane per non-empty row (and of an empty row that is taken
// alone, with the sum 0).  The rows' entries start at e0 +
// bound(0), bound(1), ..., bound(n); the term of entry first + k is load(first,
// k) -> A, then value(A) -> double, so the loads of a tile are issued before
// its gathers (first is in scalar registers).  All threads of a workgroup call,
// with the same r0 and n.  skip: nothing is done (loaded along with the
// bounds, not before them).
template <int LOADS, class Bound, class Load, class Value, class Done>
__device__ inline void sweep_bounds(int64_t r0, int n, bool skip, int64_t e0, Bound bound, Load load, Value value,
                                    Done done) {
    constexpr int TILE = LOADS * T256;
    __shared__ double prod[TILE];
    __shared__ int64_t off[T256 + 1];
    const int tid = (int)threadIdx.x;
    if (tid <= n) off[tid] = bound(tid);
    if (tid == 0 && n == T256) off[n] = bound(n);
    if (skip) return;
    __syncthreads();
    int s = 0;
    while (s < n) {
        // rows [s, e) fit in a tile
        int e = s, hi = n;
        while (e < hi) {
            const int mid = (e + hi + 1) >> 1;
            if (off[mid] - off[s] <= TILE) e = mid; else hi = mid - 1;
        }
        e = __builtin_amdgcn_readfirstlane(e);
        const int64_t first = uniform_i64(e0 + off[s]);
        if (e <= s + 1) {
            // one row: the whole group, tile by tile
            const int64_t len = uniform_i64(off[s + 1] - off[s]);
            double acc = 0.0;
            for (int64_t k0 = 0; k0 < len; k0 += TILE) {
                const int cnt = (int)(len - k0 < TILE ? len - k0 : TILE);
                decltype(load(0, 0)) a[LOADS];
#pragma unroll
                for (int u = 0; u < LOADS; ++u) {
                    const int k = tid + u * T256;
                    a[u] = load(first + k0, k < cnt ? k : cnt - 1);
                }
#pragma unroll
                for (int u = 0; u < LOADS; ++u) {
                    const double x = value(a[u]);
                    acc += tid + u * T256 < cnt ? x : 0.0;
                }
            }
            acc = wave_sum_f64(acc);
            if ((tid & 63) == 0) prod[tid >> 6] = acc;
            __syncthreads();
            acc = (prod[0] + prod[1]) + (prod[2] + prod[3]);
            if (tid == 0) done(r0 + s, acc);
            ++s;
        } else {
            const int cnt = (int)uniform_i64(off[e] - off[s]);
            if (cnt > 0) {
                decltype(load(0, 0)) a[LOADS];
#pragma unroll
                for (int u = 0; u < LOADS; ++u) {
                    const int k = tid + u * T256;
                    a[u] = load(first, k < cnt ? k : cnt - 1);
                }
#pragma unroll
                for (int u = 0; u < LOADS; ++u) prod[tid + u * T256] = value(a[u]);
            }
            __syncthreads();
            // as many lanes per row as there are for all rows at once
            int gs = 1;
            while (gs < 64 && 2 * gs * (e - s) <= T256) gs *= 2;
            const int sub = tid & (gs - 1);
            for (int r = s + tid / gs; r < e; r += T256 / gs) {
                const int k0 = (int)(off[r] - off[s]), k1 = (int)(off[r + 1] - off[s]);
                double acc = 0.0;
                for (int k = k0 + sub; k < k1; k += gs) acc += prod[k];
                for (int o = gs >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
                if (sub == 0 && k1 > k0) done(r0 + r, acc);
            }
            s = e;
        }
        __syncthreads();          // prod is written again
    }
}

template <int LOADS, class Load, class Value, class Done>
__device__ inline void sweep(int64_t r0, int n, bool skip, const int64_t* __restrict__ rp, Load load, Value value,
                             Done done) {
    const int64_t e0 = rp[r0];
    sweep_bounds<LOADS>(r0, n, skip, e0, [&](int i) { return rp[r0 + i] - e0; }, load, value, done);
}

// Bins have short rows and voxels long ones: on the matrix above eight and
// four took 156 and 274 us per sweep, four and eight 178 and 299 us.
constexpr int FORWARD_LOADS = 8, UPDATE_LOADS = 4;

// An entry and the matrix's product with a vector.
struct Entry {
    int32_t col;
    float val;
};
__device__ __forceinline__ Entry load_entry(const int32_t* __restrict__ col, const float* __restrict__ val,
                                            int64_t first, int k) {
    return Entry{*(col + first + (uint32_t)k), *(val + first + (uint32_t)k)};
}

// out[r] = sum of the row's values (sens), 0 for an empty row.
__global__ __launch_bounds__(T256) void k_sweep_sums(int64_t n_rows, int per, const int64_t* __restrict__ rp,
                                                     const float* __restrict__ v, double* __restrict__ out) {
    const int64_t r0 = sweep_chunk() * per;
    if (r0 >= n_rows) return;
    const int n = (int)std::min<int64_t>(per, n_rows - r0);
    const int i = (int)(threadIdx.x);
    if (i < n && rp[r0 + i] == rp[r0 + i + 1]) out[r0 + i] = 0.0;
    sweep<UPDATE_LOADS>(r0, n, false, rp, [&](int64_t first, int k) { return *(v + first + (uint32_t)k); },
             [](float x) { return (double)x; }, [&](int64_t r, double acc) { out[r] = acc; });
}

// ---- row lists.  The non-empty rows of T and of T^T, each in row order, made
// once per matrix: of a camera's matrix 30 to 80 % of the bins and voxels have
// no entries.  A listed row is summed by a group of lanes, one row per group and
// pass, four entries per lane in flight.

// A non-empty row: its index and entry range.
struct RowRef {
    int64_t lo;
    int32_t row, len;
};

// A workgroup takes ROW_CHUNK consecutive rows of one matrix at a time.  First
// pass: chunk[c] = non-empty rows of chunk c (T's chunks, then T^T's); the last
// workgroup does the set-up instead.  Second pass: the rows at their positions,
// and the lengths of the lists, st[ST_BINS] and st[ST_VOXS]; each workgroup adds
// up the counts before its only chunk, or (SCANNED, for more than
// ROWS_MAX_CHUNKS) finds their exclusive scan there.  In row order, so that
// the rows in flight at a time are neighbours, whose gathers meet in the caches:
// appended as the workgroups came, an iteration on 3.5e6 entries, 1.5e6 bins and
// 6.8e5 voxels took 72 us instead of 61.
constexpr int64_t ROWS_MAX_CHUNKS = 2048;
enum { ROWS_COUNT, ROWS_PLACE, ROWS_PLACE_SCANNED };

template <int PASS>
__global__ __launch_bounds__(T256) void k_mlem_rows(int64_t n_bins, int64_t n_vox, int64_t nnz,
                                                    const int64_t* __restrict__ T_rp,
                                                    const int64_t* __restrict__ Tt_rp,
                                                    RowRef* __restrict__ bins, RowRef* __restrict__ voxs,
                                                    uint64_t* __restrict__ chunk, uint32_t* __restrict__ st) {
    constexpr int WAVES = T256 / 64;
    __shared__ uint32_t before[ROWS_PER_THREAD * WAVES];
    __shared__ uint32_t total;
    __shared__ uint64_t part[WAVES];
    const int64_t n_blocks = PASS == ROWS_COUNT ? gridDim.x - 1 : gridDim.x;
    if constexpr (PASS == ROWS_COUNT) {
        if (blockIdx.x == n_blocks) {
            mlem_setup(n_bins, n_vox, nnz, T_rp, Tt_rp, st);
            return;
        }
    } else {
        if (st[ST_BAD]) return;
    }
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    const uint64_t lane_lt = (1ull << lane) - 1;
    const int64_t nbc = (n_bins + ROW_CHUNK - 1) / ROW_CHUNK;
    const int64_t nvc = (n_vox + ROW_CHUNK - 1) / ROW_CHUNK;
    for (int64_t c = blockIdx.x; c < nbc + nvc; c += n_blocks) {
        const bool vox = c >= nbc;
        const int64_t r0 = (vox ? c - nbc : c) * ROW_CHUNK, nr = vox ? n_vox : n_bins;
        const int64_t* rp = vox ? Tt_rp : T_rp;
        int64_t lo[ROWS_PER_THREAD];
        int32_t len[ROWS_PER_THREAD];
        uint64_t m[ROWS_PER_THREAD];
#pragma unroll
        for (int k = 0; k < ROWS_PER_THREAD; ++k) {
            const int64_t r = r0 + k * T256 + threadIdx.x;
            lo[k] = 0;
            len[k] = 0;
            if (r < nr) {
                lo[k] = rp[r];
                len[k] = (int32_t)(rp[r + 1] - lo[k]);
            }
        }
        uint64_t first = 0;
        if constexpr (PASS == ROWS_PLACE) {
            for (int64_t k = (vox ? nbc : 0) + threadIdx.x; k < c; k += T256) first += chunk[k];
            first = wave_sum64(first);
            if (lane == 0) part[w] = first;
        }
        if constexpr (PASS == ROWS_PLACE_SCANNED) first = chunk[c] - (vox ? chunk[nbc] : 0);
#pragma unroll
        for (int k = 0; k < ROWS_PER_THREAD; ++k) {
            m[k] = __ballot(len[k] > 0);
            if (lane == 0) before[k * WAVES + w] = (uint32_t)__popcll(m[k]);
        }
        __syncthreads();
        // exclusive scan: rows r0 + k * 256 + w * 64 + lane in (k, w, lane) order
        if (w == 0) {
            static_assert(ROWS_PER_THREAD * WAVES == 64, "one count per lane");
            const uint32_t v = before[lane];
            uint32_t x = v;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            before[lane] = x - v;
            if (lane == 63) total = x;
        }
        if constexpr (PASS == ROWS_PLACE) first = (part[0] + part[1]) + (part[2] + part[3]);
        __syncthreads();
        if constexpr (PASS == ROWS_COUNT) {
            if (threadIdx.x == 0) chunk[c] = total;
        } else {
            RowRef* out = vox ? voxs : bins;
#pragma unroll
            for (int k = 0; k < ROWS_PER_THREAD; ++k) {
                const int64_t r = r0 + k * T256 + threadIdx.x;
                const uint64_t at = first + before[k * WAVES + w] + (uint32_t)__popcll(m[k] & lane_lt);
                if (len[k] > 0) out[at] = RowRef{lo[k], (int32_t)r, len[k]};
            }
            if (threadIdx.x == 0 && (c == nbc - 1 || c == nbc + nvc - 1))
                st[vox ? ST_VOXS : ST_BINS] = (uint32_t)(first + total);
        }
        __syncthreads();     // before[] is rewritten for the next chunk
    }
}

// How a matrix's sweeps are done.  Listed rows: lanes_per_row lanes share one,
// the smallest group of 1, 4, 16 or 64 for which `each` entries per lane cover
// the mean row of `part` entries in n_rows rows.  Tiles (0):
//  * where there are few rows, too few for a wavefront each to keep the chip
//    busy (1331 voxels of 486 entries: 14.6 us per backprojection by wavefronts,
//    9.8 swept);
//  * the forward sweep of a matrix that does not stay in the caches, from
//    SWEEP_MIN_NNZ entries on (20 iterations on 2.6e7 entries, 2.5e5 bins,
//    2.6e5 voxels: 4.65 ms with listed forward sweeps, 4.32 with tiles; on
//    9.4e6 even; below, tiles lose more to their barriers and part-filled
//    tiles than a row's chain of loads costs: 2.4e6 entries, 36 iterations: 1002
//    against 1169 us);
//  * the backprojection of such a matrix if its rows are short (1.0e7 entries,
//    2.1e6 voxels: 2.40 ms swept, 2.48 listed; with longer rows listed is the
//    better: 2.6e7 entries, 2.6e5 voxels: 4.09 against 4.32 ms, 1.3e7 entries,
//    3.3e4 voxels: 1.35 against 1.86 ms).
constexpr int64_t SWEEP_MIN_NNZ = 1 << 23;
constexpr int64_t SWEEP_MIN_MEAN = 256;
constexpr int64_t SWEEP_FEW_ROWS = 1 << 15;
constexpr int64_t SWEEP_SHORT_ROW = 16;

__host__ __device__ inline int lanes_per_row(int64_t part, int64_t n_rows, int each) {
    return part <= each * n_rows ? 1 : part <= 4 * each * n_rows ? 4 : part <= 16 * each * n_rows ? 16 : 64;
}
inline bool few_long_rows(int64_t part, int64_t n_rows) {
    return n_rows < SWEEP_FEW_ROWS && part >= SWEEP_MIN_MEAN * n_rows;
}
inline int mlem_forward_lanes(int64_t nnz, int64_t n_bins) {
    return nnz >= SWEEP_MIN_NNZ || few_long_rows(nnz, n_bins) ? 0 : lanes_per_row(nnz, n_bins, 4);
}
inline int mlem_update_lanes(int64_t nnz, int64_t n_vox) {
    if (few_long_rows(nnz, n_vox) || (nnz >= SWEEP_MIN_NNZ && nnz < SWEEP_SHORT_ROW * n_vox)) return 0;
    return lanes_per_row(nnz, n_vox, 4);
}
// OSEM: 0 (tiles) for a subset's `part` of nnz entries in n_rows rows
inline int os_lanes(int64_t nnz, int64_t part, int64_t n_rows, int each) {
    if (nnz >= SWEEP_MIN_NNZ || part >= SWEEP_MIN_MEAN * n_rows) return 0;
    return lanes_per_row(part, n_rows, each);
}

// The rows of a list (at most cap, *count of them) by groups of GS lanes;
// `block` of gridDim.x workgroups.  The first row's reference is loaded along
// with the list's length, not after it.
template <int GS, class Own, class Term, class Done>
__device__ inline void sweep_list(int64_t block, const RowRef* __restrict__ L, int64_t cap,
                                  const uint32_t* __restrict__ count, const uint32_t* __restrict__ call_bad,
                                  Own own, Term term, Done done) {
    const RowGroups<GS> G(block, gridDim.x);
    if (G.first >= cap) return;
    RowRef ref = L[G.first];
    const uint32_t listed = *count, bad = *call_bad;
    // all in flight before any is used (the compiler would load the reference
    // once the length's test has passed)
    asm volatile("" ::"v"(ref.lo), "s"(listed), "s"(bad));
    const int64_t n = bad ? 0 : listed;     // a call that does not match the set-up sweeps nothing
    for (int64_t r = G.first; r < n; r += G.step) {
        if (r != G.first) ref = L[r];
        const auto o = own(ref.row);
        const double sum = group_row_sum<GS>(ref.lo, ref.lo + ref.len, G.sub, term);
        if (G.sub == 0) done(ref.row, o, sum);
    }
}

// (An XCD takes runs of consecutive rows here: 20 iterations on 5.8e6 entries,
// 9.8e5 bins and 2.1e6 voxels, whose vector no L2 holds, 2.34 ms, without 2.50.)
template <int GS>
__global__ __launch_bounds__(T256) void k_mlem_forward_rows(const RowRef* __restrict__ L, int64_t cap,
                                                            const uint32_t* __restrict__ count,
                                                            const uint32_t* __restrict__ call_bad,
                                                            const int32_t* __restrict__ col,
                                                            const float* __restrict__ val,
                                                            const double* __restrict__ S,
                                                            const float* __restrict__ P,
                                                            double* __restrict__ ratio) {
    sweep_list<GS>(sweep_chunk(), L, cap, count, call_bad, [&](int32_t r) { return P[r]; },
                   [&](int64_t k, bool ok) {
                       const double x = (double)val[k] * S[col[k]];
                       return ok ? x : 0.0;
                   },
                   [&](int32_t r, float p, double y) { ratio[r] = y > 0.0 ? (double)p / y : 0.0; });
}

template <int GS>
__global__ __launch_bounds__(T256) void k_mlem_update_rows(const RowRef* __restrict__ L, int64_t cap,
                                                           const uint32_t* __restrict__ count,
                                                           const uint32_t* __restrict__ call_bad,
                                                           const int32_t* __restrict__ col,
                                                           const float* __restrict__ val,
                                                           const double* __restrict__ ratio,
                                                           const double* __restrict__ sens,
                                                           double* __restrict__ S) {
    sweep_list<GS>(blockIdx.x, L, cap, count, call_bad, [&](int32_t r) { return double2{S[r], sens[r]}; },
                   [&](int64_t k, bool ok) {
                       const double x = (double)val[k] * ratio[col[k]];
                       return ok ? x : 0.0;
                   },
                   [&](int32_t r, double2 o, double b) { S[r] = o.y > 0.0 ? o.x * b / o.y : 0.0; });
}

// y_j = sum_i T_ij S_i; ratio_j = P_j / y_j (0 when y_j = 0), over the
// non-empty bin rows (an empty one is referred to by no entry of T^T, so its
// ratio is never read).  A call that does not match the set-up sweeps nothing.
__global__ __launch_bounds__(T256) void k_mlem_forward(int64_t n_bins, int per, const int64_t* __restrict__ rp,
                                                       const uint32_t* __restrict__ call_bad,
                                                       const int32_t* __restrict__ col,
                                                       const float* __restrict__ val,
                                                       const double* __restrict__ S,
                                                       const float* __restrict__ P,
                                                       double* __restrict__ ratio) {
    const int64_t r0 = sweep_chunk() * per;
    if (r0 >= n_bins) return;
    sweep<FORWARD_LOADS>(r0, (int)std::min<int64_t>(per, n_bins - r0), *call_bad != 0, rp,
             [&](int64_t first, int k) { return load_entry(col, val, first, k); },
             [&](Entry e) { return (double)e.val * S[e.col]; },
             [&](int64_t r, double y) { ratio[r] = y > 0.0 ? (double)P[r] / y : 0.0; });
}

// S_i <- S_i * (sum_j T_ij ratio_j) / sens_i over the non-empty voxel rows
// (an empty row has sens_i = 0, so its S_i is already 0).
__global__ __launch_bounds__(T256) void k_mlem_update(int64_t n_vox, int per, const int64_t* __restrict__ rp,
                                                      const uint32_t* __restrict__ call_bad,
                                                      const int32_t* __restrict__ col,
                                                      const float* __restrict__ val,
                                                      const double* __restrict__ ratio,
                                                      const double* __restrict__ sens,
                                                      double* __restrict__ S) {
    const int64_t r0 = sweep_chunk() * per;
    if (r0 >= n_vox) return;
    sweep<UPDATE_LOADS>(r0, (int)std::min<int64_t>(per, n_vox - r0), *call_bad != 0, rp,
             [&](int64_t first, int k) { return load_entry(col, val, first, k); },
             [&](Entry e) { return (double)e.val * ratio[e.col]; },
             [&](int64_t r, double b) { S[r] = sens[r] > 0.0 ? S[r] * b / sens[r] : 0.0; });
}

// ---- compact layout.  The non-empty rows of both matrices are listed in
// (group, length class) order; the list position of a row is the index of
// its entries in the iterated vectors.
//
// Groups.  Workgroups are handed to the 8 XCDs in turn, and workgroup b of a
// sweep works on group b mod 8, so the rows of one group are swept, and
// their vector entries written, by one XCD.  A voxel row's group is its
// eighth of the voxel index range (contiguous index ranges are slabs of
// planes); a bin row's group is that of the voxel of its first entry (for a
// parallel-hole camera, the slab its ray crosses).  Gathers then mostly read
// entries that the same XCD wrote in the previous sweep, still in its L2,
// rather than lines written back by other XCDs.  Any grouping is correct.
//
// Length classes.  Rows of at most 4, 16, 64 entries and longer ones are
// swept by groups of 1, 4, 16 and 64 lanes, one row per group and pass, so a
// row of up to 4 GS entries takes one load round of its group and a long row
// does not hold one lane for many rounds.  The lane-group size, and with it
// the summation order, depends only on the row's length.
constexpr int N_CLASS = 4;
constexpr int N_GROUP = 8;
constexpr int N_KEY = N_CLASS * N_GROUP;     // per matrix

__host__ __device__ inline int length_class(int64_t len) {
    return len <= 4 ? 0 : len <= 16 ? 1 : len <= 64 ? 2 : 3;
}

// The most rows class c can hold, of n rows and at most nnz entries.
__host__ __device__ inline int64_t class_capacity(int c, int64_t n, int64_t nnz) {
    const int64_t min_len[N_CLASS] = {1, 5, 17, 65};
    const int64_t m = nnz / min_len[c];
    return m < n ? m : n;
}

// A listed row of the compact layout (at its list position): its index and
// entry range.
struct ClassRef {
    int32_t row;
    uint32_t lo;
    int32_t len, pad;
};

// The entries of a listed row of at most four (length class 0), copied at
// its list position with columns renumbered: a sweep loads them together
// with the row's ClassRef instead of after it (one dependent load fewer).
// Slots past the row's length are unused.
struct alignas(16) ShortRow {
    int32_t col[4];
    float val[4];
};

// Compact layout (sparse matrices, nnz <= n_bins + n_vox): the iterations
// keep S, sens, P and the ratio in list order, and the column indices of both
// matrices are renumbered to list positions (Tc: voxel positions, Ttc: bin
// positions), so every gather falls in a vector of the non-empty rows only
// (a few MB at most, L2-resident) instead of a sparse scattering over the
// full bin and voxel ranges.  A column whose row in the other orientation is
// empty (the two orientations disagree) sets the bad flag.
__global__ __launch_bounds__(T256) void k_mlem_compact(int64_t nnz, const int32_t* __restrict__ T_col,
                                                       const int32_t* __restrict__ Tt_col,
                                                       const int32_t* __restrict__ bin_pos,
                                                       const int32_t* __restrict__ vox_pos,
                                                       int32_t* __restrict__ Tc, int32_t* __restrict__ Ttc,
                                                       const ClassRef* __restrict__ bins,
                                                       const ClassRef* __restrict__ voxs,
                                                       const float* __restrict__ T_val,
                                                       const float* __restrict__ Tt_val,
                                                       ShortRow* __restrict__ bin_short,
                                                       ShortRow* __restrict__ vox_short,
                                                       const double* __restrict__ sens,
                                                       double* __restrict__ sens_l, uint32_t* __restrict__ st) {
    if (st[ST_BAD]) return;
    const int64_t nb = st[ST_BINS], nv = st[ST_VOXS];
    const int64_t n = std::max(nnz, std::max(nb, nv));
    bool bad = false;
    // a short row's entries with the renumbering of Tc / Ttc (from the
    // original columns: Tc and Ttc are written by other threads of this pass)
    auto copy_short = [](const ClassRef& r, const int32_t* __restrict__ c, const float* __restrict__ v,
                         const int32_t* __restrict__ pos, ShortRow* __restrict__ out) {
        ShortRow e;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t p = k < r.len ? pos[c[r.lo + k]] : 0;
            e.col[k] = p < 0 ? 0 : p;
            e.val[k] = k < r.len ? v[r.lo + k] : 0.0f;
        }
        *out = e;
    };
    for (int64_t t = (int64_t)blockIdx.x * T256 + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * T256) {
        if (t < nnz) {
            const int32_t pv = vox_pos[T_col[t]], pb = bin_pos[Tt_col[t]];
            bad |= pv < 0 || pb < 0;
            Tc[t] = pv < 0 ? 0 : pv;
            Ttc[t] = pb < 0 ? 0 : pb;
        }
        if (t < nv) {
            const ClassRef r = voxs[t];
            sens_l[t] = sens[r.row];
            if (r.len <= 4) copy_short(r, Tt_col, Tt_val, bin_pos, vox_short + t);
        }
        if (t < nb) {
            const ClassRef r = bins[t];
            if (r.len <= 4) copy_short(r, T_col, T_val, vox_pos, bin_short + t);
        }
    }
    if (bad) atomicOr(&st[ST_BAD], 1u);
}

// Per call: the call checked against the set-up (ST_CALL_BAD), then the
// iterated vectors loaded: S = img where sens > 0, else 0, and for the
// compact layout P in list order (voxs / bins non-null).  In row order S and
// sens are indexed by voxel; in list order by list position.
__global__ __launch_bounds__(T256) void k_mlem_load(int64_t n_bins, int64_t n_vox, int64_t nnz,
                                                    const float* __restrict__ img,
                                                    const double* __restrict__ sens,
                                                    double* __restrict__ S, const float* __restrict__ P,
                                                    const ClassRef* __restrict__ bins,
                                                    const ClassRef* __restrict__ voxs,
                                                    float* __restrict__ P_l, uint32_t* __restrict__ st) {
    const bool bad = mlem_call_bad(st, n_bins, n_vox, nnz);
    if (blockIdx.x == 0 && threadIdx.x == 0) st[ST_CALL_BAD] = bad ? 1u : 0u;
    if (bad) return;
    const int64_t nv = voxs ? (int64_t)st[ST_VOXS] : n_vox, nb = bins ? (int64_t)st[ST_BINS] : 0;
    const int64_t n = std::max(nv, nb);
    for (int64_t t = (int64_t)blockIdx.x * T256 + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * T256) {
        if (t < nv) S[t] = sens[t] > 0.0 ? (double)img[voxs ? voxs[t].row : t] : 0.0;
        if (t < nb) P_l[t] = P[bins[t].row];
    }
}

// (group, class) key of a non-empty row: group by voxel index (a voxel row's
// own, a bin row's first column), class by length.
__device__ inline int row_key(int64_t vox, int64_t n_vox, int64_t len) {
    const int g = (int)(((uint64_t)vox * N_GROUP) / (uint64_t)n_vox);
    return g * N_CLASS + length_class(len);
}

// One matrix's rows in chunks of 4096 per workgroup: for each non-empty row,
// f(row, lo, len, key).  Rows of the bin matrix (col: its columns) take the
// group of their first column.
template <class F>
__device__ inline void for_listed_rows(int64_t r0, int64_t nr, const int64_t* __restrict__ rp,
                                       const int32_t* __restrict__ col, int64_t n_vox, F f) {
    // all row bounds, then all first columns, in flight before any is used
    int64_t lo[ROWS_PER_THREAD], len[ROWS_PER_THREAD];
    int32_t c0[ROWS_PER_THREAD];
#pragma unroll
    for (int k = 0; k < ROWS_PER_THREAD; ++k) {
        const int64_t r = r0 + k * T256 + threadIdx.x;
        lo[k] = 0;
        len[k] = 0;
        if (r < nr) {
            lo[k] = rp[r];
            len[k] = rp[r + 1] - lo[k];
        }
    }
#pragma unroll
    for (int k = 0; k < ROWS_PER_THREAD; ++k) c0[k] = (col && len[k] > 0) ? col[lo[k]] : 0;
#pragma unroll
    for (int k = 0; k < ROWS_PER_THREAD; ++k) {
        const int64_t r = r0 + k * T256 + threadIdx.x;
        if (len[k] > 0) f(r, lo[k], len[k], row_key(col ? (int64_t)c0[k] : r, n_vox, len[k]));
    }
}

// Pass 1: rows per (matrix, key), one workgroup histogram per chunk.
__global__ __launch_bounds__(T256) void k_mlem_count(int64_t n_bins, int64_t n_vox,
                                                     const int64_t* __restrict__ T_rp,
                                                     const int32_t* __restrict__ T_col,
                                                     const int64_t* __restrict__ Tt_rp,
                                                     uint32_t* __restrict__ st) {
    __shared__ uint32_t h[N_KEY];
    if (st[ST_BAD]) return;
    const int64_t nbc = (n_bins + ROW_CHUNK - 1) / ROW_CHUNK, nvc = (n_vox + ROW_CHUNK - 1) / ROW_CHUNK;
    for (int64_t c = blockIdx.x; c < nbc + nvc; c += gridDim.x) {
        const bool vox = c >= nbc;
        if (threadIdx.x < N_KEY) h[threadIdx.x] = 0;
        __syncthreads();
        for_listed_rows((vox ? c - nbc : c) * ROW_CHUNK, vox ? n_vox : n_bins, vox ? Tt_rp : T_rp,
                        vox ? nullptr : T_col, n_vox,
                        [&](int64_t, int64_t, int64_t, int key) { atomicAdd(&h[key], 1u); });
        __syncthreads();
        if (threadIdx.x < N_KEY && h[threadIdx.x])
            atomicAdd(&st[ST_HIST + (vox ? N_KEY : 0) + threadIdx.x], h[threadIdx.x]);
        __syncthreads();
    }
}

// Pass 2 (one thread): each key's first list position, the list lengths,
// cursors zeroed.
__global__ void k_mlem_offsets(uint32_t* __restrict__ st) {
    if (threadIdx.x != 0 || blockIdx.x != 0 || st[ST_BAD]) return;
    for (int m = 0; m < 2; ++m) {
        uint32_t at = 0;
        for (int k = 0; k < N_KEY; ++k) {
            st[ST_OFF + m * N_KEY + k] = at;
            st[ST_CUR + m * N_KEY + k] = 0;
            at += st[ST_HIST + m * N_KEY + k];
        }
        st[m == 0 ? ST_BINS : ST_VOXS] = at;
    }
}

// Pass 3: each non-empty row at the next position of its key (one atomic per
// key and workgroup chunk; the order within a key varies from call to call,
// which changes no result: every row is summed by one lane group on its
// own); pos[row] = its position, -1 for an empty row.
__global__ __launch_bounds__(T256) void k_mlem_place(int64_t n_bins, int64_t n_vox,
                                                     const int64_t* __restrict__ T_rp,
                                                     const int32_t* __restrict__ T_col,
                                                     const int64_t* __restrict__ Tt_rp,
                                                     ClassRef* __restrict__ bins, ClassRef* __restrict__ voxs,
                                                     int32_t* __restrict__ bin_pos, int32_t* __restrict__ vox_pos,
                                                     uint32_t* __restrict__ st) {
    __shared__ uint32_t h[N_KEY], base[N_KEY];
    if (st[ST_BAD]) return;
    const int64_t nbc = (n_bins + ROW_CHUNK - 1) / ROW_CHUNK, nvc = (n_vox + ROW_CHUNK - 1) / ROW_CHUNK;
    for (int64_t c = blockIdx.x; c < nbc + nvc; c += gridDim.x) {
        const bool vox = c >= nbc;
        const int64_t r0 = (vox ? c - nbc : c) * ROW_CHUNK, nr = vox ? n_vox : n_bins;
        const int64_t* rp = vox ? Tt_rp : T_rp;
        int32_t* pos = vox ? vox_pos : bin_pos;
        ClassRef* out = vox ? voxs : bins;
        const uint32_t* off = st + ST_OFF + (vox ? N_KEY : 0);
        if (threadIdx.x < N_KEY) h[threadIdx.x] = 0;
        __syncthreads();
        // rank within the chunk's rows of the same key (packed: key << 16 | rank)
        uint32_t kr[ROWS_PER_THREAD];
#pragma unroll
        for (int k = 0; k < ROWS_PER_THREAD; ++k) kr[k] = 0xFFFFFFFFu;
        for_listed_rows(r0, nr, rp, vox ? nullptr : T_col, n_vox, [&](int64_t r, int64_t, int64_t, int key) {
            kr[(r - r0) / T256] = ((uint32_t)key << 16) | atomicAdd(&h[key], 1u);
        });
        __syncthreads();
        if (threadIdx.x < N_KEY)
            base[threadIdx.x] = h[threadIdx.x] ? atomicAdd(&st[ST_CUR + (vox ? N_KEY : 0) + threadIdx.x],
                                                           h[threadIdx.x])
                                               : 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ROWS_PER_THREAD; ++k) {
            const int64_t r = r0 + k * T256 + threadIdx.x;
            if (r < nr) {
                int32_t q = -1;
                if (kr[k] != 0xFFFFFFFFu) {
                    const uint32_t key = kr[k] >> 16;
                    q = (int32_t)(off[key] + base[key] + (kr[k] & 0xFFFFu));
                    const int64_t lo = rp[r];
                    out[q] = ClassRef{(int32_t)r, (uint32_t)lo, (int32_t)(rp[r + 1] - lo), 0};
                }
                pos[r] = q;
            }
        }
        __syncthreads();     // h and base are rewritten for the next chunk
    }
}

// One (group, class) list by lane groups of GS (workgroup `block` of n_blocks
// for it), one row per group and pass.  aux(q) loads the row's own operands,
// done(q, aux, sum) runs on the group's first lane; q is the list position.
template <int GS, class Aux, class Term, class Done>
__device__ inline void sweep_key(int64_t block, int64_t n_blocks, const ClassRef* __restrict__ L,
                                 uint32_t first, uint32_t n, Aux aux, Term term, Done done) {
    const RowGroups<GS> G(block, n_blocks);
    for (int64_t r = G.first; r < (int64_t)n; r += G.step) {
        const ClassRef ref = L[first + r];
        const uint32_t q = first + (uint32_t)r;
        const auto a = aux(q);
        const double sum = group_row_sum<GS>(ref.lo, (int64_t)ref.lo + ref.len, G.sub, term);
        if (G.sub == 0) done(q, a, sum);
    }
}

// Class 0 (rows of at most four entries), one lane per row: the row's
// ClassRef and its ShortRow load together, then its (up to) four gathers.
// The terms are added in group_row_sum<1>'s order (a term past the row's
// length is 0), so the sum is the same bit for bit.
template <class Aux, class Gather, class Done>
__device__ inline void sweep_key_short(int64_t block, int64_t n_blocks, const ClassRef* __restrict__ L,
                                       const ShortRow* __restrict__ E, uint32_t first, uint32_t n, Aux aux,
                                       Gather gather, Done done) {
    const RowGroups<1> G(block, n_blocks);
    for (int64_t r = G.first; r < (int64_t)n; r += G.step) {
        const uint32_t q = first + (uint32_t)r;
        const int32_t len = L[q].len;
        const ShortRow e = E[q];
        const auto a = aux(q);
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = (double)e.val[k] * gather(e.col[k]);
            acc += k < len ? x : 0.0;
        }
        done(q, a, acc);
    }
}

// The (group, class) lists of one matrix in one launch: workgroups [b.x, b.y)
// sweep class 0, [b.y, b.z) class 1, [b.z, b.w) class 2, [b.w, gridDim.x)
// class 3 (every range a multiple of N_GROUP); within a class, workgroup b
// works on group b mod N_GROUP.  key_st: that matrix's counts (ST_HIST) and
// first positions (ST_OFF).
template <class Aux, class Term, class Gather, class Done>
__device__ inline void sweep_keys(const ClassRef* __restrict__ L, const ShortRow* __restrict__ E,
                                  const uint32_t* __restrict__ hist, const uint32_t* __restrict__ off,
                                  const uint32_t* __restrict__ call_bad, int4 b, Aux aux, Term term,
                                  Gather gather, Done done) {
    const int64_t k = blockIdx.x;
    const int g = (int)(k % N_GROUP);
    int c;
    int64_t lo, hi;
    if (k < b.y) { c = 0; lo = b.x; hi = b.y; }
    else if (k < b.z) { c = 1; lo = b.y; hi = b.z; }
    else if (k < b.w) { c = 2; lo = b.z; hi = b.w; }
    else { c = 3; lo = b.w; hi = gridDim.x; }
    const int key = g * N_CLASS + c;
    // a call that does not match the set-up sweeps nothing (the three loads
    // are independent)
    const uint32_t first = off[key], n = *call_bad ? 0u : hist[key];
    const int64_t blk = (k - lo) / N_GROUP, nblk = (hi - lo) / N_GROUP;
    if (c == 0) sweep_key_short(blk, nblk, L, E, first, n, aux, gather, done);
    else if (c == 1) sweep_key<4>(blk, nblk, L, first, n, aux, term, done);
    else if (c == 2) sweep_key<16>(blk, nblk, L, first, n, aux, term, done);
    else sweep_key<64>(blk, nblk, L, first, n, aux, term, done);
}

// Compact forward: ratio_q = P_q / (sum_k val_k S[col_k]) over the bin rows,
// S, P, ratio in list order and col renumbered to voxel list positions.
__global__ __launch_bounds__(T256) void k_mlem_forward_c(const ClassRef* __restrict__ L,
                                                         const ShortRow* __restrict__ E,
                                                         const uint32_t* __restrict__ st, int4 b,
                                                         const int32_t* __restrict__ col,
                                                         const float* __restrict__ val,
                                                         const double* __restrict__ S,
                                                         const float* __restrict__ P,
                                                         double* __restrict__ ratio) {
    sweep_keys(L, E, st + ST_HIST, st + ST_OFF, st + ST_CALL_BAD, b, [&](uint32_t q) { return P[q]; },
               [&](int64_t k, bool ok) {
                   const double x = (double)val[k] * S[col[k]];
                   return ok ? x : 0.0;
               },
               [&](int32_t c) { return S[c]; },
               [&](uint32_t q, float p, double y) { ratio[q] = y > 0.0 ? (double)p / y : 0.0; });
}

// Compact update: S_q <- S_q (sum_k val_k ratio[col_k]) / sens_q over the
// voxel rows, in list order, col renumbered to bin list positions.
__global__ __launch_bounds__(T256) void k_mlem_update_c(const ClassRef* __restrict__ L,
                                                        const ShortRow* __restrict__ E,
                                                        const uint32_t* __restrict__ st, int4 b,
                                                        const int32_t* __restrict__ col,
                                                        const float* __restrict__ val,
                                                        const double* __restrict__ ratio,
                                                        const double* __restrict__ sens,
                                                        double* __restrict__ S) {
    sweep_keys(L, E, st + ST_HIST + N_KEY, st + ST_OFF + N_KEY, st + ST_CALL_BAD, b,
               [&](uint32_t q) { return double2{S[q], sens[q]}; },
               [&](int64_t k, bool ok) {
                   const double x = (double)val[k] * ratio[col[k]];
                   return ok ? x : 0.0;
               },
               [&](int32_t c) { return ratio[c]; },
               [&](uint32_t q, double2 ss, double v) { S[q] = ss.y > 0.0 ? ss.x * v / ss.y : 0.0; });
}

// image_i = S_i (row order; vox_pos given: S in list order, 0 for an empty
// row), NaN throughout when the bad flag of st (nullable) is set.
__global__ __launch_bounds__(T256) void k_mlem_out(int64_t n_vox, const double* __restrict__ S,
                                                   const int32_t* __restrict__ vox_pos,
                                                   const uint32_t* __restrict__ st,
                                                   float* __restrict__ img) {
    const bool bad = st && (st[ST_BAD] != 0 || st[ST_CALL_BAD] != 0);
    for (int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x; i < n_vox;
         i += (int64_t)gridDim.x * T256) {
        float v;
        if (bad) {
            v = __builtin_nanf("");
        } else if (vox_pos) {
            const int32_t p = vox_pos[i];
            v = p >= 0 ? (float)S[p] : 0.0f;
        } else {
            v = (float)S[i];
        }
        img[i] = v;
    }
}

// ---- ordered subsets (OSEM; dual matrix, Eq. DMOS; additive scatter, the
// Sohlberg OS-EM equation).  Subset k holds the views v with v mod n_sub == k.

// The backprojector split by subset, built once per call, so that a subset's
// backprojection reads that subset's entries only instead of the whole of B^T
// once per subset.  A workgroup takes a chunk of consecutive rows and writes
// their entries subset by subset, within a subset row by row in their order
// in the row, into the chunk's own range of the copy: nothing has to be
// counted over the whole matrix first.  offs[(chunk n_sub + k) (per + 1) + i]:
// where row i of the chunk starts in subset k, relative to the chunk's first
// entry (i = n: its end).  Each of 16 wavefronts (4 for a small
// matrix) takes a share of the chunk's rows and goes over their entries
// 64 at a time, SPLIT_LOADS groups loaded ahead (row by row, a wavefront waits
// for each row's loads in turn); lanes of one row and subset are matched by a
// ballot per bit of the subset's number.
// Bound by reading B^T (twice, the second time from L2) and writing it once:
// 8.6e6 entries of 2.6e5 rows in 6 subsets took 230 us as a count, a scan and
// a scatter over single rows, 82 us now.
constexpr int OS_LOADS = 8;
constexpr int SPLIT_COUNTS = 4096;     // (subset, row) pairs of a chunk, counters in LDS
static_assert(OSEM_MAX_SUBSETS <= SPLIT_COUNTS, "a row's counters at least");
constexpr int SPLIT_LOADS = 4;

// Rows per chunk: a subset's share of them fills three eighths of a tile on
// average, as dense regions hold several times the mean (with twice as many rows
// the 12 updates and the split of 2.6e5 rows, 5.5 entries of each in a subset,
// took 573 against 437 us, with half 495).  Of a small matrix no more than
// leave the split enough workgroups, of 256 threads there (2e5 entries: 35 us
// with 1024).
inline int split_per(int64_t nnz, int64_t n_bins, int64_t n_vox, int n_sub) {
    int64_t per = sweep_per(OS_LOADS, nnz / n_vox * 2 / n_sub);
    if (nnz < SWEEP_MIN_NNZ) per = std::min<int64_t>(per, std::min<int64_t>(64, n_vox / 3072));
    per = std::min<int64_t>(per, SPLIT_COUNTS / n_sub);
    // a chunk's entries are counted in 32 bits
    if (nnz > INT32_MAX) per = std::min<int64_t>(per, INT32_MAX / n_bins);
    return (int)std::max<int64_t>(1, std::min<int64_t>(per, n_vox));
}

// st[2] (as for MLEM: the image is NaN when set): the entry count the caller
// gave is not B^T's own.
__global__ void k_os_check(int64_t n_vox, const int64_t* __restrict__ rp, int64_t nnz,
                           uint32_t* __restrict__ st) {
    if (blockIdx.x == 0 && threadIdx.x < 4) st[threadIdx.x] = threadIdx.x == 2 ? (rp[n_vox] != nnz) : 0u;
}

// Subset of a bin, (bin / bins_per_view) mod n_sub, with the quotients from
// products with FP64 reciprocals: (x + 1/2) / d lies at least 1 / (2 d) from
// every integer, and the product is off by less than that for x < 2^31.
struct SubsetOf {
    double inv_view, inv_sub;
    int32_t n_sub;
    __device__ SubsetOf(int32_t bins_per_view, int32_t n) : inv_view(1.0 / bins_per_view), inv_sub(1.0 / n), n_sub(n) {}
    __device__ __forceinline__ int operator()(int32_t bin) const {
        const int32_t view = (int32_t)(((double)bin + 0.5) * inv_view);
        return view - n_sub * (int32_t)(((double)view + 0.5) * inv_sub);
    }
};

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_os_split(int64_t n_vox, int per, const int64_t* __restrict__ rp,
                                                      const int32_t* __restrict__ col,
                                                      const float* __restrict__ val, int32_t bins_per_view,
                                                      int32_t n_sub, int32_t* __restrict__ offs,
                                                      int32_t* __restrict__ col_s, float* __restrict__ val_s,
                                                      const uint32_t* __restrict__ st) {
    __shared__ uint32_t cnt[SPLIT_COUNTS];      // [subset][row]: counts, then next free slots
    __shared__ uint32_t part[THREADS / 64];
    __shared__ int32_t roff[T256 + 1];           // the rows' first entries in the chunk
    const int64_t c = sweep_chunk(), r0 = c * per;
    if (r0 >= n_vox) return;
    const int n = (int)std::min<int64_t>(per, n_vox - r0), total = n * n_sub;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool bad = st[2] != 0;
    const int64_t e0 = rp[r0];
    const SubsetOf subset_of(bins_per_view, n_sub);
    for (int i = tid; i < total; i += THREADS) cnt[i] = 0;
    for (int i = tid; i <= n; i += THREADS) roff[i] = (int32_t)(rp[r0 + i] - e0);
    __syncthreads();
    // this wavefront's rows and entries
    constexpr int WAVES = THREADS / 64;
    const int ra = __builtin_amdgcn_readfirstlane(n * wave / WAVES);
    const int rb = __builtin_amdgcn_readfirstlane(n * (wave + 1) / WAVES);
    const int ea = bad ? 0 : __builtin_amdgcn_readfirstlane(roff[ra]);
    const int eb = bad ? 0 : __builtin_amdgcn_readfirstlane(roff[rb]);
    const int32_t* __restrict__ cols = col + e0;
    // the row holding entry e: the last one starting at or before it
    const auto row_of = [&](int e) {
        int lo = ra, hi = rb - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (roff[mid] <= e) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    for (int g = ea; g < eb; g += 64 * SPLIT_LOADS) {
        int32_t cc[SPLIT_LOADS];
#pragma unroll
        for (int u = 0; u < SPLIT_LOADS; ++u) {
            const int e = g + u * 64 + lane;
            cc[u] = cols[(uint32_t)(e < eb ? e : eb - 1)];
        }
#pragma unroll
        for (int u = 0; u < SPLIT_LOADS; ++u) {
            const int e = g + u * 64 + lane;
            if (e < eb) atomicAdd(&cnt[subset_of(cc[u]) * n + row_of(e)], 1u);
        }
    }
    __syncthreads();
    // exclusive scan, SPLIT_COUNTS / THREADS consecutive counters per thread
    constexpr int PER = SPLIT_COUNTS / THREADS;
    uint32_t mine[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid * PER + u;
        mine[u] = i < total ? cnt[i] : 0u;
        sum += mine[u];
    }
    uint32_t x = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t run = x - sum;
    for (int w = 0; w < wave; ++w) run += part[w];
    int32_t* out = offs + c * n_sub * (int64_t)(per + 1);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid * PER + u;
        if (i < total) {
            const int k = i / n, r = i - k * n;
            cnt[i] = run;
            out[k * (per + 1) + r] = (int32_t)run;
            run += mine[u];
            if (r == n - 1) out[k * (per + 1) + n] = (int32_t)run;
        }
    }
    __syncthreads();
    const float* __restrict__ vals = val + e0;
    int32_t* __restrict__ col_o = col_s + e0;
    float* __restrict__ val_o = val_s + e0;
    const uint64_t lane_lt = (1ull << lane) - 1ull;
    for (int g = ea; g < eb; g += 64 * SPLIT_LOADS) {
        int32_t cc[SPLIT_LOADS];
        float v[SPLIT_LOADS];
#pragma unroll
        for (int u = 0; u < SPLIT_LOADS; ++u) {
            const int e = g + u * 64 + lane;
            cc[u] = cols[(uint32_t)(e < eb ? e : eb - 1)];
            v[u] = vals[(uint32_t)(e < eb ? e : eb - 1)];
        }
#pragma unroll
        for (int u = 0; u < SPLIT_LOADS; ++u) {
            const int e = g + u * 64 + lane;
            const bool ok = e < eb;
            const int k = subset_of(cc[u]), r = row_of(ok ? e : eb - 1);
            // the lanes of this row, then of this subset
            const int first = roff[r] - (e - lane), end = roff[r + 1] - (e - lane);
            uint64_t peers = __ballot(ok) & (first > 0 ? ~0ull << first : ~0ull) & (end < 64 ? (1ull << end) - 1ull : ~0ull);
            for (int b = 0; (n_sub - 1) >> b; ++b) {
                const bool bit = (k >> b) & 1;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & lane_lt);
            if (ok) {
                const uint32_t at = cnt[k * n + r];
                col_o[at + rank] = cc[u];
                val_o[at + rank] = v[u];
                if (rank == 0) cnt[k * n + r] = at + (uint32_t)__popcll(peers);
            }
            // the next group reads the slots this one moved
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Subset k's part of chunk c of the split backprojector, swept.
template <class Load, class Value, class Done>
__device__ inline void sweep_split(int64_t c, int k, int64_t n_vox, int per, int n_sub,
                                   const int64_t* __restrict__ rp, const int32_t* __restrict__ offs, Load load,
                                   Value value, Done done) {
    const int64_t r0 = c * per;
    const int32_t* __restrict__ o = offs + (c * n_sub + k) * (int64_t)(per + 1);
    sweep_bounds<OS_LOADS>(r0, (int)std::min<int64_t>(per, n_vox - r0), false, rp[r0], [&](int i) { return (int64_t)o[i]; }, load,
                 value, done);
}

// sens[k * n_vox + i] = sum of row i's values in subset k (blockIdx.y: k)
__global__ __launch_bounds__(T256) void k_os_sums(int64_t n_vox, int per, int n_sub, const int64_t* __restrict__ rp,
                                                  const int32_t* __restrict__ offs, const float* __restrict__ val,
                                                  double* __restrict__ sens) {
    const int64_t c = sweep_chunk(), r0 = c * per;
    if (r0 >= n_vox) return;
    const int k = (int)blockIdx.y, i = (int)(threadIdx.x);
    double* out = sens + k * n_vox;
    const int32_t* o = offs + (c * n_sub + k) * (int64_t)(per + 1);
    if (i < per && r0 + i < n_vox && o[i] == o[i + 1]) out[r0 + i] = 0.0;
    sweep_split(c, k, n_vox, per, n_sub, rp, offs,
                [&](int64_t first, int e) { return *(val + first + (uint32_t)e); },
                [](float x) { return (double)x; }, [&](int64_t r, double acc) { out[r] = acc; });
}

__global__ __launch_bounds__(T256) void k_os_init(int64_t n_vox, int32_t n_sub,
                                                  const float* __restrict__ img,
                                                  const double* __restrict__ sens,
                                                  double* __restrict__ S) {
    for (int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x; i < n_vox;
         i += (int64_t)gridDim.x * T256) {
        double tot = 0.0;
        for (int k = 0; k < n_sub; ++k) tot += sens[(int64_t)k * n_vox + i];
        S[i] = tot > 0.0 ? (double)img[i] : 0.0;
    }
}

// subset k: y_j = sum_i c_ij S_i + s_j, ratio_j = P_j / y_j on the subset's
// bins: views k, k + n_sub, ..., each in chunks of `per` rows.
__global__ __launch_bounds__(T256) void k_os_forward(int64_t n_chunks, int32_t per_view, int per,
                                                     int32_t bins_per_view, int32_t n_sub, int32_t k,
                                                     const int64_t* __restrict__ rp,
                                                     const int32_t* __restrict__ col,
                                                     const float* __restrict__ val,
                                                     const double* __restrict__ S,
                                                     const float* __restrict__ P,
                                                     const float* __restrict__ scat,
                                                     double* __restrict__ ratio) {
    const int64_t c = sweep_chunk();
    if (c >= n_chunks) return;
    const int32_t in_view = (int32_t)(c % per_view) * per;
    const int64_t r0 = (k + n_sub * (c / per_view)) * bins_per_view + in_view;
    const int n = std::min(per, bins_per_view - in_view);
    const auto done = [&](int64_t j, double y) {
        y += scat ? (double)scat[j] : 0.0;
        ratio[j] = y > 0.0 ? (double)P[j] / y : 0.0;
    };
    // a bin without entries still has its scatter term
    const int i = (int)(threadIdx.x);
    if (i < n && rp[r0 + i] == rp[r0 + i + 1]) done(r0 + i, 0.0);
    sweep<OS_LOADS>(r0, n, false, rp, [&](int64_t first, int k) { return load_entry(col, val, first, k); },
             [&](Entry e) { return (double)e.val * S[e.col]; }, done);
}

// subset k: S_i <- S_i * (sum_{j in k} b_ij ratio_j) / sens_k,i (unchanged
// where sens_k,i = 0), over subset k's part of the split backprojector.
__global__ __launch_bounds__(T256) void k_os_update(int64_t n_vox, int per, int n_sub, int k,
                                                    const int64_t* __restrict__ rp,
                                                    const int32_t* __restrict__ offs,
                                                    const int32_t* __restrict__ col,
                                                    const float* __restrict__ val,
                                                    const double* __restrict__ ratio,
                                                    const double* __restrict__ sens_k,
                                                    double* __restrict__ S) {
    const int64_t c = sweep_chunk();
    if (c * per >= n_vox) return;
    sweep_split(c, k, n_vox, per, n_sub, rp, offs,
                [&](int64_t first, int e) { return load_entry(col, val, first, e); },
                [&](Entry e) { return (double)e.val * ratio[e.col]; },
                [&](int64_t i, double b) {
                    const double si = sens_k[i];
                    if (si > 0.0) S[i] = S[i] * b / si;
                });
}

// The same with a row per group of GS lanes and pass, as for MLEM: for matrices
// that stay in the caches, and for sparse ones, most of whose rows are empty
// (1.2e5 entries in 2.0e6 bins x 2.6e5 voxels, 80 subset updates: 1050 us
// with the tiles, 745 us so).
// Forward rows: row t of subset k is a bin of view k + n_sub (t / bins_per_view).
struct OsForward {
    const int64_t* __restrict__ rp;
    const int32_t* __restrict__ col;
    const float* __restrict__ val;
    const double* __restrict__ S;
    const float* __restrict__ P;
    const float* __restrict__ scat;
    double* __restrict__ ratio;
    int64_t n_rows, n_bins;
    int32_t bins_per_view, n_sub, k;

    __device__ int64_t bin(int64_t t) const {
        const uint32_t v = (uint32_t)t / (uint32_t)bins_per_view;      // fewer than 2^31 bins
        return t + (int64_t)(k + (n_sub - 1) * (int64_t)v) * bins_per_view;
    }
    template <int GS>
    __device__ void row(int64_t j, int64_t lo, int64_t hi, float p, float s, int sub) const {
        double y = 0.0;
        if (hi > lo)
            y = group_row_sum<GS>(lo, hi, sub, [&](int64_t e, bool ok) {
                const double x = (double)val[e] * S[col[e]];
                return ok ? x : 0.0;
            });
        y += scat ? (double)s : 0.0;
        if (sub == 0) ratio[j] = y > 0.0 ? (double)p / y : 0.0;
    }
};

// This group's rows; j, lo, hi: the first one's bin and bounds.
template <int GS>
__device__ inline void os_forward(const OsForward& F, const RowGroups<GS>& G, int64_t j, int64_t lo, int64_t hi) {
    for (int64_t t = G.first; t < F.n_rows; t += G.step) {
        if (t != G.first) {
            j = F.bin(t);
            lo = F.rp[j];
            hi = F.rp[j + 1];
        }
        const float p = F.P[j], s = F.scat ? F.scat[j] : 0.0f;
        F.row<GS>(j, lo, hi, p, s, G.sub);
    }
}
template <int GS>
__device__ inline void os_forward(const OsForward& F) {
    const RowGroups<GS> G(blockIdx.x, gridDim.x);
    if (G.first >= F.n_rows) return;
    const int64_t j = F.bin(G.first);
    os_forward<GS>(F, G, j, F.rp[j], F.rp[j + 1]);
}

// GS: the lanes per row for c as dense as b, whose entry count the call knows.
// c's own count is read along with the first row's bounds, and where it asks for
// other lanes (a dual matrix: c with scatter, b without), they do it, on at
// least OS_FORWARD_BLOCKS workgroups if 64 lanes per row would take as many:
// c of 6.4e6 entries with b of 1.1e5, 245760 bins, 4 updates of 1 / 24 of 6
// subsets: 399 / 755 us with b's lanes, 249 / 772 with c's on the few workgroups
// of one lane per row, 235 / 386 now.  Workgroups without rows cost nothing
// that shows (1.8e5 to 8e6 entries, b = c).
constexpr int OS_FORWARD_BLOCKS = 4096;

template <int GS>
__global__ __launch_bounds__(T256) void k_os_forward_rows(OsForward F) {
    const RowGroups<GS> G(blockIdx.x, gridDim.x);
    const int64_t c_nnz = F.rp[F.n_bins];
    const int64_t j = F.bin(G.first < F.n_rows ? G.first : F.n_rows - 1);
    const int64_t lo = F.rp[j], hi = F.rp[j + 1];
    asm volatile("" ::"s"(c_nnz), "v"(lo), "v"(hi));     // all in flight before the count is tested
    switch (lanes_per_row(c_nnz, F.n_bins, 4)) {
        case GS: os_forward<GS>(F, G, j, lo, hi); break;
        case GS == 1 ? 4 : 1: os_forward<GS == 1 ? 4 : 1>(F); break;
        case GS <= 4 ? 16 : 4: os_forward<GS <= 4 ? 16 : 4>(F); break;
        default: os_forward<GS <= 16 ? 64 : 16>(F); break;
    }
}

// Row i's entries in subset k of the split: from first + lo to first + hi.
struct SplitRow {
    int64_t first;
    int32_t lo, hi;
};
__device__ __forceinline__ SplitRow split_row(int64_t i, int k, int per, int n_sub, const int64_t* __restrict__ rp,
                                              const int32_t* __restrict__ offs) {
    const uint32_t c = (uint32_t)i / (uint32_t)per, r = (uint32_t)i - c * (uint32_t)per;
    const int32_t* __restrict__ o = offs + ((int64_t)c * n_sub + k) * (int64_t)(per + 1) + r;
    return SplitRow{rp[(int64_t)c * per], o[0], o[1]};
}

template <int GS>
__global__ __launch_bounds__(T256) void k_os_sums_rows(int64_t n_vox, int per, int n_sub,
                                                       const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ offs,
                                                       const float* __restrict__ val, double* __restrict__ sens) {
    const RowGroups<GS> G(blockIdx.x, gridDim.x);
    for (int64_t i = G.first; i < n_vox; i += G.step) {
        const SplitRow x = split_row(i, (int)blockIdx.y, per, n_sub, rp, offs);
        double b = 0.0;
        if (x.lo != x.hi)
            b = group_row_sum<GS>(x.first + x.lo, x.first + x.hi, G.sub,
                                  [&](int64_t e, bool ok) { return ok ? (double)val[e] : 0.0; });
        if (G.sub == 0) sens[(int)blockIdx.y * n_vox + i] = b;
    }
}

template <int GS>
__global__ __launch_bounds__(T256) void k_os_update_rows(int64_t n_vox, int per, int n_sub, int k,
                                                         const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ offs,
                                                         const int32_t* __restrict__ col,
                                                         const float* __restrict__ val,
                                                         const double* __restrict__ ratio,
                                                         const double* __restrict__ sens_k,
                                                         double* __restrict__ S) {
    const RowGroups<GS> G(blockIdx.x, gridDim.x);
    for (int64_t i = G.first; i < n_vox; i += G.step) {
        const SplitRow r = split_row(i, k, per, n_sub, rp, offs);
        if (r.lo == r.hi) continue;
        const double si = sens_k[i], s = S[i];
        const double b = group_row_sum<GS>(r.first + r.lo, r.first + r.hi, G.sub, [&](int64_t e, bool ok) {
            const double x = (double)val[e] * ratio[col[e]];
            return ok ? x : 0.0;
        });
        if (G.sub == 0 && si > 0.0) S[i] = s * b / si;
    }
}

}  // namespace


// OSEM workspace: per-subset sensitivities, S, the ratio, the check word,
// and the subset-split backprojector (row bounds, columns and values).
struct OsemLayout {
    size_t sens, S, ratio, st, offs, col_s, val_s, total;
};

OsemLayout osem_layout(uint64_t n_bins, uint64_t n_vox, uint32_t n_sub, uint64_t nnz) {
    OsemLayout L{};
    size_t o = 0;
    auto take = [&](uint64_t bytes) {
        const size_t at = o;
        o += (bytes + 255) & ~(uint64_t)255;
        return at;
    };
    const uint64_t rows = (uint64_t)n_sub * n_vox;
    L.sens = take(8 * rows);
    L.S = take(8 * n_vox);
    L.ratio = take(8 * n_bins);
    L.st = take(16);
    L.offs = take(8 * rows);       // (per + 1) int32 per chunk and subset: at most two per row
    L.col_s = take(4 * nnz);
    L.val_s = take(4 * nnz);
    L.total = o;
    return L;
}

size_t osem_workspace(uint64_t n_bins, uint64_t n_vox, uint32_t n_sub, uint64_t bt_nnz) {
    return osem_layout(n_bins, n_vox, n_sub, bt_nnz).total;
}

hipError_t launch_osem(int64_t n_bins, int64_t n_vox, int32_t bins_per_view, int32_t n_sub,
                       const int64_t* C_rp, const int32_t* C_col, const float* C_val,
                       const int64_t* Bt_rp, const int32_t* Bt_col, const float* Bt_val, int64_t bt_nnz,
                       const float* proj, const float* scatter, float* image, int32_t n_iter,
                       void* workspace, hipStream_t s) {
    const OsemLayout L = osem_layout((uint64_t)n_bins, (uint64_t)n_vox, (uint32_t)n_sub, (uint64_t)bt_nnz);
    char* w = (char*)workspace;
    double* sens = (double*)(w + L.sens);
    double* S = (double*)(w + L.S);
    double* ratio = (double*)(w + L.ratio);
    uint32_t* st = (uint32_t*)(w + L.st);
    int32_t* offs = (int32_t*)(w + L.offs);
    int32_t* col_s = (int32_t*)(w + L.col_s);
    float* val_s = (float*)(w + L.val_s);
    const int64_t n_views = n_bins / bins_per_view;
    const int gv = grid_for((uint64_t)n_vox, T256, 8192);
    const int per = split_per(bt_nnz, n_bins, n_vox, n_sub);
    const int64_t n_chunks = (n_vox + per - 1) / per;
    const unsigned grid_v = sweep_grid(n_chunks);
    // a subset's voxel rows are short and uneven: two entries per lane (four:
    // 11.5 us per update, 4.3e4 voxels of 4 entries)
    const int g_f = os_lanes(bt_nnz, bt_nnz, n_bins, 4), g_u = os_lanes(bt_nnz, bt_nnz / n_sub, n_vox, 2);
    const unsigned gu = g_u ? (unsigned)grid_for((uint64_t)n_vox * g_u, T256, 1 << 16) : grid_v;
    k_os_check<<<1, 64, 0, s>>>(n_vox, Bt_rp, bt_nnz, st);
    if (bt_nnz < SWEEP_MIN_NNZ)
        k_os_split<256><<<grid_v, 256, 0, s>>>(n_vox, per, Bt_rp, Bt_col, Bt_val, bins_per_view, n_sub, offs,
                                               col_s, val_s, st);
    else
        k_os_split<1024><<<grid_v, 1024, 0, s>>>(n_vox, per, Bt_rp, Bt_col, Bt_val, bins_per_view, n_sub, offs,
                                                 col_s, val_s, st);
    auto ks = g_u == 0 ? k_os_sums : g_u == 1 ? k_os_sums_rows<1> : g_u == 4 ? k_os_sums_rows<4>
            : g_u == 16 ? k_os_sums_rows<16> : k_os_sums_rows<64>;
    ks<<<dim3(gu, (unsigned)n_sub), T256, 0, s>>>(n_vox, per, n_sub, Bt_rp, offs, val_s, sens);
    k_os_init<<<gv, T256, 0, s>>>(n_vox, n_sub, image, sens, S);
    // c's entry count is not known here: tiles by b's, lanes corrected on the
    // device (tiles of a c 7 times as dense, 7.3e7 entries: 1.5 ms for 4 updates;
    // by its lanes 3.6)
    const int per_f = sweep_per(OS_LOADS, bt_nnz / n_bins);
    const int32_t per_view = (bins_per_view + per_f - 1) / per_f;
    auto kf = g_f == 1 ? k_os_forward_rows<1> : g_f == 4 ? k_os_forward_rows<4>
            : g_f == 16 ? k_os_forward_rows<16> : k_os_forward_rows<64>;
    auto ku = g_u == 0 ? k_os_update : g_u == 1 ? k_os_update_rows<1> : g_u == 4 ? k_os_update_rows<4>
            : g_u == 16 ? k_os_update_rows<16> : k_os_update_rows<64>;
    for (int it = 0; it < n_iter; ++it) {
        for (int k = 0; k < n_sub; ++k) {
            const int64_t views = (n_views - k + n_sub - 1) / n_sub, chunks = views * per_view;
            if (chunks <= 0) continue;
            if (g_f)
                kf<<<std::max(grid_for((uint64_t)(views * bins_per_view) * g_f, T256, 1 << 16),
                              grid_for((uint64_t)(views * bins_per_view) * 64, T256, OS_FORWARD_BLOCKS)),
                     T256, 0, s>>>(OsForward{C_rp, C_col, C_val, S, proj, scatter, ratio, views * bins_per_view,
                                             n_bins, bins_per_view, n_sub, k});
            else
                k_os_forward<<<sweep_grid(chunks), T256, 0, s>>>(chunks, per_view, per_f, bins_per_view, n_sub,
                                                                       k, C_rp, C_col, C_val, S, proj, scatter,
                                                                       ratio);
            ku<<<gu, T256, 0, s>>>(n_vox, per, n_sub, k, Bt_rp, offs, col_s, val_s, ratio,
                                   sens + (uint64_t)k * (uint64_t)n_vox, S);
        }
    }
    k_mlem_out<<<gv, T256, 0, s>>>(n_vox, S, nullptr, st, image);
    return hipGetLastError();
}

// Workspace of the response-matrix build (layout in sysmat_layout).
struct SysLayout {
    uint32_t* hist;        // [RADIX * n_tiles] digit histograms, then their scans
    uint32_t* tot;         // [RADIX] digit totals
    uint32_t* cnt;         // [n_runs] runs per tile of the sorted events
    uint64_t* first;       // [n_runs + 1] their exclusive scan; the last: nnz
    uint64_t* bsum;        // scan block sums
    uint64_t* keys[2];     // [cap] sort keys (double buffer), then the entries' 32-bit keys
    uint64_t* vals[2];     // [cap] weights, Q31.32, then the entries' (bin, value) pairs
    unsigned long long* a_img;   // [n_img] activity per image voxel
    unsigned long long* total;   // [TOTAL_SLOTS] partial sums of the activity
    unsigned long long* acc;     // [n_bins] summed weight per bin
    uint32_t n_tiles, n_runs;
    size_t bytes;
};

SysLayout sysmat_layout(char* w, uint64_t n_bins, uint64_t n_img, uint64_t capacity) {
    auto al = [](uint64_t x) { return (x + 255) & ~(uint64_t)255; };
    const uint64_t cap = capacity ? capacity : 1;
    SysLayout L;
    L.n_tiles = (uint32_t)((cap + RADIX_TILE - 1) / RADIX_TILE);
    L.n_runs = (uint32_t)((cap + RUN_TILE - 1) / RUN_TILE);
    char* p = w;
    auto take = [&](uint64_t bytes) { char* q = p; p += al(bytes); return q; };
    L.hist = (uint32_t*)take(4ull * RADIX * L.n_tiles);
    L.tot = (uint32_t*)take(4 * RADIX);
    L.cnt = (uint32_t*)take(4ull * L.n_runs);
    L.first = (uint64_t*)take(8 * (L.n_runs + 1ull));
    L.bsum = (uint64_t*)take(8 * (L.n_runs / SCAN_BLOCK + 1ull));
    L.keys[0] = (uint64_t*)take(8 * cap);
    L.keys[1] = (uint64_t*)take(8 * cap);
    L.vals[0] = (uint64_t*)take(8 * cap);
    L.vals[1] = (uint64_t*)take(8 * cap);
    // zeroed together: one array
    L.a_img = (unsigned long long*)take(8 * (n_img + TOTAL_SLOTS + n_bins));
    L.total = L.a_img + n_img;
    L.acc = L.total + TOTAL_SLOTS;
    L.bytes = (size_t)(p - w);
    return L;
}

// Digits of a sort over `bits` bits: the fewest passes, of equal widths.
struct Digits {
    int passes, bits;
    uint32_t mask() const { return (1u << bits) - 1u; }
};
Digits digits_of(int bits) {
    Digits d;
    d.passes = (bits + RADIX_BITS - 1) / RADIX_BITS;
    d.bits = (bits + d.passes - 1) / d.passes;
    return d;
}

size_t sysmat_workspace_bytes(uint64_t n_bins, uint64_t n_img, uint64_t capacity) {
    return sysmat_layout(nullptr, n_bins, n_img, capacity).bytes;
}

hipError_t launch_sysmat(const mc_event* events, const unsigned long long* n_events, uint64_t capacity,
                         uint32_t nx, uint32_t ny, uint32_t nz, uint32_t f, uint32_t n_views,
                         uint32_t nu, uint32_t nv, uint64_t n_hist, const uint32_t* activity,
                         uint32_t class_mask, int64_t* T_rp, int32_t* T_col, float* T_val,
                         int64_t* Tt_rp, int32_t* Tt_col, float* Tt_val, float* proj,
                         void* workspace, hipStream_t s) {
    const uint64_t n_bins = (uint64_t)n_views * nu * nv;
    const uint32_t mx = nx / f, my = ny / f, mz = nz / f;
    const uint64_t n_img = (uint64_t)mx * my * mz;
    const SysLayout L = sysmat_layout((char*)workspace, n_bins, n_img, capacity);
    const uint64_t* n_ev = (const uint64_t*)n_events;

    SysArgs a;
    a.events = events; a.n_events = n_ev; a.capacity = capacity;
    a.class_mask = class_mask;
    a.nv_nu = nu * nv;
    a.nx = nx; a.ny = ny; a.f = f; a.mx = mx; a.my = my;
    a.q_per_view = n_hist / n_views; a.r_extra = n_hist % n_views;

    const uint64_t n_zero = n_img + TOTAL_SLOTS + (proj ? n_bins : 0);
    k_fill_u64<<<grid_for(n_zero, T256, 4096), T256, 0, s>>>((uint64_t*)L.a_img, n_zero, 0);
    // an image row's f x f phantom rows in as many shares as fill the chip
    const uint64_t rows = (uint64_t)my * mz, shares = std::min<uint64_t>((uint64_t)f * f, (2047 + rows) / rows);
    k_image_activity<<<(unsigned)(rows * shares), T256, 0, s>>>(activity, nx, ny, f, mx, my, (uint32_t)shares,
                                                               L.a_img, L.total);

    // the events by (bin, voxel): rows 0..n_bins (n_bins: filtered events)
    const int col_bits = std::max(1, bit_width(n_img - 1));
    const Digits d = digits_of(col_bits + bit_width(n_bins));
    int cur = 0;
    for (int p = 0; p < d.passes; ++p) {
        if (p == 0)
            k_make_keys<<<L.n_tiles, T256, 0, s>>>(a, n_bins, col_bits, d.mask(), L.n_tiles, L.keys[0],
                                                   (int64_t*)L.vals[0], L.hist);
        else
            k_radix_hist<<<L.n_tiles, T256, 0, s>>>(L.keys[cur], n_ev, capacity, p * d.bits, d.mask(), L.n_tiles,
                                                    L.hist);
        k_digit_scan<<<RADIX, 1024, 0, s>>>(n_ev, capacity, L.n_tiles, L.hist, L.tot);
        k_radix_scatter<uint64_t><<<L.n_tiles, T256, 0, s>>>(L.keys[cur], L.vals[cur], L.keys[cur ^ 1],
                                                             L.vals[cur ^ 1], nullptr, nullptr, n_ev, capacity,
                                                             p * d.bits, d.mask(), L.n_tiles, L.hist, L.tot);
        cur ^= 1;
    }
    // merged: T, and the entries' (bin, value) pairs
    k_count_runs<<<L.n_runs, T256, 0, s>>>(L.keys[cur], a, n_bins, col_bits, L.cnt);
    hipError_t e = exclusive_scan(L.cnt, L.n_runs, L.first, L.bsum, s);
    if (e != hipSuccess) return e;
    uint64_t* pair = L.vals[cur ^ 1];
    k_emit_runs<<<L.n_runs, T256, 0, s>>>(a, L.keys[cur], (const int64_t*)L.vals[cur], L.first, n_bins, col_bits,
                                          T_col, T_val, pair, proj ? L.acc : nullptr, L.a_img, L.total);
    const uint64_t* nnz = L.first + L.n_runs;
    k_row_ptr<<<grid_for(n_bins + 1, T256, 8192), T256, 0, s>>>(pair, nnz, capacity, n_bins, T_rp,
                                                                (const int64_t*)L.acc, n_ev, proj);
    // the entries by voxel, bins in order within one: T^T
    const Digits t = digits_of(col_bits);
    const uint32_t* kin = (const uint32_t*)T_col;
    for (int p = 0; p < t.passes; ++p) {
        uint32_t* kout = (uint32_t*)L.keys[cur];
        const bool last = p == t.passes - 1;
        k_radix_hist<<<L.n_tiles, T256, 0, s>>>(kin, nnz, capacity, p * t.bits, t.mask(), L.n_tiles, L.hist);
        k_digit_scan<<<RADIX, 1024, 0, s>>>(nnz, capacity, L.n_tiles, L.hist, L.tot);
        k_radix_scatter<uint32_t><<<L.n_tiles, T256, 0, s>>>(
            kin, L.vals[cur ^ 1], kout, L.vals[cur], last ? Tt_col : nullptr, last ? Tt_val : nullptr, nnz, capacity,
            p * t.bits, t.mask(), L.n_tiles, L.hist, L.tot);
        kin = kout;
        cur ^= 1;
    }
    k_row_ptr<<<grid_for(n_img + 1, T256, 8192), T256, 0, s>>>(kin, nnz, capacity, n_img, Tt_rp,
                                                               (const int64_t*)nullptr, n_ev, (float*)nullptr);
    return hipGetLastError();
}

namespace {

// Byte offsets of mlem_iterate's workspace, for n_bins x n_vox (every array
// 256-byte aligned).  The compact layout's arrays are sized for its largest
// entry count, n_bins + n_vox.
struct MlemLayout {
    size_t sens, S, ratio, bin_rows, vox_rows, st, sens_l, P_l, bin_pos, vox_pos, Tc, Ttc, bin_short, vox_short;
    size_t total;
};

MlemLayout mlem_layout(uint64_t nb, uint64_t nv) {
    MlemLayout L{};
    size_t o = 0;
    auto take = [&](uint64_t bytes) {
        const size_t at = o;
        o += (bytes + 255) & ~(uint64_t)255;
        return at;
    };
    L.sens = take(8 * nv);
    L.S = take(8 * nv);
    L.ratio = take(8 * nb);
    L.bin_rows = take(16 * nb);
    L.vox_rows = take(16 * nv);
    L.st = take(4 * ST_WORDS);
    L.sens_l = take(8 * nv);
    L.P_l = take(4 * nb);
    L.bin_pos = take(4 * nb);
    L.vox_pos = take(4 * nv);
    L.Tc = take(4 * (nb + nv));
    L.Ttc = take(4 * (nb + nv));
    L.bin_short = take(sizeof(ShortRow) * nb);
    L.vox_short = take(sizeof(ShortRow) * nv);
    L.total = o;
    return L;
}

}  // namespace

size_t mlem_workspace(uint64_t n_bins, uint64_t n_vox) { return mlem_layout(n_bins, n_vox).total; }

hipError_t launch_mlem(int64_t n_bins, int64_t n_vox, int64_t nnz, const int64_t* T_rp,
                       const int32_t* T_col, const float* T_val, const int64_t* Tt_rp,
                       const int32_t* Tt_col, const float* Tt_val, const float* proj, float* image,
                       int32_t n_iter, void* workspace, int phases, hipStream_t s) {
    const uint64_t nb = (uint64_t)n_bins, nv = (uint64_t)n_vox;
    const MlemLayout Lo = mlem_layout(nb, nv);
    char* w = (char*)workspace;
    double* sens = (double*)(w + Lo.sens);
    double* S = (double*)(w + Lo.S);
    double* ratio = (double*)(w + Lo.ratio);
    uint32_t* st = (uint32_t*)(w + Lo.st);
    const bool setup = (phases & MLEM_SETUP) != 0, iterate = (phases & MLEM_ITERATE) != 0;
    // Layout: compact when the matrix is sparse (its renumbered columns fit
    // the workspace), else row order.
    const bool compact = nnz <= n_bins + n_vox;
    const int per_b = sweep_per(FORWARD_LOADS, nnz / n_bins);
    const int per_v = sweep_per(UPDATE_LOADS, nnz / n_vox);
    const unsigned grid_b = sweep_grid((n_bins + per_b - 1) / per_b);
    const unsigned grid_v = sweep_grid((n_vox + per_v - 1) / per_v);
    int dev = 0, n_cu = 0;
    hipError_t e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    const int gv = grid_for(nv, T256, 8192);
    const int gr = grid_for((nb + ROW_CHUNK - 1) / ROW_CHUNK + (nv + ROW_CHUNK - 1) / ROW_CHUNK, 1, 2048);
    const int g_b = compact ? 0 : mlem_forward_lanes(nnz, n_bins), g_v = compact ? 0 : mlem_update_lanes(nnz, n_vox);
    if (setup) {
        k_sweep_sums<<<grid_v, T256, 0, s>>>(n_vox, per_v, Tt_rp, Tt_val, sens);
        if (!(g_b || g_v)) k_mlem_setup<<<1, T256, 0, s>>>(n_bins, n_vox, nnz, T_rp, Tt_rp, st);
    }
    if (compact) {
        double* sens_l = (double*)(w + Lo.sens_l);
        float* P_l = (float*)(w + Lo.P_l);
        int32_t* bin_pos = (int32_t*)(w + Lo.bin_pos);
        int32_t* vox_pos = (int32_t*)(w + Lo.vox_pos);
        int32_t* Tc = (int32_t*)(w + Lo.Tc);
        int32_t* Ttc = (int32_t*)(w + Lo.Ttc);
        ClassRef* bin_list = (ClassRef*)(w + Lo.bin_rows);
        ClassRef* vox_list = (ClassRef*)(w + Lo.vox_rows);
        ShortRow* bin_short = (ShortRow*)(w + Lo.bin_short);
        ShortRow* vox_short = (ShortRow*)(w + Lo.vox_short);
        if (setup) {
            k_mlem_count<<<gr, T256, 0, s>>>(n_bins, n_vox, T_rp, T_col, Tt_rp, st);
            k_mlem_offsets<<<1, 64, 0, s>>>(st);
            k_mlem_place<<<gr, T256, 0, s>>>(n_bins, n_vox, T_rp, T_col, Tt_rp, bin_list, vox_list, bin_pos,
                                              vox_pos, st);
            k_mlem_compact<<<grid_for(std::max<uint64_t>((uint64_t)nnz, std::max(nb, nv)), T256, 8192), T256, 0,
                             s>>>(nnz, T_col, Tt_col, bin_pos, vox_pos, Tc, Ttc, bin_list, vox_list, T_val, Tt_val,
                                  bin_short, vox_short, sens, sens_l, st);
        }
        if (!iterate) return hipGetLastError();
        // Workgroups per class: each of the N_GROUP groups gets one pass over
        // a quarter of the rows the class can hold with nnz entries (groups
        // are uneven; the sweeps are grid-strided, so any count is correct),
        // the whole launch at most one resident round.
        int bpc_f = 0, bpc_u = 0;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc_f, k_mlem_forward_c, T256, 0)) != hipSuccess)
            return e;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc_u, k_mlem_update_c, T256, 0)) != hipSuccess)
            return e;
        auto ranges = [&](int64_t n_rows, int bpc, int4* b) {
            const int gs[N_CLASS] = {1, 4, 16, 64};
            const int cap = std::max(1, n_cu * bpc / (N_CLASS * N_GROUP));
            int at = 0, start[N_CLASS];
            for (int c = 0; c < N_CLASS; ++c) {
                start[c] = at;
                const uint64_t lanes = ((uint64_t)class_capacity(c, n_rows, nnz) + 3) / 4 * gs[c];
                at += N_GROUP * grid_for(lanes, T256, cap);
            }
            *b = make_int4(start[0], start[1], start[2], start[3]);
            return at;
        };
        int4 bf, bu;
        const int gf = ranges(n_bins, bpc_f, &bf), gu = ranges(n_vox, bpc_u, &bu);
        k_mlem_load<<<grid_for(std::max(nb, nv), T256, 8192), T256, 0, s>>>(n_bins, n_vox, nnz, image, sens_l, S,
                                                                            proj, bin_list, vox_list, P_l, st);
        for (int it = 0; it < n_iter; ++it) {
            k_mlem_forward_c<<<gf, T256, 0, s>>>(bin_list, bin_short, st, bf, Tc, T_val, S, P_l, ratio);
            k_mlem_update_c<<<gu, T256, 0, s>>>(vox_list, vox_short, st, bu, Ttc, Tt_val, ratio, sens_l, S);
        }
        k_mlem_out<<<gv, T256, 0, s>>>(n_vox, S, vox_pos, st, image);
        return hipGetLastError();
    }
    RowRef* bin_rows = (RowRef*)(w + Lo.bin_rows);
    RowRef* vox_rows = (RowRef*)(w + Lo.vox_rows);
    if (setup && (g_b || g_v)) {
        uint64_t* chunk = (uint64_t*)(w + Lo.Tc);       // the compact layout's, idle here
        const int64_t n_chunks = (int64_t)((nb + ROW_CHUNK - 1) / ROW_CHUNK + (nv + ROW_CHUNK - 1) / ROW_CHUNK);
        k_mlem_rows<ROWS_COUNT><<<gr + 1, T256, 0, s>>>(n_bins, n_vox, nnz, T_rp, Tt_rp, bin_rows, vox_rows, chunk, st);
        if (n_chunks > ROWS_MAX_CHUNKS) k_scan_blocks<<<1, 1024, 0, s>>>(chunk, (int)n_chunks);
        auto place = n_chunks > ROWS_MAX_CHUNKS ? k_mlem_rows<ROWS_PLACE_SCANNED> : k_mlem_rows<ROWS_PLACE>;
        place<<<gr, T256, 0, s>>>(n_bins, n_vox, nnz, T_rp, Tt_rp, bin_rows, vox_rows, chunk, st);
    }
    if (!iterate) return hipGetLastError();
    k_mlem_load<<<gv, T256, 0, s>>>(n_bins, n_vox, nnz, image, sens, S, nullptr, nullptr, nullptr, nullptr, st);
    auto kf = g_b == 1 ? k_mlem_forward_rows<1> : g_b == 4 ? k_mlem_forward_rows<4>
            : g_b == 16 ? k_mlem_forward_rows<16> : k_mlem_forward_rows<64>;
    auto ku = g_v == 1 ? k_mlem_update_rows<1> : g_v == 4 ? k_mlem_update_rows<4>
            : g_v == 16 ? k_mlem_update_rows<16> : k_mlem_update_rows<64>;
    const unsigned gf = g_b ? sweep_grid(grid_for(nb * g_b, T256, 1 << 16)) : grid_b;
    const unsigned gu = g_v ? (unsigned)grid_for(nv * g_v, T256, 1 << 16) : grid_v;
    for (int it = 0; it < n_iter; ++it) {
        if (g_b)
            kf<<<gf, T256, 0, s>>>(bin_rows, n_bins, st + ST_BINS, st + ST_CALL_BAD, T_col, T_val, S, proj, ratio);
        else
            k_mlem_forward<<<gf, T256, 0, s>>>(n_bins, per_b, T_rp, st + ST_CALL_BAD, T_col, T_val, S, proj, ratio);
        if (g_v)
            ku<<<gu, T256, 0, s>>>(vox_rows, n_vox, st + ST_VOXS, st + ST_CALL_BAD, Tt_col, Tt_val, ratio, sens, S);
        else
            k_mlem_update<<<gu, T256, 0, s>>>(n_vox, per_v, Tt_rp, st + ST_CALL_BAD, Tt_col, Tt_val, ratio, sens, S);
    }
    k_mlem_out<<<gv, T256, 0, s>>>(n_vox, S, nullptr, st, image);
    return hipGetLastError();
}

}  // namespace mcs
