// Input staging: from the caller's attenuation and activity maps to the tables
// the transport kernels read.
//
//  * max mu, input validation, the activity total and the attenuation box
//    (the voxel index range of mu > 0) in one reduction pass;
//  * accept thresholds Q_v = ceil(mu_v 2^24 / max mu) in double precision, so
//    the real/virtual decision of Woodcock tracking is an exact integer compare;
//    when the map has at most 256 distinct thresholds (segmented phantoms have
//    a handful) also one-byte codes into a palette of them, a table a quarter
//    the size that stays in L2;
//  * the runs of the activity map (maximal stretches of a grid row with one
//    weight), each with the cumulative activity before it (uint64), and a
//    table of buckets over the high bits of that sum with about two buckets
//    per run (after the guide tables of Chen & Asau 1974): an emission voxel
//    is one 8-byte bucket gather, one 16-byte run gather and a division
//    within the run, rarely a short search over runs -- the same voxel as a
//    plain inverse-CDF search over all voxels.  A segmented phantom has ~1e4
//    runs, so both tables stay in L2;
//  * (cos, sin) of each view angle;
//  * the Klein-Nishina attenuation shape sigma_KN(E)/sigma_KN(140) at 1/4 keV
//    steps, evaluated in double precision.
//
// Four launches: one over everything that only needs the inputs, one workgroup
// per problem that combines it (small problems do without), the runs and
// thresholds, the guide table and codes.
#include <algorithm>

#include "mc_internal.h"

namespace mcs {
namespace {

constexpr int RED_THREADS = 256;
constexpr int ROWS = 4;        // values a pass loads at once

__device__ inline uint64_t wave_sum_u64(uint64_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ inline uint32_t wave_max_u32(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}
__device__ inline uint32_t wave_or_u32(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v |= (uint32_t)__shfl_xor((int)v, o, 64);
    return v;
}

// Launch 1: everything that needs the caller's inputs and nothing else.  Its
// workgroups take one of the following by blockIdx.x (blockIdx.y: problem):
//  * [0, scan_blocks): SCAN_ITEMS voxels each of both maps, read once: max mu
//    (as bits: order-preserving for non-negative floats), bad-value flag and
//    attenuation box of the stretch (StagePart), its activity and the runs
//    starting in it;
//  * 1: the descriptor (passed by value, so the launch can be captured in a
//    graph), the work and chunk prefixes, the palette cleared, the view table;
//  * KN_BLOCKS: the Klein-Nishina table;
//  * the rest: the call's tallies cleared.
// One launch for up to STAGE_MAX problems, so small problems overlap instead
// of queueing.  On small problems staging is bound by its launches, 2 to 5 us
// each whatever they do: 12 of them (with the call's preparation) took 55 us
// at 32^3 and 95 us at 128^3, the three or four 19 and 45 us.
constexpr int STAGE_MAX = 8;
constexpr int KN_BLOCKS = (KN_TABLE_N + 255) / 256;

struct StageArgs {
    ProbDesc d[STAGE_MAX];
    ProbDesc* out;                  // descriptor of the launch's first problem
    uint32_t scan_blocks;
    // the call's preparation (null / 0 for replay and adjoint)
    uint64_t* work_prefix;          // [n_problems + 1], then as many of the chunk prefix
    uint64_t work0, chunks0;        // work and chunks before the launch's first problem
    uint32_t chunk;
    int first, last, n_problems;    // the launch's problems of the call
    int64_t* status;
    unsigned long long* n_events;
    int64_t* tally;
    int64_t* tally_sq;
    uint64_t tally_elems;
    uint32_t zero_blocks;           // workgroups per problem that clear tallies
};
static_assert(sizeof(StageArgs) <= 4096, "kernel arguments");

// What launch 1 finds in one stretch of voxels: max mu, STATUS flags | 1 << 31
// when mu > 0 somewhere, and the box of those voxels (10 bits per axis).
struct StagePart {
    uint32_t mx, flags, lo, hi;
};

// Where they are kept until combined: a problem of few stretches (TOP_SMALL) has
// no launch for that, so its results must outlast the threshold table's writing;
// otherwise the table's place.
constexpr int TOP_SMALL = SCAN_THREADS;
constexpr int PARTS_AT = 512;
static_assert(TOP_SMALL <= PARTS_AT && PARTS_AT + TOP_SMALL * sizeof(StagePart) / 8 <= BLOCK_SCRATCH_MIN,
              "after the stretches' sums, in the block-sum scratch");
__device__ __forceinline__ StagePart* parts_of(const ProbDesc& d) {
    const uint64_t n_blocks = (d.nvox + SCAN_ITEMS - 1) / SCAN_ITEMS;
    return n_blocks <= TOP_SMALL ? (StagePart*)(d.block_sums + PARTS_AT) : (StagePart*)d.q32;
}
constexpr uint32_t PART_ANY = 1u << 31;

// Klein-Nishina total cross-section per electron over 2 pi r_e^2 (closed form).
__device__ double kn_bracket(double e) {
    const double k = e / 510.99895;
    const double a = 1.0 + 2.0 * k;
    const double la = log(a);
    return (1.0 + k) / (k * k) * (2.0 * (1.0 + k) / a - la / k) + la / (2.0 * k)
           - (1.0 + 3.0 * k) / (a * a);
}

// Voxel i starts a run: it is active and its row neighbour on the left (none
// at ix = 0) has a different weight.
__device__ inline bool run_start(uint32_t a, uint32_t a_left, uint32_t ix) {
    return a > 0 && (ix == 0 || a_left != a);
}

__device__ inline void stage_scan(const ProbDesc& d) {
    const uint64_t nvox = d.nvox;
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_ITEMS;
    if (base >= nvox) return;               // past this problem's blocks
    constexpr int PER = SCAN_ITEMS / SCAN_THREADS;
    const float* __restrict__ mu = d.mu;
    const uint32_t* __restrict__ act = d.act;
    const uint32_t* __restrict__ prev = d.act_prev;
    const uint32_t nx = (uint32_t)d.nx, ny = (uint32_t)d.ny;
    // voxels base + j SCAN_THREADS + thread: coordinates by one division, then
    // steps of SCAN_THREADS voxels
    uint32_t i0 = (uint32_t)base + threadIdx.x;
    uint32_t ix = i0 % nx, iy = i0 / nx % ny, iz = i0 / nx / ny;
    const uint32_t sx = SCAN_THREADS % nx, sy = SCAN_THREADS / nx % ny, sz = SCAN_THREADS / nx / ny;
    uint32_t mx = 0, flags = 0, runs = 0;
    uint64_t sum = 0;
    uint32_t lo[3] = {1023u, 1023u, 1023u}, hi[3] = {0u, 0u, 0u};
#pragma unroll 4
    for (int j0 = 0; j0 < PER; j0 += 4) {
        float m[4];
        uint32_t w[4], l[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t i = base + (uint64_t)(j0 + u) * SCAN_THREADS + threadIdx.x;
            m[u] = i < nvox ? mu[i] : 0.0f;
            w[u] = i < nvox ? source_weight(act, prev, i) : 0u;
            l[u] = i < nvox && i > 0 ? source_weight(act, prev, i - 1) : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!(m[u] >= 0.0f) || !isfinite(m[u])) flags |= MC_STATUS_BAD_MU;
            else if (m[u] > 0.0f) {
                flags |= PART_ANY;
                mx = max(mx, __float_as_uint(m[u]));
                lo[0] = min(lo[0], ix); hi[0] = max(hi[0], ix);
                lo[1] = min(lo[1], iy); hi[1] = max(hi[1], iy);
                lo[2] = min(lo[2], iz); hi[2] = max(hi[2], iz);
            }
            sum += w[u];
            runs += run_start(w[u], l[u], ix);
            ix += sx; iy += sy; iz += sz;
            if (ix >= nx) { ix -= nx; ++iy; }
            if (iy >= ny) { iy -= ny; ++iz; }
        }
    }
    mx = wave_max_u32(mx);
    flags = wave_or_u32(flags);
    sum = wave_sum_u64(sum);
    runs = (uint32_t)wave_sum_u64(runs);
    for (int a = 0; a < 3; ++a) {
        for (int o = 32; o > 0; o >>= 1) {
            lo[a] = min(lo[a], (uint32_t)__shfl_xor((int)lo[a], o, 64));
            hi[a] = max(hi[a], (uint32_t)__shfl_xor((int)hi[a], o, 64));
        }
    }
    __shared__ StagePart part[SCAN_THREADS / 64];
    __shared__ uint64_t part_sum[SCAN_THREADS / 64];
    __shared__ uint32_t part_runs[SCAN_THREADS / 64];
    if ((threadIdx.x & 63) == 0) {
        const int v = threadIdx.x >> 6;
        part[v] = StagePart{mx, flags, lo[0] | lo[1] << 10 | lo[2] << 20, hi[0] | hi[1] << 10 | hi[2] << 20};
        part_sum[v] = sum;
        part_runs[v] = runs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        StagePart p = part[0];
        for (int v = 1; v < SCAN_THREADS / 64; ++v) {
            const StagePart q = part[v];
            p.mx = max(p.mx, q.mx);
            p.flags |= q.flags;
            uint32_t plo = 0, phi = 0;
            for (int a = 0; a < 30; a += 10) {
                plo |= min(p.lo >> a & 1023u, q.lo >> a & 1023u) << a;
                phi |= max(p.hi >> a & 1023u, q.hi >> a & 1023u) << a;
            }
            p.lo = plo;
            p.hi = phi;
            sum += part_sum[v];
            runs += part_runs[v];
        }
        parts_of(d)[blockIdx.x] = p;
        d.block_sums[blockIdx.x] = sum;
        d.block_cnt[blockIdx.x] = runs;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_stage_scan(StageArgs A) {
    const ProbDesc& d = A.d[blockIdx.y];
    uint32_t b = blockIdx.x;
    if (b < A.scan_blocks) {
        stage_scan(d);
        return;
    }
    b -= A.scan_blocks;
    if (b == 0) {
        __shared__ uint32_t bad_angle;
        if (threadIdx.x == 0) bad_angle = 0;
        __syncthreads();
        if (d.pal_state == 0)
            for (int k = threadIdx.x; k < PALETTE_N; k += SCAN_THREADS) d.palette[k] = PALETTE_EMPTY;
        for (int k = threadIdx.x; k < d.n_views; k += SCAN_THREADS) {
            const double a = d.angles[k];
            if (!isfinite(a)) bad_angle = 1;
            d.views[k] = make_float2((float)cos(a), (float)sin(a));
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            ProbDesc& out = A.out[blockIdx.y];
            out = d;
            if (bad_angle) out.flags |= (uint32_t)MC_STATUS_BAD_ANGLE;
            if (A.work_prefix) {
                const int p = A.first + (int)blockIdx.y;
                uint64_t w = A.work0, c = A.chunks0;
                for (int k = 0; k < (int)blockIdx.y; ++k) {
                    w += A.d[k].work_count;
                    c += (A.d[k].work_count + A.chunk - 1) / A.chunk;
                }
                uint64_t* chunk_prefix = A.work_prefix + (A.n_problems + 1);
                A.work_prefix[p] = w;
                chunk_prefix[p] = c;
                if (p + 1 == A.n_problems) {
                    A.work_prefix[p + 1] = w + d.work_count;
                    chunk_prefix[p + 1] = c + (d.work_count + A.chunk - 1) / A.chunk;
                }
                if (p == 0) {
                    for (int k = 0; k < 4; ++k) A.status[k] = 0;
                    if (A.n_events) *A.n_events = 0;
                }
            }
        }
        return;
    }
    b -= 1;
    if (b < (uint32_t)KN_BLOCKS) {
        const int i = (int)(b * SCAN_THREADS + threadIdx.x);
        if (i < KN_TABLE_N) {
            const double e = fmax((double)d.e0 - 0.25 * i, 0.5);
            d.kn_table[i] = (float)(kn_bracket(e) / kn_bracket(140.0));
        }
        return;
    }
    b -= KN_BLOCKS;
    const uint64_t stride = (uint64_t)A.zero_blocks * gridDim.y * SCAN_THREADS;
    for (uint64_t i = ((uint64_t)b * gridDim.y + blockIdx.y) * SCAN_THREADS + threadIdx.x; i < A.tally_elems;
         i += stride) {
        A.tally[i] = 0;
        if (A.tally_sq) A.tally_sq[i] = 0;
    }
}

// One workgroup per problem: the stretches' results combined into the
// descriptor (max mu, flags, box), their sums and run counts scanned (each thread
// a contiguous stretch of blocks; the prefixes put in their place with PREFIXES),
// the activity total and the number of runs.
template <int THREADS, bool PREFIXES>
__device__ inline void stage_top(ProbDesc* pd) {
    const int n_blocks = (int)((pd->nvox + SCAN_ITEMS - 1) / SCAN_ITEMS);
    __shared__ uint64_t tot[16];
    __shared__ uint32_t totc[16];
    __shared__ uint32_t s_mx, s_fl, s_lo[3], s_hi[3];
    uint64_t* __restrict__ bs = pd->block_sums;
    uint32_t* __restrict__ bc = pd->block_cnt;
    const StagePart* __restrict__ parts = parts_of(*pd);
    if (threadIdx.x < 3) { s_lo[threadIdx.x] = 1023u; s_hi[threadIdx.x] = 0u; }
    if (threadIdx.x == 3) s_mx = s_fl = 0;
    const int per = (n_blocks + THREADS - 1) / THREADS;
    const int b0 = threadIdx.x * per;
    uint64_t s = 0;
    uint32_t c = 0, mx = 0, fl = 0, lo[3] = {1023u, 1023u, 1023u}, hi[3] = {0u, 0u, 0u};
    for (int j = 0; j < per; ++j) {
        if (b0 + j >= n_blocks) break;
        s += bs[b0 + j];
        c += bc[b0 + j];
        const StagePart p = parts[b0 + j];
        mx = max(mx, p.mx);
        fl |= p.flags;
        for (int a = 0; a < 3; ++a) {
            lo[a] = min(lo[a], p.lo >> (10 * a) & 1023u);
            hi[a] = max(hi[a], p.hi >> (10 * a) & 1023u);
        }
    }
    // wavefront scans, then the wavefronts' totals
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t x = s;
    uint32_t xc = c;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = (uint64_t)__shfl_up((long long)x, o, 64);
        const uint32_t yc = (uint32_t)__shfl_up((int)xc, o, 64);
        if (lane >= o) { x += y; xc += yc; }
    }
    if (lane == 63) { tot[wave] = x; totc[wave] = xc; }
    mx = wave_max_u32(mx);
    fl = wave_or_u32(fl);
    for (int a = 0; a < 3; ++a) {
        for (int o = 32; o > 0; o >>= 1) {
            lo[a] = min(lo[a], (uint32_t)__shfl_xor((int)lo[a], o, 64));
            hi[a] = max(hi[a], (uint32_t)__shfl_xor((int)hi[a], o, 64));
        }
    }
    __syncthreads();
    if (lane == 0) {
        atomicMax(&s_mx, mx);
        atomicOr(&s_fl, fl);
        for (int a = 0; a < 3; ++a) { atomicMin(&s_lo[a], lo[a]); atomicMax(&s_hi[a], hi[a]); }
    }
    uint64_t run = x - s;                  // exclusive prefix of this thread's stretch
    uint32_t runc = xc - c;
    for (int v = 0; v < wave; ++v) { run += tot[v]; runc += totc[v]; }
    for (int j = 0; j < per; ++j) {
        if (b0 + j < n_blocks) {
            const uint64_t v = bs[b0 + j];
            const uint32_t vc = bc[b0 + j];
            if (PREFIXES) {
                bs[b0 + j] = run;
                bc[b0 + j] = runc;
            }
            run += v;
            runc += vc;
        }
    }
    __syncthreads();
    if (threadIdx.x == THREADS - 1) {
        pd->total = run;
        pd->n_runs = runc;
        pd->mu_hat_bits = s_mx;
        if (s_fl & ~PART_ANY) pd->flags |= s_fl & ~PART_ANY;
        if (s_fl & PART_ANY) {
            for (int a = 0; a < 3; ++a) {
                pd->bb_lo[a] = (int)s_lo[a];
                pd->bb_hi[a] = (int)s_hi[a];
            }
        }
    }
}

// Launch 2, where a problem has more than TOP_SMALL stretches.
__global__ __launch_bounds__(1024) void k_stage_top(ProbDesc* descs) { stage_top<1024, true>(descs + blockIdx.y); }

// A workgroup's set of the distinct thresholds it has met: open addressing in
// LDS with room for four times the palette, so a probe is short up to the
// value that makes the set too large.
constexpr uint32_t SEEN_N = 4 * PALETTE_N;

// Put q in the set (each lane its own value, no order among lanes): a value
// already there costs one LDS read, the same address for lanes with equal
// values.  *n counts the distinct values; past PALETTE_N of them the map has
// no palette (*overflow is set at once, so other workgroups stop too) and
// nothing more is added.
__device__ inline void seen_insert(uint32_t* set, uint32_t* n, uint32_t q, uint32_t* overflow) {
    uint32_t h = (q * 2654435761u) >> 22;
    while (__hip_atomic_load(n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= (uint32_t)PALETTE_N) {
        uint32_t cur = __hip_atomic_load(set + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == PALETTE_EMPTY) {
            cur = atomicCAS(set + h, PALETTE_EMPTY, q);
            if (cur == PALETTE_EMPTY) {
                if (atomicAdd(n, 1u) == (uint32_t)PALETTE_N) atomicOr(overflow, 1u);
                return;
            }
        }
        if (cur == q) return;
        h = (h + 1) & (SEEN_N - 1);
    }
}

// Put a workgroup's n (<= PALETTE_N) distinct values into the palette (all
// threads call).  Rounds of one look at the whole table (one round trip to
// memory), then one attempt per missing value at the first free slot of its
// probe order in that look.  When the values there and the missing ones are
// more than the table holds, the map has no palette, and a workgroup sees
// that in the round after the table has filled up: probing a full table slot
// by slot, a round trip each, had taken 400 us on maps whose workgroups hold
// just under 256 values each.
__device__ inline void palette_merge(uint32_t* pal, uint32_t* overflow, const uint32_t* vals, uint32_t n) {
    __shared__ uint32_t snap[PALETTE_N];
    __shared__ uint32_t n_there, n_missing;
    constexpr uint32_t PRESENT = PALETTE_N + 1;
    // where v would go: PRESENT when it is there, PALETTE_N when no slot is free
    const auto free_slot = [&](uint32_t v) -> uint32_t {
        uint32_t h = palette_hash(v);
        for (int probe = 0; probe < PALETTE_N; ++probe, h = (h + 1) & (PALETTE_N - 1)) {
            if (snap[h] == v) return PRESENT;
            if (snap[h] == PALETTE_EMPTY) return h;
        }
        return PALETTE_N;
    };
    for (;;) {
        __syncthreads();                     // the last round's reads are done
        if (threadIdx.x == 0) {
            n_missing = 0;
            // overflowed elsewhere already: nothing reads the palette
            n_there = __hip_atomic_load(overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 2u * PALETTE_N : 0u;
        }
        for (uint32_t k = threadIdx.x; k < (uint32_t)PALETTE_N; k += blockDim.x)
            snap[k] = __hip_atomic_load(pal + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < (uint32_t)PALETTE_N; k += blockDim.x)
            if (snap[k] != PALETTE_EMPTY) atomicAdd(&n_there, 1u);
        for (uint32_t k = threadIdx.x; k < n; k += blockDim.x)
            if (free_slot(vals[k]) != PRESENT) atomicAdd(&n_missing, 1u);
        __syncthreads();
        if (n_missing == 0 || n_there > (uint32_t)PALETTE_N) return;
        if (n_there + n_missing > (uint32_t)PALETTE_N) {
            // The look is not of one moment: a value can be in it behind a slot
            // of its probe order that was read before another workgroup filled
            // it.  Counted again wherever they lie, what is there and what is
            // missing are different values of the map.
            __syncthreads();
            if (threadIdx.x == 0) n_missing = 0;
            __syncthreads();
            for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) {
                bool there = false;
                for (int i = 0; i < PALETTE_N; ++i) there |= snap[i] == vals[k];
                if (!there) atomicAdd(&n_missing, 1u);
            }
            __syncthreads();
            if (n_there + n_missing > (uint32_t)PALETTE_N) {
                if (threadIdx.x == 0) atomicOr(overflow, 1u);
                return;
            }
        }
        for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) {
            const uint32_t slot = free_slot(vals[k]);
            if (slot != PRESENT && slot != (uint32_t)PALETTE_N) atomicCAS(pal + slot, PALETTE_EMPTY, vals[k]);
        }
    }
}

// Index of linear voxel i in the threshold layout.
__device__ inline uint32_t table_index(uint32_t i, uint32_t nx, uint32_t ny, int b, uint32_t m, uint32_t nbx,
                                       uint32_t nby) {
    return b == 0 ? i : brick_index(i % nx, i / nx % ny, i / nx / ny, nx, ny, b, m, nbx, nby);
}

// Q_v in double precision: mu_v * 2^24 is exact, the division is correctly
// rounded, ceil is exact.  Stored linear (b = 0) or in 2^b-voxel cubic bricks,
// so a brick is a few whole cache lines (the layout never changes a result).
// Each distinct Q also goes into the palette: a workgroup collects its distinct
// values in LDS and puts them into the global table once at its end, all at a
// time (palette_merge).  A workgroup with more than PALETTE_N of them (a
// scanned map) marks the palette as overflowed instead and leaves the table
// alone: probing a full global table value by value took 2.8 ms on a 128^3
// map of distinct values, against 26 us now (segmented map: 20 against 17 us).
template <bool OWN_TOP>
__device__ inline void stage_thresholds(ProbDesc* pd, uint32_t block, uint32_t n_blocks) {
    const uint64_t nvox = pd->nvox;
    float mu_hat;
    if constexpr (OWN_TOP) {
        __shared__ uint32_t part[SCAN_THREADS / 64];
        const uint32_t n_parts = (uint32_t)((nvox + SCAN_ITEMS - 1) / SCAN_ITEMS);
        const uint32_t mx = wave_max_u32(threadIdx.x < n_parts ? parts_of(*pd)[threadIdx.x].mx : 0u);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
        __syncthreads();
        mu_hat = __uint_as_float(max(max(part[0], part[1]), max(part[2], part[3])));
    } else {
        mu_hat = __uint_as_float(pd->mu_hat_bits);
    }
    const float* __restrict__ mu = pd->mu;
    uint32_t* __restrict__ q = pd->q32;
    const uint32_t nx = (uint32_t)pd->nx, ny = (uint32_t)pd->ny;
    const int b = pd->brick_log2;
    const uint32_t m = (1u << b) - 1u;
    const uint32_t nbx = (uint32_t)pd->nbx, nby = (uint32_t)pd->nby;
    __shared__ uint32_t seen[SEEN_N];
    __shared__ uint32_t vals[PALETTE_N];
    __shared__ uint32_t n_seen, n_vals, pal_off;
    for (uint32_t k = threadIdx.x; k < SEEN_N; k += blockDim.x) seen[k] = PALETTE_EMPTY;
    if (threadIdx.x == 0) {
        n_seen = n_vals = 0;
        pal_off = __hip_atomic_load(&pd->pal_state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const bool pal = pal_off == 0;      // one answer for the workgroup: others may set it meanwhile
    // whole wavefronts stream the map, ROWS values per thread in flight; the
    // last value a lane has put in the set is not looked up again
    uint32_t last = PALETTE_EMPTY;
    const uint64_t stride = (uint64_t)n_blocks * blockDim.x;
    for (uint64_t i0 = (uint64_t)block * blockDim.x + threadIdx.x; i0 < nvox; i0 += ROWS * stride) {
        float mv[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint64_t i = i0 + (uint64_t)u * stride;
            mv[u] = i < nvox ? mu[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint64_t i = i0 + (uint64_t)u * stride;
            if (i >= nvox) break;
            uint32_t v = 0;
            if (mu_hat > 0.0f && mv[u] > 0.0f) {
                const double t = ceil((double)mv[u] * 16777216.0 / (double)mu_hat);
                v = t >= 16777216.0 ? 16777216u : (uint32_t)t;
            }
            q[table_index((uint32_t)i, nx, ny, b, m, nbx, nby)] = v;
            if (pal && v != last) {
                seen_insert(seen, &n_seen, v, &pd->pal_state);
                last = v;
            }
        }
    }
    if (!pal) return;
    __syncthreads();
    if (n_seen > (uint32_t)PALETTE_N) return;      // *overflow is set
    for (uint32_t k = threadIdx.x; k < SEEN_N; k += blockDim.x)
        if (seen[k] != PALETTE_EMPTY) vals[atomicAdd(&n_vals, 1u)] = seen[k];
    __syncthreads();
    palette_merge(pd->palette, &pd->pal_state, vals, n_vals);
}

// One-byte palette codes in the threshold layout (skipped when the palette
// overflowed or was not requested: the kernels then read the 32-bit table).
// Table entries are taken in table order, whatever voxel they hold (padding
// of a bricked layout holds no voxel and gets some code that nothing reads).
__device__ inline void stage_codes(ProbDesc* pd, uint32_t block, uint32_t n_blocks) {
    if (pd->pal_state != 0) return;
    const int b = pd->brick_log2;
    const uint64_t n = b == 0 ? pd->nvox : (uint64_t)pd->nbx * pd->nby * pd->nbz << (3 * b);
    const uint32_t* __restrict__ q = pd->q32;
    const uint32_t* __restrict__ pal = pd->palette;
    uint8_t* __restrict__ code = pd->q8;
    const uint64_t stride = (uint64_t)n_blocks * blockDim.x;
    for (uint64_t i0 = (uint64_t)block * blockDim.x + threadIdx.x; i0 < n; i0 += ROWS * stride) {
        uint32_t v[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint64_t i = i0 + (uint64_t)u * stride;
            v[u] = i < n ? q[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint64_t i = i0 + (uint64_t)u * stride;
            if (i >= n) break;
            uint32_t h = palette_hash(v[u]);
            for (int probe = 0; probe < PALETTE_N && pal[h] != v[u]; ++probe) h = (h + 1) & (PALETTE_N - 1);
            code[i] = (uint8_t)h;
        }
    }
}

// Forced detection: the brick table of codes (in the place of the 32-bit
// thresholds) and the map value of each code.  Two map values that share a
// threshold (their difference is below 2^-24 of the maximum) cannot share a
// table entry: mu_pal_bad is set and the walks read the map itself.  A
// workgroup collects the values of its voxels in LDS and merges them into the
// problem's table once.  Threads run along x: reads and writes are whole
// brick rows.
__global__ __launch_bounds__(RED_THREADS) void k_mu_codes(ProbDesc* descs) {
    ProbDesc* pd = descs + blockIdx.y;
    if (pd->pal_state != 0) return;
    __shared__ uint32_t val[PALETTE_N];      // float bits + 1
    __shared__ uint32_t clash;
    for (int k = threadIdx.x; k < PALETTE_N; k += blockDim.x) val[k] = 0;
    if (threadIdx.x == 0) clash = 0;
    __syncthreads();
    const float* __restrict__ mu = pd->mu;
    const uint8_t* __restrict__ q8 = pd->q8;
    uint8_t* __restrict__ out = (uint8_t*)pd->q32;
    const uint32_t nx = (uint32_t)pd->nx, ny = (uint32_t)pd->ny;
    const uint32_t nrows = ny * (uint32_t)pd->nz;
    const int b = pd->brick_log2;
    const uint32_t m = (1u << b) - 1u;
    const uint32_t nbx = (uint32_t)pd->nbx, nby = (uint32_t)pd->nby;
    const uint32_t lx = mu_code_log2(pd->nx, 4), ly = mu_code_log2(pd->ny, 3);
    uint32_t last_c = PALETTE_N, last_v = 0;    // the pair this lane put in the table last
    for (uint32_t r0 = blockIdx.x; r0 < nrows; r0 += ROWS * gridDim.x)
    for (uint32_t ix = threadIdx.x; ix < nx; ix += blockDim.x) {
        uint32_t c[ROWS], v[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint32_t r = r0 + (uint32_t)u * gridDim.x;
            const bool ok = r < nrows;
            c[u] = ok ? q8[brick_index(ix, r % ny, r / ny, nx, ny, b, m, nbx, nby)] : 0u;
            v[u] = ok ? __float_as_uint(mu[(uint64_t)r * nx + ix]) + 1u : 0u;
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const uint32_t r = r0 + (uint32_t)u * gridDim.x;
            if (r >= nrows) break;
            out[mu_code_x(ix) | mu_code_y(r % ny, lx) | (r / ny) << (lx + ly)] = (uint8_t)c[u];
            if (c[u] == last_c && v[u] == last_v) continue;
            last_c = c[u];
            last_v = v[u];
            uint32_t cur = __hip_atomic_load(val + c[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == 0) cur = atomicCAS(val + c[u], 0u, v[u]);
            if (cur != 0 && cur != v[u]) clash = 1;
        }
    }
    __syncthreads();
    uint32_t* __restrict__ table = (uint32_t*)(pd->block_sums + MU_PAL_AT);
    for (int k = threadIdx.x; k < PALETTE_N; k += blockDim.x) {
        if (val[k] == 0) continue;
        uint32_t cur = __hip_atomic_load(table + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == 0) cur = atomicCAS(table + k, 0u, val[k]);
        if (cur != 0 && cur != val[k]) clash = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0 && clash) atomicOr(&pd->mu_pal_bad, 1u);
}

// Per block: 16 consecutive voxels per thread, thread-local scans, block
// exclusive scans of the thread totals, plus the block offsets; each voxel
// that starts a run writes the run (cumulative weight before it, its packed
// coordinates, its weight) at its compacted slot.
template <bool OWN_TOP>
__device__ inline void stage_runs(const ProbDesc* pd) {
    constexpr int PER = SCAN_ITEMS / SCAN_THREADS;
    const uint64_t nvox = pd->nvox;
    if ((uint64_t)blockIdx.x * SCAN_ITEMS >= nvox) return;   // past this problem's blocks
    const uint32_t* __restrict__ act = pd->act;
    const uint32_t* __restrict__ prev = pd->act_prev;
    uint4* __restrict__ runs = pd->runs;
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_ITEMS + (uint64_t)threadIdx.x * PER;
    const uint32_t nx = (uint32_t)pd->nx, ny = (uint32_t)pd->ny;
    uint32_t a[PER];
    const uint32_t left0 = (base > 0 && base < nvox) ? source_weight(act, prev, base - 1) : 0u;
    const uint32_t ix0 = (uint32_t)base % nx;
    uint64_t s = 0;
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint64_t i = base + j;
        a[j] = (i < nvox) ? source_weight(act, prev, i) : 0u;
        s += a[j];
    }
    uint32_t starts = 0;        // bit j: voxel base + j starts a run
    uint32_t rx = ix0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t l = j > 0 ? a[j - 1] : left0;
        if (base + j < nvox && run_start(a[j], l, rx)) starts |= 1u << j;
        if (++rx == nx) rx = 0;
    }
    c = __popc(starts);
    __shared__ uint64_t tot[SCAN_THREADS / 64];
    __shared__ uint32_t totc[SCAN_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t x = s;
    uint32_t xc = c;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = (uint64_t)__shfl_up((long long)x, o, 64);
        const uint32_t yc = (uint32_t)__shfl_up((int)xc, o, 64);
        if (lane >= o) { x += y; xc += yc; }
    }
    if (lane == 63) { tot[wave] = x; totc[wave] = xc; }
    __syncthreads();
    // weight and runs before the block
    uint64_t before;
    uint32_t k;
    if constexpr (OWN_TOP) {
        __shared__ uint64_t part[SCAN_THREADS / 64];
        __shared__ uint32_t partc[SCAN_THREADS / 64];
        uint64_t w = threadIdx.x < blockIdx.x ? pd->block_sums[threadIdx.x] : 0;
        uint32_t n = threadIdx.x < blockIdx.x ? pd->block_cnt[threadIdx.x] : 0;
        for (int o = 32; o > 0; o >>= 1) {
            w += (uint64_t)__shfl_xor((long long)w, o, 64);
            n += (uint32_t)__shfl_xor((int)n, o, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            part[threadIdx.x >> 6] = w;
            partc[threadIdx.x >> 6] = n;
        }
        __syncthreads();
        before = (part[0] + part[1]) + (part[2] + part[3]);
        k = (partc[0] + partc[1]) + (partc[2] + partc[3]);
    } else {
        before = pd->block_sums[blockIdx.x];
        k = pd->block_cnt[blockIdx.x];
    }
    before += x - s;                                        // weight before voxel base
    k += xc - c;
    for (int v = 0; v < wave; ++v) { before += tot[v]; k += totc[v]; }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (starts & (1u << j)) {
            const uint32_t i = (uint32_t)(base + j);
            const uint32_t ix = i % nx, iy = (i / nx) % ny, iz = i / (nx * ny);
            runs[k] = make_uint4((uint32_t)before, (uint32_t)(before >> 32),
                                 ix | (iy << 10) | (iz << 20), a[j]);   // packed 10 bits per axis
            ++k;
        }
        before += a[j];
    }
}

// Bucket table over the runs: bucket b covers t in [b 2^s, (b+1) 2^s), with
// about two buckets per run (after the guide tables of Chen & Asau 1974).
// Run r holds t in [c_r, c_{r+1}); the bucket's entry is the run holding its
// first t and the number of further runs starting inside it.
__device__ inline uint64_t run_c(const uint4* __restrict__ runs, uint64_t r) {
    const uint4 v = runs[r];
    return ((uint64_t)v.y << 32) | v.x;
}

// First run whose start is above key (R when none): the run holding key is
// the one before it (run 0 starts at 0 <= key).
__device__ inline uint64_t first_run_above(const uint4* __restrict__ runs, uint64_t R, uint64_t key) {
    uint64_t lo = 0, hi = R;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (run_c(runs, mid) > key) hi = mid; else lo = mid + 1;
    }
    return lo;
}

__device__ inline void stage_guide(ProbDesc* pd, uint32_t block, uint32_t n_blocks) {
    const uint64_t nb_cap = guide_capacity(pd->nvox);
    const uint64_t total = pd->total;
    const uint64_t R = pd->n_runs;
    if (total == 0 || R == 0) {
        if (block == 0 && threadIdx.x == 0) atomicOr(&pd->flags, (uint32_t)MC_STATUS_NO_ACTIVITY);
        return;
    }
    uint64_t cap = 1;
    while (cap < 2 * R) cap <<= 1;
    if (cap > nb_cap) cap = nb_cap;
    uint32_t s = 0;
    while (((total - 1) >> s) >= cap) ++s;
    const uint64_t B = ((total - 1) >> s) + 1;
    if (block == 0 && threadIdx.x == 0) {
        pd->shift = s;
        pd->n_buckets = (uint32_t)B;
    }
    const uint4* __restrict__ runs = pd->runs;
    uint2* __restrict__ guide = pd->guide;
    // bucket b's first t lies in run lo(b) = first_run_above(b 2^s) - 1 and
    // its last t = (b + 1) 2^s - 1 in run hi(b) = (first run starting at or
    // above (b + 1) 2^s) - 1, which is lo(b + 1), or one less when a run
    // starts exactly at (b + 1) 2^s.  A wavefront finds lo for 64
    // consecutive buckets, one search per lane, and completes 63 of them with
    // its neighbour's.
    const int lane = threadIdx.x & 63;
    const uint64_t wave = ((uint64_t)block * blockDim.x + threadIdx.x) >> 6;
    const uint64_t n_waves = ((uint64_t)n_blocks * blockDim.x) >> 6;
    for (uint64_t grp = wave; grp * 63 < B; grp += n_waves) {
        const uint64_t b = grp * 63 + (uint64_t)lane;
        const uint64_t fa = b < B ? first_run_above(runs, R, b << s) : R;   // >= 1
        const uint32_t nl = (uint32_t)__shfl_down((int)(uint32_t)fa, 1, 64);
        const uint32_t nh = (uint32_t)__shfl_down((int)(uint32_t)(fa >> 32), 1, 64);
        if (lane == 63 || b >= B) continue;
        const uint64_t lo = fa - 1;
        uint64_t hi;
        if (b + 1 < B) {
            const uint64_t fa1 = (uint64_t)nl | ((uint64_t)nh << 32);
            hi = fa1 - 1;
            if (run_c(runs, hi) == ((b + 1) << s)) --hi;
        } else {
            hi = R - 1;                        // the last bucket ends at total - 1
        }
        guide[b] = make_uint2((uint32_t)lo, (uint32_t)(hi - lo));
    }
}

// Launch 3, after the problem's maximum, total and block prefixes: the
// emission runs (workgroups [0, scan_blocks)) and the accept thresholds with
// their palette (the rest), which do not need each other.  OWN_TOP (all problems
// have at most TOP_SMALL stretches): instead of launch 2, each workgroup adds up
// what it needs of the stretches' results, one load per thread, and the last one
// fills in the descriptor (32^3: 66 us per call of 2e5 histories with launch 2,
// 60 without).
template <bool OWN_TOP>
__global__ __launch_bounds__(SCAN_THREADS) void k_stage_tables(ProbDesc* descs, uint32_t scan_blocks) {
    ProbDesc* pd = descs + blockIdx.y;
    const uint32_t end = gridDim.x - (OWN_TOP ? 1 : 0);
    if (blockIdx.x < scan_blocks) stage_runs<OWN_TOP>(pd);
    else if (blockIdx.x < end) stage_thresholds<OWN_TOP>(pd, blockIdx.x - scan_blocks, end - scan_blocks);
    else stage_top<SCAN_THREADS, false>(pd);
}

// Launch 4: the guide table over the runs ([0, guide_blocks)), the palette
// codes ([guide_blocks, gridDim.x - 1)), and the transport's totals and claim
// counters cleared (the last workgroup; the block prefixes they replace are
// not read any more).
__global__ __launch_bounds__(RED_THREADS) void k_stage_finish(ProbDesc* descs, uint32_t guide_blocks) {
    ProbDesc* pd = descs + blockIdx.y;
    if (blockIdx.x < guide_blocks) stage_guide(pd, blockIdx.x, guide_blocks);
    else if (blockIdx.x + 1 < gridDim.x) stage_codes(pd, blockIdx.x - guide_blocks, gridDim.x - 1 - guide_blocks);
    else
        for (int k = threadIdx.x; k < BLOCK_SCRATCH_MIN; k += RED_THREADS) pd->block_sums[k] = 0;
}

int grid_for(uint64_t n, int threads, int cap) {
    uint64_t g = (n + threads - 1) / threads;
    if (g > (uint64_t)cap) g = cap;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace


// Staging of n problems and, with call, the preparation of a forward call
// (work prefixes, cleared status, tallies and totals).
hipError_t launch_staging_batch(ProbDesc* d, const ProbDesc* h, int n, const CallPrep* call, hipStream_t st) {
    uint64_t max_vox = 1, max_cap = 1;
    uint64_t work0 = 0, chunks0 = 0;
    for (int i = 0; i < n; ++i) {
        max_vox = std::max<uint64_t>(max_vox, h[i].nvox);
        max_cap = std::max<uint64_t>(max_cap, guide_capacity(h[i].nvox));
    }
    const uint32_t scan_blocks = (uint32_t)((max_vox + SCAN_ITEMS - 1) / SCAN_ITEMS);
    const unsigned ny = (unsigned)n;
    for (int first = 0; first < n; first += STAGE_MAX) {
        const int cnt = std::min(STAGE_MAX, n - first);
        StageArgs a = {};
        for (int i = 0; i < cnt; ++i) a.d[i] = h[first + i];
        a.out = d + first;
        a.scan_blocks = scan_blocks;
        a.first = first;
        a.n_problems = n;
        uint32_t zero_blocks = 0;
        if (call) {
            a.work_prefix = call->work_prefix;
            a.work0 = work0;
            a.chunks0 = chunks0;
            a.chunk = call->chunk;
            a.status = call->status;
            a.n_events = call->n_events;
            if (first == 0) {
                a.tally = call->tally;
                a.tally_sq = call->tally_sq;
                a.tally_elems = call->tally_elems;
                const uint64_t g = (call->tally_elems + SCAN_THREADS - 1) / SCAN_THREADS;
                zero_blocks = (uint32_t)(std::min<uint64_t>(g, 4096) + cnt - 1) / cnt;
            }
            for (int i = 0; i < cnt; ++i) {
                work0 += a.d[i].work_count;
                chunks0 += (a.d[i].work_count + call->chunk - 1) / call->chunk;
            }
        }
        a.zero_blocks = zero_blocks;
        k_stage_scan<<<dim3(scan_blocks + 1 + KN_BLOCKS + zero_blocks, (unsigned)cnt), SCAN_THREADS, 0, st>>>(a);
    }
    const bool own_top = scan_blocks <= TOP_SMALL;
    if (!own_top) k_stage_top<<<dim3(1, ny), 1024, 0, st>>>(d);
    // each workgroup puts each threshold value it meets into the palette once
    // (a few round trips to memory): not more of them than keep the chip busy
    const uint32_t stream_blocks = (uint32_t)std::min<uint64_t>((max_vox + RED_THREADS * ROWS - 1) / (RED_THREADS * ROWS), 1024);
    if (own_top) k_stage_tables<true><<<dim3(scan_blocks + stream_blocks + 1, ny), SCAN_THREADS, 0, st>>>(d, scan_blocks);
    else k_stage_tables<false><<<dim3(scan_blocks + stream_blocks, ny), SCAN_THREADS, 0, st>>>(d, scan_blocks);
    const uint32_t guide_blocks = (uint32_t)grid_for(max_cap, RED_THREADS, 1024);
    k_stage_finish<<<dim3(guide_blocks + stream_blocks + 1, ny), RED_THREADS, 0, st>>>(d, guide_blocks);
    return hipGetLastError();
}

hipError_t launch_mu_codes(ProbDesc* d, const ProbDesc* h, int n, hipStream_t st) {
    uint64_t max_rows = 1;
    int max_nx = 1;
    for (int i = 0; i < n; ++i) {
        max_rows = std::max<uint64_t>(max_rows, (uint64_t)h[i].ny * h[i].nz);
        max_nx = std::max(max_nx, h[i].nx);
    }
    const int row_threads = (int)std::min<uint64_t>(RED_THREADS, ((uint64_t)max_nx + 63) / 64 * 64);
    const unsigned blocks = (unsigned)std::min<uint64_t>((max_rows + ROWS - 1) / ROWS, 1024);
    k_mu_codes<<<dim3(blocks, (unsigned)n), row_threads, 0, st>>>(d);
    return hipGetLastError();
}

// Entries (uint64) of a problem's block-sum scratch: the scan's block sums,
// after them the transport's totals.
size_t staging_block_scratch_u64(uint64_t nvox) {
    return (size_t)std::max<uint64_t>((nvox + SCAN_ITEMS - 1) / SCAN_ITEMS, BLOCK_SCRATCH_MIN);
}

hipError_t launch_staging(ProbDesc* d, const ProbDesc& h, hipStream_t st) {
    return launch_staging_batch(d, &h, 1, nullptr, st);
}

}  // namespace mcs
