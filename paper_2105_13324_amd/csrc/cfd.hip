// Convolution-based forced detection (CFD, paper Sec. 5.2): the collimator
// response of each depth layer, and the convolution of the sub-projection
// layers into the projection tally.
//
// A forced copy travels perpendicular to the detector and is stored, with
// its weight, in the layer of its depth (one pixel thick) at the pixel of its
// perpendicular hit (transport kernel).  The ideal cone collimator spreads a
// point at depth d over a disk of radius d tan(alpha) with plane density
// d / (2 pi (1 - cos alpha) (d^2 + r^2)^(3/2)) (directions uniform in the
// cone); integrated over each pixel (CFD_SUB^2 midpoint samples) and
// normalised, that is layer l's response at its centre depth.  The projection
// is the sum over layers of the layer convolved with its response, in FP64
// on the Q31.32 deposits, rounded once into the Q31.32 tally.
#include "mc_internal.h"

namespace mcs {
namespace {

constexpr double PI_D = 3.14159265358979323846;

__global__ __launch_bounds__(256) void k_cfd_half_widths(ProbDesc* pd) {
    for (int l = threadIdx.x; l < pd->cfd_L; l += blockDim.x)
        pd->cfd_h[l] = (uint32_t)min(cfd_half_width((l + 0.5) * pd->cfd_pix, pd->cfd_tan, pd->cfd_pix),
                                     pd->cfd_hmax);
}

// one block per layer; runs after k_cfd_half_widths
__global__ __launch_bounds__(256) void k_cfd_kernels(ProbDesc* pd) {
    const int l = blockIdx.x;
    if (l >= pd->cfd_L) return;
    const double pix = pd->cfd_pix, a = pd->alpha;
    const double d = (l + 0.5) * pix, rho = d * pd->cfd_tan, omc = 2.0 * sin(0.5 * a) * sin(0.5 * a);
    const int h = (int)pd->cfd_h[l], n = 2 * h + 1, nmax = 2 * pd->cfd_hmax + 1;
    double* k = pd->cfd_kern + (uint64_t)l * nmax * nmax;
    double part = 0.0;
    for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
        const int b = idx / n - h, c = idx % n - h;
        double acc = 0.0;
        for (int t = 0; t < CFD_SUB; ++t)
            for (int u = 0; u < CFD_SUB; ++u) {
                const double x = (c + (u + 0.5) / CFD_SUB - 0.5) * pix;
                const double y = (b + (t + 0.5) / CFD_SUB - 0.5) * pix;
                const double r2 = x * x + y * y;
                if (r2 > rho * rho) continue;
                const double q = d * d + r2;
                acc += d / (2.0 * PI_D * omc * q * sqrt(q));
            }
        acc *= (pix / CFD_SUB) * (pix / CFD_SUB);
        k[idx] = acc;
        part += acc;
    }
    __shared__ double red[256];
    red[threadIdx.x] = part;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    const double tot = red[0];
    for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x)
        k[idx] = tot > 0.0 ? k[idx] / tot : (idx == h * n + h ? 1.0 : 0.0);
}

__global__ __launch_bounds__(256) void k_fill_i64(int64_t* p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// The convolution: a block per CFD_TILE x CFD_TILE output tile of one (view,
// class).  For each layer the block stages the tile with its halo of
// half-width h and the layer's response in LDS, then adds each output's
// (2h + 1)^2 products, (b, a) in order; the next layer's values are loaded into
// registers meanwhile, and a layer whose tile and halo are all zero is skipped
// (its products are exact zeros, so the sum is the same).  Output (v, u) takes
// layer (v - b, u - a) times response (b, a).  The response is even in a and in
// b (the pixel samples are placed symmetrically; the table is so up to
// rounding), so the four layer values of (+-b, +-a) share one product.
constexpr int CFD_SMALL_H = 8;

// Output tile of this block: view and class, first column and row.  Workgroups
// are dealt to the 8 XCDs in turn: the tiles of a (view, class) go to one XCD,
// whose L2 then serves the halos they share.
struct CfdTile {
    uint64_t vc;
    int u0, v0;
};
__host__ __device__ inline uint64_t cfd_grid(uint64_t n_vc, int nu, int nv) {
    return (n_vc + 7) / 8 * 8 * ((nu + CFD_TILE - 1) / CFD_TILE) * ((nv + CFD_TILE - 1) / CFD_TILE);
}
__device__ __forceinline__ CfdTile cfd_tile(int nu, int nv) {
    const uint32_t tu = (nu + CFD_TILE - 1) / CFD_TILE, tv = (nv + CFD_TILE - 1) / CFD_TILE;
    const uint32_t b = blockIdx.x / 8, t = b % (tu * tv);
    return CfdTile{(uint64_t)(b / (tu * tv)) * 8 + blockIdx.x % 8, (int)(t % tu) * CFD_TILE, (int)(t / tu) * CFD_TILE};
}

// Half-widths up to CFD_SMALL_H: a wavefront per tile, four neighbouring
// columns per thread.  With one output per thread the LDS reads bound it, four
// per product; here a row's values serve the four columns from registers, and
// LDS and the FP64 units are about even.  The half-width is a constant of the
// code that adds a layer, so a row pair's reads are all in flight at once (with
// a loop over the columns the reads' latency took as long as before: 410 us).
// The tile's columns lie in LDS by their index mod 4, rows 12 apart, so that the
// lanes' reads of one column index mod 4 fall in distinct banks.  60 views of
// 64 x 64, 94 layers, 2 classes: 421 us with one output per thread, 262 us now.
constexpr int CFD_SMALL_W = CFD_TILE + 2 * CFD_SMALL_H;
constexpr int CFD_ROW = 12, CFD_PLANE = CFD_SMALL_W * CFD_ROW + 8;
constexpr int CFD_Q = CFD_SMALL_H + 1;         // a response's quadrant
static_assert(CFD_SMALL_W == 32 && CFD_TILE == 16, "half a wavefront per row; 4 x 16 threads");

// One layer of half-width H added to the outputs of this thread; c: its first
// column in the tile's first row.
template <int H>
__device__ __forceinline__ void cfd_layer(const double* c, const double* kt, double (&acc)[4]) {
#pragma unroll 2
    for (int bb = 0; bb <= H; ++bb) {
        // columns 4 lu - H .. 4 lu + 3 + H of the rows at -b and +b
        double up[4 + 2 * H], dn[4 + 2 * H], k[H + 1];
#pragma unroll
        for (int q = 0; q < 4 + 2 * H; ++q) {
            up[q] = c[(H - bb) * CFD_ROW + (q & 3) * CFD_PLANE + (q >> 2)];
            dn[q] = c[(H + bb) * CFD_ROW + (q & 3) * CFD_PLANE + (q >> 2)];
        }
#pragma unroll
        for (int aa = 0; aa <= H; ++aa) k[aa] = kt[bb * CFD_Q + aa];
        if (bb == 0) {
#pragma unroll
            for (int aa = 0; aa <= H; ++aa)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = fma(aa ? up[H + j - aa] + up[H + j + aa] : up[H + j], k[aa], acc[j]);
        } else {
#pragma unroll
            for (int aa = 0; aa <= H; ++aa)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = fma(aa ? (up[H + j - aa] + up[H + j + aa]) + (dn[H + j - aa] + dn[H + j + aa])
                                    : up[H + j] + dn[H + j], k[aa], acc[j]);
        }
    }
}

__global__ __launch_bounds__(64) void k_cfd_convolve_small(const ProbDesc* __restrict__ pd, int64_t* tally) {
    __shared__ double tile[4 * CFD_PLANE];
    __shared__ double kt[CFD_Q * CFD_Q];
    constexpr int PF = CFD_SMALL_W / 2;        // rows per thread
    const int nu = pd->nu, nv = pd->nv, L = pd->cfd_L;
    const int nmax = 2 * pd->cfd_hmax + 1;
    const CfdTile T = cfd_tile(nu, nv);
    if (T.vc >= 2 * (uint64_t)pd->n_views) return;
    const uint64_t view = T.vc >> 1, cls = T.vc & 1;
    const int lane = (int)threadIdx.x;
    const int col = lane & 31, row0 = lane >> 5;                   // staging
    const int lu = lane % 4, lv = lane / 4;                        // outputs (lv, 4 lu + j)
    const int64_t* __restrict__ lay = pd->layers;
    const double* __restrict__ kern = pd->cfd_kern;
    const uint32_t* __restrict__ hl = pd->cfd_h;
    int64_t nx[PF];
    double kx[2];
    auto fetch = [&](int l, int h) {
        const int w = CFD_TILE + 2 * h, n = 2 * h + 1;
        const int iu = T.u0 - h + col, v0 = T.v0 - h + row0;
        const bool in_row = col < w && iu >= 0 && iu < nu;
        const int64_t* base = lay + ((view * L + l) * 2 + cls) * (uint64_t)nv * nu;
        const double* kl = kern + (uint64_t)l * nmax * nmax;
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int iv = v0 + 2 * k;
            nx[k] = 0;
            if (in_row && row0 + 2 * k < w && iv >= 0 && iv < nv) nx[k] = base[(uint64_t)iv * nu + iu];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = lane + 64 * k, bb = i / CFD_Q, aa = i % CFD_Q;
            kx[k] = bb <= h && aa <= h ? kl[(bb + h) * n + h + aa] : 0.0;
        }
    };
    int h_next = (int)hl[0];
    fetch(0, h_next);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int l = 0; l < L; ++l) {
        const int h = h_next;
        __syncthreads();                         // the previous layer's reads are done
        bool any = false;
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            tile[(col & 3) * CFD_PLANE + (row0 + 2 * k) * CFD_ROW + (col >> 2)] = (double)nx[k];
            any |= nx[k] != 0;
        }
        kt[lane] = kx[0];
        if (lane + 64 < CFD_Q * CFD_Q) kt[lane + 64] = kx[1];
        if (l + 1 < L) {
            h_next = (int)hl[l + 1];
            fetch(l + 1, h_next);
        }
        __syncthreads();
        if (__ballot(any) == 0) continue;
        const double* c = tile + lv * CFD_ROW + lu;
        switch (h) {
        case 0: cfd_layer<0>(c, kt, acc); break;
        case 1: cfd_layer<1>(c, kt, acc); break;
        case 2: cfd_layer<2>(c, kt, acc); break;
        case 3: cfd_layer<3>(c, kt, acc); break;
        case 4: cfd_layer<4>(c, kt, acc); break;
        case 5: cfd_layer<5>(c, kt, acc); break;
        case 6: cfd_layer<6>(c, kt, acc); break;
        case 7: cfd_layer<7>(c, kt, acc); break;
        default: cfd_layer<8>(c, kt, acc); break;
        }
    }
    const int ov = T.v0 + lv;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int ou = T.u0 + 4 * lu + j;
        if (ou < nu && ov < nv)
            tally[pd->tally_offset + (T.vc * nv + ov) * (uint64_t)nu + ou] = (int64_t)llrint(acc[j]);
    }
}

// Wider responses: an output per thread, the tile in LDS sized at launch for
// the largest h (a wavefront's registers do not hold the next layer's values
// there).
constexpr int CFD_THREADS = CFD_TILE * CFD_TILE;

__global__ __launch_bounds__(CFD_THREADS) void k_cfd_convolve(const ProbDesc* __restrict__ pd, int64_t* tally) {
    constexpr int CFD_PF = ((CFD_TILE + 2 * CFD_MAX_H) * (CFD_TILE + 2 * CFD_MAX_H) + CFD_THREADS - 1) / CFD_THREADS;
    constexpr int CFD_KPF = ((2 * CFD_MAX_H + 1) * (2 * CFD_MAX_H + 1) + CFD_THREADS - 1) / CFD_THREADS;
    extern __shared__ double smem[];
    const int nu = pd->nu, nv = pd->nv, L = pd->cfd_L;
    const int hmax = pd->cfd_hmax, nmax = 2 * hmax + 1, wmax = CFD_TILE + 2 * hmax;
    double* tile = smem;                      // [wmax * wmax]
    double* kt = smem + wmax * wmax;          // [nmax * nmax]
    const CfdTile T = cfd_tile(nu, nv);
    if (T.vc >= 2 * (uint64_t)pd->n_views) return;
    const uint64_t vc = T.vc, view = vc >> 1, cls = vc & 1;
    const int tid = (int)threadIdx.x;
    const int lu = tid % CFD_TILE, lv = tid / CFD_TILE;
    const int u0 = T.u0, v0 = T.v0;
    const int64_t* __restrict__ lay = pd->layers;
    const double* __restrict__ kern = pd->cfd_kern;
    const uint32_t* __restrict__ hl = pd->cfd_h;
    int64_t nx[CFD_PF];
    double kx[CFD_KPF];
    auto fetch = [&](int l, int h) {
        const int w = CFD_TILE + 2 * h, n = 2 * h + 1;
        const int64_t* base = lay + ((view * L + l) * 2 + cls) * (uint64_t)nv * nu;
        const double* kl = kern + (uint64_t)l * nmax * nmax;
#pragma unroll
        for (int k = 0; k < CFD_PF; ++k) {
            const int i = tid + k * CFD_THREADS;
            int64_t v = 0;
            if (i < w * w) {
                const int iv = v0 - h + i / w, iu = u0 - h + i % w;
                if (iv >= 0 && iv < nv && iu >= 0 && iu < nu) v = base[(uint64_t)iv * nu + iu];
            }
            nx[k] = v;
        }
#pragma unroll
        for (int k = 0; k < CFD_KPF; ++k) {
            const int i = tid + k * CFD_THREADS;
            kx[k] = i < n * n ? kl[i] : 0.0;
        }
    };
    int h_next = (int)hl[0];
    fetch(0, h_next);
    double acc = 0.0;
    for (int l = 0; l < L; ++l) {
        const int h = h_next, n = 2 * h + 1, w = CFD_TILE + 2 * h;
        __syncthreads();                         // the previous layer's reads are done
        bool any = false;
#pragma unroll
        for (int k = 0; k < CFD_PF; ++k) {
            const int i = tid + k * CFD_THREADS;
            if (i < w * w) {
                tile[i] = (double)nx[k];
                any |= nx[k] != 0;
            }
        }
#pragma unroll
        for (int k = 0; k < CFD_KPF; ++k) {
            const int i = tid + k * CFD_THREADS;
            if (i < n * n) kt[i] = kx[k];
        }
        if (l + 1 < L) {
            h_next = (int)hl[l + 1];
            fetch(l + 1, h_next);
        }
        if (!__syncthreads_or(any)) continue;
        // layer value (v - b, u - a) sits at tile row lv + h - b, column lu + h - a
        const double* c = tile + (lv + h) * w + lu + h;
        for (int bb = 0; bb <= h; ++bb) {
            const double* up = c - bb * w;
            const double* dn = c + bb * w;
            const double* kr = kt + (bb + h) * n + h;
            double s0 = bb ? up[0] + dn[0] : up[0];
            acc = fma(s0, kr[0], acc);
#pragma unroll 4
            for (int aa = 1; aa <= h; ++aa) {
                const double s = bb ? (up[-aa] + up[aa]) + (dn[-aa] + dn[aa]) : up[-aa] + up[aa];
                acc = fma(s, kr[aa], acc);
            }
        }
    }
    const int ou = u0 + lu, ov = v0 + lv;
    if (ou < nu && ov < nv)
        tally[pd->tally_offset + (vc * nv + ov) * (uint64_t)nu + ou] = (int64_t)llrint(acc);
}

int grid_cap(uint64_t n, int cap) {
    uint64_t g = (n + 255) / 256;
    if (g < 1) g = 1;
    if (g > (uint64_t)cap) g = cap;
    return (int)g;
}

}  // namespace

hipError_t launch_cfd_setup(ProbDesc* d, const ProbDesc& h, hipStream_t s) {
    const uint64_t n_lay = (uint64_t)h.n_views * h.cfd_L * 2 * h.nv * h.nu;
    k_fill_i64<<<grid_cap(n_lay, 8192), 256, 0, s>>>(h.layers, n_lay);
    k_cfd_half_widths<<<1, 256, 0, s>>>(d);
    k_cfd_kernels<<<h.cfd_L, 256, 0, s>>>(d);
    return hipGetLastError();
}

hipError_t launch_cfd_convolve(const ProbDesc* d, const ProbDesc& h, int64_t* tally, hipStream_t s) {
    const uint64_t tiles = cfd_grid(2 * (uint64_t)h.n_views, h.nu, h.nv);
    const size_t w = CFD_TILE + 2 * (size_t)h.cfd_hmax, m = 2 * (size_t)h.cfd_hmax + 1;
    const size_t lds = 8 * (w * w + m * m);     // at most 51 KB (half-width 24)
    if (h.cfd_hmax <= CFD_SMALL_H)
        k_cfd_convolve_small<<<(unsigned)tiles, 64, 0, s>>>(d, tally);
    else
        k_cfd_convolve<<<(unsigned)tiles, CFD_THREADS, lds, s>>>(d, tally);
    return hipGetLastError();
}

}  // namespace mcs
