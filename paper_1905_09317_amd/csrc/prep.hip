// Landscape and weather preparation, and the per-cell FBP field kernel.
//
//  * cell records: fuel, burnable-neighbour mask, Horn slope numerators and
//    the FBP slope factor of every cell (Section 3.3 (i)-(ii));
//  * burnable-cell list (row-major) and the burnable cell nearest the centre
//    (ignition choices of Section 3.1, uncertainty source (1));
//  * weather table: per (scenario, period) FBP terms that do not depend on
//    the cell (Section 3.5 (iv));
//  * eval_ros: the per-cell rates of one (scenario, period, rep).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"
#include "kernels.h"
#include "types.h"

namespace c2f {

// ------------------------------------------------------------ utilities
__global__ void fill_u32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

static int fill_grid(size_t n) {
    size_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(fill_grid(n)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// -------------------------------------------------- landscape preparation

// Cell records.  Horn's 3x3 gradient numerators with replicated edges:
// gx = east column - west column (weights 1,2,1), gn = north row - south row.
// grad_from (may be NULL): take the Horn numerators from these records (a
// landscape derived from another with the same elevation) instead of elev.
__global__ void cellrec_kernel(const uint8_t* __restrict__ fuel, const int16_t* __restrict__ elev,
                               const CellRec* __restrict__ grad_from, int rows, int cols, double cell_m,
                               CellRec* __restrict__ recs, int32_t* __restrict__ overflow) {
    const size_t n = (size_t)rows * cols;
    const int DR[8] = {0, -1, -1, -1, 0, 1, 1, 1};
    const int DC[8] = {1, 1, 0, -1, -1, -1, 0, 1};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(i / cols), c = (int)(i - (size_t)r * cols);
        uint32_t mask = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int rr = r + DR[k], cc = c + DC[k];
            if (rr >= 0 && rr < rows && cc >= 0 && cc < cols && fuel[(size_t)rr * cols + cc] != 0) mask |= 1u << k;
        }
        int gx = 0, gn = 0;
        if (grad_from) {
            const uint32_t g = grad_from[i].grad;
            gx = (int)(int16_t)(g & 0xFFFFu);
            gn = (int)(int16_t)(g >> 16);
        } else if (elev) {
            const int rn = r > 0 ? r - 1 : 0, rs = r < rows - 1 ? r + 1 : rows - 1;
            const int cw = c > 0 ? c - 1 : 0, ce = c < cols - 1 ? c + 1 : cols - 1;
            auto z = [&](int rr, int cc) { return (int)elev[(size_t)rr * cols + cc]; };
            gx = (z(rn, ce) + 2 * z(r, ce) + z(rs, ce)) - (z(rn, cw) + 2 * z(r, cw) + z(rs, cw));
            gn = (z(rn, cw) + 2 * z(rn, c) + z(rn, ce)) - (z(rs, cw) + 2 * z(rs, c) + z(rs, ce));
            if (gx > 32767 || gx < -32767 || gn > 32767 || gn < -32767) {
                atomicOr(overflow, 1);
                gx = gn = 0;
            }
        }
        CellRec rec;
        const int f = fuel[i];
        rec.info = (uint32_t)f | (mask << 8);
        rec.grad = (uint32_t)(uint16_t)(int16_t)gx | ((uint32_t)(uint16_t)(int16_t)gn << 16);
        rec.ux = rec.uy = 0.f;
        if ((gx | gn) != 0) upslope_unit<float>(gx, gn, rec.ux, rec.uy);
        rec.sfc = 1.0;
        rec.sfd = 1.0;
        if ((gx | gn) != 0 && f != kNonFuel) {
            // SF^(1/c) of the rate curve(s) the cell's slope effect uses
            const double sf = slope_factor(gx, gn, cell_m);
            // mixedwoods: their conifer curve (C-2 for M-1/M-2, their own
            // dead-fir curve for M-3/M-4) and the D-1 curve
            const bool mix_pc = (f == kM1 || f == kM2), mixed = mix_pc || f == kM3 || f == kM4;
            rec.sfc = pow(sf, 1.0 / kCoef64[mix_pc ? kC2 : f].c);
            if (mixed) rec.sfd = pow(sf, 1.0 / kCoef64[kD1].c);
        }
        recs[i] = rec;
    }
}

// Burnable-cell list in row-major order: per-tile counts, one-block scan,
// ordered scatter.  A tile is kTile consecutive cells handled by one block.
constexpr int kTileThreads = 256;
constexpr int kTile = kTileThreads * 16;

__global__ void burnable_count_kernel(const uint8_t* __restrict__ fuel, int64_t n,
                                      int32_t* __restrict__ tile_counts) {
    __shared__ int s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kTile;
    int local = 0;
    for (int k = threadIdx.x; k < kTile; k += kTileThreads) {
        const int64_t i = t0 + k;
        local += (i < n && fuel[i] != 0);
    }
    atomicAdd(&s_cnt, local);
    __syncthreads();
    if (threadIdx.x == 0) tile_counts[blockIdx.x] = s_cnt;
}

__global__ void burnable_scan_kernel(int32_t* __restrict__ tile_counts, int n_tiles, LandDev* land) {
    // single block of 1024 threads: exclusive scan in place
    __shared__ int s_part[1024];
    const int per = (n_tiles + 1023) / 1024;
    const int b = threadIdx.x * per;
    int sum = 0;
    for (int k = 0; k < per && b + k < n_tiles; ++k) sum += tile_counts[b + k];
    s_part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int v = (threadIdx.x >= (unsigned)off) ? s_part[threadIdx.x - off] : 0;
        __syncthreads();
        s_part[threadIdx.x] += v;
        __syncthreads();
    }
    int run = s_part[threadIdx.x] - sum;   // exclusive prefix of this thread's range
    for (int k = 0; k < per && b + k < n_tiles; ++k) {
        const int c = tile_counts[b + k];
        tile_counts[b + k] = run;
        run += c;
    }
    if (threadIdx.x == 1023) land->n_burnable = s_part[1023];
}

__global__ void burnable_scatter_kernel(const uint8_t* __restrict__ fuel, int64_t n,
                                        const int32_t* __restrict__ tile_offsets,
                                        int32_t* __restrict__ list) {
    __shared__ int s_wave[kTileThreads / 64];
    __shared__ int s_base;
    if (threadIdx.x == 0) s_base = tile_offsets[blockIdx.x];
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k0 = 0; k0 < kTile; k0 += kTileThreads) {
        const int64_t i = t0 + k0 + threadIdx.x;
        const bool b = (i < n) && fuel[i] != 0;
        const uint64_t m = __ballot(b);
        if (lane == 0) s_wave[wave] = __popcll(m);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < kTileThreads / 64; ++w) {
            if (w < wave) before += s_wave[w];
            total += s_wave[w];
        }
        if (b) {
            const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            list[s_base + before + rank] = (int32_t)i;
        }
        __syncthreads();
        if (threadIdx.x == 0) s_base += total;
        __syncthreads();
    }
}

// Burnable cell nearest to (rows/2, cols/2); ties go to the lower index.  A
// squared distance needs up to 62 bits and an index 31, more than one atomic
// holds, so the least distance (centre_key) is found first and its lowest index
// after that.
//
// Blocks take tiles of kCentreTile consecutive cells outward from the centre
// cell, before it and behind it in turn, and a block ends at the first tile both
// of whose sides have only rows as far away as the nearest cell found so far:
// beyond the tiles of the blocks that start together little is read.  A block
// offers a distance only if it is still smaller: thousands of atomics on the one
// word were most of the time.  Bound by the launch and one tile's latency: 1500 x
// 1100 cells 5.6 us, 8192^2 7.4, 1 x 4 million 9.2, 8192^2 with fuel in one corner
// only 79 (a key of each wave through an atomic, the whole grid: 291 and 11755
// for the first two; blocks of whole rows: 6.3, 14.4, 4290 and 309).
constexpr int kCentreThreads = 256;
constexpr int kCentreTile = kCentreThreads * 16;

__global__ __launch_bounds__(kCentreThreads) void centre_kernel(const uint8_t* __restrict__ fuel, int rows, int cols,
                                                                LandDev* land) {
    __shared__ unsigned long long s_d2[kCentreThreads / 64], s_best;
    const int64_t n = (int64_t)rows * cols, n_tiles = (n + kCentreTile - 1) / kCentreTile;
    const int cr = rows / 2, cc = cols / 2;
    const int64_t tc = ((int64_t)cr * cols + cc) / kCentreTile;
    auto nearest = [&]() {
        return __hip_atomic_load(&land->centre_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // the least squared row distance of tile tc + m and those behind it, and
    // of tile tc - 1 - m and those before it
    auto behind = [&](int64_t m) -> unsigned long long {
        if (tc + m >= n_tiles) return ~0ull;
        const int64_t dr = (int64_t)((uint32_t)((tc + m) * kCentreTile) / (uint32_t)cols) - cr;
        return dr > 0 ? (unsigned long long)(dr * dr) : 0ull;
    };
    auto before = [&](int64_t m) -> unsigned long long {
        if (m >= tc) return ~0ull;
        const int64_t dr = cr - (int64_t)((uint32_t)((tc - m) * kCentreTile - 1) / (uint32_t)cols);
        return dr > 0 ? (unsigned long long)(dr * dr) : 0ull;
    };
    for (int64_t o = blockIdx.x; o < 2 * n_tiles; o += gridDim.x) {
        const int64_t m = o >> 1;
        if (threadIdx.x == 0) s_best = nearest();
        __syncthreads();
        // no cell yet: s_best is above every distance, so that only tiles
        // outside the grid end the search (the same for every thread)
        const unsigned long long b0 = behind(m), b1 = before(m), best = s_best;
        if (b0 >= best && b1 >= best) break;
        if (((o & 1) ? b1 : b0) >= best) {
            __syncthreads();
            continue;
        }
        const int64_t i0 = ((o & 1) ? tc - 1 - m : tc + m) * kCentreTile + 16 * (int64_t)threadIdx.x;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (i0 + 16 <= n) {
            const uint4 x = *(const uint4*)(fuel + i0);   // the grid starts on a 256-byte boundary
            w[0] = x.x, w[1] = x.y, w[2] = x.z, w[3] = x.w;
        } else {
            for (int u = 0; u < 16; ++u)
                if (i0 + u < n) w[u >> 2] |= (uint32_t)fuel[i0 + u] << (8 * (u & 3));
        }
        unsigned long long d2 = ~0ull;
        if ((w[0] | w[1] | w[2] | w[3]) != 0u) {
            const uint32_t r0 = (uint32_t)i0 / (uint32_t)cols;   // indices are below 2^31
            int64_t dr = (int64_t)r0 - cr, dc = i0 - (int64_t)r0 * cols - cc;
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if ((w[u >> 2] >> (8 * (u & 3))) & 0xFFu) {
                    const unsigned long long d = (unsigned long long)(dr * dr + dc * dc);
                    d2 = d < d2 ? d : d2;
                }
                if (++dc == cols - cc) dc = -cc, ++dr;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long d = __shfl_xor(d2, off);
            d2 = d < d2 ? d : d2;
        }
        if ((threadIdx.x & 63) == 0) s_d2[threadIdx.x >> 6] = d2;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < kCentreThreads / 64; ++k) d2 = s_d2[k] < d2 ? s_d2[k] : d2;
            if (d2 < nearest()) atomicMin(&land->centre_key, d2);
        }
    }
}

// Largest r with r r <= x (x < 2^62).
__device__ __forceinline__ int64_t isqrt(int64_t x) {
    int64_t r = (int64_t)sqrt((double)x);
    while (r * r > x) --r;
    while ((r + 1) * (r + 1) <= x) ++r;
    return r;
}

// The lowest index at the least distance.  In a row only the columns at
// sqrt(d^2 - dr^2) either side of the centre have it, and only the rows whose
// columns there lie in the grid are looked at.  One block.
__global__ __launch_bounds__(kCentreThreads) void centre_index_kernel(const uint8_t* __restrict__ fuel, int rows,
                                                                      int cols, LandDev* land) {
    __shared__ uint32_t s_cell;
    if (threadIdx.x == 0) s_cell = 0xFFFFFFFFu;
    __syncthreads();
    if (land->centre_key != ~0ull) {
        // cr rows and cc columns lie on the longer sides of the centre cell
        const int64_t cr = rows / 2, cc = cols / 2, d2 = (int64_t)land->centre_key;
        const int64_t near = d2 > cc * cc ? isqrt(d2 - cc * cc) : 0;
        const int64_t root = isqrt(d2), far = root < cr ? root : cr;
        auto look = [&](int64_t dr) {
            const int64_t r = cr + dr, dc2 = d2 - dr * dr;
            if (r < 0 || r >= rows || dc2 < 0) return;
            const int64_t dc = isqrt(dc2);
            if (dc * dc != dc2) return;
            if (dc <= cc && fuel[r * cols + cc - dc] != 0) atomicMin(&s_cell, (uint32_t)(r * cols + cc - dc));
            if (cc + dc < cols && fuel[r * cols + cc + dc] != 0) atomicMin(&s_cell, (uint32_t)(r * cols + cc + dc));
        };
        for (int64_t k = near + threadIdx.x; k <= far; k += kCentreThreads) {
            look(-k);
            look(k);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) land->centre_cell = (int32_t)s_cell;   // -1 if there is none
}

// Landscape constants: M-1/M-2 conifer fraction and the O-1 curing factor
// (0.005 (exp(0.061 C) - 1) below 58.8 % curing, 0.176 + 0.02 (C - 58.8)
// above); M-3/M-4 dead-fir fraction; from the foliar moisture content FMC the
// C-6 moisture effect FME = 1000 (1.5 - 0.00275 FMC)^4 / (460 + 25.9 FMC)
// over its average 0.778, and the critical surface intensity for crowning
// 0.001 CBH^1.5 (460 + 25.9 FMC)^1.5 of every fuel.
__device__ void fbp_consts(LandDev* land, float fmc_f, float pdf_f) {
    const int f = threadIdx.x;
    const double fmc = (double)fmc_f;
    const double h = pow(460.0 + 25.9 * fmc, 1.5);
    if (f < kNumFuels) {
        const double csi = 0.001 * pow(kCrown[f].cbh, 1.5) * h;
        land->csi64[f] = csi;
        land->csi32[f] = (float)csi;
    }
    if (f == 0) {
        const double fme = 1000.0 * pow(1.5 - 0.00275 * fmc, 4.0) / (460.0 + 25.9 * fmc);
        land->pdf_w64 = (double)pdf_f / 100.0;
        land->fme_r64 = fme / 0.778;
        land->pdf_w32 = pdf_f / 100.0f;
        land->fme_r32 = (float)(fme / 0.778);
    }
}

__global__ void fbpconst_kernel(LandDev* land, float fmc, float pdf) { fbp_consts(land, fmc, pdf); }

hipError_t launch_fbp_consts(LandDev* land, float fmc, float pdf, hipStream_t s) {
    hipLaunchKernelGGL(fbpconst_kernel, dim3(1), dim3(64), 0, s, land, fmc, pdf);
    return hipGetLastError();
}

// Everything of a landscape's record that its cells do not decide, and the
// start of the centre search.
__global__ void landinit_kernel(LandDev* land, float pc, float curing, int cell_m, float fmc, float pdf) {
    fbp_consts(land, fmc, pdf);
    if (threadIdx.x != 0) return;
    land->n_burnable = 0;
    land->centre_cell = -1;
    land->grad_overflow = land->pad0 = 0;
    land->centre_key = ~0ull;
    const double c = (double)curing;
    land->pc_w64 = (double)pc / 100.0;
    land->cf64 = (c < 58.8) ? 0.005 * (exp(0.061 * c) - 1.0) : 0.176 + 0.02 * (c - 58.8);
    land->cell_m64 = (double)cell_m;
    const float cf = curing;
    land->pc_w32 = pc / 100.0f;
    land->cf32 = (cf < 58.8f) ? 0.005f * (expf(0.061f * cf) - 1.0f) : 0.176f + 0.02f * (cf - 58.8f);
    land->cell_m32 = (float)cell_m;
    land->pad1 = 0.f;
}

hipError_t launch_prepare_landscape(const uint8_t* fuel, const int16_t* elev, const CellRec* grad_from,
                                    int rows, int cols, int cell_m, float pc, float curing, float fmc,
                                    float pdf, CellRec* recs, int32_t* burnable, int32_t* tile_scratch,
                                    LandDev* land, hipStream_t s) {
    const int64_t n = (int64_t)rows * cols;
    const int g = fill_grid((size_t)n);
    hipLaunchKernelGGL(landinit_kernel, dim3(1), dim3(64), 0, s, land, pc, curing, cell_m, fmc, pdf);
    hipLaunchKernelGGL(cellrec_kernel, dim3(g), dim3(256), 0, s, fuel, elev, grad_from, rows, cols,
                       (double)cell_m, recs, &land->grad_overflow);
    const int n_tiles = (int)((n + kTile - 1) / kTile);
    hipLaunchKernelGGL(burnable_count_kernel, dim3(n_tiles), dim3(kTileThreads), 0, s, fuel, n, tile_scratch);
    hipLaunchKernelGGL(burnable_scan_kernel, dim3(1), dim3(1024), 0, s, tile_scratch, n_tiles, land);
    hipLaunchKernelGGL(burnable_scatter_kernel, dim3(n_tiles), dim3(kTileThreads), 0, s, fuel, n, tile_scratch, burnable);
    const int64_t centre_tiles = 2 * ((n + kCentreTile - 1) / kCentreTile);
    hipLaunchKernelGGL(centre_kernel, dim3((unsigned)(centre_tiles < 256 ? centre_tiles : 256)), dim3(kCentreThreads),
                       0, s, fuel, rows, cols, land);
    hipLaunchKernelGGL(centre_index_kernel, dim3(1), dim3(kCentreThreads), 0, s, fuel, rows, cols, land);
    return hipGetLastError();
}

int64_t tile_scratch_entries(int64_t n_cells) { return (n_cells + kTile - 1) / kTile; }

// fuel[cells[k]] = codes[k] in the order of k: the edits of a derived landscape
// (cells are checked on the host).  Of several edits of a cell the last one
// stands: they raise a word of that cell, in owner, to the highest k, and only
// that k writes.  Bound by three launches and scattered words in L2.  Sorting
// the edits on the host took most of a derive: with 5 % of 1024^2 cells edited,
// derive and unload 2785 -> 272 us.
__global__ void edit_reset_kernel(int32_t* __restrict__ owner, const int32_t* __restrict__ cells, int32_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) owner[cells[k]] = -1;
}

__global__ void edit_claim_kernel(int32_t* __restrict__ owner, const int32_t* __restrict__ cells, int32_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) atomicMax(&owner[cells[k]], (int32_t)k);
}

__global__ void edit_apply_kernel(uint8_t* __restrict__ fuel, const int32_t* __restrict__ owner,
                                  const int32_t* __restrict__ cells, const uint8_t* __restrict__ codes, int32_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n && owner[cells[k]] == (int32_t)k) fuel[cells[k]] = codes[k];
}

// owner: scratch of one word a cell, its contents are of no account.
hipError_t launch_fuel_edits(uint8_t* fuel, int32_t* owner, const int32_t* cells, const uint8_t* codes, int32_t n,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 g((unsigned)(((int64_t)n + 255) / 256)), b(256);
    hipLaunchKernelGGL(edit_reset_kernel, g, b, 0, s, owner, cells, n);
    hipLaunchKernelGGL(edit_claim_kernel, g, b, 0, s, owner, cells, n);
    hipLaunchKernelGGL(edit_apply_kernel, g, b, 0, s, fuel, owner, cells, codes, n);
    return hipGetLastError();
}

// ------------------------------------------------------- weather table

// Surface fuel consumption (kg/m^2) of an unmixed fuel from FFMC and BUI
// (M-1/M-2 mix the C-2 and D-1 values by percent conifer where they are
// used; they get 0 here).
template <typename R>
__device__ R surface_consumption(int f, R ffmc, R bui) {
    switch (f) {
        case kC1:
            return ffmc > (R)84 ? (R)0.75 + (R)0.75 * m_sqrt((R)1 - m_exp((R)-0.23 * (ffmc - (R)84)))
                                : (R)0.75 - (R)0.75 * m_sqrt((R)1 - m_exp((R)-0.23 * ((R)84 - ffmc)));
        case kC2:
        case kM3:
        case kM4: return (R)5 * ((R)1 - m_exp((R)-0.0115 * bui));
        case kC3:
        case kC4: return (R)5 * m_pow((R)1 - m_exp((R)-0.0164 * bui), (R)2.24);
        case kC5:
        case kC6: return (R)5 * m_pow((R)1 - m_exp((R)-0.0149 * bui), (R)2.48);
        case kC7: {
            const R ffc = ffmc > (R)70 ? (R)2 * ((R)1 - m_exp((R)-0.104 * (ffmc - (R)70))) : (R)0;
            return ffc + (R)1.5 * ((R)1 - m_exp((R)-0.0201 * bui));
        }
        case kD1:
        case kD2: return (R)1.5 * ((R)1 - m_exp((R)-0.0183 * bui));
        case kS1: return (R)4 * ((R)1 - m_exp((R)-0.025 * bui)) + (R)4 * ((R)1 - m_exp((R)-0.034 * bui));
        case kS2: return (R)10 * ((R)1 - m_exp((R)-0.013 * bui)) + (R)6 * ((R)1 - m_exp((R)-0.060 * bui));
        case kS3: return (R)12 * ((R)1 - m_exp((R)-0.0166 * bui)) + (R)20 * ((R)1 - m_exp((R)-0.0210 * bui));
        case kO1a:
        case kO1b: return (R)kGrassFuelLoad;
        default: return (R)0;
    }
}

// Fill a table row from FFMC, BUI, wind speed (km/h) and the azimuth the wind
// comes from: fuels f0, f0 + step, ... of it, and with fuel 0 what the fuels
// share.  The fire heads downwind: WAZ = WD + 180 degrees.
template <typename R>
__device__ __forceinline__ void weather_row(const CoefR<R>* coef, const float* w, int f0, int step, R* row) {
    const R ffmc = (R)w[0], bui = (R)w[1], ws = (R)w[2], wd = (R)w[3];
    const R m = (R)147.2 * ((R)101 - ffmc) / ((R)59.5 + ffmc);   // fine fuel moisture
    const R ff = (R)91.9 * m_exp((R)-0.1386 * m) * ((R)1 + m_pow(m, (R)5.31) / (R)4.93e7);
    const R isz = (R)0.208 * ff;
    if (f0 == 0) {
        const R waz = m_fmod(wd + (R)180, (R)360) * (Const<R>::pi / (R)180);
        row[0] = ff;
        row[1] = isz;
        row[2] = ws * m_sin(waz);
        row[3] = ws * m_cos(waz);
    }
#pragma unroll
    for (int f = f0; f < kNumFuels; f += step) {
        const CoefR<R>& k = coef[f];
        R be = (R)1;
        if (f != kNonFuel && bui > (R)0)
            be = m_exp((R)50 * m_log(k.q) * ((R)1 / bui - (R)1 / k.bui0));
        row[kRowBE + f] = be;
        row[kRowG + f] = (k.a > (R)0) ? -m_expm1(-k.b * isz) : (R)0;
        row[kRowSFC + f] = surface_consumption<R>(f, ffmc, bui);
    }
#pragma unroll
    for (int f = f0; f < kRowLen - kRowSFC - kNumFuels; f += step) row[kRowSFC + kNumFuels + f] = (R)0;
}

// A wave a row, lane f for fuel f; blockIdx.y selects the precision.
__global__ __launch_bounds__(64) void weather_table_kernel(const float* __restrict__ wx, double* __restrict__ t64,
                                                           float* __restrict__ t32) {
    const size_t i = blockIdx.x;
    if (blockIdx.y == 0) weather_row<double>(coef_table<double>(), wx + i * 4, (int)threadIdx.x, 64, t64 + i * kRowLen);
    else weather_row<float>(coef_table<float>(), wx + i * 4, (int)threadIdx.x, 64, t32 + i * kRowLen);
}

// A lane a row: the fuels in turn, the same branch for all lanes, and the row
// written in one piece.
template <typename R>
__device__ __forceinline__ void weather_lane(const float* w, R* __restrict__ out) {
    R row[kRowLen];
    weather_row<R>(coef_table<R>(), w, 0, 1, row);
#pragma unroll
    for (int k = 0; k < kRowLen; ++k) out[k] = row[k];
}

__global__ __launch_bounds__(64) void weather_table_long_kernel(const float* __restrict__ wx, int n_rows,
                                                                double* __restrict__ t64, float* __restrict__ t32) {
    const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= (size_t)n_rows) return;
    if (blockIdx.y == 0) weather_lane<double>(wx + i * 4, t64 + i * kRowLen);
    else weather_lane<float>(wx + i * 4, t32 + i * kRowLen);
}

// Up to this many rows a wave each (one or two a SIMD in two precisions), more a
// lane each.  Bound by a row's chain of exponentials and powers, then, from about
// 2^16 rows, by the writes (768 B a row).  us for a wave / a lane a row: 48 rows
// 7.5 / 8.0, 1000 8.0 / 9.7, 2000 15.4 / 11.5, 16000 87 / 14.5, 65536 338 / 26;
// 2^20 rows 299.  (A lane a row, one launch a precision: 12.7, 17, 20, 21, 34, 300.)
// A wave each does not reach the largest table, 2^26 rows: a launch holds fewer
// than 2^32 threads along an axis.
constexpr int kWeatherWaves = 1024;

hipError_t launch_weather_table(const float* wx, int n_rows, double* t64, float* t32, hipStream_t s) {
    if (n_rows <= kWeatherWaves)
        hipLaunchKernelGGL(weather_table_kernel, dim3((unsigned)n_rows, 2), dim3(64), 0, s, wx, t64, t32);
    else
        hipLaunchKernelGGL(weather_table_long_kernel, dim3((unsigned)((n_rows + 63) / 64), 2), dim3(64), 0, s, wx,
                           n_rows, t64, t32);
    return hipGetLastError();
}

// ------------------------------------------------------------- eval_ros

template <typename R>
__global__ void eval_ros_kernel(EvalArgs a) {
    const CoefR<R>* const coef = coef_table<R>();
    const CoefR<double>* const coef64 = coef_table<double>();
    const LandR<R> L = land_consts<R>(a.land);
    const LandR<double> L64 = land_consts<double>(a.land);
    const size_t ro = ((size_t)a.scenario * a.n_wp + a.period) * kRowLen;
    const R* const row = (const R*)a.table + ro;
    const double* const row64 = a.table64 + ro;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n_cells; i += gridDim.x * blockDim.x) {
        const CellRec rec = a.cells[i];
        const int f = rec_fuel(rec.info);
        if (f == 0) {
            if (a.hros) a.hros[i] = 0;
            if (a.bros) a.bros[i] = 0;
            if (a.fros) a.fros[i] = 0;
            if (a.lb) a.lb[i] = 0;
            if (a.raz) a.raz[i] = 0;
            if (a.cfb) a.cfb[i] = 0;
            if (a.hfi) a.hfi[i] = 0;
            for (int k = 0; k < 8; ++k)
                if (a.x8) a.x8[(size_t)i * 8 + k] = 0;
            continue;
        }
        const CellRates<R> cr = cell_rates<R>(coef, coef64, rec, row, row64, L, L64);
        const R mu = noise_mult<R>(a.seed, (uint32_t)i, (uint32_t)a.period, a.rep, (R)a.sigma);
        R x[8];
        axis_rates<R>(cr, mu, x);
        if (a.hros) a.hros[i] = (double)(cr.h * mu);
        if (a.bros) a.bros[i] = (double)(cr.b * mu);
        if (a.fros) a.fros[i] = (double)((cr.h + cr.b) / ((R)2 * cr.lb) * mu);
        if (a.lb) a.lb[i] = (double)cr.lb;
        if (a.cfb || a.hfi) {
            R cfb = (R)0;
            const R hfi = head_intensity(cr, f, row, L, &cfb) * mu;
            if (a.cfb) a.cfb[i] = (double)cfb;
            if (a.hfi) a.hfi[i] = (double)hfi;
        }
        if (a.raz) {
            double az = 0.0;
            if (cr.wsv > (R)0) {
                az = (double)m_atan2(cr.wx, cr.wy) * (180.0 / 3.14159265358979323846);
                if (az < 0.0) az += 360.0;
            }
            a.raz[i] = az;
        }
        for (int k = 0; k < 8; ++k)
            if (a.x8) a.x8[(size_t)i * 8 + k] = (double)x[k];
    }
}

// The integer rates, by the evaluation of the propagation kernel: four lanes
// a cell, curves, weather row and landscape constants in LDS.
template <typename R>
__global__ __launch_bounds__(256) void eval_q8_kernel(EvalArgs a) {
    __shared__ EvalLds<double> s_x64;
    __shared__ EvalLds<float> s_x32;
    __shared__ EvalRep s_e;
    const EvalRep e{a.seed, a.rep, a.rounding, a.sigma, 0.f, mix_margin(a.sigma)};
    const int tid = (int)threadIdx.x, role = tid & 3;
    const size_t ro = ((size_t)a.scenario * a.n_wp + a.period) * kRowLen;
    if (tid < kNumCurves) {
        s_x64.coef[tid] = curve_entry<double>(tid);
        s_x32.coef[tid] = curve_entry<float>(tid);
    }
    if (tid < kNumFuels) {
        load_land<double>(a.land, s_x64.L, tid);
        load_land<float>(a.land, s_x32.L, tid);
    }
    if (tid < kRowLen) {
        s_x64.row[tid] = a.table64[ro + tid];
        s_x32.row[tid] = (float)((const R*)a.table)[ro + tid];
    }
    if (tid == 0) s_e = e;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 64 + (tid >> 2); i < a.n_cells; i += (int64_t)gridDim.x * 64) {
        const CellRec rec = a.cells[i];
        int32_t qa = 0, qb = 0;
        if (rec_fuel(rec.info) != 0)
            quad_axis_q<sizeof(R) == 8>(s_x32, s_x64, e, &s_e, rec,
                                        quad_draws<sizeof(R) == 8>(e, (uint32_t)i, (uint32_t)a.period, role), role, qa,
                                        qb);
        a.q8[(size_t)i * 8 + role] = qa;
        a.q8[(size_t)i * 8 + role + 4] = qb;
    }
}

hipError_t launch_eval_ros(int precision, const EvalArgs& a, hipStream_t s) {
    const int g = fill_grid((size_t)a.n_cells);
    if (precision == 1) hipLaunchKernelGGL(eval_ros_kernel<float>, dim3(g), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(eval_ros_kernel<double>, dim3(g), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.q8) return e;
    const int gq = (int)(((int64_t)a.n_cells + 63) / 64 < 8192 ? ((int64_t)a.n_cells + 63) / 64 : 8192);
    if (precision == 1) hipLaunchKernelGGL(eval_q8_kernel<float>, dim3(gq), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(eval_q8_kernel<double>, dim3(gq), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace c2f
