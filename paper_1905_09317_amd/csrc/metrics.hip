// Scar comparison of Section 4 (comparison methodology): per period t the
// simulated scar Y^t (cells whose arrival minute lies in [0, t P]) against a
// reference 0-1 scar X^t, by mean squared error, the structural similarity
// of Wang et al. (2004) over the whole grid (C1 = (0.01 L)^2, C2 =
// (0.03 L)^2, L = 1, N - 1 normalisation; the second denominator factor is
// sigma_x^2 + sigma_y^2 + C2, the printed formula repeating the means there)
// and the Frobenius norm of the last period's difference.
//
// For 0-1 scars every statistic follows from three counts per period: a =
// sum X, b = sum Y, c = sum X Y.  One launch counts them exactly (one 64-bit
// atomic per count and block into a zeroed buffer), and the block that
// finishes last forms the metrics in FP64 from the counts, with the products
// a b, c N and a (N - a) exact in 64-bit integers (N < 2^31), then returns
// the counts and its ticket to zero for the next launch.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.h"

namespace c2f {

// Metrics of period t from its counts (out[t] = MSE, out[T + t] = SSIM,
// out[2 T] = Frobenius norm of the last period).
__device__ void period_metrics(int64_t a, int64_t b, int64_t c, int t, int T, int64_t n, double* __restrict__ out) {
    const double N = (double)n, N1 = (double)(n - 1);
    const double C1 = 0.01 * 0.01, C2 = 0.03 * 0.03;
    const double mx = (double)a / N, my = (double)b / N;
    const double vx = (double)(a * (n - a)) / (N * N1);
    const double vy = (double)(b * (n - b)) / (N * N1);
    const double cxy = (double)(c * n - a * b) / (N * N1);
    const int64_t diff = a + b - 2 * c;   // cells where the scars differ
    out[t] = (double)diff / N;
    out[T + t] = ((2.0 * mx * my + C1) * (2.0 * cxy + C2)) / ((mx * mx + my * my + C1) * (vx + vy + C2));
    if (t == T - 1) out[2 * T] = sqrt((double)diff);
}

// Every block ends here with partial counts in LDS: part[k] adds to
// counts[base + k] for k < len.  The first wave adds them to the global
// counts, makes its atomics visible
// to the device (release fence) and takes a ticket; the block with the last
// ticket acquires, reads the finished counts, writes the metrics and clears
// counts and ticket for the next launch.  Only the first wave issues global
// atomics, so one release per block suffices; no block waits for another.
__device__ void finish_block(const uint32_t* part, int base, int len, unsigned long long* __restrict__ counts,
                             uint32_t* __restrict__ ticket, int T, int64_t n, double* __restrict__ out) {
    __shared__ bool s_last;
    __syncthreads();
    if (threadIdx.x < 64) {
        for (int k = (int)threadIdx.x; k < len; k += 64)
            if (part[k]) atomicAdd(&counts[base + k], (unsigned long long)part[k]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (threadIdx.x == 0) {
            const uint32_t nblocks = gridDim.x * gridDim.y;
            s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nblocks - 1;
        }
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // every block's counts are visible from here
    for (int t = (int)threadIdx.x; t < T; t += (int)blockDim.x) {
        unsigned long long v[3];
        for (int f = 0; f < 3; ++f) {
            v[f] = __hip_atomic_load(&counts[3 * t + f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&counts[3 * t + f], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        period_metrics((int64_t)v[0], (int64_t)v[1], (int64_t)v[2], t, T, n, out);
    }
    if (threadIdx.x == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// counts[3 t + {0, 1, 2}] += {a, b, c} of every period t in the block's range,
// streamed by each lane over 16 consecutive cells.  reference is [T][n],
// arrival [n] (-1 = unburned).  Y^t is monotone in t: cell i is in Y^t from its
// burn period k_i = ceil(m_i / P) - 1 on (0 for m_i = 0, never for
// m_i < 0), so each lane computes k_i once.  Periods go in windows of 127:
// with the bytes of kb = min(max(k_i - t_w, 0), 127) for four cells in one
// word, ((t - t_w) * 0x01010101 | 0x80808080) - kb has bit 7 of byte u set
// exactly when cell u is in Y^t (every byte stays in 1..254 for t - t_w up to 126,
// so no borrow crosses bytes; later periods of a batch are not counted); bit 7 of a byte of (((w & 0x7F..) + 0x7F..) | w) is set
// exactly when that byte of the reference word w is nonzero.  A lane's
// three counts (0..16 each) go packed in 10-bit fields through DPP sums
// over each 16-lane row (at most 256 per field), eight periods together; each
// row adds its sums to the block's counts of the periods in LDS, one 64-bit
// word with a field of 21 bits a count (a block counts at most 2^20 cells).
// Reference loads of kRowsBatch (8) periods are issued before any is used.
//
// Bound by the reference read.  The rows of a grid of n cells start n bytes
// apart, so unless n is a multiple of 16 a lane's 16 bytes straddle words:
// ALIGNED = false reads them with unaligned 16-byte loads (the last lane, whose
// cells may end the row, takes the row's last 16 bytes: byte by byte, 15 loads a
// period, it held up its block, 333 x 777 cells x 500 periods 80 us a call, 64 now).
// Periods are split over blockIdx.y in batches while blocks are fewer than the
// compute units hold.  1001 x 777 cells x 24 periods took 129 us with one block
// per 2048 cells and period, byte loads and ballots; 15.6 us here; 2048^2 x 48
// took 50.0 us with a DPP sum and LDS atomics for each period, 44.4 us with eight
// periods summed together (4.9 TB/s).
constexpr int kRowsBlock = 1024;
constexpr int kRowsPeriods = 1024;   // a block's periods at most, 20 bytes of LDS each
// kRowsMaxBlocks blocks of 16384 cells a stride reach 2^31 - 2 cells in 64
// strides, 2^20 cells a block.
constexpr int64_t kRowsMaxBlocks = 2048;
constexpr int64_t kRowsFill = 256;   // blocks that fill the compute units
constexpr int kRowsBatch = 8;
constexpr int kRowsWindow = 127;

// Bit 7 of each byte: is the byte nonzero (other bits have no meaning)?
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w) {
    return ((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}
// v of lane ^ 1, ^ 2, ^ 4 and ^ 8 (half mirror is ^ 7 and mirror ^ 15 in a row of 16)
__device__ __forceinline__ uint32_t xor1(uint32_t v) { return dpp<0xB1>(v); }
__device__ __forceinline__ uint32_t xor2(uint32_t v) { return dpp<0x4E>(v); }
__device__ __forceinline__ uint32_t xor4(uint32_t v) { return dpp<0x141>(dpp<0x1B>(v)); }
__device__ __forceinline__ uint32_t xor8(uint32_t v) { return dpp<0x140>(dpp<0x141>(v)); }

// Sums of eight values over each row of 16 lanes, value (lane & 7) in every
// lane: in three steps each lane keeps the half of its values whose number
// has its own lane bit, and adds its partner's part of them.
__device__ __forceinline__ uint32_t row_sums8(const uint32_t* r) {
    const int lane = (int)__lane_id();
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b2 = (lane & 4) != 0;
    uint32_t s[4], u[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = (b0 ? r[2 * k + 1] : r[2 * k]) + xor1(b0 ? r[2 * k] : r[2 * k + 1]);
#pragma unroll
    for (int k = 0; k < 2; ++k) u[k] = (b1 ? s[2 * k + 1] : s[2 * k]) + xor2(b1 ? s[2 * k] : s[2 * k + 1]);
    uint32_t v = (b2 ? u[1] : u[0]) + xor4(b2 ? u[0] : u[1]);
    return v + xor8(v);
}

// The bits 7 of the bytes of four words, side by side in the high halves of
// the bytes of one.
__device__ __forceinline__ uint32_t top_bits(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const uint32_t ab = (a & 0x80808080u) | (b >> 1 & ~0x80808080u), cd = (c & 0x80808080u) | (d >> 1 & ~0x80808080u);
    return ((ab & 0xC0C0C0C0u) | (cd >> 2 & ~0xC0C0C0C0u)) & 0xF0F0F0F0u;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The n < 16 bytes at p, zeros above them (a grid of fewer than 16 cells).
__device__ __forceinline__ u32x4 few_bytes(const uint8_t* p, int n) {
    uint64_t lo = 0, hi = 0;
#pragma unroll 1
    for (int u = 0; u < n; ++u) {
        const uint64_t b = p[u];
        if (u < 8) lo |= b << (8 * u);
        else hi |= b << (8 * (u - 8));
    }
    return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// Drops the lowest n of 16 bytes (0 < n < 16), zeros come in above.
__device__ __forceinline__ void drop_bytes(uint32_t* w, int n) {
    const uint64_t lo = (uint64_t)w[0] | (uint64_t)w[1] << 32, hi = (uint64_t)w[2] | (uint64_t)w[3] << 32;
    const int b = 8 * n;
    const uint64_t l = b < 64 ? lo >> b | hi << (64 - b) : hi >> (b - 64), h = b < 64 ? hi >> b : 0ull;
    w[0] = (uint32_t)l, w[1] = (uint32_t)(l >> 32), w[2] = (uint32_t)h, w[3] = (uint32_t)(h >> 32);
}

// Adds a row's packed sum to a period's count in LDS.
__device__ __forceinline__ void add_row(unsigned long long* cnt, uint32_t r) {
    atomicAdd(cnt, (unsigned long long)(r & 1023u) | (unsigned long long)((r >> 10) & 1023u) << 21 |
                       (unsigned long long)(r >> 20) << 42);
}

template <bool ALIGNED>
__global__ __launch_bounds__(kRowsBlock) void scar_counts_rows_kernel(const int32_t* __restrict__ arrival,
                                                                      const uint8_t* __restrict__ reference,
                                                                      int64_t n, int T, int per_block, int period_min,
                                                                      unsigned long long* __restrict__ counts,
                                                                      uint32_t* __restrict__ ticket,
                                                                      double* __restrict__ out) {
    typedef u32x4 u32x4_u1 __attribute__((aligned(1)));
    typedef int32_t i32x4_u4 __attribute__((ext_vector_type(4), aligned(4)));
    extern __shared__ unsigned long long s_rows[];   // [periods of the block], then 3 u32 counts of each
    const int p0 = (int)blockIdx.y * per_block, p1 = min(T, p0 + per_block), np = p1 - p0;
    for (int k = (int)threadIdx.x; k < np; k += kRowsBlock) s_rows[k] = 0;
    __syncthreads();
    const int64_t q = (n + 15) / 16;
    for (int64_t jb = (int64_t)blockIdx.x * kRowsBlock; jb < q; jb += (int64_t)gridDim.x * kRowsBlock) {
        // a wave without cells leaves its compute unit to the others
        if (jb + (int64_t)(threadIdx.x & ~63u) >= q) break;
        const int64_t j = jb + threadIdx.x;
        const int live = j < q ? (int)min((int64_t)16, n - 16 * j) : 0;   // the lane's cells (ALIGNED: all or none)
        int32_t kc[16];   // burn period of each of the lane's cells (0x7FFFFFFF = never)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int32_t m[4] = {-1, -1, -1, -1};
            if (live == 16) {
                if constexpr (ALIGNED) {
                    const int4 x = ((const int4*)arrival)[j * 4 + v];
                    m[0] = x.x, m[1] = x.y, m[2] = x.z, m[3] = x.w;
                } else {
                    const i32x4_u4 x = *(const i32x4_u4*)(arrival + 16 * j + 4 * v);
                    m[0] = x.x, m[1] = x.y, m[2] = x.z, m[3] = x.w;
                }
            } else if (!ALIGNED && live > 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = arrival[min(16 * j + 4 * v + u, n - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (4 * v + u >= live) m[u] = -1;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                kc[4 * v + u] = m[u] < 0 ? 0x7FFFFFFF : (m[u] == 0 ? 0 : (m[u] - 1) / period_min);
        }
        // the last lane's cells are read from the end of the row, and moved down
        const int over = live > 0 ? 16 - live : 0;
        for (int tw = p0; tw < p1; tw += kRowsWindow) {
            uint32_t kb[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                uint32_t w = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int32_t k = kc[4 * v + u];
                    const int32_t r = k <= tw ? 0 : (k - tw > kRowsWindow ? kRowsWindow : k - tw);
                    w |= (uint32_t)r << (8 * u);
                }
                kb[v] = w;
            }
            const int tend = min(p1, tw + kRowsWindow);
            for (int t0 = tw; t0 < tend; t0 += kRowsBatch) {
                uint32_t wb[kRowsBatch][4];
#pragma unroll
                for (int k = 0; k < kRowsBatch; ++k) {
                    u32x4 x = {0u, 0u, 0u, 0u};
                    const uint8_t* row = reference + (size_t)(t0 + k) * (size_t)n + 16 * (size_t)j;
                    if (live > 0 && t0 + k < tend) {
                        if constexpr (ALIGNED) x = *(const u32x4*)row;
                        else if (n >= 16) x = *(const u32x4_u1*)(row - over);
                        else x = few_bytes(row, live);
                    }
                    wb[k][0] = x.x, wb[k][1] = x.y, wb[k][2] = x.z, wb[k][3] = x.w;
                }
                if (!ALIGNED && over != 0 && n >= 16) {
#pragma unroll
                    for (int k = 0; k < kRowsBatch; ++k) drop_bytes(wb[k], over);
                }
                uint32_t r[kRowsBatch];
#pragma unroll
                for (int k = 0; k < kRowsBatch; ++k) {
                    const uint32_t tb = ((uint32_t)(t0 + k - tw) * 0x01010101u) | 0x80808080u;
                    const uint32_t x = top_bits(nonzero_bytes(wb[k][0]), nonzero_bytes(wb[k][1]),
                                                nonzero_bytes(wb[k][2]), nonzero_bytes(wb[k][3]));
                    const uint32_t y = top_bits(tb - kb[0], tb - kb[1], tb - kb[2], tb - kb[3]);
                    r[k] = (uint32_t)__popc(x) | (uint32_t)__popc(y) << 10 | (uint32_t)__popc(x & y) << 20;
                }
                const uint32_t v = row_sums8(r);
                const int k = (int)(threadIdx.x & 15);
                if (k < kRowsBatch && t0 + k < tend) add_row(&s_rows[t0 + k - p0], v);
            }
        }
    }
    // the block's counts as three words a period for finish_block
    uint32_t* const s_cnt = (uint32_t*)(s_rows + np);
    __syncthreads();
    for (int k = (int)threadIdx.x; k < np; k += kRowsBlock) {
        const unsigned long long v = s_rows[k];
        s_cnt[3 * k] = (uint32_t)(v & 0x1FFFFFull);
        s_cnt[3 * k + 1] = (uint32_t)((v >> 21) & 0x1FFFFFull);
        s_cnt[3 * k + 2] = (uint32_t)(v >> 42);
    }
    finish_block(s_cnt, 3 * p0, 3 * np, counts, ticket, T, n, out);
}

hipError_t launch_scar_metrics(const int32_t* arrival, const uint8_t* reference, int64_t n, int T, int period_min,
                               unsigned long long* counts, uint32_t* ticket, double* out, hipStream_t s) {
    if (n < 2 || T < 1 || T > 65535) return hipErrorInvalidValue;
    const int64_t q = (n + 15) / 16;
    const int64_t gx = (q + kRowsBlock - 1) / kRowsBlock;   // blocks over the cells
    // a block takes every period of its cells (kRowsPeriods at most), unless
    // that leaves the chip short of blocks: then fewer batches of periods each
    const int64_t batches = (T + kRowsBatch - 1) / kRowsBatch;
    const int64_t gy = std::min(batches, std::max<int64_t>(1, kRowsFill / gx));
    const int per_block = (int)std::min<int64_t>((batches + gy - 1) / gy * kRowsBatch, kRowsPeriods);
    const dim3 grid((unsigned)std::min(gx, kRowsMaxBlocks), (unsigned)((T + per_block - 1) / per_block));
    const size_t lds = (size_t)std::min(per_block, T) * 20;
    if (n % 16 == 0 && (uintptr_t)reference % 16 == 0 && (uintptr_t)arrival % 16 == 0)
        scar_counts_rows_kernel<true><<<grid, kRowsBlock, lds, s>>>(arrival, reference, n, T, per_block, period_min,
                                                                    counts, ticket, out);
    else
        scar_counts_rows_kernel<false><<<grid, kRowsBlock, lds, s>>>(arrival, reference, n, T, per_block, period_min,
                                                                     counts, ticket, out);
    return hipGetLastError();
}

}  // namespace c2f
