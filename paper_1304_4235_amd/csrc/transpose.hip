// Transposed recorded paths: the intersections grouped by the intersected
// particle, for the transposed column product of the reverse mode.
//
// Built once per geometry by a stable LSD radix sort of (particle, (row,
// factor)) pairs taken in row order, so each particle's entries stay in row
// order and every gather over them sums in a fixed order.
#include "internal.h"
#include "pair.h"

#include <algorithm>
#include <utility>

namespace rrt {

namespace {

constexpr int kBlock = 512;
constexpr int kRounds = 8;                     // items per thread per tile
constexpr int kTile = kBlock * kRounds;        // 4096 items per tile
constexpr int kWaves = kBlock / 64;
constexpr int kMaxDigitBits = 9;

template <int BITS>
__global__ void __launch_bounds__(kBlock)
k_hist32(const uint32_t* __restrict__ keys, int64_t n, int shift, uint64_t* __restrict__ hist,
         int64_t n_tiles)
{
    constexpr uint32_t kDigits = 1u << BITS;
    __shared__ uint32_t h[kDigits];
    if (threadIdx.x < kDigits) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = blockIdx.x * (int64_t)kTile;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t i = base + r * kBlock + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & (kDigits - 1)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kDigits) hist[threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// One tile's items in digit order, stable: each wave ranks its consecutive
// items with one ballot per digit bit over counts of its own (no block barrier
// between rounds), the waves' counts and the digits' are summed, and the items
// go through LDS into that order, so that the stores of a digit are consecutive
// (16 entries on average at 8 bits, where stores straight from the rounds touch
// a line each).  Bound by memory.  Measured on MI355X: 258M entries
// (16-bit index) 2 x 4.0 ms with stores from the rounds, 2 x 2.27 here; 417M
// entries (17-bit index) 3 x 5.1 ms at 8 bits, 2 x 3.9 at 9 bits a pass.
template <int BITS>
__global__ void __launch_bounds__(kBlock)
k_scatter32(const uint32_t* __restrict__ kin, const uint64_t* __restrict__ vin,
            uint32_t* __restrict__ kout, uint64_t* __restrict__ vout, int64_t n, int shift,
            const uint64_t* __restrict__ offs, int64_t n_tiles)
{
    constexpr uint32_t kDigits = 1u << BITS;
    __shared__ uint16_t s_cnt[kWaves][kDigits];   // of a wave so far, then before it
    __shared__ uint16_t s_start[kDigits];         // first place of each digit in the tile
    __shared__ uint32_t s_sum[kWaves];
    __shared__ uint64_t s_to[kDigits];            // where the tile's digits go, less s_start
    __shared__ uint64_t s_val[kTile];
    __shared__ uint32_t s_key[kTile];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (uint32_t d = lane; d < kDigits; d += 64) s_cnt[wave][d] = 0;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = blockIdx.x * (int64_t)kTile + wave * (64 * kRounds) + lane;
    uint32_t key[kRounds];
    uint64_t val[kRounds];
    uint16_t rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t i = base + r * 64;
        key[r] = i < n ? kin[i] : 0u;
        val[r] = i < n ? vin[i] : 0ull;
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool valid = base + r * 64 < n;
        const uint32_t d = (key[r] >> shift) & (kDigits - 1);
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t before = s_cnt[wave][d];
        rank[r] = (uint16_t)(before + (uint32_t)__popcll(m & lt));
        wave_sync();
        if (valid && (m & lt) == 0) s_cnt[wave][d] = (uint16_t)(before + (uint32_t)__popcll(m));
        wave_sync();
    }
    __syncthreads();
    // per digit: the waves' counts to their starts, then the digits' starts
    uint32_t total = 0;
    if (t < (int)kDigits)
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t v = s_cnt[w][t];
            s_cnt[w][t] = (uint16_t)total;
            total += v;
        }
    uint32_t incl = total;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_sum[wave] = incl;
    __syncthreads();
    uint32_t start = incl - total;
    for (int w = 0; w < wave; ++w) start += s_sum[w];
    if (t < (int)kDigits) {
        s_start[t] = (uint16_t)start;
        s_to[t] = offs[t * n_tiles + blockIdx.x] - start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (base + r * 64 < n) {
            const uint32_t d = (key[r] >> shift) & (kDigits - 1);
            const uint32_t at = (uint32_t)s_start[d] + s_cnt[wave][d] + rank[r];
            s_key[at] = key[r];
            s_val[at] = val[r];
        }
    }
    __syncthreads();
    const int64_t left = n - blockIdx.x * (int64_t)kTile;
    const int here = left < kTile ? (int)left : kTile;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int at = r * kBlock + t;
        if (at < here) {
            const uint32_t k = s_key[at];
            const uint64_t dst = s_to[(k >> shift) & (kDigits - 1)] + (uint64_t)at;
            if (dst < (uint64_t)n) {
                kout[dst] = k;
                vout[dst] = s_val[at];
            }
        }
    }
}

// start of particle j's entries: the first sorted key >= j (binary search)
__global__ void k_col_starts(const uint32_t* __restrict__ key, int64_t m, int64_t n,
                             uint64_t* __restrict__ col_off)
{
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j > n) return;
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)key[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    col_off[j] = (uint64_t)lo;
}

// y_j = sum over particle j's entries of factor * nu[row], in an order fixed by
// the entries: a wave per particle, eight streaming loads in flight per lane.
// Bound by memory and the gathers of nu.  Measured on MI355X (us with four, with
// eight loads): 258M entries 488, 473 (4.4 TB/s of entries); 417M 848, 824; two
// entries to a 16-byte load 483 and 849.
__global__ void __launch_bounds__(256)
k_gather_cols(const uint64_t* __restrict__ col_off, const uint64_t* __restrict__ ent,
              const float* __restrict__ nu, int64_t n, double* __restrict__ y)
{
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t col = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6; col < n;
         col += stride) {
        double acc = 0.0;
        const uint64_t a = col_off[col], b = col_off[col + 1];
        const long long* p = reinterpret_cast<const long long*>(ent);
        constexpr int U = 8;
        for (uint64_t e = a + lane; e < b; e += U * 64) {
            uint64_t v[U];
#pragma unroll
            for (int i = 0; i < U; ++i)
                v[i] = e + 64 * i < b ? (uint64_t)__builtin_nontemporal_load(p + e + 64 * i) : 0ull;
            float w[U];
#pragma unroll
            for (int i = 0; i < U; ++i) w[i] = nu[(uint32_t)v[i]];
#pragma unroll
            for (int i = 0; i < U; ++i)
                acc += (double)__int_as_float((int)(v[i] >> 32)) * (double)w[i];
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (lane == 0) y[col] = acc;
    }
}

}  // namespace

// Build the transposed paths into c.tpath / c.tcol_off, in the path buffer.
// Scratch: two key and one value buffer of path_hits entries, the sort
// histograms and their partial sums, also from the path buffer, released before
// returning.
// hipErrorOutOfMemory (nothing kept) when they do not fit beside the paths.
hipError_t build_transposed_paths(Ctx& c)
{
    const int64_t m = c.path_hits;
    const int64_t n = c.n;
    ws_free(c, &c.tpath);
    ws_free(c, &c.tcol_off);
    const int64_t mm = m > 0 ? m : 1;
    const int64_t n_tiles = (mm + kTile - 1) / kTile;
    // the fewest passes of at most 9 bits that cover the largest index
    int bits = 1;
    while ((int64_t(1) << bits) < n) ++bits;
    const int passes = (bits + kMaxDigitBits - 1) / kMaxDigitBits;
    const int digit = std::max((bits + passes - 1) / passes, 7);
    const size_t hn = (size_t)n_tiles << digit;
    Scratch<uint32_t> ka(c), kb(c);
    Scratch<uint64_t> vb(c), hist(c);
    hipError_t e = ws_alloc(c, &c.tpath, mm, kRegionPath);
    if (e == hipSuccess) e = ws_alloc(c, &c.tcol_off, n + 1, kRegionPath);
    if (e == hipSuccess) e = ka.get(mm, kRegionPath);
    if (e == hipSuccess) e = kb.get(mm, kRegionPath);
    if (e == hipSuccess) e = vb.get(mm, kRegionPath);
    if (e == hipSuccess) e = hist.get(hn, kRegionPath);
    if (e == hipSuccess && m > 0) {
        // (row, factor) of every recorded intersection, keyed by its particle
        e = ensure_row_offsets(c);
        if (e == hipSuccess) e = launch_expand_keys(c, ka.p, c.tpath);
    }
    uint32_t* kin = ka.p;
    uint32_t* kout = kb.p;
    uint64_t* vin = c.tpath;
    uint64_t* vout = vb.p;
    auto pass = [&](auto count, auto scatter, int shift) {
        hipLaunchKernelGGL(count, dim3((unsigned)n_tiles), dim3(kBlock), 0, c.stream, kin, m, shift,
                           hist.p, n_tiles);
        hipError_t r = hipGetLastError();
        if (r == hipSuccess)
            r = scan_exclusive_u64(c, hist.p, hist.p, (int64_t)hn, kRegionPath);
        if (r != hipSuccess) return r;
        hipLaunchKernelGGL(scatter, dim3((unsigned)n_tiles), dim3(kBlock), 0, c.stream, kin, vin,
                           kout, vout, m, shift, hist.p, n_tiles);
        return hipGetLastError();
    };
    for (int p = 0; p < passes && e == hipSuccess && m > 0; ++p) {
        e = digit == 7   ? pass(k_hist32<7>, k_scatter32<7>, digit * p)
            : digit == 8 ? pass(k_hist32<8>, k_scatter32<8>, digit * p)
                         : pass(k_hist32<9>, k_scatter32<9>, digit * p);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    // the sorted values are in vin; keep them as the transposed paths
    if (e == hipSuccess && vin != c.tpath)
        e = hipMemcpyAsync(c.tpath, vin, sizeof(uint64_t) * m, hipMemcpyDeviceToDevice, c.stream);
    // particle starts from the sorted keys
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_col_starts, dim3((unsigned)((n + 1 + 255) / 256)), dim3(256), 0,
                           c.stream, kin, m, n, c.tcol_off);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        ws_free(c, &c.tpath);
        ws_free(c, &c.tcol_off);
    }
    return e;
}

hipError_t launch_gather_cols(Ctx& c)
{
    hipLaunchKernelGGL(k_gather_cols, dim3(stride_blocks(c.n, 4)), dim3(256), 0,
                       c.stream, c.tcol_off, c.tpath, c.adj_nu, c.n, c.adj_y);
    return hipGetLastError();
}

}  // namespace rrt
