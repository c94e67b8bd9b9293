// Recorded ray paths (Sec. 4.1.1, eq. colden): the column is linear in the
// neutral fractions, so which particles a ray meets and the kernel chord
// factor K/h^2 of each are recorded once per geometry, and every column
// evaluation is a product over them.  The layout is described in internal.h:
// the 64 rays of a packet together, cut into segments.
//
//   k_build_paths    the log of the recording walk (trace.hip) into segments,
//                    with each hit's factor
//   k_path_columns   N = sum of mux_j * factor over every ray's entries
//   k_path_scatter   y_j += factor * nu over the same entries
//   k_path_rows      the entries by rows, for what needs them that way
#include "internal.h"
#include "pair.h"
#include "segment.h"

#include <algorithm>
#include <type_traits>

namespace rrt {

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

}  // namespace

int64_t path_packets(const Ctx& c) { return ((c.n + 63) / 64) * (int64_t)c.n_ray; }

// A packet is one wave's work in the walk.  With few packets for the device (6
// waves on each of 1024 SIMDs), each is split: into ranges of the tree's nodes,
// or in a periodic box into groups of its rays (so that a ray's hits stay in
// the order of one walk over its images).
//  * Node ranges, to at least 49152 units (8 a wave, as ranges differ in work):
//    the 16384-particle halo's walk 574 us at half as many units, 526 us here,
//    the 65521-particle halo's 2580 and 2323 us.
//  * Ray groups repeat the packet's node visits, and their segments are shorter,
//    which the product pays for: the 4096-particle lattice's walk and product at
//    1, 4, 8, 16 groups 698 (before the queues) and 21, 323 and 21, 360 and 27,
//    532 and 41 us.
int path_parts(const Ctx& c)
{
    const int64_t pk = path_packets(c);
    const int most = c.prm.box > 0.0 ? std::min(4, c.parts_most) : c.parts_most;
    int p = 1;
    while (p < most && pk * p < (c.prm.box > 0.0 ? 6144 : 49152)) p *= 2;
    return p;
}

// Log blocks a wave takes at once: the counter they come from is one word, on
// which the device's waves contend (what a wave holds at the end stays unused).
uint32_t log_take(const Ctx& c) { return c.packet_queue && !c.log_tight ? kLogCache : 1u; }

// ---------------------------------------------------------------------------
// the log into segments
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)

namespace {

// per wave: which hit each entry is, the rays' groups and the visits
constexpr int32_t kOwnImage = INT32_MIN;
constexpr uint32_t kPlaceFill = 0x8000u;       // no hit: slot kSegFill, factor 0

struct BuildLds {
    int32_t img[3][kSegVisits];       // periodic image, kOwnImage for none
    uint32_t vis[kSegVisits];
    float org[3 * kRayPacket];
    uint16_t place[4 * kSegGroups];   // particle of the leaf | visit << 4, by group in ray order
    uint16_t base[kSegVisits];        // first slot of each visit
    uint16_t first[kRayPacket];       // first group of each ray
    uint8_t ray[kSegGroups];
};

// One wave per segment.  The log's words spread over the lanes, each lane
// writing its ray's hits of one leaf visit into the place table (LDS); then a
// lane per group in stored order: the four chord factors (the walk's own pair
// arithmetic, so the factors are those every other evaluation of a hit
// produces) and coalesced stores.
// Bound by vector issue (80% of the SIMDs' cycles, 157 instructions to an
// intersection with the log's share): the factor's arithmetic, without the
// image shift where no lane of the wave has one.  Measured on MI355X: the 885k-
// particle field's 3.37e9 intersections 19.4 ms with the shift's adds always and
// the FP64 division, 18.2 ms here; the 262144-particle halo's 1.57e9 8.25 and
// 7.6 ms.  Not branching in the factor, so that a lane's four interleave, took
// 20.5 ms: most chords span their sphere and skip a table lookup.
template <bool NF>
__global__ void __launch_bounds__(kBlock)
k_build_paths(const uint64_t* __restrict__ log, const uint64_t* __restrict__ seg_src,
              const uint32_t* __restrict__ seg_unit, const uint64_t* __restrict__ seg_off,
              int64_t n_segs, int parts, uint4* __restrict__ packed,
              const float4* __restrict__ p4, const double* __restrict__ dirs,
              const KernelTables* __restrict__ tabs, TraceGeom g)
{
    __shared__ float4 t_erf[kTabIntervals];
    __shared__ BuildLds s_all[kWaves];
    for (int i = threadIdx.x; i < kTabIntervals; i += blockDim.x) t_erf[i] = tabs->erf_t[i];
    __syncthreads();
    const double gc = tabs->gauss_c, ga = tabs->gauss_a;
    const double L = __builtin_canonicalize(g.L), B = g.box;
    const int lane = threadIdx.x & 63;
    BuildLds& S = s_all[threadIdx.x >> 6];
    const int64_t wpd = (g.n + 63) / 64;
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    for (int64_t sg = blockIdx.x * (int64_t)kWaves + (threadIdx.x >> 6); sg < n_segs;
         sg += stride) {
        const uint64_t src = seg_src[sg];
        uint32_t blk = __builtin_amdgcn_readfirstlane((uint32_t)(src / kLogBlock));
        uint32_t pos = __builtin_amdgcn_readfirstlane((uint32_t)(src % kLogBlock));
        const int64_t pk = (int64_t)seg_unit[sg] / parts;
        const int k = __builtin_amdgcn_readfirstlane((int)(pk / wpd));
        const int ps = (int)(pk - (int64_t)k * wpd) * 64 + lane;
        const double u[3] = {dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]};
        const float4 P = p4[ps < g.n ? ps : g.n - 1];
        wave_sync();                           // the previous segment's reads are done
        S.org[lane] = P.x;
        S.org[64 + lane] = P.y;
        S.org[128 + lane] = P.z;
        uint4* dst = packed + seg_off[sg];
        uint32_t next, used;
        // the block's link word: the next block and the words used in this one
        auto load_link = [&]() {
            const uint64_t l = log[(uint64_t)blk * kLogBlock + kLogData];
            used = __builtin_amdgcn_readfirstlane((uint32_t)(l >> 32));
            next = __builtin_amdgcn_readfirstlane((uint32_t)l);
        };
        load_link();
        {
            const uint64_t* h = log + (uint64_t)blk * kLogBlock + pos;
            const uint64_t h0 = h[0];
            const uint32_t cnt = reinterpret_cast<const uint16_t*>(h + 3)[lane];
            pos += kLogHeader;
            uint32_t words = __builtin_amdgcn_readfirstlane((uint32_t)h0);
            const uint32_t n_vis =
                __builtin_amdgcn_readfirstlane((uint32_t)(h0 >> 32) & 0xffffu);
            const uint32_t slots = __builtin_amdgcn_readfirstlane((uint32_t)(h0 >> 48));
            const uint32_t gr = (cnt + 3u) >> 2;
            uint32_t incl = gr;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t y = __shfl_up(incl, off, 64);
                if (lane >= off) incl += y;
            }
            const uint32_t groups = __builtin_amdgcn_readlane(incl, 63);
            const uint32_t first = incl - gr;
            S.first[lane] = (uint16_t)first;
            for (uint32_t i = 0; i < gr; ++i) S.ray[first + i] = (uint8_t)lane;
            for (uint32_t i = cnt; i < 4u * gr; ++i) S.place[4u * first + i] = kPlaceFill;
            wave_sync();
            // the log's words, up to 64 at a time, never across a block
            while (words > 0) {
                if (pos >= used) {
                    if (next == kNoBlock) break;     // (a whole log never ends early)
                    blk = next;
                    load_link();
                    pos = 0;
                }
                uint32_t m = words < 64u ? words : 64u;
                if (m > used - pos) m = used - pos;
                const uint64_t w = (uint32_t)lane < m ? log[(uint64_t)blk * kLogBlock + pos + lane]
                                                      : 3ull << 62;
                pos += m;
                words -= m;
                const uint32_t type = (uint32_t)(w >> 62);
                const uint32_t v = (uint32_t)(w >> 43) & (kSegVisits - 1);
                if (type == (uint32_t)kLogVisit) {
                    S.vis[v] = (uint32_t)w;
                    S.img[0][v] = kOwnImage;
                }
                wave_sync();
                if (type == (uint32_t)kLogImage) {
                    const uint32_t iv = (uint32_t)(w >> 54) & (kSegVisits - 1);
                    if ((w >> 61) & 1ull) {
                        S.img[(uint32_t)(w >> 32) & 3u][iv] = (int32_t)(uint32_t)w;
                    } else {
                        S.img[0][iv] = (int)(w & 0x3ffffu) - kMaxImage;
                        S.img[1][iv] = (int)((w >> 18) & 0x3ffffu) - kMaxImage;
                        S.img[2][iv] = (int)((w >> 36) & 0x3ffffu) - kMaxImage;
                    }
                }
                if (type == (uint32_t)kLogHits) {
                    uint32_t mask = (uint32_t)w & 0xffffu;
                    const uint32_t ray = (uint32_t)(w >> 16) & 63u;
                    uint32_t i = 4u * S.first[ray] + ((uint32_t)(w >> 22) & 0xfffu);
                    const uint32_t tag = v << 4;
                    while (mask) {
                        S.place[i++] = (uint16_t)(tag | ((uint32_t)__ffs(mask) - 1u));
                        mask &= mask - 1u;
                    }
                }
            }
            wave_sync();
            // the visits' first slots
            uint32_t slot0 = 0;
            for (uint32_t v0 = 0; v0 < n_vis; v0 += 64) {
                const uint32_t v = v0 + lane;
                const uint32_t c = v < n_vis ? (S.vis[v] & (kLeafMax - 1)) + 1u : 0u;
                uint32_t in = c;
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t y = __shfl_up(in, off, 64);
                    if (lane >= off) in += y;
                }
                if (v < n_vis) S.base[v] = (uint16_t)(slot0 + in - c);
                slot0 += __builtin_amdgcn_readlane(in, 63);
            }
            wave_sync();
            if (lane == 0)
                dst[0] = make_uint4(n_vis | (slots << 16), groups, segment_words(n_vis, groups), 0u);
            uint32_t* d_vis = reinterpret_cast<uint32_t*>(dst + 1);
            for (uint32_t i = lane; i < n_vis; i += 64) d_vis[i] = S.vis[i];
            float4* d_fac = reinterpret_cast<float4*>(dst + 1 + (n_vis + 3) / 4);
            uint32_t* d_abc = reinterpret_cast<uint32_t*>(d_fac + groups);
            uint16_t* d_dr = reinterpret_cast<uint16_t*>(d_fac + groups + (groups + 3) / 4);
            for (uint32_t at = lane; at < groups; at += 64) {
                const uint32_t e = group_at(at, groups);
                const uint32_t r = S.ray[e];
                const double o0 = (double)S.org[r], o1 = (double)S.org[64 + r],
                             o2 = (double)S.org[128 + r];
                const uint64_t four = *reinterpret_cast<const uint64_t*>(S.place + 4 * e);
                uint32_t slot[4], bits[4], n_used = 0, pl = 0;
                float4 Q[4];
                uint32_t vis[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t x = (uint32_t)(four >> (16 * i)) & 0xffffu;
                    if (!(x & kPlaceFill)) {
                        pl = x;
                        ++n_used;
                    }
                    vis[i] = pl >> 4;
                    slot[i] = x & kPlaceFill ? kSegFill : S.base[vis[i]] + (pl & 15u);
                    Q[i] = p4[(S.vis[vis[i]] >> kLeafShift) + (pl & 15u)];
                }
                auto factors = [&](auto shifted_tag) {
                constexpr bool kShifted = decltype(shifted_tag)::value;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    double sh[3] = {0.0, 0.0, 0.0};
                    if (kShifted) {
                        const int s0 = S.img[0][vis[i]];
                        const bool own = s0 == kOwnImage;
                        sh[0] = own ? 0.0 : (double)s0 * B;
                        sh[1] = own ? 0.0 : (double)S.img[1][vis[i]] * B;
                        sh[2] = own ? 0.0 : (double)S.img[2][vis[i]] * B;
                    }
                    const PairGeom pg =
                        pair_geom_d<kShifted>((double)Q[i].x, (double)Q[i].y, (double)Q[i].z, o0,
                                              o1, o2, sh, u);
                    bits[i] = (uint32_t)__float_as_int(hit_factor(pg, u, Q[i].w, L, t_erf, gc, ga));
                    if (NF) {
                        const double hj = (double)Q[i].w, h2 = hj * hj;
                        if ((pg.d0 * pg.d0 + pg.d1 * pg.d1 + pg.d2 * pg.d2) < h2)
                            bits[i] |= kNearBit;
                    }
                    if ((uint32_t)i >= n_used) bits[i] = 0u;
                }
                };
                // the image shift, 0 for the source's own image as in the walk: few
                // waves hold a shifted one, the others leave its work out
                bool any = false;
                if (B > 0.0)
                    for (int i = 0; i < 4; ++i) any = any || S.img[0][vis[i]] != kOwnImage;
                if (wave_ballot(any)) factors(std::true_type{});
                else factors(std::false_type{});
                d_fac[at] = make_float4(__int_as_float((int)bits[0]), __int_as_float((int)bits[1]),
                                        __int_as_float((int)bits[2]), __int_as_float((int)bits[3]));
                d_abc[at] = slot[0] | (slot[1] << 10) | (slot[2] << 20) | ((n_used - 1u) << 30);
                d_dr[at] = (uint16_t)(slot[3] | (r << 10));
            }
        }
    }
}

}  // namespace

#pragma clang fp contract(fast)

namespace {

// The units' sizes summed.  One atomic per block and sum: they queue up on one
// word each, some 16 ns apart (the 16384-particle halo's 49152 units: 39 us with
// one per wave, 12 here).
__global__ void __launch_bounds__(kBlock)
k_sum_units(const uint64_t* __restrict__ unit_size, const uint2* __restrict__ unit_log,
            int64_t n_units, unsigned long long* __restrict__ red)
{
    __shared__ unsigned long long s_sum[kWaves][4];
    unsigned long long words = 0, blocks = 0, segs = 0, most = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_units; i += stride) {
        words += unit_size[i] & 0xffffffffull;
        blocks += unit_size[i] >> 32;
        most = std::max<unsigned long long>(most, unit_size[i] >> 32);
        if (unit_log) segs += unit_log[i].y;
    }
    for (int off = 32; off > 0; off >>= 1) {
        words += __shfl_xor(words, off, 64);
        blocks += __shfl_xor(blocks, off, 64);
        segs += __shfl_xor(segs, off, 64);
        most = std::max<unsigned long long>(most, __shfl_xor(most, off, 64));
    }
    unsigned long long* w = s_sum[threadIdx.x >> 6];
    if ((threadIdx.x & 63) == 0) {
        w[0] = words;
        w[1] = blocks;
        w[2] = segs;
        w[3] = most;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int q = 1; q < kWaves; ++q) {
        words += s_sum[q][0];
        blocks += s_sum[q][1];
        segs += s_sum[q][2];
        most = std::max(most, s_sum[q][3]);
    }
    if (words) {
        atomicAdd(red + kRedPathSize, words);
        atomicAdd(red + kRedPathBlocks, blocks);
        atomicAdd(red + kRedPathSegs, segs);
        atomicMax(red + kRedPathMost, most);
    }
}

__global__ void __launch_bounds__(kBlock)
k_unit_words(uint64_t* __restrict__ unit_off, const uint2* __restrict__ unit_log, int64_t n_units,
             uint64_t* __restrict__ unit_seg)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i > n_units) return;
    unit_off[i] = i < n_units ? unit_off[i] & 0xffffffffull : 0ull;
    unit_seg[i] = i < n_units ? unit_log[i].y : 0u;
}

// each segment's header in the log, its unit and its place, from the chain of
// its unit's headers
__global__ void __launch_bounds__(kBlock)
k_index_segments(const uint64_t* __restrict__ log, const uint2* __restrict__ unit_log,
                 const uint64_t* __restrict__ unit_off, const uint64_t* __restrict__ unit_seg,
                 int64_t unit0, int64_t n_units, uint64_t* __restrict__ seg_src,
                 uint32_t* __restrict__ seg_unit, uint64_t* __restrict__ seg_off)
{
    const int64_t u = unit0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (u >= unit0 + n_units) return;
    const uint2 ul = unit_log[u];
    uint64_t at = (uint64_t)ul.x * kLogBlock, w = unit_off[u];
    const uint64_t s = unit_seg[u];
    for (uint32_t i = 0; i < ul.y; ++i) {
        const uint64_t h0 = log[at], groups = log[at + 1], next = log[at + 2];
        seg_src[s + i] = at;
        seg_unit[s + i] = (uint32_t)u;
        seg_off[s + i] = w;
        w += segment_words((uint32_t)(h0 >> 32) & 0xffffu, (uint32_t)groups);
        at = next;
    }
}

}  // namespace

hipError_t launch_sum_units(Ctx& c, const uint64_t* unit_size, bool segments)
{
    const int64_t units = path_packets(c) * path_parts(c);
    hipLaunchKernelGGL(k_sum_units,
                       dim3((unsigned)std::min<int64_t>((units + kBlock - 1) / kBlock, 256)),
                       dim3(kBlock), 0, c.stream, unit_size, segments ? c.unit_log : nullptr, units,
                       c.red);
    return hipGetLastError();
}

hipError_t launch_unit_words(Ctx& c)
{
    const int64_t units = path_packets(c) * path_parts(c);
    hipLaunchKernelGGL(k_unit_words, dim3((unsigned)((units + kBlock) / kBlock)), dim3(kBlock), 0,
                       c.stream, c.unit_off, c.unit_log, units, c.unit_seg);
    return hipGetLastError();
}

hipError_t launch_build_paths(Ctx& c)
{
    return launch_build_range(c, 0, path_packets(c) * path_parts(c), 0, c.path_segs);
}

// the log of units unit0 and on, their segments seg0 and on
hipError_t launch_build_range(Ctx& c, int64_t unit0, int64_t units, uint64_t seg0, uint64_t n_segs)
{
    const int parts = path_parts(c);
    const int64_t segs = (int64_t)n_segs;
    if (segs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_index_segments, dim3((unsigned)((units + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, c.stream, c.path_log, c.unit_log, c.unit_off, c.unit_seg,
                       unit0, units, c.seg_src, c.seg_unit, c.seg_off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned nb = (unsigned)std::min<int64_t>((segs + kWaves - 1) / kWaves, kMaxBlocks);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, c.stream, c.path_log,
                           c.seg_src + seg0, c.seg_unit + seg0, c.seg_off + seg0, segs, parts, c.packed, c.p4, c.dirs, c.tables,
                           c.geom);
    };
    if (c.near_far) go(k_build_paths<true>);
    else go(k_build_paths<false>);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// columns from recorded paths
// ---------------------------------------------------------------------------
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// A block of W waves takes one packet, its waves every W-th segment (W = 1: a
// block of four waves takes four packets).  A segment's mux is staged in LDS
// once; then each lane takes groups, whose four products sum in FP64 and are
// added to their ray's sum in LDS.  The groups are independent, so every lane
// is busy and the loads run ahead.  A wave's instructions add in order and the
// waves' sums in theirs; the lanes of one LDS atomic that add to the same ray were
// always seen to add in the same order (no document promises it), and with that the
// columns do not depend on the run, which the tests hold to the bit.  Rows of sources
// that are not evaluated keep their columns.
__device__ __forceinline__ void lds_add(double* p, double v) { unsafeAtomicAdd(p, v); }

template <bool STREAM, typename T>
__device__ __forceinline__ T load_once(const T* p)
{
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}

template <bool NF, int W, bool STREAM>
__global__ void __launch_bounds__(W == 1 ? kBlock : 64 * W, NF ? 4 : 6)
k_path_columns(const uint64_t* __restrict__ unit_seg, const uint64_t* __restrict__ seg_off,
               const uint4* __restrict__ packed, int parts, const float* __restrict__ mux,
               int64_t n_packets, double* __restrict__ N,
               int n, const int32_t* __restrict__ seg_of, const int32_t* __restrict__ seg_active,
               const uint8_t* __restrict__ want, const unsigned long long* __restrict__ stop,
               double* __restrict__ Nn, const double* __restrict__ mu)
{
    constexpr int kW = W == 1 ? kWaves : W;
    constexpr int U = 4;                             // groups in flight per lane
    __shared__ float s_mux[kW][kSegSlots];
    __shared__ float s_mu[NF ? kW : 1][NF ? kSegSlots : 1];
    __shared__ double s_acc[kW][64];
    __shared__ double s_accn[NF ? kW : 1][NF ? 64 : 1];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t wpd = (n + 63) / 64;
    const int64_t pk = W == 1 ? blockIdx.x * (int64_t)kW + wv : (int64_t)blockIdx.x;
    if (pk >= n_packets) return;                     // whole wave (W = 1)
    const int64_t k = pk / wpd;
    const int ps = (int)(pk - k * wpd) * 64 + lane;
    bool live = ps < n;
    if (live && seg_active) live = seg_active[seg_of[ps]] != 0;
    if (live && want) live = want[ps] != 0;
    if (wave_ballot(live) == 0) return;              // the whole packet
    const bool stopped = stop && *stop != 0ull;
    s_acc[wv][lane] = 0.0;
    if (NF) s_accn[wv][lane] = 0.0;
    uint64_t sg = unit_seg[pk * parts] + (W == 1 ? 0 : wv);
    const uint64_t end = unit_seg[(pk + 1) * parts];
    float* sx = s_mux[wv];
    if (lane == 0) sx[kSegFill] = 0.0f;              // of the groups' unused entries
    float* sn = NF ? s_mu[wv] : nullptr;
    // the next segment's header and visits are loaded while one is worked on
    // (64 visits' words, of which the header says how many there are)
    uint64_t o = 0, o1 = 0;
    uint4 h = make_uint4(0, 0, 0, 0);
    uint32_t w = 0;
    if (sg < end) {
        o = seg_off[sg];
        if (sg + W < end) o1 = seg_off[sg + W];
        h = packed[o];
        w = reinterpret_cast<const uint32_t*>(packed + o + 1)[lane];
    }
    for (; sg < end; sg += W) {
        const Segment g = segment_of(packed + o, h);
        const uint32_t w0 = w;
        o = o1;
        if (sg + W < end) {
            h = packed[o];
            w = reinterpret_cast<const uint32_t*>(packed + o + 1)[lane];
            if (sg + 2 * W < end) o1 = seg_off[sg + 2 * W];
        }
        const v4f* fp = reinterpret_cast<const v4f*>(g.fac);
        v4f f[U];
        uint32_t a[U], d[U];
        auto load = [&](uint32_t at) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const uint32_t e = at + 64 * i;
                f[i] = v4f(0.0f);
                a[i] = d[i] = 0;
                if (e < g.n_groups) {
                    f[i] = load_once<STREAM>(fp + e);
                    a[i] = load_once<STREAM>(g.abc + e);
                    d[i] = load_once<STREAM>(g.dr + e);
                }
            }
        };
        load(lane);                                  // in flight while the slots are staged
        wave_sync();                                 // the previous segment's reads are done
        for_slots(g, lane, w0, [&](uint32_t slot, int j) {
            sx[slot] = mux[j];
            if (NF) sn[slot] = (float)mu[j];
        });
        wave_sync();
        for (uint32_t at = lane; at - lane < g.n_groups; at += 64 * U) {
            if (at != (uint32_t)lane) load(at);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                if (at + 64 * i >= g.n_groups) continue;
                const uint32_t sl[4] = {a[i] & 1023u, (a[i] >> 10) & 1023u, (a[i] >> 20) & 1023u,
                                        d[i] & 1023u};
                const uint32_t ray = d[i] >> 10;
                double acc = 0.0, accn = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!NF) {
                        acc += (double)(sx[sl[q]] * f[i][q]);
                    } else {
                        const uint32_t b = (uint32_t)__float_as_int(f[i][q]);
                        const float ff = __int_as_float((int)(b & ~kNearBit));
                        if (b & kNearBit) accn += (double)(sn[sl[q]] * ff);
                        else acc += (double)(sx[sl[q]] * ff);
                    }
                }
                lds_add(&s_acc[wv][ray], acc);
                if (NF) lds_add(&s_accn[wv][ray], accn);
            }
        }
    }
    const int64_t row = k * n + ps;
    if (W == 1) {
        wave_sync();
        if (live && !stopped) {
            N[row] = s_acc[wv][lane];
            if (NF) Nn[row] = s_accn[wv][lane];
        }
    } else {
        __syncthreads();
        if (wv == 0 && live && !stopped) {
            double acc = 0.0, accn = 0.0;
            for (int q = 0; q < W; ++q) {
                acc += s_acc[q][lane];
                if (NF) accn += s_accn[q][lane];
            }
            N[row] = acc;
            if (NF) Nn[row] = accn;
        }
    }
}

template <bool NF, bool STREAM>
void launch_columns_as(Ctx& c, int W)
{
    const int64_t pk = path_packets(c);
    auto go = [&](auto kernel, int64_t blocks, int threads) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, c.stream, c.unit_seg,
                           c.seg_off, c.packed, path_parts(c), c.mux_s, pk, c.N_s, (int)c.n,
                           c.geom.seg_of, c.geom.seg_active, c.geom.want, c.batch_stop, c.Nn_s,
                           c.mu_s);
    };
    if (W == 1) go(k_path_columns<NF, 1, STREAM>, (pk + kWaves - 1) / kWaves, kBlock);
    else if (W == 2) go(k_path_columns<NF, 2, STREAM>, pk, 128);
    else if (W == 4) go(k_path_columns<NF, 4, STREAM>, pk, 256);
    else go(k_path_columns<NF, 8, STREAM>, pk, 512);
}

template <bool NF>
void launch_columns_nf(Ctx& c)
{
    const int v = path_variant(c);
    if (v > 8) launch_columns_as<NF, true>(c, v - 8);
    else launch_columns_as<NF, false>(c, v);
}

// Visit every group of a packet's segments as stored, a lane per group: f(its
// place in ray order, ray, particles, factor bits, entries in use);
// begin(segment) and end(segment) are called around each by the whole wave.
// s_j: kSegSlots slots of LDS.
template <typename B, typename F, typename E>
__device__ __forceinline__ void for_groups(const uint64_t* __restrict__ unit_seg,
                                           const uint64_t* __restrict__ seg_off,
                                           const uint4* __restrict__ packed, int64_t pk, int parts,
                                           int lane, int32_t* s_j, B begin, F f, E end_seg)
{
    const uint64_t end = unit_seg[(pk + 1) * parts];
    for (uint64_t sg = unit_seg[pk * parts]; sg < end; ++sg) {
        const Segment g = segment_at(packed + seg_off[sg]);
        wave_sync();
        for_slots(g, lane, (uint32_t)lane < g.n_vis ? g.vis[lane] : 0u,
                  [&](uint32_t slot, int j) { s_j[slot] = j; });
        begin(g);
        wave_sync();
        for (uint32_t at = lane; at < g.n_groups; at += 64) {
            const uint32_t e = group_at(at, g.n_groups);
            const float4 fq = g.fac[at];
            const uint32_t a = g.abc[at], d = g.dr[at];
            const int j[4] = {s_j[a & 1023u], s_j[(a >> 10) & 1023u], s_j[(a >> 20) & 1023u],
                              s_j[d & 1023u]};
            const uint32_t b[4] = {(uint32_t)__float_as_int(fq.x), (uint32_t)__float_as_int(fq.y),
                                   (uint32_t)__float_as_int(fq.z), (uint32_t)__float_as_int(fq.w)};
            f(e, (int)(d >> 10), j, b, (a >> 30) + 1u);
        }
        wave_sync();
        end_seg(g);
    }
}

// A ray's groups are consecutive in ray order and all but its last are full, so
// entry q of group e is the ray's entry 4 (e - first) + q of the segment, with
// first its lowest group (s_first, found before the groups are visited).
__device__ __forceinline__ void find_first(const Segment& g, int lane, uint32_t* s_first)
{
    s_first[lane] = ~0u;
    wave_sync();
    for (uint32_t at = lane; at < g.n_groups; at += 64)
        atomicMin(&s_first[g.dr[at] >> 10], group_at(at, g.n_groups));
}
__device__ __forceinline__ void count_entries(const Segment& g, int lane, uint64_t* s_w)
{
    for (uint32_t at = lane; at < g.n_groups; at += 64)
        atomicAdd((unsigned long long*)&s_w[g.dr[at] >> 10],
                  (unsigned long long)((g.abc[at] >> 30) + 1u));
}

// intersections per row
__global__ void __launch_bounds__(kBlock)
k_path_row_sizes(const uint64_t* __restrict__ unit_seg, const uint64_t* __restrict__ seg_off,
             const uint4* __restrict__ packed,
                 int64_t n_packets, int parts, int n, uint64_t* __restrict__ row_cnt)
{
    __shared__ uint64_t s_w[kWaves][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t wpd = (n + 63) / 64;
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    for (int64_t pk = blockIdx.x * (int64_t)kWaves + wv; pk < n_packets; pk += stride) {
        s_w[wv][lane] = 0;
        wave_sync();
        const uint64_t end = unit_seg[(pk + 1) * parts];
        for (uint64_t sg = unit_seg[pk * parts]; sg < end; ++sg)
            count_entries(segment_at(packed + seg_off[sg]), lane, s_w[wv]);
        wave_sync();
        const int64_t k = pk / wpd;
        const int ps = (int)(pk - k * wpd) * 64 + lane;
        if (ps < n) row_cnt[k * n + ps] = s_w[wv][lane];
        wave_sync();
    }
}

// The entries by rows, at row_off: KEYS false: (tree index, factor); true: the
// tree index as a key and (factor bits << 32 | row) as its value.
// A segment's groups come in stored order (coalesced) and go through LDS into
// ray order, where consecutive lanes write consecutive entries of a row, four
// lanes to a group.  A block takes a packet, its waves every segment together:
// bound by the chain of steps in a segment, so 32 waves are to be resident.  Measured
// on MI355X, 258M intersections: a lane per group in ray order, straight from
// memory, 3.10 ms (KEYS) and 2.16 ms; here 1.78 and 1.22 ms.
struct RowsLds {
    float fac[4 * (kSegGroups + kSegGroups / 8)];
    uint32_t abc[kSegGroups];
    int32_t j[kSegSlots];
    uint16_t dr[kSegGroups];
    uint16_t first[kRayPacket];       // first group of each ray
    uint64_t to[kRayPacket];          // where its next entry goes
};

template <bool KEYS>
__global__ void __launch_bounds__(kBlock)
k_path_rows(const uint64_t* __restrict__ unit_seg, const uint64_t* __restrict__ seg_off,
            const uint4* __restrict__ packed, int64_t pk0, int64_t n_packets, int parts, int n,
            const uint64_t* __restrict__ row_off, int2* __restrict__ path,
            uint32_t* __restrict__ key, uint64_t* __restrict__ val)
{
    __shared__ RowsLds S;
    const uint32_t t = threadIdx.x;
    const int lane = t & 63;
    const int64_t wpd = (n + 63) / 64;
    for (int64_t pk = pk0 + blockIdx.x; pk < n_packets; pk += gridDim.x) {
        const int64_t k = pk / wpd, p0 = (pk - k * wpd) * 64;
        if (t < 64) S.to[t] = p0 + t < n ? row_off[k * n + p0 + t] : 0ull;
        const uint32_t row0 = (uint32_t)(k * n + p0);
        const uint64_t end = unit_seg[(pk + 1) * parts];
        for (uint64_t sg = unit_seg[pk * parts]; sg < end; ++sg) {
            const Segment g = segment_at(packed + seg_off[sg]);
            for_slots(g, lane, (uint32_t)lane < g.n_vis ? g.vis[lane] : 0u,
                      [&](uint32_t slot, int j) { S.j[slot] = j; }, t >> 6, kWaves);
            // (a gap after every eight groups spreads a lane's run over the banks)
            for (uint32_t at = t; at < g.n_groups; at += kBlock) {
                const uint32_t e = group_at(at, g.n_groups);
                const float4 f = g.fac[at];
                *reinterpret_cast<float4*>(S.fac + 4 * (e + (e >> 3))) = f;
                S.abc[e] = g.abc[at];
                S.dr[e] = g.dr[at];
            }
            __syncthreads();
            for (uint32_t e = t; e < g.n_groups; e += kBlock) {
                const uint32_t ray = S.dr[e] >> 10;
                if (e == 0 || (uint32_t)(S.dr[e - 1] >> 10) != ray) S.first[ray] = (uint16_t)e;
            }
            __syncthreads();
            for (uint32_t x = t; x < 4 * g.n_groups; x += kBlock) {
                const uint32_t e = x >> 2, q = x & 3u;
                const uint32_t a = S.abc[e], d = S.dr[e], ray = d >> 10;
                if (q > (a >> 30)) continue;
                const uint32_t slot = (q == 3u ? d : a >> (10 * q)) & 1023u;
                const uint32_t j = (uint32_t)S.j[slot];
                const uint32_t b = (uint32_t)__float_as_int(S.fac[4 * (e + (e >> 3)) + q]);
                const uint64_t w = S.to[ray] + 4u * (e - S.first[ray]) + q;
                if (KEYS) {
                    key[w] = j;
                    val[w] = ((uint64_t)b << 32) | (uint64_t)(row0 + ray);
                } else {
                    path[w] = make_int2((int)j, (int)b);
                }
            }
            __syncthreads();
            for (uint32_t e = t; e < g.n_groups; e += kBlock) {
                const uint32_t ray = S.dr[e] >> 10;
                if (e + 1 == g.n_groups || (uint32_t)(S.dr[e + 1] >> 10) != ray)
                    S.to[ray] += 4u * (e - S.first[ray]) + (S.abc[e] >> 30) + 1u;
            }
            __syncthreads();
        }
        __syncthreads();
    }
}

// Transposed product: y_j += (K/h^2) nu_row over every entry.  A wave per packet:
// a segment's entries add to its slots in LDS, then each slot that got something
// adds to its particle, 16 neighbouring ones of a visit at a time.  Bound by the
// atomics.  Measured on MI355X, the 65521-particle halo's 258M intersections in 12
// directions: 7.6 ms with a global atomic per entry (4.1 over paths by rows), 0.76
// here.
__global__ void __launch_bounds__(kBlock)
k_path_scatter(const uint64_t* __restrict__ unit_seg, const uint64_t* __restrict__ seg_off,
               const uint4* __restrict__ packed, int64_t n_packets, int parts, int n,
               const float* __restrict__ nu, double* __restrict__ y)
{
    __shared__ double s_y[kWaves][kSegSlots];
    __shared__ double s_nu[kWaves][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t wpd = (n + 63) / 64;
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    double* acc = s_y[wv];
    for (int64_t pk = blockIdx.x * (int64_t)kWaves + wv; pk < n_packets; pk += stride) {
        const int64_t k = pk / wpd, p0 = (pk - k * wpd) * 64;
        s_nu[wv][lane] = p0 + lane < n ? (double)nu[k * n + p0 + lane] : 0.0;
        const uint64_t end = unit_seg[(pk + 1) * parts];
        for (uint64_t sg = unit_seg[pk * parts]; sg < end; ++sg) {
            const Segment g = segment_at(packed + seg_off[sg]);
            const uint32_t w0 = (uint32_t)lane < g.n_vis ? g.vis[lane] : 0u;
            for (uint32_t i = lane; i < g.n_slots; i += 64) acc[i] = 0.0;
            wave_sync();
            for (uint32_t at = lane; at < g.n_groups; at += 64) {
                const float4 f = g.fac[at];
                const uint32_t a = g.abc[at], d = g.dr[at], used = (a >> 30) + 1u;
                const double v = s_nu[wv][d >> 10];
                if (v == 0.0) continue;
                const float fq[4] = {f.x, f.y, f.z, f.w};
                const uint32_t sl[4] = {a & 1023u, (a >> 10) & 1023u, (a >> 20) & 1023u, d & 1023u};
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    if (q < used) lds_add(acc + sl[q], (double)fq[q] * v);
            }
            wave_sync();
            for_slots(g, lane, w0, [&](uint32_t slot, int j) {
                if (acc[slot] != 0.0) unsafeAtomicAdd(y + j, acc[slot]);
            });
            wave_sync();
        }
    }
}

// sampled rows: entries per row, then (input index of the particle, factor
// K/h^2 without the near flag); one wave per row
__global__ void __launch_bounds__(kBlock)
k_path_sampled(const uint64_t* __restrict__ unit_seg, const uint64_t* __restrict__ seg_off,
             const uint4* __restrict__ packed, int parts,
               int n, const int32_t* __restrict__ perm, const int64_t* __restrict__ rows, int m,
               uint64_t* __restrict__ cnt, const uint64_t* __restrict__ dst_off,
               int32_t* __restrict__ hit_j, float* __restrict__ hit_fac)
{
    __shared__ int32_t s_j[kWaves][kSegSlots];
    __shared__ uint64_t s_w[kWaves][64];
    __shared__ uint32_t s_first[kWaves][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t wpd = (n + 63) / 64;
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    for (int64_t i = blockIdx.x * (int64_t)kWaves + wv; i < m; i += stride) {
        const int64_t k = rows[i] / n, ps = rows[i] - k * n;
        const int mine = (int)(ps & 63);
        s_w[wv][lane] = 0ull;
        const uint64_t to = dst_off ? dst_off[i] : 0ull;
        for_groups(
            unit_seg, seg_off, packed, k * wpd + ps / 64, parts, lane, s_j[wv],
            [&](const Segment& g) { find_first(g, lane, s_first[wv]); },
            [&](uint32_t e, int ray, const int* j, const uint32_t* b, uint32_t used) {
                if (ray != mine || !dst_off) return;
                const uint64_t w = to + s_w[wv][ray] + 4u * (e - s_first[wv][ray]);
                for (uint32_t q = 0; q < used; ++q) {
                    hit_j[w + q] = perm[j[q]];
                    hit_fac[w + q] = __int_as_float((int)(b[q] & ~kNearBit));
                }
            },
            [&](const Segment& g) { count_entries(g, lane, s_w[wv]); });
        wave_sync();
        if (lane == 0 && cnt) cnt[i] = s_w[wv][mine];
        wave_sync();
    }
}

// The rows of a density block's sources (list), G lanes per row, from the paths
// by rows: few rows of a packet run at a time there, and a packet's segments
// would be staged for each.  Without a list every row, where the paths are held by
// rows alone.
template <int G>
__global__ void __launch_bounds__(kBlock)
k_row_columns(const uint64_t* __restrict__ row_off, const int2* __restrict__ path,
              const float* __restrict__ mux, int64_t n_rows, double* __restrict__ N, int64_t n,
              const uint8_t* __restrict__ frozen, const int32_t* __restrict__ list, int64_t list_n,
              const uint8_t* __restrict__ want, const unsigned long long* __restrict__ stop)
{
    const int lane = threadIdx.x & (G - 1);
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / G);
    const long long* p = reinterpret_cast<const long long*>(path);
    const int64_t n_iter = list ? list_n * (n_rows / n) : n_rows;
    const bool stopped = stop && *stop != 0ull;
    for (int64_t v = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G; v < n_iter;
         v += stride) {
        const int64_t row = list ? (v / list_n) * n + list[v % list_n] : v;
        if (want && !want[row % n]) continue;     // not evaluated
        if (frozen && frozen[row % n]) continue;  // not updated in this step
        const uint64_t a = row_off[row], b = row_off[row + 1];
        double acc = 0.0;
        // Lanes stride through the row one entry at a time, so the particle
        // gathers of one instruction are consecutive intersections along the
        // ray and share cache lines.  Four streaming loads in flight per lane;
        // entries past the row end read as (particle 0, factor 0).
        for (uint64_t e = a + lane; e < b; e += 4 * G) {
            const long long v0 = __builtin_nontemporal_load(p + e);
            const long long v1 = e + G < b ? __builtin_nontemporal_load(p + e + G) : 0ll;
            const long long v2 = e + 2 * G < b ? __builtin_nontemporal_load(p + e + 2 * G) : 0ll;
            const long long v3 = e + 3 * G < b ? __builtin_nontemporal_load(p + e + 3 * G) : 0ll;
            const float m0 = mux[(int)v0], m1 = mux[(int)v1];
            const float m2 = mux[(int)v2], m3 = mux[(int)v3];
            acc += (double)(m0 * __int_as_float((int)(v0 >> 32)));
            acc += (double)(m1 * __int_as_float((int)(v1 >> 32)));
            acc += (double)(m2 * __int_as_float((int)(v2 >> 32)));
            acc += (double)(m3 * __int_as_float((int)(v3 >> 32)));
        }
        for (int off = G / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, G);
        if (lane == 0 && !stopped) N[row] = acc;
    }
}

unsigned packet_blocks(int64_t packets)
{
    return (unsigned)std::max<int64_t>(
        1, std::min<int64_t>((packets + kWaves - 1) / kWaves, kMaxBlocks));
}

}  // namespace

// Waves per packet, and 8 more where the paths are read past the cache.  Paths
// that stay in the 256 MB last-level cache from one sweep to the next are read with
// ordinary loads (the 16384-particle halo's 250 MB: 55 us a product against 68 with
// non-temporal ones), larger ones stream past it.
int path_variant(const Ctx& c)
{
    return path_ways(path_packets(c), c.path_live, c.path_segs) +
           (c.path_words * 16 > (uint64_t)256 << 20 ? 8 : 0);
}

hipError_t launch_path_columns(Ctx& c)
{
    if (path_packets(c) == 0) return hipSuccess;
    if (c.near_far) launch_columns_nf<true>(c);
    else launch_columns_nf<false>(c);
    return hipGetLastError();
}

hipError_t launch_row_columns(Ctx& c, int group)
{
    const int64_t n_rows = c.n * (int64_t)c.n_ray;
    const int64_t n_iter = c.row_list ? c.row_list_n * (int64_t)c.n_ray : n_rows;
    if (n_iter == 0) return hipSuccess;
    auto go = [&](auto kernel, int g) {
        hipLaunchKernelGGL(kernel, dim3(stride_blocks(n_iter, kBlock / g)), dim3(kBlock), 0,
                           c.stream, c.row_off, c.path, c.mux_s, n_rows, c.N_s, c.n, c.row_frozen,
                           c.row_list, c.row_list_n, c.row_list ? nullptr : c.geom.want,
                           c.batch_stop);
    };
    if (group == 64) go(k_row_columns<64>, 64);
    else if (group == 32) go(k_row_columns<32>, 32);
    else if (group == 16) go(k_row_columns<16>, 16);
    else go(k_row_columns<8>, 8);
    return hipGetLastError();
}

hipError_t ensure_row_offsets(Ctx& c)
{
    if (c.rows_valid) return hipSuccess;
    const int64_t n_rows = c.n * (int64_t)c.n_ray, pk = path_packets(c);
    hipLaunchKernelGGL(k_path_row_sizes, dim3(packet_blocks(pk)), dim3(kBlock), 0, c.stream,
                       c.unit_seg, c.seg_off, c.packed, pk, path_parts(c), (int)c.n, c.row_off);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemsetAsync(c.row_off + n_rows, 0, sizeof(uint64_t), c.stream);
    if (e == hipSuccess) e = scan_exclusive_u64(c, c.row_off, c.row_off, n_rows + 1);
    if (e == hipSuccess) c.rows_valid = true;
    return e;
}

hipError_t launch_expand_rows(Ctx& c, int2* path)
{
    return launch_expand_packets(c, path, 0, path_packets(c));
}

hipError_t launch_expand_packets(Ctx& c, int2* path, int64_t pk0, int64_t pk1)
{
    hipLaunchKernelGGL(k_path_rows<false>, dim3((unsigned)std::min<int64_t>(pk1 - pk0, kMaxBlocks)),
                       dim3(kBlock), 0, c.stream, c.unit_seg, c.seg_off, c.packed, pk0, pk1,
                       path_parts(c), (int)c.n, c.row_off, path, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_expand_keys(Ctx& c, uint32_t* key, uint64_t* val)
{
    const int64_t pk = path_packets(c);
    hipLaunchKernelGGL(k_path_rows<true>, dim3((unsigned)std::min<int64_t>(pk, kMaxBlocks)),
                       dim3(kBlock), 0, c.stream, c.unit_seg, c.seg_off, c.packed, (int64_t)0, pk,
                       path_parts(c), (int)c.n, c.row_off, nullptr, key, val);
    return hipGetLastError();
}

hipError_t launch_path_scatter(Ctx& c, const float* nu, double* y)
{
    hipError_t e = hipMemsetAsync(y, 0, sizeof(double) * c.n, c.stream);
    if (e != hipSuccess) return e;
    const int64_t pk = path_packets(c);
    hipLaunchKernelGGL(k_path_scatter, dim3(packet_blocks(pk)), dim3(kBlock), 0, c.stream,
                       c.unit_seg, c.seg_off, c.packed, pk, path_parts(c), (int)c.n, nu, y);
    return hipGetLastError();
}

hipError_t launch_path_rows(Ctx& c, const int64_t* rows, int m, uint64_t* cnt,
                            const uint64_t* dst_off, int32_t* hit_j, float* hit_fac)
{
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_path_sampled, dim3(packet_blocks(m)), dim3(kBlock), 0, c.stream,
                       c.unit_seg, c.seg_off, c.packed, path_parts(c), (int)c.n, c.perm, rows, m, cnt,
                       dst_off, hit_j, hit_fac);
    return hipGetLastError();
}

}  // namespace rrt
