// Ray traversal and HI column accumulation (Sec. 4.1.1, eq. colden).
//
// One thread follows one ray: source particle p (tree order), direction k and,
// in a periodic box, every image shift s whose tiles the segment can reach.
// Lanes of a wave take consecutive sources in tree order with the same
// direction, so neighbouring lanes walk nearly the same nodes.
//
// Node tests are FP32 slab tests against boxes padded outward by `pad`, which
// is far larger than any FP32 rounding in the test, so they never reject a
// particle the exact predicate accepts.  Leaf particles are decided by the
// FP64 predicate below, with a fixed operation order and no contraction, so
// that the set of intersected particles is reproducible bit for bit.
//
// A hit adds mu_j x_j / h_j^2 times the kernel chord integral K(b/h, z1/h,
// z2/h) in units of h: for the truncated Gaussian (eq. Gt) the closed form
// I(h,b,z1,z2) = (N h^3 sqrt(pi) / (2t)) e^{-t^2 q^2} [erf(t z2/h) - erf(t z1/h)] / h^2
// with t = A h = 2 pi^(1/6), q = b/h, z clipped to the sphere and to [0, L].
// erf comes from a table of cubic pieces staged in LDS; the Gaussian from the
// hardware 2^x with its exponent formed in FP64.
#include "internal.h"
#include "pair.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>

namespace rrt {

namespace {

// ---------------------------------------------------------------------------
// kernel tables (host, FP64)
// ---------------------------------------------------------------------------
struct KConst {
    double t, C;     // C = N h^3 sqrt(pi) / (2 t)
};

KConst kconst()
{
    const double pi = 3.14159265358979323846;
    double t = 2.0 * std::pow(pi, 1.0 / 6.0);
    double nh3 = (8.0 / pi) / (std::erf(t) - 2.0 * t * std::exp(-t * t) / std::sqrt(pi));
    return {t, nh3 * std::sqrt(pi) / (2.0 * t)};
}

template <typename F>
void fit_cubics(float4* out, F f)
{
    // cubic through u = 0, 1/3, 2/3, 1 on each piece, in monomial form in u
    for (int i = 0; i < kTabIntervals; ++i) {
        double a = (double)i / kTabIntervals, b = (double)(i + 1) / kTabIntervals;
        double y0 = f(a), y1 = f(a + (b - a) / 3.0), y2 = f(a + 2.0 * (b - a) / 3.0), y3 = f(b);
        // Newton divided differences on nodes 0, 1/3, 2/3, 1
        double d1 = (y1 - y0) * 3.0, d2 = (y2 - y1) * 3.0, d3 = (y3 - y2) * 3.0;
        double e1 = (d2 - d1) * 1.5, e2 = (d3 - d2) * 1.5;
        double g1 = (e2 - e1);
        // p(u) = y0 + d1 u + e1 u (u - 1/3) + g1 u (u - 1/3)(u - 2/3)
        double c0 = y0;
        double c1 = d1 - e1 / 3.0 + g1 * (2.0 / 9.0);
        double c2 = e1 - g1;
        double c3 = g1;
        out[i] = make_float4((float)c0, (float)c1, (float)c2, (float)c3);
    }
}

// column: accumulate N; count: hits per ray; record: hit lists for inspection;
// scatter: y_j += (K/h^2) nu_ray for every hit (transposed column product)
// log: the hits of the path recording, as a log of the walk's leaf visits that
// paths.hip turns into the recorded paths (wave-cooperative walk only)
// tally: the sizes the log and the recorded paths would have, nothing stored
// stats: a count pass that also tallies the walk's work (diagnostics)
enum { kModeColumn = 0, kModeCount = 1, kModeRecord = 2, kModeTally = 3, kModeScatter = 4,
       kModeLog = 5, kModeStats = 6 };

__host__ __device__ constexpr bool mode_logs(int mode)
{
    return mode == kModeLog || mode == kModeTally;
}

struct RayOut {
    double* N;              // [n_ray][n] columns (column / record modes)
    uint64_t* row_cnt;      // [n_ray * n] hits per ray (count mode)
    const uint64_t* row_off;// [n_ray * n] write offsets (record mode)
    const float* nu;        // scatter mode: adjoint of each ray's column
    double* y;              // scatter mode: accumulated per tree index
    int32_t* hit_j;         // record mode: input index of each hit
    int32_t* hit_img;       // record mode: image code of each hit
    uint64_t hit_cap;       // record mode: capacity of hit_j / hit_img
    const int32_t* perm;
    unsigned long long* hits_total;
    // near/far split (column mode): a hit is near when the
    // particle's kernel contains the source, |d|^2 < h^2 (FP64, x, y, z order)
    int near_far;
    double* Nn;             // column mode: [n_ray][n] near total-hydrogen columns
    const double* mu;       // hydrogen content per tree index (near columns use x = 1)
    // log and tally modes (the layout is described in internal.h)
    uint64_t* log;                   // the pool of log blocks
    uint64_t log_blocks;             // blocks it holds
    uint32_t log_take;               // blocks a wave takes at once
    unsigned long long* log_ctr;     // [0] next block, [1] set when the pool ran short
    uint2* unit_log;                 // per unit: first block, segments
    uint64_t* unit_size;             // per unit: recorded words | log blocks << 32
    int32_t parts;                   // units each packet's walk is split into
    int64_t unit0, unit_end;         // a part of the units (without the queues), all if 0
    // sampled sources (count and record modes): only the rays of the sorted
    // tree positions src_list[0..src_n) run, and their outputs go to row
    // i * n_ray + k for the source at src_list[i] (null = every ray, row = ray)
    const int32_t* src_list;
    int32_t src_n;
    float* hit_fac;         // record mode: K/h^2 of each hit (nullable)
    // stats mode: [rays, wave node visits, lane node visits, wave leaf visits,
    // pair tests, hits], accumulated
    unsigned long long* stats;
    // wave-cooperative walk, persistent form: a resident grid whose waves take
    // units (64 sources of one direction, over every halo) from kQueues
    // counters, kQueueStride apart, each over its share of the sources; null =
    // one wave per unit
    unsigned long long* queue;
    const unsigned long long* stop;   // column mode: holds something: nothing is written
    // the queues' share of the packets: directions and, of each, packets of 64 sources
    int32_t dir0, n_dir, pk0, n_pk;
};

// Place of tree position ps among the sorted sampled sources, or -1.
__device__ __forceinline__ int sampled_slot(const int32_t* __restrict__ list, int m, int ps)
{
    int lo = 0, hi = m;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (list[mid] < ps) lo = mid + 1;
        else hi = mid;
    }
    return (lo < m && list[lo] == ps) ? lo : -1;
}

#pragma clang fp contract(off)
template <int MODE>
__global__ void __launch_bounds__(256)
k_trace(const Node* __restrict__ nodes, const float4* __restrict__ p4,
        const float* __restrict__ mux, const double* __restrict__ dirs,
        const KernelTables* __restrict__ tabs, TraceGeom g, RayOut out)
{
    __shared__ float4 t_erf[kTabIntervals];
    if (MODE == kModeColumn && out.stop && *out.stop != 0ull) return;    // the whole grid
    constexpr bool kTerms = MODE != kModeCount;
    if (kTerms) {
        for (int i = threadIdx.x; i < kTabIntervals; i += blockDim.x) t_erf[i] = tabs->erf_t[i];
        __syncthreads();
    }
    const double gc = tabs->gauss_c, ga = tabs->gauss_a;

    const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t n_rays = (int64_t)g.n * g.n_ray;
    uint32_t cnt = 0;
    int64_t slot = gid;
    bool sampled = true;
    if (gid < n_rays && out.src_list) {
        const int k = (int)(gid / g.n);
        const int i = sampled_slot(out.src_list, out.src_n, (int)(gid - (int64_t)k * g.n));
        sampled = i >= 0;
        slot = (int64_t)i * g.n_ray + k;
    }
    if (gid < n_rays && sampled) {
        const int k = (int)(gid / g.n);
        const int ps = (int)(gid - (int64_t)k * g.n);
        const float4 P = p4[ps];
        const double rp[3] = {(double)P.x, (double)P.y, (double)P.z};
        const double u[3] = {dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]};
        const double L = g.L, B = g.box;
        const float Lf = (float)L;

        int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
        if (B > 0.0) {
            for (int a = 0; a < 3; ++a) {
                double e = rp[a] + L * u[a];
                double smin = rp[a] < e ? rp[a] : e, smax = rp[a] < e ? e : rp[a];
                lo[a] = (int)ceil((smin - g.hmax - g.phi[a]) / B - 1e-6);
                hi[a] = (int)floor((smax + g.hmax - g.plo[a]) / B + 1e-6);
            }
        }
        float inv[3];
        for (int a = 0; a < 3; ++a) {
            float ua = (float)u[a];
            if (fabsf(ua) < 1e-20f) ua = 1e-20f;
            inv[a] = 1.0f / ua;
        }
        double acc = 0.0, accn = 0.0;
        uint64_t w = MODE == kModeRecord ? out.row_off[slot] : 0;
        const double nur = (MODE == kModeScatter) ? (double)out.nu[gid] : 0.0;

        // the subtree this ray's halo owns (the whole tree for one problem)
        int root = 0, end = g.n_nodes;
        bool live = true;
        if (g.seg_root) {
            const int h = g.seg_of[ps];
            root = g.seg_root[h];
            end = g.seg_end[h];
            live = !g.seg_active || g.seg_active[h] != 0;
        }
        if (MODE == kModeColumn && g.want && !g.want[ps]) live = false;
        if (!live) lo[0] = 1, hi[0] = 0;            // no image loop at all
        for (int sx = lo[0]; sx <= hi[0]; ++sx)
        for (int sy = lo[1]; sy <= hi[1]; ++sy)
        for (int sz = lo[2]; sz <= hi[2]; ++sz) {
            double sh[3] = {(double)sx * B, (double)sy * B, (double)sz * B};
            if (!(B > 0.0)) sh[0] = sh[1] = sh[2] = 0.0;
            // the image of particle j sits at r_j + sB, i.e. the ray meets the
            // stored particles as if it started from r_p - sB
            float oai[3], obi[3];
            for (int a = 0; a < 3; ++a) {
                double o = rp[a] - sh[a];
                oai[a] = (float)(o + (double)g.pad) * inv[a];
                obi[a] = (float)(o - (double)g.pad) * inv[a];
            }
            int node = root;
            while (node < end) {
                const Node nd = nodes[node];
                float tx0 = fmaf(nd.a.x, inv[0], -oai[0]), tx1 = fmaf(nd.b.x, inv[0], -obi[0]);
                float ty0 = fmaf(nd.a.y, inv[1], -oai[1]), ty1 = fmaf(nd.b.y, inv[1], -obi[1]);
                float tz0 = fmaf(nd.a.z, inv[2], -oai[2]), tz1 = fmaf(nd.b.z, inv[2], -obi[2]);
                float tmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)),
                                   fmaxf(fminf(tz0, tz1), 0.0f));
                float tmax = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)),
                                   fminf(fmaxf(tz0, tz1), Lf));
                const int skip = __float_as_int(nd.a.w);
                const int leafw = __float_as_int(nd.b.w);
                // skip links always point past the node; max() keeps every walk finite
                if (!(tmin <= tmax)) { node = max(skip, node + 1); continue; }
                if (leafw < 0) { node = node + 1; continue; }
                const int f = leafw >> kLeafShift;
                const int c = (f + (leafw & (kLeafMax - 1)) + 1 <= g.n) ? (leafw & (kLeafMax - 1)) + 1 : 0;
                // the leaf's particles (contiguous in tree order) are loaded
                // eight at a time; p4 holds kLeafMax spare entries past n
                for (int q0 = 0; q0 < c; q0 += 8) {
                float4 Qs[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) Qs[q] = p4[f + q0 + q];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (q0 + q >= c) break;
                    const int j = f + q0 + q;
                    const float4 Q = Qs[q];
                    double d0 = ((double)Q.x - rp[0]) + sh[0];
                    double d1 = ((double)Q.y - rp[1]) + sh[1];
                    double d2 = ((double)Q.z - rp[2]) + sh[2];
                    double sp = dot_u(d0, d1, d2, u);
                    double tt = sp < 0.0 ? 0.0 : (sp > L ? L : sp);
                    double c0 = fma(-tt, u[0], d0);
                    double c1 = fma(-tt, u[1], d1);
                    double c2 = fma(-tt, u[2], d2);
                    double D2 = norm2(c0, c1, c2);
                    double hj = (double)Q.w;
                    double h2 = hj * hj;
                    if (!(D2 < h2)) continue;
                    ++cnt;
                    if (MODE == kModeCount || MODE == kModeStats) continue;
                    double px = fma(-sp, u[0], d0), py = fma(-sp, u[1], d1),
                           pz = fma(-sp, u[2], d2);
                    double b2 = norm2(px, py, pz);
                    const float gk = chord_factor(sp, b2, h2, L, Q.w, t_erf, gc, ga);
                    if (MODE == kModeRecord) {
                        if (w < out.hit_cap) {
                            out.hit_j[w] = out.perm[j];
                            out.hit_img[w] = (sx + 8) | ((sy + 8) << 4) | ((sz + 8) << 8);
                            if (out.hit_fac) out.hit_fac[w] = gk;
                        }
                        ++w;
                    }
                    bool near = false;
                    if (out.near_far) near = (d0 * d0 + d1 * d1 + d2 * d2) < h2;
                    if (MODE == kModeScatter) {
                        if (nur != 0.0) unsafeAtomicAdd(out.y + j, (double)gk * nur);
                    } else if (near) {
                        accn += (double)((float)out.mu[j] * gk);
                    } else {
                        acc += (double)(mux[j] * gk);
                    }
                }
                }   // groups of eight particles
                node = max(skip, node + 1);
            }
        }
        if ((MODE == kModeColumn || MODE == kModeRecord) && live && out.N)
            out.N[(int64_t)k * g.n + ps] = acc;
        if (MODE == kModeColumn && live && out.near_far) out.Nn[(int64_t)k * g.n + ps] = accn;
        if (MODE == kModeCount || MODE == kModeStats) out.row_cnt[slot] = cnt;
    }
    // one atomic per wave for the total intersection count
    uint64_t c64 = cnt;
    for (int off = 32; off > 0; off >>= 1) c64 += __shfl_xor(c64, off, 64);
    if ((threadIdx.x & 63) == 0 && c64) atomicAdd(out.hits_total, (unsigned long long)c64);
}
// Wave-cooperative variant: the 64 rays of a wave (same direction, sources
// adjacent in tree order) walk ONE node sequence, the depth-first union of
// their individual walks.  Node and leaf-particle loads are wave-uniform
// (scalar loads); each lane tests its own ray, and a ballot decides whether the
// wave descends or skips.  A lane only tests the particles of leaves its own
// ray's box test accepted, and sees them in depth-first order, so every lane's
// hits, counts and recorded paths equal those of its own walk.
//
// The walk is bound by vector instruction issue (the chip's VALU issue rate is
// reached with the scalar node loads hidden behind it), so the loops are
// written for instruction count:
//  * the rays share one direction, so on each axis the face a ray enters
//    through (low or high) is the same for all lanes: it is chosen once with
//    scalar selects, and the slab test needs no per-lane min/max of the pair;
//  * the node index and the walk's bounds are scalar, so the loop is too;
//  * a leaf's (ray, particle) pairs are indexed with an FP32 reciprocal (exact
//    for the at most 64 x 16 pairs); the rays' origins and the leaf's
//    particles are read, already in FP64, from LDS (each particle is loaded
//    and widened once per leaf, not once per pair);
//  * what the log modes need only when a segment opens or closes, a block ends
//    or a unit does lives in LDS: scalar registers are short, and a spilled one
//    costs two vector instructions each time;
//  * the shift of a periodic image is only formed where its pairs need it;
//  * the image shift's three adds only run for a shifted image: for the
//    unshifted one they add zero, which changes no bit of the predicate;
//  * the near test only exists in the near/far variant (NF).
// LDS per wave: origins 3 x 64 FP64, hit masks 64 x 4 B, factors 64 x 16 x
// 4 B (modes that evaluate factors in the walk, which also stage the erf
// table once per block) or the log's state, the leaf's particles 16 x 4 FP64.
// Sized per launch
// (dynamic LDS), so a 128-thread block holds two waves' buffers.
// Measured on MI355X (recording walk): the 885k-particle field 44.3 ms with one
// queue, no leaf balls and the faces swapped one axis at a time, 30.1 ms now; the
// 262144-particle halo 18.3 and 11.8 ms.  Of that halo's 14.3 ms after the log
// replaced the written entries, the balls took 1.7 (15 to 26 percent fewer
// pairs) and the queues with the scalar work 0.8.
// Six waves per SIMD (measured: the count and record passes run 4.5% faster on
// the 2.1M-particle field than at the four that ~100 VGPRs would allow, with
// a few registers spilled to scratch).
constexpr int kWaveOrgBytes = 3 * 64 * (int)sizeof(double);
constexpr int kWaveMaskBytes = 64 * (int)sizeof(unsigned int);
constexpr int kWaveGkBytes = 64 * kLeafMax * (int)sizeof(float);
constexpr int kWaveLeafBytes = kLeafMax * 4 * (int)sizeof(double);

// modes whose walk evaluates the chord factor of its hits (the path recording
// leaves it to the pass over its log)
__host__ __device__ constexpr bool mode_factors(int mode)
{
    return mode == kModeColumn || mode == kModeRecord || mode == kModeScatter;
}

// A wave's log state (wave-uniform values, read back by every lane).
struct LogState {
    uint64_t unit, hits;
    uint32_t hdr_blk, hdr_pos;       // the open segment's header
    uint32_t n_seg, size, blocks;    // of the unit: segments, recorded words, log blocks
    uint32_t first_blk;
    uint32_t c_next, c_end;          // blocks taken from the pool, not yet used
};
constexpr int kWaveLogBytes = 64;
static_assert(sizeof(LogState) <= kWaveLogBytes, "a wave's log state");

// per wave: the factor buffer or the log state of a mode
__host__ __device__ constexpr int wave_pair_bytes(int mode)
{
    return mode_factors(mode) ? kWaveGkBytes : mode_logs(mode) ? kWaveLogBytes : 0;
}

// dynamic LDS bytes of one k_trace_wave block
inline size_t wave_lds_bytes(int mode, int block)
{
    const size_t waves = (size_t)(block / 64);
    size_t b = waves * (kWaveOrgBytes + kWaveMaskBytes + wave_pair_bytes(mode) + kWaveLeafBytes);
    if (mode_factors(mode)) b += (size_t)kTabIntervals * sizeof(float4);
    return b;
}

// min(x, hi) as one instruction (fmin would first canonicalise hi, which the
// compiler redoes in every iteration)
__device__ __forceinline__ double clamp_hi(double x, double hi)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(hi));
    return r;
}

template <int MODE, bool NF, bool PQ>
__global__ void __launch_bounds__(256, 6)
k_trace_wave(const Node* __restrict__ nodes, const float4* __restrict__ leaf_ball,
             const float4* __restrict__ p4,
             const float* __restrict__ mux, const double* __restrict__ dirs,
             const KernelTables* __restrict__ tabs, TraceGeom g, RayOut out)
{
    constexpr bool kTally = mode_logs(MODE);
    constexpr bool kLog = MODE == kModeLog;
    constexpr bool kCountOnly = MODE == kModeCount || MODE == kModeStats;
    constexpr bool kTerms = mode_factors(MODE);
    extern __shared__ __align__(16) unsigned char s_dyn[];
    // the whole grid (the queues of the persistent form are spent then)
    if (MODE == kModeColumn && !PQ && out.stop && *out.stop != 0ull) return;
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int n_wv = blockDim.x >> 6;
    float4* t_erf = reinterpret_cast<float4*>(s_dyn);
    unsigned char* s_wave = s_dyn + (kTerms ? kTabIntervals * sizeof(float4) : 0);
    // per wave: the hit rays' origins (FP64, by rank among the leaf's hit rays),
    // per hit ray of the current leaf bit q set when the ray hits the leaf's
    // particle q (bit 16 + q when that hit is near), and the pairs' factors
    double* s_o = reinterpret_cast<double*>(s_wave) + wv * 3 * 64;
    unsigned int* s_mask =
        reinterpret_cast<unsigned int*>(s_wave + n_wv * kWaveOrgBytes) + wv * 64;
    float* s_gk = reinterpret_cast<float*>(s_wave + n_wv * (kWaveOrgBytes + kWaveMaskBytes)) +
                  wv * 64 * kLeafMax;
    LogState* ls = reinterpret_cast<LogState*>(
        s_wave + n_wv * (kWaveOrgBytes + kWaveMaskBytes) + wv * kWaveLogBytes);
    // the current leaf's particles: x, y, z, h in FP64
    double* s_pd = reinterpret_cast<double*>(
                       s_wave + n_wv * (kWaveOrgBytes + kWaveMaskBytes + wave_pair_bytes(MODE))) +
                   wv * kLeafMax * 4;
    if (kTerms) {
        for (int i = threadIdx.x; i < kTabIntervals; i += blockDim.x) t_erf[i] = tabs->erf_t[i];
        __syncthreads();
    }
    const double gc = tabs->gauss_c, ga = tabs->gauss_a;

    const uint64_t lt_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int64_t waves_per_dir = (g.n + 63) / 64;
    int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    // the wave's intersections over its packets, added to the total once (one
    // atomic per wave rather than per packet on the single counter)
    uint64_t hits_wave = 0;
    if (kTally && lane == 0) {
        ls->c_next = ls->c_end = 0u;             // no block taken from the pool yet
        ls->hits = 0ull;
    }
    // the recording splits a packet's walk into `parts`, each a unit of its own
    // (few packets would leave the device idle otherwise)
    const int parts = kTally ? out.parts : 1;
    // Workgroups go to the device's XCDs in turn, and each XCD has its own L2: a
    // block starts with the queue of its XCD, whose sources (and so the part of
    // the tree around them) are the same for every direction.  Every wave
    // passes over all queues before it ends.
    int que = blockIdx.x & (kQueues - 1), spent = 0;
    for (;;) {                                               // units of this wave
    int64_t unit = wave;
    int part = 0;
    if (PQ) {
        const uint32_t per = (uint32_t)(out.n_dir * parts);
        uint32_t v = 0, b0 = 0;
        for (; spent < kQueues; ++spent, que = (que + 1) & (kQueues - 1)) {
            const uint32_t n_pk = (uint32_t)out.n_pk, at = n_pk * (uint32_t)que / kQueues;
            const uint32_t len = n_pk * (uint32_t)(que + 1) / kQueues - at;
            b0 = (uint32_t)out.pk0 + at;
            unsigned long long t = 0;
            if (lane == 0) t = atomicAdd(out.queue + (size_t)que * kQueueStride, 1ull);
            t = __shfl(t, 0, 64);
            v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t < (1ull << 31) ? t : 1ull << 31));
            if ((uint64_t)v < (uint64_t)len * per) break;
        }
        const uint32_t b = v / per, kp = v - b * per;
        const uint32_t kk = kp / (uint32_t)parts;
        part = __builtin_amdgcn_readfirstlane((int)(kp - kk * (uint32_t)parts));
        // (every queue spent: past the last direction, which ends the wave)
        wave = spent < kQueues ? (int64_t)(kk + (uint32_t)out.dir0) * waves_per_dir + b0 + b
                               : (int64_t)g.n_ray * waves_per_dir;
        unit = wave * parts + part;
    } else if (kTally) {
        unit += out.unit0;
        if (out.unit_end && unit >= out.unit_end)      // past the last: ends the wave
            unit = (int64_t)g.n_ray * waves_per_dir * parts;
        wave = unit / parts;
        part = __builtin_amdgcn_readfirstlane((int)(unit - wave * parts));
    }
    if (kTally) {
        if (lane == 0) {
            ls->unit = (uint64_t)unit;
            ls->n_seg = ls->size = ls->blocks = 0u;
            ls->first_blk = kNoBlock;
        }
        wave_sync();
    }
    // the wave's direction and image range are uniform: scalar registers
    const int k = __builtin_amdgcn_readfirstlane((int)(wave / waves_per_dir));
    if (k >= g.n_ray) {                                      // whole wave
        if (kTally) hits_wave = ls->hits;
        if (lane == 0 && hits_wave) atomicAdd(out.hits_total, (unsigned long long)hits_wave);
        return;
    }
    const int ps = (int)((wave - (int64_t)k * waves_per_dir) * 64 + lane);
    // the ray's output row: the ray itself, or its sampled source's place
    int64_t slot = (int64_t)k * g.n + ps;
    bool sampled = true;
    if (out.src_list) {
        const int i = ps < g.n ? sampled_slot(out.src_list, out.src_n, ps) : -1;
        sampled = i >= 0;
        slot = (int64_t)i * g.n_ray + k;
    }
    const bool active = ps < g.n && sampled;
    const float4 P = p4[ps < g.n ? ps : g.n - 1];
    // the ray's origin: FP32 inputs, widened exactly where FP64 needs them
    const float rpf[3] = {P.x, P.y, P.z};
    const double u[3] = {dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]};
    const double B = g.box;
    // canonical once (the clamps below need canonical operands)
    const double L = __builtin_canonicalize(g.L);
    const float Lf = (float)L;
    const int64_t gid = (int64_t)k * g.n + ps;

    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    int ulo[3] = {0, 0, 0}, uhi[3] = {0, 0, 0};
    if (B > 0.0) {
        for (int a = 0; a < 3; ++a) {
            const double r = (double)rpf[a];
            double e = r + L * u[a];
            double smin = r < e ? r : e, smax = r < e ? e : r;
            lo[a] = (int)ceil((smin - g.hmax - g.phi[a]) / B - 1e-6);
            hi[a] = (int)floor((smax + g.hmax - g.plo[a]) / B + 1e-6);
            int l = active ? lo[a] : INT_MAX, h = active ? hi[a] : INT_MIN;
            for (int off = 32; off > 0; off >>= 1) {
                l = min(l, __shfl_xor(l, off, 64));
                h = max(h, __shfl_xor(h, off, 64));
            }
            ulo[a] = __builtin_amdgcn_readfirstlane(l);
            uhi[a] = __builtin_amdgcn_readfirstlane(h);
        }
    }
    // slab parameters in units of the segment length, so the segment is
    // [0, 1] and both clamps are inline constants
    float inv[3], uf[3];
    uint32_t flip[3];
    for (int a = 0; a < 3; ++a) {
        float ua = (float)u[a];
        uf[a] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ua)));
        if (fabsf(ua) < 1e-20f) ua = 1e-20f;
        inv[a] = 1.0f / (ua * Lf);
        // all ones when the ray enters boxes through the high face on axis a
        flip[a] = (uint32_t)__builtin_amdgcn_readfirstlane(inv[a] < 0.0f ? -1 : 0);
    }
    // masks that swap the faces of two axes at a time (the fourth words, skip and
    // leaf, stay); kept opaque, or the compiler turns the swaps back into
    // selects, twice as many scalar instructions
    uint64_t flip_xy = ((uint64_t)flip[1] << 32) | flip[0], flip_zw = flip[2];
    asm("" : "+s"(flip_xy), "+s"(flip_zw));
    double acc = 0.0, accn = 0.0;
    uint32_t cnt = 0;
    uint64_t w = (MODE == kModeRecord && active) ? out.row_off[slot] : 0;
    // stats mode: wave node visits, lane node visits, wave leaf visits, pair tests
    uint64_t st_nodes = 0, st_lanes = 0, st_leaves = 0, st_pairs = 0;
    // log and tally modes.  Per unit (uniform): the block and word the log has
    // reached, the open segment's header, its slots, visits, hits and words;
    // per ray: its entries in the segment.
    // (blk is kNoBlock before the first block, and once the pool ran short:
    // then only the sizes go on)
    uint32_t blk = kNoBlock, pos = kLogData;
    uint32_t g_slots = 0, g_vis = 0, g_hits = 0, g_words = 0;
    uint32_t g_cnt = 0;
    // make sure the next `need` words are in one block
    auto reserve = [&](uint32_t need) {
        if (pos + need <= kLogData) return;
        uint32_t nb = kNoBlock;
        // (a unit that has dropped out of the log has blocks counted but no block)
        const bool first = ls->blocks == 0u;
        if (kLog && (first || blk != kNoBlock)) {
            uint32_t at = ls->c_next, end = ls->c_end;
            if (at == end) {
                unsigned long long b = 0;
                const uint32_t n_take = out.log_take;
                if (lane == 0) b = atomicAdd(out.log_ctr, (unsigned long long)n_take);
                b = __shfl(b, 0, 64);
                if (b >= out.log_blocks) {
                    at = end = kNoBlock;
                    if (lane == 0) out.log_ctr[1] = 1ull;
                } else {
                    at = (uint32_t)b;
                    const uint64_t room = out.log_blocks - b;
                    end = at + (uint32_t)(room < n_take ? room : n_take);
                }
            }
            nb = __builtin_amdgcn_readfirstlane(at);
            if (lane == 0) {
                if (nb != kNoBlock) {
                    ls->c_next = at + 1u;
                    ls->c_end = end;
                }
                if (first) ls->first_blk = nb;
                else if (nb != kNoBlock)
                    out.log[(uint64_t)blk * kLogBlock + kLogData] =
                        (uint64_t)nb | ((uint64_t)pos << 32);
            }
        }
        if (lane == 0) ls->blocks += 1u;
        wave_sync();
        blk = nb;
        pos = 0;
    };
    auto open_segment = [&]() {
        reserve(kLogHeader);
        if (kLog && blk != kNoBlock && lane == 0) {
            // the header before points at this one
            if (ls->n_seg)
                out.log[(uint64_t)ls->hdr_blk * kLogBlock + ls->hdr_pos + 2] =
                    (uint64_t)blk * kLogBlock + pos;
            ls->hdr_blk = blk;
            ls->hdr_pos = pos;
        }
        wave_sync();
        pos += kLogHeader;
    };
    auto close_segment = [&]() {
        uint32_t groups = (g_cnt + 3u) >> 2, hits = g_cnt;
        for (int off = 32; off > 0; off >>= 1) {
            groups += __shfl_xor(groups, off, 64);
            hits += __shfl_xor(hits, off, 64);
        }
        if (kLog && blk != kNoBlock) {
            uint64_t* h = out.log + ((uint64_t)ls->hdr_blk * kLogBlock + ls->hdr_pos);
            if (lane == 0) {
                h[0] = (uint64_t)g_words | ((uint64_t)g_vis << 32) | ((uint64_t)g_slots << 48);
                h[1] = groups;
            }
            reinterpret_cast<uint16_t*>(h + 3)[lane] = (uint16_t)g_cnt;
        }
        if (lane == 0) {
            ls->n_seg += 1u;
            ls->size += segment_words(g_vis, groups);
            ls->hits += hits;
        }
        wave_sync();
        g_slots = g_vis = g_hits = g_words = 0;
        g_cnt = 0;
    };
    const double nur = (MODE == kModeScatter && active) ? (double)out.nu[gid] : 0.0;

    // lanes of one wave can belong to two halos (at a halo boundary in tree
    // order): walk each halo's subtree in turn with that halo's lanes
    int root = 0, end = g.n_nodes;
    bool live = active;
    if (g.seg_root && active) {
        const int h = g.seg_of[ps];
        root = g.seg_root[h];
        end = g.seg_end[h];
        live = !g.seg_active || g.seg_active[h] != 0;
    }
    if (MODE == kModeColumn && g.want && active && !g.want[ps]) live = false;
    if (kTally && parts > 1 && B > 0.0 && lane * parts / 64 != part) live = false;
    uint64_t pending = wave_ballot(live);
    while (pending) {
    const int leader = __ffsll((unsigned long long)pending) - 1;
    const int sroot = __builtin_amdgcn_readfirstlane(__shfl(root, leader, 64));
    const int send = __builtin_amdgcn_readfirstlane(__shfl(end, leader, 64));
    const bool in_seg = live && root == sroot;
    pending &= ~wave_ballot(in_seg);
    // This unit's part of the packet's walk: a range of the subtree's nodes (a
    // depth-first walk may start at any node: it visits the leaves from there
    // on, whose ancestors' tests would only have spared it some of its own), or
    // in a periodic box, where every ray's images follow one another, some of
    // the rays.  Either way a ray's hits stay in the order of one walk.
    int n_from = sroot, n_to = send;
    if (kTally && parts > 1 && !(B > 0.0)) {
        n_from = sroot + (int)((int64_t)(send - sroot) * part / parts);
        n_to = sroot + (int)((int64_t)(send - sroot) * (part + 1) / parts);
    }
    for (int sx = ulo[0]; sx <= uhi[0]; ++sx)
    for (int sy = ulo[1]; sy <= uhi[1]; ++sy)
    for (int sz = ulo[2]; sz <= uhi[2]; ++sz) {
        const bool mine = in_seg && sx >= lo[0] && sx <= hi[0] && sy >= lo[1] && sy <= hi[1] &&
                          sz >= lo[2] && sz <= hi[2];
        if (wave_ballot(mine) == 0) continue;
        // the segment's end in the slab test; below the start for lanes that
        // do not walk this image, so their test always fails
        const float t_end = mine ? 1.0f : -1.0f;
        // the log's words of a visit before its rays': one, two with a shifted image,
        // four with one that does not fit a word (wave-uniform)
        const uint32_t hw = (sx | sy | sz) == 0 ? 1u
                            : max(max(abs(sx), abs(sy)), abs(sz)) <= kMaxImage ? 2u : 4u;
        const bool shifted = hw > 1u;
        // slab offsets of the entry and exit faces: the low face is padded
        // by -pad, the high face by +pad
        float oin[3], oout[3], of[3];
        for (int a = 0; a < 3; ++a) {
            const int sa = a == 0 ? sx : a == 1 ? sy : sz;
            const double o = (double)rpf[a] - (B > 0.0 ? (double)sa * B : 0.0);
            of[a] = (float)o;
            const float oa = (float)(o + (double)g.pad) * inv[a];
            const float ob = (float)(o - (double)g.pad) * inv[a];
            oin[a] = flip[a] ? ob : oa;
            oout[a] = flip[a] ? oa : ob;
        }
        // the wave walks one node sequence: the index is scalar, nodes are
        // read with scalar loads and the slab test takes its bounds from
        // scalar registers
        int node = n_from;
        for (;;) {
            // the next leaf that any of the wave's rays reach
            uint64_t hm = 0;
            int leafw = -1;
            while (node < n_to) {
                const uint64_t* np = reinterpret_cast<const uint64_t*>(nodes + (uint32_t)node);
                const uint64_t a_xy = np[0], a_zw = np[1], b_xy = np[2], b_zw = np[3];
                // entry and exit faces: a ^ ((a ^ b) & flip) swaps the pair in
                // scalar registers
                const uint64_t d_xy = (a_xy ^ b_xy) & flip_xy, d_zw = (a_zw ^ b_zw) & flip_zw;
                const uint64_t e_xy = a_xy ^ d_xy, f_xy = b_xy ^ d_xy;
                const uint64_t e_zw = a_zw ^ d_zw, f_zw = b_zw ^ d_zw;
                const float ex = __uint_as_float((uint32_t)e_xy);
                const float ey = __uint_as_float((uint32_t)(e_xy >> 32));
                const float ez = __uint_as_float((uint32_t)e_zw);
                const float fx = __uint_as_float((uint32_t)f_xy);
                const float fy = __uint_as_float((uint32_t)(f_xy >> 32));
                const float fz = __uint_as_float((uint32_t)f_zw);
                const float tmin = fmaxf(fmaxf(fmaxf(fmaf(ex, inv[0], -oin[0]),
                                                     fmaf(ey, inv[1], -oin[1])),
                                               fmaf(ez, inv[2], -oin[2])), 0.0f);
                const float tmax = fminf(fminf(fminf(fmaf(fx, inv[0], -oout[0]),
                                                     fmaf(fy, inv[1], -oout[1])),
                                               fmaf(fz, inv[2], -oout[2])), t_end);
                hm = wave_ballot(tmin <= tmax);
                if (MODE == kModeStats) {
                    st_nodes += 1;
                    st_lanes += __popcll(hm);
                }
                // (moved out of the pair, which the compiler would compare in vector code)
                const int skip = (int)(uint32_t)(e_zw >> 32);
                asm("s_mov_b32 %0, %1" : "=s"(leafw) : "s"((uint32_t)(f_zw >> 32)));
                // skip links always point past the node; max() keeps every walk finite
                if (hm == 0) {
                    node = max(skip, node + 1);
                    leafw = -1;
                    continue;
                }
                if (leafw < 0) {
                    ++node;
                    continue;
                }
                node = max(skip, node + 1);
                break;
            }
            if (leafw < 0) break;
            const int f = leafw >> kLeafShift;
            // A kernel sphere is round, its box is not: of the rays that reach a
            // leaf's box, those that pass by the ball around its spheres have
            // no hit there.  (FP32 with the same pad as the boxes, which is more
            // than ten times this test's rounding.)
            {
                const float4 ball = leaf_ball[f];
                const float b0 = ball.x - of[0], b1 = ball.y - of[1], b2 = ball.z - of[2];
                const float bp = fmaf(b2, uf[2], fmaf(b1, uf[1], b0 * uf[0]));
                const float bt = __builtin_amdgcn_fmed3f(bp, 0.0f, Lf);
                const float e0 = fmaf(-bt, uf[0], b0), e1 = fmaf(-bt, uf[1], b1),
                            e2 = fmaf(-bt, uf[2], b2);
                hm &= wave_ballot(fmaf(e2, e2, fmaf(e1, e1, e0 * e0)) <= ball.w);
                if (hm == 0) continue;
            }
            const int c = (f + (leafw & (kLeafMax - 1)) + 1 <= g.n) ? (leafw & (kLeafMax - 1)) + 1 : 0;
            // Leaf work compacted over the wave: the (hit ray, leaf particle)
            // pairs are spread over all 64 lanes, so a leaf that few of the
            // wave's rays reach costs few wave instructions.  Pair t is hit
            // ray t mod k_hit (by rank) and leaf particle t / k_hit; its lane
            // evaluates the canonical predicate and the chord factor and sets
            // the pair's bit in its ray's hit mask; each ray then takes its
            // hits in particle order, exactly as if it had looped over them.
            const bool hit = (hm >> lane) & 1ull;
            const int k_hit = __popcll(hm);
            const int rank = __popcll(hm & lt_mask);
            if (lane < c) {
                const float4 Q = p4[f + lane];
                s_pd[4 * lane] = (double)Q.x;
                s_pd[4 * lane + 1] = (double)Q.y;
                s_pd[4 * lane + 2] = (double)Q.z;
                s_pd[4 * lane + 3] = (double)Q.w;
            }
            if (hit) {
                s_o[rank] = (double)rpf[0];
                s_o[64 + rank] = (double)rpf[1];
                s_o[128 + rank] = (double)rpf[2];
                s_mask[rank] = 0u;
            }
            wave_sync();
            const int pairs = k_hit * c;
            if (MODE == kModeStats) {
                st_leaves += 1;
                st_pairs += (uint64_t)pairs;
            }
            // t / k_hit as (t + 1/2) / k_hit rounded down in FP32: the
            // quotient is at least 1/(2 k_hit) >= 1/128 away from an integer,
            // far beyond the error of the reciprocal and product (< 2^-12)
            const float rk = __builtin_amdgcn_rcpf((float)k_hit);
            uint32_t v_hits = 0;           // at least this visit's hits (log modes)
            // two copies of the pair loop: with and without the image shift
            // (a select per component would cost more than the adds it saves)
            auto pair_loop = [&](auto shifted_tag) {
            constexpr bool kShifted = decltype(shifted_tag)::value;
            double sh[3] = {0.0, 0.0, 0.0};
            if (kShifted) {
                sh[0] = (double)sx * B;
                sh[1] = (double)sy * B;
                sh[2] = (double)sz * B;
            }
            // Every lane runs every iteration; spare lanes repeat the last pair,
            // which changes no hit (the same bit, the same factor) but counts in
            // v_hits.
            for (int t0 = 0; t0 < pairs; t0 += 64) {
                const int t = min(t0 + lane, pairs - 1);
                const int q = (int)(((float)t + 0.5f) * rk);
                const int r = t - q * k_hit;
                const double* pq = s_pd + 4 * q;
                const PairGeom pg = pair_geom_d<kShifted>(pq[0], pq[1], pq[2], s_o[r],
                                                          s_o[64 + r], s_o[128 + r], sh, u);
                // clamp to [0, L]; a zero's sign cannot change |c|^2
                const double tt = clamp_hi(fmax(pg.sp, 0.0), L);
                double c0 = fma(-tt, u[0], pg.d0);
                double c1 = fma(-tt, u[1], pg.d1);
                double c2 = fma(-tt, u[2], pg.d2);
                double D2 = norm2(c0, c1, c2);
                double hj = pq[3];
                double h2 = hj * hj;
                const bool in = D2 < h2;
                if (kTally) v_hits += (uint32_t)__popcll(wave_ballot(in));
                if (in) {
                    bool near = false;
                    if (NF) near = (pg.d0 * pg.d0 + pg.d1 * pg.d1 + pg.d2 * pg.d2) < h2;
                    if (kTerms) s_gk[t] = hit_factor(pg, u, (float)hj, L, t_erf, gc, ga);
                    atomicOr(&s_mask[r], (near ? 0x10001u : 1u) << q);
                }
            }
            };
            if (shifted) pair_loop(std::true_type{});
            else pair_loop(std::false_type{});
            wave_sync();
            if (kTally) {
                // the visit's hits go to the log: one word for the visit (a second
                // for a shifted image) and one for each ray that hits, in
                // lane order
                const uint32_t m = hit ? s_mask[rank] & 0xffffu : 0u;
                const uint64_t rays = wave_ballot(m != 0u);
                if (rays) {
                    bool full = g_slots + c > kSegFill || g_vis == kSegVisits;
                    if (!full && g_hits + v_hits > kSegHits) {
                        // with the spare lanes' repeats: the hits themselves decide
                        uint32_t hits = g_cnt + (uint32_t)__popc(m);
                        for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off, 64);
                        hits = (uint32_t)__builtin_amdgcn_readfirstlane((int)hits);
                        full = hits > kSegHits;
                        g_hits = hits - v_hits;
                    }
                    if (g_vis && full) close_segment();
                    if (g_vis == 0) open_segment();
                    const uint32_t need = hw + (uint32_t)__popcll(rays);
                    reserve(need);
                    if (kLog && blk != kNoBlock) {
                        uint64_t* at = out.log + ((uint64_t)blk * kLogBlock + pos);
                        if (lane == 0) at[0] = log_visit_word(leafw, g_vis);
                        if (hw == 2u && lane == 1) at[1] = log_image_word(sx, sy, sz, g_vis);
                        if (hw == 4u && lane > 0 && lane < 4)
                            at[lane] = log_axis_word(lane == 1 ? sx : lane == 2 ? sy : sz,
                                                     lane - 1, g_vis);
                        if (m)
                            at[hw + (uint32_t)__popcll(rays & lt_mask)] =
                                log_hits_word(m, lane, g_cnt, g_vis);
                    }
                    g_cnt += (uint32_t)__popc(m);
                    pos += need;
                    g_words += need;
                    g_slots += c;
                    g_hits += v_hits;
                    ++g_vis;
                }
            }
            if (!kTally && hit) {
                const unsigned int m = s_mask[rank];
                if (kCountOnly) cnt += __popc(m & 0xffffu);
                for (unsigned int hb = kCountOnly ? 0u : m & 0xffffu; hb; hb &= hb - 1) {
                    const int q = __ffs(hb) - 1;
                    const int j = f + q;
                    const float gk = kTerms ? s_gk[q * k_hit + rank] : 0.0f;
                    ++cnt;
                    if (MODE == kModeRecord) {
                        if (w < out.hit_cap) {
                            out.hit_j[w] = out.perm[j];
                            out.hit_img[w] = (sx + 8) | ((sy + 8) << 4) | ((sz + 8) << 8);
                            if (out.hit_fac) out.hit_fac[w] = gk;
                        }
                        ++w;
                    }
                    const bool near = NF && ((m >> (16 + q)) & 1u);
                    if (MODE == kModeScatter) {
                        if (nur != 0.0) unsafeAtomicAdd(out.y + j, (double)gk * nur);
                    } else if (near) {
                        accn += (double)((float)out.mu[j] * gk);
                    } else {
                        acc += (double)(mux[j] * gk);
                    }
                }
            }
            wave_sync();                  // the pair buffers are reused by the next leaf
        }
    }
    }   // halos of this wave
    if (active) {
        if ((MODE == kModeColumn || MODE == kModeRecord) && live && out.N) out.N[gid] = acc;
        if (MODE == kModeColumn && live && NF) out.Nn[gid] = accn;
        if (MODE == kModeCount || MODE == kModeStats) out.row_cnt[slot] = cnt;
    }
    if (kTally) {
        if (g_vis) close_segment();
        if (lane == 0) {
            const uint64_t un = ls->unit;
            if (out.unit_log) out.unit_log[un] = make_uint2(ls->first_blk, ls->n_seg);
            if (kLog) {
                if (blk != kNoBlock)
                    out.log[(uint64_t)blk * kLogBlock + kLogData] =
                        (uint64_t)kNoBlock | ((uint64_t)kLogData << 32);
            }
            if (out.unit_size)
                out.unit_size[un] = (uint64_t)ls->size | ((uint64_t)ls->blocks << 32);
        }
        wave_sync();
    }
    uint64_t c64 = cnt;
    if (!kTally) {
        for (int off = 32; off > 0; off >>= 1) c64 += __shfl_xor(c64, off, 64);
        hits_wave += c64;
    }
    const uint64_t rays = MODE == kModeStats ? (uint64_t)__popcll(wave_ballot(active)) : 0;
    if (MODE == kModeStats && lane == 0) {
        atomicAdd(out.stats + 0, (unsigned long long)rays);
        atomicAdd(out.stats + 1, (unsigned long long)st_nodes);
        atomicAdd(out.stats + 2, (unsigned long long)st_lanes);
        atomicAdd(out.stats + 3, (unsigned long long)st_leaves);
        atomicAdd(out.stats + 4, (unsigned long long)st_pairs);
        atomicAdd(out.stats + 5, (unsigned long long)c64);
    }
    if (!PQ) {
        if (kTally) hits_wave = ls->hits;
        if (lane == 0 && hits_wave) atomicAdd(out.hits_total, (unsigned long long)hits_wave);
        return;
    }
    }   // units of this wave
}

#pragma clang fp contract(on)

// Every queue from its start, or spent where a column evaluation is stopped (the
// walk itself reads no more than its queues: the test there cost it 2%).
__global__ void k_zero_queues(unsigned long long* p, const unsigned long long* stop)
{
    const unsigned long long from = stop && *stop != 0ull ? 1ull << 31 : 0ull;
    if (threadIdx.x < kQueues) p[(size_t)threadIdx.x * kQueueStride] = from;
}

}  // namespace

void fill_kernel_tables(KernelTables* host)
{
    const KConst kc = kconst();
    const double t = kc.t, C = kc.C;
    fit_cubics(host->erf_t, [&](double z) { return std::erf(t * z); });
    host->gauss_c = C;
    host->gauss_a = t * t / std::log(2.0);
}

// The wave-cooperative walk: one wave per 64 sources of one direction, or
// (packet queue) a resident grid taking packets from a counter.  The near/far
// variant only for the modes that split near hits.
template <int MODE, bool NF>
static void launch_wave_nf(Ctx& c, RayOut o, int bs, size_t lds, int64_t waves)
{
    const unsigned nb = (unsigned)((waves * 64 + bs - 1) / bs);
    // the persistent form for the walks that record, count or evaluate
    constexpr bool kQueued = MODE == kModeColumn || MODE == kModeCount || mode_logs(MODE);
    if (kQueued && c.packet_queue && o.unit_end == 0) {
        // a kernel, not a memset, clears the counters (the launch may be captured)
        hipLaunchKernelGGL(k_zero_queues, dim3(1), dim3(64), 0, c.stream, c.queue,
                           o.stop);
        o.queue = c.queue;
        int per_cu = 0, cus = 0, dev = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_trace_wave<MODE, NF, kQueued>,
                                                         bs, lds) != hipSuccess || per_cu < 1)
            per_cu = 1;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                hipSuccess || cus < 1)
            cus = 1;
        const unsigned resident = (unsigned)std::min<int64_t>(nb, (int64_t)per_cu * cus);
        hipLaunchKernelGGL((k_trace_wave<MODE, NF, kQueued>), dim3(resident), dim3(bs), lds,
                           c.stream, c.nodes, c.leaf_ball, c.p4, c.mux_s, c.dirs, c.tables, c.geom, o);
        return;
    }
    hipLaunchKernelGGL((k_trace_wave<MODE, NF, false>), dim3(nb), dim3(bs), lds, c.stream,
                       c.nodes, c.leaf_ball, c.p4, c.mux_s, c.dirs, c.tables, c.geom, o);
}

// (units: of a range of them, whose part of the packets is in o already)
template <int MODE>
static void launch_wave(Ctx& c, RayOut o, int64_t units = 0)
{
    const int bs = c.prm.block_size > 0 ? c.prm.block_size : 128;
    const int64_t waves = units ? units : path_packets(c) * (mode_logs(MODE) ? o.parts : 1);
    if (!units) {
        o.n_dir = c.n_ray;
        o.n_pk = (int32_t)((c.n + 63) / 64);
    }
    const size_t lds = wave_lds_bytes(MODE, bs);
    constexpr bool kSplit = MODE == kModeColumn;
    if (kSplit && o.near_far) launch_wave_nf<MODE, kSplit>(c, o, bs, lds, waves);
    else launch_wave_nf<MODE, false>(c, o, bs, lds, waves);
}

template <int MODE>
static void launch_one(Ctx& c, RayOut o)
{
    if (c.prm.traversal == 1) {
        const int bs = c.prm.block_size > 0 ? c.prm.block_size : 128;
        const int64_t n_rays = c.n * (int64_t)c.n_ray;
        const unsigned nb = (unsigned)((n_rays + bs - 1) / bs);
        hipLaunchKernelGGL(k_trace<MODE>, dim3(nb), dim3(bs), 0, c.stream, c.nodes, c.p4, c.mux_s,
                           c.dirs, c.tables, c.geom, o);
    } else {
        launch_wave<MODE>(c, o);
    }
}

static hipError_t launch_mode(Ctx& c, int mode, RayOut o)
{
    if (mode == kModeColumn) launch_one<kModeColumn>(c, o);
    else if (mode == kModeCount) launch_one<kModeCount>(c, o);
    else if (mode == kModeRecord) launch_one<kModeRecord>(c, o);
    else if (mode == kModeStats) {
        // the counters are those of the wave-cooperative walk
        launch_wave<kModeStats>(c, o);
    } else launch_one<kModeScatter>(c, o);
    return hipGetLastError();
}

hipError_t launch_columns(Ctx& c)
{
    RayOut o{};
    o.N = c.N_s;
    o.perm = c.perm;
    o.hits_total = c.red + kRedHits;
    o.near_far = c.near_far;
    o.Nn = c.Nn_s;
    o.mu = c.mu_s;
    o.stop = c.batch_stop;
    return launch_mode(c, kModeColumn, o);
}

hipError_t launch_count_hits(Ctx& c, uint64_t* row_cnt)
{
    RayOut o{};
    o.row_cnt = row_cnt;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;   // counting is not a column evaluation
    return launch_mode(c, kModeCount, o);
}

hipError_t launch_count_rows(Ctx& c, const int32_t* src_list, int32_t src_n, uint64_t* row_cnt)
{
    RayOut o{};
    o.row_cnt = row_cnt;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    o.src_list = src_list;
    o.src_n = src_n;
    return launch_mode(c, kModeCount, o);
}

hipError_t launch_record_rows(Ctx& c, const int32_t* src_list, int32_t src_n,
                              const uint64_t* row_off, int32_t* hit_j, int32_t* hit_img,
                              float* hit_fac, uint64_t cap)
{
    RayOut o{};
    o.hit_cap = cap;
    o.row_off = row_off;
    o.hit_j = hit_j;
    o.hit_img = hit_img;
    o.hit_fac = hit_fac;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    o.src_list = src_list;
    o.src_n = src_n;
    return launch_mode(c, kModeRecord, o);
}

hipError_t launch_trace_stats(Ctx& c, uint64_t* row_cnt, unsigned long long* stats)
{
    RayOut o{};
    o.row_cnt = row_cnt;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    o.stats = stats;
    return launch_mode(c, kModeStats, o);
}

hipError_t launch_record_hits(Ctx& c, const uint64_t* row_off, int32_t* hit_j, int32_t* hit_img,
                              uint64_t cap)
{
    RayOut o{};
    o.hit_cap = cap;
    o.row_off = row_off;
    o.hit_j = hit_j;
    o.hit_img = hit_img;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    return launch_mode(c, kModeRecord, o);
}

hipError_t launch_log_walk(Ctx& c, bool store, uint64_t* unit_size)
{
    RayOut o{};
    o.perm = c.perm;
    o.hits_total = c.red + kRedPathHits;
    o.log = c.path_log;
    o.log_blocks = c.log_blocks;
    o.log_take = log_take(c);
    o.log_ctr = c.log_ctr;
    o.unit_log = c.unit_log;
    o.unit_size = unit_size;
    o.parts = path_parts(c);
    if (store) launch_wave<kModeLog>(c, o);
    else launch_wave<kModeTally>(c, o);
    return hipGetLastError();
}

// The log of a range of the units, whose sizes and segments are known: by the queues
// where it is whole directions or whole packets of one, else a wave to a unit (whose
// kernel spills and is three times as slow on many units).
hipError_t launch_log_range(Ctx& c, int64_t unit0, int64_t units, uint32_t take)
{
    RayOut o{};
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    o.log = c.path_log;
    o.log_blocks = c.log_blocks;
    o.log_take = take;
    o.log_ctr = c.log_ctr;
    o.unit_log = c.unit_log;
    o.parts = path_parts(c);
    const int64_t wpd = (c.n + 63) / 64, per_dir = wpd * o.parts, last = unit0 + units - 1;
    const bool packets = unit0 % o.parts == 0 && units % o.parts == 0;
    o.dir0 = (int32_t)(unit0 / per_dir);
    if (c.packet_queue && unit0 % per_dir == 0 && units % per_dir == 0) {
        o.n_dir = (int32_t)(units / per_dir);
        o.n_pk = (int32_t)wpd;
    } else if (c.packet_queue && packets && unit0 / per_dir == last / per_dir) {
        o.n_dir = 1;
        o.pk0 = (int32_t)(unit0 % per_dir / o.parts);
        o.n_pk = (int32_t)(units / o.parts);
    } else {
        o.unit0 = unit0;
        o.unit_end = unit0 + units;
        o.log_take = 1;                   // a wave's blocks end with its unit
    }
    launch_wave<kModeLog>(c, o, units);
    return hipGetLastError();
}

hipError_t launch_scatter_traverse(Ctx& c, const float* nu, double* y)
{
    RayOut o{};
    o.nu = nu;
    o.y = y;
    o.perm = c.perm;
    o.hits_total = c.red + kRedScratch;
    return launch_mode(c, kModeScatter, o);
}

}  // namespace rrt
