// su3_bwd.hip -- adjoint of the SU(3) link multiply on gfx950.
//
// For the real loss Re sum conj(dC) * C with C[s][j] = A[s][j] B[j]:
//   dA[s][j] = dC[s][j] B[j]^H             (per site, streamed like the forward)
//   dB[j]    = sum_s A[s][j]^H dC[s][j]     (a sum over every site)
// The paper has no adjoint; these are the two contractions of its product.
//
// Stage 1 (bwd_tiles). A lane owns one row (3 complex) of a link at a time,
// 48 B in FP64 and 24 B in FP32, and a wavefront streams steps of 3 chunks
// per lane of dC and A (whole 1 KiB global runs; one 64-row tile in FP64,
// two in FP32), transposed to one row per lane through LDS. Per row k of
// link j it writes row k of dA and adds conj(A(k, m)) dC(k, l) (m, l = 0..2)
// to 18 FP64 accumulators. The tiles of a wavefront are spaced a multiple of
// 3 tiles (192 rows, a multiple of the 12 rows of a site) apart, so a lane
// keeps one row position, hence one link and one accumulator set, on every
// tile. A workgroup of 3 wavefronts takes kSteps steps each, 1, 2 or 4 by the
// lattice size; in most forms the workgroups are taken in batches of 256 and
// step k of every workgroup of a batch lies in one contiguous block (phase
// striping), which keeps the workgroups that run together on one contiguous
// front.
// At the end the lanes' accumulators are summed in a fixed order: per row
// position within the wavefront (lanes in increasing order), then per link
// over the workgroup's wavefronts and the link's three rows. Each workgroup
// writes one 4x3x3 complex FP64 partial. Partials are stored in quads of
// components: quad u = q / 4 holds, for every workgroup g, the 4 doubles of
// components 4u .. 4u+3 at 4 (u * groups + g), so each workgroup writes 18
// whole 32-byte sectors rather than 72 scattered doubles (a scattered
// 8-byte store costs a whole sector of HBM writes).
// Stage 2 (bwd_sum) reduces the partials of each of the 72 real components in
// two fixed-order levels in one launch: runs of kChunk consecutive partials
// of a quad's 4 components, one workgroup each, then the run sums, by the
// last workgroup of the quad to arrive. Both levels keep every load of a
// thread in flight at once, so stage 2 costs a few microseconds at any
// lattice size.
// The number of workgroups of every stage depends only on the number of sites,
// the precision and which of two sizes the workspace has, so the rounding sequence, and every bit of dB, is the same on
// every run and every device. The only atomics are stage 2's arrival counts,
// which decide who adds the run sums, not in which order.
#include "su3_internal.hpp"

namespace su3 {

constexpr int kBwdWaves = 3;                 // wavefronts per workgroup
constexpr int kBwdThreads = 64 * kBwdWaves;
// Forms of stage 1: kSub 64-row tiles per step (3 chunks per lane of each
// array), kSteps steps per wavefront, at most kWaves resident wavefronts per CU.
// More steps amortise the closing reduction and cut the partials stage 2
// reads; fewer shorten the drain at the end of the grid and spread a small
// lattice over more CUs.
// kBatch, phase striping (0: off): the workgroups are taken in batches of
// kBatch, and step k of every workgroup of a batch lies in one contiguous
// block of the batch's tiles, so the workgroups that run at the same time
// stream one contiguous front instead of each its own run.
// kEarly: a wavefront's first loads are issued before the barrier that
// publishes b, so they do not wait for it.
// kGroup: the workgroups take the groups in the grouped order, 16 consecutive
// per XCD (each group's work and partial slot stay, so dB does too).
template <typename S_, int kSub_, int kSteps_, int kBatch_, bool kEarly_, int kWaves_, bool kGroup_ = false>
struct BwdForm {
    typedef S_ S;
    static constexpr int kSub = kSub_, kSteps = kSteps_, kBatch = kBatch_, kWaves = kWaves_;
    static constexpr bool kEarly = kEarly_, kGroup = kGroup_;
    static constexpr int kTiles = kBwdWaves * kSub * kSteps;   // 64-row tiles per workgroup
};
// 64-row tiles per workgroup of the forms that the smallest workspace holds the
// partials of; the others (`spread`) take 3 or 6, and need up to 4 times as much.
// Spreading through more wavefronts per workgroup instead, 12 of one step or 6
// of two on 12 tiles, needs no more but loses what it is for: FP64 4,096 sites
// 8.1 us against 6.3, 20,000 12.8 against 10.8, 160,000 55 against 50.
constexpr int kCompactTiles = 12;
// Which form takes which lattice, by the last site count of each (sweeps of 1,
// 2 and 4 steps, caps of 9 and 12, batches of 0 and 256 and both kEarly at 16
// sizes; microseconds, both stages, against 4 steps, a cap of 9 and a batch of
// 256 in FP64 and 2 steps and a cap of 12 in FP32, both without kEarly).
// The lines at 16,384 and 32,768 sites lie where the whole grid is resident at
// once, 4 workgroups per CU, with 1 and 2 steps. 131,072 is where the partials of 4
// steps still are one run of stage 2 (2,048): up to there 4 steps are the faster
// (against 2 grouped steps 65,537 sites 1.08, 98,304 1.03, 131,072 1.01), past it 2
// (131,073 1.02-1.03, 160,000 1.02-1.03, 200,000 1.03-1.04).
//  FP64: 4,096 sites 6.2 / 8.4, 16,384 9.6 / 10.2, 20,000 10.8 / 12.0, 131,072
//  42.6 / 43.2, 160,000 49.9 / 52.1, 331,776 96 / 98, 2^20 288 / 292, 2,000,000
//  542 / 556 (2 steps there: 567).
//  FP32: 4,096 sites 6.6 / 7.5, 32,768 9.9 / 10.7, 100,000 20.7 / 21.2, 331,776
//  52.3 / 52.9; above 700,000 sites kEarly loses 1-5% and a batch 1-2%.
// kGroup is worth 1-2% in FP64 from 131,072 sites (331,776: 97.2 -> 96.0,
// 2,560,000: 711 -> 702) and 0-1.5% in FP32 from 700,000; below, it loses up to
// 5%, as does a run-time choice of the order. Groups of 2 to 64, and batches of
// 128 and 512 with them, were level or slower, and one contiguous eighth of
// the groups per XCD 4-8% slower.
typedef BwdForm<double, 1, 1, 0, true, 12> BwdF64x1;            // spread, to 16,384 sites
typedef BwdForm<double, 1, 2, 256, true, 12> BwdF64x2;          // spread, to 32,768
typedef BwdForm<double, 1, 4, 256, true, 9> BwdF64x4;           // to 131,072; compact, to 400,000
typedef BwdForm<double, 1, 2, 256, true, 12, true> BwdF64x2g;   // spread, to 400,000
typedef BwdForm<double, 1, 4, 256, true, 9, true> BwdF64x4g;    // above
typedef BwdForm<float, 2, 1, 0, true, 12> BwdF32x1;             // spread, to 32,768
typedef BwdForm<float, 2, 2, 256, true, 12> BwdF32x2;           // to 700,000
typedef BwdForm<float, 2, 2, 0, false, 12, true> BwdF32x2g;     // above
// dB alone (kSteps 0: the step count is a launch argument, db_steps).
typedef BwdForm<double, 1, 0, 256, true, 9> DbF64;
typedef BwdForm<float, 2, 0, 256, true, 9> DbF32;
constexpr int64_t kLast64[] = {16384, 32768, 131072, 400000};
constexpr int64_t kLast32[] = {32768, 700000};
constexpr int kRowsPerSite = 12;

// Stage 2: threads per workgroup and partials per thread of one run.
#ifndef SU3_BWD_CHUNK_THREADS
#define SU3_BWD_CHUNK_THREADS 256
#endif
#ifndef SU3_BWD_CHUNK_LOADS
#define SU3_BWD_CHUNK_LOADS 8
#endif
constexpr int kChunkThreads = SU3_BWD_CHUNK_THREADS;
constexpr int kChunkLoads = SU3_BWD_CHUNK_LOADS;
constexpr int64_t kChunk = (int64_t)kChunkThreads * kChunkLoads;

// Row `lane` of sub-tile q of a staged step, as 6 interleaved re/im values.
__device__ __forceinline__ void row_from_stage(const u4 *st, int q, int lane, double (&v)[6])
{
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const d2 w = __builtin_bit_cast(d2, st[192 * q + 3 * lane + e]);
        v[2 * e] = w.x;
        v[2 * e + 1] = w.y;
    }
}
__device__ __forceinline__ void row_from_stage(const u4 *st, int q, int lane, float (&v)[6])
{
    const f2 *p = reinterpret_cast<const f2 *>(st) + 192 * q + 3 * lane;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const f2 w = p[e];
        v[2 * e] = w.x;
        v[2 * e + 1] = w.y;
    }
}
__device__ __forceinline__ void row_to_stage(u4 *st, int q, int lane, const double (&v)[6])
{
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const d2 w = {v[2 * e], v[2 * e + 1]};
        st[192 * q + 3 * lane + e] = __builtin_bit_cast(u4, w);
    }
}
__device__ __forceinline__ void row_to_stage(u4 *st, int q, int lane, const float (&v)[6])
{
    f2 *p = reinterpret_cast<f2 *>(st) + 192 * q + 3 * lane;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const f2 w = {v[2 * e], v[2 * e + 1]};
        p[e] = w;
    }
}

// kDa: form and store dA as well as dB's partials; without it b and da are not
// touched. `steps` is the step count of the forms without one.
template <class F, bool kDa>
__global__ __launch_bounds__(kBwdThreads) void bwd_tiles(const u4 *__restrict__ a, const typename F::S *__restrict__ b,
                                                         const u4 *__restrict__ dc, u4 *__restrict__ da,
                                                         double *__restrict__ ws, uint32_t *__restrict__ counts,
                                                         int64_t rows, int64_t groups, int steps)
{
    typedef typename F::S S;
    constexpr int kSub = F::kSub;                     // 64-row tiles per step
    const int nsteps = F::kSteps > 0 ? F::kSteps : steps;
    constexpr int CT = 64 * 6 * (int)sizeof(S) / 16;  // chunks per 64-row tile: 192 or 96
    constexpr int kStageBytes = 2 * 3 * 64 * 16;      // a and dC, 3 chunks per lane each
    constexpr int kRedBytes = 64 * 19 * 8;            // 18 accumulators per lane, padded
    constexpr int kBytes = kStageBytes > kRedBytes ? kStageBytes : kRedBytes;
    // per-wavefront LDS: step staging in the loop, reduction after it
    __shared__ __attribute__((aligned(16))) char tilebuf[kBwdWaves][kBytes];
    __shared__ double rowsum[kBwdWaves][kRowsPerSite * 18];
    __shared__ S bsh[72];

    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    u4 *stg = reinterpret_cast<u4 *>(tilebuf[wv]);    // dC at [0, 192), A at [192, 384)
    double *red = reinterpret_cast<double *>(tilebuf[wv]);
    // this workgroup's tile group; its partial goes to slot grp
    const int64_t grp = F::kGroup ? group_order<16>(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    // the wavefront's first 64-row tile t0; it takes t0 + D i for
    // i < kSub * nsteps (D a multiple of 3)
    const int64_t per = (int64_t)kBwdWaves * kSub * nsteps;   // tiles of a workgroup
    int64_t t0, D;
    if constexpr (F::kBatch > 0) {
        constexpr int kB = F::kBatch;
        const int64_t bt = grp / kB, lam = grp - bt * kB;
        const int64_t nb = groups - bt * kB < kB ? groups - bt * kB : (int64_t)kB;
        t0 = bt * per * kB + kBwdWaves * lam + wv;
        D = kBwdWaves * nb;
    } else {
        t0 = grp * per + wv;
        D = kBwdWaves;
    }
    const int64_t nchunks = rows * 6 * (int64_t)sizeof(S) / 16;

    // Global chunk of step-chunk c (c = 64 i + lane, i < 3) of the step that
    // starts at tile ts: sub-tile c / CT, chunk c mod CT of it.
    auto gchunk = [&](int64_t ts, int i) -> int64_t {
        const int c = 64 * i + lane, q = c / CT;
        return (ts + D * q) * CT + (c - q * CT);
    };
    // Step loads: chunks past the end re-read the last chunk (in bounds; they
    // are cleared before use, and store nothing). The loads of the next step
    // are issued as soon as the current step sits in LDS, so they are in
    // flight while the current step is computed and stored.
    u4 va[3], vg[3];
    auto load_step = [&](int64_t ts) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int64_t g = gchunk(ts, i);
            const int64_t gc = g < nchunks ? g : nchunks - 1;
            vg[i] = ld_stream(dc + gc);
            va[i] = ld_stream(a + gc);
        }
    };
    // b before the first step: vector memory operations retire in order, so the
    // barrier that publishes b in LDS waits for the b load only while the step
    // is in flight.
    const S bv = kDa && threadIdx.x < 72 ? b[threadIdx.x] : S(0);
    if (F::kEarly)
        load_step(t0);
    if (blockIdx.x == 0 && threadIdx.x < 18)
        counts[threadIdx.x] = 0;   // for stage 2
    S br[9], bi[9];
    if constexpr (kDa) {
        if (threadIdx.x < 72)
            bsh[threadIdx.x] = bv;
        __syncthreads();
        const int pos = (int)((t0 * 64 + lane) % kRowsPerSite);   // row position in the site
        const int j = pos / 3;                                     // its link
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            br[q] = bsh[2 * (9 * j + q)];
            bi[q] = bsh[2 * (9 * j + q) + 1];
        }
    }
    double acc[18];
#pragma unroll
    for (int v = 0; v < 18; ++v)
        acc[v] = 0.0;
    if (!F::kEarly)
        load_step(t0);
    for (int k = 0; k < nsteps; ++k) {
        const int64_t ts = t0 + D * kSub * k;   // the step's first tile
        if (ts * 64 >= rows)
            break;                              // wave-uniform
        // every row of the step's last tile is in the lattice
        const bool whole = (ts + D * (kSub - 1) + 1) * 64 <= rows;
        // Rows past the end of the lattice hold re-read data, of another link
        // even, and have to add exact zeros to dB: both factors are cleared,
        // as 0 times a non-finite dC would be NaN. A row past the end is whole
        // chunks past the end (rows come in twelves, chunks in rows or pairs).
        if (!whole) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (gchunk(ts, i) >= nchunks)
                    vg[i] = va[i] = u4{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            stg[64 * i + lane] = vg[i];
            stg[192 + 64 * i + lane] = va[i];
        }
        wave_sync();
        if (k + 1 < nsteps && (ts + D * kSub) * 64 < rows)
            load_step(ts + D * kSub);
        S o[kSub][6];
#pragma unroll
        for (int q = 0; q < kSub; ++q) {
            S g[6], x[6];     // interleaved re/im of dC and A row `lane` of sub-tile q
            row_from_stage(stg, q, lane, g);
            row_from_stage(stg + 192, q, lane, x);
            // dA(k, m) = sum_l dC(k, l) conj(B(m, l))
#pragma unroll
            for (int m = 0; kDa && m < 3; ++m) {
                S re = 0, im = 0;
#pragma unroll
                for (int l = 0; l < 3; ++l)
                    cmac(re, im, g[2 * l], g[2 * l + 1], br[3 * m + l], -bi[3 * m + l]);
                o[q][2 * m] = re;
                o[q][2 * m + 1] = im;
            }
            // dB(m, l) += conj(A(k, m)) dC(k, l), in FP64
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int l = 0; l < 3; ++l)
                    cmac(acc[6 * m + 2 * l], acc[6 * m + 2 * l + 1], (double)x[2 * m], -(double)x[2 * m + 1],
                         (double)g[2 * l], (double)g[2 * l + 1]);
        }
        wave_sync();
        if constexpr (!kDa)
            continue;
#pragma unroll
        for (int q = 0; q < kSub; ++q)
            row_to_stage(stg, q, lane, o[q]);
        wave_sync();
        // store the dA step as 3 whole-wavefront runs, guarded past the end
        u4 w[3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            w[i] = stg[64 * i + lane];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int64_t g = gchunk(ts, i);
            if (whole || g < nchunks)
                st_stream(da + g, w[i]);
        }
        wave_sync();
    }

    // ---- fixed-order reduction --------------------------------------------
    // The lanes' 18 accumulators go to LDS (row stride 19 doubles); then the
    // sums of the 12 row positions r are formed: output 18*r + e adds the
    // lanes at position r, (r - base) mod 12 and every 12th lane after it,
    // in increasing order. Every load of a lane is issued before the first
    // add (fixed trip counts; a lane index past 63 reads lane 63 and adds an
    // exact zero instead).
    const int base = (int)((t0 * 64) % kRowsPerSite);
    constexpr int kLanesPerPos = (64 + kRowsPerSite - 1) / kRowsPerSite;   // 6
    constexpr int kOut = kRowsPerSite * 18;                                 // 216
#pragma unroll
    for (int v = 0; v < 18; ++v)
        red[lane * 19 + v] = acc[v];
    wave_sync();
#pragma unroll
    for (int it = 0; it < (kOut + 63) / 64; ++it) {
        const int o3 = lane + 64 * it;
        if (o3 < kOut) {
            const int r = o3 / 18, e = o3 % 18;
            const int l0 = ((r - base) % kRowsPerSite + kRowsPerSite) % kRowsPerSite;
            double x[kLanesPerPos];
#pragma unroll
            for (int i = 0; i < kLanesPerPos; ++i) {
                const int l = l0 + kRowsPerSite * i;
                const double y = red[(l < 64 ? l : 63) * 19 + e];
                x[i] = l < 64 ? y : 0.0;
            }
            double sum = x[0];
#pragma unroll
            for (int i = 1; i < kLanesPerPos; ++i)
                sum += x[i];
            rowsum[wv][o3] = sum;
        }
    }
    __syncthreads();
    // workgroup partial of component q = 18*j + e: wavefronts in order, then
    // the link's three rows in order
    if (threadIdx.x < 72) {
        const int jj = threadIdx.x / 18, e = threadIdx.x % 18;
        double sum = 0.0;
        for (int w2 = 0; w2 < kBwdWaves; ++w2)
            for (int r = 3 * jj; r < 3 * jj + 3; ++r)
                sum += rowsum[w2][18 * r + e];
        ws[4 * ((int64_t)(threadIdx.x >> 2) * groups + grp) + (threadIdx.x & 3)] = sum;
    }
}

// Stage 2, grid = (chunks, 18): workgroup (c, u) adds partials c*kChunk ..
// c*kChunk + kChunk - 1 of the 4 components of quad u. Thread t adds partials
// t, t + kChunkThreads, ... in order; then, per component, a binary tree across
// the lanes of each wavefront pairs lane t with t + w for w = 32, 16, ..., 1,
// and the wavefront sums are added in wavefront order. With one run that is
// dB. Otherwise the workgroup leaves its run's 4 sums in the run's first
// partial slot, whose contents it has read, and counts itself in; the last
// one of quad u adds the run sums in the same fixed order, whichever
// workgroup it is: lane t of wavefront e takes runs t, t + 64, ... of component
// e in order, then the tree.
// Run sums and counts move at agent scope (write-through stores, loads and
// atomics at the memory side), each store complete before the count, so no
// cache has to be written back or invalidated; a release fence would write
// back the XCD's whole L2 in every workgroup, which made one launch slower
// than two. The order of sum and count rests on the hardware, not on the
// language's memory model, which grants relaxed accesses none: a store at agent
// scope writes through, vmcnt counts it until it has reached the memory side, and
// the loads that follow the last arrival's count read there. Two launches took 9.3 us (4.7 and 4.6) after stage 1 in FP64, at
// L = 32 and at 24^4 alike; this one takes 5.8 and 5.4.
// T: the type dB is stored in, double, or float for the FP64 sum rounded once.
template <typename T>
__global__ __launch_bounds__(kChunkThreads) void bwd_sum(double *__restrict__ ws, T *__restrict__ db,
                                                         uint32_t *__restrict__ counts, int64_t groups,
                                                         int64_t chunks)
{
    constexpr int kW = kChunkThreads / 64;
    static_assert(kW >= 4, "one wavefront per component in the last workgroup");
    __shared__ double red[4][kW];
    __shared__ uint32_t arrived;
    const int64_t c = blockIdx.x;
    const int u = blockIdx.y, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double *quad = ws + 4 * (int64_t)u * groups;   // 4 doubles per workgroup of stage 1
    const d2 *src = reinterpret_cast<const d2 *>(quad);
    d2 v[kChunkLoads][2];
#pragma unroll
    for (int i = 0; i < kChunkLoads; ++i) {
        const int64_t g = c * kChunk + (int64_t)kChunkThreads * i + threadIdx.x;
        const d2 z = {0.0, 0.0};
        v[i][0] = g < groups ? src[2 * g] : z;
        v[i][1] = g < groups ? src[2 * g + 1] : z;
    }
    double sum[4] = {v[0][0].x, v[0][0].y, v[0][1].x, v[0][1].y};
#pragma unroll
    for (int i = 1; i < kChunkLoads; ++i) {
        sum[0] += v[i][0].x;
        sum[1] += v[i][0].y;
        sum[2] += v[i][1].x;
        sum[3] += v[i][1].y;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            sum[e] += __shfl_down(sum[e], w, 64);
    if (lane == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            red[e][wv] = sum[e];
    }
    __syncthreads();
    double total = 0.0;
    if (threadIdx.x < 4) {
        total = red[threadIdx.x][0];
#pragma unroll
        for (int w2 = 1; w2 < kW; ++w2)
            total += red[threadIdx.x][w2];
    }
    if (chunks == 1) {
        if (threadIdx.x < 4)
            db[4 * u + threadIdx.x] = (T)total;
        return;
    }
    if (wv == 0) {
        if (lane < 4)
            __hip_atomic_store(quad + 4 * c * kChunk + lane, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the sums have reached memory
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(counts + u, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (arrived != (uint32_t)chunks - 1 || wv >= 4)
        return;
    double x = 0.0;
    for (int64_t k = lane; k < chunks; k += 64)
        x += __hip_atomic_load(quad + 4 * k * kChunk + wv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1)
        x += __shfl_down(x, w, 64);
    if (lane == 0)
        db[4 * u + wv] = (T)x;
}

// dB of an empty lattice.
template <typename T>
__global__ __launch_bounds__(128) void bwd_zero(T *__restrict__ db)
{
    if (threadIdx.x < 72)
        db[threadIdx.x] = T(0);
}

static_assert(BwdF64x4::kTiles == kCompactTiles && BwdF64x4g::kTiles == kCompactTiles &&
                  BwdF32x2::kTiles == kCompactTiles && BwdF32x2g::kTiles == kCompactTiles,
              "the compact forms have one count of partials");

// The 64-row tiles of one workgroup of stage 1 for a lattice of n sites.
static int64_t tiles_per_group(int64_t n, int precision, bool spread)
{
    if (!spread)
        return kCompactTiles;
    if (precision == 0)
        return n <= kLast64[0]   ? BwdF64x1::kTiles
               : n <= kLast64[1] ? BwdF64x2::kTiles
               : n <= kLast64[2] ? BwdF64x4::kTiles
               : n <= kLast64[3] ? BwdF64x2g::kTiles
                                 : BwdF64x4g::kTiles;
    return n <= kLast32[0] ? BwdF32x1::kTiles : n <= kLast32[1] ? BwdF32x2::kTiles : BwdF32x2g::kTiles;
}

// Workgroups of stage 1 for `sites`, spread or not.
int64_t bwd_groups(int64_t sites, int precision, bool spread)
{
    const int64_t tiles = (sites * kRowsPerSite + 63) / 64, per = tiles_per_group(sites, precision, spread);
    return (tiles + per - 1) / per;
}

static int64_t bwd_chunks(int64_t groups) { return (groups + kChunk - 1) / kChunk; }

// Steps of dB alone: nothing is written per site, so long-lived workgroups
// cost nothing and save closing reductions and partials. About 512
// workgroups, two per CU, of at most 32 steps (microseconds, both stages,
// against the steps of the whole adjoint): FP64 131,072 sites 27 / 30,
// 331,776 63 / 70, 2^20 182 / 218 (6.6 TB/s), 2,560,000 448 / 538; FP32 2^20 96
// / 111. Fewer or more workgroups at mid-sized lattices and caps of 12 or 15
// were 0-3% slower.
static int db_steps(int64_t sites, int precision)
{
    const int64_t tiles = (sites * kRowsPerSite + 63) / 64;
    const int64_t per_step = kBwdWaves * (precision == 0 ? DbF64::kSub : DbF32::kSub);
    const int64_t steps = (tiles + 512 * per_step - 1) / (512 * per_step);
    return (int)(steps < 32 ? steps : 32);
}

// The partials, and as many doubles as there are run sums: stage 2 keeps its
// 18 counts (4 bytes each) there. A form with fewer steps makes more groups,
// so the groups do not grow with the sites everywhere; the workspace does, and
// one that is large enough for a lattice is large enough for any smaller one.
int64_t bwd_workspace_doubles(int64_t sites, int precision, bool spread)
{
    int64_t groups = bwd_groups(sites, precision, spread);
    auto at_least = [&](const int64_t *last, int count) {
        for (int i = 0; i < count; ++i)
            if (last[i] < sites && bwd_groups(last[i], precision, spread) > groups)
                groups = bwd_groups(last[i], precision, spread);
    };
    if (precision == 0)
        at_least(kLast64, sizeof(kLast64) / sizeof(kLast64[0]));
    else
        at_least(kLast32, sizeof(kLast32) / sizeof(kLast32[0]));
    return 72 * (groups + bwd_chunks(groups));
}

int bwd_block_threads() { return kBwdThreads; }

template <class F, bool kDa>
static hipError_t launch_tiles_f(const void *a, const void *b, const void *dc, void *da, int64_t sites, double *ws,
                                 uint32_t *counts, int64_t groups, int steps, hipStream_t s)
{
    static PadCache cache;
    const LaunchPlan plan =
        launch_plan(reinterpret_cast<const void *>(bwd_tiles<F, kDa>), F::kWaves, kBwdThreads, groups, cache);
    return launch_k(bwd_tiles<F, kDa>, dim3((unsigned)groups), dim3(kBwdThreads), s, plan.pad, (const u4 *)a,
                    (const typename F::S *)b, (const u4 *)dc, (u4 *)da, ws, counts, sites * kRowsPerSite, groups, steps);
}

// Stage 2 over `groups` partials; db in double, or in float for `db_float`.
static hipError_t launch_sum(double *ws, uint32_t *counts, int64_t groups, void *db, bool db_float, hipStream_t s)
{
    const int64_t chunks = bwd_chunks(groups);
    const dim3 grid((unsigned)chunks, 18);
    if (db_float)
        return launch_k(bwd_sum<float>, grid, dim3(kChunkThreads), s, 0, ws, (float *)db, counts, groups, chunks);
    return launch_k(bwd_sum<double>, grid, dim3(kChunkThreads), s, 0, ws, (double *)db, counts, groups, chunks);
}

hipError_t launch_bwd(const void *a, const void *b, const void *dc, void *da, void *db, bool db_float, int64_t sites,
                      int precision, bool spread, double *ws, hipStream_t s)
{
    const int64_t groups = bwd_groups(sites, precision, spread);
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + 72 * groups);
    auto *launch = precision != 0 ? (spread && sites <= kLast32[0] ? launch_tiles_f<BwdF32x1, true>
                                     : sites <= kLast32[1]         ? launch_tiles_f<BwdF32x2, true>
                                                                   : launch_tiles_f<BwdF32x2g, true>)
                   : sites > kLast64[3]                        ? launch_tiles_f<BwdF64x4g, true>
                   : !spread                                   ? launch_tiles_f<BwdF64x4, true>
                   : sites <= kLast64[0]                       ? launch_tiles_f<BwdF64x1, true>
                   : sites <= kLast64[1]                       ? launch_tiles_f<BwdF64x2, true>
                   : sites <= kLast64[2]                       ? launch_tiles_f<BwdF64x4, true>
                                                               : launch_tiles_f<BwdF64x2g, true>;
    const hipError_t e = launch(a, b, dc, da, sites, ws, counts, groups, 0, s);
    return e != hipSuccess ? e : launch_sum(ws, counts, groups, db, db_float, s);
}

// Its groups are never more than those of the whole adjoint, spread or not, whose
// workspace therefore serves it.
hipError_t launch_db(const void *a, const void *dc, void *db, bool db_float, int64_t sites, int precision, bool spread,
                     double *ws, hipStream_t s)
{
    const int per_step = kBwdWaves * (precision == 0 ? DbF64::kSub : DbF32::kSub);
    int steps = db_steps(sites, precision);
    if (!spread && steps * per_step < kCompactTiles)
        steps = kCompactTiles / per_step;
    const int64_t tiles = (sites * kRowsPerSite + 63) / 64;
    const int64_t per = (int64_t)per_step * steps;
    const int64_t groups = (tiles + per - 1) / per;
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + 72 * groups);
    const hipError_t e = (precision == 0 ? launch_tiles_f<DbF64, false> : launch_tiles_f<DbF32, false>)(
        a, nullptr, dc, nullptr, sites, ws, counts, groups, steps, s);
    return e != hipSuccess ? e : launch_sum(ws, counts, groups, db, db_float, s);
}

// An empty lattice has dB = 0 (a kernel rather than a memset, so the call is
// safe to capture).
hipError_t launch_bwd_zero(void *db, bool db_float, hipStream_t s)
{
    if (db_float)
        return launch_k(bwd_zero<float>, dim3(1), dim3(128), s, 0, (float *)db);
    return launch_k(bwd_zero<double>, dim3(1), dim3(128), s, 0, (double *)db);
}

// ---- the library-owned workspace of su3_mult_nn_bwd_noalloc ---------------
// A fixed device array (each device the library runs on holds its own copy
// until the process ends). Its name is only a host-side handle: host code
// uses the device address that hipGetSymbolAddress returns for the current
// device, kept per device in scratch_ptr.
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];
static std::atomic<double *> scratch_ptr[kMaxDevices];

hipError_t bwd_scratch(double **ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= kMaxDevices)
        return hipErrorInvalidDevice;
    double *p = scratch_ptr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        // racing first calls on one device get the same address
        e = hipGetSymbolAddress(reinterpret_cast<void **>(&p), HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return e;
        if (p == nullptr)
            return hipErrorInvalidSymbol;
        scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

} // namespace su3
