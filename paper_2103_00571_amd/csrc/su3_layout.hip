// su3_layout.hip -- data movement around the link multiply on gfx950:
// AoS <-> SoA transposes, FP64 <-> storage-form conversion (pack/unpack),
// and the plain streaming copy used as the bandwidth reference.
#include "su3_internal.hpp"

#include <type_traits>

namespace su3 {

// Resident wavefronts per CU of the reconstruct-12 conversions, with FP32 and
// FP64 rows. The unpack has 9 KiB of stores and 3 or 6 KiB of loads per
// wavefront (FP64, 100,000 sites: 16.1 us with 7 and 16.7 with 6, 2,560,000: 391
// and 385). The pack has 9 KiB of loads (FP32, 100,000 sites: 13.6 with 12 and
// 14.5 with 6; from 1,000,000, with nontemporal stores, 5% faster with 6 than
// with 4; FP64, 200,000: 28.8 with 6, 29.8 with 4; 2,560,000, write-through: 377
// and 367).
constexpr WaveCaps kUnpackR12F32 = one_cap(7);
constexpr WaveCaps kUnpackR12F64 = {{130000000, INT64_MAX}, {7, 6, 6}};
constexpr WaveCaps kPackR12F32 = {{260000000, INT64_MAX}, {12, 6, 6}};
constexpr WaveCaps kPackR12F64 = {{kThroughAgain / 384 * 960, INT64_MAX}, {6, 4, 4}, 75};

// Bytes written by the reconstruct-12 unpack up to which, and with FP32 rows past
// which, its stores write through (launch_unpack_r12).
constexpr int64_t kFitUnpackR12 = 155000000, kThroughAgainUnpackR12 = 750000000;

// The FP32 pack and unpack and the general transposes loop over their items
// with a grid stride, on a grid of up to kOnePass workgroups: one pass for
// all but the largest lattices, which streams faster than fewer workgroups
// looping.
constexpr int64_t kOnePass = (int64_t)1 << 24;

// ------------------------------------------------------------ AoS <-> SoA
// One workgroup moves a tile of 64 sites at a time through LDS: the site-
// major side is read or written as one contiguous run of 64*36 elements, the
// plane side as 36 contiguous runs of 64 elements. The LDS row has one
// element of padding so that the column walk does not hit one bank.
// A whole tile is moved with every load of a thread issued before the first
// LDS write (9 elements per thread), nontemporal loads and stores, and, in
// FP64, the XCD-contiguous tile order (each XCD one contiguous eighth of the
// tiles; a one-pass grid). The last, ragged tile moves element by element.
// This is the path of the small lattices (of any too large for the one-pass grids
// below, and of some between); launch_aos_soa has the rule.
constexpr int kTileSites = 64;

template <typename V, bool kToSoa, bool kXcd>
__global__ __launch_bounds__(kBlock) void transpose_aos_soa(const V *__restrict__ src, V *__restrict__ dst,
                                                            int64_t n, int64_t pitch)
{
    __shared__ V tile[36][kTileSites + 1];
    constexpr int kPer = 36 * kTileSites / kBlock;
    static_assert(kPer * kBlock == 36 * kTileSites, "a tile splits evenly over the workgroup");
    const int64_t tiles = (n + kTileSites - 1) / kTileSites;
    // the XCD order needs the one-pass grid (one workgroup per tile)
    int64_t t = blockIdx.x;
    if (kXcd && (int64_t)gridDim.x >= tiles)
        t = xcd_order(blockIdx.x, gridDim.x);
    for (; t < tiles; t += gridDim.x) {
        const int64_t s0 = t * kTileSites;
        const int ns = (int)((n - s0) < kTileSites ? (n - s0) : kTileSites);
        if (ns == kTileSites) {
            V v[kPer];
            if (kToSoa) {
#pragma unroll
                for (int i = 0; i < kPer; ++i)
                    v[i] = ld_stream(src + s0 * 36 + threadIdx.x + i * kBlock);
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    tile[e % 36][e / 36] = v[i];
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    v[i] = tile[e / kTileSites][e % kTileSites];
                }
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    st_stream(dst + (int64_t)(e / kTileSites) * pitch + s0 + e % kTileSites, v[i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    v[i] = ld_stream(src + (int64_t)(e / kTileSites) * pitch + s0 + e % kTileSites);
                }
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    tile[e / kTileSites][e % kTileSites] = v[i];
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = threadIdx.x + i * kBlock;
                    v[i] = tile[e % 36][e / 36];
                }
#pragma unroll
                for (int i = 0; i < kPer; ++i)
                    st_stream(dst + s0 * 36 + threadIdx.x + i * kBlock, v[i]);
            }
        } else if (kToSoa) {
            for (int e = threadIdx.x; e < ns * 36; e += kBlock)
                tile[e % 36][e / 36] = src[s0 * 36 + e];
            __syncthreads();
            for (int e = threadIdx.x; e < 36 * kTileSites; e += kBlock) {
                const int p = e / kTileSites, sl = e % kTileSites;
                if (sl < ns)
                    dst[(int64_t)p * pitch + s0 + sl] = tile[p][sl];
            }
        } else {
            for (int e = threadIdx.x; e < 36 * kTileSites; e += kBlock) {
                const int p = e / kTileSites, sl = e % kTileSites;
                if (sl < ns)
                    tile[p][sl] = src[(int64_t)p * pitch + s0 + sl];
            }
            __syncthreads();
            for (int e = threadIdx.x; e < ns * 36; e += kBlock)
                dst[s0 * 36 + e] = tile[e % 36][e / 36];
        }
        __syncthreads();
    }
}

// The same transforms for the larger lattices, one tile of TS sites per
// workgroup of B threads. What bounds them is the 36 plane streams: a kernel
// that only copies the same addresses (36 KiB per workgroup in and out, no
// LDS, nontemporal stores, workgroup order) peaks at 6.0 (to planes) and 6.2 TB/s
// (from planes) at 2,560,000 FP64 sites, with one such workgroup per CU, and falls
// to 5.6 and 5.9 with two to four; the run length on the planes (1 to 16 KiB) does
// not matter. So the tile and the number of resident workgroups set the bytes in
// flight, and many threads with few elements each keep a tile's life short. Write-
// through stores in the grouped order pass that copy (6.1 and 6.3 TB/s); the bound
// with them has not been probed.
// launch_aos_soa states which tile serves which size.
// kThrough: write-through stores (OutWindow) instead of nontemporal ones.
// kGroup: the grouped tile order (group_order), which alone is worth 1-2% and
// with these stores 4-5% (groups of 2, 4, 16, 32 and 64 and all the tiles of an
// XCD together were 0 to 4% slower). To planes the groups collide where the
// plane stride is near a power of two (0.84 to 0.98 of the speed from 2^17 to
// 2^21 sites) and gain nothing up to a million sites; they gain 1-6% beyond.
//
// kHalo, for planes that do not start on 128-byte lines (a site count that
// is no multiple of 8 in FP64 or 16 in FP32, dense): a run cut at the tile's
// own sites would begin and end inside a line that the neighbouring
// workgroup writes too, and two partial writes of a line cost far more than
// one whole one (at 31^4 sites 4.4 TB/s in FP64 and 3.7 in FP32, and 5.5 and
// 5.1 with the halo). The workgroup instead reads
// one line's worth of sites past its tile and moves each plane's window up to
// that plane's next line boundary, so that every line is written whole by one
// workgroup; the first tile also writes the sites before its window.
template <typename V, int TS, int B, bool kHalo, bool kThrough, bool kGroup>
__global__ __launch_bounds__(B) void to_soa_tile(const V *__restrict__ src, V *__restrict__ dst, int64_t n,
                                                 int64_t pitch)
{
    constexpr int H = kHalo ? 128 / (int)sizeof(V) : 1;   // sites per line
    constexpr int W = kHalo ? TS + H : TS;                // sites read
    constexpr int kIn = (36 * W + B - 1) / B, kOut = 36 * TS / B;
    static_assert(kOut * B == 36 * TS && TS % H == 0, "a tile splits evenly over the workgroup and into lines");
    __shared__ V tile[36][W + 1];
    const int64_t t = kGroup ? group_order(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    const int64_t s0 = t * TS, nin = n * 36;
    V v[kIn];
#pragma unroll
    for (int i = 0; i < kIn; ++i) {
        const int e = threadIdx.x + i * B;
        const int64_t g = s0 * 36 + e;
        if (36 * W % B == 0 || e < 36 * W)
            v[i] = ld_stream(src + (g < nin ? g : nin - 1));   // in bounds; unused past the end
    }
#pragma unroll
    for (int i = 0; i < kIn; ++i) {
        const int e = threadIdx.x + i * B;
        if (36 * W % B == 0 || e < 36 * W)
            tile[e % 36][e / 36] = v[i];
    }
    __syncthreads();
    // sites from s0 up to plane p's next line boundary
    const unsigned at = kHalo ? (unsigned)(((uintptr_t)dst / sizeof(V) + (uint64_t)s0) % H) : 0;
    const unsigned step = kHalo ? (unsigned)(pitch % H) : 0;
    auto shift = [=](int p) { return (int)((H - (at + (unsigned)p * step) % H) % H); };
    V o[kOut];
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int e = threadIdx.x + i * B, p = e / TS;
        o[i] = tile[p][e % TS + shift(p)];
    }
    const OutWindow out = out_window(dst, 36 * pitch * (int64_t)sizeof(V));   // kThrough: below 4 GiB
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int e = threadIdx.x + i * B, p = e / TS;
        const int64_t s = s0 + e % TS + shift(p);
        if constexpr (kThrough) {
            if (s < n)
                st_out<true>(out, ((uint32_t)p * (uint32_t)pitch + (uint32_t)s) * (uint32_t)sizeof(V), o[i]);
        } else if (s < n) {
            st_stream(dst + (int64_t)p * pitch + s, o[i]);
        }
    }
    if (kHalo && t == 0) {
        for (int e = threadIdx.x; e < 36 * H; e += B) {
            const int p = e / H, s = e % H;
            if (s < shift(p) && s < n)
                dst[(int64_t)p * pitch + s] = tile[p][s];
        }
    }
}

// kNt: nontemporal plane loads. Where planes do not start on lines, two
// workgroups read the line at a tile's edge, and FP32 keeps it in the cache.
// Write-through stores go with the grouped order here.
template <typename V, int TS, int B, bool kNt, bool kThrough>
__global__ __launch_bounds__(B) void to_aos_tile(const V *__restrict__ src, V *__restrict__ dst, int64_t n,
                                                 int64_t pitch)
{
    constexpr int kPer = 36 * TS / B;
    static_assert(kPer * B == 36 * TS, "a tile splits evenly over the workgroup");
    __shared__ V tile[36][TS + 1];
    const int64_t t = kThrough ? group_order(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    const int64_t s0 = t * TS, nout = n * 36;
    V v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = threadIdx.x + i * B;
        const int64_t s = s0 + e % TS;
        const V *q = src + (int64_t)(e / TS) * pitch + (s < n ? s : n - 1);   // in bounds; unused past the end
        v[i] = kNt ? ld_stream(q) : *q;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = threadIdx.x + i * B;
        tile[e / TS][e % TS] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = threadIdx.x + i * B;
        v[i] = tile[e % 36][e / 36];
    }
    const OutWindow out = out_window(dst + s0 * 36, (nout - s0 * 36) * (int64_t)sizeof(V));
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        st_out<kThrough>(out, (uint32_t)((threadIdx.x + i * B) * sizeof(V)), v[i]);
}

// FP32 with both sides in 16-byte accesses: two elements of a site on the
// site-major side, two sites of a plane on the plane side (every plane on a
// 128-byte boundary, so pairs of sites are 16-byte aligned). Half the
// memory instructions of 8-byte elements: 7.2 against 10.5 us at 65,536
// sites. Padding is neither read nor written.
template <int TS, int B>
__global__ __launch_bounds__(B) void to_soa_pairs(const f4 *__restrict__ src, f2 *__restrict__ dst, int64_t n,
                                                  int64_t pitch)
{
    constexpr int kPer = 18 * TS / B;
    static_assert(kPer * B == 18 * TS && TS % 2 == 0, "a tile splits evenly over the workgroup");
    __shared__ __attribute__((aligned(16))) f2 tile[36][TS + 2];   // even rows keep pairs aligned
    const int64_t s0 = (int64_t)blockIdx.x * TS, nin = n * 18;
    f4 v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int64_t g = s0 * 18 + threadIdx.x + i * B;
        v[i] = ld_stream(src + (g < nin ? g : nin - 1));   // in bounds; unused past the end
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = 2 * (threadIdx.x + i * B);
        tile[e % 36][e / 36] = f2{v[i].x, v[i].y};
        tile[e % 36 + 1][e / 36] = f2{v[i].z, v[i].w};
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = 2 * (threadIdx.x + i * B);
        v[i] = *reinterpret_cast<const f4 *>(&tile[e / TS][e % TS]);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = 2 * (threadIdx.x + i * B);
        const int64_t s = s0 + e % TS;
        f2 *q = dst + (int64_t)(e / TS) * pitch + s;
        if (s + 1 < n)
            st_stream(reinterpret_cast<f4 *>(q), v[i]);
        else if (s < n)
            *q = f2{v[i].x, v[i].y};
    }
}

template <int TS, int B>
__global__ __launch_bounds__(B) void to_aos_pairs(const f2 *__restrict__ src, f4 *__restrict__ dst, int64_t n,
                                                  int64_t pitch)
{
    constexpr int kPer = 18 * TS / B;
    static_assert(kPer * B == 18 * TS && TS % 2 == 0, "a tile splits evenly over the workgroup");
    __shared__ __attribute__((aligned(16))) f2 tile[36][TS + 2];
    const int64_t s0 = (int64_t)blockIdx.x * TS, nout = n * 18;
    f4 v[kPer];
    if (s0 + TS <= n) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = 2 * (threadIdx.x + i * B);
            v[i] = ld_stream(reinterpret_cast<const f4 *>(src + (int64_t)(e / TS) * pitch + s0 + e % TS));
        }
    } else {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = 2 * (threadIdx.x + i * B);
            const int64_t s = s0 + e % TS;
            const f2 *q = src + (int64_t)(e / TS) * pitch;
            const f2 x = q[s < n ? s : n - 1], y = q[s + 1 < n ? s + 1 : n - 1];
            v[i] = f4{x.x, x.y, y.x, y.y};
        }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = 2 * (threadIdx.x + i * B);
        *reinterpret_cast<f4 *>(&tile[e / TS][e % TS]) = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = 2 * (threadIdx.x + i * B);
        const f2 x = tile[e % 36][e / 36], y = tile[e % 36 + 1][e / 36];
        v[i] = f4{x.x, x.y, y.x, y.y};
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int64_t g = s0 * 18 + threadIdx.x + i * B;
        if (g < nout)
            st_stream(dst + g, v[i]);
    }
}

// ------------------------------------------------------------ pack
// FP64 complex -> FP32 complex, round to nearest even (v_cvt_f32_f64), one
// complex per thread: 16 bytes in, 8 out. Nontemporal loads and write-through
// stores: 6.97 against 6.49 TB/s with plain ones at 2^20 sites, 6.4 against
// 5.9 at 160,000. Small grids take them too, unlike the BF16 pack's: up to 8,192
// sites they are level (3.3 us), at 16,384 3.5 us against 3.9 over one and three
// inputs in turn and 4.0 against 3.9 over ten, at 32,768 5.4-6.1 against 6.0-6.6.
template <int B>
__global__ __launch_bounds__(B) void pack_f32(const d2 *__restrict__ src, f2 *__restrict__ dst, int64_t n)
{
    for (int64_t t = blockIdx.x; t * B < n; t += gridDim.x) {
        const int64_t e = t * B + threadIdx.x;
        const d2 v = ld_stream(src + (e < n ? e : n - 1));
        const f2 o = {(float)v.x, (float)v.y};
        st_out<true>(out_window(dst + t * B, 8 * (n - t * B)), 8 * threadIdx.x, o);
    }
}

// The BF16 conversions: a wavefront moves 64 chunks (16 bytes, 4 complex) of
// the BF16 side and the 4 KiB of FP64 they stand for, every access of it one
// whole 1 KiB run; a private LDS slice turns one chunk per lane into one
// complex per lane and back. With one or two complex per thread and no LDS
// the BF16 side moved as 4- or 8-byte words and the FP64 side in strides of
// 32 bytes: 2^20 sites took 124 (pack) and 126 us (unpack), now 113 and 116;
// 24^4 sites 42 and 45, now 37 and 38. The caps are from a sweep of 8 to 20
// wavefronts per CU, or none, at 49,152 to 2,560,000 sites; three or four
// chunks per lane, 256 threads and the XCD order were slower. Without kThrough
// the loads are cached: the input of a grid that is resident at once is small
// enough to be found in the caches, and nontemporal loads cost the pack of 16,384
// sites 15% there.
#ifndef SU3_WAVES_BF16_CONV
#define SU3_WAVES_BF16_CONV 14
#endif
constexpr int kPackBf16Block = 64, kUnpackBf16Block = 128;

// FP64 complex -> BF16 (re, im), through FP32, each step to nearest even.
template <bool kThrough>
__global__ __launch_bounds__(kPackBf16Block) void pack_bf16(const d2 *__restrict__ src, u4 *__restrict__ dst,
                                                            int64_t chunks)
{
    __shared__ u4 stage[kPackBf16Block];
    const int lane = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * kPackBf16Block, n = 4 * chunks;
    d2 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t g = 4 * c0 + 64 * i + lane;
        const d2 *p = src + (g < n ? g : n - 1);   // in bounds; dropped past the end
        v[i] = kThrough ? ld_stream(p) : *p;
    }
    uint32_t *words = reinterpret_cast<uint32_t *>(stage);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        words[64 * i + lane] = pack_bf16x2((float)v[i].x, (float)v[i].y);
    wave_sync();
    store_runs<kThrough, 1>(dst, stage, c0, lane, chunks);
}

// FP64 links -> rows 0 and 1 in FP32 (V = f2, round to nearest even) or FP64
// (V = d2), the reconstruct-12 storage. One wavefront per tile of 64 links:
// whole-wavefront 1 KiB runs of the tile's links (9 chunks each) in, the
// rows 0-1 of each (3 or 6 chunks) out, through a private LDS slice.
template <typename V, bool kThrough>
__global__ __launch_bounds__(64) void pack_r12(const u4 *__restrict__ src, u4 *__restrict__ dst, int64_t links)
{
    constexpr int kOut = sizeof(V) == 8 ? 3 : 6;   // output chunks per link
    __shared__ u4 stage[64 * 9];
    const int lane = threadIdx.x;
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t nin = links * 9, nout = links * kOut;
    u4 v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int64_t g = t * 64 * 9 + 64 * i + lane;
        v[i] = ld_stream(src + (g < nin ? g : nin - 1));   // in bounds; unused past the end
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
        stage[64 * i + lane] = v[i];
    wave_sync();
    typedef typename std::conditional<sizeof(V) == 8, float, double>::type E;   // element of V
    V o[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const d2 w = __builtin_bit_cast(d2, stage[9 * lane + q]);
        o[q] = V{(E)w.x, (E)w.y};
    }
    wave_sync();
    V *out = reinterpret_cast<V *>(stage) + 6 * lane;
#pragma unroll
    for (int q = 0; q < 6; ++q)
        out[q] = o[q];
    wave_sync();
    if constexpr (kThrough)
        store_runs<true, kOut>(dst, stage, t * 64 * kOut, lane, nout);
    else
        store_each<kOut>(dst, stage, t * 64 * kOut, lane, nout);
}

// ------------------------------------------------------------ unpack
// FP32 complex -> FP64, exact, one complex per thread; nontemporal loads and
// stores: 6.70 against 6.47 TB/s with plain ones at 2^20 sites, level up to 16,384
// (3.4 us at 8,192, 4.4 at 16,384), 6.4-6.8 us against 6.9-7.7 at 32,768. Only one
// input unpacked again and again at 200,000 to 280,000 sites loses (1-2.5%).
template <int B>
__global__ __launch_bounds__(B) void unpack_f32(const f2 *__restrict__ src, d2 *__restrict__ dst, int64_t n)
{
    for (int64_t e = (int64_t)blockIdx.x * B + threadIdx.x; e < n; e += (int64_t)gridDim.x * B) {
        const f2 v = ld_stream(src + e);
        const d2 o = {(double)v.x, (double)v.y};
        st_stream(dst + e, o);
    }
}

// BF16 -> FP64, exact.
template <bool kThrough>
__global__ __launch_bounds__(kUnpackBf16Block) void unpack_bf16(const u4 *__restrict__ src, d2 *__restrict__ dst,
                                                                int64_t chunks)
{
    __shared__ u4 stage[kUnpackBf16Block];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * kUnpackBf16Block + 64 * wave, n = 4 * chunks;
    u4 *my = stage + 64 * wave;
    const u4 *p = src + (c0 + lane < chunks ? c0 + lane : chunks - 1);   // in bounds; dropped past the end
    my[lane] = kThrough ? ld_stream(p) : *p;
    wave_sync();
    const uint32_t *words = reinterpret_cast<const uint32_t *>(my);
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = words[64 * i + lane];
    const OutWindow out = out_window(dst + 4 * c0, 16 * (n - 4 * c0));
#pragma unroll
    for (int i = 0; i < 4; ++i)
        st_out<kThrough>(out, 16 * (64 * i + lane), d2{(double)bf16_lo(w[i]), (double)bf16_hi(w[i])});
}

// Rows 0-1 (FP32 or FP64) -> full FP64 link; row 2 = conj(row0 x row1) evaluated in
// FP64 without contraction, each product and difference rounded on its own,
// in the order (r0_p r1_q) - (r0_q r1_p) with each complex product formed as
// (re*re - im*im, re*im + im*re). The result is then a fixed function of the
// stored rows, independent of compiler contraction choices.
// One wavefront per tile of 64 links, the streaming pattern of the product
// kernels: the tile's rows 0-1 (3 chunks per link in FP32, 6 in FP64) and its
// full FP64 links (9 chunks each) move in whole-wavefront 1 KiB runs, and a
// private LDS slice turns them into one link per lane. Row 2 is rebuilt in
// FP64 with contraction off, in the oracle's operation order, so the result
// is bit-exact.
template <typename V, bool kThrough>
__global__ __launch_bounds__(64) void unpack_r12(const u4 *__restrict__ src, u4 *__restrict__ dst, int64_t links)
{
#pragma clang fp contract(off)
    constexpr int kIn = sizeof(V) == 8 ? 3 : 6;   // input chunks per link
    __shared__ u4 stage[64 * 9];
    const int lane = threadIdx.x;
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t nin = links * kIn, nout = links * 9;
    u4 v[kIn];
#pragma unroll
    for (int i = 0; i < kIn; ++i) {
        const int64_t g = t * 64 * kIn + 64 * i + lane;
        v[i] = ld_stream(src + (g < nin ? g : nin - 1));   // in bounds; unused past the end
    }
#pragma unroll
    for (int i = 0; i < kIn; ++i)
        stage[64 * i + lane] = v[i];
    wave_sync();
    double r[12];
    const V *in = reinterpret_cast<const V *>(stage) + 6 * lane;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const V w = in[q];
        r[2 * q] = (double)w.x;
        r[2 * q + 1] = (double)w.y;
    }
    d2 o[9];
#pragma unroll
    for (int q = 0; q < 6; ++q)
        o[q] = d2{r[2 * q], r[2 * q + 1]};
    const double *r0 = r, *r1 = r + 6;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const int p = (l + 1) % 3, q = (l + 2) % 3;
        const double pr = r0[2 * p] * r1[2 * q] - r0[2 * p + 1] * r1[2 * q + 1];
        const double pi = r0[2 * p] * r1[2 * q + 1] + r0[2 * p + 1] * r1[2 * q];
        const double qr = r0[2 * q] * r1[2 * p] - r0[2 * q + 1] * r1[2 * p + 1];
        const double qi = r0[2 * q] * r1[2 * p + 1] + r0[2 * q + 1] * r1[2 * p];
        o[6 + l] = d2{pr - qr, -(pi - qi)};
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < 9; ++q)
        stage[9 * lane + q] = __builtin_bit_cast(u4, o[q]);
    wave_sync();
    store_runs<kThrough, 9>(dst, stage, t * 64 * 9, lane, nout);
}

// ------------------------------------------------------------ stream copy
// dst[i] = src[i] over 16-byte elements, one element per thread, with
// nontemporal loads; the grid covers the buffer once, so the dispatcher streams
// it in address order. Workgroups of one wavefront. Stores write through
// (kThrough), or are nontemporal where the grid is at most 24 wavefronts per CU,
// all resident at once.
// Write-through against nontemporal, 576 B FP64 sites: 20,000 4.6 / 4.9 us,
// 65,536 11.9 / 12.5, 663,552 112.6 / 114.5, 4,200,000 713 / 718 (6.79 TB/s). At
// most 24 wavefronts per CU above 600 MB: 1% faster there, 2-6% slower below.
// 2, 3 or 4 elements per thread, capped or not, and tiles in XCD order were 0
// to 15% slower.
constexpr int kCopyBlock = 64;
constexpr int kCopyWaves = 24;
constexpr int64_t kCopyCapBytes = 600000000;

template <bool kThrough>
__global__ __launch_bounds__(kCopyBlock) void stream_copy(const u4 *__restrict__ src, u4 *__restrict__ dst, int64_t n)
{
    const int64_t base = (int64_t)blockIdx.x * kCopyBlock, i = base + threadIdx.x;
    if constexpr (kThrough) {
        const OutWindow out = out_window(dst + base, 16 * kCopyBlock);
        if (i < n)
            st_out<true>(out, 16 * threadIdx.x, ld_stream(src + i));
    } else if (i < n) {
        st_stream(dst + i, ld_stream(src + i));
    }
}

// Access-shape probe: wavefront w (the workgroup index, or with order 1 its
// XCD-contiguous tile, xcd_order) reads chunks w*64*RA + 64 i + lane of a
// (i < RA) and likewise of b, and writes chunks w*64*W + 64 i + lane of c,
// the same whole-wavefront 1 KiB runs and per-lane chunk counts as the
// kernels it stands beside and their write-through stores, with no arithmetic
// beyond folding the loads into the stored values (so that no load is dead).
template <int RA, int RB, int W>
__global__ __launch_bounds__(64) void stream_shape(const u4 *__restrict__ a, const u4 *__restrict__ b,
                                                   u4 *__restrict__ c, int order)
{
    const int64_t w = order ? xcd_order(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    const int lane = threadIdx.x;
    u4 va[RA], vb[RB > 0 ? RB : 1];
#pragma unroll
    for (int i = 0; i < RA; ++i)
        va[i] = ld_stream(a + w * 64 * RA + 64 * i + lane);
#pragma unroll
    for (int i = 0; i < RB; ++i)
        vb[i] = ld_stream(b + w * 64 * RB + 64 * i + lane);
    const OutWindow out = out_window(c + w * 64 * W, 16 * 64 * W);
    u4 x = va[0];
#pragma unroll
    for (int i = 1; i < RA; ++i)
        x ^= va[i];
#pragma unroll
    for (int i = 0; i < RB; ++i)
        x ^= vb[i];
#pragma unroll
    for (int i = 0; i < W; ++i) {
        u4 o = x;
        o.x += (uint32_t)i;
        st_out<true>(out, 16 * (64 * i + lane), o);
    }
}

// ------------------------------------------------------------ launchers
static unsigned grid_for(int64_t items, int64_t per_block, int64_t cap = kOnePass)
{
    int64_t g = (items + per_block - 1) / per_block;
    if (g > cap)
        g = cap;
    if (g < 1)
        g = 1;
    return (unsigned)g;
}

// K on tiles of TS sites, one workgroup of B threads each, at most kPerCU
// workgroups resident per CU (0: as many as fit).
template <auto K, int TS, int B, int kPerCU, typename VS, typename VD>
static hipError_t launch_tiles(const VS *src, VD *dst, int64_t n, int64_t pitch, hipStream_t s)
{
    static PadCache cache;
    const int64_t grid = (n + TS - 1) / TS;
    const LaunchPlan plan = launch_plan(reinterpret_cast<const void *>(K), kPerCU * (B / 64), B, grid, cache);
    return launch_k(K, dim3((unsigned)grid), dim3(B), s, plan.pad, src, dst, n, pitch);
}
template <typename V, int TS, int B, bool kHalo, bool kThrough, bool kGroup, int kPerCU>
static hipError_t launch_to_soa(const void *src, void *dst, int64_t n, int64_t pitch, hipStream_t s)
{
    return launch_tiles<to_soa_tile<V, TS, B, kHalo, kThrough, kGroup>, TS, B, kPerCU>((const V *)src, (V *)dst, n,
                                                                                      pitch, s);
}
template <typename V, int TS, int B, bool kNt, bool kThrough, int kPerCU>
static hipError_t launch_to_aos(const void *src, void *dst, int64_t n, int64_t pitch, hipStream_t s)
{
    return launch_tiles<to_aos_tile<V, TS, B, kNt, kThrough>, TS, B, kPerCU>((const V *)src, (V *)dst, n, pitch, s);
}
// The general path: any size, a grid of 64-site tiles that loops past kOnePass.
template <typename V, bool kXcd>
static hipError_t launch_general(const void *src, void *dst, int64_t n, int64_t pitch, bool to_soa, hipStream_t s)
{
    const dim3 g(grid_for(n, kTileSites));
    if (to_soa)
        return launch_k(transpose_aos_soa<V, true, kXcd>, g, dim3(kBlock), s, 0, (const V *)src, (V *)dst, n, pitch);
    return launch_k(transpose_aos_soa<V, false, kXcd>, g, dim3(kBlock), s, 0, (const V *)src, (V *)dst, n, pitch);
}

// Which transpose serves which lattice (microseconds, this path / the general
// one, on random data in rotating buffers). `lines`: every plane starts on a
// 128-byte line.
//  FP64, up to 49,152 sites: the general path; its 64-site tiles give more CUs
//    work than larger ones, and its XCD order collides less at 2^15 sites.
//  FP64 to planes, on lines: up to 65,536 sites 128-site tiles, the whole grid
//    resident at two per CU (65,536: 13.3 / 15.6); above, 32-site tiles: up to
//    262,144 sites 384 threads, three per CU, write-through (81,920: 17.0,
//    160,000: 30.4, 230,400: 46.8; 1.00 to 1.17 times the next form at 8
//    sizes, dense and padded), beyond that 576 threads, nontemporal (24^4: 64 /
//    78; the form before it is level there and 5% slower at 2^20), and above
//    1,100,000 sites grouped and write-through (40^4: 490 / 565, 48^4: 1018 /
//    1150; against nontemporal in order 0.98 at 2^21 padded and 1.01 to 1.07
//    elsewhere, 2^20 * 9/8 to 2^22 * 5/4 sites, 2^22 padded 1.05 among them: no
//    line by the plane stride follows; 0.91 to 1.0 at 262,656 to 663,552
//    sites). Off lines, 128-site tiles with the
//    halo, two per CU up to 131,072 sites (65,537: 13.5 / 15.9) and one
//    above (31^4: 193 / 250, 2,560,001: 533 / 630).
//  FP64 from planes, on lines: up to 65,536 sites as above; beyond, 32-site
//    tiles of 384 threads, three per CU, grouped and write-through (160,000:
//    30.1 / 35.2, 24^4: 60.4 / 72, 40^4: 472 / 523). Against 128-site tiles in
//    order with nontemporal stores, the former choice there: 1.02 to 1.15 at
//    14 sizes, dense and padded, and 0.97 at one (230,400 padded). Off lines
//    the general path up to 196,608 sites and 128-site tiles above, one per CU,
//    also grouped and write-through (31^4: 175 / 208; 0.99 to 1.10 times
//    the tiles in order at 7 sizes).
//  FP32 on lines: pairs on 64-site tiles of 128 threads up to 131,072 sites
//    (65,536: 7.2 / 10.5). Above, to planes, single elements on 64-site tiles
//    of 256 threads, three per CU, write-through, up to 400,000 sites (230,400:
//    24.9, 24^4: 32.6; 0.98 to 1.25 times the next form) and pairs on 64-site
//    tiles of 576 threads beyond (40^4: 234 / 257, 48^4: 516 / 558; the form
//    before it is level there and 3% slower at 2^20 and 2^21). From planes,
//    64-site tiles of 768 threads, grouped and write-through (160,000: 17.4,
//    24^4: 32.4, 1,736,096: 157 / 159, 40^4: 232 / 250), except between 500,000 and
//    1,450,000 sites (144 MB, where conversions stop to write through, and 418 MB
//    of output): there the general path is on the whole faster (520,000: 49.0 /
//    48.8, 700,000: 68.6 / 67.5, 900,000: 85.2 / 83.7, 1,400,000: 126.8 / 123.9;
//    1,200,000: 110 / 111, 1,500,000 padded: 140 / 147), and the same tiles with
//    nontemporal stores are 0-5% slower than it. Where a dense plane stride lies
//    within 128 KiB of a multiple of 4 MiB its planes collide, and the tiles stay
//    (2^20: 98 / 105).
//  FP32 off lines: up to 49,152 sites the general path; above, 128-site tiles
//    of 256 threads, to planes with the halo, two per CU (65,537: 9.3 / 10.7,
//    31^4: 105 / 142, 2,560,001: 266 / 381), from planes with cached loads
//    (65,537: 8.6 / 11.1, 31^4: 94 / 105, 2,560,001: 251 / 280).
//  Write-through stores to planes take 32-bit offsets from the first plane, so
//    those forms need all planes within 4 GiB: pitches of at most 7 * 2^20
//    (longer ones, far beyond those sizes, take the nontemporal form).
//  Over 2^27 sites, where a one-pass grid could pass 2^32 threads: the general
//    path, which loops.
hipError_t launch_aos_soa(const void *src, void *dst, int64_t sites, int64_t pitch, int elem_bytes, bool to_soa,
                          hipStream_t s)
{
    const int64_t n = sites;
    const bool lines = pitch * elem_bytes % 128 == 0 && (uintptr_t)(to_soa ? dst : src) % 128 == 0;
    const bool huge = n > (int64_t)1 << 27, window = pitch <= (int64_t)7 << 20;
    if (elem_bytes == 16) {
        if (n <= 49152 || huge || (!to_soa && !lines && n <= 196608))
            return launch_general<d2, true>(src, dst, n, pitch, to_soa, s);
        if (to_soa && !lines)
            return n <= 131072 ? launch_to_soa<d2, 128, 768, true, false, false, 0>(src, dst, n, pitch, s)
                               : launch_to_soa<d2, 128, 768, true, false, false, 1>(src, dst, n, pitch, s);
        if (to_soa)
            return n <= 65536               ? launch_to_soa<d2, 128, 768, false, false, false, 0>(src, dst, n, pitch, s)
                   : n <= 262144 && window  ? launch_to_soa<d2, 32, 384, false, true, false, 3>(src, dst, n, pitch, s)
                   : n <= 1100000 || !window ? launch_to_soa<d2, 32, 576, false, false, false, 0>(src, dst, n, pitch, s)
                                            : launch_to_soa<d2, 32, 576, false, true, true, 3>(src, dst, n, pitch, s);
        return n <= 65536 ? launch_to_aos<d2, 128, 768, true, false, 0>(src, dst, n, pitch, s)
               : lines    ? launch_to_aos<d2, 32, 384, true, true, 3>(src, dst, n, pitch, s)
                          : launch_to_aos<d2, 128, 768, true, true, 1>(src, dst, n, pitch, s);
    }
    if (huge || (!lines && n <= 49152))
        return launch_general<f2, false>(src, dst, n, pitch, to_soa, s);
    if (!lines)
        return to_soa ? launch_to_soa<f2, 128, 256, true, false, false, 2>(src, dst, n, pitch, s)
                      : launch_to_aos<f2, 128, 256, false, false, 0>(src, dst, n, pitch, s);
    if (n <= 131072)
        return to_soa ? launch_tiles<to_soa_pairs<64, 128>, 64, 128, 0>((const f4 *)src, (f2 *)dst, n, pitch, s)
                      : launch_tiles<to_aos_pairs<64, 128>, 64, 128, 0>((const f2 *)src, (f4 *)dst, n, pitch, s);
    if (!to_soa) {
        const int64_t m = pitch * 8 % ((int64_t)4 << 20), near = (int64_t)128 << 10;
        const bool collide = pitch == n && (m < near || m > ((int64_t)4 << 20) - near);
        return n * 288 <= kFitConversion || n > 1450000 || collide
                   ? launch_to_aos<f2, 64, 768, true, true, 0>(src, dst, n, pitch, s)
                   : launch_general<f2, false>(src, dst, n, pitch, to_soa, s);
    }
    return n <= 400000 && window ? launch_to_soa<f2, 64, 256, false, true, false, 3>(src, dst, n, pitch, s)
                                 : launch_tiles<to_soa_pairs<64, 576>, 64, 576, 0>((const f4 *)src, (f2 *)dst, n, pitch, s);
}

hipError_t launch_stream_copy(const void *src, void *dst, int64_t bytes, hipStream_t s)
{
    const int64_t n = bytes / 16;
    const int64_t grid = (n + kCopyBlock - 1) / kCopyBlock;
    static PadCache cache;
    size_t pad = 0;
    if (2 * bytes > kCopyCapBytes)
        pad = launch_plan(reinterpret_cast<const void *>(stream_copy<true>), kCopyWaves, kCopyBlock, grid, cache).pad;
    return launch_k(grid <= kCopyWaves * kCUs ? stream_copy<false> : stream_copy<true>, dim3((unsigned)grid),
                    dim3(kCopyBlock), s, pad, (const u4 *)src, (u4 *)dst, n);
}

bool stream_shape_supported(int in_a, int in_b, int out)
{
    return (in_a == 1 && in_b == 0 && out == 1) || (in_a == 3 && in_b == 0 && out == 3) ||
           (in_a == 3 && in_b == 3 && out == 3) || (in_a == 6 && in_b == 0 && out == 9) ||
           (in_a == 9 && in_b == 0 && out == 9);
}

template <int RA, int RB, int W>
static hipError_t launch_shape_k(const void *a, const void *b, void *c, int64_t tiles, int waves, int order,
                                 hipStream_t s)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return hipErrorInvalidDevice;
    const size_t pad = occupancy_pad_for(reinterpret_cast<const void *>(stream_shape<RA, RB, W>), waves, 64, dev);
    return launch_k(stream_shape<RA, RB, W>, dim3((unsigned)tiles), dim3(64), s, pad, (const u4 *)a, (const u4 *)b,
                    (u4 *)c, order);
}

hipError_t launch_stream_shape(const void *a, const void *b, void *c, int64_t tiles, int in_a, int in_b, int out,
                               int waves_per_cu, int tile_order, hipStream_t s)
{
    if (in_a == 1 && in_b == 0 && out == 1)
        return launch_shape_k<1, 0, 1>(a, b, c, tiles, waves_per_cu, tile_order, s);
    if (in_a == 3 && in_b == 0 && out == 3)
        return launch_shape_k<3, 0, 3>(a, b, c, tiles, waves_per_cu, tile_order, s);
    if (in_a == 3 && in_b == 3 && out == 3)
        return launch_shape_k<3, 3, 3>(a, b, c, tiles, waves_per_cu, tile_order, s);
    if (in_a == 6 && in_b == 0 && out == 9)
        return launch_shape_k<6, 0, 9>(a, b, c, tiles, waves_per_cu, tile_order, s);
    if (in_a == 9 && in_b == 0 && out == 9)
        return launch_shape_k<9, 0, 9>(a, b, c, tiles, waves_per_cu, tile_order, s);
    return hipErrorInvalidValue;
}

template <typename V>
static hipError_t launch_pack_r12(const void *src, void *dst, int64_t links, hipStream_t s)
{
    static PadCache cache[3];
    const int64_t grid = (links + 63) / 64, bytes = links * (144 + 6 * (int)sizeof(V));
    const LaunchPlan plan =
        launch_plan(reinterpret_cast<const void *>(pack_r12<V, true>), sizeof(V) == 8 ? kPackR12F32 : kPackR12F64,
                    bytes, 64, grid, cache);
    // FP32 rows, a third of the bytes read, do not gain again past the cache (290
    // MB written 0.98, 1 GB 0.99)
    const bool through = write_through(plan, links * (6 * (int)sizeof(V)), kFitConversion,
                                       sizeof(V) == 8 ? INT64_MAX : kThroughAgain);
    return launch_k(through ? pack_r12<V, true> : pack_r12<V, false>, dim3((unsigned)grid), dim3(64), s,
                    plan.pad, (const u4 *)src, (u4 *)dst, links);
}

template <typename V>
static hipError_t launch_unpack_r12(const void *src, void *dst, int64_t links, hipStream_t s)
{
    static PadCache cache[3];
    const int64_t grid = (links + 63) / 64;
    const LaunchPlan plan =
        launch_plan(reinterpret_cast<const void *>(unpack_r12<V, true>), sizeof(V) == 8 ? kUnpackR12F32 : kUnpackR12F64,
                    links * (144 + 6 * (int)sizeof(V)), 64, grid, cache);
    // a quarter (FP32 rows) and two fifths of the traffic are read: the first line
    // lies a little higher than the pack's (150 MB written 1.05-1.08 and 1.00-1.05,
    // 160 MB 1.02-1.09 and 0.97-1.01), the second where FP32 rows stop to lose when
    // one input is unpacked again and again (450 MB 0.99, 750 MB 1.00)
    const bool through =
        write_through(plan, links * 144, kFitUnpackR12, sizeof(V) == 8 ? kThroughAgainUnpackR12 : kThroughAgain);
    return launch_k(through ? unpack_r12<V, true> : unpack_r12<V, false>, dim3((unsigned)grid), dim3(64), s, plan.pad,
                    (const u4 *)src, (u4 *)dst, links);
}

// The BF16 conversions of `chunks` 16-byte chunks of the BF16 side (9 per
// site), in launches of at most 2^31 threads: one for any lattice of up to 238
// million sites (a loop inside the pack cost it 7%).
constexpr int64_t kBf16Chunks = (int64_t)1 << 31;

static hipError_t launch_pack_bf16(const d2 *src, u4 *dst, int64_t chunks, hipStream_t s)
{
    static PadCache cache;
    hipError_t e = hipSuccess;
    for (int64_t c = 0; c < chunks && e == hipSuccess; c += kBf16Chunks) {
        const int64_t m = chunks - c < kBf16Chunks ? chunks - c : kBf16Chunks;
        const int64_t grid = (m + kPackBf16Block - 1) / kPackBf16Block;
        const LaunchPlan plan = launch_plan(reinterpret_cast<const void *>(pack_bf16<true>), SU3_WAVES_BF16_CONV,
                                            kPackBf16Block, grid, cache);
        e = launch_k(plan.one_generation ? pack_bf16<false> : pack_bf16<true>, dim3((unsigned)grid),
                     dim3(kPackBf16Block), s, plan.pad, src + 4 * c, dst + c, m);
    }
    return e;
}

static hipError_t launch_unpack_bf16(const u4 *src, d2 *dst, int64_t chunks, hipStream_t s)
{
    static PadCache cache;
    hipError_t e = hipSuccess;
    for (int64_t c = 0; c < chunks && e == hipSuccess; c += kBf16Chunks) {
        const int64_t m = chunks - c < kBf16Chunks ? chunks - c : kBf16Chunks;
        const int64_t grid = (m + kUnpackBf16Block - 1) / kUnpackBf16Block;
        const LaunchPlan plan = launch_plan(reinterpret_cast<const void *>(unpack_bf16<true>), SU3_WAVES_BF16_CONV,
                                            kUnpackBf16Block, grid, cache);
        // cached loads and nontemporal stores between the lines too: 160 MB written
        // 1.04-1.06 and 1.37 times the plain kernel's speed with one and three inputs
        // in turn, where write-through gives 0.97 and 1.22
        const bool through = write_through(plan, m * 64, kFitConversion);
        e = launch_k(through ? unpack_bf16<true> : unpack_bf16<false>, dim3((unsigned)grid),
                     dim3(kUnpackBf16Block), s, plan.pad, src + c, dst + 4 * c, m);
    }
    return e;
}

// precision codes as in su3.h: 0 F64, 1 F32, 2 BF16, 3 R12_F32 (rows 0-1 FP32
// in, full FP32 out), 4 R12C_F32 (rows 0-1 FP32 in and out), 5 R12_F64 (rows
// 0-1 FP64 in, full FP64 out). Codes 3 and 4 share the storage of a.
hipError_t launch_pack(const void *src, void *dst, int64_t sites, int precision, hipStream_t s)
{
    const int64_t elems = sites * 36, links = sites * 4;
    switch (precision) {
    case 1:
        return launch_k(pack_f32<64>, dim3(grid_for(elems, 64, kOnePass)), dim3(64), s, 0, (const d2 *)src,
                        (f2 *)dst, elems);
    case 2:
        return launch_pack_bf16((const d2 *)src, (u4 *)dst, elems / 4, s);
    case 3:
    case 4:
        return launch_pack_r12<f2>(src, dst, links, s);
    case 5:
        return launch_pack_r12<d2>(src, dst, links, s);
    default:
        return launch_stream_copy(src, dst, elems * 16, s);
    }
}

hipError_t launch_unpack(const void *src, void *dst, int64_t sites, int precision, hipStream_t s)
{
    const int64_t elems = sites * 36, links = sites * 4;
    switch (precision) {
    case 1:
        return launch_k(unpack_f32<64>, dim3(grid_for(elems, 64, kOnePass)), dim3(64), s, 0, (const f2 *)src, (d2 *)dst,
                        elems);
    case 2:
        return launch_unpack_bf16((const u4 *)src, (d2 *)dst, elems / 4, s);
    case 3:
    case 4:
        return launch_unpack_r12<f2>(src, dst, links, s);
    case 5:
        return launch_unpack_r12<d2>(src, dst, links, s);
    default:
        return launch_stream_copy(src, dst, elems * 16, s);
    }
}

} // namespace su3
