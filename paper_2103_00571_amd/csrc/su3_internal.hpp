// su3_internal.hpp -- device helpers and launcher declarations shared by the
// kernel files of libsu3 (gfx950). Not part of the public ABI (include/su3.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <tuple>

namespace su3 {

// 16-byte vector types as clang ext vectors, so that __builtin_nontemporal_*
// accept them and the compiler emits one global_load/store_dwordx4 each.
typedef double d2 __attribute__((ext_vector_type(2)));   // one complex double
typedef float f4 __attribute__((ext_vector_type(4)));    // two complex float
typedef float f2 __attribute__((ext_vector_type(2)));    // one complex float
typedef uint32_t u4 __attribute__((ext_vector_type(4))); // eight bf16
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// Streaming accesses: a and c are touched once per call, so loads and stores
// carry the nontemporal hint (global_load/store ... nt) and do not displace
// the b links or other data from the caches.
template <typename T>
__device__ __forceinline__ T ld_stream(const T *p) { return __builtin_nontemporal_load(p); }
template <typename T>
__device__ __forceinline__ void st_stream(T *p, T v) { __builtin_nontemporal_store(v, p); }

// complex multiply-accumulate acc += x * y, four fused multiply-adds
__device__ __forceinline__ void cmac(double &re, double &im, double xr, double xi, double yr, double yi)
{
    re = __builtin_fma(xr, yr, re);
    re = __builtin_fma(-xi, yi, re);
    im = __builtin_fma(xr, yi, im);
    im = __builtin_fma(xi, yr, im);
}
__device__ __forceinline__ void cmac(float &re, float &im, float xr, float xi, float yr, float yi)
{
    re = __builtin_fmaf(xr, yr, re);
    re = __builtin_fmaf(-xi, yi, re);
    im = __builtin_fmaf(xr, yi, im);
    im = __builtin_fmaf(xi, yr, im);
}

// BF16 <-> FP32. Widening is a shift; narrowing rounds to nearest even
// (v_cvt_pk_bf16_f32 on gfx950 under the default rounding mode).
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    f2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2));
}

// Order LDS traffic between the lanes of one wavefront (LDS operations of a
// wavefront execute in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// XCD-contiguous tile order of a one-pass grid of nb workgroups. The
// dispatcher deals workgroups round-robin to MI355X's 8 XCDs (workgroup i to
// XCD i mod 8); here the k-th workgroup of XCD x takes tile
// x*q + min(x, r) + k (q = nb / 8, r = nb mod 8), so each XCD streams one
// contiguous eighth of the buffers in address order instead of every eighth
// tile. A bijection on [0, nb) for any nb: XCD x owns q tiles, plus one if
// x < r. The 8 is the XCD count of one device in the single-partition mode;
// under another partitioning the order is still a bijection, so results do
// not change, only the streaming rate may.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_order(int64_t bid, int64_t nb)
{
    const int64_t q = nb / kXcds, r = nb % kXcds, x = bid % kXcds;
    return x * q + (x < r ? x : r) + bid / kXcds;
}

// Grouped tile order: within every 8 * kGroup tiles each XCD takes kGroup
// consecutive ones, so that its runs join up while the whole grid still walks
// the array in order. A bijection on [0, nb): the tail of less than 8 * kGroup
// keeps the index.
template <int kGroup = 8>
__device__ __forceinline__ int64_t group_order(int64_t bid, int64_t nb)
{
    constexpr int kSpan = kXcds * kGroup;
    const int64_t k = bid / kSpan;
    const int r = (int)(bid - k * kSpan);
    return (k + 1) * kSpan > nb ? bid : k * kSpan + r % kXcds * kGroup + r / kXcds;
}

// The tile of this workgroup in the site-major products, the matrix-vector
// product and the reconstruct-12 pack and unpack: XCD-contiguous (at L = 48
// it streams 3-5% faster than tile = workgroup index at the best cap of
// each). SU3_XCD_ORDER 0 restores tile = workgroup index.
#ifndef SU3_XCD_ORDER
#define SU3_XCD_ORDER 1
#endif
__device__ __forceinline__ int64_t xcd_tile(int64_t bid, int64_t nb)
{
    return SU3_XCD_ORDER ? xcd_order(bid, nb) : bid;
}

// Output stores of the streaming kernels go through a buffer resource over a
// window of the output: its base is wave-uniform (scalar registers), a lane
// adds a 32-bit byte offset, and the hardware drops stores at or past the
// window's end, so ragged tiles need no branches. The resource also lets the
// kernel choose the cache policy (kThrough):
//  * write-through to memory (sc1), for grids of more than one generation.
//    Nothing reads the output back, and dirty lines left in the 8 L2s only
//    have to be evicted later, between other reads. Against nontemporal stores
//    (L2 write-back), L = 48: FP64 936 -> 917 us, FP32 470 -> 462, BF16 237 -> 235,
//    reconstruct-12 403 -> 395, a^H b FP64 968 -> 957. Mid-sized lattices
//    gain more, as their outputs stay in the Infinity Cache: over three and
//    over ten buffers, FP64 at 98,304 sites 1.13x and 1.05x, FP32 at 24^4 1.11x
//    and 1.05x, BF16 at 663,552 sites 1.17x and 1.04x.
//  * nontemporal otherwise: a grid that is resident at once would end with
//    the write-through of its whole output, and cold outputs of 9 MB (BF16 at
//    65,536 sites over 24 buffers) took 5.2 instead of 4.5 us.
// The policy is a template parameter, not an argument: with both sets of
// stores in one kernel the smallest grids were up to 15% slower.
struct OutWindow {
    __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ OutWindow out_window(void *base, int64_t bytes)
{
    const uint64_t p = (uint64_t)base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    const int64_t most = 0xfffffff0;
    const uint32_t size =
        __builtin_amdgcn_readfirstlane((uint32_t)(bytes < 0 ? 0 : bytes < most ? bytes : most));
    // word 3: 32-bit data format, no swizzle
    return {__builtin_amdgcn_make_buffer_rsrc((void *)((uint64_t)hi << 32 | lo), 0, size, 0x00020000)};
}
// Store the 8 or 16 bytes of v at byte `off` of the window.
template <bool kThrough, typename T>
__device__ __forceinline__ void st_out(const OutWindow &w, uint32_t off, T v)
{
    constexpr int kPolicy = kThrough ? 16 : 2;   // cache policy bits of buffer stores: sc1, nt
    static_assert(sizeof(T) == 8 || sizeof(T) == 16, "one store");
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), w.r, off, 0, kPolicy);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), w.r, off, 0, kPolicy);
}

// Store N whole-wavefront runs from a wavefront's LDS slice: chunk 64 i + lane
// (i < N) of the tile that starts at chunk `base` (wave-uniform) of dst;
// chunks at or past n are dropped. Every LDS read is issued before the first
// store, so the wavefront waits for LDS once.
template <bool kThrough, int N>
__device__ __forceinline__ void store_runs(u4 *__restrict__ dst, const u4 *slice, int64_t base, int lane, int64_t n)
{
    u4 w[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        w[i] = slice[64 * i + lane];
    const int64_t left = n - base;
    const OutWindow out = out_window(dst + base, 16 * (left < 64 * N ? left : 64 * N));
#pragma unroll
    for (int i = 0; i < N; ++i)
        st_out<kThrough>(out, 16 * (64 * i + lane), w[i]);
}

// The same with nontemporal stores to global addresses, one by one as their LDS
// reads arrive: 1-2% faster than store_runs with nontemporal stores in the
// matrix-vector product (750,000 sites FP64 96.9 us against 98.7) and in the
// reconstruct-12 pack (FP32 1,041,664 sites 0.99-1.0 against 0.98 of the
// speed without buffer resources); the products and the unpack are 0-2% slower.
template <int N>
__device__ __forceinline__ void store_each(u4 *__restrict__ dst, const u4 *slice, int64_t base, int lane, int64_t n)
{
    const bool whole = base + 64 * N <= n;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (whole || base + 64 * i + lane < n)
            st_stream(dst + base + 64 * i + lane, slice[64 * i + lane]);
}

// Threads per workgroup of the streaming kernels: four wave64s.
constexpr int kBlock = 256;

// Compute units of an MI355X.
constexpr int kCUs = 256;

// Devices per process for the per-device caches.
constexpr int kMaxDevices = 64;

// Launch a kernel through hipLaunchKernel, which reports a failed launch in
// its return value; each argument is converted to the kernel's parameter type.
// dyn_lds is the dynamic LDS size in bytes.
template <typename... KArgs, typename... Args>
inline hipError_t launch_k(void (*k)(KArgs...), dim3 grid, dim3 block, hipStream_t s, size_t dyn_lds, Args... args)
{
    static_assert(sizeof...(KArgs) == sizeof...(Args), "argument count");
    struct Pack {
        std::tuple<KArgs...> t;
    };
    Pack p{std::tuple<KArgs...>(static_cast<KArgs>(args)...)};
    void *argv[sizeof...(KArgs)];
    std::apply([&](auto &...e) {
        int i = 0;
        ((argv[i++] = (void *)&e), ...);
    }, p.t);
    return hipLaunchKernel(reinterpret_cast<const void *>(k), grid, block, argv, dyn_lds, s);
}

// Per-kernel, per-device launch facts, looked up on the first call (0: not
// yet): the dynamic LDS that enforces the occupancy cap, plus 1, in the low
// 32 bits and the workgroups one CU holds without it, of at most 24
// wavefronts, in the high 32.
typedef std::atomic<int64_t> PadCache[kMaxDevices];
// How to launch a streaming kernel: the dynamic LDS to add to each workgroup
// so that at most `waves` wavefronts are resident per CU (0 for no cap), and
// whether the whole grid is resident at once without a cap. The caps keep the
// bytes in flight at the rate's peak while workgroup follows workgroup; a grid
// that is resident at once has nothing to follow it, and a cap would only
// hold part of it back for a second generation. Uncapped against capped, at
// 65,536 sites: reconstruct-12 5.8 against 8.6 us, a^H b FP32 6.7 against 9.1;
// at 32,768 sites: reconstruct-12 FP64 5.7 against 8.2, a^H b FP64 6.6 against
// 8.8; BF16 at 100,000 sites 5.8 against 7.4. Past residency (reconstruct-12
// FP64 at 69,632 sites), and past 24 wavefronts per CU where more fit (FP64
// at 40,960 sites, FP32 at 81,920), the cap is as fast or up to 3% faster.
// Some kernels lose that already when their last CUs fill up (`share`, the percent
// of what is resident at once up to which a grid goes uncapped; the speed of a cap
// alone over three inputs in turn, uncapped -> capped with write-through): FP64
// products at 28,832 sites (88%) 0.94 -> 1.03, FP32 61,600 (94%) 0.98 -> 1.05, a^H
// b FP32 139,264 (100%) 0.96 -> 1.04 and FP64 59,632 (91%) 0.98 -> 1.05, the
// reconstruct-12 pack with FP64 rows 69,632 (100%) 0.97 -> 1.05. Others gain to the
// last CU (BF16 at 99,600 sites 1.32 -> 1.06).
struct LaunchPlan {
    size_t pad = 0;
    bool one_generation = false;
};
LaunchPlan launch_plan(const void *kernel, int waves, int block, int64_t grid, PadCache &cache, int share = 100);
// Caps by the bytes a call moves: waves[0] up to upto[0], waves[1] up to
// upto[1], waves[2] beyond, each with its own PadCache. A long stream runs best
// with few wavefronts resident; a short one spends more of its time filling
// and draining the CUs, where more of them help. The limits were placed by
// runs over 1, 3 and 10 buffers in turn, so that no size loses with any.
struct WaveCaps {
    int64_t upto[2];
    int waves[3];
    int share = 100;
};
constexpr WaveCaps one_cap(int waves, int share = 100)
{
    return {{INT64_MAX, INT64_MAX}, {waves, waves, waves}, share};
}
inline LaunchPlan launch_plan(const void *kernel, const WaveCaps &caps, int64_t bytes, int block, int64_t grid,
                              PadCache (&cache)[3])
{
    const int k = bytes <= caps.upto[0] ? 0 : bytes <= caps.upto[1] ? 1 : 2;
    return launch_plan(kernel, caps.waves[k], block, grid, cache[k], caps.share);
}
// Where the stores of a grid of more than one generation write through, by the
// bytes a call writes. The lines are measured ones, from runs of 10 ms over 1, 3
// and 10 inputs in turn, each with an output of its own or into new outputs, of
// which two are then in turn.
//  * Small outputs come back to a 256 MiB Infinity Cache that still holds part of
//    them: how much depends on how many the caller has in turn, which a call
//    cannot know. The product's line is where three outputs stop to gain (FP64,
//    FP32, BF16, reconstruct-12 and a^H b, write-through against nontemporal: 97 MB
//    1.10-1.13, 100 MB 1.03-1.04, 102 MB 0.99-1.02, 108 MB 0.98-0.995). With two it
//    would lie at 150 MB (1.07-1.18 up to there), and ten lose up to 2% from 72 MB.
//    Matrix-vector: 97 MB 1.05, 100 MB 0.99. A conversion writes a new output each
//    time: 140 MB 1.02-1.18, 150 MB 0.98-1.05, 160 MB 0.96-1.00.
//  * Outputs past the whole cache find nothing of it again, and write-through
//    saves the eviction: 282 MB 0.97-1.01, 290 MB 1.00-1.03, in every form.
constexpr int64_t kFitProduct = 100000000, kFitConversion = 144000000, kThroughAgain = 286000000;
inline bool write_through(const LaunchPlan &plan, int64_t written, int64_t fit, int64_t again = kThroughAgain)
{
    return !plan.one_generation && (written <= fit || written > again);
}
// The dynamic LDS of a cap of `waves` wavefronts per CU on device `dev`,
// computed on every call (no cache).
size_t occupancy_pad_for(const void *kernel, int waves, int block, int dev);

// ---- launchers (each returns hipSuccess or the launch error) --------------
// Forward products. The grid covers the lattice once; *_grid report it.
int64_t fwd_aos_grid(int precision, int64_t sites);
int64_t fwd_soa_grid(int64_t sites, int64_t pitch, int elem_bytes);
// Plane pitch (elements) of the padded SoA layout that streams at the site-major rate.
int64_t soa_pitch(int64_t sites, int elem_bytes);
int soa_block_threads();
hipError_t launch_fwd_aos(const void *a, const void *b, void *c, int64_t sites, int precision, hipStream_t s);
// The a b^H and a^H b products (FP64 = 0, FP32 = 1).
int64_t fwd_an_grid(int precision, int64_t sites);
hipError_t launch_fwd_na(const void *a, const void *b, void *c, int64_t sites, int precision, hipStream_t s);
hipError_t launch_fwd_an(const void *a, const void *b, void *c, int64_t sites, int precision, hipStream_t s);
// Matrix times colour vector, w[s][j] = a[s][j] v[s] (FP64 = 0, FP32 = 1).
int64_t mat_vec_grid(int precision, int64_t sites);
hipError_t launch_mat_vec(const void *a, const void *v, void *w, int64_t sites, int precision, hipStream_t s);
// SoA product; plane p of a and c starts at element p * pitch (pitch >= sites).
hipError_t launch_fwd_soa(const void *a, const void *b, void *c, int64_t sites, int64_t pitch, int elem_bytes,
                          hipStream_t s);
int aos_block_threads();
// Layout and storage-form conversions.
hipError_t launch_aos_soa(const void *src, void *dst, int64_t sites, int64_t pitch, int elem_bytes, bool to_soa,
                          hipStream_t s);
hipError_t launch_pack(const void *src, void *dst, int64_t sites, int precision, hipStream_t s);
hipError_t launch_unpack(const void *src, void *dst, int64_t sites, int precision, hipStream_t s);
hipError_t launch_stream_copy(const void *src, void *dst, int64_t bytes, hipStream_t s);
// Streaming probe of an access shape: per wavefront tile, in_a (and in_b)
// 16-byte chunks per lane read, out chunks per lane written. False for a
// shape it does not implement.
bool stream_shape_supported(int in_a, int in_b, int out);
hipError_t launch_stream_shape(const void *a, const void *b, void *c, int64_t tiles, int in_a, int in_b, int out,
                               int waves_per_cu, int tile_order, hipStream_t s);
// Adjoint: stage 1 writes per-workgroup partial sums of db into ws (72 x
// bwd_groups doubles, in 32-byte quads of components), stage 2 reduces them
// in a fixed order; bwd_workspace_doubles is the workspace of both. db is
// stored in double, or in float (rounded once) for db_float. launch_db forms
// db alone. spread: small lattices take more workgroups, and more workspace.
int64_t bwd_groups(int64_t sites, int precision, bool spread);
int64_t bwd_workspace_doubles(int64_t sites, int precision, bool spread);
int bwd_block_threads();
hipError_t launch_bwd(const void *a, const void *b, const void *dc, void *da, void *db, bool db_float, int64_t sites,
                      int precision, bool spread, double *ws, hipStream_t s);
hipError_t launch_db(const void *a, const void *dc, void *db, bool db_float, int64_t sites, int precision, bool spread,
                     double *ws, hipStream_t s);
hipError_t launch_bwd_zero(void *db, bool db_float, hipStream_t s);
// Bytes of the library-owned adjoint workspace (one static device array per
// device) and its device address on the current device, looked up on the
// first call per device.
constexpr size_t kScratchBytes = (size_t)64 << 20;
hipError_t bwd_scratch(double **ptr);

} // namespace su3
