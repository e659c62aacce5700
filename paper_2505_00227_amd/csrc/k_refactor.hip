// Refactor kernels for gfx950: level statistics, bitplane encoding with the
// per-plane error table and per-group lossless statistics, and the device-side
// hybrid selection of Alg. 2 (Sec. 4.2) with its Huffman codebook.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "device_bits.hpp"
#include "mdr_internal.hpp"

namespace mdr {
namespace {

// rows a general-path encoder workgroup stages in LDS at once
constexpr uint32_t kPassRows = 33;

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ int frexp_exp_f32(uint32_t absbits)
{
    uint32_t eb = absbits >> 23;
    if (eb) return (int)eb - 126;
    return -117 - (int)__clz(absbits & 0x7FFFFFu);
}

__device__ __forceinline__ int frexp_exp_f64(uint64_t absbits)
{
    uint32_t eb = (uint32_t)(absbits >> 52);
    if (eb) return (int)eb - 1022;
    return -1010 - (int)__clzll(absbits & 0xFFFFFFFFFFFFFull);
}

__device__ __forceinline__ uint64_t order_key_f32(uint32_t bits)
{
    return (bits >> 31) ? (uint64_t)(~bits) : (uint64_t)(bits | 0x80000000u);
}

__device__ __forceinline__ uint64_t order_key_f64(uint64_t bits)
{
    return (bits >> 63) ? ~bits : (bits | 0x8000000000000000ull);
}

template <typename T>
__device__ __forceinline__ T wave_max(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        T o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_min(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        T o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int l)
{
    return ((uint64_t)lane_value((uint32_t)(v >> 32), l) << 32) | lane_value((uint32_t)v, l);
}

// orders LDS traffic between the lanes of one wavefront
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ fills
__global__ void k_fill_u32(uint32_t* p, uint64_t count, uint32_t value)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
        p[i] = value;
}

// Copy from pinned host memory, read through its device address, into device
// memory on the stream's own queue.  System-scope loads go past any cache the
// host's writes could miss.
__global__ void k_copy_in(const uint64_t* src, uint64_t* __restrict__ dst, uint64_t count)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
        dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Start of a refactor pass, in one launch: the descriptor from pinned host
// memory (as k_copy_in), the level statistics to their neutral values and a
// region of accumulators to zero.  The first workgroups copy, the others fill.
// Both are bound by a launch: 2 launches took 7 us of a pass, this one 4
// (refactor of 32768 f32 values and its retrieval: 158 -> 153 us).
__global__ void k_begin_pass(const uint64_t* src, uint64_t* __restrict__ dst, uint64_t words, uint32_t copy_wg,
                             LevelStats* st, uint32_t count, u32x4* z, uint64_t n4)
{
    if (blockIdx.x < copy_wg) {
        const uint64_t stride = (uint64_t)copy_wg * blockDim.x;
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride)
            dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    const uint64_t i0 = (uint64_t)(blockIdx.x - copy_wg) * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)(gridDim.x - copy_wg) * blockDim.x;
    for (uint64_t i = i0; i < count; i += stride) {
        st[i].minkey = ~0ull;
        st[i].maxkey = 0;
        st[i].maxabs_bits = 0;
    }
    for (uint64_t i = i0; i < n4; i += stride) z[i] = u32x4{0u, 0u, 0u, 0u};
}

// ------------------------------------------------------------------ level statistics
// One streaming pass: min / max / max|x| (max |x| gives Alg. 1's alignment
// exponent and the non-finite check).  Each thread folds 16-byte vectors, the
// workgroup reduces in LDS, and one lane per workgroup publishes with three
// device atomics.  Atomics on one address serialize in the memory system, so
// a level gets few large workgroups (kStatsThreads threads, at most
// kStatsMaxWg of them).  Per thread: the largest |x| bit pattern and the float
// minimum / maximum (zeros of either sign are reported as +0.0, so their order
// does not matter).
template <bool F64>
struct StatAcc {
    using U = std::conditional_t<F64, uint64_t, uint32_t>;
    using T = std::conditional_t<F64, double, float>;
    U amax = 0;
    T vmin = __builtin_huge_val(), vmax = -__builtin_huge_val();
    __device__ __forceinline__ void add(U b)
    {
        const U ab = b & (F64 ? 0x7FFFFFFFFFFFFFFFull : 0x7FFFFFFFu);
        amax = ab > amax ? ab : amax;
        T v;
        __builtin_memcpy(&v, &b, sizeof(T));
        vmin = __builtin_fmin(vmin, v);
        vmax = __builtin_fmax(vmax, v);
    }
};

// One launch covers every level of a batch: workgroup -> job through wg_job,
// then a grid-stride loop over that level with the job's own workgroup count.
template <bool F64, bool VEC>
__global__ __launch_bounds__(kStatsThreads) void k_stats(const StatsJob* __restrict__ jobs,
                                                    const uint32_t* __restrict__ wg_job)
{
    using U = typename StatAcc<F64>::U;
    using T = typename StatAcc<F64>::T;
    constexpr int PER = 16 / sizeof(U);  // values per 16-byte vector
    const StatsJob& job = jobs[wg_job[blockIdx.x]];
    const auto x = gmem(static_cast<const U*>(job.x));
    const uint64_t n = job.n;
    LevelStats* st = job.stats;
    StatAcc<F64> acc;
    const uint64_t stride = (uint64_t)job.grid * blockDim.x;
    const uint64_t tid0 = (uint64_t)(blockIdx.x - job.wg_base) * blockDim.x + threadIdx.x;
    uint64_t done = 0;
    if (VEC) {
        const uint64_t nvec = n / PER;
        const auto xv4 = gmem(reinterpret_cast<const u32x4*>(job.x));
#pragma unroll 4
        for (uint64_t i = tid0; i < nvec; i += stride) {
            const u32x4 q = __builtin_nontemporal_load(&xv4[i]);
            if constexpr (F64) {
                acc.add(((uint64_t)q.y << 32) | q.x);
                acc.add(((uint64_t)q.w << 32) | q.z);
            } else {
                acc.add(q.x);
                acc.add(q.y);
                acc.add(q.z);
                acc.add(q.w);
            }
        }
        done = nvec * PER;
    }
    for (uint64_t i = done + tid0; i < n; i += stride) acc.add(x[i]);

    __shared__ unsigned long long s_amax[kStatsThreads / 64];
    __shared__ T s_min[kStatsThreads / 64], s_max[kStatsThreads / 64];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t amax = wave_max((uint64_t)acc.amax);
    T vmin = wave_min(acc.vmin), vmax = wave_max(acc.vmax);
    if (lane == 0) {
        s_amax[wave] = amax;
        s_min[wave] = vmin;
        s_max[wave] = vmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kStatsThreads / 64; ++w) {
            amax = s_amax[w] > amax ? s_amax[w] : amax;
            vmin = s_min[w] < vmin ? s_min[w] : vmin;
            vmax = s_max[w] > vmax ? s_max[w] : vmax;
        }
        U bmin, bmax;
        __builtin_memcpy(&bmin, &vmin, sizeof(T));
        __builtin_memcpy(&bmax, &vmax, sizeof(T));
        const uint64_t kmin = F64 ? order_key_f64(bmin) : order_key_f32((uint32_t)bmin);
        const uint64_t kmax = F64 ? order_key_f64(bmax) : order_key_f32((uint32_t)bmax);
        atomicMin((unsigned long long*)&st->minkey, (unsigned long long)kmin);
        atomicMax((unsigned long long*)&st->maxkey, (unsigned long long)kmax);
        if (amax) atomicMax((unsigned long long*)&st->maxabs_bits, (unsigned long long)amax);
    }
}

// ------------------------------------------------------------------ bitplane encoder
// One thread owns one block of 32 consecutive values (one u32 word of every
// plane); a workgroup covers a tile of 256 blocks and walks a contiguous range
// of tiles.  Per block:
//   y = |x| * 2^(B-e) (exact), mag = floor(y), sign bit;
//   error keys: key_k = fract(y * 2^(k-B)) = (|x| mod 2^(e-k)) / 2^(e-k); the
//     workgroup keeps max_k key_k in LDS.  Values with mag = 0 lie below every
//     cut: their error is |x| for every k (tracked as `small`);
//   32x32 in-register bit transpose (two for f64) -> plane words;
//   coalesced stores of each plane row, per-unit byte histograms (LDS), and
//   counts of W-bit word transitions for the run-length estimate.
//
// Exact pruning of the f32 error keys.  Let K_k be the workgroup's running
// maximum.  When K_k >= 1 - 2^-t (its binary fraction starts with t ones), a
// value can exceed it only if the t bits just below the cut, in y's binary
// expansion, are all ones.  With Y = (mag << 32) | top 32 fraction bits, bit p
// of r_t = AND_{i<t} (Y << i) says "bits p..p-t+1 of Y are ones"; r_1, r_2,
// r_4, r_8, r_12 come from four shift-ANDs, and each cut c = B-k (bit c-1 of
// the high word) is tested with the longest of them its K_k allows, so one
// pass flags every candidate cut of a value.  Only flagged cuts are evaluated
// and folded in with an LDS max; the others cannot change the result.  Cuts
// with K_k < 1/2 take the direct per-block maximum; k = 0 is max |x|, known from
// the statistics.  Stale maxima only add candidates, so the result is exact.
//
// f64 FAST takes the same test to the plane words from a workgroup's second tile
// on: after the transpose a run of ones below a cut is an AND of plane words,
// one operation for 32 values (with 16 more planes of fraction bits for the
// lowest cuts), against 46 per value.  A word of flagged values comes out of
// it; their keys are then taken from the values, loaded again while the rows go
// out (a few a tile, and the values need not stay in registers: 128 of them
// against 168).  Cuts with no bit below them so far are checked by one key, and
// the cuts above them whose keys cannot rise while that holds are left out, so
// data of few significant bits does not fall back to the per-value test.
// 2^27 values: exponents over 100 binades 867 -> 810 us, uniform 1311 -> 707,
// 10-bit values 2164 -> 629; 2^30 values of 32 slabs 5.36 -> 4.95 ms, of which
// the loads and stores alone take 4.0 and the histograms most of the rest.  In
// f32 the per-value test costs half as much and hides under the histograms: the
// plane test changed 2^27 values by -1 to +5%, so it is not used there.
// FAST: 32 planes of f32 or 64 planes of f64, in groups of 4 (every row, its
// unit and its histogram offset known at compile time): rows go from registers
// straight to memory, neighbours come by lane shuffle, runs are counted per
// thread (f32) or per wavefront (f64) and unit.
template <bool F64, bool VEC, bool FAST>
__device__ __forceinline__ void encode_body(const EncodeJob& job, const uint32_t wg)
{
    using T = std::conditional_t<F64, double, float>;
    constexpr int G = F64 ? 2 : 1;  // u32 words per W-bit word
    constexpr int NROW = F64 ? 65 : 33;
    // dynamic LDS (general path only): [nunits][256] byte histograms, then the
    // tile's plane words [rows][256]
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_prev[kMaxRows][G];  // last word(s) of the previous tile, per row
    __shared__ uint32_t s_trans[kMaxRows];
    __shared__ uint32_t s_key32[F64 ? 1 : kKeyStride];
    __shared__ unsigned long long s_key64[F64 ? kKeyStride : 1];
    __shared__ uint32_t s_zero[FAST && !F64 ? 1 : kThreads];  // sink for zero bytes (one slot per thread)
    // FAST: the byte histograms at fixed LDS addresses, so each unit's offset is
    // an instruction immediate
    constexpr int FUNITS = F64 ? 17 : 9;  // FAST: units (sign + 16 or 8 groups)
    // f64 FAST: each unit's 256 bins are followed by one sink slot per lane for
    // zero bytes (counted by difference), at the same offset from every unit
    constexpr int HSTRIDE = F64 ? 320 : 256;
    __shared__ uint32_t s_hist_fast[FAST ? FUNITS * HSTRIDE : 1];

    __shared__ uint32_t s_hoff[kMaxRows];  // row -> its unit's histogram offset
    // FAST: each wave's last words of every row for the next wave's first lanes
    // (f32: lane 63's; f64: lanes 62 and 63, the two halves of its last W-bit word)
    __shared__ uint32_t s_edge[FAST && !F64 ? 4 : 1][kThreads / 64][FAST && !F64 ? 33 : 1];
    // f64: every wave's first (lanes 0, 1) and last (lanes 62, 63) words per row
    __shared__ uint32_t s_first64[FAST && F64 ? 4 : 1][kThreads / 64][2][FAST && F64 ? 65 : 1];
    __shared__ uint32_t s_last64[FAST && F64 ? 4 : 1][kThreads / 64][2][FAST && F64 ? 65 : 1];
    uint32_t edge_trc[2] = {0, 0};  // f64 FAST: transitions at the wave's left edge, rows lane and lane + 64
    uint32_t trc[FAST && !F64 ? 9 : 1];  // f32 FAST: this thread's word transitions per unit
#pragma unroll
    for (int i = 0; i < (FAST && !F64 ? 9 : 1); ++i) trc[i] = 0;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    // every field the tile loop needs, in registers: stores through the row
    // pointer could otherwise alias the job table and force reloads
    const uint32_t B = job.B, nbd = job.nbd, m = job.m, nunits = job.nunits;
    const uint32_t ntiles = job.ntiles, tpw = job.tiles_per_wg;
    const uint64_t n = job.n;
    const uint64_t amax = job.stats->maxabs_bits;  // 0: every value is zero
    const int e = amax == 0 ? 0 : (F64 ? frexp_exp_f64(amax) : frexp_exp_f32((uint32_t)amax));
    const T* xg = static_cast<const T*>(job.x);
    const auto x = gmem(xg);
    const auto rows = gmem(job.rows);
    const auto recs = gmem(job.recs);
    if (tid < kMaxRows) s_hoff[tid] = job.hist_off[tid];
    (void)m;
    uint32_t* s_hist = FAST ? s_hist_fast : s_dyn;
    uint32_t* s_pl = FAST ? s_dyn : s_dyn + nunits * 256;  // [rows of one pass][256]

    for (uint32_t i = tid; i < nunits * (FAST ? HSTRIDE : 256); i += kThreads) s_hist[i] = 0;
    if (tid < kMaxRows) s_trans[tid] = 0;
    if (tid < kKeyStride) {
        if constexpr (F64)
            s_key64[tid] = 0;
        else
            s_key32[tid] = 0;
    }

    uint32_t frac_max = 0;  // f32: bits of max fract(y) = the k = B key (nonnegative: bits order as values)
    uint64_t frac_max64 = 0;  // the same for f64
    T small = 0;
    uint32_t per_value = 0;  // FAST: tiles to go before the plane test is tried again

    // y < 1, the values below every cut, in terms of |x|
    const T tiny_below = F64 ? (T)__builtin_amdgcn_ldexp(1.0, e - (int)B) : (T)__builtin_amdgcn_ldexpf(1.0f, e - (int)B);
    uint32_t tiny_high;  // its high word
    if constexpr (F64)
        tiny_high = (uint32_t)((uint64_t)__double_as_longlong(tiny_below) >> 32);
    else
        tiny_high = __float_as_uint(tiny_below);
    const auto fabs_t = [](T a) -> T {
        if constexpr (F64)
            return __builtin_fabs(a);
        else
            return __builtin_fabsf(a);
    };
    const uint32_t t0 = wg * tpw;
    const uint32_t t1 = min(ntiles, t0 + tpw);
    const uint32_t last_blk = min(nbd, t1 * kTileBlocks) - 1;
    // the zeroed histograms and key maxima must be visible to every wave
    // before any reads or updates them (the fast path has no barrier at the
    // top of a tile)
    __syncthreads();

    // ---- 32 consecutive values of tile tt (zeros past the level's end)
    // the u32 word of the tile this thread encodes: its own index, except on
    // the f64 fast path, where lane l of a wave takes half l / 32 (low half
    // first) of the wave's W-bit word l % 32, so that the same half of the
    // previous word is one lane down
    const uint32_t slot = (FAST && F64) ? ((tid & ~63u) | ((lane & 31u) << 1) | (lane >> 5)) : tid;
    auto load_tile = [&](uint32_t tt, T (&vv)[32]) {
        const uint32_t b = tt * kTileBlocks + slot;
        const uint64_t bs = (uint64_t)b * 32;
        if (VEC && b < nbd && bs + 32 <= n) {
            if constexpr (F64) {
                const auto p = gmem(reinterpret_cast<const f64x2*>(xg + bs));
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const f64x2 q = p[j];
                    vv[2 * j] = q.x;
                    vv[2 * j + 1] = q.y;
                }
            } else {
                const auto p = gmem(reinterpret_cast<const f32x4*>(xg + bs));
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const f32x4 q = p[j];
                    vv[4 * j] = q.x;
                    vv[4 * j + 1] = q.y;
                    vv[4 * j + 2] = q.z;
                    vv[4 * j + 3] = q.w;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 32; ++j) vv[j] = (b < nbd && bs + j < n) ? x[bs + j] : T(0);
        }
    };
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t blk = t * kTileBlocks + slot;
        const bool valid = blk < nbd;
        // the fast path shares nothing between tiles but the edge buffers (four
        // of them), so its waves need no barrier here
        if constexpr (!FAST) __syncthreads();  // the previous tile's rows have been consumed
        T v[32];
        load_tile(t, v);

        // ---- align to the level exponent: y = |x| 2^(B-e), mag = floor(y)
        uint32_t sgn = 0;
        uint32_t lo[32];
        uint32_t hi[F64 ? 32 : 1];
        if constexpr (FAST) {
            uint32_t least = ~0u;  // of the high words of |x|: tells whether any value may lie below every cut
#pragma unroll
            for (int j = 31; j >= 0; --j) {
                uint32_t h;
                if constexpr (F64)
                    h = (uint32_t)((uint64_t)__double_as_longlong(v[j]) >> 32);
                else
                    h = __float_as_uint(v[j]);
                sgn = __builtin_amdgcn_alignbit(sgn, h, 31);
                least = min(least, h & 0x7FFFFFFFu);
            }
            asm volatile("" : "+v"(sgn));  // here, or the raw values would live on
            if (__ballot(least <= tiny_high)) {
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    // mag = floor(y) = 0: |x| to `small`, the value to zero.  By
                    // mask: two selects in a row on one condition take 23 cycles
                    const T a = fabs_t(v[j]);
                    uint32_t mask = a < tiny_below ? ~0u : 0u;
                    asm volatile("" : "+v"(mask));
                    if constexpr (F64) {
                        const uint64_t b = (uint64_t)__double_as_longlong(a), mask2 = (uint64_t)mask << 32 | mask;
                        small = __builtin_fmax(small, __longlong_as_double((long long)(b & mask2)));
                        v[j] = __longlong_as_double((long long)(b & ~mask2));
                    } else {
                        const uint32_t b = __float_as_uint(a);
                        small = __builtin_fmaxf(small, __uint_as_float(b & mask));
                        v[j] = __uint_as_float(b & ~mask);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                if constexpr (F64)
                    v[j] = __builtin_amdgcn_ldexp(fabs_t(v[j]), (int)B - e);
                else
                    v[j] = __builtin_amdgcn_ldexpf(fabs_t(v[j]), (int)B - e);
            }
        } else
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            if constexpr (F64) {
                uint64_t bits = (uint64_t)__double_as_longlong(v[j]);
                sgn |= (uint32_t)(bits >> 63) << j;
                double a = __longlong_as_double((long long)(bits & 0x7FFFFFFFFFFFFFFFull));
                double y = __builtin_amdgcn_ldexp(a, (int)B - e);
                bool tiny = y < 1.0;  // mag = floor(y) = 0
                small = (tiny && a > small) ? a : small;
                v[j] = tiny ? 0.0 : y;
            } else {
                uint32_t bits = __float_as_uint(v[j]);
                sgn |= (bits >> 31) << j;
                float a = __uint_as_float(bits & 0x7FFFFFFFu);
                float y = __builtin_amdgcn_ldexpf(a, (int)B - e);
                bool tiny = y < 1.0f;  // mag = floor(y) = 0
                small = (tiny && a > small) ? a : small;
                v[j] = tiny ? 0.0f : y;
            }
        }

        // materialise y and the running `small` here, so the raw values die
        // before the key loop instead of being carried through it
#pragma unroll
        for (int j = 0; j < 32; ++j) asm volatile("" : "+v"(v[j]));
        asm volatile("" : "+v"(small));
        // ---- exact error keys, k = 0..B
        // f64 FAST: by plane words once the running maxima are high (see above)
        constexpr bool PLANES = FAST && F64;
        bool by_plane = false;
        uint64_t free8 = 0, free12 = 0, free16 = 0;  // cuts (bit c) that need no run of 8, 12, 16 ones
        if constexpr (PLANES) {
            if (t > t0) {
                uint32_t tl = 0;  // lane c: the leading ones of cut c's running maximum
                const double M = __longlong_as_double((long long)s_key64[64 - lane]);
                if (M >= 0.5) tl = __clz(~(uint32_t)(M * 0x1p32));
                uint64_t s4 = __ballot(tl >= 4);
                const uint64_t s8 = __ballot(tl >= 8);
                // Cuts 0 .. z without a bit below them so far.  While that stays
                // so, cut c's key has c - z bits: at all ones it cannot rise
                const uint64_t none = __ballot(M == 0.0);
                uint64_t done = none;
                if (none) {
                    const int z = 63 - __clzll((long long)none);
                    double km = 0.0;
#pragma unroll
                    for (int j = 0; j < 32; ++j)
                        km = __builtin_fmax(km, __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(v[j], -z)));
                    done = __ballot(km != 0.0) ? 0 : none | __ballot((int)lane > z && (int)tl >= (int)lane - z);
                }
                by_plane = __popcll(s4 | done) >= 56 && __popcll(s8 | done) >= 48 && per_value == 0;
                per_value -= per_value ? 1u : 0u;
                uint64_t direct = ~(s4 | done);
                s4 &= ~done;
                free8 = s4 & ~s8;
                free12 = s4 & ~__ballot(tl >= 12);
                free16 = s4 & ~__ballot(tl >= 16);
                if (by_plane) {
                    // the few cuts whose maximum is below 1 - 2^-4: directly, from
                    // the highest: no bit below a cut, none below the lower ones
                    while (direct) {
                        const int c = 63 - __clzll((long long)direct);
                        direct &= ~(1ull << c);
                        double km = 0.0;
#pragma unroll
                        for (int j = 0; j < 32; ++j)
                            km = __builtin_fmax(km, __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(v[j], -c)));
                        if (!__ballot(km != 0.0)) break;
                        km = wave_max(km);
                        if (lane == 0) atomicMax(&s_key64[64 - c], (unsigned long long)__double_as_longlong(km));
                    }
                }
            }
        }
        if (by_plane) {
        } else if constexpr (F64) {
            // The f32 pruning below on the 128-bit fixed point of y: words
            // X3:X2 = magnitude (hi[j]:lo[j]), X1 = the top 32 fraction bits.
            // Cut c (1..B-1) is bit 64+c-1; a tested run is at most 12 bits
            // long, so it never reaches below bit 53 and the word below X1 is
            // not needed (the runs computed for X1's low bits, which take
            // zeros from below, are never used).  Lane l decides cut l+1.
            uint64_t S1, S2, S4, S8, S12;
            if (t == t0 && B > 1) {
                const int c = (int)(lane % (B - 1)) + 1;  // seeds, as for f32
                double km = 0.0;
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    km = __builtin_fmax(km, __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(v[j], -c)));
                }
                atomicMax(&s_key64[B - c], (unsigned long long)__double_as_longlong(km));
                __syncthreads();
            }
            {
                const uint32_t c = lane + 1;
                uint32_t tl = 0;
                if (c < B) {
                    const double M = __longlong_as_double((long long)s_key64[B - c]);
                    if (M >= 0.5) tl = __clz(~(uint32_t)(M * 0x1p32));
                }
                const bool live = c < B;
                S12 = __ballot(live && tl >= 12);
                S8 = __ballot(live && tl >= 8 && tl < 12);
                S4 = __ballot(live && tl >= 4 && tl < 8);
                S2 = __ballot(live && tl >= 2 && tl < 4);
                S1 = __ballot(live && tl == 1);
            }
            const uint64_t strong = S1 | S2 | S4 | S8 | S12;
            const uint32_t S1l = (uint32_t)S1, S2l = (uint32_t)S2, S4l = (uint32_t)S4, S8l = (uint32_t)S8,
                           S12l = (uint32_t)S12;
            const uint32_t S1h = (uint32_t)(S1 >> 32), S2h = (uint32_t)(S2 >> 32), S4h = (uint32_t)(S4 >> 32),
                           S8h = (uint32_t)(S8 >> 32), S12h = (uint32_t)(S12 >> 32);
            // ALL12: every cut's maximum already starts with 12 ones (the usual
            // case past a workgroup's first tile), so the 12-bit runs alone flag
            // the candidates and the shorter runs' masks drop out
            auto key_pass = [&](auto all12_t) {
                constexpr bool ALL12 = decltype(all12_t)::value;
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    const double y = v[j];
                    const double f = __builtin_amdgcn_fract(y);
                    frac_max64 = (uint64_t)__double_as_longlong(__builtin_fmax(__longlong_as_double((long long)frac_max64), f));
                    asm volatile("" : "+v"(frac_max64));  // fold in now, not at the end
                    const double yh = __builtin_trunc(y * 0x1p-32);
                    const uint32_t X3 = (uint32_t)yh, X2 = (uint32_t)(y - yh * 0x1p32), X1 = (uint32_t)(f * 0x1p32);
                    // (word << k) = alignbit(word, word below, 32 - k)
                    const uint32_t r2_3 = X3 & __builtin_amdgcn_alignbit(X3, X2, 31);
                    const uint32_t r2_2 = X2 & __builtin_amdgcn_alignbit(X2, X1, 31);
                    const uint32_t r2_1 = X1 & (X1 << 1);
                    const uint32_t r4_3 = r2_3 & __builtin_amdgcn_alignbit(r2_3, r2_2, 30);
                    const uint32_t r4_2 = r2_2 & __builtin_amdgcn_alignbit(r2_2, r2_1, 30);
                    const uint32_t r4_1 = r2_1 & (r2_1 << 2);
                    const uint32_t r8_3 = r4_3 & __builtin_amdgcn_alignbit(r4_3, r4_2, 28);
                    const uint32_t r8_2 = r4_2 & __builtin_amdgcn_alignbit(r4_2, r4_1, 28);
                    const uint32_t r8_1 = r4_1 & (r4_1 << 4);
                    const uint32_t r12_3 = r8_3 & __builtin_amdgcn_alignbit(r8_3, r8_2, 28);
                    const uint32_t r12_2 = r8_2 & __builtin_amdgcn_alignbit(r8_2, r8_1, 28);
                    uint32_t ca, cb;
                    if constexpr (ALL12) {
                        ca = r12_2 & S12l;
                        cb = r12_3 & S12h;
                    } else {
                        ca = (X2 & S1l) | (r2_2 & S2l) | (r4_2 & S4l) | (r8_2 & S8l) | (r12_2 & S12l);
                        cb = (X3 & S1h) | (r2_3 & S2h) | (r4_3 & S4h) | (r8_3 & S8h) | (r12_3 & S12h);
                    }
                    uint64_t cand = ((uint64_t)cb << 32) | ca;  // bit c-1: cut c
                    while (cand) {
                        const int c = __ffsll((unsigned long long)cand);
                        cand &= cand - 1;
                        const double key = __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(y, -c));
                        atomicMax(&s_key64[B - c], (unsigned long long)__double_as_longlong(key));
                    }
                }
            };
            if (!FAST && S12 == (B > 1 ? (1ull << (B - 1)) - 1ull : 0ull)) {
                if constexpr (!FAST) key_pass(std::true_type{});
            } else {
                key_pass(std::false_type{});
                const uint64_t all = B > 1 ? (1ull << (B - 1)) - 1ull : 0ull;  // cuts 1 .. B-1
                uint64_t weak = all & ~strong;
                while (weak) {  // from the highest: no bit below a cut, none below the lower ones
                    const int c = 64 - __clzll((long long)weak);
                    weak &= ~(1ull << (c - 1));
                    double km = 0.0;
#pragma unroll
                    for (int j = 0; j < 32; ++j) {
                        km = __builtin_fmax(km, __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(v[j], -c)));
                    }
                    if (!__ballot(km != 0.0)) break;
                    km = wave_max(km);
                    if (lane == 0) atomicMax(&s_key64[B - c], (unsigned long long)__double_as_longlong(km));
                }
            }
        } else {
            // Cut c = B - k (k = 1..B-1) is bit c-1 of y; k = B is the fraction
            // itself (frac_max).  A value can raise the running maximum M_c only
            // if its key exceeds M_c; when M_c has t leading ones (M_c >= 1 - 2^-t)
            // that needs bits c-1 .. c-t of y to be ones.  Each cut is tested with
            // the longest run in {12, 8, 4, 2, 1} that its M_c allows; cuts with
            // M_c < 1/2 take the direct maximum.  Lane l decides cut l+1.
            uint32_t S1, S2, S4, S8, S12;
            if (t == t0 && B > 1) {
                // Seed the workgroup's running maxima before its first tile:
                // lane l takes the exact maximum over its own 32 values for
                // one cut, so every cut starts from the largest of about 256
                // actual keys.  Without it every cut would take the direct
                // maximum below (about three times the work of a pruned tile);
                // seeds are keys of actual values, so the pruning stays exact.
                const int c = (int)(lane % (B - 1)) + 1;
                float km = 0.0f;
#pragma unroll
                for (int j = 0; j < 32; ++j)
                    km = fmaxf(km, __builtin_amdgcn_fractf(__builtin_amdgcn_ldexpf(v[j], -c)));
                atomicMax(&s_key32[B - c], __float_as_uint(km));
                __syncthreads();
            }
            {
                const uint32_t c = lane + 1;
                uint32_t tl = 0;
                if (c < B) {
                    const float M = __uint_as_float(s_key32[B - c]);
                    if (M >= 0.5f) tl = __clz(~(uint32_t)(M * 0x1p32f));
                }
                const bool live = c < B;
                S12 = (uint32_t)__ballot(live && tl >= 12);
                S8 = (uint32_t)__ballot(live && tl >= 8 && tl < 12);
                S4 = (uint32_t)__ballot(live && tl >= 4 && tl < 8);
                S2 = (uint32_t)__ballot(live && tl >= 2 && tl < 4);
                S1 = (uint32_t)__ballot(live && tl == 1);
            }
            const uint32_t strong = S1 | S2 | S4 | S8 | S12;
            auto one = [&](float y) {
                const float f = __builtin_amdgcn_fractf(y);
                frac_max = max(frac_max, __float_as_uint(f));
                asm volatile("" : "+v"(frac_max));  // fold in now, not at the end
                const uint64_t Y = ((uint64_t)(uint32_t)y << 32) | (uint32_t)(f * 0x1p32f);
                const uint64_t r2 = Y & (Y << 1);    // bit p: bits p, p-1 are ones
                const uint64_t r4 = r2 & (r2 << 2);  // p .. p-3
                const uint64_t r8 = r4 & (r4 << 4);  // p .. p-7
                const uint64_t r12 = r8 & (r8 << 4); // p .. p-11
                uint32_t cand = ((uint32_t)(Y >> 32) & S1) | ((uint32_t)(r2 >> 32) & S2) |
                                ((uint32_t)(r4 >> 32) & S4) | ((uint32_t)(r8 >> 32) & S8) |
                                ((uint32_t)(r12 >> 32) & S12);
                while (cand) {
                    const int c = __ffs(cand);  // 1-based bit index == cut
                    cand &= cand - 1;
                    const float key = __builtin_amdgcn_fractf(__builtin_amdgcn_ldexpf(y, -c));
                    atomicMax(&s_key32[B - c], __float_as_uint(key));
                }
            };
#pragma unroll
            for (int j = 0; j < 32; ++j) one(v[j]);
            const uint32_t all = (1u << (B - 1)) - 1u;  // cuts 1 .. B-1
            uint32_t weak = all & ~strong;
            while (weak) {  // from the highest, as for f64
                const int c = 32 - __clz(weak);
                weak &= ~(1u << (c - 1));
                float km = 0.0f;
#pragma unroll
                for (int j = 0; j < 32; ++j)
                    km = fmaxf(km, __builtin_amdgcn_fractf(__builtin_amdgcn_ldexpf(v[j], -c)));
                if (!__ballot(km != 0.0f)) break;
                km = wave_max(km);
                if (lane == 0) atomicMax(&s_key32[B - c], __float_as_uint(km));
            }
        }

        if constexpr (PLANES) {
            // the maximum fraction (cut 0) too is in LDS after every tile
            if (!by_plane) {
                const uint64_t fm = wave_max(frac_max64);
                if (lane == 0) atomicMax(&s_key64[64], (unsigned long long)fm);
            }
        }
        // ---- mag = hi:lo (0 when tiny), converted afresh: reusing the key
        // pass's conversions would keep 32 or 64 more registers alive through it.
        // PLANES: and the top 16 bits of the fractions of values p and p + 16 in fr[p]
        uint32_t fr[PLANES ? 16 : 1];
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            uint32_t f2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = p + 16 * h;
                asm volatile("" : "+v"(v[j]));
                if constexpr (F64) {
                    const double yh = __builtin_trunc(v[j] * 0x1p-32), yl = v[j] - yh * 0x1p32;
                    hi[j] = (uint32_t)yh;
                    lo[j] = (uint32_t)yl;
                    if constexpr (PLANES) f2[h] = (uint32_t)(__builtin_amdgcn_fract(yl) * 0x1p16);
                } else {
                    lo[j] = (uint32_t)v[j];
                }
            }
            if constexpr (PLANES) {
                fr[p] = f2[0] | (f2[1] << 16);
                asm volatile("" : "+v"(fr[p]));  // here, or the values would live through the transposes
            }
        }
        // ---- bit transpose: lo[c] (and hi[c]) become the plane words of bit c (32 + c);
        // row 0 = sign, row r >= 1 = plane r-1 = bit B-r
        transpose32(lo);
        if constexpr (F64) transpose32(hi);
        uint32_t raised = 0;  // PLANES: this block's values that may raise a key maximum
        T raise_x = 0;        // the first of them
        if constexpr (PLANES) {
            if (by_plane) {
                transpose16(fr);  // fr[i]: bit i - 16
                // X(i): the plane word of bit i - 16; cut c's key begins with bit c - 1
                auto X = [&](int i) -> uint32_t { return i < 16 ? fr[i & 15] : i < 48 ? lo[(i - 16) & 31] : hi[(i - 48) & 31]; };
                uint32_t r2[79], r4[79];  // runs of 2 and 4 ones down from a bit
#pragma unroll
                for (int i = 1; i < 79; ++i) {
                    r2[i] = X(i) & X(i - 1);
                    if (i >= 3) r4[i] = r2[i] & r2[i - 2];
                    if (i >= 15) {
                        const int c = i - 15;
                        auto ones_if = [&](uint64_t cuts) -> uint32_t {  // all ones if it holds cut c
                            return 0u - ((uint32_t)(cuts >> (c & 32)) >> (c & 31) & 1u);
                        };
                        const uint32_t f8 = ones_if(free8), f12 = ones_if(free12), f16 = ones_if(free16);
                        raised |= r4[i] & (r4[i - 4] | f8) & (r4[i - 8] | f12) & (r4[i - 12] | f16);
                        asm volatile("" : "+v"(raised));
                    }
                }
                // its value again, in flight while the rows go out
                if (raised) raise_x = x[(uint64_t)blk * 32 + (__ffs(raised) - 1)];
            }
        }
        // the flagged values' keys, a value of every lane at a time
        auto raise_keys = [&]() {
            // many flagged values: the per-value test is faster, for some tiles
            if (__ballot(__popc(raised) > 8)) per_value = 7;
            while (raised) {
                const double y = __builtin_amdgcn_ldexp(__builtin_fabs(raise_x), (int)B - e);
                raised &= raised - 1;
                if (raised) raise_x = x[(uint64_t)blk * 32 + (__ffs(raised) - 1)];
                // the same runs along this value's bits: Y.F its integer and 32 fraction bits
                const double f = __builtin_amdgcn_fract(y), yh = __builtin_trunc(y * 0x1p-32);
                const uint64_t Y = (uint64_t)(uint32_t)yh << 32 | (uint32_t)(y - yh * 0x1p32);
                const uint64_t F = (uint64_t)(uint32_t)(f * 0x1p32) << 32;
                atomicMax(&s_key64[64], (unsigned long long)__double_as_longlong(f));
                const uint64_t F2 = F & (F << 1), F4 = F2 & (F2 << 2);
                const uint64_t Y2 = Y & (Y << 1 | F >> 63), Y4 = Y2 & (Y2 << 2 | F2 >> 62);
                uint64_t cand = Y4 & ((Y4 << 4 | F4 >> 60) | free8 >> 1) & ((Y4 << 8 | F4 >> 56) | free12 >> 1) &
                                ((Y4 << 12 | F4 >> 52) | free16 >> 1) & (~0ull >> 1);  // bit c - 1: cut c
                while (cand) {
                    const int c = __ffsll((unsigned long long)cand);
                    cand &= cand - 1;
                    const double key = __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(y, -c));
                    atomicMax(&s_key64[64 - c], (unsigned long long)__double_as_longlong(key));
                }
            }
        };
        if constexpr (FAST && F64) {
            // row r (0..64) is sgn, hi[32 - r] (r <= 32) or lo[64 - r]; unit
            // of row r is (r + 3) / 4.  Lanes l and l + 32 hold the halves of
            // the wave's W-bit word l (l < 32), so the same half of the
            // previous word comes by one wave shift.  At the wave's left edge:
            // lanes 0 and 32 (its first word) and 31 and 63 (its last) leave
            // their words in LDS, and after the tile's barrier lane r of each
            // wave compares row r of its first word with the left wave's last
            // (wave 0: wave 3 of the previous tile), so the row loop reads no LDS.
            const uint32_t wave = tid >> 6, h = lane >> 5, lw32 = lane & 31u;
            const uint32_t par = (t - t0) & 3;  // edge buffers in use, as for f32
#define MDR_ROW64(r) ((r) == 0 ? sgn : ((r) <= 32 ? hi[32 - (r)] : lo[64 - (r)]))
            if (lw32 == 0 || lw32 == 31) {
                uint32_t* dst = lw32 == 0 ? &s_first64[par][wave][h][0] : &s_last64[par][wave][h][0];
#pragma unroll
                for (int r = 0; r <= 64; ++r) dst[r] = MDR_ROW64(r);
            }
            if (t == t0 && wave == 0 && lw32 == 0) {
#pragma unroll
                for (int r = 0; r <= 64; ++r) recs[((uint64_t)wg * kMaxRows + r) * 4 + h] = MDR_ROW64(r);
            }
            if (valid && blk + 2 > last_blk) {
#pragma unroll
                for (int r = 0; r <= 64; ++r)
                    recs[((uint64_t)wg * kMaxRows + r) * 4 + 2 + (blk + 1 - last_blk)] = MDR_ROW64(r);
            }
            __syncthreads();  // edges written; every thread is done with its y values
            {
                // the wave's first word against its left neighbour; the range's
                // first word (wave 0 of its first tile) has none
                const uint32_t first_blk = t * kTileBlocks + wave * 64;
                if (first_blk < nbd && (wave > 0 || t > t0)) {
                    const uint32_t lp = wave ? par : ((par + 3) & 3), lwv = wave ? wave - 1 : 3;
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
                        const uint32_t r = lane + 64u * hh;
                        if (r <= 64) {
                            const bool ne = s_first64[par][wave][0][r] != s_last64[lp][lwv][0][r] ||
                                            s_first64[par][wave][1][r] != s_last64[lp][lwv][1][r];
                            edge_trc[hh] += ne ? 1u : 0u;
                        }
                    }
                }
            }
            const uint32_t zsink = (256u + lane) * 4u;  // this lane's sink, bytes past a unit's bins
            auto rows_out = [&](auto full_tile) {
                constexpr bool FULL = decltype(full_tile)::value;
                uint64_t rb = reinterpret_cast<uint64_t>(job.rows);
                asm volatile("" : "+s"(rb));
                const uint32_t boff = blk * 4u;
                // lanes whose word has a left neighbour in the wave
                const unsigned long long keep = __ballot((FULL || valid) && lw32 != 0);
                uint32_t ucnt = 0;  // the current unit's transitions (wave-wide)
#pragma unroll
                for (int r = 0; r <= 64; ++r) {
                    const uint32_t w = MDR_ROW64(r);
                    const int unit = (r + 3) / 4;
                    if (FULL || valid) {
                        *gmem(reinterpret_cast<uint32_t*>(rb + boff)) = w;
                        // nonzero bytes into the unit's bins, zero bytes into this
                        // lane's sink slot after them (no branches)
                        uint8_t* hb = reinterpret_cast<uint8_t*>(&s_hist_fast[unit * HSTRIDE]);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t byte = (w >> (8 * q)) & 0xFFu;
                            atomicAdd(reinterpret_cast<uint32_t*>(hb + (byte ? byte * 4u : zsink)), 1u);
                        }
                    }
                    // the same half of the previous word: one wave_shr:1 (lanes 0
                    // and 32 compare at the edge above instead)
                    const int p1 = __builtin_amdgcn_update_dpp((int)w, (int)w, 0x138, 0xF, 0xF, false);
                    const unsigned long long ne = __ballot((int)w != p1) & keep;
                    // a word differs if either half does; a unit's count goes to
                    // its first row's slot (the selection sums a unit's rows)
                    ucnt += (uint32_t)__popc((uint32_t)ne | (uint32_t)(ne >> 32));
                    if (r == 0 || r % 4 == 0) {
                        if (lane == 0 && ucnt) atomicAdd(&s_trans[r == 0 ? 0 : r - 3], ucnt);
                        ucnt = 0;
                    }
                    rb += 4ull * nbd;
                }
            };
            if ((t + 1) * kTileBlocks <= nbd)
                rows_out(std::true_type{});
            else
                rows_out(std::false_type{});
            raise_keys();
#undef MDR_ROW64
            continue;
        } else if constexpr (FAST) {
            // row r (0..32) is sgn or lo[32 - r]; unit of row r is (r + 3) / 4
            const uint32_t wave = tid >> 6;
            // four buffers: without a barrier at the top of the tile, a wave can
            // be one tile ahead of another, never two (the edge barrier below)
            const uint32_t par = (t - t0) & 3;
            if (lane == 63) {
                s_edge[par][wave][0] = sgn;
#pragma unroll
                for (int r = 1; r <= 32; ++r) s_edge[par][wave][r] = lo[32 - r];
            }
            if (t == t0 && tid == 0) {
                // the first block of the range has no left neighbour: it sees its
                // own words there (no transition).  Slot 3 of wave 3 is next
                // written three tiles later, after this tile's barrier.
                s_edge[3][3][0] = sgn;
#pragma unroll
                for (int r = 1; r <= 32; ++r) s_edge[3][3][r] = lo[32 - r];
                recs[((uint64_t)wg * kMaxRows) * 2] = sgn;
#pragma unroll
                for (int r = 1; r <= 32; ++r) recs[((uint64_t)wg * kMaxRows + r) * 2] = lo[32 - r];
            }
            __syncthreads();  // edges written; every thread is done with its y values
            const uint32_t* edge = wave ? &s_edge[par][wave - 1][0] : &s_edge[(par + 3) & 3][3][0];
            if (valid && blk == last_blk) {
                recs[((uint64_t)wg * kMaxRows) * 2 + 1] = sgn;
#pragma unroll
                for (int r = 1; r <= 32; ++r) recs[((uint64_t)wg * kMaxRows + r) * 2 + 1] = lo[32 - r];
            }
            // per row: coalesced store, nonzero bytes into the unit's histogram
            // (zero bytes are counted by difference later), and a transition
            // against the left neighbour's word, which the wave shift brings
            // from lane l-1 (lane 0: the previous wave's last word)
            auto rows_out = [&](auto full_tile) {
                constexpr bool FULL = decltype(full_tile)::value;
                // row base in scalar registers, advanced per row (kept out of the
                // tile loop's invariants, which would not fit), plus a 32-bit
                // byte offset: a level holds < 2^32 values, so blk * 4 < 2^29
                uint64_t rb = reinterpret_cast<uint64_t>(job.rows);
                asm volatile("" : "+s"(rb));
                const uint32_t boff = blk * 4u;
#pragma unroll
                for (int r = 0; r <= 32; ++r) {
                    const uint32_t w = r == 0 ? sgn : lo[32 - r];
                    const int unit = (r + 3) / 4;
                    if (FULL || valid) {
                        *gmem(reinterpret_cast<uint32_t*>(rb + boff)) = w;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t byte = (w >> (8 * q)) & 0xFFu;
                            if (byte) atomicAdd(&s_hist_fast[unit * 256 + byte], 1u);
                        }
                    }
                    // wave_shr:1 (lane l <- lane l-1); lane 0 keeps `old`
                    const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp((int)edge[r], (int)w, 0x138, 0xF, 0xF, false);
                    trc[unit] += ((FULL || valid) && w != nb) ? 1u : 0u;
                    rb += 4ull * nbd;
                }
            };
            if ((t + 1) * kTileBlocks <= nbd)
                rows_out(std::true_type{});
            else
                rows_out(std::false_type{});
            continue;
        }
        // Rows go through LDS in passes of at most kPassRows (f64's 65 rows in
        // two), so that two f64 workgroups fit a CU.
        const uint32_t nrows = B + 1;
        const uint32_t npass = nrows > kPassRows ? 2u : 1u;
        const uint32_t per = (nrows + npass - 1) / npass;
        const bool have_prev = t > t0;
        const bool lead = valid && (tid % G) == 0 && (tid >= G || have_prev);
        for (uint32_t pass = 0; pass < npass; ++pass) {
            const uint32_t rlo = pass * per, rhi = min(nrows, rlo + per);
            __syncthreads();  // every thread is done with its y values / the previous pass's rows
            if (rlo == 0) s_pl[tid] = sgn;
#pragma unroll
            for (int c = 0; c < 32; ++c) {
                const uint32_t r = B - (uint32_t)c;  // row of bit c (when c < B)
                if (c < (int)B && r >= rlo && r < rhi) s_pl[(r - rlo) * kTileBlocks + tid] = lo[c];
            }
            if constexpr (F64) {
#pragma unroll
                for (int c = 0; c < 32; ++c) {
                    const uint32_t r = B - 32u - (uint32_t)c;  // row of bit 32 + c
                    if (32 + c < (int)B && r >= rlo && r < rhi) s_pl[(r - rlo) * kTileBlocks + tid] = hi[c];
                }
            }
            __syncthreads();

            // ---- per row: coalesced store, byte histogram, word transitions.
            // Rows go four at a time so their LDS reads overlap; zero bytes are
            // counted by difference later and go to this thread's sink slot here.
            for (uint32_t r0 = rlo; r0 < rhi; r0 += 4) {
                uint32_t w[4], pv[4], pv1[4], nx[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t r = min(r0 + i, rhi - 1);
                    const uint32_t* row = s_pl + (r - rlo) * kTileBlocks;
                    w[i] = row[tid];
                    pv[i] = tid >= G ? row[tid - G] : s_prev[r][tid];
                    if constexpr (G == 2) {
                        nx[i] = row[tid + 1 < kTileBlocks ? tid + 1 : tid];
                        pv1[i] = tid >= G ? row[tid - 1] : s_prev[r][1];
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t r = r0 + i;
                    if (r >= rhi) break;
                    if (valid) {
                        rows[(uint64_t)r * nbd + blk] = w[i];
                        uint32_t* h = s_hist + s_hoff[r];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t byte = (w[i] >> (8 * q)) & 0xFFu;
                            atomicAdd(byte ? &h[byte] : &s_zero[tid], 1u);
                        }
                    }
                    bool flag = w[i] != pv[i];
                    if constexpr (G == 2) flag = flag || nx[i] != pv1[i];
                    unsigned long long bal = __ballot(lead && flag);
                    if (lane == 0 && bal) atomicAdd(&s_trans[r], (uint32_t)__popcll(bal));
                }
            }
            // first / last words of this workgroup's range, for the boundaries
            if (t == t0 && tid < G)
                for (uint32_t r = rlo; r < rhi; ++r)
                    recs[((uint64_t)wg * kMaxRows + r) * 2 * G + tid] = s_pl[(r - rlo) * kTileBlocks + tid];
            if (valid && blk + G > last_blk)
                for (uint32_t r = rlo; r < rhi; ++r)
                    recs[((uint64_t)wg * kMaxRows + r) * 2 * G + G + (blk - (last_blk + 1 - G))] =
                        s_pl[(r - rlo) * kTileBlocks + tid];
            __syncthreads();
            if (tid >= kTileBlocks - G)
                for (uint32_t r = rlo; r < rhi; ++r)
                    s_prev[r][tid - (kTileBlocks - G)] = s_pl[(r - rlo) * kTileBlocks + tid];
        }
        (void)NROW;
    }

    // ---- flush: per-workgroup partials (reduced by the selection kernel)
    if constexpr (FAST && F64) {
        // the rows' counts are in their slots already; the edge counts go to their row's
        if (edge_trc[0]) atomicAdd(&s_trans[lane], edge_trc[0]);
        if (lane == 0 && edge_trc[1]) atomicAdd(&s_trans[64], edge_trc[1]);
    } else if constexpr (FAST) {
        // a unit's transitions go to its first row's slot (the selection sums a unit's rows)
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            uint32_t v = trc[i];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (lane == 0 && v) atomicAdd(&s_trans[i == 0 ? 0 : 1 + (i - 1) * 4], v);
        }
    }
    small = wave_max(small);
    if constexpr (F64) {
        frac_max64 = wave_max(frac_max64);
        if (lane == 0) {
            atomicMax(&s_key64[B], (unsigned long long)frac_max64);
            atomicMax(&s_key64[kKeyStride - 1], (unsigned long long)__double_as_longlong(small));
        }
    } else {
        frac_max = wave_max(frac_max);
        if (lane == 0) {
            atomicMax(&s_key32[B], frac_max);
            atomicMax(&s_key32[kKeyStride - 1], __float_as_uint(small));
        }
    }
    __syncthreads();
    // fold this workgroup's results into its copy of the level totals (zeroed
    // before the pass): key maxima (nonnegative float bits order as integers),
    // nonzero byte counts and transitions
    const uint32_t copy = wg & (job.copies - 1);
    if (tid < kKeyStride) {
        const unsigned long long kv = F64 ? s_key64[tid] : (unsigned long long)s_key32[tid];
        if (kv) atomicMax(&job.keys[copy * kKeyStride + tid], kv);
    }
    for (uint32_t i = tid; i < nunits * 256; i += kThreads) {
        const uint32_t hv = s_hist[FAST ? (i >> 8) * HSTRIDE + (i & 255u) : i];
        if (hv) atomicAdd(&job.hist[copy * nunits * 256 + i], hv);
    }
    if (tid < kMaxRows && s_trans[tid]) atomicAdd(&job.trans[copy * kMaxRows + tid], s_trans[tid]);
}

// f32 fits five waves per SIMD (96 registers) with LDS to spare; general f64 two
// (256 registers, without spills: left alone the compiler takes 259 and one)
template <bool VEC, bool FAST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_encode_f32(
    const EncodeJob* __restrict__ jobs, const uint32_t* __restrict__ wg_job)
{
    const EncodeJob& job = jobs[wg_job[blockIdx.x]];
    encode_body<false, VEC, FAST>(job, blockIdx.x - job.wg_base);
}

template <bool VEC, bool FAST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_encode_f64(
    const EncodeJob* __restrict__ jobs, const uint32_t* __restrict__ wg_job)
{
    const EncodeJob& job = jobs[wg_job[blockIdx.x]];
    encode_body<true, VEC, FAST>(job, blockIdx.x - job.wg_base);
}

// the f64 fast path: four waves per SIMD (128 registers; a few scalars spill),
// as many as its LDS allows; within 2% of three (140 registers) from 2^28 values
// on, 4 to 8% faster on 2^23 and 2^24
template <bool VEC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_encode_f64_fast(
    const EncodeJob* __restrict__ jobs, const uint32_t* __restrict__ wg_job)
{
    const EncodeJob& job = jobs[wg_job[blockIdx.x]];
    encode_body<true, VEC, true>(job, blockIdx.x - job.wg_base);
}

// ------------------------------------------------------------------ bitplane encoder, small passes
// The same results for a pass of few values, where the kernels above leave most
// of the chip idle and a thread's 32 values, one after the other through 20 to
// 70 KB of unrolled code fetched cold, are the pass's latency (32768 values:
// 25 us in f32, 40 in f64, against 7 and 13 here).  Eight lanes share a block of 32 values,
// four values each (a wavefront reads 1 or 2 KiB in one go); the bit transpose
// exchanges words between the eight lanes in three rounds and finishes in
// registers; the tile's rows go through LDS and are stored, counted and compared
// by a rolled loop; and the error keys are taken directly: lane c walks the
// wavefront's aligned values in LDS and keeps the largest fraction at cut c.
// About twice the instructions a value of the kernels above, a sixth of the
// code.
template <bool F64>
__global__ __launch_bounds__(kThreads) void k_encode_small(const EncodeJob* __restrict__ jobs,
                                                           const uint32_t* __restrict__ wg_job)
{
    using T = std::conditional_t<F64, double, float>;
    constexpr int G = F64 ? 2 : 1;
    constexpr uint32_t kPad = kSmallTileBlocks + 1;
    extern __shared__ uint32_t s_dyn[];  // [nunits][256] byte histograms, then three tiles' rows [B + 1][kPad]
    __shared__ __align__(16) T s_y[kThreads / 64][256];
    __shared__ unsigned long long s_key[kKeyStride];
    __shared__ uint32_t s_trans[kMaxRows];
    __shared__ uint32_t s_hoff[kMaxRows];
    const EncodeJob& job = jobs[wg_job[blockIdx.x]];
    const uint32_t wg = blockIdx.x - job.wg_base;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = lane & 7;
    const uint32_t B = job.B, nbd = job.nbd, nunits = job.nunits;
    const uint64_t n = job.n;
    const uint64_t amax = job.stats->maxabs_bits;  // 0: every value is zero
    const int e = amax == 0 ? 0 : (F64 ? frexp_exp_f64(amax) : frexp_exp_f32((uint32_t)amax));
    const T* xg = static_cast<const T*>(job.x);
    const auto rows = gmem(job.rows);
    const auto recs = gmem(job.recs);
    uint32_t* s_hist = s_dyn;
    uint32_t* s_pl0 = s_dyn + nunits * 256;
    const uint32_t pl_words = (B + 1) * kPad;
    for (uint32_t i = tid; i < nunits * 256; i += kThreads) s_hist[i] = 0;
    if (tid < kMaxRows) {
        s_trans[tid] = 0;
        s_hoff[tid] = job.hist_off[tid];
    }
    if (tid < kKeyStride) s_key[tid] = 0;
    // exchange rounds with the lane 4, 2, 1 away: a lane keeps the bits of `keep`
    // and takes the others from its partner's word turned by `turn`
    const uint32_t keep16 = sub & 4 ? 0xFFFF0000u : 0x0000FFFFu, turn16 = 16;
    const uint32_t keep8 = sub & 2 ? 0xFF00FF00u : 0x00FF00FFu, turn8 = sub & 2 ? 8 : 24;
    const uint32_t keep4 = sub & 1 ? 0xF0F0F0F0u : 0x0F0F0F0Fu, turn4 = sub & 1 ? 4 : 28;
    auto transpose = [&](uint32_t (&a)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_ds_swizzle((int)a[i], 0x101F);  // lane ^ 4
            a[i] = (a[i] & keep16) | (__builtin_amdgcn_alignbit(o, o, turn16) & ~keep16);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a[i], 0x4E, 0xF, 0xF, false);  // lane ^ 2
            a[i] = (a[i] & keep8) | (__builtin_amdgcn_alignbit(o, o, turn8) & ~keep8);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a[i], 0xB1, 0xF, 0xF, false);  // lane ^ 1
            a[i] = (a[i] & keep4) | (__builtin_amdgcn_alignbit(o, o, turn4) & ~keep4);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t x = a[i], y = a[i + 2];
            a[i] = (x & 0x33333333u) | ((y << 2) & 0xCCCCCCCCu);
            a[i + 2] = ((x >> 2) & 0x33333333u) | (y & 0xCCCCCCCCu);
        }
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            const uint32_t x = a[i], y = a[i + 1];
            a[i] = (x & 0x55555555u) | ((y << 1) & 0xAAAAAAAAu);
            a[i + 1] = ((x >> 1) & 0x55555555u) | (y & 0xAAAAAAAAu);
        }
    };
    const uint32_t t0 = wg * job.tiles_per_wg, t1 = min(job.ntiles, t0 + job.tiles_per_wg);
    const uint32_t nrows = B + 1;
    // f32: two halves of a wavefront walk its values for the same 32 cuts
    constexpr uint32_t kWalk = F64 ? 256 : 128;
    const uint32_t cut = F64 ? lane : lane & 31;
    T km = 0, small = 0;
    __syncthreads();
    for (uint32_t t = t0; t < t1; ++t) {
        // three buffers: a wavefront may fill the next tile's while another
        // still reads this one's and the last words of the one before
        uint32_t* s_pl = s_pl0 + (t - t0) % 3 * pl_words;
        const uint32_t* s_before = s_pl0 + (t - t0 + 2) % 3 * pl_words;
        const uint32_t blk0 = t * kSmallTileBlocks, lblk = wave * 8 + (lane >> 3);
        // ---- four values a lane, aligned: y = |x| 2^(B-e), mag = floor(y)
        const uint64_t i0 = (uint64_t)(blk0 + lblk) * 32 + 4 * sub;
        T v[4];
        if (i0 + 4 <= n) {
            constexpr int W = sizeof(T) / 4;  // 16-byte pieces of four values
            uint32_t w[4 * W];
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const u32x4_any q = gmem(reinterpret_cast<const u32x4_any*>(xg + i0))[k];
                w[4 * k] = q.x, w[4 * k + 1] = q.y, w[4 * k + 2] = q.z, w[4 * k + 3] = q.w;
            }
            __builtin_memcpy(v, w, sizeof w);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = i0 + j < n ? gmem(xg)[i0 + j] : T(0);
        }
        uint32_t sgn = 0, lo[4], hi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T y;
            if constexpr (F64) {
                const uint64_t bits = (uint64_t)__double_as_longlong(v[j]);
                sgn |= (uint32_t)(bits >> 63) << j;
                const double a = __longlong_as_double((long long)(bits & 0x7FFFFFFFFFFFFFFFull));
                y = __builtin_amdgcn_ldexp(a, (int)B - e);
                if (y < 1.0) {  // mag = 0: below every cut
                    small = a > small ? a : small;
                    y = 0.0;
                }
                const double yh = __builtin_trunc(y * 0x1p-32);
                hi[j] = (uint32_t)yh;
                lo[j] = (uint32_t)(y - yh * 0x1p32);
            } else {
                const uint32_t bits = __float_as_uint(v[j]);
                sgn |= (bits >> 31) << j;
                const float a = __uint_as_float(bits & 0x7FFFFFFFu);
                y = __builtin_amdgcn_ldexpf(a, (int)B - e);
                if (y < 1.0f) {
                    small = a > small ? a : small;
                    y = 0.0f;
                }
                lo[j] = (uint32_t)y;
                hi[j] = 0;
            }
            s_y[wave][(lane << 2) + j] = y;
        }
        // ---- the block's sign word, then the plane words of bits 4 sub .. 4 sub + 3 (and 32 more)
        sgn <<= 4 * sub;
        sgn |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sgn, 0xB1, 0xF, 0xF, false);
        sgn |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sgn, 0x4E, 0xF, 0xF, false);
        sgn |= (uint32_t)__builtin_amdgcn_ds_swizzle((int)sgn, 0x101F);
        transpose(lo);
        if constexpr (F64) transpose(hi);
        if (sub == 0) s_pl[lblk] = sgn;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t c = 4 * sub + i;  // bit c is row B - c
            if (c < B) s_pl[(B - c) * kPad + lblk] = lo[i];
            if (F64 && 32 + c < B) s_pl[(B - 32 - c) * kPad + lblk] = hi[i];
        }
        // ---- error keys: cut c = B - k (k = 1 .. B) of the wavefront's values
        wave_fence();
        if (cut < B) {
            const T* yw = s_y[wave] + (F64 ? 0 : (lane >> 5) * kWalk);
#pragma unroll 4
            for (uint32_t i = 0; i < kWalk; i += 16 / sizeof(T)) {
#pragma unroll
                for (uint32_t q = 0; q < 16 / sizeof(T); ++q) {
                    T key;
                    if constexpr (F64) {
                        key = __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(yw[i + q], -(int)cut));
                        km = __builtin_fmax(km, key);
                    } else {
                        key = __builtin_amdgcn_fractf(__builtin_amdgcn_ldexpf(yw[i + q], -(int)cut));
                        km = __builtin_fmaxf(km, key);
                    }
                }
            }
        }
        __syncthreads();  // the tile's rows are in LDS
        // ---- per row: store, count the nonzero bytes, compare with the left neighbour
        for (uint32_t i = tid; i < nrows * kSmallTileBlocks; i += kThreads) {
            const uint32_t r = i / kSmallTileBlocks, b = i % kSmallTileBlocks, blk = blk0 + b;
            const uint32_t* row = s_pl + r * kPad;
            const uint32_t w = row[b];
            const bool valid = blk < nbd;
            bool flag = false;
            if (valid) {
                rows[(uint64_t)r * nbd + blk] = w;
                uint32_t* h = s_hist + s_hoff[r];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t byte = (w >> (8 * q)) & 0xFFu;
                    if (byte) atomicAdd(&h[byte], 1u);
                }
                if (b % G == 0 && (b >= G || t > t0)) {  // a W-bit word against the one before it
                    const uint32_t* left = b >= G ? row + b : s_before + r * kPad + kSmallTileBlocks;
                    flag = w != left[-G];
                    if (G == 2) flag = flag || row[b + 1] != left[-1];
                }
                // the range's first and last words, for the boundaries between ranges
                if (t == t0 && b < G) recs[((uint64_t)wg * kMaxRows + r) * 2 * G + b] = w;
                const uint32_t last = min(nbd, t1 * kSmallTileBlocks);
                if (blk + G >= last) recs[((uint64_t)wg * kMaxRows + r) * 2 * G + G + (blk + G - last)] = w;
            }
            // a row's 32 words sit in one half of a wavefront
            const unsigned long long bal = __ballot(flag);
            const uint32_t cnt = (uint32_t)__popc((uint32_t)(bal >> (lane & 32)));
            if (b == 0 && cnt) atomicAdd(&s_trans[r], cnt);
        }
    }
    // ---- flush: the workgroup's results into its copy of the level totals (zeroed before the pass)
    if (cut < B) {
        if constexpr (F64)
            atomicMax(&s_key[B - cut], (unsigned long long)__double_as_longlong(km));
        else
            atomicMax(&s_key[B - cut], (unsigned long long)__float_as_uint(km));
    }
    small = wave_max(small);
    if (lane == 0) {
        if constexpr (F64)
            atomicMax(&s_key[kKeyStride - 1], (unsigned long long)__double_as_longlong(small));
        else
            atomicMax(&s_key[kKeyStride - 1], (unsigned long long)__float_as_uint(small));
    }
    __syncthreads();
    const uint32_t copy = wg & (job.copies - 1);
    if (tid < kKeyStride && s_key[tid]) atomicMax(&job.keys[copy * kKeyStride + tid], s_key[tid]);
    for (uint32_t i = tid; i < nunits * 256; i += kThreads)
        if (s_hist[i]) atomicAdd(&job.hist[copy * nunits * 256 + i], s_hist[i]);
    if (tid < kMaxRows && s_trans[tid]) atomicAdd(&job.trans[copy * kMaxRows + tid], s_trans[tid]);
}

// ------------------------------------------------------------------ hybrid selection
// Working memory of one code construction (one wavefront).  W: the weights'
// type, 32 bits while a unit has fewer than 2^30 bytes.
template <typename W>
struct CodeScratch {
    W w[512];            // node weights: leaves [0, nl) ascending, merged nodes from nl
    W ow[128];           // a round's nodes in merged order: weights
    uint32_t ord[128];   // ... and node numbers
    uint32_t par[512];   // parent of every node; then depth << 16 | ancestor of merged nodes
    uint32_t bits[256];  // codes per length
};

// Code lengths of the nl >= 2 symbols sym[0, nl) (ascending (count, symbol)
// order, weights in cs.w): the two-queue Huffman tree, leaf queue first on
// weight ties, then the count adjustment of ITU-T T.81 Annex K when it is
// deeper than lmax.  Runs on one wavefront; returns the longest length.
//
// The tree is built in rounds instead of one merge at a time: with t the sum
// of the two smallest nodes, every node of weight <= t goes before any node
// that is yet to be made (a new node weighs at least t, and on a tie leaves
// and older nodes go first), so all of them pair up at once in merged order; an
// odd last one waits for the next round.  A round looks at the first 64 of
// each queue; what lies past a full window bounds what the other may give.
// Serial merging on one lane, with its dependent LDS picks, was most of a
// selection launch: 71 us for the 45 units of a 32768-value variable.
template <typename W>
__device__ __forceinline__ uint32_t huf_lengths(CodeScratch<W>& cs, const uint32_t* sym, int nl, uint32_t lmax, uint8_t* len, uint32_t lane)
{
    constexpr W kNone = ~W(0) >> 1;   // above any weight; the sum of two does not wrap
    int q1 = 0, q2 = nl, next = nl;  // heads of the leaf and merged queues, end of the latter
    while ((nl - q1) + (next - q2) > 1) {
        const int nlf = nl - q1, nin = next - q2;
        const W wl = (int)lane < nlf ? cs.w[q1 + lane] : kNone;
        const W wi = (int)lane < nin ? cs.w[q2 + lane] : kNone;
        const W l0 = lane_value(wl, 0), l1 = lane_value(wl, 1);
        const W i0 = lane_value(wi, 0), i1 = lane_value(wi, 1);
        W t = l0 + l1;
        t = l0 + i0 < t ? l0 + i0 : t;
        t = i0 + i1 < t ? i0 + i1 : t;
        // a window that is full to its end (more nodes <= t may follow): leaves
        // past it go before merged nodes of at least their weight, merged nodes
        // past it before leaves of more than theirs
        const W lw = lane_value(wl, 63), iw = lane_value(wi, 63);
        const bool sat_l = nlf > 64 && lw <= t, sat_i = nin > 64 && iw <= t;
        const bool in_l = wl <= t && (!sat_i || wl <= iw);
        const bool in_i = wi <= t && (!sat_l || wi < lw);
        const int cl = __popcll(__ballot(in_l)), ci = __popcll(__ballot(in_i));
        if (cl + ci <= 3) {  // a single merge, of the two smallest: leaves first on a tie
            const int leaves = l0 <= i0 ? (l1 <= i0 ? 2 : 1) : (l0 <= i1 ? 1 : 0);
            if (lane < 2) cs.par[(int)lane < leaves ? q1 + (int)lane : q2 + (int)lane - leaves] = (uint32_t)next;
            if (lane == 2) cs.w[next] = t;
            q1 += leaves;
            q2 += 2 - leaves;
            ++next;
            wave_fence();
            continue;
        }
        // positions in merged order, by a walk over the shorter side
        int pl = (int)lane, pi = (int)lane;
        if (ci <= cl) {
            for (int j = 0; j < ci; ++j) {
                const W v = lane_value(wi, j);
                const int before = __popcll(__ballot(in_l && wl <= v));
                pl += v < wl ? 1 : 0;
                pi = (int)lane == j ? j + before : pi;
            }
        } else {
            for (int j = 0; j < cl; ++j) {
                const W v = lane_value(wl, j);
                const int before = __popcll(__ballot(in_i && wi < v));
                pi += v <= wi ? 1 : 0;
                pl = (int)lane == j ? j + before : pl;
            }
        }
        if (in_l) {
            cs.ord[pl] = (uint32_t)(q1 + (int)lane);
            cs.ow[pl] = wl;
        }
        if (in_i) {
            cs.ord[pi] = (uint32_t)(q2 + (int)lane);
            cs.ow[pi] = wi;
        }
        wave_fence();
        const int P = cl + ci, np = P >> 1;
        if ((int)lane < np) {
            // all four reads before the writes: one LDS round trip
            const uint32_t node = (uint32_t)(next + (int)lane), na = cs.ord[2 * lane], nb = cs.ord[2 * lane + 1];
            const W wa = cs.ow[2 * lane], wb = cs.ow[2 * lane + 1];
            cs.w[node] = wa + wb;
            cs.par[na] = node;
            cs.par[nb] = node;
        }
        const bool odd_leaf = cl > 0 && __builtin_amdgcn_readlane(pl, cl - 1) == P - 1;
        q1 += cl - ((P & 1) && odd_leaf ? 1 : 0);
        q2 += ci - ((P & 1) && !odd_leaf ? 1 : 0);
        next += np;
        wave_fence();
    }

    // depths of the merged nodes (numbers nl .. 2 nl - 2, the last the root) by
    // pointer jumping, four nodes a lane; then each leaf's is its parent's plus one
    const uint32_t root = (uint32_t)(2 * nl - 2);
    uint32_t dp[4], lp[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const uint32_t leaf = lane + 64 * h, v = (uint32_t)nl + leaf;
        lp[h] = (int)leaf < nl ? cs.par[leaf] : 0u;
        dp[h] = v < root ? (1u << 16) | cs.par[v] : root;  // depth so far << 16 | ancestor at that distance
    }
    wave_fence();
    for (;;) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t v = (uint32_t)nl + lane + 64 * h;
            if (v <= root) cs.par[v] = dp[h];
        }
        wave_fence();
        bool open = false;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t v = (uint32_t)nl + lane + 64 * h;
            open = open || (v < root && (dp[h] & 0xFFFFu) != root);
        }
        if (__ballot(open) == 0) break;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t a = cs.par[dp[h] & 0xFFFFu];
            dp[h] = (dp[h] & 0xFFFF0000u) + a;
        }
        wave_fence();  // everyone has read before the next round writes
    }
    uint32_t d[4], most = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const uint32_t leaf = lane + 64 * h;
        d[h] = (int)leaf < nl ? (cs.par[lp[h]] >> 16) + 1 : 0u;
        most = d[h] > most ? d[h] : most;
    }
    most = wave_max(most);
    if (most > lmax) {
#pragma unroll
        for (int h = 0; h < 4; ++h) cs.bits[lane + 64 * h] = 0;
        wave_fence();
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if (d[h]) atomicAdd(&cs.bits[d[h]], 1u);
        wave_fence();
        // Lane l holds the count of length l.  Lengths stay below 64: a tree of
        // depth d takes weights of Fibonacci(d + 2) in all, and a unit has at
        // most 2^35 bytes (64 rows of 2^27 words): d <= 50.
        int b = (int)cs.bits[lane];
        // Per step, two codes of the deepest length i: one moves up to i - 1,
        // the other to a code split at the longest shorter length j <= i - 2
        // that has one (j -> two of j + 1).  Splitting one code of length j
        // all the way down to i - 1, as consecutive steps do, takes
        // T = 2^(i-1-j) - 1 steps and leaves 2^(i-1-j) codes there, so
        // codes are split whole while the steps last; of the next one the
        // steps left split a path (at each length one code stays, or is
        // split whole).  (One step at a time was up to 50 us of a large
        // skewed unit's selection.)
        const int l = (int)lane;
        for (int i = (int)most; i > (int)lmax; --i) {
            int left = __builtin_amdgcn_readlane(b, i) >> 1;  // steps at this length, at most 127
            b += (l == i ? -2 * left : 0) + (l == i - 1 ? left : 0);
            while (left > 0) {
                const unsigned long long nzm = __ballot(b != 0) & ((1ull << (i - 1)) - 1);
                if (!nzm) break;  // cannot happen for a full tree
                const int j = 63 - __clzll((long long)nzm);
                int d = i - 1 - j, T = (1 << min(d, 16)) - 1;  // 16 levels stand for more: T > left
                const int bj = __builtin_amdgcn_readlane(b, j);
                // left / T, exact for these small numbers
                int q = (int)((float)left * __builtin_amdgcn_rcpf((float)T) + 1e-3f);
                q = min(__builtin_amdgcn_readfirstlane(q), bj);
                left -= q * T;
                int deep = q << min(d, 16);       // codes left at i - 1
                unsigned long long stay = 0;      // lengths that keep one code of the split path
                if (q < bj && left > 0) {
                    ++q;                          // the partly split code
                    for (int c = j; left > 0;) {
                        --left;                   // split: two of length c + 1
                        ++c;
                        --d;
                        T = (1 << min(d, 16)) - 1;
                        if (left >= T) {          // one of them whole (T = 0 at c = i - 1)
                            left -= T;
                            deep += 1 << d;
                        } else {
                            stay |= 1ull << c;
                        }
                        if (left == 0) {          // the other stays as it is
                            if (d == 0)
                                ++deep;
                            else
                                b += l == c ? 1 : 0;
                        }
                    }
                }
                b += (l == j ? -q : 0) + (l == i - 1 ? deep : 0) + (int)((stay >> l) & 1);
            }
        }
        // hand the lengths out again, the heaviest leaf (last) the shortest
        uint32_t cum = 0, nd[4] = {1, 1, 1, 1};
        for (uint32_t L = 1; L < lmax; ++L) {
            cum += (uint32_t)__builtin_amdgcn_readlane(b, (int)L);
#pragma unroll
            for (int h = 0; h < 4; ++h) nd[h] += (uint32_t)(nl - 1) - (lane + 64 * h) >= cum ? 1u : 0u;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) d[h] = nd[h];
        most = lmax;
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const uint32_t leaf = lane + 64 * h;
        if ((int)leaf < nl) len[sym[leaf]] = (uint8_t)d[h];
    }
    return most;
}

// One workgroup of NT threads per (unit, level) (Alg. 2): gather the byte
// histogram and the run count, build length-limited Huffman code lengths with
// the two-queue construction, canonical codes, both size estimates, and the
// method decision.  Units that Alg. 2 can only copy (S <= T_s) skip the
// codebook, and so do units whose entropy already rules Huffman out: every
// prefix code takes at least the entropy, so when that (less a margin far above
// its rounding) plus the stream's overhead fails Alg. 2's test, the code's own
// estimate fails it too, and nothing else reads the code.
// NT = 256, 512 or 1024 threads (a launch knob): the code is built by one
// wavefront, so smaller workgroups let more units build theirs at once, while
// the boundary and rank steps of a few large units go faster with more threads.
template <int NT, typename W>
__global__ __launch_bounds__(NT) void k_select(const SelectParams job, const SelectLevel* __restrict__ levels)
{
    constexpr uint32_t kWaves = NT / 64;
    __shared__ __align__(16) unsigned long long s_key[256];  // count << 8 | symbol, ~0 when absent
    __shared__ CodeScratch<W> s_cs;
    __shared__ uint32_t s_rank[256];
    __shared__ uint32_t s_sorted[256];
    __shared__ uint8_t s_len[256];
    __shared__ unsigned long long s_red[kWaves], s_red2[kWaves];
    __shared__ unsigned long long s_bits[4];
    __shared__ double s_redf[4];
    __shared__ uint32_t s_cnt[4][kLutBitsMax + 1];
    __shared__ uint32_t s_maxlen;

    const SelectLevel& lv = levels[blockIdx.y];
    const uint32_t u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t B = job.B, m = job.m, G = job.G, grid = lv.grid;
    const uint32_t r0 = u == 0 ? 0 : 1 + (u - 1) * m;
    const uint32_t r1 = u == 0 ? 1 : min(B + 1, r0 + m);
    const uint64_t S = (uint64_t)(r1 - r0) * lv.nbd * 4;
    if (lv.nbd == 0) {
        // empty level: no planes; every unit is an empty stream of the forced
        // method (direct copy under Alg. 2)
        if (tid < 256) {
            lv.lens[u * 256 + tid] = 0;
            lv.codes[u * 256 + tid] = 0;
        }
        if (tid == 0) {
            UnitInfo ui;
            ui.S = 0;
            ui.est_huf = 8 + 256 + 4;
            ui.est_rle = 8;
            ui.nruns = 0;
            ui.method = job.force_method >= 0 ? (uint32_t)job.force_method : 0u;
            ui.nchunks = 0;
            ui.maxlen = 0;
            ui.pad = 0;
            lv.units[u] = ui;
            lv.work[u] = (uint64_t)ui.method << 62;
            lv.bytes[u] = ui.method == 2 ? kHufHeaderBytes + 4 : ui.method == 1 ? 8 : 0;
        }
        return;
    }

    auto wave_sum64 = [](unsigned long long v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        return v;
    };

    // ---- byte histogram (the copies of the level's totals from the encoder)
    const uint32_t copies = lv.copies;
    unsigned long long f = 0;
    if (tid < 256) {
        const auto h = gmem(lv.hist) + u * 256 + tid;
#pragma unroll 8
        for (uint32_t c = 0; c < copies; ++c) f += h[(uint64_t)c * job.nunits * 256];
    }
    if (u == 0 && tid < kKeyStride) {
        unsigned long long k = 0;
#pragma unroll 8
        for (uint32_t c = 0; c < copies; ++c) {
            const unsigned long long v = gmem(lv.keys)[c * kKeyStride + tid];
            k = v > k ? v : k;
        }
        lv.keys_out[tid] = k;
    }

    // ---- runs of equal W-bit words: transitions inside workgroup ranges (level
    // totals from the encoder), at range boundaries, and between consecutive
    // planes of the group
    const uint32_t nrow = r1 - r0;
    unsigned long long tr = 0;
    for (uint32_t i = tid; i < nrow * copies; i += NT) tr += gmem(lv.trans)[i / nrow * kMaxRows + r0 + i % nrow];
    {
        // boundary i: first word(s) of range w = 1 + i / nrow against the last
        // of range w - 1, row r0 + i % nrow, eight boundaries a thread in
        // flight; a record holds a row's first and last word (G = 1), or its
        // first two and last two, in 8-byte pieces
        constexpr int kFly = 8;
        const auto recs = gmem(lv.recs);
        const auto pieces = gmem(reinterpret_cast<const uint64_t*>(lv.recs));
        const uint32_t nbnd = (grid - 1) * nrow;
        // i / nrow by a multiplication: exact while i * nrow < 2^32, and
        // i < 65536 * 65 (encoder workgroups of a level, rows)
        const uint32_t inv = 0xFFFFFFFFu / nrow + 1;
        for (uint32_t i0 = tid; i0 < nbnd; i0 += kFly * NT) {
            uint64_t cw[kFly], pw[kFly];
#pragma unroll
            for (int k = 0; k < kFly; ++k) {
                const uint32_t i = min(i0 + k * NT, nbnd - 1);
                const uint32_t w = nrow == 1 ? i : __umulhi(i, inv), r = r0 + i - w * nrow;  // range w + 1
                cw[k] = pieces[((uint64_t)(w + 1) * kMaxRows + r) * G];
                pw[k] = pieces[((uint64_t)w * kMaxRows + r) * G + G - 1];
            }
#pragma unroll
            for (int k = 0; k < kFly; ++k) {
                const bool ne = G == 1 ? (uint32_t)cw[k] != (uint32_t)(pw[k] >> 32) : cw[k] != pw[k];
                tr += i0 + k * NT < nbnd && ne ? 1u : 0u;
            }
        }
        for (uint32_t r = r0 + 1 + tid; r < r1; r += NT) {
            const uint64_t cur = (uint64_t)r * 2 * G;
            const uint64_t prv = ((uint64_t)(grid - 1) * kMaxRows + (r - 1)) * 2 * G;
            bool ne = false;
            for (uint32_t g = 0; g < G; ++g) ne = ne || recs[cur + g] != recs[prv + G + g];
            tr += ne ? 1 : 0;
        }
    }
    {
        const unsigned long long nzw = wave_sum64(tid > 0 && tid < 256 ? f : 0);
        const unsigned long long trw = wave_sum64(tr);
        if (lane == 0) {
            s_red[wave] = nzw;
            s_red2[wave] = trw;
        }
        if (tid < 256) {
            s_rank[tid] = 0;
            s_len[tid] = 0;
        }
        if (tid == 0) s_maxlen = 0;
    }
    __syncthreads();
    unsigned long long nz = 0, trans = 0;
    for (uint32_t w = 0; w < kWaves; ++w) {
        nz += s_red[w];
        trans += s_red2[w];
    }
    if (tid == 0) f = S - nz;  // zero bytes are not counted by the encoder
    const unsigned long long nruns = 1 + trans;
    const uint64_t nchunks = (S + job.huf_chunk - 1) / job.huf_chunk;
    bool need_code = job.force_method == 2 || (job.force_method < 0 && S > job.t_s);
    double ent = 0.0;
    if (need_code) {
        if (tid < 256) {
            s_key[tid] = f ? (f << 8) | tid : ~0ull;
            // entropy in bits (float logarithms: a relative error of about 1e-6)
            double h = f ? (double)f * (double)(__log2f((float)S) - __log2f((float)f)) : 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) h += __shfl_xor(h, off, 64);
            const unsigned long long pm = __ballot(f != 0);
            if (lane == 0) {
                s_redf[wave] = h;
                s_cnt[wave][0] = (uint32_t)__popcll(pm);
            }
        }
        __syncthreads();
        ent = (s_redf[0] + s_redf[1]) + (s_redf[2] + s_redf[3]);
        if (job.force_method < 0) {
            const double low = ent * (0.9999 / 8) + (double)(8 + 256 + 4 * (nchunks + 1)) - 1e-4 * (double)S;
            need_code = !(1000.0 * (double)S < (double)job.t_cr_milli * low);
        }
    }

    // ---- Huffman code lengths
    if (need_code) {
        // rank of each present symbol in (count, symbol) order: kRankParts
        // threads per symbol, 256 / kRankParts comparisons each
        constexpr uint32_t kRankParts = kWaves / 4;
        constexpr uint32_t kSpan = 256 / kRankParts;
        const uint32_t s = tid & 255, part = tid >> 8;
        const unsigned long long key = s_key[s];
        uint32_t r = 0;
#pragma unroll 8
        for (uint32_t q = part * kSpan; q < part * kSpan + kSpan; ++q) r += s_key[q] < key ? 1u : 0u;
        if (kRankParts > 1) {
            if (r) atomicAdd(&s_rank[s], r);
            __syncthreads();
            r = s_rank[s];
        }
        const int nl = (int)(s_cnt[0][0] + s_cnt[1][0] + s_cnt[2][0] + s_cnt[3][0]);
        if (part == 0 && key != ~0ull) {
            s_sorted[r] = s;
            s_cs.w[r] = (W)(key >> 8);
        }
        __syncthreads();
        if (wave == 0) {
            if (nl == 1) {  // a phantom partner, the smallest other symbol
                if (lane == 0) {
                    const uint32_t s0 = s_sorted[0];
                    s_len[s0] = 1;
                    s_len[s0 == 0 ? 1 : 0] = 1;
                    s_maxlen = 1;
                }
            } else {
                const uint32_t most = huf_lengths(s_cs, s_sorted, nl, job.huf_lmax, s_len, lane);
                if (lane == 0) s_maxlen = most;
            }
        }
        __syncthreads();
    }

    // ---- canonical codes: (length, symbol) order.  A symbol's place among the
    // codes of its length: ballots within its wavefront, then the earlier ones'
    const uint32_t L = tid < 256 ? s_len[tid] : 0;
    uint32_t before = 0;
    unsigned long long bits = 0;
    if (tid < 256) {
        if (need_code) {
            uint32_t mine = 0;  // lane l: this wavefront's symbols of length l
#pragma unroll
            for (uint32_t l = 1; l <= (uint32_t)kLutBitsMax; ++l) {
                const unsigned long long bl = __ballot(L == l);
                mine = lane == l ? (uint32_t)__popcll(bl) : mine;
                if (L == l) before = (uint32_t)__popcll(bl & ((1ull << lane) - 1));
            }
            if (lane >= 1 && lane <= (uint32_t)kLutBitsMax) s_cnt[wave][lane] = mine;
        }
        bits = wave_sum64(f * (unsigned long long)L);
        if (lane == 0) s_bits[wave] = bits;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t code = 0;
        if (need_code) {
            // lane l: symbols of length l in all, and in the earlier wavefronts
            uint32_t all = 0, earlier = 0;
            if (lane >= 1 && lane <= (uint32_t)kLutBitsMax) {
#pragma unroll
                for (uint32_t w = 0; w < 4; ++w) {
                    const uint32_t c = s_cnt[w][lane];
                    all += c;
                    earlier += w < wave ? c : 0u;
                }
            }
            uint32_t first = 0;
#pragma unroll
            for (uint32_t l = 1; l <= (uint32_t)kLutBitsMax; ++l) {
                if (L == l) code = first + lane_value(earlier, (int)l) + before;
                first = (first + lane_value(all, (int)l)) << 1;
            }
        }
        lv.lens[u * 256 + tid] = (uint8_t)L;
        lv.codes[u * 256 + tid] = code;
    }

    // ---- estimates and the decision
    if (tid == 0) {
        bits = s_bits[0] + s_bits[1] + s_bits[2] + s_bits[3];
        // (0 for a unit without a code: its Huffman estimate is not needed)
        const uint64_t est_huf = need_code ? (bits + 7) / 8 + 8 + 256 + 4 * (nchunks + 1) : 0;
        const uint64_t est_rle = 8 + nruns * (4ull * G + 4);
        uint32_t method;
        if (job.force_method >= 0) {
            method = (uint32_t)job.force_method;
        } else if (S > job.t_s) {
            if (need_code && 1000ull * S > (uint64_t)job.t_cr_milli * est_huf)
                method = 2;  // MDR_HUF
            else if (1000ull * S > (uint64_t)job.t_cr_milli * est_rle)
                method = 1;  // MDR_RLE
            else
                method = 0;  // MDR_DC
        } else {
            method = 0;
        }
        UnitInfo ui;
        ui.S = S;
        ui.est_huf = est_huf;
        ui.est_rle = est_rle;
        ui.nruns = nruns;
        ui.method = method;
        ui.nchunks = (uint32_t)nchunks;
        ui.maxlen = s_maxlen;
        ui.pad = 0;
        lv.units[u] = ui;
        const uint64_t tiles = (S / (4ull * G) + kRleTileWords - 1) / kRleTileWords;
        lv.work[u] = (uint64_t)method << 62 | (method == 2 ? nchunks : method == 1 ? tiles << 32 : 0);
        lv.bytes[u] = method == 2 ? kHufHeaderBytes + 4 * (nchunks + 1) : method == 1 ? est_rle : S;
    }
}

}  // namespace

// ------------------------------------------------------------------ launchers
static unsigned grid_for(uint64_t items, unsigned per_block, unsigned cap)
{
    uint64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t count, uint32_t value, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(count, kThreads, 4096)), dim3(kThreads), 0, s, p,
                       count, value);
    return hipGetLastError();
}

hipError_t launch_copy_in(void* dst, const void* host, uint64_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    if (bytes % 8) return hipErrorInvalidValue;
    void* src = nullptr;
    hipError_t e = hipHostGetDevicePointer(&src, const_cast<void*>(host), 0);
    if (e != hipSuccess) return e;
    const uint64_t count = bytes / 8;
    hipLaunchKernelGGL(k_copy_in, dim3(grid_for(count, kThreads, 1024)), dim3(kThreads), 0, s,
                       static_cast<const uint64_t*>(src), static_cast<uint64_t*>(dst), count);
    return hipGetLastError();
}

hipError_t launch_begin_pass(void* dst, const void* host, uint64_t bytes, LevelStats* st, uint32_t count, void* z,
                             uint64_t zbytes, hipStream_t s)
{
    if (bytes == 0 || bytes % 8 || zbytes % 16) return hipErrorInvalidValue;
    void* src = nullptr;
    hipError_t e = hipHostGetDevicePointer(&src, const_cast<void*>(host), 0);
    if (e != hipSuccess) return e;
    const uint64_t words = bytes / 8, n4 = zbytes / 16;
    const unsigned copy_wg = grid_for(words, kThreads, 1024);
    const unsigned fill_wg = grid_for(std::max<uint64_t>(count, n4), kThreads, 3072);
    hipLaunchKernelGGL(k_begin_pass, dim3(copy_wg + fill_wg), dim3(kThreads), 0, s, static_cast<const uint64_t*>(src),
                       static_cast<uint64_t*>(dst), words, copy_wg, st, count, static_cast<u32x4*>(z), n4);
    return hipGetLastError();
}

hipError_t launch_stats_batch(const StatsJob* jobs, const uint32_t* wg_job, uint32_t grid, bool f64,
                              bool vec, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    if (f64) {
        if (vec)
            hipLaunchKernelGGL((k_stats<true, true>), dim3(grid), dim3(kStatsThreads), 0, s, jobs, wg_job);
        else
            hipLaunchKernelGGL((k_stats<true, false>), dim3(grid), dim3(kStatsThreads), 0, s, jobs, wg_job);
    } else {
        if (vec)
            hipLaunchKernelGGL((k_stats<false, true>), dim3(grid), dim3(kStatsThreads), 0, s, jobs, wg_job);
        else
            hipLaunchKernelGGL((k_stats<false, false>), dim3(grid), dim3(kStatsThreads), 0, s, jobs, wg_job);
    }
    return hipGetLastError();
}

size_t encode_lds_bytes(uint32_t nunits, uint32_t B, uint32_t m, bool f64)
{
    if ((!f64 && B == 32 && m == 4) || (f64 && B == 64 && m == 4)) return 0;  // the fast paths: static LDS only
    const uint32_t npass = B + 1 > kPassRows ? 2u : 1u;  // as the kernel stages its rows
    const size_t planes = (size_t)((B + 1 + npass - 1) / npass) * kTileBlocks * sizeof(uint32_t);
    return (size_t)nunits * 256 * sizeof(uint32_t) + planes;
}

size_t encode_small_lds_bytes(uint32_t nunits, uint32_t B)
{
    return (size_t)nunits * 256 * sizeof(uint32_t) + 3ull * (B + 1) * (kSmallTileBlocks + 1) * sizeof(uint32_t);
}

hipError_t encode_set_lds(uint32_t nunits, uint32_t B, uint32_t m, bool f64, bool small)
{
    if (small) {
        if (encode_small_lds_bytes(nunits, B) <= 48 * 1024) return hipSuccess;  // beside up to 10 KB of its own
        const void* fn = f64 ? (const void*)k_encode_small<true> : (const void*)k_encode_small<false>;
        return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)encode_small_lds_bytes(nunits, B));
    }
    const size_t shmem = encode_lds_bytes(nunits, B, m, f64);
    if (shmem <= 64 * 1024) return hipSuccess;  // the fast path always fits
    const void* fns[2] = {f64 ? (const void*)k_encode_f64<true, false> : (const void*)k_encode_f32<true, false>,
                          f64 ? (const void*)k_encode_f64<false, false> : (const void*)k_encode_f32<false, false>};
    for (const void* fn : fns) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_encode_batch(const EncodeJob* jobs, const uint32_t* wg_job, uint32_t grid,
                               uint32_t nunits, uint32_t B, uint32_t m, bool f64, bool vec, hipStream_t s)
{
    const bool fast = (!f64 && B == 32 && m == 4) || (f64 && B == 64 && m == 4);
    if (grid == 0) return hipSuccess;
    const size_t shmem = encode_lds_bytes(nunits, B, m, f64);
    dim3 g(grid), b(kThreads);
    if (f64) {
        if (fast) {
            if (vec)
                hipLaunchKernelGGL((k_encode_f64_fast<true>), g, b, shmem, s, jobs, wg_job);
            else
                hipLaunchKernelGGL((k_encode_f64_fast<false>), g, b, shmem, s, jobs, wg_job);
        } else {
            if (vec)
                hipLaunchKernelGGL((k_encode_f64<true, false>), g, b, shmem, s, jobs, wg_job);
            else
                hipLaunchKernelGGL((k_encode_f64<false, false>), g, b, shmem, s, jobs, wg_job);
        }
    } else {
        if (fast) {
            if (vec)
                hipLaunchKernelGGL((k_encode_f32<true, true>), g, b, shmem, s, jobs, wg_job);
            else
                hipLaunchKernelGGL((k_encode_f32<false, true>), g, b, shmem, s, jobs, wg_job);
        } else {
            if (vec)
                hipLaunchKernelGGL((k_encode_f32<true, false>), g, b, shmem, s, jobs, wg_job);
            else
                hipLaunchKernelGGL((k_encode_f32<false, false>), g, b, shmem, s, jobs, wg_job);
        }
    }
    return hipGetLastError();
}

hipError_t launch_encode_small(const EncodeJob* jobs, const uint32_t* wg_job, uint32_t grid, uint32_t nunits, uint32_t B,
                               bool f64, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    const size_t shmem = encode_small_lds_bytes(nunits, B);
    if (f64)
        hipLaunchKernelGGL(k_encode_small<true>, dim3(grid), dim3(kThreads), shmem, s, jobs, wg_job);
    else
        hipLaunchKernelGGL(k_encode_small<false>, dim3(grid), dim3(kThreads), shmem, s, jobs, wg_job);
    return hipGetLastError();
}

hipError_t launch_select_batch(const SelectParams& p, const SelectLevel* lv, uint32_t nlev,
                               hipStream_t s)
{
    if (nlev == 0) return hipSuccess;
    const dim3 g(p.nunits, nlev);
    switch (p.threads) {
    case 256:
        if (p.wide)
            hipLaunchKernelGGL((k_select<256, uint64_t>), g, dim3(256), 0, s, p, lv);
        else
            hipLaunchKernelGGL((k_select<256, uint32_t>), g, dim3(256), 0, s, p, lv);
        break;
    case 1024:
        if (p.wide)
            hipLaunchKernelGGL((k_select<1024, uint64_t>), g, dim3(1024), 0, s, p, lv);
        else
            hipLaunchKernelGGL((k_select<1024, uint32_t>), g, dim3(1024), 0, s, p, lv);
        break;
    default:
        if (p.wide)
            hipLaunchKernelGGL((k_select<512, uint64_t>), g, dim3(512), 0, s, p, lv);
        else
            hipLaunchKernelGGL((k_select<512, uint32_t>), g, dim3(512), 0, s, p, lv);
        break;
    }
    return hipGetLastError();
}

}  // namespace mdr
