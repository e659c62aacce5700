// Squared L2 error of a level after k planes, k = 0..B: the L2 error table
// that MDR offers beside the L-infinity one (the paper controls L-infinity
// error throughout).  E2[k] = sum_i (|x_i| - xhat_k(|x_i|))^2 with
// xhat_k(a) = floor(a 2^(k-e)) 2^(e-k), the magnitude the retrieval rebuilds
// from k planes of the level aligned to exponent e.  Every residual is exact
// in fp64 (it is a run of the value's own significand bits); each square is
// added with one rounding and the sums run in fp64 in a fixed order (per
// thread, then a fixed tree per workgroup, then workgroups in a fixed order),
// so the table is the same on every run.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "mdr_internal.hpp"

namespace mdr {
namespace {

constexpr uint32_t kL2 = 256;  // threads per workgroup

// One launch covers up to kL2LaunchLevels levels, passed by value.
struct L2Args {
    L2Level lv[kL2LaunchLevels];
};

// Partial rows of every workgroup (B + 2 entries: E2[0..B], then the largest
// |x| the workgroup read).
//
// A value's residual after k planes, in units of 2^(e-k), is fract(z 2^k) with
// z = |x| 2^-e in [0, 1): exact (z's significand bits below the cut), so an
// entry costs a scaling, a fract and a fused multiply-add into its accumulator,
// and the accumulators are scaled back by 2^(2(e-k)) once per workgroup.  (A
// floor and two scalings per entry, unfused, were six operations: the f32
// launches of a 512^3 field took 1.34 ms, this one 0.50.)  The bound is fp64
// issue, three operations of about 4.8 cycles a wavefront and entry.  Values
// with z < 2^-400, whose scaled squares could underflow, lie below every cut:
// their residual is |x| itself and they are summed unscaled.
// KN: accumulators a thread holds, the first of 17, 33, 65 that covers B + 1
// entries (entries past B are computed and dropped).
template <typename T, int KN>
__global__ __launch_bounds__(kL2) void k_l2_partial(const L2Args A, uint32_t nlev, uint32_t B,
                                                    double* __restrict__ part)
{
    __shared__ double red[kL2 / 64][KN + 2];  // entries, sum of tiny values' squares, max |x|
    uint32_t l = 0;
    while (l + 1 < nlev && blockIdx.x >= A.lv[l + 1].wg_base) ++l;
    const T* __restrict__ x = static_cast<const T*>(A.lv[l].x);
    const uint64_t n = A.lv[l].n;
    const int e = A.lv[l].e;
    double acc[KN];
#pragma unroll
    for (int j = 0; j < KN; ++j) acc[j] = 0.0;
    double amax = 0.0, tiny = 0.0;
    const uint64_t stride = (uint64_t)A.lv[l].nwg * kL2;
    auto add = [&](T xv) {
        const double a = __builtin_fabs((double)xv);
        amax = __builtin_fmax(amax, a);
        double z = __builtin_amdgcn_ldexp(a, -e);
        const bool low = z < 0x1p-400;
        const double t = low ? a : 0.0;
        z = low ? 0.0 : z;
        asm volatile("" : "+v"(z));  // select once: the compiler would move it past every entry's scaling
        tiny = __builtin_fma(t, t, tiny);
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            const double y = __builtin_amdgcn_fract(__builtin_amdgcn_ldexp(z, k));
            acc[k] = __builtin_fma(y, y, acc[k]);
        }
    };
    uint64_t i = (uint64_t)(blockIdx.x - A.lv[l].wg_base) * kL2 + threadIdx.x;
    // the next value is loaded while this one's entries are summed
    T next = i < n ? x[i] : T(0);
    while (i < n) {
        const T cur = next;
        i += stride;
        if (i < n) next = x[i];
        add(cur);
    }
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < KN; ++j) {
        double v = acc[j];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) red[wave][j] = v;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        tiny += __shfl_xor(tiny, o, 64);
        amax = __builtin_fmax(amax, __shfl_xor(amax, o, 64));
    }
    if (lane == 0) {
        red[wave][KN] = tiny;
        red[wave][KN + 1] = amax;
    }
    __syncthreads();
    const uint32_t k = threadIdx.x;
    double* row = part + (uint64_t)blockIdx.x * (B + 2);
    if (k <= B) {
        double v = 0.0, t = 0.0;
#pragma unroll
        for (uint32_t w = 0; w < kL2 / 64; ++w) {
            v += red[w][k];
            t += red[w][KN];
        }
        row[k] = __builtin_amdgcn_ldexp(v, 2 * (e - (int)k)) + t;
    } else if (k == B + 1) {
        double m = 0.0;
        for (uint32_t w = 0; w < kL2 / 64; ++w) m = __builtin_fmax(m, red[w][KN + 1]);
        row[k] = m;
    }
}

// out[l][0..B]: the tables; out[l][B + 1]: the largest |x| read, which the
// caller checks against the refactored level's.  A workgroup per level: wave w
// adds the level's rows w, w + 16, ... in order (lanes over the entries), then
// the 16 waves' sums are added in order.  (One thread an entry over all the
// rows took 87 us a level, a chain of a thousand loads.)
constexpr uint32_t kL2Final = 1024;
__global__ __launch_bounds__(kL2Final) void k_l2_final(const L2Args A, uint32_t B, const double* __restrict__ part,
                                                       double* __restrict__ out)
{
    __shared__ double red[kL2Final / 64][kL2RowMax];
    const uint32_t l = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (A.lv[l].n == 0) return;  // its row is not read
    const uint32_t nwg = A.lv[l].nwg;
    const double* p = part + (uint64_t)A.lv[l].wg_base * (B + 2);
    for (uint32_t k = lane; k < B + 2; k += 64) {
        double v = 0.0;
#pragma unroll 4
        for (uint32_t w = wave; w < nwg; w += kL2Final / 64) {
            const double q = p[(uint64_t)w * (B + 2) + k];
            v = k <= B ? v + q : __builtin_fmax(v, q);
        }
        red[wave][k] = v;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < B + 2; k += kL2Final) {
        double v = 0.0;
        for (uint32_t w = 0; w < kL2Final / 64; ++w) v = k <= B ? v + red[w][k] : __builtin_fmax(v, red[w][k]);
        out[(uint64_t)A.lv[l].row * (B + 2) + k] = v;
    }
}

// Fixed scratch of mdr_l2_table_noalloc: the partial rows of at most kL2MaxWg
// workgroups, then the rows of at most kL2NoAllocLevels levels, kL2RowMax
// entries (B + 2 for B <= 64) each: 574,464 bytes per device, held until the
// process ends.  Host code never passes this name to a kernel: it is a
// host-side stand-in; the device address comes from hipGetSymbolAddress, per
// device.
constexpr uint64_t kL2PartDoubles = (uint64_t)kL2MaxWg * kL2RowMax;
constexpr uint64_t kL2ScratchDoubles = kL2PartDoubles + (uint64_t)kL2NoAllocLevels * kL2RowMax;
__device__ __align__(256) double scratch[kL2ScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

hipError_t l2_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) {
        e = hipSetDevice(device);
        if (e != hipSuccess) return e;
    }
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double*>(p);
    return hipSuccess;
}

hipError_t l2_scratch(int device, double** part, double** out)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    double* p;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        p = g_scratch_ptr[device];
    }
    if (!p) return hipErrorNotInitialized;
    *part = p;
    *out = p + kL2PartDoubles;
    return hipSuccess;
}

// Workgroups of a launch's levels: in proportion to their values, at least 8
// values a thread, at most kL2MaxWg in all (every workgroup resident at once: a
// level's share ends when the others do).  A 65-entry table's accumulators
// leave room for three workgroups a CU instead of four.
static uint32_t plan_workgroups(L2Args& A, uint32_t cnt, uint32_t B)
{
    const uint64_t most = B > 32 ? kL2MaxWg * 3 / 4 : kL2MaxWg;
    uint64_t total = 0;
    for (uint32_t l = 0; l < cnt; ++l) total += A.lv[l].n;
    uint32_t base = 0;
    for (uint32_t l = 0; l < cnt; ++l) {
        L2Level& v = A.lv[l];
        v.wg_base = base;
        v.nwg = 0;
        if (v.n) {
            const uint64_t share = 1 + (uint64_t)((double)(most - cnt) * ((double)v.n / (double)total));
            const uint64_t useful = (v.n + kL2 * 8 - 1) / (kL2 * 8);
            v.nwg = (uint32_t)(share < useful ? share : useful);
        }
        base += v.nwg;
    }
    return base;
}

template <typename T, int KN>
static hipError_t launch_tables(const L2Args& A, uint32_t cnt, uint32_t nwg, uint32_t B, double* part, double* out,
                                hipStream_t s)
{
    hipLaunchKernelGGL((k_l2_partial<T, KN>), dim3(nwg), dim3(kL2), 0, s, A, cnt, B, part);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_l2_final, dim3(cnt), dim3(kL2Final), 0, s, A, B, part, out);
    return hipGetLastError();
}

hipError_t launch_l2_tables(bool f64, const L2Level* levels, uint32_t nlevels, uint32_t B, double* part, double* out,
                            hipStream_t s)
{
    // empty levels have no workgroups (their rows are not written)
    L2Args A;
    uint32_t cnt = 0;
    hipError_t err = hipSuccess;
    for (uint32_t l = 0; l < nlevels && err == hipSuccess; ++l) {
        if (levels[l].n) {
            A.lv[cnt] = levels[l];
            A.lv[cnt++].row = l;
        }
        if (cnt == 0 || (cnt < kL2LaunchLevels && l + 1 < nlevels)) continue;
        // the next launch reuses the partial rows: launches stay in stream order
        const uint32_t nwg = plan_workgroups(A, cnt, B);
        if (f64)
            err = B < 17 ? launch_tables<double, 17>(A, cnt, nwg, B, part, out, s)
                  : B < 33 ? launch_tables<double, 33>(A, cnt, nwg, B, part, out, s)
                           : launch_tables<double, 65>(A, cnt, nwg, B, part, out, s);
        else
            err = B < 17 ? launch_tables<float, 17>(A, cnt, nwg, B, part, out, s)
                         : launch_tables<float, 33>(A, cnt, nwg, B, part, out, s);
        cnt = 0;
    }
    return err;
}

}  // namespace mdr
