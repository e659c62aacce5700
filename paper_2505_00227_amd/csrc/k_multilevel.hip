// Multilevel decomposition and recomposition of a row-major n0 x n1 x n2 field
// (n2 fastest) into coefficient levels, the input form of Sec. 2/3.  The
// decomposition is prior work that the paper does not spell out; this is the
// hierarchical multilinear interpolation decomposition (MGARD's interpolation
// step without its L2-projection correction).  Step j works on the stride
// h = 2^j grid: a node of it that is not on the stride-2h grid stores
// u - P, where P refines the stride-2h values along x, then y, then z, each
// time taking (a + b) * 0.5 of the two neighbours on the axis, or the left
// neighbour alone past the last coarse node of the line.  Level 0 holds the raw
// values of the stride-2^nsteps grid; level l >= 1 holds the nodes of step
// nsteps - l in the row-major order of their grid.  Arithmetic stays in the
// field's type, one rounding per operation (no contraction), so coefficients
// are reproducible bit for bit.
//
// A wavefront covers cells of a step's grid: a cell is the 2 x 2 rows
// (2A, 2B) .. (2A + 1, 2B + 1) of it, and a lane takes four consecutive nodes of
// each of them.  The four rows share the coarse rows they refine from, so a
// cell reads seven rows (decomposition) or four and its coefficients
// (recomposition) with every load in flight at once, where row by row it was
// twelve.  Rows shorter than a wavefront's 256 nodes are packed side by side
// into its lanes.  A decomposition step reads only the input field, so all
// steps run in one launch; a recomposition step reads the nodes of every
// coarser step, so they run coarsest first, the small grids together in one
// workgroup's LDS.
//
// Bound: HBM (2 n values), with the neighbour rows from L2: consecutive
// workgroups are placed on one XCD, a contiguous range of the grid each.  The
// decomposition of a 512^3 f32 field went from 0.54 ms (a row segment a
// wavefront, a launch a step) to 0.21, 5.1 TB/s of its 2 n values, 0.92 of a
// large copy's rate; the recomposition of a 301 x 402 x 503 f64 one from 0.48
// to 0.29.
// 16-byte accesses need only the value's alignment here, so rows of any length
// and level offsets of any alignment take the same path.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_bits.hpp"
#include "mdr_internal.hpp"

namespace mdr {
namespace {

constexpr uint32_t kMl = 256;       // threads per workgroup: four wavefronts
constexpr uint32_t kMlNodes = 256;  // nodes of a row a wavefront covers: four a lane
constexpr uint32_t kMlXcds = 8;

__host__ __device__ __forceinline__ uint64_t axis_nodes(uint32_t n, uint32_t j)
{
    return n == 0 ? 0 : (uint64_t)((n - 1) >> j) + 1;
}

// One step's work: its grid, level offset and wavefront units.
struct MlStep {
    uint64_t coef;     // offset of the step's level in the coefficient buffer
    uint64_t coef1;    // and of the level its coarse nodes come from, if not the field
    uint32_t m0, m1, m2;
    uint32_t j;
    uint32_t segs;     // wavefronts along a row
    uint32_t pack;     // cells along y a wavefront packs (segs == 1), a power of two
    uint32_t groups;   // wavefronts along y
    uint32_t blk0;     // first workgroup of the step in its launch
    uint32_t blocks;   // workgroups
};

// NT: touched once, kept out of the way of the rows that neighbours share
template <typename T, int N, bool NT = false>
__device__ __forceinline__ void load_vec(const T* p, T* o)
{
    constexpr int W = N * sizeof(T) / 4;
    uint32_t w[W];
    if constexpr (W == 2) {
        const u32x2_any q = *gmem(reinterpret_cast<const u32x2_any*>(p));
        w[0] = q.x, w[1] = q.y;
    } else {
#pragma unroll
        for (int i = 0; i < W / 4; ++i) {
            const auto at = gmem(reinterpret_cast<const u32x4_any*>(p)) + i;
            u32x4_any q;
            if constexpr (NT)
                q = __builtin_nontemporal_load(at);
            else
                q = *at;
            w[4 * i] = q.x, w[4 * i + 1] = q.y, w[4 * i + 2] = q.z, w[4 * i + 3] = q.w;
        }
    }
    __builtin_memcpy(o, w, sizeof w);
}

template <typename T, int N, bool NT = false>
__device__ __forceinline__ void store_vec(T* p, const T* v)
{
    constexpr int W = N * sizeof(T) / 4;
    uint32_t w[W];
    __builtin_memcpy(w, v, sizeof w);
    if constexpr (W == 2) {
        *gmem(reinterpret_cast<u32x2_any*>(p)) = u32x2_any{w[0], w[1]};
    } else {
#pragma unroll
        for (int i = 0; i < W / 4; ++i) {
            const u32x4_any q = u32x4_any{w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]};
            if constexpr (NT)
                __builtin_nontemporal_store(q, gmem(reinterpret_cast<u32x4_any*>(p)) + i);
            else
                gmem(reinterpret_cast<u32x4_any*>(p))[i] = q;
        }
    }
}

// nodes x .. x + 3 (cnt of them exist) of a grid row that starts at `row`,
// 2^j values apart; J = 0, 1: the step index at compile time, whole vectors
template <typename T, int J, bool NT = false>
__device__ __forceinline__ void load_nodes(const T* row, uint32_t x, uint32_t cnt, uint32_t n2, uint32_t j, T (&v)[4])
{
    if (J == 0 && cnt == 4) {
        load_vec<T, 4, NT>(row + x, v);
    } else if (J == 1 && cnt == 4 && 2ull * x + 8 <= n2) {
        T w[8];
        load_vec<T, 8>(row + 2ull * x, w);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = w[2 * k];
    } else {
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = k < cnt ? gmem(row)[(uint64_t)(x + k) << j] : T(0);
    }
}

// the next lane's value (the last lane's own is returned in its place)
__device__ __forceinline__ float next_lane(float v)
{
    const int b = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(b, b, 0x130, 0xF, 0xF, false));  // wave_shl:1
}
__device__ __forceinline__ double next_lane(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x130, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(lo, lo, 0x130, 0xF, 0xF, false));
}

// P along x of a coarse row's nodes x .. x + 3 from its even ones (v[0], v[2]
// and nx, the node x + 4)
template <typename T>
__device__ __forceinline__ void refine_x(const T (&v)[4], T nx, bool has2, bool has4, T (&p)[4])
{
#pragma clang fp contract(off)
    p[0] = v[0];
    p[1] = has2 ? (v[0] + v[2]) * T(0.5) : v[0];
    p[2] = v[2];
    p[3] = has4 ? (v[2] + nx) * T(0.5) : v[2];
}

template <typename T>
__device__ __forceinline__ T mean(T a, T b)
{
#pragma clang fp contract(off)
    return (a + b) * T(0.5);
}

// The stride-2 nodes x and x + 2 (v[0], v[2]) of a cell's four coarse rows
// (2A + 2da, 2B + 2db), rebuilt from the stride-4 nodes and step 1's
// coefficients: the recomposition's last two steps in one pass, so that step
// 1's nodes, every second value of every fourth row, are never written and
// read back as partial lines (65 of 340 us on a 301 x 402 x 503 f64 field).
template <typename T>
__device__ __forceinline__ void stride2_rows(const T* __restrict__ lv1, const T* field, uint32_t n1, uint32_t n2,
                                             uint32_t m0, uint32_t m1, uint32_t m2, uint32_t A, uint32_t B, uint32_t x,
                                             bool live, bool has2, bool has4, T (&e)[2][2][4])
{
#pragma clang fp contract(off)
    const uint32_t h0 = (m0 + 1) >> 1, h1 = (m1 + 1) >> 1, h2 = (m2 + 1) >> 1;  // stride-2 grid
    const uint32_t q0 = (h0 + 1) >> 1, q1 = (h1 + 1) >> 1, q2 = (h2 + 1) >> 1;  // stride-4 grid
    const uint32_t zl = A >> 1, yl = B >> 1;
    const bool zh = zl + 1 < q0, yh = yl + 1 < q1;
    const bool a_odd = A & 1, b_odd = B & 1;
    T n[2][2][2] = {};  // stride-4 rows [z][y], refined along x: stride-2 nodes x / 2, x / 2 + 1
    T c[2][2][2] = {};  // step 1's coefficients of the four rows
    if (live) {
#pragma unroll
        for (uint32_t z = 0; z < 2; ++z)
#pragma unroll
            for (uint32_t y = 0; y < 2; ++y)
                if ((z == 0 || zh) && (y == 0 || yh))
                    n[z][y][0] = gmem(field)[((uint64_t)(zl + z) * 4 * n1 + (uint64_t)(yl + y) * 4) * n2 + x];
#pragma unroll
        for (uint32_t da = 0; da < 2; ++da)
#pragma unroll
            for (uint32_t db = 0; db < 2; ++db) {
                const uint32_t a = A + da, b = B + db;
                if (a >= h0 || b >= h1) continue;
                uint64_t at = ((uint64_t)a * h1 + b) * h2 - (uint64_t)((a + 1) >> 1) * q1 * q2;
                if (!(a & 1)) at -= (uint64_t)((b + 1) >> 1) * q2;
                if (!((a | b) & 1)) {  // only its odd nodes are new
                    if (has2) c[da][db][1] = gmem(lv1)[at + x / 4];
                } else if (has2) {
                    load_vec<T, 2>(lv1 + at + x / 2, c[da][db]);
                } else {
                    c[da][db][0] = gmem(lv1)[at + x / 2];
                }
            }
    }
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const T nx = next_lane(n[z][y][0]);
            n[z][y][1] = has4 ? mean(n[z][y][0], nx) : n[z][y][0];
        }
#pragma unroll
    for (int da = 0; da < 2; ++da)
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            // row A + da lies on the stride-4 grid where that is even: rows zl
            // (A even) or zl + 1 (A odd); else between the two
            const bool z_between = da ? !a_odd : a_odd, y_between = db ? !b_odd : b_odd;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                T w[2];
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    const T lo = n[z][0][k], hi = n[z][1][k];
                    w[z] = y_between ? (yh ? mean(lo, hi) : lo) : (b_odd ? hi : lo);
                }
                const T P = z_between ? (zh ? mean(w[0], w[1]) : w[0]) : (a_odd ? w[1] : w[0]);
                const bool raw = k == 0 && !z_between && !y_between;
                e[da][db][2 * k] = raw ? P : c[da][db][k] + P;
            }
        }
}

// One wavefront unit of a step.  DEC: field -> coefficients; else the other
// way, writing the nodes of the step (j = 0: whole rows).  FROM (j = 0 of a
// recomposition), where the coarse nodes come from and what else is written:
// kField, the field, which holds them; kStep1, step 1 is done too, its level at
// coef1; kRaw, level 0 at coef1, the only step (with a copy of level 0 into every
// second value of the field first, partial lines that were read back as such,
// 4000 x 4000 f64 values took 80 us, now 54: a copy of them takes 41).
enum { kField, kStep1, kRaw };
template <typename T, bool DEC, int J, int FROM>
__device__ __forceinline__ void ml_unit(const MlStep& st, T* __restrict__ coeffs, T* field, uint32_t n1, uint32_t n2,
                                        uint32_t unit)
{
#pragma clang fp contract(off)
    constexpr bool FUSED = FROM == kStep1, RAW = FROM == kRaw;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t j = J < 2 ? (uint32_t)J : st.j;
    const uint32_t seg = unit % st.segs, yz = unit / st.segs;
    const uint32_t A = yz / st.groups, g = yz % st.groups;
    const uint32_t per = 64 / st.pack;  // lanes a row takes
    const uint32_t B = g * st.pack + lane / per;
    // FUSED: the last lane of a segment that the row goes on after only
    // supplies its neighbour's next node
    const uint32_t span = FUSED && st.segs > 1 ? kMlNodes - 4 : kMlNodes;
    const uint32_t x = seg * span + 4 * (lane % per);
    const uint32_t m0 = st.m0, m1 = st.m1, m2 = st.m2;
    const bool live = 2 * B < m1 && x < m2;
    const uint32_t cnt = live ? min(4u, m2 - x) : 0u;
    const bool zo = 2 * A + 1 < m0, yo = 2 * B + 1 < m1;  // the cell's odd planes / rows exist
    const bool z2 = 2 * A + 2 < m0, y2 = 2 * B + 2 < m1;  // and the coarse ones past them
    auto row = [&](uint32_t a, uint32_t b) { return field + (((uint64_t)a << j) * n1 + ((uint64_t)b << j)) * n2; };
    const T* const c00 = row(2 * A, 2 * B);
    T e[2][2][4] = {};                 // coarse rows [z][y]
    T(&e00)[4] = e[0][0];
    T(&e01)[4] = e[0][1];
    T(&e10)[4] = e[1][0];
    T(&e11)[4] = e[1][1];
    T u01[4], u10[4], u11[4];          // DEC: the cell's other rows; else their coefficients
    T k0[2] = {T(0), T(0)};            // else: the first row's odd coefficients
    const uint32_t e1 = (m1 + 1) >> 1, e2 = (m2 + 1) >> 1;
    auto raw = [&](uint32_t a, uint32_t b) { return coeffs + st.coef1 + ((uint64_t)a * e1 + b) * e2; };
    // coefficients of the cell's rows: position of each row's first in the level
    const uint64_t pl0 = (uint64_t)2 * A * m1 * m2 - (uint64_t)A * e1 * e2;
    const uint64_t pl1 = (uint64_t)(2 * A + 1) * m1 * m2 - (uint64_t)(A + 1) * e1 * e2;
    T* const lv = coeffs + st.coef;
    T* const r00 = lv + pl0 + (uint64_t)2 * B * m2 - (uint64_t)B * e2 + x / 2;
    T* const r01 = lv + pl0 + (uint64_t)(2 * B + 1) * m2 - (uint64_t)(B + 1) * e2 + x;
    T* const r10 = lv + pl1 + (uint64_t)2 * B * m2 + x;
    T* const r11 = lv + pl1 + (uint64_t)(2 * B + 1) * m2 + x;
    const uint32_t odd = cnt >> 1;  // odd nodes among the lane's
    T nx00 = T(0), nx01 = T(0), nx10 = T(0), nx11 = T(0);
    const bool edge = !FUSED && lane == 63 && x + 4 < m2;  // the next node is in the next wavefront's segment
    const bool has2 = x + 2 < m2, has4 = x + 4 < m2;
    if (live) {
        if (RAW) {
#pragma unroll
            for (uint32_t da = 0; da < 2; ++da)
#pragma unroll
                for (uint32_t db = 0; db < 2; ++db) {
                    if ((da && !z2) || (db && !y2)) continue;
                    const T* c = raw(A + da, B + db) + x / 2;
                    T w[2] = {T(0), T(0)};
                    if (has2)
                        load_vec<T, 2>(c, w);
                    else
                        w[0] = *gmem(c);
                    e[da][db][0] = w[0], e[da][db][2] = w[1];
                }
        } else if (!FUSED) {
            load_nodes<T, J>(c00, x, cnt, n2, j, e00);
            if (y2) load_nodes<T, J>(row(2 * A, 2 * B + 2), x, cnt, n2, j, e01);
            if (z2) load_nodes<T, J>(row(2 * A + 2, 2 * B), x, cnt, n2, j, e10);
            if (y2 && z2) load_nodes<T, J>(row(2 * A + 2, 2 * B + 2), x, cnt, n2, j, e11);
        }
        if (DEC) {
            if (yo) load_nodes<T, J, J == 0>(row(2 * A, 2 * B + 1), x, cnt, n2, j, u01);
            if (zo) load_nodes<T, J, J == 0>(row(2 * A + 1, 2 * B), x, cnt, n2, j, u10);
            if (yo && zo) load_nodes<T, J, J == 0>(row(2 * A + 1, 2 * B + 1), x, cnt, n2, j, u11);
        } else {
            if (odd == 2)
                load_vec<T, 2>(r00, k0);
            else if (odd == 1)
                k0[0] = *gmem(r00);
            if (yo) load_nodes<T, 0, true>(r01 - x, x, cnt, m2, 0, u01);
            if (zo) load_nodes<T, 0, true>(r10 - x, x, cnt, m2, 0, u10);
            if (yo && zo) load_nodes<T, 0, true>(r11 - x, x, cnt, m2, 0, u11);
        }
        if (RAW && edge) {
            const uint32_t at = x / 2 + 2;
            nx00 = gmem(raw(A, B))[at];
            if (y2) nx01 = gmem(raw(A, B + 1))[at];
            if (z2) nx10 = gmem(raw(A + 1, B))[at];
            if (y2 && z2) nx11 = gmem(raw(A + 1, B + 1))[at];
        } else if (edge) {
            const uint64_t at = (uint64_t)(x + 4) << j;
            nx00 = gmem(c00)[at];
            if (y2) nx01 = gmem(row(2 * A, 2 * B + 2))[at];
            if (z2) nx10 = gmem(row(2 * A + 2, 2 * B))[at];
            if (y2 && z2) nx11 = gmem(row(2 * A + 2, 2 * B + 2))[at];
        }
    }
    if constexpr (FUSED) stride2_rows(coeffs + st.coef1, field, n1, n2, m0, m1, m2, A, B, x, live, has2, has4, e);
    T p00[4], p01[4], p10[4], p11[4];
    {
        const T s00 = next_lane(e00[0]), s01 = next_lane(e01[0]), s10 = next_lane(e10[0]), s11 = next_lane(e11[0]);
        refine_x(e00, edge ? nx00 : s00, has2, has4, p00);
        refine_x(e01, edge ? nx01 : s01, has2, has4, p01);
        refine_x(e10, edge ? nx10 : s10, has2, has4, p10);
        refine_x(e11, edge ? nx11 : s11, has2, has4, p11);
    }
    if (!live || (FUSED && st.segs > 1 && lane == 63)) return;
    // along y, then z: P of rows (even, odd), (odd, even) and (odd, odd)
    T q01[4], q10[4], q11[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        q01[k] = y2 ? mean(p00[k], p01[k]) : p00[k];
        const T far = y2 ? mean(p10[k], p11[k]) : p10[k];
        q10[k] = z2 ? mean(p00[k], p10[k]) : p00[k];
        q11[k] = z2 ? mean(q01[k], far) : q01[k];
    }
    if (DEC) {
        T o[4];
        o[0] = e00[1] - p00[1], o[1] = e00[3] - p00[3];
        if (odd == 2)
            store_vec<T, 2>(r00, o);
        else if (odd == 1)
            *gmem(r00) = o[0];
        auto put = [&](T* r, const T (&u)[4], const T (&q)[4]) {
#pragma clang fp contract(off)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = u[k] - q[k];
            if (cnt == 4) {
                store_vec<T, 4, true>(r, o);
            } else {
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (k < cnt) gmem(r)[k] = o[k];
            }
        };
        if (yo) put(r01, u01, q01);
        if (zo) put(r10, u10, q10);
        if (yo && zo) put(r11, u11, q11);
    } else {
        T* const f00 = row(2 * A, 2 * B);
        T o[4] = {e00[0], k0[0] + p00[1], e00[2], k0[1] + p00[3]};
        if (J == 0 && cnt == 4) {
            // the even values too (kField: again, unchanged): whole lines, where single odd
            // values would be partial ones (readers of the row see the same bits)
            store_vec<T, 4>(f00 + x, o);
        } else {
            // (not from the field: the even nodes are new to it)
#pragma unroll
            for (uint32_t k = FROM != kField ? 0 : 1; k < 4; k += FROM != kField ? 1 : 2)
                if (k < cnt) gmem(f00)[(uint64_t)(x + k) << j] = o[k];
        }
        auto put = [&](T* r, const T (&c)[4], const T (&q)[4]) {
#pragma clang fp contract(off)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = c[k] + q[k];
            if (J == 0 && cnt == 4) {
                store_vec<T, 4, true>(r + x, o);
            } else {
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (k < cnt) gmem(r)[(uint64_t)(x + k) << j] = o[k];
            }
        };
        if (yo) put(row(2 * A, 2 * B + 1), u01, q01);
        if (zo) put(row(2 * A + 1, 2 * B), u10, q10);
        if (yo && zo) put(row(2 * A + 1, 2 * B + 1), u11, q11);
    }
}

// workgroup -> its place in a launch of `blocks`, consecutive ones on one XCD
// (the hardware deals workgroups to the XCDs in turn); ~0 past the end
__device__ __forceinline__ uint32_t xcd_block(uint32_t id, uint32_t blocks)
{
    const uint32_t per = (blocks + kMlXcds - 1) / kMlXcds;
    const uint32_t at = (id % kMlXcds) * per + id / kMlXcds;
    return id / kMlXcds < per && at < blocks ? at : ~0u;
}

// this workgroup's number in its launch, and how many there are (see ml_grid)
__device__ __forceinline__ uint32_t ml_id() { return blockIdx.y * gridDim.x + blockIdx.x; }
__device__ __forceinline__ uint32_t ml_launched() { return gridDim.y * gridDim.x; }

template <typename T, bool DEC, int J, int FROM = kField>
__device__ __forceinline__ void ml_block(const MlStep& st, T* coeffs, T* field, uint32_t n1, uint32_t n2, uint32_t blk)
{
    const uint32_t at = xcd_block(blk, st.blocks);
    const uint32_t unit = at * (kMl / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t cells0 = (st.m0 + 1) >> 1;
    if (at == ~0u || unit >= cells0 * st.groups * st.segs) return;
    ml_unit<T, DEC, J, FROM>(st, coeffs, field, n1, n2, unit);
}

// The decomposition: every step and the raw coarsest grid in one launch.
struct MlSteps {
    MlStep st[kMlMaxSteps];
    uint32_t count;  // steps, finest first
    uint32_t blk_raw;
};

// coarsest grid (stride 2^nsteps): DEC copies field -> level 0, else back
template <typename T, bool DEC>
__device__ __forceinline__ void ml_raw(T* coeffs, T* field, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t nsteps,
                                       uint64_t first, uint64_t stride)
{
    const uint64_t m0 = axis_nodes(n0, nsteps), m1 = axis_nodes(n1, nsteps), m2 = axis_nodes(n2, nsteps);
    for (uint64_t c = first; c < m0 * m1 * m2; c += stride) {
        const uint64_t b2 = c % m2, b1 = c / m2 % m1, b0 = c / m2 / m1;
        const uint64_t f = ((b0 << nsteps) * n1 + (b1 << nsteps)) * n2 + (b2 << nsteps);
        if (DEC)
            gmem(coeffs)[c] = gmem(field)[f];
        else
            gmem(field)[f] = gmem(coeffs)[c];
    }
}

template <typename T>
__global__ __launch_bounds__(kMl) void k_ml_decompose(const MlSteps S, T* field, T* coeffs, uint32_t n0, uint32_t n1,
                                                      uint32_t n2, uint32_t nsteps)
{
    const uint32_t blk = ml_id();
    if (blk >= S.blk_raw) {
        ml_raw<T, true>(coeffs, field, n0, n1, n2, nsteps, (uint64_t)(blk - S.blk_raw) * kMl + threadIdx.x,
                        (uint64_t)(ml_launched() - S.blk_raw) * kMl);
        return;
    }
    uint32_t i = 0;
    while (i + 1 < S.count && blk >= S.st[i + 1].blk0) ++i;
    const MlStep& st = S.st[i];
    if (st.j == 0)
        ml_block<T, true, 0>(st, coeffs, field, n1, n2, blk - st.blk0);
    else if (st.j == 1)
        ml_block<T, true, 1>(st, coeffs, field, n1, n2, blk - st.blk0);
    else
        ml_block<T, true, 2>(st, coeffs, field, n1, n2, blk - st.blk0);
}

// One step of the recomposition (FROM: see ml_unit).
template <typename T, int J, int FROM>
__global__ __launch_bounds__(kMl) void k_ml_recompose(const MlStep st, T* coeffs, T* field, uint32_t n1, uint32_t n2)
{
    ml_block<T, false, J, FROM>(st, coeffs, field, n1, n2, ml_id());
}

template <typename T>
__global__ __launch_bounds__(kMl) void k_ml_raw(T* coeffs, T* field, uint32_t n0, uint32_t n1, uint32_t n2,
                                                uint32_t nsteps)
{
    ml_raw<T, false>(coeffs, field, n0, n1, n2, nsteps, (uint64_t)blockIdx.x * kMl + threadIdx.x,
                     (uint64_t)gridDim.x * kMl);
}

// The recomposition's first steps, in one workgroup: the raw grid and `steps`
// refinements of it (each of at most kMlSmall nodes) in LDS, the last one's
// nodes then written to the field.  (A launch each, they cost about 5 us.)
constexpr uint32_t kMlSmallThreads = 1024;
constexpr uint32_t kMlSmallBytes = 32768;  // of one grid; two in LDS
template <typename T>
__global__ __launch_bounds__(kMlSmallThreads) void k_ml_recompose_small(const MlOffsets off, const T* coeffs, T* field,
                                                                        uint32_t n0, uint32_t n1, uint32_t n2,
                                                                        uint32_t nsteps, uint32_t steps)
{
#pragma clang fp contract(off)
    constexpr uint32_t kMlSmall = kMlSmallBytes / sizeof(T);
    __shared__ T s_g[2][kMlSmall];
    const uint32_t tid = threadIdx.x;
    uint32_t o0 = (uint32_t)axis_nodes(n0, nsteps), o1 = (uint32_t)axis_nodes(n1, nsteps),
             o2 = (uint32_t)axis_nodes(n2, nsteps);
    for (uint32_t i = tid; i < o0 * o1 * o2; i += kMlSmallThreads) s_g[0][i] = gmem(coeffs)[off.off[0] + i];
    __syncthreads();
    uint32_t cur = 0;
    for (uint32_t l = 1; l <= steps; ++l) {
        const uint32_t j = nsteps - l;
        const uint32_t m0 = (uint32_t)axis_nodes(n0, j), m1 = (uint32_t)axis_nodes(n1, j),
                       m2 = (uint32_t)axis_nodes(n2, j);
        const uint32_t e1 = (m1 + 1) >> 1, e2 = (m2 + 1) >> 1;
        const T* g = s_g[cur];
        T* out = s_g[cur ^ 1];
        const auto lv = gmem(coeffs + off.off[l]);
        for (uint32_t i = tid; i < m0 * m1 * m2; i += kMlSmallThreads) {
            const uint32_t c = i % m2, b = i / m2 % m1, a = i / m2 / m1;
            const uint32_t z0 = a >> 1, y0 = b >> 1, x0 = c >> 1;
            const bool zm = (a & 1) && z0 + 1 < o0, ym = (b & 1) && y0 + 1 < o1, xm = (c & 1) && x0 + 1 < o2;
            auto line = [&](uint32_t z, uint32_t y) {
                const T* r = g + (z * o1 + y) * o2 + x0;
                return xm ? mean(r[0], r[1]) : r[0];
            };
            auto plane = [&](uint32_t z) { return ym ? mean(line(z, y0), line(z, y0 + 1)) : line(z, y0); };
            T v = zm ? mean(plane(z0), plane(z0 + 1)) : plane(z0);
            if ((a | b | c) & 1) {
                uint32_t skipped = ((a + 1) >> 1) * e1 * e2;  // nodes of the coarser grid before this one
                if (!(a & 1)) {
                    skipped += ((b + 1) >> 1) * e2;
                    if (!(b & 1)) skipped += (c + 1) >> 1;
                }
                v = lv[i - skipped] + v;
            }
            out[i] = v;
        }
        __syncthreads();
        cur ^= 1;
        o0 = m0, o1 = m1, o2 = m2;
    }
    const uint32_t j = nsteps - steps;
    for (uint32_t i = tid; i < o0 * o1 * o2; i += kMlSmallThreads) {
        const uint64_t c = i % o2, b = i / o2 % o1, a = i / o2 / o1;
        gmem(field)[((a << j) * n1 + (b << j)) * n2 + (c << j)] = s_g[cur][i];
    }
}

// host: the work of step j; false if its grid has no new nodes beyond the
// coarser one (a step past the grid's extent: an empty level)
bool plan_step(uint32_t n0, uint32_t n1, uint32_t n2, uint32_t j, uint64_t coef, MlStep& st, bool fused = false)
{
    st.m0 = (uint32_t)axis_nodes(n0, j);
    st.m1 = (uint32_t)axis_nodes(n1, j);
    st.m2 = (uint32_t)axis_nodes(n2, j);
    st.j = j;
    st.coef = coef;
    st.coef1 = 0;
    st.blk0 = 0;
    if (st.m0 == 1 && st.m1 == 1 && st.m2 == 1) return false;
    const uint32_t lanes = (st.m2 + 3) / 4;
    st.segs = (st.m2 + kMlNodes - 1) / kMlNodes;
    if (fused && st.segs > 1) st.segs = (st.m2 + kMlNodes - 5) / (kMlNodes - 4);
    st.pack = 1;
    while (st.segs == 1 && st.pack < 64 && lanes * st.pack * 2 <= 64) st.pack *= 2;
    const uint32_t cells0 = (st.m0 + 1) >> 1, cells1 = (st.m1 + 1) >> 1;
    st.groups = (cells1 + st.pack - 1) / st.pack;
    const uint64_t units = (uint64_t)cells0 * st.groups * st.segs;
    st.blocks = (uint32_t)((units + kMl / 64 - 1) / (kMl / 64));
    return true;
}

// workgroups a step is launched with: whole rounds over the XCDs
uint32_t launch_blocks(const MlStep& st) { return (st.blocks + kMlXcds - 1) / kMlXcds * kMlXcds; }

// The grid of a launch of `blocks` workgroups.  x may hold 2^32 - 1 threads
// (more are taken modulo 2^32, without an error), so from 2^24 workgroups on
// they go in rows of 2^20; what the last row has too many finds no work.
// Fields of about 3 x 10^10 values get there whose rows fill little more than
// half of their wavefronts.
dim3 ml_grid(uint32_t blocks)
{
    constexpr uint32_t kRow = 1u << 20;  // whole rounds over the XCDs
    if ((uint64_t)blocks * kMl <= 0xFFFFFFFFull) return dim3(blocks);
    return dim3(kRow, (blocks + kRow - 1) / kRow);
}

uint32_t raw_blocks(uint64_t nodes)
{
    const uint64_t b = (nodes + kMl - 1) / kMl;
    return (uint32_t)(b < 4096 ? b : 4096);
}

template <typename T>
hipError_t ml_decompose(T* field, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t nsteps, const MlOffsets& off,
                        T* coeffs, hipStream_t s)
{
    MlSteps S{};
    uint32_t blk = 0;
    for (uint32_t j = 0; j < nsteps; ++j) {
        MlStep& st = S.st[S.count];
        if (!plan_step(n0, n1, n2, j, off.off[nsteps - j], st)) continue;
        st.blk0 = blk;
        blk += launch_blocks(st);
        ++S.count;
    }
    S.blk_raw = blk;
    blk += raw_blocks(axis_nodes(n0, nsteps) * axis_nodes(n1, nsteps) * axis_nodes(n2, nsteps));
    hipLaunchKernelGGL(k_ml_decompose<T>, ml_grid(blk), dim3(kMl), 0, s, S, field, coeffs, n0, n1, n2, nsteps);
    return hipGetLastError();
}

template <typename T>
hipError_t ml_recompose(T* coeffs, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t nsteps, const MlOffsets& off,
                        T* field, hipStream_t s)
{
    auto nodes = [&](uint32_t j) { return axis_nodes(n0, j) * axis_nodes(n1, j) * axis_nodes(n2, j); };
    // the raw grid and as many steps as fit one workgroup's LDS; a grid too
    // large for it is copied by a launch of its own
    uint32_t l = 0;
    if (nsteps == 1 && nodes(0) > kMlSmallBytes / sizeof(T)) {
        MlStep st;
        plan_step(n0, n1, n2, 0, off.off[1], st);
        st.coef1 = off.off[0];
        hipLaunchKernelGGL((k_ml_recompose<T, 0, kRaw>), ml_grid(launch_blocks(st)), dim3(kMl), 0, s, st, coeffs, field,
                           n1, n2);
        return hipGetLastError();
    }
    if (nodes(nsteps) <= kMlSmallBytes / sizeof(T)) {
        while (l < nsteps && nodes(nsteps - l - 1) <= kMlSmallBytes / sizeof(T)) ++l;
        hipLaunchKernelGGL(k_ml_recompose_small<T>, dim3(1), dim3(kMlSmallThreads), 0, s, off, coeffs, field, n0, n1, n2,
                           nsteps, l);
    } else {
        hipLaunchKernelGGL(k_ml_raw<T>, dim3(raw_blocks(nodes(nsteps))), dim3(kMl), 0, s, coeffs, field, n0, n1, n2,
                           nsteps);
    }
    hipError_t e = hipGetLastError();
    while (l < nsteps && e == hipSuccess) {
        const uint32_t j = nsteps - ++l;
        const bool fused = j == 1;
        MlStep st;
        if (fused) ++l;
        if (!plan_step(n0, n1, n2, fused ? 0 : j, off.off[l], st, fused)) continue;
        st.coef1 = fused ? off.off[l - 1] : 0;
        const dim3 g = ml_grid(launch_blocks(st));
        if (fused)
            hipLaunchKernelGGL((k_ml_recompose<T, 0, kStep1>), g, dim3(kMl), 0, s, st, coeffs, field, n1, n2);
        else if (j == 0)
            hipLaunchKernelGGL((k_ml_recompose<T, 0, kField>), g, dim3(kMl), 0, s, st, coeffs, field, n1, n2);
        else
            hipLaunchKernelGGL((k_ml_recompose<T, 2, kField>), g, dim3(kMl), 0, s, st, coeffs, field, n1, n2);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

// (the kernels share one unit for both directions, so they take the input
// unqualified; only the output is written)
hipError_t launch_decompose(bool f64, const void* u, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t nsteps,
                            const MlOffsets& off, void* out, hipStream_t s)
{
    if ((uint64_t)n0 * n1 * n2 == 0) return hipSuccess;
    void* in = const_cast<void*>(u);
    return f64 ? ml_decompose(static_cast<double*>(in), n0, n1, n2, nsteps, off, static_cast<double*>(out), s)
               : ml_decompose(static_cast<float*>(in), n0, n1, n2, nsteps, off, static_cast<float*>(out), s);
}

hipError_t launch_recompose(bool f64, const void* c, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t nsteps,
                            const MlOffsets& off, void* u, hipStream_t s)
{
    if ((uint64_t)n0 * n1 * n2 == 0) return hipSuccess;
    void* in = const_cast<void*>(c);
    return f64 ? ml_recompose(static_cast<double*>(in), n0, n1, n2, nsteps, off, static_cast<double*>(u), s)
               : ml_recompose(static_cast<float*>(in), n0, n1, n2, nsteps, off, static_cast<float*>(u), s);
}

}  // namespace mdr
