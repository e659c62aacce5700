// Lossless kernels for gfx950 (Sec. 4.1): device-wide exclusive scan, chunked
// canonical Huffman coding of byte symbols, and run-length coding of W-bit
// plane words.  Direct copy needs no kernel: its payload is the plane rows.
#include "device_bits.hpp"
#include "mdr_internal.hpp"

namespace mdr {
namespace {

constexpr int kScanItems = 4;                          // per thread
constexpr int kScanTile = kThreads * kScanItems;       // per workgroup

// Inclusive scan over the wavefront with data-parallel moves between lanes (no
// LDS traffic): within each row of 16 lanes by shifts of 1, 2, 4 and 8 (a lane
// whose source lies before its row adds 0), then row 0's last lane into row 1
// and row 2's into row 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, uint32_t lane)
{
    (void)lane;
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
    return (uint32_t)x;
}

// exclusive scan of one tile; returns the tile total
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_wave, uint32_t& excl)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t inc = wave_incl_scan(v, lane);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t wbase = 0, total = 0;
    for (uint32_t w = 0; w < kThreads / 64; ++w) {
        wbase += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    excl = wbase + inc - v;
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(kThreads) void k_scan_tiles(const uint32_t* in, uint32_t* out,
                                                         uint64_t n, uint32_t* sums)
{
    __shared__ uint32_t s_wave[kThreads / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems], sum = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        v[j] = base + j < n ? in[base + j] : 0;
        sum += v[j];
    }
    uint32_t excl;
    uint32_t total = block_excl_scan(sum, s_wave, excl);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (base + j < n) out[base + j] = excl;
        excl += v[j];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void k_scan_add(uint32_t* out, uint64_t n,
                                                       const uint32_t* sums)
{
    const uint32_t add = sums[blockIdx.x];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j)
        if (base + j < n) out[base + j] += add;
}

// ------------------------------------------------------------------ batch encode
// Huffman payload: u64 nsym | u8 len[256] | u32 off[nchunks+1] | u32 words[].
// Chunk c (huf_chunk symbols) starts at word off[c]; code bits are packed most
// significant first.  Run-length payload: u32 nruns | u32 wbytes |
// symbols[nruns] (W-bit) | u32 lengths[nruns].
//
// Every kernel below has a fixed grid and reads its amount of work from device
// memory (counts[]), so the whole stage runs without the host learning which
// units chose which method.
constexpr uint64_t kHufHeader = kHufHeaderBytes;

__device__ __forceinline__ uint64_t wave_incl_scan64(uint64_t v, uint32_t lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint64_t o = __shfl_up(v, off, 64);
        if (lane >= (uint32_t)off) v += o;
    }
    return v;
}

// exclusive scan across a workgroup of NT threads (64-bit); returns the total
template <int NT>
__device__ uint64_t block_scan64(uint64_t v, uint64_t* s_wave, uint64_t& excl)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint64_t inc = wave_incl_scan64(v, lane);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint64_t wbase = 0, total = 0;
    for (uint32_t w = 0; w < NT / 64; ++w) {
        wbase += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    excl = wbase + inc - v;
    __syncthreads();
    return total;
}

// largest u in [0, U) with base[u] <= c, for a non-decreasing base with base[0] = 0
__device__ __forceinline__ uint32_t find_unit(const uint32_t* base, uint32_t U, uint32_t c)
{
    uint32_t lo = 0, hi = U;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (base[mid] <= c)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// first plane row of unit u (its rows are contiguous in the level's row array)
__device__ __forceinline__ const uint32_t* unit_rows(const LosslessArgs& A, uint32_t u)
{
    const uint32_t i = u % A.nunits;
    const EncodeJob& job = A.jobs[u / A.nunits];
    const uint32_t r0 = i == 0 ? 0 : 1 + (i - 1) * A.m;
    return job.rows + (uint64_t)r0 * job.nbd;
}

// Threads of the two one-workgroup kernels take consecutive units each, from
// compact arrays, four units' loads at a time: one scan for all of them (1024
// units a scan, from the 48-byte unit records, a batch of 11520 took 36 and 43 us).
constexpr uint32_t kUnitFly = 4;

// Every unit's first Huffman chunk and run-length tile, by a workgroup of NT
// threads: put(unit, first chunk | first tile << 32); returns the totals.
template <int NT, typename Put>
__device__ __forceinline__ uint64_t plan_units(const LosslessArgs& A, uint64_t* s_wave, Put put)
{
    const uint32_t per = (A.U + NT - 1) / NT, u0 = min(threadIdx.x * per, A.U), u1 = min(u0 + per, A.U);
    const auto work = gmem(A.work);
    uint64_t sum = 0;  // chunks (low half) and run-length tiles (high half) of the thread's units
    for (uint32_t u = u0; u < u1; u += kUnitFly) {
        uint64_t w[kUnitFly];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) w[k] = work[min(u + k, u1 - 1)];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) sum += u + k < u1 ? w[k] & kWorkCounts : 0;
    }
    uint64_t at;
    const uint64_t total = block_scan64<NT>(sum, s_wave, at);
    for (uint32_t u = u0; u < u1; u += kUnitFly) {
        uint64_t w[kUnitFly];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) w[k] = work[min(u + k, u1 - 1)];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) {
            if (u + k >= u1) break;
            put(u + k, at);
            at += w[k] & kWorkCounts;
        }
    }
    if (threadIdx.x == 0) put(A.U, total);
    return total;
}

// writes the plan where the later launches read it
__device__ __forceinline__ void store_plan(const LosslessArgs& A, uint32_t u, uint64_t at)
{
    gmem(A.chunk_base)[u] = (uint32_t)at;
    gmem(A.tile_base)[u] = (uint32_t)(at >> 32);
    if (u == A.U) {
        A.counts[0] = (uint32_t)at;
        A.counts[1] = (uint32_t)(at >> 32);
        A.counts[2] = 0;
    }
}

// Up to this many units (four a thread) every workgroup of the counting launch
// makes the plan for itself in LDS, where its wavefronts then look their units
// up: 6.7 us instead of 4.4 + 6.4 in two launches for 9 units, 25.0 instead of
// 4.6 + 24.6 for 81.  Past it the plan grows with the units (18 us for 11520),
// and one workgroup makes it for all.
constexpr uint32_t kPlanUnits = 1024;

__global__ __launch_bounds__(1024) void k_unit_plan(const LosslessArgs* __restrict__ Ap)
{
    __shared__ uint64_t s_wave[16];
    const LosslessArgs& A = *Ap;
    plan_units<1024>(A, s_wave, [&](uint32_t u, uint64_t at) { store_plan(A, u, at); });
}

// Huffman chunks are split among wavefronts in contiguous shares; a wavefront
// walks its share in batches of kHufLoads wave-wide loads of 256 words (lane l
// takes words 4l .. 4l+3 of each: sixteen consecutive symbols), never crossing
// a unit.  A chunk of huf_chunk symbols is huf_chunk / 4 words: 16, 32 or 64
// lanes of one load (chunks of 256, 512, 1024 symbols) or 2 or 4 whole loads
// (2048, 4096), so a batch holds 16 / (huf_chunk / 256) chunks.  Code lengths
// and codes of the current unit are cached in LDS.
constexpr uint32_t kHufLoads = 4;
static_assert(4096 / 256 <= 4 * kHufLoads, "a chunk of the largest size fits one batch");

// inclusive scan of v over segments of `seg` lanes (16, 32 or 64: a uniform
// value), by data-parallel moves: rows of 16 by shifts of 1, 2, 4, 8, then
// row 0's last lane into row 1 and row 2's into row 3, then lane 31 into rows
// 2 and 3
__device__ __forceinline__ uint32_t seg_incl_scan(uint32_t v, uint32_t seg)
{
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
    if (seg >= 32) x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    if (seg >= 64) x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return (uint32_t)x;
}

// a batch's words, lane l's four of each load (0 past the batch's chunks or
// the unit's end; `valid` counts the lane's words that are in)
struct HufBatch {
    uint32_t w[kHufLoads][4];
    uint32_t valid[kHufLoads];
};

__device__ __forceinline__ bool huf_load_batch(const uint32_t* g, uint64_t wb, uint32_t nwb, uint64_t nwu,
                                               uint32_t lane, HufBatch& hb)
{
    // a whole batch from a 16-byte boundary: one 16-byte load per lane and load
    if (nwb == 256 * kHufLoads && wb + 256 * kHufLoads <= nwu &&
        (reinterpret_cast<uintptr_t>(g + wb) & 15u) == 0) {
        const auto p = gmem(reinterpret_cast<const u32x4*>(g + wb));
#pragma unroll
        for (uint32_t r = 0; r < kHufLoads; ++r) {
            const u32x4 q = p[r * 64 + lane];
            hb.w[r][0] = q.x;
            hb.w[r][1] = q.y;
            hb.w[r][2] = q.z;
            hb.w[r][3] = q.w;
            hb.valid[r] = 4;
        }
        return true;
    }
    const auto gg = gmem(g);
#pragma unroll
    for (uint32_t r = 0; r < kHufLoads; ++r) {
        const uint32_t i0 = r * 256 + 4 * lane;
        uint32_t nv = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const bool ok = i0 + i < nwb && wb + i0 + i < nwu;
            hb.w[r][i] = ok ? gg[wb + i0 + i] : 0u;
            nv += ok ? 1u : 0u;
        }
        hb.valid[r] = nv;
    }
    return false;
}

// chunks a wavefront takes of `total`, and the tiles a workgroup takes: the
// counting and the writing launch share them out alike (kPersistWg workgroups)
constexpr uint32_t kPersistWaves = kPersistWg * (kThreads / 64);
__host__ __device__ __forceinline__ uint32_t chunk_share(uint32_t total)
{
    return (total + kPersistWaves - 1) / kPersistWaves;
}
__host__ __device__ __forceinline__ uint32_t tile_share(uint32_t total) { return (total + kPersistWg - 1) / kPersistWg; }

__device__ __forceinline__ void wave_share(uint32_t total, uint32_t& w, uint32_t& c0, uint32_t& c1)
{
    w = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    const uint32_t per = chunk_share(total);
    c0 = min(w * per, total);
    c1 = min(c0 + per, total);
}

// Words of every wavefront's share of the Huffman chunks -> wave_part, and where
// each unit's first chunk starts and its last one ends within its wavefront's
// share: per lane the code lengths of its sixteen symbols, summed over each
// chunk's lanes by a segmented scan (chunks over several loads carry their sum
// across them).  The writing launch walks the same shares, so these are all the
// offsets it needs: no word count is kept per chunk.
__device__ __forceinline__ void huf_count_body(const LosslessArgs& A, const uint32_t* chunk_base, const uint32_t total)
{
    // a byte a symbol: the table's 64 words lie in as many banks, so lanes
    // reading different symbols do not wait on each other (a word a symbol: the
    // counts of 1.07 GB took 274 us; now 252, 4.3 TB/s)
    __shared__ __align__(4) uint8_t s_len[kThreads / 64][256];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint8_t* L = s_len[wave];
    const uint32_t cw = A.huf_chunk / 4, wpl = A.huf_chunk / 256;  // words, 256-symbol groups per chunk
    const uint32_t cpb = 4 * kHufLoads / wpl;                       // chunks per batch
    const uint32_t seg = min(64u, 16 * wpl), lpc = wpl > 4 ? wpl / 4 : 1;  // lanes a chunk takes of a load; loads a chunk
    uint32_t wv, c0, c1, acc = 0;  // acc: words of the share so far
    wave_share(total, wv, c0, c1);
    uint32_t u = 0, cb_lo = 1, cb_hi = 0;  // chunks [cb_lo, cb_hi) belong to unit u
    uint64_t nwu = 0;                      // words of unit u
    for (uint32_t c = c0; c < c1;) {
        if (c < cb_lo || c >= cb_hi) {
            u = find_unit(chunk_base, A.U, c);
            cb_lo = chunk_base[u];
            cb_hi = chunk_base[u + 1];
            nwu = A.units[u].S / 4;
            reinterpret_cast<uint32_t*>(L)[lane] = reinterpret_cast<const uint32_t*>(A.lens + (uint64_t)u * 256)[lane];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if (c == cb_lo && lane == 0) A.huf_lo[u] = acc;
        const uint32_t nbt = min(cpb, min(c1, cb_hi) - c);  // chunks in this batch
        HufBatch hb;
        huf_load_batch(unit_rows(A, u), (uint64_t)(c - cb_lo) * cw, nbt * cw, nwu, lane, hb);
        uint32_t run = 0;  // bits of the chunk's earlier loads (chunks over several loads)
#pragma unroll
        for (uint32_t r = 0; r < kHufLoads; ++r) {
            uint32_t T = 0;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t w = hb.w[r][i];
                const uint32_t bits = (uint32_t)L[w & 0xFF] + L[(w >> 8) & 0xFF] + L[(w >> 16) & 0xFF] + L[w >> 24];
                T += i < hb.valid[r] ? bits : 0u;
            }
            const uint32_t x = seg_incl_scan(T, seg);
            if (lpc == 1) {
                for (uint32_t k = 0; k < 64 / seg; ++k)  // no chunk: no bits
                    acc += ((uint32_t)__builtin_amdgcn_readlane((int)x, (int)(k * seg + seg - 1)) + 31) / 32;
            } else {
                if (r % lpc == 0) run = 0;
                run += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
                if (r % lpc == lpc - 1) acc += (run + 31) / 32;
            }
        }
        if (c + nbt == cb_hi && lane == 0) A.huf_hi[u] = acc;
        c += nbt;
    }
    if (lane == 0) A.wave_part[wv] = acc;
}

__device__ __forceinline__ bool word_ne(const uint32_t* g, uint64_t i, uint64_t j, uint32_t G)
{
    bool ne = g[i * G] != g[j * G];
    if (G == 2) ne = ne || g[i * G + 1] != g[j * G + 1];
    return ne;
}

// A workgroup takes a contiguous share of the tiles: its runs -> tile_part, the
// runs before each unit's first tile within the share -> rle_lo, and every
// tile's first run start, counted from the tile's first word -> tile_first
// (kNoStart: none starts in it).
constexpr uint32_t kNoStart = ~0u;
__device__ __forceinline__ void rle_count_body(const LosslessArgs& A, const uint32_t* tile_base, const uint32_t total)
{
    __shared__ uint32_t s_cnt[kThreads / 64], s_first[kThreads / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t t0 = min(blockIdx.x * tile_share(total), total), t1 = min(t0 + tile_share(total), total);
    uint32_t u = 0, tb_lo = 1, tb_hi = 0, acc = 0;  // tiles [tb_lo, tb_hi) belong to unit u
    for (uint32_t t = t0; t < t1; ++t) {
        if (t < tb_lo || t >= tb_hi) {
            u = find_unit(tile_base, A.U, t);
            tb_lo = tile_base[u];
            tb_hi = tile_base[u + 1];
        }
        if (t == tb_lo && tid == 0) A.rle_lo[u] = acc;
        const uint32_t* g = unit_rows(A, u);
        const uint64_t nw = A.units[u].S / (4ull * A.G);
        const uint64_t i0 = (uint64_t)(t - tb_lo) * kRleTileWords;
        const uint64_t i1 = min(nw, i0 + kRleTileWords);
        uint32_t cnt = 0, first = kNoStart;
        for (uint64_t i = i0 + tid; i < i1; i += kThreads)
            if (i == 0 || word_ne(g, i, i - 1, A.G)) {
                ++cnt;
                first = min(first, (uint32_t)(i - i0));
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            cnt += __shfl_xor(cnt, o, 64);
            first = min(first, (uint32_t)__shfl_xor((int)first, o, 64));
        }
        if (lane == 0) {
            s_cnt[wave] = cnt;
            s_first[wave] = first;
        }
        __syncthreads();
        for (int w = 0; w < kThreads / 64; ++w) acc += s_cnt[w];
        if (tid == 0) A.tile_first[t] = min(min(s_first[0], s_first[1]), min(s_first[2], s_first[3]));
        __syncthreads();
    }
    if (tid == 0) A.tile_part[blockIdx.x] = acc;
}

// Both statistics of the planned units in one launch: Huffman chunk sizes, then
// run counts per run-length tile.  FEW: at most kPlanUnits units.
template <bool FEW>
__global__ __launch_bounds__(kThreads) void k_counts(const LosslessArgs* __restrict__ Ap)
{
    const LosslessArgs& A = *Ap;
    if constexpr (FEW) {
        __shared__ uint32_t s_chunk[kPlanUnits + 1], s_tile[kPlanUnits + 1];
        __shared__ uint64_t s_wave[kThreads / 64];
        const uint64_t total = plan_units<kThreads>(A, s_wave, [&](uint32_t u, uint64_t at) {
            s_chunk[u] = (uint32_t)at;
            s_tile[u] = (uint32_t)(at >> 32);
            if (blockIdx.x == 0) store_plan(A, u, at);
        });
        __syncthreads();
        huf_count_body(A, s_chunk, (uint32_t)total);
        rle_count_body(A, s_tile, (uint32_t)(total >> 32));
    } else {
        huf_count_body(A, A.chunk_base, A.counts[0]);
        rle_count_body(A, A.tile_base, A.counts[1]);
    }
}

// The shares' totals to their exclusive scans, each unit's first word / run to
// its absolute place, then every unit's stream bytes and arena offset (exclusive
// scan of the 256-byte-aligned sizes), and the headers of empty streams.
__global__ __launch_bounds__(1024) void k_unit_sizes(const LosslessArgs* __restrict__ Ap)
{
    __shared__ uint64_t s_wave[16];
    __shared__ uint32_t s_part[kPersistWaves];
    const LosslessArgs& A = *Ap;
    const uint32_t tid = threadIdx.x;
    static_assert(kPersistWaves == 4096 && kPersistWg == 1024, "four shares and one a thread");
    {
        const u32x4 p = reinterpret_cast<const u32x4*>(A.wave_part)[tid];
        const uint32_t q = A.tile_part[tid];
        // words (low half; sums may wrap, only differences are used) and runs
        uint64_t ex;
        block_scan64<1024>(((uint64_t)q << 32) | 0u, s_wave, ex);
        A.tile_part[tid] = (uint32_t)(ex >> 32);
        block_scan64<1024>((uint64_t)p.x + p.y + p.z + p.w, s_wave, ex);
        const uint32_t b = (uint32_t)ex;
        const u32x4 o = u32x4{b, b + p.x, b + p.x + p.y, b + p.x + p.y + p.z};
        reinterpret_cast<u32x4*>(A.wave_part)[tid] = o;
        reinterpret_cast<u32x4*>(s_part)[tid] = o;
    }
    __syncthreads();  // (also the tile parts: read back below by other threads of this workgroup)
    const uint32_t cs = max(1u, chunk_share(A.counts[0])), ts = max(1u, tile_share(A.counts[1]));
    const uint32_t per = (A.U + 1023) / 1024, u0 = min(tid * per, A.U), u1 = min(u0 + per, A.U);
    const auto work = gmem(A.work);
    const auto ubytes = gmem(A.unit_bytes);  // Huffman: without its words so far
    const auto hlo = gmem(A.huf_lo);
    const auto hhi = gmem(A.huf_hi);
    const auto cbase = gmem(A.chunk_base);
    uint64_t sum = 0;
    for (uint32_t u = u0; u < u1; u += kUnitFly) {
        uint64_t w[kUnitFly], by[kUnitFly];
        uint32_t lo[kUnitFly], hi[kUnitFly], c0[kUnitFly];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) {
            const uint32_t i = min(u + k, u1 - 1);
            w[k] = work[i], by[k] = ubytes[i], lo[k] = hlo[i], hi[k] = hhi[i], c0[k] = cbase[i];
        }
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) {
            if (u + k >= u1) break;
            const uint32_t nch = (uint32_t)w[k], tiles = (uint32_t)((w[k] & kWorkCounts) >> 32);
            if (nch) {
                const uint32_t first = s_part[c0[k] / cs] + lo[k];
                by[k] += 4ull * (s_part[(c0[k] + nch - 1) / cs] + hi[k] - first);
                hlo[u + k] = first;
                ubytes[u + k] = by[k];
            }
            if (tiles) A.rle_lo[u + k] += A.tile_part[A.tile_base[u + k] / ts];
            sum += w[k] >> 62 ? (by[k] + 255) & ~255ull : 0;
        }
    }
    uint64_t at;
    const uint64_t total = block_scan64<1024>(sum, s_wave, at);
    const bool over = total > A.cap;
    for (uint32_t u = u0; u < u1; u += kUnitFly) {
        uint64_t w[kUnitFly], by[kUnitFly];
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) {
            const uint32_t i = min(u + k, u1 - 1);
            w[k] = work[i], by[k] = ubytes[i];
        }
#pragma unroll
        for (uint32_t k = 0; k < kUnitFly; ++k) {
            if (u + k >= u1) break;
            gmem(A.pay_off)[u + k] = at;
            const uint32_t method = (uint32_t)(w[k] >> 62);
            if (method == 0) continue;
            if ((w[k] & kWorkCounts) == 0 && !over) {  // an empty stream's header
                uint32_t* p = reinterpret_cast<uint32_t*>(A.arena + at);
                if (method == 2) {  // nsym 0, no code lengths, off[0] = 0
                    for (uint32_t q = 0; q < (kHufHeader + 4) / 4; ++q) p[q] = 0;
                } else {
                    p[0] = 0;
                    p[1] = 4 * A.G;
                }
            }
            at += (by[k] + 255) & ~255ull;
        }
    }
    if (tid == 0) {
        A.counts[2] = over ? 1u : 0u;
        A.counts[4] = (uint32_t)total;
        A.counts[5] = (uint32_t)(total >> 32);
    }
}

// Huffman payloads.  A batch's chunks go back to back into the wave's LDS
// buffer, each from a word boundary as in the stream: a lane's bits start at
// its chunk's word offset (the batch's earlier chunks, from their segment
// totals) plus the exclusive scan of its group plus the bits of the chunk's
// earlier loads.  A lane's sixteen codes go in as eight pairs (at most 24 bits,
// so one or two words each) with atomic ORs; the batch then leaves as one
// coalesced run of words, and each chunk's first lane writes its offset.  The
// first chunk's wavefront writes the header, the last one's the closing offset.
template <bool FULL>
__device__ __forceinline__ void huf_emit_load(const HufBatch& hb, uint32_t r, const uint32_t* LC, uint32_t* buf,
                                              uint32_t seg, uint32_t lpc, uint32_t nbt, uint32_t lane,
                                              uint32_t& boff, uint32_t& run, uint32_t* off, uint32_t gw)
{
    // the lane's eight code pairs (code, length), in stream order
    uint32_t cp[8], lp[8], T = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t w = hb.w[r][i];
        const bool in = FULL || i < hb.valid[r];
#pragma unroll
        for (uint32_t p = 0; p < 2; ++p) {
            const uint32_t a = LC[(w >> (16 * p)) & 0xFF], b = LC[(w >> (16 * p + 8)) & 0xFF];
            const uint32_t lb = b >> 16, L = (a >> 16) + lb;
            cp[2 * i + p] = in ? ((a & 0xFFFFu) << lb) | (b & 0xFFFFu) : 0u;
            lp[2 * i + p] = in ? L : 0u;
            T += in ? L : 0u;
        }
    }
    const uint32_t x = seg_incl_scan(T, seg);
    uint32_t pos;
    if (lpc == 1) {
        // chunks of this load: one per segment; the lane's chunk starts after
        // the earlier segments' words
        const uint32_t sg = lane / seg;
        uint32_t coff = boff, add = 0;
        for (uint32_t k = 0; k < 64 / seg; ++k) {
            const uint32_t wk = ((uint32_t)__builtin_amdgcn_readlane((int)x, (int)(k * seg + seg - 1)) + 31) / 32;
            coff += sg > k ? wk : 0u;
            add += wk;
        }
        const uint32_t cj = r * (64 / seg) + sg;
        if ((lane & (seg - 1)) == 0 && cj < nbt) *gmem(off + cj) = gw + coff;
        pos = 32 * coff + x - T;
        boff += add;
    } else {
        if (r % lpc == 0) {
            run = 0;
            if (lane == 0 && r / lpc < nbt) *gmem(off + r / lpc) = gw + boff;
        }
        pos = 32 * boff + run + x - T;
        run += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        if (r % lpc == lpc - 1) boff += (run + 31) / 32;
    }
    if (T != 0) {
        uint32_t P = pos;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            // bits [P, P + lp) of the stream, most significant first: in the
            // 64-bit window of words P / 32 and P / 32 + 1 the pair's last bit
            // sits 64 - lp - P % 32 bits up (an empty pair adds nothing)
            const uint64_t v = (uint64_t)cp[k] << ((64u - lp[k] - (P & 31u)) & 63u);
            uint32_t* q = buf + (P >> 5);
            atomicOr(q, (uint32_t)(v >> 32));
            atomicOr(q + 1, (uint32_t)v);
            P += lp[k];
        }
    }
}

// LDS words of one wave's batch buffer: cpb chunks of at most chunk * 12 bits,
// plus the word after the last (a pair's second OR may touch it), in 16-byte units
__host__ __device__ constexpr uint32_t huf_buf_words(uint32_t huf_chunk)
{
    return ((4 * kHufLoads / (huf_chunk / 256)) * ((huf_chunk * kLutBitsMax + 31) / 32) + 4 + 3) / 4 * 4;
}

__device__ __forceinline__ void huf_write_body(const LosslessArgs& A, uint32_t buf_words)
{
    extern __shared__ __align__(16) uint32_t s_buf[];  // [kThreads / 64][buf_words]
    __shared__ uint32_t s_lc[kThreads / 64][256];      // code | length << 16 of each symbol
    if (A.counts[2]) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t total = A.counts[0];
    uint32_t* LC = s_lc[wave];
    const uint32_t cw = A.huf_chunk / 4, wpl = A.huf_chunk / 256;
    const uint32_t cpb = 4 * kHufLoads / wpl;  // chunks per batch
    const uint32_t seg = min(64u, 16 * wpl), lpc = wpl > 4 ? wpl / 4 : 1;
    const uint32_t cmax = (A.huf_chunk * kLutBitsMax + 31) / 32;  // words of a chunk at most
    uint32_t* buf = s_buf + wave * buf_words;
    uint32_t wv, c0, c1;
    wave_share(total, wv, c0, c1);
    uint32_t acc = c0 < c1 ? A.wave_part[wv] : 0u;  // words before the batch, over every unit
    uint32_t u = 0, cb_lo = 1, cb_hi = 0, nch = 0, base = 0;
    uint64_t nwu = 0;
    uint8_t* pay = nullptr;
    auto sync_wave = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (uint32_t c = c0; c < c1;) {
        if (c < cb_lo || c >= cb_hi) {
            u = find_unit(A.chunk_base, A.U, c);
            cb_lo = A.chunk_base[u];
            cb_hi = A.chunk_base[u + 1];
            nwu = A.units[u].S / 4;
            nch = A.units[u].nchunks;
            base = A.huf_lo[u];
            pay = A.arena + A.pay_off[u];
            for (uint32_t k = lane; k < 256; k += 64)
                LC[k] = A.codes[(uint64_t)u * 256 + k] | ((uint32_t)A.lens[(uint64_t)u * 256 + k] << 16);
        }
        const uint32_t nbt = min(cpb, min(c1, cb_hi) - c);
        // zero the batch's words (and the one after them) for the ORs
        const uint32_t nclr = (nbt * cmax + 4) / 4;
        for (uint32_t i = lane; i < nclr; i += 64) reinterpret_cast<u32x4*>(buf)[i] = u32x4{0u, 0u, 0u, 0u};
        sync_wave();
        HufBatch hb;
        const bool full = huf_load_batch(unit_rows(A, u), (uint64_t)(c - cb_lo) * cw, nbt * cw, nwu, lane, hb);
        const uint32_t lc0 = c - cb_lo;               // the batch's first chunk in the unit
        const uint32_t gw = acc - base;               // and its first word in the stream
        uint32_t* const poff = reinterpret_cast<uint32_t*>(pay + kHufHeader);
        const auto off = gmem(poff);
        const auto words = off + nch + 1;
        uint32_t boff = 0, run = 0;  // words of the batch's finished chunks; bits of the chunk's earlier loads
        if (full) {
#pragma unroll
            for (uint32_t r = 0; r < kHufLoads; ++r)
                huf_emit_load<true>(hb, r, LC, buf, seg, lpc, nbt, lane, boff, run, poff + lc0, gw);
        } else {
#pragma unroll
            for (uint32_t r = 0; r < kHufLoads; ++r)
                huf_emit_load<false>(hb, r, LC, buf, seg, lpc, nbt, lane, boff, run, poff + lc0, gw);
        }
        sync_wave();
        for (uint32_t i = lane; i < boff; i += 64) words[gw + i] = buf[i];
        if (lane == 0 && lc0 + nbt == nch) off[nch] = gw + boff;
        if (lc0 == 0) {
            const UnitInfo& ui = A.units[u];
            if (lane == 0) *reinterpret_cast<uint64_t*>(pay) = ui.S;
            const uint32_t b4 = lane * 4;
            reinterpret_cast<uint32_t*>(pay + 8)[lane] = (LC[b4] >> 16) | ((LC[b4 + 1] >> 16) << 8) |
                                                         ((LC[b4 + 2] >> 16) << 16) | ((LC[b4 + 3] >> 16) << 24);
        }
        sync_wave();  // the buffer is cleared again by the next batch
        c += nbt;
        acc += boff;
    }
}

// Run-length payloads: every run start stores its symbol and its length, the
// distance to the next run's start.  Run r of a unit = the runs of its earlier
// tiles + starts before the word inside the tile; the next start is the
// thread's, else the first of a later thread of the tile, else the first of a
// later tile (tile_first), else the unit's end.  A tile that starts no run has
// nothing to write and is left out, so only tiles with a start look ahead, each
// up to the next of them: the search is linear in the unit's tiles.  (With
// every tile searching, constant units took steps in the square of theirs: the
// stage over 2^28 f32 zeros in one unit of 32 planes, 65536 tiles, 5.95 ms, now
// 0.80; with values that alternate from tile to tile 2.64 and 1.50.)
constexpr int kRlePer = kRleTileWords / kThreads;  // consecutive words per thread

__device__ __forceinline__ void rle_write_body(const LosslessArgs& A)
{
    __shared__ uint32_t s_wave[kThreads / 64];
    __shared__ uint32_t s_first[kThreads], s_wfirst[kThreads / 64 + 1];
    if (A.counts[2]) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t total = A.counts[1], G = A.G;
    const uint32_t t0 = min(blockIdx.x * tile_share(total), total), t1 = min(t0 + tile_share(total), total);
    uint32_t acc = t0 < t1 ? A.tile_part[blockIdx.x] : 0u;  // runs before the tile, over every unit
    uint32_t u = 0, tb_lo = 1, tb_hi = 0;                   // tiles [tb_lo, tb_hi) belong to unit u
    for (uint32_t t = t0; t < t1; ++t) {
        if (t < tb_lo || t >= tb_hi) {
            u = find_unit(A.tile_base, A.U, t);
            tb_lo = A.tile_base[u];
            tb_hi = A.tile_base[u + 1];
        }
        if (A.tile_first[t] == kNoStart) continue;  // the whole workgroup
        const UnitInfo& ui = A.units[u];
        const uint32_t* g = unit_rows(A, u);
        const uint64_t nw = ui.S / (4ull * G), nruns = ui.nruns;
        uint8_t* pay = A.arena + A.pay_off[u];
        uint32_t* sym = reinterpret_cast<uint32_t*>(pay + 8);
        uint32_t* lens = reinterpret_cast<uint32_t*>(pay + 8 + 4ull * G * nruns);
        const uint32_t lt = t - tb_lo;
        const uint64_t i0 = (uint64_t)lt * kRleTileWords + (uint64_t)tid * kRlePer;
        uint32_t flags = 0;
        for (int k = 0; k < kRlePer; ++k) {
            const uint64_t i = i0 + k;
            const bool f = i < nw && (i == 0 || word_ne(g, i, i - 1, G));
            flags |= f ? (1u << k) : 0u;
        }
        // the first start past this tile: later tiles of the unit, 256 at a time
        uint32_t past = (uint32_t)nw;
        for (uint32_t q = t + 1; q < tb_hi; q += kThreads) {
            const unsigned long long has = __ballot(q + tid < tb_hi && A.tile_first[q + tid] != kNoStart);
            if (lane == 0) s_wave[wave] = has ? q + 64 * wave + (uint32_t)__ffsll(has) - 1 : kNoStart;
            __syncthreads();
            const uint32_t with = min(min(s_wave[0], s_wave[1]), min(s_wave[2], s_wave[3]));
            __syncthreads();
            if (with != kNoStart) {
                past = (with - tb_lo) * kRleTileWords + A.tile_first[with];
                break;
            }
        }
        const uint32_t first = flags ? (uint32_t)i0 + (uint32_t)__ffs(flags) - 1 : kNoStart;
        const unsigned long long any = __ballot(flags != 0);
        s_first[tid] = first;
        if (lane == 0) s_wfirst[wave] = any ? (uint32_t)__ffsll(any) - 1 + 64 * wave : kNoStart;  // a thread
        uint32_t excl;
        const uint32_t tile_total = block_excl_scan((uint32_t)__popc(flags), s_wave, excl);  // (a barrier inside)
        uint32_t next = past;  // the first start after this thread's words
        {
            const unsigned long long later = lane == 63 ? 0 : any >> (lane + 1);
            uint32_t th = later ? tid + (uint32_t)__ffsll(later) : kNoStart;
            for (uint32_t w = wave + 1; w < kThreads / 64 && th == kNoStart; ++w) th = s_wfirst[w];
            if (th != kNoStart) next = s_first[th];
        }
        uint64_t r = (uint64_t)(acc - A.rle_lo[u]) + excl;
        if (lt == 0 && tid == 0) {
            reinterpret_cast<uint32_t*>(pay)[0] = (uint32_t)nruns;
            reinterpret_cast<uint32_t*>(pay)[1] = 4 * G;
        }
        while (flags) {
            const uint32_t k = (uint32_t)__ffs(flags) - 1;
            flags &= flags - 1;
            const uint32_t i = (uint32_t)i0 + k, end = flags ? (uint32_t)i0 + (uint32_t)__ffs(flags) - 1 : next;
            if (r < nruns) {
                sym[r * G] = g[(uint64_t)i * G];
                if (G == 2) sym[r * G + 1] = g[(uint64_t)i * G + 1];
                lens[r] = end - i;
            }
            ++r;
        }
        acc += tile_total;
        __syncthreads();  // s_first, s_wfirst are written again by the next tile
    }
}

// Payload writes: Huffman streams, then run-length ones (different units).
__global__ __launch_bounds__(kThreads) void k_write(const LosslessArgs* __restrict__ Ap, uint32_t buf_words)
{
    const LosslessArgs& A = *Ap;
    huf_write_body(A, buf_words);
    rle_write_body(A);
}

// ------------------------------------------------------------------ Huffman decode
// The first-code table of a stream, built in LDS by a workgroup of kTabThreads
// from the 256 code lengths of its header: entry i of the 2^lmax-entry table
// holds (length << 8) | symbol of the code that the lmax-bit window i starts
// with (codes are prefix-free, so the bits after it do not matter).  A window
// that starts with no code (possible only for an incomplete code) consumes
// lmax bits as symbol 0.  Ends with a barrier.
constexpr int kTabThreads = 1024;  // four windows a thread: a launch of few streams waits on their chains

__device__ __forceinline__ void build_first_code_table(const uint8_t* __restrict__ payload, uint32_t lmax,
                                       uint16_t* s_one, uint32_t (*s_wcnt)[kLutBitsMax + 1],
                                       uint8_t* s_sym)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t nent = 1u << lmax;
    // canonical code of symbol `tid`: the first code of its length plus the
    // smaller symbols of that length (wavefront ballots, then the counts of
    // the earlier wavefronts)
    const uint32_t L = tid < 256 ? payload[8 + tid] : 0u;
    const bool has = L != 0 && L <= lmax;
    uint32_t before = 0, mine = 0;  // lane l of mine: this wavefront's symbols of length l
#pragma unroll
    for (uint32_t l = 1; l <= (uint32_t)kLutBitsMax; ++l) {
        const unsigned long long bl = __ballot(has && L == l);
        mine = lane == l ? (uint32_t)__popcll(bl) : mine;
        if (has && L == l) before = (uint32_t)__popcll(bl & ((1ull << lane) - 1));
    }
    if (wave < 4 && lane >= 1 && lane <= (uint32_t)kLutBitsMax) s_wcnt[wave][lane] = mine;
    __syncthreads();
    uint32_t all = 0, earlier = 0;  // lane l: symbols of length l in all, and in the earlier wavefronts
    if (lane >= 1 && lane <= (uint32_t)kLutBitsMax) {
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            const uint32_t c = s_wcnt[w][lane];
            all += c;
            earlier += w < wave ? c : 0u;
        }
    }
    // per length l (all in registers): lim[l] = end of the lmax-bit windows
    // whose first code has length <= l (non-decreasing in l); base[l] = index
    // of the first symbol of length l minus the first code of that length
    uint32_t lim[kLutBitsMax + 1], base[kLutBitsMax + 1], lim_all = 0;
    {
        uint32_t first = 0, idx = 0;
#pragma unroll
        for (int l = 1; l <= kLutBitsMax; ++l) {
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)all, l);  // 0 past lmax
            const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)earlier, l);
            if (has && (uint32_t)l == L) s_sym[idx + e + before] = (uint8_t)tid;
            base[l] = idx - first;
            lim[l] = l <= (int)lmax ? (first + cnt) << (lmax - l) : nent;
            if (l == (int)lmax) lim_all = lim[l];
            idx += cnt;
            first = (first + cnt) << 1;
        }
    }
    __syncthreads();
    // first code of every window (independent entries)
    for (uint32_t i = tid; i < nent; i += kTabThreads) {
        uint32_t Lx = 1, bx = base[1];
#pragma unroll
        for (int l = 1; l < kLutBitsMax; ++l) {
            const bool past = l < (int)lmax && lim[l] <= i;
            Lx += past ? 1u : 0u;
            bx = past ? base[l + 1] : bx;
        }
        const bool code = i < lim_all;  // then Lx is the leading code's length
        s_one[i] = code ? (uint16_t)((Lx << 8) | s_sym[bx + (i >> (lmax - Lx))]) : (uint16_t)(lmax << 8);
    }
    __syncthreads();
}

// The decode tables of a launch, one workgroup per stream, built once and
// stored to the job's table slot (the decoders' workgroups copy them to LDS
// instead of each building them).  The multi-symbol table: 2^lmax entries
// mapping the next lmax bits to up to three symbols (every code lying wholly
// inside the window is decoded by that one lookup): symbols | count << 24 |
// bits << 26.  COUNT (the G-lane decoder): behind it the counting table, all
// whole codes of the window (up to lmax) and the first one's length: count |
// bits << 4 | first << 8, 16 bits an entry.
// The first launch to need the descriptor can also bring it: with `words`, the
// jobs are read from pinned host memory and the workgroups past them copy the
// descriptor from src to dst (a launch of its own took 4 us).
__device__ __forceinline__ uint32_t spread(uint32_t i) { return i ^ (i >> 6); }

template <bool COUNT>
__global__ __launch_bounds__(kTabThreads) void k_huf_tables(const DecodeJob* jobs, uint32_t njobs, const uint64_t* src,
                                                            uint64_t* __restrict__ dst, uint64_t words)
{
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x >= njobs) {
        const uint64_t stride = (uint64_t)(gridDim.x - njobs) * kTabThreads;
        for (uint64_t i = (uint64_t)(blockIdx.x - njobs) * kTabThreads + tid; i < words; i += stride)
            dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    __shared__ DecodeJob s_job;
    static_assert(sizeof(DecodeJob) % 8 == 0 && sizeof(DecodeJob) / 8 <= 64, "a job is a few 64-bit words");
    if (tid < sizeof(DecodeJob) / 8)
        reinterpret_cast<uint64_t*>(&s_job)[tid] = __hip_atomic_load(
            reinterpret_cast<const uint64_t*>(jobs + blockIdx.x) + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __syncthreads();
    const DecodeJob job = s_job;
    const uint32_t lmax = job.lmax, nent = 1u << lmax, mask = nent - 1;
    __shared__ uint16_t s_one[1 << kLutBitsMax];
    __shared__ uint32_t s_three[COUNT ? 1 << kLutBitsMax : 1];
    __shared__ uint32_t s_wcnt[4][kLutBitsMax + 1];
    __shared__ uint8_t s_sym[256];
    build_first_code_table(job.payload, lmax, s_one, s_wcnt, s_sym);
    // up to three whole codes per window: chains of first-code lookups, four
    // windows at a time so their LDS latencies overlap
    const auto t = gmem(reinterpret_cast<uint32_t*>(job.table));
    for (uint32_t i0 = tid; i0 < nent; i0 += 4 * kTabThreads) {
        uint32_t syms[4] = {0, 0, 0, 0}, k[4] = {0, 0, 0, 0}, used[4] = {0, 0, 0, 0};
#pragma unroll
        for (uint32_t step = 0; step < 3; ++step) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t i = i0 + q * kTabThreads;
                const uint32_t e = s_one[(i << used[q]) & mask];
                const uint32_t l = e >> 8;
                if (k[q] == step && used[q] + l <= lmax) {  // no earlier code ended the chain, and this one fits
                    syms[q] |= (e & 0xFFu) << (8 * step);
                    ++k[q];
                    used[q] += l;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = i0 + q * kTabThreads;
            if (i >= nent) continue;
            const uint32_t e = syms[q] | (k[q] << 24) | (used[q] << 26);
            t[i] = e;
            if (COUNT) s_three[spread(i)] = e;
        }
    }
    if (!COUNT) return;
    __syncthreads();
    // all whole codes: three at a time while they fit, then one at a time.  What
    // consecutive windows look up after one-bit codes lies 8 and then 64 entries
    // apart, in few banks; `spread` puts it in all of them (retrieval of 2^18
    // constant f32 values 46.3 -> 42.8 us, of 2^21 f64 ones 63.9 -> 60.5)
    const auto tc = gmem(reinterpret_cast<uint16_t*>(job.table) + 2 * nent);
    for (uint32_t i0 = tid; i0 < nent; i0 += 4 * kTabThreads) {
        uint32_t k[4], used[4];
        bool open[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t e = s_three[spread((i0 + q * kTabThreads) & mask)];
            k[q] = (e >> 24) & 3u;
            used[q] = e >> 26;
            open[q] = k[q] == 3 && used[q] < lmax;  // fewer than three: the next code does not fit
        }
        while (__ballot(open[0] || open[1] || open[2] || open[3])) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t at = ((i0 + q * kTabThreads) << used[q]) & mask;
                const uint32_t e = s_three[spread(at)], left = lmax - used[q];
                uint32_t dk = (e >> 24) & 3u, du = e >> 26;
                if (du > left) {
                    dk = 1;
                    du = (uint32_t)s_one[at] >> 8;
                }
                const bool fits = open[q] && du <= left;
                k[q] += fits ? dk : 0u;
                used[q] += fits ? du : 0u;
                // a group of fewer than three that fits was cut by the window's
                // end or its last code's: one code at a time finds what is left
                open[q] = fits && used[q] < lmax;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = i0 + q * kTabThreads;
            if (i < nent) tc[i] = (uint16_t)(k[q] | (used[q] << 4) | (((uint32_t)s_one[i] >> 8) << 8));
        }
    }
}

// copies a job's table of `words` 32-bit words to LDS with 16-byte loads
// (tables sit at kHufTableBytes strides, and 2^lmax words are a multiple of 8 for lmax >= 3)
template <int NT>
__device__ __forceinline__ void load_table(const void* table, uint32_t words, uint32_t* lds)
{
    const auto src = gmem(reinterpret_cast<const u32x4*>(table));
    u32x4* dst = reinterpret_cast<u32x4*>(lds);
    for (uint32_t i = threadIdx.x; i < (words + 3) / 4; i += NT) dst[i] = src[i];
}

// One thread per chunk, kThreads chunks per workgroup (the launch for many
// chunks), through the multi-symbol table: skewed groups, whose frequent
// symbols have 1-3 bit codes, take a third of the dependent lookups of a
// one-symbol table; a 4-byte entry keeps the table at 16 KiB, so that eight
// workgroups fit a CU.  Compressed words arrive in 16-byte blocks one block
// ahead of their use, each iteration takes at most one word and makes two
// lookups, and decoded bytes leave in 64-byte pieces.
__global__ __launch_bounds__(kThreads) void k_huf_decode(const DecodeJob* __restrict__ jobs,
                                                         const uint32_t* __restrict__ wg_job)
{
    const DecodeJob& job = jobs[wg_job[blockIdx.x]];
    const uint8_t* payload = job.payload;
    const uint64_t S = job.S;
    const uint32_t chunk = job.chunk, lmax = job.lmax, nchunks = job.nchunks;
    __shared__ __align__(16) uint32_t s_multi[1 << kLutBitsMax];  // symbols | count << 24 | bits << 26
    const uint32_t tid = threadIdx.x;
    load_table<kThreads>(job.table, 1u << lmax, s_multi);
    __syncthreads();  // the only barrier

    const uint32_t c = (blockIdx.x - job.wg_base) * kThreads + tid;
    if (c >= nchunks) return;
    const auto off = gmem(reinterpret_cast<const uint32_t*>(payload + kHufHeader));
    const uint32_t wb = off[c], we = off[c + 1];
    // words past the chunk's end are never decoded: read the last one instead
    const uint32_t wl = we > wb ? we - 1 : wb;
    const uint64_t lo = (uint64_t)c * chunk;
    const uint32_t cnt = (uint32_t)((lo + chunk <= S) ? chunk : S - lo);  // a multiple of 4
    const auto dst4 = gmem(reinterpret_cast<u32x4*>(job.out + lo));
    // Compressed words arrive as aligned 16-byte blocks, two in flight: a
    // thread's stream is its own, and with one word per load every line came
    // from memory several times over before the thread had used it up.  Block
    // k holds words 4k - delta .. 4k - delta + 3 of the chunk data (delta puts
    // the data's start on its 16-byte grid); the first block may begin before
    // the chunk and the last may end past it (a stream's allocation is padded
    // to 256 bytes), but no block past the one holding word wl is read.
    const uintptr_t wbase = reinterpret_cast<uintptr_t>(payload + kHufHeader + 4ull * (nchunks + 1));
    const uint32_t delta = (uint32_t)((wbase & 15u) >> 2);
    const auto blk4 = gmem(reinterpret_cast<const u32x4*>(wbase & ~(uintptr_t)15));
    const uint32_t b0 = (wb + delta) >> 2, j0 = (wb + delta) & 3u, bl = (wl + delta) >> 2;
    u32x4 qa = blk4[b0], qb = blk4[min(b0 + 1, bl)];
    uint32_t bnext = b0 + 2, jq = j0;  // qa's next word (the first block may begin before the chunk)
    uint64_t buf = 0;
    int nb = 0;
    uint64_t pend = 0;  // decoded bytes not yet in a whole word (at most three between lookups)
    uint32_t npend = 0, done = 0, wo = 0, nob = 0, nsl = 0;
    // decoded words leave in whole 64-byte pieces: ob collects four words, the
    // slots s0..s2 the three vectors before it (a line written at once is
    // written once; 16-byte pieces of lines far apart were written back piecemeal)
    u32x4 ob = {0, 0, 0, 0}, s0 = {0, 0, 0, 0}, s1 = {0, 0, 0, 0}, s2 = {0, 0, 0, 0};
    // One lookup: up to three symbols into pend, and a whole word out of it
    // when there is one.  The window is whole: at least lmax bits are in the
    // buffer (or the chunk's data has ended; symbols from the bits past it lie
    // past its end, never complete a word, and are never stored).
    auto lookup = [&]() {
        const uint32_t e = s_multi[buf >> (64 - lmax)];
        const uint32_t k = (e >> 24) & 3u, used = e >> 26;
        pend |= (uint64_t)(e & 0xFFFFFFu) << (8 * npend);  // bytes past the k symbols are 0
        npend += k;
        done += k;
        buf <<= used;
        nb -= (int)used;
        if (npend >= 4) {
            ob = u32x4{ob.y, ob.z, ob.w, (uint32_t)pend};  // oldest word first once full
            pend >>= 32;
            npend -= 4;
            if (++nob == 4) {
                nob = 0;
                if (nsl == 3) {
                    dst4[wo] = s0;
                    dst4[wo + 1] = s1;
                    dst4[wo + 2] = s2;
                    dst4[wo + 3] = ob;
                    wo += 4;
                    nsl = 0;
                } else {
                    // the held vectors move down one slot: after three, s0..s2 hold them in order
                    s0 = s1;
                    s1 = s2;
                    s2 = ob;
                    ++nsl;
                }
            }
        }
    };
    // Every lane takes at most one word and makes two lookups per iteration
    // (a lookup uses at most lmax <= 12 bits, and after the refill at least 32
    // are held), so a wavefront iterates as often as its longest chunk needs
    // lookups, halved, instead of the sum over words of each word's slowest lane.
    while (done < cnt) {
        if (nb <= 32) {
            const uint32_t w = jq == 0 ? qa.x : jq == 1 ? qa.y : jq == 2 ? qa.z : qa.w;
            buf |= (uint64_t)w << (32 - nb);
            nb += 32;
            if (++jq == 4) {
                jq = 0;
                qa = qb;
                qb = blk4[min(bnext++, bl)];
            }
        }
        lookup();
        if (done < cnt) lookup();
    }
    // a chunk ends on a word: the whole vectors held in the slots, then up to
    // three words, the newest nob of ob (in order)
    if (nsl > 2) dst4[wo++] = s0;
    if (nsl > 1) dst4[wo++] = s1;
    if (nsl > 0) dst4[wo++] = s2;
    const auto dst = gmem(reinterpret_cast<uint32_t*>(job.out + lo)) + 4 * wo;
    if (nob == 3) {
        dst[0] = ob.y;
        dst[1] = ob.z;
        dst[2] = ob.w;
    } else if (nob == 2) {
        dst[0] = ob.z;
        dst[1] = ob.w;
    } else if (nob == 1) {
        dst[0] = ob.w;
    }
}

// ------------------------------------------------------------------ Huffman decode, G lanes a chunk
// For launches with too few chunks to fill the chip, where one thread per
// chunk leaves a 256-symbol chain of dependent lookups as the launch's
// latency.  A chunk's compressed bits are cut into G equal ranges and lane g
// of the chunk's G lanes decodes the codes that start in range g.  Only lane 0
// knows where its first code starts; lane g > 0 starts at its range's first
// bit, decodes to past its range's end, and the end it reaches becomes lane
// g+1's next start, until no start moves.  The chain of starts is then the
// one a serial decode passes through (lane 0's is right from the first round,
// and each round makes at least one more lane right, so G rounds always end
// it; a prefix code falls back into step with the true boundaries within a
// few codes, so two or three rounds are usual).  A prefix sum of the lanes'
// counts places their symbols, a last walk writes them to LDS, and the
// workgroup stores its chunks' bytes with 16-byte stores.
// Bound by the walks' dependent LDS lookups: the counting walks take all whole
// codes of a 12-bit window at once, the last one up to three symbols (one code
// a lookup, a workgroup took 45000 cycles instead of 24000, and the smallest
// launch 21 us instead of 14).
constexpr uint32_t kSplitOut = 16384;                            // decoded bytes a workgroup holds
constexpr uint32_t kSplitWords = kSplitOut * kLutBitsMax / 32;   // their compressed words, at most

// The bits of a chunk (words W[qb..ql], MSB first) from bit `pos` on: at least
// 32 valid at a lookup, the next word loaded ahead of its use.
struct BitReader {
    const uint32_t* W;
    uint32_t q, ql, next, nb;
    uint64_t buf;
    __device__ __forceinline__ BitReader(const uint32_t* W_, uint32_t qb, uint32_t ql_, uint32_t pos) : W(W_), ql(ql_)
    {
        q = qb + (pos >> 5);
        const uint32_t sh = pos & 31u;
        buf = ((((uint64_t)W[min(q, ql)]) << 32) | W[min(q + 1, ql)]) << sh;
        next = W[min(q + 2, ql)];
        nb = 64 - sh;
        q += 3;
    }
    __device__ __forceinline__ uint32_t window(uint32_t lmax)
    {
        if (nb < 32) {
            buf |= (uint64_t)next << (32 - nb);
            nb += 32;
            next = W[min(q++, ql)];
        }
        return (uint32_t)(buf >> (64 - lmax));
    }
    __device__ __forceinline__ void skip(uint32_t n)
    {
        buf <<= n;
        nb -= n;
    }
};

// Counts the codes that start in [pos, hi); returns where the walk stops, the
// start of the first code at or past hi.  A lookup takes all whole codes of its
// window while the window ends before hi, then one at a time.
__device__ __forceinline__ uint32_t huf_count(const uint32_t* W, uint32_t qb, uint32_t ql, const uint16_t* tab,
                                              uint32_t lmax, uint32_t pos, uint32_t hi, uint32_t& n)
{
    BitReader br(W, qb, ql, pos);
    n = 0;
    while (pos < hi) {
        const uint32_t e = tab[br.window(lmax)];
        const bool whole = pos + lmax <= hi;
        const uint32_t L = whole ? (e >> 4) & 15u : e >> 8;
        n += whole ? e & 15u : 1u;
        br.skip(L);
        pos += L;
    }
    return pos;
}

// Writes the `n` symbols from bit pos on to out, up to three a lookup.
__device__ __forceinline__ void huf_symbols(const uint32_t* W, uint32_t qb, uint32_t ql, const uint32_t* tab,
                                            uint32_t lmax, uint32_t pos, uint32_t n, uint8_t* out)
{
    BitReader br(W, qb, ql, pos);
    for (uint32_t j = 0; j < n;) {
        const uint32_t e = tab[br.window(lmax)];
        const uint32_t k = (e >> 24) & 3u;
        out[j] = (uint8_t)e;
        if (k > 1 && j + 1 < n) out[j + 1] = (uint8_t)(e >> 8);
        if (k > 2 && j + 2 < n) out[j + 2] = (uint8_t)(e >> 16);
        br.skip(e >> 26);
        j += k;
    }
}

// Dynamic LDS of a launch whose largest chunk is cap_chunk symbols: the
// multi-symbol and the counting table, then the compressed words and the decoded bytes of the
// workgroup's chunks.
constexpr uint32_t kSplitTables = (4u << kLutBitsMax) + (2u << kLutBitsMax);
__host__ __device__ constexpr uint32_t split_words_cap(uint32_t cpw, uint32_t cap_chunk)
{
    return cpw * cap_chunk * kLutBitsMax / 32;
}
__host__ __device__ constexpr uint32_t split_lds_bytes(uint32_t cpw, uint32_t cap_chunk)
{
    return kSplitTables + 4 * split_words_cap(cpw, cap_chunk) + cpw * cap_chunk;
}

template <int G, int NT>
__global__ __launch_bounds__(NT) void k_huf_decode_split(const DecodeJob* __restrict__ jobs,
                                                               const uint32_t* __restrict__ wg_job,
                                                               uint32_t cap_chunk)
{
    static_assert(G >= 4 && G <= 64 && (G & (G - 1)) == 0, "G lanes a chunk: 4..64, a power of two");
    constexpr uint32_t kCpw = NT / G;  // chunks per workgroup
    const DecodeJob& job = jobs[wg_job[blockIdx.x]];
    const uint8_t* payload = job.payload;
    const uint64_t S = job.S;
    const uint32_t chunk = job.chunk, lmax = job.lmax, nchunks = job.nchunks;
    // the launcher sizes LDS for cap_chunk and raises G so that kCpw * cap_chunk <= kSplitOut
    if (chunk > cap_chunk || kCpw * cap_chunk > kSplitOut) return;
    extern __shared__ __align__(16) uint8_t s_dyn[];
    uint32_t* s_multi = reinterpret_cast<uint32_t*>(s_dyn);
    const uint16_t* s_count = reinterpret_cast<const uint16_t*>(s_dyn + (4u << lmax));
    const uint32_t wcap = split_words_cap(kCpw, cap_chunk);
    uint32_t* s_words = reinterpret_cast<uint32_t*>(s_dyn + kSplitTables);
    uint8_t* s_out = s_dyn + kSplitTables + 4 * wcap;
    const uint32_t tid = threadIdx.x;
    const uint32_t c0 = (blockIdx.x - job.wg_base) * kCpw, c1 = min(c0 + kCpw, nchunks);
    const auto off = gmem(reinterpret_cast<const uint32_t*>(payload + kHufHeader));
    const auto wp = gmem(reinterpret_cast<const uint32_t*>(payload + kHufHeader + 4ull * (nchunks + 1)));
    // the workgroup's compressed words (its chunks are adjacent) and the
    // stream's table, both loads in flight at once
    const uint32_t w0 = off[c0], nw = min(off[c1] - w0, wcap);
    constexpr uint32_t kPer = kSplitWords / NT;
    uint32_t held[kPer];
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint32_t i = tid + r * NT;
        held[r] = i < nw ? wp[w0 + i] : 0u;
    }
    load_table<NT>(job.table, (1u << lmax) + (1u << lmax) / 2, s_multi);
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint32_t i = tid + r * NT;
        if (i < nw) s_words[i] = held[r];
    }
    __syncthreads();

    const uint32_t g = tid % G, cl = tid / G, c = c0 + cl;
    const bool live = c < c1;
    uint32_t qb = 0, ql = 0, nbits = 0, cnt = 0;
    if (live) {
        qb = min(off[c] - w0, wcap - 1);
        const uint32_t qe = min(off[c + 1] - w0, wcap);
        ql = qe > qb ? qe - 1 : qb;
        nbits = (qe > qb ? qe - qb : 0) * 32;
        const uint64_t lo = (uint64_t)c * chunk;
        cnt = (uint32_t)(lo + chunk <= S ? chunk : S - lo);
    }
    const uint32_t Lb = (nbits + G - 1) / G;
    const uint32_t lo_g = min(g * Lb, nbits), hi_g = min(lo_g + Lb, nbits);
    uint32_t start = lo_g, n = 0;
    for (int round = 0; round < G; ++round) {
        const uint32_t end = huf_count(s_words, qb, ql, s_count, lmax, start, hi_g, n);
        const uint32_t prev = __shfl_up(end, 1, G);
        // a lane whose range is empty (past the chunk's bits) decodes nothing
        // from any start: left out, it cannot hold the others up
        const bool moved = live && g != 0 && lo_g < hi_g && prev != start;
        if (__ballot(moved) == 0) break;  // every start is the end of the lane before
        if (moved) start = prev;
    }
    uint32_t incl = n;  // inclusive prefix sum of the counts over the chunk's lanes
#pragma unroll
    for (uint32_t d = 1; d < (uint32_t)G; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d, G);
        if (g >= d) incl += t;
    }
    const uint32_t o = incl - n;
    if (live && o < cnt)
        huf_symbols(s_words, qb, ql, s_multi, lmax, start, min(n, cnt - o), s_out + cl * chunk + o);
    __syncthreads();
    // the chunks' bytes are adjacent in the output too: a multiple of 4 bytes
    const uint64_t lo0 = (uint64_t)c0 * chunk;
    const uint32_t T = (uint32_t)(min((uint64_t)c1 * chunk, S) - lo0);
    const auto dst4 = gmem(reinterpret_cast<u32x4*>(job.out + lo0));
    const u32x4* src4 = reinterpret_cast<const u32x4*>(s_out);
    for (uint32_t i = tid; i < T / 16; i += NT) dst4[i] = src4[i];
    const uint32_t tw = (T & 15u) / 4;
    if (tid < tw) {
        const uint32_t i = (T & ~15u) / 4 + tid;
        gmem(reinterpret_cast<uint32_t*>(job.out + lo0))[i] = reinterpret_cast<const uint32_t*>(s_out)[i];
    }
}

// ------------------------------------------------------------------ RLE decode
// Every run-length group of a retrieval in one pass of three launches: the run
// lengths of all groups are gathered into one array, one exclusive scan turns
// them into run starts (a group's starts are its entries minus its first, so
// the scan's sums may wrap), and every W-bit word of every group finds its run
// by binary search over its group's starts.
__global__ __launch_bounds__(kThreads) void k_rle_gather(const RleJob* __restrict__ jobs,
                                                         const uint32_t* __restrict__ wg_job,
                                                         uint32_t* __restrict__ lens)
{
    const RleJob& job = jobs[wg_job[blockIdx.x]];
    const uint64_t r0 = (uint64_t)(blockIdx.x - job.wg_gather) * kRlePerWg;
    const uint64_t r1 = min(r0 + kRlePerWg, job.nruns);
    const auto src = gmem(reinterpret_cast<const uint32_t*>(job.payload + 8 + 4ull * job.G * job.nruns));
    for (uint64_t r = r0 + threadIdx.x; r < r1; r += kThreads) lens[job.run_base + r] = src[r];
}

__global__ __launch_bounds__(kThreads) void k_rle_expand(const RleJob* __restrict__ jobs,
                                                         const uint32_t* __restrict__ wg_job,
                                                         const uint32_t* __restrict__ starts)
{
    const RleJob& job = jobs[wg_job[blockIdx.x]];
    const uint32_t* st = starts + job.run_base;
    const uint32_t s0 = st[0];
    const auto sym = gmem(reinterpret_cast<const uint32_t*>(job.payload + 8));
    const auto g = gmem(reinterpret_cast<uint32_t*>(job.out));
    const uint32_t G = job.G;
    const uint64_t i0 = (uint64_t)(blockIdx.x - job.wg_expand) * kRlePerWg;
    const uint64_t i1 = min(i0 + kRlePerWg, job.nwords);
    for (uint64_t i = i0 + threadIdx.x; i < i1; i += kThreads) {
        // last run whose start is <= i (starts relative to the group's first)
        uint64_t lo = 0, hi = job.nruns;  // invariant: start[lo] <= i, answer in [lo, hi)
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if ((uint64_t)(uint32_t)(st[mid] - s0) <= i)
                lo = mid;
            else
                hi = mid;
        }
        for (uint32_t q = 0; q < G; ++q) g[i * G + q] = sym[lo * G + q];
    }
}

}  // namespace

// ------------------------------------------------------------------ launchers
static unsigned blocks_for(uint64_t items, uint64_t per, unsigned cap)
{
    uint64_t b = (items + per - 1) / per;
    if (b < 1) b = 1;
    return (unsigned)(b > cap ? cap : b);
}

uint64_t scan_temp_words(uint64_t n)
{
    uint64_t t = 0;
    while (n > 1) {
        n = (n + kScanTile - 1) / kScanTile;
        t += n + 64;
    }
    return t + 64;
}

hipError_t launch_scan_exclusive(const uint32_t* in, uint32_t* out, uint64_t n, uint32_t* temp,
                                 hipStream_t s)
{
    if (n == 0) return hipSuccess;
    uint64_t tiles = (n + kScanTile - 1) / kScanTile;
    uint32_t* sums = temp;
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(kThreads), 0, s, in, out, n, sums);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || tiles == 1) return err;
    err = launch_scan_exclusive(sums, sums, tiles, temp + tiles + 64, s);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)tiles), dim3(kThreads), 0, s, out, n, sums);
    return hipGetLastError();
}

hipError_t launch_lossless_batch(const LosslessArgs& a, const LosslessArgs* a_dev, hipStream_t s)
{
    if (a.U == 0) return hipSuccess;
    const dim3 P(kPersistWg), T(kThreads);
    if (a.U <= kPlanUnits) {
        hipLaunchKernelGGL(k_counts<true>, P, T, 0, s, a_dev);
    } else {
        hipLaunchKernelGGL(k_unit_plan, dim3(1), dim3(1024), 0, s, a_dev);
        hipLaunchKernelGGL(k_counts<false>, P, T, 0, s, a_dev);
    }
    hipLaunchKernelGGL(k_unit_sizes, dim3(1), dim3(1024), 0, s, a_dev);
    const uint32_t buf_words = huf_buf_words(a.huf_chunk);
    const size_t shmem = (size_t)(kThreads / 64) * buf_words * sizeof(uint32_t);
    hipLaunchKernelGGL(k_write, P, T, shmem, s, a_dev, buf_words);
    return hipGetLastError();
}

hipError_t launch_huf_decode_batch(const DecodeJob* jobs, uint32_t njobs, const uint32_t* wg_job,
                                   uint32_t grid, uint32_t lanes, uint32_t threads, uint32_t cap_chunk, hipStream_t s,
                                   const DescCopy& desc)
{
    if (grid == 0 || njobs == 0) return hipSuccess;
    const dim3 P(grid), T(threads);
    const uint64_t words = desc.bytes / 8;
    const DecodeJob* first = jobs;  // where the tables' launch reads the jobs
    void* src = nullptr;
    if (words) {
        const hipError_t e = hipHostGetDevicePointer(&src, const_cast<void*>(desc.host), 0);
        if (e != hipSuccess) return e;
        const uint64_t at = reinterpret_cast<const uint8_t*>(jobs) - static_cast<const uint8_t*>(desc.dev);
        first = reinterpret_cast<const DecodeJob*>(static_cast<const uint8_t*>(src) + at);
    }
    const dim3 PT(njobs + (words ? blocks_for(words, kTabThreads, 256) : 0));
    const uint64_t* from = static_cast<const uint64_t*>(src);
    uint64_t* to = static_cast<uint64_t*>(desc.dev);
    if (lanes == 1) {
        hipLaunchKernelGGL(k_huf_tables<false>, PT, dim3(kTabThreads), 0, s, first, njobs, from, to, words);
        hipLaunchKernelGGL(k_huf_decode, P, T, 0, s, jobs, wg_job);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_huf_tables<true>, PT, dim3(kTabThreads), 0, s, first, njobs, from, to, words);
    const size_t shmem = split_lds_bytes(threads / lanes, cap_chunk);
    if (threads == kSplitThreadsMax && lanes == 16) {
        hipLaunchKernelGGL((k_huf_decode_split<16, kSplitThreadsMax>), P, T, shmem, s, jobs, wg_job, cap_chunk);
        return hipGetLastError();
    }
    if (threads != kThreads) return hipErrorInvalidValue;
    switch (lanes) {
    case 4: hipLaunchKernelGGL((k_huf_decode_split<4, kThreads>), P, T, shmem, s, jobs, wg_job, cap_chunk); break;
    case 8: hipLaunchKernelGGL((k_huf_decode_split<8, kThreads>), P, T, shmem, s, jobs, wg_job, cap_chunk); break;
    case 16: hipLaunchKernelGGL((k_huf_decode_split<16, kThreads>), P, T, shmem, s, jobs, wg_job, cap_chunk); break;
    case 32: hipLaunchKernelGGL((k_huf_decode_split<32, kThreads>), P, T, shmem, s, jobs, wg_job, cap_chunk); break;
    case 64: hipLaunchKernelGGL((k_huf_decode_split<64, kThreads>), P, T, shmem, s, jobs, wg_job, cap_chunk); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

uint32_t huf_decode_lanes(uint32_t want, uint64_t total_chunks, uint32_t max_chunk)
{
    uint32_t g = want;
    if (g == 0) {
        // measured on 256-symbol chunks: 16 lanes (16 symbols a lane) are
        // fastest from few chunks to 163840 (72 us against 86 with one thread
        // a chunk); at 294912 one thread a chunk is (147 us against 178)
        if (total_chunks * max_chunk >= kHufOneLaneSymbols) return 1;
        g = min(64u, 16 * max(1u, max_chunk / 256));
    }
    if (g == 1) return 1;
    while (g < 64 && (uint64_t)g * kSplitOut < (uint64_t)kThreads * max_chunk) g <<= 1;  // staging fits
    return g;
}

uint32_t huf_decode_threads(uint32_t lanes, uint64_t total_chunks, uint32_t max_chunk)
{
    return lanes == 16 && max_chunk == 256 && total_chunks >= kHufWideChunks ? kSplitThreadsMax : kThreads;
}

hipError_t launch_rle_decode_batch(const RleJob* jobs, const uint32_t* wg_gather, uint32_t n_gather,
                                   const uint32_t* wg_expand, uint32_t n_expand, uint64_t total_runs,
                                   uint32_t* lens, uint32_t* starts, uint32_t* temp, hipStream_t s)
{
    if (n_gather == 0 || n_expand == 0 || total_runs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rle_gather, dim3(n_gather), dim3(kThreads), 0, s, jobs, wg_gather, lens);
    hipError_t err = launch_scan_exclusive(lens, starts, total_runs, temp, s);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_rle_expand, dim3(n_expand), dim3(kThreads), 0, s, jobs, wg_expand, starts);
    return hipGetLastError();
}

}  // namespace mdr
