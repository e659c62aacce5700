// Container format (serialization, Sec. 5.1) and CRC-32.
//
// Little-endian throughout.
//   header (56 B): u32 magic 0x3152444D ("MDR1") | u8 version=1 | u8 dtype | u8 B | u8 m
//                  | u32 nlevels | u32 t_cr_milli | u64 t_s | u32 huf_chunk | u32 huf_lmax
//                  | i32 force_method | u32 0 | u64 blob bytes | u32 crc32(bytes 0..47) | u32 0
//   per level:     u64 n | i32 e | u32 nstreams=1+B | f64 min | f64 max | f64 max|x|
//                  | f64 E[B+1] | nstreams x {u8 method, u8[3] 0, u32 crc32, u64 bytes}
//                  | u32 crc32(record so far) | u32 0
//                  | payloads in table order, each zero padded to a multiple of 8 bytes
#include <cmath>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "api_internal.hpp"

namespace mdr {

// ---- CRC-32 (reflected polynomial 0xEDB88320), eight table lookups per 8 bytes
namespace {
struct CrcTables {
    uint32_t t[8][256];
    CrcTables()
    {
        for (uint32_t i = 0; i < 256; ++i) {
            uint32_t c = i;
            for (int k = 0; k < 8; ++k) c = (c & 1u) ? (c >> 1) ^ 0xEDB88320u : (c >> 1);
            t[0][i] = c;
        }
        for (int s = 1; s < 8; ++s)
            for (uint32_t i = 0; i < 256; ++i) t[s][i] = (t[s - 1][i] >> 8) ^ t[0][t[s - 1][i] & 0xFFu];
    }
};
const CrcTables& crc_tables()
{
    static const CrcTables tables;
    return tables;
}
}  // namespace

uint32_t crc32(const uint8_t* p, uint64_t n)
{
    const auto& T = crc_tables().t;
    uint32_t c = 0xFFFFFFFFu;
    while (n >= 8) {
        uint32_t a, b;
        std::memcpy(&a, p, 4);
        std::memcpy(&b, p + 4, 4);
        a ^= c;
        c = T[7][a & 0xFF] ^ T[6][(a >> 8) & 0xFF] ^ T[5][(a >> 16) & 0xFF] ^ T[4][a >> 24] ^
            T[3][b & 0xFF] ^ T[2][(b >> 8) & 0xFF] ^ T[1][(b >> 16) & 0xFF] ^ T[0][b >> 24];
        p += 8;
        n -= 8;
    }
    while (n--) c = (c >> 8) ^ T[0][(c ^ *p++) & 0xFFu];
    return c ^ 0xFFFFFFFFu;
}

namespace {
constexpr uint32_t kMagic = 0x3152444Du;
constexpr uint64_t kHeader = 56;

uint64_t pad8(uint64_t v) { return (v + 7) & ~(uint64_t)7; }

template <typename T>
void put(uint8_t* p, T v)
{
    std::memcpy(p, &v, sizeof(T));
}
template <typename T>
T get(const uint8_t* p)
{
    T v;
    std::memcpy(&v, p, sizeof(T));
    return v;
}

uint64_t record_bytes(uint32_t B) { return 16 + 24 + 8ull * (B + 1) + 16ull * (1 + B) + 8; }

uint64_t blob_size(const mdr_refactored* r)
{
    uint64_t t = kHeader;
    for (const LevelRec& L : r->levels) {
        t += record_bytes(r->B);
        for (uint32_t s = 0; s <= r->B; ++s)
            if (L.units[s].method != MDR_PLACEHOLDER) t += pad8(L.units[s].bytes);
    }
    return t;
}

mdr_status corrupt(const std::string& what) { return fail(MDR_ERR_CORRUPT_STREAM, what); }

uint64_t S_of(const mdr_refactored* r, const LevelRec& L, uint32_t slot)
{
    uint32_t r0, r1;
    slot_rows(slot, r->B, r->m, r0, r1);
    return 4ull * (r1 - r0) * L.nbd;
}

// structural checks of one payload (host bytes) so that decoding stays in bounds
mdr_status check_payload(const mdr_refactored* r, const LevelRec& L, uint32_t slot,
                         const uint8_t* p, uint64_t bytes, UnitRec& u)
{
    const uint64_t S = S_of(r, L, slot);
    u.S = S;
    if (u.method == MDR_DC) {
        if (bytes != S) return corrupt("direct-copy payload size does not match its planes");
        return MDR_OK;
    }
    if (u.method == MDR_RLE) {
        if (bytes < 8) return corrupt("RLE payload too short");
        uint64_t nr = get<uint32_t>(p);
        if (get<uint32_t>(p + 4) != 4 * r->G) return corrupt("RLE word width mismatch");
        if (bytes != 8 + nr * (4ull * r->G + 4)) return corrupt("RLE payload size mismatch");
        const uint64_t nwords = S / 4 / r->G;
        uint64_t total = 0;
        const uint8_t* lens = p + 8 + 4ull * r->G * nr;
        for (uint64_t i = 0; i < nr; ++i) {
            uint32_t len = get<uint32_t>(lens + 4 * i);
            if (len == 0) return corrupt("RLE run of length 0");
            total += len;
        }
        if (total != nwords) return corrupt("RLE runs do not cover the group");
        u.nruns = nr;
        return MDR_OK;
    }
    if (u.method == MDR_HUF) {
        const uint32_t chunk = r->prm.huf_chunk;
        const uint64_t nc = (S + chunk - 1) / chunk;
        if (bytes < 8 + 256 + 4 * (nc + 1)) return corrupt("Huffman payload too short");
        if (get<uint64_t>(p) != S) return corrupt("Huffman symbol count mismatch");
        uint32_t maxlen = 0;
        for (int s = 0; s < 256; ++s) {
            uint32_t l = p[8 + s];
            if (l > r->prm.huf_lmax) return corrupt("Huffman code longer than the limit");
            maxlen = l > maxlen ? l : maxlen;
        }
        const uint8_t* off = p + 8 + 256;
        const uint64_t words = (bytes - (8 + 256 + 4 * (nc + 1))) / 4;
        if (8 + 256 + 4 * (nc + 1) + 4 * words != bytes) return corrupt("Huffman payload not word aligned");
        uint32_t prev = 0;
        for (uint64_t c = 0; c <= nc; ++c) {
            uint32_t o = get<uint32_t>(off + 4 * c);
            if (o < prev || o > words) return corrupt("Huffman chunk offsets out of range");
            prev = o;
        }
        if (get<uint32_t>(off) != 0 || prev != words) return corrupt("Huffman chunk offsets inconsistent");
        u.nchunks = (uint32_t)nc;
        u.maxlen = maxlen;
        return MDR_OK;
    }
    return corrupt("unknown lossless method");
}

// One payload between its place in device memory and its place in the blob.
struct Span {
    uint8_t* dev;
    uint64_t at;     // offset in the blob
    uint64_t bytes;  // a multiple of 4, > 0
    uint32_t crc;    // filled by move_payloads
};

// Payloads below this go through one staging buffer, laid out as in the blob:
// a copy per run of them instead of one each (about 13 us whatever its size).
constexpr uint64_t kStagedPayload = 256u << 10;

// Every payload from the device into the blob (to_host) or the other way, and
// its CRC-32 computed on the device: one pass over the bytes there, which also
// moves the small ones between their places and the staging buffer.
// hipErrorOutOfMemory (nothing done) when the staging does not fit.
hipError_t move_payloads(mdr_context* ctx, std::vector<Span>& sp, uint8_t* blob, bool to_host)
{
    if (sp.empty()) return hipSuccess;
    struct Run {
        uint64_t at, bytes, stage;  // of the blob, and where it starts in the staging buffer
    };
    std::vector<Run> runs;
    std::vector<CrcJob> jobs(sp.size());
    uint64_t staged = 0, blocks = 0;
    bool open = false;
    for (size_t i = 0; i < sp.size(); ++i) {
        CrcJob& j = jobs[i];
        j = {reinterpret_cast<const uint32_t*>(sp[i].dev), nullptr, sp[i].bytes / 4, (uint32_t)blocks, 0};
        blocks += (j.words + kCrcBlockWords - 1) / kCrcBlockWords;
        if (sp[i].bytes >= kStagedPayload) {
            open = false;
            continue;
        }
        // a level's record lies between two levels' payloads: a run goes on over it
        if (!open) runs.push_back({sp[i].at, 0, staged});
        open = true;
        runs.back().bytes = sp[i].at + sp[i].bytes - runs.back().at;
        staged = align256(runs.back().stage + runs.back().bytes);
    }
    PoolBuf stage, meta;
    hipError_t e = stage.alloc(ctx->pool, staged);
    if (e != hipSuccess) return e;
    const uint64_t o_out = align256(sizeof(CrcJob) * jobs.size());
    e = meta.alloc(ctx->pool, o_out + 4 * blocks);
    if (e != hipSuccess) return e;
    uint8_t* st = static_cast<uint8_t*>(stage.p);
    {
        size_t r = 0;
        for (size_t i = 0; i < sp.size(); ++i) {
            if (sp[i].bytes >= kStagedPayload) continue;
            while (sp[i].at >= runs[r].at + runs[r].bytes) ++r;
            uint32_t* p = reinterpret_cast<uint32_t*>(st + runs[r].stage + (sp[i].at - runs[r].at));
            if (to_host) {
                jobs[i].dst = p;
            } else {
                jobs[i].dst = const_cast<uint32_t*>(jobs[i].src);
                jobs[i].src = p;
            }
        }
    }
    auto big = [&]() -> hipError_t {
        for (const Span& s : sp) {
            if (s.bytes < kStagedPayload) continue;
            const hipError_t ce = to_host ? hipMemcpy(blob + s.at, s.dev, s.bytes, hipMemcpyDeviceToHost)
                                          : hipMemcpy(s.dev, blob + s.at, s.bytes, hipMemcpyHostToDevice);
            if (ce != hipSuccess) return ce;
        }
        return hipSuccess;
    };
    auto small = [&]() -> hipError_t {
        for (const Run& r : runs) {
            const hipError_t ce = to_host ? hipMemcpy(blob + r.at, st + r.stage, r.bytes, hipMemcpyDeviceToHost)
                                          : hipMemcpy(st + r.stage, blob + r.at, r.bytes, hipMemcpyHostToDevice);
            if (ce != hipSuccess) return ce;
        }
        return hipSuccess;
    };
    e = hipMemcpy(meta.p, jobs.data(), sizeof(CrcJob) * jobs.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !to_host) e = big();
    if (e == hipSuccess && !to_host) e = small();
    uint32_t* out = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(meta.p) + o_out);
    (void)hipGetLastError();  // only this launch is checked
    if (e == hipSuccess)
        e = launch_crc_blocks(static_cast<const CrcJob*>(meta.p), (uint32_t)jobs.size(), (uint32_t)blocks, out, nullptr);
    if (e == hipSuccess && to_host) e = big();
    if (e == hipSuccess && to_host) e = small();
    std::vector<uint32_t> rem(blocks);
    if (e == hipSuccess) e = hipMemcpy(rem.data(), out, 4 * blocks, hipMemcpyDeviceToHost);
    // the buffers go back to the pool: nothing may still use them
    const hipError_t es = hipStreamSynchronize(nullptr);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return e == hipErrorOutOfMemory ? hipErrorUnknown : e;
    for (size_t i = 0; i < sp.size(); ++i) {
        const uint64_t b1 = i + 1 < sp.size() ? jobs[i + 1].block0 : blocks;
        sp[i].crc = crc_join(rem.data() + jobs[i].block0, (uint32_t)(b1 - jobs[i].block0), jobs[i].words);
    }
    return hipSuccess;
}
}  // namespace

}  // namespace mdr

using namespace mdr;

extern "C" {

mdr_status mdr_serialize(const mdr_refactored* r, void* host, uint64_t cap, uint64_t* used)
{
    set_error("");
    if (!r || !used) return fail(MDR_ERR_INVALID_ARG, "NULL argument");
    const uint64_t total = blob_size(r);
    *used = total;
    if (cap == 0) return MDR_OK;
    if (!host) return fail(MDR_ERR_INVALID_ARG, "host is NULL");
    if (cap < total) return fail(MDR_ERR_INVALID_ARG, "cap is smaller than the serialized size");
    hipError_t he = hipSetDevice(r->ctx->device);
    if (he != hipSuccess) return hip_fail(he, "hipSetDevice");
    he = hipDeviceSynchronize();
    if (he != hipSuccess) return hip_fail(he, "hipDeviceSynchronize");
    uint8_t* out = static_cast<uint8_t*>(host);
    std::memset(out, 0, kHeader);
    const uint32_t B = r->B;
    put<uint32_t>(out, kMagic);
    out[4] = 1;
    out[5] = (uint8_t)r->dtype;
    out[6] = (uint8_t)B;
    out[7] = (uint8_t)r->m;
    put<uint32_t>(out + 8, (uint32_t)r->levels.size());
    put<uint32_t>(out + 12, r->prm.t_cr_milli);
    put<uint64_t>(out + 16, r->prm.t_s_bytes);
    put<uint32_t>(out + 24, r->prm.huf_chunk);
    put<uint32_t>(out + 28, r->prm.huf_lmax);
    put<int32_t>(out + 32, r->prm.force_method);
    put<uint64_t>(out + 40, total);
    put<uint32_t>(out + 48, crc32(out, 48));
    // payloads first (their CRCs go into the tables); they start behind each
    // level's record, in slot order
    std::vector<Span> sp;
    uint64_t pos = kHeader;
    for (const LevelRec& L : r->levels) {
        pos += record_bytes(B);
        for (uint32_t s = 0; s <= B; ++s) {
            const UnitRec& u = L.units[s];
            if (u.method == MDR_PLACEHOLDER) continue;
            if (u.bytes) sp.push_back({u.dev, pos, u.bytes, 0});
            pos += pad8(u.bytes);
        }
    }
    he = move_payloads(r->ctx, sp, out, true);
    if (he == hipErrorOutOfMemory) {  // no room for the staging: one by one, CRCs on the host
        (void)hipGetLastError();
        for (Span& x : sp) {
            he = hipMemcpy(out + x.at, x.dev, x.bytes, hipMemcpyDeviceToHost);
            if (he != hipSuccess) break;
            x.crc = crc32(out + x.at, x.bytes);
        }
    }
    if (he != hipSuccess) return hip_fail(he, "hipMemcpy(payload)");
    pos = kHeader;
    size_t next = 0;
    for (const LevelRec& L : r->levels) {
        const uint64_t rec = pos;
        std::memset(out + rec, 0, record_bytes(B));
        put<uint64_t>(out + pos, L.n);
        put<int32_t>(out + pos + 8, L.e);
        put<uint32_t>(out + pos + 12, 1 + B);
        put<double>(out + pos + 16, L.vmin);
        put<double>(out + pos + 24, L.vmax);
        put<double>(out + pos + 32, L.vmaxabs);
        pos += 40;
        for (uint32_t k = 0; k <= B; ++k, pos += 8) put<double>(out + pos, L.E[k]);
        const uint64_t table = pos;
        pos += 16ull * (1 + B) + 8;
        for (uint32_t s = 0; s <= B; ++s) {
            const UnitRec& u = L.units[s];
            uint8_t* ent = out + table + 16ull * s;
            ent[0] = (uint8_t)u.method;
            const uint64_t nb = u.method == MDR_PLACEHOLDER ? 0 : u.bytes;
            put<uint64_t>(ent + 8, nb);
            put<uint32_t>(ent + 4, nb ? sp[next++].crc : 0);
            if (u.method == MDR_PLACEHOLDER) continue;
            if (pad8(nb) != nb) std::memset(out + pos + nb, 0, pad8(nb) - nb);
            pos += pad8(nb);
        }
        const uint64_t rec_end = table + 16ull * (1 + B);
        put<uint32_t>(out + rec_end, crc32(out + rec, rec_end - rec));
    }
    if (pos != total) return fail(MDR_ERR_HIP, "internal: serialized size mismatch");
    return MDR_OK;
}

mdr_status mdr_deserialize(mdr_context* ctx, const void* host, uint64_t bytes, mdr_refactored** out)
{
    set_error("");
    if (!out) return fail(MDR_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!ctx || !host) return fail(MDR_ERR_INVALID_ARG, "NULL argument");
    const uint8_t* in = static_cast<const uint8_t*>(host);
    if (bytes < kHeader) return corrupt("blob shorter than its header");
    if (get<uint32_t>(in) != kMagic) return corrupt("bad magic");
    if (in[4] != 1) return corrupt("unknown container version");
    if (get<uint32_t>(in + 48) != crc32(in, 48)) return corrupt("header CRC mismatch");
    if (get<uint64_t>(in + 40) != bytes) return corrupt("blob size mismatch");
    auto R = std::make_unique<mdr_refactored>();
    R->ctx = ctx;
    if (in[5] > 1) return corrupt("bad dtype");
    R->dtype = (mdr_dtype)in[5];
    R->B = in[6];
    R->m = in[7];
    R->G = R->dtype == MDR_F64 ? 2 : 1;
    const uint32_t W = 32 * R->G, B = R->B, m = R->m;
    if (B < 1 || B > W || m < 1 || m > B) return corrupt("bad plane count or group size");
    const uint32_t nlevels = get<uint32_t>(in + 8);
    R->prm.group_planes = m;
    R->prm.t_cr_milli = get<uint32_t>(in + 12);
    R->prm.t_s_bytes = get<uint64_t>(in + 16);
    R->prm.huf_chunk = get<uint32_t>(in + 24);
    R->prm.huf_lmax = get<uint32_t>(in + 28);
    R->prm.force_method = get<int32_t>(in + 32);
    if (R->prm.huf_chunk < 256 || R->prm.huf_chunk > 4096 || (R->prm.huf_chunk & (R->prm.huf_chunk - 1)) ||
        R->prm.huf_lmax < 8 || R->prm.huf_lmax > (uint32_t)kLutBitsMax)
        return fail(MDR_ERR_UNSUPPORTED, "Huffman parameters not supported by this build");
    if (nlevels == 0 || nlevels > (bytes - kHeader) / record_bytes(B)) return corrupt("bad level count");
    R->levels.resize(nlevels);

    // ---- parse and validate everything but the payloads' CRCs on the host first
    struct Src {
        uint32_t level, slot;
        const uint8_t* p;
        uint32_t crc;  // as recorded
    };
    std::vector<Src> srcs;
    // an error past some payloads: the first of them whose CRC is wrong comes before it
    auto after_crcs = [&](mdr_status st) {
        const std::string what = mdr_last_error();
        for (const Src& sr : srcs)
            if (crc32(sr.p, R->levels[sr.level].units[sr.slot].bytes) != sr.crc) return corrupt("payload CRC mismatch");
        return fail(st, what);
    };
    uint64_t pos = kHeader, rows_bytes = 0, pay_bytes = 0;
    for (uint32_t l = 0; l < nlevels; ++l) {
        LevelRec& L = R->levels[l];
        if (bytes - pos < record_bytes(B)) return after_crcs(corrupt("truncated level record"));
        const uint64_t rec = pos;
        L.n = get<uint64_t>(in + pos);
        L.e = get<int32_t>(in + pos + 8);
        if (get<uint32_t>(in + pos + 12) != 1 + B) return after_crcs(corrupt("stream count mismatch"));
        if (L.n > 0xFFFFFFFFull) return after_crcs(corrupt("level too large"));
        L.nbd = R->G == 2 ? (uint32_t)(2 * ((L.n + 63) / 64)) : (uint32_t)((L.n + 31) / 32);
        L.vmin = get<double>(in + pos + 16);
        L.vmax = get<double>(in + pos + 24);
        L.vmaxabs = get<double>(in + pos + 32);
        pos += 40;
        L.E.resize(B + 1);
        for (uint32_t k = 0; k <= B; ++k, pos += 8) {
            L.E[k] = get<double>(in + pos);
            if (!(L.E[k] >= 0.0) || std::isinf(L.E[k])) return after_crcs(corrupt("bad error table"));
        }
        const uint64_t table = pos;
        const uint64_t rec_end = table + 16ull * (1 + B);
        if (get<uint32_t>(in + rec_end) != crc32(in + rec, rec_end - rec)) return after_crcs(corrupt("level record CRC mismatch"));
        pos = rec_end + 8;
        L.units.init(B, m);
        for (uint32_t s = 0; s <= B; ++s) {
            const uint8_t* ent = in + table + 16ull * s;
            const uint64_t nb = get<uint64_t>(ent + 8);
            const bool leader = s == 0 || (s - 1) % m == 0;
            if (!leader) {
                if (ent[0] != MDR_PLACEHOLDER || nb != 0) return after_crcs(corrupt("bad placeholder slot"));
                continue;
            }
            UnitRec& u = L.units.unit(s == 0 ? 0 : 1 + (s - 1) / m);
            u.method = ent[0];
            if (u.method > MDR_HUF) return after_crcs(corrupt("bad method in a leading slot"));
            if (nb > bytes - pos) return after_crcs(corrupt("payload runs past the end of the blob"));
            u.bytes = nb;
            srcs.push_back({l, s, in + pos, get<uint32_t>(ent + 4)});
            mdr_status st = check_payload(R.get(), L, s, in + pos, nb, u);
            if (st) return after_crcs(st);
            if (nb == 0 && srcs.back().crc != 0) return after_crcs(corrupt("payload CRC mismatch"));
            if (u.method != MDR_DC) pay_bytes += (nb + 255) & ~255ull;
            pos += pad8(nb);
            if (pos > bytes) return after_crcs(corrupt("payload padding runs past the end of the blob"));
        }
        rows_bytes += (4ull * (B + 1) * L.nbd + 255) & ~255ull;
    }
    if (pos != bytes) return after_crcs(corrupt("trailing bytes after the last level"));

    // ---- upload: direct-copy payloads become plane rows, others go to the payload arena
    hipError_t he = hipSetDevice(ctx->device);
    if (he != hipSuccess) return after_crcs(hip_fail(he, "hipSetDevice"));
    R->rows_arena = std::make_shared<PoolBuf>();
    R->payload_arena = std::make_shared<PoolBuf>();
    he = R->rows_arena->alloc(ctx->pool, rows_bytes);
    if (he != hipSuccess) return after_crcs(hip_fail(he, "hipMalloc(planes)"));
    he = R->payload_arena->alloc(ctx->pool, pay_bytes + 256);  // padded for the Huffman decoder's block reads
    if (he != hipSuccess) return after_crcs(hip_fail(he, "hipMalloc(payloads)"));
    uint8_t* rb = static_cast<uint8_t*>(R->rows_arena->p);
    for (uint32_t l = 0; l < nlevels; ++l) {
        R->levels[l].rows = reinterpret_cast<uint32_t*>(rb);
        rb += (4ull * (B + 1) * R->levels[l].nbd + 255) & ~255ull;
    }
    uint8_t* pb = static_cast<uint8_t*>(R->payload_arena->p);
    std::vector<Span> sp;
    for (const Src& sr : srcs) {
        LevelRec& L = R->levels[sr.level];
        UnitRec& u = L.units.unit(sr.slot == 0 ? 0 : 1 + (sr.slot - 1) / m);
        if (u.method == MDR_DC) {
            uint32_t r0, r1;
            slot_rows(sr.slot, B, m, r0, r1);
            u.dev = reinterpret_cast<uint8_t*>(L.rows + (uint64_t)r0 * L.nbd);
        } else {
            u.dev = pb;
            pb += (u.bytes + 255) & ~255ull;
        }
        if (u.bytes) sp.push_back({u.dev, (uint64_t)(sr.p - in), u.bytes, sr.crc});
    }
    std::vector<uint32_t> want;
    for (const Span& x : sp) want.push_back(x.crc);
    he = move_payloads(ctx, sp, const_cast<uint8_t*>(in), false);
    if (he == hipErrorOutOfMemory) {  // no room for the staging: CRCs on the host, one by one
        (void)hipGetLastError();
        for (Span& x : sp) {
            x.crc = crc32(in + x.at, x.bytes);
            he = hipMemcpy(x.dev, in + x.at, x.bytes, hipMemcpyHostToDevice);
            if (he != hipSuccess) break;
        }
    }
    if (he != hipSuccess) return after_crcs(hip_fail(he, "hipMemcpy(payload)"));
    for (size_t i = 0; i < sp.size(); ++i)
        if (sp[i].crc != want[i]) return corrupt("payload CRC mismatch");
    *out = R.release();
    return MDR_OK;
}

}  // extern "C"
