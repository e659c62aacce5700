// Launch rules of the refactor pass's encoder (host only).
#pragma once
#include <cstdint>

namespace mdr {

// Passes of at most this many values take the small passes' encoder (eight
// lanes a block, tiles of 32 blocks).  Its advantage is latency (2^18 values: 9
// against 26 us in f32, 16 against 41 in f64; 2^21 f32 values 19 against 28,
// 2^20 f64 ones 28 against 42), its cost instructions a value (2^22: 33 against
// 35, a unit per plane 46 against 46; f64 78 against 57).
constexpr uint64_t small_pass_values(bool f64) { return f64 ? 1u << 20 : 1u << 21; }
// and aims for this many workgroups at most: each ends by adding its
// histograms into the level's, a KiB a unit (2^21 f32 values in 9 units: 22 us
// at 1024, 25 at 512; in 33 units: 43 and 33; 2^20 f64 in 17: 36 and 30)
constexpr uint32_t small_target_wg(uint32_t nunits) { return nunits <= 12 ? 1024 : 512; }

// A pass of up to this many tiles in the register fast paths aims for one round
// of workgroups, as many as are resident at once (four a CU in f64): a
// workgroup's first tile and its end cost more than the others, and a second
// round of as few tiles is not full (2^25 f64 values, 4096 tiles: 233 us with 1024
// workgroups, 251 with 2048; 12288 tiles: 535 and 562; 2^24 f32 values: 66 and 71,
// 4096 tiles: 106 and 110).  Past it more workgroups spread the load better
// (2^28 f64 values: 1330 us with 1024, 1288 to 1310 with 2048 and 2185; 6144 f32
// tiles: 154 and 151).
constexpr uint32_t kOneRoundWg = 1024;
constexpr uint64_t one_round_tiles(bool f64) { return f64 ? 12288 : 4096; }

// The context's default target, which stands for the rules above; a target
// asked for by mdr_context_set_launch or a tuning table is taken as it is.
constexpr uint32_t kEncTargetDefault = 2304;

// Workgroups the encoder's tiles are split over.  small: the small passes'
// encoder, tiles of 32 blocks, else of 256.
constexpr uint32_t encode_target_wg(uint32_t asked, bool f64, uint32_t B, uint32_t m, uint32_t nunits, bool small,
                                    uint64_t tiles)
{
    if (asked != kEncTargetDefault) return asked;
    if (small) return small_target_wg(nunits);
    const bool fast = m == 4 && B == (f64 ? 64u : 32u);
    return fast && tiles <= one_round_tiles(f64) ? kOneRoundWg : kEncTargetDefault;
}

}  // namespace mdr
