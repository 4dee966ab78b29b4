// Block order of a launch that holds prefill-shaped tiles and block decodes
// (attn_mixed_kernel): a first round of prefill blocks, as many decodes, then
// groups of kMixedGroup blocks of either kind in the ratio of what is left.
// Host and device code, so that the blocks of any mix can be listed on a CPU.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define SANGAM_HD __host__ __device__
#else
#define SANGAM_HD
#endif

namespace sangam {

constexpr int kMixedGroup = 8;  // blocks of one kind in a row: one per XCD

struct MixedOrder {
    int32_t n_prefill;      // blocks of prefill tiles
    int32_t n_decode;
    int32_t first_prefill;  // of the first round
    int32_t first_decode;
    uint64_t share;         // of prefills in the later groups, in 1 / 2^32, rounded up
};

// A block's tile, or index -1 (the last group of a kind may not be full).
struct MixedBlock {
    int32_t index;
    bool decode;
};

// Fills in the order and returns its number of blocks, fewer than
// 2 kMixedGroup of which find no tile. With G later groups, P of them of
// prefills, the share is ceil(P 2^32 / G): as G < 2^32, floor(G share / 2^32)
// is P exactly, so the G groups hold every block of both kinds.
inline int64_t mixed_order(MixedOrder* m, int64_t n_prefill, int64_t n_decode, int64_t round) {
    m->n_prefill = int32_t(n_prefill);
    m->n_decode = int32_t(n_decode);
    m->first_prefill = int32_t(n_prefill < round ? n_prefill : round);
    m->first_decode = int32_t(n_decode < round ? n_decode : round);
    const uint64_t p = uint64_t(n_prefill - m->first_prefill + kMixedGroup - 1) / kMixedGroup;
    const uint64_t groups = p + uint64_t(n_decode - m->first_decode + kMixedGroup - 1) / kMixedGroup;
    m->share = groups ? ((p << 32) + groups - 1) / groups : 0;
    return int64_t(m->first_prefill) + m->first_decode + int64_t(kMixedGroup * groups);
}

SANGAM_HD inline MixedBlock mixed_block(const MixedOrder& m, uint32_t block) {
    const uint32_t head = uint32_t(m.first_prefill) + uint32_t(m.first_decode);
    uint32_t index = block;
    bool decode = block >= uint32_t(m.first_prefill);
    if (block >= head) {
        const uint32_t g = (block - head) / kMixedGroup;
        const uint32_t before = uint32_t((g * m.share) >> 32);  // groups of prefills
        decode = uint32_t(((g + 1) * m.share) >> 32) == before;
        index = (decode ? uint32_t(m.first_decode) : uint32_t(m.first_prefill)) +
                (decode ? g - before : before) * kMixedGroup + (block - head) % kMixedGroup;
    } else if (decode) {
        index -= uint32_t(m.first_prefill);
    }
    const int32_t n = decode ? m.n_decode : m.n_prefill;
    return {index < uint32_t(n) ? int32_t(index) : -1, decode};
}

}  // namespace sangam
