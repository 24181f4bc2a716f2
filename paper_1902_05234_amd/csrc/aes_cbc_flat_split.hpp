// aes_cbc_flat_split.hpp -- which messages of a set a wave of the block-by-block
// CBC decryption (aes_cbc_dec_flat.hip) takes.  Plain arithmetic, shared by the
// kernel, its launcher and a host test.
#pragma once
#include <algorithm>
#include <cstdint>

namespace aesgpu {

struct FlatSplit {
    uint64_t groups;     // of messages, one record per lane
    uint32_t per_group;  // messages of a group, at most 64
    uint32_t slices;     // waves that share a group, each taking every slices-th step of it
    uint32_t run_log2;   // a group's messages come in runs of 2^run_log2 consecutive ones
    uint32_t skew;       // groups by which each band of runs is turned against the one before
    uint32_t inverse;    // 2^32 / groups, rounded up, for up to 2^12 groups
};

// Message of lane `lane` (below per_group) of group g; past the end of the set
// for a lane without one.  The set is cut into bands of one run per group, and
// a group takes a run of every band: lengths that grow along the set, or a
// stretch of long messages, then fall on all groups alike.  The runs of a group
// lie groups + skew runs apart, a number without small factors, so lengths that
// repeat with a small period do too.
constexpr uint64_t flat_message(const FlatSplit& s, uint64_t g, uint32_t lane)
{
    const uint32_t band = lane >> s.run_log2, first = band << s.run_log2;
    const uint32_t rest = s.per_group - first, run = rest >> s.run_log2 ? 1u << s.run_log2 : rest;
    if (band == 0)
        return g * run + lane;
    // modulo groups by multiplication (exact: both numbers are below 2^13), or
    // by one subtraction where the bands together turn by less than the groups
    const uint32_t groups = static_cast<uint32_t>(s.groups), at = static_cast<uint32_t>(g) + band * s.skew;
    const uint32_t wraps = s.inverse != 0 ? static_cast<uint32_t>((uint64_t{at} * s.inverse) >> 32) : at >= groups;
    return s.groups * first + uint64_t{at - wraps * groups} * run + (lane - first);
}

// nmsgs > 0 messages over an input arena of in_blocks blocks, on cus CUs of 16
// resident waves; one_arena: no message may be shared by waves.  The lengths
// are on the device, so the arena's blocks per message stand in for their mean.
inline FlatSplit flat_split(uint64_t nmsgs, uint64_t in_blocks, bool one_arena, int cus)
{
    const uint64_t resident = 16u * (uint64_t)cus, mean = std::max<uint64_t>(1, in_blocks / nmsgs);
    uint64_t per_group = 0, slices = 1;
    if (!one_arena) {
        // Groups as near to 64 messages as fill the device, each shared by as
        // many waves as that leaves, down to one step each: the waves of a
        // group have equally many steps, whatever its messages' lengths.
        slices = std::max<uint64_t>(1, 64u * resident / nmsgs);
        per_group = slices > 1 ? (nmsgs * slices + resident - 1) / resident : 0;
    }
    if (slices == 1) {
        // A wave per group: as many messages as give every resident wave one
        // group, in as many rounds as groups of 64 need, and at least a step.
        const uint64_t rounds = (nmsgs + 64u * resident - 1) / (64u * resident);
        per_group = std::max((nmsgs + resident * rounds - 1) / (resident * rounds), (64u + mean - 1) / mean);
    }
    per_group = std::min<uint64_t>({per_group, 64u, nmsgs});
    const uint64_t groups = (nmsgs + per_group - 1) / per_group;
    if (slices > 1)
        slices = std::min<uint64_t>(std::max<uint64_t>(1, mean * per_group / 64u),
                                    std::max<uint64_t>(1, resident / groups));
    // Runs of about a step's 64 blocks: shorter ones scatter a step's memory
    // accesses, longer ones leave fewer bands.
    uint32_t run_log2 = 0;
    while (run_log2 < 6u && (mean << run_log2) < 64u)
        ++run_log2;
    if (nmsgs >> 32 || groups == 1)  // more than the kernel keeps message numbers for; nothing to deal
        run_log2 = 6;
    uint32_t skew = 1;
    while ((groups + skew) % 2 == 0 || (groups + skew) % 3 == 0 || (groups + skew) % 5 == 0 || (groups + skew) % 7 == 0)
        ++skew;  // 10 at most: such numbers lie no further apart
    return FlatSplit{groups, (uint32_t)per_group, (uint32_t)slices, run_log2, skew,
                     groups > 1 && groups <= 4096u ? (uint32_t)(((uint64_t)1 << 32) / groups + 1) : 0u};
}

}  // namespace aesgpu
