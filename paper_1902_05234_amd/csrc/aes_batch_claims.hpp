// aes_batch_claims.hpp -- how the batched launch (aes_batch.hip) hands out the
// claims of a work list.  Plain arithmetic, shared by the kernel and a host
// test that plays lists through it.
#pragma once
#include <cstdint>

namespace aesgpu {

// Most claims worth taking with one update of a list's counter, for n claims
// over `blocks` blocks in all: as many as hold the 1200 blocks that the device
// walks (at 1330 GB/s) in the 14 ns of an update.  Longer items cost nothing
// one by one, and several in one wave's hands do: 20,000 messages of up to 8
// MiB that are an item each 20.7 ms one by one, 25.5 in runs.  Lists near 2^32
// claims go one by one: the counter passes the end of a list by at most the
// last claims of every wave, and must not wrap.
constexpr uint32_t claims_worth(uint64_t blocks, uint64_t n)
{
    if (n >> 31)
        return 1u;
    const uint64_t mean = n != 0 ? blocks / n : 0;
    return 1u + static_cast<uint32_t>(1200u / (mean != 0 ? mean : 1u));
}

// The claims of one list, an item each, of which the first `dealt` go to the
// `waves` waves that start on the list, in turn, and the rest to whichever
// wave asks, through the list's counter.  An update of the counter takes
// about 14 ns in which no other is served: 1000 items of one unit on 1008
// waves took 43 us, the time of their 3000 updates.  So a list that one claim
// per wave covers is dealt whole.  Of a longer one every wave gets one claim,
// as it would at once from the counter, and more only up to five eighths of
// its share, 8, and what is worth an update: dealt claims stay with their
// wave, and dealt waves drift apart over the arenas.  (us; one by one, the
// five eighths rounded up and of any length, and so: 20,000 messages of up to
// 8 MiB in items of 2048 blocks 9685, 10181, 9556; of up to 4 KiB 327, 165,
// 146; 10,000 items of 4 blocks, one in a hundred of 20,000, 612, 787, 568;
// 8192 items of 2048 blocks beside as many of one block 371, 349, 309.)
struct Claims {
    uint32_t n, dealt;
};

constexpr Claims claims_of(uint32_t n, uint32_t waves, uint32_t worth)
{
    if (n <= waves || waves == 0)
        return Claims{n, waves == 0 ? 0u : n};
    const uint32_t share = n / waves, part = share < 13u ? share * 5u / 8u : 8u;
    const uint32_t turns = part < worth ? part : worth;
    return Claims{n, (turns != 0 ? turns : 1u) * waves};
}

// Waves that a list's claims are to last for: those that start on it, or half
// of the launch where these are fewer, because the others come over once
// their own list is dry.  (With the starting waves of a wave's own list for
// both, 10 encryption and 50,000 decryption items of 256 blocks left 17,360
// claims to sixteen helping waves in runs of 68: 679 us one by one, 945 so, 233
// now.)
constexpr uint32_t claim_waves(uint32_t own, uint32_t all) { return own > all / 2u ? own : (all + 1u) / 2u; }

// What a launch hands its kernel for one list: the claims, and the claims that
// each of claim_waves is to have, as a factor over 2^32.
struct ListClaims {
    uint32_t n, dealt, per_wave;
};

constexpr ListClaims list_claims(uint32_t n, uint32_t own, uint32_t all, uint32_t worth)
{
    const Claims c = claims_of(n, own, worth);
    return ListClaims{c.n, c.dealt, UINT32_MAX / claim_waves(own, all)};
}

// Claims taken with one update of the counter when `left` are left, per_wave as
// above: a sixteenth of a wave's share and one, and twice as many as the last
// time, up to two fifths of the share, where none of those was over 512 blocks
// (100,000 messages of up to 1 KiB 1238 us one by one, 300 so; of up to 8 KiB
// 1247 -> 330; half the share: 282 and 310, but its last runs end unevenly).
constexpr uint32_t claims_at_once(uint32_t left, uint32_t per_wave, uint32_t taken, uint32_t longest, uint32_t worth)
{
    const uint32_t share = static_cast<uint32_t>((uint64_t{left} * per_wave) >> 32);
    const uint32_t few = 1u + share / 16u, most = 1u + (share + 1u) * 2u / 5u;
    const uint32_t more = longest > 512u ? few : 2u * taken < most ? 2u * taken : most;
    const uint32_t n = few > more ? few : more;
    return n < worth ? n : worth;
}

// Launch shape of lists that one claim per resident wave covers: every item in
// as many parts (up to 32) as leave every wave one claim at most, so that a
// short list spreads over all CUs and nothing goes through the claim counters.
// max_grid: workgroups that the caller allows, resident: that the device holds
// at once; a list that does not fit both gets grid 0.  The parts of all items
// are no more than the resident waves.
struct ShortList {
    uint32_t parts_log2, grid, enc_groups;
};

constexpr ShortList short_list(uint64_t n_enc, uint64_t n_dec, uint32_t waves_per_group, uint64_t max_grid,
                               uint64_t resident)
{
    const uint64_t room = max_grid < resident ? max_grid : resident;
    ShortList s{0u, 0u, 0u};
    for (uint32_t p = 0; p <= 5u; ++p) {
        const uint64_t need_e = ((n_enc << p) + waves_per_group - 1) / waves_per_group;
        const uint64_t need_d = ((n_dec << p) + waves_per_group - 1) / waves_per_group;
        if (need_e + need_d > room)
            break;
        s = ShortList{p, static_cast<uint32_t>(need_e + need_d), static_cast<uint32_t>(need_e)};
    }
    return s;
}

}  // namespace aesgpu
