// aes_cbc_dec_flat.hip -- CBC decryption of a message set, walked block by
// block whatever the messages' lengths.
//
// Decryption has no chain (section 3.1.2, eq 2: P_i = invcipher(C_i) XOR
// C_{i-1}), so any 64 blocks of a message set can be a wave's work.  A wave
// takes a group of up to 64 messages, one record per lane, drops the empty and
// the refused ones, and numbers the group's blocks from 0 by a prefix sum over
// the lengths.  It then walks those numbers 64 at a time, one block per lane,
// so every lane has a block however short or ragged the messages are.  Which
// message a lane's block belongs to follows from one 64-bit mask per step, the
// bit of every number at which a message starts: the count of bits up to the
// lane gives the message, a lane permute its offsets.  The block before a
// message's first one is its IV, read from the record.
//
// A group's messages come from all over the list (aes_cbc_flat_split.hpp), so
// that a list sorted by length, or one with its long messages in a row, keeps
// all waves busy equally long.  With 64 consecutive messages to a group such
// lists took (AES-128, us; consecutive -> spread; one wave per message between
// them): 2^16 of 1 ... 4096 blocks sorted 2516 -> 415 (483), 2^14 of 1 ... 65536
// sorted 9975 -> 1288 (2942), 2^16 with 64 of 65536 blocks in a row 22476 -> 644
// (2550), 2^16 of 0 ... 256 sorted 175 -> 102 (115); in random order 104 -> 103.
//
// Short lists of long messages split the other way: `slices` waves share a
// group (then one message) and take every slices-th step of it.  Block b
// reads ciphertext block b - 1, which another wave may own, so slices need
// separate arenas; a single wave loads a step's blocks, and the blocks before
// them, ahead of the stores of the step before, so in place is safe.
#include <algorithm>

#include "aes_cbc_flat_split.hpp"
#include "aes_cbc_msgs.hpp"
#include "aes_ecb_kernel.hpp"

namespace aesgpu {

namespace {

// Layout of aes_cbc_msg (aesgpu.h).
struct FlatMsg {
    uint64_t in_block;
    uint64_t out_block;
    uint64_t nblocks;
    uint64_t reserved;
    uint4 iv;
};
static_assert(sizeof(FlatMsg) == 48, "aes_cbc_msg layout");

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

__device__ __forceinline__ uint64_t pull(uint32_t from, uint64_t v)
{
    const int a = static_cast<int>(from << 2);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(a, static_cast<int>(v)));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(a, static_cast<int>(v >> 32)));
    return lo | (static_cast<uint64_t>(hi) << 32);
}

// v of a uniform lane, as a uniform value.
__device__ __forceinline__ uint64_t lane_value(uint64_t v, uint32_t from)
{
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(v), from)) |
           ((uint64_t) static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), from)) << 32);
}

__device__ __forceinline__ uint64_t push(uint32_t to, uint64_t v)
{
    const int a = static_cast<int>(to << 2);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(a, static_cast<int>(v)));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(a, static_cast<int>(v >> 32)));
    return lo | (static_cast<uint64_t>(hi) << 32);
}

template <int NR, int PL>
__global__ __launch_bounds__(1024) void cbc_dec_flat_kernel(const FlatMsg* __restrict__ msgs, uint64_t nmsgs,
                                                            FlatSplit split, const uint4* in, uint64_t in_blocks,
                                                            uint4* out, uint64_t out_blocks, uint32_t* rejected,
                                                            RoundKeys rk)
{
    __shared__ __align__(16) uint32_t lds[Layout<PL, true>::words];
    fill_tables<PL, true>(lds, &c_tables);
    __syncthreads();
    const LaneBases<PL, true> lb(threadIdx.x);
    auto key = [&](int i) { return rk.w[i]; };

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t groups = split.groups;
    const uint32_t per_group = split.per_group, slices = split.slices;
    const uint64_t step = (uint64_t)slices * 64u;
    const uint64_t units = groups * slices;  // below 2^32 where slices > 1
    // a workgroup's waves that walk units; the others only help with the tables
    const uint64_t walk = min((uint64_t)(blockDim.x >> 6), (units + gridDim.x - 1) / gridDim.x);
    for (uint64_t u = wave < walk ? blockIdx.x * walk + wave : units; u < units; u += gridDim.x * walk) {
        const uint64_t g = slices > 1 ? static_cast<uint32_t>(u) / slices : u;
        const uint32_t slice = static_cast<uint32_t>(u - g * slices);
        // 32 bits number the group's messages from m0 on
        const uint64_t m0 = split.run_log2 == 6u ? g * per_group : 0;
        const uint64_t m = flat_message(split, g, min(lane, per_group - 1u));
        // one record per lane; a lane without one, or with one that is refused, has no blocks
        uint64_t nb = 0, d_in = 0, d_out = 0;
        if (lane < per_group && m < nmsgs) {
            const FlatMsg* d = msgs + m;
            const uint64_t n = d->nblocks, ib = d->in_block, ob = d->out_block;
            if (d->reserved == 0 && ib <= in_blocks && n <= in_blocks - ib && ob <= out_blocks &&
                n <= out_blocks - ob) {
                nb = n, d_in = ib, d_out = ob;
            } else if (rejected != nullptr && slice == 0) {
                atomicAdd(rejected, 1u);
            }
        }
        // numbers of the group's blocks: message of lane l has [start, start + nb)
        uint64_t end = nb;
        for (uint32_t s = 1; s < per_group; s <<= 1) {
            const uint64_t below = pull(lane - s, end);
            end += lane >= s ? below : 0u;
        }
        const uint64_t total = lane_value(end, per_group - 1);
        uint64_t start = end - nb;
        d_in -= start;
        d_out -= start;
        uint32_t rec = static_cast<uint32_t>(m - m0);
        // messages with blocks move to lanes 0 .. have - 1, in order
        const uint64_t some = __ballot(nb != 0);
        const uint32_t have = static_cast<uint32_t>(__popcll(some));
        if (some & (some + 1)) {
            const uint32_t below = lanes_below(some);
            const uint32_t to = nb != 0 ? below : have + (lane - below);
            start = push(to, start);
            d_in = push(to, d_in);
            d_out = push(to, d_out);
            rec = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(static_cast<int>(to << 2), static_cast<int>(rec)));
        }
        if (lane >= have)
            start = ~(uint64_t)0 >> 1;  // behind every block

        uint4 c, p, *to = out;  // the lane's block of a step, the ciphertext before it, its place
        bool on = false;
        // Each turn loads one step and then finishes the one loaded before it.
        // seen: messages whose start lies below the step's base
        uint32_t seen = 0;
        for (uint64_t base = (uint64_t)slice * 64u;; base += step) {
            uint4 nc, np, *nto = out;
            bool non = false;
            if (base < total) {
                const uint64_t n = base + lane;
                non = n < total;
                seen = static_cast<uint32_t>(__popcll(__ballot(start < base)));
                const uint32_t rel = start - base < 64u ? static_cast<uint32_t>(start - base) : 64u;
                const uint4* prev;
                uint64_t bi, bo;
                uint64_t left = __ballot(rel < 64u);
                if (left == 0) {
                    // the whole step inside one message
                    const uint32_t o = seen - 1u;
                    bi = lane_value(d_in, o) + n;
                    bo = lane_value(d_out, o) + n;
                    prev = in + bi - 1;
                } else {
                    uint64_t starts = 0;  // gathered on the scalar unit, which is idle here
                    do {
                        starts |= 1ull << __builtin_amdgcn_readlane(rel, __builtin_ctzll(left));
                        left &= left - 1;
                    } while (left != 0);
                    const bool first = (starts >> lane) & 1u;
                    const uint32_t owner = seen + lanes_below(starts) + (first ? 1u : 0u) - 1u;
                    bi = pull(owner, d_in) + n;
                    bo = pull(owner, d_out) + n;
                    const uint32_t r = static_cast<uint32_t>(
                        __builtin_amdgcn_ds_bpermute(static_cast<int>(owner << 2), static_cast<int>(rec)));
                    prev = first ? &msgs[m0 + r].iv : in + bi - 1;
                }
                nto = out + bo;
                if (non) {
                    nc = in[bi];
                    np = *prev;
                }
            }
            if (on) {
                const uint4 x = crypt_block<NR, true, PL>(c, lds, lb, key);
                *to = make_uint4(x.x ^ p.x, x.y ^ p.y, x.z ^ p.z, x.w ^ p.w);
            }
            if (base >= total)
                break;
            c = nc, p = np, to = nto, on = non;
        }
    }
}

template <int NR, int PL>
hipError_t launch_flat(const FlatMsg* msgs, uint64_t nmsgs, const FlatSplit& split, const void* in, uint64_t in_blocks,
                       void* out, uint64_t out_blocks, uint32_t* rejected, const RoundKeys& rk, int wg, int max_grid,
                       hipStream_t stream)
{
    const uint64_t grid = std::min<uint64_t>((uint64_t)max_grid, split.groups * split.slices);
    hipLaunchKernelGGL((cbc_dec_flat_kernel<NR, PL>), dim3((uint32_t)grid), dim3(wg), 0, stream, msgs, nmsgs, split,
                       static_cast<const uint4*>(in), in_blocks, static_cast<uint4*>(out), out_blocks, rejected, rk);
    return hipGetLastError();
}

}  // namespace

// The decryption tables fill a CU's LDS (160 KiB), so a CU holds one
// workgroup, of at most 16 waves.
hipError_t launch_cbc_dec_flat(int nr, const void* msgs, uint64_t nmsgs, const void* in, uint64_t in_blocks,
                               void* out, uint64_t out_blocks, uint32_t* rejected, const RoundKeys& rk, int cus,
                               hipStream_t stream)
{
    const FlatSplit split = flat_split(nmsgs, in_blocks, in == out, cus);
    // At least 8 waves, which fill the tables in one memory round trip (16
    // messages of 4 blocks 13.4 -> 6.1 us per launch against one wave).
    const uint64_t c = (uint64_t)cus, per_cu = (split.groups * split.slices + c - 1) / c;
    const int wg = (int)std::min<uint64_t>(1024, std::max<uint64_t>(512, 64u * per_cu));
    const FlatMsg* m = static_cast<const FlatMsg*>(msgs);
    switch (nr) {
    case 10:
        return launch_flat<10, kPlace4>(m, nmsgs, split, in, in_blocks, out, out_blocks, rejected, rk, wg, cus, stream);
    case 12:
        return launch_flat<12, kPlace4>(m, nmsgs, split, in, in_blocks, out, out_blocks, rejected, rk, wg, cus, stream);
    case 14:
        return launch_flat<14, kPlace4>(m, nmsgs, split, in, in_blocks, out, out_blocks, rejected, rk, wg, cus, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace aesgpu
