// aes_cbc_enc_row.hip -- CBC encryption of few messages: sixteen lanes per
// message, one table lookup per lane per round.
//
// CBC encryption is one chain per message (section 3.1.2, eq 2), so a short
// list of messages is bound by the latency of a round, not by any rate.  The
// round is eq 26, e_j = T0[b0(W_j)] ^ T1[b1(W_{j+1})] ^ T2[b2(W_{j+2})] ^
// T3[b3(W_{j+3})] ^ k_j: here every one of its sixteen lookups has a lane of
// its own, in a row of 16 (a DPP row, so a wave walks four messages).
//
// A lane whose lookup counts for column j keeps column j: the sum of a
// column's four terms is formed in all four of its lanes, which then look up
// one byte each of that column in the next round.  Two XORs with a DPP move
// do it when the four lanes are a coset of a plane in the lane number's bits
// and the moves XOR the lane number with two vectors that span it.  The
// rounds alternate between two planes that share only 0, so that a column's
// lanes of one round are spread over all four columns of the next: {0, 1, 2,
// 3} (quad permutes by XOR 1 and 2) and {0, 7, 8, 15} (row half mirror is XOR
// 7, row rotation by 8 is XOR 8).  With q = lane / 4 (mod 4) the coset of the
// first and h of the second, a lane that holds column h and adds up over the
// first plane looks up byte h - q, and the other way round byte q - h (eq
// 19's shift: byte t of column x counts for column x - t).  Nr is even, so
// every block starts and ends with column h.
//
// A round's critical path is one byte permute, one LDS read and two XORs (the
// key is added in the wait states before the second), against three quad
// moves, four permutes, four reads and two XORs with a lane per column.  A
// lane needs one word of each entry for either kind of round, T_t of its t:
// 256 entries x 2 x 32 words, 64 KiB, conflict free, with the lookup address
// one v_perm_b32 as in the other kernels (entry in address bits 8 .. 15).
//
// Bound: that latency, 42 ns or 100 cycles a round, most of it the LDS read.
// AES-128, against four lanes per message: 16 messages of 4 KiB 149 -> 110 us,
// 1024 of 16 KiB 590 -> 427, 8192 of 4 KiB 162 -> 118.  A first form with the
// sum in one lane of four and a quad broadcast behind it took 46 ns; loads
// under a condition per block, each waited for at once, another 10.
#include <algorithm>

#include "aes_cbc_msgs.hpp"
#include "aes_device.hpp"

namespace aesgpu {

namespace {

// Layout of aes_cbc_msg (aesgpu.h).
struct RowMsg {
    uint64_t in_block;
    uint64_t out_block;
    uint64_t nblocks;
    uint64_t reserved;
    uint32_t iv[4];
};
static_assert(sizeof(RowMsg) == 48, "aes_cbc_msg layout");

// x of the lane that DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ uint32_t lane_move(uint32_t x)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true));
}

// v over the lanes of a coset, plus k: of {0, 1, 2, 3} and of {0, 7, 8, 15}.
__device__ __forceinline__ uint32_t sum_q(uint32_t v, uint32_t k)
{
    v ^= lane_move<0xb1>(v);            // quad_perm [1, 0, 3, 2]
    return v ^ k ^ lane_move<0x4e>(v);  // quad_perm [2, 3, 0, 1]
}

__device__ __forceinline__ uint32_t sum_h(uint32_t v, uint32_t k)
{
    v ^= lane_move<0x141>(v);            // row_half_mirror
    return v ^ k ^ lane_move<0x128>(v);  // row_ror:8
}

// The two cosets of a lane.
__device__ __forceinline__ uint32_t coset_q(uint32_t lane) { return (lane >> 2) & 3u; }
__device__ __forceinline__ uint32_t coset_h(uint32_t lane) { return (lane ^ ((lane & 4u) ? 3u : 0u)) & 3u; }

constexpr int kRowGroup = 8;  // blocks loaded and stored at once (one 128-byte line)

template <int NR>
__global__ __launch_bounds__(1024) void cbc_enc_msgs_row_kernel(const RowMsg* __restrict__ msgs, uint64_t nmsgs,
                                                                const uint32_t* in, uint64_t in_blocks,
                                                                uint32_t* out, uint64_t out_blocks,
                                                                uint32_t* rejected, RoundKeys rk)
{
    __shared__ __align__(16) uint32_t lds[256 * 64];
    {
        // words 4f .. 4f + 3 of every entry, f the same for all of a thread's entries
        const uint32_t f = threadIdx.x & 15u;
        uint32_t turn[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t l = (4u * f + i) & 31u, t = f < 8u ? coset_h(l) - coset_q(l) : coset_q(l) - coset_h(l);
            turn[i] = 8u * (t & 3u);
        }
        for (uint32_t i = threadIdx.x; i < 256u * 16u; i += blockDim.x) {
            const uint32_t v = c_tables.te0[i >> 4];
            *reinterpret_cast<uint4*>(lds + 4u * i) =
                make_uint4(__builtin_rotateleft32(v, turn[0]), __builtin_rotateleft32(v, turn[1]),
                           __builtin_rotateleft32(v, turn[2]), __builtin_rotateleft32(v, turn[3]));
        }
    }
    const uint32_t lane = threadIdx.x & 63u, q = coset_q(lane), h = coset_h(lane);
    uint32_t kc[NR + 1];  // odd rounds end in column q, even ones in column h
#pragma unroll
    for (int r = 0; r <= NR; ++r) {
        const uint32_t j = r % 2 ? q : h;
        kc[r] = j == 0 ? rk.w[4 * r] : j == 1 ? rk.w[4 * r + 1] : j == 2 ? rk.w[4 * r + 2] : rk.w[4 * r + 3];
    }
    // the round's byte of the word to bits 8 .. 15, the lane's place below it
    const uint32_t tq = (h - q) & 3u, th = (q - h) & 3u, base = (lane & 31u) << 2;
    const uint32_t sel_q = 0x0c0c0000u | ((4u + tq) << 8), sel_h = 0x0c0c0000u | ((4u + th) << 8);
    // last round: T_t has the S-box byte in byte t + 1 (mod 4); it moves to byte t, the others clear
    const uint32_t last = (0x0c0c0c0cu & ~(0xffu << (8u * th))) | (((th + 1u) & 3u) << (8u * th));
    __syncthreads();

    auto lookup_q = [&](uint32_t w) { return lds_word(lds, __builtin_amdgcn_perm(w, base, sel_q)); };
    auto lookup_h = [&](uint32_t w) { return lds_word(lds, __builtin_amdgcn_perm(w, base, sel_h) + 128u); };

    const uint64_t units = (nmsgs + 3u) / 4u;
    // a workgroup's waves that walk messages; the others only help with the table
    const uint64_t walk = min((uint64_t)(blockDim.x >> 6), (units + gridDim.x - 1) / gridDim.x);
    const uint32_t wave = threadIdx.x >> 6;
    for (uint64_t wv = wave < walk ? blockIdx.x * walk + wave : units; wv < units; wv += gridDim.x * walk) {
        const uint64_t m = wv * 4u + (lane >> 4);
        uint64_t nb = 0;
        const uint32_t* src = in;
        uint32_t* dst = out;
        uint32_t chain = 0;
        if (m < nmsgs) {
            const RowMsg& d = msgs[m];  // the sixteen lanes of a row read the same record
            const uint64_t n = d.nblocks, ib = d.in_block, ob = d.out_block;
            if (d.reserved == 0 && ib <= in_blocks && n <= in_blocks - ib && ob <= out_blocks &&
                n <= out_blocks - ob) {
                nb = n;
                src = in + 4u * ib + h;
                dst = out + 4u * ob + h;
                chain = d.iv[h];
            } else if (rejected != nullptr && (lane & 15u) == 0) {
                atomicAdd(rejected, 1u);
            }
        }
        uint32_t nxt[kRowGroup];
#pragma unroll
        for (uint32_t k = 0; k < kRowGroup; ++k)
            nxt[k] = 0u;
        if (nb != 0) {
#pragma unroll
            for (uint32_t k = 0; k < kRowGroup; ++k)
                nxt[k] = src[4u * (k < nb ? k : (uint32_t)nb - 1u)];
        }
        const uint32_t mine = (lane >> 2) & 3u;  // of four blocks, the one whose word this lane stores
        auto block = [&](uint32_t p) {
            uint32_t w = chain ^ (p ^ kc[0]);
#pragma unroll
            for (int round = 1; round < NR; round += 2) {
                w = sum_q(lookup_q(w), kc[round]);
                if (round + 1 < NR)
                    w = sum_h(lookup_h(w), kc[round + 1]);
            }
            chain = sum_h(__builtin_amdgcn_perm(0u, lookup_h(w), last), kc[NR]);
        };
        // a row's lanes share nb, so a row is wholly active or wholly idle
        for (uint64_t g = 0; g < nb; g += kRowGroup) {
            const uint32_t left = (uint32_t)(nb - g < 2u * kRowGroup ? nb - g : 2u * kRowGroup);  // of two groups
            uint32_t cur[kRowGroup], keep[kRowGroup / 4];
            const uint32_t* ahead = src + 4u * g;
#pragma unroll
            for (uint32_t k = 0; k < kRowGroup; ++k)
                cur[k] = nxt[k];
            // Unconditional loads (the last block again past the end): a
            // load under a condition of its own is waited for at once.
#pragma unroll
            for (uint32_t k = 0; k < kRowGroup; ++k) {
                const uint32_t i = kRowGroup + k < left ? kRowGroup + k : left - 1u;
                nxt[k] = ahead[4u * i];
            }
            if (__all(left >= kRowGroup)) {
#pragma unroll
                for (uint32_t k = 0; k < kRowGroup; ++k) {
                    block(cur[k]);
                    keep[k / 4] = k % 4 == 0 || mine == k % 4 ? chain : keep[k / 4];
                }
#pragma unroll
                for (uint32_t k = 0; k < kRowGroup; k += 4)
                    dst[4u * (g + k + mine)] = keep[k / 4];
            } else {
#pragma unroll
                for (uint32_t k = 0; k < kRowGroup; ++k) {
                    if (k < left) {
                        block(cur[k]);
                        if (mine == k % 4)
                            dst[4u * (g + k)] = chain;
                    }
                }
            }
        }
    }
}

template <int NR>
hipError_t launch_row(const void* msgs, uint64_t nmsgs, const void* in, uint64_t in_blocks, void* out,
                      uint64_t out_blocks, uint32_t* rejected, const RoundKeys& rk, int cus, hipStream_t stream)
{
    // Four messages per wave, spread evenly over the CUs: one workgroup per CU
    // up to 16 waves, two beyond.  At least 8 waves, which share the table's
    // fill (16 messages of 4 blocks 9.5 -> 5.4 us per launch against one).
    const uint64_t c = (uint64_t)cus, waves = (nmsgs + 3u) / 4u, per_cu = (waves + c - 1) / c;
    const uint64_t groups = per_cu <= 16u ? c : 2u * c;
    const uint64_t wg = std::min<uint64_t>(1024, std::max<uint64_t>(512, 64u * ((waves + groups - 1) / groups)));
    const uint64_t grid = std::min(groups, waves);
    hipLaunchKernelGGL(cbc_enc_msgs_row_kernel<NR>, dim3((uint32_t)grid), dim3((uint32_t)wg), 0, stream,
                       static_cast<const RowMsg*>(msgs), nmsgs, static_cast<const uint32_t*>(in), in_blocks,
                       static_cast<uint32_t*>(out), out_blocks, rejected, rk);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cbc_enc_row(int nr, const void* msgs, uint64_t nmsgs, const void* in, uint64_t in_blocks,
                              void* out, uint64_t out_blocks, uint32_t* rejected, const RoundKeys& rk, int cus,
                              hipStream_t stream)
{
    switch (nr) {
    case 10: return launch_row<10>(msgs, nmsgs, in, in_blocks, out, out_blocks, rejected, rk, cus, stream);
    case 12: return launch_row<12>(msgs, nmsgs, in, in_blocks, out, out_blocks, rejected, rk, cus, stream);
    case 14: return launch_row<14>(msgs, nmsgs, in, in_blocks, out, out_blocks, rejected, rk, cus, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace aesgpu
