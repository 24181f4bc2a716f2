// aes_ctr.hip -- counter mode on the same round core as ECB.
//
// CTR (section 3.1.5, eq 5; marked parallel in Table 1): data block j is
// XORed with the cipher of a counter block, and counter blocks of successive
// data blocks are successive 128-bit big-endian integers c0 + j (mod 2^128),
// so every block is independent, as in ECB.  Each lane builds its counter
// block from the block index (no memory read), runs the encryption rounds
// and XORs the result into the data it loaded: the same 32 bytes of HBM per
// block as an ECB encryption, and fewer LDS lookups (counter-mode caching,
// below).  Decryption is the same operation.  A partial last block is read and written byte by byte and
// uses the leading bytes of its key-stream block.
#include "aes_col_round.hpp"
#include "aes_ecb_kernel.hpp"

namespace aesgpu {

// State words of counter block c0 + b: byte 0 of the block is the most
// significant byte, and state word c holds bytes 4c..4c+3 little-endian.
__device__ __forceinline__ uint4 counter_state(const Counter128& c0, uint64_t b)
{
    const uint64_t lo = c0.lo + b;
    const uint64_t hi = c0.hi + (lo < c0.lo ? 1u : 0u);
    return make_uint4(__builtin_bswap32(static_cast<uint32_t>(hi >> 32)), __builtin_bswap32(static_cast<uint32_t>(hi)),
                      __builtin_bswap32(static_cast<uint32_t>(lo >> 32)), __builtin_bswap32(static_cast<uint32_t>(lo)));
}

__device__ __forceinline__ uint4 xor4(uint4 a, uint4 b) { return make_uint4(a.x ^ b.x, a.y ^ b.y, a.z ^ b.z, a.w ^ b.w); }

// Counter-mode caching (rounds 1 and 2).  The kernel walks the counters in
// units of span = 64 * BPT consecutive values that start at a multiple of
// span, so within a unit bytes 0..14 of the counter block are the same for
// every lane and only byte 15 (the top byte of state word 3) differs.  In
// round 1 (eq 26) byte 15 feeds one lookup, T3 of output column 0; the
// other 15 lookups and output columns 1..3 are the same for the whole unit.
// In round 2 every output column then has exactly one lookup that depends
// on the lane (a byte of column 0) and three that do not.  The 27 shared
// lookups of a wave's next 64 units are done side by side, one unit per lane,
// and handed out as uniform values.  A lane's own 1 + 4 lookups
// depend, beside its counters' low byte, on column 0 alone, whose other
// inputs are bytes 0, 5 and 10 of the counter: byte 10 moves every 2^40
// blocks.  So a lane keeps their four words per block (ctr_lane_words) over
// the units it walks and renews them only when column 0's shared part or the
// unit's low byte differs: rounds 1-2 cost a block four XORs and no lookup,
// 16 Nr - 32 in all, 128 for AES-128 instead of 160.
// Bound: as ECB, with fewer lookups.  AES-128 1 GiB 632 -> 606 us, 16 MiB 15.3
// -> 14.5, against a unit's shared lookups as scalar loads and a lane's own
// five for every block.  (1 GiB takes 3.55 us per lookup of a block and 154
// us beside them, here as for ECB with 10 and 14 rounds.)

// T_t[byte t of w] for a per-lane w, from the tables of placement PL in LDS.
template <int PL, int T>
__device__ __forceinline__ uint32_t lane_lookup(const uint32_t* lds, const LaneBases<PL, false>& lb, uint32_t w)
{
    if (PL == kPlace4)
        return lds_word(lds, addr_of<256, T>(w, lb.m7, lb.b[T]));
    if (PL == kPlace2) {
        const uint32_t v = lds_word(lds, addr_of<256, T>(w, lb.m7, lb.b[T]));  // T0 or T2 as stored
        return (T & 1) ? rotl8(v) : v;
    }
    const uint32_t v = lds_word(lds, addr_of<128, T>(w, lb.m7, lb.b[T]));      // T0
    return T == 0 ? v : T == 1 ? rotl8(v) : T == 2 ? rotl16(v) : rotl24(v);
}

// T_t[byte t of w] for a uniform w, from the source table (scalar load).
template <int T>
__device__ __forceinline__ uint32_t uniform_lookup(uint32_t w)
{
    const uint32_t v = c_tables.te0[(w >> (8 * T)) & 255u];
    return T == 0 ? v : (v << (8 * T)) | (v >> (32 - 8 * T));
}

// Rounds 1-2 of a unit, the part its blocks share: w0 .. w3 = state words of
// the unit's first counter; rk(i) = round-key word i as used in eq 26.
struct CtrShared {
    uint32_t u0, v0, v1, v2, v3;  // round 1 column 0 without its lane lookup; round 2 without theirs
};

template <int PL, bool kUniform, class K>
__device__ __forceinline__ CtrShared ctr_shared(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3,
                                                const uint32_t* lds, const LaneBases<PL, false>& lb, const K& rk)
{
    const uint32_t x0 = w0 ^ rk(0), x1 = w1 ^ rk(1), x2 = w2 ^ rk(2), x3 = w3 ^ rk(3);  // byte 15 of x3 unused
    auto t0 = [&](uint32_t w) { return kUniform ? uniform_lookup<0>(w) : lane_lookup<PL, 0>(lds, lb, w); };
    auto t1 = [&](uint32_t w) { return kUniform ? uniform_lookup<1>(w) : lane_lookup<PL, 1>(lds, lb, w); };
    auto t2 = [&](uint32_t w) { return kUniform ? uniform_lookup<2>(w) : lane_lookup<PL, 2>(lds, lb, w); };
    auto t3 = [&](uint32_t w) { return kUniform ? uniform_lookup<3>(w) : lane_lookup<PL, 3>(lds, lb, w); };
    CtrShared c;
    c.u0 = t0(x0) ^ t1(x1) ^ t2(x2) ^ rk(4);
    const uint32_t u1 = t0(x1) ^ t1(x2) ^ t2(x3) ^ t3(x0) ^ rk(5);
    const uint32_t u2 = t0(x2) ^ t1(x3) ^ t2(x0) ^ t3(x1) ^ rk(6);
    const uint32_t u3 = t0(x3) ^ t1(x0) ^ t2(x1) ^ t3(x2) ^ rk(7);
    c.v0 = t1(u1) ^ t2(u2) ^ t3(u3) ^ rk(8);
    c.v1 = t0(u1) ^ t1(u2) ^ t2(u3) ^ rk(9);
    c.v2 = t0(u2) ^ t1(u3) ^ t3(u1) ^ rk(10);
    c.v3 = t0(u3) ^ t2(u1) ^ t3(u2) ^ rk(11);
    return c;
}

// A lane's terms of the four columns after round 2: u0 is round 1's column 0
// without its lane lookup, w3 the lane's state word 3 (its top byte is read).
template <int PL>
__device__ __forceinline__ uint4 ctr_lane_words(uint32_t u0, uint32_t w3, const uint32_t* lds,
                                                const LaneBases<PL, false>& lb, uint32_t k3)
{
    const uint32_t a = u0 ^ lane_lookup<PL, 3>(lds, lb, w3 ^ k3);
    return make_uint4(lane_lookup<PL, 0>(lds, lb, a), lane_lookup<PL, 3>(lds, lb, a),
                      lane_lookup<PL, 2>(lds, lb, a), lane_lookup<PL, 1>(lds, lb, a));
}

// One unit the fast path cannot take (the first, when the counters start
// inside a unit, and the last, partial one): lane by lane, with the whole
// cipher on each counter; a partial last block is read and written byte by
// byte and uses the leading bytes of its key-stream block.
template <int NR, int BPT, int PL, class K>
__device__ __forceinline__ void ctr_edge_unit(const uint4* __restrict__ in, uint4* __restrict__ out, uint64_t nbytes,
                                              const Counter128& c0, uint64_t u, uint32_t d, const uint32_t* lds,
                                              const LaneBases<PL, false>& lb, const K& key)
{
    const uint64_t span = 64u * BPT;
    const uint64_t nfull = nbytes / 16u, nblocks = (nbytes + 15u) / 16u;
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const uint64_t i = u * span + lane + 64u * k;  // counter offset from c0 - d
        if (i < d)
            continue;
        const uint64_t b = i - d;
        if (b < nfull) {
            store_block(out + b, xor4(in[b], crypt_block<NR, false, PL>(counter_state(c0, b), lds, lb, key)));
        } else if (b < nblocks) {
            const uint4 ks = crypt_block<NR, false, PL>(counter_state(c0, b), lds, lb, key);
            const uint32_t kw[4] = {ks.x, ks.y, ks.z, ks.w};
            const uint8_t* src = reinterpret_cast<const uint8_t*>(in) + 16u * b;
            uint8_t* dst = reinterpret_cast<uint8_t*>(out) + 16u * b;
            const uint32_t rem = static_cast<uint32_t>(nbytes - 16u * b);  // 1..15
            for (uint32_t t = 0; t < rem; ++t)
                dst[t] = static_cast<uint8_t>(src[t] ^ (kw[t >> 2] >> (8u * (t & 3u))));
        }
    }
}

// CTR over nbytes.  Counter of data block b: c0 + b.  With d = c0 mod span
// (span a power of two), block b belongs to unit (b + d) / span, and unit u
// holds the counters c0 - d + u * span + i, i < span, whose bytes 0..14 do
// not change.  Units 1 .. end_full - 1 (and unit 0 when d = 0) hold whole
// blocks only and take the cached path; the first unit (d > 0) and the last
// one (partial blocks) take ctr_edge_unit.
// kSingle: for launches whose waves walk at most one whole unit each, where
// there is nothing to keep: the unit's shared words as scalar loads, no look at
// whether the lane's words still hold (AES-256, 4 MiB 7.63 -> 7.44 us, AES-128
// 6.47 -> 6.35, against the general form).
template <int NR, int BPT, int PL, bool kSingle>
__global__ __launch_bounds__(1024) void ctr_kernel(const uint4* __restrict__ in, uint4* __restrict__ out,
                                                   uint64_t nbytes, Counter128 c0, RoundKeys rk)
{
    __shared__ __align__(16) uint32_t lds[Layout<PL, false>::words];
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t waves_per_grid = (uint64_t)gridDim.x * (blockDim.x >> 6);
    // uniform across the wave (made explicit, so the unit's counter and the
    // shared lookups live in scalar registers)
    const uint64_t wave_id =
        (uint64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr uint64_t span = 64u * BPT;
    const uint64_t nfull = nbytes / 16u;                  // whole blocks
    const uint64_t nblocks = (nbytes + 15u) / 16u;        // including a partial last block
    const uint32_t d = static_cast<uint32_t>(c0.lo & (span - 1u));
    const uint64_t first_full = d ? 1u : 0u;
    const uint64_t end_full = (nfull + d) / span;          // units [first_full, end_full) are whole
    const uint64_t n_units = (nblocks + d + span - 1u) / span;
    const uint64_t base_lo = c0.lo - d;                    // counter of unit 0, slot 0 (no borrow)
    uint64_t u = first_full + wave_id;
    // the data of the first unit is requested before the table fill
    uint4 cur[BPT];
    if (u < end_full) {
#pragma unroll
        for (int k = 0; k < BPT; ++k)
            cur[k] = in[u * span - d + lane + 64u * k];
    }
    fill_tables<PL, false>(lds, &c_tables);
    __syncthreads();
    const LaneBases<PL, false> lb(threadIdx.x);
    auto key = [&](int i) { return rk.w[i]; };
    // rounds 1-2 of the shared part need eq 26's keys as they are (the
    // 2-table kernels receive the inner-round words turned right by 8)
    auto key12 = [&](int i) { return (PL == kPlace2 && i >= 4) ? rotl8(rk.w[i]) : rk.w[i]; };
    uint4 mine[BPT];  // ctr_lane_words of column 0's shared part `of` and low byte `low`
    uint32_t of = 0, low = ~0u;
    CtrShared ahead{};
    uint32_t turn = 0;
    for (; u < end_full; u += waves_per_grid) {
        const uint64_t first = u * span - d + lane;
        const uint64_t un = u + waves_per_grid;
        uint4 nxt[BPT];
        if (un < end_full) {
#pragma unroll
            for (int k = 0; k < BPT; ++k)
                nxt[k] = in[un * span - d + lane + 64u * k];
        }
        CtrShared c;
        if constexpr (kSingle) {
            const uint64_t lo = base_lo + u * span, hi = c0.hi + (lo < base_lo ? 1u : 0u);
            c = ctr_shared<PL, true>(__builtin_bswap32(static_cast<uint32_t>(hi >> 32)),
                                     __builtin_bswap32(static_cast<uint32_t>(hi)),
                                     __builtin_bswap32(static_cast<uint32_t>(lo >> 32)),
                                     __builtin_bswap32(static_cast<uint32_t>(lo)), lds, lb, key12);
        } else {
            if ((turn & 63u) == 0) {
                // the shared words of the wave's next 64 units, one unit per lane
                // (the low byte of a unit's first counter is a multiple of span)
                const uint64_t lo = base_lo + (u + lane * waves_per_grid) * span;
                const uint64_t hi = c0.hi + (lo < base_lo ? 1u : 0u);
                ahead = ctr_shared<PL, false>(__builtin_bswap32(static_cast<uint32_t>(hi >> 32)),
                                              __builtin_bswap32(static_cast<uint32_t>(hi)),
                                              __builtin_bswap32(static_cast<uint32_t>(lo >> 32)),
                                              __builtin_bswap32(static_cast<uint32_t>(lo)), lds, lb, key12);
            }
            auto of_unit = [&](uint32_t v) {
                return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), turn & 63u));
            };
            c = {of_unit(ahead.u0), of_unit(ahead.v0), of_unit(ahead.v1), of_unit(ahead.v2), of_unit(ahead.v3)};
            ++turn;
        }
        const uint32_t w3 = __builtin_bswap32(static_cast<uint32_t>(base_lo + u * span));
        if (kSingle || c.u0 != of || (w3 >> 24) != low) {
            of = c.u0;
            low = w3 >> 24;
            // slot lane + 64k: only byte 15 (bits 24..31 of word 3) moves, with no carry
#pragma unroll
            for (int k = 0; k < BPT; ++k)
                mine[k] = ctr_lane_words<PL>(c.u0, w3 + ((lane + 64u * k) << 24), lds, lb, rk.w[3]);
        }
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const uint4 s = make_uint4(c.v0 ^ mine[k].x, c.v1 ^ mine[k].y, c.v2 ^ mine[k].z, c.v3 ^ mine[k].w);
            store_block(out + first + 64u * k, xor4(cur[k], crypt_rounds<NR, false, PL, 3>(s, lds, lb, key)));
        }
#pragma unroll
        for (int k = 0; k < BPT; ++k)
            cur[k] = nxt[k];
    }
    // the edge units: the first (counters start inside it) on wave 0, the
    // last (holds the end of the data) on the grid's last wave
    if (d && wave_id == 0)
        ctr_edge_unit<NR, BPT, PL>(in, out, nbytes, c0, 0, d, lds, lb, key);
    const uint64_t back = first_full > end_full ? first_full : end_full;
    if (back < n_units && !(d && back == 0) && wave_id == waves_per_grid - 1)
        ctr_edge_unit<NR, BPT, PL>(in, out, nbytes, c0, back, d, lds, lb, key);
}

// CTR with one column word per lane (four lanes per block), for the sizes
// where ECB takes that form: a launch bound by the latency of one block's
// rounds.  Lane l of a wave holds word l of the unit's 16 blocks (256 bytes).
// The quad of a partial last block computes all of its key stream and its
// lanes move the words and bytes that exist.
// Against one state per lane, AES-256: 18,602 bytes 6.9 -> 3.8 us per launch
// (replayed graph), 512 KiB 7.7 -> 4.1; AES-128: 64 KiB 6.2 -> 3.5.
template <int NR, int PL>
__global__ __launch_bounds__(1024) void ctr_col_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                       uint64_t nbytes, Counter128 c0, RoundKeys rk)
{
    __shared__ __align__(16) uint32_t lds[Layout<PL, false>::words];
    const uint32_t lane = threadIdx.x & 63u, j = lane & 3u;
    const uint64_t waves_per_grid = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t nwords = nbytes / 4u;                       // whole words
    const uint64_t nblocks = (nbytes + 15u) / 16u;             // including a partial last block
    const uint64_t units = (nblocks + 15u) / 16u;
    uint64_t wv = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    auto word_at = [&](uint64_t unit) { return in[min(unit * 64u + lane, nwords - 1u)]; };
    uint32_t cur = 0;
    if (wv < units && nwords != 0)
        cur = word_at(wv);
    fill_tables<PL, false>(lds, &c_tables);
    const uint32_t j_hi = j & 2u, j_lo = j & 1u;
    uint32_t kc[NR + 1];
#pragma unroll
    for (int r = 0; r <= NR; ++r)
        kc[r] = j == 0 ? rk.w[4 * r] : j == 1 ? rk.w[4 * r + 1] : j == 2 ? rk.w[4 * r + 2] : rk.w[4 * r + 3];
    __syncthreads();
    const LaneBases<PL, false> lb(threadIdx.x);
    for (; wv < units; wv += waves_per_grid) {
        const uint64_t wn = wv + waves_per_grid;
        uint32_t nxt = 0;
        if (wn < units && nwords != 0)
            nxt = word_at(wn);
        const uint64_t i = wv * 64u + lane, b = i / 4u;
        if (b < nblocks) {
            const uint64_t lo = c0.lo + b, hi = c0.hi + (lo < c0.lo ? 1u : 0u), half = j_hi ? lo : hi;
            const uint32_t w = __builtin_bswap32(static_cast<uint32_t>(j_lo ? half : half >> 32));
            const uint32_t ks = col_block<NR, false, PL>(w, lds, lb, kc);
            if (i < nwords) {
                __builtin_nontemporal_store(cur ^ ks, out + i);
            } else if (4u * i < nbytes) {
                const uint8_t* src = reinterpret_cast<const uint8_t*>(in + i);
                uint8_t* dst = reinterpret_cast<uint8_t*>(out + i);
                for (uint32_t t = 0; t < static_cast<uint32_t>(nbytes - 4u * i); ++t)
                    dst[t] = static_cast<uint8_t>(src[t] ^ (ks >> (8u * t)));
            }
        }
        cur = nxt;
    }
}

template <int NR, int PL>
hipError_t launch_ctr_col(const void* in, void* out, uint64_t nbytes, const Counter128& c0, const RoundKeys& rk,
                          const LaunchShape& shape, int cus, hipStream_t stream)
{
    auto kern = ctr_col_kernel<NR, PL>;
    int grid = 0;
    hipError_t e = col_grid_for(reinterpret_cast<const void*>(kern), shape, cus, (nbytes + 15u) / 16u, &grid);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(shape.wg), 0, stream, static_cast<const uint32_t*>(in),
                       static_cast<uint32_t*>(out), nbytes, c0, rk);
    return hipGetLastError();
}

template <int NR, int BPT, int PL>
hipError_t launch_ctr_one(const void* in, void* out, uint64_t nbytes, const Counter128& c0, const RoundKeys& rk,
                          const LaunchShape& shape, int cus, hipStream_t stream)
{
    auto kern = ctr_kernel<NR, BPT, PL, false>;
    int grid = 0;
    const uint64_t nblocks = (nbytes + 15u) / 16u;
    hipError_t e = grid_for(reinterpret_cast<const void*>(kern), shape, cus, nblocks, &grid);
    if (e != hipSuccess)
        return e;
    if (nblocks <= (uint64_t)grid * (uint64_t)shape.wg * BPT)  // whole units: no more than waves
        kern = ctr_kernel<NR, BPT, PL, true>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(shape.wg), 0, stream, static_cast<const uint4*>(in),
                       static_cast<uint4*>(out), nbytes, c0, rk);
    return hipGetLastError();
}

template <int BPT, int PL>
hipError_t launch_ctr_nr(int nr, const void* in, void* out, uint64_t nbytes, const Counter128& c0,
                         const RoundKeys& rk, const LaunchShape& shape, int cus, hipStream_t stream)
{
    if constexpr (BPT == AES_BPT_COLUMN) {
        switch (nr) {
        case 10: return launch_ctr_col<10, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        case 12: return launch_ctr_col<12, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        case 14: return launch_ctr_col<14, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (nr) {
        case 10: return launch_ctr_one<10, BPT, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        case 12: return launch_ctr_one<12, BPT, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        case 14: return launch_ctr_one<14, BPT, PL>(in, out, nbytes, c0, rk, shape, cus, stream);
        default: return hipErrorInvalidValue;
        }
    }
}

template <int PL>
hipError_t launch_ctr_bpt(int nr, const void* in, void* out, uint64_t nbytes, const Counter128& c0,
                          const RoundKeys& rk, const LaunchShape& shape, int cus, hipStream_t stream)
{
    switch (shape.bpt) {
    case AES_BPT_COLUMN:
        return launch_ctr_nr<AES_BPT_COLUMN, PL>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    case 1: return launch_ctr_nr<1, PL>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    case 2: return launch_ctr_nr<2, PL>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    case 4: return launch_ctr_nr<4, PL>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ctr(const LaunchShape& shape, int placement, int nr, const void* in, void* out, uint64_t nbytes,
                      const Counter128& c0, const RoundKeys& rk, int cus, hipStream_t stream)
{
    switch (placement) {
    case kPlace4: return launch_ctr_bpt<kPlace4>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    case kPlace2: return launch_ctr_bpt<kPlace2>(nr, in, out, nbytes, c0, inner_keys_rotr8(rk, nr), shape, cus, stream);
    case kPlace1: return launch_ctr_bpt<kPlace1>(nr, in, out, nbytes, c0, rk, shape, cus, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace aesgpu
