// Prune a dense matrix to Balanced-Sparsity form and pack it
// (arXiv 1811.00206: Sec. 3.1 pattern; Sec. 3.2 / Algorithm 1, the per-block
// "order by absolute magnitude, drop the smallest" step, taken in one shot to
// exactly k survivors per bank).
//
// Selection never sorts and never touches floating point:
//   * key = bit pattern of |w| (monotone in |w| for finite values);
//   * the k-th largest key T is built bit by bit from the top: the bit is set if
//     at least k keys have the prefix built so far with that bit set;
//   * every key > T survives; of the keys == T the first k - #(key > T) in
//     offset order survive, which is the lower-offset tie rule;
//   * survivors get their output slot from prefix counts in offset order, so
//     offsets come out ascending; values are copied bit for bit.
// Algorithm 1 compares against a threshold with "<", which would keep every
// element tied with the threshold; counting keeps exactly k instead.
//
// LPB lanes share a bank, each owning C consecutive elements of it (C <= 32, 64 in banks over
// 1024), so a wavefront works on 64/LPB banks at once.  Two things bound this kernel: the stream of
// W and the vector ALU, which overlap only across the wavefronts that are resident (a wavefront
// copies, waits, then selects), so every step is built to touch an element few times:
//   * the wavefront's banks are one contiguous piece of W; it goes to LDS with
//     direct-to-LDS loads (no registers) and stays there, so that a kept value is fetched
//     by its offset at the very end and nothing else carries values around;
//   * the keys are bit-sliced a byte at a time, from the top: eight masks (one bit per
//     element of the lane) come out of a byte gather and an 8 x 8 bit transpose, and a
//     select step costs one AND and one popcount per 32 elements plus the exchange over the
//     LPB lanes.  As soon as every bank of the wavefront needs all of its remaining
//     candidates the lower bytes are never looked at: for Gaussian fp32 weights the cut is
//     settled after 8 exponent and about 12 mantissa bits, so the last byte is skipped;
//   * lanes own consecutive elements, so a lane's survivors are consecutive in the output:
//     one prefix over the LPB lanes, then a walk over the set bits that writes offsets
//     only (k steps for a whole bank in one lane);
//   * offsets and values leave as whole words: four outputs per lane and step, the values
//     gathered from LDS through the offsets just written.
// Measured (MI355X, back to back over three matrices), before and now; before, 16-byte pieces
// striped over the lanes were transposed whole and every element was written or sent to a
// trash slot: 6000 x 3000 fp32, 10 of 100 kept: 22.4 -> 16.8 us (4.8 TB/s of W, vals and idx);
// 4096 x 25088 binary16, 6 of 64: 62.9 -> 46.6 us (5.0 TB/s); 11908 x 7616 binary16, 18 of 64:
// 63.5 -> 52.7 us.  Vector instructions on the first: 12.9 M -> 6.6 M, 585 per wavefront, 11
// wavefronts per SIMD: 10.7 of the 16.8 us; its bytes alone take 13.3 us at the 6.1 TB/s at which
// a product streams weights here.
// Re-pruning a packed matrix to fewer weights per bank (one more round of
// Algorithm 1's loop) runs the same kernel on the stored values, k per bank: 10 -> 5 of 100 on the
// 6000 x 3000 matrix 7.9 us (9.6 with one byte fetched per lane and step, 9.5 with the kernel before
// the bit-sliced bytes), 128 -> 64 of 256 on 16384 x 8192 90 us (134, 144).
#pragma once
#include "bs_internal.h"

namespace bs {
namespace {

// ---- bit-sliced selection ---------------------------------------------------
// 8 x 8 bit transpose inside each of the four byte columns of q[0..7]: afterwards bit
// 8j+g of q[t] is what bit 8j+t of q[g] was.
template <int J, uint32_t M>
__device__ __forceinline__ void swap_bits(uint32_t (&q)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if ((i & J) == 0) {
            const uint32_t a = q[i], b = q[i + J];
            q[i] = (a & M) | ((b << J) & ~M);
            q[i + J] = ((a >> J) & M) | (b & ~M);
        }
    }
}
__device__ __forceinline__ void transpose8(uint32_t (&q)[8]) {
    swap_bits<4, 0x0F0F0F0Fu>(q);
    swap_bits<2, 0x33333333u>(q);
    swap_bits<1, 0x55555555u>(q);
    // kept opaque: merged into the select steps the last stage loses its bit-field inserts
#pragma unroll
    for (int i = 0; i < 8; ++i) asm("" : "+v"(q[i]));
}

// State of a lane's search: candidates (keys that agree with the threshold so far), keys
// known to be greater, and how many more survivors the candidates must give, minus one.
template <int NM>
struct Select {
    uint32_t cand[NM], gt[NM];
    int r1;
};

// One bit of the threshold, s[m] = that bit of the lane's elements 32m .. 32m+31.
template <int LPB, int NM>
__device__ __forceinline__ void select_bit(Select<NM>& t, const uint32_t (&s)[NM]) {
    uint32_t ones[NM];
    int c = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        ones[m] = t.cand[m] & s[m];
        c += __popc(ones[m]);
    }
    // (kept opaque: folded into the exchange the popcount would be computed twice)
    if constexpr (LPB > 1) asm("" : "+v"(c));
    c = group_sum_i<LPB>(c);
    // take = all ones if enough keys have the bit set (the threshold has it), else zero
    const int left = t.r1 - c;
    uint32_t take = (uint32_t)(left >> 31);
    asm("" : "+v"(take));   // stays a mask: turned back into compares it costs three more per bit
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        t.gt[m] |= ones[m] & ~take;
        t.cand[m] &= ~(s[m] ^ take);
    }
    t.r1 = (int)(((uint32_t)t.r1 & take) | ((uint32_t)left & ~take));
}

// Byte `BYTE` of fp32 keys (3: the sign bit is skipped).  w[e] = the lane's element e.
template <int BYTE, int LPB, int NE, int NM>
__device__ __forceinline__ void select_byte(Select<NM>& t, const uint32_t (&w)[NE]) {
    uint32_t q[NM][8];
    constexpr uint32_t kPair = 0x0c0c0000u | ((4u + BYTE) << 8) | BYTE;   // {a.byte, b.byte, 0, 0}
#pragma unroll
    for (int m = 0; m < NM; ++m) {
#pragma unroll
        for (int g = 0; g < 8; ++g) {   // bytes of elements 32m + {g, 8+g, 16+g, 24+g}
            const int e = 32 * m + g;
            if (e >= NE) { q[m][g] = 0u; continue; }
            const uint32_t u = __builtin_amdgcn_perm(w[e + 8 < NE ? e + 8 : e], w[e], e + 8 < NE ? kPair : 0x0c0c0c00u | BYTE);
            uint32_t v = 0u;
            if (e + 16 < NE) v = __builtin_amdgcn_perm(w[e + 24 < NE ? e + 24 : e + 16], w[e + 16],
                                                       e + 24 < NE ? kPair : 0x0c0c0c00u | BYTE);
            q[m][g] = e + 16 < NE ? __builtin_amdgcn_perm(v, u, 0x05040100u) : u;
        }
        transpose8(q[m]);
    }
#pragma unroll
    for (int b = BYTE == 3 ? 6 : 7; b >= 0; --b) {
        uint32_t s[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) s[m] = q[m][b];
        select_bit<LPB, NM>(t, s);
    }
}

// Byte `BYTE` of binary16 keys (1: the sign bit is skipped).  w[i] = elements 2i, 2i+1.
template <int BYTE, int LPB, int NE, int NM, int NW>
__device__ __forceinline__ void select_byte16(Select<NM>& t, const uint32_t (&w)[NW]) {
    uint32_t q[NM][8];
    // {a.even, b.even, a.odd, b.odd}
    constexpr uint32_t kFour = ((6u + BYTE) << 24) | ((2u + BYTE) << 16) | ((4u + BYTE) << 8) | BYTE;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
#pragma unroll
        for (int g = 0; g < 8; g += 2) {
            const int i = 16 * m + g / 2;   // words of elements 32m + g + {0, 8, 16, 24}
            const uint32_t u = __builtin_amdgcn_perm(i + 4 < NW ? w[i + 4 < NW ? i + 4 : i] : 0u, w[i], kFour);
            uint32_t v = 0u;
            if (i + 8 < NW)
                v = __builtin_amdgcn_perm(i + 12 < NW ? w[i + 12 < NW ? i + 12 : i] : 0u, w[i + 8 < NW ? i + 8 : i], kFour);
            q[m][g] = __builtin_amdgcn_perm(v, u, 0x05040100u);
            q[m][g + 1] = __builtin_amdgcn_perm(v, u, 0x07060302u);
        }
        transpose8(q[m]);
    }
#pragma unroll
    for (int b = BYTE == 1 ? 6 : 7; b >= 0; --b) {
        uint32_t s[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) s[m] = q[m][b];
        select_bit<LPB, NM>(t, s);
    }
}

// every bank of the wavefront needs all of its remaining candidates
template <int LPB, int NM>
__device__ __forceinline__ bool settled(const Select<NM>& t) {
    int n = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) n += __popc(t.cand[m]);
    return __all(group_sum_i<LPB>(n) == t.r1 + 1);
}

// mask with the n lowest bits set (0 <= n <= 32)
__device__ __forceinline__ uint32_t low_bits(int n) { return n >= 32 ? 0xFFFFFFFFu : (1u << n) - 1u; }

// How a lane's elements lie in LDS.
//   kAligned   C elements, C*sizeof(VT) a power of two of 64 bytes or more: lanes would start
//              on the same LDS banks, so 16-byte piece p of a lane sits at p ^ (its 256-byte
//              window's number), which spreads 16 lanes over all LDS banks;
//   kWords     as in memory; elements start on 4-byte boundaries;
//   kHalves    as in memory; binary16 with an odd bank.
enum LaneLayout { kAligned, kWords, kHalves };

// The offsets that go out with the survivors: their positions in the bank or, re-pruning, the
// offsets that the packed matrix holds there.  Those are fetched by position where a wavefront
// keeps at most kFewOutputs (a lane's four together: one round trip); with more it would be several
// dependent round trips, and all stored offsets come to LDS while the keys are searched
// (2048 x 8192, 100 -> 90 of 256: 26.3 -> 17.8 us; where few are kept the copy costs up to 15 %:
// 4096 x 4096, 32 -> 2 of 64: 12.1 against 11.4 us).
enum Offsets { kPositions, kStored, kStoredInLds };
constexpr int kFewOutputs = 4 * kWave;

struct PruneArgs {
    const void* W;
    void* vals;
    void* idx;
    const void* remap;     // re-pruning: the stored offsets; else null
    int64_t n_banks;
    int B, k;
    int C;                 // elements per lane: LPB * C >= B, C <= NE
    uint32_t magic_k;      // magic_u32(k)
    int raw_bytes;         // LDS bytes of the wavefront's banks; its offsets follow
    int stored_at;         // kStoredInLds: where the stored offsets lie behind those
    int wave_bytes;        // all of them, a multiple of 256
    int streamed;          // W is larger than the last-level cache
};

// Wavefronts per workgroup at most; they share nothing.  1 / 2 / 4 on the 6000 x 3000 matrix:
// 18.6 / 18.5 / 16.9 us (11250 wavefronts of short life: fewer workgroups to dispatch).
constexpr int kPruneWaves = 4;

// n bytes from memory to LDS by one wavefront, P (4 or 16) at a time and the last ones singly;
// direct-to-LDS loads, so the caller waits.
template <int P>
__device__ __forceinline__ void copy_bytes(const unsigned char* src, unsigned char* dst, int n, int lane) {
    const int pieces = n / P;
    for (int p0 = 0; p0 < pieces; p0 += kWave)
        if (p0 + lane < pieces) {
            const auto from = (const __attribute__((address_space(1))) void*)(src + (size_t)(p0 + lane) * P);
            const auto to = (__attribute__((address_space(3))) void*)(dst + p0 * P);
            if constexpr (P == 16) __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
            else __builtin_amdgcn_global_load_lds(from, to, 4, 0, 0);
        }
    const int done = pieces * P;
    if (lane < n - done) dst[done + lane] = src[done + lane];
}

// The wavefront's banks to LDS: piece place(p) to place p.  POLICY: 0, or 2 for non-temporal loads.
template <int POLICY, typename F>
__device__ __forceinline__ void copy_places(const unsigned char* src, unsigned char* dst, int places, int pieces, int lane, F place) {
    for (int p0 = 0; p0 < places; p0 += kWave) {
        const int p = (int)place((uint32_t)(p0 + lane));
        if (p0 + lane < places && p < pieces)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(src + (size_t)p * 16),
                (__attribute__((address_space(3))) void*)(dst + p0 * 16), 16, 0, POLICY);
    }
}

// A group of 64/LPB banks per wavefront, no loop.
template <typename VT, typename IT, int LPB, int NE, LaneLayout LAYOUT, Offsets OFFSETS>
__global__ __launch_bounds__(kWave * kPruneWaves) void prune_pack_kernel(PruneArgs a) {
    constexpr int S = sizeof(VT);
    constexpr int NM = NE > 32 ? 2 : 1;           // mask words
    constexpr int NW = NE * S / 4;                // words of a lane's elements
    constexpr int BPW = kWave / LPB;              // banks per wavefront
    constexpr int PPL = NE * S / 16;              // kAligned: 16-byte pieces per lane
    static_assert(NE <= 64 && (NE % 16 == 0 || (NE == 4 && S == 4)), "lane shape");
    extern __shared__ __align__(256) unsigned char pp_shared[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    unsigned char* pp_lds = pp_shared + wave * a.wave_bytes;
    const int64_t grp = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (blockDim.x / kWave) + wave;
    const int64_t first = grp * BPW;
    if (first >= a.n_banks) return;
    const int n_ok = a.n_banks - first < BPW ? (int)(a.n_banks - first) : BPW;
    const int B = a.B, k = a.k;

    // ---- the banks -> LDS --------------------------------------------------
    // Where 16-byte piece p of the group sits, and (the same map) which piece sits at p.
    auto place = [](uint32_t p) -> uint32_t {
        if constexpr (LAYOUT == kAligned) return p ^ ((p >> 4) & (uint32_t)(PPL - 1));
        else return p;
    };
    const unsigned char* src = static_cast<const unsigned char*>(a.W) + first * B * S;
    const int bytes = n_ok * B * S;
    const int pieces = bytes >> 4;
    const int places = LAYOUT == kAligned ? (pieces + 15) & ~15 : pieces;
    // A matrix that the last-level cache (256 MB) cannot hold is read past it: 336 MB 72.3 -> 63.4 us (4.9 -> 5.6 TB/s), 537 MB
    // 117 -> 109; 206 MB used again 45.0 -> 52.4, so the line is the cache's size.
    if (a.streamed) copy_places<2>(src, pp_lds, places, pieces, lane, place);
    else copy_places<0>(src, pp_lds, places, pieces, lane, place);
    // the matrix's last group may end inside a 16-byte piece (never kAligned)
    const int rest = bytes & 15;
    if (lane * S < rest)
        *reinterpret_cast<VT*>(pp_lds + (bytes - rest) + lane * S) =
            *reinterpret_cast<const VT*>(src + (bytes - rest) + lane * S);
    // direct-to-LDS loads are not tracked by the compiler; only this wavefront reads them
    pin_order();
    wait_vm_and_lds<0>();
    pin_order();

    // ---- this lane's elements ----------------------------------------------
    const int q = lane % LPB, bank = lane / LPB;
    const int e0 = q * a.C;                                   // first element inside the bank
    const int n_mine = max(0, min(a.C, B - e0));
    uint32_t w[NW];
    if constexpr (LAYOUT == kAligned) {
        const uint32_t p0 = (uint32_t)lane * PPL, x = (p0 >> 4) & (PPL - 1);
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
            const uint4 t = *reinterpret_cast<const uint4*>(pp_lds + ((p0 + ((uint32_t)p ^ x)) << 4));
            w[4 * p] = t.x; w[4 * p + 1] = t.y; w[4 * p + 2] = t.z; w[4 * p + 3] = t.w;
        }
    } else {
        // past the lane's own elements this reads neighbours' (or bytes past the group, which
        // the launcher allocates): masked out below
        const unsigned char* mine = pp_lds + (bank * B + e0) * S;
        if constexpr (LAYOUT == kWords) {
#pragma unroll
            for (int i = 0; i < NW; ++i) w[i] = reinterpret_cast<const uint32_t*>(mine)[i];
        } else {
#pragma unroll
            for (int i = 0; i < NW; ++i)
                w[i] = (uint32_t)reinterpret_cast<const uint16_t*>(mine)[2 * i] |
                       ((uint32_t)reinterpret_cast<const uint16_t*>(mine)[2 * i + 1] << 16);
        }
    }

    // ---- the stored offsets -> LDS ----------------------------------------------
    const unsigned char* idx_src = static_cast<const unsigned char*>(a.remap) + first * B;
    unsigned char* stored = pp_lds + a.stored_at;
    if constexpr (OFFSETS == kStoredInLds) {
        static_assert(sizeof(IT) == 1 && BPW >= 8, "byte offsets, groups of 8 banks or more");
        pin_order();
        // pieces that every group starts on
        if (BPW % 16 == 0 || B % 2 == 0) copy_bytes<16>(idx_src, stored, n_ok * B, lane);
        else copy_bytes<4>(idx_src, stored, n_ok * B, lane);
        pin_order();
    }

    // ---- the k largest keys --------------------------------------------------
    Select<NM> t;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        t.cand[m] = low_bits(min(32, max(0, n_mine - 32 * m)));
        t.gt[m] = 0u;
    }
    t.r1 = k - 1;
    if constexpr (S == 4) {
        select_byte<3, LPB, NE, NM>(t, w);
        select_byte<2, LPB, NE, NM>(t, w);
        if (!settled<LPB, NM>(t)) {
            select_byte<1, LPB, NE, NM>(t, w);
            if (!settled<LPB, NM>(t)) select_byte<0, LPB, NE, NM>(t, w);
        }
    } else {
        select_byte16<1, LPB, NE, NM, NW>(t, w);
        if (!settled<LPB, NM>(t)) select_byte16<0, LPB, NE, NM, NW>(t, w);
    }
    // candidates beyond the r1 + 1 still needed are ties with the threshold: the lowest
    // offsets stay, i.e. the first lanes of the bank and each lane's lowest bits
    {
        int own = 0;
#pragma unroll
        for (int m = 0; m < NM; ++m) own += __popc(t.cand[m]);
        const int room = t.r1 + 1 - group_prefix_i<LPB>(own, q);   // ties this lane may keep
        if (__any(own > room)) {
            const int want = max(0, min(own, room));
            int left = want;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int here = __popc(t.cand[m]);
                if (left < here) {
                    // smallest n with `left` candidates among the n lowest bits
                    int n = 0;
#pragma unroll
                    for (int step = 16; step > 0; step >>= 1)
                        if (__popc(t.cand[m] & low_bits(n + step)) <= left) n += step;
                    t.cand[m] &= low_bits(n);
                    left = 0;
                } else {
                    left -= here;
                }
            }
        }
    }

    // ---- offsets of the survivors, in order ----------------------------------
    IT* out_i = reinterpret_cast<IT*>(pp_lds + a.raw_bytes);
    {
        int own = 0;
#pragma unroll
        for (int m = 0; m < NM; ++m) own += __popc(t.gt[m] | t.cand[m]);
        IT* dst = out_i + bank * k + group_prefix_i<LPB>(own, q);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            uint32_t keep = t.gt[m] | t.cand[m];
            while (keep) {
                *dst++ = (IT)(e0 + 32 * m + __builtin_ctz(keep));
                keep &= keep - 1u;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // ---- values and offsets out ------------------------------------------------
    auto value = [&](int slot, uint32_t off) -> VT {
        const uint32_t e = div_magic((uint32_t)slot, (uint32_t)k, a.magic_k) * (uint32_t)B + off;
        uint32_t at = e * S;
        if constexpr (LAYOUT == kAligned) at = (place(at >> 4) << 4) | (at & 15u);
        return *reinterpret_cast<const VT*>(pp_lds + at);
    };
    VT* vout = static_cast<VT*>(a.vals) + first * k;
    IT* iout = static_cast<IT*>(a.idx) + first * k;
    const int n_out = n_ok * k;
    // the offset that goes out for the survivor at position `off` of its bank
    auto offset = [&](int slot, uint32_t off) -> IT {
        if constexpr (OFFSETS == kPositions) return (IT)off;
        const uint32_t at = div_magic((uint32_t)slot, (uint32_t)k, a.magic_k) * (uint32_t)B + off;
        return OFFSETS == kStoredInLds ? stored[at] : idx_src[at];
    };
    if constexpr (OFFSETS == kStoredInLds) {   // the copies above are not tracked by the compiler
        pin_order();
        wait_vm_and_lds<0>();
        pin_order();
    }
    // four outputs per lane and step; a group starts on a multiple of four outputs unless
    // it holds two banks (LPB == 32), and only the matrix's last group may end elsewhere.
    // Offsets that are fetched by position: one per lane where that takes one step.
    int quads = LPB <= 16 || k % 2 == 0 ? n_out >> 2 : 0;
    if (OFFSETS == kStored && n_out <= kWave) quads = 0;
    using Quad = typename RawBytes<4 * S>::type;
    using IQuad = typename RawBytes<4 * sizeof(IT)>::type;
    for (int s = lane; s < quads; s += kWave) {
        IQuad o = reinterpret_cast<const IQuad*>(out_i)[s];
        VT v[4];
        IT out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t off = sizeof(IT) == 1 ? (word_of(o, 0) >> (8 * i)) & 0xffu
                                                 : (word_of(o, i >> 1) >> (16 * (i & 1))) & 0xffffu;
            v[i] = value(4 * s + i, off);
            if constexpr (OFFSETS != kPositions) out[i] = offset(4 * s + i, off);
        }
        if constexpr (OFFSETS != kPositions) __builtin_memcpy(&o, out, sizeof(o));
        Quad vq;
        __builtin_memcpy(&vq, v, sizeof(vq));
        reinterpret_cast<Quad*>(vout)[s] = vq;
        reinterpret_cast<IQuad*>(iout)[s] = o;
    }
    for (int s = 4 * quads + lane; s < n_out; s += kWave) {
        const uint32_t off = out_i[s];
        vout[s] = value(s, off);
        iout[s] = offset(s, off);
    }
}

template <typename VT, typename IT, int LPB, int NE, LaneLayout LAYOUT, Offsets OFFSETS>
int prune_launch_kernel(PruneArgs a, hipStream_t st) {
    constexpr int BPW = kWave / LPB, S = sizeof(VT);
    // the banks, and what the last lane's fixed-size read may reach past them
    a.raw_bytes = (BPW * a.B * S + (LAYOUT == kAligned ? 0 : (LPB * a.C - a.B + NE) * S) + 15) / 16 * 16;
    a.stored_at = (a.raw_bytes + BPW * a.k * (int)sizeof(IT) + 15) / 16 * 16;
    a.wave_bytes = (a.stored_at + (OFFSETS == kStoredInLds ? BPW * a.B : 0) + 255) / 256 * 256;
    int waves = kPruneWaves;
    while (waves * a.wave_bytes > 48 * 1024) waves >>= 1;   // at most 24.5 KB per wavefront
    const int64_t groups = (a.n_banks + BPW - 1) / BPW;
    const int64_t wgs = (groups + waves - 1) / waves;
    const int64_t gx = wgs < ((int64_t)1 << 20) ? wgs : ((int64_t)1 << 20);
    const int64_t gy = (wgs + gx - 1) / gx;
    if (gy > 65535) return BS_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((prune_pack_kernel<VT, IT, LPB, NE, LAYOUT, OFFSETS>), dim3((unsigned)gx, (unsigned)gy),
                       dim3(kWave * waves), (size_t)waves * a.wave_bytes, st, a);
    return hip_status(hipGetLastError());
}

template <typename VT, typename IT, int LPB, int NE, LaneLayout LAYOUT>
int prune_launch_one(const PruneArgs& a, hipStream_t st) {
    if constexpr (sizeof(IT) == 1) {
        if (a.remap && kWave / LPB * a.k <= kFewOutputs)
            return prune_launch_kernel<VT, IT, LPB, NE, LAYOUT, kStored>(a, st);
        if (a.remap) return prune_launch_kernel<VT, IT, LPB, NE, LAYOUT, kStoredInLds>(a, st);
    }
    return prune_launch_kernel<VT, IT, LPB, NE, LAYOUT, kPositions>(a, st);
}

template <typename VT, typename IT, int LPB, int NE>
int prune_launch_layout(const PruneArgs& a, hipStream_t st) {
    if constexpr (NE * sizeof(VT) >= 64)
        if (a.B == LPB * a.C && a.C == NE) return prune_launch_one<VT, IT, LPB, NE, kAligned>(a, st);
    if constexpr (sizeof(VT) == 2 && sizeof(IT) == 1)   // wide banks are whole 16-byte pieces
        if (a.B % 2 != 0) return prune_launch_one<VT, IT, LPB, NE, kHalves>(a, st);
    return prune_launch_one<VT, IT, LPB, NE, kWords>(a, st);
}

// W viewed as n_banks banks of `bank` elements, k kept per bank.  As few lanes per bank as 32
// elements per lane allow (one mask word): a select step costs a wavefront the same whatever
// its lanes hold, and up to 64 per lane would need a third fewer instructions, but the LDS a
// wavefront holds doubles and the wavefronts that are left hide less of the stream
// (one wavefront per workgroup:
// 19.5 against 18.4 us on the 6000 x 3000 matrix, 48.0 against 44.5 us on the binary16 one).  Banks over 1024 elements: 32 lanes of up to 64.
template <typename VT, typename IT>
int prune_banks(const void* W, int64_t n_banks, int bank, int k, void* vals, IT* idx,
                const IT* remap, hipStream_t st) {
    constexpr bool kWide = sizeof(IT) == 2;
    PruneArgs a;
    a.W = W; a.vals = vals; a.idx = idx; a.remap = remap;
    a.n_banks = n_banks; a.B = bank; a.k = k;
    a.magic_k = magic_u32((uint32_t)k);
    a.raw_bytes = a.stored_at = a.wave_bytes = 0;
    a.streamed = (double)n_banks * bank * sizeof(VT) > kLastLevelBytes;
    int lpb = 1;
    while (lpb < 32 && (bank + lpb - 1) / lpb > 32) lpb <<= 1;
    a.C = (bank + lpb - 1) / lpb;
    if (sizeof(VT) == 2 && lpb > 1) a.C = (a.C + 1) & ~1;   // binary16: a lane starts on a word
    if (a.C > 64) return BS_ERR_UNSUPPORTED;
    switch (lpb) {
        case 1:
            // up to four fp32: half the transpose of each byte is of zeros and goes (3627 x 1024,
            // 1 of 4, ties, so that all four bytes are looked at: 20.4 -> 16.7 us)
            if constexpr (sizeof(VT) == 4)
                if (a.C <= 4) return prune_launch_layout<VT, IT, 1, 4>(a, st);
            if (a.C <= 16) return prune_launch_layout<VT, IT, 1, 16>(a, st);
            return prune_launch_layout<VT, IT, 1, 32>(a, st);
        case 2: return prune_launch_layout<VT, IT, 2, 32>(a, st);
        case 4: return prune_launch_layout<VT, IT, 4, 32>(a, st);
        case 8: return prune_launch_layout<VT, IT, 8, 32>(a, st);
        case 16: if constexpr (kWide) return prune_launch_layout<VT, IT, 16, 32>(a, st); break;
        case 32:
            if constexpr (kWide) {
                if (a.C <= 32) return prune_launch_layout<VT, IT, 32, 32>(a, st);
                return prune_launch_layout<VT, IT, 32, 64>(a, st);
            }
    }
    return BS_ERR_UNSUPPORTED;
}

}  // namespace
}  // namespace bs
