// Y = W_sparse . X for products in which the gathers are most of the work (arXiv 1811.00206,
// Sec. 3.4 with a batch; im2col convolutions of Sec. 4.2).
//
// A workgroup owns a tile of 16 columns and a range of rows of W and walks K (or a slab of it)
// in stages: some wavefronts copy the next stage's rows of X into one half of LDS while the
// others walk their rows of W against the other half; one barrier per stage.  With K walked
// inside the workgroup there is usually one slab, so no partial sums pass through memory and
// no second kernel adds them.
//
// As in the paper a thread owns a bank, and rows of X lie in LDS so that its threads never meet
// in an LDS bank: see SpmmStream layout below.  What bounds it, counted per entry and 16 columns
// of a wavefront: 4 reads of 1 KB (LDS: 1.9 ns each for the compute unit when nothing collides,
// measured), 16 multiply-adds (1.05 ns of a SIMD each), 1 dot product for the address (1.8 ns) and
// 3 exclusive ors (1 ns each): LDS 7.6 ns against 5.4 ns of vector instructions per compute unit;
// measured 11 ns with 12 wavefronts.  On the way here, 6000 x 3000 at 90 % and N = 128 (main kernel):
//   one lane per row and 4 columns, quads sharing the weights by DPP (the tile kernels)  23.6 us
//   the same walk in stages, addresses by one dot product                               21.3
//   8 columns per lane, banks side by side (no collisions, but DPP at 1.8 ns per value)  21.7
//   a bank per lane, 16 columns (no value passes between lanes)                           18.5
//   the first stage copied by all wavefronts, whole words only in the weights' ring       17.4
// Beside them the weights: a lane reads its own bank, so a load instruction makes about three accesses of
// 64 bytes per four lanes, 240 per 64 banks of 10, and the address unit is busy 24 of 36 thousand cycles (N = 128).
// The accumulators of columns 2i and 2i+1 are kept in each other's place: a multiply-add whose
// addend and X operand are both in even or both in odd registers takes 1.4 ns instead of 1.
// Tried and not kept: more than 14 walking wavefronts (the copies fall behind), the gathers of
// a unit's first entries issued before the last multiply-adds of the unit before (spills), 32 columns per lane (half
// the weights' accesses, but three to six wavefronts then walk: 25.9 us against 19.5), offsets in one load that
// reaches back into the bank before (18.1 us against 17.9).
#pragma once
#include "bs_spmm_kernel.h"

namespace bs {

// SpmmStream layout.  A tile is 16 columns of X: four pieces of 16 bytes.  In LDS the same row of four banks lies side by
// side in 256 bytes, the width of the 64 LDS banks.  A lane owns one bank of a row of W and reads the four pieces
// of an entry's row of X; of 16 neighbouring lanes, four work on different banks and four on different
// rows of W, which start at different pieces: every read touches each LDS bank once, whatever
// the offsets.
constexpr int kStreamPieces = 4, kStreamColumns = 4 * kStreamPieces;
constexpr int kStreamBanks = 16 / kStreamPieces;         // banks side by side = lanes per row of W
constexpr int kStreamRows = kWave / kStreamBanks;        // rows of W per wavefront
constexpr int kStreamPitch = 256;
constexpr int kStreamMinK = 4;    // the fewest entries per bank (a word of byte offsets)
constexpr int kStreamMaxK = 16;   // up to here the kernel knows k at compile time
// entries of a bank that a lane loads at once
constexpr int stream_unit(int kc) { return kc > 0 ? kc : -kc; }

struct SpmmStreamArgs {
    const void* vals;
    const void* idx;
    const float* X;
    float* out;            // Y (one slab) or the workspace [n_slabs][M][N]
    int64_t ldx;
    int64_t ld_out;        // ldy, or N for the workspace
    int64_t slab_stride;   // M*N for the workspace, 0 for Y
    int M, K, B, k, N;
    int nb;
    int n_tiles;           // tiles of 16 columns
    int slab_banks, n_slabs;   // banks of K per workgroup
    int sb;                // banks per stage
    int n_bufs;            // halves of LDS: 2, or 1 where only one stage's tile fits
    int buf_bytes;
    int rows_per_wg, row_groups;
    int ksplit, row_waves; // wavefronts that walk rows: ksplit groups of row_waves
    int rounds;            // units per bank
    int last;              // entries of a bank's last unit
    int tiles_fast;        // consecutive workgroups share the row group (else the column tile)
    int total_wgs, wgs_per_xcd;
    uint32_t magic_inner, magic_slab;   // magic_u32 of the faster index's count, of tiles * row groups
    uint32_t magic_sb, magic_rw;
    int by_registers;      // X is copied through registers: rows that start at any multiple of 4 bytes, or lie so far
                           // apart that four banks of them span 2 GB
    int vec_out;
};

struct SpmmStreamPlan {
    bool ok;
    int n_tiles, slab_banks, n_slabs, sb, n_bufs, buf_bytes;
    int rows_per_wg, row_groups, ksplit, row_waves, copy_waves;
    size_t lds_bytes;
    double ns;                               // expected time, the slab sums included
};
// The rounding error of a sum, as its variance over that of its terms' own rounding when all terms are of one size: an
// addition rounds its result, so it counts as many times as the result has terms, over the number of terms
// of the whole sum.  Of `n` terms (or sums of equally many terms each, exact themselves) added one after the other:
inline double chain_rounding(double n, bool terms) { return (n + 1) / 2 - (terms ? 0 : 1 / n); }
enum SpmmFit { kFirstFit, kSecondFit };          // whose factors an expected time is made of
// The best launch for a shape (of any row pitch of X: a product's sums are in the same order whatever the
// pitch), with at most max_slabs slabs (looked for from min_slabs on), max_lds bytes of LDS and sums whose rounding is at most max_rounding,
// expected to take less than max_ns; ok = false where there is none or the kernels do not apply.
SpmmStreamPlan spmm_stream_plan(SpmmFit fit, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, int min_slabs, int max_slabs,
                                int max_lds, double max_rounding, double max_ns);
double spmm_stream_rounding(const SpmmStreamPlan& p, int nb, int k);
double spmm_stream_ns(const SpmmStreamPlan& p, SpmmFit fit, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N);
// t: the operands as for the tile kernels, out and slab_stride for p's number of slabs
int spmm_stream_launch(const SpmmStreamPlan& p, const SpmmArgs& t, int dtype, int isize, hipStream_t st);
int spmm_stream_launch_f32(const SpmmStreamArgs& a, const SpmmLaunch& l);
int spmm_stream_launch_f16(const SpmmStreamArgs& a, const SpmmLaunch& l);
int spmm_stream_launch_wide(int dtype, const SpmmStreamArgs& a, const SpmmLaunch& l);

#ifdef __HIPCC__

typedef __attribute__((address_space(3))) const char* LdsBytes;
typedef __attribute__((address_space(3))) const SpmmAcc LdsFour;

// Words at the address of any entry.
template <int N, int ALIGN>
struct __attribute__((packed, aligned(ALIGN))) WordsAt { uint32_t w[N]; };

// N consecutive values or offsets (at least four bytes) in words.  The last word ends with the last
// entry, so with a remainder it repeats bytes of the word before: loads of less than a word
// would be widened at the end of the loop that carries them, which waits for them.
template <typename T, int N>
struct EntryWords {
    static constexpr int kBytes = (int)sizeof(T) * N, kWhole = kBytes / 4, kWords = (kBytes + 3) / 4;
    static_assert(kWhole > 0, "at least one word");
    uint32_t w[kWords];
    __device__ __forceinline__ void load(const char* p) {
        const auto whole = *reinterpret_cast<const WordsAt<kWhole, sizeof(T)>*>(p);
#pragma unroll
        for (int i = 0; i < kWhole; ++i) w[i] = whole.w[i];
        if constexpr (kWords > kWhole) w[kWhole] = reinterpret_cast<const WordsAt<1, sizeof(T)>*>(p + kBytes - 4)->w[0];
    }
    static constexpr int word(int i) { return i * (int)sizeof(T) / 4; }
    // place of entry i inside its word, in entries
    static constexpr int place(int i) {
        return word(i) < kWhole ? i % (4 / (int)sizeof(T)) : i - (N - 4 / (int)sizeof(T));
    }
};

// LDS operations of this wavefront are finished (its direct-to-LDS loads are not among them)
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// One stage's banks of X (`banks` from bank `bank0`; columns n0 .. n0+16) to LDS, by the `waves`
// copying wavefronts: four LDS rows at a time.
__device__ __forceinline__ void spmm_stream_copy(const SpmmStreamArgs& a, char* dst, int bank0, int banks, int n0, int ntw,
                                                 int wave, int waves, int lane) {
    constexpr int P = kStreamPieces, kBanks = kStreamBanks;
    const int B = a.B;
    const int p = (lane & 15) / P, c = lane & (P - 1), lrow = lane >> 4;
    const int groups = (banks + kBanks - 1) / kBanks, spare = groups * kBanks - banks;
    const int quads = (B + 3) >> 2;              // of rows, per group of banks
    // Rows of X are read in pieces of 16 bytes, which may reach up to 12 bytes past a row's last
    // column: into the next row, but not past the last row of X, which is brought in by itself.
    const bool ragged_end = bank0 + banks == a.nb && (ntw & 3);
    const uint32_t lane_off = ((uint32_t)(p * B + lrow) * (uint32_t)a.ldx + (uint32_t)min(c * 4, (ntw - 1) & ~3)) * 4u;   // below 2 GB, or not used
    const char* X0 = reinterpret_cast<const char*>(a.X + (size_t)bank0 * B * a.ldx + n0);
    const size_t group_step = (size_t)kBanks * B * a.ldx * 4, quad_step = (size_t)4 * a.ldx * 4;
    // rows of this lane's bank in the last group: none if there is no such bank
    const int last_rows = p >= kBanks - spare ? 0 : ragged_end && p == kBanks - spare - 1 ? B - 1 : B;
    int g = 0, rq = wave;
    while (rq >= quads) { rq -= quads; ++g; }
    if (!a.by_registers) {
        while (g < groups) {
            const int r = rq * 4 + lrow;
            if (r < (g == groups - 1 ? last_rows : B))
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(X0 + g * group_step + rq * quad_step + lane_off),
                    (__attribute__((address_space(3))) void*)(dst + (size_t)(g * B + rq * 4) * kStreamPitch), 16, 0, 0);
            rq += waves;
            while (rq >= quads) { rq -= quads; ++g; }
        }
    } else {
        // Eight loads are in flight before the first LDS store.  Lanes without a row read one that
        // is there: no branch comes between the loads.
        constexpr int kBatch = 8;
        using Four = WordsAt<4, 4>;
        // not `lane_off` itself in 64 bits: fc6 at N = 16, which is copied the other way, then takes 18.78 us instead of 18.65
        const size_t far_off = ((size_t)(p * B + lrow) * (size_t)a.ldx + (size_t)min(c * 4, (ntw - 1) & ~3)) * 4u;
        while (g < groups) {
            Four t[kBatch];
            int at[kBatch];                      // LDS row of each piece, or -1
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int r = rq * 4 + lrow, end = g < groups ? g == groups - 1 ? last_rows : B : 0;
                at[u] = r < end ? g * B + r : -1;
                t[u] = *reinterpret_cast<const Four*>(r < end ? X0 + g * group_step + rq * quad_step + far_off : X0);
                rq += waves;
                while (rq >= quads) { rq -= quads; ++g; }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (at[u] >= 0)
                    *reinterpret_cast<uint4*>(dst + at[u] * kStreamPitch + (lane & 15) * 16) = make_uint4(t[u].w[0], t[u].w[1], t[u].w[2], t[u].w[3]);
        }
    }
    if (ragged_end && wave == 0 && lane < 4 * P) {
        const int j = banks - 1;
        const float x = a.X[(size_t)(a.K - 1) * a.ldx + n0 + min(lane, ntw - 1)];
        *reinterpret_cast<float*>(dst + (size_t)((j / kBanks) * B + B - 1) * kStreamPitch + (j % kBanks) * (16 * P) + lane * 4) = x;
    }
}

// A lane's offsets as pairs of 16 bits, the operands of a two-way dot product with (256, 0) or
// (0, 256): LDS address = base + offset * 256 in one instruction.
template <typename IT, int U>
struct StreamOffsets {
    using Words = EntryWords<IT, U>;
    uint32_t w[Words::kWords * (sizeof(IT) == 1 ? 2 : 1)];
    __device__ __forceinline__ explicit StreamOffsets(const Words& o) {
#pragma unroll
        for (int i = 0; i < Words::kWords; ++i) {
            if constexpr (sizeof(IT) == 1) {
                w[2 * i] = o.w[i] & 0x00ff00ffu;
                w[2 * i + 1] = (o.w[i] >> 8) & 0x00ff00ffu;
            } else {
                w[i] = o.w[i];
            }
        }
    }
    __device__ __forceinline__ uint32_t address(int i, uint32_t base) const {
        typedef unsigned short U2 __attribute__((ext_vector_type(2)));
        const int at = Words::place(i);
        const int word = sizeof(IT) == 1 ? Words::word(i) * 2 + (at & 1) : Words::word(i), half = sizeof(IT) == 1 ? at >> 1 : at;
        return __builtin_amdgcn_udot2(__builtin_bit_cast(U2, w[word]), __builtin_bit_cast(U2, (uint32_t)kStreamPitch << (16 * half)), base, false);
    }
};

template <typename VT, int U>
__device__ __forceinline__ float stream_value(const EntryWords<VT, U>& v, int i) {
    using Words = EntryWords<VT, U>;
    const uint32_t word = v.w[Words::word(i)];
    if constexpr (sizeof(VT) == 4) return __builtin_bit_cast(float, word);
    else return __half2float(__builtin_bit_cast(__half, (uint16_t)(Words::place(i) ? word >> 16 : word & 0xffffu)));
}

// Entries E0 .. U-1 of the unit, the gathers of D entries ahead of the multiply-adds (left to itself
// the compiler waits for each gather by itself).
__device__ __forceinline__ void spmm_stream_gather(uint32_t at, SpmmAcc (&x)[kStreamPieces]) {
#pragma unroll
    for (int j = 0; j < kStreamPieces; ++j) x[j] = *reinterpret_cast<LdsFour*>(at ^ (16u * j));
}
template <typename VT, typename IT, int U, int D, int E0>
__device__ __forceinline__ void spmm_stream_walk(uint32_t base, const EntryWords<VT, U>& v, const StreamOffsets<IT, U>& o, SpmmAcc (&acc)[kStreamPieces]) {
    SpmmAcc x[D][kStreamPieces];
#pragma unroll
    for (int e = E0; e < E0 + D && e < U; ++e) spmm_stream_gather(o.address(e, base), x[(e - E0) % D]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = E0; e < U; ++e) {
        const float w = stream_value<VT, U>(v, e);
        uint32_t at = 0;
        if (e + D < U) at = o.address(e + D, base);   // its result cannot be used at once
#pragma unroll
        for (int j = 0; j < kStreamPieces; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[j][i ^ 1] = fmaf(w, x[(e - E0) % D][j][i], acc[j][i ^ 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (e + D < U) {
            spmm_stream_gather(at, x[(e - E0) % D]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}
// ... of which the last n (1 .. U) count: known only at run time, the same for every lane
template <typename VT, typename IT, int U, int D, int LO, int HI>
__device__ __forceinline__ void spmm_stream_walk_n(uint32_t base, const EntryWords<VT, U>& v, const StreamOffsets<IT, U>& o, int n, SpmmAcc (&acc)[kStreamPieces]) {
    if constexpr (LO == HI) {
        spmm_stream_walk<VT, IT, U, D, U - LO>(base, v, o, acc);
    } else {
        constexpr int kMid = (LO + HI + 1) / 2;
        if (n >= kMid) spmm_stream_walk_n<VT, IT, U, D, kMid, HI>(base, v, o, n, acc);
        else spmm_stream_walk_n<VT, IT, U, D, LO, kMid - 1>(base, v, o, n, acc);
    }
}

// KC = k, or -U for any k >= U, walked in units of U entries.
template <typename VT, typename IT, int KC>
__global__ __launch_bounds__(1024) void spmm_stream_kernel(SpmmStreamArgs a) {
    extern __shared__ __align__(16) char Xs[];
    constexpr int U = stream_unit(KC), P = kStreamPieces, kBanks = kStreamBanks;
    constexpr int kRing = U > 4 ? 2 : 4;         // units in flight per lane
    constexpr int kAhead = U * sizeof(VT) > 48 || KC < 0 ? 2 : 3;   // gathered entries in flight
    using VR = EntryWords<VT, U>;
    using IR = EntryWords<IT, U>;

    const int bid = blockIdx.x;
    const int wg = (bid % kXcds) * a.wgs_per_xcd + bid / kXcds;
    if (wg >= a.total_wgs) return;
    const int inner = a.tiles_fast ? a.n_tiles : a.row_groups, outer = a.tiles_fast ? a.row_groups : a.n_tiles;
    const int s = (int)div_magic_any((uint32_t)wg, (uint32_t)(inner * outer), a.magic_slab);
    const int in_slab = wg - s * inner * outer;
    const int wo = (int)div_magic_any((uint32_t)in_slab, (uint32_t)inner, a.magic_inner);
    const int wi = in_slab - wo * inner;
    const int z = a.tiles_fast ? wi : wo, g = a.tiles_fast ? wo : wi;

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n0 = z * kStreamColumns, ntw = min(kStreamColumns, a.N - n0);
    const int bank0 = s * a.slab_banks, banks = min(a.slab_banks, a.nb - bank0);
    const int stages = (int)div_magic((uint32_t)(banks + a.sb - 1), (uint32_t)a.sb, a.magic_sb);
    const int row_waves = a.row_waves;
    const int walkers = a.ksplit * row_waves;

    const int kq = (int)div_magic((uint32_t)wave, (uint32_t)row_waves, a.magic_rw);
    const int wr = wave - kq * row_waves;
    const int p = lane & (kBanks - 1), turn = (lane & 15) / kBanks;   // bank of a group; which piece comes first
    const int r0 = g * a.rows_per_wg, r_end = min(a.M, r0 + a.rows_per_wg);
    const int row = r0 + wr * kStreamRows + (lane >> 4) * P + turn;
    const int k = KC > 0 ? KC : a.k;
    const int groups = (banks + kBanks - 1) / kBanks, spare = groups * kBanks - banks;
    const char* vbase = static_cast<const char*>(a.vals) + ((size_t)r0 * a.nb + bank0) * k * sizeof(VT);
    const char* ibase = static_cast<const char*>(a.idx) + ((size_t)r0 * a.nb + bank0) * k * sizeof(IT);
    const uint32_t lane_e = (uint32_t)((min(row, r_end - 1) - r0) * a.nb + p) * (uint32_t)k;
    // a lane without a bank in the last group re-reads one that is there, and adds nothing
    const uint32_t lane_e_last = lane_e - (uint32_t)((p >= kBanks - spare ? p - (kBanks - spare - 1) : 0) * k);

    VR vr[kRing];
    IR ir[kRing];
    int ld_g = kq, ld_r = 0;
    auto issue = [&](VR& v, IR& o) {
        const int lg = min(ld_g, groups - 1);
        const uint32_t at = (uint32_t)(lg * kBanks * k) + (KC > 0 ? 0u : (uint32_t)min(ld_r * U, k - U));
        const uint32_t e = lg == groups - 1 ? lane_e_last : lane_e;
        v.load(vbase + (size_t)at * sizeof(VT) + (uint32_t)(e * (uint32_t)sizeof(VT)));
        o.load(ibase + (size_t)at * sizeof(IT) + (uint32_t)(e * (uint32_t)sizeof(IT)));
        if (KC > 0 || ++ld_r == a.rounds) { ld_r = 0; ld_g += a.ksplit; }
    };
    // the first stage's tile by all wavefronts, behind the first weights
    if (wave < walkers) {
#pragma unroll
        for (int u = 0; u < kRing; ++u) issue(vr[u], ir[u]);
    }
    pin_order();
    spmm_stream_copy(a, Xs, bank0, min(a.sb, banks), n0, ntw, wave, (int)(blockDim.x >> 6), lane);
    pin_order();
    wait_vm_and_lds<0>();
    __builtin_amdgcn_s_barrier();
    pin_order();
    if (wave >= walkers) {
        for (int st = 1; st < stages; ++st) {
            if (a.n_bufs == 1) __builtin_amdgcn_s_barrier();
            const int b0 = st * a.sb;
            spmm_stream_copy(a, Xs + (a.n_bufs == 2 && (st & 1) ? a.buf_bytes : 0), bank0 + b0, min(a.sb, banks - b0), n0, ntw,
                                wave - walkers, (int)(blockDim.x >> 6) - walkers, lane);
            pin_order();
            wait_vm_and_lds<0>();
            pin_order();
            __builtin_amdgcn_s_barrier();
        }
        return;
    }

    SpmmAcc acc[P] = {}, tot[P] = {};
    const int stage_groups = a.sb / kBanks;      // where there is more than one stage
    int gi = kq, r = 0, st = 0, stage_g0 = 0, stage_end = stages > 1 ? stage_groups : groups;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsBytes)Xs + (uint32_t)(p * 16 * P + turn * 16);
    const uint32_t group_bytes = (uint32_t)(a.B * kStreamPitch);
    uint32_t buf = 0;
    auto next_stage = [&]() {
        ++st;
        wait_lds();
        __builtin_amdgcn_s_barrier();
        if (a.n_bufs == 1) __builtin_amdgcn_s_barrier();
        stage_g0 = stage_end;
        stage_end = min(stage_end + stage_groups, groups);
        buf = a.n_bufs == 2 && (st & 1) ? (uint32_t)a.buf_bytes : 0u;
    };
    while (gi < groups) {
#pragma unroll
        for (int u = 0; u < kRing; ++u) {
            if (gi < groups) {
                if (gi >= stage_end) {           // every stage but the last holds a unit of every wavefront
#pragma unroll
                    for (int j = 0; j < P; ++j) { tot[j] += acc[j]; acc[j] = SpmmAcc{0.f, 0.f, 0.f, 0.f}; }
                    pin_order();
                    next_stage();
                    pin_order();
                }
                const StreamOffsets<IT, U> o(ir[u]);
                const uint32_t base = lds0 + (buf + (uint32_t)(gi - stage_g0) * group_bytes);
                if (gi < groups - 1 || p < kBanks - spare) {
                    if (KC > 0 || r + 1 < a.rounds) spmm_stream_walk<VT, IT, U, kAhead, 0>(base, vr[u], o, acc);
                    else if constexpr (KC <= 0) spmm_stream_walk_n<VT, IT, U, kAhead, 1, U>(base, vr[u], o, a.last, acc);
                }
            }
            pin_order();
            issue(vr[u], ir[u]);
            pin_order();
            if (KC > 0 || ++r == a.rounds) { r = 0; gi += a.ksplit; }
        }
    }
#pragma unroll
    for (int j = 0; j < P; ++j) tot[j] += acc[j];
    while (st + 1 < stages) next_stage();

    // the sums of a row's four lanes, then one piece per lane
    static_assert(P == kBanks, "as many pieces as lanes of a row");
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[j][i] = group_sum<kBanks>(tot[j][i]);
    SpmmAcc t = tot[0];
#pragma unroll
    for (int j = 1; j < P; ++j)
        if (j == p) t = tot[j];
    SpmmAcc mine = {t[1], t[0], t[3], t[2]};
    if (a.ksplit > 1) {
        SpmmAcc* part = reinterpret_cast<SpmmAcc*>(Xs);
        const int at = wr * kWave + lane, per = row_waves * kWave;
        pin_order();
        wait_lds();
        __builtin_amdgcn_s_barrier();
        pin_order();
        if (kq > 0) part[(kq - 1) * per + at] = mine;
        pin_order();
        wait_lds();
        __builtin_amdgcn_s_barrier();
        pin_order();
        if (kq > 0) return;
        for (int o = 0; o + 1 < a.ksplit; ++o) mine += part[o * per + at];
    }
    if (row < r_end) {
        float* dst = a.out + (size_t)s * a.slab_stride + (size_t)row * a.ld_out + n0;
        const int c = (p ^ turn) * 4;
        if (a.vec_out && c + 4 <= ntw) {
            *reinterpret_cast<SpmmAcc*>(dst + c) = mine;
        } else {
#pragma unroll
            for (int n = 0; n < 4; ++n)
                if (c + n < ntw) dst[c + n] = mine[n];
        }
    }
}

template <typename VT, typename IT, int KC>
int spmm_stream_launch_one(const SpmmStreamArgs& a, const SpmmLaunch& l) {
    constexpr auto kern = spmm_stream_kernel<VT, IT, KC>;
    if (l.lds > kLdsWithoutLimit) {
        const int st_code = ensure_lds_limit(LdsKernelOf<kern, kStageGroup<VT, IT>>::reg, l.st);
        if (st_code != BS_OK) return st_code;
    }
    hipLaunchKernelGGL(kern, dim3(a.wgs_per_xcd * kXcds), dim3(l.threads), l.lds, l.st, a);
    return hip_status(hipGetLastError());
}

template <typename VT, typename IT, int KC = kStreamMaxK>
int spmm_stream_launch_k(const SpmmStreamArgs& a, const SpmmLaunch& l) {
    if constexpr (KC == kStreamMaxK) {
        if (a.k > KC) return spmm_stream_launch_one<VT, IT, -8>(a, l);
    }
    if (a.k == KC) return spmm_stream_launch_one<VT, IT, KC>(a, l);
    if constexpr (KC > kStreamMinK) return spmm_stream_launch_k<VT, IT, KC - 1>(a, l);
    return BS_ERR_UNSUPPORTED;
}

#endif  // __HIPCC__
}  // namespace bs
