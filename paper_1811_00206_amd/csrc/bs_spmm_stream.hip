// Host side of the SpMM kernels that walk K in stages (bs_spmm_stream_kernel.h): the launch and what it
// is expected to take.
#include <algorithm>
#include <cmath>

#include "bs_spmm_stream_kernel.h"

namespace bs {
namespace {

constexpr int kCus = 256, kWavesPerCu = 16;  // wavefronts: by the kernels' registers
constexpr int kMaxWalkers = 14;
constexpr double kStagesWorth = 1.02;         // of the best launch's time: more than that shorter stages hardly take off

template <typename I>
constexpr I div_up(I a, I b) { return (a + b - 1) / b; }

// entries of a bank that a lane loads at once (the kernel's U)
int unit_of(int isize, int k) { return isize == 2 ? (k < 8 ? 4 : 8) : k > kStreamMaxK ? 8 : k; }

// Expected time of a launch in ns.  The terms are the kernel's own steps; their factors are fits to timed launches on
// MI355X.  kFirst: 1332 launches of random shapes and plans, operands repeated, both offset widths (median error 6 %, 11 %
// rms).  kSecond: 19233 launches of 11000 random products with 8-bit offsets whose operands change from call to call (5 %, 8 %;
// without the term of a SIMD 10 %).  Wavefront w of a workgroup runs on SIMD w % 4 and a stage waits for the busiest
// of the four, so 5 walking wavefronts take as long as 8.  Which of them says what: stream_choice in bs_spmm.hip.
struct Factors {
    double alone, shared, simd;      // of an entry: a wavefront by itself, each that shares the compute unit, a SIMD
    double slow;                     // factor of an entry above k = kStreamMaxK and with 16-bit offsets
    double launch, round, first_copy, unit;
    double wave_copy, cu_copy;       // bytes per ns that a wavefront, a compute unit copies
    double by_registers;             // of the bytes that no direct copy moves
    double not_overlapped;           // of the shorter of a stage's walk and the next one's copy
    double slabs, slab_rate;         // of the sum over slabs: ns, bytes per ns
    double memory, memory_rate;      // passing all operands once
    double beside;                   // of the shorter of that and of the workgroups' own time
};
constexpr Factors kFirst{66.0, 13.7, 0, 1.24, 1670, 1800, 874, 29, 15.7, 82.0, 1.57, 0, 2700, 3750, 3000, 3835, 0};
constexpr Factors kSecond{50.7, 10.9, 35.4, 1.36, 1810, 2190, 662, 31, 15.7, 59.9, 1.55, 0.43, 2600, 4550, 0, 3506, 0.08};

struct Expectation {
    const Factors& f;
    double slow, memory, slab;   // factor of an entry; what passing all operands once takes; the slab sums, per slab
    double least;                // what every launch takes: its fixed times and the walk of all entries, spread over the chip
    double group;                // bytes of a group of banks, weighted by the way it is copied
    int k;

    Expectation(SpmmFit fit, int vsize, int isize, int64_t M, int64_t K, int bank, int k_, int64_t N, int64_t n_tiles)
        : f(fit == kFirstFit ? kFirst : kSecond), k(k_) {
        const double w_bytes = (double)M * (K / bank) * k * (vsize + isize), y_bytes = 4.0 * M * N;
        slow = isize == 2 || k > kStreamMaxK ? f.slow : 1.0;
        memory = f.memory + (w_bytes * std::min<int64_t>(n_tiles, 2) + 4.0 * K * N + y_bytes) / f.memory_rate;
        slab = 2.0 * y_bytes / f.slab_rate;
        const double entries = (double)div_up(M, (int64_t)kStreamRows) * n_tiles * div_up(K / bank, (int64_t)kStreamBanks) * k;
        least = std::max(memory, f.launch + f.round + f.first_copy + entries * slow * std::max(f.shared, f.simd * 0.25) / kCus);
        group = (double)bank * kStreamPitch * (N % 4 == 0 ? 1.0 : f.by_registers);   // as in the usual X, whose rows are adjacent
    }
    double slabs(int n) const { return n > 1 ? f.slabs + n * slab : 0.0; }
    // No launch of so many slabs takes less, ...
    double at_least(int n_slabs) const { return least + slabs(n_slabs); }
    // ... nor one of so many wavefronts side by side (as many entries and copies in all, whatever ks), ...
    double at_least(int n_slabs, int slab_groups, int row_waves, double rounds, double per_cu) const {
        const double walk = slab_groups * k * slow * row_waves * std::max({f.alone / kMaxWalkers, f.shared * per_cu, f.simd * per_cu * 0.25});
        return total(n_slabs, rounds, std::max(walk, slab_groups * group * per_cu * (1.0 / f.cu_copy)));
    }
    // ... nor with ks groups of those and so many groups of banks in the first stage.
    double at_least(int n_slabs, int slab_groups, int row_waves, double rounds, double per_cu, int ks, int first) const {
        const double unit = k * slow * std::max({f.alone, f.shared * ks * row_waves * per_cu, f.simd * (int)(ks * row_waves * per_cu * 0.25 + 0.9999)}) + f.unit;
        return total(n_slabs, rounds, first * group * per_cu * (1.0 / f.cu_copy) + div_up(slab_groups, ks) * unit);
    }
    double total(int n_slabs, double rounds, double ns) const { return f.launch + rounds * (f.round + f.first_copy + ns) + slabs(n_slabs); }
    double operator()(const SpmmStreamPlan& p, int slab_groups, int wgs) const {
        const int walkers = p.ksplit * p.row_waves, waves = walkers + p.copy_waves, sg = p.sb / kStreamBanks, stages = div_up(slab_groups, sg);
        const int per_cu = std::max(1, std::min({kMaxLdsBytes / (int)p.lds_bytes, kWavesPerCu / waves, div_up(wgs, kCus)}));
        const double entry = std::max({f.alone, f.shared * walkers * per_cu, f.simd * div_up(walkers * per_cu, 4)}) * slow;
        const double unit = k * entry + f.unit * std::max(1.0, walkers * per_cu / 4.0);
        const double walk = div_up(std::min(sg, slab_groups), p.ksplit) * unit;
        const double first = f.first_copy + std::min(sg, slab_groups) * group * per_cu / std::min(f.wave_copy * waves * per_cu, f.cu_copy);
        double t = first + walk;
        if (stages > 1) {
            const double tail = div_up(slab_groups - (stages - 1) * sg, p.ksplit) * unit;
            const double copy = f.first_copy + sg * group * per_cu / std::min(f.wave_copy * p.copy_waves * per_cu, f.cu_copy);
            t = first + tail + (stages - 1) * (p.n_bufs == 2 ? std::max(walk, copy) + f.not_overlapped * std::min(walk, copy) : walk + copy);
        }
        t = f.launch + div_up(wgs, kCus * per_cu) * (t + f.round);
        return std::max(t, memory) + f.beside * std::min(t, memory) + slabs(p.n_slabs);
    }
};

// A lane adds its banks' entries of a stage, then the stages; then come the banks side by side, the wavefronts
// along K and the slabs.
double rounding(const SpmmStreamPlan& p, int slab_groups, int k) {
    const int sg = p.sb / kStreamBanks;
    return chain_rounding((double)k * div_up(std::min(sg, slab_groups), p.ksplit), true) + chain_rounding(div_up(slab_groups, sg), false) +
           std::log2(kStreamBanks) + chain_rounding(p.ksplit, false) + chain_rounding(p.n_slabs, false);
}

}  // namespace

// As rounding(), with the stages, slabs and lanes that are not full counted as what they are.
double spmm_stream_rounding(const SpmmStreamPlan& p, int nb, int k) {
    const int sg = p.sb / kStreamBanks, ks = p.ksplit;
    auto sums = [&](double n) { return (n - 1) * (n + 2) / 2; };               // 2 + 3 + ... + n
    auto stage = [&](int groups) {                                             // of its terms, in ks wavefronts
        const int n = groups / ks, longer = groups % ks;
        auto chain = [&](double terms) { return terms * (terms + 1) / 2; };
        return kStreamBanks * (longer * chain((double)(n + 1) * k) + (ks - longer) * chain((double)n * k));
    };
    auto slab = [&](int groups) {                                              // its stages, and those added
        const int full = std::max(groups - 1, 0) / sg;
        return full * stage(std::min(sg, groups)) + stage(groups - full * sg) + (full > 0 ? (double)kStreamBanks * k * (sg * sums(full) + groups) : 0.0);
    };
    const int rest = nb - (p.n_slabs - 1) * p.slab_banks, last = div_up(rest, kStreamBanks);
    const double spare = last - rest * (1.0 / kStreamBanks);                    // share of the lanes that the last group leaves out
    double all = (p.n_slabs - 1) * slab(p.slab_banks / kStreamBanks) + (1 - spare) * slab(last) + spare * slab(last - 1);
    if (p.n_slabs > 1) all += k * (p.slab_banks * sums(p.n_slabs - 1) + nb);
    return all / ((double)nb * k) + std::log2(kStreamBanks) + chain_rounding(ks, false);
}

double spmm_stream_ns(const SpmmStreamPlan& p, SpmmFit fit, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N) {
    return Expectation(fit, vsize, isize, M, K, bank, k, N, p.n_tiles)(p, p.slab_banks / kStreamBanks, p.n_tiles * p.n_slabs * p.row_groups);
}

// This runs in every call, so most launches are passed over by what they take at least: 3000 random products are
// planned in 0.42 us in the mean and 1.6 at the 99th percentile, fc6 (4096 x 25088, banks of 64) at N = 16 in 1.2, the tile kernels included.
SpmmStreamPlan spmm_stream_plan(SpmmFit fit_of, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, int min_slabs, int max_slabs, int max_lds,
                                double max_rounding, double max_ns) {
    SpmmStreamPlan best{};
    constexpr int ib = kStreamBanks, rows = kStreamRows;
    const int64_t tiles = div_up(N, (int64_t)kStreamColumns);
    if (k < kStreamMinK || tiles > INT32_MAX / 2) return best;
    const int nb = (int)(K / bank), n_tiles = (int)tiles, group = bank * kStreamPitch;
    const int fit = max_lds / group, fit_half = max_lds / 2 / group, fit_one = std::min(max_lds, kMaxLdsBytes / 2) / group;
    if (fit < 1) return best;
    const int most_per_cu = fit_of == kFirstFit ? 4 : 1;     // with more the second fit found 6 % of its launches
    const Expectation expected(fit_of, vsize, isize, M, K, bank, k, N, tiles);
    best.ns = max_ns;
    const double most_terms = 2 * max_rounding;      // added by a lane in a stage: with more the first term of rounding() is too large
    // First the slabs that give every compute unit a workgroup of 12 wavefronts, most often the best or near it.
    auto more = [&](int s) { return s < 4 ? s + 1 : fit_of == kFirstFit ? s + s / 2 : s + (s + 1) / 3; };
    const int64_t enough = std::min<int64_t>(kCus / std::max<int64_t>(1, n_tiles * div_up(M, (int64_t)12 * rows)), max_slabs);
    int likely = min_slabs;
    while (more(likely) <= enough) likely = more(likely);
    for (int s = likely, next = min_slabs; s <= max_slabs; s = next, next = more(next)) {
        if (s == likely && next > likely) continue;       // looked at already
        const int slab_groups = div_up(div_up(nb, s), ib), slabs = div_up(nb, slab_groups * ib);
        if (expected.at_least(slabs) >= best.ns) {
            if (next > s) break;          // more slabs take longer still
            continue;
        }
        const int per_group = (int)std::min<int64_t>((int64_t)n_tiles * slabs, INT32_MAX);      // workgroups
        int seen_waves = 0, seen_rows = 0;
        for (int c = 1; c <= most_per_cu; ++c) {           // workgroups per compute unit to aim at
            const int target = std::max(1, kCus * c / per_group), m = div_up((int)M, target);
            const int row_waves = std::min(div_up(m, rows), 12), rpwg = std::min(m, row_waves * rows);
            if (row_waves == seen_waves && rpwg == seen_rows) continue;
            seen_waves = row_waves;
            seen_rows = rpwg;
            const int groups = div_up((int)M, rpwg);
            if ((double)rpwg * nb * k * 4 > UINT32_MAX || (double)n_tiles * slabs * groups > INT32_MAX / 2) continue;
            const int wgs = n_tiles * slabs * groups;
            // several stages fill more than half of LDS, whatever ks: one workgroup per compute unit at a time
            const bool alone = slab_groups > fit_half && max_lds == kMaxLdsBytes;
            const double rounds = alone ? div_up(wgs, kCus) : 1, per_cu = alone ? 1 : std::max(1.0, wgs * (1.0 / kCus));
            if (expected.at_least(slabs, slab_groups, row_waves, rounds, per_cu) >= best.ns) continue;
            for (int ks = 1; ks * row_waves <= kMaxWalkers && ks <= slab_groups; ks = ks < 4 ? ks + 1 : ks + ks / 2) {
                if (fit_of == kFirstFit && k * (std::min(slab_groups, fit_half) - ks + 1) > most_terms * ks) continue;
                if (expected.at_least(slabs, slab_groups, row_waves, rounds, per_cu, ks, slab_groups <= fit_one ? slab_groups : ks) >= best.ns) continue;
                // a stage holds a group of banks for each of the ks; two of them side by side
                int sg = std::min(slab_groups, fit_half / ks * ks);
                int bufs = sg >= slab_groups ? 1 : 2;
                if (sg < 1 || (sg < slab_groups && slab_groups <= fit_one)) {
                    sg = std::min(slab_groups, fit / ks * ks);
                    bufs = 1;
                }
                if (sg < 1) continue;
                SpmmStreamPlan p{};
                p.ok = true;
                p.n_tiles = n_tiles; p.n_slabs = slabs; p.slab_banks = slab_groups * ib;
                p.sb = sg * ib; p.n_bufs = bufs; p.buf_bytes = sg * group;
                p.rows_per_wg = rpwg; p.row_groups = groups;
                p.ksplit = ks; p.row_waves = row_waves;
                p.copy_waves = std::min(4, kWavesPerCu - ks * row_waves);
                p.lds_bytes = std::max<size_t>((size_t)bufs * p.buf_bytes, (size_t)(ks - 1) * row_waves * 1024);
                if (p.lds_bytes > (size_t)max_lds) continue;
                p.ns = expected(p, slab_groups, wgs);
                if (fit_of == kFirstFit) {
                    if (p.ns < best.ns && rounding(p, slab_groups, k) <= max_rounding) best = p;
                    continue;
                }
                // The second fit looks at shorter stages too, whose sums round less: the first copy is shorter, the later ones are
                // more (512 x 4608 at N = 196, stages of 8 banks instead of 16: 14.7 us as well, 14.8 against 22.2 in rounding).
                for (int n = div_up(sg, ks); p.ns >= best.ns || spmm_stream_rounding(p, nb, k) > max_rounding;) {
                    const double longer = p.ns;
                    n = (n + 1) / 2;
                    p.sb = n * ks * ib; p.n_bufs = 2; p.buf_bytes = n * ks * group;
                    p.lds_bytes = std::max<size_t>((size_t)2 * p.buf_bytes, (size_t)(ks - 1) * row_waves * 1024);
                    p.ok = p.sb < sg * ib && longer < kStagesWorth * best.ns && p.lds_bytes <= (size_t)max_lds;
                    if (!p.ok) break;
                    sg = n * ks;
                    p.ns = expected(p, slab_groups, wgs);
                }
                if (p.ok) best = p;
            }
        }
    }
    return best;
}

int spmm_stream_launch(const SpmmStreamPlan& p, const SpmmArgs& t, int dtype, int isize, hipStream_t st) {
    SpmmStreamArgs a{};
    a.vals = t.vals; a.idx = t.idx; a.X = t.X; a.out = t.out;
    a.ldx = t.ldx; a.ld_out = t.ld_out; a.slab_stride = t.slab_stride;
    a.M = t.M; a.K = t.K; a.B = t.B; a.k = t.k; a.N = t.N; a.nb = t.nb;
    a.n_tiles = p.n_tiles; a.slab_banks = p.slab_banks; a.n_slabs = p.n_slabs; a.sb = p.sb; a.n_bufs = p.n_bufs; a.buf_bytes = p.buf_bytes;
    a.rows_per_wg = p.rows_per_wg; a.row_groups = p.row_groups; a.ksplit = p.ksplit; a.row_waves = p.row_waves;
    const int unit = unit_of(isize, t.k);
    a.rounds = (t.k + unit - 1) / unit;
    a.last = t.k - unit * (a.rounds - 1);
    // Consecutive workgroups run on one XCD and share its L2: the order that fetches fewer bytes from
    // memory (each of the 8 XCDs sees all of what varies slowest).
    const double x = 4.0 * t.K * t.N, w = (double)t.M * t.nb * t.k * ((dtype == BS_F16 ? 2 : 4) + isize);
    a.tiles_fast = w + x * std::min(kXcds, p.row_groups) <= x + w * std::min(kXcds, p.n_tiles);
    a.total_wgs = p.n_tiles * p.n_slabs * p.row_groups;
    a.wgs_per_xcd = (a.total_wgs + kXcds - 1) / kXcds;
    a.magic_inner = magic_u32(a.tiles_fast ? p.n_tiles : p.row_groups);
    a.magic_slab = magic_u32(p.n_tiles * p.row_groups);
    a.magic_sb = magic_u32(p.sb);
    a.magic_rw = magic_u32(p.row_waves);
    // the direct copies' 32-bit offsets inside a group of banks
    a.by_registers = t.ldx % 4 != 0 || (double)(kStreamBanks * t.B + 4) * (double)t.ldx * 4 > INT32_MAX;
    a.vec_out = t.vec_out;
    const SpmmLaunch l{64 * (p.ksplit * p.row_waves + p.copy_waves), p.lds_bytes, st, false};
    if (isize == 2) return spmm_stream_launch_wide(dtype, a, l);
    return dtype == BS_F16 ? spmm_stream_launch_f16(a, l) : spmm_stream_launch_f32(a, l);
}

}  // namespace bs
