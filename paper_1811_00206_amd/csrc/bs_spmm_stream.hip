// Host side of the SpMM kernels that walk K in stages (bs_spmm_stream_kernel.h): the launch and what it
// is expected to take.
#include <algorithm>
#include <cmath>

#include "bs_spmm_stream_kernel.h"

namespace bs {
namespace {

constexpr int kP = 4;                        // pieces of 4 columns per tile
constexpr int kCus = 256, kWavesPerCu = 16;  // wavefronts: by the kernels' registers
constexpr int kMaxWalkers = 14;

int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

// entries of a bank that a lane loads at once (the kernel's U)
int unit_of(int isize, int k) { return isize == 2 ? (k < 8 ? 4 : 8) : k > kStreamMaxK ? 8 : k; }

// Expected time of a launch in ns.  The terms are the kernel's own steps; their factors are a fit to
// 1332 launches of random shapes and plans on MI355X (median error 6 %, 11 % rms).
double expected_ns(const SpmmStreamPlan& p, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, bool aligned) {
    const int walkers = p.ksplit * p.row_waves, waves = walkers + p.copy_waves;
    const int64_t wgs = (int64_t)p.n_tiles * p.n_slabs * p.row_groups;
    const int64_t slab_groups = div_up(std::min<int64_t>(p.slab_banks, K / bank), stream_banks(kP)), sg = p.sb / stream_banks(kP);
    const int64_t stages = div_up(slab_groups, sg);
    double per_cu = std::max<int64_t>(1, std::min<int64_t>({(int64_t)(kMaxLdsBytes / p.lds_bytes), kWavesPerCu / waves, div_up(wgs, kCus)}));
    const double rounds = std::ceil(wgs / (kCus * per_cu));
    // an entry costs a wavefront 66 ns by itself, and 13.7 ns for each that shares the compute unit
    const double entry = std::max(66.0, 13.7 * walkers * per_cu) * (isize == 2 || k > kStreamMaxK ? 1.24 : 1.0);
    const double unit = k * entry + 29.0 * std::max(1.0, walkers * per_cu / 4);
    const double walk = std::ceil((double)std::min(sg, slab_groups) / p.ksplit) * unit;
    const double tail = std::ceil((double)(slab_groups - (stages - 1) * sg) / p.ksplit) * unit;
    const double group = (double)bank * kStreamPitch * per_cu * (aligned ? 1.0 : 1.57);
    const double first = 874 + std::min(sg, slab_groups) * group / std::min(15.7 * waves * per_cu, 82.0);
    const double copy = 874 + sg * group / std::min(15.7 * p.copy_waves * per_cu, 82.0);
    double t = first + walk;
    if (stages > 1) t = first + tail + (stages - 1) * (p.n_bufs == 2 ? std::max(walk, copy) : walk + copy);
    t = 1670 + rounds * (t + 1800);
    const double w_bytes = (double)M * (K / bank) * k * (vsize + isize), y_bytes = 4.0 * M * N;
    t = std::max(t, 3000 + (w_bytes * std::min(p.n_tiles, 2) + 4.0 * K * N + y_bytes) / 3835);
    if (p.n_slabs > 1) t += 2700 + 2.0 * p.n_slabs * y_bytes / 3750;
    return t;
}

// A lane adds its banks' entries of a stage, then the stages; then come the banks side by side, the wavefronts
// along K and the slabs.
double rounding(const SpmmStreamPlan& p, int64_t nb, int k) {
    const int64_t groups = div_up(std::min<int64_t>(p.slab_banks, nb), stream_banks(kP)), sg = p.sb / stream_banks(kP);
    return chain_rounding((double)k * div_up(std::min(sg, groups), p.ksplit), true) + chain_rounding((double)div_up(groups, sg), false) +
           std::log2(stream_banks(kP)) + chain_rounding(p.ksplit, false) + chain_rounding(p.n_slabs, false);
}

}  // namespace

SpmmStreamPlan spmm_stream_plan(int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, int max_slabs,
                                int max_lds, double max_rounding) {
    SpmmStreamPlan best{};
    constexpr int ib = stream_banks(kP), rows = stream_rows(kP);
    if (k < kStreamMinK) return best;
    const bool aligned = N % 4 == 0;         // as in the usual X, whose rows are adjacent
    const int64_t nb = K / bank;
    const int64_t group = (int64_t)bank * kStreamPitch;
    const int64_t n_tiles = div_up(N, 4 * kP);
    for (int s = 1; s <= max_slabs; s = s < 4 ? s + 1 : s + s / 2) {
        const int64_t slab = div_up(div_up(nb, s), ib) * ib, slabs = div_up(nb, slab), slab_groups = slab / ib;
        int64_t seen_waves = 0;
        for (int c = 1; c <= 4; ++c) {           // workgroups per compute unit to aim at
            int64_t groups = std::max<int64_t>(1, (int64_t)kCus * c / (n_tiles * slabs));
            const int64_t row_waves = std::min<int64_t>(div_up(div_up(M, groups), rows), 12);
            const int64_t rpwg = std::min(div_up(M, groups), row_waves * rows);
            if (row_waves * 4096 + rpwg == seen_waves) continue;
            seen_waves = row_waves * 4096 + rpwg;
            groups = div_up(M, rpwg);
            if ((double)rpwg * nb * k * 4 > UINT32_MAX || (double)n_tiles * slabs * groups > INT32_MAX / 2) continue;
            for (int ks = 1; ks * row_waves <= kMaxWalkers && ks <= slab_groups; ks = ks < 4 ? ks + 1 : ks + ks / 2) {
                // a stage holds a group of banks for each of the ks; two of them side by side
                int64_t sg = std::min(slab_groups, (max_lds / 2 / group) / ks * ks);
                int bufs = sg >= slab_groups ? 1 : 2;
                if (sg < 1 || (sg < slab_groups && slab_groups * group <= std::min(max_lds, kMaxLdsBytes / 2))) {
                    sg = std::min(slab_groups, (max_lds / group) / ks * ks);
                    bufs = 1;
                }
                if (sg < 1) continue;
                SpmmStreamPlan p{};
                p.ok = true;
                p.n_tiles = (int)n_tiles; p.n_slabs = (int)slabs; p.slab_banks = (int)slab;
                p.sb = (int)(sg * ib); p.n_bufs = bufs; p.buf_bytes = (int)(sg * group);
                p.rows_per_wg = (int)rpwg; p.row_groups = (int)groups;
                p.ksplit = ks; p.row_waves = (int)row_waves;
                p.copy_waves = std::min(4, kWavesPerCu - ks * (int)row_waves);
                p.lds_bytes = std::max<size_t>((size_t)bufs * p.buf_bytes, (size_t)(ks - 1) * row_waves * 1024);
                if (p.lds_bytes > (size_t)max_lds) continue;
                p.ns = expected_ns(p, vsize, isize, M, K, bank, k, N, aligned);
                if ((!best.ok || p.ns < best.ns) && rounding(p, nb, k) <= max_rounding) best = p;
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
    a.by_registers = t.ldx % 4 != 0 || (double)(stream_banks(kP) * t.B + 4) * (double)t.ldx * 4 > INT32_MAX;
    a.vec_out = t.vec_out;
    const SpmmLaunch l{64 * (p.ksplit * p.row_waves + p.copy_waves), p.lds_bytes, st, false};
    if (isize == 2) return spmm_stream_launch_wide(dtype, a, l);
    return dtype == BS_F16 ? spmm_stream_launch_f16(a, l) : spmm_stream_launch_f32(a, l);
}

}  // namespace bs
