// Host side of bs_spmm: tiling plan, launch, and the kernel that adds slab
// partial sums (see bs_spmm_kernel.h for the design of the main kernel).
#include <algorithm>
#include <cmath>

#include "bs_spmm_rows_kernel.h"
#include "bs_spmm_stream_kernel.h"

namespace bs {
namespace {

constexpr size_t kTileBudget = 128 * 1024;   // LDS bytes for the tile of X
constexpr int kCus = 256;

struct SpmmPlan {
    bool ok;
    int ch;            // entries per value/offset chunk
    int q;             // float4 quads per lane (1, 2 or 4)
    int nl;            // column groups of 4*q columns per tile (power of two, at most 8)
    int nt, n_tiles;   // columns per tile
    int sb, n_slabs;   // banks per slab
    int lpr, u;        // lanes per (row, column group), chunk slots per lane
    bool rows;         // one lane per (row, column group): bs_spmm_rows_kernel.h
    int row_threads;   // lanes of a workgroup that walk rows; launched_threads() adds those that only copy X
    int max_threads;
    int rows_per_wg, row_groups;
    int table_off;
    size_t tile_bytes, lds_bytes;
    size_t ws_bytes;
    double cost;
};

int64_t gcd64(int64_t a, int64_t b) { while (b) { int64_t t = a % b; a = b; b = t; } return a; }

// One candidate: tiles of `quads` groups of 4 columns (a power of two).  Cost = bytes moved through L2 (tiles of
// X staged by every workgroup, W once per column tile, slab partial sums twice).
// isize: bytes per stored offset; with 2 the kernels exist for the widest chunk and for
// single entries only.
SpmmPlan plan_for(int quads, int dtype, int64_t M, int64_t K, int bank, int k, int64_t N, int isize) {
    SpmmPlan p{};
    // one float4 per lane and entry: the lanes of a column group then read one
    // contiguous piece of an LDS row, which costs the fewest bank conflicts
    // (measured: 2 quads per lane equal, 4 quads per lane 1.6x slower)
    const int q = 1;
    const int nl = quads / q;
    const int64_t nb = K / bank;
    const int64_t row_len = nb * k;
    const int vsize = dtype == BS_F16 ? 2 : 4;
    const size_t per_bank = (size_t)bank * quads * 16;
    int64_t sb = (int64_t)(kTileBudget / per_bank);
    if (sb < 1) return p;
    if (sb > nb) sb = nb;

    // chunk width: divides the row; slab starts must stay chunk-aligned
    int ch = 16 / vsize;
    while (ch > 1 && row_len % ch != 0) ch >>= 1;
    if (sb < nb) {
        const int64_t q = ch / gcd64(k, ch);   // sb multiple of q keeps sb*k % ch == 0
        if (sb >= 2 * q) sb = sb / q * q;
        while (ch > 1 && (sb * k) % ch != 0) ch >>= 1;
    }
    // the position table (one word per entry of a row inside the slab) sits behind the tile
    while (sb > 1 && sb * per_bank + (size_t)sb * k * 4 > (size_t)kMaxLdsBytes) --sb;
    if (sb * per_bank + (size_t)sb * k * 4 > (size_t)kMaxLdsBytes) return p;
    if (sb < nb) while (ch > 1 && (sb * k) % ch != 0) ch >>= 1;
    if (isize == 2 && ch != 16 / vsize) ch = 1;

    p.ch = ch;
    p.q = q;
    p.nl = nl;
    p.nt = 4 * quads;
    p.n_tiles = (int)((N + p.nt - 1) / p.nt);
    p.sb = (int)sb;
    p.n_slabs = (int)((nb + sb - 1) / sb);
    const size_t tile_bytes = (size_t)sb * per_bank;
    p.tile_bytes = tile_bytes;
    p.table_off = (int)(tile_bytes / 4);
    p.lds_bytes = tile_bytes + (size_t)sb * k * 4;

    const int64_t cps = sb * k / ch;
    // lanes per (row, column group): as few idle lane-slots as possible (slots past
    // the end of the run are skipped only when they are empty for every lane); among
    // equals the narrowest group that needs one round of 4 slots, else two rounds
    int lpr = 0;
    int64_t best_slots = 0;
    auto better = [&](int cand, int64_t slots) {
        if (lpr == 0) return true;
        const int64_t w_new = slots * cand, w_old = best_slots * lpr;
        if (w_new != w_old) return w_new < w_old;
        const bool one_new = slots <= 4, one_old = best_slots <= 4;
        if (one_new != one_old) return one_new;
        return one_new ? cand < lpr : cand > lpr;
    };
    for (int cand = 4; cand <= kWave / nl; cand <<= 1) {
        const int64_t slots = (cps + cand - 1) / cand;
        if (slots > 8 && cand < kWave / nl) continue;
        if (better(cand, slots)) { lpr = cand; best_slots = slots; }
    }
    p.lpr = lpr;
    p.u = best_slots <= 2 ? 2 : 4;
    // tiles of 16 columns and more: one lane per (row, column group); measured on the
    // 6000 x 3000 matrix 13.9 / 27.4 us against 14.9 / 34.7 us at N = 32 / 128, and
    // 25.0 against 39.5 us on the 128 x 576 convolution with 12544 columns
    p.rows = nl >= 4;
    if (p.rows) { p.lpr = lpr = 1; p.u = 4; }
    const int max_threads = p.lds_bytes > 80 * 1024 ? 1024 : p.lds_bytes > 40 * 1024 ? 512 : 256;

    int wg_per_cu = (int)((size_t)kMaxLdsBytes / p.lds_bytes);
    if (wg_per_cu > 2048 / max_threads) wg_per_cu = 2048 / max_threads;
    if (wg_per_cu < 1) wg_per_cu = 1;
    int64_t groups = (int64_t)kCus * wg_per_cu / ((int64_t)p.n_slabs * p.n_tiles);
    if (groups < 1) groups = 1;
    if (groups > M) groups = M;
    const int64_t rpw = (M + groups - 1) / groups;
    p.rows_per_wg = (int)rpw;
    p.row_groups = (int)((M + rpw - 1) / rpw);
    // workgroup size: equal row passes (no half-empty last pass), whole wavefronts
    const int lanes_per_row = lpr * nl;
    const int64_t passes = (rpw * lanes_per_row + max_threads - 1) / max_threads;
    const int64_t rows_per_pass = (rpw + passes - 1) / passes;
    int64_t threads = (rows_per_pass * lanes_per_row + kWave - 1) / kWave * kWave;
    if (threads > max_threads) threads = max_threads;
    p.row_threads = (int)threads;
    p.max_threads = max_threads;
    p.ws_bytes = p.n_slabs > 1 ? (size_t)p.n_slabs * M * N * 4 : 0;
    const double w_bytes = (double)M * row_len * (vsize + isize);
    p.cost = (double)p.row_groups * p.n_tiles * p.n_slabs * tile_bytes + p.n_tiles * w_bytes +
             2.0 * p.ws_bytes;
    p.ok = true;
    return p;
}

// 16-byte direct-to-LDS copies need 16-byte aligned row pieces and whole groups of 4 columns.
// One or two columns, and three in adjacent rows, go through registers: 4441 x 736 at N = 2:
// 5.4 -> 4.7 us, 11772 x 3072 at N = 3: 11.0 -> 7.1 us; with three in a wider pitch each load would
// touch as many cache lines as it has lanes for few bytes (2182 x 2704, ldx = 4: 6.4 against 9.0 us).
SpmmCopy copy_kind(int64_t N, int64_t ldx) {
    if (N % 4 == 0 && ldx % 4 == 0) return kCopyWide;
    return N <= 2 || (N == 3 && ldx == 3) ? kCopyRegisters : kCopyNarrow;
}

// Threads of a workgroup.  With few rows per workgroup the wavefronts that walk them are too few
// to bring the tile in: each more copies a share of it and leaves.
//   * Pieces of 16 bytes, up to 8 of them per lane: 1024 x 1024 at N = 40: 12.8 -> 11.2 us.  Where
//     half of that many wavefronts walk rows already, the others cost more than they bring
//     (6000 x 3000 at N = 40: 17.0 -> 17.7 us).
//   * Pieces of 4 bytes are four times as many, so up to four times the lanes (300 x 320 at N = 8
//     with an odd row pitch, 304 workgroups: 5.5 -> 3.6 us), as far as the chip has room for them:
//     512 per compute unit, or two wavefronts per workgroup (3723 x 600 at N = 37, 1960 workgroups:
//     6.7 us with 128 lanes each, 8.4 with 256).
int launched_threads(const SpmmPlan& p, SpmmCopy copy) {
    const bool wide = copy == kCopyWide;
    auto whole = [](int64_t lanes) { return (lanes + kWave - 1) / kWave * kWave; };
    int64_t copy_threads = whole((int64_t)p.tile_bytes / (8 * 16));
    if (!wide) {
        const int64_t wgs = (int64_t)p.n_tiles * p.n_slabs * p.row_groups;
        const int64_t room = std::max<int64_t>((int64_t)kCus * 512 / wgs / kWave * kWave, 2 * kWave);
        copy_threads = std::max(copy_threads, std::min(whole((int64_t)p.tile_bytes / (8 * 4)), room));
    }
    if (copy_threads > p.max_threads) copy_threads = p.max_threads;
    return (int)(p.row_threads * (wide ? 2 : 1) < copy_threads ? copy_threads : p.row_threads);
}

SpmmPlan make_plan(int dtype, int64_t M, int64_t K, int bank, int k, int64_t N, int isize = 1) {
    SpmmPlan best{};
    // Tiles of at most 32 columns: with 64 the LDS rows are 256 bytes, half as many banks of
    // X fit a slab and a wavefront holds 4 rows instead of 8; measured on ten shapes the
    // wider tile won twice by 2-3 % and lost up to 18 % (4096 x 4096 at N = 64: 20.6 against
    // 17.8 us; 1024 x 1024 at N = 512: 15.9 against 13.0 us).
    for (int quads = 1; quads <= 8; quads <<= 1) {
        if (quads > 1 && 4 * (quads / 2) >= N) break;   // the narrower tile already covers N
        SpmmPlan p = plan_for(quads, dtype, M, K, bank, k, N, isize);
        if (p.ok && (!best.ok || p.cost < best.cost)) best = p;
    }
    return best;
}

// What the tile kernels are expected to take for a plan of more than 8 columns, in ns, the slab sums included.  Fits to
// random products on MI355X.  kFirst: 442 of them, operands repeated (median error 5 %, 9 % rms); kSecond: 2656 with 8-bit
// offsets whose operands change from call to call (4.4 %, 8.7 %).
struct TileFactors {
    double rows_alone, rows_shared, rows_simd, load, row;    // lane per row: of an entry as in bs_spmm_stream.hip; of 16 chunks; of a pass
    double rows_ch2, rows_ch1, rows_half;
    double alone, shared, simd, pass, few;                   // several lanes per row; `few`: chunks of at most 2 entries
    double tile, unaligned, wave_copy, cu_copy, launch, memory, memory_rate, slabs, slab_rate;
};
constexpr TileFactors kFirst{14.2, 3.68, 0, 530, 223, 0.94, 0.9, 1.07, 41.3, 2.84, 0, 629, 1.4,
                                104, 1.37, 15, 54.2, 2930, 2500, 3019, 1920, 4800};
constexpr TileFactors kSecond{16.05, 3.42, 13.3, 439, 0, 0.94, 0.96, 1.05, 46.8, 6.22, 14.36, 686, 1.24,
                             0, 1.61, 550, 65.2, 3460, 3739, 2972, 2324, 4069};
double tiles_ns(const SpmmPlan& p, SpmmFit fit, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, SpmmCopy copy) {
    const TileFactors& f = fit == kFirstFit ? kFirst : kSecond;
    const int threads = launched_threads(p, copy);
    const int64_t wgs = (int64_t)p.n_tiles * p.n_slabs * p.row_groups, nb = K / bank;
    const double per_cu = (double)std::max<int64_t>(1, std::min<int64_t>({(int64_t)(kMaxLdsBytes / p.lds_bytes), 1024 / threads, (wgs + kCus - 1) / kCus}));
    const double rounds = std::ceil(wgs / (kCus * per_cu)), walkers = p.row_threads / 64.0 * per_cu, simd = std::ceil(walkers * 0.25);
    const int64_t run = std::min<int64_t>(p.sb, nb) * k;      // entries of a row inside a slab
    const int rows_per_pass = p.row_threads / (p.nl * p.lpr);
    double pass;
    if (p.rows) {
        pass = run * std::max({f.rows_alone, f.rows_shared * walkers, f.rows_simd * simd}) + f.load * std::ceil(run / (16.0 * p.ch)) + f.row;
        pass *= (p.ch == 2 ? f.rows_ch2 : p.ch == 1 ? f.rows_ch1 : 1.0) * (vsize == 2 ? f.rows_half : 1.0);
    } else {
        const int64_t slots = (run / p.ch + p.lpr - 1) / p.lpr;
        pass = (slots * p.ch * std::max({f.alone, f.shared * walkers, f.simd * simd}) + f.pass) * (p.ch <= 2 ? f.few : 1.0);
    }
    const double tile = f.tile + (double)p.tile_bytes * per_cu * (copy == kCopyWide ? 1.0 : f.unaligned) / std::min(f.wave_copy * threads / 64 * per_cu, f.cu_copy);
    double t = f.launch + rounds * (tile + (p.rows_per_wg + rows_per_pass - 1) / rows_per_pass * pass);
    const double w_bytes = (double)M * nb * k * (vsize + isize), y_bytes = 4.0 * M * N;
    t = std::max(t, f.memory + (w_bytes * std::min(p.n_tiles, 2) + 4.0 * K * N + y_bytes) / f.memory_rate);
    if (p.n_slabs > 1) t += f.slabs + 2.0 * p.n_slabs * y_bytes / f.slab_rate;
    return t;
}

// The rounding error of the tile kernels' sums (chain_rounding): `lpr` lanes walk every lpr-th chunk of a slab's run.
double tiles_rounding(const SpmmPlan& p, int64_t nb, int k) {
    const int64_t run = nb * k / p.n_slabs, chunks = std::max<int64_t>(1, run / p.ch), slots = chunks / p.lpr, longer = chunks - slots * p.lpr;
    auto lanes = [&](int64_t n, int64_t entries) { return n * entries * chain_rounding((double)entries, true); };
    return (lanes(longer, (slots + 1) * p.ch) + lanes(p.lpr - longer, slots * p.ch)) / (double)(chunks * p.ch) +
           std::log2((double)std::min<int64_t>(p.lpr, chunks)) + chain_rounding(p.n_slabs, false);
}

// The stage kernels are taken, for every row pitch of X alike, where they are expected to be faster.  The first fit says
// whether and with which launch, by a line at 0.93 that was chosen with both kernels of 1050 random products timed.  Products
// expected below kStreamWorthNs are not worth the planning.  With 8-bit offsets the second fit then looks for another stage
// launch: one that it expects to take less than the first one (both times by the second fit, so much of what that is off by
// is common to the two) and whose sums round no worse.  Without that condition 5 % of random products got sums
// of a larger error (512 x 4608 at N = 784 1.4 times; up to 2.3 times where a product went back to the tile kernels, which
// now none does).  How much less, from 3700 random products with both launches timed:
//   * With more slabs than the first launch 0.97, with as many 0.95: of those expected at 0.98 to 1 every fifth loses more than 8 %.
//   * Instead of tiles of 16 and 32 columns 1, above kStreamMaxK 0.96.  There the stream of W again divides the products: of
//     74 with more than 10 MB of it 34 gain and 28 lose more than 8 % (3833 x 5120, 95 entries per bank, N = 30: 27.4 -> 42.7 us).
//   * Tiles of 4 and 8 columns stay: of 414 products 243 would gain, but 66 lose more than 8 % (520 x 400, N = 5799: 21.0 -> 30.2).
// Of 4500 other products that the second fit alone would plan anew, 1765 are: 0.915 of the time (geometric mean), 1305 gain more
// than 3 %, 192 lose that, 77 more than 8 %.  By itself it plans all of them anew and 388 lose more than 8 %.
// The terms below are what the expectations leave out:
//   * Banks of more than 32 entries and one tile of columns stay on the tile kernels.  What divides these products
//     is the stream of W: all 4 of the 27 timed ones with more than 64 MB of it lose (15947 x 6144, 124 entries
//     per bank, N = 12: 40.1 us by tiles, 68.7 in stages), 11 of the 23 with at most 42 MB gain up to three times
//     (251 x 12500, k = 39, N = 10: 43.1 against 14.2), the others run as long or have no stage launch.  So the line
//     is safe, and further in than it has to be.
//   * More workgroups than compute units: copies of the first stage have nothing to hide behind, unaligned
//     ones the longest (303 x 350 at N = 5687, 28.1 against 34.6 us).
//   * An X of more than 128 MB comes from memory in rows of 64 bytes: of nine timed three lose (142 x 12900 at N = 4846:
//     112.8 against 141.3 us), two gain (65 x 12500 at N = 3963: 85.9 against 67.7), four have no other launch or
//     run as long.
// A launch whose sums would round worse than the tile kernels' is not looked at: those walk an odd row length or a small
// tile with up to 64 lanes per row, so their sums are short (6722 x 144, banks of 16, k = 13, N = 40: 4 entries per lane and
// an exchange, against 39 in a lane of the stage kernels, 1.5 times the error).  Of 4000 random products, 4 %.
constexpr double kStreamMargin = 0.93, kStreamWorthNs = 6000;
constexpr double kSecondMoreSlabs = 0.97, kSecondSameSlabs = 0.95, kSecondFromTiles = 1.0, kSecondFromTilesLong = 0.96, kSecondMaxWBytes = 10e6;
constexpr double kStreamManyAligned = 1.05, kStreamManyUnaligned = 1.2, kStreamLongBank = 1.1;
constexpr int kStreamLongK = 32;
constexpr double kStreamMaxXBytes = 128e6;
SpmmStreamPlan stream_choice(const SpmmPlan& p, int vsize, int isize, int64_t M, int64_t K, int bank, int k, int64_t N) {
    if (N <= 8 || k < kStreamMinK) return {};
    if ((k > kStreamLongK && N <= 16) || 4.0 * K * N > kStreamMaxXBytes) return {};
    // a product whose tile kernel needs no LDS limit raised can be captured as the first of all, so this one may not need it either
    const int max_lds = p.lds_bytes > kLdsWithoutLimit ? kMaxLdsBytes : (int)kLdsWithoutLimit;
    const double longer = k > kStreamLongK ? kStreamLongBank : 1.0;
    auto tiles = [&](SpmmFit fit) { return tiles_ns(p, fit, vsize, isize, M, K, bank, k, N, copy_kind(N, N)); };
    // a launch to be taken instead of the tile kernels
    auto instead = [&](SpmmFit fit, double max_rounding, double max_ns, double many_ns) {
        const SpmmStreamPlan sp = spmm_stream_plan(fit, vsize, isize, M, K, bank, k, N, 1, p.n_slabs, max_lds, max_rounding, max_ns);
        const bool many = (int64_t)sp.n_tiles * sp.n_slabs * sp.row_groups > kCus;
        return sp.ok && many && sp.ns * (N % 4 == 0 ? kStreamManyAligned : kStreamManyUnaligned) >= many_ns ? SpmmStreamPlan{} : sp;
    };
    const double first_tiles = tiles(kFirstFit), max_ns = kStreamMargin * first_tiles / longer;
    SpmmStreamPlan first{};
    if (first_tiles > kStreamWorthNs) first = instead(kFirstFit, tiles_rounding(p, K / bank, k), max_ns, max_ns);
    if (isize == 2) return first;
    if (!first.ok) {
        const bool long_banks = k > kStreamMaxK;
        if (!p.rows || (long_banks && (double)M * (K / bank) * k * (vsize + 1) > kSecondMaxWBytes)) return first;
        const double ns = tiles(kSecondFit) / longer;
        return ns > kStreamWorthNs ? instead(kSecondFit, tiles_rounding(p, K / bank, k), (long_banks ? kSecondFromTilesLong : kSecondFromTiles) * ns, ns) : first;
    }
    const double ns = spmm_stream_ns(first, kSecondFit, vsize, isize, M, K, bank, k, N);
    if (ns <= kStreamWorthNs) return first;
    const SpmmStreamPlan second = spmm_stream_plan(kSecondFit, vsize, isize, M, K, bank, k, N, first.n_slabs, std::min(p.n_slabs, std::max(3, 2 * first.n_slabs)),
                                                   max_lds, spmm_stream_rounding(first, (int)(K / bank), k), kSecondMoreSlabs * ns);
    if (second.n_slabs == first.n_slabs && second.ns >= kSecondSameSlabs * ns) return first;
    return second.ok ? second : first;
}

// Y[r][n] = sum over slabs, in slab order.  magic_n = magic_u32(N): rows from element
// numbers without a 64-bit division (M*N < 2^32 is checked by the caller).
// V = floats per lane and step: 4 when M, N, ldy and Y's address allow 16-byte accesses.
// The kernel is one round trip to memory long, so the loads of up to kBatch slabs are
// issued together and only then added, in slab order (one load after the other made
// three slabs cost three round trips: 4.5 us for a kernel with nothing to compute).
template <int V>
__global__ __launch_bounds__(256) void spmm_reduce_kernel(const float* __restrict__ P,
                                                          float* __restrict__ Y, int64_t M,
                                                          int64_t N, int64_t ldy, int n_slabs,
                                                          uint32_t magic_n) {
    constexpr int kBatch = 8;
    using Vec = typename std::conditional<V == 4, float4, float>::type;
    const int64_t total = M * N;
    const int64_t steps = total / V;                       // V divides N, or M*N if ldy = N
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < steps;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = j * V;
        float acc[V];
#pragma unroll
        for (int n = 0; n < V; ++n) acc[n] = 0.f;
        for (int s0 = 0; s0 < n_slabs; s0 += kBatch) {
            Vec t[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int s = s0 + b < n_slabs ? s0 + b : n_slabs - 1;   // a re-read, never added
                t[b] = *reinterpret_cast<const Vec*>(P + (int64_t)s * total + i);
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (s0 + b < n_slabs) {
                    if constexpr (V == 4) {
                        if (s0 + b == 0) { acc[0] = t[b].x; acc[1] = t[b].y; acc[2] = t[b].z; acc[3] = t[b].w; }
                        else { acc[0] += t[b].x; acc[1] += t[b].y; acc[2] += t[b].z; acc[3] += t[b].w; }
                    } else {
                        if (s0 + b == 0) acc[0] = t[b];
                        else acc[0] += t[b];
                    }
                }
            }
        }
        int64_t o = i;
        if (ldy != N) {
            const uint32_t r = div_magic_any((uint32_t)i, (uint32_t)N, magic_n);
            o = (int64_t)r * ldy + ((uint32_t)i - r * (uint32_t)N);
        }
        if constexpr (V == 4) *reinterpret_cast<float4*>(Y + o) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        else Y[o] = acc[0];
    }
}

// ---- scratch for callers that cannot allocate (bs_spmm_static) -------------------
// The slab partial sums of such a call live in this array.  In host code the array's
// name is only a stand-in: the address kernels and copies may use is what
// hipGetSymbolAddress reports, once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::atomic<void*> g_scratch_ptr[64];

}  // namespace

int static_scratch_lookup() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) return BS_ERR_HIP;
    if (g_scratch_ptr[dev].load(std::memory_order_acquire)) return BS_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return BS_ERR_HIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    return BS_OK;
}

int launch_spmm_static(const void* vals, const uint8_t* idx, int dtype, int64_t M, int64_t K, int bank,
                       int k, const float* X, int64_t N, int64_t ldx, float* Y, int64_t ldy,
                       hipStream_t st) {
    if (M > INT32_MAX / 4 || N > INT32_MAX / 4) return BS_ERR_UNSUPPORTED;
    const SpmmPlan p = make_plan(dtype, M, K, bank, k, N);
    if (!p.ok) return BS_ERR_UNSUPPORTED;
    if (p.ws_bytes > kStaticScratchBytes) return BS_ERR_SCRATCH_LIMIT;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) return BS_ERR_HIP;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        // first call on this device: look the address up, but never inside a capture
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cs) != hipSuccess) return BS_ERR_HIP;
        if (cs != hipStreamCaptureStatusNone) return BS_ERR_NOT_INITIALISED;
        const int rc = static_scratch_lookup();
        if (rc != BS_OK) return rc;
        ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    }
    return launch_spmm(vals, idx, dtype, M, K, bank, k, X, N, ldx, Y, ldy, ptr, kStaticScratchBytes, st);
}

size_t spmm_workspace_bytes(int dtype, int64_t M, int64_t K, int bank, int k, int64_t N) {
    const SpmmPlan p = make_plan(dtype, M, K, bank, k, N);
    return p.ok ? p.ws_bytes : 0;
}

int spmm_plan_describe(int dtype, int isize, int64_t M, int64_t K, int bank, int k, int64_t N, int64_t* out,
                       int n_out) {
    if (M > INT32_MAX / 4 || N > INT32_MAX / 4) return BS_ERR_UNSUPPORTED;
    const SpmmPlan p = make_plan(dtype, M, K, bank, k, N, isize);
    if (!p.ok || p.lds_bytes > (size_t)kMaxLdsBytes) return BS_ERR_UNSUPPORTED;
    const int64_t total = (int64_t)p.n_tiles * p.n_slabs * p.row_groups;
    if (total > INT32_MAX / 2) return BS_ERR_UNSUPPORTED;
    if (p.ws_bytes && M * N > (int64_t)UINT32_MAX) return BS_ERR_UNSUPPORTED;
    const int rows_per_pass = p.row_threads / (p.nl * p.lpr);
    const SpmmStreamPlan sp = stream_choice(p, dtype == BS_F16 ? 2 : 4, isize, M, K, bank, k, N);
    const int64_t v[30] = {p.rows ? 1 : 0, p.ch, p.nl, p.nt, p.n_tiles, p.sb, p.n_slabs, p.lpr, p.u,
                           p.row_threads, p.rows_per_wg, p.row_groups,
                           (p.rows_per_wg + rows_per_pass - 1) / rows_per_pass,
                           (int64_t)p.lds_bytes, (total + kXcds - 1) / kXcds * kXcds, p.table_off,
                           launched_threads(p, copy_kind(N, N)),
                           sp.ok ? 1 : 0, sp.n_tiles, sp.n_slabs, sp.slab_banks, sp.sb, sp.n_bufs, sp.buf_bytes,
                           sp.rows_per_wg, sp.row_groups, sp.ksplit, sp.row_waves, sp.copy_waves, (int64_t)sp.lds_bytes};
    for (int i = 0; i < n_out && i < 30; ++i) out[i] = v[i];
    return BS_OK;
}

namespace {
int launch_spmm_any(const void* vals, const void* idx, int isize, int dtype, int64_t M, int64_t K, int bank,
                    int k, const float* X, int64_t N, int64_t ldx, float* Y, int64_t ldy,
                    void* workspace, size_t workspace_bytes, hipStream_t st) {
    if (M > INT32_MAX / 4 || N > INT32_MAX / 4) return BS_ERR_UNSUPPORTED;
    const SpmmPlan p = make_plan(dtype, M, K, bank, k, N, isize);
    if (!p.ok || p.lds_bytes > (size_t)kMaxLdsBytes) return BS_ERR_UNSUPPORTED;
    if (p.ws_bytes) {
        if (M * N > (int64_t)UINT32_MAX) return BS_ERR_UNSUPPORTED;   // the reduce kernel's 32-bit rows
        if (!workspace || workspace_bytes < p.ws_bytes) return BS_ERR_WORKSPACE;
        if ((uintptr_t)workspace % 16) return BS_ERR_ALIGN;
    }
    const int64_t total = (int64_t)p.n_tiles * p.n_slabs * p.row_groups;
    if (total > INT32_MAX / 2) return BS_ERR_UNSUPPORTED;

    SpmmArgs a;
    a.vals = vals; a.idx = idx; a.X = X;
    a.ldx = ldx;
    if (p.n_slabs > 1) { a.out = static_cast<float*>(workspace); a.ld_out = N; a.slab_stride = M * N; }
    else { a.out = Y; a.ld_out = ldy; a.slab_stride = 0; }
    a.M = (int)M; a.K = (int)K; a.B = bank; a.k = k; a.N = (int)N;
    a.nb = (int)(K / bank);
    a.sb = p.sb; a.n_slabs = p.n_slabs; a.nt = p.nt; a.n_tiles = p.n_tiles; a.nl = p.nl;
    a.rows_per_wg = p.rows_per_wg; a.row_groups = p.row_groups;
    a.total_wgs = (int)total;
    a.wgs_per_xcd = (int)((total + kXcds - 1) / kXcds);
    a.table_off = p.table_off;
    a.magic_k = magic_u32((uint32_t)k);
    a.magic_rg = magic_u32((uint32_t)p.row_groups);
    a.magic_rgs = magic_u32((uint32_t)(p.row_groups * p.n_slabs));
    a.copy = copy_kind(N, ldx);
    const int rows_per_pass = p.row_threads / (p.nl * p.lpr);
    a.row_threads = p.row_threads;
    a.n_passes = (p.rows_per_wg + rows_per_pass - 1) / rows_per_pass;
    a.vec_out = (a.ld_out % 4 == 0 && a.slab_stride % 4 == 0 && (uintptr_t)a.out % 16 == 0) ? 1 : 0;

    auto tiles = [&](bool prepare_only) {
        const SpmmLaunch l{launched_threads(p, copy_kind(N, ldx)), p.lds_bytes, st, prepare_only};
        return isize == 2 ? spmm_launch_wide(dtype, p.rows, p.ch, p.lpr, p.u, a, l)
               : p.rows ? spmm_rows_launch(dtype, p.ch, a, l)
               : dtype == BS_F16 ? spmm_launch_f16(p.ch, p.lpr, p.u, p.q, a, l)
                                 : spmm_launch_f32(p.ch, p.lpr, p.u, p.q, a, l);
    };
    int n_slabs = p.n_slabs, st_code;
    const SpmmStreamPlan sp = stream_choice(p, dtype == BS_F16 ? 2 : 4, isize, M, K, bank, k, N);
    if (sp.ok) {
        SpmmArgs t = a;
        if (sp.n_slabs == 1 && p.n_slabs > 1) {
            t.out = Y; t.ld_out = ldy; t.slab_stride = 0;
            t.vec_out = ldy % 4 == 0 && (uintptr_t)Y % 16 == 0;
        }
        // A first use inside a capture is answered as for the tile kernel of this shape, whose preparation includes
        // every stage kernel of these types: which kernel runs does not depend on what has run before.
        st_code = tiles(true);
        if (st_code == BS_OK) st_code = spmm_stream_launch(sp, t, dtype, isize, st);
        n_slabs = sp.n_slabs;
    } else {
        st_code = tiles(false);
    }
    if (st_code != BS_OK) return st_code;
    if (n_slabs > 1) {
        // 16 bytes per lane where rows of Y and of the workspace allow it (the workspace is
        // 16-byte aligned, its rows are N floats; with rows of Y as long, both are one piece)
        const bool vec = (uintptr_t)Y % 16 == 0 &&
                         (ldy == N ? M * N % 4 == 0 : N % 4 == 0 && ldy % 4 == 0);
        const int64_t steps = M * N / (vec ? 4 : 1);
        int64_t grid = (steps + 255) / 256;
        if (grid > 256 * 16) grid = 256 * 16;
        auto kern = vec ? spmm_reduce_kernel<4> : spmm_reduce_kernel<1>;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), 0, st,
                           static_cast<const float*>(workspace), Y, M, N, ldy, n_slabs,
                           magic_u32((uint32_t)N));
        return hip_status(hipGetLastError());
    }
    return BS_OK;
}
}  // namespace

int launch_spmm(const void* vals, const uint8_t* idx, int dtype, int64_t M, int64_t K, int bank,
                int k, const float* X, int64_t N, int64_t ldx, float* Y, int64_t ldy,
                void* workspace, size_t workspace_bytes, hipStream_t st) {
    return launch_spmm_any(vals, idx, 1, dtype, M, K, bank, k, X, N, ldx, Y, ldy, workspace,
                           workspace_bytes, st);
}

int launch_spmm_wide(const void* vals, const uint16_t* idx, int dtype, int64_t M, int64_t K, int bank,
                     int k, const float* X, int64_t N, int64_t ldx, float* Y, int64_t ldy,
                     void* workspace, size_t workspace_bytes, hipStream_t st) {
    return launch_spmm_any(vals, idx, 2, dtype, M, K, bank, k, X, N, ldx, Y, ldy, workspace,
                           workspace_bytes, st);
}

size_t spmm_workspace_bytes_wide(int dtype, int64_t M, int64_t K, int bank, int k, int64_t N) {
    const SpmmPlan p = make_plan(dtype, M, K, bank, k, N, 2);
    return p.ok ? p.ws_bytes : 0;
}

}  // namespace bs
