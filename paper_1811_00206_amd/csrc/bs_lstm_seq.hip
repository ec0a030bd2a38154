// Host side of bs_lstm_sequence: one kernel for all steps (bs_lstm_seq_kernel.h), or a launch per step.
#include <hip/hip_ext.h>

#include <algorithm>

#include "bs_lstm_seq_kernel.h"

namespace bs {
namespace {

// The kernels ahead and behind and the first loads cost about two launched steps: T = 3 takes as long either way (16.5 against
// 17.2 us over fourteen matrices), T = 4 16.5 against 20.
constexpr int64_t kMinSteps = 4;
constexpr int64_t kWaitTicks = 2000000;          // 20 ms
constexpr int kLookTicks = 14;                   // of a look that finds nothing new: 135 to 138 ns with 1 to 128 workgroups
// Units per workgroup: with fewer than 8 the stores of many workgroups meet in one line of H_all (512 units, 512 lanes
// each: 64 workgroups 65 us for 32 steps, 128 79 us).
constexpr int kMaxWgs = 128, kFewestUnits = 8;
// Lanes: 512 up to this many entries each, else 768 if that goes (1024 x 2048, 16 entries: 62 against 67 us for 32 steps;
// 6000 x 3000, 36 or 24 entries: 78 against 72).
constexpr int kFewEntries = 16;

bool overlap(const void* p, int64_t pn, const void* q, int64_t qn) {
    const uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return a < b + (uint64_t)qn * 4 && b < a + (uint64_t)pn * 4;
}

// Compute units of the current device, 0 where that cannot be told.
int compute_units() {
    static std::atomic<int> known[64];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) return 0;
    if ((n = known[dev].load(std::memory_order_relaxed)) > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    known[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Whether the stream's kernels may run on all of them (a query of 0.2 us, as good inside a capture).
bool on_all_units(hipStream_t st, int units) {
    uint32_t mask[32] = {};
    const uint32_t words = ((uint32_t)units + 31) / 32;
    if (words > 32) return false;
    if (st == hipStreamLegacy || st == hipStreamPerThread) return true;       // names of streams that have no mask of their own
    if (hipExtStreamGetCUMask(st, words, mask) != hipSuccess) {
        (void)hipGetLastError();                 // the launch says what is wrong with the stream
        return true;
    }
    for (int i = 0; i < units; ++i)
        if (!(mask[i / 32] >> (i % 32) & 1)) return false;
    return true;
}

}  // namespace

// threads, workgroups: 0, or the shape to launch
static LstmSeqPlan lstm_seq_plan(int dtype, int64_t H, int64_t I, int bank, int k, int threads, int workgroups) {
    LstmSeqPlan p{};
    const int64_t K = H + I, row_len = K / bank * k;
    if (H % 4 || I % 4 || K * 4 > 0xffff || (double)H * 4 * row_len * 4 > INT32_MAX) return p;
    if (!lstm_step_lanes(dtype, H, I, bank, k, &p.ch, &p.lpr)) return p;
    const int64_t cpr = row_len / p.ch;
    p.slots = (int)std::min<int64_t>((cpr + p.lpr - 1) / p.lpr, INT32_MAX);
    if (p.slots > kLstmSeqMost) return p;
    const int max_wgs = workgroups ? workgroups : (int)std::min<int64_t>(kMaxWgs, std::max<int64_t>(1, H / kFewestUnits));
    auto rows_of = [&](int thr) {                // per lane, 0 where that does not go
        const int groups = thr / p.lpr;
        if (thr % (4 * p.lpr) || I > 4 * thr) return 0;
        const int64_t rows = (4 * ((H + max_wgs - 1) / max_wgs) + groups - 1) / groups, chunks = rows * p.slots;
        return rows <= kLstmSeqMost && chunks <= kLstmSeqSlots && chunks * p.ch <= kLstmSeqEntries && thr <= lstm_seq_threads((int)chunks * p.ch) ? (int)rows : 0;
    };
    p.threads = threads;
    if (threads == 0) {
        const int rows = rows_of(512);
        p.threads = (rows == 0 || rows * p.slots * p.ch > kFewEntries) && rows_of(768) ? 768 : 512;
    }
    p.rows = rows_of(p.threads);
    if (p.rows == 0) return p;
    p.units = p.rows * (p.threads / p.lpr) / 4;
    p.grid = (int)((H + p.units - 1) / p.units);
    p.x_slots = (int)std::min<int64_t>(I / bank * k / p.ch / p.lpr, p.slots);   // chunks of which every entry's bank lies in x
    p.lds = ((size_t)2 * (K + 4) + 4 * p.units) * 4 + 16;
    p.finish_lds = (size_t)(K + 4 + 4 * H) * 4 + H;
    p.ok = p.lds <= kLdsWithoutLimit && p.finish_lds <= kLdsWithoutLimit;
    return p;
}

void lstm_seq_plan_describe(int dtype, int64_t H, int64_t I, int bank, int k, int threads, int workgroups, int64_t* out, int n_out) {
    const LstmSeqPlan p = lstm_seq_plan(dtype, H, I, bank, k, threads, workgroups);
    const int64_t v[11] = {p.ok, p.ch, p.lpr, p.slots, p.rows, p.units, p.x_slots, p.threads, p.grid, (int64_t)p.lds, (int64_t)p.finish_lds};
    for (int i = 0; i < n_out && i < 11; ++i) out[i] = v[i];
}

static int launch_plan(const LstmSeqPlan& p, const void* vals, const uint8_t* idx, int dtype, int64_t H, int64_t I, int bank, int k,
                       const float* X, int64_t T, const float* h0, const float* bias, float* c, float* H_all, int64_t wait_ticks,
                       hipStream_t st) {
    LstmSeqArgs a{};
    a.vals = vals; a.idx = idx; a.X = X; a.h0 = h0; a.bias = bias; a.c = c; a.H_all = H_all;
    a.T = T; a.H = (int)H; a.I = (int)I; a.B = bank; a.k = k;
    a.row_len = (int)((H + I) / bank * k);
    a.chunks_per_row = a.row_len / p.ch;
    a.magic_k = magic_u32((uint32_t)k);
    a.units = p.units;
    a.lpr = p.lpr;
    while ((1 << a.lpr_shift) < p.lpr) ++a.lpr_shift;
    a.x_slots = p.x_slots;
    a.vec = (int)(H + I) + 4;
    a.wait_looks = (int)std::min<int64_t>((wait_ticks < 0 ? kWaitTicks : wait_ticks) / kLookTicks, INT32_MAX);
    return dtype == BS_F16 ? lstm_seq_launch_f16(p, a, st) : lstm_seq_launch_f32(p, a, st);
}

int launch_lstm_finish(const void* vals, const uint8_t* idx, int dtype, int64_t H, int64_t I, int bank, int k, const float* X,
                       int64_t T, const float* h0, const float* bias, float* c, float* H_all, hipStream_t st) {
    LstmSeqPlan p = lstm_seq_plan(dtype, H, I, bank, k, 0, 0);
    if (!p.ok) return BS_ERR_UNSUPPORTED;
    p.finish_only = true;
    return launch_plan(p, vals, idx, dtype, H, I, bank, k, X, T, h0, bias, c, H_all, -1, st);
}

int launch_lstm_sequence(const void* vals, const uint8_t* idx, int dtype, int64_t H, int64_t I, int bank, int k,
                         const float* X, int64_t T, const float* h0, const float* bias, float* c, float* H_all,
                         int threads, int workgroups, int64_t wait_ticks, hipStream_t st) {
    const LstmSeqPlan p = T >= kMinSteps || threads ? lstm_seq_plan(dtype, H, I, bank, k, threads, workgroups) : LstmSeqPlan{};
    // H_all is filled ahead of the first step, c is written behind the last
    const bool apart = !overlap(H_all, T * H, X, T * I) && !overlap(H_all, T * H, h0, H) && !overlap(H_all, T * H, bias, 4 * H) &&
                       !overlap(H_all, T * H, c, H) && !overlap(c, H, X, T * I) && !overlap(c, H, bias, 4 * H);
    const int units = compute_units();
    if (!p.ok || !apart || p.grid * 2 > units || !on_all_units(st, units)) {
        for (int64_t t = 0; t < T; ++t) {
            const float* h_in = t == 0 ? h0 : H_all + (t - 1) * H;
            const int rc = launch_lstm_step(vals, idx, dtype, H, I, bank, k, X + t * I, h_in, bias, c, c, H_all + t * H, st);
            if (rc != BS_OK) return rc;
        }
        return BS_OK;
    }
    return launch_plan(p, vals, idx, dtype, H, I, bank, k, X, T, h0, bias, c, H_all, wait_ticks, st);
}

}  // namespace bs
