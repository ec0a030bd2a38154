// T dependent LSTM steps (arXiv 1811.00206, Sec. 4.3's recurrent models; eq. (1) with bias) in one kernel.
//
// Launched one by one, a step is bound by its launch: it waits for the whole grid of the step before, reads the weights
// again and copies [x ; h] again: 3.6 us each on the 6000 x 3000 matrix at 90 %, whose 9 MB pass in 1.5.  Here up to
// 128 workgroups stay for all T steps.  A workgroup keeps the weights of its hidden units in registers, with
// the LDS address of every entry's operand, and the units' cell state.  What a step waits for is the hidden
// state of the step before, and that carries its own flag: H_all is filled with a word that no hidden state
// is (kAbsent) ahead of the kernel, a unit's owner stores its value past the caches, and every workgroup reads row
// t-1 of H_all, each lane its two words, until none is absent.  No barrier, counter or fence: a step costs one store's
// and one load's latency (measured without the products, 1500 units: 1.4 us with 63 workgroups, 1.5 with 125, 1.75 with
// 250; through one atomic counter, 10 with 256).  The chunks of a row that need only x are done before the wait.
// 32 steps of 1500 / 1024 / 512 / 128 units (I = H), launched and here: 113 -> 68, 101 -> 60, 92 -> 64, 91 -> 45 us, 6 of them
// the first loads and the kernels ahead and behind.  What is left of a step is those latencies; polling with
// two loads in flight instead of one takes 3 % longer.
//
// Sums are those of spmv_kernel<..., LSTM = true>, bit for bit: same lanes per row, chunks and order.  So which of
// the two runs may depend on T and on the number of compute units.
//
// No workgroup relies on the others being there.  The launch is small enough for four such kernels at a time, as many as
// a process has hardware queues: at most half as many workgroups as compute units, two of which share one's registers and LDS.
// A stream that is bound to some of the compute units gets launched steps.  Where the workgroups do not get there all the same
// (another process, a captured launch on such a stream) a step's wait ends after wait_looks (looks and not time, which passes
// while a queue is switched out too): the workgroup marks its units of that step kGivenUp, on which the others stop too, leaves
// their cell state as it was, and the kernel ends.  lstm_finish_kernel, one workgroup that waits for nobody, comes behind it:
// it does nothing where the last row is whole, and otherwise repeats the sequence for the units that are missing there.
// That costs far more than launched steps would have: 20 ms and, for 1500 units, 156 us a step.
#pragma once
#include <algorithm>

#include "bs_spmv_kernel.h"

namespace bs {

constexpr uint32_t kAbsent = 0xffffffffu, kGivenUp = 0xfffffffeu;   // above every other word; no hidden state: lstm_state()

struct LstmSeqArgs {
    const void* vals;
    const uint8_t* idx;
    const float* X;
    const float* h0;
    const float* bias;
    float* c;
    float* H_all;
    int64_t T;
    int H, I, B, k;
    int row_len, chunks_per_row;
    uint32_t magic_k;
    int units;             // hidden units per workgroup
    int lpr, lpr_shift;    // lanes per row, and its logarithm
    int x_slots;           // of a row's chunks in a lane, the first ones that read x alone, in every lane
    int vec;               // floats of one copy of [x ; h], with a zero behind it
    int wait_looks;        // of a lane in a step, before it gives up
};

struct LstmSeqPlan {
    bool ok;
    int ch, lpr, slots, rows;   // chunks of a row per lane, rows per lane
    int units, x_slots, threads, grid;
    size_t lds, finish_lds;
    bool finish_only;
};

int lstm_seq_launch_f32(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st);
int lstm_seq_launch_f16(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st);

// Entries that a lane can hold (a value and half an address each), by the workgroup's size: two workgroups of 768 or 512
// lanes share a compute unit's registers, 80 or 128 of them per lane.
constexpr int lstm_seq_threads(int entries) { return entries <= 24 ? 768 : 512; }
// 36: as far as was measured (6000 x 3000 at 90 %, 512 lanes: 78 us for 32 steps).  The fp32 kernels then use 95 of their 128
// registers, the binary16 ones 77, so more would fit; 1500 units at 80 % and every eighth random model of up to 1536 units
// go step by step.
constexpr int kLstmSeqEntries = 36, kLstmSeqSlots = 12, kLstmSeqMost = 4;    // the most; of chunks, and of one row
constexpr int kLstmFinishThreads = 1024;

#ifdef __HIPCC__

__device__ __forceinline__ bool lstm_there(uint32_t w) { return w < kGivenUp; }

// The cell update of one unit from its four rows' sums; c and h as they are stored.
__device__ __forceinline__ float lstm_cell(const float4 sum, const float4 bias, float& c) {
    const float gi = logistic_fast(sum.x + bias.x), gf = logistic_fast(sum.y + bias.y);
    const float gg = tanh_fast(sum.z + bias.z), go = logistic_fast(sum.w + bias.w);
    c = lstm_state(fmaf(gf, c, gi * gg));
    return lstm_state(go * tanh_fast(c));
}

// An LDS operation of this wavefront is finished for all the others behind this; global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
    pin_order();
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    pin_order();
}

template <typename T>
__device__ __forceinline__ void keep_packed(T& w) {
    if constexpr (sizeof(T) <= 4) {
        uint32_t x = word_of(w, 0);
        asm volatile("" : "+v"(x));
        w = (T)x;
    } else {
        asm volatile("" : "+v"(w.x));
        asm volatile("" : "+v"(w.y));
        if constexpr (sizeof(T) == 16) {
            asm volatile("" : "+v"(w.z));
            asm volatile("" : "+v"(w.w));
        }
    }
}

// The sums of R values over the a.lpr lanes of a row, as group_sum<a.lpr> adds them.
template <int R>
__device__ __forceinline__ void lstm_row_sums(float (&v)[R], int lpr) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = group_sum<8>(v[r]);
    if (lpr < 16) return;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] += dpp_move<0x140>(v[r]);
    if (lpr < 32) return;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = add_across_16(v[r]);
    if (lpr < 64) return;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = add_across_32(v[r]);
}

// VT, CH as in spmv_kernel; a lane has U chunks of each of R rows.
template <typename VT, int CH, int U, int R>
__global__ __launch_bounds__(lstm_seq_threads(U * R * CH), lstm_seq_threads(U * R * CH) / 128) void lstm_seq_kernel(LstmSeqArgs a) {
    extern __shared__ __align__(16) float lds[];
    using VRaw = typename RawBytes<CH * sizeof(VT)>::type;
    using IRaw = typename IdxChunk<uint8_t, CH>::type;
    constexpr int S = U * R, kAddr = (CH + 1) / 2;
    const int tid = threadIdx.x, lane_in_row = tid & (a.lpr - 1), group = tid >> a.lpr_shift, groups = (int)blockDim.x >> a.lpr_shift;
    const int unit0 = blockIdx.x * a.units, units = min(a.units, a.H - unit0);
    float* const sums = lds + 2 * a.vec;         // of the workgroup's rows, four per unit
    int* const stop = reinterpret_cast<int*>(sums + a.units * 4);

    // the weights: row `group + r * groups` of the workgroup (gate i % 4 of unit i / 4) has slots r * U and on
    VRaw v[S];
    uint32_t at[S][kAddr];                       // LDS bytes from the start of [x ; h], two in a word
    {
        IRaw o[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int i = group + s / U * groups, cc = min(lane_in_row + s % U * a.lpr, a.chunks_per_row - 1);
            const uint32_t e = (i < units * 4 ? (uint32_t)((i & 3) * a.H + unit0 + (i >> 2)) * (uint32_t)a.row_len : 0u) + (uint32_t)cc * CH;
            v[s] = *reinterpret_cast<const VRaw*>(static_cast<const char*>(a.vals) + e * (uint32_t)sizeof(VT));
            o[s] = *reinterpret_cast<const IRaw*>(a.idx + e);
            pin_order();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = lane_in_row + u * a.lpr;
            uint32_t bank[CH];                   // of an entry: its bank's first place
#pragma unroll
            for (int j = 0; j < CH; ++j) bank[j] = div_magic((uint32_t)(c * CH + j), (uint32_t)a.k, a.magic_k) * (uint32_t)a.B;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int s = r * U + u;
                const bool there = group + r * groups < units * 4 && c < a.chunks_per_row;     // else: zero times the zero behind [x ; h]
                if (!there) v[s] = zero_raw<VRaw>();
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const uint32_t b = there ? (bank[j] + offset_at(o[s], j)) * 4u : (uint32_t)(a.H + a.I) * 4u;
                    if (j & 1) at[s][j / 2] |= b << 16;
                    else at[s][j / 2] = b;
                }
                pin_order();
            }
        }
    }
    float cell = 0.f;
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < units) {
        const int unit = unit0 + tid;
        cell = a.c[unit];
        bias = make_float4(a.bias[unit], a.bias[a.H + unit], a.bias[2 * a.H + unit], a.bias[3 * a.H + unit]);
    }
    if (tid == 0) *stop = 0;
    if (tid < 2) lds[tid * a.vec + a.H + a.I] = 0.f;
    const int x4 = a.I >> 2;
    float4 xr = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < x4) {
        reinterpret_cast<float4*>(lds)[tid] = reinterpret_cast<const float4*>(a.X)[tid];
        if (a.T > 1) xr = reinterpret_cast<const float4*>(a.X + a.I)[tid];
    }
    __syncthreads();

    // Values and addresses are unpacked where they are used: the compiler would do so once, ahead of the loop, and spill.
    auto keep = [&]() {
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int j = 0; j < kAddr; ++j) asm volatile("" : "+v"(at[s][j]));
            if constexpr (sizeof(VT) == 2) keep_packed(v[s]);
        }
    };
    uint32_t base = 0;                           // LDS bytes of this step's [x ; h]
    const uint32_t other = (uint32_t)a.vec * 4u;
    for (int64_t t = 0; t < a.T; ++t, base ^= other) {
        const char* const xh = reinterpret_cast<const char*>(lds) + base;
        keep();
        float part[S];
        auto dot = [&](int s) {
            float p = 0.f;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const uint32_t b = (j & 1) ? at[s][j / 2] >> 16 : at[s][j / 2] & 0xffffu;
                p = fmaf(value_at<VT>(v[s], j), *reinterpret_cast<const float*>(xh + b), p);
            }
            return p;
        };
        // what needs only x, the same slots in every lane: scalar branches
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (s % U < a.x_slots) part[s] = dot(s);
        keep();
        pin_order();
        // the hidden state of the step before
        {
            uint64_t* const to = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(lds) + base + (uint32_t)a.I * 4u);
            const uint64_t* from = reinterpret_cast<const uint64_t*>(t == 0 ? a.h0 : a.H_all + (t - 1) * a.H);
            int looks = a.wait_looks;            // left to this lane in this step
            for (int i = tid; i < (a.H >> 1) && looks >= 0; i += (int)blockDim.x) {
                uint64_t w;
                if (t == 0) {
                    w = from[i];
                } else {
                    for (;;) {
                        w = __hip_atomic_load(from + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (lstm_there(max((uint32_t)w, (uint32_t)(w >> 32)))) break;
                        if ((uint32_t)w == kGivenUp || (uint32_t)(w >> 32) == kGivenUp) looks = 0;
                        if (--looks < 0) {
                            *stop = 1;
                            break;
                        }
                    }
                }
                to[i] = w;
            }
        }
        lds_barrier();
        const int stopped = *stop;
        // x of the next step to the other copy, which nobody reads any more; the one after that is on its way
        if (tid < x4 && t + 1 < a.T) {
            *reinterpret_cast<float4*>(reinterpret_cast<char*>(lds) + (base ^ other) + tid * 16) = xr;
            if (t + 2 < a.T) xr = reinterpret_cast<const float4*>(a.X + (t + 2) * a.I)[tid];
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (s % U >= a.x_slots) part[s] = dot(s);
        float sum[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sum[r] = part[r * U];
#pragma unroll
            for (int u = 1; u < U; ++u) sum[r] += part[r * U + u];
        }
        lstm_row_sums(sum, a.lpr);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (lane_in_row == 0 && group + r * groups < a.units * 4) sums[group + r * groups] = sum[r];
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(stopped)) {   // the same in every wavefront: written only ahead of the first barrier
            if (tid < units)
                __hip_atomic_store(reinterpret_cast<uint32_t*>(a.H_all) + t * a.H + unit0 + tid, kGivenUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (tid < units) {
            const float h = lstm_cell(reinterpret_cast<const float4*>(sums)[tid], bias, cell);
            __hip_atomic_store(reinterpret_cast<uint32_t*>(a.H_all) + t * a.H + unit0 + tid, __builtin_bit_cast(uint32_t, h), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (tid < units) a.c[unit0 + tid] = cell;
}

// What lstm_seq_kernel left out, if anything: one workgroup.  Units whose last row is there are finished, their cell state
// included; the others have theirs as it was before step 0.  A step passes all weights through one compute unit, so the
// chunks of several rows are in flight together, and the banks of a lane's operands are counted once: a step of
// 1500 / 1024 / 512 / 128 units takes 156 / 90 / 24 / 3.0 us (entry by entry 748 / 385 / 84 / 8.2; in lstm_seq_kernel 1.2 to 2.0).
template <typename VT, int CH, int U>
__global__ __launch_bounds__(kLstmFinishThreads) void lstm_finish_kernel(LstmSeqArgs a) {
    extern __shared__ __align__(16) float lds[];
    using VRaw = typename RawBytes<CH * sizeof(VT)>::type;
    using IRaw = typename IdxChunk<uint8_t, CH>::type;
    constexpr int R = 8 / U;
    const int tid = threadIdx.x, lane_in_row = tid & (a.lpr - 1), group = tid >> a.lpr_shift, groups = (int)blockDim.x >> a.lpr_shift;
    const uint32_t* const last = reinterpret_cast<const uint32_t*>(a.H_all) + (a.T - 1) * a.H;
    int missing = 0;
    for (int u = tid; u < a.H; u += kLstmFinishThreads) missing |= !lstm_there(last[u]);
    if (!__syncthreads_or(missing)) return;

    float* const sums = lds + a.vec;
    uint8_t* const todo = reinterpret_cast<uint8_t*>(sums + 4 * a.H);
    for (int u = tid; u < a.H; u += kLstmFinishThreads) todo[u] = !lstm_there(last[u]);
    uint32_t bank[U][CH];                        // of an entry: its bank's first place in [x ; h]
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < CH; ++j)
            bank[u][j] = div_magic((uint32_t)(min(lane_in_row + u * a.lpr, a.chunks_per_row - 1) * CH + j), (uint32_t)a.k, a.magic_k) * (uint32_t)a.B;
    for (int64_t t = 0; t < a.T; ++t) {
        const float* const h_in = t == 0 ? a.h0 : a.H_all + (t - 1) * a.H;
        for (int i = tid; i < a.I; i += kLstmFinishThreads) lds[i] = a.X[t * a.I + i];
        for (int i = tid; i < a.H; i += kLstmFinishThreads) lds[a.I + i] = h_in[i];
        __syncthreads();
        // row i is gate i % 4 of unit i / 4: the lanes of a row are of one mind, those of a wavefront need not be
        for (int i0 = group; i0 < 4 * a.H; i0 += R * groups) {
            VRaw v[R][U];
            IRaw o[R][U];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = min(i0 + r * groups, 4 * a.H - 1);
                if (!todo[i >> 2]) continue;
                const uint32_t row = (uint32_t)((i & 3) * a.H + (i >> 2)) * (uint32_t)a.row_len;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t e = row + (uint32_t)min(lane_in_row + u * a.lpr, a.chunks_per_row - 1) * CH;
                    v[r][u] = *reinterpret_cast<const VRaw*>(static_cast<const char*>(a.vals) + e * (uint32_t)sizeof(VT));
                    o[r][u] = *reinterpret_cast<const IRaw*>(a.idx + e);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = i0 + r * groups;
                if (i >= 4 * a.H || !todo[i >> 2]) continue;
                float sum[1] = {0.f};
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float p = 0.f;
#pragma unroll
                    for (int j = 0; j < CH; ++j) p = fmaf(value_at<VT>(v[r][u], j), lds[bank[u][j] + offset_at(o[r][u], j)], p);
                    if (lane_in_row + u * a.lpr < a.chunks_per_row) sum[0] = u == 0 ? p : sum[0] + p;
                }
                lstm_row_sums(sum, a.lpr);
                if (lane_in_row == 0) sums[i] = sum[0];
            }
        }
        __syncthreads();
        for (int u = tid; u < a.H; u += kLstmFinishThreads) {
            if (!todo[u]) continue;
            const float4 bias = make_float4(a.bias[u], a.bias[a.H + u], a.bias[2 * a.H + u], a.bias[3 * a.H + u]);
            a.H_all[t * a.H + u] = lstm_cell(reinterpret_cast<const float4*>(sums)[u], bias, a.c[u]);
        }
        __syncthreads();                         // of its own workgroup's stores the next step reads
    }
}

// H_all without a hidden state in it (rows are whole pieces of 16 bytes)
static __global__ __launch_bounds__(256) void lstm_absent_kernel(uint4* H_all, int64_t pieces) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pieces; i += (int64_t)gridDim.x * 256)
        H_all[i] = make_uint4(kAbsent, kAbsent, kAbsent, kAbsent);
}

template <typename VT, int CH, int U, int R>
int lstm_seq_launch_one(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st) {
    const int64_t pieces = a.T * a.H / 4;
    if (!p.finish_only) {
        hipLaunchKernelGGL(lstm_absent_kernel, dim3((unsigned)std::min<int64_t>((pieces + 255) / 256, 1024)), dim3(256), 0, st,
                           reinterpret_cast<uint4*>(a.H_all), pieces);
        hipLaunchKernelGGL((lstm_seq_kernel<VT, CH, U, R>), dim3(p.grid), dim3(p.threads), p.lds, st, a);
    }
    hipLaunchKernelGGL((lstm_finish_kernel<VT, CH, U>), dim3(1), dim3(kLstmFinishThreads), p.finish_lds, st, a);
    return hip_status(hipGetLastError());
}

template <typename VT, int CH, int UR = kLstmSeqMost * kLstmSeqMost - 1>
int lstm_seq_launch_slots(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st) {
    constexpr int U = UR / kLstmSeqMost + 1, R = UR % kLstmSeqMost + 1;
    if constexpr (U * R * CH <= kLstmSeqEntries && U * R <= kLstmSeqSlots)
        if (p.slots == U && p.rows == R) return lstm_seq_launch_one<VT, CH, U, R>(p, a, st);
    if constexpr (UR > 0) return lstm_seq_launch_slots<VT, CH, UR - 1>(p, a, st);
    return BS_ERR_UNSUPPORTED;
}

#endif
}  // namespace bs
