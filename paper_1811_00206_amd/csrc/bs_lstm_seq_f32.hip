// Whole LSTM sequences on fp32 values (see bs_lstm_seq_kernel.h for the design).
#include "bs_lstm_seq_kernel.h"

namespace bs {
int lstm_seq_launch_f32(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st) {
    switch (p.ch) {
        case 4: return lstm_seq_launch_slots<float, 4>(p, a, st);
        case 2: return lstm_seq_launch_slots<float, 2>(p, a, st);
        case 1: return lstm_seq_launch_slots<float, 1>(p, a, st);
    }
    return BS_ERR_UNSUPPORTED;
}
}  // namespace bs
