// Whole LSTM sequences on binary16 values (see bs_lstm_seq_kernel.h for the design).
#include "bs_lstm_seq_kernel.h"

namespace bs {
int lstm_seq_launch_f16(const LstmSeqPlan& p, const LstmSeqArgs& a, hipStream_t st) {
    switch (p.ch) {
        case 8: return lstm_seq_launch_slots<__half, 8>(p, a, st);
        case 4: return lstm_seq_launch_slots<__half, 4>(p, a, st);
        case 2: return lstm_seq_launch_slots<__half, 2>(p, a, st);
        case 1: return lstm_seq_launch_slots<__half, 1>(p, a, st);
    }
    return BS_ERR_UNSUPPORTED;
}
}  // namespace bs
