// bs_prune_pack and bs_reprune with byte offsets (banks of up to 256 elements); the kernel is
// in bs_prune_pack_kernel.h.
#include "bs_prune_pack_kernel.h"

namespace bs {

int launch_prune_pack(const void* W, int dtype, int64_t M, int64_t K, int bank, int k,
                      void* vals, uint8_t* idx, hipStream_t st) {
    const int64_t n_banks = M * (K / bank);
    if (dtype == BS_F16) return prune_banks<__half, uint8_t>(W, n_banks, bank, k, vals, idx, nullptr, st);
    return prune_banks<float, uint8_t>(W, n_banks, bank, k, vals, idx, nullptr, st);
}

// Re-prune: the k stored values of a bank are a bank of k elements themselves; the
// survivors carry the offsets the packed matrix already holds instead of their slots.
int launch_reprune(const void* vals, const uint8_t* idx, int dtype, int64_t n_banks, int k, int k2,
                   void* vals2, uint8_t* idx2, hipStream_t st) {
    if (dtype == BS_F16) return prune_banks<__half, uint8_t>(vals, n_banks, k, k2, vals2, idx2, idx, st);
    return prune_banks<float, uint8_t>(vals, n_banks, k, k2, vals2, idx2, idx, st);
}

}  // namespace bs
