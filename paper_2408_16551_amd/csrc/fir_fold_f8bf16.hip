// Folded polyphase FIR (values rounded to E4M3's four significant bits, parts in
// bf16): see fir_fold.h.  Instantiated apart from BF16: with the rounding behind a
// branch of the same kernels both forms lose where the ring is long (2048 complex
// channels, 12 taps, 2^25 samples 260 -> 317 us; 512, 24 taps, 2^24 200 -> 281).
#include "fir_fold.h"

namespace tina {
hipError_t launch_fold_f8bf16(const FirArgs& a, hipStream_t s) { return launch_fold_qm<QM_F8BF16>(a, s); }
hipError_t launch_fold_batch_f8bf16(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s) {
    return launch_fold_batch_qm<QM_F8BF16>(t, max_m, split, grid, s);
}
}  // namespace tina
