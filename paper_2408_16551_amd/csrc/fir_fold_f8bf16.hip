// Folded polyphase FIR (values rounded to E4M3, parts in bf16): see fir_fold.h.
#include "fir_fold.h"

namespace tina {
hipError_t launch_fold_f8bf16(const FirArgs& a, hipStream_t s) { return launch_fold_qm<QM_F8BF16>(a, s); }
hipError_t launch_fold_batch_f8bf16(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s) {
    return launch_fold_batch_qm<QM_F8BF16>(t, max_m, split, grid, s);
}
}  // namespace tina
