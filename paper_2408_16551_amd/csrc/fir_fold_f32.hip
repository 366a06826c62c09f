// Folded polyphase FIR (FP32 parts): see fir_fold.h.
#include "fir_fold.h"

namespace tina {
hipError_t launch_fold_f32(const FirArgs& a, hipStream_t s) { return launch_fold_qm<QM_NONE>(a, s); }
hipError_t launch_fold_batch_f32(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s) {
    return launch_fold_batch_qm<QM_NONE>(t, max_m, split, grid, s);
}
}  // namespace tina
