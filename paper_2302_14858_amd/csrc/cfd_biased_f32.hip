// FP32 instances of the biased wave kernel (cfd_biased_wave.h), compiled on
// their own so the build runs both types in parallel.
#include "cfd_biased_wave.h"

namespace cfd {
const void *biased_wave_fn_f32(int hb, int emb) { return wave_fn<float, false, uint32_t>(hb, emb); }
}  // namespace cfd
