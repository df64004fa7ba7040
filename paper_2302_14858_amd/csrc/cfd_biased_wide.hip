// FP64 instances of the biased wave kernel (cfd_biased_wave.h) for x lines of
// more than 64 columns, compiled on their own so the build runs them in parallel.
#include "cfd_biased_wave.h"

namespace cfd {
const void *biased_wide_fn_f64(int hb, int emb) { return wave_fn<double, true, uint32_t>(hb, emb); }
}  // namespace cfd
