// FP64 instances of the biased wave kernel (cfd_biased_wave.h) for fields of
// 4 GiB and more, compiled on their own so the build runs them in parallel.
#include "cfd_biased_wave.h"

namespace cfd {
const void *biased_big_fn_f64(int hb, int emb) { return wave_fn<double, false, uint64_t>(hb, emb); }
}  // namespace cfd
