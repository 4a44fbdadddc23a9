// Batched list scan of 3 stored bits per coordinate.
#include "batch_scan.h"

namespace ivftq {

hipError_t batch_scan_b3(const BatchScanArgs& a, int dp, hipStream_t st) { return run_batch_width<3>(a, dp, st); }

}  // namespace ivftq
