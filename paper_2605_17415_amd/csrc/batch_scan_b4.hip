// Batched list scan of 4 stored bits per coordinate.
#include "batch_scan.h"

namespace ivftq {

hipError_t batch_scan_b4(const BatchScanArgs& a, int dp, hipStream_t st) { return run_batch_width<4>(a, dp, st); }

}  // namespace ivftq
