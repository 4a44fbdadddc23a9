// Batched list scan of 8 stored bits per coordinate.
#include "batch_scan.h"

namespace ivftq {

hipError_t batch_scan_b8(const BatchScanArgs& a, int dp, hipStream_t st) { return run_batch_width<8>(a, dp, st); }

}  // namespace ivftq
