// Batched list scan of 5 stored bits per coordinate.
#include "batch_scan.h"

namespace ivftq {

hipError_t batch_scan_b5(const BatchScanArgs& a, int dp, int max_tiles, hipStream_t st) { return run_batch_width<5>(a, dp, max_tiles, st); }

}  // namespace ivftq
