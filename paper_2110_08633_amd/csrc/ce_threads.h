// Choice of the threads per row of the bf16 cross-entropy kernel (host only, no HIP).
#pragma once
#include <stdint.h>

namespace hydra {

// The fewer threads hold a row, the more rows a CU has in flight - if there are more rows than CUs.  With a row per CU or less
// nothing overlaps, and the row itself should be short: us, 1024 threads / 256 or 512: 64 rows of 5000 columns 4.0 / 4.6, of
// 20000 8.0 / 8.6, 256 of 8000 5.8 / 6.2; 288 of 5000 the same, of 20000 12 % faster with 512.  Up to 2048 columns 1024 threads
// have less than a vector each: 64 rows of 1500 3 % faster with 256.
inline int ce_row_threads(int M, int64_t ld) {
  if (ld <= 2048) return 256;
  if (M <= 256) return 1024;
  return ld <= 8192 ? 256 : ld <= 32768 ? 512 : 1024;
}

}  // namespace hydra
