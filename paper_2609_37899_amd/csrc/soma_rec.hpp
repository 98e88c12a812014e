// soma_rec.hpp -- the exchange recurrence's instances (soma_rec.hip).
#pragma once

namespace soma {

// The k_rec_xchg instance for hidden width H (H % 64 == 0, 128 <= H <= 704),
// the generator family (Rademacher or Gaussian) and the layer (layer 1 reads
// the folded table); nullptr for other widths.
const void* xchg_kernel_for(int H, bool rademacher, bool layer1);

// Its instance on pre-formed weights (H % 64 == 0, H <= 512).
const void* xchg_pre_kernel_for(int H);

}  // namespace soma
