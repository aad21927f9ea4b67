// Matrix-core variants of the measured configurations for batches whose sequences differ in length.
#include "decode_mfma_table.h"

namespace mixkvq {

bool try_main_table_any_lengths(const GenericArgs& a, hipError_t* err) { return try_main_table<SeqCounts>(a, err); }

}  // namespace mixkvq
