// Instantiates the bulk hash for one (vector type, weight type) pair (see hash_bulk.h).
#include "hash_bulk.h"

namespace spotlight {
template int run_bulk_hash<hashdev::bf16_raw, hashdev::bf16_raw>(spotlight_ctx*, const hashdev::HashArgs&, int, int);
}  // namespace spotlight
