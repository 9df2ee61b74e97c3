// Instantiates the bulk hash for one (vector type, weight type) pair (see hash_bulk.h).
#include "hash_bulk.h"

namespace spotlight {
template int run_bulk_hash<float, float>(spotlight_ctx*, const hashdev::HashArgs&, int, int);
}  // namespace spotlight
