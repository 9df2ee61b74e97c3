// Bulk hashing in two passes: hash_screen.h settles most keys, hash_bulk.h hashes the others with the chain.
#include "hash_open.h"

namespace spotlight {
using namespace hashdev;
extern template int run_bulk_hash<bf16_raw, bf16_raw>(spotlight_ctx*, const HashArgs&, int, int);

bool screen_serves(int hidden, int W) { return screen::serves(hidden, W); }

size_t screen_operand_bytes(int hidden, int W)
{
    return screen::serves(hidden, W) && !screen::resident(hidden, W) ? static_cast<size_t>(screen::blocks_of(hidden)) * screen::operands_of(screen::words_for(W)) * 64 * sizeof(uint4) : 0;
}

size_t screen_scale_bytes(int heads, int W) { return screen::scale_bytes(heads, W); }

bool screened_hash_applies(const spotlight_ctx* ctx, const HashArgs& a, int n_xheads) { return screen::applies(ctx, a, n_xheads); }

int run_screened_hash(spotlight_ctx* ctx, const HashArgs& job, int n_xheads, int stage)
{
    HashArgs a = job;
    if (!bulk::counts_open_rows(a, n_xheads, ctx->n_cus)) a.open_counts = nullptr;
    const int rc = screen::launch(ctx, a, n_xheads, stage);
    if (rc != SPOTLIGHT_OK) return rc;
    if (!a.audit && screen::open_serves(a.hidden, a.W)) return screen::launch_open(ctx, a, n_xheads, stage);
    // audited: every row with the chain, which also counts what the first pass settled wrongly
    return a.audit ? run_bulk_hash<bf16_raw, bf16_raw>(ctx, a, n_xheads, stage) : run_open_hash(ctx, a, n_xheads, stage);
}

}  // namespace spotlight
