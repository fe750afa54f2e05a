// Prints the decode plans of the built library, for tests that run without a GPU: one problem per
// input line, "batch n_q_heads n_kv_heads n_kept bits group outliers decode_splits workspace_bytes key_axis counts"
// (workspace_bytes 0: as many as the library states; counts 0: the priced plan itself, 1: as a call launches it on a cache of
// equal heads, 2: on a cache with head-level counts), one answer per line, "accepted n_splits n_waves
// part_bytes part_off counter_bytes stated_bytes half chunks_per_split least_bytes".
// Test infrastructure only.
#include <cstdio>

#include "kvqp_internal.h"

int main() {
    int batch, hq, hkv, n, bits, group, outliers, splits, axis, counts;
    size_t bytes;
    while (std::scanf("%d %d %d %d %d %d %d %d %zu %d %d", &batch, &hq, &hkv, &n, &bits, &group, &outliers, &splits, &bytes, &axis, &counts) == 11) {
        kvqp_cfg c{};
        c.batch = batch; c.n_q_heads = hq; c.n_kv_heads = hkv; c.head_dim = 128; c.bits = bits; c.group_size = group;
        c.key_axis = axis;
        c.outlier_threshold = outliers ? 6.0f : 0.0f; c.decode_splits = splits; c.sm_scale = 0.088f;
        const size_t stated = kvqp::decode_ws_bound(c);
        kvqp::DecodePlan p = kvqp::plan_decode(c, n);
        if (counts == 1) p.take_half();
        if (counts == 2) p.take_plain();
        const size_t least = p.least_bytes();
        const bool ok = p.fit(bytes ? bytes : stated);
        std::printf("%d %d %d %zu %zu %zu %zu %d %d %zu\n", (int)ok, p.n_splits, p.n_waves, p.part_bytes, p.part_off,
                    kvqp::decode_ws_header_bytes(c), stated, (int)p.half, p.chunks_per_split, least);
    }
    return 0;
}
