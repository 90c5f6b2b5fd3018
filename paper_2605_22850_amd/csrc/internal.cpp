// What the tests ask of the library's dispatch rules (no GPU needed).  Not
// part of the C ABI.
#include <algorithm>

#include "common.hpp"

using namespace oc;

extern "C" {

// Whether the few-row kernels take a product, and how many ranges they split
// its K into.
int oc_internal_gemm_rows(int64_t M, int64_t K, int64_t N, int has_workspace, int64_t *n_split) {
    const bool ours = gemm_rows_applies(M, K, N, has_workspace != 0);
    *n_split = ours ? gemm_rows_splits(M, K, N) : 0;
    return ours;
}

// The plan of one request's attention: out = tile rows, row tiles, key blocks,
// splits, blocks per split.  An oc_status.
int oc_internal_attention_plan(const oc_layout *layout, int64_t prefix_tokens, int64_t suffix_tokens, int64_t *out) {
    AttnPlan p;
    const int rc = check_attention_args(*layout, prefix_tokens, suffix_tokens, &p);
    if (rc) return rc;
    const int64_t v[5] = {p.tile_rows, p.m_tiles, p.n_blocks, p.n_split, p.blocks_per_split};
    std::copy(v, v + 5, out);
    return OC_OK;
}

// The same of n requests whose attention is one launch, five values each.
int oc_internal_attention_batch_plan(const oc_layout *layout, int32_t n, const int64_t *prefix_tokens,
                                     const int64_t *suffix_tokens, int64_t *out) {
    if (n < 1 || n > MAX_ATTN_BATCH) return OC_EINVAL;
    AttnPlan p[MAX_ATTN_BATCH];
    const int rc = plan_attention_batch(*layout, prefix_tokens, suffix_tokens, n, p);
    for (int32_t i = 0; i < n && !rc; ++i) {
        const int64_t v[5] = {p[i].tile_rows, p[i].m_tiles, p[i].n_blocks, p[i].n_split, p[i].blocks_per_split};
        std::copy(v, v + 5, out + 5 * i);
    }
    return rc;
}

// The row tiles in the order of an attention launch's workgroups: out[2 * w]
// the (KV head, split) group and out[2 * w + 1] the row tile of workgroup w, -1
// where it has none.  Returns the number of workgroups; fills at most `max`.
int64_t oc_internal_attention_tiles(int32_t tile_rows, int32_t m_tiles, int32_t nkv, int32_t n_split, int32_t *out,
                                    int64_t max) {
    AttnPlan p{};
    p.tile_rows = tile_rows;
    p.m_tiles = m_tiles;
    p.nkv = nkv;
    p.n_split = n_split;
    const int64_t n = attention_grid(p);
    for (int64_t w = 0; w < n && w < max; ++w) {
        int group, mt;
        const bool has = attention_tile((int)w, p, &group, &mt);
        out[2 * w] = has ? group : -1;
        out[2 * w + 1] = has ? mt : -1;
    }
    return n;
}

// LDS that an attention workgroup holds, and what an ingest workgroup next to it
// reserves.
void oc_internal_lds(int32_t tile_rows, int32_t head_dim, int64_t *attention, int64_t *ingest) {
    AttnPlan p{};
    p.tile_rows = tile_rows;
    p.d = head_dim;
    *attention = (int64_t)attention_lds_bytes(p);
    *ingest = (int64_t)ingest_reservation(attention_lds_bytes(p));
}

// VGPRs of an attention kernel and of the ingest kernel that runs next to it (a
// GPU must be present).
void oc_internal_registers(int32_t tile_rows, int32_t head_dim, int pow2_ingest, int32_t *attention, int32_t *ingest) {
    AttnPlan p{};
    p.tile_rows = tile_rows;
    p.d = head_dim;
    *attention = attention_registers(p);
    *ingest = ingest_registers(pow2_ingest != 0);
}

}  // extern "C"
