// Arguments of the key-stationary pass of the backward (dK / dV).
#pragma once
#include "moc_attn_common.h"

namespace moc {

struct KvArgs {
    const void *q, *k, *v, *d_o;
    // per query (lse * log2(e), delta), an extra pair (+inf, 0) at the end; beside wide tiles records of four words (see store_stats)
    const float *stats2;
    const float *gstats2;              // the same gathered in the order of the inverse lists
    void *dk, *dv;
    float *tpart_k, *tpart_v;
    const KvItem *items;
    const int32_t *list_off, *qlist;
    int N, C, topk, n_partials, BH;
    int n_items, n_text;               // work list of a head: items, caption items among them (of `join` segments each)
    int text_tiles, join, text_seg, video_at;    // caption tiles; queries of `join` segments; first video item of `items`
    int key_tile;                      // rows of a partial
    float scale, scale_log2;
};

hipError_t launch_dkdv_wide(const KvArgs &kv, int dtype, hipStream_t st);

}  // namespace moc
