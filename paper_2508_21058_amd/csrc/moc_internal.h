// Host-side structures and kernel launchers of libmoc (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "../../include/moc.h"

namespace moc {

constexpr int kBM = 128;         // queries per workgroup in the query-stationary passes
// Keys per workgroup in the key-stationary pass: 4 score waves of 32, or, where whole tiles of calls with many of them go
// to the kernel of their own, 4 waves of 64.
constexpr int kKeyTile = 128, kWideTile = 256;
constexpr int kWideMin = 160;    // fewer keys left of a chunk go to the other kernel (one of four waves of 64 would idle, another be half empty)
constexpr int kWideFull = 193;   // from here on a wide tile fills all four waves
// Queries per partial of a text key tile in the key-stationary pass. A caption tile is attended by all
// N queries, so its items are the longest of the pass: a quarter of the stream keeps the longest item
// well under a compute unit's share of short streams (6,256 tokens: a whole-stream item is 196 steps
// where a video item is 33 and a unit's share 182), 16384 bounds the partials of long ones (4096, 8192
// and 16384 take the same time there), 256 keeps a segment's partial cheaper than its products.
constexpr int kTextSegMin = 256, kTextSegMax = 16384, kTextItems = 512;
inline int text_segments(int N) {
    const int target = N / 4 < kTextSegMin ? kTextSegMin : (N / 4 > kTextSegMax ? kTextSegMax : (N + 3) / 4);
    return (N + target - 1) / target;
}
// Neighbouring segments of a caption tile that one workgroup walks, leaving one partial for all of them. Segments
// balance calls of few caption items; where a call has an item per compute unit anyway, more partials (a tile in
// fp32 each, written and summed) only cost. So a tile keeps as many as leave fewer than two items per unit (but
// no more than kTextSegMax queries in one). dK/dV and the sums of the partials with four partials a tile / with this rule (one
// where not given): 16 heads of 10k tokens with a 2,000-token caption (256 whole-stream items) 576 / 533 us, 32 heads
// 1,156 / 1,068, eight 300-token captions of 24 heads (576) 1,568 / 1,507; six heads of them (144, four partials)
// 294, with two 323.
inline int text_join(int N, int n_tiles, int BH, int nseg) {
    const long long items = (long long)n_tiles * BH;
    int want = items > 0 ? (int)std::min<long long>((kTextItems - 1) / items, nseg) : 1;
    want = std::max(std::max(want, 1), (N + kTextSegMax - 1) / kTextSegMax);
    return std::max(1, nseg / want);
}
constexpr int kRowsPerBlk = 256, kRowsPerBlkMin = 64;   // queries per block of the list builder (one wave and one histogram row each)
constexpr int kMaxListChunks = 16384;   // chunks the list builder's LDS histogram holds

// One query tile of the forced-link pass: queries [q_start, q_start+q_count)
// all belong to window `win` and share its key ranges.
struct AnchorTile { int32_t q_start, q_count, win, pad; };

// A contiguous key range [start, start+len).
struct KeyRange { int32_t start, len; };

// One workgroup of the key-stationary backward pass.
//   keys [key_start, key_start+key_len), key_len <= kKeyTile, or kWideTile in the list of wide tiles
//   contiguous query source [q_start, q_start+q_len)
//   chunk >= 0: additionally the routed-query list of that chunk
//   partial >= 0: write fp32 partial sums to that slot instead of dk/dv
struct KvItem { int32_t key_start, key_len, q_start, q_len, chunk, partial, pad0, pad1; };

// A text key tile and the partial slots to sum for it.
struct TextTile { int32_t key_start, key_len, first_partial, n_partials; };

// A work list of the key-stationary pass: n_text caption items, then the video items.
struct KvList {
    int32_t n_items = 0, n_text = 0, n_text_tiles = 0;
    KvItem *d_items = nullptr;
};
// The caption tiles of a pass and the rows of partials they need.
struct TextTiles {
    int32_t n = 0, n_partials = 0;
    TextTile *d = nullptr;
};

}  // namespace moc

struct moc_meta {
    int32_t N = 0, C = 0, T = 0, W = 0;
    int32_t n_atiles = 0, n_ranges = 0;
    int32_t text_seg = 0;            // queries per caption item (the last of a tile may have fewer)
    int32_t max_routed_len = 0;      // longest chunk that is not a caption
    void *d_base = nullptr;
    size_t d_bytes = 0;
    int32_t *d_off = nullptr;        // [C+1]
    int32_t *d_kind = nullptr;       // [C] 1 = text
    int32_t *d_win = nullptr;        // [C] dense window id
    int32_t *d_rwin = nullptr;       // [C] window id of a video chunk, -1 for a caption chunk
    int32_t *d_wfirst = nullptr;     // [W] first chunk of window
    int32_t *d_wlast = nullptr;      // [W] last chunk of window (inclusive)
    int32_t *d_chunk_of = nullptr;   // [N]
    uint32_t *d_textmask = nullptr;  // [ceil(C/32)] bit j%32 of word j/32 set: chunk j is text
    int32_t *d_ntb = nullptr;        // [C+1] number of non-text chunks with index < j
    int32_t *d_video = nullptr;      // the non-text chunks, ascending
    int32_t *d_arange_off = nullptr; // [W+1] into d_aranges
    moc::KeyRange *d_aranges = nullptr;
    moc::AnchorTile *d_atiles = nullptr;
    moc::KvList kv_all, kv_wide, kv_rest;      // every tile of kKeyTile keys; tiles of kWideTile, and what they leave
    moc::TextTiles tt_all, tt_wide;            // caption tiles of kv_all; of kv_wide and kv_rest
    int64_t wide_queries[2] = {};              // forced queries of the wide tiles of kWideFull keys and more, and of the others
    int32_t wide_video[2] = {};                // ... and how many of them are not captions'
    int32_t n_video = 0;                       // chunks that are not captions
    std::vector<int32_t> h_off, h_kind, h_win;
};

namespace moc {

// Optional per-kernel timing with HIP events on the launch stream (off by
// default; switched on through moc_prof_enable). A Scope brackets one launch and closes its own record, so scopes
// may nest or overlap those of another thread.
bool prof_on();
hipEvent_t prof_begin(const char *name, hipStream_t st);      // -> the event that ends the record
void prof_end(hipEvent_t end, hipStream_t st);
struct ProfScope {
    hipStream_t st;
    hipEvent_t end;
    ProfScope(const char *name, hipStream_t s) : st(s), end(prof_on() ? prof_begin(name, s) : nullptr) {}
    ~ProfScope() { if (end) prof_end(end, st); }
};
#define MOC_PROF(name, st) ::moc::ProfScope moc_prof_scope_(name, st)

// Drop-off / drop-in on rows of width topk + max_in whose first topk columns hold the routed chunks.
hipError_t launch_perturb(const moc_meta *m, int BH, int topk, int max_in, int causal, float p_max,
                          const uint64_t *thr, uint64_t seed, int32_t *sel, hipStream_t st);

// Outer-loop routing over [N, D] features: per-segment means, scores against segment g, top-M on the device.
constexpr int kMaxSegments = 4096;
hipError_t launch_outer(int D, int dtype, const void *x, int P, int max_tiles, int g, int M, const int32_t *d_seg_off,
                        const int32_t *d_tile_base, const int32_t *d_cand, float *partial, float *mean,
                        float *scores, int32_t *d_selected, hipStream_t st);
// dst[o][..] = rows of src[o] listed by `n_ranges` host records; d_ranges: device room for them (used when
// they are too many to travel with the launch; the records must then outlive the copy).
struct GatherRange { int32_t src, len, dst, pad; };
constexpr int kGatherArgRanges = 64;
struct GatherTable { GatherRange r[kGatherArgRanges]; };
hipError_t launch_gather(int outer, long long n_src_rows, long long n_dst_rows, int row_bytes, const void *src,
                         void *dst, const GatherRange *ranges, int n_ranges, void *d_ranges, hipStream_t st);

// Machine probes (streaming copy, MFMA loop); see moc_probe.
constexpr int kProbeMfmaGrid = 256;
hipError_t launch_probe(int kind, void *buf, size_t bytes, int iters, hipStream_t st, hipEvent_t e0, hipEvent_t e1,
                        double *units);

// Whether the key-stationary pass takes the wide tiles: only with heads of 128 features, and where the items are many rounds
// of the chip, since they are twice as long as the others', and more where a second launch has to take what they leave.
// dK/dV without them / with them, at so many wide items, us. Nothing left: 546 items (23k tokens, six heads, 1,280-key
// chunks) 3,180 / 3,455, 576 (6k, 24 heads, 256-key) 291 / 312, 720, 996 and 1,248 (15k to 27k, twelve heads, 256-key) 304 / 330,
// 403 / 462 and 517 / 495, 1,456 (23k, 16 heads, 256-key) 926 / 912, 1,512 (16k, 24 heads, 1,280-key) 1,402 / 1,325, 2,184 (23k, 24
// heads, 1,280-key) 11,557 / 10,635. With a rest: 660 (14k, 12 heads, 260-key) 613 / 672, 1,320 (29k, 12 heads, 260-key) 1,698 / 1,774,
// 2,208 (57k, 12 heads, 312-key) 3,019 / 3,166, 2,976 (41k, 24 heads, ragged) 3,322 / 3,219, 7,008 (57k, 24 heads, 195-key) 5,687 / 5,269.
// The line does not look at how much of the work the rest is. Where that is much, either kernel may be ahead by a part of a round
// (24 heads, k = 4, own-chunk windows, 2,640 and 6,000 items: chunks of 256 and 128 keys in turn 1,099 / 1,172 and 2,435 / 2,495, of 256
// and 130 1,642 / 1,436 and 4,288 / 3,316, of 256 and eight times 64 1,819 / 1,859 and 4,186 / 4,284, of 256, 64 and 64 1,071 / 936 and
// 2,490 / 2,121; 2,640 of them in one window 38,028 / 37,601, 45,354 / 45,405, 202,330 / 187,856 and 43,313 / 42,002).
constexpr int kWideItems = 1408, kWideItemsRest = 2560;
// A tile of three filled waves costs what a full one does. On long contiguous streams of queries that is more than the two items of the
// other kernel it stands for: 24 heads, 120 chunks of 160, 176, 192 keys in one window, k = 1, 10.3 / 11.6, 11.8 / 12.6, 13.1 / 13.9 ms (208 and
// 224 keys 15.8 / 15.4, 16.9 / 16.5); 32 captions of 160 keys and 130-key chunks, 454k tokens, six heads, 19.8 / 21.7. On gathered lists it is
// less: windows of a chunk, k = 4, 250 chunks of them 1,353 / 1,322, 1,489 / 1,419, 1,565 / 1,564 us. So the queries that full tiles stream,
// and half of those in the lists of the others, have to be as many as there are in the windows of the others. With 16 captions of 256 keys,
// 229k tokens, twelve heads, 160-, 180- and 192-key chunks 14.0 / 13.0, 13.9 / 12.9, 13.8 / 12.8 ms, k = 16 20.7 / 20.7, 21.3 / 20.6, 21.2 / 20.6; in
// windows of 14k tokens, which the line leaves to the other kernel, 55.8 / 57.0, 54.3 / 53.1, 51.8 / 50.7.
inline bool wide_tiles(const moc_meta *m, int BH, int d, int topk) {
    if (d != 128 || (long long)m->kv_wide.n_items * BH < (m->kv_rest.n_items > 0 ? kWideItemsRest : kWideItems)) return false;
    const long long list = m->n_video > 0 ? (long long)m->N * topk / m->n_video : 0;        // of a chunk, on average
    return 2 * (m->wide_queries[0] + m->wide_video[0] * list) + m->wide_video[1] * list >= 2 * m->wide_queries[1];
}

// Layout of the attention workspace (byte offsets); shared by fwd and bwd.
struct AttnWs {
    size_t cnt, list_off, tile_off, vmask, gsum, cnt_blk, qlist, plse, po, cnt_fine, cvt, delta, stats2, gstats2, tpart_k, tpart_v, total;
};
AttnWs attn_ws_layout(const moc_meta *m, int BH, int d, int topk, int dtype, bool with_bwd);

// Route workspace: pooled keys split into three bf16 planes (hi, mid, lo with
// hi + mid + lo == the fp32 value), [BH][3][Cpad][d], Cpad = C rounded up to 32, pad rows zero.
struct RouteWs { size_t kb_split, total; int Cpad; };
RouteWs route_ws_layout(const moc_meta *m, int BH, int d, int topk, int dtype);

hipError_t launch_chunk_of(const moc_meta *m, hipStream_t st);

hipError_t launch_pool(const moc_meta *m, int BH, int d, int dtype, const void *k, float *kbar, void *kb_split,
                       int Cpad, hipStream_t st);

hipError_t launch_route(const moc_meta *m, int BH, int d, int dtype, const void *q, const void *kb_split, int Cpad,
                        int topk, int causal, int32_t *sel, int sel_stride, hipStream_t st);

// pooling + scoring + top-k in one launch (bf16 storage); see route_fused_kernel
hipError_t launch_route_fused(const moc_meta *m, int BH, int d, const void *q, const void *k, float *kbar,
                              void *kb_split, int Cpad, int topk, int causal, int32_t *sel, hipStream_t st);
hipError_t fused_wait_flag(int *timed_out);

// bf16 copies of `count` (0: none) fp32 tensors of n elements each (n a multiple of 8), back to back in `out`. They ride
// with a launch that does not need them, as its last workgroups: per_tensor of them a tensor.
struct CvtArgs {
    const float *x[3] = {};
    void *out = nullptr;
    size_t n = 0;
    int count = 0;
    uint32_t per_tensor = 0;
};
constexpr int kCvtUnroll = 4;           // words of 8 elements a thread
inline CvtArgs cvt_args(const void *x0, const void *x1, const void *x2, void *out, size_t n) {
    CvtArgs c;
    c.x[0] = static_cast<const float *>(x0); c.x[1] = static_cast<const float *>(x1); c.x[2] = static_cast<const float *>(x2);
    c.out = out; c.n = n; c.count = x2 ? 3 : 2;
    return c;
}
// the workgroups of `threads` threads it adds to a launch
inline uint32_t cvt_grid(CvtArgs &c, int threads) {
    const size_t per_wg = (size_t)threads * kCvtUnroll * 8;
    c.per_tensor = (uint32_t)((c.n + per_wg - 1) / per_wg);
    return c.per_tensor * c.count;
}
// ... in a launch of their own
hipError_t launch_to_bf16(CvtArgs c, hipStream_t st);

// room for the histograms of the list builder's two launches, in calls that take them
size_t list_fine_bytes(const moc_meta *m, int BH, int topk);
// counts -> offsets -> inverse lists (per head and chunk: the queries that routed to it); cvt: conversions that ride
// with its first launch
hipError_t launch_build_lists(const moc_meta *m, int BH, int topk, const int32_t *sel, char *ws,
                              const AttnWs &L, CvtArgs cvt, hipStream_t st);

// (both read the lists and the slot masks launch_build_lists left in the workspace)
hipError_t launch_attn_fwd(const moc_meta *m, int BH, int d, int dtype, const void *q, const void *k,
                           const void *v, int topk, float scale, void *o, float *lse, char *ws, const AttnWs &L,
                           hipStream_t st);

hipError_t launch_attn_bwd(const moc_meta *m, int BH, int d, int dtype, const void *q, const void *k,
                           const void *v, const void *o, const float *lse, const void *d_o, int topk, float scale,
                           void *dq, void *dk, void *dv, char *ws, const AttnWs &L, hipStream_t st);

}  // namespace moc
