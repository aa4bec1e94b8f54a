// Work-item decoding and global->LDS staging shared by the attention passes.
#pragma once
#include "moc_device.h"
#include "moc_internal.h"

namespace moc {

// compile-time integer tag (selects an LDS buffer in the unrolled pipelines)
template <int V> struct IC { static constexpr int value = V; };

constexpr int MODE_ANCHOR = 0;  // forced links: window query tile x (text spans + window)
constexpr int MODE_ROUTED = 1;  // routed links: gathered queries of a chunk x that chunk

// Arguments of the query-stationary passes (forward, and dQ of the backward).
struct FwdArgs {
    const void *q, *k, *v;
    bf16_t *po;        // [BH, N, slots, D] partial outputs (forward) / partial dQ (backward)
    float *plse;       // [BH, N, slots]   partial log-sum-exp (forward only)
    int N, C, topk, slots;
    int BH, items_per_head;   // work list of the launch: items_per_head entries per (batch, head)
    float scale, scale_log2;
    const AnchorTile *atiles;
    const int32_t *arange_off;
    const KeyRange *aranges;
    const int32_t *off, *list_off, *tile_off, *qlist;
    // backward only
    const void *d_o;
    const float *lse, *delta;
    const float *gstats2;   // [BH, N*topk] (lse * log2 e, delta) in inverse-list order: pairs, with `rec` the first two words of records
    // sums of the caption tiles' partials, which the last workgroups of the forced-link dQ launch make
    const float *tpart_k, *tpart_v;
    const TextTile *text_tiles;
    void *dk, *dv;
    int n_text_tiles, n_partials, join, reduce_at, key_tile;
    bool rec;               // statistics in records of four words (see store_stats)
    // forced-link forward items with the merge fused into their epilogue
    int slice_heads;        // see heads_per_slice
    const uint32_t *vmask;  // [BH, N] bit r: routed slot r of the query counts (set by the list builder)
    void *o_out;            // [BH, N, D] final output, in the caller's storage type
    float *lse_out;         // [BH, N] final log-sum-exp
};

// Chunk-stationary routed items (forward and dQ pass): a workgroup keeps the keys and values of one
// chunk in LDS and serves a group of that chunk's query tiles from them.
// Resident keys, of K and of V: 144 KB of LDS at d = 128. Only chunks that can be routed to count: captions are
// forced links and may be longer (512-token captions kept a 33k-token layer of 260-key chunks off this path: 7.51 ->
// 7.32 ms a training step with it). At d = 64 twice the rows would fit, but longer chunks gain nothing over the tiled
// kernels there: forward / dQ of 340-key chunks, 24 heads of 114k tokens, k = 8, 3,181 / 3,764 us in 576 resident rows,
// 3,046 / 4,115 tiled; 512-key chunks, 24 heads of 33k, k = 5, 729 / 899 against 593 / 916.
constexpr int kChunkRows = 288;
constexpr int kGroupTiles = 16;       // query tiles (of kBM list entries) per workgroup: they amortise the copy
constexpr int kComputeUnits = 256;
// Which kernels take the routed items. A workgroup of the chunk-stationary ones fills a compute unit and waits
// for its chunk's copy and its first queries with nothing beside it, and its last round is long: they need many
// rounds. The tiled kernels run two independent workgroups on a unit, an item each. Forward + dQ of the routed
// items, chunk-stationary / tiled, at so many query tiles per compute unit (heads of 128 features):
//   13 tiles  (6k tokens, 24 heads, k = 3)   40-key chunks 268 / 158 us, 260-key 227 / 166
//   29 tiles  (10k, 16 heads, k = 6)         409 / 307, 407 / 362
//   66 tiles  (60k, six heads, k = 6)        64-key 871 / 865, 260-key 1,064 / 1,079
//   88 tiles  (24k, 24 heads, k = 5)         1,049 / 981, 1,408 / 1,348
//   95 tiles  (130k, two heads, k = 12)      1,076 / 1,098, 1,480 / 1,548
//   120 tiles (33k, 24 heads, k = 5)         1,416 / 1,365, 1,856 / 1,897
//   293 tiles (200k, six heads, k = 8)       3,451 / 3,731, 4,629 / 5,011
// Smaller groups (one to fourteen tiles) gain on sixteen below 60 tiles, but stay behind the tiled kernels.
constexpr int kStationaryTiles = 92;
inline bool chunk_stationary(const moc_meta *m, int topk, int BH) {
    return m->max_routed_len <= kChunkRows &&
           (long long)m->N * topk * BH >= (long long)kStationaryTiles * kComputeUnits * kBM;
}

// The GPU has 8 XCDs with private L2 caches and hands consecutive workgroups to
// them round-robin. Work lists are ordered so that neighbours share K/V (or
// Q/dO), hence XCD x takes the contiguous slice [x*per, (x+1)*per) of the list.
// Launch ceil(total/8)*8 workgroups on a 1-D grid; returns false for padding.
constexpr int kXcds = 8;
__host__ __device__ inline int xcd_grid(long long total) { return (int)((total + kXcds - 1) / kXcds) * kXcds; }
__device__ __forceinline__ bool xcd_remap(long long total, int &logical) {
    const int L = blockIdx.x;
    const int per = (int)((total + kXcds - 1) / kXcds);
    logical = (L % kXcds) * per + L / kXcds;
    return logical < total;
}
// The forced-link items take the heads of a slice from the last one: the routed launch before them left the partials of an
// XCD's last heads in its L2, and those are then read first. Only where slices are whole heads, and each head's items stay
// in their order, so that the items come in the sequence of sizes they had: which of them end a launch of few items decides
// more than the L2 gives (all items walked backwards: forced forward of sixteen heads of 6,543 tokens in ragged windows
// 74 -> 82 us, of 24 heads of 7,399 tokens 154 -> 136). Forced forward / dQ of 24 heads of 6,256 tokens, k = 3, 84.6 -> 83.3 /
// 100.5 -> 94.4 us, of 32 fp32 heads of 3,577 tokens, k = 8, 104.6 -> 94.0 / 103.9 -> 98.1, forward of 48 heads of 64
// features, 11.6k tokens, k = 11, 286 -> 272; 24 heads of 33k tokens 953 -> 951 / 1,169 -> 1,180, no difference.
inline int heads_per_slice(int BH) { return BH % kXcds == 0 ? BH / kXcds : 0; }      // 0: slices are not whole heads
__device__ __forceinline__ int head_from_last(int bh, int per_slice) {
    return per_slice ? (int)(blockIdx.x % kXcds) * 2 * per_slice + per_slice - 1 - bh : bh;
}

// The key-stationary work list of a head holds its caption items (n_text, the long ones) before its
// video items. Both kinds are dealt to the XCDs separately, caption items of every head first: a
// slice of the plain head-major list would give some XCDs the caption items of a head and others none
// (six heads of a 457k-token stream: 1.30 M against 0.53 M query tiles), and start the caption items of
// its last head when the rest is nearly done. With the shorter caption segments of text_segments() this
// took the 32-shot layer of six heads from 104.4 to 99.6 ms, 13k tokens of six fp32 heads from 1,435 to
// 1,217 us and the 1,088-token fp32 layer from 119 to 104 us. Caption items cost alike and go out as one
// slice per XCD. Video items do not: under the causal mask early chunks are routed to by more queries. Whole
// heads balance that and share their queries in an XCD's L2 (two samples of eight ragged heads: 367 us, dealt
// out eight items at a time 408), so XCDs take equal numbers of heads. The BH % 8 heads left are dealt out two
// neighbours at a time: slices of those left some XCDs the long lists of a head. dK/dV of one head of 80k tokens
// in 5,244-key chunks 2,225 us in slices, 976 dealt out; two heads of 311k tokens 41.3 -> 26.7 ms; six heads of 457k
// tokens 39.4 -> 37.2 ms. But heads shorter than a round of the chip (an item per compute unit) go out in slices when
// they are more than a few: dealt out, several at a time would pass through every L2 (six fp32 heads of 13k ragged
// tokens 247 us in slices, 257 dealt out; six heads of 14k 353 / 405; three heads of 25k 1,471 / 1,134). 499 layers of
// random layouts, all dealt out: 0.84 times their time in slices with one head, 0.88 two, 0.91 three, 0.96 four,
// 0.99 six and twelve, 0.44 to 1.17 one by one; 363 by this rule 0.91, 0.44 to 1.09. Three to eight items at a time
// do as well as two, twenty-four 2 % worse, one loses 2.5 ms of the 457k tokens. Launch kv_grid() workgroups;
// returns false for padding.
constexpr int kVideoTurn = 2, kFewHeads = 3;
__host__ __device__ inline int kv_grid(int n_items, int n_text, int BH) {
    return xcd_grid((long long)n_text * BH) + xcd_grid((long long)(n_items - n_text) * BH);
}
__device__ __forceinline__ bool kv_item(int n_items, int n_text, int BH, int &bh, int &item) {
    const long long tot_t = (long long)n_text * BH, tot_v = (long long)(n_items - n_text) * BH;
    const int per_t = (int)((tot_t + kXcds - 1) / kXcds);
    const int x = blockIdx.x % kXcds, p = blockIdx.x / kXcds;
    const bool text = p < per_t;
    int l = x * per_t + p;
    if (!text) {
        const int whole = BH / kXcds * (n_items - n_text);                                        // an XCD's items of whole heads
        const int left = (BH % kXcds) * (n_items - n_text);                                       // items of the other heads
        const bool deal = BH % kXcds <= kFewHeads || n_items - n_text >= kComputeUnits;
        const int turns = deal ? left / (kXcds * kVideoTurn) * kVideoTurn : 0;                    // an XCD's of them in whole turns
        const int rest = (left - turns * kXcds + kXcds - 1) / kXcds;                              // and in a slice
        const int v = p - per_t, u = v - whole;
        l = u < 0 ? x * whole + v
                  : whole * kXcds + (u < turns ? (u / kVideoTurn * kXcds + x) * kVideoTurn + u % kVideoTurn
                                               : turns * kXcds + x * rest + (u - turns));
    }
    if (l >= (text ? tot_t : tot_v)) return false;
    const int per_head = text ? n_text : n_items - n_text;
    bh = l / per_head;
    item = l - bh * per_head + (text ? 0 : n_text);
    return true;
}

// Workgroup `wg` of the conversions that ride with a launch of THREADS threads; bound by HBM.
template <int THREADS> __device__ __forceinline__ void convert_workgroup(const CvtArgs &c, uint32_t wg) {
    const uint32_t t = wg / c.per_tensor;
    const float *x = t == 0 ? c.x[0] : (t == 1 ? c.x[1] : c.x[2]);
    bf16_t *out = static_cast<bf16_t *>(c.out) + t * c.n;
    const size_t i0 = ((size_t)(wg - t * c.per_tensor) * THREADS * kCvtUnroll + threadIdx.x) * 8;
    bf16x8 v[kCvtUnroll];
#pragma unroll
    for (int u = 0; u < kCvtUnroll; ++u) v[u] = Io<float>::load8(x + min(i0 + (size_t)u * THREADS * 8, c.n - 8));
#pragma unroll
    for (int u = 0; u < kCvtUnroll; ++u)
        if (i0 + (size_t)u * THREADS * 8 < c.n) *reinterpret_cast<bf16x8 *>(out + i0 + (size_t)u * THREADS * 8) = v[u];
}

struct ItemDesc {
    int q_start, q_count;
    const int32_t *entries;   // gathered rows ((query << 5) | slot) or nullptr
    int nranges;
    const KeyRange *ranges;   // nullptr: use `single`
    KeyRange single;
    __device__ __forceinline__ KeyRange range(int r) const { return ranges ? ranges[r] : single; }
};

template <int MODE>
__device__ __forceinline__ bool decode_item(const FwdArgs &a, int bh, int t, ItemDesc &it) {
    if (MODE == MODE_ANCHOR) {
        const AnchorTile at = a.atiles[t];
        it.q_start = at.q_start;
        it.q_count = at.q_count;
        it.entries = nullptr;
        const int r0 = a.arange_off[at.win];
        it.nranges = a.arange_off[at.win + 1] - r0;
        it.ranges = a.aranges + r0;
        it.single = KeyRange{0, 0};
        return true;
    } else {
        const int C = a.C;
        const int32_t *toff = a.tile_off + (size_t)bh * (C + 1);
        if (t >= toff[C]) return false;
        int lo = 0, hi = C;   // largest j with toff[j] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (toff[mid] <= t) lo = mid; else hi = mid;
        }
        const int j = lo;
        const int32_t *loff = a.list_off + (size_t)bh * (C + 1);
        const int tl = t - toff[j];
        const int cnt = loff[j + 1] - loff[j];
        it.q_start = 0;
        it.q_count = min(kBM, cnt - tl * kBM);
        it.entries = a.qlist + (size_t)bh * a.N * a.topk + loff[j] + tl * kBM;
        it.nranges = 1;
        it.ranges = nullptr;
        it.single = KeyRange{a.off[j], a.off[j + 1] - a.off[j]};
        return true;
    }
}

// Walks the key ranges of an item in tiles of BN keys; the last tile of every
// range may be ragged (valid() < BN).
template <int BN> struct TileIter {
    const ItemDesc &it;
    int r, pos;
    KeyRange cur;
    __device__ __forceinline__ explicit TileIter(const ItemDesc &d) : it(d), r(0), pos(0), cur(d.range(0)) {}
    // In a scalar register before any address is made of it: the tile copies (inline assembly, which gets no
    // wait states from the compiler) take their base from scalar registers, and one that a vector instruction
    // has just written may only be read five wait states later; scalar results may be read at once.
    __device__ __forceinline__ int start() const { return __builtin_amdgcn_readfirstlane(cur.start + pos); }
    __device__ __forceinline__ int valid() const { return min(BN, cur.len - pos); }
    __device__ __forceinline__ bool next() {
        pos += BN;
        if (pos >= cur.len) {
            ++r;
            pos = 0;
            if (r >= it.nranges) return false;
            cur = it.range(r);
        }
        return true;
    }
};

// Where the epilogues of the forced-link items put the forced-link part among the routed partials of a query. At
// d = 128 with bf16 storage it comes first and, in the forward, is weighted before it is rounded to bf16; for d = 64
// and fp32 storage it comes last and is rounded before it is weighted, as if it had gone through a slot of its own.
// Both are as exact; either order is kept where it has always been, so that results stay the same.
template <int D, typename OT> __device__ constexpr bool forced_last() { return D == 64 || sizeof(OT) == 4; }

// Epilogue of the query-stationary passes. A transposed accumulator holds, per
// lane, 4-feature pieces of ONE row; storing those directly scatters 8-byte
// writes over 32 rows per instruction and the L2 writes partial lines back
// several times. Instead every wave transposes its 32 x D tile through its own
// 32 x (D + 4) bf16 patch of LDS and stores whole 16-byte groups, 16 lanes per
// 256-byte row. `dst_row` is this lane's destination row index (in rows of D
// bf16) or -1 if its row is not to be written; `scale` multiplies the values.
// All waves of the workgroup must have finished reading `smem` (barrier before).
template <int D>
__device__ __forceinline__ void store_rows_bf16(char *smem, int wave, int lane, const f32x16 *acc, float scale,
                                                int dst_row, bf16_t *out) {
    constexpr int DB = D / 32, RS = D + 4;             // padded row: consecutive rows shift by 2 banks
    const int half = lane >> 5, l32 = lane & 31;
    bf16_t *patch = reinterpret_cast<bf16_t *>(smem) + wave * (32 * RS + 64);
    int32_t *rowidx = reinterpret_cast<int32_t *>(patch + 32 * RS);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            Io<bf16_t>::store4(patch + l32 * RS + b * 32 + g * 8 + half * 4, acc[b][4 * g] * scale,
                               acc[b][4 * g + 1] * scale, acc[b][4 * g + 2] * scale, acc[b][4 * g + 3] * scale);
    if (half == 0) rowidx[l32] = dst_row;
    __builtin_amdgcn_wave_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    constexpr int LPR = D / 8, RPI = 64 / LPR;          // lanes per row, rows per instruction
    const int cg = lane % LPR, r0 = lane / LPR;
#pragma unroll
    for (int it = 0; it < 32 / RPI; ++it) {
        const int r = it * RPI + r0;
        const int dr = rowidx[r];
        const u32x2 lo2 = *reinterpret_cast<const u32x2 *>(patch + r * RS + cg * 8);
        const u32x2 hi2 = *reinterpret_cast<const u32x2 *>(patch + r * RS + cg * 8 + 4);
        if (dr >= 0) {
            u32x4 v = {lo2[0], lo2[1], hi2[0], hi2[1]};
            *reinterpret_cast<u32x4 *>(out + (size_t)dr * D + cg * 8) = v;
        }
    }
}

// A wave's 32 x D transposed accumulator, scaled, to 32 scattered rows of bf16 without a way through LDS. A lane holds
// 4-feature pieces of one row, its counterpart in the other half-wave the pieces between them: exchanged across the
// halves they make 16-byte words, and exchanged with the row 16 lanes on, four lanes hold 64 contiguous bytes of a row.
// Stored after the first exchange already, in 32-byte pieces of 32 rows at a time, the address unit and the L2 saw twice
// the requests: routed forward / dQ of 457k tokens, six heads, 130-key chunks, k = 16, 7,457 / 9,116 us against 7,229 /
// 8,648 now; 114k tokens, 24 heads, 260-key chunks, k = 8, 4,316 / 5,579 against 4,304 / 5,529. (Non-temporal stores
// lose: 4,410 / 5,762.) prow: the lane's row (in rows of D); rows >= valid are not written.
template <int D>
__device__ __forceinline__ void scatter_rows_bf16(const f32x16 *acc, float scale, int prow, int valid, int lane, bf16_t *out) {
    const int l16 = lane & 15, quad = ((lane >> 4) & 1) * 2 + (lane >> 5);       // 16-byte word of the lane within a 64-byte piece
    const auto rows = __builtin_amdgcn_permlane16_swap((uint32_t)prow, (uint32_t)prow, false, false);
    bf16_t *d0 = out + (size_t)rows[0] * D + quad * 8, *d1 = out + (size_t)rows[1] * D + quad * 8;
    const bool ok0 = l16 < valid, ok1 = l16 + 16 < valid;
#pragma unroll
    for (int b = 0; b < D / 32; ++b) {
        u32x4 w[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = 8 * u;
            const uint32_t x0 = pack_bf16(acc[b][i] * scale, acc[b][i + 1] * scale);
            const uint32_t x1 = pack_bf16(acc[b][i + 2] * scale, acc[b][i + 3] * scale);
            const uint32_t y0 = pack_bf16(acc[b][i + 4] * scale, acc[b][i + 5] * scale);
            const uint32_t y1 = pack_bf16(acc[b][i + 6] * scale, acc[b][i + 7] * scale);
            const auto r0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
            w[u] = u32x4{r0[0], r1[0], r0[1], r1[1]};
        }
        u32x4 p0, p1;                     // rows 0 .. 15, rows 16 .. 31
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto r = __builtin_amdgcn_permlane16_swap(w[0][e], w[1][e], false, false);
            p0[e] = r[0];
            p1[e] = r[1];
        }
        if (ok0) *reinterpret_cast<u32x4 *>(d0 + b * 32) = p0;
        if (ok1) *reinterpret_cast<u32x4 *>(d1 + b * 32) = p1;
    }
}

// Moves ROWS source rows of D features into a swizzled LDS tile (SwTile<D>).
//   issue_rows(tile, valid, lds)  starts the transfer of a tile into `lds`
//   commit()                      waits for this wave's copies (before the barrier that publishes `lds`)
// Asynchronous global->LDS loads (global_load_lds_dwordx4): no staging registers, no
// LDS store instructions. One wave instruction fills 1 KB of LDS, lane l writing
// bytes [16 l, 16 l + 16), so each lane fetches the global element that belongs at
// its swizzled LDS position.
template <int D, int ROWS> struct TileLoader {
    static constexpr int NW = 4;                        // waves of the workgroup that share the loads
    static constexpr int RPI = 512 / D;                 // rows per wave instruction
    static constexpr int NI = ROWS / RPI;               // wave instructions per tile
    static constexpr int P = (NI + NW - 1) / NW;        // per wave
    static_assert(NI % NW == 0, "tile rows must divide evenly among the waves");
    int wave, rlo, cgp;
    __device__ __forceinline__ int slot(int p) const { return wave + NW * p; }
    __device__ __forceinline__ explicit TileLoader(int tid)
        : wave(__builtin_amdgcn_readfirstlane(tid >> 6)), rlo((tid & 63) / (D / 8)), cgp((tid & 63) % (D / 8)) {}
    // contiguous rows [0, valid) of a tile whose first row is at `tile` (a
    // wave-uniform pointer): scalar base + one 32-bit lane offset per load
    __device__ __forceinline__ void issue_rows(const bf16_t *tile, int valid, bf16_t *lds) const {
        const uint32_t at = lds_address(lds);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int n = slot(p);
            const int row = n * RPI + rlo;
            const int cg = cgp ^ SwTile<D>::sw(row);
            const uint32_t off = (uint32_t)(min(row, valid - 1) * D + cg * 8) * 2u;
            async_copy16_at(tile, off, at + n * 1024);
        }
    }
    // the tile is complete once this wave's copies have landed (and the workgroup has met at a barrier)
    __device__ __forceinline__ void commit() const { wait_vmcnt<0>(); }
};

}  // namespace moc
