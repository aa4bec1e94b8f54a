// Inverse routing lists: for every (head, chunk) the queries that routed to it.
//
// Routing is per query (Eq. 3), so under incoherent selections a tile of
// neighbouring queries touches far more chunks than k. The attention passes
// therefore visit routed work chunk-major: the rows gathered through these
// lists form dense query tiles against one chunk's keys - the packing the
// paper obtains from a variable-length attention call (Sec. 3.3).
//
// A stable counting sort on the device, no host synchronisation, no global
// atomics, so every list is in ascending query order and the same input gives
// the same lists (and the same summation order in dK / dV) on every call:
//   count  one wave per block of queries (64 to 256): which entries of a
//          row count at all (see entry_ok), an LDS histogram over the chunks,
//          written out whole as row `block` of a [blocks][C] table;
//   scan   down the blocks of every chunk (a block's first position inside the
//          chunk's list), then across the chunks (list offsets, tile offsets);
//   fill   one wave per block walks its queries in order and takes their
//          positions from LDS cursors (see fill_rows), so they do not depend on
//          scheduling.
// Calls with few entries do all three in one workgroup per head; where the table is small, the workgroups of
// the fill scan it themselves.
// An entry packs query and slot as (i << 5) | r (r < MOC_MAX_TOPK = 32).
//
// Which entries of a selection row count (Sec. 3.3 pre-routing mask): forced
// links are attended anyway, so an entry naming a caption chunk or a chunk of
// the query's own window is dropped, as is the second mention of a chunk in a
// row and anything outside [0, C). The union M(i) + R(i) is a set. Bit r of
// vmask[query] says whether slot r counts; the attention epilogues read the
// same word, so a dropped slot is never merged.
#include "moc_attn_common.h"
#include "moc_internal.h"

namespace moc {

// The passes below walk their queries 64 / topk at a time: lane L holds entry L of the step's rows
// (query L / topk, slot L % topk), read with one coalesced load. The loads of kListUnroll steps are in
// flight together: a step is a chain of two dependent loads, and small calls have few waves to cover it.
constexpr int kListUnroll = 4;

struct ListLane {
    int rpb, mu, r;      // queries per step (topk <= 32: at least two), this lane's query of the step and its slot
    bool on;
    __device__ __forceinline__ explicit ListLane(int topk, int lane)
        : rpb(64 / topk), mu(lane / topk), r(lane - lane / topk * topk), on(lane / topk < 64 / topk) {}
};

// The lanes among `who` that name the same chunk as this one, by one ballot per bit of the chunk index.
__device__ __forceinline__ unsigned long long same_chunk(int j, unsigned long long who, int bits) {
    for (int b = 0; b < bits; ++b) {
        const bool bit = (j >> b) & 1;
        const unsigned long long bal = __ballot(bit);
        who &= bit ? bal : ~bal;
    }
    return who;
}

// Counts the entries of queries [i0, i0 + nrow) into hist and writes their slot masks. An entry counts
// if it names a video chunk (rw >= 0) outside the query's own window that no earlier slot of the row
// names (the row-mates sit in the neighbouring lanes; topk - 1 shuffles, each an LDS round trip, took
// 97 us at 5,606 tokens, three heads and k = 16, the ballots take 16). sel and vmask point at the
// head's first query.
__device__ __forceinline__ void count_rows(const int32_t *__restrict__ sel, int i0, int nrow, int topk, int C, int bits, int lane,
                                           const int32_t *__restrict__ chunk_of, const int32_t *__restrict__ win,
                                           const int32_t *__restrict__ rw, uint32_t *__restrict__ vmask,
                                           int32_t *hist) {
    const ListLane L(topk, lane);
    const int32_t *src = sel + (size_t)i0 * topk;
    uint32_t *vm = vmask + i0;
    const uint32_t rowbits = topk >= 32 ? 0xffffffffu : ((1u << topk) - 1u);
    const unsigned long long earlier = (unsigned long long)((1u << L.r) - 1u) << (lane - L.r);      // earlier slots of the row
    for (int u0 = 0; u0 < nrow; u0 += kListUnroll * L.rpb) {
        int j[kListUnroll], wq[kListUnroll], w[kListUnroll];
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            const int u = u0 + t * L.rpb + L.mu;
            const bool in = L.on && u < nrow;
            const int jt = src[in ? u * topk + L.r : 0];       // (plain loads: a load inside a branch is waited for there)
            wq[t] = chunk_of[i0 + (in ? u : 0)];
            j[t] = in ? jt : -1;
        }
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            wq[t] = win[wq[t]];
            const bool known = j[t] >= 0 && j[t] < C;
            const int wt = rw[known ? j[t] : 0];
            w[t] = known ? wt : -1;
        }
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            const int u = u0 + t * L.rpb + L.mu;
            const bool link = w[t] >= 0 && w[t] != wq[t];
            bool ok = link;
            if (topk > 4) {
                ok = link && !(same_chunk(j[t], __ballot(link), bits) & earlier);
            } else {                               // at most three neighbours: fewer shuffles than ballots
                for (int p = 1; p < topk; ++p) {
                    const int other = __shfl_up(j[t], p, 64);
                    if (p <= L.r && other == j[t]) ok = false;
                }
            }
            if (ok) atomicAdd(&hist[j[t]], 1);
            const unsigned long long bal = __ballot(ok);
            if (L.on && u < nrow && L.r == 0) vm[u] = (uint32_t)(bal >> (L.mu * topk)) & rowbits;
        }
    }
}

// Writes the list entries of queries [i0, i0 + nrow); cursor[j] is the next free position of chunk j's
// list for them. Lanes of one step that name the same chunk belong to different queries (the slots that
// count name distinct chunks) and take consecutive positions in lane order, that is in query order: each
// adds its rank among them to the cursor, and the last of them moves it. LDS operations of a wave complete in program order, so the
// next step reads what this one wrote. (One LDS add per query of the step, the obvious way to the same
// order, waits for LDS up to 64 / topk times a step: 24.3 us against 17.0 at 9k tokens, sixteen heads and k = 6.
// At 114k tokens the scattered 4-byte stores bound the pass, 200 us either way.)
__device__ __forceinline__ void fill_rows(const int32_t *__restrict__ sel, int i0, int nrow, int topk, int bits, int lane,
                                          const uint32_t *__restrict__ vmask, int32_t *cursor,
                                          int32_t *qlist) {
    const ListLane L(topk, lane);
    const int32_t *src = sel + (size_t)i0 * topk;
    const uint32_t *vm = vmask + i0;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int u0 = 0; u0 < nrow; u0 += kListUnroll * L.rpb) {
        int j[kListUnroll];
        uint32_t used[kListUnroll];
        bool ok[kListUnroll];
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            const int u = u0 + t * L.rpb + L.mu;
            const bool in = L.on && u < nrow;
            j[t] = src[in ? u * topk + L.r : 0];
            used[t] = vm[in ? u : 0];
        }
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            const int u = u0 + t * L.rpb + L.mu;
            ok[t] = L.on && u < nrow && ((used[t] >> L.r) & 1u);
        }
#pragma unroll
        for (int t = 0; t < kListUnroll; ++t) {
            const unsigned long long same = same_chunk(j[t], __ballot(ok[t]), bits);
            if (ok[t]) {
                const int pos = cursor[j[t]] + __popcll(same & below);
                if ((same >> lane) == 1ull) cursor[j[t]] = pos + 1;
                qlist[pos] = ((i0 + u0 + t * L.rpb + L.mu) << 5) | L.r;
            }
            asm volatile("" ::: "memory");      // another lane may have moved the cursor this lane reads next
        }
    }
}

// One wave per block of `rows` queries. CVT: conversions ride (an instance of its own: the code of the others does not grow).
template <bool CVT>
__global__ __launch_bounds__(64) void list_count_kernel(const int32_t *__restrict__ sel, int N, int topk, int C, int bits,
                                                        const int32_t *__restrict__ chunk_of,
                                                        const int32_t *__restrict__ win,
                                                        const int32_t *__restrict__ rw, int rows, int NB, int BH,
                                                        uint32_t *__restrict__ vmask, int32_t *__restrict__ cnt_blk,
                                                        CvtArgs cvt) {
    extern __shared__ int32_t hist[];    // [C]
    const int mine = xcd_grid((long long)NB * BH);
    if constexpr (CVT)
        if ((int)blockIdx.x >= mine) { convert_workgroup<64>(cvt, blockIdx.x - mine); return; }
    int logical;
    if (!xcd_remap((long long)NB * BH, logical)) return;
    const int bh = logical / NB, blk = logical - bh * NB, lane = threadIdx.x;
    const int i0 = blk * rows, nrow = min(rows, N - i0);
    for (int b = lane; b < C; b += 64) hist[b] = 0;
    __syncthreads();
    count_rows(sel + (size_t)bh * N * topk, i0, nrow, topk, C, bits, lane, chunk_of, win, rw, vmask + (size_t)bh * N, hist);
    __syncthreads();
    int32_t *out = cnt_blk + ((size_t)bh * NB + blk) * C;
    for (int b = lane; b < C; b += 64) out[b] = hist[b];
}

// Down the blocks in two levels (the table is [block][chunk], so neighbouring threads read
// neighbouring words): the blocks are cut into kScanGroups groups; pass 1 sums every chunk's
// entries per group, pass 2 turns the group's entries into the number of entries of that chunk
// in all earlier blocks and leaves the chunk's total behind.
constexpr int kScanGroups = 32;
__global__ __launch_bounds__(256) void list_group_sum_kernel(const int32_t *__restrict__ cnt_blk, int NB, int C,
                                                             int32_t *__restrict__ gsum) {
    const int bh = blockIdx.z, g = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= C) return;
    const int per = (NB + kScanGroups - 1) / kScanGroups;
    const int b0 = g * per, b1 = min(NB, b0 + per);
    const int32_t *col = cnt_blk + (size_t)bh * NB * C + j;
    int sum = 0;
    for (int b = b0; b < b1; ++b) sum += col[(size_t)b * C];
    gsum[((size_t)bh * kScanGroups + g) * C + j] = sum;
}
__global__ __launch_bounds__(256) void list_block_scan_kernel(int32_t *__restrict__ cnt_blk, int NB, int C,
                                                              const int32_t *__restrict__ gsum,
                                                              int32_t *__restrict__ cnt) {
    const int bh = blockIdx.z, g = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= C) return;
    const int per = (NB + kScanGroups - 1) / kScanGroups;
    const int b0 = g * per, b1 = min(NB, b0 + per);
    const int32_t *gs = gsum + (size_t)bh * kScanGroups * C + j;
    int run = 0;
    for (int u = 0; u < g; ++u) run += gs[(size_t)u * C];
    int32_t *col = cnt_blk + (size_t)bh * NB * C + j;
    for (int b = b0; b < b1; ++b) {
        const int c = col[(size_t)b * C];
        col[(size_t)b * C] = run;
        run += c;
    }
    if (g == kScanGroups - 1) cnt[(size_t)bh * C + j] = run;
}

// per head: list_off = exclusive scan of cnt, tile_off = exclusive scan of ceil(cnt / kBM)
__global__ __launch_bounds__(256) void list_scan_kernel(const int32_t *__restrict__ cnt, int C,
                                                        int32_t *__restrict__ list_off,
                                                        int32_t *__restrict__ tile_off) {
    __shared__ int32_t sa[256], sb[256];
    const int bh = blockIdx.x;
    const int32_t *c = cnt + (size_t)bh * C;
    int32_t *lo = list_off + (size_t)bh * (C + 1);
    int32_t *to = tile_off + (size_t)bh * (C + 1);
    const int seg = (C + 255) / 256;
    const int b0 = threadIdx.x * seg, b1 = min(C, b0 + seg);
    int a = 0, b = 0;
    for (int j = b0; j < b1; ++j) { a += c[j]; b += (c[j] + kBM - 1) / kBM; }
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        int ra = 0, rb = 0;
        for (int t = 0; t < 256; ++t) {
            const int xa = sa[t], xb = sb[t];
            sa[t] = ra; sb[t] = rb;
            ra += xa; rb += xb;
        }
        lo[C] = ra;
        to[C] = rb;
    }
    __syncthreads();
    a = sa[threadIdx.x];
    b = sb[threadIdx.x];
    for (int j = b0; j < b1; ++j) {
        lo[j] = a;
        to[j] = b;
        a += c[j];
        b += (c[j] + kBM - 1) / kBM;
    }
}

// One wave per block. A block writes a few words into every chunk's list; neighbouring blocks of a head
// write the words next to them, so they run on one XCD, whose L2 then holds whole lines (203 -> 197 us at
// 114k tokens, 24 heads, k = 8; 1,034 -> 866 at 457k tokens, six heads, k = 16).
__global__ __launch_bounds__(64) void list_fill_kernel(const int32_t *__restrict__ sel, int N, int topk, int C, int bits,
                                                       const uint32_t *__restrict__ vmask, int NB, int BH,
                                                       const int32_t *__restrict__ cnt_blk,
                                                       const int32_t *__restrict__ list_off,
                                                       int32_t *__restrict__ qlist) {
    extern __shared__ int32_t cursor[];  // [C]
    int logical;
    if (!xcd_remap((long long)NB * BH, logical)) return;
    const int bh = logical / NB, blk = logical - bh * NB, lane = threadIdx.x;
    const int i0 = blk * kRowsPerBlk, nrow = min(kRowsPerBlk, N - i0);
    const int32_t *base = cnt_blk + ((size_t)bh * NB + blk) * C;
    const int32_t *lo = list_off + (size_t)bh * (C + 1);
    for (int b = lane; b < C; b += 64) cursor[b] = lo[b] + base[b];
    __syncthreads();
    fill_rows(sel + (size_t)bh * N * topk, i0, nrow, topk, bits, lane, vmask + (size_t)bh * N, cursor,
              qlist + (size_t)bh * N * topk);
}

// Scan and fill in one launch, for tables that are cheap to read whole: every workgroup (sixteen blocks of a head, a
// wave each) sums the head's table itself, thread (g, j) every G-th row of chunk j, instead of three launches that pass
// the sums on. Counting and this against the launches before (one workgroup a head at 6,256 tokens, else the five of the
// general way): 29 -> 15 us at 6,256 tokens, 24 heads, k = 3; 57 -> 26 at 15.5k tokens, sixteen ragged heads, k = 6; 47 -> 19
// at 12.9k, six heads, k = 5; 66 -> 49 at 33k, 24 heads, k = 5; 155 -> 144 at 182k, 24 heads, k = 5.
constexpr int kFillWaves = 16;
constexpr int kFillChunks = 880;          // its cursors and sums: 64 KB of LDS
__global__ __launch_bounds__(kFillWaves * 64) void list_scan_fill_kernel(const int32_t *__restrict__ sel, int N, int topk, int C,
                                                                         int bits, const uint32_t *__restrict__ vmask,
                                                                         int rows, int NB, int BH,
                                                                         const int32_t *__restrict__ cnt_blk,
                                                                         int32_t *__restrict__ list_off,
                                                                         int32_t *__restrict__ tile_off,
                                                                         int32_t *__restrict__ qlist) {
    extern __shared__ int32_t cursor[];  // [kFillWaves][C]
    __shared__ int32_t part[2][kFillWaves * 64];
    static_assert(kFillWaves * kFillChunks * 4 + 2 * kFillWaves * 65 * 4 <= 65536, "LDS of a launch");
    __shared__ int32_t wsum[2][kFillWaves];
    const int groups = (NB + kFillWaves - 1) / kFillWaves;
    int logical;
    if (!xcd_remap((long long)groups * BH, logical)) return;
    const int bh = logical / groups, b0 = (logical - bh * groups) * kFillWaves;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t *tab = cnt_blk + (size_t)bh * NB * C;
    // ---- per chunk: entries in the blocks before this workgroup's, entries in all
    const int G = kFillWaves * 64 / C, g = tid / C, j = tid - g * C;
    int before = 0, tot = 0;
    if (g < G) {
#pragma unroll 8
        for (int b = g; b < NB; b += G) {
            const int c = tab[(size_t)b * C + j];
            tot += c;
            before += b < b0 ? c : 0;
        }
        part[0][tid] = before;
        part[1][tid] = tot;
    }
    __syncthreads();
    before = tot = 0;
    const int used = min(G, NB);         // a thread past the last row has summed none
    if (tid < C)
        for (int u = 0; u < used; ++u) { before += part[0][u * C + tid]; tot += part[1][u * C + tid]; }
    // ---- thread j owns chunk j: an exclusive scan over the chunks
    int a = tot, t = (tot + kBM - 1) / kBM;
    const int tiles = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int xa = __shfl_up(a, o, 64), xt = __shfl_up(t, o, 64);
        if (lane >= o) { a += xa; t += xt; }
    }
    if (lane == 63) { wsum[0][wave] = a; wsum[1][wave] = t; }
    __syncthreads();
    for (int w = 0; w < wave; ++w) { a += wsum[0][w]; t += wsum[1][w]; }
    if (tid < C) {
        if (b0 == 0) {
            int32_t *lo = list_off + (size_t)bh * (C + 1), *to = tile_off + (size_t)bh * (C + 1);
            lo[tid] = a - tot;
            to[tid] = t - tiles;
            if (tid == C - 1) { lo[C] = a; to[C] = t; }
        }
        int c[kFillWaves], at = a - tot + before;
#pragma unroll
        for (int w = 0; w < kFillWaves; ++w) c[w] = tab[(size_t)min(b0 + w, NB - 1) * C + tid];
#pragma unroll
        for (int w = 0; w < kFillWaves; ++w) { cursor[w * C + tid] = at; at += c[w]; }
    }
    __syncthreads();
    const int i0 = (b0 + wave) * rows;
    if (i0 < N)
        fill_rows(sel + (size_t)bh * N * topk, i0, min(rows, N - i0), topk, bits, lane, vmask + (size_t)bh * N, cursor + wave * C,
                  qlist + (size_t)bh * N * topk);
}

// The whole list builder for a head in one workgroup: sixteen waves take consecutive sixteenths of the
// queries, count into histograms of their own, scan them and fill. The smallest calls are bound by their
// launches, not by work: 38 us in five, 7 in one at 1,088 tokens.
constexpr int kHeadWaves = 16, kHeadChunks = 1000;      // 62.5 KB of histograms
template <bool CVT>
__global__ __launch_bounds__(kHeadWaves * 64) void list_head_kernel(const int32_t *__restrict__ sel, int N, int topk,
                                                                    int C, int bits,
                                                                    const int32_t *__restrict__ chunk_of,
                                                                    const int32_t *__restrict__ win,
                                                                    const int32_t *__restrict__ rw,
                                                                    uint32_t *__restrict__ vmask,
                                                                    int32_t *__restrict__ list_off,
                                                                    int32_t *__restrict__ tile_off,
                                                                    int32_t *__restrict__ qlist, int BH, CvtArgs cvt) {
    extern __shared__ int32_t hist[];    // [kHeadWaves][C]
    __shared__ int32_t wsum[2][kHeadWaves];
    if constexpr (CVT)
        if ((int)blockIdx.x >= BH) { convert_workgroup<kHeadWaves * 64>(cvt, blockIdx.x - BH); return; }
    const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (N + kHeadWaves - 1) / kHeadWaves;
    const int i0 = min(N, wave * per), nrow = min(per, N - i0);
    for (int b = tid; b < kHeadWaves * C; b += kHeadWaves * 64) hist[b] = 0;
    __syncthreads();
    sel += (size_t)bh * N * topk;
    vmask += (size_t)bh * N;
    count_rows(sel, i0, nrow, topk, C, bits, lane, chunk_of, win, rw, vmask, hist + wave * C);
    __syncthreads();
    // thread j owns chunk j: entries of the earlier waves, then an exclusive scan over the chunks
    int tot = 0;
    if (tid < C)
        for (int w = 0; w < kHeadWaves; ++w) {
            const int c = hist[w * C + tid];
            hist[w * C + tid] = tot;
            tot += c;
        }
    int a = tot, b = (tot + kBM - 1) / kBM;          // inclusive scans within the wave
    const int tiles = b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int xa = __shfl_up(a, o, 64), xb = __shfl_up(b, o, 64);
        if (lane >= o) { a += xa; b += xb; }
    }
    if (lane == 63) { wsum[0][wave] = a; wsum[1][wave] = b; }
    __syncthreads();
    for (int w = 0; w < wave; ++w) { a += wsum[0][w]; b += wsum[1][w]; }
    if (tid < C) {
        int32_t *lo = list_off + (size_t)bh * (C + 1), *to = tile_off + (size_t)bh * (C + 1);
        lo[tid] = a - tot;
        to[tid] = b - tiles;
        if (tid == C - 1) { lo[C] = a; to[C] = b; }
        for (int w = 0; w < kHeadWaves; ++w) hist[w * C + tid] += a - tot;
    }
    __syncthreads();
    fill_rows(sel, i0, nrow, topk, bits, lane, vmask, hist + wave * C, qlist + (size_t)bh * N * topk);
}

// How a call's lists are built: a workgroup a head, count and scan + fill over blocks of `rows` queries, or the five
// launches of the general way.
enum ListWay { LIST_HEAD, LIST_TWO, LIST_GENERAL };
struct ListPlan { ListWay way; int rows, NB; };
constexpr int kFillTable = 49152;         // words of a head's table up to which two launches are used (192 KB read by each workgroup)
constexpr int kFillSpread = 4096;         // waves of the count kernel up to which smaller blocks gain
static ListPlan list_plan(int N, int C, int topk, int BH) {
    const long long entries = (long long)N * topk;
    ListPlan p{LIST_GENERAL, kRowsPerBlk, (N + kRowsPerBlk - 1) / kRowsPerBlk};
    bool two = C <= kFillChunks && (long long)p.NB * C <= kFillTable;
    if (two) {
        // Blocks shrink until the count has some 4,096 waves: with 2,048 of them 33k tokens (24 heads, k = 5) take 52 us for 49,
        // with 1,024 6,256 tokens (24 heads, k = 3) 18 for 15 and 15.5k tokens (sixteen heads, k = 6) 34 for 26.
        int rows = p.rows, NB = p.NB;
        while (rows > kRowsPerBlkMin && (long long)NB * BH < kFillSpread && (long long)((N + rows / 2 - 1) / (rows / 2)) * C <= kFillTable) {
            rows /= 2;
            NB = (N + rows - 1) / rows;
        }
        // Sixteen waves a workgroup fill slower than waves spread over the chip, which shows where each has many steps: with blocks of
        // 256 queries, k = 16 112 us for 102 (one head, 16k tokens) and 121 for 110 (six, 50k), but 135 for 146 with 24 heads; k = 32
        // 231 for 208 there; k = 8 63 for 67 (six heads, 8k). With 128 queries k = 32 105 for 164 (one head, 12k).
        two = rows < kRowsPerBlk || topk <= 8 || (topk <= 16 && BH >= 24);
        if (two) p = ListPlan{LIST_TWO, rows, NB};
    }
    if (C > kHeadChunks || entries > 32768) return p;
    const bool head =
        // one launch for two, or as long: 24 heads of 4,096 entries 11 us for 14, of 8,192 at k = 8 17 for 19, at k = 1 15 for 15, of
        // 8,400 20 for 14
        entries <= 8192
        // one launch for five: a sixteenth of the head is up to as many steps as the general way's blocks, or the heads are many
        // (960 chunks: 4,096 tokens, k = 3 28 us for 40; 16k, k = 1 27 for 30; 32k, k = 1 51 for 34 with two heads, 61 for 81 with 64)
        || (!two && (BH >= 48 || (long long)(N - 4096) * topk <= 12288))
        // 200 heads fill the chip with one workgroup each (32k tokens, two chunks, k = 1 38 us for 49; 128 heads take as long)
        || (BH >= 192 && C <= 20);
    if (head) p = ListPlan{LIST_HEAD, 0, 0};
    return p;
}

size_t list_fine_bytes(const moc_meta *m, int BH, int topk) {
    const ListPlan p = list_plan(m->N, m->C, topk, BH);
    return p.way == LIST_TWO ? (size_t)BH * p.NB * m->C * 4 : 0;
}

// Conversions ride with the first launch, but not
//   beside the histograms of more chunks than this: their waves get the count's LDS too, 4 KB let 32 run on a compute unit;
constexpr int kCvtChunks = 1024;
//   where the selections are large: the fill reads them a second time, and the conversions, which stream behind the count,
//   have by then pushed them out of the caches. Lists and conversions of 24 heads, d = 64, riding / alone: 101 MB of
//   selections (66k tokens, k = 16) 841 / 733 us (the fill 480 / 295), 51 MB (33k) 348 / 321, 25 MB (16k) 137 / 133; eight heads
//   34 MB (66k tokens) 267 / 281; with d = 128 506 / 493, 218 / 220 and 384 / 395 for the last three.
constexpr long long kCvtEntries = 10000000;
hipError_t launch_build_lists(const moc_meta *m, int BH, int topk, const int32_t *sel, char *ws, const AttnWs &L,
                              CvtArgs cvt, hipStream_t st) {
    const int C = m->C, N = m->N;
    int32_t *cnt = reinterpret_cast<int32_t *>(ws + L.cnt);
    int32_t *cnt_blk = reinterpret_cast<int32_t *>(ws + L.cnt_blk);
    uint32_t *vmask = reinterpret_cast<uint32_t *>(ws + L.vmask);
    int32_t *list_off = reinterpret_cast<int32_t *>(ws + L.list_off);
    int32_t *tile_off = reinterpret_cast<int32_t *>(ws + L.tile_off);
    int32_t *qlist = reinterpret_cast<int32_t *>(ws + L.qlist);
    if (cvt.count && (C > kCvtChunks || (long long)BH * N * topk > kCvtEntries)) {
        const hipError_t e = launch_to_bf16(cvt, st);
        if (e != hipSuccess) return e;
        cvt.count = 0;
    }
    MOC_PROF("build_lists", st);
    int bits = 0;
    while ((1 << bits) < C) ++bits;
    const ListPlan plan = list_plan(N, C, topk, BH);
    if (plan.way == LIST_HEAD) {
        const uint32_t extra = cvt_grid(cvt, kHeadWaves * 64);
        const auto kernel = cvt.count ? list_head_kernel<true> : list_head_kernel<false>;
        kernel<<<dim3(BH + extra), dim3(kHeadWaves * 64), (size_t)kHeadWaves * C * 4, st>>>(
            sel, N, topk, C, bits, m->d_chunk_of, m->d_win, m->d_rwin, vmask, list_off, tile_off, qlist, BH, cvt);
        return hipGetLastError();
    }
    const int rows = plan.rows, NB = plan.NB;
    if (plan.way == LIST_TWO) cnt_blk = reinterpret_cast<int32_t *>(ws + L.cnt_fine);
    const size_t shm = (size_t)C * 4;
    const uint32_t extra = cvt_grid(cvt, 64);
    const auto count = cvt.count ? list_count_kernel<true> : list_count_kernel<false>;
    count<<<dim3(xcd_grid((long long)NB * BH) + extra), dim3(64), shm, st>>>(
        sel, N, topk, C, bits, m->d_chunk_of, m->d_win, m->d_rwin, rows, NB, BH, vmask, cnt_blk, cvt);
    if (plan.way == LIST_TWO) {
        const long long wgs = (long long)((NB + kFillWaves - 1) / kFillWaves) * BH;
        list_scan_fill_kernel<<<dim3(xcd_grid(wgs)), dim3(kFillWaves * 64), kFillWaves * shm, st>>>(
            sel, N, topk, C, bits, vmask, rows, NB, BH, cnt_blk, list_off, tile_off, qlist);
        return hipGetLastError();
    }
    int32_t *gsum = reinterpret_cast<int32_t *>(ws + L.gsum);
    const dim3 sgrid((C + 255) / 256, kScanGroups, BH);
    list_group_sum_kernel<<<sgrid, dim3(256), 0, st>>>(cnt_blk, NB, C, gsum);
    list_block_scan_kernel<<<sgrid, dim3(256), 0, st>>>(cnt_blk, NB, C, gsum, cnt);
    list_scan_kernel<<<dim3(BH), dim3(256), 0, st>>>(cnt, C, list_off, tile_off);
    list_fill_kernel<<<dim3(xcd_grid((long long)NB * BH)), dim3(64), shm, st>>>(sel, N, topk, C, bits, vmask, NB, BH, cnt_blk, list_off, qlist);
    return hipGetLastError();
}

}  // namespace moc
