// Routing regularisers applied to the routed set of every (head, query) row
// (Sec. 3.2, "Context Drop-off" and "Context Drop-in"): a random number of the
// routed chunks is removed, a Poisson number of further candidates is added.
//
// One lane per row. Random words come from Philox4x32-10 (Salmon et al., SC'11)
// with counter (query, head, block, 0) and the 64-bit seed as key; draw t of a
// row is word t mod 4 of block t / 4: draw 0 sets the drop probability, draw 1
// the Poisson count, the next draws pick what to remove and then what to add.
// Both picks are uniform without replacement by rank: floor(draw * n / 2^32)
// among the n entries still alive (routed order), respectively among the n
// candidates not routed and not yet added (ascending chunk index). The rank of
// a candidate is found without enumerating candidates: a prefix count of
// non-text chunks gives the rank of any chunk among the query's candidates, the
// ranks already excluded are kept sorted in registers, and a table of the
// non-text chunks turns the final rank back into a chunk index.
//
// Bound by vector instructions: two or three Philox blocks and the bookkeeping of
// the slowest of 64 lanes. So the lists live in registers with fixed bounds (a
// sorting network, unrolled inserts) instead of LDS lists walked at run time, and
// rows travel through LDS only to be read and written in whole lines: 194 -> 118 us at
// 114k tokens, 24 heads, 8 + 4 slots (45 of it from the table in place of a search). The draws' blocks made once
// for all picks and the words of a row found without divisions: 116 -> 104, 12 heads with 20 + 12 slots 216 -> 195. (The
// chunk's tables and the first block ahead of the rows' loads: no difference, latency is not the bound.)
#include "moc_internal.h"
#include "moc_device.h"

namespace moc {

struct PerturbArgs {
    int32_t *sel;                          // [BH][N][width], the first topk columns hold the routed chunks
    const int32_t *chunk_of, *win, *wfirst, *wlast;
    const int32_t *ntb;                    // [C+1] number of non-text chunks with index < j
    const int32_t *video;                  // the non-text chunks, ascending (the inverse of ntb)
    int N, C, topk, max_in, causal;
    float p_max;
    uint32_t key0, key1;
    uint64_t thr[MOC_MAX_TOPK];            // floor(CDF(j) * 2^32) of the Poisson law, j < max_in
};

// block `blk` of the row with counter words c0, c1
struct Philox { uint32_t w[4]; };
__device__ __forceinline__ Philox philox(uint32_t c0, uint32_t c1, uint32_t blk, uint32_t k0, uint32_t k1) {
    uint32_t x0 = c0, x1 = c1, x2 = blk, x3 = 0;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * x0, m1 = (uint64_t)0xCD9E8D57u * x2;
        const uint32_t h0 = (uint32_t)(m0 >> 32), l0 = (uint32_t)m0;
        const uint32_t h1 = (uint32_t)(m1 >> 32), l1 = (uint32_t)m1;
        x0 = h1 ^ x1 ^ k0; x1 = l1; x2 = h0 ^ x3 ^ k1; x3 = l0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return Philox{{x0, x1, x2, x3}};
}

constexpr int kPerturbThreads = 128;

// One row, in place: routed chunks best first and -1 behind them on entry, survivors, added chunks and -1
// on return.
template <int K, int W>
__device__ __forceinline__ void perturb_row(const PerturbArgs &a, int i, int bh, int width, int32_t *row) {
    constexpr int kNone = 0x7fffffff;
    const int cq = a.chunk_of[i];
    const int w = a.win[cq];
    const int limit = a.causal ? cq : a.C;
    const int wf = min(a.wfirst[w], limit), wl1 = min(a.wlast[w] + 1, limit);   // own window inside [0, limit)
    const int nt_wf = a.ntb[wf];
    const int win_nt = a.ntb[wl1] - nt_wf;                                      // its non-text chunks
    const int n_elig = a.ntb[limit] - win_nt;

    int ent[K];
    int nv = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        ent[r] = r < a.topk ? row[r] : -1;
        nv += ent[r] >= 0 ? 1 : 0;
    }

    const Philox first = philox((uint32_t)i, (uint32_t)bh, 0, a.key0, a.key1);
    const uint32_t r_drop = first.w[0], r_in = first.w[1];

    // ---- drop-off: floor(p k) of the routed chunks, p = u p_max, single precision
    const float u = (float)(r_drop >> 8) * 0x1p-24f;
    const float pk = (u * a.p_max) * (float)a.topk;
    const int nd = min((int)floorf(pk), nv);
    // ---- drop-in: m ~ Poisson by inversion, truncated, capped by what is available
    int m = 0;
    for (int j = 0; j < a.max_in; ++j) m += (uint64_t)r_in >= a.thr[j] ? 1 : 0;
    m = min(m, n_elig - nv);

    // The words of all picks are made before the first of them: made as the picks come to a new block, each block would
    // be evaluated again for every count of removed entries among the 64 rows, six times a wave instead of two or three.
    // They wait in the row itself, whose entries are in registers: those of the removals at its front, where survivors come
    // after the last removal, those of the additions at its end, never in front of the place the next addition goes to.
    // (In LDS of their own, twice the row's, they cost more waves than they gain: 114.9 -> 136.9 us.)
    const int picks = nd + m, add_at = width - picks;
    if (picks > 0) row[nd > 0 ? 0 : add_at] = (int32_t)first.w[2];
    if (picks > 1) row[1 + (nd > 1 ? 0 : add_at)] = (int32_t)first.w[3];
    for (int j = 2; j < picks; j += 4) {                   // pick j takes draw j + 2
        const Philox b = philox((uint32_t)i, (uint32_t)bh, (uint32_t)((j + 2) >> 2), a.key0, a.key1);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j + e < picks) row[j + e + (j + e < nd ? 0 : add_at)] = (int32_t)b.w[e];
    }

    uint32_t alive = nv >= 32 ? 0xffffffffu : ((1u << nv) - 1u);
    for (int s = 0; s < nd; ++s) {
        const int t = (int)__umulhi((uint32_t)row[s], (uint32_t)(nv - s));
        uint32_t b = alive;
        for (int x = 0; x < t; ++x) b &= b - 1;            // skip t alive entries
        alive &= ~(b & (0u - b));                          // clear the lowest remaining one
    }

    // ranks (among the query's candidates) that are taken, ascending: the routed chunks first
    int ex[W];
#pragma unroll
    for (int r = 0; r < W; ++r) ex[r] = kNone;
#pragma unroll
    for (int r = 0; r < K; ++r)
        if (r < W) ex[r] = ent[r] >= 0 ? a.ntb[ent[r]] - (ent[r] >= wl1 ? win_nt : 0) : kNone;
#pragma unroll
    for (int p = 1; p < K; p *= 2)                          // Batcher's odd-even merge sort
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int x = 0; x < K - 1; ++x)
                if (x + k < K && x >= k % p && ((x - k % p) / k) % 2 == 0 && x / (2 * p) == (x + k) / (2 * p)) {
                    const int t = min(ex[x], ex[x + k]);
                    ex[x + k] = max(ex[x], ex[x + k]);
                    ex[x] = t;
                }
    // survivors first, in routed order
    int out = 0;
#pragma unroll
    for (int r = 0; r < K; ++r)
        if ((alive >> r) & 1u) row[out++] = ent[r];
    for (int s = 0; s < m; ++s) {
        int t = (int)__umulhi((uint32_t)row[width - m + s], (uint32_t)(n_elig - nv - s));
#pragma unroll
        for (int p = 0; p < W; ++p) t += ex[p] <= t ? 1 : 0;      // step over excluded ranks
#pragma unroll
        for (int p = W - 1; p >= 1; --p) ex[p] = min(ex[p], max(ex[p - 1], t));
        ex[0] = min(ex[0], t);
        const int nt_rank = t < nt_wf ? t : t + win_nt;    // rank among all non-text chunks
        row[out++] = a.video[nt_rank];
    }
    for (; out < width; ++out) row[out] = -1;
}

// K: at least topk, a power of two; W: at least topk + max_in. Dynamic LDS: one padded row per lane.
template <int K, int W>
__global__ __launch_bounds__(kPerturbThreads) void perturb_kernel(PerturbArgs a) {
    extern __shared__ int32_t lds[];
    const int tid = threadIdx.x;
    const int width = a.topk + a.max_in;
    const int rs = width | 1;                                  // LDS row stride: odd, free of bank conflicts
    const int i0 = blockIdx.x * kPerturbThreads, nrow = min(kPerturbThreads, a.N - i0);
    const int bh = blockIdx.y;
    int32_t *rows = a.sel + ((size_t)bh * a.N + i0) * width;
    // word e of the rows is word c of row r; a step of a workgroup's width moves both on without a division
    const int r0 = tid / width, c0 = tid - r0 * width, dr = kPerturbThreads / width, dc = kPerturbThreads - dr * width;
    auto words = [&](auto f) {
        for (int e = tid, r = r0, c = c0; e < nrow * width; e += kPerturbThreads) {
            f(rows[e], lds[r * rs + c]);
            r += dr;
            c += dc;
            if (c >= width) { c -= width; ++r; }
        }
    };
    if (a.topk > 0) words([](int32_t &g, int32_t &l) { l = g; });      // (with topk == 0 the rows hold nothing yet)
    __syncthreads();
    if (tid < nrow) perturb_row<K, W>(a, i0 + tid, bh, width, lds + tid * rs);
    __syncthreads();
    words([](int32_t &g, int32_t &l) { g = l; });
}

hipError_t launch_perturb(const moc_meta *m, int BH, int topk, int max_in, int causal, float p_max,
                          const uint64_t *thr, uint64_t seed, int32_t *sel, hipStream_t st) {
    PerturbArgs a{};
    a.sel = sel;
    a.chunk_of = m->d_chunk_of; a.win = m->d_win; a.wfirst = m->d_wfirst; a.wlast = m->d_wlast; a.ntb = m->d_ntb;
    a.video = m->d_video;
    a.N = m->N; a.C = m->C; a.topk = topk; a.max_in = max_in; a.causal = causal != 0;
    a.p_max = p_max;
    a.key0 = (uint32_t)seed; a.key1 = (uint32_t)(seed >> 32);
    for (int j = 0; j < max_in; ++j) a.thr[j] = thr[j];
    dim3 grid((m->N + kPerturbThreads - 1) / kPerturbThreads, BH);
    const int width = topk + max_in;
    if (width == 0) return hipSuccess;         // no columns
    MOC_PROF("route_perturb", st);
    const size_t lds_bytes = (size_t)(width | 1) * kPerturbThreads * sizeof(int32_t);   // <= 16.5 KB
    if (topk <= 8 && width <= 12) perturb_kernel<8, 12><<<grid, kPerturbThreads, lds_bytes, st>>>(a);
    else if (topk <= 16 && width <= 20) perturb_kernel<16, 20><<<grid, kPerturbThreads, lds_bytes, st>>>(a);
    else perturb_kernel<32, 32><<<grid, kPerturbThreads, lds_bytes, st>>>(a);
    return hipGetLastError();
}

}  // namespace moc
