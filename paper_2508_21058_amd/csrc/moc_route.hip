// Stages (b2)+(c): routing scores and per-query top-k (Eq. 3; Sec. 3.2 causal
// routing mask; Sec. 3.3 pre-routing mask that removes forced links from the
// candidates).
//
// Scores on matrix cores at fp32 accuracy: the fp32 pooled keys arrive split
// into three bf16 planes (hi + mid + lo == value); a bf16 query is exact, an
// fp32 query is split the same way, and all partial products of order <= 2 are
// accumulated in fp32, so a score differs from the exact inner product only by
// accumulation rounding. S^T[chunk][query] tiles of 32 chunks x 32 queries put
// one query in each lane (two half-waves share a query and own 16 chunks of a
// tile each); the [N, C] score matrix never exists in memory.
//
// Per-lane top-k without branches: a candidate is one 64-bit word, (score, chunk), whose
// order as a double is the order of the selection: higher score first, lower chunk on a
// tie (see entry()). The 16 words of a tile go through a sorting network and are merged
// into the lane's sorted list, v_max_f64 / v_min_f64 pairs that run at the full vector
// rate here; at the end the two half-waves merge their lists. One pass over the chunks;
// any data (ties, few tiles) stays exact, and the time does not depend on the data.
//
// Bound by the sum of these vector instructions, about 260 per tile of 32 x 32 scores (k <= 8, 193 of them the selection), and
// of its 24 matrix instructions, which hardly run side by side: 1,040 and 768 cycles of the 1,700 that a tile takes. Neither
// half the LDS reads nor dealing the ones between the others gains more than 7 % (see launch_route). Against queues of the scores above the k-th best so far,
// inserted entry by entry (divergent, two LDS rows per entry, two waves per SIMD): 1,313
// -> 684 us at 114k tokens, 24 heads, 440 chunks, k = 8; 7,074 -> 4,552 us at 457k tokens,
// six heads, 3,488 chunks, k = 16; 26 -> 15 us at 6,256 tokens, k = 3. The queues cost less per tile the
// longer the scan, as ever fewer scores beat the k-th best; without a causal mask they meet the networks near
// 9,000 chunks (fp32, d = 64, k = 16: 1,260 -> 1,183 us at 5,210 chunks, 3,561 -> 3,720 at 9,418).
#include "moc_attn_common.h"
#include "moc_pool_unit.h"

namespace moc {

// f(IC<0>), f(IC<1>), ..., f(IC<N - 1>)
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F f) {
    if constexpr (I < N) { f(IC<I>{}); static_for<N, I + 1>(f); }
}

struct RouteArgs {
    const void *q;
    const bf16_t *split;          // [BH][3][Cpad][D]
    const int32_t *chunk_of, *win, *wfirst, *wlast;
    const uint32_t *textmask;
    int32_t *sel;
    int N, C, Cpad, topk, causal;
    int turn;                     // blocks of queries from the last one on
    int stride;                   // int32 words between consecutive rows of sel (>= topk)
};

// Under the causal mask the last queries have the most tiles: first, so that a launch ends on short workgroups (457k tokens,
// k = 16: 4,373 -> 4,270 us; four heads of 60k tokens, 968 chunks, k = 11 140 -> 126). Not for wide lists over few tiles where
// a head fills the chip: all of its workgroups then scan at one time and write their rows at another (sixteen heads of
// 100k tokens, k = 11 in rows of 15 words: 120 chunks 194 us in order, 225 turned round, 248 chunks 268 / 289, 488 chunks
// 424 / 423; of 80k tokens 154 / 156, 214 / 214, 344 / 339; k = 8 turned round 2 % faster at any of these).
static int from_last(int N, int C, int topk, int causal) { return causal && (topk <= 8 || C >= 384 || N < 80000); }

// The entry of a candidate: the score's bits as the high word of a double, which read as one is finite
// for every score but a NaN (+-inf become exponent 0x7f8) and ordered like the scores; the low word
// orders equal scores by chunk, ascending (a negative double falls as its low word grows, hence the
// sign mask). A NaN counts as -inf, which is no candidate. (A score is never -0: its sum starts at +0.)
// The score is read straight from a matrix accumulator, so its first reader is a builtin: the compiler puts
// the wait states such a read needs in front of instructions it knows, not in front of inline assembly. The
// infinities come in registers whose values the compiler does not know (see Infinities): of a median with
// constants it makes a minimum, which turns a NaN into +inf.
struct Infinities {
    float neg = -INFINITY, pos = INFINITY;
    __device__ __forceinline__ Infinities() { asm("" : "+s"(neg)); asm("" : "+v"(pos)); }
};
// `chunk` comes as two words whose bits do not overlap, the second a constant: one three-way instruction joins them with
// the sign. Written as operators that took three, 80 of 222 vector instructions a tile at k = 8, now 48: 114k tokens, 24 heads,
// k = 8 565 -> 540 us; 457k tokens, six heads, k = 16 4,155 -> 4,006; d = 64 365 -> 342; 6,256 tokens, k = 8 28.8 -> 27.2.
__device__ __forceinline__ double entry(float score, uint32_t chunk, uint32_t low, const Infinities &inf) {
    // median of score, -inf and +inf: the score, or for a NaN the least of the other two
    const uint32_t hi = __float_as_uint(__builtin_amdgcn_fmed3f(score, inf.neg, inf.pos));
    const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)((int32_t)hi >> 31), chunk, low, 0x69);    // ~(sign ^ chunk ^ low)
    return __hiloint2double((int)hi, (int)lo);
}
// the chunk, or -1 if the entry is no candidate (masked scores are -inf)
__device__ __forceinline__ int entry_chunk(double e) {
    const int hi = __double2hiint(e);
    return __int_as_float(hi) >= -3.0e38f ? __double2loint(e) ^ ~(hi >> 31) : -1;
}

// v_max_f64 / v_min_f64 as they are: fmax() would first quiet signalling NaNs, which entries never are
__device__ __forceinline__ double max64(double a, double b) { double r; asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
__device__ __forceinline__ double min64(double a, double b) { double r; asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }

__device__ __forceinline__ void order2(double &a, double &b) {      // a >= b
    const double t = max64(a, b);
    b = min64(a, b);
    a = t;
}
// the best K of two descending lists of K, descending again: the pairwise
// maxima of one list against the other reversed are the best K as a bitonic sequence
template <int K> __device__ __forceinline__ void merge_entries(double (&list)[K], const double *x) {
#pragma unroll
    for (int p = 0; p < K; ++p) list[K - 1 - p] = max64(list[K - 1 - p], x[p]);
#pragma unroll
    for (int k = K / 2; k >= 1; k /= 2)
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (!(i & k)) order2(list[i], list[i + k]);
}

// The selection of a tile as a list of steps, known at compile time, so that they can be dealt between the matrix
// instructions of the next tile. Per M = min(K, 16) scores: their entries are made, sorted by Batcher's odd-even merge
// network, descending (5 / 19 / 63 pairs for 4 / 8 / 16 entries), and merged into the list, as merge_entries() does.
struct NetStep { uint8_t op, i, j; };
enum : uint8_t { NET_ENTRY, NET_SORT, NET_TAKE, NET_MERGE };
constexpr int net_cost(uint8_t op) { return op == NET_ENTRY ? 3 : (op == NET_TAKE ? 1 : 2); }     // vector instructions
template <int K> struct Net {
    static constexpr int M = K < 16 ? K : 16, kMax = 256;
    NetStep s[kMax];
    int n, cost;
    constexpr void add(uint8_t op, int i, int j) {
        s[n++] = NetStep{op, (uint8_t)i, (uint8_t)j};
        cost += net_cost(op);
    }
    constexpr Net() : s{}, n(0), cost(0) {
        for (int r = 0; r < 16; r += M) {
            for (int i = 0; i < M; ++i) add(NET_ENTRY, r + i, 0);
            for (int p = 1; p < M; p *= 2)
                for (int k = p; k >= 1; k /= 2)
                    for (int i = 0; i < M - 1; ++i)       // pairs (i, i + k) inside blocks of 2 p
                        if (i + k < M && i >= k % p && ((i - k % p) / k) % 2 == 0 && i / (2 * p) == (i + k) / (2 * p))
                            add(NET_SORT, r + i, r + i + k);
            for (int p = 0; p < M; ++p) add(NET_TAKE, K - 1 - p, r + p);
            for (int k = K / 2; k >= 1; k /= 2)
                for (int i = 0; i < K; ++i)
                    if (!(i & k)) add(NET_MERGE, i, i + k);
        }
    }
    // the first step that does not belong to the first `part` of `parts` shares of the cost
    constexpr int cut(int part, int parts) const {
        int i = 0;
        for (int c = 0; i < n && c * parts < cost * part; ++i) c += net_cost(s[i].op);
        return i;
    }
};
template <int K> struct NetOf { static constexpr Net<K> net{}; };

// steps [AT, END) of the network over one lane's scores `sc` of a tile, x being its entries
template <int K, int AT, int END>
__device__ __forceinline__ void net_run(double (&list)[K], double (&x)[16], const f32x16 &sc, uint32_t jb, const Infinities &inf) {
    if constexpr (AT < END) {
        constexpr NetStep st = NetOf<K>::net.s[AT];
        if constexpr (st.op == NET_ENTRY) x[st.i] = entry(sc[st.i], jb, (uint32_t)((st.i >> 2) * 8 + (st.i & 3)), inf);
        else if constexpr (st.op == NET_SORT) order2(x[st.i], x[st.j]);
        else if constexpr (st.op == NET_TAKE) list[st.i] = max64(list[st.i], x[st.j]);
        else order2(list[st.i], list[st.j]);
        net_run<K, AT + 1, END>(list, x, sc, jb, inf);
    }
}

// Four waves x 32 (or 64) queries per workgroup, three workgroups per CU with bf16 queries (120 to 154 registers at
// d = 128), two with fp32 ones of 128 features (three planes of query fragments, 236 to 256 registers) or with 64 queries,
// two staged tiles of pooled keys (one in use, one in flight).
constexpr int kRouteThreads = 256;
constexpr int kRouteStages = 2;

// QG groups of 32 queries a wave: see launch_route.
template <int D, typename T, int KMAX, int QG>
__device__ __forceinline__ void route_body(const RouteArgs &a, char *smem) {
    constexpr int KS = D / 16;
    constexpr int NQ = sizeof(T) == 2 ? 1 : 3;       // query planes
    constexpr int PB = 32 * D * 2;                   // bytes of one plane tile (32 chunks)
    constexpr int TB = 3 * PB;                       // bytes of one staged tile
    constexpr int NWV = kRouteThreads / 64;
    constexpr int QPW = NWV * 32 * QG;               // queries per workgroup

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int bh = blockIdx.y, N = a.N, C = a.C;
    // From the last queries on (see from_last) within every eighth block, so that a block of queries keeps its XCD: the pooling
    // pass before and the perturbed rows' pass behind have the same blocks there, in its L2 (three heads of 8,000 tokens,
    // k = 8: routing 9.8 us and perturbed rows 12.2 turned round as a whole, 9.3 and 10.0 so).
    const int nb = gridDim.x, bx = blockIdx.x, b8 = bx % kXcds;
    const int q0 = (a.turn ? b8 + kXcds * ((nb - b8 + kXcds - 1) / kXcds - 1 - bx / kXcds) : bx) * QPW;
    const int topk = a.topk;
    int i[QG], limit[QG], wf[QG], wl[QG], lim_lo[QG], wf_lo[QG], wl_hi[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        i[g] = q0 + (wave * QG + g) * 32 + l32;
        const int cq = a.chunk_of[min(i[g], N - 1)], w = a.win[cq];
        wf[g] = a.wfirst[w];
        wl[g] = a.wlast[w];
        limit[g] = a.causal ? cq : C;                                   // candidates have index < limit
        // queries ascend with the lane, so do chunk, window and limit
        lim_lo[g] = __builtin_amdgcn_readlane(limit[g], 0);             // smallest limit of the 32 queries
        wf_lo[g] = __builtin_amdgcn_readlane(wf[g], 0);                 // chunks that may be forced links of one of them
        wl_hi[g] = __builtin_amdgcn_readlane(wl[g], 31);
    }
    const int lim_wg = __builtin_amdgcn_readfirstlane(a.causal ? a.chunk_of[min(q0 + QPW - 1, N - 1)] : C);  // uniform: largest limit in the workgroup
    const int ntiles = (lim_wg + 31) >> 5;
    auto out_row = [&](int g) { return a.sel + ((size_t)bh * N + i[g]) * a.stride; };
    if (ntiles == 0) {                                                  // no candidates at all
#pragma unroll
        for (int g = 0; g < QG; ++g)
            if (i[g] < N && half == 0)
                for (int r = 0; r < topk; ++r) out_row(g)[r] = -1;
        return;
    }

    // query operand planes (B operand: lane -> query column)
    bf16x8 qf[QG][NQ][KS];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        const T *qp = static_cast<const T *>(a.q) + ((size_t)bh * N + min(i[g], N - 1)) * D;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (NQ == 1) {
                qf[g][0][s] = Io<T>::load8(qp + s * 16 + half * 8);
            } else {
                float f[8];
                Io<T>::load8f(qp + s * 16 + half * 8, f);
                float hi[8], mid[8], lo[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bf16_t h = (bf16_t)f[e];
                    const float r1 = f[e] - (float)h;
                    const bf16_t m = (bf16_t)r1;
                    hi[e] = (float)h; mid[e] = (float)m; lo[e] = r1 - (float)m;
                }
                u32x4 ph, pm, pl;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ph[e] = pack_bf16(hi[2 * e], hi[2 * e + 1]);
                    pm[e] = pack_bf16(mid[2 * e], mid[2 * e + 1]);
                    pl[e] = pack_bf16(lo[2 * e], lo[2 * e + 1]);
                }
                qf[g][0][s] = __builtin_bit_cast(bf16x8, ph);
                qf[g][NQ > 1 ? 1 : 0][s] = __builtin_bit_cast(bf16x8, pm);
                qf[g][NQ > 2 ? 2 : 0][s] = __builtin_bit_cast(bf16x8, pl);
            }
        }
    }
    // The query fragments are consumed here, before the first tile copy is issued: the waits the
    // compiler needs for their loads then sit in front of the loop, not inside it, where they would
    // also wait for the tile copies in flight.
#pragma unroll
    for (int g = 0; g < QG; ++g)
#pragma unroll
        for (int qa = 0; qa < NQ; ++qa)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                u32x4 w = __builtin_bit_cast(u32x4, qf[g][qa][s]);
                asm volatile("" : "+v"(w));
                qf[g][qa][s] = __builtin_bit_cast(bf16x8, w);
            }
    LaneOffs<D> lo;
    lo.init(lane);

    // Copies of one staged tile (3 planes x 32 rows), spread over the four waves: a wave instruction moves
    // 1 KB (512 / D rows). Every wave issues the same number of copies per tile, six or three, so that one
    // vmcnt bound fits all.
    constexpr int RPI = 512 / D, NI = 32 / RPI, TOT = 3 * NI, PW = (TOT + NWV - 1) / NWV;
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    const int rlo = lane / (D / 8), cgp = lane % (D / 8);
    const bf16_t *sp = a.split + (size_t)bh * 3 * a.Cpad * D;
    auto issue = [&](int t, int buf) {
        const uint32_t at = lds_address(smem + buf * TB);
#pragma unroll
        for (int p = 0; p < PW; ++p) {
            const int n = (uwave + NWV * p) % TOT;
            const int plane = n / NI, sub = n % NI;
            const int row = sub * RPI + rlo;
            const int cg = cgp ^ SwTile<D>::sw(row);
            const bf16_t *src = sp + ((size_t)plane * a.Cpad + (size_t)t * 32) * D;
            async_copy16_at(src, (uint32_t)(row * D + cg * 8) * 2u, at + plane * PB + sub * 1024);
        }
    };
    const Infinities inf;
    double list[QG][KMAX], x[16];        // a lane's best KMAX candidates so far, best first; entries of a tile
#pragma unroll
    for (int g = 0; g < QG; ++g)
#pragma unroll
        for (int p = 0; p < KMAX; ++p) list[g][p] = entry(-INFINITY, 0xffffffffu, 0u, inf);

    // One pass over the products of a staged tile, in the order (query plane, key plane, features); row fragments are
    // read kAhead products ahead. With SELECT the selection over `sc`, the scores of the tile before (whose first chunk
    // for this lane is jb), is dealt between the products.
    struct Scores { f32x16 g[QG]; };
    constexpr int NM = (NQ == 1 ? 3 : 6) * KS, kAhead = 2;
    auto plane_of = [](int m) constexpr { return m / KS < 3 ? m / KS : (m / KS < 5 ? m / KS - 3 : 0); };
    auto qplane_of = [](int m) constexpr { return m / KS < 3 ? 0 : (m / KS < 5 ? 1 : 2); };
    auto tile_pass = [&](auto cur, auto select, const Scores &sc, uint32_t jb) -> Scores {
        constexpr int CUR = decltype(cur)::value;
        constexpr bool SELECT = decltype(select)::value != 0;
        lo.pin_rows();
        Scores acc;
#pragma unroll
        for (int g = 0; g < QG; ++g) acc.g[g] = zero16();
        bf16x8 kf[kAhead + 1];
        auto read = [&](auto m) {
            constexpr int MI = decltype(m)::value;
            if constexpr (MI < NM) kf[MI % (kAhead + 1)] = lo.template frag<CUR * TB + plane_of(MI) * PB>(smem, MI % KS);
        };
        static_for<kAhead>([&](auto m) { read(m); });
        static_for<NM>([&](auto m) {
            constexpr int MI = decltype(m)::value;
            read(IC<MI + kAhead>{});
#pragma unroll
            for (int g = 0; g < QG; ++g) acc.g[g] = mfma32(kf[MI % (kAhead + 1)], qf[g][qplane_of(MI)][MI % KS], acc.g[g]);
            if constexpr (SELECT) {
                constexpr int PG = NM / QG, G = MI / PG;
                constexpr int A = NetOf<KMAX>::net.cut(MI % PG, PG), B = NetOf<KMAX>::net.cut(MI % PG + 1, PG);
                net_run<KMAX, A, B>(list[G], x, sc.g[G], jb, inf);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        return acc;
    };
    // scores of chunks that are no candidates become -inf
    auto mask = [&](Scores &acc, int t) {
        const int j0 = t * 32;
        const uint32_t tm = uniform_load_u32(a.textmask, t);
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            // the tile's chunks but text are candidates for every one of the 32 queries
            const bool inside = j0 + 32 <= lim_lo[g] && (j0 + 32 <= wf_lo[g] || j0 > wl_hi[g]);
            const bool clean = tm == 0 && inside;
            if (!clean) {
                // One 32-bit word per lane, bit b = chunk j0 + b is a candidate of this lane's query:
                // below the causal limit, outside the own window [wf, wl], not text; it differs from text alone only
                // where the limit or the window cuts the tile. The lane takes its 16 bits, (r >> 2) * 8 + half * 4 +
                // (r & 3), at compile-time positions, each as a mask of its score: two instructions where a test and a
                // choice take three. Both together, k = 16: 114k tokens, six heads 177 -> 172 us, 24 heads 647 -> 630, 457k
                // tokens, six heads, 872 chunks 1,117 -> 1,099. (With two groups, k = 8 and all 256 registers taken, the masks
                // cost 106 spills.)
                uint32_t okm = ~tm;
                if (!inside) {
                    auto below = [](int n) { return n >= 32 ? 0xffffffffu : (n <= 0 ? 0u : ((1u << n) - 1u)); };
                    okm &= below(limit[g] - j0) & (below(wf[g] - j0) | ~below(wl[g] - j0 + 1));
                }
                const uint32_t mine = okm >> (half * 4);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    constexpr uint32_t kNegInf = 0xff800000u;
                    const int bit = (r >> 2) * 8 + (r & 3);
                    if constexpr (QG == 1) {
                        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)mine, bit, 1);               // all ones or zero
                        acc.g[g][r] = __uint_as_float((__float_as_uint(acc.g[g][r]) & m) | (kNegInf & ~m));
                    } else if (!((mine >> bit) & 1u)) {
                        acc.g[g][r] = -INFINITY;
                    }
                }
            }
        }
    };
    auto select_all = [&](const Scores &sc, int t) {
        static_for<QG>([&](auto g) {
            constexpr int G = decltype(g)::value;
            net_run<KMAX, 0, NetOf<KMAX>::net.n>(list[G], x, sc.g[G], (uint32_t)(t * 32 + half * 4), inf);
        });
    };

    issue(0, 0);
    if constexpr (QG == 2) {
        if (ntiles > 1) { issue(1, 1); wait_vmcnt<PW>(); } else wait_vmcnt<0>();
        __syncthreads();
        Scores sc = tile_pass(IC<0>{}, IC<0>{}, Scores{}, 0u);
        mask(sc, 0);
        wait_vmcnt<0>();
        __syncthreads();
        // the scores of tile t are in `sc`, tile t + 1 has landed in the other stage
        auto step = [&](auto next, int t) {
            constexpr int NEXT = decltype(next)::value;
            if (t + 1 == ntiles) { select_all(sc, t); return false; }
            const bool more = t + 2 < ntiles;
            if (more) issue(t + 2, NEXT ^ 1);
            sc = tile_pass(next, IC<1>{}, sc, (uint32_t)(t * 32 + half * 4));
            mask(sc, t + 1);
            if (more) { wait_vmcnt<0>(); __syncthreads(); }
            return true;
        };
        for (int t = 0;;) {
            if (!step(IC<1>{}, t++)) break;
            if (!step(IC<0>{}, t++)) break;
        }
    } else {
        wait_vmcnt<0>();
        __syncthreads();
        auto step = [&](auto cur, int t) {
            constexpr int CUR = decltype(cur)::value;
            const bool more = t + 1 < ntiles;
            if (more) issue(t + 1, CUR ^ 1);
            Scores sc = tile_pass(cur, IC<0>{}, Scores{}, 0u);
            mask(sc, t);
            select_all(sc, t);
            if (more) { wait_vmcnt<0>(); __syncthreads(); }
            return more;
        };
        for (int t = 0;;) {
            if (!step(IC<0>{}, t++)) break;
            if (!step(IC<1>{}, t++)) break;
        }
    }

    // ---------------- the upper half-wave's list into the lower one's
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        double up[KMAX];
#pragma unroll
        for (int p = 0; p < KMAX; ++p) {
            const uint32_t h = (uint32_t)__double2hiint(list[g][p]), l = (uint32_t)__double2loint(list[g][p]);
            const auto rh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
            const auto rl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
            up[p] = __hiloint2double((int)rh[1], (int)rl[1]);
        }
        merge_entries<KMAX>(list[g], up);
        if (i[g] >= N || half != 0) continue;
        int32_t *out = out_row(g);
        if ((topk | a.stride) % 4 == 0) {      // rows of whole 16-byte words
#pragma unroll
            for (int p = 0; p < KMAX; p += 4) {
                const u32x4 w = {(uint32_t)entry_chunk(list[g][p]), (uint32_t)entry_chunk(list[g][p + 1]),
                                 (uint32_t)entry_chunk(list[g][p + 2]), (uint32_t)entry_chunk(list[g][p + 3])};
                if (p < topk) *reinterpret_cast<u32x4 *>(out + p) = w;
            }
        } else {
#pragma unroll
            for (int p = 0; p < KMAX; ++p)
                if (p < topk) out[p] = entry_chunk(list[g][p]);
        }
    }
}

template <int D, typename T, int KMAX, int QG>
__global__ __launch_bounds__(kRouteThreads, 2) void route_kernel(RouteArgs a) {
    __shared__ __attribute__((aligned(1024))) char smem[kRouteStages * 3 * 32 * D * 2];
    route_body<D, T, KMAX, QG>(a, smem);
}

// ---------------------------------------------------------------------------------------------
// Pooling, scoring and top-k in ONE launch (the fusion the paper lists as future work, Sec. 5).
// Every query needs the mean key of every earlier chunk, so the scoring part of every workgroup
// depends on the whole pooling pass: the first kFusePoolWgs workgroups of the launch (they are
// dispatched first and never wait before they pool) share the chunks among themselves, count the
// chunks they have finished in a device word, and every workgroup waits for that count before it
// scores. The wait is bounded (kFuseSpinLimit sleeps of a few hundred cycles): if it runs out, a
// flag is raised, the workgroup scores whatever the planes hold, and every wave still exits.
// The words live in a static device array (zero when the module loads); the last workgroup of a
// launch clears them again, so launches must not overlap on one GPU.
// Only the pooling workgroups release and only the end of a wait acquires, since both write back or drop whole
// caches: with an acquire at every look at the count and a release at the end of every workgroup 114k tokens, 24
// heads and k = 8 took 2,697 us, 14k tokens 357, now 1,557 and 169 (as two launches 778 and 46).
constexpr int kFusePoolWgs = 256;
constexpr long long kFuseSpinLimit = 20000000;
static __device__ unsigned int g_fuse_sync[4];       // [0] chunks pooled, [1] workgroups finished, [2] a wait ran out

struct FuseArgs {
    const void *k;
    const int32_t *off;
    float *kbar;
    bf16_t *split;
    unsigned int units;      // Cpad * BH (chunk, head) pairs to pool
};

template <int D, typename T, int KMAX>
__global__ __launch_bounds__(kRouteThreads, 2) void route_fused_kernel(RouteArgs a, FuseArgs f) {
    static_assert(kRouteThreads == 256, "the pooling unit is written for 256 threads");
    __shared__ __attribute__((aligned(1024))) char smem[kRouteStages * 3 * 32 * D * 2];
    static_assert(PoolShape<D, T>::kRedFloats * 4 <= kRouteStages * 3 * 32 * D * 2, "pooling scratch fits the tile buffers");
    const unsigned int wg = blockIdx.y * gridDim.x + blockIdx.x, nwg = gridDim.x * gridDim.y;
    const unsigned int npool = min(nwg, (unsigned int)kFusePoolWgs);
    if (wg < npool) {
        unsigned int done = 0;
        for (unsigned int u = wg; u < f.units; u += npool) {
            pool_unit<D, T>(static_cast<const T *>(f.k), f.off, a.N, a.C, a.Cpad, f.kbar, f.split, (int)(u % a.Cpad),
                            (int)(u / a.Cpad), reinterpret_cast<float *>(smem));
            ++done;
        }
        __syncthreads();                                       // every thread's stores are issued
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(&g_fuse_sync[0], done, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x == 0) {
        long long spins = 0;
        while (__hip_atomic_load(&g_fuse_sync[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < f.units) {
            if (++spins > kFuseSpinLimit) { g_fuse_sync[2] = 1u; break; }
            __builtin_amdgcn_s_sleep(8);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");     // once, not per look: each would drop the L1 of the pooling waves
    }
    __syncthreads();
    route_body<D, T, KMAX, 1>(a, smem);
    __syncthreads();
    if (threadIdx.x == 0) {
        // (no data passes here: the end of the launch publishes the selections)
        const unsigned int fin = __hip_atomic_fetch_add(&g_fuse_sync[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (fin == nwg - 1) {                                  // the last one out: every workgroup is past its wait
            __hip_atomic_store(&g_fuse_sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&g_fuse_sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

hipError_t launch_route_fused(const moc_meta *m, int BH, int d, const void *q, const void *k, float *kbar,
                              void *kb_split, int Cpad, int topk, int causal, int32_t *sel, hipStream_t st) {
    RouteArgs a{};
    a.q = q;
    a.split = static_cast<const bf16_t *>(kb_split);
    a.chunk_of = m->d_chunk_of; a.win = m->d_win; a.wfirst = m->d_wfirst; a.wlast = m->d_wlast;
    a.textmask = m->d_textmask;
    a.sel = sel;
    a.N = m->N; a.C = m->C; a.Cpad = Cpad; a.topk = topk; a.causal = causal != 0;
    a.turn = from_last(a.N, a.C, topk, a.causal);
    a.stride = topk;
    FuseArgs f{k, m->d_off, kbar, static_cast<bf16_t *>(kb_split), (unsigned int)Cpad * (unsigned int)BH};
    dim3 grid((m->N + kRouteThreads / 2 - 1) / (kRouteThreads / 2), BH), block(kRouteThreads);
    MOC_PROF("route_fused", st);
#define MOC_FUSED(DD, KK) route_fused_kernel<DD, bf16_t, KK><<<grid, block, 0, st>>>(a, f)
#define MOC_FUSED_K(DD)                         \
    do {                                        \
        if (topk <= 4) MOC_FUSED(DD, 4);        \
        else if (topk <= 8) MOC_FUSED(DD, 8);   \
        else if (topk <= 16) MOC_FUSED(DD, 16); \
        else MOC_FUSED(DD, 32);                 \
    } while (0)
    if (d == 128) MOC_FUSED_K(128); else MOC_FUSED_K(64);
#undef MOC_FUSED_K
#undef MOC_FUSED
    return hipGetLastError();
}

// blocking: has any wait of a fused launch run out since the module was loaded? (also clears the flag)
hipError_t fused_wait_flag(int *timed_out) {
    unsigned int w[4] = {};
    hipError_t e = hipMemcpyFromSymbol(w, HIP_SYMBOL(g_fuse_sync), sizeof(w), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    *timed_out = w[2] != 0;
    if (w[2]) {
        const unsigned int zero = 0;
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_fuse_sync), &zero, sizeof(zero), 2 * sizeof(unsigned int), hipMemcpyHostToDevice);
    }
    return e;
}

// Two groups of 32 queries a wave read a tile's fragments once for both and have registers left (227 to 256, two
// workgroups a compute unit) for the scores of a tile and of the next, so that the selection of one runs between the
// products of the other. 24 heads, bf16, d = 128, causal, one group / two: 114k tokens, k = 8, 440 chunks 549 / 538 us, 872
// 962 / 921, k = 3, 440 chunks 502 / 476; 457k tokens, six heads, 3,488 chunks, k = 8 3,466 / 3,253. It needs a chip full
// several times over with half the workgroups (6,256 tokens, 600 of them: 15 / 18). Below 80,000 tokens it also needs
// - under the causal mask: workgroups that are short against a head, since they end at their own tile and every eighth
//   is on one XCD (8,000 tokens, 144 heads, 136 chunks, k = 8 116 / 157; 64 chunks 88 / 93; 424 242 / 327; 16,000 tokens,
//   72 heads, 440 chunks 241 / 246), and one or two tiles, or a dozen (33k tokens, 48 heads, k = 8: 64 chunks
//   117 / 118, 136 149 / 157, 264 222 / 224, 328 263 / 264, 440 327 / 324, 696 476 / 468; k = 3: 113 / 109, 140 / 143, 203 / 200, 240 / 237,
//   299 / 290, 435 / 418; 66k tokens, 24 heads, 136 chunks, k = 8 149 / 156);
// - without it: not four or five tiles (8,000 tokens, 300 heads, k = 8: 64 chunks 188 / 182, 104 282 / 299, 136 341 / 358;
//   33k tokens, 48 heads, 136 chunks 223 / 223, 200 300 / 298, 440 564 / 544).
// Wider lists spill (k = 16: 4,270 / 15,809), d = 64 gains nothing (375 / 374 at k = 8), nor does fp32 there (116 / 165,
// spills). One group with the selection dealt takes as long as without, or longer (457k tokens, k = 16: 4,380 / 4,547).
constexpr long long kPairWgs = 4096;
static bool pair_of_groups(int N, int C, long long wgs, int causal) {
    if (wgs < kPairWgs) return false;
    if (N >= 80000) return true;
    return causal ? N >= 32768 && (C <= 64 || C >= 384) : C <= 96 || C > 160;
}

hipError_t launch_route(const moc_meta *m, int BH, int d, int dtype, const void *q, const void *kb_split, int Cpad,
                        int topk, int causal, int32_t *sel, int sel_stride, hipStream_t st) {
    RouteArgs a{};
    a.q = q;
    a.split = static_cast<const bf16_t *>(kb_split);
    a.chunk_of = m->d_chunk_of; a.win = m->d_win; a.wfirst = m->d_wfirst; a.wlast = m->d_wlast;
    a.textmask = m->d_textmask;
    a.sel = sel;
    a.N = m->N; a.C = m->C; a.Cpad = Cpad; a.topk = topk; a.causal = causal != 0;
    a.turn = from_last(a.N, a.C, topk, a.causal);
    a.stride = sel_stride;
    MOC_PROF("route_topk", st);
    auto run = [&](auto dd, auto kk, auto tt) {
        constexpr int DD = decltype(dd)::value, KK = decltype(kk)::value;
        using T = decltype(tt);
        if constexpr (KK <= 8 && sizeof(T) == 2 && DD == 128) {
            const int wgs = (m->N + kRouteThreads - 1) / kRouteThreads;
            if (pair_of_groups(m->N, m->C, (long long)wgs * BH, causal)) {
                route_kernel<DD, T, KK, 2><<<dim3(wgs, BH), dim3(kRouteThreads), 0, st>>>(a);
                return;
            }
        }
        route_kernel<DD, T, KK, 1><<<dim3((m->N + kRouteThreads / 2 - 1) / (kRouteThreads / 2), BH), dim3(kRouteThreads), 0, st>>>(a);
    };
    auto by_k = [&](auto dd, auto tt) {
        if (topk <= 4) run(dd, IC<4>{}, tt);
        else if (topk <= 8) run(dd, IC<8>{}, tt);
        else if (topk <= 16) run(dd, IC<16>{}, tt);
        else run(dd, IC<32>{}, tt);
    };
    if (dtype == MOC_BF16) { if (d == 128) by_k(IC<128>{}, bf16_t{}); else by_k(IC<64>{}, bf16_t{}); }
    else { if (d == 128) by_k(IC<128>{}, float{}); else by_k(IC<64>{}, float{}); }
    return hipGetLastError();
}

}  // namespace moc
