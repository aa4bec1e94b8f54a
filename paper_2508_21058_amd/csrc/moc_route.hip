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
// Bound by these vector instructions: about 240 per tile of 32 x 32 scores (k <= 8) beside
// its 24 matrix instructions. Against queues of the scores above the k-th best so far,
// inserted entry by entry (divergent, two LDS rows per entry, two waves per SIMD): 1,313
// -> 684 us at 114k tokens, 24 heads, 440 chunks, k = 8; 7,074 -> 4,552 us at 457k tokens,
// six heads, 3,488 chunks, k = 16; 26 -> 15 us at 6,256 tokens, k = 3. The queues cost less per tile the
// longer the scan, as ever fewer scores beat the k-th best; without a causal mask they meet the networks near
// 9,000 chunks (fp32, d = 64, k = 16: 1,260 -> 1,183 us at 5,210 chunks, 3,561 -> 3,720 at 9,418).
#include "moc_attn_common.h"
#include "moc_pool_unit.h"

namespace moc {

struct RouteArgs {
    const void *q;
    const bf16_t *split;          // [BH][3][Cpad][D]
    const int32_t *chunk_of, *win, *wfirst, *wlast;
    const uint32_t *textmask;
    int32_t *sel;
    int N, C, Cpad, topk, causal;
    int stride;                   // int32 words between consecutive rows of sel (>= topk)
};

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
__device__ __forceinline__ double entry(float score, uint32_t chunk, const Infinities &inf) {
    // median of score, -inf and +inf: the score, or for a NaN the least of the other two
    const uint32_t hi = __float_as_uint(__builtin_amdgcn_fmed3f(score, inf.neg, inf.pos));
    const uint32_t lo = chunk ^ ~(uint32_t)((int32_t)hi >> 31);
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
// Batcher's odd-even merge sort, descending: 5 / 19 / 63 pairs for 4 / 8 / 16 entries
template <int M> __device__ __forceinline__ void sort_entries(double *x) {
#pragma unroll
    for (int p = 1; p < M; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int i = 0; i < M - 1; ++i)       // pairs (i, i + k) inside blocks of 2 p
                if (i + k < M && i >= k % p && ((i - k % p) / k) % 2 == 0 && i / (2 * p) == (i + k) / (2 * p))
                    order2(x[i], x[i + k]);
}
// the best K of a descending list of K and a descending list of M <= K, descending again: the pairwise
// maxima of one list against the other reversed are the best K as a bitonic sequence
template <int K, int M> __device__ __forceinline__ void merge_entries(double (&list)[K], const double *x) {
#pragma unroll
    for (int p = 0; p < M; ++p) list[K - 1 - p] = max64(list[K - 1 - p], x[p]);
#pragma unroll
    for (int k = K / 2; k >= 1; k /= 2)
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (!(i & k)) order2(list[i], list[i + k]);
}

// Four waves x 32 queries per workgroup, three workgroups per CU with bf16 queries (132 to 166 registers at d = 128),
// two with fp32 ones of 128 features (three planes of query fragments, 232 to 256 registers), two staged tiles of
// pooled keys (one in use, one in flight). The pass is bound by the selection's vector instructions, not by the latency
// of the tile copies.
constexpr int kRouteThreads = 256;
constexpr int kRouteStages = 2;

template <int D, typename T, int KMAX>
__device__ __forceinline__ void route_body(const RouteArgs &a, char *smem) {
    constexpr int KS = D / 16;
    constexpr int NQ = sizeof(T) == 2 ? 1 : 3;       // query planes
    constexpr int PB = 32 * D * 2;                   // bytes of one plane tile (32 chunks)
    constexpr int TB = 3 * PB;                       // bytes of one staged tile
    constexpr int NWV = kRouteThreads / 64;
    constexpr int QPW = kRouteThreads / 2;           // queries per workgroup

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int bh = blockIdx.y, N = a.N, C = a.C;
    const int q0 = blockIdx.x * QPW;
    const int i = q0 + wave * 32 + l32;
    const bool valid = i < N;
    const int ic = valid ? i : N - 1;
    const int cq = a.chunk_of[ic];
    const int w = a.win[cq];
    const int wf = a.wfirst[w], wl = a.wlast[w];
    const int limit = a.causal ? cq : C;                               // candidates have index < limit
    // queries ascend with the lane, so do chunk, window and limit
    const int lim_wg = __builtin_amdgcn_readfirstlane(a.causal ? a.chunk_of[min(q0 + QPW - 1, N - 1)] : C);  // uniform: largest limit in the workgroup
    const int ntiles = (lim_wg + 31) >> 5;
    const int lim_lo = __shfl(limit, 0, 64);                            // smallest limit in the wave
    const int wf_lo = __shfl(wf, 0, 64), wl_hi = __shfl(wl, 31, 64);    // chunks that may be forced links in the wave
    const int topk = a.topk;
    int32_t *out = a.sel + ((size_t)bh * N + ic) * a.stride;
    if (ntiles == 0) {                                                  // no candidates at all
        if (valid && half == 0)
            for (int r = 0; r < topk; ++r) out[r] = -1;
        return;
    }

    // query operand planes (B operand: lane -> query column)
    bf16x8 qf[NQ][KS];
    {
        const T *qp = static_cast<const T *>(a.q) + ((size_t)bh * N + ic) * D;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (NQ == 1) {
                qf[0][s] = Io<T>::load8(qp + s * 16 + half * 8);
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
                qf[0][s] = __builtin_bit_cast(bf16x8, ph);
                qf[NQ > 1 ? 1 : 0][s] = __builtin_bit_cast(bf16x8, pm);
                qf[NQ > 2 ? 2 : 0][s] = __builtin_bit_cast(bf16x8, pl);
            }
        }
    }
    // The query fragments are consumed here, before the first tile copy is issued: the waits the
    // compiler needs for their loads then sit in front of the loop, not inside it, where they would
    // also wait for the tile copies in flight.
#pragma unroll
    for (int qa = 0; qa < NQ; ++qa)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            u32x4 w = __builtin_bit_cast(u32x4, qf[qa][s]);
            asm volatile("" : "+v"(w));
            qf[qa][s] = __builtin_bit_cast(bf16x8, w);
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
    // tile t + 1 has landed once at most the copies of the tiles after it are still in flight
    constexpr int DIST = kRouteStages - 1;           // tiles issued ahead of the one in use
    auto landed = [&](int t_next) {
        if (DIST > 1 && t_next + DIST - 1 < ntiles) wait_vmcnt<(DIST - 1) * PW>(); else wait_vmcnt<0>();
    };

    // scores of tile t for this lane: 16 chunks, ineligible ones set to -inf
    auto scores = [&](auto cur, int t) -> f32x16 {
        constexpr int CUR = decltype(cur)::value;
        lo.pin();
        f32x16 acc = zero16();
#pragma unroll
        for (int qa = 0; qa < NQ; ++qa)
#pragma unroll
            for (int kp = 0; kp < 3; ++kp) {
                if (qa + kp > 2) continue;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    bf16x8 kf;
                    if (kp == 0) kf = lo.template frag<CUR * TB>(smem, s);
                    else if (kp == 1) kf = lo.template frag<CUR * TB + PB>(smem, s);
                    else kf = lo.template frag<CUR * TB + 2 * PB>(smem, s);
                    acc = mfma32(kf, qf[qa][s], acc);
                }
            }
        const int j0 = t * 32;
        const uint32_t tm = uniform_load_u32(a.textmask, t);
        // fast path: the whole tile is a candidate for every query of the wave
        const bool clean = tm == 0 && j0 + 32 <= lim_lo && (j0 + 32 <= wf_lo || j0 > wl_hi);
        if (!clean) {
            // One 32-bit word per lane, bit b = chunk j0 + b is a candidate of this lane's query:
            // below the causal limit, outside the own window [wf, wl], not text. The lane then
            // tests its 16 bits, (r >> 2) * 8 + half * 4 + (r & 3), at compile-time positions.
            auto below = [](int n) { return n >= 32 ? 0xffffffffu : (n <= 0 ? 0u : ((1u << n) - 1u)); };
            const uint32_t okm = below(limit - j0) & (below(wf - j0) | ~below(wl - j0 + 1)) & ~tm;
            const uint32_t mine = okm >> (half * 4);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!((mine >> ((r >> 2) * 8 + (r & 3))) & 1u)) acc[r] = -INFINITY;
        }
        return acc;
    };

    // ---------------- the lane's best KMAX candidates so far, best first
    const Infinities inf;
    double list[KMAX];
#pragma unroll
    for (int p = 0; p < KMAX; ++p) list[p] = entry(-INFINITY, 0xffffffffu, inf);
    auto scan = [&](auto cur, int t) {
        constexpr int CUR = decltype(cur)::value;
        constexpr int M = KMAX < 16 ? KMAX : 16;       // entries sorted and merged at a time
        const bool more = t + 1 < ntiles;
        if (t + DIST < ntiles) issue(t + DIST, (CUR + DIST) % kRouteStages);
        const f32x16 sc = scores(cur, t);
        const uint32_t jb = (uint32_t)(t * 32 + half * 4);
        double x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = entry(sc[r], jb ^ (uint32_t)((r >> 2) * 8 + (r & 3)), inf);
#pragma unroll
        for (int r = 0; r < 16; r += M) {
            sort_entries<M>(x + r);
            merge_entries<KMAX, M>(list, x + r);
        }
        if (more) { landed(t + 1); __syncthreads(); }
        return more;
    };
#pragma unroll
    for (int u = 0; u < DIST; ++u)
        if (u < ntiles) issue(u, u);
    landed(0);
    __syncthreads();
    for (int t = 0;;) {
        if (!scan(IC<0>{}, t++)) break;
        if (!scan(IC<1 % kRouteStages>{}, t++)) break;
        if (kRouteStages > 2 && !scan(IC<2 % kRouteStages>{}, t++)) break;
    }

    // ---------------- the upper half-wave's list into the lower one's
    double up[KMAX];
#pragma unroll
    for (int p = 0; p < KMAX; ++p) {
        const uint32_t h = (uint32_t)__double2hiint(list[p]), l = (uint32_t)__double2loint(list[p]);
        const auto rh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
        const auto rl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
        up[p] = __hiloint2double((int)rh[1], (int)rl[1]);
    }
    merge_entries<KMAX, KMAX>(list, up);
    if (valid && half == 0) {
        if ((topk | a.stride) % 4 == 0) {      // rows of whole 16-byte words
#pragma unroll
            for (int p = 0; p < KMAX; p += 4) {
                const u32x4 w = {(uint32_t)entry_chunk(list[p]), (uint32_t)entry_chunk(list[p + 1]),
                                 (uint32_t)entry_chunk(list[p + 2]), (uint32_t)entry_chunk(list[p + 3])};
                if (p < topk) *reinterpret_cast<u32x4 *>(out + p) = w;
            }
        } else {
#pragma unroll
            for (int p = 0; p < KMAX; ++p)
                if (p < topk) out[p] = entry_chunk(list[p]);
        }
    }
}

template <int D, typename T, int KMAX>
__global__ __launch_bounds__(kRouteThreads, kRouteThreads == 256 ? 2 : 1) void route_kernel(RouteArgs a) {
    __shared__ __attribute__((aligned(1024))) char smem[kRouteStages * 3 * 32 * D * 2];
    route_body<D, T, KMAX>(a, smem);
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
    route_body<D, T, KMAX>(a, smem);
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

hipError_t launch_route(const moc_meta *m, int BH, int d, int dtype, const void *q, const void *kb_split, int Cpad,
                        int topk, int causal, int32_t *sel, int sel_stride, hipStream_t st) {
    RouteArgs a{};
    a.q = q;
    a.split = static_cast<const bf16_t *>(kb_split);
    a.chunk_of = m->d_chunk_of; a.win = m->d_win; a.wfirst = m->d_wfirst; a.wlast = m->d_wlast;
    a.textmask = m->d_textmask;
    a.sel = sel;
    a.N = m->N; a.C = m->C; a.Cpad = Cpad; a.topk = topk; a.causal = causal != 0;
    a.stride = sel_stride;
    dim3 grid((m->N + kRouteThreads / 2 - 1) / (kRouteThreads / 2), BH), block(kRouteThreads);
    MOC_PROF("route_topk", st);
#define MOC_ROUTE(DD, TT, KK) route_kernel<DD, TT, KK><<<grid, block, 0, st>>>(a)
#define MOC_ROUTE_K(DD, TT)                         \
    do {                                            \
        if (topk <= 4) MOC_ROUTE(DD, TT, 4);        \
        else if (topk <= 8) MOC_ROUTE(DD, TT, 8);   \
        else if (topk <= 16) MOC_ROUTE(DD, TT, 16); \
        else MOC_ROUTE(DD, TT, 32);                 \
    } while (0)
    if (dtype == MOC_BF16) { if (d == 128) MOC_ROUTE_K(128, bf16_t); else MOC_ROUTE_K(64, bf16_t); }
    else { if (d == 128) MOC_ROUTE_K(128, float); else MOC_ROUTE_K(64, float); }
#undef MOC_ROUTE_K
#undef MOC_ROUTE
    return hipGetLastError();
}

}  // namespace moc
