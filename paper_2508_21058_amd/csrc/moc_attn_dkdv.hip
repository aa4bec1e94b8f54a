// dK / dV of whole key tiles (256 keys of one chunk, or its last 160 to 255), heads of 128 features: the key-stationary pass for calls with
// many of them. The ragged rest of such calls, heads of 64 features and small calls take attn_bwd_dkdv_pipe_kernel.
//
// A workgroup is four waves, one per SIMD with all 512 of its registers: a wave owns 64 keys, holds their dK^T and dV^T
// (the 256 accumulation registers) and the operands of K (64 vector registers), and streams every query that attends
// them past, 16 at a time. P and dS never leave the wave: the scores are formed as 16 x 16 blocks (queries x keys), whose
// accumulators become operands of the gradient products by exchanging half of their words with the lanes 16 away. Against
// two roles of waves of 32 keys (the other kernel) a tile row is read from LDS once per 64 keys instead of 32, nothing waits for
// another wave's P, and a chunk's queries are fetched once per 256 keys instead of 128. dK/dV of 24 heads, the other kernel
// alone / with this one: 181,760 tokens, 1,280- to 10,240-key chunks 154.4 / 140.5 ms (1,120 -> 1,230 TFLOP/s), 114k tokens,
// 260-key chunks (whose last four keys stay with the other kernel) 17.05 / 16.22, 33k tokens 3.20 / 3.04, six heads of 457k
// tokens in 130-key chunks (captions only) 36.6 / 34.6.
//
// What bounds it is that a SIMD has one wave to issue from, an instruction every four cycles at best: 16 queries against 64
// keys are 1,024 cycles of the matrix pipe and 225 instructions (900 cycles of issue), 48 of them its own, and take 1,550. On
// 181,760 tokens it issues 56 % of its cycles, has an instruction that the pipe or its operands hold back 32 % and waits for copies
// or a barrier 12 %; the matrix pipe is busy 66 % (63 % on 114k tokens of 260-key chunks, whose items are shorter). Hence the step
// is written out in slots, and what is issued in the shadow of which product matters: scheduling left to the compiler within a slot
// 13 % slower; LDS reads behind the 16-cycle score products instead of the 32-cycle gradient product 3 %; a barrier every 16 queries
// instead of every 32 1 %. Without the exponentials a timing-only build takes 5 % less, without the reads of V 6 %.
#include "moc_attn_bwd.h"

namespace moc {

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The accumulation registers are named in the assembly: given variables, the compiler copies half of them to vector registers
// and back around every product. It is told that each of these statements destroys all of them, so nothing of its own
// lives there across one (tests/test_asm_wait_states.py reads the assembly for it: nothing else touches them).
#define MOC_ACC_REGS \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", \
    "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", \
    "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", \
    "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", \
    "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", \
    "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", \
    "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", \
    "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", \
    "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", \
    "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", \
    "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", \
    "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", \
    "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", \
    "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", \
    "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", \
    "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
// a[REG .. REG + 15] += A * B
template <int REG> __device__ __forceinline__ void mfma32_acc(bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" :: "v"(a), "v"(b), "n"(REG), "n"(REG + 15) : MOC_ACC_REGS);
}
// ... whose operands a vector instruction may just have written: two wait states, which the compiler does not add for
// inline assembly
template <int REG> __device__ __forceinline__ void mfma32_acc_late(bf16x8 a, bf16x8 b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" :: "v"(a), "v"(b), "n"(REG), "n"(REG + 15) : MOC_ACC_REGS);
}
template <int REG> __device__ __forceinline__ void acc_zero4() {
    asm volatile("v_accvgpr_write_b32 a[%0], 0\n\tv_accvgpr_write_b32 a[%1], 0\n\tv_accvgpr_write_b32 a[%2], 0\n\tv_accvgpr_write_b32 a[%3], 0"
                 :: "n"(REG), "n"(REG + 1), "n"(REG + 2), "n"(REG + 3) : MOC_ACC_REGS);
}
template <int REG> __device__ __forceinline__ float acc_read() {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(REG) : MOC_ACC_REGS);
    return v;
}
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F f) {
    if constexpr (I < N) { f(IC<I>{}); static_for<I + 1, N>(f); }
}

// The copies of moc_device.h with bases and destinations that are in scalar registers already (asked for again in every step,
// the compiler keeps them in vector registers and reads them back right in front of the copy).
__device__ __forceinline__ void copy16(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void copy16(const void *at, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(at), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void copy4(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void copy4(const void *at, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" :: "v"(at), "s"(lds) : "memory", "m0");
}

namespace wide {
constexpr int D = 128, KS = D / 32, DB = D / 32;        // feature steps of the score products, feature blocks of the gradients
constexpr int NB = 4, KB = NB / 2, KW = NB * 16;        // 16- and 32-key blocks of a wave, its keys
constexpr int R = 16, RB = D * 2;                       // queries of a stage, bytes of a row
constexpr int TB = R * RB, SB = 2 * TB;                 // bytes of a stage's Q (or dO) rows, of a stage
// Eight stages: 64 KB, the reach of an LDS instruction's offset, so that a step (eight of them make the loop's body) needs
// no address arithmetic. Rows of stage n + L go out in step n, statistics 2 L ahead.
constexpr int NST = 8, L = NST - 3;
constexpr int RECB = R * 16, RECN = 2 * NST;            // bytes of a stage's records, stages of their ring
constexpr int LPT = 3;                                  // vector-memory operations of a wave and stage: Q, dO, records
constexpr int RECS = NST * SB, VALUES = RECS + RECN * RECB, LDS = VALUES + 4 * NB * KS * 1024;
constexpr int AK = KB * DB * 16;                        // dV^T in a[0 ..], dK^T in a[AK ..]; block (x, y) at (x * DB + y) * 16
constexpr int NF = 2 * DB;                              // transposed fragments of a stage: dO, Q of feature block 0, 1 ..
constexpr int J = 16;                                   // slots of a step: a gradient product, a pair of score products, a 64th of the exponentials
constexpr int DG = 3;                                   // slots by which the gradient products of a stage reach into the next step
constexpr int LA = 4;                                   // slots between a transposed read and its first product
constexpr int VA = 4;                                   // fragments of V held: each is read VA - 1 slots ahead
static_assert(NF * KB == J && NB * KS == J && NB * 4 == J && LDS <= 160 * 1024);
}  // namespace wide

// OT: storage type of dK and dV. BIG: rows beyond the reach of 32-bit byte offsets
template <typename OT, bool BIG>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkdv_wide_kernel(KvArgs a) {
    using namespace wide;
    typedef bf16_t T;
    __shared__ __attribute__((aligned(1024))) char smem[LDS];     // stages; records; V
    int bh, item_no;
    if (!kv_item(a.n_items, a.n_text, a.BH, bh, item_no)) return;
    // scalars before any address is made of them (see TileIter::start)
    bh = __builtin_amdgcn_readfirstlane(bh);
    item_no = __builtin_amdgcn_readfirstlane(item_no);
    const bool caption = item_no < a.n_text;
    KvItem item = a.items[caption ? item_no + item_no / a.text_tiles * (a.join - 1) * a.text_tiles : item_no - a.n_text + a.video_at];
    if (caption) item.q_len = min(a.text_seg, a.N - item.q_start);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31, l16 = lane & 15, quad = lane >> 4;
    const int N = a.N;

    const bool routed = item.chunk >= 0 && a.topk > 0;
    const int32_t *loff = a.list_off + (size_t)bh * (a.C + 1);
    const int lbeg = __builtin_amdgcn_readfirstlane(routed ? loff[item.chunk] : 0);
    const int n_list = __builtin_amdgcn_readfirstlane(routed ? loff[item.chunk + 1] : 0) - lbeg;
    const int n_win = (item.q_len + R - 1) / R;                   // stages of the window's queries; the list's follow
    const int n_st = n_win + (n_list + R - 1) / R;
    if (n_st == 0) return;

    // ---- copies: a wave moves four rows of Q and of dO a stage
    const char *const qbase = static_cast<const char *>(uniform_ptr(static_cast<const char *>(a.q) + (size_t)bh * N * RB));
    const char *const dobase = static_cast<const char *>(uniform_ptr(static_cast<const char *>(a.d_o) + (size_t)bh * N * RB));
    const int rlo = lane >> 4;
    const uint32_t vcol = (uint32_t)(((lane & 15) ^ SwTile<D>::sw(wave * 4 + rlo)) * 16);
    const uint32_t smem_at = lds_address(smem) + wave * 1024, recs_at = lds_address(smem) + RECS;
    auto issue_rows = [&](int word, int slot) {
        const uint32_t dst = smem_at + slot * SB;
        if constexpr (BIG) {
            const size_t off = ((size_t)(uint32_t)(word >> 5) * RB) | vcol;
            copy16(qbase + off, dst);
            copy16(dobase + off, dst + TB);
        } else {
            const uint32_t off = ((uint32_t)(word & ~31) * (RB / 32)) | vcol;
            copy16(qbase, off, dst);
            copy16(dobase, off, dst + TB);
        }
    };
    // Records, in LDS [stage & 15][group of four queries][lse2, delta, list word, spare: four each]. Every wave copies those of
    // the whole stage, a dword a lane (the four write the same words), so that it may read the list words as soon as its own
    // copies have landed. Padding rows, past the last stage too, repeat the last record of their window or list with lse2 = +inf
    // (P = dS = 0): rows and records go out in every step, and a vmcnt bound counts whole stages. Zero times a NaN or an infinity
    // is not zero, so a padding row may only be one that attends these keys anyway (its own would leave the same NaN there).
    const int rec_row = rlo * 4 + (lane & 3), rec_sel = ((lane >> 2) & 3) * 4;
    const uint32_t rec_off = (uint32_t)(rec_row * 16 + rec_sel);
    const char *const inf_rec = reinterpret_cast<const char *>(a.stats2) + (size_t)a.BH * N * 16;
    const char *rec_ptr = reinterpret_cast<const char *>(a.stats2) + ((size_t)bh * N + item.q_start) * 16;
    const char *const rec_list = reinterpret_cast<const char *>(a.gstats2) + ((size_t)bh * N * a.topk + lbeg) * 16;
    int rec_left = item.q_len, rec_more = n_list;
    uint32_t rec_slot = 0;
    auto issue_record = [&]() {
        const uint32_t dst = recs_at + rec_slot;
        rec_slot = (rec_slot + RECB) & (RECN * RECB - 1);
        if (rec_left >= R) {
            copy4(rec_ptr, rec_off, dst);
        } else {
            if (rec_left <= 0 && rec_more > 0) { rec_ptr = rec_list; rec_left = rec_more; rec_more = 0; }
            // (past the last stage rec_left - 1 is negative and leads back to the last record)
            const char *const at = rec_ptr + (min(rec_row, rec_left - 1) * 16 + rec_sel);
            copy4(rec_row >= rec_left && rec_sel == 0 ? inf_rec : at, dst);
        }
        rec_ptr += RECB;
        rec_left -= R;
    };
    auto word_of = [&](int at) {
        return *reinterpret_cast<const __attribute__((address_space(3))) int *>((uintptr_t)(recs_at + wave * 64 + 32 + rlo * 4 + at));
    };
    for (int u = 0; u < L; ++u) issue_record();

    // ---- keys and values of the wave: K in registers, -V in LDS (for want of 64 more registers), both as operands
    char *const vals = smem + VALUES + wave * (NB * KS * 1024) + lane * 16;
    bf16x8 kf[NB][KS];
    {
        const char *kbase = static_cast<const char *>(a.k) + (size_t)bh * N * RB;
        const char *vbase = static_cast<const char *>(a.v) + (size_t)bh * N * RB;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const size_t row = (size_t)(item.key_start + min(wave * KW + b * 16 + l16, item.key_len - 1)) * RB + quad * (KS * 16);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                kf[b][s] = Io<T>::load8(reinterpret_cast<const T *>(kbase + row + s * 16));
                u32x4 v = __builtin_bit_cast(u32x4, Io<T>::load8(reinterpret_cast<const T *>(vbase + row + s * 16)));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] ^= 0x80008000u;
                *reinterpret_cast<u32x4 *>(vals + (s * NB + b) * 1024) = v;
            }
        }
    }
    // the stage "before the first", whose gradients the first step adds with P = dS = 0
#pragma unroll
    for (int x = 0; x < SB / 4096; ++x) *reinterpret_cast<u32x4 *>(smem + (NST - 1) * SB + x * 4096 + tid * 16) = u32x4{0, 0, 0, 0};
    if (n_win < L) wait_vmcnt<0>();           // list words of the first stages
    for (int u = 0; u < L; ++u) {
        issue_rows(u < n_win ? (item.q_start + min(u * R + wave * 4 + rlo, item.q_len - 1)) << 5 : word_of(u * RECB), u);
        issue_record();
    }
    static_for<0, AK / 2>([](auto r) { acc_zero4<4 * decltype(r)::value>(); });

    // Lane offsets: rows as operands, transposed pieces, records of the lane's four queries. Contraction step s of the scores
    // takes the 16-byte groups KS * quad + s of a row (K and V alike): with neighbouring groups in a step two rows of every
    // sixteen lanes that read together would share banks.
    int rowa[KS], tra[2 * DB];
#pragma unroll
    for (int s = 0; s < KS; ++s) rowa[s] = l16 * RB + (((KS * quad + s) ^ SwTile<D>::sw(l16)) << 4);
#pragma unroll
    for (int u = 0; u < 2 * DB; ++u) {
        const int x = 32 * (u >> 1) + 16 * (quad & 1) + 4 * (l16 & 3), r0 = 8 * half + (l16 >> 2) + 4 * (u & 1);
        tra[u] = (SwTile<D>::off(r0, x >> 3) + (x & 7)) * 2;
    }
    int par = 0;                               // first stage of the loop's body in the ring of records, in bytes
    const float c = a.scale_log2;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    auto rowfrag = [&](int at) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(smem + at)); };
    auto trfrag = [&](int f, int at) {         // fragment f of the stage at byte `at`
        const int t = at + ((f & 1) ? 0 : TB);
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + tra[f & ~1] + t));
        const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + tra[f | 1] + t));
        return __builtin_bit_cast(bf16x8, s16x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]});
    };
    auto vload = [&](int y) { return *reinterpret_cast<const bf16x8 *>(vals + y * 1024); };
    auto stat = [&](int at, int sel) { return *reinterpret_cast<const f32x4 *>(smem + RECS + quad * 64 + sel * 16 + at); };
    // Two 16-key blocks' P (or dS), four queries a lane each, become an operand of eight queries a lane: words 0, 1 are the
    // first block's, 2, 3 the second's; `h` exchanges word h of both.
    auto exchange = [](uint32_t (&w)[4], int h) {
        const auto r = __builtin_amdgcn_permlane16_swap(w[h], w[2 + h], false, false);
        w[h] = r[0];
        w[2 + h] = r[1];
    };
    auto operand = [](const uint32_t (&w)[4]) { return __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]}); };

    bf16x8 tf[4], rq[2], rd[2], vq[VA];
    f32x4 SA[NB], PA[NB], SBb[NB], PB[NB], lse, del;
    bf16x8 pf[KB], df[KB];                     // P and dS operands of the stage whose gradient products are running
    uint32_t pn[KB][4], dn[KB][4];             // ... of the stage behind it (scalars: a vector built over two steps spills)
    float p_last[2], d_last[2];                // its last two elements
#pragma unroll
    for (int x = 0; x < KB; ++x) {
        pf[x] = df[x] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
#pragma unroll
        for (int i = 0; i < 4; ++i) pn[x][i] = dn[x][i] = 0u;
    }
    p_last[0] = p_last[1] = d_last[0] = d_last[1] = 0.f;
    int word;                                  // list word of the lane's row of the stage to be copied

    // One step (n % 8 = H): vector half of stage n (S, Pd -> P, dS), score products of stage n + 1 (Sn, Pn), gradient products
    // of stage n - 1, the last DG of them in the next step. The scheduling barriers keep the order of issue.
    auto step = [&](auto hc, f32x4 *S, f32x4 *Pd, f32x4 *Sn, f32x4 *Pn) {
        constexpr int H = decltype(hc)::value;
        constexpr int PRV = (H + NST - 1) % NST * SB, CUR = H * SB, NXT = (H + 1) % NST * SB, NX2 = (H + 2) % NST * SB;
        auto rec_at = [&](auto k) {            // records of stage n + k
            constexpr int u = H + decltype(k)::value;
            return (u >= NST ? par ^ (NST * RECB) : par) + u % NST * RECB;
        };
        if constexpr (H % 2 == 0) {            // stages n + 2 and n + 3 have landed: all copies but those of n + 4
            wait_vmcnt<LPT>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        issue_record();
        uint32_t pw[KB][4], dw[KB][4];
        float ps[J];
        f32x4 lse_next;
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, J>([&](auto jc) {
            constexpr int j = decltype(jc)::value, g = (j + J - DG) % J, f = g / KB, kb = g % KB, s = j / NB, b = j % NB;
            Sn[b] = mfma16(rq[s & 1], kf[b][s], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : Sn[b]);
            __builtin_amdgcn_sched_barrier(0);
            ps[j] = __builtin_amdgcn_exp2f(fmaf(S[j >> 2][j & 3], c, -lse[j & 3]));
            __builtin_amdgcn_sched_barrier(0);
            Pn[b] = mfma16(rd[s & 1], vq[j % VA], s == 0 ? del : Pn[b]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j == 0) {            // the stage before: its last elements
                pn[KB - 1][3] = pack_bf16(p_last[0], p_last[1]);
                dn[KB - 1][3] = pack_bf16(d_last[0], d_last[1]);
            } else {
                constexpr int e = j - 1, eb = e >> 2, i = e & 3;
                Pd[eb][i] *= ps[e];
                if constexpr (e & 1) {
                    pw[eb >> 1][(eb & 1) * 2 + (i >> 1)] = pack_bf16(ps[e - 1], ps[e]);
                    dw[eb >> 1][(eb & 1) * 2 + (i >> 1)] = pack_bf16(Pd[eb][i - 1], Pd[eb][i]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            mfma32_acc<(f & 1) * AK + (kb * DB + (f >> 1)) * 16>(tf[f & 3], (f & 1) ? df[kb] : pf[kb]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j == 1 || j == 2) { exchange(pn[KB - 1], j - 1); exchange(dn[KB - 1], j - 1); }
            if constexpr (j == 9 || j == 10) { exchange(pw[0], j - 9); exchange(dw[0], j - 9); }
            if constexpr (j == DG - 1)
#pragma unroll
                for (int x = 0; x < KB; ++x) pf[x] = operand(pn[x]);
            if constexpr (b == 0) {
                constexpr int at = s + 1 < KS ? NXT : NX2;
                rq[(s + 1) & 1] = rowfrag(rowa[(s + 1) % KS] + at);
                rd[(s + 1) & 1] = rowfrag(rowa[(s + 1) % KS] + at + TB);
            }
            vq[(j + VA - 1) % VA] = vload((j + VA - 1) % J);
            constexpr int jl = j + LA - DG;    // transposed fragment read ahead, at the end the next stage's first
            if constexpr (jl % KB == 0) tf[jl / KB & 3] = trfrag(jl / KB % NF, jl < J ? PRV : CUR);
            if constexpr (j == J - 3) lse_next = stat(rec_at(IC<1>{}), 0);
            if constexpr (j == J - 2) del = stat(rec_at(IC<2>{}), 1);
            if constexpr (j == J - 6) word = word_of(rec_at(IC<L>{}));
            if constexpr (j == J - 1) issue_rows(word, (H + L) % NST);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j == DG - 1)
#pragma unroll
                for (int x = 0; x < KB; ++x) df[x] = operand(dn[x]);
        });
        p_last[0] = ps[J - 2]; p_last[1] = ps[J - 1];
        d_last[0] = Pd[NB - 1][2]; d_last[1] = Pd[NB - 1][3] * ps[J - 1];
#pragma unroll
        for (int x = 0; x < KB; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (x < KB - 1 || i < 3) pn[x][i] = pw[x][i], dn[x][i] = dw[x][i];
        lse = lse_next;
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- scores of the first stage, and what the first step expects in registers
    wait_vmcnt<0>();
    __syncthreads();
    del = stat(0, 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8 q8 = rowfrag(rowa[s]), d8 = rowfrag(rowa[s] + TB);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            SA[b] = mfma16(q8, kf[b][s], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : SA[b]);
            PA[b] = mfma16(d8, vload(s * NB + b), s == 0 ? del : PA[b]);
        }
    }
    lse = stat(0, 0);
    del = stat(RECB, 1);
    rq[0] = rowfrag(rowa[0] + SB);
    rd[0] = rowfrag(rowa[0] + SB + TB);
#pragma unroll
    for (int y = 0; y < VA; ++y) vq[y] = vload(y);
#pragma unroll
    for (int f = 0; f < 4; ++f) tf[f] = trfrag(0, (NST - 1) * SB);
    // whole turns of the ring (an exit between two steps makes the compiler spill); the steps past the last stage add zeros
    for (int n = 0; n < n_st; n += NST) {
        step(IC<0>{}, SA, PA, SBb, PB);
        step(IC<1>{}, SBb, PB, SA, PA);
        step(IC<2>{}, SA, PA, SBb, PB);
        step(IC<3>{}, SBb, PB, SA, PA);
        step(IC<4>{}, SA, PA, SBb, PB);
        step(IC<5>{}, SBb, PB, SA, PA);
        step(IC<6>{}, SA, PA, SBb, PB);
        step(IC<7>{}, SBb, PB, SA, PA);
        par ^= NST * RECB;
    }
    // the last gradient products of the stage before the last, and those of the last
    static_for<0, DG>([&](auto jc) {
        constexpr int g = J - DG + decltype(jc)::value, f = g / KB, kb = g % KB;
        mfma32_acc_late<(f & 1) * AK + (kb * DB + (f >> 1)) * 16>(tf[f & 3], (f & 1) ? df[kb] : pf[kb]);
    });
    pn[KB - 1][3] = pack_bf16(p_last[0], p_last[1]);
    dn[KB - 1][3] = pack_bf16(d_last[0], d_last[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) { exchange(pn[KB - 1], h); exchange(dn[KB - 1], h); }
#pragma unroll
    for (int x = 0; x < KB; ++x) pf[x] = operand(pn[x]), df[x] = operand(dn[x]);
    static_for<0, J>([&](auto jc) {
        constexpr int g = decltype(jc)::value, f = g / KB, kb = g % KB;
        if (kb == 0) tf[0] = trfrag(f, (NST - 1) * SB);
        mfma32_acc_late<(f & 1) * AK + (kb * DB + (f >> 1)) * 16>(tf[0], (f & 1) ? df[kb] : pf[kb]);
    });
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // the last products are in their registers
    wait_vmcnt<0>();                                        // the copies past the last stage

    // ---- results: lane = key, registers = features; the accumulator holds -dK
    const float dks = -a.scale;
    static_for<0, KB * DB * 4>([&](auto w) {
        constexpr int r = 4 * decltype(w)::value, x = r / (DB * 16), y = r / 16 % DB, g = r / 4 % 4;
        const int kr = wave * KW + x * 32 + l32, col = y * 32 + g * 8 + half * 4;
        const f32x4 v4 = {acc_read<r>(), acc_read<r + 1>(), acc_read<r + 2>(), acc_read<r + 3>()};
        const f32x4 k4 = {acc_read<AK + r>() * dks, acc_read<AK + r + 1>() * dks, acc_read<AK + r + 2>() * dks, acc_read<AK + r + 3>() * dks};
        if (kr < item.key_len) {
            if (item.partial < 0) {
                const size_t row = ((size_t)bh * N + item.key_start + kr) * D + col;
                Io<OT>::store4(static_cast<OT *>(a.dk) + row, k4[0], k4[1], k4[2], k4[3]);
                Io<OT>::store4(static_cast<OT *>(a.dv) + row, v4[0], v4[1], v4[2], v4[3]);
            } else {
                const size_t row = (((size_t)bh * a.n_partials + item.partial) * a.key_tile + kr) * D + col;
                *reinterpret_cast<f32x4 *>(a.tpart_k + row) = k4;
                *reinterpret_cast<f32x4 *>(a.tpart_v + row) = v4;
            }
        }
    });
}

hipError_t launch_dkdv_wide(const KvArgs &kv, int dtype, hipStream_t st) {
    const dim3 grid(kv_grid(kv.n_items, kv.n_text, kv.BH)), block(256);
    const bool big = (long long)kv.N * wide::RB >= (1ll << 32);
    if (dtype == MOC_BF16) {
        if (big) attn_bwd_dkdv_wide_kernel<bf16_t, true><<<grid, block, 0, st>>>(kv);
        else attn_bwd_dkdv_wide_kernel<bf16_t, false><<<grid, block, 0, st>>>(kv);
    } else {
        if (big) attn_bwd_dkdv_wide_kernel<float, true><<<grid, block, 0, st>>>(kv);
        else attn_bwd_dkdv_wide_kernel<float, false><<<grid, block, 0, st>>>(kv);
    }
    return hipGetLastError();
}

}  // namespace moc
