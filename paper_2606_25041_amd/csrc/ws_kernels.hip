// gfx950 (MI355X) kernels for block-causal streaming attention.
//
// Block-causal rule (Wan-Streamer v0.1, Abstract; Sec. 1 with Fig. 1): a
// token sees its whole own block and every earlier block; a block may end in
// a token-causal segment (the thinker's language and state slots, Sec. 1 and
// Sec. 2.4) whose tokens see the segment only up to themselves.  The step
// kernel runs the current unit against its full-history cache (Sec. 2.4);
// the prefill kernel covers whole sequences (Sec. 2.4, system prefill); the
// append kernel commits a KV slice to the paged cache (Sec. 2.4).  The
// gradient kernels, which serve training in the same causal format
// (Sec. 2.3), are in ws_bwd.hip.
//
// Attention kernel design (one work-group = one work item: a tile of 256
// query rows of one (stream, KV head) group and one KV split, 8 waves x 32
// rows; in the prefill the rows are tokens of one query head of the group,
// in a step they are packed (token, query head) rows, every query head of
// the group for consecutive new tokens):
//  * S^T = K Q^T on v_mfma_f32_32x32x16_bf16: K (A operand) from LDS, Q (B
//    operand) resident in registers.  In the 32x32 accumulator layout a lane
//    owns one query column and 16 keys, so row max/sum are in-lane plus one
//    v_permlane32_swap per 64-key tile.
//  * Online softmax in the log2 domain (scale*log2(e) folded into one FMA),
//    fp32 running max/sum per lane, lazy rescale of O; a tile's max is only
//    taken when some row may need a larger running max.
//  * O^T += V^T P^T on the same MFMA: P stays in registers (the accumulator
//    layout of S^T is exactly the B-operand layout once the 16 keys of each
//    MFMA step are permuted consistently on both operands); V is read with
//    ds_read_b64_tr_b16 from a row-major LDS tile, so no transpose pass.
//  * K/V tiles of 64 keys (= one cache page) go from global memory straight
//    into a 5-stage LDS ring (global_load_lds_dwordx4), three tiles in flight
//    while the current one is used; rows are XOR-swizzled in 16-byte chunks
//    so both the K reads and the V transpose reads are bank-conflict free.
//  * Two waves share each SIMD and run the same loop one block apart: while
//    one issues the MFMAs of a tile (S^T of this one, P V of the previous
//    tile), the other computes its softmax; a work-group barrier separates
//    the blocks.
//  * Tiles past the last visible key of the query tile are never loaded
//    (block-granularity skip); tiles fully visible to every row of the query
//    tile run without element masks; only the tiles straddling a block
//    boundary (or the end of the keys) apply per-element masks.
//  * Work items are ordered by KV group (stream, KV head) and mapped
//    XCD-aware: consecutive logical items land on the same XCD so query heads
//    and query tiles that read the same K/V share that XCD's L2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "ws_kernels.h"
#include "ws_device_util.h"

namespace ws {
namespace {

constexpr int KT = 64;        // keys per tile (= page size)
constexpr float RESCALE_LOG2 = 8.f;  // lazy-rescale threshold (log2 units)
constexpr float RESCALE_BOUND = 256.f;  // 2^RESCALE_LOG2
constexpr int NSTAGE = 5;            // K/V tiles resident in the LDS ring (loads three tiles ahead)
constexpr int RAHEAD = 4;            // LDS operand reads issued this many MFMAs ahead

// The fused append's share of step work item ai of the napp items of its
// (stream, KV head): they split the new tokens evenly; tokens t >= nl are
// padding and not committed.  One 16-byte chunk per thread.
template <int D, int NT>
__device__ __forceinline__ void append_share(const AttnArgs &a, int b, int kvh, int ai, int napp, int n_pool, int nl,
                                             const int32_t *ptab, int tid) {
    constexpr int CH = D / 8;
    const int s0 = (int)((int64_t)ai * a.Lq / napp);
    const int n = max(min((int)((int64_t)(ai + 1) * a.Lq / napp), nl) - s0, 0) * CH;
    for (int u = tid; u < n; u += NT) {
        const int t = s0 + u / CH, c = u % CH;
        const int pos = n_pool + t;
        const int64_t dst = (((int64_t)ptab[pos >> 6] * a.Hkv + kvh) * KT + (pos & 63)) * D + 8 * c;
        *(u32x4 *)(a.kpool + dst) = *(const u32x4 *)(a.kc + b * a.kc_sb + (int64_t)t * a.kc_st + kvh * a.kc_sh + 8 * c);
        *(u32x4 *)(a.vpool + dst) = *(const u32x4 *)(a.vc + b * a.vc_sb + (int64_t)t * a.vc_st + kvh * a.vc_sh + 8 * c);
    }
}

// What a launch does, fixed at compile time: a kernel that serves one kind of
// call carries fewer scalars through its loop (spilled: contiguous prefill 14,
// split step 22, per-stream 45 to 49; one kernel for all had 22) and none of
// the others' code through the instruction cache, where short launches spend
// their time.  Prefill of 2 x 16384 tokens 3.93 -> 3.76 ms; its loop still reads
// five spilled scalars back per tile.
enum Kind { PREFILL_CONTIGUOUS, PREFILL_PAGED, STEP, STEP_SPLIT, STEP_RAGGED };

// STEP_SPLIT: every item writes partials, none rows of the output.
// STEP_RAGGED: the streams have their own split counts (rp).
struct NoPlan {};
template <bool RAGGED>
using Plan = std::conditional_t<RAGGED, RaggedPlan, NoPlan>;

//
// KG = 2 (prefill): the work-group takes 128 query rows, and its two halves of
// four waves the even and the odd key tiles of the same rows, merged through
// LDS at the end.  Twice the work items, each half as long, for the same
// matrix work, at twice the tile loads per query row: for sequences whose
// 256-row items leave compute units idle.
template <int D, int NW, int NB, int KIND, bool F32, int KG>
__global__ __launch_bounds__(NW * 64) void attn_kernel(const AttnArgs a, const Plan<KIND == STEP_RAGGED> rp) {
    constexpr bool step = KIND == STEP || KIND == STEP_SPLIT || KIND == STEP_RAGGED;
    constexpr bool RAGGED = KIND == STEP_RAGGED;
    constexpr int NT = NW * 64;
    constexpr int QT = NW * 32 * NB / KG;  // query rows per work-group
    static_assert(KG == 1 || (KG == 2 && !step), "key groups: prefill only");
    constexpr int ROWB = 2 * D;            // bytes of one key row
    constexpr int TILEB = KT * ROWB;       // bytes of one K (or V) tile
    constexpr int RPW = 1024 / ROWB;       // key rows per wave-wide 16-byte load
    constexpr int LPR = ROWB / 16;         // lanes per key row in such a load
    constexpr int NWD = NW / 2;            // waves that load tiles (the leading half)
    constexpr int NI = TILEB / (NWD * 1024);  // wave-wide loads per loading wave per tile, each of K and V
    constexpr int KK = D / 16;             // MFMA k-steps over head_dim for S^T
    constexpr int MD = D / 32;             // 32-row blocks of head_dim for O^T
    constexpr int VRING = NSTAGE * TILEB;  // byte offset of the V ring
    static_assert(NI >= 1 && TILEB % (NWD * 1024) == 0, "a tile splits into wave-wide loads");
    __shared__ __attribute__((aligned(1024))) char smem[2 * NSTAGE * TILEB];

    // ---- work item ------------------------------------------------------
    // The launch parameters the decode and the query loads need are read in
    // one batch (the asm makes them all live at once, so the compiler issues
    // their loads together and waits once, instead of one round trip per
    // field as each is first used); divisions use the host's dividers.
    const uint32_t bid = blockIdx.x;
    uint32_t per_xcd = a.per_xcd, n_work = a.n_work, per_group = a.per_group, per_qt = a.per_qt;
    uint32_t G = a.G, gi = a.gi, Hkv = a.Hkv, nqt = a.nqt, nrows = a.nrows, lens0 = a.lens_arg[0];
    uint32_t has_nl = a.has_new_lens;
    FastDiv fd_group = a.fd_group, fd_qt = a.fd_qt, fd_g = a.fd_g, fd_hkv = a.fd_hkv, fd_split = a.fd_split;
    FastDiv fd_gq = a.fd_gq;
    const uint16_t *qptr = a.q;
    int64_t q_sb = a.q_sb, q_st = a.q_st, q_sh = a.q_sh;
    asm volatile("" : "+s"(per_xcd), "+s"(n_work), "+s"(per_group), "+s"(per_qt), "+s"(G), "+s"(gi), "+s"(Hkv),
                      "+s"(nqt), "+s"(nrows), "+s"(lens0), "+s"(fd_group.mul), "+s"(fd_group.shift),
                      "+s"(fd_qt.mul), "+s"(fd_qt.shift), "+s"(fd_g.mul), "+s"(fd_g.shift), "+s"(fd_hkv.mul),
                      "+s"(fd_hkv.shift), "+s"(fd_split.mul), "+s"(fd_split.shift), "+s"(fd_gq.mul),
                      "+s"(fd_gq.shift), "+s"(qptr), "+s"(q_sb), "+s"(q_st), "+s"(q_sh), "+s"(has_nl));
    // Ragged: lane p of each half-wave reads plan position p in the same
    // round trip; the item's stream is then picked by a ballot and its fields
    // by lane reads, so no load depends on the item.
    i32x4 pos[3];
    if constexpr (RAGGED) {
#pragma unroll
        for (int i = 0; i < 3; ++i) pos[i] = ((const i32x4 *)&rp.pos[threadIdx.x & 31])[i];
        asm volatile("" : "+v"(pos[0]), "+v"(pos[1]), "+v"(pos[2]));
    }
    // Work-group i runs on XCD i mod 8, which takes the contiguous items
    // [x, x + 1) * per_xcd: whole KV groups, so that an XCD's work-groups share
    // their keys in its L2.  A prefill of few rounds (units > 0) takes the
    // groups' items dealt to `deal` classes and the classes of an XCD in turn,
    // so that its longest items start first and every XCD has its share.
    uint32_t group, idx;
    if (!step && a.units > 0) {
        const uint32_t j = bid / NUM_XCD, pos = fastdiv(j, a.fd_units);
        const uint32_t unit = (bid % NUM_XCD) * (uint32_t)a.units + (j - pos * (uint32_t)a.units);
        group = unit >> a.deal_log2;
        idx = (pos << a.deal_log2) + (unit & ((1u << a.deal_log2) - 1));
        if (idx >= per_group) return;
    } else {
        const uint32_t w = (bid % NUM_XCD) * per_xcd + bid / NUM_XCD;
        if (w >= n_work) return;
        group = fastdiv(w, fd_group);
        idx = w - group * per_group;
    }
    uint32_t qi, split;
    int b, kvh, hh = 0, ppos = 0;
    auto field = [&](int i) -> int { return __builtin_amdgcn_readlane(pos[i >> 2][i & 3], ppos); };
    if constexpr (RAGGED) {
        kvh = (int)group;
        const uint32_t cls = fastdiv(idx, rp.fd_class);
        idx = (idx - cls * (uint32_t)rp.per_class) * (uint32_t)rp.deal + cls;
        if (idx >= (uint32_t)rp.n_items) return;
        ppos = (__builtin_popcountll(__builtin_amdgcn_ballot_w64((uint32_t)pos[0][0] <= idx)) >> 1) - 1;
        b = field(1);
        idx -= (uint32_t)field(0);
        fd_split.mul = (uint32_t)field(8);
        fd_split.shift = (uint32_t)field(9);
        qi = fastdiv(idx, fd_split);
        split = idx - qi * (uint32_t)field(2);
    } else {
        qi = fastdiv(idx, fd_qt);
        const uint32_t rem = idx - qi * per_qt;
        split = fastdiv(rem, fd_g);
        hh = (int)(rem - split * gi);
        // Groups are taken stream-major; a step over blocks of different
        // lengths takes them KV-head-major instead, so that the contiguous
        // range of items each XCD runs mixes long and short streams rather
        // than holding a few streams only.
        if (has_nl) {
            kvh = (int)fastdiv(group, a.fd_b);
            b = (int)(group - (uint32_t)kvh * (uint32_t)a.B);
        } else {
            b = (int)fastdiv(group, fd_hkv);
            kvh = (int)(group - b * Hkv);
        }
    }
    const int hq = kvh * (int)G + hh;   // (prefill; a step's rows span the group's heads)
    // token and query head of packed row p (see AttnArgs)
    auto row_token = [&](int p) -> int { return step ? (int)fastdiv((uint32_t)p, fd_gq) : p; };
    auto row_head = [&](int p, int t) -> int { return step ? kvh * (int)G + (p - t * (int)G) : hq; };
    const int qt = step ? (int)qi : (int)(nqt - 1 - qi);  // prefill: heaviest tiles first
    const int q0 = qt * QT;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hf = lane >> 5;     // which half of the wave
    const int l32 = lane & 31;
    // 32-row block of the tile this wave computes: the trailing waves (which
    // issue no tile loads) take the first blocks, so a small block's rows go
    // to waves without load duty
    const int rblk = KG == 2 ? wave % (NW / 2) : (wave + NW / 2) % NW;
    const int kg = KG == 2 ? wave / (NW / 2) : 0;   // key group: tiles t_begin + kg, + 2, ...

    // A step tile whose first token lies past its stream's new block (blocks
    // of different lengths, padded) holds no real row: it computes nothing
    // and leaves its rows' outputs unwritten, but still does its share of
    // the fused append.  Decided before any load is issued.
    if (!RAGGED && step && has_nl) {
        const int nl0 = a.lens_in_args ? a.nl_arg[b] : ld_uniform(a.new_lens, b);
        if ((int)fastdiv((uint32_t)q0, fd_gq) >= nl0) {
            if (a.fuse_append) {
                const int np0 = a.lens_in_args ? a.lens_arg[b] : ld_uniform(a.cache_lens, b);
                append_share<D, NT>(a, b, kvh, (int)(qi * a.nsplit + split), a.nqt * a.nsplit, np0, nl0,
                                    a.page_table + (int64_t)b * a.max_pages, tid);
            }
            return;
        }
    }

    // Query rows of this wave go global -> LDS -> registers, issued first
    // thing: the direct loads stay in order with the tile loads, so one
    // counted wait covers both.  They are staged in the last two ring stages
    // (of the K ring for waves 0..3, of the V ring for waves 4..7), which are
    // first refilled in loop steps t_begin and t_begin + 1, after every wave
    // has passed the prologue barrier.  The layout is that of a key tile, so the fragments
    // are read like K.
    static_assert(NB == 1, "query staging holds 32 rows per wave");
    constexpr int QI = 32 * ROWB / 1024;   // wave-wide loads per wave
    const uint32_t q_stage = (uint32_t)((wave < 4 ? 0 : VRING) + (NSTAGE - 2) * TILEB + (wave & 3) * 32 * ROWB);
    {
        const char *qg = (const char *)(qptr + b * q_sb);
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            const int r = i * RPW + lane / LPR;   // row within the wave's 32
            const int ch = (lane % LPR) ^ swz<D>(r);
            const int p = min(q0 + rblk * 32 + r, (int)nrows - 1);
            const int t = row_token(p);
            const int h = row_head(p, t);
            dma16(qg + (int64_t)t * (2 * q_st) + (int64_t)h * (2 * q_sh) + 16 * ch, lds_addr(smem) + q_stage + i * 1024);
        }
    }

    // ---- key range ------------------------------------------------------
    // Every row sees a prefix [0, kend) of the keys, and kend does not
    // decrease along the rows of a tile, so the tile's first and last rows
    // give the keys all rows see (kfull) and the keys any row sees (k_hi).
    const int32_t *offs = step ? nullptr : a.offsets + (int64_t)b * (a.nb + 1);
    const int32_t *text = (!step && a.has_text) ? a.text_starts + (int64_t)b * a.nb : nullptr;
    int n_pool, k_hi, kfull, ts = 0, nl = 0;
    BlockWindow win;   // (prefill)
    if constexpr (RAGGED) {
        n_pool = field(4);
        nl = field(5);
        ts = field(6);
    } else if (step) {
        n_pool = !a.lens_in_args ? ld_uniform(a.cache_lens, b) : b == 0 ? (int)lens0 : a.lens_arg[b];
        // start of the new block's token-causal segment (Lq: none) and the
        // block's length (Lq: no padding); new token t sees
        // n_pool + min(nl, max(ts, t + 1)) keys
        ts = a.lens_in_args ? a.text_arg[b] : a.has_text ? ld_uniform(a.text_starts, b) : a.Lq;
        nl = a.lens_in_args ? a.nl_arg[b] : a.has_new_lens ? ld_uniform(a.new_lens, b) : a.Lq;
    }
    if (step) {
        const int t_last = (int)fastdiv((uint32_t)(min(q0 + QT, (int)nrows) - 1), fd_gq);
        k_hi = n_pool + min(nl, max(ts, t_last + 1));
        kfull = n_pool + min(nl, max(ts, (int)fastdiv((uint32_t)q0, fd_gq) + 1));
    } else {
        n_pool = KIND == PREFILL_PAGED ? a.Lq : 0;
        const int q_last = min(q0 + QT, a.Lq) - 1;
        win = block_window(offs, text, a.nb, q0, lane);
        k_hi = token_key_end(win, q_last, lane);
        kfull = token_key_end(win, q0, lane);
    }
    const int ntile = (k_hi + KT - 1) / KT;
    // (split * ntile < 2^31: ntile < 2^25 and split < MAX_SPLITS = 32)
    const int t_begin = (int)fastdiv(split * (uint32_t)ntile, fd_split);
    const int t_end = (int)fastdiv((split + 1) * (uint32_t)ntile, fd_split);

    // ---- page ids -------------------------------------------------------
    // The first four tiles' pages are read up front; later ones one loop
    // step before their tile's loads are issued (a scalar load, waited for
    // with the tile loads), so no page-table read sits in front of them.
    const int32_t *ptab = a.page_table + (int64_t)b * a.max_pages;
    const int tp_end = min(t_end, (n_pool + KT - 1) / KT);   // tiles with cache rows
    auto page_glb = [&](int t) -> int { return KIND != PREFILL_CONTIGUOUS && t < tp_end ? ld_uniform(ptab, t) : 0; };

    // ---- this lane's query rows -------------------------------------------
    // row n of the lane: q0 + rblk * 32 * NB + 32 * n + l32 (the fragments
    // are staged through LDS in the pipeline prologue, below)
    int row[NB], kend[NB], tok[NB], hqr[NB];
    bf16x8 qf[NB][KK];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        row[n] = q0 + rblk * 32 * NB + 32 * n + l32;
        const int pc = min(row[n], (int)nrows - 1);
        tok[n] = row_token(pc);
        hqr[n] = row_head(pc, tok[n]);
        if constexpr (step) kend[n] = n_pool + min(nl, max(ts, tok[n] + 1));
        else kend[n] = lane_key_end(win, min(q0 + rblk * 32 * NB + 32 * n, (int)nrows - 1), tok[n], lane);
    }

    // ---- direct-to-LDS tile loads -----------------------------------------
    // The leading waves (wave < NWD) load the tiles.  Wave-wide load i of
    // such a wave fills tile bytes [(i * NWD + wave) * 1024, +1024): lane
    // `lane` writes 16 bytes at +16 * lane, i.e. slot lane % LPR of key row
    // lrow0 + i * NWD * RPW, and so fetches the chunk that belongs there,
    // lch = slot ^ swz(row).  The swizzle depends on the row modulo 16 only,
    // so lch is the same for all i.
    static_assert((NWD * RPW) % 16 == 0, "the swizzle must repeat across a wave's loads");
    const int lwave = KG == 2 ? wave % NWD : wave;   // (two key groups: either half loads)
    const int lrow0 = lwave * RPW + lane / LPR;
    const int lch = (lane % LPR) ^ swz<D>(lrow0);
    const char *kpool_b = (const char *)a.kpool;
    const char *vpool_b = (const char *)a.vpool;
    const char *kc_b = (const char *)(a.kc + b * a.kc_sb + kvh * a.kc_sh);
    const char *vc_b = (const char *)(a.vc + b * a.vc_sb + kvh * a.vc_sh);
    const int64_t kst2 = 2 * a.kc_st, vst2 = 2 * a.vc_st;
    // per-lane byte offsets: within a (page, KV head) tile, and within the
    // contiguous rows starting at this wave's first row (token strides are
    // below 2^24 elements, checked on the host)
    uint32_t lofs_p = (uint32_t)(lrow0 * ROWB + 16 * lch);
    uint32_t lofs_k = (uint32_t)((lane / LPR) * kst2 + 16 * lch);
    uint32_t lofs_v = (uint32_t)((lane / LPR) * vst2 + 16 * lch);
    // Loads of one tile u (its physical page, if cached, is `page`,
    // wave-uniform) into ring stage s: NI wave-wide loads for K and for V.
    // A tile inside one cache page or inside the contiguous keys is loaded
    // from a wave-uniform base + i * step and a per-lane offset, so its loads
    // can be spread out (issue_part); a tile straddling the cache end or the
    // last key is loaded at once with per-lane addresses (issue_straddle).
    struct TileLoad {
        const char *bk, *bv;   // wave-uniform bases of load 0
        int64_t sk, sv;        // base step per load
        uint32_t ok, ov;       // per-lane byte offsets
        uint32_t kd, vd;       // LDS destination of load 0 of this wave
        bool straddle;
    };
    auto plan_tile = [&](int u, int s, int page) -> TileLoad {
        const int kt = u * KT;
        TileLoad t;
        t.kd = lds_addr(smem) + s * TILEB + lwave * 1024;
        t.vd = t.kd + VRING;
        t.straddle = false;
        if (KIND != PREFILL_CONTIGUOUS && kt + KT <= n_pool) {
            // whole tile in one cache page
            const int64_t tb = ((int64_t)page * a.Hkv + kvh) * TILEB;
            t.bk = kpool_b + tb;
            t.bv = vpool_b + tb;
            t.sk = t.sv = NWD * 1024;
            t.ok = t.ov = lofs_p;
        } else if (KIND != PREFILL_PAGED && kt >= n_pool && kt + KT <= k_hi) {
            // whole tile in the contiguous keys
            const int64_t j0 = kt - n_pool + lwave * RPW;
            t.bk = kc_b + j0 * kst2;
            t.bv = vc_b + j0 * vst2;
            t.sk = NWD * RPW * kst2;
            t.sv = NWD * RPW * vst2;
            t.ok = lofs_k;
            t.ov = lofs_v;
        } else {
            t.straddle = true;
        }
        return t;
    };
    auto issue_part = [&](const TileLoad &t, int i) {
        dma16s(t.bk + i * t.sk, t.ok, t.kd + i * NWD * 1024);
        dma16s(t.bv + i * t.sv, t.ov, t.vd + i * NWD * 1024);
    };
    // rows past the end repeat the last key (their scores are masked)
    auto issue_straddle = [&](int u, int s, int page) {
        const int kt = u * KT;
        const uint32_t kd = lds_addr(smem) + s * TILEB + lwave * 1024;
        const uint32_t vd = kd + VRING;
        const int64_t tb = ((int64_t)page * a.Hkv + kvh) * TILEB;
        const char *kg = kpool_b + tb, *vg = vpool_b + tb;
        const int64_t c0 = (int64_t)(kt - n_pool);   // contiguous row of the tile's first key
        const char *kcg = kc_b + c0 * kst2, *vcg = vc_b + c0 * vst2;
        const uint32_t lofs_c = lofs_p - lrow0 * ROWB;   // the chunk's byte offset in a row
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = min(lrow0 + i * NWD * RPW, k_hi - 1 - kt);   // row within the tile
            const char *gk, *gv;
            if (KIND == PREFILL_PAGED || (step && kt + r < n_pool)) {
                gk = kg + (uint32_t)(r * ROWB) + lofs_c;
                gv = vg + (uint32_t)(r * ROWB) + lofs_c;
            } else {
                gk = kcg + (uint32_t)(r * kst2) + lofs_c;
                gv = vcg + (uint32_t)(r * vst2) + lofs_c;
            }
            dma16(gk, kd + i * NWD * 1024);
            dma16(gv, vd + i * NWD * 1024);
        }
    };
    // all loads of tile u at once
    auto issue_tile = [&](int u, int s, int page) {
        const TileLoad t = plan_tile(u, s, page);
        if (t.straddle) {
            issue_straddle(u, s, page);
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) issue_part(t, i);
        }
        // the waits count this tile's loads as one group: keep later memory
        // operations from being moved in between
        asm volatile("" ::: "memory");
    };
    // wait until at most `younger` tiles' loads are still in flight
    auto wait_tiles = [&](int younger) {
        if (younger >= 2) wait_vm_lgkm<4 * NI>();
        else if (younger == 1) wait_vm_lgkm<2 * NI>();
        else wait_vm_lgkm<0>();
    };

    // ---- LDS read addresses -----------------------------------------------
    // K (A operand of S^T = K Q^T): lane (l32, hf) reads key row 32 * mb + l32,
    // chunk 2 * kk + hf, at kbase ^ (32 * kk): the row offset has no bits
    // below 128 and chunk 2 * kk ^ swz only changes bits 5.. of the slot.
    uint32_t kbase = l32 * ROWB + 16 * (hf ^ swz<D>(l32));
    // V^T fragments (A operand of O^T += V^T P^T) by transpose reads: lane
    // reads key rows 16 * ks4 + vr and +8, 4 head-dim columns of chunk
    // 4 * md + vc, at vbase[e] ^ (64 * md).
    const int j16 = lane & 15;
    uint32_t vbase[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int vr = 4 * hf + (j16 >> 2) + 8 * e;
        const int vc = 2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1);
        vbase[e] = VRING + vr * ROWB + 16 * (vc ^ swz<D>(vr)) + 8 * (j16 & 1);
    }

    auto read_q = [&]() {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            qf[0][kk] = *(const bf16x8 *)(smem + q_stage + (kbase ^ (32 * kk)));
    };

    const float c2 = a.scale_log2;
    f32x16 o[NB][MD];
    float m[NB], l[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        m[n] = -INFINITY;
        l[n] = 0.f;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[n][md][v] = 0.f;
    }

    constexpr int NQK = 2 * KK;       // K fragments (steps) of S^T per tile; NB MFMAs each
    constexpr int NPV = 4 * MD;       // V fragments (steps) of O^T per tile; NB MFMAs each
    constexpr int SPQ = 32 * NB / NQK;   // softmax scores per S^T step
    constexpr int SPV = 32 * NB / NPV;   // scores per O^T step folded into the next row max
    static_assert(SPQ % 2 == 0 && SPV % 2 == 0, "scores go in pairs");
    typedef f32x16 Tile[NB][2];      // S^T of one tile: per query block, two 32-key blocks

    // (soff: byte offset of a ring stage, a multiple of TILEB, so adding it
    // commutes with the XORs on the low address bits)
    // K fragment of S^T step i (kk = i / 2, key block mb = i % 2)
    auto kread = [&](uint32_t kb, int i) -> bf16x8 {
        return *(const bf16x8 *)(smem + (i & 1) * 32 * ROWB + (kb ^ (32 * (i >> 1))));
    };
    // V^T fragment of O^T step i (ks4 = i / MD, md = i % MD) by two
    // transpose reads
    auto vread = [&](uint32_t v0, uint32_t v1, int i) -> bf16x8 {
        const int ks4 = i / MD, md = i % MD;
        const i16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_i16x4 *)(smem + ks4 * 16 * ROWB + (v0 ^ (64 * md))));
        const i16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_i16x4 *)(smem + ks4 * 16 * ROWB + (v1 ^ (64 * md))));
        // whole-vector reinterpretation: element-wise bf16 casts of the
        // transpose-read result were lowered to a splat
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // score e (0..32*NB-1) of a tile: query block n = e / 32, and within it
    // in P's B-operand order (fragment ks4 = e % 32 / 8 holds keys
    // 8 * (ks4 & 1) + e % 8 of key block ks4 / 2)
    auto score = [&](const Tile &sc, int e) -> float { return sc[e >> 5][(e >> 4) & 1][e & 15]; };
    // P weights of a tile: 2^(s * c2 - m), rounded to bf16 for P.V, and their
    // fp32 lane sums ls (so lse is exact to fp32 rounding).  One straight block:
    // all exponents, then all exps, then the packs and a pairwise sum, so
    // the dependent steps of different scores overlap.
    auto softmax_weights = [&](const Tile &sc, bf16x8 (&pf)[NB][4], const float (&m_use)[NB], float (&ls)[NB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            float x[32];
#pragma unroll
            for (int f = 0; f < 32; ++f) x[f] = __builtin_fmaf(score(sc, 32 * n + f), c2, -m_use[n]);
#pragma unroll
            for (int f = 0; f < 32; ++f) x[f] = fast_exp2(x[f]);
#pragma unroll
            for (int f = 0; f < 32; ++f) pf[n][f >> 3][f & 7] = (__bf16)x[f];
            // pairwise sum in a fixed order (the same for every tile)
#pragma unroll
            for (int w = 1; w < 32; w *= 2)
#pragma unroll
                for (int f = 0; f < 32; f += 2 * w) x[f] += x[f + w];
            ls[n] = x[0];
        }
    };
    // in-lane max of a tile's scores per query block; the other half-wave's
    // keys are folded in by update_max
    auto lane_max = [&](const Tile &sc, float (&mx)[NB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            mx[n] = -INFINITY;
#pragma unroll
            for (int e = 0; e < 32; ++e) mx[n] = fmaxf(mx[n], score(sc, 32 * n + e));
        }
    };
    // element masks only where the tile is not visible to every row
    auto mask = [&](int t, Tile &sc) {
        const int kt = t * KT;
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = kt + mb * 32 + (v >> 2) * 8 + 4 * hf + (v & 3);
                    if (key >= kend[n]) sc[n][mb][v] = -INFINITY;
                }
    };
    // Running max (log2 domain) from a tile's in-lane max, with lazy rescale:
    // m only moves when the tile max exceeds it by more than 2^RESCALE_LOG2,
    // so most tiles skip rescaling O and l (a wave-uniform branch).  Weights
    // stay <= 2^RESCALE_LOG2; O and l share the same m, so the quotient is
    // exact.
    auto update_max = [&](const float (&mx_lane)[NB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const float mx = halves_max(mx_lane[n]) * c2;
            const bool grow = mx > m[n] + RESCALE_LOG2;
            if (__builtin_amdgcn_ballot_w64(grow)) {
                // lanes that keep m scale by 1 (also while m is still -inf:
                // a row that sees no key of this tile); 0 from -inf
                const float m_new = grow ? mx : m[n];
                const float alpha = grow ? fast_exp2(m[n] - m_new) : 1.f;
                m[n] = m_new;
                l[n] *= alpha;
#pragma unroll
                for (int md = 0; md < MD; ++md)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[n][md][v] *= alpha;
            }
        }
    };
    auto max_shift = [&](float (&m_use)[NB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n) m_use[n] = (m[n] == -INFINITY) ? 0.f : m[n];
    };
    // S^T[key][query] = K Q^T for the 64 keys of a stage x this wave's
    // 32 * NB queries.  Each step is fenced so the reads stay RAHEAD steps
    // ahead of their MFMAs.
    auto qk = [&](uint32_t soff, Tile &sn) {
        const uint32_t kb = kbase + soff;
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) sn[n][mb][v] = 0.f;
        bf16x8 kf[RAHEAD + 1];
#pragma unroll
        for (int i = 0; i < RAHEAD; ++i) kf[i] = kread(kb, i);
#pragma unroll
        for (int i = 0; i < NQK; ++i) {
            if (i + RAHEAD < NQK) kf[(i + RAHEAD) % (RAHEAD + 1)] = kread(kb, i + RAHEAD);
#pragma unroll
            for (int n = 0; n < NB; ++n)
                sn[n][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % (RAHEAD + 1)], qf[n][i >> 1], sn[n][i & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // softmax of a tile: mask, running max, P weights and their sum
    auto softmax = [&](int t, Tile &sc, bf16x8 (&pf)[NB][4]) {
        if ((t + 1) * KT > kfull) {
            // (a real branch: the compiler would otherwise turn this rare
            // path into selects executed on every tile)
            asm volatile("" ::: "memory");
            mask(t, sc);
        }
        // Weights at the running max as it stands; the tile's max is only
        // taken when some row may need a larger one: a row that has seen no
        // key yet, or whose lane sum of weights exceeds 2^RESCALE_LOG2 (a
        // necessary condition for a score above m + RESCALE_LOG2; inf and
        // NaN land here too).  That path is the lazy-rescale update and the
        // weights again, so every weight stays <= 2^RESCALE_LOG2 either way.
        float m_use[NB], ls[NB];
        max_shift(m_use);
        softmax_weights(sc, pf, m_use, ls);
        bool slow = false;
#pragma unroll
        for (int n = 0; n < NB; ++n) slow = slow || m[n] == -INFINITY || !(ls[n] <= RESCALE_BOUND);
        if (__builtin_amdgcn_ballot_w64(slow)) {
            float mx[NB];
            lane_max(sc, mx);
            update_max(mx);
            max_shift(m_use);
            softmax_weights(sc, pf, m_use, ls);
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) l[n] += ls[n];
    };
    // O^T[d][query] += V^T P^T from the V tile of a stage; V reads RAHEAD
    // steps ahead of their MFMAs
    auto pv = [&](uint32_t soff, const bf16x8 (&pf)[NB][4]) {
        const uint32_t v0 = vbase[0] + soff, v1 = vbase[1] + soff;
        bf16x8 vf[RAHEAD + 1];
#pragma unroll
        for (int i = 0; i < RAHEAD; ++i) vf[i] = vread(v0, v1, i);
#pragma unroll
        for (int i = 0; i < NPV; ++i) {
            if (i + RAHEAD < NPV) vf[(i + RAHEAD) % (RAHEAD + 1)] = vread(v0, v1, i + RAHEAD);
#pragma unroll
            for (int n = 0; n < NB; ++n)
                o[n][i % MD] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i % (RAHEAD + 1)], pf[n][i / MD], o[n][i % MD], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- pipeline ---------------------------------------------------------
    // Tile t lives in ring stage (t - t_begin) % NSTAGE.  Every wave runs
    // the same loop: step j is an MFMA block (S^T of tile j, then O += P V
    // of tile j-1), a work-group barrier, the VALU block (softmax of tile j)
    // and another barrier.  The second wave on each SIMD (waves NWD..NW-1,
    // SIMD = wave % 4) enters the loop one barrier late, so on every SIMD one
    // wave's softmax overlaps the other wave's MFMAs.  The leading waves
    // issue the loads of tile j+3 at the start of step j and wait for tile
    // j+1 before its last barrier: a stage is refilled only after the
    // trailing waves' last read of its tile, and its loads have three steps
    // to land.
    static_assert(NW == 8, "two waves per SIMD");
    const bool lead = wave < NWD;
    // a wave whose 32 rows all lie past the last row (a small block's tile)
    // only takes part in the loads and barriers
    const bool busy = q0 + rblk * 32 < (int)nrows;
    Tile S;
    bf16x8 pf[NB][4];
    const int n_tiles = t_end - t_begin;
    auto stage_off = [&](int t) -> uint32_t { return (uint32_t)((t - t_begin) % NSTAGE) * TILEB; };
    if constexpr (KG == 2) {
        // (below)
    } else if (n_tiles > 0) {
        // Prologue: the leading waves issue the first three tiles and wait
        // for the first and their query rows (the other two stay in flight
        // into loop step t_begin, as in the steady state); the trailing
        // waves wait for their query rows.  The page-id reads are the only
        // loads the compiler sees here, so its own waits never cover the
        // tile loads.
        int pg_next = 0;   // page of tile j+3, read one step ahead
        if (lead) {
            const int pg0 = page_glb(t_begin), pg1 = page_glb(t_begin + 1), pg2 = page_glb(t_begin + 2);
            pg_next = page_glb(t_begin + 3);
            issue_tile(t_begin, 0, pg0);
            if (n_tiles > 1) issue_tile(t_begin + 1, 1, pg1);
            if (n_tiles > 2) issue_tile(t_begin + 2, 2, pg2);
            wait_tiles(min(2, n_tiles - 1));
        } else {
            wait_vm_lgkm<0>();
        }
        read_q();
        wait_vm_lgkm<63>();   // (LDS reads and writes complete; no vector-memory wait)
        wg_barrier();
        if (!lead) wg_barrier();
        for (int j = t_begin; j <= t_end; ++j) {
            // Addresses derived from these per-lane bases are cheap to
            // recompute; hidden from the optimiser here so that it does not
            // hoist them out of the loop and hold them in registers the
            // pipeline needs.
            asm volatile("" : "+v"(kbase), "+v"(vbase[0]), "+v"(vbase[1]), "+v"(lofs_p), "+v"(lofs_k), "+v"(lofs_v));
            if (busy) {
                // S^T of tile j first: its accumulators are complete long
                // before the softmax reads them after the barrier
                if (j < t_end) qk(stage_off(j), S);
                if (j > t_begin) pv(stage_off(j - 1), pf);
            }
            wg_barrier();
            // the leading waves issue the loads of tile j+3 here, ahead of
            // their softmax, rather than ahead of their MFMA block
            if (lead && j + 3 < t_end) issue_tile(j + 3, (j + 3 - t_begin) % NSTAGE, pg_next);
            if (busy && j < t_end) softmax(j, S, pf);
            // (read here, under the wait below: a scalar read left in flight
            // across the MFMA block would force full LDS drains there)
            if (lead && j + 4 < t_end) pg_next = page_glb(j + 4);
            // tile j+1 landed; tiles j+2 and j+3 may stay in flight
            if (lead && j + 1 < t_end) wait_tiles(min(2, t_end - 2 - j));
            wg_barrier();
        }
        if (lead) wg_barrier();
    } else {
        wait_vm_lgkm<0>();   // (the query loads)
    }

    // Two key groups.  Phase p (between two barriers) is the leading waves'
    // MFMA block of step p / 2 (p even) or the trailing waves' (p odd), while
    // the others run their softmax: K of tile t_begin + p is read in phase p
    // and V of it in phase p + 2.  In its softmax phase each half issues the
    // tile three past its own, into the stage whose V was read one phase
    // before, and waits for it after its next MFMA block, one phase before
    // it is read.
    if constexpr (KG == 2) {
        if (n_tiles > 0) {
            int pg_next = page_glb(t_begin + kg + 3);   // page of the tile issued next
            if (kg == 0) {
                const int pg0 = page_glb(t_begin), pg2 = page_glb(t_begin + 2);
                issue_tile(t_begin, 0, pg0);
                if (n_tiles > 2) issue_tile(t_begin + 2, 2, pg2);
                wait_tiles(n_tiles > 2 ? 1 : 0);
            } else {
                const int pg1 = page_glb(t_begin + 1);
                if (n_tiles > 1) issue_tile(t_begin + 1, 1, pg1);
                wait_vm_lgkm<0>();
            }
            read_q();
            wait_vm_lgkm<63>();
            wg_barrier();
            if (!lead) wg_barrier();
            const int nj = (n_tiles + 1) / 2;
            for (int j = 0; j <= nj; ++j) {
                asm volatile("" : "+v"(kbase), "+v"(vbase[0]), "+v"(vbase[1]), "+v"(lofs_p), "+v"(lofs_k), "+v"(lofs_v));
                const int t = t_begin + 2 * j + kg;
                if (busy) {
                    if (t < t_end) qk(stage_off(t), S);
                    if (j > 0 && t - 2 < t_end) pv(stage_off(t - 2), pf);
                }
                wait_vm_lgkm<0>();   // the tile issued in the last softmax phase landed
                wg_barrier();
                if (t + 3 < t_end) issue_tile(t + 3, (t + 3 - t_begin) % NSTAGE, pg_next);
                if (busy && t < t_end) softmax(t, S, pf);
                if (t + 5 < t_end) pg_next = page_glb(t + 5);
                wait_vm_lgkm<63>();
                wg_barrier();
            }
            if (lead) wg_barrier();
        } else {
            wait_vm_lgkm<0>();   // (the query loads)
            wg_barrier();
        }
        // The odd tiles' sums go to the leading wave of the same rows, in
        // register order; every tile and query read is behind the last barrier.
        char *xch = smem + VRING + rblk * (32 * D * 4 + 512);
        if (kg == 1) {
#pragma unroll
            for (int md = 0; md < MD; ++md)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 val;
#pragma unroll
                    for (int e = 0; e < 4; ++e) val[e] = o[0][md][4 * g + e];
                    *(f32x4 *)(xch + ((md * 4 + g) * 64 + lane) * 16) = val;
                }
            *(float *)(xch + 32 * D * 4 + 4 * lane) = m[0];
            *(float *)(xch + 32 * D * 4 + 256 + 4 * lane) = l[0];
        }
        wait_vm_lgkm<0>();
        wg_barrier();
        if (kg == 1) return;
        // rows that saw no key of a half have m = -inf there: weight 0
        const float m1 = *(const float *)(xch + 32 * D * 4 + 4 * lane), l1 = *(const float *)(xch + 32 * D * 4 + 256 + 4 * lane);
        const float mm = fmaxf(m[0], m1);
        const float a0 = m[0] == -INFINITY ? 0.f : fast_exp2(m[0] - mm), a1 = m1 == -INFINITY ? 0.f : fast_exp2(m1 - mm);
        m[0] = mm;
        l[0] = l[0] * a0 + l1 * a1;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 val = *(const f32x4 *)(xch + ((md * 4 + g) * 64 + lane) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[0][md][4 * g + e] = o[0][md][4 * g + e] * a0 + val[e] * a1;
            }
    }

    // ---- epilogue -----------------------------------------------------------
    // (the plan's fields are read again here rather than held over the loop)
    int nsplit = 1, slot = 0, napp = 1;
    if constexpr (RAGGED) {
        asm volatile("" : "+s"(ppos));
        nsplit = rp.pos[ppos].ns;
        slot = rp.pos[ppos].slot + (int)split;
        napp = rp.pos[ppos].items;
    } else if constexpr (step) {
        nsplit = a.nsplit;
        slot = b * nsplit + (int)split;
        napp = a.nqt * nsplit;
    }
    // Output rows of an unsplit item leave through LDS, so that a store covers
    // 16-byte pieces of 4 (D = 64: 8) whole rows rather than of 32: a wave's
    // own query stage holds its 32 rows (f32: half of the head dims at a
    // time), and after the loop's last barrier nothing else touches it.
    // 3.3k tokens, GQA 40/8 x 128: 136 -> 131 us; GQA 64/8, 2 x 1.4k: 118 ->
    // 112 us; unchanged where an item runs many tiles.
    // A step of at most 64 packed rows stores them from the registers instead:
    // one or two waves hold them, and the exchange is latency at the end of the
    // launch (32 streams of 24 rows over 1000 keys: 30.1 us through LDS, 29.3
    // direct; f32 30.3 and 29.4; 64 rows 10.4 and 9.8, 128 rows 10.8 and 12.0).
    const bool whole = KIND != STEP_SPLIT && (!step || nsplit == 1);   // this item's rows are final
    const bool direct = KIND == STEP && a.nrows <= 64;
    if (whole && busy && !direct) {
        // (the lane is hidden from the optimiser, so that nothing derived from
        // it here is computed ahead of the loop and held in registers there)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        char *stage = smem + q_stage;
        const int er = ln & 31, eh = ln >> 5, c = ln % LPR;
        const float lt = halves_sum(l[0]);
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        // the stage's rows to out + ofs bytes, 16 bytes per lane
        // (written and read by this wave only; the compiler orders them)
        auto store_rows = [&](auto elem, int64_t ofs) {
            using E = decltype(elem);
#pragma unroll
            for (int i = 0; i < 32 / RPW; ++i) {
                const int rr = i * RPW + ln / LPR;
                const int p = q0 + rblk * 32 + rr;
                const u32x4 val = *(const u32x4 *)(stage + rr * ROWB + 16 * (c ^ swz<D>(rr)));
                if (p < (int)nrows) {
                    const int t = row_token(p), h = row_head(p, t);
                    *(u32x4 *)((char *)((E *)a.out + b * a.o_sb + (int64_t)t * a.o_st + h * a.o_sh) + ofs + 16 * c) = val;
                }
            }
        };
        if constexpr (F32) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int m2 = 0; m2 < MD / 2; ++m2)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        f32x4 val;
#pragma unroll
                        for (int e = 0; e < 4; ++e) val[e] = o[0][half * (MD / 2) + m2][4 * g + e] * inv;
                        *(f32x4 *)(stage + er * ROWB + 16 * ((8 * m2 + 2 * g + eh) ^ swz<D>(er))) = val;
                    }
                store_rows(0.f, half * ROWB);
            }
        } else {
#pragma unroll
            for (int md = 0; md < MD; ++md)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    u32x2 val;
                    val[0] = pack_bf16x2(o[0][md][4 * g + 0] * inv, o[0][md][4 * g + 1] * inv);
                    val[1] = pack_bf16x2(o[0][md][4 * g + 2] * inv, o[0][md][4 * g + 3] * inv);
                    *(u32x2 *)(stage + er * ROWB + 16 * ((4 * md + g) ^ swz<D>(er)) + 8 * eh) = val;
                }
            store_rows((uint16_t)0, 0);
        }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const float lt = halves_sum(l[n]);
        const int r = row[n];
        if (r >= (int)nrows) continue;
        const int t = tok[n], h = hqr[n];
        if (whole) {
            if (direct) {
                const float inv = lt > 0.f ? 1.f / lt : 0.f;
                const int64_t ofs = b * a.o_sb + (int64_t)t * a.o_st + h * a.o_sh + 4 * hf;
#pragma unroll
                for (int md = 0; md < MD; ++md)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        if constexpr (F32) {
                            f32x4 val;
#pragma unroll
                            for (int e = 0; e < 4; ++e) val[e] = o[n][md][4 * g + e] * inv;
                            *(f32x4 *)((float *)a.out + ofs + 32 * md + 8 * g) = val;
                        } else {
                            u32x2 val;
                            val[0] = pack_bf16x2(o[n][md][4 * g + 0] * inv, o[n][md][4 * g + 1] * inv);
                            val[1] = pack_bf16x2(o[n][md][4 * g + 2] * inv, o[n][md][4 * g + 3] * inv);
                            *(u32x2 *)((uint16_t *)a.out + ofs + 32 * md + 8 * g) = val;
                        }
                    }
            }
            if (a.lse && hf == 0)
                a.lse[((int64_t)b * a.Hq + h) * a.Lq + t] = (m[n] + __builtin_amdgcn_logf(lt)) * 0.69314718055994531f;
        } else if constexpr (!F32) {
            // bf16 output: o / l rounded to bf16 and the split's log2-domain
            // lse; register order, two accumulator groups (16 bytes) per
            // lane, so each store instruction writes 1 KB contiguous.
            // Partials are stored non-temporally (read once, by the combine
            // launch)
            const int64_t blk = ((int64_t)slot * a.Hkv + kvh) * a.nrb + (r >> 5);
            const float inv = lt > 0.f ? 1.f / lt : 0.f;
            uint16_t *op = (uint16_t *)a.part_o + blk * (32 * D) + 8 * lane;
#pragma unroll
            for (int pg = 0; pg < 2 * MD; ++pg) {
                const int md = pg >> 1, g0 = 2 * (pg & 1);
                u32x4 val;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    val[2 * h + 0] = pack_bf16x2(o[n][md][4 * (g0 + h) + 0] * inv, o[n][md][4 * (g0 + h) + 1] * inv);
                    val[2 * h + 1] = pack_bf16x2(o[n][md][4 * (g0 + h) + 2] * inv, o[n][md][4 * (g0 + h) + 3] * inv);
                }
                __builtin_nontemporal_store(val, (u32x4 *)(op + pg * 512));
            }
            if (hf == 0) __builtin_nontemporal_store(lt > 0.f ? m[n] + __builtin_amdgcn_logf(lt) : -INFINITY, a.part_ml + blk * 32 + l32);
        } else {
            // register order: each store instruction writes 1 KB contiguous
            const int64_t blk = ((int64_t)slot * a.Hkv + kvh) * a.nrb + (r >> 5);
            float *op = a.part_o + blk * (32 * D) + 4 * lane;
#pragma unroll
            for (int md = 0; md < MD; ++md)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 val;
#pragma unroll
                    for (int e = 0; e < 4; ++e) val[e] = o[n][md][4 * g + e];
                    __builtin_nontemporal_store(val, (f32x4 *)(op + (md * 4 + g) * 256));
                }
            if (hf == 0) {
                __builtin_nontemporal_store(m[n], a.part_ml + 2 * (blk * 32 + l32) + 0);
                __builtin_nontemporal_store(lt, a.part_ml + 2 * (blk * 32 + l32) + 1);
            }
        }
    }

    // ---- fused append -----------------------------------------------------
    // Step items cover every query head of their KV group (packed rows),
    // so the items of a (stream, KV head) group split the new tokens evenly
    // among them; padding tokens (t >= nl) are not committed.
    // This kernel reads the new block from kc/vc, never from the slots being
    // written, so the append can trail the attention; it comes after the
    // epilogue's stores so that its loads overlap their drain.
    if (step && a.fuse_append && hh == 0)
        append_share<D, NT>(a, b, kvh, (int)(qi * nsplit + split), napp, n_pool, nl, ptab, tid);
}

// The merge is bound by latency: one round trip of loads behind the work
// item's decode, on work-groups that hardly fill the chip (256-token block, 24
// heads, 10 splits: 19 MB in 6 us).  A work-group is therefore a part of one
// 32-row block, so that the decode is a few scalar multiplications by the
// host's dividers; 64-bit divisions per thread stood before the first load
// (6.3 -> 5.8 us with the 16-byte stores and the 12-split loop; the step 26.0
// -> 25.5 us, solver loop of 8 steps 211.0 -> 208.0 us).
// Threads of a work-group (NT), bf16: 128 while such work-groups are one per
// compute unit, which spreads the loads over twice the units (21 splits of 64
// blocks, head dim 128: 5.0 us against 5.4; 32 of 128, head dim 64: 5.7 against
// 6.4); past that a unit's second work-group runs after its first, and 256 are
// faster (21 splits of 76 blocks, head dim 128: 7.1 against 5.6 us, 16 of 128:
// 6.0 against 5.3; 18 of 160, head dim 64: 6.8 against 5.7).  Blocks of streams
// with one split do not count (24 of 72 merged, up to 29 splits: 5.4 against
// 6.1).  f32: 256 (128 measured 5 to 20 % slower from 76 blocks on, a few tenths
// of a us faster below).

// bf16 output: split s holds o_s / l_s (bf16) and lse_s = m_s + log2(l_s);
//   M = max_s lse_s,  L = sum_s 2^(lse_s - M),  o = sum_s 2^(lse_s - M) o_s / L.
// A thread owns the 8 elements (two accumulator groups) one writer lane
// stored with one 16-byte store, for every split.
// VARLEN: blocks of different lengths; padding rows are skipped (their
// partials may not exist).  SMAX >= nsplit: the split loops are unrolled
// SMAX times (the launch takes the smallest of 4, 8, 12, 16, 32).
// RAGGED: the streams have their own split counts and slots (rp); a stream
// with one split was written by the attention launch.
template <int D, bool VARLEN, bool RAGGED, int SMAX, int NT>
__global__ __launch_bounds__(NT) void combine16_kernel(const AttnArgs a, const Plan<RAGGED> rp) {
    static_assert(SMAX <= MAX_SPLITS, "at most MAX_SPLITS partials");
    constexpr int MD = D / 32;
    constexpr int PER_BLK = 2 * MD * 64;      // 16-byte items per 32-row block
    static_assert(PER_BLK % NT == 0, "a work-group stays within one block");
    const uint32_t blk = blockIdx.x / (PER_BLK / NT);
    const int item = (int)(blockIdx.x % (PER_BLK / NT) * NT + threadIdx.x);
    const int lane = item & 63;
    const int pg = item >> 6;                 // md * 2 + g0 / 2
    const uint32_t grp = fastdiv(blk, a.fd_nrb);
    const int r = (int)(blk - grp * (uint32_t)a.nrb) * 32 + (lane & 31);   // packed row
    if (r >= a.nrows) return;
    const int b = (int)fastdiv(grp, a.fd_hkv);
    const int kvh = (int)(grp - (uint32_t)b * (uint32_t)a.Hkv);
    const int t = (int)fastdiv((uint32_t)r, a.fd_gq);
    if (VARLEN && t >= a.new_lens[b]) return;   // padding row: left unwritten
    const int hq = kvh * a.G + (r - t * a.G);
    int S = a.nsplit, slot = b * S;
    if constexpr (RAGGED) {
        S = rp.ns[b];
        slot = rp.slot[b];
        if (S == 1) return;
    }
    const int64_t sb = (int64_t)a.Hkv * a.nrb;   // blocks per slot
    const int64_t pb = slot * sb + (int64_t)(blk - (uint32_t)b * (uint32_t)sb);
    const float *pl = a.part_ml + pb * 32 + (lane & 31);
    const uint16_t *po = (const uint16_t *)a.part_o + pb * (32 * D) + pg * 512 + 8 * lane;
    const int64_t ls = sb * 32;               // split stride of lse
    const int64_t ps = sb * 32 * D;           // split stride of o
    // all loads first (one round trip), then the arithmetic
    float lse[SMAX];
    u32x4 ov[SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        if (s < S) {
            lse[s] = pl[s * ls];
            ov[s] = *(const u32x4 *)(po + s * ps);
        } else {
            lse[s] = -INFINITY;
            ov[s] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    float M = -INFINITY;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) M = fmaxf(M, lse[s]);
    const float Mu = (M == -INFINITY) ? 0.f : M;
    float L = 0.f;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        const float wgt = __builtin_amdgcn_exp2f(lse[s] - Mu);   // 0 for absent splits
        L += wgt;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[2 * k + 0] += __uint_as_float(ov[s][k] << 16) * wgt;
            acc[2 * k + 1] += __uint_as_float(ov[s][k] & 0xFFFF0000u) * wgt;
        }
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    // the halves of the wave hold 4 elements each of two 8-element groups of
    // a row; after the swap each holds one group whole: one 16-byte store
    u32x4 val;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32x2 x = __builtin_amdgcn_permlane32_swap(pack_bf16x2(acc[2 * h] * inv, acc[2 * h + 1] * inv),
                                                         pack_bf16x2(acc[4 + 2 * h] * inv, acc[5 + 2 * h] * inv), false, false);
        val[h] = x[0];
        val[2 + h] = x[1];
    }
    *(u32x4 *)((uint16_t *)a.out + b * a.o_sb + (int64_t)t * a.o_st + hq * a.o_sh + 16 * pg + 8 * (lane >> 5)) = val;
    if (a.lse && pg == 0 && lane < 32)
        a.lse[((int64_t)b * a.Hq + hq) * a.Lq + t] = (M + __builtin_amdgcn_logf(L)) * 0.69314718055994531f;
}

// Merge the KV-split partials of every query row: with per-split running
// max m_s (log2 domain), sum l_s and unnormalised o_s,
//   M = max_s m_s,  L = sum_s l_s 2^(m_s - M),  o = sum_s o_s 2^(m_s - M) / L.
// Splits are visited in a fixed order, so the result is deterministic.  A
// thread owns the 4 elements one accumulator lane holds for one (md, g), so
// its partial reads are the writer's contiguous 1 KB runs; the split loops
// are unrolled (as in combine16_kernel), so that all loads are in flight
// together: 20 splits of 240 blocks, head dim 64: 11.3 us as a rolled loop
// over the splits.
template <int D, bool VARLEN, bool RAGGED, int SMAX, int NT>
__global__ __launch_bounds__(NT) void combine_kernel(const AttnArgs a, const Plan<RAGGED> rp) {
    constexpr int MD = D / 32;
    constexpr int PER_BLK = MD * 4 * 64;      // float4 items per 32-row block
    static_assert(PER_BLK % NT == 0, "a work-group stays within one block");
    const uint32_t blk = blockIdx.x / (PER_BLK / NT);
    const int item = (int)(blockIdx.x % (PER_BLK / NT) * NT + threadIdx.x);
    const int lane = item & 63;
    const int mg = item >> 6;                 // md * 4 + g
    const uint32_t grp = fastdiv(blk, a.fd_nrb);
    const int r = (int)(blk - grp * (uint32_t)a.nrb) * 32 + (lane & 31);   // packed row
    if (r >= a.nrows) return;
    const int b = (int)fastdiv(grp, a.fd_hkv);
    const int kvh = (int)(grp - (uint32_t)b * (uint32_t)a.Hkv);
    const int t = (int)fastdiv((uint32_t)r, a.fd_gq);
    if (VARLEN && t >= a.new_lens[b]) return;   // padding row: left unwritten
    const int hq = kvh * a.G + (r - t * a.G);
    const int d0 = 32 * (mg >> 2) + 8 * (mg & 3) + 4 * (lane >> 5);
    int S = a.nsplit, slot = b * S;
    if constexpr (RAGGED) {
        S = rp.ns[b];
        slot = rp.slot[b];
        if (S == 1) return;
    }
    const int64_t sb = (int64_t)a.Hkv * a.nrb;   // blocks per slot
    const int64_t pb = slot * sb + (int64_t)(blk - (uint32_t)b * (uint32_t)sb);
    const float2 *ml = (const float2 *)a.part_ml + pb * 32 + (lane & 31);
    const float *po = a.part_o + pb * (32 * D) + (int64_t)mg * 256 + 4 * lane;
    const int64_t mls = sb * 32;              // split stride of (m, l)
    const int64_t ps = sb * 32 * D;           // split stride of o
    // all loads first (one round trip), then the arithmetic
    float2 m_l[SMAX];
    f32x4 ov[SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        if (s < S) {
            m_l[s] = ml[s * mls];
            ov[s] = *(const f32x4 *)(po + s * ps);
        } else {
            m_l[s] = float2{-INFINITY, 0.f};
            ov[s] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    float M = -INFINITY;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) M = fmaxf(M, m_l[s].x);
    const float Mu = (M == -INFINITY) ? 0.f : M;
    float L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        const float wgt = __builtin_amdgcn_exp2f(m_l[s].x - Mu);   // 0 for absent splits
        L += m_l[s].y * wgt;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += ov[s][e] * wgt;
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    float *op = (float *)a.out + b * a.o_sb + (int64_t)t * a.o_st + hq * a.o_sh + d0;
    f32x4 val;
#pragma unroll
    for (int e = 0; e < 4; ++e) val[e] = acc[e] * inv;
    *(f32x4 *)op = val;
    if (a.lse && mg == 0 && lane < 32)
        a.lse[((int64_t)b * a.Hq + hq) * a.Lq + t] = (M + __builtin_amdgcn_logf(L)) * 0.69314718055994531f;
}

// Copy new tokens' K/V rows into their cache slots: one 16-byte chunk per
// thread; consecutive threads walk one token row, so reads and writes are
// contiguous 256-byte runs (head_dim 128).
__global__ __launch_bounds__(256) void append_kernel(const AppendArgs a) {
    const int CH = a.D / 8;
    const int b = blockIdx.y;
    const int64_t total = (int64_t)(a.new_lens ? a.new_lens[b] : a.Ln) * a.Hkv * CH;
    for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < total; u += (int64_t)gridDim.x * 256) {
        const int c = (int)(u % CH);
        const int h = (int)((u / CH) % a.Hkv);
        const int t = (int)(u / ((int64_t)CH * a.Hkv));
        const int pos = a.cache_lens[b] + t;
        const int page = a.page_table[(int64_t)b * a.max_pages + (pos >> 6)];
        const int64_t dst = (((int64_t)page * a.Hkv + h) * KT + (pos & 63)) * a.D + 8 * c;
        *(u32x4 *)(a.kpool + dst) = *(const u32x4 *)(a.kn + b * a.kn_sb + (int64_t)t * a.kn_st + h * a.kn_sh + 8 * c);
        *(u32x4 *)(a.vpool + dst) = *(const u32x4 *)(a.vn + b * a.vn_sb + (int64_t)t * a.vn_st + h * a.vn_sh + 8 * c);
    }
}

template <int D, int KIND, int KG>
int launch_attn_t(const AttnArgs &a, const Plan<KIND == STEP_RAGGED> &rp, hipStream_t st) {
    const dim3 grid(a.per_xcd * NUM_XCD), block(8 * 64);
    if (a.out_f32)
        hipLaunchKernelGGL((attn_kernel<D, 8, 1, KIND, true, KG>), grid, block, 0, st, a, rp);
    else
        hipLaunchKernelGGL((attn_kernel<D, 8, 1, KIND, false, KG>), grid, block, 0, st, a, rp);
    return (int)hipGetLastError();
}

template <int D, int KIND>
int launch_prefill_t(const AttnArgs &a, int key_groups, hipStream_t st) {
    return key_groups == 2 ? launch_attn_t<D, KIND, 2>(a, NoPlan{}, st) : launch_attn_t<D, KIND, 1>(a, NoPlan{}, st);
}

template <int D>
int launch_attn_d(const AttnArgs &a, const RaggedPlan *rag, TileShape shape, hipStream_t st) {
    return rag ? launch_attn_t<D, STEP_RAGGED, 1>(a, *rag, st)
         : a.mode == MODE_STEP ? shape.parts_only ? launch_attn_t<D, STEP_SPLIT, 1>(a, NoPlan{}, st)
                                                  : launch_attn_t<D, STEP, 1>(a, NoPlan{}, st)
         : a.paged ? launch_prefill_t<D, PREFILL_PAGED>(a, shape.kg, st)
                   : launch_prefill_t<D, PREFILL_CONTIGUOUS>(a, shape.kg, st);
}

template <int D, bool VL, bool RAGGED>
int launch_combine_t(const AttnArgs &a, const Plan<RAGGED> &rp, int nsplit, hipStream_t st) {
    const int per_blk = D / 32 * (a.out_f32 ? 4 : 2) * 64;   // items per 32-row block
    const int64_t blocks = (int64_t)a.B * a.Hkv * a.nrb;
    int cus = 0;
    if (int e = current_device_cus(&cus)) return e;
    int64_t merged = blocks;   // those that are not of a stream with one split
    if constexpr (RAGGED) merged = std::count_if(rp.ns, rp.ns + a.B, [](int32_t n) { return n > 1; }) * (int64_t)a.Hkv * a.nrb;
    const int nt = !a.out_f32 && merged * (per_blk / 128) <= cus ? 128 : 256;
    const dim3 grid((unsigned)(blocks * (per_blk / nt)));
    auto launch = [&](auto smax) {
        constexpr int SMAX = decltype(smax)::value;
        if (a.out_f32)
            hipLaunchKernelGGL((combine_kernel<D, VL, RAGGED, SMAX, 256>), grid, dim3(256), 0, st, a, rp);
        else if (nt == 128)
            hipLaunchKernelGGL((combine16_kernel<D, VL, RAGGED, SMAX, 128>), grid, dim3(128), 0, st, a, rp);
        else
            hipLaunchKernelGGL((combine16_kernel<D, VL, RAGGED, SMAX, 256>), grid, dim3(256), 0, st, a, rp);
    };
    if (nsplit <= 4) launch(std::integral_constant<int, 4>{});
    else if (nsplit <= 8) launch(std::integral_constant<int, 8>{});
    else if (nsplit <= 12) launch(std::integral_constant<int, 12>{});
    else if (nsplit <= 16) launch(std::integral_constant<int, 16>{});
    else launch(std::integral_constant<int, MAX_SPLITS>{});
    return (int)hipGetLastError();
}

template <int D>
int launch_combine_d(const AttnArgs &a, const RaggedPlan *rag, hipStream_t st) {
    if (rag)
        return a.has_new_lens ? launch_combine_t<D, true, true>(a, *rag, rag->max_nsplit, st)
                              : launch_combine_t<D, false, true>(a, *rag, rag->max_nsplit, st);
    return a.has_new_lens ? launch_combine_t<D, true, false>(a, NoPlan{}, a.nsplit, st)
                          : launch_combine_t<D, false, false>(a, NoPlan{}, a.nsplit, st);
}

}  // namespace

int launch_attention(const AttnArgs &a, const RaggedPlan *rag, int head_dim, TileShape shape, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (shape.nw != 8 || shape.nb != 1) return (int)hipErrorInvalidValue;
    if (head_dim == 128) return launch_attn_d<128>(a, rag, shape, st);
    if (head_dim == 64) return launch_attn_d<64>(a, rag, shape, st);
    return (int)hipErrorInvalidValue;
}

int launch_combine(const AttnArgs &a, const RaggedPlan *rag, int head_dim, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (head_dim == 128) return launch_combine_d<128>(a, rag, st);
    if (head_dim == 64) return launch_combine_d<64>(a, rag, st);
    return (int)hipErrorInvalidValue;
}

int launch_append(const AppendArgs &a, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    const int64_t total = (int64_t)a.Ln * a.Hkv * (a.D / 8);
    int64_t gx = (total + 255) / 256;
    if (gx > 4096) gx = 4096;
    if (gx < 1) gx = 1;
    hipLaunchKernelGGL(append_kernel, dim3((unsigned)gx, (unsigned)a.B), dim3(256), 0, st, a);
    return (int)hipGetLastError();
}


}  // namespace ws
