// gfx950 (MI355X) kernels for the gradients of whole-sequence block-causal
// attention (training uses the same causal format as generation,
// Wan-Streamer v0.1, Sec. 2.3): a query-major dQ kernel, which also leaves
// each row's D and key end for the key-major dK/dV kernel after it; both
// deterministic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ws_kernels.h"
#include "ws_device_util.h"

namespace ws {
namespace {

constexpr int KB_DKDV = 16;   // key tiles of one group taken together on an XCD (dK/dV)
constexpr int AH = 2;         // LDS operand reads issued this many MFMAs ahead

// ---------------------------------------------------------------------------
// Gradients of the whole-sequence path (training shares the causal format,
// Sec. 2.3).  With the forward's lse, P_ij = exp(s_ij - lse_i) needs no
// running max:
//   D_i = <dO_i, O_i>,  dS_ij = P_ij (<dO_i, v_j> - D_i),
//   dQ_i = scale sum_j dS_ij k_j,  dK_j = scale sum_i dS_ij q_i,
//   dV_j = sum_i P_ij dO_i.
// Two kernels: a query-major one for dQ (like the forward, with dS^T in place
// of P^T), which forms D_i from the rows of dO it holds anyway and stores it
// (a pass of its own over O and dO took 10 us at 2.4k tokens, 119 us at
// 2 x 16384), then a key-major one for dK and dV
// (S = Q K^T with the keys as columns, so P and dS are B operands of
// dV^T += dO^T P and dK^T += Q^T dS).  Each sums in a fixed order: the
// gradients are deterministic, and dK/dV sum the G query heads of their KV
// head inside one work-group.

// byte offset of 16-byte chunk c of row r in an LDS tile of [rows][D] bf16
// (the forward's swizzle)
template <int D>
__device__ __forceinline__ uint32_t tile_off(int r, int c) {
    return (uint32_t)(r * 2 * D + 16 * (c ^ swz<D>(r)));
}

// A fragment of (tile rows 16 ks .. 16 ks + 15)^T for head-dim block md, by
// two transpose reads; tb[] are the lane's bases (as the forward's V^T reads)
template <int D>
__device__ __forceinline__ bf16x8 tr_frag(const char *tile, const uint32_t (&tb)[2], int ks, int md) {
    const i16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4 *)(tile + ks * 16 * 2 * D + (tb[0] ^ (64 * md))));
    const i16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4 *)(tile + ks * 16 * 2 * D + (tb[1] ^ (64 * md))));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int D>
__device__ __forceinline__ void tr_bases(int lane, uint32_t (&tb)[2]) {
    const int j16 = lane & 15, hf = lane >> 5;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int vr = 4 * hf + (j16 >> 2) + 8 * e;
        const int vc = 2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1);
        tb[e] = (uint32_t)(vr * 2 * D + 16 * (vc ^ swz<D>(vr)) + 8 * (j16 & 1));
    }
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Loads rows [r0, r0 + nrows) of a [rows][D] bf16 tile (row r of the tile
// = global row min(r0 + r, rmax), at least 0) straight into LDS at `lds` in the
// swizzled layout, spread over NWV waves: wave-wide load i of wave w fills
// tile bytes [(i * NWV + w) * 1024, +1024), lane l the 16 bytes at +16 l,
// so it fetches the chunk that belongs there.  The caller waits for them
// (s_waitcnt vmcnt) before the barrier that publishes the tile.
template <int D, int NWV, int ROWS>
__device__ __forceinline__ void dma_rows(const char *g, int64_t st_bytes, int r0, int rmax, uint32_t lds,
                                         int wave, int lane) {
    constexpr int ROWB = 2 * D, RPW = 1024 / ROWB, LPR = ROWB / 16;
    constexpr int NI = ROWS * ROWB / (NWV * 1024);
    static_assert(NI >= 1 && ROWS * ROWB % (NWV * 1024) == 0, "the tile splits into wave-wide loads");
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int r = (i * NWV + wave) * RPW + lane / LPR;
        const int ch = (lane % LPR) ^ swz<D>(r);
        const int gr = max(min(r0 + r, rmax), 0);
        dma16(g + (int64_t)gr * st_bytes + 16 * ch, lds + (i * NWV + wave) * 1024);
    }
}

// dQ: one work-group = (stream, query head, 128 query rows), 4 waves x 32
// rows; K/V tiles of 64 keys go straight to LDS (two stages); tiles past
// the last row's key end are never loaded.  Registers are held to two waves
// per SIMD, so two independent work-groups share a CU.  As in the dK/dV
// kernel, every vector instruction and load stands beside an MFMA that does
// not need it (the second half's S beside the first half's dS), and element
// masks run only on the tiles that straddle some row's key end: 2 x 16384
// tokens, GQA 32/8 x 128: 6.1 -> 5.4 ms, bitwise the same dQ.  Two MFMAs of
// read-ahead and three measured the same.
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dq_kernel(const BwdArgs a) {
    constexpr int ROWB = 2 * D, KK = D / 16, MD = D / 32;
    constexpr int TILEB = 64 * ROWB;
    __shared__ __attribute__((aligned(1024))) char smem[2 * 2 * TILEB];   // [stage][K, V]
    const int nqt = (a.L + 127) / 128;
    const int wid = blockIdx.x;
    // query tiles heaviest first over all (stream, head) pairs, so the
    // dispatch order is longest-first across the whole launch and the last
    // round of work-groups holds the shortest tiles; within a tile level the
    // (stream, KV head) group is the fast digit, so with work-group i on XCD
    // i mod 8 the G query heads of a group share an XCD (and its L2) for
    // the whole launch
    const int qt = nqt - 1 - wid / (a.B * a.Hq);
    const int kq = wid % (a.B * a.Hq);
    const int grp = kq % (a.B * a.Hkv), hhq = kq / (a.B * a.Hkv);
    const int b = grp / a.Hkv;
    const int h = (grp % a.Hkv) * a.G + hhq;
    const int g = h / a.G;
    const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q0 = qt * 128;
    const int row = q0 + 32 * wave + l32;
    const int rc = min(row, a.L - 1);
    const int32_t *offs = a.offsets + (int64_t)b * (a.nb + 1);
    const int32_t *text = a.text_starts ? a.text_starts + (int64_t)b * a.nb : nullptr;
    const BlockWindow win = block_window(offs, text, a.nb, q0, lane);
    const int k_hi = token_key_end(win, min(q0 + 127, a.L - 1), lane);
    const int kfull = token_key_end(win, q0, lane);
    const int my_kend = lane_key_end(win, min(q0 + 32 * wave, a.L - 1), rc, lane);
    const float lse2 = a.lse[((int64_t)b * a.Hq + h) * a.L + rc] * 1.4426950408889634f;
    const float c2 = a.scale_log2;

    // B fragments of the lane's query row: q and dO, head dims 16 kk + 8 hf +
    // [0, 8), and -D = -<dO, O> from the row's output
    bf16x8 qf[KK], dof[KK];
    float nD;
    {
        const uint16_t *qp = a.q + b * a.q_sb + (int64_t)rc * a.q_st + h * a.q_sh + 8 * hf;
        const uint16_t *dp = a.dout + b * a.do_sb + (int64_t)rc * a.do_st + h * a.do_sh + 8 * hf;
        const uint16_t *op = a.o + b * a.o_sb + (int64_t)rc * a.o_st + h * a.o_sh + 8 * hf;
        u32x4 ov[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            ov[kk] = *(const u32x4 *)(op + 16 * kk);
            dof[kk] = *(const bf16x8 *)(dp + 16 * kk);
            qf[kk] = *(const bf16x8 *)(qp + 16 * kk);
        }
        float part[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const u32x4 dv = __builtin_bit_cast(u32x4, dof[kk]);
            part[kk] = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                part[kk] += bf16_lo(ov[kk][k]) * bf16_lo(dv[k]) + bf16_hi(ov[kk][k]) * bf16_hi(dv[k]);
        }
#pragma unroll
        for (int w = 1; w < KK; w *= 2)
#pragma unroll
            for (int kk = 0; kk < KK; kk += 2 * w) part[kk] += part[kk + w];
        nD = -halves_sum(part[0]);
    }
    // the row data of the dK/dV launch: lse2 and -D of this head's row and,
    // once per token, its key end
    if (row < a.L && hf == 0) {
        float *dl = a.dl + 2 * ((int64_t)b * a.Hq + h) * a.L + row;
        dl[0] = lse2;
        dl[a.L] = nD;
        if (h == 0) a.kend[(int64_t)b * a.L + row] = my_kend;
    }
    const char *kg = (const char *)(a.k + b * a.k_sb + g * a.k_sh);
    const char *vg = (const char *)(a.v + b * a.v_sb + g * a.v_sh);
    const int64_t kst = 2 * a.k_st, vst = 2 * a.v_st;
    // K and V rows of tile t + 1 go straight to LDS while tile t is used: part
    // i (0 .. 2 NI - 1) is one wave-wide load from a wave-uniform base and a
    // per-lane 32-bit offset (the swizzle repeats every 16 rows), issued
    // between MFMAs.  The tile holding the last key, or rows too far apart for
    // 32-bit offsets, is loaded whole in part 0 with per-lane addresses.
    constexpr int RPW = 1024 / ROWB, LPR = ROWB / 16, NI = TILEB / 4096;
    static_assert(4 * RPW % 16 == 0, "the swizzle must repeat across a wave's loads");
    const int lrow = RPW * wave + lane / LPR;
    const uint32_t lch = (uint32_t)(16 * ((lane % LPR) ^ swz<D>(lrow)));
    const uint32_t kofs = (uint32_t)lrow * (uint32_t)kst + lch, vofs = (uint32_t)lrow * (uint32_t)vst + lch;
    const bool wide = a.wide_strides != 0;
    auto issue_part = [&](int t, int i) {
        const uint32_t kl = lds_addr(smem) + (t & 1) * 2 * TILEB;
        if ((t + 1) * 64 > k_hi || wide) {
            if (i || t * 64 >= k_hi) return;
            // (the lane is hidden from the optimiser, so that what this rare
            // path derives from it is not hoisted and held in registers)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            dma_rows<D, 4, 64>(kg, kst, t * 64, k_hi - 1, kl, wave, ln);
            dma_rows<D, 4, 64>(vg, vst, t * 64, k_hi - 1, kl + TILEB, wave, ln);
        } else if (i < NI) {
            dma16s(kg + (t * 64 + i * 4 * RPW) * kst, kofs, kl + i * 4096 + wave * 1024);
        } else {
            dma16s(vg + (t * 64 + (i - NI) * 4 * RPW) * vst, vofs, kl + TILEB + (i - NI) * 4096 + wave * 1024);
        }
    };
    uint32_t kbase = (uint32_t)(l32 * ROWB + 16 * (hf ^ swz<D>(l32)));
    uint32_t tb[2];
    tr_bases<D>(lane, tb);

    f32x16 acc[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[md][v] = 0.f;
    const int ntile = (k_hi + 63) / 64;
#pragma unroll
    for (int i = 0; i < 2 * NI; ++i) issue_part(0, i);
    wait_vm_lgkm<0>();
    wg_barrier();
    for (int t = 0; t < ntile; ++t) {
        const char *kt = smem + (t & 1) * 2 * TILEB, *vt = kt + TILEB;
        // One MFMA stream over the tile's two halves of 32 keys, every vector
        // instruction beside a matrix instruction that does not need it:
        // S0; dP0 beside P0 = exp2(S0 c2 - lse2); S1 beside dS0 = P0 (dP0 -
        // D); dP1 beside P1; dQ += K^T dS (half 0) beside dS1; dQ (half 1).
        // Operands are read AH steps ahead; the fences keep this order.
        f32x16 S[2], dPt[2];
        bf16x8 dsf[2][2], fr[AH + 1];
        // A operand of step i: K of a half (S^T), V of a half (dP^T), K^T
        auto rd = [&](int i) {
            const int h = i / (2 * KK), j = i % (2 * KK), jj = i - 4 * KK;
            if (i < 4 * KK)
                fr[i % (AH + 1)] = *(const bf16x8 *)((j < KK ? kt : vt) + h * 32 * ROWB + (kbase ^ (uint32_t)(32 * (j % KK))));
            else
                fr[i % (AH + 1)] = tr_frag<D>(kt, tb, jj / MD, jj % MD);
        };
        auto weights = [&](int h, int v) { S[h][v] = fast_exp2(__builtin_fmaf(S[h][v], c2, -lse2)); };
        auto grads = [&](int h, int v) { dsf[h][v >> 3][v & 7] = (__bf16)(S[h][v] * (dPt[h][v] + nD)); };
        // weights of keys past the row's end are 0, in the tiles that straddle
        // some row's end only (a real branch: the compiler would otherwise
        // turn this rare path into selects executed on every tile)
        auto mask = [&](int h) {
            if ((t + 1) * 64 > kfull) {
                asm volatile("" ::: "memory");
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (t * 64 + h * 32 + 8 * (v >> 2) + 4 * hf + (v & 3) >= my_kend) S[h][v] = 0.f;
            }
        };
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int v = 0; v < 16; ++v) S[h][v] = dPt[h][v] = 0.f;
#pragma unroll
        for (int i = 0; i < AH; ++i) rd(i);
        constexpr int PS = 16 / KK;   // elements per step of a half's S or dP
#pragma unroll
        for (int i = 0; i < 4 * KK; ++i) {
            rd(i + AH);
            const int h = i / (2 * KK), j = i % (2 * KK);
            if (j < KK)
                S[h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (AH + 1)], qf[j % KK], S[h], 0, 0, 0);
            else
                dPt[h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (AH + 1)], dof[j % KK], dPt[h], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < PS; ++u) {
                if (j >= KK) weights(h, PS * (j - KK) + u);
                else if (h == 1) grads(0, PS * j + u);
            }
            if (i >= 1 && i <= 2 * NI) issue_part(t + 1, i - 1);
            __builtin_amdgcn_sched_barrier(0);
            if (j == 2 * KK - 1) mask(h);
        }
        constexpr int PG = 8 / MD;    // elements of dS1 per step of dQ (half 0)
#pragma unroll
        for (int i = 0; i < 4 * MD; ++i) {
            const int n = 4 * KK + i;
            if (i + AH < 4 * MD) rd(n + AH);
            acc[i % MD] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % (AH + 1)], dsf[i / (2 * MD)][i / MD % 2],
                                                                 acc[i % MD], 0, 0, 0);
            if (i < 2 * MD) {
#pragma unroll
                for (int u = 0; u < PG; ++u) grads(1, PG * i + u);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_vm_lgkm<0>();   // tile t + 1 landed (and this tile's LDS reads are done)
        wg_barrier();
    }
    if (row < a.L) {
        float *op = a.dq + b * a.dq_sb + (int64_t)row * a.dq_st + h * a.dq_sh;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                f32x4 val;
#pragma unroll
                for (int e = 0; e < 4; ++e) val[e] = acc[md][4 * gq + e] * a.scale;
                *(f32x4 *)(op + 32 * md + 8 * gq + 4 * hf) = val;
            }
    }
}

// dK and dV: one work-group = (stream, KV head, 128 keys), 8 waves: wave w
// owns keys 32 (w % 4) .. + 31 and belongs to group w / 4.  The
// work-group's K and V stay in LDS; the chunks of 32 query rows (every row
// that sees any of these keys, for every query head of the KV group, walked
// from the sequence end) alternate between the two groups, each with its own
// two LDS stages, so two waves share every SIMD.  At the end group 1 hands its
// partial sums to group 0 through LDS (fixed order: group 0's + group 1's).
//
// A chunk costs a wave 32 MFMAs (1024 cycles) and, as straight code, half
// as many cycles again of vector work that both waves of a SIMD reach
// together; so every vector instruction, address step and load stands in the
// shadow of an MFMA that does not need it (chunk() below), element masks run
// only on the chunks that straddle a block end, and the loads take
// wave-uniform bases advanced by additions.  2 x 16384 tokens, GQA 32/8 x
// 128: 9.0 -> 7.8 ms (cycles -15 %; the clock is power-limited there, 1.74
// to 1.86 GHz, and MFMA busy 48 -> 59 %).  Two MFMAs of read-ahead and three
// measured the same.  A barrier per group of four waves instead of the
// work-group's, with or without a half-step offset between the groups,
// measured the same too.
template <int D>
__global__ __launch_bounds__(512) void bwd_dkdv_kernel(const BwdArgs a) {
    constexpr int ROWB = 2 * D, KK = D / 16, MD = D / 32;
    constexpr int TILEK = 128 * ROWB, TILEC = 32 * ROWB;
    constexpr int CPR = ROWB / 16, RPP = 512 / CPR, NPK = 128 / RPP;
    constexpr int SMEM = 2 * TILEK + 2 * 2 * 2 * TILEC;   // K, V; [group][stage][Q, dO]
    static_assert(2 * 4 * MD * 16 * 64 * 4 <= SMEM, "the partial sums fit the tiles' space");
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    __shared__ __attribute__((aligned(256))) float srow[2][2][128];   // [group][stage][lse2, -D, key end (twice) of 32 rows]
    const int nkt = (a.L + 127) / 128;
    const int wid = blockIdx.x;
    // Key tiles from the first keys (seen by the most rows: the heaviest)
    // over all (stream, KV head) groups, so the dispatch order is
    // longest-first across the whole launch.  Work-group i runs on XCD
    // i mod 8: when the group count is a multiple of 8, XCD x keeps groups
    // x, x + 8, ... for the whole launch and takes their key tiles in blocks
    // of KB_DKDV, the tiles of a block of one group one after another, so
    // they start together and walk the same rows at about the same time
    // (one L2 read serves them); the launch is rounded up to whole blocks
    // and work-groups past the last key tile exit at once.
    const int ngrp = a.B * a.Hkv;
    int kt, grpi, split = 0, nsplit = 1;
    if (a.split_tiles) {
        // items in tile order, the groups as the fast digit (with a multiple
        // of 8 groups each stays on one XCD)
        const int it = wid / ngrp;
        grpi = wid - it * ngrp;
        int lo = 0, hi = nkt - 1;   // the last tile that starts at or before it
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.tile_start[mid] <= it) lo = mid; else hi = mid - 1;
        }
        kt = lo;
        split = it - a.tile_start[kt];
        nsplit = a.tile_start[kt + 1] - a.tile_start[kt];
    } else if (ngrp % NUM_XCD == 0) {
        const int gpx = ngrp / NUM_XCD, x = wid % NUM_XCD, l = wid / NUM_XCD;
        const int kb = l / (gpx * KB_DKDV), r = l - kb * gpx * KB_DKDV;
        const int gi = r / KB_DKDV;
        kt = kb * KB_DKDV + (r - gi * KB_DKDV);
        grpi = x + NUM_XCD * gi;
        if (kt >= nkt) return;
    } else {
        kt = wid / ngrp;
        grpi = wid % ngrp;
    }
    const int kvh = grpi % a.Hkv;
    const int b = grpi / a.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, sub = wave & 3;
    const int kw0 = kt * 128;
    const int key = kw0 + 32 * sub + l32;
    const float c2 = a.scale_log2;
    // the work-group's K and V (rows past the end repeat the last key)
    {
        const int lr = tid / CPR, lc = tid % CPR;
        const uint16_t *kg = a.k + b * a.k_sb + kvh * a.k_sh + 8 * lc;
        const uint16_t *vg = a.v + b * a.v_sb + kvh * a.v_sh + 8 * lc;
#pragma unroll
        for (int p = 0; p < NPK; ++p) {
            const int r = lr + p * RPP;
            const int kr = min(kw0 + r, a.L - 1);
            *(u32x4 *)(smem + tile_off<D>(r, lc)) = *(const u32x4 *)(kg + (int64_t)kr * a.k_st);
            *(u32x4 *)(smem + TILEK + tile_off<D>(r, lc)) = *(const u32x4 *)(vg + (int64_t)kr * a.v_st);
        }
    }
    // first row that sees any of these keys (key ends do not decrease)
    const int32_t *kend_b = a.kend + (int64_t)b * a.L;
    int lo = 0, hi = a.L - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ld_uniform(kend_b, mid) > kw0) hi = mid; else lo = mid + 1;
    }
    const int i0 = lo;
    // Chunks of 32 query rows counted from the sequence end, down to row i0,
    // with the query heads innermost: chunk it holds rows L - 32 (c + 1) ..
    // L - 32 c - 1 (c = it / G) of head it % G.  The work-groups of a KV head
    // (different key tiles, running side by side) then read the same rows at
    // about the same time and the L2 serves them once.  Rows before i0 see
    // none of these keys, so the masking zeroes their terms.
    // A split takes a contiguous share [first, total) of the chunks; group grp
    // takes chunks first + grp, first + grp + 2, ...
    const int nch = (a.L - i0 + 31) / 32;
    const int first = (int)((int64_t)a.G * nch * split / nsplit);
    const int total = (int)((int64_t)a.G * nch * (split + 1) / nsplit);
    const int nstep = (total - first + 1) / 2;

    // Rows from im on see every key of this wave, so a chunk whose first row
    // is at or past im needs no element masks (key ends do not decrease).
    int im;
    {
        const int kl = min(kw0 + 32 * sub + 31, a.L - 1);
        int mlo = i0, mhi = a.L;
        while (mlo < mhi) {
            const int mid = (mlo + mhi) >> 1;
            if (ld_uniform(kend_b, mid) > kl) mhi = mid; else mlo = mid + 1;
        }
        im = mlo;
    }
    // Q and dO rows of one chunk go straight to LDS: wave-wide load i of wave
    // `sub` fills rows 4 RPW i + RPW sub .. + RPW - 1 of the tile, from a
    // wave-uniform base and a per-lane 32-bit offset (the swizzle repeats
    // every 16 rows, so the offset serves every i).
    constexpr int RPW = 1024 / ROWB, LPR = ROWB / 16, NI = TILEC / 4096;
    static_assert(4 * RPW % 16 == 0, "the swizzle must repeat across a wave's loads");
    const int64_t qst = 2 * a.q_st, dst = 2 * a.do_st;
    const int lrow = RPW * sub + lane / LPR;
    const uint32_t lch = (uint32_t)(16 * ((lane % LPR) ^ swz<D>(lrow)));
    const uint32_t qofs = (uint32_t)(lrow * (uint32_t)qst) + lch, dofs = (uint32_t)(lrow * (uint32_t)dst) + lch;
    // lanes 0..31 fetch lse2 and lanes 32..63 -D of the chunk's rows
    const uint32_t rofs = 4u * (uint32_t)(l32 + hf * a.L), eofs = 4u * (uint32_t)l32;
    const bool wide = a.wide_strides != 0;   // 32-bit row offsets do not reach
    // Next chunk to load (chunk ni of the tile): its
    // first row (may be negative: rows before 0 are no rows), its query head
    // within the group, and that row's addresses in Q, dO and the row data
    // (lse2 of a head, then -D).  Advanced by additions only.
    const int64_t qsh = 2 * a.q_sh, dsh = 2 * a.do_sh, rsh = 8 * (int64_t)a.L;
    const int64_t qwrap = a.G * qsh + 32 * qst, dwrap = a.G * dsh + 32 * dst, rwrap = a.G * rsh + 128;
    int ni = first + grp, nh = ni % a.G, nr0 = a.L - 32 * (ni / a.G + 1);
    const char *nq = (const char *)(a.q + b * a.q_sb) + (kvh * a.G + nh) * qsh + nr0 * qst;
    const char *nd = (const char *)(a.dout + b * a.do_sb) + (kvh * a.G + nh) * dsh + nr0 * dst;
    const char *nr = (const char *)a.dl + ((int64_t)b * a.Hq + kvh * a.G + nh) * rsh + 4 * (int64_t)nr0;
    auto advance = [&]() {
        ni += 2;
        nh += 2;
        nq += 2 * qsh;
        nd += 2 * dsh;
        nr += 2 * rsh;
        while (nh >= a.G) {
            nh -= a.G;
            nr0 -= 32;
            nq -= qwrap;
            nd -= dwrap;
            nr -= rwrap;
        }
    };
    // Load part i (0 .. 2 NI) of the next chunk into stage st: the parts are
    // issued between the MFMAs of the current chunk.  A chunk with rows
    // before 0, or rows too far apart, is loaded whole in part 0 with
    // per-lane addresses.
    constexpr int NPART = 2 * NI + 1;
    auto issue_part = [&](int i, int st) {
        if (ni >= total) return;
        const uint32_t base = lds_addr(smem) + (uint32_t)(2 * TILEK + (grp * 2 + st) * 2 * TILEC);
        const uint32_t rl = lds_addr((const char *)&srow[grp][st][0]);
        if (nr0 < 0 || wide) {
            if (i) return;
            // (the lane is hidden from the optimiser, so that what this rare
            // path derives from it is not hoisted and held in registers)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            dma_rows<D, 4, 32>(nq - nr0 * qst, qst, nr0, a.L - 1, base, sub, ln);
            dma_rows<D, 4, 32>(nd - nr0 * dst, dst, nr0, a.L - 1, base + TILEC, sub, ln);
            const int64_t r = max(nr0 + (ln & 31), 0);
            if (sub == 0) dma4(nr + 4 * (r - nr0 + (ln >> 5) * (int64_t)a.L), rl);
            if (sub == 1) dma4(kend_b + r, rl + 256);
        } else if (i < NI) {
            dma16s(nq + i * (4 * RPW) * qst, qofs, base + i * 4096 + sub * 1024);
        } else if (i < 2 * NI) {
            dma16s(nd + (i - NI) * (4 * RPW) * dst, dofs, base + TILEC + (i - NI) * 4096 + sub * 1024);
        } else {
            if (sub == 0) dma4s(nr, rofs, rl);
            if (sub == 1) dma4s((const char *)(kend_b + nr0), eofs, rl + 256);
        }
    };
    // LDS read addresses: Q / dO fragments (row l32, chunk 2 kk + hf) relative
    // to this group's stage 0, K / V fragments of this wave's keys, and the
    // transpose reads of dO / Q
    const uint32_t kbase = (uint32_t)(l32 * ROWB + 16 * (hf ^ swz<D>(l32)));
    uint32_t tb[2];
    tr_bases<D>(lane, tb);
    const char *ctile = smem + 2 * TILEK + grp * 4 * TILEC;
    const char *ktile = smem + 32 * sub * ROWB, *vtile = ktile + TILEK;

    f32x16 dk[MD], dv[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
        for (int v = 0; v < 16; ++v) dk[md][v] = dv[md][v] = 0.f;
    // One chunk of 32 query rows (from row r0) in stage st
    auto chunk = [&](int st, int r0) {
        const char *qt = ctile + st * 2 * TILEC, *dt = qt + TILEC;
        const float *ri = &srow[grp][st][4 * hf];
        // One MFMA stream in which every vector instruction stands beside a
        // matrix instruction that does not need it: S = Q K^T; then
        // dP - D = dO V^T - D (accumulated from -D) beside P = exp2(S c2 -
        // lse2); then dV^T += dO^T P beside dS = P (dP - D); then dK^T +=
        // Q^T dS.  Operands are read AH steps ahead; the fences keep this
        // order.
        f32x16 S, dP;
        f32x4 l4[4];
#pragma unroll
        for (int v = 0; v < 16; ++v) S[v] = 0.f;
        bf16x8 fa[AH + 1], fb[AH + 1];
        auto rd = [&](int i) {
            const char *ct = i < KK ? qt : dt, *ot = i < KK ? ktile : vtile;
            const uint32_t x = kbase ^ (uint32_t)(32 * (i % KK));
            fa[i % (AH + 1)] = *(const bf16x8 *)(ct + x);
            fb[i % (AH + 1)] = *(const bf16x8 *)(ot + x);
        };
#pragma unroll
        for (int i = 0; i < AH; ++i) rd(i);
#pragma unroll
        for (int i = 0; i < 2 * KK; ++i) {
            if (i + AH < 2 * KK) rd(i + AH);
            if (i >= KK - 4 && i < KK) {
                const int gq = i - (KK - 4);
                l4[gq] = *(const f32x4 *)(ri + 8 * gq);
                const f32x4 d4 = *(const f32x4 *)(ri + 32 + 8 * gq);
#pragma unroll
                for (int e = 0; e < 4; ++e) dP[4 * gq + e] = d4[e];
            }
            if (i < KK) {
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i % (AH + 1)], fb[i % (AH + 1)], S, 0, 0, 0);
            } else {
                dP = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i % (AH + 1)], fb[i % (AH + 1)], dP, 0, 0, 0);
                constexpr int PS = 16 / KK;
#pragma unroll
                for (int u = 0; u < PS; ++u) {
                    const int v = PS * (i - KK) + u;
                    S[v] = fast_exp2(__builtin_fmaf(S[v], c2, -l4[v >> 2][v & 3]));
                }
            }
            if (i >= 1 && i <= NPART) issue_part(i - 1, st ^ 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (r0 < im) {
            // (a real branch: the compiler would otherwise turn this rare
            // path into selects executed on every chunk)
            int ln = lane;
            asm volatile("" : "+v"(ln) :: "memory");
            const int ky = kw0 + 32 * sub + (ln & 31);
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const int r = 8 * gq + 4 * (ln >> 5);
                const i32x4 ke = *(const i32x4 *)&srow[grp][st][64 + r];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    S[4 * gq + e] = ((r0 + r + e >= 0) & (ky < ke[e])) ? S[4 * gq + e] : 0.f;
            }
        }
        // P (rows 8 (v / 4) + 4 hf + v % 4 of the lane's key) as B fragments
        bf16x8 pf[2], dsf[2], fr[AH + 1];
#pragma unroll
        for (int i = 0; i < AH; ++i) fr[i] = tr_frag<D>(dt, tb, i / MD, i % MD);
#pragma unroll
        for (int v = 0; v < 16; ++v) pf[v >> 3][v & 7] = (__bf16)S[v];
#pragma unroll
        for (int i = 0; i < 4 * MD; ++i) {
            const int n = i + AH;
            if (n < 4 * MD) fr[n % (AH + 1)] = tr_frag<D>(n < 2 * MD ? dt : qt, tb, n / MD % 2, n % MD);
            const int ks = i / MD % 2, md = i % MD;
            if (i < 2 * MD) {
                dv[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (AH + 1)], pf[ks], dv[md], 0, 0, 0);
                constexpr int PS = 8 / MD;
#pragma unroll
                for (int u = 0; u < PS; ++u) {
                    const int v = PS * i + u;
                    dsf[v >> 3][v & 7] = (__bf16)(S[v] * dP[v]);
                }
            } else {
                dk[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (AH + 1)], dsf[ks], dk[md], 0, 0, 0);
            }
            if (i == 2 * MD) advance();   // (the loads of the current next chunk are all issued)
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const bool any = first + grp < total;
    int r0 = nr0;   // first row of the current step's chunk
    if (any) {
#pragma unroll
        for (int i = 0; i < NPART; ++i) issue_part(i, 0);
        advance();
    }
    wait_vm_lgkm<0>();
    wg_barrier();
    for (int s = 0; s < nstep; ++s) {
        // (a group without a chunk in the last step has nothing left to load)
        const int rn = nr0;
        if (first + 2 * s + grp < total) chunk(s & 1, r0);
        r0 = rn;
        wait_vm_lgkm<0>();   // the next chunks landed; this step's LDS reads are done
        wg_barrier();
    }
    // group 1 -> LDS -> group 0, in register order (conflict-free)
    float *part = (float *)smem;
    const int pbase = (sub * MD) * 16 * 64 + lane;
    if (grp == 1) {
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                part[pbase + (md * 16 + v) * 64] = dk[md][v];
                part[4 * MD * 16 * 64 + pbase + (md * 16 + v) * 64] = dv[md][v];
            }
    }
    wait_vm_lgkm<0>();
    wg_barrier();
    if (grp == 0 && nsplit > 1) {
        // this split's sums, unscaled, in register order (1 KB per store)
        float *pp = a.part + (((int64_t)(a.tile_start[kt] + split) * ngrp + grpi) * 2 * 128 + 32 * sub) * D + 4 * lane;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                f32x4 kv, vv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = 4 * gq + e;
                    kv[e] = dk[md][v] + part[pbase + (md * 16 + v) * 64];
                    vv[e] = dv[md][v] + part[4 * MD * 16 * 64 + pbase + (md * 16 + v) * 64];
                }
                *(f32x4 *)(pp + (md * 4 + gq) * 256) = kv;
                *(f32x4 *)(pp + 128 * D + (md * 4 + gq) * 256) = vv;
            }
        return;
    }
    if (grp == 0 && key < a.L) {
        float *kp = a.dk + b * a.dk_sb + (int64_t)key * a.dk_st + kvh * a.dk_sh;
        float *vp = a.dv + b * a.dv_sb + (int64_t)key * a.dv_st + kvh * a.dv_sh;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                f32x4 kv, vv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = 4 * gq + e;
                    kv[e] = (dk[md][v] + part[pbase + (md * 16 + v) * 64]) * a.scale;
                    vv[e] = dv[md][v] + part[4 * MD * 16 * 64 + pbase + (md * 16 + v) * 64];
                }
                *(f32x4 *)(kp + 32 * md + 8 * gq + 4 * hf) = kv;
                *(f32x4 *)(vp + 32 * md + 8 * gq + 4 * hf) = vv;
            }
    }
}

// Adds the partial sums of the split key tiles in split order and writes dK
// and dV.  One thread per 4 elements (one register group of one lane of the
// kernel above); bound by reading the partials.
template <int D>
__global__ __launch_bounds__(256) void bwd_sum_kernel(const BwdArgs a) {
    constexpr int PER = 128 * D / 4 / 256;   // blocks per (tile, group, dK or dV)
    const int ngrp = a.B * a.Hkv;
    const int blk = blockIdx.x % PER, wh = blockIdx.x / PER % 2, tg = blockIdx.x / (2 * PER);
    const int kt = tg / ngrp, grpi = tg - kt * ngrp;
    const int s0 = a.tile_start[kt], ns = a.tile_start[kt + 1] - s0;
    const int u = blk * 256 + threadIdx.x;   // ((sub * MD + md) * 4 + gq) * 64 + lane
    const int64_t stride = (int64_t)ngrp * 2 * 128 * D;
    const float *pp = a.part + (((int64_t)s0 * ngrp + grpi) * 2 + wh) * 128 * D + 4 * u;
    f32x4 x[BWD_MAX_SPLITS];
#pragma unroll
    for (int s = 0; s < BWD_MAX_SPLITS; ++s)
        if (s < ns) x[s] = *(const f32x4 *)(pp + s * stride);
    f32x4 sum = x[0];
#pragma unroll
    for (int s = 1; s < BWD_MAX_SPLITS; ++s)
        if (s < ns)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += x[s][e];
    const int lane = u & 63, gq = (u >> 6) & 3, md = (u >> 8) % (D / 32), sub = (u >> 8) / (D / 32);
    const int key = kt * 128 + 32 * sub + (lane & 31);
    if (key >= a.L) return;
    const int b = grpi / a.Hkv, kvh = grpi - b * a.Hkv;
    const int d0 = 32 * md + 8 * gq + 4 * (lane >> 5);
    float *op = wh ? a.dv + b * a.dv_sb + (int64_t)key * a.dv_st + kvh * a.dv_sh
                   : a.dk + b * a.dk_sb + (int64_t)key * a.dk_st + kvh * a.dk_sh;
    if (!wh)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] *= a.scale;
    *(f32x4 *)(op + d0) = sum;
}

template <int D>
int launch_bwd_t(const BwdArgs &a, hipStream_t st) {
    const int64_t nqt = (a.L + 127) / 128;
    hipLaunchKernelGGL(bwd_dq_kernel<D>, dim3((unsigned)(a.B * a.Hq * nqt)), dim3(256), 0, st, a);
    if (int e = (int)hipGetLastError()) return e;
    const int64_t ngrp = (int64_t)a.B * a.Hkv;
    if (a.split_tiles) {
        hipLaunchKernelGGL(bwd_dkdv_kernel<D>, dim3((unsigned)(ngrp * a.tile_start[nqt])), dim3(512), 0, st, a);
        if (int e = (int)hipGetLastError()) return e;
        constexpr int64_t PER = 128 * D / 4 / 256;
        hipLaunchKernelGGL(bwd_sum_kernel<D>, dim3((unsigned)(a.split_tiles * ngrp * 2 * PER)), dim3(256), 0, st, a);
        return (int)hipGetLastError();
    }
    const int64_t grid = ngrp % NUM_XCD == 0 ? ngrp * ((nqt + KB_DKDV - 1) / KB_DKDV) * KB_DKDV : ngrp * nqt;
    hipLaunchKernelGGL(bwd_dkdv_kernel<D>, dim3((unsigned)grid), dim3(512), 0, st, a);
    return (int)hipGetLastError();
}

}  // namespace

int launch_prefill_bwd(const BwdArgs &a, int head_dim, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (head_dim == 128) return launch_bwd_t<128>(a, st);
    if (head_dim == 64) return launch_bwd_t<64>(a, st);
    return (int)hipErrorInvalidValue;
}

}  // namespace ws
