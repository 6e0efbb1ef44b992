// The library's host side (ws_api.cpp) over launchers that record what they
// are given instead of enqueueing it: the tests read the plan of a call from
// it, on the CPU, for any number of compute units.
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/ws_attn.h"
#include "../../paper_2606_25041_amd/csrc/ws_kernels.h"

namespace {
int g_cus = 256;
struct Seen {
    ws::AttnArgs attn;
    ws::RaggedPlan rag;
    ws::BwdArgs bwd;
    int kg, ragged, combined;
} g_seen;
alignas(16) char g_mem[16];   // stands for every device pointer

ws_tensor4 tensor(int32_t dtype, int64_t tokens, int64_t heads, int64_t d) {
    return ws_tensor4{g_mem, dtype, tokens * heads * d, heads * d, d};
}
}  // namespace

namespace ws {
int launch_attention(const AttnArgs &a, const RaggedPlan *rag, int, TileShape shape, void *) {
    g_seen.attn = a;
    g_seen.ragged = rag != nullptr;
    if (rag) g_seen.rag = *rag;
    g_seen.kg = shape.kg;
    return 0;
}
int launch_combine(const AttnArgs &, const RaggedPlan *, int, void *) { return g_seen.combined = 1, 0; }
int launch_append(const AppendArgs &, void *) { return 0; }
int launch_prefill_bwd(const BwdArgs &a, int, void *) { return g_seen.bwd = a, 0; }
int current_device_cus(int *cus) { return g_cus > 0 ? (*cus = g_cus, 0) : 1; }
int scratch_address(void **p) { return *p = g_mem, 0; }
}  // namespace ws

extern "C" {

// compute units of the pretended device (0: no device)
void probe_cus(int cus) { g_cus = cus; }

// Plans a step; lens, nl (nullable) and ns are [batch].  Returns the status;
// *ragged: every stream has its own split count; ns: those counts; work: work
// items, grid work-groups.
int probe_step(int batch, int hq, int hkv, int d, int new_len, const int32_t *lens, const int32_t *nl, int f32, int *ragged,
               int32_t *ns, int64_t *work) {
    int64_t pages = 1;
    for (int b = 0; b < batch; ++b) pages = std::max<int64_t>(pages, lens[b] / 64 + 1);
    const std::vector<int32_t> table((size_t)(batch * pages), 0);
    const ws_paged_kv kv{g_mem, g_mem, (int32_t *)g_mem, table.data(), 1, WS_PAGE_SIZE, (int32_t)pages, hkv, d};
    const ws_tensor4 q = tensor(WS_DTYPE_BF16, new_len, hq, d), k = tensor(WS_DTYPE_BF16, new_len, hkv, d),
                     out = tensor(f32 ? WS_DTYPE_F32 : WS_DTYPE_BF16, new_len, hq, d);
    memset(&g_seen, 0, sizeof g_seen);
    const int32_t *dev = (const int32_t *)g_mem;
    const int rc = nl ? ws_block_causal_attn_fwd_varlen(q, k, k, &kv, lens, dev, nl, dev, nullptr, nullptr, batch, new_len,
                                                        hq, 0.1f, 0, out, nullptr, g_mem, (size_t)1 << 60, nullptr)
                      : ws_block_causal_attn_fwd(q, k, k, &kv, lens, dev, batch, new_len, hq, 0.1f, 0, out, nullptr, g_mem,
                                                 (size_t)1 << 60, nullptr);
    *ragged = g_seen.ragged;
    for (int b = 0; b < batch; ++b) ns[b] = g_seen.ragged ? g_seen.rag.ns[b] : g_seen.attn.nsplit;
    work[0] = g_seen.attn.n_work;
    work[1] = (int64_t)g_seen.attn.per_xcd * ws::NUM_XCD;
    return rc;
}

// Plans a contiguous prefill in blocks of `block` tokens.  out: key groups,
// units, deal_log2, per_group; work: work items, grid work-groups.
int probe_prefill(int batch, int hq, int hkv, int d, int seq, int block, int *out, int64_t *work) {
    const int nb = (seq + block - 1) / block;
    std::vector<int32_t> off;
    for (int b = 0; b < batch; ++b)
        for (int n = 0; n <= nb; ++n) off.push_back(std::min(n * block, seq));
    const ws_tensor4 q = tensor(WS_DTYPE_BF16, seq, hq, d), k = tensor(WS_DTYPE_BF16, seq, hkv, d);
    memset(&g_seen, 0, sizeof g_seen);
    const int rc = ws_block_causal_prefill(q, k, k, nullptr, off.data(), (const int32_t *)g_mem, batch, seq, nb, hq, hkv, d,
                                           0.1f, q, nullptr, nullptr);
    out[0] = g_seen.kg;
    out[1] = g_seen.attn.units;
    out[2] = g_seen.attn.deal_log2;
    out[3] = g_seen.attn.per_group;
    work[0] = g_seen.attn.n_work;
    work[1] = (int64_t)g_seen.attn.per_xcd * ws::NUM_XCD;
    return rc;
}

}  // extern "C"
