// moe_layer_forward: the calls of one expert layer in sequence; a short batch is sorted by the first contraction's
// workgroups instead of a launch of its own, and a handful of tokens is routed by them as well.  The same goes for the separate calls:
// the sorted copies of the rows that these write are by-products of the contractions, and the combine of a top-1 layer is the epilogue of the second one.
// Small layers are bound by their launches (and by the host, about 4 us each): one token, 5 experts of 896 x 3584 19.0 us in five
// launches, 10.0 in two; 38 tokens, 8 of 1152 x 4608 46.6 and 39.3; 46 tokens in fp32, 5 of 44 x 812 20.5 and 15.1; with a dispatch of its own, 2759
// tokens, 7 of 1856 x 5184 171.0 and 166.2.  What sorts in tiles besides: routed_tiles_fit().
#include "ffn_common.hpp"

extern "C" int moe_layer_forward(const exf_moe_layer* layer, void* stream)
{
    EXF_REQUIRE_PTR(layer);
    const exf_moe_layer& l = *layer;
    const bool fused = l.fused != 0;
    void* x_sorted = fused ? nullptr : l.x_sorted;
    const int32_t* idx = l.forced_idx != nullptr ? l.forced_idx : l.topk_idx;
    // everything the calls refuse, before anything is launched
    if (int bad = exf::check_gate(l.x, l.w_gate, l.T, l.d, l.E, l.k, l.dt, l.topk_idx, l.topk_w)) return bad;
    if (int bad = exf::check_dispatch(l.x, idx, l.T, l.d, l.k, l.E, l.E_local, l.dt, x_sorted, l.src_of_sorted, l.sorted_of_src, l.expert_counts,
                                      l.expert_offsets, l.dispatch_workspace, l.dispatch_workspace_bytes))
        return bad;
    if (fused) {
        if (int bad = exf::check_ffn_fused(l.x, l.src_of_sorted, l.sorted_of_src, l.topk_w, l.expert_offsets, l.w1, l.w2, l.T, l.k, l.d, l.f,
                                           l.E_local, l.act, l.dt, l.out, l.ffn_workspace, l.ffn_workspace_bytes))
            return bad;
    } else {
        if (int bad = exf::check_ffn(l.x_sorted, l.expert_offsets, l.w1, l.w2, l.T * l.k, l.d, l.f, l.E_local, l.act, l.dt, l.y_sorted,
                                     l.ffn_workspace, l.ffn_workspace_bytes))
            return bad;
        if (int bad = exf::check_combine(l.y_sorted, l.sorted_of_src, l.topk_w, l.T, l.d, l.k, l.dt, l.out)) return bad;
    }
    // A first contraction that sorts reads the ids, and x where separate calls read their sorted copy, while hidden activations are written.  Calls in sequence
    // may have these in the workspace of a later one: there they stay calls in sequence.
    const int64_t A = l.T * l.k;
    const size_t elem = l.dt == EXF_BF16 ? 2 : 4;
    const size_t hidden = fused ? moe_expert_ffn_fused_workspace_bytes(l.T, l.k, l.d, l.f, l.E_local, l.dt) : moe_expert_ffn_workspace_bytes(A, l.d, l.f, l.E_local, l.dt);
    auto apart = [&](const void* p, size_t n) { return exf::lie_apart(p, n, l.ffn_workspace, hidden); };
    const bool free = apart(idx, A * sizeof(int32_t)) && apart(l.expert_map, l.E * sizeof(int32_t)) && (fused || apart(l.x, l.T * l.d * elem));
    const bool streamed = free && exf::routed_path_fits(A, l.d, l.f, l.E_local, l.dt);
    const bool routed = streamed || (free && !fused && exf::routed_tiles_fit(A, l.d, l.f, l.E, l.E_local, l.dt));
    const bool gated = streamed && exf::gate_joins_layer(l.T, l.d, l.E, l.dt, idx != l.topk_idx) && apart(l.w_gate, l.E * l.d * elem);
    int rc = EXF_OK;
    if (!gated) rc = moe_gate_topk(l.x, l.w_gate, l.T, l.d, l.E, l.k, l.renormalize, l.dt, nullptr, l.topk_idx, l.topk_w, stream);
    if (rc != EXF_OK) return rc;
    if (routed) {
        exf::FfnRouting r{idx,          l.expert_map, l.E, l.src_of_sorted, l.sorted_of_src, l.expert_counts, l.expert_offsets, gated ? l.w_gate : nullptr,
                          l.renormalize, l.topk_idx,   l.topk_w, x_sorted, fused ? nullptr : l.y_sorted};
        return exf::ffn_fused_routed(r, l.x, l.topk_w, l.w1, l.w2, l.T, l.k, l.d, l.f, l.E_local, l.act, l.dt, l.out, l.ffn_workspace,
                                     l.ffn_workspace_bytes, stream);
    }
    rc = moe_dispatch(l.x, idx, l.expert_map, l.T, l.d, l.k, l.E, l.E_local, l.dt, x_sorted, l.src_of_sorted,
                      l.sorted_of_src, l.expert_counts, l.expert_offsets, l.dispatch_workspace, l.dispatch_workspace_bytes, stream);
    if (rc != EXF_OK) return rc;
    if (fused)
        return moe_expert_ffn_fused(l.x, l.src_of_sorted, l.sorted_of_src, l.topk_w, l.expert_offsets, l.w1, nullptr, l.w2, nullptr, l.T,
                                    l.k, l.d, l.f, l.E_local, l.act, l.dt, l.out, l.ffn_workspace, l.ffn_workspace_bytes, stream);
    if (l.k == 1)  // (several contributions to an output row: from different workgroups)
        return exf::ffn_combined(l.x_sorted, l.src_of_sorted, l.sorted_of_src, l.topk_w, l.expert_offsets, l.w1, l.w2, l.T, l.d, l.f, l.E_local, l.act,
                                 l.dt, l.y_sorted, l.out, l.ffn_workspace, stream);
    rc = moe_expert_ffn(l.x_sorted, l.expert_offsets, l.w1, nullptr, l.w2, nullptr, l.T * l.k, l.d, l.f, l.E_local, l.act, l.dt,
                        l.y_sorted, l.ffn_workspace, l.ffn_workspace_bytes, stream);
    if (rc != EXF_OK) return rc;
    return moe_combine(l.y_sorted, l.sorted_of_src, l.topk_w, l.T, l.d, l.k, l.dt, l.out, stream);
}
