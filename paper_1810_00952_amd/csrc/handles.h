// The opaque handles of the C ABI as the library's own sources see them.
#pragma once
#include <memory>

#include "plan.h"

struct rl_ctx { std::shared_ptr<rl::ErrBox> err; };
struct rl_graph { rl::Graph g; };
// small: the same graph for the built-in workspace, where p does not fit into it and a plan that spends less does (else null).
// A param that the two read laid out differently has both forms in its packed buffer: p's and, behind it at small_offset, small's.
struct rl_plan {
    rl::Plan p;
    std::unique_ptr<rl::Plan> small;
};

namespace rl {
// small's layout of param v where it differs from p's, else null
inline const PackSpec *second_pack(const rl_plan &plan, int v)
{
    if (!plan.small) return nullptr;
    auto own = plan.p.packs.find(v);
    return own == plan.p.packs.end() || plan.small->packs.at(v) == own->second ? nullptr : &plan.small->packs.at(v);
}
inline size_t small_offset(const PackSpec &of_p) { return (of_p.bytes + 255) & ~(size_t)255; }
rl_status run_bound(const Plan &p, const rl_binding *bindings, int32_t n_bindings, void *ws, size_t ws_bytes, void *stream);
}
