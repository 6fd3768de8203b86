// The opaque handles of the C ABI as the library's own sources see them.
#pragma once
#include <memory>

#include "plan.h"

struct rl_ctx { std::shared_ptr<rl::ErrBox> err; };
struct rl_graph { rl::Graph g; };
// small: the same graph for the built-in workspace, where p does not fit into it and a plan that spends less does (else null).
// A param's packed buffer then holds p's weights and, behind them at small_offset, small's.
struct rl_plan {
    rl::Plan p;
    std::unique_ptr<rl::Plan> small;
};

namespace rl {
inline size_t small_offset(const PackSpec &of_p) { return (of_p.bytes + 255) & ~(size_t)255; }
rl_status run_bound(const Plan &p, const rl_binding *bindings, int32_t n_bindings, void *ws, size_t ws_bytes, void *stream);
}
