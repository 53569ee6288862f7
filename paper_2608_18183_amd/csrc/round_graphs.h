// The captured rounds a context keeps (host code, no device types).
#pragma once
#include <cstddef>
#include <cstdint>
#include <utility>
#include <vector>

namespace hbsjd {

// Pairs of graphs (buffer parity 0 and 1), each with the kernels its products
// were captured with. They are valid while the launch arguments they bake in
// stay the same (the signature); a pair serves a round whose row bound gives
// each of its products the same kernels.
template <typename Plan, typename Exec>
class RoundGraphPool {
  public:
    struct Pair {
        std::vector<Plan> plan;
        int bound = 0;   // the row bound it was captured under
        Exec exec[2] = {};
    };

    explicit RoundGraphPool(size_t limit) : limit_(limit) {}

    // before a round: pairs of another signature go, through destroy(exec)
    template <typename F>
    void match(std::vector<uint64_t> signature, F destroy) {
        if (signature == signature_) return;
        drop(destroy);
        signature_ = std::move(signature);
    }
    // the first pair whose grids cover the bound and whose plan holds, or null
    template <typename F>
    Pair* find(int bound, F holds) {
        for (Pair& p : pairs_)
            if (p.bound >= bound && holds(p.plan)) return &p;
        return nullptr;
    }
    // before a capture: at the limit every pair has to go (drop), the
    // signature, which the next pair shares, stays
    bool full() const { return pairs_.size() >= limit_; }
    Pair* add(Pair pair) {
        pairs_.push_back(std::move(pair));
        return &pairs_.back();
    }
    template <typename F>
    void drop(F destroy) {
        for (Pair& p : pairs_)
            for (Exec& e : p.exec)
                if (e) destroy(e);
        pairs_.clear();
    }

  private:
    size_t limit_;
    std::vector<Pair> pairs_;
    std::vector<uint64_t> signature_;
};

}  // namespace hbsjd
