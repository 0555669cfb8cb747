// Ranks of a pool's slots and whether any of them is below the pool's (host side).
//
// Calls on different slots may come from different threads, and a compute call on a third may ask for any_lower()
// meanwhile: a call touches its own slot's entry and a counter of the slots below the pool's rank, and no entry of
// another slot.
#pragma once
#include <atomic>
#include <cstdint>
#include <vector>

namespace lora {

class AdapterRanks {
public:
    // r: ranks of the n slots, or null: the pool's
    void init(int pool_rank, int n, const int32_t *r)
    {
        pool_rank_ = pool_rank;
        rank_.assign(n, pool_rank);
        n_lower_ = 0;
        for (int a = 0; r && a < n; ++a) set(a, r[a]);
    }
    int operator[](int adapter) const { return rank_[adapter]; }
    void set(int adapter, int rank)
    {
        const int change = (rank < pool_rank_) - (rank_[adapter] < pool_rank_);
        rank_[adapter] = rank;
        if (change) n_lower_.fetch_add(change, std::memory_order_relaxed);
    }
    bool any_lower() const { return n_lower_.load(std::memory_order_relaxed) > 0; }

private:
    int pool_rank_ = 0;
    std::vector<int32_t> rank_;
    std::atomic<int> n_lower_{0};
};

}  // namespace lora
