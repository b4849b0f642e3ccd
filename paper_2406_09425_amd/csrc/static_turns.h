// Whose turn it is in sgprs_pool_run_static: host logic without HIP, so that it can be checked without a GPU.
#pragma once
#include <vector>

namespace sgprs {

// Partitions with work take turns on the `max_busy` places (0: a place for each).  While a partition is
// active, up to kStaticDepth inferences are queued on its stream, so the next one starts without a host
// round trip behind the one before (with one at a time, the event poll and the launch lay between them:
// eight tasks on 8 x 32 CUs, four busy, 68 us per inference against 37).  After kStaticTurn inferences
// it makes room, if one that waits could take its place.
constexpr int kStaticDepth = 2, kStaticTurn = 8;

class StaticTurns {
public:
    // left[p]: inferences pinned to partition p.  Partitions p and p + pipes share a dispatch pipe: with a
    // gate of up to `pipes`, no two busy partitions may share one.
    StaticTurns(const std::vector<long long>& left, int max_busy, int pipes)
        : parts_(left.size()), max_busy_(max_busy), pipes_(pipes), per_pipe_(max_busy > 0 && max_busy <= pipes),
          pipe_busy_(pipes, 0)
    {
        for (size_t p = 0; p < left.size(); ++p) {
            parts_[p].left = left[p];
            if (left[p]) waiting_.push_back((int)p);
        }
    }
    bool finished() const { return waiting_.empty() && active_.empty(); }
    const std::vector<int>& active() const { return active_; }  // in the order they are served
    int queued(int p) const { return parts_[p].queued; }

    // Fills the free places, whoever has waited longest first.  (Going round by index instead, one that
    // shares its pipe can find it taken every time its number comes up.)
    void admit()
    {
        for (size_t w = 0; w < waiting_.size() && !(max_busy_ && (int)active_.size() >= max_busy_);) {
            const int p = waiting_[w], pipe = p % pipes_;
            if (per_pipe_ && pipe_busy_[pipe]) {
                ++w;
                continue;
            }
            parts_[p].turn = kStaticTurn;
            active_.push_back(p);
            ++pipe_busy_[pipe];
            waiting_.erase(waiting_.begin() + w);
        }
    }
    // May active partition p queue another inference?  A turn that nobody could use begins anew.
    bool may_launch(int p)
    {
        Part& q = parts_[p];
        if (!wanted(p)) q.turn = kStaticTurn;
        return q.queued < kStaticDepth && q.left && q.turn;
    }
    void launched(int p) { ++parts_[p].queued, --parts_[p].left, --parts_[p].turn; }
    void completed(int p) { --parts_[p].queued; }
    // Gives p's place back if its turn is over and its stream empty; with work left it queues up again.
    bool release(int p)
    {
        Part& q = parts_[p];
        if (q.queued || (q.left && q.turn)) return false;
        --pipe_busy_[p % pipes_];
        if (q.left) waiting_.push_back(p);
        for (size_t a = 0; a < active_.size(); ++a)
            if (active_[a] == p) {
                active_.erase(active_.begin() + a);
                break;
            }
        return true;
    }

private:
    struct Part {
        long long left = 0;        // inferences not yet launched
        int queued = 0, turn = 0;  // in flight; launches left in this turn
    };
    // Does a waiting partition fit the place that p would leave?  Those on a pipe without a busy partition
    // count too: with a gate below the number of pipes it is the gate that they wait for.
    bool wanted(int p) const
    {
        for (int w : waiting_)
            if (!per_pipe_ || !pipe_busy_[w % pipes_] || w % pipes_ == p % pipes_) return true;
        return false;
    }
    std::vector<Part> parts_;
    int max_busy_, pipes_;
    bool per_pipe_;
    std::vector<int> pipe_busy_, active_, waiting_;
};

}  // namespace sgprs
