// The turn-taking of the static executor, driven as the executor drives it, with inferences of one time
// unit: every partition gets its inferences, the gate and the pipe rule hold, no partition waits longer
// than the others' turns, and the makespan is what rotating turns give.  Prints "ok <cases>" or the
// first failure.
#include <algorithm>
#include <cstdio>
#include <initializer_list>

#include "static_turns.h"

using sgprs::kStaticDepth;
using sgprs::kStaticTurn;

static int fail(const char* what, int n_p, int gate, int rounds, long v)
{
    printf("FAIL %s: %d partitions, gate %d, %d rounds (%ld)\n", what, n_p, gate, rounds, v);
    return 1;
}

int main()
{
    constexpr int kPipes = 4;
    long cases = 0;
    for (int n_p = 1; n_p <= 9; ++n_p)
        for (int gate = 0; gate <= 9; ++gate)
            for (int rounds : {1, 3, 4, 5, 8, 9, 20, 100}) {
                std::vector<long long> left(n_p, rounds);
                sgprs::StaticTurns turns(left, gate, kPipes);
                std::vector<long> launched(n_p, 0), done_at(n_p, 0), waited(n_p, 0);
                long now = 0;
                for (; !turns.finished(); ++now) {
                    if (now > 1000000) return fail("never ends", n_p, gate, rounds, now);
                    // a time unit: everybody launches what they may, then the oldest of each stream completes
                    for (bool more = true; more;) {
                        more = false;
                        turns.admit();
                        for (size_t a = 0; a < turns.active().size();) {
                            const int p = turns.active()[a];
                            if (turns.may_launch(p)) {
                                turns.launched(p);
                                ++launched[p];
                                more = true;
                            }
                            if (turns.queued(p) > kStaticDepth) return fail("queue too long", n_p, gate, rounds, p);
                            if (!turns.release(p)) ++a;
                            else more = true;
                        }
                    }
                    const std::vector<int> busy = turns.active();
                    if (gate && (int)busy.size() > gate) return fail("gate", n_p, gate, rounds, (long)busy.size());
                    if (gate && gate <= kPipes)
                        for (size_t i = 0; i < busy.size(); ++i)
                            for (size_t j = 0; j < i; ++j)
                                if (busy[i] % kPipes == busy[j] % kPipes) return fail("two on one pipe", n_p, gate, rounds, busy[i]);
                    std::vector<bool> on(n_p, false);
                    for (int p : busy) {
                        on[p] = true;
                        turns.completed(p);
                        ++done_at[p];
                    }
                    for (int p = 0; p < n_p; ++p) {
                        waited[p] = on[p] || done_at[p] == rounds ? 0 : waited[p] + 1;
                        // all others may get two turns each before it, however many places there are
                        if (waited[p] > 2L * n_p * (kStaticTurn + kStaticDepth)) return fail("starved", n_p, gate, rounds, p);
                    }
                    for (size_t a = 0; a < turns.active().size();)
                        if (!turns.release(turns.active()[a])) ++a;
                }
                for (int p = 0; p < n_p; ++p)
                    if (launched[p] != rounds || done_at[p] != rounds) return fail("inferences", n_p, gate, rounds, launched[p]);
                // lower bound: the places, and (under a gate of up to four) the busiest pipe; a last turn or two
                // may run alone
                const long places = gate == 0 || gate > n_p ? n_p : gate;
                long bound = ((long)n_p * rounds + places - 1) / places;
                if (gate && gate <= kPipes) bound = std::max(bound, (long)((n_p + kPipes - 1) / kPipes) * rounds);
                bound = std::max(bound, (long)rounds);
                if (now > bound + 2 * kStaticTurn) return fail("makespan", n_p, gate, rounds, now);
                ++cases;
            }
    printf("ok %ld\n", cases);
    return 0;
}
