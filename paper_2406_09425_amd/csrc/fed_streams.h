// Does a thread feed one stream or several?  Host logic without HIP, so that it can be checked without a GPU.
#pragma once

namespace sgprs {

// One per thread.  It steers how work is launched, never what is computed: a stream that was destroyed
// and whose handle is used again costs at most a few launches of the slower kind.
class FedStreams {
public:
    static constexpr int kRuns = 8;  // as many as a turn of the static executor
    // The thread launches work on `stream` (NULL: on several at once).  True unless one of its last kRuns
    // launches went elsewhere; a thread's first stream is not a change.
    bool only(const void* stream)
    {
        if (stream && (stream == last_ || !last_)) {
            if (since_ < kRuns) ++since_;
        } else {
            since_ = 0;
        }
        if (stream) last_ = stream;
        return since_ >= kRuns;
    }

private:
    const void* last_ = nullptr;
    int since_ = kRuns;  // launches since the last change
};

}  // namespace sgprs
