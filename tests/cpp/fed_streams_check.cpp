// FedStreams: one stream from the start, two in turn, bursts, work on several at once.
// Prints "ok" or the first failure.
#include <cstdio>

#include "fed_streams.h"

static const int a = 0, b = 0;
#define CHECK(c) do { if (!(c)) { printf("FAIL line %d: %s\n", __LINE__, #c); return 1; } } while (0)

int main()
{
    constexpr int K = sgprs::FedStreams::kRuns;
    {   // one stream, from the first launch on
        sgprs::FedStreams f;
        for (int i = 0; i < 100; ++i) CHECK(f.only(&a));
    }
    {   // two in turn: the first launch cannot know, all others do
        sgprs::FedStreams f;
        CHECK(f.only(&a));
        for (int i = 0; i < 100; ++i) {
            CHECK(!f.only(&b));
            CHECK(!f.only(&a));
        }
        // from then on one of them: after kRuns launches the other is forgotten
        for (int i = 0; i < K - 1; ++i) CHECK(!f.only(&a));
        for (int i = 0; i < 100; ++i) CHECK(f.only(&a));
    }
    {   // bursts of kRuns launches never look like one stream
        sgprs::FedStreams f;
        for (int i = 0; i < K; ++i) CHECK(f.only(&a));
        for (int k = 0; k < 10; ++k) {
            for (int i = 0; i < K; ++i) CHECK(!f.only(&b));
            for (int i = 0; i < K; ++i) CHECK(!f.only(&a));
        }
    }
    {   // a task spread over several streams, between launches on one
        sgprs::FedStreams f;
        CHECK(f.only(&a));
        CHECK(!f.only(nullptr));
        CHECK(!f.only(&a));
    }
    {
        sgprs::FedStreams f;
        CHECK(!f.only(nullptr));
        CHECK(!f.only(&a));
    }
    printf("ok\n");
    return 0;
}
