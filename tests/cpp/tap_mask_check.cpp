// tap_mask against its definition: every window position from far before the image to far past it,
// for image sizes 1..70; the bits of a filter of up to 15 taps are exact, and no bit reaches the next mask.
// Prints "ok <cases>" or the first failure.
#include <cstdio>

#include "tap_mask.h"

int main()
{
    long cases = 0;
    for (int size = 1; size <= 70; ++size)
        for (int first = -150; first <= 220; ++first) {
            const unsigned got = sgprs::tap_mask(first, size);
            unsigned want = 0;
            for (int t = 0; t < sgprs::kTapMaskBits - 1; ++t) {
                const bool in = first + t >= 0 && first + t < size;
                if (in) want |= 1u << t;
            }
            if (got != want) {
                printf("FAIL size %d first %d: %#x, expected %#x\n", size, first, got, want);
                return 1;
            }
            ++cases;
        }
    printf("ok %ld\n", cases);
    return 0;
}
