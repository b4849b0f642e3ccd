// tap_mask against its definition: every window position from far before the image to far past it,
// for image sizes 1..70 and filters of 1 and 3 taps; the mask may hold no bit beyond the filter.
// Prints "ok <cases>" or the first failure.
#include <cstdio>
#include <initializer_list>

#include "tap_mask.h"

int main()
{
    long cases = 0;
    for (int taps : {1, 3})
        for (int size = 1; size <= 70; ++size)
            for (int first = -150; first <= 220; ++first) {
                unsigned want = 0;
                for (int t = 0; t < taps; ++t)
                    if (first + t >= 0 && first + t < size) want |= 1u << t;
                const unsigned got = sgprs::tap_mask(first, size, taps);
                if (got != want) {
                    printf("FAIL taps %d size %d first %d: %#x, expected %#x\n", taps, size, first, got, want);
                    return 1;
                }
                ++cases;
            }
    printf("ok %ld\n", cases);
    return 0;
}
