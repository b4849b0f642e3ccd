// Prints the plan of a down-sampling block's paired launch, kind and variant, for every "h cin n cus" on standard input
// (bf16, weights in fragment order too).
#include <cstdio>

#include "internal.h"

int main()
{
    int h, cin, n, cus;
    while (scanf("%d %d %d %d", &h, &cin, &n, &cus) == 4) {
        const sgprs_conv_desc_t d0 = {n, h, h, cin, 2 * cin, 3, 3, 2, 1, SGPRS_BF16, 1}, d1 = {n, h, h, cin, 2 * cin, 1, 1, 2, 0, SGPRS_BF16, 0};
        const sgprs::ConvPlan p = sgprs::plan_conv_pair(d0, d1, cus, true);
        printf("%d %d\n", p.kind, p.variant);
    }
    return 0;
}
