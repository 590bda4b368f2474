// One line per call on stdin (rule and its arguments): the rule's answer.
#include <stdio.h>
#include <string.h>
#include "rules.h"

int main() {
    char rule[32];
    long long a, b, c, d, e;
    while (scanf("%31s %lld %lld %lld %lld %lld", rule, &a, &b, &c, &d, &e) == 6) {
        if (!strcmp(rule, "quantize_wide")) printf("%d\n", (int)quantize_wide(a, (int)b, (int)c, (int)d, e != 0));
        else if (!strcmp(rule, "calib_threads")) printf("%d\n", calib_threads((int)a));
        else if (!strcmp(rule, "pilot_for_results")) printf("%lld\n", (long long)pilot_for_results(a, (int)b, (int)c));
        else if (!strcmp(rule, "ivf_shared_pays")) printf("%d\n", (int)ivf_shared_pays(a, b));
        else if (!strcmp(rule, "scan_blocks_most")) printf("%d\n", scan_blocks_most((int)a, b, c != 0));
        else return 1;
    }
    return 0;
}
