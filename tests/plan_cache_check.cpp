// Counts what csrc/plan_cache.h plans: every pass of a descriptor once, when it is first asked for, as long as the descriptor is remembered.
#include <stdio.h>
#include "plan_cache.h"

struct Plans { int K, pass[3]; };
static mcn::PlanCache<Plans, 8> cache;            // all zero is empty
static int begun, made[3];

static Plans *ask(int K, int pass) {
    mcn_conv_desc d;
    memset(&d, 0, sizeof d);
    d.K = K;
    Plans *p = cache.get(d, pass, [&](Plans &q) { ++begun; if (q.K | q.pass[0] | q.pass[1] | q.pass[2]) puts("another layer's plans"), ++begun; q.K = K; }, [&](Plans &q, int s) { ++made[s]; ++q.pass[s]; });
    if (p->K != K || p->pass[pass] != 1) { printf("layer %d, pass %d: plans of layer %d, made %d times\n", K, pass, p->K, p->pass[pass]); return nullptr; }
    return p;
}
static bool counts(const char *what, int b, int m0, int m1, int m2) {
    const bool ok = begun == b && made[0] == m0 && made[1] == m1 && made[2] == m2;
    if (!ok) printf("%s: %d begun, %d %d %d planned, not %d, %d %d %d\n", what, begun, made[0], made[1], made[2], b, m0, m1, m2);
    return ok;
}

int main() {
    bool ok = true;
    for (int round = 0; round < 5; ++round)
        for (int k = 1; k <= 8; ++k) ok &= ask(k, 0) != nullptr;
    ok &= counts("eight layers in turn, one pass", 8, 8, 0, 0);
    for (int k = 8; k >= 1; --k) ok &= ask(k, 2) != nullptr && ask(k, 1) != nullptr;
    ok &= counts("the other passes, in reverse", 8, 8, 8, 8);
    ok &= ask(9, 1) != nullptr;                   // in the place of layer 1, asked for first
    for (int k = 2; k <= 8; ++k) ok &= ask(k, 0) != nullptr;
    ok &= counts("a ninth layer", 9, 8, 9, 8);
    ok &= ask(1, 0) != nullptr && ask(9, 1) != nullptr && ask(3, 2) != nullptr;      // layer 1 in the place of layer 2
    ok &= counts("the first again", 10, 9, 9, 8);
    ok &= ask(2, 0) != nullptr;
    ok &= counts("the second again", 11, 10, 9, 8);
    Plans *p = ask(5, 0);
    ok &= p && ask(5, 1) == p && ask(5, 2) == p;       // one place for all passes
    puts(ok ? "OK" : "FAILED");
    return !ok;
}
