// The plans of the descriptors asked for last.  Plain C++ (tests/plan_cache_check.cpp counts what is planned).
#pragma once
#include <string.h>
#include <type_traits>
#include "../../include/mcnconv.h"

namespace mcn {

// N descriptors, first in first out; the plan of a pass is made when that pass is first asked for.  Planning takes 5 to 400 us a pass,
// as long as many a kernel: a call must not wait for the plans of another pass.  All zero is empty, so that a thread's own one needs no constructor.
template <class Plans, int N>
struct PlanCache {
    static_assert(std::is_trivially_copyable<Plans>::value, "plans are plain values");
    struct Slot {
        mcn_conv_desc d;
        unsigned made;             // bit p: pass p is planned
        Plans plans;
    };
    Slot slots[N];
    int used, last, oldest;

    // begin(plans): of a descriptor that is not remembered, all zero (nothing of the one whose place it takes); make(plans, pass): a
    // pass that is not planned yet
    template <class Begin, class Make>
    Plans *get(const mcn_conv_desc &d, int pass, Begin begin, Make make) {
        int at = -1;
        for (int i = 0, j = last; i < used; ++i, j = j + 1 < used ? j + 1 : 0)       // the same one again or, in a network, the next
            if (memcmp(&slots[j].d, &d, sizeof(d)) == 0) { at = j; break; }
        if (at < 0) {
            if (used < N) at = used++;
            else { at = oldest; oldest = oldest + 1 < N ? oldest + 1 : 0; }
            slots[at].d = d;
            slots[at].made = 0;
            memset(&slots[at].plans, 0, sizeof(Plans));
            begin(slots[at].plans);
        }
        last = at;
        Slot &s = slots[at];
        if (!(s.made >> pass & 1)) {
            make(s.plans, pass);
            s.made |= 1u << pass;
        }
        return &s.plans;
    }
};

}  // namespace mcn
