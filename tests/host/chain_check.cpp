// Host check of the step machines' rotating counters (cm_steps.h), built with
// hipcc as host code and run by tests/test_chain.py: a workgroup that looks at
// the counters late -- at any point of the steps that workgroup 0 runs before
// it waits for the others -- sees what the early ones saw; how often a chain
// looks at its time slice.
#include <cstdio>

#include "../../paper_1612_09368_amd/csrc/cm_steps.h"

using namespace cm;

static int fails = 0;
#define CHECK(c)                                             \
    do {                                                     \
        if (!(c)) {                                          \
            std::printf("FAIL line %d: %s\n", __LINE__, #c); \
            ++fails;                                         \
        }                                                    \
    } while (0)

int main() {
    for (int32_t r = 0; r < 12; ++r) {
        // the three slots of a step differ, and what it pushes the next reads
        CHECK(slot_read(r) != slot_push(r) && slot_push(r) != slot_clear(r) && slot_clear(r) != slot_read(r));
        CHECK(slot_push(r) == slot_read(r + 1));
        CHECK(slot_clear(r) == slot_push(r + 1));
        // tails as the barrier before step r left them: items for step r, the
        // slot it pushes to empty, the last step's own slot still full
        for (int links = 0; links <= CHAIN_FREE; ++links) {
            int tail[3];
            tail[slot_read(r)] = 5;
            tail[slot_push(r)] = 0;
            tail[slot_clear(r)] = 7;
            const int seen = tail[slot_read(r)];
            for (int32_t l = r; l < r + links; ++l) {
                CHECK(tail[slot_push(l)] == 0);  // cleared before it is pushed to
                tail[slot_clear(l)] = 0;
                CHECK(tail[slot_read(r)] == seen);
                for (int p = 1; p <= 4; ++p) {
                    tail[slot_push(l)] = p;
                    CHECK(tail[slot_read(r)] == seen);  // a look between any two of its writes
                }
            }
        }
    }
    // the slice: every 16 steps for the default bounds and for tuned ones, after
    // each step where a bound lets one step walk for milliseconds
    CHECK(slice_mask(2048, 128, 16384) == 15 && slice_mask(8192, 1024, 1 << 18) == 15);
    CHECK(slice_mask(0x7fffffff, 128, 16384) == 0);
    CHECK(slice_mask(2048, 0x7fffffff, 16384) == 0);
    CHECK(slice_mask(2048, 128, 0x7fffffff) == 0);
    std::printf(fails ? "chain: %d failures\n" : "chain: ok\n", fails);
    return fails ? 1 : 0;
}
