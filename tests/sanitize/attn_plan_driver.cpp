// Drives the device code that divides the verify attention's work (csrc/rows.h, attn_plan.h) on
// the host, under AddressSanitizer and UndefinedBehaviorSanitizer without recovery: what a run
// reads from a workspace that holds no plan is arbitrary, and no arithmetic on it may wrap past a
// check.
#include <climits>
#include <cstdio>
#include <cstdlib>

#include "attn_plan.h"

namespace {

uint64_t g_state = 0x9E3779B97F4A7C15ull;
uint64_t next_u64() {  // splitmix64
    uint64_t z = (g_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
int below(int n) { return (int)(next_u64() % (uint64_t)n); }

void expect(bool ok, const char* what) {
    if (!ok) {
        std::fprintf(stderr, "FAILED: %s\n", what);
        std::exit(2);
    }
}

const int kWords[] = {INT_MIN, INT_MIN + 1, -65536, -16, -1, 0, 1, 2, 3, 15, 16, 17, 63, 64, 65, 1000, 65536,
                      1 << 22, INT_MAX - 16, INT_MAX - 1, INT_MAX};
constexpr int kNumWords = sizeof(kWords) / sizeof(kWords[0]);

// a word as garbage or a stale plan may hold it
int word(int near) {
    switch (below(16)) {
        case 0: return kWords[below(kNumWords)];
        case 1: return (int)(uint32_t)next_u64();
        default: return below(2 * near + 2) - 1;
    }
}

// ---- the row and length checks at every extreme, against 64-bit arithmetic ----
void check_ranges_of_words() {
    for (int q0 : kWords)
        for (int k : kWords)
            for (int total : kWords)
                for (int block : {1, 5, 16}) {
                    const bool in = k >= 1 && k <= block && q0 >= 0 && (long long)q0 + k <= total;
                    if (total < 0) continue;
                    expect(sv::rows_in_batch(q0, k, block, total) == in, "rows_in_batch");
                    for (int kv : kWords)
                        for (int cap : {1, 64, 65, 1 << 22}) {
                            const long long n = kv > cap ? cap : kv;
                            const long long want = in && n >= k ? (n + 63) / 64 : 0;
                            expect(sv::plan_tiles(block, total, cap, q0, k, kv) == want, "plan_tiles");
                        }
                }
}

// ---- the number of items of any stored count: within the items of the longest plan ----
void check_item_counts() {
    for (int it = 0; it < 100000; it++) {
        const int heads = 1 + below(511), most = 1 + below(0x7FFFFFF0 / heads);
        const int stored = word(most < 1 << 20 ? most : 1 << 20);
        const int n = sv::plan_ranges(stored, most) * heads;
        expect(n >= 0 && n <= most * heads, "item count");
        if (stored >= 0 && stored <= most) expect(n == stored * heads, "a built plan keeps its count");
    }
}

// ---- every item is taken by exactly one workgroup, whatever the grid ----
void check_items_of_grids() {
    for (int grid = 1; grid <= 320; grid++)
        for (int n = 0; n <= 2 * grid + 9; n++) {
            const bool one_pass = sv::plan_one_pass(n, grid);
            std::vector<int> seen(n, 0);
            // without one pass, the claims follow the workgroups' own indices without a gap
            for (int index = 0; index < (one_pass ? grid : n + grid); index++) {
                const int item = sv::plan_item(index, n, one_pass);
                expect(item >= -1 && item < n, "an existing item");
                if (item >= 0) seen[item]++;
            }
            for (int i = 0; i < n; i++) expect(seen[i] == 1, "each item once");
        }
    for (int w : kWords)
        for (int n : {0, 1, 255, 256, 257, 0x7FFFFFF0})
            for (bool one_pass : {false, true}) {
                const int item = sv::plan_item(w, n, one_pass && sv::plan_one_pass(n, 256));
                expect(item >= -1 && item < n, "an existing item for any claim");
            }
    expect(sv::plan_one_pass(256, 256) && !sv::plan_one_pass(0x7FFFFFF0, 256), "one pass");
}

struct Shape {
    int R, block, total_q, max_kv_len, G, nrb, ranges;
};

// ---- the walk between cuts of arbitrary words: existing rows and tiles only ----
void check_walk_of_words() {
    long pieces = 0;
    for (int it = 0; it < 200000; it++) {
        Shape a{};
        a.R = 1 + below(6);
        a.block = 1 + below(16);
        a.total_q = 1 + below(a.R * a.block);
        a.max_kv_len = it % 2 ? 1 + below(300) : 1 << below(23);
        a.G = 1 + below(16);
        const int rb_rows = a.G * a.block > 128 ? 256 : 128;
        a.nrb = (a.G * a.block + rb_rows - 1) / rb_rows;
        a.ranges = 1 + below(3);
        const int tiles = (a.max_kv_len + 63) / 64;
        auto cut = [&] {
            return sv::AttnRange{word(a.R), word(a.nrb), word(tiles), word(a.total_q), word(a.block),
                                 word(a.max_kv_len), word(1), word(1)};
        };
        const sv::AttnRange r0 = cut(), r1 = cut();
        const int q_of = word(a.total_q), k_of = word(a.block), kv_of = word(a.max_kv_len);
        int calls = 0;
        sv::walk_range(a, r0, r1, rb_rows, [&](int i, int& q0, int& k_i, int& kv) {
            expect(i >= 0 && i < a.R, "request");
            q0 = q_of;
            k_i = k_of;
            kv = kv_of;
        }, [&](int i, int row0, int q0, int k_i, int kv, int t0, int t1, int nt) {
            calls++;
            pieces++;
            expect(i >= 0 && i < a.R, "request of a piece");
            expect(k_i >= 1 && k_i <= a.block && q0 >= 0 && (long long)q0 + k_i <= a.total_q, "rows");
            expect(row0 >= 0 && row0 % rb_rows == 0 && row0 < a.G * k_i, "first row");
            expect(kv >= k_i && kv <= a.max_kv_len && nt == (kv + 63) / 64, "keys");
            expect(t0 >= 0 && t0 < t1 && t1 <= nt, "tiles");
        });
        expect(calls <= a.R * a.nrb, "number of pieces");
    }
    expect(pieces > 10000, "the words gave pieces");
}

}  // namespace

int main() {
    check_ranges_of_words();
    check_item_counts();
    check_items_of_grids();
    check_walk_of_words();
    std::printf("ok\n");
    return 0;
}
