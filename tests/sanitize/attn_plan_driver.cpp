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

// ---- whole plans: the cuts of 64-bit arithmetic, every tile once, every partial result merged ----
struct Round {
    sv::AttnPlanArgs a{};
    std::vector<int> q0, k, kv;
};

uint64_t unit_cost(int M, int nt) {
    if (M <= 0 || nt <= 0) return 0;
    return (M > 64 ? 144 : 100) + (uint64_t)nt * (M > 128 ? 32 : M > 64 ? 20 : 16);
}

int tiles_of(const Round& r, int i) {
    const int kv = std::min(r.kv[i], r.a.max_kv_len);
    const bool ok = r.k[i] >= 1 && r.k[i] <= r.a.block && r.q0[i] >= 0 && (long long)r.q0[i] + r.k[i] <= r.a.total_q;
    return ok && kv >= r.k[i] ? (kv + 63) / 64 : 0;
}

// the cuts by their definition: cut c at c equal parts of the line's cost (with the odd XCDs'
// parts 17/1024 shorter where the ranges are shared out evenly), moved onto a unit's end within
// two tiles of it; on a short line moved onto the start of a unit of fewer than 12 tiles
std::vector<sv::AttnRange> cuts_of(const Round& r) {
    const sv::AttnPlanArgs& a = r.a;
    uint64_t W = 0;
    std::vector<uint64_t> before;
    for (int i = 0; i < a.R; i++) {
        before.push_back(W);
        for (int rb = 0; rb < a.nrb; rb++) W += unit_cost(a.G * r.k[i] - rb * a.rb_rows, tiles_of(r, i));
    }
    const uint64_t step = std::max<uint64_t>((W + a.ranges - 1) / a.ranges, (100 + 6 * 16) / 2);
    const bool brief = step < 100 + 6 * 16;
    const int n = (int)((W + step - 1) / step);
    std::vector<sv::AttnRange> out(n + 1, sv::AttnRange{a.R, 0, 0, 0, 0, 0, 0, 0});
    for (int c = 0; c < n; c++) {
        uint64_t at = c * step;
        if (n % 8 == 0 && n * a.heads <= 256) {
            const int per = n / 8, x = c / per, part = c % per;
            at += (uint64_t)(x % 2 ? per - part : part) * (step * 17 / 1024);
        }
        if (at >= W) continue;
        int i = 0;
        while (i + 1 < a.R && before[i + 1] <= at) i++;
        uint64_t x = at - before[i];
        const int nt = tiles_of(r, i);
        int rb = 0;
        while (rb + 1 < a.nrb && x >= unit_cost(a.G * r.k[i] - rb * a.rb_rows, nt))
            x -= unit_cost(a.G * r.k[i] - rb++ * a.rb_rows, nt);
        const int M = a.G * r.k[i] - rb * a.rb_rows;
        const uint64_t start = M > 64 ? 144 : 100;
        int t = x > start ? (int)((x - start) / (M > 128 ? 32 : M > 64 ? 20 : 16)) : 0;
        if (t <= 2 || (brief && nt < 12)) t = 0;
        if (t >= nt || (t > 0 && nt - t <= 2)) t = 0, rb++;
        out[c] = sv::AttnRange{i, rb, t, r.q0[i], r.k[i], r.kv[i], 0, 0};
    }
    return out;
}

template <int NT>
void check_plan(Round& r) {
    sv::AttnPlanArgs& a = r.a;
    std::vector<sv::AttnRange> recs(a.ranges + 1);
    int32_t ctr[3] = {-7, -7, -7};
    a.recs = recs.data();
    a.ctr = ctr;
    std::vector<uint32_t> pre(a.R + 1), wsum(NT / 64);
    hosthip::run_workgroup(NT, [&] {
        sv::build_attn_plan<NT>(a, [&](int i, int& q0, int& k, int& kv) {
            q0 = r.q0[i];
            k = r.k[i];
            kv = r.kv[i];
        }, pre.data(), wsum.data());
    });
    const std::vector<sv::AttnRange> want = cuts_of(r);
    const int n = ctr[0];
    expect(n == (int)want.size() - 1 && n <= a.ranges && ctr[1] == 0 && ctr[2] == 0, "the counts of a plan");
    for (int c = 0; c <= n; c++)
        expect(recs[c].req == want[c].req && recs[c].block == want[c].block && recs[c].tile == want[c].tile &&
                   recs[c].q0 == want[c].q0 && recs[c].k == want[c].k && recs[c].kv == want[c].kv, "the cuts");
    // the walk: per unit, its pieces in order
    std::vector<int> next(a.R * a.nrb, 0);
    std::vector<int> cut_slot(2 * a.ranges, -1);  // the unit whose piece a partial result holds
    for (int c = 0; c < n; c++)
        sv::walk_range(a, recs[c], recs[c + 1], a.rb_rows, [&](int i, int& q0, int& k, int& kv) {
            q0 = r.q0[i];
            k = r.k[i];
            kv = r.kv[i];
        }, [&](int i, int row0, int q0, int k, int, int t0, int t1, int nt) {
            const int unit = i * a.nrb + row0 / a.rb_rows;
            expect(q0 == r.q0[i] && k == r.k[i] && nt == tiles_of(r, i), "a piece's request");
            expect(t0 == next[unit], "the tiles of a unit follow each other");
            next[unit] = t1;
            if (t1 - t0 == nt) return;
            const int slot = 2 * c + (t0 == 0);
            expect(cut_slot[slot] == -1, "one piece per partial result");
            cut_slot[slot] = unit;
        });
    for (int i = 0; i < a.R; i++)
        for (int rb = 0; rb < a.nrb; rb++)
            expect(next[i * a.nrb + rb] == (a.G * r.k[i] > rb * a.rb_rows ? tiles_of(r, i) : 0), "every tile once");
    // the merge: from the first cut inside a unit on, the piece that starts it and one per cut
    for (int c = 1; c < n; c++) {
        if (recs[c].tile <= 0) continue;
        const int unit = recs[c].req * a.nrb + recs[c].block;
        const bool first = recs[c - 1].tile <= 0 || recs[c - 1].req * a.nrb + recs[c - 1].block != unit;
        if (!first) continue;
        expect(cut_slot[2 * (c - 1) + 1] == unit, "the start of a cut unit");
        cut_slot[2 * (c - 1) + 1] = -1;
        for (int s = c; s < n && recs[s].req == recs[c].req && recs[s].block == recs[c].block; s++) {
            expect(cut_slot[2 * s] == unit, "the further pieces of a cut unit");
            cut_slot[2 * s] = -1;
        }
    }
    for (int slot : cut_slot) expect(slot == -1, "every partial result is merged");
}

void check_plans() {
    const int kHeads[] = {1, 2, 3, 4, 7, 8, 16, 24, 100, 200};
    for (int it = 0; it < 150; it++) {
        Round r;
        sv::AttnPlanArgs& a = r.a;
        a.heads = kHeads[below(10)];
        a.G = 1 << below(7);
        a.block = 1 + below(16);
        const bool wide = a.G * a.block > 128;
        a.rb_rows = wide ? 256 : 128;
        a.nrb = (a.G * a.block + a.rb_rows - 1) / a.rb_rows;
        const int most = std::max(1, 511 / (a.heads * a.nrb));
        a.R = it % 5 ? 1 + below(most) : most;
        a.max_kv_len = it % 7 == 0 ? 1 << 22 : 1 << (1 + below(18));
        int per_head = a.heads <= 256 ? 256 / a.heads : 0;
        if (per_head * a.heads * 10 < 256 * 9) per_head = (4 * 256 + a.heads - 1) / a.heads;
        a.ranges = (int)std::min<long long>(per_head, (long long)a.R * a.nrb * ((a.max_kv_len + 63) / 64));
        int q = 0;
        for (int i = 0; i < a.R; i++) {
            r.q0.push_back(q);
            r.k.push_back(1 + below(a.block));
            const int top = it % 3 ? a.max_kv_len : 1 << below(23);  // (longer contexts are cut to the longest)
            r.kv.push_back(it % 7 == 0 ? a.max_kv_len : r.k[i] + below(top));
            if (it % 11 == 0 && i % 3 == 1) r.k[i] = word(a.block) % 1000000;  // malformed
            if (it % 13 == 0 && i % 4 == 2) r.kv[i] = word(a.max_kv_len);
            q += std::max(0, std::min(r.k[i], a.block));
        }
        a.total_q = std::max(1, it % 17 ? q : q - 2);
        if (it % 25) check_plan<64>(r);
        else check_plan<512>(r);
    }
}

// ---- a run on the words of stdin: R block total_q max_kv_len G nrb heads ranges, qo, kv_lens, the
// count and the cuts; prints the number of pieces and of merged units ----
void check_run_on_words() {
    auto in = [] {
        int v = 0;
        expect(std::scanf("%d", &v) == 1, "a word on stdin");
        return v;
    };
    Shape a{};
    a.R = in();
    a.block = in();
    a.total_q = in();
    a.max_kv_len = in();
    a.G = in();
    a.nrb = in();
    const int heads = in();
    a.ranges = in();
    const int rb_rows = a.G * a.block > 128 ? 256 : 128;
    const int slot_rows = std::min(a.G * a.block, rb_rows);
    std::vector<int> qo(a.R + 1), kv(a.R);
    for (int& v : qo) v = in();
    for (int& v : kv) v = in();
    const int n = sv::plan_ranges(in(), a.ranges) * heads;
    std::vector<sv::AttnRange> recs(a.ranges + 1);
    for (auto& r : recs)
        for (int* w : {&r.req, &r.block, &r.tile, &r.q0, &r.k, &r.kv, &r.pad0, &r.pad1}) *w = in();
    std::vector<char> slots(2 * (size_t)a.ranges * heads * slot_rows);  // the rows of the partial results
    long pieces = 0;
    const bool one_pass = sv::plan_one_pass(n, 256);
    for (int index = 0; index < (one_pass ? 256 : n + 256); index++) {
        const int item = sv::plan_item(index, n, one_pass);
        if (item < 0) continue;
        const int rng = item / heads, h = item % heads;
        sv::walk_range(a, recs.at(rng), recs.at(rng + 1), rb_rows, [&](int i, int& q0, int& k, int& kv_len) {
            q0 = qo.at(i);
            k = qo.at(i + 1) - q0;
            kv_len = kv.at(i);
        }, [&](int i, int row0, int q0, int k, int kv_len, int t0, int t1, int nt) {
            pieces++;
            expect(i >= 0 && i < a.R && row0 >= 0 && row0 < a.G * k, "a piece's request and rows");
            expect(q0 >= 0 && k >= 1 && k <= a.block && (long long)q0 + k <= a.total_q, "rows of the batch");
            expect(kv_len >= k && kv_len <= a.max_kv_len && 0 <= t0 && t0 < t1 && t1 <= nt, "tiles");
            if (t1 - t0 == nt) return;
            const size_t slot = 2 * ((size_t)rng * heads + h) + (t0 == 0);
            for (int r = 0; r < std::min(a.G * k - row0, rb_rows); r++) slots.at(slot * slot_rows + r) = 1;
        });
    }
    std::printf("ok %ld\n", pieces);
}

}  // namespace

int main(int argc, char**) {
    if (argc > 1) {
        check_run_on_words();
        return 0;
    }
    check_ranges_of_words();
    check_item_counts();
    check_items_of_grids();
    check_walk_of_words();
    check_plans();
    std::printf("ok\n");
    return 0;
}
