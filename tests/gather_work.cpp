// Replay of the gather kernels' work arrangement on the CPU, from the code that the kernels and their launches use
// (plan_gather, block_work, wave_work): every (batch item, head, query, sample part) has to be one wave's
// work, and no wave may get a batch item or head that does not exist. Built once as it is and once with each
// macro that arranges the work in another way. Prints "failures: 0" when every check holds.
#include <cstdio>
#include <vector>

#include "msda_internal.h"

namespace {

struct Case {
    const char* name;
    int N, M, D, elem, P;
    std::vector<int> hw;  // H, W per level
    int Lq;               // 0: as many queries as pixels
};

int failures = 0;

void check(const Case& c, int ppw, int k_split_max) {
    msda::Params p = {};
    p.n_batch = c.N;
    p.M = c.M;
    p.D = c.D;
    p.P = c.P;
    p.L = (int)c.hw.size() / 2;
    p.K = p.L * p.P;
    p.k_split_max = k_split_max;
    for (int l = 0; l < p.L; ++l) {
        p.H[l] = c.hw[2 * l];
        p.W[l] = c.hw[2 * l + 1];
        p.start[l] = p.S;
        p.S += p.H[l] * p.W[l];
    }
    p.Lq = c.Lq ? c.Lq : p.S;
    const msda::GatherLaunch g = msda::plan_gather(p, ppw, c.elem);
    // the query order and the head pairs do not depend on the arrangement
    const bool pairs = g.waves > 1 && c.M % 2 == 0 && c.D * c.elem == 64;
    const bool strips = g.waves > 1 && p.Lq == p.S && c.D * c.elem <= 128 && p.K >= 4;
    if ((p.head_group == 2) != pairs || (p.strips != 0) != strips) {
        ++failures;
        std::printf("%s: strips %d, head group %d\n", c.name, p.strips, p.head_group);
    }
    std::vector<int> times((size_t)c.N * c.M * p.Lq * p.k_split, 0);
    int64_t outside = 0, wrong = 0;
    for (int b = 0; b < g.grid; ++b) {
        int slab, chunk;
        if (!msda::block_work(p, (uint32_t)b, (uint32_t)g.grid, slab, chunk)) continue;
        for (int w = 0; w < g.waves; ++w) {
            const msda::Tile t = msda::wave_work(p, ppw, slab, chunk, w);
            if (t.n < 0 || t.n >= c.N || t.m < 0 || t.m >= c.M || t.q0 < 0 || t.part < 0 || t.part >= p.k_split) {
                ++outside;
                continue;
            }
            for (int q = t.q0; q < t.q0 + ppw && q < p.Lq; ++q)
                ++times[(((size_t)t.n * c.M + t.m) * p.Lq + q) * p.k_split + t.part];
        }
    }
    for (int x : times) wrong += x != 1;
    if (outside || wrong) {
        ++failures;
        std::printf("%s: %lld waves outside, %lld pieces of work not done once\n", c.name, (long long)outside,
                    (long long)wrong);
    }
}

}  // namespace

int main() {
    const std::vector<Case> cases = {
        {"pairs, one batch item", 1, 8, 32, 2, 4, {160, 160, 80, 80, 40, 40}, 0},
        {"pairs, odd batch", 3, 8, 32, 2, 4, {120, 120}, 0},
        {"pairs, cross-attention", 3, 6, 16, 4, 4, {100, 100, 50, 50}, 4500},
        {"odd heads", 2, 5, 32, 2, 3, {90, 70, 45, 35}, 0},
        {"long rows", 2, 5, 36, 4, 3, {90, 70, 45, 35}, 0},
        {"few samples", 2, 8, 32, 4, 3, {150, 90}, 0},
        {"wide rows", 2, 8, 32, 4, 4, {100, 150, 50, 75, 25, 38, 13, 19}, 0},
        {"cross-attention", 2, 8, 32, 4, 8, {116, 200, 58, 100}, 10000},
        {"decoder", 2, 8, 32, 4, 4, {100, 150, 50, 75, 25, 38, 13, 19}, 300},
        {"small", 1, 2, 32, 2, 4, {9, 7, 3, 2}, 0},
        {"one query", 1, 1, 64, 4, 1, {3, 3}, 1},
    };
    for (const Case& c : cases)
        for (int ppw : {1, 4, 8, 16, 64})
            for (int ks : {1, 8}) check(c, ppw, ks);
    std::printf("failures: %d\n", failures);
    return failures != 0;
}
