// The dispatch's XCD choice (a2a_order.h) against the general planner on the same workload: one threadblock per
// row copy, touching its source row and its destination row, unit bytes.
#include <cstdio>
#include <random>
#include <vector>

#include "a2a_order.h"
#include "nap_planner.h"

int main() {
    std::mt19937_64 rng(11);
    long long cases = 0, bad = 0;
    for (int it = 0; it < 400; ++it) {
        const int P = 1 + static_cast<int>(rng() % 64), T = static_cast<int>(rng() % 40);
        const int k = 1 + static_cast<int>(rng() % (it % 3 ? 8 : 64));
        const int64_t ntok = static_cast<int64_t>(P) * T;
        std::vector<uint64_t> mask(static_cast<size_t>(ntok));
        for (auto& m : mask) {
            const int n = it % 5 == 0 ? k : 1 + static_cast<int>(rng() % k);  // ties, and mixed sizes
            for (int j = 0; j < n; ++j) m |= uint64_t(1) << (rng() % P);
        }
        std::vector<int64_t> rows(static_cast<size_t>(P), 0), start(static_cast<size_t>(P) + 1, 0), next(rows);
        for (uint64_t m : mask)
            for (int d = 0; d < P; ++d) rows[static_cast<size_t>(d)] += m >> d & 1u;
        for (int d = 0; d < P; ++d) start[static_cast<size_t>(d) + 1] = start[static_cast<size_t>(d)] + rows[static_cast<size_t>(d)];
        std::vector<int64_t> off{0}, chunk, token;
        for (int64_t i = 0; i < ntok; ++i)
            for (int d = 0; d < P; ++d)
                if (mask[static_cast<size_t>(i)] >> d & 1u) {
                    chunk.push_back(i);
                    chunk.push_back(ntok + start[static_cast<size_t>(d)] + next[static_cast<size_t>(d)]++);
                    off.push_back(static_cast<int64_t>(chunk.size()));
                    token.push_back(i);
                }
        const std::vector<int64_t> unit(token.size(), 1);
        const nuna::NapPlan plan = nuna::nap_plan(nuna::nap_topology_mi355x(), nuna::kNumXcd,
                                                  static_cast<int64_t>(token.size()), off.data(), chunk.data(),
                                                  unit.data(), nullptr);
        std::vector<uint8_t> xcd(static_cast<size_t>(ntok));
        int64_t copies[nuna::kNumXcd], want[nuna::kNumXcd] = {};
        nuna::a2a_token_xcds(mask.data(), ntok, xcd.data(), copies);
        bad += static_cast<int64_t>(plan.groups.size()) != ntok;
        for (size_t c = 0; c < token.size(); ++c, ++cases) {
            // Group g is token g: the lists in group order are the lists in token order.
            bad += plan.tb_domain[c] != xcd[static_cast<size_t>(token[c])] || plan.tb_group[c] != token[c];
            ++want[plan.tb_domain[c]];
        }
        for (int x = 0; x < nuna::kNumXcd; ++x) bad += want[x] != copies[x];
    }
    std::printf("%lld copies, %lld mismatches\n", cases, bad);
    return bad != 0;
}
