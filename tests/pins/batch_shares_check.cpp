// Driver for the CPU check of split_work_shrinking
// (paper_2202_01753_amd/csrc/batch_plan.hpp): reads "<n> <each> <levels>", the
// shares and n lines "<m> <cost>"; prints a line "<item> <t0> <t1>" per piece and
// then one with every integral's first piece.
#include <cstdio>
#include <iostream>

#include "batch_plan.hpp"

int main() {
    int n, levels;
    long long each;
    std::cin >> n >> each >> levels;
    std::vector<double> shares(levels), cost(n);
    std::vector<int64_t> m(n);
    for (double &s : shares) std::cin >> s;
    for (int i = 0; i < n; ++i) std::cin >> m[i] >> cost[i];
    std::vector<mcubes::plan::Piece> out;
    std::vector<int32_t> first(n, -1);
    mcubes::plan::split_work_shrinking(m.data(), cost.data(), 0, n, shares.data(), levels, each, out, first.data());
    for (const auto &p : out) std::printf("%d %lld %lld\n", p.item, (long long)p.t0, (long long)p.t1);
    for (int i = 0; i < n; ++i) std::printf("%d ", first[i]);
    std::printf("\n");
}
