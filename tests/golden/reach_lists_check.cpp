// Checks the sphere lists of ckv_reach (host builder) against brute force: for random
// ground points and every level, a point inside the level's grid finds in its cell's list,
// ascending and padded, every sphere whose centre is within the level's radius, and a point
// outside has none within it.  The lookup is the step setup's.  Prints the number of
// (point, level) pairs and exits 0, or names the first miss and exits 1.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "ckv_tables.cpp"

namespace ckv {
void set_error(const std::string&) {}
}

int main(int argc, char** argv)
{
    const int n = std::atoi(argv[1]);
    const double half = std::atof(argv[2]), cx = std::atof(argv[3]);
    std::mt19937_64 g(5);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    ckv_array arr;
    arr.n_tel = n;
    for (int k = 0; k < n; ++k) {
        arr.x.push_back(cx + half * u(g));
        arr.y.push_back(half * u(g));
    }
    ckv_reach r;
    std::vector<uint32_t> data;
    ckv::build_reach(&arr, &r, &data);
    if (n <= ckv::kReachMinTel || !(2.0 * half < 1e6)) {
        if (!data.empty()) return 1;
        std::puts("0");
        return 0;
    }
    const ReachLevel* lev = reinterpret_cast<const ReachLevel*>(data.data());
    const uint32_t* rec = data.data() + r.rec_at;
    const uint16_t* list = reinterpret_cast<const uint16_t*>(data.data() + r.list_at);
    const size_t entries = 2 * (data.size() - r.list_at);
    if (r.levels < ckv::kReachLevels && ckv::kReachMin * std::pow(2.0, 0.5 * (r.levels - 1)) < 0.4 * half)
        return std::puts("too few levels"), 1;
    long pairs = 0;
    for (int q = 0; q < 4000; ++q) {
        const double spread = std::pow(10.0, 1.5 * u(g)) * (half + 100.0);
        const double X = cx + spread * u(g), Y = spread * u(g);
        for (int l = 0; l < r.levels; ++l) {
            const double radius = ckv::kReachMin * std::pow(2.0, 0.5 * l);
            const ReachLevel& v = lev[l];
            const double fx = (X - v.x0) * (double)v.inv_cell, fy = (Y - v.y0) * (double)v.inv_cell;
            const bool in = fx >= 0.0 && fy >= 0.0 && fx < (double)v.nx && fy < (double)v.ny;
            uint32_t at = 0, cnt = 0;
            if (in) {
                const uint32_t c = v.rec + (uint32_t)((int)fx * v.ny + (int)fy);
                if (r.rec_at + 2 * (size_t)c + 2 > r.list_at) return std::puts("record out of range"), 1;
                at = rec[2 * c];
                cnt = rec[2 * c + 1];
                const uint32_t end = at + (cnt + ckv::kReachPad - 1) / ckv::kReachPad * ckv::kReachPad;
                if (at % ckv::kReachPad || end > entries) return std::puts("list out of range"), 1;
                for (uint32_t i = at; i < end; ++i) {
                    const bool ok = i >= at + cnt ? list[i] == 0xFFFF
                                                  : list[i] < n && (i == at || list[i] > list[i - 1]);
                    if (!ok) return std::printf("bad entry, level %d\n", l), 1;
                }
            }
            for (int k = 0; k < n; ++k) {
                if (std::hypot(arr.x[k] - X, arr.y[k] - Y) > radius) continue;
                bool found = false;
                for (uint32_t i = at; i < at + cnt && !found; ++i) found = list[i] == k;
                if (!found) return std::printf("sphere %d missing: level %d, point %.3f %.3f\n", k, l, X, Y), 1;
            }
            ++pairs;
        }
    }
    std::printf("%ld\n", pairs);
    return 0;
}
