// Host check of the launch rules: where the lane-quad plane kernel is taken.  Prints the
// number of failed checks.
#include <cstdio>

#include "../paper_1601_07378_amd/csrc/kernels.hpp"
#include "../paper_1601_07378_amd/csrc/plan.hpp"

using namespace vloc;

// The automatic FP64 plan of a sphere that reaches the fraction f of every axis.
static bool setup(const int (&n)[3], double f, Geometry &g, LaneQuads &lq, HostPlan &h)
{
    const double two_pi = 6.283185307179586, R = f * n[0], k[3] = {0, 0, 0};
    const double cell[9] = {two_pi, 0, 0, 0, two_pi * n[1] / n[0], 0, 0, 0, two_pi * n[2] / n[0]};
    const int32_t grid[3] = {n[0], n[1], n[2]};
    std::string err;
    if (build_host_plan(h, grid, cell, 0.5 * R * R, k, nullptr, err) != VLOC_OK) return false;
    g = Geometry{};
    g.N1 = n[0];
    g.N2 = n[1];
    g.N3 = n[2];
    g.L1x = h.sx.L1;
    g.L2x = h.sx.L2;
    g.L1y = h.sy.L1;
    g.L2y = h.sy.L2;
    g.full = h.plane_full;
    lq = LaneQuads{};
    lq.q = n[0] / 4;
    lq.cus = 256;
    lq.planes = 1;
    lq.nxo = h.nxo;
    lq.cls = f >= 0.19 && f <= 0.32;
    return true;
}

int main()
{
    int bad = 0;
    // shapes that lose on lane quads, and shapes that gain (times in kernels.hpp)
    const struct {
        int n[3];
        double f;
        bool pays, dens;
    } shapes[] = {
        {{80, 80, 80}, 0.4, false, false},    {{96, 72, 96}, 0.4, false, false},
        {{96, 80, 96}, 0.4, false, false},    {{108, 90, 64}, 0.4, false, false},
        {{100, 36, 100}, 0.4, false, false},  {{64, 64, 64}, 0.4, false, true},
        {{128, 64, 128}, 0.4, false, true},   {{100, 100, 100}, 0.4, false, true},
        {{96, 72, 96}, 0.12, false, true},    {{108, 90, 64}, 0.12, false, true},
        {{108, 108, 64}, 0.12, false, true},  {{120, 80, 64}, 0.12, false, true},
        {{120, 80, 64}, 0.25, false, false},  {{32, 32, 32}, 0.4, true, true},
        {{48, 48, 48}, 0.4, true, true},      {{72, 135, 64}, 0.4, true, true},
        {{64, 150, 64}, 0.4, true, true},     {{32, 64, 64}, 0.12, true, true},
        {{80, 80, 80}, 0.12, true, true},     {{96, 32, 64}, 0.12, true, true},
        {{128, 128, 16}, 0.12, true, true},   {{64, 64, 64}, 0.25, true, true},
        {{80, 80, 80}, 0.25, true, true},     {{96, 96, 96}, 0.25, true, true},
        {{128, 128, 128}, 0.25, true, true},  {{60, 60, 100}, 0.25, true, true},
        {{120, 120, 64}, 0.12, true, true},   {{128, 72, 128}, 0.25, true, true},
        {{128, 18, 64}, 0.4, true, true},
    };
    for (const auto &s : shapes) {
        Geometry g;
        LaneQuads lq;
        HostPlan h;
        if (!setup(s.n, s.f, g, lq, h) ||
            lq_pays(g, lq, s.f * s.n[0], MODE_APPLY) != s.pays ||
            lq_pays(g, lq, s.f * s.n[0], MODE_DENSITY) != s.dens) {
            std::printf("lq_pays %d x %d x %d reach %.2f\n", s.n[0], s.n[1], s.n[2], s.f);
            ++bad;
        }
    }
    std::printf("%d failed\n", bad);
    return bad != 0;
}
