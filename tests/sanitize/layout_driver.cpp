// Checks the layouts that build_layout makes, on the CPU: every node that is not solid
// lies in exactly one tile of the step's list and of the read pass' list, no part of
// the arena overlaps the next, the total stays within lbm_footprint, and the layout
// is the one that the rules state.  Built host-only with sanitizers by
// tests/test_layout_rules.py; no device call is made.
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/lbm.h"
#include "../../paper_2512_01032_amd/csrc/lattice_host.hpp"

using namespace pflbm;

static int bad = 0;
#define CHECK(c, ...) do { if (!(c)) { bad = 1; printf("FAILED %s: ", #c); printf(__VA_ARGS__); printf("\n"); } } while (0)

static lbm_params params(int nx, int ny, int nz, int storage) {
    lbm_params p;
    memset(&p, 0, sizeof(p));
    p.nx = nx; p.ny = ny; p.nz = nz; p.storage = storage;
    p.rho_l = 1.0; p.rho_g = 0.001; p.nu_l = 0.01; p.nu_g = 0.1; p.sigma = 1e-3; p.W = 4.0; p.M = 1.0 / 6.0;
    p.eps = 1e-10; p.P_ref = 1.0 / 3.0; p.q_phase = 7; p.hyst_beta = 0.95;
    return p;
}

// walls: 0 none, 1 the layers y = 0 and z = 0, 2 a random third of the nodes,
// 3 all but a column of 3 x 3 nodes
static void check(const char* name, lbm_params p, int walls, int want_fused, int want_back) {
    const int64_t N = (int64_t)p.nx * p.ny * p.nz;
    std::vector<uint8_t> solid(N, 0);
    uint64_t r = 12345;
    for (int64_t n = 0; n < N; ++n) {
        const int64_t x = n % p.nx, y = n / p.nx % p.ny, z = n / ((int64_t)p.nx * p.ny);
        r = r * 6364136223846793005ull + 1442695040888963407ull;
        if (walls == 1) solid[n] = y == 0 || z == 0;
        if (walls == 2) solid[n] = (r >> 33) % 3 == 0;
        if (walls == 3) solid[n] = !(x >= 5 && x < 8 && y >= 5 && y < 8);
    }
    lbm_geometry g;
    memset(&g, 0, sizeof(g));
    for (int k = 0; k < 16; ++k) g.theta_deg[k] = 90.0;
    g.solid = walls ? solid.data() : nullptr;
    for (int fused = 0; fused < 2; ++fused) {
        LatticeLayout L;
        const int rc = build_layout(&p, &g, 0, fused != 0, &L);
        CHECK(rc == LBM_OK, "%s rc %d", name, rc);
        if (rc != LBM_OK) return;
        if (fused) {
            CHECK((int)L.fused == want_fused, "%s fused %d", name, (int)L.fused);
            CHECK((int)L.back == want_back, "%s back %d", name, (int)L.back);
        } else {
            CHECK(!L.fused && !L.back && L.rtiles.empty(), "%s", name);
        }
        CHECK(L.total <= footprint_bytes(&p), "%s %zu > %zu", name, L.total, footprint_bytes(&p));
        CHECK(L.rtiles.empty() == !L.back, "%s", name);
        for (const auto* list : {&L.tiles, &L.rtiles}) {
            if (list->empty()) continue;
            std::vector<uint8_t> seen(N, 0);
            for (size_t k = 0; k < list->size(); ++k) {
                const Tile& t = (*list)[k];
                CHECK(t.tile_in_lat == (int)k, "%s tile %zu", name, k);
                CHECK(t.z0 >= 0 && t.zn >= 1 && t.z0 + t.zn <= p.nz && t.x0 % L.tx == 0 && t.y0 % L.ty == 0, "%s tile %zu", name, k);
                for (int z = t.z0; z < t.z0 + t.zn; ++z)
                    for (int y = t.y0; y < std::min(p.ny, t.y0 + L.ty); ++y)
                        for (int x = t.x0; x < std::min(p.nx, t.x0 + L.tx); ++x) ++seen[x + (int64_t)p.nx * (y + (int64_t)p.ny * z)];
            }
            int64_t wrong = 0;
            for (int64_t n = 0; n < N; ++n) wrong += solid[n] ? seen[n] > 1 : seen[n] != 1;
            CHECK(wrong == 0, "%s %lld nodes", name, (long long)wrong);
        }
        // arena: the parts in order, each before the next
        std::vector<size_t> o = {L.off_desc, L.off_pop0};
        if (L.fused) {
            if (L.off_pop1 != L.off_pop0) o.push_back(L.off_pop1);
            for (size_t v : {L.off_h0, L.off_h1, L.off_flag, L.off_link, L.off_tiles, L.off_rtiles, L.off_partials, L.off_wrefs, L.off_wslot, L.off_hyst})
                o.push_back(v);
            CHECK(L.off_h1 - L.off_h0 >= L.h_bytes && L.off_flag - L.off_h1 >= L.h_bytes, "%s h", name);
            CHECK(L.off_partials - L.off_rtiles >= L.rtiles.size() * sizeof(Tile), "%s rtiles", name);
            CHECK(L.off_wslot - L.off_wrefs >= L.walls.size() * sizeof(WallRef), "%s walls", name);
            // phi and the near-wall sums of a read pass fit an h buffer
            int sh, sg, sphi;
            storage_sizes(p.storage, &sh, &sg, &sphi);
            CHECK(!L.back || L.h_bytes >= (size_t)((N + 3) / 4 * 4 + (L.n_wall ? 4 * N : 0)) * sphi, "%s read pass", name);
            CHECK(L.tiles.size() >= L.rtiles.size(), "%s partials", name);
        }
        o.push_back(L.total);
        CHECK(std::is_sorted(o.begin(), o.end()), "%s offsets", name);
        CHECK(L.wmat.size() == (L.fused ? 0 : 3 * (size_t)L.n_wall), "%s", name);
        CHECK((int64_t)L.walls.size() == (L.fused && !L.back ? 0 : L.n_wall), "%s", name);
        std::vector<uint8_t> slot(L.n_wall, 0);
        for (const WallRef& w : L.walls) {
            CHECK(w.slot >= 0 && w.slot < L.n_wall && !slot[w.slot], "%s slot", name);
            slot[w.slot] = 1;
        }
    }
    printf("%s ok\n", name);
}

int main() {
    const int F8 = LBM_FP64, F4 = LBM_FP32_SHIFT, F2 = LBM_FP16_SHIFT_G;
    check("one node", params(1, 1, 1, F4), 0, 1, 0);
    check("ragged", params(67, 13, 9, F8), 1, 1, 0);
    check("flat", params(130, 1, 31, F8), 0, 1, 0);
    check("porous", params(35, 20, 18, F2), 2, 1, 0);
    check("column", params(70, 40, 30, F4), 3, 1, 0);
    check("cube within the cache", params(120, 120, 120, F4), 0, 1, 0);
    check("cube beyond", params(128, 128, 128, F4), 0, 1, 1);
    check("depth that leaves a short read tile", params(131, 129, 131, F4), 1, 1, 1);
    check("fewer planes than a read tile", params(1100, 1000, 3, F4), 0, 1, 1);
    check("narrow, lines beyond", params(17, 256, 256, F4), 0, 1, 1);
    check("narrow porous", params(33, 200, 300, F2), 2, 1, 1);
    check("mostly solid, few lines", params(160, 160, 120, F4), 3, 1, 1);
    check("FP64 beyond", params(104, 104, 104, F8), 1, 1, 1);
    lbm_params p = params(104, 104, 104, F8);
    p.hysteresis = 1;
    check("FP64 hysteresis beyond", p, 1, 0, 0);
    p = params(131, 129, 131, F4);
    p.hysteresis = 2;
    check("FP32 hysteresis beyond", p, 2, 1, 1);
    p = params(64, 60, 50, F2);
    p.hysteresis = 1;
    check("hysteresis within", p, 1, 1, 0);
    p = params(40, 30, 20, F4);
    p.q_phase = 19;
    check("D3Q19", p, 1, 0, 0);
    p = params(40, 30, 20, F4);
    p.face_bc[4] = LBM_BC_PRESSURE;
    check("one face, wrap", p, 0, 0, 0);
    p.face_bc[5] = LBM_BC_PRESSURE;
    check("two faces", p, 0, 1, 0);
    printf(bad ? "FAILED\n" : "OK\n");
    return bad;
}
