// The matrix-core plan of random and named NBB fractals, driven lane by lane
// as the kernel drives it (operands, record writes and reads, halo blocks of
// the neighbour tiles), against neighbour counts taken cell by cell through
// lambda and nu, for both stencils.  Prints what was compared and the shapes.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <string>
#include <vector>

#include "plan.hpp"
using namespace nbb;

static int count_ref(const Fractal &f, const std::vector<uint8_t> &st, uint64_t i, bool edge) {
    int64_t x, y;
    lambda_levels(f, f.r, i, &x, &y);
    int n = 0;
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
            if (!dx && !dy) continue;
            if (edge && dx && dy) continue;
            const int64_t v = nu_levels(f, f.r, x + dx, y + dy);
            if (v >= 0) n += st[size_t(v)];
        }
    return n;
}

// D[row][col] = sum over quarters and bytes of A and B, lanes as the kernel's
static void contract(const int8_t *A, const std::vector<uint8_t> &B, int (&D)[64][4]) {
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * (l / 16) + i, col = l % 16;
            for (int q = 0; q < 4; ++q)
                for (int j = 0; j < 16; ++j) D[l][i] += A[(q * 16 + row) * 16 + j] * B[(q * 16 + col) * 16 + j];
        }
}

// Byte i of record dword t of a lane whose 16 cells are x.
static uint8_t pick(const std::vector<uint32_t> &sel, uint32_t t, uint32_t sub, int i, const uint8_t *x) {
    const uint32_t a = sel[2 * (4 * t + sub)] >> (8 * i) & 0xFF, b = sel[2 * (4 * t + sub) + 1] >> (8 * i) & 0xFF;
    if ((a > 7 && a != 12) || (b > 7 && b != 12) || (a < 8 && b < 8)) std::abort();
    return a < 8 ? x[a] : (b < 8 ? x[8 + b] : 0);
}

// `inst`: the same fractal at a level below the plan's tile, as a batch's
// instance is one cut tile without neighbours, with live bytes behind it.
static void check(const Fractal &f, const MatPlan &p, std::mt19937 &rng, bool edge, const Fractal *inst = nullptr) {
    const Fractal &of = inst ? *inst : f;
    const uint64_t ntiles = inst ? 1 : p.ntiles;
    const uint32_t bytes = uint32_t(std::min<uint64_t>(p.K, of.cells));
    std::vector<uint8_t> st(std::max<uint64_t>(of.cells, p.K), 1);
    for (uint64_t i = 0; i < of.cells; ++i) st[i] = rng() & 1;
    const uint32_t bpg = 64 / p.lanes;
    for (uint64_t tile = 0; tile < ntiles; ++tile) {
        if (ntiles > 40 && rng() % (p.ntiles / 20)) continue;
        std::vector<uint8_t> lds(p.buf_bytes, 0xEE);
        const uint32_t zero = (p.lanes * p.nr * p.nrecs) * 4;
        if (zero + 4 > p.buf_bytes) std::abort();
        for (int i = 0; i < 4; ++i) lds[zero + i] = 0;
        auto load = [&](uint64_t t, uint32_t b, uint32_t sub, uint8_t *dst) {
            const uint32_t off = mat_first_cell(sub, p.CB);
            if (inst && !mat_lane_owns(b, p.CB, off, bytes)) return;  // loads as zeros
            for (uint32_t j = 0; j < 16; ++j) dst[j] = st[t * p.K + b * p.CB + off + j];
        };
        auto publish = [&](const std::vector<uint8_t> &B, const std::vector<int64_t> &rec) {
            for (uint32_t t = 0; t < p.nr; ++t) {
                for (int l = 0; l < 64; ++l) {
                    const uint32_t in = (l / 16) / p.lanes * 16 + l % 16, sub = (l / 16) % p.lanes;
                    if (rec[in] < 0) continue;
                    for (int i = 0; i < 4; ++i)
                        lds[4 * ((t * p.lanes + sub) * p.nrecs + rec[in]) + i] =
                            pick(p.sel, t, sub, i, B.data() + 16 * l);
                }
            }
        };
        auto gather = [&](uint32_t n, auto block_of, std::vector<uint8_t> *B, std::vector<int64_t> *rec, uint32_t g,
                          uint32_t rec0) {
            B->assign(1024, 0);
            rec->assign(bpg, -1);
            for (int l = 0; l < 64; ++l) {
                const uint32_t in = (l / 16) / p.lanes * 16 + l % 16, sub = (l / 16) % p.lanes;
                const uint32_t b = g * bpg + in;
                if (b >= n) continue;
                (*rec)[in] = rec0 + b;
                uint64_t t;
                uint32_t lb;
                if (block_of(b, &t, &lb)) load(t, lb, sub, B->data() + 16 * l);
            }
        };
        std::vector<uint8_t> B;
        std::vector<int64_t> rec;
        auto own = [&](uint32_t b, uint64_t *t, uint32_t *lb) {
            *t = tile;
            *lb = b;
            return true;
        };
        auto halo = [&](uint32_t h, uint64_t *t, uint32_t *lb) {
            const uint32_t nt = inst ? 0xFFFFFFFFu : p.nbr[tile * 8 + (p.halo[h] >> 29)];
            *t = nt;
            *lb = p.halo[h] & 0x1FFFFFFFu;
            return nt != 0xFFFFFFFFu;
        };
        for (uint32_t g = 0; g < p.groups; ++g) {
            gather(p.nblk, own, &B, &rec, g, 0);
            publish(B, rec);
        }
        for (uint32_t g = 0; g * bpg < p.nhalo; ++g) {
            if (g >= p.waves) std::abort();
            gather(p.nhalo, halo, &B, &rec, g, p.nblk);
            publish(B, rec);
        }
        if (p.groups > p.waves * p.gpw) std::abort();
        for (uint32_t g = 0; g < p.groups; ++g) {
            gather(p.nblk, own, &B, &rec, g, 0);
            for (uint32_t t = 0; t < 2; ++t) {
                int D[64][4] = {};
                contract(p.A.data() + mat_self_off(p.nh, edge, t), B, D);
                for (uint32_t h = 0; h < p.nh; ++h) {
                    std::vector<uint8_t> R(1024);
                    for (int l = 0; l < 64; ++l)
                        for (int d = 0; d < 4; ++d) {
                            const uint32_t w = p.raddr[(size_t(g) * 64 + l) * 2 * p.nh + 2 * h + d / 2];
                            const uint32_t a = d & 1 ? w >> 16 : w & 0xFFFFu;
                            if (a + 4 > p.buf_bytes) std::abort();
                            for (int i = 0; i < 4; ++i) R[16 * l + 4 * d + i] = lds[a + i];
                        }
                    contract(p.A.data() + mat_halo_off(p.nh, edge, h, t), R, D);
                }
                for (int l = 0; l < 64; ++l) {
                    const uint32_t in = (l / 16) / p.lanes * 16 + l % 16, sub = (l / 16) % p.lanes;
                    const uint32_t b = g * bpg + in;
                    if (b >= p.nblk) continue;
                    for (int i = 0; i < 4; ++i)
                        for (int hi = 0; hi < 2; ++hi) {
                            const uint32_t c = mat_first_cell(sub, p.CB) + 8 * t + 4 * hi + i;
                            if (b * p.CB + c >= bytes) continue;
                            const int want = count_ref(of, st, tile * p.K + b * p.CB + c, edge);
                            const int got = hi ? D[l][i] >> 4 : D[l][i] & 15;
                            if (want != got || D[l][i] < 0 || D[l][i] > 255) {
                                std::printf("mismatch k %u s %u r %u m %u tile %llu block %u cell %u: %d %d\n", f.k, f.s,
                                            f.r, p.m, (unsigned long long)tile, b, c, want, got);
                                std::exit(1);
                            }
                        }
                }
            }
        }
    }
}

// Several generations of a random rule on tiles held with their rings.
static void check_hold(const Fractal &f, const HoldPlan &p, std::mt19937 &rng, const Fractal *inst = nullptr) {
    const Fractal &of = inst ? *inst : f;
    const uint64_t ntiles = inst ? 1 : p.ntiles;
    const uint32_t bytes = uint32_t(std::min<uint64_t>(p.K, of.cells));
    const uint32_t rule = rng() & 0x01FF01FFu;
    const bool edge = rng() & 1;
    const uint32_t gens = std::min(p.gens, 10u), bpg = 64 / p.lanes;
    std::vector<uint8_t> st(std::max<uint64_t>(of.cells, p.K), 1);
    for (uint64_t i = 0; i < of.cells; ++i) st[i] = rng() & 1;
    std::vector<uint8_t> ref(st.begin(), st.begin() + std::ptrdiff_t(of.cells));
    for (uint32_t g = 0; g < gens; ++g) {
        std::vector<uint8_t> next(of.cells);
        for (uint64_t i = 0; i < of.cells; ++i) {
            const int n = count_ref(of, ref, i, edge);
            next[i] = (rule >> (ref[i] ? 16 + n : n)) & 1;
        }
        ref.swap(next);
    }
    std::vector<uint32_t> nbr;
    if (inst) nbr.assign(8, 0xFFFFFFFFu);
    else neighbour_table(f, f.r - p.m, &nbr);
    for (uint64_t tile = 0; tile < ntiles; ++tile) {
        if (ntiles > 4 && rng() % (ntiles / 2)) continue;
        const uint32_t groups = p.waves * p.gpw;
        std::vector<std::vector<uint8_t>> X(groups, std::vector<uint8_t>(1024));
        std::vector<uint8_t> live(groups * 64);
        for (uint32_t g = 0; g < groups; ++g)
            for (int l = 0; l < 64; ++l) {
                const uint32_t in = (l / 16) / p.lanes * 16 + l % 16, sub = (l / 16) % p.lanes, b = g * bpg + in;
                if (b >= p.ntot) continue;
                uint64_t t = tile;
                uint32_t lb = b;
                if (b >= p.nblk) {
                    const uint32_t item = p.halo[b - p.nblk];
                    t = nbr[tile * 8 + (item >> 29)];
                    lb = item & 0x1FFFFFFFu;
                    if (t == 0xFFFFFFFFu) continue;
                } else if (!mat_lane_owns(b, p.CB, mat_first_cell(sub, p.CB), bytes)) {
                    continue;
                }
                live[g * 64 + l] = 1;
                for (uint32_t j = 0; j < 16; ++j)
                    X[g][16 * l + j] = st[t * p.K + lb * p.CB + mat_first_cell(sub, p.CB) + j];
            }
        for (uint32_t gen = 0; gen < gens; ++gen) {
            std::vector<uint8_t> lds(p.zero + 4, 0xEE);
            for (int i = 0; i < 4; ++i) lds[p.zero + i] = 0;
            for (uint32_t g = 0; g < groups; ++g)
                for (uint32_t t = 0; t < p.nr; ++t) {
                    for (int l = 0; l < 64; ++l) {
                        const uint32_t in = (l / 16) / p.lanes * 16 + l % 16, sub = (l / 16) % p.lanes;
                        const uint32_t a = 4 * (std::min(g * bpg + in, p.ntot) * p.rs + sub * p.nr + t);
                        if (a + 4 > p.zero) std::abort();
                        for (int i = 0; i < 4; ++i) lds[a + i] = pick(p.sel, t, sub, i, X[g].data() + 16 * l);
                    }
                }
            for (uint32_t g = 0; g < groups; ++g) {
                std::vector<uint8_t> N(1024);
                for (uint32_t t = 0; t < 2; ++t) {
                    int D[64][4] = {};
                    contract(p.A.data() + mat_self_off(p.nh, edge, t), X[g], D);
                    for (uint32_t h = 0; h < p.nh; ++h) {
                        std::vector<uint8_t> R(1024);
                        for (int l = 0; l < 64; ++l)
                            for (int d = 0; d < 4; ++d) {
                                const uint32_t w = p.raddr[(size_t(g) * 64 + l) * 2 * p.nh + 2 * h + d / 2];
                                const uint32_t a = d & 1 ? w >> 16 : w & 0xFFFFu;
                                if (a > p.zero) std::abort();
                                for (int i = 0; i < 4; ++i) R[16 * l + 4 * d + i] = lds[a + i];
                            }
                        contract(p.A.data() + mat_halo_off(p.nh, edge, h, t), R, D);
                    }
                    for (int l = 0; l < 64; ++l)
                        for (int i = 0; i < 4; ++i)
                            for (int hi = 0; hi < 2; ++hi) {
                                const int n = hi ? D[l][i] >> 4 : D[l][i] & 15;
                                const int j = 16 * l + 8 * t + 4 * hi + i;
                                N[j] = live[g * 64 + l] && n <= 8 && (rule >> (X[g][j] ? 16 + n : n)) & 1;
                            }
                }
                X[g].swap(N);
            }
        }
        for (uint32_t b = 0; b < p.nblk; ++b)
            for (uint32_t sub = 0; sub < p.lanes; ++sub)
                for (uint32_t j = 0; j < 16; ++j) {
                    const uint32_t c = mat_first_cell(sub, p.CB) + j, in = b % bpg;
                    if (b * p.CB + c >= bytes) continue;
                    const uint32_t lane = (in / 16 * p.lanes + sub) * 16 + in % 16;
                    if (X[b / bpg][16 * lane + j] != ref[tile * p.K + b * p.CB + c]) {
                        std::printf("held mismatch k %u s %u r %u m %u gens %u tile %llu block %u cell %u\n", f.k, f.s, f.r,
                                    p.m, gens, (unsigned long long)tile, b, c);
                        std::exit(1);
                    }
                }
    }
}

static bool make(uint32_t s, const std::vector<int32_t> &off, uint32_t r, Fractal *f) {
    std::string msg;
    return validate_fractal(uint32_t(off.size() / 2), s, off.data(), r, f, &msg) == 0;
}

int main(int argc, char **argv) {
    std::mt19937 rng(7);
    int plans = 0, held = 0;
    std::vector<std::pair<uint32_t, std::vector<int32_t>>> named = {
        {2, {0, 0, 1, 0, 0, 1}},                                      // triangle
        {3, {0, 0, 1, 0, 2, 0, 0, 1, 2, 1, 0, 2, 1, 2, 2, 2}},        // carpet
        {3, {0, 0, 0, 1, 0, 2, 1, 1, 2, 0, 2, 1, 2, 2}},              // H
        {3, {0, 0, 1, 0, 2, 0, 1, 1}},                                // chandelier-like
        {2, {0, 0, 1, 0, 0, 1, 1, 1}},                                // full square
        {3, {1, 0, 0, 1, 1, 1, 2, 1, 1, 2}},                          // Vicsek
        {3, {0, 0, 2, 0, 1, 1, 0, 2, 2, 2}},                          // X
        {3, {0, 0, 2, 0, 0, 2, 2, 2}},                                // Cantor dust
        {3, {0, 0, 2, 0}},                                            // Cantor set
    };
    for (auto &n : named)
        for (uint32_t r = 2; r <= 7; ++r) {
            Fractal f;
            if (!make(n.first, n.second, r, &f) || f.cells > 60000) continue;
            for (uint32_t m = 1; m <= r; ++m) {
                MatPlan p;
                std::string msg;
                if (!build_mat_plan(f, m, rng() % 2 ? 0 : 1u << rng() % 3, &p, &msg)) continue;
                for (bool edge : {false, true}) check(f, p, rng, edge);
                ++plans;
                for (uint32_t rings = 0; rings <= 2; ++rings) {
                    HoldPlan h;
                    if (f.cells > 20000 || !build_hold_plan(f, m, rings, rng() % 2 ? 0 : 1u << rng() % 3, &h, &msg))
                        continue;
                    check_hold(f, h, rng);
                    ++held;
                    if (argc > 1)
                        std::printf("# held k %u r %u m %u rings %u: nblk %u ntot %u groups %u gpw %u waves %u zero %u\n",
                                    f.k, f.r, m, rings, h.nblk, h.ntot, h.groups, h.gpw, h.waves, h.zero);
                }
                if (r == 7 || argc > 1)
                    std::printf("# k %u s %u r %u m %u: q %u CB %u lanes %u nblk %u nhalo %u nr %u nh %u gpw %u waves %u buf %u\n",
                                f.k, f.s, r, m, p.q, p.CB, p.lanes, p.nblk, p.nhalo, p.nr, p.nh, p.gpw, p.waves,
                                p.buf_bytes);
            }
        }
    // instances below the tile level of the launch's plan, of every level that
    // has a plan of its own; block levels differ between them for k = 2 and 4
    int cut = 0;
    named.push_back({2, {0, 0, 1, 1}});                               // diagonal
    for (auto &n : named)
        for (uint32_t r = 2; r <= 9; ++r) {
            Fractal f, low;
            if (!make(n.first, n.second, r, &f) || f.cells > 5000) continue;
            for (uint32_t lr = 1; lr < r; ++lr) {
                MatPlan p;
                HoldPlan h;
                std::string msg;
                make(n.first, n.second, lr, &low);
                if (mat_dims(low).empty()) continue;
                for (uint32_t m = lr + 1; m <= r; ++m) {
                    if (build_mat_plan(f, m, 0, &p, &msg))
                        for (bool edge : {false, true}) check(f, p, rng, edge, &low);
                    if (build_hold_plan(f, m, m == r ? 0 : 1, 0, &h, &msg)) {
                        for (int i = 0; i < 4; ++i) check_hold(f, h, rng, &low);
                        ++cut;
                    }
                }
            }
        }
    std::printf("cut %d\n", cut);
    // few blocks in a wide square
    for (const auto &n : std::vector<std::pair<uint32_t, std::vector<int32_t>>>{{3, {0, 0, 2, 0}}, {4, {0, 0, 1, 1}}}) {
        Fractal f;
        const uint32_t r = n.first == 3 ? 12 : 11;
        if (!make(n.first, n.second, r, &f)) std::abort();
        for (uint32_t m = r - 1; m <= r; ++m) {
            MatPlan p;
            HoldPlan h;
            std::string msg;
            if (!build_mat_plan(f, m, 0, &p, &msg) || !build_hold_plan(f, m, m < r ? 2 : 0, 0, &h, &msg)) std::abort();
            check(f, p, rng, false);
            check_hold(f, h, rng);
        }
    }
    for (int it = 0; it < 300; ++it) {
        const uint32_t s = 2 + rng() % 3, k = 1 + rng() % (s * s);
        std::vector<int> cells(s * s);
        for (uint32_t i = 0; i < s * s; ++i) cells[i] = int(i);
        std::shuffle(cells.begin(), cells.end(), rng);
        std::vector<int32_t> off;
        for (uint32_t j = 0; j < k; ++j) {
            off.push_back(int32_t(cells[j] % s));
            off.push_back(int32_t(cells[j] / s));
        }
        Fractal f;
        if (!make(s, off, 1 + rng() % 7, &f) || f.cells > 20000) continue;
        for (uint32_t m = 1; m <= f.r; ++m) {
            MatPlan p;
            std::string msg;
            if (!build_mat_plan(f, m, rng() % 2 ? 0 : 1u << rng() % 3, &p, &msg)) continue;
            check(f, p, rng, rng() & 1);
            ++plans;
            HoldPlan h;
            if (f.cells <= 5000 && build_hold_plan(f, m, m == f.r ? 0 : 1 + rng() % 2, 0, &h, &msg)) {
                check_hold(f, h, rng);
                ++held;
            }
        }
        // whatever level and groups per wavefront a launch picks can be built
        const std::vector<MatDims> dims = mat_dims(f);
        for (uint32_t cus : {1u, 256u}) {
            uint32_t gpw = 0;
            const uint32_t a = pick_mat_level(dims, f.k, {f.r, f.r, uint32_t(1 + rng() % f.r)}, cus, &gpw);
            MatPlan p;
            std::string msg;
            if (a && (!build_mat_plan(f, a, gpw, &p, &msg, false) || p.gpw != gpw)) std::abort();
        }
    }
    std::printf("held %d plans %d\n", held, plans);
    return 0;
}
