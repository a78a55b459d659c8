// Host-side plan of the matrix-core form of the tiled step.  See MatParams in
// params.hpp for the scheme.
#include <stddef.h>

#include <algorithm>

#include "plan.hpp"

namespace nbb {

namespace {

uint64_t ipow(uint64_t b, uint32_t e) {
    uint64_t p = 1;
    while (e--) p *= b;
    return p;
}

const int kDirX[8] = {-1, 0, 1, -1, 1, -1, 0, 1};  // as the neighbour tables: row-major without the centre
const int kDirY[8] = {-1, -1, -1, 0, 0, 1, 1, 1};

// What a block of level q needs from its neighbours and how its record holds
// what they need from it.
struct BlockShape {
    uint32_t q = 0, CB = 0, BS = 0, lanes = 0, nr = 0, nh = 0;
    std::vector<int64_t> x, y;               // the block's cells
    std::vector<std::vector<uint32_t>> need;  // per direction: cells of that neighbour next to one of ours
    std::vector<int32_t> rec;                // lanes * nr * 4 record bytes: cell or -1; dword t lanes + sub is lane sub's t-th
    std::vector<std::pair<uint32_t, uint32_t>> reads;  // (direction, record dword)
};

// The record dwords that hold all of `cells`, first found first.
void reads_of(const std::vector<int32_t> &rec, uint32_t dir, const std::vector<uint32_t> &cells,
              std::vector<std::pair<uint32_t, uint32_t>> *reads) {
    std::vector<uint32_t> left = cells;
    while (!left.empty()) {
        // the dword with the most of what is left
        size_t best = 0, most = 0;
        for (size_t d = 0; d < rec.size() / 4; ++d) {
            size_t n = 0;
            for (size_t b = 0; b < 4; ++b)
                n += rec[4 * d + b] >= 0 && std::count(left.begin(), left.end(), uint32_t(rec[4 * d + b]));
            if (n > most) {
                most = n;
                best = d;
            }
        }
        reads->push_back({dir, uint32_t(best)});
        std::vector<uint32_t> rest;
        for (uint32_t c : left) {
            bool in = false;
            for (size_t b = 0; b < 4; ++b) in |= rec[4 * best + b] == int32_t(c);
            if (!in) rest.push_back(c);
        }
        left.swap(rest);
    }
}

bool block_shape(const Fractal &f, uint32_t q, BlockShape *s) {
    s->q = q;
    s->CB = uint32_t(ipow(f.k, q));
    s->BS = uint32_t(ipow(f.s, q));
    s->lanes = s->CB <= 16 ? 1 : (s->CB <= 32 ? 2 : 4);
    s->x.resize(s->CB);
    s->y.resize(s->CB);
    for (uint32_t c = 0; c < s->CB; ++c) lambda_levels(f, q, c, &s->x[c], &s->y[c]);
    s->need.assign(8, {});
    size_t total = 0;
    for (uint32_t d = 0; d < 8; ++d)
        for (uint32_t e = 0; e < s->CB; ++e) {
            const int64_t ex = s->x[e] + kDirX[d] * int64_t(s->BS), ey = s->y[e] + kDirY[d] * int64_t(s->BS);
            for (uint32_t c = 0; c < s->CB; ++c)
                if (std::abs(ex - s->x[c]) <= 1 && std::abs(ey - s->y[c]) <= 1) {
                    s->need[d].push_back(e);
                    ++total;
                    break;
                }
        }
    // The record: dwords of up to four needed cells held by one lane each.  A
    // direction's cells of one lane go four at a time into a dword that has
    // them or room for them, else into a new one, so that a direction is read
    // in few dwords; cells that two lanes hold (the last lane overlaps the one
    // before) go to the lane with fewer dwords.
    std::vector<std::vector<std::vector<uint32_t>>> dw(s->lanes);
    auto first_cell = [&](uint32_t sub) { return std::min(16 * sub, s->CB - 16); };
    std::vector<uint32_t> order = {0, 1, 2, 3, 4, 5, 6, 7};
    std::stable_sort(order.begin(), order.end(),
                     [&](uint32_t a, uint32_t b) { return s->need[a].size() > s->need[b].size(); });
    for (uint32_t d : order)
        for (uint32_t sub = 0; sub < s->lanes; ++sub) {
            std::vector<uint32_t> mine;
            for (uint32_t e : s->need[d])
                if (e / 16 == sub) mine.push_back(e);
            for (size_t i = 0; i < mine.size(); i += 4) {
                const std::vector<uint32_t> part(mine.begin() + ptrdiff_t(i),
                                                 mine.begin() + ptrdiff_t(std::min(i + 4, mine.size())));
                std::vector<uint32_t> *home = nullptr;
                size_t grow = 5;
                uint32_t fresh = sub;
                for (uint32_t l = 0; l < s->lanes; ++l) {
                    if (part.front() < first_cell(l) || part.back() >= first_cell(l) + 16) continue;
                    if (dw[l].size() < dw[fresh].size()) fresh = l;
                    for (auto &w : dw[l]) {
                        size_t more = 0;
                        for (uint32_t e : part) more += !std::count(w.begin(), w.end(), e);
                        if (w.size() + more > 4 || more >= grow) continue;
                        grow = more;
                        home = &w;
                    }
                }
                if (!home) {
                    dw[fresh].emplace_back();
                    home = &dw[fresh].back();
                }
                for (uint32_t e : part)
                    if (!std::count(home->begin(), home->end(), e)) home->push_back(e);
            }
        }
    s->nr = 1;
    for (const auto &l : dw) s->nr = std::max<uint32_t>(s->nr, uint32_t(l.size()));
    s->rec.assign(size_t(s->nr) * s->lanes * 4, -1);
    for (uint32_t l = 0; l < s->lanes; ++l)
        for (size_t t = 0; t < dw[l].size(); ++t)
            for (size_t j = 0; j < dw[l][t].size(); ++j)
                s->rec[4 * (t * s->lanes + l) + j] = int32_t(dw[l][t][j]);
    for (uint32_t d = 0; d < 8; ++d) reads_of(s->rec, d, s->need[d], &s->reads);
    s->nh = std::max<uint32_t>(1, uint32_t((s->reads.size() + 4 * s->lanes - 1) / (4 * s->lanes)));
    return s->nr <= 3 && s->nh <= 2;
}

// The largest block level with 16 to 64 cells whose ring fits.
bool pick_shape(const Fractal &f, BlockShape *s) {
    if (!tiled_supported(f) || f.k < 2) return false;
    uint32_t q = 0;
    while (q < f.r && ipow(f.k, q + 1) <= 64) ++q;
    for (; q >= 1 && ipow(f.k, q) >= 16; --q) {
        BlockShape t;
        if (block_shape(f, q, &t)) {
            *s = std::move(t);
            return true;
        }
    }
    return false;
}

}  // namespace

const uint32_t kNone = 0xFFFFFFFFu;

// Numbers by place in [lo, hi)^2, at most `most` of them: a table of the whole
// square up to 1 MB, else a hash table, as a sparse fractal has few blocks in a
// square of any side (the Cantor set 1,024 in a row of 59,049, whose square
// would take 14 GB).  The plans of the triangle r16 and the chandelier r9 take
// 0.4 and 0.5 ms from tables, 1.1 and 1.3 from hash tables.
class PlaceMap {
   public:
    PlaceMap(int64_t lo, int64_t hi, uint64_t most) : lo_(lo), side_(uint64_t(hi - lo)) {
        dense_ = side_ <= 512;
        uint64_t n = dense_ ? side_ * side_ : 16;
        for (; !dense_ && n < 2 * most; n *= 2) --shift_;
        if (!dense_) key_.assign(size_t(n), 0);
        val_.assign(size_t(n), kNone);
    }
    // the number at (x, y), or kNone; a reference to set it (to anything else)
    uint32_t &at(int64_t x, int64_t y) {
        const uint64_t u = uint64_t(x - lo_), v = uint64_t(y - lo_);
        if (dense_) return val_[size_t(v * side_ + u)];
        const uint64_t key = v << 32 | u;
        size_t i = size_t((key * 0x9E3779B97F4A7C15ull) >> shift_);
        while (val_[i] != kNone && key_[i] != key) i = (i + 1) & (val_.size() - 1);
        key_[i] = key;
        return val_[i];
    }

   private:
    int64_t lo_;
    uint64_t side_;
    bool dense_ = false;
    uint32_t shift_ = 60;
    std::vector<uint64_t> key_;
    std::vector<uint32_t> val_;
};

// The places of the blocks of a tile, `levels` block levels: the numbers by
// place and the places by number.
static void tile_places(const Fractal &f, uint32_t levels, PlaceMap *block,
                        std::vector<std::pair<int64_t, int64_t>> *at) {
    const uint64_t nb = ipow(f.k, levels);
    for (uint64_t b = 0; b < nb; ++b) {
        int64_t X, Y;
        lambda_levels(f, levels, b, &X, &Y);
        block->at(X, Y) = uint32_t(b);
        at->push_back({X, Y});
    }
}

// The blocks of the tile at level m and of its neighbour tiles: `source`
// gets the record of every read of every block (an own block, a halo block
// numbered as first met, or none).
static bool build_ring(const Fractal &f, const BlockShape &s, uint32_t m, MatPlan *p, std::vector<uint32_t> *source,
                       std::string *msg) {
    *p = MatPlan();
    if (m < s.q || m > f.r) {
        *msg = "the matrix form needs q <= m <= r";
        return false;
    }
    const uint32_t bpg = 64 / s.lanes;
    const uint64_t nb = ipow(f.k, m - s.q);
    if (nb > uint64_t(4) * kMatMaxWaves * bpg) {
        *msg = "more groups than a work-group takes";
        return false;
    }
    p->m = m;
    p->q = s.q;
    p->K = uint32_t(ipow(f.k, m));
    p->CB = s.CB;
    p->lanes = s.lanes;
    p->nblk = uint32_t(nb);
    p->nr = s.nr;
    p->nh = s.nh;
    p->groups = (p->nblk + bpg - 1) / bpg;
    p->ntiles = ipow(f.k, f.r - m);
    const int64_t G = int64_t(ipow(f.s, m - s.q));
    PlaceMap block(0, G, nb), ring(-1, G + 1, 8 * nb);  // ring: the halo block at a place around the tile
    std::vector<std::pair<int64_t, int64_t>> at;
    tile_places(f, m - s.q, &block, &at);
    source->assign(size_t(p->nblk) * s.reads.size(), kNone);
    for (uint32_t b = 0; b < p->nblk; ++b)
        for (size_t i = 0; i < s.reads.size(); ++i) {
            const uint32_t d = s.reads[i].first;
            const int64_t nx = at[b].first + kDirX[d], ny = at[b].second + kDirY[d];
            const int tx = nx < 0 ? -1 : (nx >= G ? 1 : 0), ty = ny < 0 ? -1 : (ny >= G ? 1 : 0);
            const uint32_t v = block.at(nx - tx * G, ny - ty * G);
            if (v == kNone) continue;
            uint32_t &src = (*source)[b * s.reads.size() + i];
            if (!tx && !ty) {
                src = v;
                continue;
            }
            uint32_t &h = ring.at(nx, ny);
            if (h == kNone) {
                uint32_t dir = 0;
                while (kDirX[dir] != tx || kDirY[dir] != ty) ++dir;
                h = p->nblk + uint32_t(p->halo.size());
                p->halo.push_back(dir << 29 | v);
            }
            src = h;
        }
    p->nhalo = uint32_t(p->halo.size());
    if (p->halo.empty()) p->halo.push_back(0);
    p->nrecs = p->nblk + p->nhalo + 1;
    const uint64_t words = uint64_t(s.lanes) * s.nr * p->nrecs + 1;  // and one dword of zeros
    p->buf_bytes = uint32_t((words * 4 + 15) & ~uint64_t(15));
    if (p->buf_bytes > 32 * 1024 - 16) {  // two buffers, 16-bit offsets
        *msg = "records beyond 32 KiB";
        return false;
    }
    return true;
}

// Groups per wavefront: the most of 4, 2, 1 that leaves two wavefronts per
// work-group and, with the tiles at hand, six per CU (a wavefront with more
// groups has more loads in flight and does the tile's uniform work less
// often: triangle r16 at level 8, 1 / 2 / 4 groups per wavefront 18.3 / 16.2 /
// 15.8 us; carpet r7, two tiles per CU, 3.70 / 3.85 / 4.66); each wavefront
// also takes at most one group of halo blocks.  0 if none fits.
static uint32_t pick_gpw(uint32_t groups, uint32_t hgroups, uint64_t tiles, uint32_t cus) {
    const uint64_t per_cu = (tiles + cus - 1) / cus;
    uint32_t gpw = 0;
    for (uint32_t g : {4u, 2u, 1u}) {
        const uint32_t w = std::max((groups + g - 1) / g, hgroups);
        if (w > kMatMaxWaves) break;
        gpw = g;
        if (w >= 2 && w * per_cu >= 6) break;
    }
    return gpw;
}

// The constant operands of a block shape (MatParams::A).
static void mat_operands(const BlockShape &s, std::vector<int8_t> *A) {
    // operands: lane l of an operand holds row l % 16, products 16 (l / 16) ..
    const uint32_t nh = s.nh;
    A->assign(size_t(1024) * 2 * (2 + 2 * nh), 0);
    auto first_cell = [&](uint32_t sub) { return std::min(16 * sub, s.CB - 16); };
    auto put = [&](uint32_t off, uint32_t row, uint32_t quarter, uint32_t byte, int w) {
        (*A)[off + (quarter * 16 + row) * 16 + byte] = int8_t((*A)[off + (quarter * 16 + row) * 16 + byte] + w);
    };
    for (int edge = 0; edge < 2; ++edge) {
        auto adjacent = [&](int64_t dx, int64_t dy) {
            dx = std::abs(dx);
            dy = std::abs(dy);
            return edge ? dx + dy == 1 : (dx <= 1 && dy <= 1 && dx + dy != 0);
        };
        for (uint32_t g = 0; g < 4; ++g)
            for (uint32_t row = 4 * g; row < 4 * g + 4; ++row)
                for (uint32_t t = 0; t < 2; ++t)
                    for (uint32_t hi = 0; hi < 2; ++hi) {
                        const uint32_t c = first_cell(g % s.lanes) + 8 * t + 4 * hi + row % 4;
                        const int w = hi ? 16 : 1;
                        for (uint32_t sub = 0; sub < s.lanes; ++sub) {
                            const uint32_t quarter = g / s.lanes * s.lanes + sub;
                            for (uint32_t j = 0; j < 16; ++j) {
                                const uint32_t e = first_cell(sub) + j;
                                if (e < 16 * sub) continue;  // held by an earlier lane
                                if (adjacent(s.x[e] - s.x[c], s.y[e] - s.y[c]))
                                    put(mat_self_off(nh, edge, t), row, quarter, j, w);
                            }
                        }
                        std::vector<std::pair<uint32_t, int32_t>> seen;
                        for (size_t i = 0; i < s.reads.size(); ++i)
                            for (uint32_t b = 0; b < 4; ++b) {
                                const uint32_t dir = s.reads[i].first;
                                const int32_t e = s.rec[4 * s.reads[i].second + b];
                                if (e < 0 || !std::count(s.need[dir].begin(), s.need[dir].end(), uint32_t(e))) continue;
                                const std::pair<uint32_t, int32_t> id{dir, e};
                                if (std::count(seen.begin(), seen.end(), id)) continue;
                                seen.push_back(id);
                                const int64_t ex = s.x[e] + kDirX[dir] * int64_t(s.BS);
                                const int64_t ey = s.y[e] + kDirY[dir] * int64_t(s.BS);
                                if (!adjacent(ex - s.x[c], ey - s.y[c])) continue;
                                const uint32_t h = uint32_t(i) / (4 * s.lanes), sub = uint32_t(i) / 4 % s.lanes;
                                put(mat_halo_off(nh, edge, h, t), row, g / s.lanes * s.lanes + sub,
                                    4 * (uint32_t(i) % 4) + b, w);
                            }
                    }
    }
}

// Selectors of record dword t of lane sub, at 2 (4 t + sub): its bytes out of
// the lane's first two dwords and out of its last two (12: a zero byte).
static void mat_selectors(const BlockShape &s, std::vector<uint32_t> *sel) {
    sel->assign(size_t(8) * s.nr, 0x0C0C0C0Cu);
    for (uint32_t t = 0; t < s.nr; ++t)
        for (uint32_t sub = 0; sub < s.lanes; ++sub)
            for (uint32_t j = 0; j < 4; ++j) {
                const int32_t e = s.rec[4 * (t * s.lanes + sub) + j];
                if (e < 0) continue;
                const uint32_t at = uint32_t(e) - std::min(16 * sub, s.CB - 16);  // the lane's byte
                uint32_t &w = (*sel)[2 * (4 * t + sub) + (at >= 8)];
                w = (w & ~(0xFFu << (8 * j))) | (at & 7) << (8 * j);
            }
}

static bool build_mat_shape(const Fractal &f, const BlockShape &s, uint32_t m, uint32_t gpw, MatPlan *p,
                            std::string *msg, bool with_nbr) {
    std::vector<uint32_t> source;
    if (!build_ring(f, s, m, p, &source, msg)) return false;
    const uint32_t bpg = 64 / s.lanes, hgroups = (p->nhalo + bpg - 1) / bpg;
    p->gpw = gpw ? gpw : pick_gpw(p->groups, hgroups, p->ntiles, 256);
    p->waves = p->gpw ? std::max((p->groups + p->gpw - 1) / p->gpw, hgroups) : 0;
    if (!p->gpw || p->waves > kMatMaxWaves) {
        *msg = "more groups than a work-group takes";
        return false;
    }
    // record reads: read i is dword i % 4 of lane (i / 4) % lanes, halo operand i / (4 lanes)
    const uint32_t zero = 4 * s.lanes * s.nr * p->nrecs;
    p->raddr.assign(size_t(p->waves) * p->gpw * 64 * 2 * p->nh, zero | zero << 16);
    for (uint32_t b = 0; b < p->nblk; ++b)
        for (size_t i = 0; i < s.reads.size(); ++i) {
            const uint32_t src = source[b * s.reads.size() + i];
            if (src == kNone) continue;
            const uint32_t h = uint32_t(i) / (4 * s.lanes), sub = uint32_t(i) / 4 % s.lanes, d = uint32_t(i) % 4;
            const uint32_t in = b % bpg;  // block of the group: 16 columns by 4 / lanes
            const uint32_t lane = (in / 16 * s.lanes + sub) * 16 + in % 16;
            uint32_t &w = p->raddr[((size_t(b / bpg) * 64 + lane) * 2 * p->nh) + 2 * h + d / 2];
            const uint32_t addr = 4 * (s.reads[i].second * p->nrecs + src);
            w = d % 2 ? (w & 0xFFFFu) | addr << 16 : (w & 0xFFFF0000u) | addr;
        }
    mat_operands(s, &p->A);
    mat_selectors(s, &p->sel);
    if (with_nbr) neighbour_table(f, f.r - m, &p->nbr);
    p->ok = true;
    return true;
}

// The members of the tile at level m: its own blocks, then every block of
// the neighbour tiles within `rings` blocks of one of them.
static bool hold_members(const Fractal &f, const BlockShape &s, uint32_t m, uint32_t rings, HoldPlan *p,
                         std::vector<std::pair<int64_t, int64_t>> *at, std::string *msg) {
    *p = HoldPlan();
    const int64_t G = m < s.q || m > f.r ? 0 : int64_t(ipow(f.s, m - s.q));
    if (!G || rings > G || (rings == 0 && m != f.r)) {
        *msg = "q <= m <= r, at most a tile's side of rings, and none only for a tile that is the whole state";
        return false;
    }
    const uint32_t bpg = 64 / s.lanes, most = kHoldMaxWaves * 4 * bpg;
    const uint64_t nb = ipow(f.k, m - s.q);
    if (nb > most) {
        *msg = "more groups than a work-group holds";
        return false;
    }
    p->m = m;
    p->q = s.q;
    p->K = uint32_t(ipow(f.k, m));
    p->CB = s.CB;
    p->lanes = s.lanes;
    p->nr = s.nr;
    p->nh = s.nh;
    p->nblk = uint32_t(nb);
    p->ntiles = ipow(f.k, f.r - m);
    p->gens = rings ? rings * s.BS : kHoldMaxGens;
    const int64_t D = rings;
    PlaceMap block(-2 * D, G + 2 * D, nb);
    tile_places(f, m - s.q, &block, at);
    auto near = [&](int64_t x, int64_t y) {
        for (int64_t v = y - D; v <= y + D; ++v)
            for (int64_t u = x - D; u <= x + D; ++u)
                if (block.at(u, v) != kNone) return true;
        return false;
    };
    for (uint32_t d = 0; d < 8 && D; ++d)
        for (uint64_t b = 0; b < nb; ++b) {
            const int64_t X = (*at)[b].first + kDirX[d] * G, Y = (*at)[b].second + kDirY[d] * G;
            if (X < -D || Y < -D || X >= G + D || Y >= G + D || !near(X, Y)) continue;
            p->halo.push_back(d << 29 | uint32_t(b));
            at->push_back({X, Y});
        }
    p->ntot = uint32_t(at->size());
    p->groups = (p->ntot + bpg - 1) / bpg;
    // A record in consecutive dwords, one more of them where their number is a
    // multiple of four: the 32 banks of a half wavefront's read then serve
    // records at an odd distance (a bank model that agrees with the conflict
    // counters gives 5.3 -> 4.0 cycles per read on H, 6.4 -> 4.6 on the carpet).
    p->rs = s.lanes * s.nr + (s.lanes * s.nr % 4 == 0 ? 1 : 0);
    const uint64_t words = uint64_t(p->ntot + 1) * p->rs + 1;  // one record never read, one dword of zeros
    p->zero = uint32_t(4 * (words - 1));
    if (p->ntot > most || words * 4 > kHoldBuf) {
        *msg = "more groups or records than a work-group holds";
        return false;
    }
    return true;
}

// Groups per wavefront: one up to five groups, two up to 24, else four (four
// wavefronts or more share the groups, registers for several work-groups per
// CU).  One / two / four: triangle r16 at level 8 (8 groups, 97 generations)
// 515 / 409 / 441 us, at 9 (24 groups) - / 394 / 464, carpet r9 at 4 (7
// groups, 46 generations) 1,069 / 933 / 953, H r8 at 4 (5 groups, 91) 167 /
// 171 / 229, H r10 at 5 (27 groups, 46) - / 2,519 / 2,029.
static uint32_t hold_gpw(uint32_t groups) { return groups <= 5 ? 1 : (groups <= 24 ? 2 : 4); }

bool build_hold_plan(const Fractal &f, uint32_t m, uint32_t rings, uint32_t gpw, HoldPlan *p, std::string *msg,
                     bool operands) {
    BlockShape s;
    if (!pick_shape(f, &s)) {
        *msg = "no block level of this fractal fits the matrix form";
        return false;
    }
    std::vector<std::pair<int64_t, int64_t>> at;
    if (!hold_members(f, s, m, rings, p, &at, msg)) return false;
    p->gpw = gpw ? gpw : hold_gpw(p->groups);
    p->waves = (p->groups + p->gpw - 1) / p->gpw;
    if (p->waves > kHoldMaxWaves) {
        *msg = "more groups than a work-group holds";
        return false;
    }
    const int64_t E = int64_t(rings) + 1;  // looked up to a block outside the rings
    PlaceMap member(-E, int64_t(ipow(f.s, m - s.q)) + E, p->ntot);
    for (uint32_t b = 0; b < p->ntot; ++b) member.at(at[b].first, at[b].second) = b;
    const uint32_t bpg = 64 / s.lanes;
    p->raddr.assign(size_t(p->waves) * p->gpw * 64 * 2 * p->nh, p->zero | p->zero << 16);
    for (uint32_t b = 0; b < p->ntot; ++b)
        for (size_t i = 0; i < s.reads.size(); ++i) {
            const uint32_t src = member.at(at[b].first + kDirX[s.reads[i].first], at[b].second + kDirY[s.reads[i].first]);
            if (src == kNone) continue;
            const uint32_t h = uint32_t(i) / (4 * s.lanes), sub = uint32_t(i) / 4 % s.lanes, d = uint32_t(i) % 4;
            const uint32_t in = b % bpg, lane = (in / 16 * s.lanes + sub) * 16 + in % 16;
            uint32_t &w = p->raddr[((size_t(b / bpg) * 64 + lane) * 2 * p->nh) + 2 * h + d / 2];
            const uint32_t rd = s.reads[i].second;
            const uint32_t addr = 4 * (src * p->rs + rd % s.lanes * s.nr + rd / s.lanes);
            w = d % 2 ? (w & 0xFFFFu) | addr << 16 : (w & 0xFFFF0000u) | addr;
        }
    if (operands) {
        mat_operands(s, &p->A);
        mat_selectors(s, &p->sel);
    }
    if (p->halo.empty()) p->halo.push_back(0);
    p->ok = true;
    return true;
}

std::vector<HoldDims> hold_dims(const Fractal &f) {
    std::vector<HoldDims> out;
    BlockShape s;
    if (!pick_shape(f, &s)) return out;
    for (uint32_t m = s.q; m <= f.r; ++m)
        for (uint32_t rings = m == f.r ? 0 : 1; rings <= (m == f.r ? 0u : kHoldMaxRings); ++rings) {
            HoldPlan p;
            std::vector<std::pair<int64_t, int64_t>> at;
            std::string msg;
            if (!hold_members(f, s, m, rings, &p, &at, &msg)) continue;
            out.push_back({m, rings, p.groups, p.gens, 0.0});
        }
    return out;
}

// Estimated time per generation in us: a launch (4 us, and the state through
// memory once) over its generations (counted up to 24 for small states, where
// the launch is what counts, up to 12 for others: a call may ask for fewer),
// and a generation: 0.2 us for the barrier and the round through LDS and 0.02
// us per group on the busiest CU, 15 % more where a work-group has more than
// 16 groups, 75 % more beyond 30 (one or two work-groups per CU).  Fitted to
// sweeps over triangle r7 - r16, carpet r5 - r9, H r5 - r10, Vicsek r10,
// chandelier r13 and full square r12; more rings only for a gain of 5 %.
bool pick_hold(const std::vector<HoldDims> &dims, uint32_t k, const std::vector<uint32_t> &levels, uint32_t cus,
               HoldDims *out, uint32_t *gpw) {
    cus = std::max(cus, 1u);
    uint64_t cells = 0;
    for (uint32_t r : levels) cells += ipow(k, r);
    bool found = false;
    double best = 0.0;
    for (const HoldDims &d : dims) {
        uint64_t tiles = 0;
        for (uint32_t r : levels) tiles += r > d.m ? ipow(k, r - d.m) : 1;
        const double work = double((tiles + cus - 1) / cus) * d.groups;
        const double gen = std::max(0.2 + (d.groups > 30 ? 0.035 : (d.groups > 16 ? 0.023 : 0.02)) * work,
                                    0.03 * d.groups);
        const double t = (4.0 + double(cells) * 1.6e-7) / (d.rings ? std::min(d.gens, cells < 4000000 ? 24u : 12u) : 64u) +
                         gen;
        if (found && t >= (d.rings > out->rings ? 0.95 * best : best)) continue;
        found = true;
        best = t;
        *out = d;
        out->gen_us = gen;
        *gpw = hold_gpw(d.groups);
    }
    return found;
}

bool build_mat_plan(const Fractal &f, uint32_t m, uint32_t gpw, MatPlan *p, std::string *msg, bool with_nbr) {
    BlockShape s;
    if (!pick_shape(f, &s)) {
        *msg = "no block level of this fractal fits the matrix form";
        return false;
    }
    return build_mat_shape(f, s, m, gpw, p, msg, with_nbr);
}

std::vector<MatDims> mat_dims(const Fractal &f) {
    std::vector<MatDims> out;
    BlockShape s;
    if (!pick_shape(f, &s)) return out;
    for (uint32_t m = s.q; m <= f.r; ++m) {
        MatPlan p;
        std::vector<uint32_t> source;
        std::string msg;
        if (!build_ring(f, s, m, &p, &source, &msg)) break;  // larger tiles do not fit either
        const uint32_t bpg = 64 / s.lanes;
        out.push_back({m, p.groups, (p.nhalo + bpg - 1) / bpg, double(p.nhalo) / bpg});
    }
    return out;
}

// The level with the least work on the busiest CU: its tiles times the
// groups of a tile, a group of halo blocks (loaded and published, no rule and
// no store) counted half.  Of the measured best levels (triangle r14 and r16:
// 8, carpet r7: 4, r9: 5, H r9 and r10: 5, Vicsek r10: 5, chandelier r13: 7,
// each against its neighbours) it picks every one.
uint32_t pick_mat_level(const std::vector<MatDims> &dims, uint32_t k, const std::vector<uint32_t> &levels, uint32_t cus,
                        uint32_t *gpw) {
    cus = std::max(cus, 1u);
    uint32_t best = 0;
    double best_cost = 0.0;
    for (const MatDims &d : dims) {
        uint64_t tiles = 0;
        for (uint32_t r : levels) tiles += r > d.m ? ipow(k, r - d.m) : 1;
        const uint32_t g = pick_gpw(d.groups, d.hgroups, tiles, cus);
        if (!g) continue;
        const uint32_t waves = std::max((d.groups + g - 1) / g, d.hgroups);
        const double cost = double((tiles + cus - 1) / cus) * (waves * g + 0.5 * d.halo);
        if (!best || cost < best_cost) {
            best = d.m;
            best_cost = cost;
            *gpw = g;
        }
    }
    return best;
}

}  // namespace nbb
