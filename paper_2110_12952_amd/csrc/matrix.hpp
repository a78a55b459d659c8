// The compact step on the matrix cores (k_step_matrix) and its launchers.
// Included by matrix_inst.hip, which is compiled once per (BATCH, RULE, AL).
//
// Section 3's stencil procedure on the blocked approach, for compact storage,
// with the neighbour counts of a level-q block (CB consecutive compact cells,
// 16 to 64 of them) as a contraction of the block's bytes with a constant
// matrix.  A wavefront holds 64 / L blocks (a group), L lanes per block, lane
// `sub` the 16 cells from min(16 sub, CB - 16) (the last lane's cells overlap
// the lane's before where CB is no multiple of 16: both compute and store the
// same bytes, so that every load and store is a whole 16 bytes inside the
// block).  A lane's 16 bytes are loaded as they lie and are its share of the
// B operand of v_mfma_i32_16x16x64_i8 (column = lane % 16, products of quarter
// lane / 16); the operand A is block-diagonal over the blocks that share a
// column.  Row 4 g + i of result t holds the counts of cells 8 t + i (weight
// 1) and 8 t + 4 + i (weight 16) of the lanes of quarter g, so a lane
// receives the counts of its own 16 cells, eight neighbours at most in each
// nibble, in the order of its own bytes: no cross-lane move, no unpacking into
// rows and no packing back.
//
// Per tile a work-group
//   1. publishes the record of every block (the cells its neighbours need, as
//      bytes; two v_perm per dword pick them) in LDS, own blocks and
//      the blocks of the eight neighbour tiles that a block of the tile reads
//      (zeros where a neighbour tile does not exist: their loads are out of
//      the buffer's range, which ends with the aligned dword that holds the
//      state's or arena's last byte);
//   2. reads, per lane, 4 NH record dwords of the neighbouring blocks
//      (addresses from the plan), which are the B operand of the halo's
//      contraction, adds both, applies the rule (v_perm tables on four counts
//      per dword) and stores the lane's 16 next states.
// Work-groups are persistent over XCD-contiguous tile ranges; the next tile's
// loads are issued before the barrier of the current one, the records are
// double-buffered (one barrier per tile), and lanes without a block load and
// store out of the buffers' range (dropped by the hardware), so that no
// memory operation sits behind a branch.
//
// What bounds it: memory.  One generation per launch, before (the vector
// forms) and now: triangle r16 (43 MB of state, in the Infinity Cache) 17.1 ->
// 15.7 us (a copy of the state takes 12.8), carpet r9 (134 MB) 50 -> 40 (a
// copy 47), H r10 (282 MB) 161 -> 112 (a copy in this layout 105, of aligned
// blocks 99), Vicsek r10 14.6 -> 7.6.
//
// BATCH: tiles of many instances of one plan in an arena: batch tile g is
// local tile rec[4g+1] of the state of rec[4g+2] cells at byte 16 rec[4g].  An
// instance of a lower level than the tile (its cells are the first copy of
// that level in a tile) is one tile without neighbours whose blocks past the
// last cell load as zeros and are not stored.
// RULE: 0 = B3/S23, 1 = any rule (tables, or bit extract where an entry at
// eight neighbours is set).
// AL: alignment of the blocks in a state: 16 or 4 bytes, or 1 (loads then
// take five aligned dwords and v_alignbyte: measured 103 to 106 us for a copy
// of 282 MB in this layout at 27 and 49 bytes per block against 111 to 116
// with unaligned 16-byte loads and 99 for aligned blocks).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "occupancy_cache.hpp"
#include "plan.hpp"

namespace nbb {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A voffset beyond every state (k^r stays below it for every fractal the
// form takes): loads there return 0 and stores are dropped, since no resource
// covers it.
constexpr uint32_t kNowhere = 0xFFFFFE00u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t mat_rsrc(const uint8_t *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, int(bytes), 0x00020000);
}

template <int AL>
struct MatRaw {
    u32x4 v;
    uint32_t hi;  // the fifth dword (AL 1)
};
template <int AL>
__device__ __forceinline__ MatRaw<AL> mat_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    MatRaw<AL> m;
    m.hi = 0;
    if (AL == 1) {
        const uint32_t s = off & ~3u;
        m.v = __builtin_amdgcn_raw_buffer_load_b128(r, s, 0, 0);
        m.hi = __builtin_amdgcn_raw_buffer_load_b32(r, s + 16, 0, 0);
    } else {
        m.v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    }
    return m;
}
// The 16 bytes at byte off % 4 of the loaded dwords.
template <int AL>
__device__ __forceinline__ u32x4 mat_align(const MatRaw<AL> &m, uint32_t off) {
    if (AL != 1) return m.v;
    u32x4 x;
    x[0] = alignbyte(m.v[1], m.v[0], off);
    x[1] = alignbyte(m.v[2], m.v[1], off);
    x[2] = alignbyte(m.v[3], m.v[2], off);
    x[3] = alignbyte(m.hi, m.v[3], off);
    return x;
}

__device__ __forceinline__ i32x4 mat_mul(u32x4 a, u32x4 b, i32x4 c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
}
// Four results of at most 255 each as the bytes of a dword, in three
// instructions (left to itself the compiler regroups the shifts into four).
__device__ __forceinline__ uint32_t mat_bytes(i32x4 d) {
    const uint32_t lo = uint32_t(d[0]) | uint32_t(d[1]) << 8, hi = uint32_t(d[2]) | uint32_t(d[3]) << 8;
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// LDS by address: kept in a register as it is (left to itself the compiler
// keeps packed 16-bit offsets and unpacks them at every use).
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ uint32_t lds_at(const uint8_t *base, uint32_t off) {
    uint32_t a = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const uint8_t *)base)) + off;
    asm("" : "+v"(a));
    return a;
}
__device__ __forceinline__ uint32_t lds_get(uint32_t a) { return *reinterpret_cast<lds_u32 *>(uintptr_t(a)); }
__device__ __forceinline__ void lds_put(uint32_t a, uint32_t v) { *reinterpret_cast<lds_u32 *>(uintptr_t(a)) = v; }

// A record dword out of a lane's 16 cells.
__device__ __forceinline__ uint32_t mat_pick(const u32x4 &x, uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_perm(x[1], x[0], lo) | __builtin_amdgcn_perm(x[3], x[2], hi);
}

// Next states of four cells: n their live-neighbour counts, o the cells.
template <int RULE>
__device__ __forceinline__ uint32_t mat_rule(uint32_t n, uint32_t o, uint32_t rule, const RuleTables &RT, bool tables) {
    if (RULE == 0) return __builtin_amdgcn_perm(0u, 0x01000000u, n | o);
    if (tables) {  // uniform
        const uint32_t born = __builtin_amdgcn_perm(RT.born_hi, RT.born_lo, n);
        const uint32_t surv = __builtin_amdgcn_perm(RT.surv_hi, RT.surv_lo, n);
        const uint32_t smask = __builtin_amdgcn_perm(0u, 0x0000FF00u, o);  // 0xFF where alive
        return (surv & smask) | (born & ~smask);
    }
    const uint32_t I = n + (o << 4);  // v_bfe takes its offset from the low 5 bits
    uint32_t v = __builtin_amdgcn_ubfe(rule, I, 1);
#pragma unroll
    for (int c = 1; c < 4; ++c) v |= __builtin_amdgcn_ubfe(rule, I >> (8 * c), 1) << (8 * c);
    return v;
}

template <int AL, int NR, int NH, int GPW, bool BATCH, int RULE>
__global__ __launch_bounds__(64 * kMatMaxWaves) void k_step_matrix(MatParams E, const uint8_t *__restrict__ in,
                                                                   uint8_t *__restrict__ out, uint32_t rule,
                                                                   const uint32_t *__restrict__ rec) {
    extern __shared__ __align__(16) uint8_t lds_m[];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    const XcdRange R64 = xcd_range(blockIdx.x, gridDim.x, E.ntiles);
    const uint32_t first = uint32_t(R64.first), end = uint32_t(R64.end), step = uint32_t(R64.step);
    if (first >= end) return;
    // the work-group's tiles are first + i step; loads past the last read it again
    const uint32_t last = first + (end - 1 - first) / step * step;
    auto tile = [&](uint32_t i) -> uint32_t { return min(first + i * step, last); };

    // This lane's share of its wavefront's groups: quarter = lane / 16 holds
    // lane `sub` of block in / of the group's 64 / L blocks.
    const uint32_t L = E.lanes, quarter = lane >> 4, col = lane & 15;
    const uint32_t sub = quarter & (L - 1), bpg = 64 / L;
    const uint32_t slot = (L == 4 ? 0u : (L == 2 ? quarter >> 1 : quarter)) * 16 + col;
    const uint32_t coff = mat_first_cell(sub, E.CB);
    const bool edge = (rule >> 31) != 0;
    const uint8_t *A8 = reinterpret_cast<const uint8_t *>(E.A) + 16 * lane;
    auto operand = [&](uint32_t off) -> u32x4 { return *reinterpret_cast<const u32x4 *>(A8 + off); };
    u32x4 Aself[2], Ahalo[NH][2];
    uint32_t sel[NR][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) Aself[t] = operand(mat_self_off(NH, edge, t));
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int t = 0; t < 2; ++t) Ahalo[h][t] = operand(mat_halo_off(NH, edge, h, t));
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int d = 0; d < 2; ++d) sel[t][d] = E.sel[2 * (4 * t + sub) + d];
    const uint32_t rstride = 4 * L * E.nrecs;  // from one record result's dwords to the next's
    uint32_t voff[GPW], waddr[GPW], raddr[GPW][2 * NH];
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const uint32_t g = wave * GPW + u, b = g * bpg + slot;
        const bool ok = b < E.nblk;
        voff[u] = ok ? b * E.CB + coff : kNowhere;
        waddr[u] = 4 * (sub * E.nrecs + (ok ? b : E.nrecs - 1));
#pragma unroll
        for (int d = 0; d < 2 * NH; ++d) raddr[u][d] = E.raddr[(g * 64 + lane) * (2 * NH) + d];
    }
    const uint32_t h = wave * bpg + slot;
    const bool hlane = h < E.nhalo;
    const uint32_t hitem = E.halo[hlane ? h : 0u];
    const uint32_t hoff = (hitem & 0x1FFFFFFFu) * E.CB + coff, hdir = hitem >> 29;
    uint32_t hwaddr = 4 * (sub * E.nrecs + (hlane ? E.nblk + h : E.nrecs - 1));
    if (tid < 2) *reinterpret_cast<uint32_t *>(lds_m + tid * E.buf_bytes + 4 * (L * NR * E.nrecs)) = 0;

    const RuleTables RT = rule_tables(rule);
    const bool tables = RT.perm || edge;

    // A tile's loads.
    struct Pending {
        MatRaw<AL> raw[GPW], hraw;
        uint32_t hpos;    // halo block's offset in its state
        uint32_t phase;   // the tile's first byte in its dword
        uint8_t *dst;     // the tile's output
        uint32_t bytes;   // and its length
    } P;
    // A tile's record, read one tile before its loads.
    struct Where {
        uint32_t base16, local, cells;
    };
    auto where = [&](uint32_t t) -> Where {
        if (!BATCH) return {0, t, 0};
        const uint32_t *r = rec + 4 * uint64_t(t);
        return {r[0], r[1], r[2]};
    };
    auto prefetch = [&](const Where &w, uint32_t nt) {
        const uint64_t base = uint64_t(w.base16) << 4;
        const uint32_t local = w.local, cells = w.cells;
        const uint8_t *src = in + base;
        const uint64_t room = (E.limit - base + 3) & ~uint64_t(3);  // whole dwords
        const uint32_t lim = room > kNowhere ? kNowhere : uint32_t(room);
        const uint32_t toff = local * E.K, tal = toff & ~3u;
        P.phase = toff & 3;
        P.dst = out + base + toff;
        P.bytes = BATCH ? min(E.K, cells) : E.K;
        const __amdgpu_buffer_rsrc_t own = mat_rsrc(src + tal, lim - tal), all = mat_rsrc(src, lim);
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            const uint32_t off = BATCH && voff[u] >= P.bytes ? kNowhere : voff[u];
            P.raw[u] = mat_load<AL>(own, AL == 1 ? off + P.phase : off);
        }
        P.hpos = hlane && nt != kOutside ? nt * E.K + hoff : kNowhere;
        P.hraw = mat_load<AL>(all, P.hpos);
    };
    auto entry = [&](uint32_t t) -> uint32_t { return E.nbr[uint64_t(t) * 8 + hdir]; };

    uint32_t nt = entry(tile(1));
    Where wh = where(tile(1));
    prefetch(where(tile(0)), entry(tile(0)));
    // As many stores after the first tile's loads as after any later tile's
    // (into an empty range, so dropped): the compiler then counts the same
    // outstanding operations on both ways into the loop and waits for the
    // loads alone, not for the stores behind them.
#pragma unroll
    for (int u = 0; u < GPW; ++u)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{0, 0, 0, 0}, mat_rsrc(P.dst, 0), voff[u], 0, 0);
    int32_t delta = int32_t(E.buf_bytes);  // to the other record buffer
    for (uint32_t i = 0;; ++i) {
        // step 1: the records
        u32x4 x[GPW];
        const i32x4 zero = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            x[u] = mat_align<AL>(P.raw[u], AL == 1 ? voff[u] + P.phase : 0u);
#pragma unroll
            for (int t = 0; t < NR; ++t)
                *reinterpret_cast<uint32_t *>(lds_m + waddr[u] + t * rstride) = mat_pick(x[u], sel[t][0], sel[t][1]);
        }
        const u32x4 hx = mat_align<AL>(P.hraw, P.hpos);
#pragma unroll
        for (int t = 0; t < NR; ++t)
            *reinterpret_cast<uint32_t *>(lds_m + hwaddr + t * rstride) = mat_pick(hx, sel[t][0], sel[t][1]);
        const __amdgpu_buffer_rsrc_t gout = mat_rsrc(P.dst, P.bytes);
        // the next tile's loads, the neighbour tile of the one after it
        const uint32_t nt1 = nt;
        const Where wh1 = wh;
        nt = entry(tile(i + 2));
        wh = where(tile(i + 2));
        prefetch(wh1, nt1);
        __syncthreads();
        // step 2: counts and rule
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            i32x4 d0 = mat_mul(Aself[0], x[u], zero), d1 = mat_mul(Aself[1], x[u], zero);
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                u32x4 r;
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const uint32_t a = raddr[u][2 * hh + d];
                    r[2 * d] = *reinterpret_cast<const uint32_t *>(lds_m + (a & 0xFFFFu));
                    r[2 * d + 1] = *reinterpret_cast<const uint32_t *>(lds_m + (a >> 16));
                }
                d0 = mat_mul(Ahalo[hh][0], r, d0);
                d1 = mat_mul(Ahalo[hh][1], r, d1);
            }
            const uint32_t c0 = mat_bytes(d0), c1 = mat_bytes(d1);
            u32x4 w;
            w[0] = mat_rule<RULE>(c0 & 0x0F0F0F0Fu, x[u][0], rule, RT, tables);
            w[1] = mat_rule<RULE>((c0 >> 4) & 0x0F0F0F0Fu, x[u][1], rule, RT, tables);
            w[2] = mat_rule<RULE>(c1 & 0x0F0F0F0Fu, x[u][2], rule, RT, tables);
            w[3] = mat_rule<RULE>((c1 >> 4) & 0x0F0F0F0Fu, x[u][3], rule, RT, tables);
            __builtin_amdgcn_raw_buffer_store_b128(w, gout, voff[u], 0, 0);
        }
        if (first + (i + 1) * step >= end) break;
        // the other record buffer: its reads ended before the barrier above
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            waddr[u] += delta;
#pragma unroll
            for (int d = 0; d < 2 * NH; ++d) raddr[u][d] += uint32_t(delta) * 0x10001u;
        }
        hwaddr += delta;
        delta = -delta;
    }
}

// Persistent launch: as many work-groups as can be resident at once, capped
// by the tiles.
template <int AL, int NR, int NH, int GPW, bool BATCH, int RULE>
static hipError_t launch_matrix_t(const MatParams &E, const uint8_t *in, uint8_t *out, uint32_t rule,
                                  const uint32_t *rec, int cu_count, hipStream_t st) {
    const uint32_t lds = 2 * E.buf_bytes, threads = 64 * E.waves;
    static OccupancyCache cache;
    int per_cu = 0;
    hipError_t e = cache.get(lds, threads, &per_cu, [&](int *n) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, k_step_matrix<AL, NR, NH, GPW, BATCH, RULE>, int(threads),
                                                            lds);
    });
    if (e != hipSuccess) return e;
    // Work-groups per CU: the fewest tile rounds times work-groups (the tiles
    // the busiest CU works through) that leaves six wavefronts on a CU, fewer
    // work-groups first.  Triangle r16 (6,561 tiles, two wavefronts each) with
    // 2 / 3 / 4 / 6 / 8: 17.6 / 15.9 / 15.8 / 17.4 / 17.0 us; Vicsek r10
    // (3,125 tiles) 7.2 / 6.5 / 6.7 / 7.5 / 8.5; H r10 with 1 / 2: 115.6 / 117.9.
    uint64_t best = 0;
    int use = per_cu;
    for (int c = 1; c <= per_cu; ++c) {
        if (c < per_cu && uint32_t(c) * E.waves < 6) continue;
        const uint64_t wgs = uint64_t(c) * cu_count, work = (E.ntiles + wgs - 1) / wgs * c;
        if (best && work >= best) continue;
        best = work;
        use = c;
    }
    const uint64_t grid = std::min<uint64_t>(uint64_t(use) * cu_count, E.ntiles);
    if (!grid) return hipSuccess;
    hipLaunchKernelGGL((k_step_matrix<AL, NR, NH, GPW, BATCH, RULE>), dim3(uint32_t(grid)), dim3(threads), lds, st, E,
                       in, out, rule, rec);
    return hipGetLastError();
}

// Several generations of the matrix form per launch (HoldParams): a work-group
// per tile holds the tile's blocks and those around it in registers, 16 cells
// per lane as above, for all of the launch's generations; only the records go
// through LDS (double-buffered, one barrier per generation).  The state is
// read and written once per launch instead of once per generation, and a
// generation of a small state costs a barrier instead of a launch.
// What bounds it: instruction issue.  A group's generation is 16 + 3 NR vector
// instructions and four MFMAs of 16 cycles, and on the workloads the vector
// and the matrix pipes are busy for about 85 % of the time together (H r10,
// nine generations per launch: 237 + 110 of 410 us), the LDS for half of it.
// Per launch: triangle r16 33.2 us for 8 generations (one per launch: 126),
// carpet r9 185 us for 9 (360), H r10 419 us for 9 (1,008).  Measured and not
// kept: every LDS read of a generation issued before the first use (H r10
// 518 -> 547 us for 10 generations: registers), records picked by a third
// contraction (548).
//   BUF: the second record buffer's offset (an instruction offset).
//   AL 0: the state at one bit per cell (in and out are words, E.limit their
//   bytes; not BATCH).  A lane's 16 bits come out of two words and spread to
//   bytes once per launch; the next states are gathered as the tile's words
//   in LDS, and the words shared with the neighbouring tiles are stored by an
//   atomic AND and OR of the tile's own bits.
//   BATCH: rec as above; word 3 of a tile's record indexes steps_of, the
//   generations n its instance takes in the whole call (steps_of NULL: every
//   instance takes `gens` now).  mode says which of a call's launches it is:
//     kHoldMost  number `launch` (from 0) of those that take all but the last
//                generation, in as few launches as E.gens allows plus one where
//                their number would not have the parity of n - 1 (launches
//                alternate the buffers); nothing past an instance's own
//     kHoldLast  the last generation: from `in` to `out` for odd n, from `out`
//                to `in` for even n
//     kHoldWhole  number `launch` of those that take all n (tiles that are
//                whole instances): in place in `in` for even n, for odd n from
//                `in` to `out` by the first and in place there by the others,
//                so that the other arena is untouched
//   Not BATCH, kHoldWhole (the state is one tile): the whole call in one
//   launch, generation `gens` to out if odd, else to in, and the generation
//   before it to the other (every load has ended before the first barrier).
template <int AL, int NR, int NH, int GPW, int BUF, bool BATCH, int RULE>
__global__ __launch_bounds__(64 * kHoldMaxWaves) void k_step_hold(HoldParams E, uint8_t *in, uint8_t *out,
                                                                  uint32_t rule, uint32_t gens,
                                                                  const uint32_t *__restrict__ rec,
                                                                  const uint32_t *__restrict__ steps_of,
                                                                  uint32_t launch, uint32_t mode) {
    extern __shared__ __align__(16) uint8_t lds_m[];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    // work-groups go round-robin over the 8 XCDs: each takes consecutive tiles
    const uint32_t xcd = blockIdx.x & 7, share = E.ntiles >> 3, more = E.ntiles & 7;
    const uint32_t t = xcd * share + min(xcd, more) + (blockIdx.x >> 3);
    uint64_t base = 0;
    uint32_t local = t, bytes = E.K;
    if (BATCH) {
        const uint32_t *r = rec + 4 * uint64_t(t);
        base = uint64_t(r[0]) << 4;
        local = r[1];
        bytes = min(E.K, r[2]);
        if (steps_of) {
            const uint32_t n = steps_of[r[3]];
            if (mode == kHoldLast) {
                if (n == 0) return;
                gens = 1;
                if (!(n & 1)) {
                    uint8_t *o = out;
                    out = in;
                    in = o;
                }
            } else {
                const uint32_t T = mode == kHoldWhole ? n : max(n, 1u) - 1;
                uint32_t L = T / E.gens + (T % E.gens != 0);
                if (mode == kHoldMost) L += (L ^ T) & 1;
                if (launch >= L) return;
                gens = T / L + (launch < T % L ? 1u : 0u);
                if (mode == kHoldWhole && !(n & 1)) out = in;
                if (mode == kHoldWhole && launch) in = out;
            }
        }
    }
    const uint32_t L = E.lanes, quarter = lane >> 4, col = lane & 15;
    const uint32_t sub = quarter & (L - 1), bpg = 64 / L;
    const uint32_t slot = (L == 4 ? 0u : (L == 2 ? quarter >> 1 : quarter)) * 16 + col;
    const uint32_t coff = mat_first_cell(sub, E.CB);
    const uint8_t *src = in + base;
    const uint64_t room = (E.limit - base + 3) & ~uint64_t(3);
    const __amdgpu_buffer_rsrc_t all = mat_rsrc(src, room > kNowhere ? kNowhere : uint32_t(room));
    const uint32_t toff = local * E.K;
    // the blocks: own ones, those of the neighbour tiles, none
    uint32_t soff[GPW], live[GPW];
    u32x4 x[GPW];
    MatRaw<AL> raw[GPW];
    uint32_t pos[GPW];
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const uint32_t b = (wave * GPW + u) * bpg + slot;
        // (a whole tile's lanes all own theirs)
        const bool own = b < E.nblk && mat_lane_owns(b, E.CB, BATCH ? coff : 0u, bytes), ring = b >= E.nblk && b < E.ntot;
        const uint32_t item = E.halo[ring ? b - E.nblk : 0u];
        const uint32_t nt = E.nbr[uint64_t(t) * 8 + (item >> 29)];
        soff[u] = own ? b * E.CB + coff : kNowhere;
        pos[u] = own ? toff + b * E.CB + coff
                     : (ring && nt != kOutside ? nt * E.K + (item & 0x1FFFFFFFu) * E.CB + coff : kNowhere);
        live[u] = pos[u] != kNowhere ? 0xFFFFFFFFu : 0u;
        if (AL == 0) {
            const uint32_t w = pos[u] == kNowhere ? kNowhere : pos[u] >> 5 << 2;
            raw[u].v[0] = __builtin_amdgcn_raw_buffer_load_b32(all, w, 0, 0);
            raw[u].hi = __builtin_amdgcn_raw_buffer_load_b32(all, w + 4, 0, 0);
        } else {
            raw[u] = mat_load<AL>(all, pos[u]);
        }
    }
    const bool edge = (rule >> 31) != 0;
    const uint8_t *A8 = reinterpret_cast<const uint8_t *>(E.A) + 16 * lane;
    auto operand = [&](uint32_t off) -> u32x4 { return *reinterpret_cast<const u32x4 *>(A8 + off); };
    u32x4 Aself[2], Ahalo[NH][2];
    uint32_t sel[NR][2];
#pragma unroll
    for (int k = 0; k < NR; ++k)
#pragma unroll
        for (int d = 0; d < 2; ++d) sel[k][d] = E.sel[2 * (4 * k + sub) + d];
#pragma unroll
    for (int k = 0; k < 2; ++k) Aself[k] = operand(mat_self_off(NH, edge, k));
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int k = 0; k < 2; ++k) Ahalo[h][k] = operand(mat_halo_off(NH, edge, h, k));
    uint32_t waddr[GPW], raddr[GPW][4 * NH];
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const uint32_t g = wave * GPW + u, b = g * bpg + slot;
        waddr[u] = lds_at(lds_m, 4 * (min(b, E.ntot) * E.rs + sub * NR));
#pragma unroll
        for (int d = 0; d < 2 * NH; ++d) {
            const uint32_t a = E.raddr[(g * 64 + lane) * (2 * NH) + d];
            raddr[u][2 * d] = lds_at(lds_m, a & 0xFFFFu);
            raddr[u][2 * d + 1] = lds_at(lds_m, a >> 16);
        }
    }
    if (tid < 2) *reinterpret_cast<uint32_t *>(lds_m + tid * BUF + E.zero) = 0;
    const RuleTables RT = rule_tables(rule);
    const bool tables = RT.perm || edge;
    const bool all_live = (wave * GPW + GPW) * bpg <= E.nblk && (wave * GPW + GPW) * bpg * E.CB <= bytes;
    // A wavefront without a block (of an instance below the tile level) leaves
    // its blocks' records at zero and only keeps the barriers.
    if (BATCH && wave * GPW * bpg * E.CB >= bytes && (wave * GPW + GPW) * bpg <= E.nblk) {
#pragma unroll
        for (int u = 0; u < GPW; ++u)
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                lds_put(waddr[u] + 4 * k, 0);
                lds_put(waddr[u] + BUF + 4 * k, 0);
            }
        for (uint32_t g = 0; g < gens; ++g) __syncthreads();
        return;
    }
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        if (AL == 0) {
            const uint32_t bits = __builtin_amdgcn_alignbit(raw[u].hi, raw[u].v[0], pos[u]);
#pragma unroll
            for (int d = 0; d < 4; ++d) x[u][d] = nibble_to_bytes((bits >> (4 * d)) & 15u);
        } else {
            x[u] = mat_align<AL>(raw[u], pos[u]);
        }
    }

    auto generation = [&](auto parity) {
        constexpr int P = decltype(parity)::value * BUF;
        const i32x4 zero = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < GPW; ++u)
#pragma unroll
            for (int k = 0; k < NR; ++k)
                lds_put(waddr[u] + P + 4 * k, mat_pick(x[u], sel[k][0], sel[k][1]));
        __syncthreads();
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            i32x4 d0 = mat_mul(Aself[0], x[u], zero), d1 = mat_mul(Aself[1], x[u], zero);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                u32x4 r;
#pragma unroll
                for (int d = 0; d < 4; ++d) r[d] = lds_get(raddr[u][4 * h + d] + P);
                d0 = mat_mul(Ahalo[h][0], r, d0);
                d1 = mat_mul(Ahalo[h][1], r, d1);
            }
            const uint32_t c0 = mat_bytes(d0), c1 = mat_bytes(d1);
            x[u][0] = mat_rule<RULE>(c0 & 0x0F0F0F0Fu, x[u][0], rule, RT, tables);
            x[u][1] = mat_rule<RULE>((c0 >> 4) & 0x0F0F0F0Fu, x[u][1], rule, RT, tables);
            x[u][2] = mat_rule<RULE>(c1 & 0x0F0F0F0Fu, x[u][2], rule, RT, tables);
            x[u][3] = mat_rule<RULE>((c1 >> 4) & 0x0F0F0F0Fu, x[u][3], rule, RT, tables);
        }
        // blocks that do not exist stay dead (uniform branch)
        if (!all_live)
#pragma unroll
            for (int u = 0; u < GPW; ++u)
#pragma unroll
                for (int d = 0; d < 4; ++d) x[u][d] &= live[u];
    };
    uint8_t *before = nullptr;
    if (!BATCH && AL != 0 && mode == kHoldWhole) {
        before = gens & 1 ? in : out;
        if (!(gens & 1)) out = in;
        if (gens < 2) before = nullptr;  // (it is there already)
    }
    auto keep = [&](uint32_t g) {  // the generation before the last (uniform)
        if (BATCH || AL == 0 || !before || g + 1 != gens) return;
        const __amdgpu_buffer_rsrc_t r = mat_rsrc(before, bytes);
#pragma unroll
        for (int u = 0; u < GPW; ++u) __builtin_amdgcn_raw_buffer_store_b128(x[u], r, soff[u], 0, 0);
    };
    for (uint32_t g = 0; g < gens; g += 2) {
        keep(g);
        generation(std::integral_constant<int, 0>());
        if (g + 1 < gens) {
            keep(g + 1);
            generation(std::integral_constant<int, 1>());
        }
    }
    if (AL == 0) {
        // the tile's words in LDS (over the records), then to memory
        uint32_t *words = reinterpret_cast<uint32_t *>(lds_m);
        const uint32_t ph = toff & 31, nw = (ph + E.K + 31) >> 5;
        __syncthreads();
        for (uint32_t w = tid; w < nw; w += 64 * E.waves) words[w] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            if (soff[u] == kNowhere) continue;
            uint32_t bits = 0;
#pragma unroll
            for (int d = 0; d < 4; ++d) bits |= (x[u][d] * 0x01020408u >> 24) << (4 * d);
            const uint32_t at = ph + soff[u];
            const uint64_t v = uint64_t(bits) << (at & 31);
            atomicOr(words + (at >> 5), uint32_t(v));
            if (v >> 32) atomicOr(words + (at >> 5) + 1, uint32_t(v >> 32));
        }
        __syncthreads();
        uint32_t *dst = reinterpret_cast<uint32_t *>(out) + (toff >> 5);
        for (uint32_t w = tid; w < nw; w += 64 * E.waves) {
            const uint32_t lo = w == 0 ? ph : 0u, hi = min(ph + E.K - 32 * w, 32u);  // the tile's bits of the word
            const uint32_t mask = (hi == 32 ? 0xFFFFFFFFu : (1u << hi) - 1) & ~((1u << lo) - 1);
            if (mask == 0xFFFFFFFFu) {
                dst[w] = words[w];
            } else {
                atomicAnd(dst + w, ~mask);
                atomicOr(dst + w, words[w] & mask);
            }
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t gout = mat_rsrc(out + base + toff, bytes);
#pragma unroll
    for (int u = 0; u < GPW; ++u) __builtin_amdgcn_raw_buffer_store_b128(x[u], gout, soff[u], 0, 0);
}

template <int AL, int NR, int NH, int GPW, int BUF, bool BATCH, int RULE>
static hipError_t launch_hold_t(const HoldParams &E, uint8_t *in, uint8_t *out, uint32_t rule, uint32_t gens,
                                const uint32_t *rec, const uint32_t *steps_of, uint32_t launch, uint32_t mode,
                                hipStream_t st) {
    if (!E.ntiles) return hipSuccess;
    uint32_t lds = hold_lds_bytes(E.zero);  // (BUF is hold_buf(E.zero))
    if (AL == 0) lds = std::max(lds, 4 * ((E.K + 62) / 32 + 1));
    hipLaunchKernelGGL((k_step_hold<AL, NR, NH, GPW, BUF, BATCH, RULE>), dim3(E.ntiles), dim3(64 * E.waves), lds, st, E,
                       in, out, rule, gens, rec, steps_of, launch, mode);
    return hipGetLastError();
}

// The instantiation for a plan: exact operand counts (the kernel's operand
// offsets follow them).
template <int AL, bool BATCH, int RULE>
static hipError_t launch_matrix_shape(const MatParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, const uint8_t *in,
                                      uint8_t *out, uint32_t rule, const uint32_t *rec, int cu_count, hipStream_t st) {
#define NBB_MAT_CASE(R, H, G)           \
    if (nr == R && nh == H && gpw == G) \
    return launch_matrix_t<AL, R, H, G, BATCH, RULE>(E, in, out, rule, rec, cu_count, st)
#define NBB_MAT_CASES(R, H)  \
    NBB_MAT_CASE(R, H, 1);   \
    NBB_MAT_CASE(R, H, 2);   \
    NBB_MAT_CASE(R, H, 4)
    NBB_MAT_CASES(1, 1);
    NBB_MAT_CASES(2, 1);
    NBB_MAT_CASES(3, 1);
    NBB_MAT_CASES(1, 2);
    NBB_MAT_CASES(2, 2);
    NBB_MAT_CASES(3, 2);
#undef NBB_MAT_CASES
#undef NBB_MAT_CASE
    return hipErrorInvalidValue;
}
template <int AL, bool BATCH, int RULE>
static hipError_t launch_hold_shape(const HoldParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, uint8_t *in,
                                    uint8_t *out, uint32_t rule, uint32_t gens, const uint32_t *rec,
                                    const uint32_t *steps_of, uint32_t launch, uint32_t mode, hipStream_t st) {
    const bool small = hold_buf(E.zero) == kHoldBufSmall;
#define NBB_HOLD_CASE(R, H, G)                                                                                    \
    if (nr == R && nh == H && gpw == G)                                                                           \
    return small ? launch_hold_t<AL, R, H, G, int(kHoldBufSmall), BATCH, RULE>(E, in, out, rule, gens, rec,       \
                                                                               steps_of, launch, mode, st)      \
                 : launch_hold_t<AL, R, H, G, int(kHoldBuf), BATCH, RULE>(E, in, out, rule, gens, rec, steps_of,  \
                                                                          launch, mode, st)
#define NBB_HOLD_CASES(R, H) \
    NBB_HOLD_CASE(R, H, 1);  \
    NBB_HOLD_CASE(R, H, 2);  \
    NBB_HOLD_CASE(R, H, 4)
    NBB_HOLD_CASES(1, 1);
    NBB_HOLD_CASES(2, 1);
    NBB_HOLD_CASES(3, 1);
    NBB_HOLD_CASES(1, 2);
    NBB_HOLD_CASES(2, 2);
    NBB_HOLD_CASES(3, 2);
#undef NBB_HOLD_CASES
#undef NBB_HOLD_CASE
    return hipErrorInvalidValue;
}

}  // namespace nbb
