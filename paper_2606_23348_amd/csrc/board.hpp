// board.hpp -- one environment's board in LDS and what a wave does to it:
// map generation, the moves of a turn, the random legal actor
// (arxiv 2606.23348, Sections III and IV).
#pragma once

#include "device.hpp"
#include "internal.hpp"

namespace gen {

// ---------------------------------------------------------------- LDS carve-up
// Per env, S = padded cells per row (multiple of 16):
//   owner int8 [S] | type uint8 [S] | armyc uint8 [S] + 16
//   obm   u64 [P][16]                 (cells owned by each player)
//   vis   u64 [P][16]                 (visible cell bitmaps)
//   gbm   u64 [3][16] + int32 [8]      (passable and army > 1 bitmaps; map generator scratch; army totals)
//         + u64 [4]                    (the actor's Philox block, computed early)
//   army  int32 [S]                   (last: dead after growth, when the dense
//                                      observation writer stages its bytes there and in what follows)
struct Lds {
    int32_t *army;
    int8_t *owner;
    uint8_t *type;
    uint8_t *armyc;
    uint64_t *obm, *vis, *gbm;
};

__device__ __forceinline__ Lds carve(uint8_t *smem, const Geom &g)
{
    Lds L;
    uint32_t o = 0;
    L.owner = reinterpret_cast<int8_t *>(smem + o); o += g.S;
    L.type = smem + o; o += g.S;
    L.armyc = smem + o; o += g.S + 16;
    L.obm = reinterpret_cast<uint64_t *>(smem + o); o += 8 * 16 * g.P;
    L.vis = reinterpret_cast<uint64_t *>(smem + o); o += 8 * 16 * g.P;
    L.gbm = reinterpret_cast<uint64_t *>(smem + o); o += 8 * 16 * 3 + 32 + 32;
    L.army = reinterpret_cast<int32_t *>(smem + o);
    return L;
}

// ---------------------------------------------------------------- map generation
// The generator works on row bitmaps: lane r holds row r of the board as 32
// bits (bit = column), so the 4-neighbour step is two shifts and two wave
// shifts, a Manhattan ball is one mask per row, and a uniform pick is a
// prefix sum over the rows' populations and one ballot.  It is bound by
// vector issue and, in small batches, by its serial chain.  A Philox4x64
// block costs a wave about 2,000 clocks and gives every lane 8 draws, so
// the draws after the cells' come from the block round that drew the last
// cells, one per lane, rather than from a block each.  Measured with the
// observation: 65,536 maps of 24x24 1,229 -> 178 us, 512 official 23x23
// maps 55 -> 18 us (before: cell bitmaps of 64-bit words in LDS, a Philox
// block per draw, the plain cells balloted again for every city).

// Bits [lane W, lane W + W) of a cell bitmap in LDS: row `lane` of the board
// (0 past the last row).  Reads at most one dword past the bitmap's last.
__device__ __forceinline__ uint32_t row_bits(const uint32_t *bm, uint32_t rowm, const Geom &g)
{
    const int o = (rowm ? lane_id() : 0) * g.W;
    const uint64_t v = (uint64_t)bm[o >> 5] | ((uint64_t)bm[(o >> 5) + 1] << 32);
    return (uint32_t)(v >> (o & 31)) & rowm;
}

// One cell and its place: row and column (wave-uniform).
struct RowCol { int r, c; };

// The cell at position idx (row-major order) of a row bitmap whose rows'
// inclusive population prefix is `incl`; idx < population.
__device__ __forceinline__ RowCol row_select(uint32_t row, uint32_t incl, uint32_t idx)
{
    const uint32_t excl = incl - (uint32_t)__popc(row);
    const int r = __builtin_ctzll(ballot(excl <= idx && idx < incl));
    const uint32_t word = (uint32_t)readlane((int)row, r), t = idx - (uint32_t)readlane((int)excl, r);
    const bool hit = lane_id() < 32 && ((word >> (lane_id() & 31)) & 1u) && __builtin_amdgcn_mbcnt_lo(word, 0u) == t;
    return {r, __builtin_ctzll(ballot(hit))};
}

// Cells within BFS distance r of a cell (4-neighbour steps over `pass`).
__device__ uint32_t row_reach(uint32_t pass, RowCol src, int radius)
{
    uint32_t cw = lane_id() == src.r ? 1u << src.c : 0u;
    for (int r = 1; r <= radius; ++r) {
        const uint32_t n = (cw | (cw << 1) | (cw >> 1) | wave_shr1(cw, 0u) | wave_shl1(cw, 0u)) & pass;
        const bool changed = ballot(n != cw) != 0ull;
        cw = n;
        if (!changed) break;
    }
    return cw;
}

// The 4-connected component of a cell: one row up and down per round, and
// each row's runs filled at once (adding the seeds to the passable bits
// carries through a run to its end; the other direction on reversed rows).
__device__ uint32_t row_component(uint32_t pass, RowCol src)
{
    const uint32_t rp = __brev(pass);
    uint32_t cw = lane_id() == src.r ? 1u << src.c : 0u;
    for (;;) {
        uint32_t n = (cw | wave_shr1(cw, 0u) | wave_shl1(cw, 0u)) & pass;
        n |= pass & ~(pass + n);
        uint32_t b = __brev(n);
        b |= rp & ~(rp + b);
        n = __brev(b);
        if (ballot(n != cw) == 0ull) return n;
        cw = n;
    }
}

// Section IV-A generator family (readings R14, R18).  Executed by the whole
// wave with uniform control flow; every random choice is a Philox draw
// indexed exactly as the generator's draw order defines.  Leaves the grid in
// LDS and the scalars in `s`.
__device__ void mapgen_wave(const Lds &L, const Geom &g, const GenParamsDev &prm, uint64_t seed, uint64_t env_id,
                            uint32_t episode, EnvScalars &s)
{
    const int lane = lane_id();
    const int HW = g.HW, W = g.W, H = g.H;
    const uint32_t rowm = lane < H ? (W == 32 ? ~0u : (1u << W) - 1u) : 0u;     // the columns of row `lane`
    uint8_t *mt8 = reinterpret_cast<uint8_t *>(L.gbm);                           // mountain bitmap, a byte per block
    int gpv = 0;                                                                 // lane i: cell of general i
    bool placed = false;

    // LDS rows of a map without owners: types from the mountain bitmap
    auto blank = [&](bool mountains) {
        for (int q = lane; q * 4 < g.S; q += kWave) {
            const uint32_t m4 = mountains ? ((uint32_t)mt8[q >> 1] >> ((q & 1) * 4)) & 0xFu : 0u;
            reinterpret_cast<uint32_t *>(L.type)[q] = spread4(m4) * (uint32_t)MOUNTAIN;
            reinterpret_cast<uint32_t *>(L.owner)[q] = 0xFFFFFFFFu;
            reinterpret_cast<uint4 *>(L.army)[q] = make_uint4(0u, 0u, 0u, 0u);
        }
        wave_sync();
    };

    for (int attempt = 0; attempt < 128 && !placed; ++attempt) {
        const uint32_t T = attempt < 64 ? prm.thresh : 0u;
        // G1: one draw per cell; a Philox block gives the draws of 8 cells.
        uint32_t v[8];
        int base = 0;                                  // block of lane 0 in the last round
        for (;; base += kWave) {
            const int b = base + lane;
            uint64_t x0 = env_id, x1 = episode, x2 = (uint64_t)attempt, x3 = (uint64_t)b;
            philox4x64_10(x0, x1, x2, x3, seed, DOM_MAPGEN);
            v[0] = (uint32_t)x0; v[1] = (uint32_t)(x0 >> 32); v[2] = (uint32_t)x1; v[3] = (uint32_t)(x1 >> 32);
            v[4] = (uint32_t)x2; v[5] = (uint32_t)(x2 >> 32); v[6] = (uint32_t)x3; v[7] = (uint32_t)(x3 >> 32);
            uint32_t m8 = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) m8 |= (v[t] < T ? 1u : 0u) << t;
            const int left = HW - b * 8;
            if (left < 8) m8 &= left > 0 ? (1u << left) - 1u : 0u;
            if (b * 8 < g.S) mt8[b] = (uint8_t)m8;
            if ((base + kWave) * 8 >= HW) break;
        }
        // The draws after the cells': draw HW + t on lane t.  The last
        // round's blocks hold the next ones (up to 512).  A longer sequence
        // is drawn 64 at a time, each lane the block of its own draw: before
        // the cities of a board that leaves fewer than the 32 draws that
        // come before them, and between the cities.
        uint32_t D = 0, j = 0, dn = (uint32_t)min(kWave, (base + kWave) * 8 - HW);   // draws j .. dn - 1 are on hand
        uint32_t d0 = (uint32_t)HW;                    // first draw of the window
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t x = shfl32(v[t], ((HW + lane) >> 3) - base);
            if (((HW + lane) & 7) == t) D = x;
        }
        auto refill = [&]() {
            d0 += j;
            j = 0;
            dn = kWave;
            D = draw32(seed, DOM_MAPGEN, env_id, episode, (uint64_t)attempt, d0 + (uint32_t)lane);
        };
        auto draw = [&]() -> uint32_t { return (uint32_t)readlane((int)D, (int)(j++)); };
        if (dn < 32u) refill();
        wave_sync();
        const uint32_t pass = ~row_bits(reinterpret_cast<const uint32_t *>(mt8), rowm, g) & rowm;
        uint32_t incl = wave_incl_scan((uint32_t)__popc(pass));
        uint32_t n = (uint32_t)readlane((int)incl, kWave - 1);
        if (n == 0) continue;
        // G2: first general over the non-mountain cells in row-major order
        RowCol at = row_select(pass, incl, pick(draw(), n));
        if (lane == 0) gpv = at.r * W + at.c;
        uint32_t gens = lane == at.r ? 1u << at.c : 0u;
        // G3: its 4-connected component; further generals stay inside it
        // (with a cap on the BFS distance the reach takes its place)
        const bool official = prm.generator == 1;
        uint32_t room = official && prm.dmax > 0 ? pass : row_component(pass, at);
        // G4: each further general far enough from all earlier ones: in
        // Manhattan distance, or (R18) in BFS steps, at most dmax if set
        bool ok = true;
        for (int i = 1; i < g.P; ++i) {
            if (official) {
                if (prm.dmin > 0) room &= ~row_reach(pass, at, prm.dmin - 1);
                if (prm.dmax > 0) room &= row_reach(pass, at, prm.dmax);
            } else {
                const int k = prm.dmin - 1 - abs(lane - at.r);       // columns at.c - k .. at.c + k are too near
                if (k >= 0) room &= ~(((2u << min(at.c + k, 31)) - 1u) & ~((1u << max(at.c - k, 0)) - 1u));
            }
            room &= ~gens;
            incl = wave_incl_scan((uint32_t)__popc(room));
            n = (uint32_t)readlane((int)incl, kWave - 1);
            if (n == 0) { ok = false; break; }
            at = row_select(room, incl, pick(draw(), n));
            if (lane == i) gpv = at.r * W + at.c;
            if (lane == at.r) gens |= 1u << at.c;
        }
        if (!ok) continue;
        // G5: cities; under the official rules one within the radius of
        // every general first, then the rest on plain cells anywhere
        blank(true);
        uint32_t plain = pass & ~gens, cas = 0u;
        const int ncity = prm.cmin + (int)pick(draw(), (uint32_t)(prm.cmax - prm.cmin + 1));
        auto city = [&](uint32_t among) -> bool {
            incl = wave_incl_scan((uint32_t)__popc(among));
            n = (uint32_t)readlane((int)incl, kWave - 1);
            if (n == 0) return false;
            at = row_select(among, incl, pick(draw(), n));
            const int32_t a = prm.amin + (int32_t)pick(draw(), (uint32_t)(prm.amax - prm.amin + 1));
            const int c = at.r * W + at.c;
            if (lane == 0) { L.type[c] = CASTLE; L.army[c] = a; }
            if (lane == at.r) { cas |= 1u << at.c; plain &= ~(1u << at.c); }
            return true;
        };
        int t = 0;
        if (official) {
            for (int i = 0; i < g.P && ok; ++i) {
                const int c = readlane(gpv, i), r = div_w(c, g);
                const uint32_t near = row_reach(pass, {r, c - r * W}, prm.radius);
                if (ballot((near & cas) != 0u) != 0ull) continue;
                ok = city(near & plain);
                ++t;
            }
            if (!ok) continue;
        }
        for (; t < ncity; ++t) {
            if (j + 2u > dn) refill();
            if (!city(plain)) break;
        }
        placed = true;
    }
    if (!placed) {
        // deterministic last resort: no mountains, no cities, fixed border cells
        blank(false);
        const int r = (lane == 0 || lane == 2 || lane == 4) ? 0 : (lane == 1 || lane == 3 || lane == 5) ? H - 1 : H / 2;
        const int c = (lane == 0 || lane == 3 || lane == 6) ? 0 : (lane == 1 || lane == 2 || lane == 7) ? W - 1 : W / 2;
        gpv = r * W + c;
    }
    wave_sync();
    // G6: generals (plus pre-grown armies on the overflow-stress workload)
    int32_t a = 1;
    if (prm.pregrow && episode == 0 && (env_id & 3) == 0)
        a = 100000 + (int32_t)pick(draw32(seed, DOM_PREGROW, env_id, 0, 0, (uint32_t)(lane & 7)), 900001u);
    for (int i = 0; i < g.P; ++i) {                    // in order: the last resort's cells may coincide
        if (lane == i) {
            L.type[gpv] = GENERAL;
            L.owner[gpv] = (int8_t)i;
            L.army[gpv] = a;
        }
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < kMaxP; ++i) s.gpos[i] = (int16_t)(i < g.P ? readlane(gpv, i) : -1);
    s.turn = 0;
    s.episode = episode;
    s.alive = (uint8_t)((1u << g.P) - 1u);
    s.finished = 0;
    wave_sync();
}

// ---------------------------------------------------------------- moves (Section IV-D)
__device__ __forceinline__ bool is_ally(int mode, int a, int b) { return mode == MODE_2V2 && a != b && ((a ^ b) & 1) == 0; }

// Decode one action (on the lane of its player): source and destination
// cells and the half flag packed as src | dst << 10 | half << 20, or -1 when
// the code can never be legal (out of range, k = 0, off the grid, into a
// mountain -- mountains never change during a step).
__device__ __forceinline__ int decode_action(const Lds &L, const Geom &g, int32_t a)
{
    if (a < 0 || a >= g.HW * 9) return -1;
    const int src = a / 9, k = a - src * 9;
    if (k == 0) return -1;
    const int dir = (k - 1) & 3;
    int r = div_w(src, g), c = src - r * g.W;
    r += dir == 0 ? -1 : dir == 1 ? 1 : 0;
    c += dir == 2 ? -1 : dir == 3 ? 1 : 0;
    if (r < 0 || r >= g.H || c < 0 || c >= g.W) return -1;
    const int dst = r * g.W + c;
    if (L.type[dst] == MOUNTAIN) return -1;
    return src | (dst << 10) | ((k >= 5 ? 1 : 0) << 20);
}

// Apply player i's decoded move (a wave-uniform value), re-validating
// ownership and army at application time (R4/R5).  The five LDS values the
// move can need are read at once and made scalar, the decision runs on the
// scalar unit, and lane 0 writes the cells that change.  Returns the player
// whose general was captured (-1 if none); the captured general becomes a
// castle here.
__device__ int apply_move(const Lds &L, const Geom &g, const EnvScalars &s, int i, int packed)
{
    if (packed < 0 || !((s.alive >> i) & 1)) return -1;
    const int src = packed & 1023, dst = (packed >> 10) & 1023;     // neighbours, never equal
    const bool half = (packed >> 20) & 1;
    const int o_src = readfirst(L.owner[src]);
    const int32_t have = readfirst(L.army[src]);
    const int o = readfirst(L.owner[dst]);
    const int32_t d = readfirst(L.army[dst]);
    const int t = readfirst(L.type[dst]);
    if (o_src != i || have <= 1) return -1;
    const int32_t m = half ? (have >> 1) : have - 1;
    int o_new = o, victim = -1;
    int32_t d_new;
    if (o == i) {
        d_new = sat_add(d, m);
    } else if (o >= 0 && is_ally(g.mode, o, i)) {
        d_new = sat_add(d, m);
        o_new = i;
    } else if (m > d) {
        o_new = i;
        d_new = m - d;
        if (t == GENERAL) {
#pragma unroll
            for (int v = 0; v < kMaxP; ++v) {
                if (v < g.P && victim < 0 && s.gpos[v] == dst && ((s.alive >> v) & 1) && v != i &&
                    !is_ally(g.mode, v, i))
                    victim = v;
            }
        }
    } else {
        d_new = d - m;
    }
    if (lane_id() == 0) {
        L.army[src] = have - m;
        L.army[dst] = d_new;
        L.owner[dst] = (int8_t)o_new;
        if (victim >= 0) L.type[dst] = CASTLE;
    }
    return readfirst(victim);
}

// All players' moves in rotating priority (reading R5), captures applied at
// once by the whole wave (Section IV-E transfer, reading R9 halving).
// Returns true if a general was captured (the type row then changed).
//
// Moves whose four, six, ... cells are all different and none of which takes
// a general do not depend on their order: they are decided and applied in
// one pass, lane p player p's.  Each lane claims its two cells in a byte row
// (the last writer of a cell keeps it, so at least one lane of a clash reads
// another's claim).  Any clash or capture leaves the board untouched and
// goes through the moves one by one, about 800 clocks each against 1,100 for
// the pass (8 players: 6,700 -> 1,300 clocks of a wave alone).
__device__ bool resolve_moves(const Lds &L, const Geom &g, EnvScalars &s, int32_t my_action, uint8_t *claim)
{
    const int lane = lane_id();
    const int my_move = lane < g.P && ((s.alive >> lane) & 1) ? decode_action(L, g, my_action) : -1;
    if (ballot(my_move >= 0) == 0ull) return false;
    {
        const int src = my_move & 1023, dst = (my_move >> 10) & 1023;
        bool slow = false, moves = false;
        int32_t have = 0, d = 0, m = 0;
        int o = 0;
        if (my_move >= 0) {
            claim[src] = (uint8_t)lane;
            claim[dst] = (uint8_t)lane;
        }
        wave_sync();
        if (my_move >= 0) {
            slow = claim[src] != lane || claim[dst] != lane;
            have = L.army[src];
            d = L.army[dst];
            o = L.owner[dst];
            m = (my_move >> 20) & 1 ? have >> 1 : have - 1;
            moves = L.owner[src] == lane && have > 1;
            // a won attack on a general may be a capture
            slow = slow || (moves && o != lane && L.type[dst] == GENERAL && !(o >= 0 && is_ally(g.mode, o, lane)) && m > d);
        }
        if (ballot(slow) == 0ull) {
            if (moves) {
                const bool join = o == lane || (o >= 0 && is_ally(g.mode, o, lane));
                L.army[src] = have - m;
                L.army[dst] = join ? sat_add(d, m) : m > d ? m - d : d - m;
                if (join || m > d) L.owner[dst] = (int8_t)lane;
            }
            wave_sync();
            return false;
        }
    }
    bool captured = false;
    for (int j = 0; j < g.P; ++j) {
        const int i = (s.turn + j) % g.P;
        const int packed = readlane(my_move, i);
        const int victim = apply_move(L, g, s, i, packed);
        wave_sync();
        if (victim >= 0) {
            for (int c = lane; c < g.HW; c += kWave) {
                if (L.owner[c] == victim) {
                    L.owner[c] = (int8_t)i;
                    L.army[c] = L.army[c] >> 1;
                }
            }
            s.alive = (uint8_t)(s.alive & ~(1u << victim));
            captured = true;
            wave_sync();
        }
    }
    return captured;
}

// Cell bitmaps of the board, eight cells a thread (threads tid, tid + nt, ...):
// those of each player, and with ACT the passable cells and those with more
// than one unit, as bytes of the row-major bitmaps (bit = cell).  many(b): the
// armies of cells 8 b to 8 b + 7 clamped to bytes.  (A ballot per player and
// 64 cells took 580 clocks a word of a wave alone: 5,200 of the 17,800 of a
// 24x24 step, with 8 players 14,000 of 40,000.)
template <bool ACT, class Many>
__device__ __forceinline__ void cell_bitmaps(const Geom &g, const int8_t *owner, const uint8_t *type, uint64_t *own,
                                             uint64_t *pass, uint64_t *big, int tid, int nt, Many &&many)
{
    for (int b = tid; b < 8 * g.NW; b += nt) {
        const int left = g.HW - 8 * b;                 // bytes past the map are read and masked
        const uint32_t real = left >= 8 ? 0xFFu : left > 0 ? (1u << left) - 1u : 0u;
        const uint2 o = *reinterpret_cast<const uint2 *>(owner + 8 * b);
        for (int p = 0; p < g.P; ++p)
            reinterpret_cast<uint8_t *>(own + p * 16)[b] =
                (uint8_t)(bits8(bytes_eq(o.x, (uint32_t)p), bytes_eq(o.y, (uint32_t)p)) & real);
        if (ACT) {
            const uint2 t = *reinterpret_cast<const uint2 *>(type + 8 * b), m = many(b);
            const uint32_t mt = bits8(t.x & ~(t.x >> 1) & 0x01010101u, t.y & ~(t.y >> 1) & 0x01010101u);
            reinterpret_cast<uint8_t *>(pass)[b] = (uint8_t)(~mt & real);
            reinterpret_cast<uint8_t *>(big)[b] = (uint8_t)(bits8(bytes_gt1(m.x), bytes_gt1(m.y)) & real);
        }
    }
}

// Four armies clamped to bytes.
__device__ __forceinline__ uint32_t clamp4(int4 a)
{
    return (uint32_t)min(a.x, 255) | ((uint32_t)min(a.y, 255) << 8) | ((uint32_t)min(a.z, 255) << 16) | ((uint32_t)min(a.w, 255) << 24);
}

// ---------------------------------------------------------------- random legal actor (reading R15)
// Lane (p, w) holds word w of player p's bitmaps.  The legal moves of one
// direction are the player's cells with more than one unit whose neighbour
// in that direction is on the grid and not a mountain: one AND with the
// shifted passable bitmap.  A cell with d legal directions contributes 2d
// entries (all-but-one, then half) to the list [pass, (cell, k)...]; the
// uniform pick is located by a prefix over words and a binary search over
// the bits of one word.  own: [P][16] words, pass/big: [16] words in LDS;
// blk: the actor's two Philox4x32 blocks if the caller computed them.
__device__ void actor_wave(const Geom &g, const uint64_t *own, const uint64_t *pass, const uint64_t *big,
                           uint32_t alive, uint64_t actor_seed, uint64_t step_idx, uint64_t env_id, int32_t *act_out,
                           const uint64_t *blk = nullptr)
{
    const int lane = lane_id();
    const int NW = g.NW, W = g.W;
    const int lp = lane_player(NW), w = lane - lp * NW;
    const int ppr = readlane(lp, kWave - 1) + ((readlane(w, kWave - 1) == NW - 1) ? 1 : 0);     // 64 / NW
    const ColMasks cm = col_masks(w, g);
    const uint64_t pw = pass[w];
    const uint64_t pprev = w > 0 ? pass[w - 1] : 0ull, pnext = w < NW - 1 ? pass[w + 1] : 0ull;
    const uint64_t up_ok = (pw << W) | (pprev >> (64 - W));          // cell c with c - W passable
    const uint64_t dn_ok = (pw >> W) | (pnext << (64 - W));          // c + W passable
    const uint64_t lf_ok = ((pw << 1) | (pprev >> 63)) & ~cm.col0;   // c - 1 passable, same row
    const uint64_t rt_ok = ((pw >> 1) | (pnext << 63)) & ~cm.colL;   // c + 1 passable, same row
    const uint64_t bw = big[w];
    // the actor's draws (reading R15): player p takes 32-bit half p % 2 of
    // r[p / 2], r0 r1 from the block of players 0..3, r2 r3 from that of 4..7
    uint64_t r0, r1, r2, r3;
    if (blk != nullptr) {                        // computed earlier by the caller (in LDS)
        r0 = blk[0]; r1 = blk[1]; r2 = blk[2]; r3 = blk[3];
    } else {
        uint64_t w0, w1;
        actor_block(actor_seed, env_id, step_idx, w0, w1);
        r0 = shfl64(w0, 0); r1 = shfl64(w1, 0); r2 = shfl64(w0, 32); r3 = shfl64(w1, 32);
    }
    for (int p0 = 0; p0 < g.P; p0 += ppr) {
        const int p = p0 + lp;
        const bool valid = lp < ppr && p < g.P;
        const uint64_t src = (valid && ((alive >> p) & 1u)) ? (own[p * 16 + w] & bw) : 0ull;
        const uint64_t lu = src & up_ok, ld = src & dn_ok, ll = src & lf_ok, lr = src & rt_ok;
        const uint32_t cnt = 2u * (uint32_t)(__popcll(lu) + __popcll(ld) + __popcll(ll) + __popcll(lr));
        const uint32_t incl = wave_incl_scan(cnt);
        const int first = lp * NW;
        // every lane takes part in both shuffles (an inactive source lane would read as 0)
        const uint32_t below = shfl32(incl, first - 1);
        const uint32_t upto = shfl32(incl, first + NW - 1);
        const uint32_t before = first > 0 ? below : 0u;
        const uint32_t total = upto - before;
        const uint32_t excl = incl - cnt - before;
        const uint64_t rw = (p >> 1) == 0 ? r0 : (p >> 1) == 1 ? r1 : (p >> 1) == 2 ? r2 : r3;
        const uint32_t r = (p & 1) ? (uint32_t)(rw >> 32) : (uint32_t)rw;
        const uint32_t idx = pick(r, 1u + total);
        const bool mine = valid && idx > 0 && excl <= idx - 1 && idx - 1 < excl + cnt;
        if (mine) {
            // entry t of this word lies in the last cell b whose earlier cells
            // hold at most t entries.  A cell's move count n = lu + ld + ll + lr
            // (0..4) as three bit planes, n = s0 + 2 s1 + 4 s2 (full adders; a
            // carry of the second level excludes those of the first), so the
            // entries of a set of cells are 2 (|s0| + 2 |s1| + 4 |s2|); the
            // search halves the word, then works on 32-bit halves.
            uint32_t t = idx - 1 - excl;
            const uint64_t xa = lu ^ ld, xb = ll ^ lr, c1 = lu & ld, c2 = ll & lr;
            const uint64_t s0 = xa ^ xb, c3 = xa & xb;
            const uint64_t s1 = c1 ^ c2 ^ c3, s2 = c1 & c2;
            uint32_t h0 = (uint32_t)s0, h1 = (uint32_t)s1, h2 = (uint32_t)s2;
            const uint32_t lo = 2u * (uint32_t)(__popc(h0) + 2 * __popc(h1) + 4 * __popc(h2));
            int b = 0;
            if (lo <= t) {
                b = 32;
                t -= lo;
                h0 = (uint32_t)(s0 >> 32); h1 = (uint32_t)(s1 >> 32); h2 = (uint32_t)(s2 >> 32);
            }
            int bl = 0;
            for (int st = 16; st >= 1; st >>= 1) {
                const uint32_t m = (1u << (bl + st)) - 1u;
                const uint32_t pre = 2u * (uint32_t)(__popc(h0 & m) + 2 * __popc(h1 & m) + 4 * __popc(h2 & m));
                if (pre <= t) bl += st;
            }
            b += bl;
            const uint32_t ml = (1u << bl) - 1u;
            uint32_t j = t - 2u * (uint32_t)(__popc(h0 & ml) + 2 * __popc(h1 & ml) + 4 * __popc(h2 & ml));
            const uint32_t dirs = (uint32_t)((lu >> b) & 1ull) | ((uint32_t)((ld >> b) & 1ull) << 1) |
                                  ((uint32_t)((ll >> b) & 1ull) << 2) | ((uint32_t)((lr >> b) & 1ull) << 3);
            const uint32_t nd = (uint32_t)__popc(dirs);
            int kbase = 1;
            if (j >= nd) { j -= nd; kbase = 5; }
            int dir = 0;
            for (int d = 0, seen = 0; d < 4; ++d) {
                if ((dirs >> d) & 1u) {
                    if ((uint32_t)seen == j) { dir = d; break; }
                    ++seen;
                }
            }
            act_out[p] = (w * 64 + b) * 9 + kbase + dir;
        } else if (valid && w == 0 && idx == 0) {
            act_out[p] = 0;
        }
    }
}

// ---------------------------------------------------------------- one turn on the LDS grid
// What a step does before growth: the moves, the turn counter, terminal and
// rewards (Section III, Section IV-E; reading R11), the next map where a
// finished game restarts.  Executed by one wave; `act` is lane p's action,
// `claim` S bytes of LDS for the moves, src.map() the generator's settings.
struct MapArgs {
    GenParamsDev prm;
    uint64_t seed, env_id;
};

struct Turn {
    bool write_type = false;     // the type row (and the general cells) changed
    bool grow2 = false, grow50 = false, done = false;
    uint32_t win = 0, lose = 0;  // player masks
};

template <class Src>
__device__ __forceinline__ Turn advance(const Lds &L, const Geom &g, const Src &src, EnvScalars &s, int32_t act,
                                        uint8_t *claim)
{
    Turn r;
    if (s.finished) {
        r.done = true;
        return r;
    }
    const uint32_t alive0 = s.alive;
    r.write_type = resolve_moves(L, g, s, act, claim);
    s.turn += 1;
    r.grow2 = (s.turn & 1) == 0;
    r.grow50 = (s.turn % 50) == 0;
    const uint32_t alive = s.alive;
    if (g.mode == MODE_2V2) {
        const bool t0 = (alive & 0x5u) != 0, t1 = (alive & 0xAu) != 0;
        if (!t0 || !t1) {
            r.done = true;
            const uint32_t winners = t0 ? 0x5u : 0xAu;
            r.win = winners;
            r.lose = 0xFu & ~winners;
        }
    } else {
        r.lose = alive0 & ~alive;
        if (__popc(alive) == 1) { r.done = true; r.win = alive; }
    }
    if (r.done) {
        const MapArgs m = src.map();
        if (m.prm.auto_reset) {
            mapgen_wave(L, g, m.prm, m.seed, m.env_id, s.episode + 1u, s);
            r.write_type = true;
            r.grow2 = r.grow50 = false;
        } else {
            s.finished = 1;
        }
    }
    return r;
}

// One 0x01 per growing cell byte of a quad (Section IV-C), without branches:
// owned (the owner byte's sign bit clear) and a castle or general (type bit
// 1) on even turns or plain (type 0) on multiples of 50.
__device__ __forceinline__ uint32_t growing4(uint32_t o4, uint32_t t4, bool grow2, bool grow50)
{
    const uint32_t gm2 = grow2 ? 0x01010101u : 0u, gm50 = grow50 ? 0x01010101u : 0u;
    return (~o4 >> 7) & (((t4 >> 1) & gm2) | (~(t4 | (t4 >> 1)) & gm50));
}

}  // namespace gen
