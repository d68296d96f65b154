// kernels.hip -- gfx950 kernels of the batched Generals.io environment step
// (arxiv 2606.23348, Section IV).  One wave64 owns one environment: the grid
// (owner int8, type uint8, army int32) is loaded from HBM into LDS once, the
// whole step runs on it, and owner/army plus the uint8 observation stream
// back out.  No MFMA: nothing here is a contraction.
#include <algorithm>

#include "board.hpp"
#include "device.hpp"
#include "internal.hpp"

namespace gen {

// ---------------------------------------------------------------- LDS size of one env (board.hpp, Lds)
uint32_t lds_bytes_for(int S, int P)
{
    return (uint32_t)(4 * S + S + S + (S + 16) + 8 * 16 * (2 * P + 3) + 32 + 32);
}

// The staged writer's runs: four planes of a player, or all eight where the
// quads of a plane (and one more for a shifted one) fit half a wave.
constexpr int kSmallBoard = 121;
__host__ __device__ static inline int planes_per_run(int PS) { return PS <= kSmallBoard ? 8 : 4; }

// Its staging of one wave: a run, the line carried from the run before, the
// bytes a quad at the end writes past them.
__host__ __device__ static inline uint32_t stage_bytes(const Geom &g)
{
    return (uint32_t)(planes_per_run(g.PS) * ((g.PS + 15) & ~15) + 128 + 48);
}

// ---------------------------------------------------------------- fused env kernel
enum { K_STEP = 0, K_RESET = 1, K_OBSERVE = 2 };
// Observation writers: planes of a multiple of 4 cells (dword aligned) stored
// where they lie, any other size staged in LDS, planes padded to a multiple
// of 4 bytes (the layout of a pool's ragged observations, so envs of every
// shape take the dword writer), or aligned planes staged.
enum { OBS_QUAD = 0, OBS_STREAM = 1, OBS_PADDED = 2, OBS_STAGED = 3 };

// Player-independent bits of the four cells of quad q, one 0x01 per cell
// byte (SWAR over the owner and type bytes).
struct QuadCells {
    uint32_t o4;        // owner bytes
    uint32_t neutral;   // no owner
    uint32_t plain_n;   // no owner and not a mountain
    uint32_t mtn, cas, gen;
};

__device__ __forceinline__ QuadCells quad_cells(const Lds &L, int q)
{
    QuadCells c;
    c.o4 = reinterpret_cast<const uint32_t *>(L.owner)[q];
    const uint32_t t4 = reinterpret_cast<const uint32_t *>(L.type)[q];
    c.neutral = (c.o4 >> 7) & 0x01010101u;
    c.mtn = t4 & ~(t4 >> 1) & 0x01010101u;
    c.cas = (t4 >> 1) & ~t4 & 0x01010101u;
    c.gen = t4 & (t4 >> 1) & 0x01010101u;
    c.plain_n = c.neutral & ~c.mtn;
    return c;
}

// The eight observation dwords of quad q for player p (reading R16): one
// byte per cell, channel k in v[k].  ac: the quad's army bytes clamped to
// 255.  In 2v2 `ally` is p's teammate, otherwise p itself.
__device__ __forceinline__ void quad_planes(const Lds &L, const QuadCells &c, uint32_t ac, int p, uint32_t ally,
                                            int q, uint32_t v[8])
{
    const uint32_t vb = (uint32_t)(L.vis[p * 16 + (q >> 4)] >> ((q & 15) * 4)) & 0xFu;
    const uint32_t visb = spread4(vb);
    const uint32_t eqp = bytes_eq(c.o4, (uint32_t)p);
    const uint32_t eqa = ally == (uint32_t)p ? eqp : bytes_eq(c.o4, ally);
    v[0] = eqp;
    v[1] = (c.neutral ^ 0x01010101u) & ~eqp & ~eqa & visb;
    v[2] = c.plain_n & visb;
    v[3] = c.mtn & visb;
    v[4] = c.cas & visb;
    v[5] = c.gen & visb;
    v[6] = visb ^ 0x01010101u;
    v[7] = ac & (visb * 0xFFu);
}

// Quad q's dwords of player p's eight planes into the env's observation
// block ([P][8] planes of PS bytes), nontemporal; `keep` masks the bytes of
// cells past the map in a padded plane's last quad to zero.
// ro: buffer descriptor of the env's block; the plane offset is a scalar
// operand and 4q the one vector offset of all eight stores.
// Nontemporal also for dense planes, whose first and last sectors belong to
// two planes (us per step, plain and nontemporal: 2v2 14x14, 50,000 envs 119,
// 70; FFA-8 12x13, 32,768 envs 115, 77; 1v1 10x10, 65,536 envs 81.5, 80.3; of
// whole sectors, 2v2 16x16, 65,536 envs 161, 94).
__device__ __forceinline__ void quad_store(const Lds &L, const Geom &g, const Rsrc &ro, const QuadCells &qc,
                                           uint32_t ac, int p, int q, int PS, uint32_t keep = ~0u)
{
    const uint32_t ally = g.mode == MODE_2V2 ? (uint32_t)(p ^ 2) : (uint32_t)p;
    uint32_t v[8];
    quad_planes(L, qc, ac, p, ally, q, v);
#pragma unroll
    for (int ch = 0; ch < 8; ++ch)
        __builtin_amdgcn_raw_buffer_store_b32(v[ch] & keep, ro, 4 * q, (p * 8 + ch) * PS, kAuxNT);
}

// Two waves per env: wave 0 writes the planes of players 0 .. obs_split(P) - 1
// and then runs the actor, wave 1 the rest (3 of 8 and 5 of 8 players
// balance the two).
__device__ __forceinline__ int obs_split(int P) { return (P * 3) >> 3; }

// Waves per env in the staged writer: its n runs shared out, fewer for wave 0,
// which goes on to the actor (about one run's time).
struct RunRange { int begin, end; };

__device__ __forceinline__ RunRange wave_runs(const Geom &g, int wave, int nwv, bool act)
{
    const int n = g.P * 8 / planes_per_run(g.PS), own = act ? 1 : 0;
    if (nwv == 1) return {0, n};
    const int c0 = max(0, (n + own) / nwv - own);
    if (wave == 0) return {0, c0};
    return {c0 + (n - c0) * (wave - 1) / (nwv - 1), c0 + (n - c0) * wave / (nwv - 1)};
}

// Dense planes, runs [runs.begin, runs.end), by one wave: the bytes are put
// together in LDS and leave in the tensor's order as whole 128-byte lines, 16
// bytes a lane; the bytes of a line that the next run finishes are carried
// over, and only the range's first and last lines (shared with a neighbour)
// are written in part.  Planes of an odd number of cells start anywhere in a
// dword (WHOLE: they never do): each dword is realigned with the lane before
// and added to a cleared stage, so the dwords across two planes need no case
// of their own.  The cells are decoded once for all players: R rounds of 64
// quads, or with HALF lanes 32 to 63 take channels 4 to 7 of the quads of
// lanes 0 to 31.  (Before, every plane's dwords were stored where they lie,
// each plane's first and last lines in parts: us per step: FFA-8 25x25, 16,384 envs 215 -> 129; 2v2 17x19, 30,000 envs
// 134 -> 90; 1v1 25x25, 65,536 envs 278 -> 200; 9x11, 124 -> 98.)
template <bool WHOLE, int R, bool HALF>
__device__ __forceinline__ void stage_runs(const Lds &L, const Geom &g, uint8_t *obs, RunRange runs, uint8_t *stage)
{
    constexpr int kPlanes = HALF ? 8 : 4;
    const int lane = lane_id(), HW = g.HW, PS = g.PS;                  // cells, bytes from plane to plane
    const int cells = (HW + 3) >> 2, nq = (PS + 3) >> 2;               // quads of cells, of bytes
    const uint32_t tail = (HW & 3) ? (1u << (8 * (HW & 3))) - 1u : ~0u;
    const int d = (int)(reinterpret_cast<uintptr_t>(obs) & 127u);
    const Rsrc ro = buffer_rsrc(obs - d, (uint32_t)(d + g.P * 8 * PS));
    const int first = d + runs.begin * kPlanes * PS;   // from the line at or before the block
    QuadCells qc[R];
    uint32_t ac[R], keep[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int q = HALF ? lane & 31 : kWave * k + lane, qi = min(q, cells - 1);
        keep[k] = q < cells - 1 ? ~0u : q == cells - 1 ? tail : 0u;
        qc[k] = quad_cells(L, qi);
        ac[k] = reinterpret_cast<const uint32_t *>(L.armyc)[qi];
    }
    if (!WHOLE)
        for (int i = lane; i < (int)(stage_bytes(g) >> 4); i += kWave)
            reinterpret_cast<uint4 *>(stage)[i] = make_uint4(0u, 0u, 0u, 0u);
    uint32_t carry = 0u;                               // lane i: dword i of the line the last run left unfinished
    for (int n = runs.begin; n < runs.end; ++n) {
        const int p = HALF ? n : n >> 1;
        const bool upper = HALF ? lane >= 32 : (n & 1) != 0;           // channels 4 to 7
        const uint32_t ally = g.mode == MODE_2V2 ? (uint32_t)(p ^ 2) : (uint32_t)p;
        const int at = d + n * kPlanes * PS, line = at & ~127, end = at + kPlanes * PS;
        uint32_t visb[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int qi = min(HALF ? lane & 31 : kWave * k + lane, cells - 1);
            visb[k] = spread4((uint32_t)(L.vis[p * 16 + (qi >> 4)] >> ((qi & 15) * 4)) & 0xFu);
        }
        wave_sync();
        if (lane < 32) reinterpret_cast<uint32_t *>(stage)[lane] = carry;
        wave_sync();
        [[maybe_unused]] uint32_t before[4] = {0u, 0u, 0u, 0u};         // the last quad of the round before
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int q = HALF ? lane & 31 : kWave * k + lane;
            uint32_t v[4] = {0u, 0u, 0u, 0u}, u[4] = {0u, 0u, 0u, 0u};
            if (HALF || upper) {
                u[0] = qc[k].cas & visb[k];
                u[1] = qc[k].gen & visb[k];
                u[2] = visb[k] ^ 0x01010101u;
                u[3] = ac[k] & (visb[k] * 0xFFu);
            }
            if (HALF || !upper) {
                const uint32_t eqp = bytes_eq(qc[k].o4, (uint32_t)p);
                const uint32_t eqa = ally == (uint32_t)p ? eqp : bytes_eq(qc[k].o4, ally);
                v[0] = eqp;
                v[1] = (qc[k].neutral ^ 0x01010101u) & ~eqp & ~eqa & visb[k];
                v[2] = qc[k].plain_n & visb[k];
                v[3] = qc[k].mtn & visb[k];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int x = at - line + j * PS;      // the plane's place in the stage, m bytes into a dword
                const uint32_t m = (uint32_t)x & 3u, c = (upper ? u[j] : v[j]) & keep[k];
                uint32_t *to = reinterpret_cast<uint32_t *>(stage + ((HALF && upper ? x + 4 * PS : x) & ~3)) + q;
                if (WHOLE) {
                    if (q < nq) *to = c;
                    continue;
                }
                uint32_t out = c;
                if (m != 0u) out = __builtin_amdgcn_alignbyte(c, wave_shr1(c, before[j]), 4u - m);
                if (k + 1 < R) before[j] = (uint32_t)readlane((int)c, kWave - 1);
                if (q <= nq) atomicOr(to, out);
            }
        }
        wave_sync();
        // whole lines out; a cleared stage is left for the next run
        const int whole = (end & ~127) - line, shared = line < first ? 128 : 0;
        const int i = 4 * lane, rest = end - line - whole;   // bytes of the line the next run finishes
        const bool last = n + 1 == runs.end;
        carry = i < rest ? *reinterpret_cast<const uint32_t *>(stage + whole + i) : 0u;
        if (shared != 0 && (whole > 0 || last) && i >= first - line && i < (whole > 0 ? 128 : end - line))
            __builtin_amdgcn_raw_buffer_store_b32(*reinterpret_cast<const uint32_t *>(stage + i), ro, i, line, 0);
        for (int j = 16 * lane; j < end - line; j += 16 * kWave) {
            u32x4 *x = reinterpret_cast<u32x4 *>(stage + j);
            const u32x4 v = *x;
            if (j >= shared && j < whole) __builtin_amdgcn_raw_buffer_store_b128(v, ro, j, line, kAuxNT);
            if (!WHOLE) *x = u32x4{0u, 0u, 0u, 0u};
        }
        if (last && whole >= shared && i < rest) __builtin_amdgcn_raw_buffer_store_b32(carry, ro, i, line + whole, 0);
    }
}

template <bool WHOLE>
__device__ __forceinline__ void obs_dense_planes(const Lds &L, const Geom &g, uint8_t *obs, RunRange runs, uint8_t *stage)
{
    const int quads = (g.PS + 3) / 4 + (WHOLE ? 0 : 1);
    if (g.PS <= kSmallBoard) stage_runs<WHOLE, 1, true>(L, g, obs, runs, stage);
    else if (quads <= 64) stage_runs<WHOLE, 1, false>(L, g, obs, runs, stage);
    else if (quads <= 128) stage_runs<WHOLE, 2, false>(L, g, obs, runs, stage);
    else if (quads <= 192) stage_runs<WHOLE, 3, false>(L, g, obs, runs, stage);
    else stage_runs<WHOLE, 4, false>(L, g, obs, runs, stage);
}

// Padded planes (plane stride g.PS, a multiple of 32 bytes): the dword
// writer for players p_begin .. p_end - 1, quads outer (a quad's cells
// decoded once for all those players; measured on the mixed pool: 286 ->
// 273 us per step against players outer); the bytes of cells past the map
// in a plane's last quads are written as zero.
__device__ __forceinline__ void obs_padded_planes(const Lds &L, const Geom &g, uint8_t *obs, int p_begin, int p_end)
{
    const int lane = lane_id();
    const int PS = g.PS;
    const int nq = PS >> 2;
    const int nfull = ((g.HW + 3) >> 2) - 1;                          // last quad holding map cells
    const uint32_t tail = (g.HW & 3) ? (1u << (8 * (g.HW & 3))) - 1u : ~0u;
    const Rsrc ro = buffer_rsrc(obs, (uint32_t)(g.P * 8 * PS));
    for (int q = lane; q < nq; q += kWave) {
        const QuadCells qc = quad_cells(L, q);
        const uint32_t ac = reinterpret_cast<const uint32_t *>(L.armyc)[q];
        const uint32_t keep = q < nfull ? ~0u : q == nfull ? tail : 0u;
        for (int p = p_begin; p < p_end; ++p) quad_store(L, g, ro, qc, ac, p, q, PS, keep);
    }
}

// Dense planes that end in the middle of a line, two at a time: channels 2 i
// and 2 i + 1 are one run of whole lines, stored 64 quads at a time, so that
// the line they share is one store's (HALF: whether a store's quads are the
// first plane's, the second's or both).  Plane by plane that line is written
// in halves two rounds apart; together in LDS (the staged writer) the run
// costs instructions that a launch after a pause, at lower clocks, feels.
// us per step of 1v1 24x24, 65,536 envs, plane by plane, staged, in pairs:
// one batch after a pause 132, 172, 131; on and on 138, 144, 130; several
// batches in turn 224, 203, 203.
template <int HALF>
__device__ __forceinline__ void pair_stores(const Lds &L, const Geom &g, const Rsrc &ro, int Q, int n)
{
    const bool odd = HALF == 2 ? Q >= n : HALF == 1;       // the run's quad Q is of the second plane
    const int q = odd ? Q - n : Q;
    const QuadCells qc = quad_cells(L, q);
    const uint32_t ac = reinterpret_cast<const uint32_t *>(L.armyc)[q];
    for (int p = 0; p < g.P; ++p) {
        const uint32_t ally = g.mode == MODE_2V2 ? (uint32_t)(p ^ 2) : (uint32_t)p;
        uint32_t v[8];
        quad_planes(L, qc, ac, p, ally, q, v);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = HALF == 0 ? v[2 * i] : HALF == 1 ? v[2 * i + 1] : odd ? v[2 * i + 1] : v[2 * i];
            __builtin_amdgcn_raw_buffer_store_b32(x, ro, 4 * Q, (p * 8 + 2 * i) * g.HW, kAuxNT);
        }
    }
}

__device__ __forceinline__ void obs_paired_planes(const Lds &L, const Geom &g, const Rsrc &ro)
{
    const int n = g.HW >> 2;
    for (int at = 0; at < 2 * n; at += kWave) {
        const int Q = at + lane_id();
        if (Q >= 2 * n) continue;
        if (at + kWave <= n) pair_stores<0>(L, g, ro, Q, n);
        else if (at >= n) pair_stores<1>(L, g, ro, Q, n);
        else pair_stores<2>(L, g, ro, Q, n);
    }
}

// Per-env inputs and outputs of one step (pointers into this env's rows).
struct EnvIO {
    EnvScalars *sc;
    int8_t *owner;
    uint8_t *type;
    int32_t *army;
    const int32_t *actions;     // P actions of this step
    int32_t *next_actions;      // fused actor output (ACT)
    int32_t *rewards;
    uint8_t *done;
    uint8_t *obs;               // this env's [P][8][H][W] block, nullptr = no observation
    int32_t *land;              // scoreboard (SB)
    int64_t *army_tot;
    uint64_t env_id;            // global id (keys every draw)
    uint64_t actor_seed;
    uint64_t actor_step;        // actor step index when the tick is not used
    bool use_tick;              // keep the per-env step counter; the actor draws with it
    int nwv = 1;                // waves of the workgroup sharing the observation planes
    bool stage = false;         // padded planes may go through the staged writer
    bool paired = false;        // EnvArgs::paired
};

// One environment step (or reset / observation) on one wave.  OBSV selects
// the observation writer and layout at compile time (OBS_PADDED for the
// mixed shapes of a pool).  src.io() and src.map() read the env's arguments
// where they are needed (see fresh).
template <int KIND, int OBSV, bool SB, bool ACT, class Src>
__device__ __forceinline__ void env_body(uint8_t *smem, const Geom &g, const Src &src)
{
    const int lane = lane_id();
    const Lds L = carve(smem, g);

    EnvScalars s;
    bool write_type = false, grow2 = false, grow50 = false, done = false;
    uint32_t win = 0, lose = 0;

    if (KIND == K_RESET) {
        const MapArgs m = src.map();
        mapgen_wave(L, g, m.prm, m.seed, m.env_id, 0u, s);
        s.tick = 0;
        write_type = true;
    } else {
        const EnvIO io = src.io();
        s = *io.sc;
        const int n16 = g.S >> 4;
        const uint4 *go = reinterpret_cast<const uint4 *>(io.owner);
        const uint4 *gt = reinterpret_cast<const uint4 *>(io.type);
        const uint4 *ga = reinterpret_cast<const uint4 *>(io.army);
        int32_t act = 0;
        if constexpr (ACT) {
            // state HBM -> registers (16-byte loads; S <= 1024 cells, so one
            // owner and one type chunk and at most four army chunks per
            // lane; indexes are clamped rather than the loads predicated:
            // lanes past the end re-read the last chunk and skip the store)
            const int na = 4 * n16;
            // two-wave envs issue their state loads at raised wave priority,
            // so a new env's loads are not queued behind older waves' work
            // (FFA-8 25x25: 216 -> 211 us; one-wave shapes unchanged)
            if (io.nwv > 1) __builtin_amdgcn_s_setprio(3);
            const uint4 vo = go[min(lane, n16 - 1)];
            const uint4 vt = gt[min(lane, n16 - 1)];
            const uint4 va0 = ga[min(lane, na - 1)];
            const uint4 va1 = ga[min(lane + 64, na - 1)];
            const uint4 va2 = ga[min(lane + 128, na - 1)];
            const uint4 va3 = ga[min(lane + 192, na - 1)];
            if (KIND == K_STEP && lane < g.P) act = io.actions[lane];
            if (io.nwv > 1) __builtin_amdgcn_s_setprio(0);
            // the actor's Philox blocks do not depend on the state:
            // computing them while the loads are in flight hides their
            // latency; they wait in LDS until the actor runs
            if (io.next_actions != nullptr) {
                const uint64_t tick = (uint64_t)s.tick + ((KIND == K_STEP && io.use_tick) ? 1u : 0u);
                uint64_t w0, w1;
                actor_block(io.actor_seed, io.env_id, io.use_tick ? tick : io.actor_step, w0, w1);
                if ((lane & 31) == 0) {
                    uint64_t *pb = L.gbm + 52 + (lane >> 4);
                    pb[0] = w0;
                    pb[1] = w1;
                }
            }
            if (lane < n16) {
                reinterpret_cast<uint4 *>(L.owner)[lane] = vo;
                reinterpret_cast<uint4 *>(L.type)[lane] = vt;
            }
            uint4 *la = reinterpret_cast<uint4 *>(L.army);
            if (lane < na) la[lane] = va0;
            if (lane + 64 < na) la[lane + 64] = va1;
            if (lane + 128 < na) la[lane + 128] = va2;
            if (lane + 192 < na) la[lane + 192] = va3;
        } else {
            // state HBM -> LDS, 16-byte loads
            for (int i = lane; i < n16; i += kWave) {
                reinterpret_cast<uint4 *>(L.owner)[i] = go[i];
                reinterpret_cast<uint4 *>(L.type)[i] = gt[i];
            }
            for (int i = lane; i < 4 * n16; i += kWave) reinterpret_cast<uint4 *>(L.army)[i] = ga[i];
            if (KIND == K_STEP && lane < g.P) act = io.actions[lane];
        }
        wave_sync();
        if (KIND == K_STEP) {
            if (io.use_tick) s.tick += 1;
            const Turn r = advance(L, g, src, s, act, L.armyc);
            write_type = r.write_type;
            grow2 = r.grow2;
            grow50 = r.grow50;
            done = r.done;
            win = r.win;
            lose = r.lose;
        }
    }

    const EnvIO io = src.io();

    // ---- growth (Section IV-C), state store, army clamp, scoreboard
    unsigned long long *const tot = reinterpret_cast<unsigned long long *>(L.gbm + 32);    // army totals (SB)
    if (SB) {
        if (lane < kMaxP) tot[lane] = 0ull;
        wave_sync();
    }
    {
        const int nq = g.S >> 2;
        uint32_t *go = reinterpret_cast<uint32_t *>(io.owner);
        uint32_t *gt = reinterpret_cast<uint32_t *>(io.type);
        int4 *ga = reinterpret_cast<int4 *>(io.army);
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t o4 = reinterpret_cast<const uint32_t *>(L.owner)[q];
            const uint32_t t4 = reinterpret_cast<const uint32_t *>(L.type)[q];
            int4 a4 = reinterpret_cast<const int4 *>(L.army)[q];
            int32_t av[4] = {a4.x, a4.y, a4.z, a4.w};
            // the army never wraps (saturating add, reading R12)
            const uint32_t inc = growing4(o4, t4, grow2, grow50);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                [[maybe_unused]] const int o = (int8_t)(o4 >> (8 * k));
                av[k] = __builtin_elementwise_add_sat(av[k], (int32_t)((inc >> (8 * k)) & 1u));
                // one LDS addition per owned cell (a wave sum per player took
                // 1,100 clocks each)
                // (the address is from the state's bytes: only a player's is one of the totals)
                if (SB && (uint32_t)o < (uint32_t)kMaxP) atomicAdd(&tot[o], (unsigned long long)(long long)av[k]);
            }
            if (KIND != K_OBSERVE) {
                st_nt(reinterpret_cast<uint4 *>(ga + q),
                      make_uint4((uint32_t)av[0], (uint32_t)av[1], (uint32_t)av[2], (uint32_t)av[3]));
                st_nt(go + q, o4);
                if (write_type) st_nt(gt + q, t4);
            }
            uint32_t ac = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) ac |= (uint32_t)(av[k] > 255 ? 255 : av[k]) << (8 * k);
            reinterpret_cast<uint32_t *>(L.armyc)[q] = ac;
        }
    }
    // ---- per-player owned-cell bitmaps, with the fused actor also the
    // passable and army > 1 bitmaps
    wave_sync();
    auto many = [&](int b) { return reinterpret_cast<const uint2 *>(L.armyc)[b]; };
    cell_bitmaps<ACT>(g, L.owner, L.type, L.obm, L.gbm, L.gbm + 16, lane, kWave, many);
    wave_sync();

    if (SB && lane < g.P) {
        int land = 0;
        for (int w = 0; w < g.NW; ++w) land += __popcll(L.obm[lane * 16 + w]);
        io.land[lane] = land;
        io.army_tot[lane] = (int64_t)tot[lane];
    }

    // ---- fog (Section IV-B, team vision R10)
    team_vision(L.obm, L.vis, g);
    wave_sync();
    // the workgroup's further waves, which only write planes, wait here
    // for the state and the vision, then writes the later players' planes
    if (OBSV != OBS_QUAD && io.nwv > 1) __syncthreads();

    // Planes of a multiple of 4 cells: each lane takes 4 cells, computes their
    // bytes of all 8 channel planes in registers and stores them directly
    // (4-byte stores, 256 contiguous bytes per wave store).  Other shapes
    // stage the bytes in LDS.
    if (OBSV == OBS_QUAD || OBSV == OBS_PADDED) {
        if (io.obs != nullptr) {
            // Quads outer: a quad's owner and type bits decoded once for
            // all players.
            if (OBSV == OBS_QUAD) {
                const int nq = g.HW >> 2;
                const Rsrc ro = buffer_rsrc(io.obs, (uint32_t)(g.P * 8 * g.HW));
                if (io.paired) obs_paired_planes(L, g, ro);
                else for (int q = lane; q < nq; q += kWave) {
                    const QuadCells qc = quad_cells(L, q);
                    const uint32_t ac = reinterpret_cast<const uint32_t *>(L.armyc)[q];
                    for (int p = 0; p < g.P; ++p) quad_store(L, g, ro, qc, ac, p, q, g.HW);
                }
            } else if (io.stage && io.nwv == 1 && g.HW > kOneRound && (g.PS & 127) != 0) {
                obs_dense_planes<true>(L, g, io.obs, wave_runs(g, 0, 1, ACT), reinterpret_cast<uint8_t *>(L.army));
            } else {
                obs_padded_planes(L, g, io.obs, 0, io.nwv > 1 ? obs_split(g.P) : g.P);
            }
        }
    } else if (io.obs != nullptr) {
        obs_dense_planes<OBSV == OBS_STAGED>(L, g, io.obs, wave_runs(g, 0, io.nwv, ACT), reinterpret_cast<uint8_t *>(L.army));
    }
    wave_sync();

    // ---- fused random actor for the next step, on the final state
    if (ACT && io.next_actions != nullptr)
        actor_wave(g, L.obm, L.gbm, L.gbm + 16, s.alive, io.actor_seed, io.use_tick ? s.tick : io.actor_step, io.env_id,
                   io.next_actions, KIND != K_RESET ? L.gbm + 52 : nullptr);

    // ---- rewards, done, scalars
    if (KIND == K_STEP) {
        if (lane < g.P) io.rewards[lane] = ((win >> lane) & 1u) ? 1 : (((lose >> lane) & 1u) ? -1 : 0);
        if (lane == 0) *io.done = done ? 1 : 0;
    }
    if (KIND != K_OBSERVE && lane == 0) {
        EnvScalars *d = io.sc;
        d->turn = s.turn;
        d->episode = s.episode;
        d->alive = s.alive;
        d->finished = s.finished;
        if (io.use_tick || KIND == K_RESET) d->tick = s.tick;
        if (write_type) {
#pragma unroll
            for (int i = 0; i < kMaxP; ++i) d->gpos[i] = s.gpos[i];
        }
    }
}

// The step kernels for planes of a multiple of 4 cells without the
// scoreboard are limited to the registers of 8 waves per SIMD (the default
// budget of 106 scalar registers allows 7); the extra scalar spills go to
// vector-register lanes and cost less than the lost occupancy (measured).
// The scoreboard kernels would spill vector registers to scratch under that
// limit, and the other plane sizes measured slower at 25x25; they keep the
// default.
// NWV = 2 (steps of more than 4 players with padded planes): a second wave per
// env writes the planes of the players from obs_split(P) on.  NWV = 8: up to 8
// waves share the staged writer's runs (odd planes).
struct EnvSrc {
    int e, nwv;

    __device__ __forceinline__ EnvIO io() const
    {
        const EnvArgs &a = fresh_args<EnvArgs>();
        const size_t cell0 = (size_t)e * a.g.S, player0 = (size_t)e * a.g.P;
        EnvIO io;
        io.sc = a.sc + e;
        io.owner = a.owner + cell0;
        io.type = a.type + cell0;
        io.army = a.army + cell0;
        io.actions = a.actions + player0;
        io.next_actions = a.next_actions + player0;
        io.rewards = a.rewards + player0;
        io.done = a.dones + e;
        io.obs = a.obs != nullptr ? a.obs + (size_t)e * (size_t)(a.g.P * 8 * a.g.PS) : nullptr;
        io.land = a.land + player0;
        io.army_tot = a.army_tot + player0;
        io.env_id = a.env_base + (uint64_t)e;
        io.actor_seed = a.actor_seed;
        io.actor_step = a.step_idx;
        io.use_tick = false;
        io.nwv = nwv;
        io.paired = a.paired != 0u;
        return io;
    }

    __device__ __forceinline__ MapArgs map() const
    {
        const EnvArgs &a = fresh_args<EnvArgs>();
        return {a.prm, a.seed, a.env_base + (uint64_t)e};
    }
};

template <int KIND, int OBSV, bool SB, bool ACT, int NWV>
__global__ __launch_bounds__(64 * NWV)
__attribute__((amdgpu_waves_per_eu((SB || (OBSV != OBS_QUAD && OBSV != OBS_STAGED)) ? 1 : 8, 8))) void k_env(EnvArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const Geom g = a.g;
    EnvSrc src{(int)xcd_env(blockIdx.x, gridDim.x), 1};
    if (NWV > 1) {
        static_assert(NWV == 1 || OBSV != OBS_QUAD, "further waves only share the staged and padded-plane writers");
        const int wv = readfirst((int)(threadIdx.x >> 6));
        src.nwv = OBSV == OBS_PADDED ? 2 : readfirst((int)(blockDim.x >> 6));
        if (wv > 0) {
            // exactly one barrier, matching the one wave 0 passes after the vision
            const Lds L = carve(smem, g);
            __syncthreads();
            uint8_t *obs = src.io().obs;
            if (obs != nullptr) {
                if (OBSV == OBS_STREAM || OBSV == OBS_STAGED)
                    obs_dense_planes<OBSV == OBS_STAGED>(L, g, obs, wave_runs(g, wv, src.nwv, ACT),
                                                         reinterpret_cast<uint8_t *>(L.army) + (uint32_t)wv * stage_bytes(g));
                else obs_padded_planes(L, g, obs, obs_split(g.P), g.P);
            }
            return;
        }
    }
    env_body<KIND, OBSV, SB, ACT>(smem, g, src);
}

// ---------------------------------------------------------------- batched pool (mixed shapes)
// One wave per env, `wpg` envs per workgroup, envs taken in the order of a
// work list (slots slot_begin .. slot_end - 1 of it: a launch covers one
// segment of envs that share a packing); each env's shape, mode, generator
// settings and buffer offsets come from its 32-byte descriptor.  With a
// grid smaller than the segment the workgroups loop (persistent form).
// With two waves per env (NWV = 2, one env per workgroup) the second wave
// writes the observation planes of the later players, as in the plain
// two-wave step.
// One pool env on the calling wave (slot = position in the work list;
// wave = the wave's index within the env, of nwv).
// Args: fresh() of the launch's arguments as PoolArgs.
template <class Args, bool STAGE>
struct PoolSrc {
    Args args;
    PoolDesc d;
    int nwv;

    __device__ __forceinline__ EnvIO io() const
    {
        const PoolArgs &a = args.fresh();
        EnvIO io;
        io.sc = a.sc + d.env;
        io.owner = a.owner + d.cell_off;
        io.type = a.type + d.cell_off;
        io.army = a.army + d.cell_off;
        io.actions = a.actions + d.act_off;
        io.next_actions = a.actor ? a.actions + d.act_off : nullptr;
        io.rewards = a.rewards + d.act_off;
        io.done = a.dones + d.env;
        io.obs = a.obs != nullptr ? a.obs + (size_t)d.obs_off16 * 16 : nullptr;
        io.land = nullptr;
        io.army_tot = nullptr;
        io.env_id = a.env_base + d.env;
        io.actor_seed = a.actor_seed;
        io.actor_step = 0;
        io.use_tick = true;
        io.nwv = nwv;
        io.stage = STAGE && a.stage != 0u;
        return io;
    }

    __device__ __forceinline__ MapArgs map() const
    {
        const PoolArgs &a = args.fresh();
        MapArgs m{a.prm, a.seed, a.env_base + d.env};
        m.prm.cmin = d.cmin;
        m.prm.cmax = d.cmax;
        m.prm.dmin = d.dmin;
        return m;
    }
};

struct PoolLaunch {
    __device__ __forceinline__ const PoolArgs &fresh() const { return fresh_args<PoolArgs>(); }
};

template <int KIND, bool ACT, bool STAGE, class Args>
__device__ __forceinline__ void pool_env_d(const Args &args, uint8_t *smem, const PoolDesc &d, int nwv = 1,
                                           int wave = 0)
{
    Geom g;
    g.H = d.H;
    g.W = d.W;
    g.HW = d.H * d.W;
    g.S = (g.HW + 15) & ~15;
    g.P = d.P;
    g.mode = d.mode;
    g.NW = (g.HW + 63) >> 6;
    g.magic_w = d.magic_w;
    g.PS = pool_plane_stride(g.HW, g.P);
    const PoolSrc<Args, STAGE> src{args, d, nwv};
    if (wave > 0) {
        // exactly one barrier, matching the one wave 0 passes after the vision
        const Lds L = carve(smem, g);
        __syncthreads();
        uint8_t *obs = src.io().obs;
        if (obs != nullptr) obs_padded_planes(L, g, obs, obs_split(g.P), g.P);
        return;
    }
    env_body<KIND, OBS_PADDED, false, ACT>(smem, g, src);
}

// PERSIST = false: one env per wave (per workgroup with NWV = 2), the grid
// covers the segment.  PERSIST = true (NWV = 1 only: the two waves of an env
// would need a second barrier before reusing the LDS for the next env): a
// smaller grid whose waves stride over the segment.
template <int KIND, bool ACT, bool PERSIST, int NWV>
__global__ __launch_bounds__(256) void k_pool(PoolArgs a)
{
    static_assert(NWV == 1 || !PERSIST, "two waves per env only in the one-shot grid");
    extern __shared__ __align__(16) uint8_t smem[];
    // wave index as a scalar: everything derived from the env id stays wave-uniform
    const uint32_t wave = (uint32_t)readfirst((int)(threadIdx.x >> 6));
    if (NWV == 2) {
        const uint32_t slot = a.slot_begin + blockIdx.x;
        if (slot < a.slot_end) pool_env_d<KIND, ACT, false>(PoolLaunch{}, smem, a.desc[slot], 2, (int)wave);
        return;
    }
    uint8_t *mine = smem + wave * a.lds_per_wave;
    if (PERSIST) {
        for (uint32_t slot = a.slot_begin + blockIdx.x * a.wpg + wave; slot < a.slot_end; slot += gridDim.x * a.wpg)
            pool_env_d<KIND, ACT, false>(PoolLaunch{}, mine, a.desc[slot]);
    } else {
        const uint32_t slot = a.slot_begin + xcd_chunk32(blockIdx.x, gridDim.x) * a.wpg + wave;
        if (slot < a.slot_end) pool_env_d<KIND, ACT, true>(PoolLaunch{}, mine, a.desc[slot]);
    }
}

// ---------------------------------------------------------------- standalone actor
__global__ __launch_bounds__(64) void k_sample(SampleArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = lane_id();
    const int e = blockIdx.x;
    const Geom g = a.g;
    const Lds L = carve(smem, g);
    const uint64_t env_id = a.env_base + (uint64_t)e;
    const size_t cell0 = (size_t)e * g.S;
    const uint32_t alive = a.sc[e].alive;
    // owner and type rows into LDS; armies clamped to a byte
    const int n16 = g.S >> 4;
    for (int i = lane; i < n16; i += kWave) {
        reinterpret_cast<uint4 *>(L.owner)[i] = reinterpret_cast<const uint4 *>(a.owner + cell0)[i];
        reinterpret_cast<uint4 *>(L.type)[i] = reinterpret_cast<const uint4 *>(a.type + cell0)[i];
    }
    for (int q = lane; q < 4 * n16; q += kWave) {
        reinterpret_cast<uint32_t *>(L.armyc)[q] = clamp4(reinterpret_cast<const int4 *>(a.army + cell0)[q]);
    }
    wave_sync();
    auto many = [&](int b) { return reinterpret_cast<const uint2 *>(L.armyc)[b]; };
    cell_bitmaps<true>(g, L.owner, L.type, L.obm, L.gbm, L.gbm + 16, lane, kWave, many);
    wave_sync();
    actor_wave(g, L.obm, L.gbm, L.gbm + 16, alive, a.actor_seed, a.step_idx, env_id, a.actions + (size_t)e * g.P);
}

// ---------------------------------------------------------------- launchers
uint32_t lds_bytes(const Geom &g) { return lds_bytes_for(g.S, g.P); }

// Waves per env of the staged writer for odd planes: as many as the batch
// leaves room for, up to a wave per run; two where an env has 10 or more runs
// (us per step with 1, 2, 4, 8 waves: FFA-8 25x25, 500 envs 28.6, 20.3, 16.0,
// 14.5; 2,000 envs 31.1, 26.0, 28.1, 34.2; 16,384 envs 143, 129, 152, 228;
// 2v2 17x19, 500 envs 13.2, 10.5, 9.3, 9.2; 2,000 envs 15.6, 13.7, 16.7, 23.5;
// 4,096 envs 19.8, 21.8, 26.8, 43.0).
static int dense_waves(const EnvArgs &a, int n_envs)
{
    if (a.obs == nullptr) return 1;
    const int runs = a.g.P * 8 / planes_per_run(a.g.PS);
    if (n_envs <= 512) return std::min(8, runs);
    if (n_envs <= 1024) return std::min(4, runs);
    return n_envs <= 2048 || (runs >= 10 && n_envs <= 16384) ? 2 : 1;
}

// Aligned planes through the staged writer: where a plane takes more than one
// round of stores its last line meets the next plane's first one eight planes
// later, and the line leaves the L2 in parts.  Planes of whole lines have no
// such line; planes of whole 64-byte halves lose only when the batch's
// observation is beyond the Infinity Cache.  (us per step, stored where they
// lie and staged: 1v1 20x20, 65,536 envs 233, 143; 2v2 20x20, 40,000 envs 250,
// 102; 1v1 18x18, 8,000 envs 25.6, 21.1; 14x20, 8,192 envs 21.8, 20.2; 16x16,
// 65,536 envs 80, 98; 28x32, 8,000 envs 31, 36; 2v2 21x21 padded to 448, 28,000
// envs 87, 78.  A second round of a few cells pays later: 13x20, 8,192 envs
// 18.6, 20.8; 20,000 envs 44.4, 40.4; 65,536 envs 135, 114; held to 18 waves a
// CU the dword stores take 112 there, 40.2 and, at 17x16, 114 against 112, so
// two cell counts do not get a rule of their own.  A reset's maps keep the
// waves apart, so it gains nothing: 24x24 177, 238.)
static bool stage_whole(const EnvArgs &a, int n_envs, int kind)
{
    if (kind == K_RESET || a.obs == nullptr || a.g.HW <= kOneRound || a.g.PS % 128 == 0) return false;
    const uint64_t bytes = (uint64_t)n_envs * (uint64_t)(a.g.P * 8 * a.g.PS);
    const uint64_t parts = a.g.HW <= kOneRound + 16 ? 64000000ull : 30000000ull;
    return bytes >= (a.g.PS % 64 != 0 ? parts : 400000000ull);
}

// Dense planes in pairs: those of more than a round of stores that end in the
// middle of a line, where the observation no longer sits in the L2s (us per
// step, plane by plane and in pairs: 24x24 1v1, 2,048 envs 9.7, 9.9; 4,096
// envs 14.0, 13.6; 8,192 envs 24.3, 21.6; FFA-8 24x24, 1,024 envs 15.9, 16.5;
// 2,048 envs 23.4, 22.0; 2v2 24x24, 28,000 envs 118, 99; FFA-6 16x20, 16,384
// envs 60, 53; 26x32 1v1, 30,000 envs 147, 129; 14x32 1v1, 8,192 envs 18.5,
// 17.7; FFA-3 10x32, 8,192 envs 19.3, 17.8; two players' planes of 320 cells
// have too little to store per decoded cell, in each of four shapes: 9,000
// envs 17.6, 18.6; 32,768 envs 46.0, 48.3; 65,536 envs 85, 89; 78,000 envs,
// 400 MB 172, 143; boards of one round: 12x16 1v1, 65,536 envs 77, 82).
static bool pair_planes(const EnvArgs &a, int n_envs)
{
    if (a.obs == nullptr || a.g.PS != a.g.HW || a.g.HW <= kOneRound || a.g.HW % 128 != 64 || n_envs < 2048) return false;
    const uint64_t bytes = (uint64_t)n_envs * (uint64_t)(a.g.P * 8 * a.g.PS);
    return bytes >= (a.g.P * a.g.HW < 800 ? 400000000ull : 35000000ull);
}

// LDS of the dword writers by one wave: with more than 4 players and planes of
// more than one line a batch is held to 16 waves a CU, since the lines that
// two planes share leave the L2 in parts when the 32 waves that would fit all
// store (us per step with 32 and 16 waves: FFA-8 12x12, 32,768 envs 92, 75;
// FFA-8 12x13 108, 86; FFA-8 14x14, 16,384 envs 68, 63; FFA-6 14x14, 32,768
// envs 93, 71; FFA-5 14x14 74, 64; FFA-8 12x12 padded, 32,768 envs 94, 77;
// planes within a line or fewer players need the waves: FFA-8 10x10 62, 74;
// 2v2 14x14, 50,000 envs 73, 88; below 8,192 envs the same either way).
constexpr uint32_t kSixteenWavesLds = 10240;

static uint32_t dword_lds(const EnvArgs &a, int n_envs, uint32_t lds)
{
    const bool held = a.obs != nullptr && a.g.P > 4 && a.g.HW > 128 && n_envs >= 8192;
    return held ? std::max(lds, kSixteenWavesLds) : lds;
}

template <int KIND, bool SB, bool ACT>
static hipError_t launch_kind(const EnvArgs &a, int n_envs, hipStream_t stream)
{
    const dim3 grid((unsigned)n_envs), block(kWave);
    const uint32_t lds = lds_bytes(a.g), lds_dense = lds - 4u * (uint32_t)a.g.S + stage_bytes(a.g);
    if (a.g.PS != a.g.HW) {
        // planes padded to 32 bytes: the dword writer for every shape; more
        // than 4 players share it between two waves
        if constexpr (KIND == K_STEP) {
            if (a.g.P > 4 && a.obs != nullptr && n_envs <= 16384) {
                hipLaunchKernelGGL((k_env<KIND, OBS_PADDED, SB, ACT, 2>), grid, dim3(2 * kWave), lds, stream, a);
                return hipGetLastError();
            }
        }
        if (stage_whole(a, n_envs, KIND))
            hipLaunchKernelGGL((k_env<KIND, OBS_STAGED, SB, ACT, 1>), grid, block, lds_dense, stream, a);
        else
            hipLaunchKernelGGL((k_env<KIND, OBS_PADDED, SB, ACT, 1>), grid, block, dword_lds(a, n_envs, lds), stream, a);
        return hipGetLastError();
    }
    const int nwv = KIND == K_RESET ? 1 : dense_waves(a, n_envs);
    const bool staged = a.g.HW % 4 != 0, paired = pair_planes(a, n_envs);
    if (staged && nwv > 1) {
        if constexpr (KIND != K_RESET)
            hipLaunchKernelGGL((k_env<KIND, OBS_STREAM, SB, ACT, 8>), grid, dim3(kWave * nwv),
                               lds_dense + (uint32_t)(nwv - 1) * stage_bytes(a.g), stream, a);
    } else if (staged) {
        hipLaunchKernelGGL((k_env<KIND, OBS_STREAM, SB, ACT, 1>), grid, block, lds_dense, stream, a);
    } else if (!paired && stage_whole(a, n_envs, KIND)) {
        hipLaunchKernelGGL((k_env<KIND, OBS_STAGED, SB, ACT, 1>), grid, block, lds_dense, stream, a);
    } else {
        EnvArgs b = a;
        b.paired = paired ? 1u : 0u;
        hipLaunchKernelGGL((k_env<KIND, OBS_QUAD, SB, ACT, 1>), grid, block, dword_lds(a, n_envs, lds), stream, b);
    }
    return hipGetLastError();
}

hipError_t launch_step(const EnvArgs &a, int n_envs, hipStream_t stream)
{
    if (a.next_actions != nullptr)
        return (a.land != nullptr) ? launch_kind<K_STEP, true, true>(a, n_envs, stream)
                                   : launch_kind<K_STEP, false, true>(a, n_envs, stream);
    return (a.land != nullptr) ? launch_kind<K_STEP, true, false>(a, n_envs, stream)
                               : launch_kind<K_STEP, false, false>(a, n_envs, stream);
}

hipError_t launch_reset(const EnvArgs &a, int n_envs, hipStream_t stream)
{
    return launch_kind<K_RESET, false, false>(a, n_envs, stream);
}

hipError_t launch_observe(const EnvArgs &a, int n_envs, hipStream_t stream)
{
    return launch_kind<K_OBSERVE, false, false>(a, n_envs, stream);
}

// ---------------------------------------------------------------- served batches
// One launch steps the envs of many requests (each request = one step of a
// group, a pool of its own), one workgroup per env of the launch; a
// workgroup finds its request by a binary search over the requests' first
// workgroups (at most 9 scalar loads from the argument segment), so no
// workgroup is launched for nothing when request sizes differ.
// Buffers are addressed as arena + offset so that every pointer derives from
// a kernel argument (global address space, scalar base + vector offset).
// The request list travels in the kernel argument (scalar loads from the
// argument segment), the group records stay resident in the arena.
// UNI: every request of the launch is a uniform group (its record says so),
// whose descriptors the kernel derives instead of loading; a launch with any
// other group loads every descriptor (one copy of the step per kernel: with
// both forms in one kernel the served mix ran 5-13% slower).
// The uniform instance budgets registers for 8 waves per SIMD (uniform 24x24
// 1v1 groups fit 8 in LDS); the other keeps the default budget, since the
// LDS of its largest board limits it to fewer waves anyway (served mix
// 401.5 -> 410 M frames/s without the 8-wave budget's spills).
struct ServeLaunchOf {
    const ServeReq *req;

    __device__ __forceinline__ PoolArgs fresh() const
    {
        const ServeReq &r = gen::fresh<ServeReq>(req);
        uint8_t *const arena = fresh_args<ServeLaunch>().arena;
        PoolArgs a;
        a.prm = r.prm;
        a.seed = r.seed;
        a.env_base = r.env_base;
        a.actor_seed = r.actor_seed;
        a.actor = r.actor;
        a.stage = 0;
        a.sc = reinterpret_cast<EnvScalars *>(arena + r.off_sc);
        a.owner = reinterpret_cast<int8_t *>(arena + r.off_owner);
        a.type = arena + r.off_type;
        a.army = reinterpret_cast<int32_t *>(arena + r.off_army);
        a.actions = reinterpret_cast<int32_t *>(arena + r.off_actions);
        a.rewards = reinterpret_cast<int32_t *>(arena + r.off_rewards);
        a.dones = arena + r.off_dones;
        a.obs = r.off_obs != ~0ull ? arena + r.off_obs : nullptr;
        return a;
    }
};

template <bool UNI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(UNI ? 8 : 1, 8))) void k_serve(ServeLaunch la)
{
    extern __shared__ __align__(16) uint8_t smem[];
    uint8_t *const arena = la.arena;
    // the request holding this workgroup: binary search over the ascending
    // first[] (wave-uniform, scalar loads), first[lo] <= b < first[hi]
    const uint32_t b = blockIdx.x;
    uint32_t lo = 0, hi = la.n_req;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (la.first[mid] <= b) lo = mid;
        else hi = mid;
    }
    const ServeReq &r = la.groups[la.idx[lo]];
    const uint32_t slot = b - la.first[lo];
    if (slot >= r.n_envs) return;
    if (UNI) {
        // every env of a uniform group has the template's shape and
        // settings: its descriptor follows from the slot
        PoolDesc d = r.tmpl;
        d.cell_off = slot * r.cells_per_env;
        d.obs_off16 = slot * r.obs16_per_env;
        d.act_off = slot * d.P;
        d.env = slot;
        pool_env_d<K_STEP, true, false>(ServeLaunchOf{&r}, smem, d);
    } else {
        pool_env_d<K_STEP, true, false>(ServeLaunchOf{&r}, smem, reinterpret_cast<const PoolDesc *>(arena + r.off_desc)[slot]);
    }
}

hipError_t launch_serve(const ServeLaunch &la, uint32_t total_envs, uint32_t lds, bool all_uniform, hipStream_t stream)
{
    if (la.n_req == 0 || la.n_req > kServeMaxReqs || total_envs == 0) return hipErrorInvalidValue;
    if (all_uniform) hipLaunchKernelGGL(k_serve<true>, dim3(total_envs), dim3(kWave), lds, stream, la);
    else hipLaunchKernelGGL(k_serve<false>, dim3(total_envs), dim3(kWave), lds, stream, la);
    return hipGetLastError();
}

template <int KIND, bool ACT, bool PERSIST, int NWV>
static hipError_t launch_pool_kind(const PoolArgs &a, uint32_t grid, hipStream_t stream)
{
    const uint32_t threads = NWV == 2 ? 2 * kWave : kWave * a.wpg;
    const uint32_t lds = NWV == 2 ? a.lds_per_wave : a.lds_per_wave * a.wpg;
    hipLaunchKernelGGL((k_pool<KIND, ACT, PERSIST, NWV>), dim3(grid), dim3(threads), lds, stream, a);
    return hipGetLastError();
}

template <int KIND, bool ACT>
static hipError_t launch_pool_act(const PoolArgs &a, uint32_t grid, uint32_t nwv, hipStream_t stream)
{
    const uint32_t n = a.slot_end - a.slot_begin;
    if (nwv == 2) return launch_pool_kind<KIND, ACT, false, 2>(a, n, stream);
    const uint32_t full = (n + a.wpg - 1) / a.wpg;
    if (grid != 0 && grid < full) return launch_pool_kind<KIND, ACT, true, 1>(a, grid, stream);
    PoolArgs b = a;
    b.stage = a.stage != 0u && a.obs != nullptr ? 1u : 0u;
    b.lds_per_wave += b.stage != 0u ? kStageExtra : 0u;
    return launch_pool_kind<KIND, ACT, false, 1>(b, full, stream);
}

// One segment of the work list [a.slot_begin, a.slot_end): grid == 0 one
// wave (nwv waves) per env, else persistent (nwv == 1 only).
hipError_t launch_pool(const PoolArgs &a, int kind, bool act, uint32_t grid, uint32_t nwv, hipStream_t stream)
{
    if (a.slot_end <= a.slot_begin) return hipSuccess;
    if (kind == K_RESET)
        return act ? launch_pool_act<K_RESET, true>(a, grid, 1, stream) : launch_pool_act<K_RESET, false>(a, grid, 1, stream);
    return act ? launch_pool_act<K_STEP, true>(a, grid, nwv, stream) : launch_pool_act<K_STEP, false>(a, grid, nwv, stream);
}

hipError_t launch_sample(const SampleArgs &a, int n_envs, hipStream_t stream)
{
    hipLaunchKernelGGL(k_sample, dim3((unsigned)n_envs), dim3(kWave), lds_bytes(a.g), stream, a);
    return hipGetLastError();
}

}  // namespace gen
