// features.hip -- the paper's full feature tensor (Appendix A, table of
// observation channels; reading R17 of this library): 38 float32 maps per
// player and env, and whole rollouts that record them, by one workgroup per
// env.
//
// The output alone is 152 bytes per cell and player, so the kernels are
// built around its stores.  The env's state and its memory in HBM (persistent
// masks, the last enemy sighting per cell, a ring of the last 8 frames) are
// read once into LDS with 16-byte loads, the memory is updated there, and
// then each wave writes whole planes: one (player, channel) at a time, so
// the channel is wave-uniform, four consecutive cells per lane, 16-byte
// nontemporal stores in runs on 128-byte boundaries whatever the board's
// size, the waves of a workgroup side by side.  A lane per cell that writes
// all channels with 4-byte stores leaves every line in parts where planes are
// no multiple of 128 bytes; it stays for outputs that the last-level cache
// puts together (cell_task, by_cells).  Features and step, us, all by cells
// before: FFA-8 25x25, 1,024 envs, 347 -> 195 (24x24 178 -> 167); 1v1 25x25,
// 8,192 envs, 665 -> 445; 24x24, 460 -> 385; 10x10, 163 -> 113; 24x24 with
// tokens, 65,536 envs, 3,400 -> 3,100, where constant planes take 2,600: the
// stores bound it.
// Measured and not kept: runs of 2 to 4 planes per wave with the values at
// their seams carried over (10 to 25% slower: the waves write further apart).
#define GEN_LANE_PER_USE        // see lane_id()
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "board.hpp"
#include "device.hpp"
#include "internal.hpp"

namespace gen {

// log(1 + dt) / 5 (channel 21) for dt in [0, kAgeTable): filled once per
// device by host code from the host C library's double log1p, divided by 5
// in double and rounded once to float32; larger gaps are computed here in
// double the same way.
__device__ float g_age_table[kAgeTable];

namespace {

constexpr int kFeatC = 38;
constexpr int kHist = 7;
constexpr int kEdge = 0;          // cache policy of the part stores at a plane's ends: plain, so the cache merges them
constexpr uint32_t kOnes = 0x01010101u;          // one per cell byte
constexpr int kFeatWaves = 8, kFeatMostWaves = 16;

// Bits of a player's byte per cell.  The first five are the memory (channels
// 4 to 8); the others only stand in LDS, for the turn's planes: visible now;
// channel 9 where visible, channel 13 in the fog; visible and neutral.
enum : int { B_SEEN = 0, B_ENEMY, B_GENERAL, B_CASTLE, B_MOUNTAIN, B_NOW, B_PLACE, B_NEUTRAL };
constexpr uint32_t kMemoryBits = 0x1F1F1F1Fu;

// Barrier of the workgroup that orders LDS only: a full __syncthreads would
// also wait for the wave's outstanding stores to HBM, which no other wave
// reads.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------- LDS of one env
// `mem` mirrors the env's memory block from its `bits` section to the end of
// the frame ring (FeatBlock: bits | last | lturn | fowner | fvis | farmy), so
// block and mirror are copied as one run.  The frame of turn t sits in ring
// slot t mod 8.  The planes read a frame as its armies and two masks per
// cell: own (bit p: owned by player p) and foe (bit p: seen by p on an
// enemy's cell), both 0 in a slot that holds no frame of the last 8 turns.
struct FeatLds {
    uint8_t *mem;            // 9 P S + 48 S bytes
    uint8_t *bits;           // [P][S]
    int32_t *last, *lturn;   // [P][S]
    int8_t *fowner;          // [8][S]
    uint8_t *fvis;           // [8][S]
    int32_t *farmy;          // [8][S]
    uint8_t *own, *foe;      // [8][S] masks (k_features: in the place of fowner and fvis)
    int8_t *owner;           // [S] the board of this turn
    uint8_t *type;           // [S]
    int32_t *army;           // [S] (k_features: the ring slot of this turn)
    uint64_t *obm, *vis;     // [P][16]
    unsigned long long *armt;    // [8] army totals
    int32_t *land;           // [8]
    float *flat;             // [8][6] channels 14 to 19 by player
    float *cx, *cy;          // [32] channels 22 and 23 by column, row
};

__host__ __device__ inline uint32_t feat_lds_bytes(int S, int P)
{
    return (uint32_t)(16 + 9 * P * S + 48 * S + 2 * S + 2 * P * 128 + 64 + 32 + 192 + 256);
}

__device__ __forceinline__ FeatLds feat_carve(uint8_t *smem, int S, int P)
{
    FeatLds F;
    F.mem = smem + 16;                                 // an unaligned quad at a row's start stays inside
    F.bits = F.mem;
    F.last = reinterpret_cast<int32_t *>(F.mem + P * S);
    F.lturn = F.last + P * S;
    F.fowner = reinterpret_cast<int8_t *>(F.lturn + P * S);
    F.fvis = reinterpret_cast<uint8_t *>(F.fowner + 8 * S);
    F.farmy = reinterpret_cast<int32_t *>(F.fvis + 8 * S);
    F.own = reinterpret_cast<uint8_t *>(F.fowner);
    F.foe = F.fvis;
    F.army = F.farmy;
    F.owner = reinterpret_cast<int8_t *>(F.farmy + 8 * S);
    F.type = reinterpret_cast<uint8_t *>(F.owner + S);
    F.obm = reinterpret_cast<uint64_t *>(F.type + S);
    F.vis = F.obm + P * 16;
    F.armt = reinterpret_cast<unsigned long long *>(F.vis + P * 16);
    F.land = reinterpret_cast<int32_t *>(F.armt + 8);
    F.flat = reinterpret_cast<float *>(F.land + 8);
    F.cx = F.flat + 48;
    F.cy = F.cx + 32;
    return F;
}

// The workgroup's copy of n 16-byte chunks, four loads in flight per thread.
__device__ __forceinline__ void copy16(void *dst, const void *src, int n, int tid, int nt)
{
    const u32x4 *sp = static_cast<const u32x4 *>(src);
    u32x4 *dp = static_cast<u32x4 *>(dst);
    for (int i = tid; i < n; i += 4 * nt) {
        const int i1 = i + nt, i2 = i1 + nt, i3 = i2 + nt;
        const u32x4 v0 = sp[i], v1 = sp[min(i1, n - 1)], v2 = sp[min(i2, n - 1)], v3 = sp[min(i3, n - 1)];
        dp[i] = v0;
        if (i1 < n) dp[i1] = v1;
        if (i2 < n) dp[i2] = v2;
        if (i3 < n) dp[i3] = v3;
    }
}

// ---------------------------------------------------------------- one turn's frame
struct FrameCtx {
    Geom g;
    int t = 0, slot = 0;     // turn, its ring slot
    bool fresh = true;       // the block holds another episode (or nothing): an empty memory
};

// Bit j: ring slot j holds the frame of one of the 7 turns before t
// (stamp[j]: turn of the frame in slot j, -1 none).
__device__ __forceinline__ uint32_t slots_held(const int32_t (&stamp)[8], int t)
{
    uint32_t h = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int32_t d = t - stamp[j];
        if (stamp[j] >= 0 && (stamp[j] & 7) == j && d >= 1 && d <= kHist) h |= 1u << j;
    }
    return h;
}

// The two masks of a quad (see FeatLds) from its owner and visibility bytes.
// A byte that is no player (0xFF: none; 8 and up never stand in a valid
// state) sets no bit.
__device__ __forceinline__ uint32_t own_mask(uint32_t o4)
{
    const uint32_t m = (1u << (o4 & 7u)) | ((1u << ((o4 >> 8) & 7u)) << 8) | ((1u << ((o4 >> 16) & 7u)) << 16) |
                       ((1u << ((o4 >> 24) & 7u)) << 24);
    return m & (bytes_eq(o4 & 0xF8F8F8F8u, 0u) * 0xFFu);
}

__device__ __forceinline__ uint32_t foe_mask(uint32_t o4, uint32_t own, uint32_t vis, int mode)
{
    const uint32_t owned = (~(o4 >> 7) & kOnes) * 0xFFu;
    const uint32_t team = mode == MODE_2V2 ? own | ((own << 2) & 0x0C0C0C0Cu) | ((own >> 2) & 0x03030303u) : own;
    return vis & owned & ~team;
}

// The masks of the ring's earlier frames (0 for a slot that holds none).
__device__ __forceinline__ void ring_masks(const FeatLds &F, const FrameCtx &f, uint32_t held, int tid, int nt)
{
    const int nq = f.g.S >> 2;
    const uint32_t magic = ((1u << 20) + (uint32_t)nq - 1) / (uint32_t)nq;
    for (int n = tid; n < 8 * nq; n += nt) {
        const int j = (int)(((uint32_t)n * magic) >> 20);
        const uint32_t o4 = reinterpret_cast<const uint32_t *>(F.fowner)[n], v4 = reinterpret_cast<const uint32_t *>(F.fvis)[n];
        const bool have = (held >> j) & 1u;
        const uint32_t own = have ? own_mask(o4) : 0u;
        const uint32_t foe = have ? foe_mask(o4, own, v4, f.g.mode) : 0u;
        reinterpret_cast<uint32_t *>(F.own)[n] = own;
        reinterpret_cast<uint32_t *>(F.foe)[n] = foe;
    }
}

// Army totals (zeroed before), one LDS addition per owned cell: 64 of them to
// few addresses cost less than a wave sum per player.
__device__ __forceinline__ void army_totals(const FeatLds &F, const Geom &g, int tid, int nt)
{
    for (int c = tid; c < g.HW; c += nt) {
        const int o = F.owner[c];
        if ((uint32_t)o < (uint32_t)kMaxP) atomicAdd(&F.armt[o], (unsigned long long)(long long)F.army[c]);
    }
}

// Memory update of a (player, quad of cells) per thread and that player's
// masks of this turn; the row after the last player puts the quad's frame
// into its ring slot.  MIRROR: the memory stays in LDS (the caller writes it
// back later, so the raw frame is kept beside its masks), else it goes to
// HBM at once.
template <bool MIRROR>
__device__ __forceinline__ void frame_update(const FeatLds &F, const FrameCtx &f, const Rsrc &rm, const FeatBlock &fb,
                                             int tid, int nt)
{
    const Geom &g = f.g;
    const int nq = g.S >> 2;
    const uint32_t magic = ((1u << 20) + (uint32_t)nq - 1) / (uint32_t)nq;    // n / nq, exact for n < 9 * 256
    for (int n = tid; n < nq * (g.P + 1); n += nt) {
        const int p = (int)(((uint32_t)n * magic) >> 20), q = n - p * nq;
        const int w = q >> 4, sh = (q & 15) * 4;
        const uint32_t o4 = reinterpret_cast<const uint32_t *>(F.owner)[q];
        const int4 a = reinterpret_cast<const int4 *>(F.army)[q];
        if (p == g.P) {
            uint32_t vb = 0;
            for (int k = 0; k < g.P; ++k) vb |= spread4((uint32_t)(F.vis[k * 16 + w] >> sh) & 0xFu) << k;
            const uint32_t own = own_mask(o4);
            const int at = f.slot * nq + q;
            if (MIRROR) {
                reinterpret_cast<uint32_t *>(F.fowner)[at] = o4;
                reinterpret_cast<uint32_t *>(F.fvis)[at] = vb;
            } else {
                const u32x4 x = {(uint32_t)a.x, (uint32_t)a.y, (uint32_t)a.z, (uint32_t)a.w};
                __builtin_amdgcn_raw_buffer_store_b32(o4, rm, 4 * q, (int)fb.fowner + f.slot * g.S, kAuxNT);
                __builtin_amdgcn_raw_buffer_store_b32(vb, rm, 4 * q, (int)fb.fvis + f.slot * g.S, kAuxNT);
                __builtin_amdgcn_raw_buffer_store_b128(x, rm, 16 * q, (int)fb.farmy + 4 * f.slot * g.S, kAuxNT);
            }
            reinterpret_cast<uint32_t *>(F.own)[at] = own;
            reinterpret_cast<uint32_t *>(F.foe)[at] = foe_mask(o4, own, vb, g.mode);
            reinterpret_cast<int4 *>(F.farmy)[at] = a;
            continue;
        }
        const uint32_t t4 = reinterpret_cast<const uint32_t *>(F.type)[q];
        const uint32_t v = spread4((uint32_t)(F.vis[p * 16 + w] >> sh) & 0xFu);
        const uint32_t mate = g.mode == MODE_2V2 ? (uint32_t)(p ^ 2) : (uint32_t)p;
        const uint32_t none = (o4 >> 7) & kOnes, mine = bytes_eq(o4, (uint32_t)p);
        const uint32_t ve = v & ~none & ~mine & ~bytes_eq(o4, mate);
        const uint32_t mtn = t4 & ~(t4 >> 1), cas = (t4 >> 1) & ~t4, gnl = t4 & (t4 >> 1);
        uint32_t *pb = reinterpret_cast<uint32_t *>(F.bits + p * g.S) + q;
        int4 *pl = reinterpret_cast<int4 *>(F.last + p * g.S) + q, *pt = reinterpret_cast<int4 *>(F.lturn + p * g.S) + q;
        uint32_t bits = f.fresh ? 0u : *pb & kMemoryBits;
        int4 last = f.fresh ? make_int4(0, 0, 0, 0) : *pl, lt = f.fresh ? make_int4(0, 0, 0, 0) : *pt;
        bits |= (v << B_SEEN) | (ve << B_ENEMY) | ((v & gnl) << B_GENERAL) | ((v & cas) << B_CASTLE) | ((v & mtn) << B_MOUNTAIN);
        if (v & 0x00000001u) last.x = (ve & 0x00000001u) ? a.x : 0;
        if (v & 0x00000100u) last.y = (ve & 0x00000100u) ? a.y : 0;
        if (v & 0x00010000u) last.z = (ve & 0x00010000u) ? a.z : 0;
        if (v & 0x01000000u) last.w = (ve & 0x01000000u) ? a.w : 0;
        if (ve & 0x00000001u) lt.x = f.t;
        if (ve & 0x00000100u) lt.y = f.t;
        if (ve & 0x00010000u) lt.z = f.t;
        if (ve & 0x01000000u) lt.w = f.t;
        const uint32_t fog = v ^ kOnes;
        *pb = bits | (v << B_NOW) | ((v & none) << B_NEUTRAL) |
              (((v & none & ~mtn) | (fog & (mtn | cas | (bits >> B_GENERAL)))) << B_PLACE);
        *pl = last;
        *pt = lt;
        if (!MIRROR) {
            const u32x4 xl = {(uint32_t)last.x, (uint32_t)last.y, (uint32_t)last.z, (uint32_t)last.w};
            const u32x4 xt = {(uint32_t)lt.x, (uint32_t)lt.y, (uint32_t)lt.z, (uint32_t)lt.w};
            __builtin_amdgcn_raw_buffer_store_b32(bits, rm, 4 * q, (int)fb.bits + p * g.S, kAuxNT);
            __builtin_amdgcn_raw_buffer_store_b128(xl, rm, 16 * q, (int)fb.last + 4 * p * g.S, kAuxNT);
            __builtin_amdgcn_raw_buffer_store_b128(xt, rm, 16 * q, (int)fb.lturn + 4 * p * g.S, kAuxNT);
        }
    }
}

// Four cells' bytes and int32 values in LDS, from any cell (ANY) or a multiple of 4.
template <bool ANY>
__device__ __forceinline__ uint32_t ld4(const void *p)
{
    if (!ANY) return *static_cast<const uint32_t *>(p);
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

template <bool ANY>
__device__ __forceinline__ int4 ld16(const int32_t *p)
{
    if (!ANY) return *reinterpret_cast<const int4 *>(p);
    return make_int4(p[0], p[1], p[2], p[3]);
}

// v where bit `at` of m is set, else 0.
__device__ __forceinline__ int keep(int v, uint32_t m, int at) { return v & __builtin_amdgcn_sbfe((int)m, at, 1); }

__device__ __forceinline__ int4 keep4(int4 a, uint32_t m, int bit)
{
    return make_int4(keep(a.x, m, bit), keep(a.y, m, bit + 8), keep(a.z, m, bit + 16), keep(a.w, m, bit + 24));
}

__device__ __forceinline__ float4 bytes_to_f(uint32_t m)
{
    return make_float4((float)(m & 0xFFu), (float)((m >> 8) & 0xFFu), (float)((m >> 16) & 0xFFu), (float)(m >> 24));
}

// Channel ch (wave-uniform) of player p at the quads of cells c[0], c[1], ...
// (any cell with ANY, else multiples of 4; with N players those
// of player p first, then p + 1's and so on, the last player's again after it): the channel is decided once
// for all R quads of a lane, whose LDS reads are then in flight together.
template <bool ANY, int N, int R>
__device__ __forceinline__ void channel(const FeatLds &F, const FrameCtx &f, int p0, int ch, const int (&c)[R], float4 (&x)[R])
{
    const Geom &g = f.g;
    const int S = g.S;
    auto player = [&](int k) { return N == 1 ? p0 : min(p0 + k / (R / N), g.P - 1); };
    auto each = [&](auto &&value) {
#pragma unroll
        for (int k = 0; k < R; ++k) x[k] = value(c[k], player(k));
    };
    if (ch >= 24) {
        // army of the frame of turn t - k minus that of t - k - 1 on the
        // player's (resp. visible enemies') cells; an absent frame is empty
        const int k = ch - (ch >= 24 + kHist ? 24 + kHist : 24);
        const uint8_t *mask = ch >= 24 + kHist ? F.foe : F.own;
        const int o0 = ((f.t - k) & 7) * S, o1 = ((f.t - k - 1) & 7) * S;
        each([&](int q, int p) {
            const int4 u = keep4(ld16<ANY>(F.farmy + o0 + q), ld4<ANY>(mask + o0 + q), p);
            const int4 v = keep4(ld16<ANY>(F.farmy + o1 + q), ld4<ANY>(mask + o1 + q), p);
            return make_float4((float)(u.x - v.x), (float)(u.y - v.y), (float)(u.z - v.z), (float)(u.w - v.w));
        });
        return;
    }
    const int now = f.slot * S;
    switch (ch) {
    case 0: case 1: case 2: case 3: {
        const uint8_t *mask = ch == 1 ? F.own + now : ch == 2 ? F.foe + now : F.bits;
        const bool own = ch == 1 || ch == 2;
        each([&](int q, int p) {
            const int4 v = keep4(ld16<ANY>(F.farmy + now + q), ld4<ANY>(mask + (own ? 0 : p * S) + q),
                                 own ? p : ch == 0 ? (int)B_NOW : (int)B_NEUTRAL);
            return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
        });
        break;
    }
    case 4: case 5: case 6: case 7: case 8:
        each([&](int q, int p) { return bytes_to_f((ld4<ANY>(F.bits + p * S + q) >> (ch - 4)) & kOnes); });
        break;
    case 10: case 11: {
        const uint8_t *mask = ch == 10 ? F.own + now : F.foe + now;
        each([&](int q, int p) { return bytes_to_f((ld4<ANY>(mask + q) >> p) & kOnes); });
        break;
    }
    case 9: case 12: case 13: {
        const uint32_t in = ch == 9 ? 0u : kOnes, all = ch == 12 ? kOnes : 0u;     // not visible; every such cell
        each([&](int q, int p) {
            const uint32_t b = ld4<ANY>(F.bits + p * S + q);
            return bytes_to_f(((b >> B_NOW) ^ in) & ((b >> B_PLACE) | all) & kOnes);
        });
        break;
    }
    case 14: case 15: case 16: case 17: case 18: case 19: {
        each([&](int, int p) {
            const float v = F.flat[p * 6 + ch - 14];
            return make_float4(v, v, v, v);
        });
        break;
    }
    case 20:
        each([&](int q, int p) {
            const int4 v = ld16<ANY>(F.last + p * S + q);
            return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
        });
        break;
    case 21: {
        // age of the sightings before, not visible now; gaps beyond the
        // table are computed in a loop of their own (one copy of log1p)
        bool far = false;
        each([&](int q, int p) {
            const uint32_t b = ld4<ANY>(F.bits + p * S + q), m = ~(b >> B_NOW) & (b >> B_ENEMY);
            const int4 lt = ld16<ANY>(F.lturn + p * S + q);
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            auto age = [&](uint32_t bit, int32_t then, float &to) {
                if (!(m & bit)) return;
                const uint32_t dt = (uint32_t)(f.t - then);
                to = g_age_table[min(dt, (uint32_t)kAgeTable - 1u)];
                far = far || dt >= (uint32_t)kAgeTable;
            };
            age(0x00000001u, lt.x, v.x);
            age(0x00000100u, lt.y, v.y);
            age(0x00010000u, lt.z, v.z);
            age(0x01000000u, lt.w, v.w);
            return v;
        });
        // wait for the table here: left to the store below, which every
        // channel shares, the wait would hold each plane's store until all
        // stores before it have reached memory (they count together)
#pragma unroll
        for (int k = 0; k < R; ++k) asm volatile("" : "+v"(x[k].x), "+v"(x[k].y), "+v"(x[k].z), "+v"(x[k].w));
        if (ballot(far) != 0ull) {
#pragma nounroll
            for (int n = 0; n < 4 * R; ++n) {
                int q = 0;
#pragma unroll
                for (int k = 0; k < R; ++k) q = n >> 2 == k ? max(c[k] + (n & 3), 0) : q;
                const int p = player(n >> 2);
                const uint32_t b = F.bits[p * S + q];
                const uint32_t dt = (uint32_t)(f.t - F.lturn[p * S + q]);
                if (((b >> B_NOW) & 1u) || !((b >> B_ENEMY) & 1u) || dt < (uint32_t)kAgeTable) continue;
                const float v = (float)(log1p((double)(int32_t)dt) / 5.0);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    if (n == 4 * k) x[k].x = v;
                    if (n == 4 * k + 1) x[k].y = v;
                    if (n == 4 * k + 2) x[k].z = v;
                    if (n == 4 * k + 3) x[k].w = v;
                }
            }
        }
        break;
    }
    default: {
        const float *v = ch == 22 ? F.cx : F.cy;
        each([&](int q, int p) {
            int r[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int row = div_w(max(q + k, 0), g);
                r[k] = (ch == 22 ? q + k - g.W * row : row) & 31;
            }
            return make_float4(v[r[0]], v[r[1]], v[r[2]], v[r[3]]);
        });
    }
    }
}

// Shift a wave's run of quads (quad 64 k + lane in x[k]) up by r values: each
// quad takes the last r values of the one before it, one DPP move each.
template <int r, int R>
__device__ __forceinline__ void shift_run(float4 (&x)[R])
{
#pragma unroll
    for (int k = R - 1; k >= 0; --k) {
        auto prev = [&](float v, float before) {
            const int first = k > 0 ? readlane(__float_as_int(before), kWave - 1) : 0;
            return __uint_as_float(wave_shr1(__float_as_uint(v), (uint32_t)first));
        };
        const float4 u = x[k], l = x[k > 0 ? k - 1 : 0];
        const float w = prev(u.w, l.w);
        if (r == 1) {
            x[k] = make_float4(w, u.x, u.y, u.z);
        } else {
            const float z = prev(u.z, l.z);
            x[k] = r == 2 ? make_float4(z, w, u.x, u.y) : make_float4(prev(u.y, l.y), z, w, u.x);
        }
    }
}

// The quads x of one plane, shifted where they have to be, to its place: sh
// floats past the byte offset base of ro.
template <bool SHIFT, int G, int R>
__device__ __forceinline__ void plane_store(float4 *px, int sh, int base, int HW, int gl, const Rsrc &ro)
{
    const int vo = G == kWave ? 0 : base, so = G == kWave ? base : 0;
    float4 x[R];
#pragma unroll
    for (int k = 0; k < R; ++k) x[k] = px[k];
    if (SHIFT && G == kWave) {
        if ((sh & 3) == 1) shift_run<1>(x);
        else if ((sh & 3) == 2) shift_run<2>(x);
        else if ((sh & 3) == 3) shift_run<3>(x);
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int c0 = 4 * (kWave * k + gl) - sh, at = vo + 16 * (kWave * k + gl);
        const u32x4 v = {__float_as_uint(x[k].x), __float_as_uint(x[k].y), __float_as_uint(x[k].z), __float_as_uint(x[k].w)};
        if (c0 >= 0 && c0 + 4 <= HW) __builtin_amdgcn_raw_buffer_store_b128(v, ro, at, so, kAuxNT);
        if (!SHIFT) continue;
        if (G == kWave) {                              // how much of an end's quad is the same for the wave
            const int head = sh & 3, tail = (HW + sh) & 3;
            if (k == 0 && head != 0) {
                if (c0 < 0 && c0 > -4) {
                    if (head == 1) __builtin_amdgcn_raw_buffer_store_b96(u32x3{v.y, v.z, v.w}, ro, at + 4, so, kEdge);
                    else if (head == 2) __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.z, v.w}, ro, at + 8, so, kEdge);
                    else __builtin_amdgcn_raw_buffer_store_b32(v.w, ro, at + 12, so, kEdge);
                }
            }
            if (tail != 0 && k == (HW + sh) >> 8) {
                if (c0 < HW && c0 + 4 > HW) {
                    if (tail == 1) __builtin_amdgcn_raw_buffer_store_b32(v.x, ro, at, so, kEdge);
                    else if (tail == 2) __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, ro, at, so, kEdge);
                    else __builtin_amdgcn_raw_buffer_store_b96(u32x3{v.x, v.y, v.z}, ro, at, so, kEdge);
                }
            }
        } else if ((c0 < 0 && c0 > -4) || (c0 < HW && c0 + 4 > HW)) {
            if (c0 >= 0) __builtin_amdgcn_raw_buffer_store_b32(v.x, ro, at, so, kEdge);
            if (c0 + 1 >= 0 && c0 + 1 < HW) __builtin_amdgcn_raw_buffer_store_b32(v.y, ro, at + 4, so, kEdge);
            if (c0 + 2 >= 0 && c0 + 2 < HW) __builtin_amdgcn_raw_buffer_store_b32(v.z, ro, at + 8, so, kEdge);
            if (c0 + 3 < HW) __builtin_amdgcn_raw_buffer_store_b32(v.w, ro, at + 12, so, kEdge);
        }
    }
}

// Plane (p, ch) of one player (of 64 / G players, G lanes each: boards whose
// planes leave most of a wave idle; of N players, one after the other), by one wave, in
// 16-byte stores on 16-byte boundaries, each round's run of 1 KB on a 128-byte
// one: lane i stores the quad of cells from 4 i - sh on, sh the floats between
// that boundary and the plane.  Where planes start inside 16 bytes (SHIFT) a
// lane reads the quad at the multiple of 4 above that and the wave shifts
// (reading LDS off its boundaries: 23x23 rollout 1,295 -> 1,400 us; small
// boards, G < 64, do, their players' shifts differ), and the quads across a
// plane's ends are written in part.  ro: the env's block from the 128-byte
// boundary at or before its first float, d floats into it.
// R: rounds of 64 quads that cover a plane (G < 64: one).
template <bool SHIFT, int G, int R, int N>
__device__ __forceinline__ void plane_out(const FeatLds &F, const FrameCtx &f, int p0, int ch, const Rsrc &ro, int d)
{
    const Geom &g = f.g;
    const int HW = g.HW, lane = lane_id(), gl = lane & (G - 1);
    const int p = G == kWave ? p0 : min(p0 + lane / G, g.P - 1);
    int sh[N], base[N], c[N * R];
    float4 x[N * R];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int fo = d + ((p + n) * kFeatC + ch) * HW;   // the plane's first float
        sh[n] = fo & (G == kWave ? 31 : 3);
        base[n] = 4 * (fo - sh[n]);
#pragma unroll
        for (int k = 0; k < R; ++k)
            c[n * R + k] = G == kWave ? min(max(4 * (kWave * k + gl) - (sh[n] & ~3), 0), g.S - 4)
                                      : min(max(4 * gl - sh[n], SHIFT ? -3 : 0), SHIFT ? HW - 1 : HW - 4);
    }
    channel<SHIFT && G != kWave, N, N * R>(F, f, p, ch, c, x);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (G == kWave ? p0 + n < g.P : p0 + lane / G < g.P) plane_store<SHIFT, G, R>(x + n * R, sh[n], base[n], HW, gl, ro);
    }
}

// The env's planes as tasks for one wave each, in the order of the tensor:
// the waves of a workgroup then write next to each other.
template <int G, int N>
__device__ __forceinline__ int plane_tasks(int P)
{
    constexpr int n = N * (kWave / G);                 // players to a task
    return (P + n - 1) / n * kFeatC;
}

template <bool SHIFT, int G, int R, int N>
__device__ __forceinline__ void plane_task(const FeatLds &F, const FrameCtx &f, int k, float *fe)
{
    const int d = (int)(((uintptr_t)fe >> 2) & 31);
    const Rsrc ro = buffer_rsrc(fe - d, 4u * (uint32_t)(d + f.g.P * kFeatC * f.g.HW));
    const int grp = k / kFeatC;
    plane_out<SHIFT, G, R, N>(F, f, grp * N * (kWave / G), k - grp * kFeatC, ro, d);
}

// The planes by a lane per cell, which writes every channel of its cell in
// dwords: about 20 vector instructions a plane and 64 cells, against 60 to
// 100 for each round of a plane task, which boards of few cells (or a second
// round of few) and batches that do not fill the chip pay in full.  The lines
// are written in parts, so large outputs are for the planes (see by_cells).
// A wave's task is 64 cells and one of `groups` parts of the players; a
// channel 21 value that comes from HBM is loaded before the stores of the
// player before it (loads and stores count together, so a later wait would be
// one for those stores).
__device__ __forceinline__ int cell_groups(const Geom &g, int nwv) { return min(g.P, max(1, nwv / g.NW)); }

__device__ __forceinline__ void cell_task(const FeatLds &F, const FrameCtx &f, int k, int groups, float *fe)
{
    const Geom &g = f.g;
    const int HW = g.HW, S = g.S, P = g.P;
    const int grp = k / g.NW, c = (k - grp * g.NW) * kWave + lane_id();
    const Rsrc ro = buffer_rsrc(fe, 4u * (uint32_t)(P * kFeatC * HW));
    if (c < HW) {
        // the frames of turns t, t - 1, ..., t - 7
        int32_t army[kHist + 1];
        uint32_t own[kHist + 1], foe[kHist + 1];
#pragma unroll
        for (int j = 0; j <= kHist; ++j) {
            const int at = ((f.t - j) & 7) * S + c;
            army[j] = F.farmy[at];
            own[j] = F.own[at];
            foe[j] = F.foe[at];
        }
        const int row = div_w(c, g);
        const float cx = F.cx[c - row * g.W], cy = F.cy[row];
        auto age = [&](int p) {                        // channel 21
            const uint32_t b = F.bits[p * S + c];
            const uint32_t dt = (uint32_t)(f.t - F.lturn[p * S + c]);
            if (!(~(b >> B_NOW) & (b >> B_ENEMY) & 1u)) return 0.0f;
            return dt < (uint32_t)kAgeTable ? g_age_table[dt] : (float)(log1p((double)(int32_t)dt) / 5.0);
        };
        const int end = (grp + 1) * P / groups;
        int p = grp * P / groups;
        float next = age(p);
#pragma nounroll
        for (; p < end; ++p) {
            const float aged = next;
            next = age(min(p + 1, end - 1));
            const uint32_t b = F.bits[p * S + c], now = b >> B_NOW, place = b >> B_PLACE;
            auto put = [&](int ch, float x) {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), ro, 4 * c, 4 * (p * kFeatC + ch) * HW, kEdge);
            };
            auto bit = [](uint32_t m, int at) { return (float)((m >> at) & 1u); };
            put(0, (float)keep(army[0], b, B_NOW));
            put(1, (float)keep(army[0], own[0], p));
            put(2, (float)keep(army[0], foe[0], p));
            put(3, (float)keep(army[0], b, B_NEUTRAL));
#pragma unroll
            for (int j = 0; j < 5; ++j) put(4 + j, bit(b, j));
            put(9, bit(now & place, 0));
            put(10, bit(own[0], p));
            put(11, bit(foe[0], p));
            put(12, bit(~now, 0));
            put(13, bit(~now & place, 0));
#pragma unroll
            for (int j = 0; j < 6; ++j) put(14 + j, F.flat[p * 6 + j]);
            put(20, (float)F.last[p * S + c]);
            put(21, aged);
            put(22, cx);
            put(23, cy);
            int32_t o0 = keep(army[0], own[0], p), f0 = keep(army[0], foe[0], p);
#pragma unroll
            for (int j = 0; j < kHist; ++j) {
                const int32_t o1 = keep(army[j + 1], own[j + 1], p), f1 = keep(army[j + 1], foe[j + 1], p);
                put(24 + j, (float)(o0 - o1));
                put(24 + kHist + j, (float)(f0 - f1));
                o0 = o1;
                f0 = f1;
            }
        }
    }
}

// Token windows: 64 of the 512 turns of `players` players' two rows (the
// enemies' army and land) per task.  Two players share the turns' stamps and
// halve the tasks, which small boards' 2 or 4 waves and many players feel (one
// player to a task and two, features and step, us: 8x8 FFA-3, 3,426 envs 78 ->
// 62; 10x10 1v1, 30,000 envs 552 -> 515; 12x12 FFA-8, 3,996 envs 283 -> 270; 32
// turns of rollout of 23x23, 512 envs 661 -> 642; 16 of 17x19 2v2, 400 envs 394
// -> 386).
template <int players>
struct TokenLoad {
    int32_t stamp, land[players];
    u32x2 army[players];
};

template <int players>
__device__ __forceinline__ int token_tasks(int P) { return (P + players - 1) / players * (kTokenWindow / kWave); }

// The turn of this lane in task k (before the episode: negative).
__device__ __forceinline__ int32_t token_turn(const FrameCtx &f, int k)
{
    return f.t - (kTokenWindow - 1) + (k & 7) * kWave + lane_id();
}

// Whether some turn of task k may be in the ring (wave-uniform).
__device__ __forceinline__ bool token_some(const FrameCtx &f, int k)
{
    return !f.fresh && f.t - (kTokenWindow - 1) + (k & 7) * kWave + kWave - 1 >= 0;
}

// The turn that the lane's slot of the ring holds.
__device__ __forceinline__ int32_t token_stamp(const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm, int k)
{
    return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rm, 4 * (token_turn(f, k) & (kTokenWindow - 1)), (int)fb.tstamp, 0);
}

template <int players>
__device__ __forceinline__ void token_values(const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm, int k, TokenLoad<players> &v)
{
    const int p0 = (k >> 3) * players, sl = token_turn(f, k) & (kTokenWindow - 1);
#pragma unroll
    for (int i = 0; i < players; ++i) {
        const int p = min(p0 + i, f.g.P - 1);          // an odd last player's twice
        v.army[i] = __builtin_amdgcn_raw_buffer_load_b64(rm, 8 * sl, (int)fb.tarmy + 8 * p * kTokenWindow, 0);
        v.land[i] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rm, 4 * sl, (int)fb.tland + 4 * p * kTokenWindow, 0);
    }
}

template <int players>
__device__ __forceinline__ TokenLoad<players> token_load(const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm, int k)
{
    TokenLoad<players> v{};
    v.stamp = -1;
    if (token_some(f, k)) {
        v.stamp = token_stamp(f, fb, rm, k);
        token_values(f, fb, rm, k, v);
    }
    return v;
}

template <int players>
__device__ __forceinline__ void token_store(const FeatLds &F, const FrameCtx &f, const TokenLoad<players> &v, int k, float *te)
{
    const int p0 = (k >> 3) * players, j = (k & 7) * kWave + lane_id();
    const int32_t tau = token_turn(f, k);
    const bool now = j == kTokenWindow - 1;                  // this turn: channels 19 and 18
    const bool have = !f.fresh && tau >= 0 && v.stamp == tau;
#pragma unroll
    for (int i = 0; i < players; ++i) {
        const int p = p0 + i;
        if (p >= f.g.P) break;
        const Rsrc rt = buffer_rsrc(te + (size_t)p * 2 * kTokenWindow, 8u * kTokenWindow);
        const float army = now ? F.flat[p * 6 + 5] : have ? (float)(int64_t)(((uint64_t)v.army[i].y << 32) | v.army[i].x) : 0.0f;
        const float land = now ? F.flat[p * 6 + 4] : have ? (float)v.land[i] : 0.0f;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(army), rt, 4 * j, 0, kAuxNT);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(land), rt, 4 * j, 4 * kTokenWindow, kAuxNT);
    }
}

// The windows of one wave where few envs share a CU (boards of three rounds
// and more): the loads of its first two tasks are issued before the
// turn's memory update and their values stored after it, so the ring's latency
// is hidden (as a last task of a few waves the windows cost 1.1 ms of the 3.9
// of 65,536 envs of 24x24); those left are loaded two at a time.  Feature
// launches keep one player to a task: 24x24, 65,536 envs 3,192, 3,289 with two.
template <int players>
struct TokenWave {
    TokenLoad<players> v0{}, v1{};
    int n = 0;               // tasks, 0 without tokens

    __device__ __forceinline__ void start(const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm, bool tokens, int wv, int nwv)
    {
        n = tokens ? token_tasks<players>(f.g.P) : 0;
        if (wv < n) v0 = token_load<players>(f, fb, rm, wv);
        if (wv + nwv < n) v1 = token_load<players>(f, fb, rm, wv + nwv);
    }

    __device__ __forceinline__ void finish(const FeatLds &F, const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm,
                                           float *te, int wv, int nwv)
    {
        if (wv < n) token_store(F, f, v0, wv, te);
        if (wv + nwv < n) token_store(F, f, v1, wv + nwv, te);
        for (int k = wv + 2 * nwv; k < n; k += 2 * nwv) {
            v0 = token_load<players>(f, fb, rm, k);
            if (k + nwv < n) v1 = token_load<players>(f, fb, rm, k + nwv);
            token_store(F, f, v0, k, te);
            if (k + nwv < n) token_store(F, f, v1, k + nwv, te);
        }
    }
};

// The windows of one wave where several envs share a CU, whose phases hide the
// latency: all of them after the update, two tasks at a time, their stamps
// first, and only turns that the ring holds are loaded (a ring that few turns
// were recorded in: 8x16 2v2, 6,000 envs with every turn loaded 192, 151;
// 16x16 2v2, 2,600 envs 115, 107).  Every load is waited for here: one left
// pending at the end is waited for in each plane after it, together with that
// plane's stores (12x12 1v1, 12,000 envs without tokens 182 us, with such a
// load 235; 8 turns of rollout of 13x15 2v2, 600 envs 226, 245).
template <int players>
__device__ __forceinline__ void token_windows(const FeatLds &F, const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm,
                                              float *te, int wv, int nwv)
{
    auto stamp = [&](int k) {
        TokenLoad<players> v{};
        v.stamp = token_some(f, k) ? token_stamp(f, fb, rm, k) : -1;
        return v;
    };
    auto values = [&](int k, TokenLoad<players> &v) {
        if (v.stamp == token_turn(f, k) && v.stamp >= 0) token_values(f, fb, rm, k, v);
    };
    auto settle = [](TokenLoad<players> &v) {
#pragma unroll
        for (int i = 0; i < players; ++i) asm volatile("" : "+v"(v.land[i]), "+v"(v.army[i].x), "+v"(v.army[i].y));
    };
    const int n = token_tasks<players>(f.g.P);
    for (int k = wv; k < n; k += 2 * nwv) {
        const int k1 = min(k + nwv, n - 1);
        TokenLoad<players> v0 = stamp(k), v1 = stamp(k1);
        asm volatile("" : "+v"(v0.stamp), "+v"(v1.stamp));
        values(k, v0);
        values(k1, v1);
        settle(v0);
        token_store(F, f, v0, k, te);
        settle(v1);
        if (k + nwv < n) token_store(F, f, v1, k + nwv, te);
    }
}

// Channels 14 to 19 of each player, and this turn's entry of the scoreboard
// ring (Section V-A: the two temporal tokens), by one wave; a fresh block's
// ring is emptied.
__device__ __forceinline__ void scoreboard_out(const FeatLds &F, const FrameCtx &f, const FeatBlock &fb, const Rsrc &rm)
{
    const int lane = lane_id(), ts = f.t & (kTokenWindow - 1);
    for (int j = lane; j < kTokenWindow; j += kWave)
        if (f.fresh || j == ts)
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(j == ts ? f.t : -1), rm, 4 * j, (int)fb.tstamp, 0);
    if (lane < f.g.P) {
        int32_t n = 0;
        for (int w = 0; w < f.g.NW; ++w) n += __popcll(F.obm[lane * 16 + w]);
        F.land[lane] = n;
    }
    wave_sync();
    if (lane < f.g.P) {
        int32_t ol = 0;
        int64_t oa = 0;
        for (int q = 0; q < f.g.P; ++q) {              // the enemies' totals
            if (q == lane || (f.g.mode == MODE_2V2 && q == (lane ^ 2))) continue;
            ol += F.land[q];
            oa += (int64_t)F.armt[q];
        }
        float *to = F.flat + 6 * lane;
        to[0] = (float)f.t;
        to[1] = (float)((double)(f.t % 50) / 50.0);
        to[2] = (float)F.land[lane];
        to[3] = (float)(int64_t)F.armt[lane];
        to[4] = (float)ol;
        to[5] = (float)oa;
        const int off = lane * kTokenWindow + ts;
        const u32x2 v = {(uint32_t)(uint64_t)oa, (uint32_t)((uint64_t)oa >> 32)};
        __builtin_amdgcn_raw_buffer_store_b64(v, rm, 8 * off, (int)fb.tarmy, 0);
        __builtin_amdgcn_raw_buffer_store_b32((uint32_t)ol, rm, 4 * off, (int)fb.tland, 0);
    }
}

}  // namespace

// G, R, N, SHIFT: see plane_out; G = 1: a lane per cell (cell_task).
template <bool SHIFT, int G, int R, int N>
__global__ __launch_bounds__(64 * kFeatMostWaves) void k_features(FeatArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int e = (int)xcd_env(blockIdx.x, gridDim.x), lane = lane_id();   // see xcd_env
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const int wv = readfirst(tid >> 6), nwv = nt >> 6;
    const FeatBlock fb = a.blk;
    FrameCtx f;
    f.g = a.g;
    const Geom &g = f.g;
    const int S = g.S, P = g.P;
    FeatLds F = feat_carve(smem, S, P);
    uint8_t *blk = a.mem + (size_t)e * fb.bytes;

    const int n16 = S >> 4;
    const size_t cell0 = (size_t)e * S;
    const EnvScalars s = a.sc[e];
    uint32_t *hdr = reinterpret_cast<uint32_t *>(blk);
    f.t = s.turn;
    f.slot = f.t & 7;
    F.army = F.farmy + f.slot * S;
    // The header and the state first, in one wait; memory and ring only where
    // they are this episode's.  What LDS then holds in their place is not
    // read: frame_update starts from 0, and an earlier frame's masks are 0.
    // First call after a reset, us, with the copies before the header and so:
    // 24x24 1v1, 65,536 envs 2,958, 2,487; 23x23 1v1, 512 envs 32.4, 29.9;
    // 28x32 FFA-7, 2,385 envs 566, 504; a later one 2,965, 2,902; 30.3, 29.3;
    // 545, 548 (8x8 1v1, 16 envs 8.2, 7.6).
    const u32x4 *header = reinterpret_cast<const u32x4 *>(blk);
    const u32x4 h0 = header[0], h1 = header[1], h2 = header[2];
    const int na = 4 * n16, mine = f.slot * na;
    u32x4 *la = reinterpret_cast<u32x4 *>(F.farmy);    // this turn's slot is the state's
    const u32x4 *so = reinterpret_cast<const u32x4 *>(a.owner + cell0), *st = reinterpret_cast<const u32x4 *>(a.type + cell0);
    const u32x4 *sa = reinterpret_cast<const u32x4 *>(a.army + cell0);
    for (int i = tid; i < na; i += nt) {
        const int j = min(i, n16 - 1);
        const u32x4 o = so[j], t = st[j], v = sa[i];
        la[mine + i] = v;
        if (i < n16) {
            reinterpret_cast<u32x4 *>(F.owner)[i] = o;
            reinterpret_cast<u32x4 *>(F.type)[i] = t;
        }
    }
    f.fresh = readfirst((int)h0[0]) != (int)kFeatMagic || (uint32_t)readfirst((int)h0[1]) != s.episode;
    int32_t stamp[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) stamp[j] = f.fresh ? -1 : readfirst((int)(j < 2 ? h0[j + 2] : j < 6 ? h1[j - 2] : h2[j - 6]));
    if (!f.fresh) {
        copy16(F.mem, blk + fb.bits, (9 * P + 16) * n16, tid, nt);
        const u32x4 *fa = reinterpret_cast<const u32x4 *>(blk + fb.farmy);
        for (int i = tid; i < 8 * na; i += 2 * nt) {
            const int j = min(i + nt, 8 * na - 1);
            const u32x4 v = fa[i], w = fa[j];
            if (i < mine || i >= mine + na) la[i] = v;
            if (j < mine || j >= mine + na) la[j] = w;
        }
    }
    // Every load has come, so that no plane waits for one and with it for the
    // stores before it (12x12 1v1, 12,000 envs: 212 us with one pending, 160 without).
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt 0, the others at most
    if (tid < 8) F.armt[tid] = 0;
    if (wv == nwv - 1 && lane < 32) {
        F.cx[lane] = (float)((double)lane / (double)(g.W - 1));
        F.cy[lane] = (float)((double)lane / (double)(g.H - 1));
    }
    lds_barrier();
    ring_masks(F, f, slots_held(stamp, f.t), tid, nt);
    cell_bitmaps<false>(g, F.owner, F.type, F.obm, nullptr, nullptr, tid, nt, [](int) { return make_uint2(0u, 0u); });
    army_totals(F, g, tid, nt);
    lds_barrier();
    if (wv == 0) team_vision(F.obm, F.vis, g);
    const Rsrc rm = buffer_rsrc(blk, fb.bytes);
    if (wv == nwv - 1) scoreboard_out(F, f, fb, rm);
    // every wave has read the header
    if (wv == nwv - 1 && lane == 0) {
        hdr[0] = kFeatMagic;
        hdr[1] = s.episode;
#pragma unroll
        for (int j = 0; j < 8; ++j) hdr[2 + j] = (uint32_t)(j == f.slot ? f.t : stamp[j]);
    }
    lds_barrier();
    const bool tokens = a.tokens != nullptr;
    float *te = tokens ? a.tokens + (size_t)e * P * 2 * kTokenWindow : nullptr;
    if constexpr (R >= 3) {
        TokenWave<1> tw;
        tw.start(f, fb, rm, tokens, wv, nwv);
        frame_update<false>(F, f, rm, fb, tid, nt);
        lds_barrier();
        if (tokens) tw.finish(F, f, fb, rm, te, wv, nwv);
    } else {
        frame_update<false>(F, f, rm, fb, tid, nt);
        lds_barrier();
        if (tokens) token_windows<2>(F, f, fb, rm, te, wv, nwv);
    }
    float *fe = a.feat + (size_t)e * (size_t)P * kFeatC * g.HW;
    if constexpr (G == 1) {
        const int groups = cell_groups(g, nwv);
        for (int k = wv; k < g.NW * groups; k += nwv) cell_task(F, f, k, groups, fe);
    } else {
        for (int k = wv; k < plane_tasks<G, N>(P); k += nwv) plane_task<SHIFT, G, R, N>(F, f, k, fe);
    }
}

// ---------------------------------------------------------------- rollouts
// T turns of one env by one workgroup: features of the state, random actor,
// step, as gen_features, gen_sample_actions and gen_step called in turn.
// Envs are independent, so no launch boundary is needed between the turns:
// the board, the feature memory and the frame ring stay in LDS, and per turn
// only the outputs go to HBM (512 envs of 23x23 with tokens: 48.0 -> 19.5 us
// a turn against two launches; 24x24 without: 35.0 -> 17.3 us, 17.2 with
// constant planes, so it is bound by the stores).
// Wave 0 plays the turn while the others write its planes; these tasks are
// handed out by a counter, so wave 0 joins when it is done.
struct RollLds {
    Lds L;                   // the live board
    EnvScalars *s;           // its scalars after the last turn
    int32_t *hdr;            // the memory block's header: magic, episode, stamp[8]
    int32_t *act;            // [8] this turn's actions
    int32_t *next;           // next task to hand out
    uint8_t *claim;          // [S] for the moves
};

constexpr int kRollExtra = 8 * 56 + 32 + 48 + 32 + 16 + 2 * 96;

__host__ __device__ inline uint32_t roll_lds_bytes(int S, int P) { return feat_lds_bytes(S, P) + (uint32_t)(21 * S + kRollExtra); }

// The next map's settings, read where a game ends (see fresh).
struct RolloutSrc {
    int e;
    __device__ __forceinline__ MapArgs map() const
    {
        const RolloutArgs &a = fresh_args<RolloutArgs>();
        return {a.prm, a.seed, a.env_base + (uint64_t)e};
    }
};

template <bool SHIFT, int G, int R, int N>
__global__ __launch_bounds__(64 * kFeatMostWaves) void k_rollout(RolloutArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int e = (int)xcd_env(blockIdx.x, gridDim.x), lane = lane_id();
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const int wv = readfirst(tid >> 6), nwv = nt >> 6;
    const FeatBlock fb = a.blk;
    FrameCtx f;
    f.g = a.g;
    const Geom &g = f.g;
    const int S = g.S, P = g.P, n16 = S >> 4, nq = S >> 2;
    FeatLds F = feat_carve(smem, S, P);
    RollLds rl;
    {
        uint8_t *x = smem + feat_lds_bytes(S, P);
        F.own = x; x += 8 * S;
        F.foe = x; x += 8 * S;
        F.army = reinterpret_cast<int32_t *>(x); x += 4 * S;
        rl.claim = x; x += S;
        rl.L.army = F.army;
        rl.L.owner = F.owner;
        rl.L.type = F.type;
        rl.L.armyc = nullptr;
        rl.L.obm = F.obm;
        rl.L.vis = F.vis;
        rl.L.gbm = reinterpret_cast<uint64_t *>(x); x += 8 * 56;
        rl.s = reinterpret_cast<EnvScalars *>(x); x += 32;
        rl.hdr = reinterpret_cast<int32_t *>(x); x += 48;
        rl.act = reinterpret_cast<int32_t *>(x); x += 32;
        rl.next = reinterpret_cast<int32_t *>(x); x += 16;
    }
    unsigned long long *const armt0 = reinterpret_cast<unsigned long long *>(rl.next + 4);   // totals, turn about
    const size_t cell0 = (size_t)e * S;
    uint8_t *blk = a.mem + (size_t)e * fb.bytes;
    const Rsrc rm = buffer_rsrc(blk, fb.bytes);
    copy16(rl.L.army, a.army + cell0, 4 * n16, tid, nt);
    copy16(rl.L.owner, a.owner + cell0, n16, tid, nt);
    copy16(rl.L.type, a.type + cell0, n16, tid, nt);
    copy16(F.mem, blk + fb.bits, (9 * P + 48) * n16, tid, nt);
    if (tid < 10) rl.hdr[tid] = reinterpret_cast<const int32_t *>(blk)[tid];
    if (wv == 1 && lane < 8) reinterpret_cast<uint32_t *>(rl.s)[lane] = reinterpret_cast<const uint32_t *>(a.sc + e)[lane];
    if (wv == 2 && lane < 24) reinterpret_cast<uint64_t *>(armt0)[lane] = 0ull;
    if (wv == nwv - 1 && lane < 32) {
        F.cx[lane] = (float)((double)lane / (double)(g.W - 1));
        F.cy[lane] = (float)((double)lane / (double)(g.H - 1));
    }
    lds_barrier();
    {
        int32_t stamp[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) stamp[j] = readfirst(rl.hdr[2 + j]);
        ring_masks(F, f, slots_held(stamp, readfirst(rl.s->turn)), tid, nt);
    }

    const uint64_t env_id = a.env_base + (uint64_t)e;
    const int groups = cell_groups(g, nwv), n_tasks = G == 1 ? g.NW * groups : plane_tasks<G, N>(P);
    for (int step = 0; step < a.n_steps; ++step) {
        // what follows from the geometry is computed anew each turn: kept
        // over the loop it costs more scalar registers than there are
        asm volatile("" : "+s"(f.g.S), "+s"(f.g.HW), "+s"(f.g.P), "+s"(f.g.W), "+s"(f.g.H), "+s"(f.g.NW));
        // ---- this turn's frame: the live board into its ring slot
        EnvScalars s;
        {
            uint32_t w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = (uint32_t)readfirst((int)reinterpret_cast<const uint32_t *>(rl.s)[k]);
            __builtin_memcpy(&s, w, 32);
        }
        f.t = s.turn;
        f.slot = f.t & 7;
        f.fresh = readfirst(rl.hdr[0]) != (int)kFeatMagic || (uint32_t)readfirst(rl.hdr[1]) != s.episode;
        if (f.fresh) ring_masks(F, f, 0u, tid, nt);    // no earlier frames
        F.armt = armt0 + 12 * (step & 1);
        F.land = reinterpret_cast<int32_t *>(F.armt + 8);
        cell_bitmaps<true>(g, F.owner, F.type, F.obm, rl.L.gbm, rl.L.gbm + 16, tid, nt, [&](int b) {
            const int4 *x = reinterpret_cast<const int4 *>(F.army) + 2 * b;
            return make_uint2(clamp4(x[0]), clamp4(x[1]));
        });
        army_totals(F, g, tid, nt);
        lds_barrier();
        // ---- vision; the actor's draws; the scoreboard ring; the header
        if (wv == 0) {
            team_vision(F.obm, F.vis, g);
        } else if (wv == 1) {
            actor_wave(g, F.obm, rl.L.gbm, rl.L.gbm + 16, s.alive, a.actor_seed, a.step0 + (uint64_t)step, env_id, rl.act);
            wave_sync();
            if (lane < P) a.actions[((size_t)step * gridDim.x + (size_t)e) * P + lane] = rl.act[lane];
        } else if (wv == 2) {
            // the ring in HBM is read by the other waves in later turns
            scoreboard_out(F, f, fb, rm);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        } else if (wv == 3) {
            if (lane < 8) rl.hdr[2 + lane] = lane == f.slot ? f.t : f.fresh ? -1 : rl.hdr[2 + lane];
            if (lane == 0) {
                rl.hdr[0] = (int)kFeatMagic;
                rl.hdr[1] = (int)s.episode;
                *rl.next = 0;
            }
            if (lane < 12) reinterpret_cast<uint64_t *>(armt0 + 12 * ((step & 1) ^ 1))[lane] = 0ull;
        }
        lds_barrier();
        float *te = a.tokens != nullptr ? a.tokens + ((size_t)step * gridDim.x + (size_t)e) * P * 2 * kTokenWindow : nullptr;
        if constexpr (R >= 3) {
            TokenWave<2> tw;
            tw.start(f, fb, rm, te != nullptr, wv, nwv);
            frame_update<true>(F, f, rm, fb, tid, nt);
            lds_barrier();
            if (te != nullptr) tw.finish(F, f, fb, rm, te, wv, nwv);
        } else {
            frame_update<true>(F, f, rm, fb, tid, nt);
            lds_barrier();
            if (te != nullptr) token_windows<2>(F, f, fb, rm, te, wv, nwv);
        }
        // ---- wave 0 plays the turn on the live board, the others write
        if (wv == 0) {
            const Turn r = advance(rl.L, g, RolloutSrc{e}, s, lane < P ? rl.act[lane] : 0, rl.claim);
            if (r.grow2 || r.grow50) {
                for (int q = lane; q < nq; q += kWave) {
                    const uint32_t inc = growing4(reinterpret_cast<const uint32_t *>(rl.L.owner)[q],
                                                  reinterpret_cast<const uint32_t *>(rl.L.type)[q], r.grow2, r.grow50);
                    int4 x = reinterpret_cast<int4 *>(rl.L.army)[q];
                    x.x = __builtin_elementwise_add_sat(x.x, (int)(inc & 1u));
                    x.y = __builtin_elementwise_add_sat(x.y, (int)((inc >> 8) & 1u));
                    x.z = __builtin_elementwise_add_sat(x.z, (int)((inc >> 16) & 1u));
                    x.w = __builtin_elementwise_add_sat(x.w, (int)(inc >> 24));
                    reinterpret_cast<int4 *>(rl.L.army)[q] = x;
                }
            }
            if (lane < P)
                a.rewards[((size_t)step * gridDim.x + (size_t)e) * P + lane] =
                    ((r.win >> lane) & 1u) ? 1 : (((r.lose >> lane) & 1u) ? -1 : 0);
            if (lane == 0) {
                a.dones[(size_t)step * gridDim.x + (size_t)e] = r.done ? 1 : 0;
                *rl.s = s;
            }
        }
        float *fe = a.feat + ((size_t)step * gridDim.x + (size_t)e) * (size_t)P * kFeatC * g.HW;
        auto hand = [&]() { return lane == 0 ? atomicAdd(rl.next, 1) : 0; };
        for (int k = readfirst(hand()); k < n_tasks;) {
            const int k2 = hand();                         // the next one, while this one is written
            if constexpr (G == 1) cell_task(F, f, k, groups, fe);
            else plane_task<SHIFT, G, R, N>(F, f, k, fe);
            k = readfirst(k2);
        }
        lds_barrier();
    }
    // ---- the board and the memory back to HBM
    copy16(a.army + cell0, rl.L.army, 4 * n16, tid, nt);
    copy16(a.owner + cell0, rl.L.owner, n16, tid, nt);
    copy16(a.type + cell0, rl.L.type, n16, tid, nt);
    for (int i = tid; i < P * nq; i += nt) reinterpret_cast<uint32_t *>(F.bits)[i] &= kMemoryBits;
    lds_barrier();
    copy16(blk + fb.bits, F.mem, (9 * P + 48) * n16, tid, nt);
    if (tid < 10) reinterpret_cast<int32_t *>(blk)[tid] = rl.hdr[tid];
    if (wv == 1 && lane < 8) reinterpret_cast<uint32_t *>(a.sc + e)[lane] = reinterpret_cast<const uint32_t *>(rl.s)[lane];
}

namespace {
std::mutex g_age_mu;
bool g_age_ready[kMaxDevices] = {};
}  // namespace

hipError_t feature_tables_ready()
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_age_mu);
    if (g_age_ready[dev]) return hipSuccess;
    std::vector<float> t(kAgeTable);
    for (int dt = 0; dt < kAgeTable; ++dt) t[(size_t)dt] = (float)(std::log1p((double)dt) / 5.0);
    e = hipMemcpyToSymbol(HIP_SYMBOL(g_age_table), t.data(), t.size() * sizeof(float), 0, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) g_age_ready[dev] = true;
    return e;
}

// How a board's planes lie in the tensor: the quads of 4 cells of one, shifted
// where it starts inside 16 bytes, and the rounds of 64 that they take on
// 128-byte lines.
struct PlaneLayout {
    bool shift;
    int quads, rounds;
};

static PlaneLayout plane_layout(int HW, const float *feat)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(feat);
    PlaneLayout l;
    l.shift = HW % 4 != 0 || (at & 15) != 0;
    l.quads = l.shift ? (HW + 3) / 4 + 1 : HW / 4;
    const int before = HW % 32 == 0 && (at & 127) == 0 ? 0 : 7;    // quads of the first line before the plane
    l.rounds = (l.quads + before + kWave - 1) / kWave;
    return l;
}

// The instance for a board: planes on 16-byte boundaries or not, two players
// to a wave where a plane (shifted or not) takes at most half of one, rounds
// of 64 quads of a plane.  Up to two rounds a wave takes the planes of
// several players one after the other: finding a channel's branch costs it about
// as much as a round (features and step with one player to a task and two:
// 16x16 1v1, 32,000 envs 890, 705 us; 13x15 1v1, 20,000 envs 512, 464; 17x19
// 2v2, 2,000 envs 120, 115; with three rounds the same either way: 25x25,
// 3,000 envs of 3 players 232, 234).  Of one round it takes two players' of 2,
// three of 3, 5 or 6, four of 4, 7 or 8: no more than one place is idle (two
// and three or four: 13x15 FFA-7 with tokens, 338 envs 48.0, 44.9; 8x20 FFA-3,
// 5,225 envs 111, 108; 14x14 FFA-8, 2,000 envs 150, 148; 16x16 2v2, 16,000 envs
// 610, 617; 16 turns of rollout of 12x16 2v2, 400 envs 224, 207).
template <class F>
static void by_layout(const PlaneLayout &l, int P, F &&go)
{
    auto pick = [&](auto shift) {
        constexpr std::integral_constant<int, 64> wave{};
        constexpr std::integral_constant<int, 1> one{};
        constexpr std::integral_constant<int, 2> two{};
        constexpr std::integral_constant<int, 3> three{};
        constexpr std::integral_constant<int, 4> four{};
        constexpr std::integral_constant<int, 5> five{};
        if (l.quads <= 32) go(shift, std::integral_constant<int, 32>{}, one, one);
        else if (l.rounds == 1 && P == 2) go(shift, wave, one, two);
        else if (l.rounds == 1 && (P == 4 || P > 6)) go(shift, wave, one, four);
        else if (l.rounds == 1) go(shift, wave, one, three);
        else if (l.rounds == 2) go(shift, wave, two, two);
        else if (l.rounds == 3) go(shift, wave, three, one);
        else if (l.rounds == 4) go(shift, wave, four, one);
        else go(shift, wave, five, one);
    };
    if (l.shift) pick(std::true_type{});
    else pick(std::false_type{});
}

// Whether a batch's features go out by cells (cell_task) rather than by plane
// tasks: outputs that the 256 MB last-level cache holds, whose lines in parts
// it puts together, of boards on which a plane task works for few cells.
// Measured on 1,300 boards and batches (features and step, us, by planes and
// by cells; more than these sizes cost the cells up to 1.3 times the planes):
// - planes that start inside 16 bytes, up to 256 cells: 15x15 FFA-8, 300 envs
//   49.8, 33.2; 13x15 FFA-7 with tokens, 338 envs 45.9, 33.8; 15x15 2v2, 1,500
//   envs (205 MB) 85.6, 70.2; 410 MB 143, 135 and 1v1 144, 156;
// - the same with up to 350 cells: 17x17 FFA-8, 300 envs 54.9, 40; 17x17 1v1,
//   1,500 envs (132 MB) 58.0, 61.3; 23x23, 621 envs 43, 45;
// - aligned planes where a task leaves more than 40% of its lanes idle (8x8
//   FFA-3, 1,500 envs 35.4, 25.2; or a second round of few quads:
//   12x20 FFA-8, 100 envs 27.6, 25.4), or more than 20% and the output is not
//   a matter of latency (10x10 2v2, 1,500 envs 48.5, 37.7; 300 envs 20.7, 20.5);
// - others are the same or slower by cells (16x16 2v2, 642 envs 36.5, 43.2;
//   24x24 1v1, 1,140 envs 63, 75).
static bool by_cells(const Geom &g, const PlaneLayout &l, int n_envs)
{
    const uint64_t bytes = 4ull * kFeatC * (uint64_t)n_envs * (uint64_t)(g.P * g.HW);
    if (l.shift && g.HW <= 256) return bytes <= 200000000ull;
    if (bytes > 110000000ull) return false;
    if (l.shift) return g.HW <= 350;
    if (l.quads > 32) return l.rounds == 2 && g.HW <= 272;
    const int used = g.P * l.quads, lanes = kWave * ((g.P + 1) / 2);
    return 5 * used < 3 * lanes || (5 * used < 4 * lanes && bytes > 50000000ull);
}

// Workgroups that one round over the chip holds, one to a CU.
constexpr int kCUs = 256;

hipError_t launch_features(const FeatArgs &a, int n_envs, hipStream_t stream)
{
    const PlaneLayout layout = plane_layout(a.g.HW, a.feat);
    const uint32_t lds = feat_lds_bytes(a.g.S, a.g.P);
    if (by_cells(a.g, layout, n_envs)) {
        // A wave's tasks are 64 cells of some players: 8 waves while a CU holds
        // one or two envs, then 4, or 2 on boards of few tasks (8, 4 and 2
        // waves: 15x15 1v1, 800 envs 32.0, 25.1, 26.9; 300 envs 20.1, 20.0,
        // 22; 9x9 1v1, 6,000 envs 152, 92, 77; 13x15 1v1, 5,058 envs 160, 157, 178).
        const int nwv = n_envs <= 2 * kCUs ? 8 : a.g.NW <= 2 && a.g.P <= 4 && n_envs > 8 * kCUs ? 2 : 4;
        hipLaunchKernelGGL((k_features<true, 1, 1, 1>), dim3((unsigned)n_envs), dim3(kWave * nwv), lds, stream, a);
        return hipGetLastError();
    }
    // Waves per env: as many as fill a CU's 32 with the envs that fit its
    // LDS, so that a small board's phases overlap other envs' (10x10 1v1,
    // 30,000 envs: 8 waves 545 us, 4 waves 426, 2 waves 365; 16x16 2v2,
    // 16,000 envs: 764, 645, 910; 25x25 FFA-8, 2,000 envs: 387, 467, 810);
    // 8 where the batch leaves the chip idle anyway (16x16 1v1, 64 envs:
    // 16.8, 20.2, 27.9; 700 envs: 24.8, 25.4, 32.5), and 16 where every env
    // has a CU of its own (28x14 FFA-8, 60 envs: 39.0 -> 33.7; 24x24 1v1, 64
    // envs: 21.6 -> 19.9; but 500 envs: 34.7 -> 39.1; features and step).
    // 16 also where the LDS leaves room for one env, or for two of more than
    // 4 players (8 and 16 waves: 31x31 FFA-8, 800 envs 285, 259; 28x32 FFA-7
    // with tokens, 2,385 envs 630, 548; 31x31 2v2, 1,500 envs 252, 224; 25x25
    // FFA-8, 1,024 envs 209, 196; but 31x30 1v1, 6,000 envs 490, 552).
    const uint32_t fit = 160u * 1024u / lds;
    const bool most = n_envs <= kCUs || fit == 1 || (fit == 2 && a.g.P > 4);
    // 12 below 512 envs, where some CUs hold one env and some two (8, 12 and 16
    // waves, features alone: 24x24 1v1, 320 envs 20.3, 19.9, 25.3; 25x25 FFA-4
    // with tokens, 300 envs 44.5, 42.4, 48.0; FFA-8 16x16, 300 envs 29.2, 28.6,
    // 32.7; 23x23 1v1, 450 envs 25.5, 25.0, 28.3; 12x12 1v1, 400 envs 11.4,
    // 11.3, 15.1; 28x28 2v2, 260 envs 41.6, 41.8, 46.9).
    int nwv = fit < 6 || n_envs <= 1024 ? kFeatWaves : fit < 16 ? 4 : 2;
    if (most) nwv = kFeatMostWaves;
    else if (n_envs < 2 * kCUs) nwv = 12;
    by_layout(layout, a.g.P, [&](auto shift, auto lanes, auto rounds, auto players) {
        hipLaunchKernelGGL((k_features<shift.value, lanes.value, rounds.value, players.value>), dim3((unsigned)n_envs),
                           dim3(kWave * nwv), lds, stream, a);
    });
    return hipGetLastError();
}

// The same for rollouts, whose turns write on and on: less of a turn's output
// stays in the cache, and more where a board is few cells and players (us of 4
// to 10 turns by planes and by cells, and the output of a turn: 8x8 FFA-3,
// 1,500 envs 271, 137, 43 MB; 8,000 envs 921, 525, 233 MB; 9x9 2v2, 8,000 envs
// 775, 631, 393 MB; 15x15 FFA-8, 300 envs 392, 314, 82 MB; 512 envs 409, 510,
// 140 MB; 17x17 2v2, 300 envs 218, 140, 52 MB; 17x19 FFA-8, 200 envs 232, 281,
// 78 MB; aligned planes of more than 32 quads: 12x20 2v2, 512 envs 160, 196).
// Of larger boards, whose plane tasks take three rounds and more, only outputs
// of a few turns stay (8 turns by planes and by cells: 19x21 2v2, 144 envs (35
// MB) 106.5, 82.4; 267 envs (65 MB) 193, 234; 25x25 1v1, 105 envs 87.8, 77.0;
// 25x25 FFA-8, 46 envs 227, 159; 31x31 1v1, 119 envs 96.9, 86.9; 210 envs of
// 29x27 (50 MB) 104.5, 113.8), and of the aligned ones only those whose third
// round is half empty (24x24 FFA-8, 42 envs 176, 151; 24x24 1v1, 114 envs 75.8,
// 77.2, 171 envs 74.4, 71.0; but 20x20 1v1, 164 envs 65.2, 72.3; 28x28 1v1, 83
// envs 84.2, 90.2; 32x32 FFA-8, 24 envs 206, 215).
static bool turns_by_cells(const Geom &g, const PlaneLayout &l, uint64_t bytes)
{
    const uint64_t most = g.HW > 350         ? 45000000ull
                          : g.NW * g.P <= 8  ? 400000000ull
                          : g.HW <= 256      ? 110000000ull
                                             : 60000000ull;
    if (bytes > most) return false;
    if (l.shift) return true;
    if (l.rounds == 3) return 5 * l.quads < 4 * kWave * 3;
    return l.quads <= 32 && 5 * g.P * l.quads < 3 * kWave * ((g.P + 1) / 2);
}

// Waves 0 to 3 have parts of a turn of their own.
constexpr int kRollLeastWaves = 4;
static_assert(kRollLeastWaves >= 4 && kFeatWaves >= kRollLeastWaves && kFeatMostWaves >= kRollLeastWaves, "a wave per part of a turn");

hipError_t launch_rollout(const RolloutArgs &a, int n_envs, hipStream_t stream)
{
    const PlaneLayout layout = plane_layout(a.g.HW, a.feat);
    const uint32_t lds = roll_lds_bytes(a.g.S, a.g.P);
    const uint64_t bytes = 4ull * kFeatC * (uint64_t)n_envs * (uint64_t)(a.g.P * a.g.HW);
    if (turns_by_cells(a.g, layout, bytes)) {
        // (4, 8 and 16 waves: 15x15 2v2, 200 envs 144, 108, 103; 300 envs 134,
        // 115, 163; 512 envs (70 MB) 251, 236, 170; 8x8 1v1, 1,500 envs 127,
        // 188, 331; 9x9 FFA-8, 1,500 envs 563, 394, 487; 13x15 2v2, 800 envs
        // 411, 339, 389)
        const bool one = n_envs <= kCUs || (n_envs <= 2 * kCUs && bytes > 60000000ull);
        const int nwv = one ? kFeatMostWaves : n_envs > 2 * kCUs && a.g.NW * a.g.P <= 8 ? kRollLeastWaves : kFeatWaves;
        hipLaunchKernelGGL((k_rollout<true, 1, 1, 1>), dim3((unsigned)n_envs), dim3(kWave * nwv), lds, stream, a);
        return hipGetLastError();
    }
    // Waves per env: 16 where a CU has one env, by the batch or by the LDS;
    // 4 in larger batches of boards of which many fit, so that more envs'
    // serial parts run side by side, as long as a turn has little to write
    // (us of 3 to 16 turns with 4, 8 and 16 waves: 8x8 FFA-3, 5,000 envs 749,
    // 934, -; 10x10 1v1, 600 envs 108, 128, -; 13x15 1v1, 5,000 envs 705, 845, -;
    // but 16x16 1v1, 1,000 envs 179, 170; 10x10 2v2, 1,500 envs 327, 302; 13x15
    // 2v2, 1,500 envs 571, 498; 25x25 FFA-8, 512 envs 607, 369, 320; 31x31 1v1
    // 215, 146, 136; 23x23 1v1 218, 167, 185).
    const uint32_t fit = 160u * 1024u / lds;
    const bool few = a.g.P == 2 ? fit >= 7 : a.g.P <= 4 && fit >= 12;
    const int nwv = n_envs <= kCUs || fit == 1 ? kFeatMostWaves : n_envs > 2 * kCUs && few ? kRollLeastWaves : kFeatWaves;
    by_layout(layout, a.g.P, [&](auto shift, auto lanes, auto rounds, auto players) {
        hipLaunchKernelGGL((k_rollout<shift.value, lanes.value, rounds.value, players.value>), dim3((unsigned)n_envs),
                           dim3(kWave * nwv), lds, stream, a);
    });
    return hipGetLastError();
}

}  // namespace gen
