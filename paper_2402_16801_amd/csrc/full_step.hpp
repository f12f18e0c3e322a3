// One step of one full-Craftax environment by one wavefront.
//
// The player's state is wave-uniform and stays packed as in the record (every lane computes the same
// values, so the compiler keeps them in scalar registers and branches on them without divergence; see
// Player); lane k < 14 holds mob slot k of the current floor as one word, lane k < 10 plant slot k.
// The phases follow section "Craftax: An Extension of Crafter ..." for what exists (floors,
// ladders, combat with three damage elements, bow, spells, potions, enchanting, attributes,
// boss waves); their order and every constant are this library's own frozen reading:
// action -> mobs (melee, passive, mob projectiles, player projectiles, ranged) -> despawn /
// spawn -> plants -> needs -> reward, done.
#pragma once

#include "full_common.hpp"

namespace cf {

// The player's state stays packed as the record holds it, except what nearly every step touches: the 43
// actions and the needs take single fields out with a shift and a mask.  Unpacked it is 55 scalars,
// more than the scalar registers hold beside the rest of the step, and every one that is spilled
// costs two vector instructions (to a lane of a vector register and back).  Packed, with mob slots as
// single words: 1,027 -> 788 vector instructions per environment and step, no scratch; a step of 4,096
// environments 16.7 -> 15.3 us, of 32,768 109 -> 103, a rollout of 64 steps and 4,096 environments 807 -> 728.
// Kills, the floors visited, the potion map, the time and the seed stay in the LDS copy of the record.
struct Flags {   // record word R_FLAGS
    uint32_t sleeping : 1, resting : 1, fireball : 1, iceball : 1, book : 2, pickaxe : 3, sword : 3, sword_ench : 2, bow : 1, bow_ench : 2,
             boss_vulnerable : 1, boss_hits : 4, unused : 10;
};
struct Attr { uint32_t armour : 8, armour_ench : 8, xp : 4, dex : 3, str : 3, intel : 3, unused : 3; };   // R_ATTR; armour: 4 x 2 bits each
static_assert(sizeof(Flags) == 4 && sizeof(Attr) == 4, "one record word each");
struct Items {   // R_INV .. R_POT: ten counts, then the six potions, a byte each
    uint64_t lo, hi;
    __device__ int get(int i) const { return (int)((i < 8 ? lo >> (8 * i) : hi >> (8 * (i - 8))) & 0xFFu); }
    __device__ void add(int i, int d) { if (i < 8) lo += (uint64_t)(int64_t)d << (8 * i); else hi += (uint64_t)(int64_t)d << (8 * (i - 8)); }   // the byte must neither under- nor overflow
};
constexpr int I_POTION = 10;
static_assert(I_WOOD == 0 && I_STONE == 1 && I_COAL == 2 && I_IRON == 3 && I_DIAMOND == 4, "crafting costs are packed in this order");
struct Player {
    int px, py, dir, floor;
    Flags f;
    Attr a;
    Items inv;
    int vit[5];
    uint32_t cnt;                      // R_CNT: hunger, thirst, fatigue, recover as signed bytes
    uint32_t mana_word;                // R_MANA: its mana byte is vit[V_MANA]; mana counter (signed byte), day phase
    uint32_t ach[3];
};

__device__ inline int sext8(uint32_t v) { return (int)(int8_t)(v & 0xFFu); }

// The record as it was before the step: a whole wavefront holds word l of it in lane l, from where a word is one
// instruction away; a group of lanes reads it in LDS.
template <int GW>
struct RecordWords {
    const uint32_t* rec;
    uint32_t mine;
    __device__ __forceinline__ uint32_t operator[](int i) const { return GW == 64 ? (uint32_t)lane_get((int)mine, i) : rec[i]; }
};
static_assert(REC_DWORDS == 64, "a record word per lane");
template <int GW>
__device__ __forceinline__ void unpack_player(const RecordWords<GW>& old, Player& P)
{
    const uint32_t pos = old[R_POS];
    P.px = pos & 0xFF; P.py = (pos >> 8) & 0xFF; P.dir = (pos >> 16) & 0xFF; P.floor = (pos >> 24) & 0xF;
    P.f = __builtin_bit_cast(Flags, old[R_FLAGS]);
    P.a = __builtin_bit_cast(Attr, old[R_ATTR]);
    P.inv.lo = (uint64_t)old[R_INV] | ((uint64_t)old[R_INV + 1] << 32);
    P.inv.hi = (uint64_t)old[R_INV + 2] | ((uint64_t)old[R_POT] << 32);
    const uint32_t v = old[R_VIT];
    P.mana_word = old[R_MANA];
#pragma unroll
    for (int i = 0; i < 4; ++i) P.vit[i] = (v >> (8 * i)) & 0xFF;
    P.vit[V_MANA] = P.mana_word & 0xFF;
    P.cnt = old[R_CNT];
#pragma unroll
    for (int i = 0; i < 3; ++i) P.ach[i] = old[R_ACH + i];
}

// packs everything that can change back into the LDS copy of the record (one lane writes); t: the new time
__device__ __forceinline__ void pack_player(uint32_t* rec, const Player& P, uint32_t t)
{
    rec[R_POS] = (uint32_t)P.px | ((uint32_t)P.py << 8) | ((uint32_t)P.dir << 16) | ((uint32_t)P.floor << 24);
    rec[R_FLAGS] = __builtin_bit_cast(uint32_t, P.f);
    rec[R_ATTR] = __builtin_bit_cast(uint32_t, P.a);
    rec[R_INV] = (uint32_t)P.inv.lo; rec[R_INV + 1] = (uint32_t)(P.inv.lo >> 32);
    rec[R_INV + 2] = (uint32_t)P.inv.hi; rec[R_POT] = (uint32_t)(P.inv.hi >> 32);
    rec[R_VIT] = (uint32_t)P.vit[0] | ((uint32_t)P.vit[1] << 8) | ((uint32_t)P.vit[2] << 16) | ((uint32_t)P.vit[3] << 24);
    rec[R_MANA] = (P.mana_word & ~0xFFu) | (uint32_t)P.vit[V_MANA];
    rec[R_CNT] = P.cnt;
    rec[R_ACH] = P.ach[0]; rec[R_ACH + 1] = P.ach[1]; rec[R_ACH + 2] = P.ach[2];
    rec[R_T] = t;
}
static_assert(R_POT == R_INV + 3, "sixteen item bytes in a row");

__device__ inline void clear_counter(Player& P, int k) { P.cnt &= ~(0xFFu << (8 * k)); }
__device__ inline void unlock(Player& P, int a)
{
    const uint32_t bit = 1u << (a & 31);
    const int w = a >> 5;
    P.ach[0] |= w == 0 ? bit : 0u; P.ach[1] |= w == 1 ? bit : 0u; P.ach[2] |= w == 2 ? bit : 0u;
}
__device__ inline int cap_health(const Player& P) { return 9 + (5 * ((int)P.a.str - 1)) / 4; }
__device__ inline int cap_need(const Player& P) { return 9 + 2 * ((int)P.a.dex - 1); }
__device__ inline int cap_mana(const Player& P) { return 9 + 3 * ((int)P.a.intel - 1); }
__device__ inline int toward(int dx, int dy) { const bool along = iabs(dx) >= iabs(dy); return (along ? 2 : 4) + ((along ? dx : dy) >> 31); }   // 1 left, 2 right, 3 up, 4 down
// damage after defence: every element is reduced by its own percentage, integer parts
__device__ inline int through(int ap, int af, int ai, int dp, int df, int di)
{
    return ap * (100 - dp) / 100 + af * (100 - df) / 100 + ai * (100 - di) / 100;
}

// The window of floor f around (px, py), of both maps, its load and its arrival in LDS apart: a dword of
// each map per lane and turn (a byte per lane, as 13 columns in three turns: steps of 4,096 environments 14.6 us, now 14.2,
// of 32,768 94.0 and 89.9).
template <int GW = 64>
struct Window {
    static constexpr int TURNS = (WIN_DWORDS + GW - 1) / GW;
    uint32_t b[TURNS], il[TURNS];
    __device__ __forceinline__ void fetch(int l, const uint8_t* __restrict__ maps, int f, int px, int py)
    {
#pragma unroll
        for (int it = 0; it < TURNS; ++it) {
            const int i = l + GW * it, x = win_x0(px) + 4 * (i & 3), y = win_y0(py) + (i >> 2);
            b[it] = 0x01010101u * (uint32_t)B_OOB; il[it] = 0x01010101u * (uint32_t)(MAX_LIGHT << 3);
            if (i < WIN_DWORDS && inb(x, y)) {
                const uint32_t* cells = reinterpret_cast<const uint32_t*>(maps + block_off(f, x, y));
                b[it] = cells[0]; il[it] = cells[CELLS / 4];
            }
        }
    }
    __device__ __forceinline__ void park(int l, uint32_t* wb, uint32_t* wi) const
    {
#pragma unroll
        for (int it = 0; it < TURNS; ++it) if (l + GW * it < WIN_DWORDS) { wb[l + GW * it] = b[it]; wi[l + GW * it] = il[it]; }
    }
};
template <int GW = 64>
__device__ __forceinline__ void load_window(int l, const uint8_t* __restrict__ maps, int f, int px, int py, uint32_t* e)
{
    Window<GW> w;
    w.fetch(l, maps, f, px, py);
    w.park(l, e + L_WB, e + L_WI);
}

// A mob slot in its packed form (0 when empty): bit 0 alive, bits 1..12 the cell, so "is this live slot
// on that cell" is one AND and one compare against cell_key, a move one bit-field insert, a kill "= 0".
struct MobRegs {
    uint32_t w;
    __device__ uint32_t alive() const { return w & 1u; }
    __device__ int x() const { return (int)__builtin_amdgcn_ubfe(w, 1, 6); }
    __device__ int y() const { return (int)__builtin_amdgcn_ubfe(w, 7, 6); }
    __device__ int dir() const { return (int)__builtin_amdgcn_ubfe(w, 13, 3); }
    __device__ int cd() const { return (int)__builtin_amdgcn_ubfe(w, 21, 4); }
    __device__ int type() const { return (int)__builtin_amdgcn_ubfe(w, 25, 5); }
};
constexpr uint32_t KEY_MASK = 0x1FFFu, HP_SHIFT = 16, CD_SHIFT = 21, TYPE_SHIFT = 25;
__device__ inline uint32_t cell_key(int x, int y) { return 1u | ((uint32_t)x << 1) | ((uint32_t)y << 7); }
__device__ inline void set_cooldown(MobRegs& m, int cd) { m.w = (m.w & ~(15u << CD_SHIFT)) | ((uint32_t)cd << CD_SHIFT); }
__device__ inline void clear_mob(MobRegs& m) { m.w = 0u; }

struct StepOut { bool done; float reward; int wx0, wy0; uint32_t t; uint32_t unlocked[3]; };   // t: time after the step; unlocked: achievement bits new after this step

enum Intent : int { N_NONE = 0, N_DAMAGE, N_DAMAGE_DIE, N_DIE, N_MOVE, N_SHOOT, N_FLY, N_PPROJ };

// e: this wave's LDS area with the record loaded; old: the record once more, as it was.  genv: the environment's 1024-byte block in
// HBM.  maps: its floors.  m, qw: this lane's mob slot (current floor) and plant word.
// KEEP (kernels that keep an environment from step to step): m comes in as the last step left it, and the
// windows are only loaded if those in LDS (kept: their window_key, or 0) are not the ones around the player's current position (a step to the side
// leaves them as they are three times out of four);
// every change a step makes to the maps inside the windows is made in the windows too, so kept ones
// equal fresh ones.
// table: lane 0 holds the zombie threshold of the day phase (see day_table).
// after_load: called once the loads of the current window have been issued and stored, before the
// wave waits for them (the caller parks data it fetched earlier there).
__device__ inline uint32_t window_key(int f, int px, int py) { return 0x80000000u | ((uint32_t)win_x0(px) & 0xFFu) | ((uint32_t)py << 8) | ((uint32_t)f << 16); }
template <int GW = 64, bool KEEP = false, typename AfterLoad>
__device__ __forceinline__ StepOut step_env(const int l, const uint32_t env, uint32_t* e, const RecordWords<GW>& old, uint32_t* __restrict__ genv,
                                   uint8_t* __restrict__ maps, const int action_in,
                                   const uint32_t table, const Params& p, MobRegs& m, uint32_t& qw, Player& P, uint32_t& kept, AfterLoad&& after_load)
{
    using G = Lanes<GW>;
    uint32_t* rec = e + L_REC;
    uint8_t* wb = reinterpret_cast<uint8_t*>(e + L_WB);
    uint8_t* wi = reinterpret_cast<uint8_t*>(e + L_WI);
    unpack_player<GW>(old, P);
    const int phase = (int)(P.mana_word >> 16);
    const uint32_t seed_lo = old[R_SEED_LO], seed_hi = old[R_SEED_HI];

    // this step's draws: lane k computes Philox block k = (move k, decision k, plant-eaten k, misc k)
    const U4 rnd = philox4x32_10(env, old[R_T], old[R_EPISODE], (cx::DOM_STEP << 16) | (uint32_t)(l < NSLOT ? l : 0), seed_lo, seed_hi);
    auto misc = [&](int i) { return (uint32_t)G::get((int)rnd.w[3], i); };

    // mob table of the current floor and the window around the player
    if (!KEEP) m.w = l < NSLOT ? genv[REC_DWORDS + P.floor * MOBTAB_DWORDS + l] : 0u;
    qw = l < NPLANT ? rec[R_PLANT + l] : 0u;
    // block under every plant (floor 0), fetched before anything is stored this step
    int q_block = B_INVALID;
    if (qw & 1u) q_block = maps[block_off(0, (int)((qw >> 1) & 63u), (int)((qw >> 7) & 63u))];
    int wx0 = win_x0(P.px), wy0 = win_y0(P.py);
    if (!KEEP || kept != window_key(P.floor, P.px, P.py)) {
        load_window<GW>(l, maps, P.floor, P.px, P.py, e);
        kept = window_key(P.floor, P.px, P.py);
    }
    after_load();
    wave_sync();

    auto win_b = [&](int x, int y) { return G::uni((int)wb[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)]); };
    auto win_i = [&](int x, int y) { return G::uni((int)wi[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)]); };
    auto in_win = [&](int x, int y) { return (unsigned)(x - wx0) < (unsigned)WIN_COLS && (unsigned)(y - wy0) < (unsigned)WIN_ROWS; };
    auto occ_mask = [&](int x, int y) -> uint32_t { return (uint32_t)G::ballot((m.w & KEY_MASK) == cell_key(x, y)); };
    // the one block cell the player may change this step; mobs read their terrain from HBM and
    // take this cell from here instead
    int patch_f = -1, patch_x = -1, patch_y = -1, patch_b = 0;
    auto set_block = [&](int x, int y, int b) {
        if (l == 0) {
            maps[block_off(P.floor, x, y)] = (uint8_t)b;
            if (in_win(x, y)) wb[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)] = (uint8_t)b;
        }
        wave_sync();
    };
    auto set_facing_block = [&](int x, int y, int b) {
        patch_f = P.floor; patch_x = x; patch_y = y; patch_b = b;
        set_block(x, y, b);
    };
    const int health0 = P.vit[V_HEALTH];

    // the player hurts mob slot k; returns true when it died
    auto hurt_mob = [&](int k, int ap, int af, int ai) -> bool {
        if (k >= S_MPROJ0) return false;                       // projectiles cannot be hit
        const uint32_t hit = (uint32_t)G::get((int)m.w, k);
        const CreatureRow c = creature((int)((hit >> TYPE_SHIFT) & 31u));
        const int nhp = (int)((hit >> HP_SHIFT) & 31u) - through(ap, af, ai, c.Dp, c.Df, c.Di);
        if (nhp > 0) { if (l == k) m.w = (m.w & ~(31u << HP_SHIFT)) | ((uint32_t)nhp << HP_SHIFT); return false; }
        if (l == k) clear_mob(m);
        unlock(P, c.ach);
        if (k >= S_PASSIVE0) { P.vit[V_FOOD] = min(cap_need(P), P.vit[V_FOOD] + FOOD_MEAT); clear_counter(P, K_HUNGER); }
        else {
            const int f = P.floor;
            const uint32_t counts = G::uniu(rec[R_KILLS + (f >> 2)]);
            int kf = (int)((counts >> (8 * (f & 3))) & 0xFFu);
            if (kf < 255) {
                ++kf;
                if (l == 0) rec[R_KILLS + (f >> 2)] = counts + (1u << (8 * (f & 3)));
                wave_sync();
            }
            // the way down opens once enough enemies of this floor are gone
            if (f >= 1 && f < FLOORS - 1 && kf >= KILLS_TO_CLEAR) {
                const uint32_t lw = G::uniu(rec[R_LADDER + f]);
                const int lx = (lw >> 16) & 0xFF, ly = (lw >> 24) & 0xFF;
                int il;
                if (in_win(lx, ly)) il = win_i(lx, ly);
                else {
                    __threadfence();                           // a torch placed this step may have lit that cell
                    il = G::uni((int)__hip_atomic_load(maps + il_off(f, lx, ly), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
                if ((il & 7) == IT_LADDER_DOWN_BLOCKED) {
                    const int nil = (il & ~7) | IT_LADDER_DOWN;
                    if (l == 0) {
                        maps[il_off(f, lx, ly)] = (uint8_t)nil;
                        if (in_win(lx, ly)) wi[CX_IDX((ly - wy0) * WIN_PITCH + (lx - wx0), WIN_ROWS * WIN_PITCH)] = (uint8_t)nil;
                    }
                    wave_sync();
                }
            }
        }
        return true;
    };
    auto spawn_mob = [&](int slot, int x, int y, int dir, int type, int hp) {
        if (l == slot) m.w = cell_key(x, y) | ((uint32_t)dir << 13) | ((uint32_t)hp << HP_SHIFT) | ((uint32_t)type << TYPE_SHIFT);
    };
    auto shot_attack = [&](int kind, int& ap, int& af, int& ai) {
        ap = af = ai = 0;
        if (kind == PP_ARROW) { ap = 2 + ((int)P.a.dex - 1); if (P.f.bow_ench == 1) af = 4; if (P.f.bow_ench == 2) ai = 4; }
        else if (kind == PP_FIREBALL) af = 4 + 2 * ((int)P.a.intel - 1);
        else ai = 4 + 2 * ((int)P.a.intel - 1);
    };

    // ---- phase 1: the player's action -------------------------------------------------------
    int a = (action_in < 0 || action_in >= A_COUNT) ? A_NOOP : action_in;
    if (P.f.sleeping || P.f.resting) a = A_NOOP;
    // table / furnace within one cell of the player (crafting never moves, so this is final)
    bool near_table, near_furnace;
    {
        int b = B_INVALID;
        if (l < 9) b = wb[CX_IDX((P.py - wy0 - 1 + l / 3) * WIN_PITCH + (P.px - wx0 - 1 + l % 3), WIN_ROWS * WIN_PITCH)];
        near_table = G::ballot(b == B_TABLE) != 0;
        near_furnace = G::ballot(b == B_FURNACE) != 0;
    }
    auto try_craft = [&](bool need_furnace, int wood, int stone, int coal, int iron, int diamond) -> bool {
        if (!near_table || (need_furnace && !near_furnace)) return false;
        if (P.inv.get(I_WOOD) < wood || P.inv.get(I_STONE) < stone || P.inv.get(I_COAL) < coal || P.inv.get(I_IRON) < iron || P.inv.get(I_DIAMOND) < diamond) return false;
        P.inv.lo -= (uint64_t)((uint32_t)wood | ((uint32_t)stone << 8) | ((uint32_t)coal << 16) | ((uint32_t)iron << 24)) | ((uint64_t)diamond << 32);
        return true;
    };
    auto change_floor = [&](int nf, int x, int y) {
        const uint32_t nw = l < NSLOT ? genv[REC_DWORDS + nf * MOBTAB_DWORDS + l] : 0u;
        if (G::ballot((nw & KEY_MASK) == cell_key(x, y))) return;         // the far end of the ladder must be free
        if (l < NSLOT) genv[REC_DWORDS + P.floor * MOBTAB_DWORDS + l] = m.w;
        m.w = nw;
        P.floor = nf; P.px = x; P.py = y;
        const uint32_t perm_visited = G::uniu(rec[R_PERM]);
        if (!((perm_visited >> (18 + nf)) & 1u)) {
            if (l == 0) rec[R_PERM] = perm_visited | (1u << (18 + nf));
            if (P.a.xp < 15) ++P.a.xp;                                   // section "Attributes": a point per new floor
            const int ea = enter_ach(nf);
            if (ea >= 0) unlock(P, ea);
        }
        wave_sync();
        wx0 = win_x0(x); wy0 = win_y0(y);
        load_window<GW>(l, maps, nf, x, y, e);
        kept = window_key(nf, x, y);
        wave_sync();
    };
    auto stock = [&](int item, int n) { const int have = P.inv.get(item); P.inv.add(item, min(INV_MAX, have + n) - have); };
    // a projectile of the player leaves the facing cell
    auto shoot = [&](int kind, int tx, int ty, bool t_ok) -> bool {
        if (!t_ok) return false;
        const uint32_t om = occ_mask(tx, ty);
        if (om) {
            const int k = __builtin_ctz(om);
            if (k >= S_MPROJ0) return false;
            int ap, af, ai;
            shot_attack(kind, ap, af, ai);
            hurt_mob(k, ap, af, ai);
            return true;
        }
        const uint32_t free_slots = ~(uint32_t)G::ballot(m.alive() != 0u) & (7u << S_PPROJ0);
        if (!free_slots || !in_set(FLYABLE, win_b(tx, ty))) return false;
        spawn_mob(__builtin_ctz(free_slots), tx, ty, P.dir, kind, 0);
        return true;
    };

    if (a >= A_LEFT && a <= A_DOWN) {
        P.dir = a;
        const int tx = P.px + dir_dx(a), ty = P.py + dir_dy(a);
        if (inb(tx, ty) && occ_mask(tx, ty) == 0) {
            const int b = win_b(tx, ty);
            if (in_set(WALKABLE, b)) { P.px = tx; P.py = ty; }
            else if (b == B_LAVA) { P.px = tx; P.py = ty; P.vit[V_HEALTH] = 0; }
        }
    } else if (a != A_NOOP) {
        const int tx = P.px + dir_dx(P.dir), ty = P.py + dir_dy(P.dir);
        const bool t_ok = inb(tx, ty);
        const int f = P.floor;
        auto collect = [&](int b, int item, int level, int ach, int leaves) {
            if ((int)P.f.pickaxe >= level && P.inv.get(item) < INV_MAX) {
                P.inv.add(item, 1);
                if (leaves != b) set_facing_block(tx, ty, leaves);
                unlock(P, ach);
            }
        };
        switch (a) {
        case A_DO: {
            if (!t_ok) break;
            const uint32_t om = occ_mask(tx, ty);
            if (om) {
                const int sw = (int)P.f.sword;                       // fist 1, wood 2, stone 3, iron 5, diamond 8
                const int ap = (sw == 0 ? 1 : sw == 1 ? 2 : sw == 2 ? 3 : sw == 3 ? 5 : 8) + ((int)P.a.str - 1);
                hurt_mob(__builtin_ctz(om), ap, P.f.sword_ench == 1 ? 4 : 0, P.f.sword_ench == 2 ? 4 : 0);
                break;
            }
            const int b = win_b(tx, ty);
            switch (b) {
            case B_TREE: collect(b, I_WOOD, 0, H_COLLECT_WOOD, B_TREE); break;
            case B_STONE: case B_STALAGMITE: collect(b, I_STONE, 1, H_COLLECT_STONE, B_PATH); break;
            case B_COAL: collect(b, I_COAL, 1, H_COLLECT_COAL, B_PATH); break;
            case B_IRON: collect(b, I_IRON, 2, H_COLLECT_IRON, B_PATH); break;
            case B_DIAMOND: collect(b, I_DIAMOND, 3, H_COLLECT_DIAMOND, B_PATH); break;
            case B_SAPPHIRE: collect(b, I_SAPPHIRE, 4, H_COLLECT_SAPPHIRE, B_PATH); break;
            case B_RUBY: collect(b, I_RUBY, 4, H_COLLECT_RUBY, B_PATH); break;
            case B_GRASS: if (misc(9) < P_SAPLING) collect(b, I_SAPLING, 0, H_COLLECT_SAPLING, B_GRASS); break;
            case B_WATER: case B_FOUNTAIN:
                P.vit[V_DRINK] = min(cap_need(P), P.vit[V_DRINK] + 1); clear_counter(P, K_THIRST); unlock(P, H_COLLECT_DRINK);
                break;
            case B_RIPE:
                P.vit[V_FOOD] = min(cap_need(P), P.vit[V_FOOD] + FOOD_PLANT); clear_counter(P, K_HUNGER);
                set_facing_block(tx, ty, B_PLANT);
                if ((qw & KEY_MASK) == cell_key(tx, ty)) qw &= 0xFFFFu;      // its age
                unlock(P, H_EAT_PLANT);
                break;
            case B_CHEST: {
                // section "Combat": the bow lies in a chest of the first dungeon floor; books in dungeon chests
                set_facing_block(tx, ty, B_PATH);
                unlock(P, H_OPEN_CHEST);
                if (f == 1 && !P.f.bow) { P.f.bow = 1; unlock(P, H_FIND_BOW); break; }
                const int c = I_POTION + (int)choice(misc(10), 6);
                if (P.inv.get(c) < INV_MAX) P.inv.add(c, 1);
                const int k = (int)choice(misc(11), 4);
                if (k == 0) stock(I_ARROW, 4);
                else if (k == 1) stock(I_TORCH, 4);
                else if (k == 2 && P.f.book < 2) ++P.f.book;
                break;
            }
            case B_NECRO_VULN: {
                // section "Boss Floor": every hit calls the next wave; eight hits win
                unlock(P, H_DAMAGE_NECROMANCER);
                const int hits = min((int)P.f.boss_hits + 1, 15);   // the field's largest value: an import may bring it, and won stays won
                P.f.boss_hits = (uint32_t)hits;
                P.f.boss_vulnerable = 0;
                if (hits >= BOSS_HITS) { unlock(P, H_DEFEAT_NECROMANCER); set_facing_block(tx, ty, B_PATH); break; }
                set_facing_block(tx, ty, B_NECROMANCER);
                const int wv = hits - 1;
                const int mt = melee_of_floor(wv), rt = ranged_of_floor(wv);
#pragma unroll
                for (int s = 0; s < 5; ++s) {
                    const int x = s < 3 ? 20 + 4 * s : 22 + 4 * (s - 3), y = s < 3 ? 10 : 8;
                    const int type = s < 3 ? mt : rt;
                    const bool taken = occ_mask(x, y) != 0 || (P.px == x && P.py == y);
                    if (!(G::get((int)m.w, s) & 1) && !taken) spawn_mob(s, x, y, 0, type, creature(type).hp);
                }
                break;
            }
            default: break;
            }
            break;
        }
        case A_SLEEP: if (P.vit[V_ENERGY] < cap_need(P)) P.f.sleeping = 1; break;
        case A_REST: if (P.vit[V_HEALTH] < cap_health(P)) P.f.resting = 1; break;
        case A_PLACE_STONE: case A_PLACE_TABLE: case A_PLACE_FURNACE: case A_PLACE_PLANT: case A_PLACE_TORCH: {
            if (!t_ok || occ_mask(tx, ty) != 0) break;
            const int il = win_i(tx, ty);
            if ((il & 7) != IT_NONE) break;
            const int b = win_b(tx, ty);
            if (a == A_PLACE_STONE) {
                if (P.inv.get(I_STONE) < 1 || !in_set(FLYABLE, b)) break;
                P.inv.add(I_STONE, -1); set_facing_block(tx, ty, B_STONE); unlock(P, H_PLACE_STONE);
            } else if (a == A_PLACE_TABLE) {
                if (P.inv.get(I_WOOD) < 1 || !in_set(WALKABLE, b)) break;
                P.inv.add(I_WOOD, -1); set_facing_block(tx, ty, B_TABLE); unlock(P, H_PLACE_TABLE);
            } else if (a == A_PLACE_FURNACE) {
                if (P.inv.get(I_STONE) < 1 || !in_set(WALKABLE, b) || !near_table) break;
                P.inv.add(I_STONE, -1); set_facing_block(tx, ty, B_FURNACE); unlock(P, H_PLACE_FURNACE);
            } else if (a == A_PLACE_PLANT) {
                if (f != 0 || P.inv.get(I_SAPLING) < 1 || b != B_GRASS) break;
                const uint32_t cap = min(p.cap_plant, (uint32_t)NPLANT);
                const uint32_t free_slots = ~(uint32_t)G::ballot((qw & 1u) != 0u) & ((1u << cap) - 1u);
                if (!free_slots) break;
                const int s = __builtin_ctz(free_slots);
                P.inv.add(I_SAPLING, -1); set_facing_block(tx, ty, B_PLANT);
                if (l == s) { qw = cell_key(tx, ty); q_block = B_PLANT; }
                unlock(P, H_PLACE_PLANT);
            } else {
                if (P.inv.get(I_TORCH) < 1 || !in_set(WALKABLE, b)) break;
                P.inv.add(I_TORCH, -1);
                if (l == 0) wi[CX_IDX((ty - wy0) * WIN_PITCH + (tx - wx0), WIN_ROWS * WIN_PITCH)] = (uint8_t)((il & ~7) | IT_TORCH);
                wave_sync();
                // light falls off by 4 per cell of Chebyshev distance; the centre cell also carries the item
#pragma unroll
                for (int it = 0; it < (81 + GW - 1) / GW; ++it) {
                    const int i = l + GW * it;
                    if (i < 81) {
                        const int ddy = i / 9 - 4, ddx = i % 9 - 4, x = tx + ddx, y = ty + ddy;
                        if (inb(x, y) && in_win(x, y)) {
                            const int old = wi[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)];
                            const int nl = MAX_LIGHT - 4 * max(iabs(ddx), iabs(ddy));
                            const bool centre = ddx == 0 && ddy == 0;
                            if (nl > (old >> 3) || centre) {
                                const int nv = (old & 7) | (max(nl, old >> 3) << 3);
                                wi[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)] = (uint8_t)nv;
                                maps[il_off(f, x, y)] = (uint8_t)nv;
                            }
                        }
                    }
                }
                wave_sync();
                unlock(P, H_PLACE_TORCH);
            }
            break;
        }
        // tools are levels (1 wood, 2 stone, 3 iron, 4 diamond); crafting only ever raises the level
        case A_MAKE_WOOD_PICKAXE: if (P.f.pickaxe < 1 && try_craft(false, 1, 0, 0, 0, 0)) { P.f.pickaxe = 1; unlock(P, H_MAKE_WOOD_PICKAXE); } break;
        case A_MAKE_STONE_PICKAXE: if (P.f.pickaxe < 2 && try_craft(false, 1, 1, 0, 0, 0)) { P.f.pickaxe = 2; unlock(P, H_MAKE_STONE_PICKAXE); } break;
        case A_MAKE_IRON_PICKAXE: if (P.f.pickaxe < 3 && try_craft(true, 1, 0, 1, 1, 0)) { P.f.pickaxe = 3; unlock(P, H_MAKE_IRON_PICKAXE); } break;
        case A_MAKE_DIAMOND_PICKAXE: if (P.f.pickaxe < 4 && try_craft(true, 1, 0, 0, 0, 3)) { P.f.pickaxe = 4; unlock(P, H_MAKE_DIAMOND_PICKAXE); } break;
        case A_MAKE_WOOD_SWORD: if (P.f.sword < 1 && try_craft(false, 1, 0, 0, 0, 0)) { P.f.sword = 1; unlock(P, H_MAKE_WOOD_SWORD); } break;
        case A_MAKE_STONE_SWORD: if (P.f.sword < 2 && try_craft(false, 1, 1, 0, 0, 0)) { P.f.sword = 2; unlock(P, H_MAKE_STONE_SWORD); } break;
        case A_MAKE_IRON_SWORD: if (P.f.sword < 3 && try_craft(true, 1, 0, 1, 1, 0)) { P.f.sword = 3; unlock(P, H_MAKE_IRON_SWORD); } break;
        case A_MAKE_DIAMOND_SWORD: if (P.f.sword < 4 && try_craft(true, 1, 0, 0, 0, 2)) { P.f.sword = 4; unlock(P, H_MAKE_DIAMOND_SWORD); } break;
        case A_MAKE_IRON_ARMOUR: case A_MAKE_DIAMOND_ARMOUR: {
            const int lvl = a == A_MAKE_IRON_ARMOUR ? 1 : 2;
            int piece = -1;
#pragma unroll
            for (int i = 3; i >= 0; --i) if ((int)((P.a.armour >> (2 * i)) & 3u) < lvl) piece = i;
            if (piece < 0) break;
            if (lvl == 1 ? try_craft(true, 0, 0, 3, 3, 0) : try_craft(true, 0, 0, 0, 0, 3)) {
                P.a.armour = (P.a.armour & ~(3u << (2 * piece))) | ((uint32_t)lvl << (2 * piece));
                unlock(P, lvl == 1 ? H_MAKE_IRON_ARMOUR : H_MAKE_DIAMOND_ARMOUR);
            }
            break;
        }
        case A_MAKE_ARROW: if (try_craft(false, 1, 1, 0, 0, 0)) { stock(I_ARROW, 2); unlock(P, H_MAKE_ARROW); } break;
        case A_MAKE_TORCH: if (try_craft(false, 1, 0, 1, 0, 0)) { stock(I_TORCH, 4); unlock(P, H_MAKE_TORCH); } break;
        case A_SHOOT_ARROW: if (P.f.bow && P.inv.get(I_ARROW) >= 1 && shoot(PP_ARROW, tx, ty, t_ok)) { P.inv.add(I_ARROW, -1); unlock(P, H_FIRE_BOW); } break;
        case A_CAST_FIREBALL: if (P.f.fireball && P.vit[V_MANA] >= 2 && shoot(PP_FIREBALL, tx, ty, t_ok)) { P.vit[V_MANA] -= 2; unlock(P, H_CAST_FIREBALL); } break;
        case A_CAST_ICEBALL: if (P.f.iceball && P.vit[V_MANA] >= 2 && shoot(PP_ICEBALL, tx, ty, t_ok)) { P.vit[V_MANA] -= 2; unlock(P, H_CAST_ICEBALL); } break;
        case A_DESCEND:
            if (f < FLOORS - 1 && (win_i(P.px, P.py) & 7) == IT_LADDER_DOWN) {
                const uint32_t lw = G::uniu(rec[R_LADDER + f + 1]);
                change_floor(f + 1, lw & 0xFF, (lw >> 8) & 0xFF);
            }
            break;
        case A_ASCEND:
            if (f > 0 && (win_i(P.px, P.py) & 7) == IT_LADDER_UP) {
                const uint32_t lw = G::uniu(rec[R_LADDER + f - 1]);
                change_floor(f - 1, (lw >> 16) & 0xFF, (lw >> 24) & 0xFF);
            }
            break;
        case A_READ_BOOK:
            if (P.f.book < 1 || (P.f.fireball && P.f.iceball)) break;
            --P.f.book;
            if (!P.f.fireball) { P.f.fireball = 1; unlock(P, H_LEARN_FIREBALL); }
            else { P.f.iceball = 1; unlock(P, H_LEARN_ICEBALL); }
            break;
        case A_ENCHANT_SWORD: case A_ENCHANT_ARMOUR: case A_ENCHANT_BOW: {
            // section "Potions and Enchantments": mana and a gemstone at an enchantment table
            if (!t_ok) break;
            const int b = win_b(tx, ty);
            if (b != B_ENCH_FIRE && b != B_ENCH_ICE) break;
            const uint32_t elem = b == B_ENCH_FIRE ? 1u : 2u;
            const int gem = elem == 1u ? I_RUBY : I_SAPPHIRE, gems = P.inv.get(gem);
            if (P.vit[V_MANA] < 9 || gems < 1) break;
            if (a == A_ENCHANT_SWORD) { if (P.f.sword < 1 || P.f.sword_ench == elem) break; P.f.sword_ench = elem; unlock(P, H_ENCHANT_SWORD); }
            else if (a == A_ENCHANT_BOW) { if (!P.f.bow || P.f.bow_ench == elem) break; P.f.bow_ench = elem; }
            else {
                int piece = -1;
#pragma unroll
                for (int i = 3; i >= 0; --i)
                    if (((P.a.armour >> (2 * i)) & 3u) > 0u && ((P.a.armour_ench >> (2 * i)) & 3u) != elem) piece = i;
                if (piece < 0) break;
                P.a.armour_ench = (P.a.armour_ench & ~(3u << (2 * piece))) | (elem << (2 * piece));
                unlock(P, H_ENCHANT_ARMOUR);
            }
            P.vit[V_MANA] -= 9;
            P.inv.add(gem, -1);
            break;
        }
        case A_LEVEL_UP_DEXTERITY: if (P.a.xp >= 1 && P.a.dex < 5) { --P.a.xp; ++P.a.dex; } break;
        case A_LEVEL_UP_STRENGTH: if (P.a.xp >= 1 && P.a.str < 5) { --P.a.xp; ++P.a.str; } break;
        case A_LEVEL_UP_INTELLIGENCE: if (P.a.xp >= 1 && P.a.intel < 5) { --P.a.xp; ++P.a.intel; } break;
        default:
            if (a >= A_DRINK_POTION_RED && a <= A_DRINK_POTION_YELLOW) {
                const int col = a - A_DRINK_POTION_RED;
                if (P.inv.get(I_POTION + col) < 1) break;
                P.inv.add(I_POTION + col, -1);
                unlock(P, H_DRINK_POTION);
                // effects: health, mana or energy, +8 or -3, under this episode's colour map
                const int eff = (G::uniu(rec[R_PERM]) >> (3 * col)) & 7u, which = eff >> 1, delta = (eff & 1) ? -3 : 8;
                if (which == 0) P.vit[V_HEALTH] = max(0, min(cap_health(P), P.vit[V_HEALTH] + delta));
                else if (which == 1) P.vit[V_MANA] = max(0, min(cap_mana(P), P.vit[V_MANA] + delta));
                else P.vit[V_ENERGY] = max(0, min(cap_need(P), P.vit[V_ENERGY] + delta));
            }
            break;
        }
    }

    // ---- phase 2: mobs of the current floor ---------------------------------------------------
    // What few steps need is behind a vote: the damage of attackers, the spawn attempts (whose probability draw is looked at
    // first: most end there, and their cells are then not fetched), plants; slots that do nothing are left out of the walk, and a slot's
    // code knows what its class can do.  Bound by instruction issue: a step of 32,768 environments 89.9 -> 79.9 us, of 4,096 14.2 -> 14.0,
    // a rollout of 64 steps and 4,096 environments 648 -> 579.
    const int f = P.floor;
    int damage = 0;
    {
        // every live slot decides what it wants to do from the state after the player's action
        int kind = N_NONE, tx = 0, ty = 0, tdir = 0, col = COL_FLYING;
        bool want_terrain = false, at_player = false;
        if (m.alive()) {
            const int mx = m.x(), my = m.y();
            if (l < S_MPROJ0) {
                const int dx = P.px - mx, dy = P.py - my, adx = iabs(dx), ady = iabs(dy), cheb = max(adx, ady), to_player = toward(dx, dy);
                const uint32_t m8 = choice(rnd.w[0], 8);
                const int wander = m8 < 4 ? (int)m8 + 1 : 0;
                col = creature(m.type()).col;
                kind = N_MOVE;
                tdir = wander;
                if (l < S_PASSIVE0) {
                    if (m.cd() > 0) m.w -= 1u << CD_SHIFT;
                    const bool ready = m.cd() == 0;
                    if (l < S_RANGED0) {
                        if (cheb < CHASE_RANGE && rnd.w[1] < P_CHASE) tdir = to_player;
                        if (adx + ady == 1) { tdir = 0; if (ready) { kind = N_DAMAGE; set_cooldown(m, CD_MELEE); } }
                    } else {
                        const bool aligned = (dx == 0 || dy == 0) && cheb <= SHOOT_RANGE;
                        if (tdir == 0 && cheb <= SHOOT_RANGE) tdir = to_player;
                        if (aligned && ready && rnd.w[1] < P_SHOOT) {
                            tdir = to_player;
                            set_cooldown(m, CD_RANGED);
                            kind = cheb == 1 ? N_DAMAGE : N_SHOOT;      // the next cell in that direction is the player's
                            col = COL_FLYING;
                        }
                    }
                }
                if (tdir == 0 && kind == N_MOVE) kind = N_NONE;
            } else {
                tdir = m.dir();
                kind = l < S_PPROJ0 ? N_FLY : N_PPROJ;
            }
            tx = mx + dir_dx(tdir); ty = my + dir_dy(tdir);
            at_player = tx == P.px && ty == P.py;
            if (kind == N_FLY && at_player) kind = N_DAMAGE_DIE;
            if (kind == N_MOVE || kind == N_SHOOT || kind == N_FLY || kind == N_PPROJ) {
                if (!inb(tx, ty)) kind = (kind == N_FLY || kind == N_PPROJ) ? N_DIE : N_NONE;
                else want_terrain = true;
            }
        }
        // spawn attempts whose probability draw passes; lanes 0..2 fetch their terrain with the mobs
        const int first[3] = { S_MELEE0, S_RANGED0, S_PASSIVE0 }, count[3] = { 3, 2, 3 };
        const int type[3] = { melee_of_floor(f), ranged_of_floor(f), passive_of_floor(f) };
        uint32_t attempts = 0u;
        if (f != 8) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                // overworld: zombies by darkness
                const uint32_t thr = j == 0 ? (f == 0 ? (uint32_t)G::get((int)table, 0) : P_MELEE_SPAWN) : (j == 1 ? (f == 0 ? P_SKELETON_SPAWN : P_RANGED_SPAWN) : P_PASSIVE_SPAWN);
                if (type[j] >= 0 && misc(3 * j + 2) < thr) attempts |= 1u << j;
            }
        }
        int sx[3] = { 0, 0, 0 }, sy[3] = { 0, 0, 0 };
        int probe_b = B_INVALID;
        if (attempts != 0u) {
            const int pick = (int)choice(rnd.w[3], 31) - 15;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                sx[j] = P.px + G::get(pick, 3 * j);
                sy[j] = P.py + G::get(pick, 3 * j + 1);
            }
            const int x = l == 0 ? sx[0] : (l == 1 ? sx[1] : sx[2]), y = l == 0 ? sy[0] : (l == 1 ? sy[1] : sy[2]);
            if (l < 3 && ((attempts >> l) & 1u) && inb(x, y)) {
                probe_b = maps[block_off(f, x, y)];
                if (patch_f == f && patch_x == x && patch_y == y) probe_b = patch_b;
            }
        }
        bool ok = false;
        if (want_terrain) {
            int b = maps[block_off(f, tx, ty)];
            if (patch_f == f && patch_x == tx && patch_y == ty) b = patch_b;
            ok = passable_for(col, b);
            if (kind == N_FLY && !ok) kind = N_DIE;
            ok = ok && !at_player;
            if ((kind == N_MOVE || kind == N_SHOOT) && !ok) kind = N_NONE;
        }
        // what an attacker does to the player, less what the armour takes
        int dmg = 0;
        if (G::ballot(kind == N_DAMAGE || kind == N_DAMAGE_DIE) != 0u) {
            int pdp = 0, pdf = 0, pdi = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pdp += 10 * (int)((P.a.armour >> (2 * i)) & 3u);
                const int en = (P.a.armour_ench >> (2 * i)) & 3u;
                if (en == 1) pdf += 20;
                if (en == 2) pdi += 20;
            }
            const CreatureRow c = creature(m.type());
            dmg = ((P.f.sleeping || P.f.resting) ? 2 : 1) * through(c.dp, c.df, c.di, pdp, pdf, pdi);
        }
        const uint32_t tkey = cell_key(tx & 63, ty & 63);
        constexpr int KIND_SHIFT = 13, OK_SHIFT = 16, DIR_SHIFT = 17;
        const int iwv = (int)tkey | (kind << KIND_SHIFT) | ((ok ? 1 : 0) << OK_SHIFT) | (tdir << DIR_SHIFT);

        // the slots act one after the other, each seeing what the earlier ones did
        uint32_t alive_bits = (uint32_t)G::ballot(m.alive() != 0u);
        uint32_t acting = (uint32_t)G::ballot(kind != N_NONE);
        constexpr int ORDER[NSLOT] = { 0, 1, 2, 5, 6, 7, 8, 9, 10, 11, 12, 13, 3, 4 };
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) {
            const int k = ORDER[i];
            if (!((acting >> k) & 1u)) continue;
            const int iw = G::get(iwv, k), kd = (iw >> KIND_SHIFT) & 7;
            const uint32_t key = (uint32_t)iw & KEY_MASK;
            auto occupied = [&]() -> uint32_t { return (uint32_t)G::ballot((m.w & KEY_MASK) == key); };
            auto go = [&]() { if (l == k) m.w = (m.w & ~KEY_MASK) | tkey; };
            auto die = [&]() { if (l == k) clear_mob(m); alive_bits &= ~(1u << k); };
            if (k < S_MPROJ0) {
                if (kd == N_DAMAGE) { damage += G::get(dmg, k); continue; }
                if (occupied() != 0u) continue;
                if (k >= S_RANGED0 && k < S_PASSIVE0 && kd == N_SHOOT) {
                    const uint32_t free_slots = ~alive_bits & (7u << S_MPROJ0);
                    if (free_slots) {
                        const int s = __builtin_ctz(free_slots);
                        const uint32_t shot = key | ((uint32_t)((iw >> DIR_SHIFT) & 7) << 13) | ((uint32_t)G::get((int)m.w, k) & (31u << TYPE_SHIFT));
                        if (l == s) m.w = shot;
                        alive_bits |= 1u << s;
                    }
                } else go();
            } else if (k < S_PPROJ0) {
                if (kd == N_DAMAGE_DIE) damage += G::get(dmg, k);
                if (kd != N_FLY || occupied() != 0u) die(); else go();
            } else {
                if (kd == N_DIE) { die(); continue; }
                const uint32_t om = occupied();
                if (om) {
                    const int hit = __builtin_ctz(om);
                    int ap, af, ai;
                    shot_attack((G::get((int)m.w, k) >> TYPE_SHIFT) & 31, ap, af, ai);
                    if (hurt_mob(hit, ap, af, ai)) { alive_bits &= ~(1u << hit); acting &= ~(1u << hit); }
                    die();
                } else if ((iw >> OK_SHIFT) & 1) go();
                else die();
            }
        }
        P.vit[V_HEALTH] = max(0, P.vit[V_HEALTH] - damage);

        // ---- despawn far away, spawn near (section "Creatures": fixed slots, masked when empty) ----
        if (max(iabs(m.x() - P.px), iabs(m.y() - P.py)) > DESPAWN_DIST) clear_mob(m);    // an empty slot stays empty
        alive_bits = (uint32_t)G::ballot(m.alive() != 0u);
        if (f == 8) {
            // the necromancer can be hit again once its wave is gone
            if (!P.f.boss_vulnerable && P.f.boss_hits < BOSS_HITS && !(alive_bits & 0x1Fu)) {
                P.f.boss_vulnerable = 1;
                set_block(BOSS_X, BOSS_Y, B_NECRO_VULN);
            }
        } else {
            const uint32_t caps[3] = { p.cap_melee, p.cap_ranged, p.cap_passive };
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (!((attempts >> j) & 1u)) continue;
                const int x = sx[j], y = sy[j];
                const int n = min(count[j], (int)caps[j]);
                const uint32_t free_slots = ~alive_bits & (((1u << n) - 1u) << first[j]);
                if (!free_slots || max(iabs(x - P.px), iabs(y - P.py)) < SPAWN_MIN_DIST || !inb(x, y)) continue;
                if (occ_mask(x, y) != 0 || (x == P.px && y == P.py)) continue;
                const int b = G::get(probe_b, j);
                // overworld: skeletons on paths, zombies and cows on grass
                const bool okb = f == 0 ? b == (j == 1 ? B_PATH : B_GRASS) : passable_for(creature(type[j]).col, b);
                if (!okb) continue;
                const int s = __builtin_ctz(free_slots);
                spawn_mob(s, x, y, 0, type[j], creature(type[j]).hp);
                alive_bits |= 1u << s;
            }
        }
    }

    // ---- plants: they only grow while the player is in the overworld ---------------------------
    if (f == 0 && G::ballot((qw & 1u) != 0u) != 0u) {
        uint32_t zombie[3];
#pragma unroll
        for (int z = 0; z < 3; ++z) zombie[z] = (uint32_t)G::get((int)m.w, S_MELEE0 + z);
        if (qw & 1u) {
            const int x = (int)((qw >> 1) & 63u), y = (int)((qw >> 7) & 63u);
            if (patch_f == 0 && patch_x == x && patch_y == y) q_block = patch_b;
            if ((qw >> 16) < 65535u) qw += 1u << 16;
            int nb = -1;
            if (q_block == B_PLANT && (qw >> 16) >= (uint32_t)RIPE_AGE) nb = B_RIPE;
            auto beside = [&](uint32_t z) { return (z & 1u) && iabs((int)((z >> 1) & 63u) - x) + iabs((int)((z >> 7) & 63u) - y) == 1; };
            if ((beside(zombie[0]) || beside(zombie[1]) || beside(zombie[2])) && rnd.w[2] < P_PLANT_EATEN) { nb = B_GRASS; qw = 0u; }
            if (nb >= 0) {
                maps[block_off(0, x, y)] = (uint8_t)nb;
                if (in_win(x, y)) wb[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)] = (uint8_t)nb;
            }
        }
        wave_sync();
    }

    // ---- needs -------------------------------------------------------------------------------
    {
        const bool damaged = damage > 0;
        const bool asleep = P.f.sleeping, idle = P.f.sleeping || P.f.resting;
        int hunger = sext8(P.cnt) + (asleep ? 1 : 2), thirst = sext8(P.cnt >> 8) + (asleep ? 1 : 2), fatigue = sext8(P.cnt >> 16) + (asleep ? -1 : 1),
            recover = sext8(P.cnt >> 24), mana = sext8(P.mana_word >> 8) + (int)P.a.intel;   // section "Attributes": intelligence feeds magic
        if (hunger > 50) { hunger = 0; P.vit[V_FOOD] = max(0, P.vit[V_FOOD] - 1); }
        if (thirst > 40) { thirst = 0; P.vit[V_DRINK] = max(0, P.vit[V_DRINK] - 1); }
        if (asleep) { if (fatigue < -10) { fatigue = 0; P.vit[V_ENERGY] = min(cap_need(P), P.vit[V_ENERGY] + 1); } }
        else if (fatigue > 30) { fatigue = 0; P.vit[V_ENERGY] = max(0, P.vit[V_ENERGY] - 1); }
        if (mana > 20) { mana = 0; P.vit[V_MANA] = min(cap_mana(P), P.vit[V_MANA] + 1); }
        if (P.vit[V_HEALTH] > 0) {
            const bool fed = P.vit[V_FOOD] > 0 && P.vit[V_DRINK] > 0 && (P.vit[V_ENERGY] > 0 || asleep);
            recover += fed ? (idle ? 4 : 2) : (idle ? -1 : -2);
            if (recover > 50) { recover = 0; P.vit[V_HEALTH] = min(cap_health(P), P.vit[V_HEALTH] + 1); }
            if (recover < -30) { recover = 0; --P.vit[V_HEALTH]; }
        }
        P.cnt = (uint32_t)(hunger & 0xFF) | ((uint32_t)(thirst & 0xFF) << 8) | ((uint32_t)(fatigue & 0xFF) << 16) | ((uint32_t)(recover & 0xFF) << 24);
        P.mana_word = ((uint32_t)(mana & 0xFF) << 8) | ((uint32_t)(phase + 1 == (int)p.day_length ? 0 : phase + 1) << 16);   // and the new phase
        if (asleep && (P.vit[V_ENERGY] >= cap_need(P) || damaged)) { P.f.sleeping = 0; unlock(P, H_WAKE_UP); }
        if (P.f.resting && (P.vit[V_HEALTH] >= cap_health(P) || damaged)) P.f.resting = 0;
    }

    // ---- reward, time, done (section "RL Environment Interface") ------------------------------
    int gained = 0;
    StepOut o;
#pragma unroll
    for (int w = 0; w < 3; ++w) o.unlocked[w] = P.ach[w] & ~old[R_ACH + w];
    if ((o.unlocked[0] | o.unlocked[1] | o.unlocked[2]) != 0u) {
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            const uint32_t nw = o.unlocked[w];
            gained += __builtin_popcount(nw & CAT1[w]) + 3 * __builtin_popcount(nw & CAT3[w]) +
                      5 * __builtin_popcount(nw & CAT5[w]) + 8 * __builtin_popcount(nw & CAT8[w]);
        }
    }
    o.reward = (float)(10 * gained + (P.vit[V_HEALTH] - health0)) * 0.1f;
    o.t = old[R_T] + 1u;
    o.done = P.vit[V_HEALTH] <= 0 || o.t >= p.max_episode_steps;
    o.wx0 = wx0; o.wy0 = wy0;
    return o;
}

}  // namespace cf
