// Symbolic observation of full Craftax (appendix "Observation Space"): 9 x 11 cells around the
// player, per cell one-hot block (37) + item (5) + creature (40: five slot classes of eight
// types) + light; cells darker than 0.05 are blank; then the 51 scalars of the inventory table.
// The wave stages the bytes in LDS and streams them out as whole cache lines (byte layout) or floats
// (flat layout).
#pragma once

#include "full_common.hpp"

namespace cf {

constexpr int VEC_DAY = 43;      // the scalar that is the daylight
// Where scalar i of the observation comes from: record word, shift, mask, and how the raw
// integer becomes a float.  Direction, daylight and "floor cleared" are handled apart.
enum Conv : int { CV_SQRT10 = 0, CV_TENTH, CV_HALF, CV_QUARTER, CV_RAW, CV_SPECIAL };
struct ScalarSpec { uint8_t word, shift, mask, conv; };
constexpr ScalarSpec SCALAR_ROWS[NVEC] = {
    { R_INV, 0, 255, CV_SQRT10 }, { R_INV, 8, 255, CV_SQRT10 }, { R_INV, 16, 255, CV_SQRT10 }, { R_INV, 24, 255, CV_SQRT10 },
    { R_INV + 1, 0, 255, CV_SQRT10 }, { R_INV + 1, 8, 255, CV_SQRT10 }, { R_INV + 1, 16, 255, CV_SQRT10 }, { R_INV + 1, 24, 255, CV_SQRT10 },
    { R_INV + 2, 0, 255, CV_SQRT10 }, { R_INV + 2, 8, 255, CV_SQRT10 },
    { R_INV + 2, 16, 255, CV_SQRT10 }, { R_INV + 2, 24, 255, CV_SQRT10 },                                  // potions 0, 1
    { R_POT, 0, 255, CV_SQRT10 }, { R_POT, 8, 255, CV_SQRT10 }, { R_POT, 16, 255, CV_SQRT10 }, { R_POT, 24, 255, CV_SQRT10 },
    { R_FLAGS, 4, 3, CV_HALF },        // book n/2
    { R_FLAGS, 6, 7, CV_QUARTER },     // pickaxe level/4
    { R_FLAGS, 9, 7, CV_QUARTER },     // sword level/4
    { R_FLAGS, 12, 3, CV_RAW },        // sword enchantment: fire 1, ice 2
    { R_FLAGS, 14, 1, CV_RAW },        // bow
    { R_FLAGS, 15, 3, CV_RAW },        // bow enchantment
    { R_ATTR, 0, 3, CV_HALF }, { R_ATTR, 2, 3, CV_HALF }, { R_ATTR, 4, 3, CV_HALF }, { R_ATTR, 6, 3, CV_HALF },       // armour level/2
    { R_ATTR, 8, 3, CV_RAW }, { R_ATTR, 10, 3, CV_RAW }, { R_ATTR, 12, 3, CV_RAW }, { R_ATTR, 14, 3, CV_RAW },        // armour enchantments
    { R_VIT, 0, 255, CV_TENTH }, { R_VIT, 8, 255, CV_TENTH }, { R_VIT, 16, 255, CV_TENTH }, { R_VIT, 24, 255, CV_TENTH },
    { R_MANA, 0, 255, CV_TENTH },
    { R_ATTR, 16, 15, CV_TENTH },      // experience
    { R_ATTR, 20, 7, CV_TENTH }, { R_ATTR, 23, 7, CV_TENTH }, { R_ATTR, 26, 7, CV_TENTH },                           // dexterity strength intelligence
    { R_POS, 16, 255, CV_SPECIAL }, { R_POS, 16, 255, CV_SPECIAL }, { R_POS, 16, 255, CV_SPECIAL }, { R_POS, 16, 255, CV_SPECIAL },   // facing one-hot
    { R_MANA, 16, 255, CV_SPECIAL },   // daylight
    { R_FLAGS, 0, 1, CV_RAW },         // sleeping
    { R_FLAGS, 1, 1, CV_RAW },         // resting
    { R_FLAGS, 2, 1, CV_RAW },         // learned fireball
    { R_FLAGS, 3, 1, CV_RAW },         // learned iceball
    { R_POS, 24, 15, CV_TENTH },       // floor / 10
    { R_POS, 24, 15, CV_SPECIAL },     // floor cleared
    { R_FLAGS, 17, 1, CV_RAW },        // boss vulnerable
};

// The same as the renderer of a step reads it, in one dword: the field (record word, shift, width) and where its value's float lies in
// the tables in LDS (LUT_FLOATS below), which go up to `limit` there: a lookup without branches.
constexpr int LUT_SQRT10 = 0, LUT_TENTH = 100, LUT_LIGHT20 = 132, LUT_HALF = 164, LUT_QUARTER = 168, LUT_RAW = 176, LUT_FLOATS = 180, LUT_COPIED = 164;
struct ScalarTables { ScalarSpec rows[NVEC]; uint32_t fields[NVEC]; };
constexpr ScalarTables scalar_tables()
{
    ScalarTables t{};
    for (int i = 0; i < NVEC; ++i) {
        const ScalarSpec s = SCALAR_ROWS[i];
        uint32_t width = 0;
        while ((s.mask >> width) != 0) ++width;
        const uint32_t at = s.conv == CV_SQRT10 ? LUT_SQRT10 : s.conv == CV_TENTH ? LUT_TENTH : s.conv == CV_HALF ? LUT_HALF : s.conv == CV_QUARTER ? LUT_QUARTER : LUT_RAW;
        const uint32_t limit = s.conv == CV_SQRT10 ? 99 : s.conv == CV_TENTH ? 31 : s.conv == CV_QUARTER ? 7 : 3;
        t.rows[i] = s;
        t.fields[i] = (uint32_t)s.word | ((uint32_t)s.shift << 6) | (width << 11) | (at << 16) | (limit << 24);
    }
    return t;
}
__device__ __constant__ const ScalarTables SCALARS = scalar_tables();

// scalar `i` of the observation from the packed record in LDS
__device__ __forceinline__ float scalar_value(int i, const uint32_t* rec, const Luts* __restrict__ luts)
{
    const ScalarSpec s = SCALARS.rows[i];
    const uint32_t raw = (rec[s.word] >> s.shift) & s.mask;
    if (s.conv == CV_SQRT10) return luts->sqrt10[min(raw, 99u)];
    if (s.conv == CV_TENTH) return luts->tenth[min(raw, 31u)];
    if (s.conv == CV_HALF) return (float)raw * 0.5f;
    if (s.conv == CV_QUARTER) return (float)raw * 0.25f;
    if (s.conv == CV_RAW) return (float)raw;
    if (i >= 39 && i < 43) return (int)raw == i - 38 ? 1.0f : 0.0f;
    if (i == VEC_DAY) return luts->daylight[rec[R_MANA] >> 16];
    // floor cleared: the overworld always, deeper floors after enough kills
    const int f = (int)raw;
    const int kills = (int)((rec[R_KILLS + (f >> 2)] >> (8 * (f & 3))) & 0xFFu);
    return (f == 0 || kills >= KILLS_TO_CLEAR) ? 1.0f : 0.0f;
}

// What the step kernels fetch ahead of the renderer, so that it waits for no table in memory: the
// fields of the scalars this lane writes (scalar l, l + GW, ...), the small conversion tables
// in LDS, and the daylight value of the observation's phase.
template <int GW>
struct RenderAux {
    uint32_t field[(NVEC + 1 + GW - 1) / GW];   // of scalar l + GW * it
    const float* lut;                           // LDS: sqrt10[100], tenth[32], light20[32], n / 2, n / 4, n
    float day;                                  // in the lane that writes it: daylight[phase of the rendered state]
};
// What a step looks up by day phase, in one load: lane 0 gets the zombie threshold of the phase, the lane that writes the daylight
// that of the next phase, lane 1 that of a fresh episode.  (Loads to scalar registers, one for each, held up the step: they are waited for
// with the next access to LDS.)
template <int GW>
__device__ __forceinline__ uint32_t day_table(int l, uint32_t phase, uint32_t day_length, const Luts* __restrict__ luts)
{
    static_assert(VEC_DAY % GW > 1 && offsetof(Luts, zombie_thr) == offsetof(Luts, daylight) + 4 * MAX_DAY, "lanes of their own, one table after the other");
    const uint32_t next = phase + 1u == day_length ? 0u : phase + 1u;
    return reinterpret_cast<const uint32_t*>(luts->daylight)[l == 0 ? MAX_DAY + phase : l == VEC_DAY % GW ? next : 0u];
}
// the daylight of the rendered state in the lane that writes it
template <int GW>
__device__ __forceinline__ float day_of(uint32_t table, bool fresh) { return __uint_as_float(fresh ? (uint32_t)Lanes<GW>::get((int)table, 1) : table); }
template <int GW>
__device__ __forceinline__ void fetch_scalar_fields(int l, RenderAux<GW>& aux)
{
#pragma unroll
    for (int it = 0; it < (NVEC + 1 + GW - 1) / GW; ++it) aux.field[it] = SCALARS.fields[min(l + GW * it, NVEC - 1)];
}
// entry i < LUT_FLOATS of the tables in LDS
__device__ __forceinline__ float lut_entry(int i, const Luts* __restrict__ luts)
{
    if (i < LUT_COPIED) return luts->sqrt10[i];          // sqrt10, tenth and light20 lie one after the other
    return i < LUT_QUARTER ? (float)(i - LUT_HALF) * 0.5f : i < LUT_RAW ? (float)(i - LUT_QUARTER) * 0.25f : (float)(i - LUT_RAW);
}
__device__ __forceinline__ float scalar_value_fast(int i, uint32_t field, const uint32_t* rec, const float* lut, float day)
{
    const uint32_t raw = __builtin_amdgcn_ubfe(rec[field & 63u], (field >> 6) & 31u, (field >> 11) & 31u);
    float v = lut[((field >> 16) & 0xFFu) + min(raw, field >> 24)];
    // facing, daylight, floor cleared (the overworld always, deeper floors after enough kills)
    if (i >= 39 && i < 43) v = (int)raw == i - 38 ? 1.0f : 0.0f;
    if (i == VEC_DAY) v = day;
    if (i == 49) v = raw == 0u || ((rec[R_KILLS + ((raw >> 2) & 3u)] >> (8 * (raw & 3u))) & 0xFFu) >= (uint32_t)KILLS_TO_CLEAR ? 1.0f : 0.0f;
    return v;
}

// Observation channel of the creature in slot k (class by slot range, type slot by creature).
__device__ inline int creature_channel(int k, int type)
{
    if (k < S_RANGED0) return 42 + melee_type_slot(type);
    if (k < S_PASSIVE0) return 42 + 16 + ranged_type_slot(type);
    if (k < S_MPROJ0) return 42 + 8 + (type == C_COW ? 0 : (type == C_SNAIL ? 1 : 2));
    if (k < S_PPROJ0) {
        const CreatureRow c = creature(type);
        return 42 + 24 + (c.df > 0 ? (c.di > 0 ? 3 : 1) : (c.di > 0 ? 2 : 0));
    }
    return 42 + 32 + type;
}

// one-hot nibble -> four bytes of 0/1
__device__ inline uint32_t spread4(uint32_t nibble) { return (nibble * 0x00204081u) & 0x01010101u; }

// The observation of one environment by a whole wavefront.  e: its LDS area (staged_dwords<HALVES>) with the
// packed record (current) and the two windows with origin (wx0, wy0) on the current floor; m_*:
// this lane's mob slot.  F32 = false: writes the 8448-byte layout; F32 = true: writes float[8268]
// (+ zero padding to 33152 bytes).
//
// An observation of 8217 cell bytes holds at most 396 that are not zero.  They are set one by one in a
// cleared LDS area, which the lanes then read back in 16-byte pieces and store as whole cache lines.
// LDS moves 128 bytes per clock beside the vector units, which bound the step kernels; in the earlier form
// (the channels as single bits, every piece expanded from 16 of them) a quarter of the vector
// instructions of a step expanded bits.  Measured, before the player's state was kept packed: a step of
// 4,096 environments 18.3 -> 16.7 us, of 32,768 115 -> 110, a rollout of 64 steps and 4,096 environments
// 897 -> 805 us.  The area covers 5,120 bytes at a time, or (HALVES) half of them, with which eight blocks of the step kernel share
// a compute unit (see step_bound); that takes a store more (rollout of 64 steps and 4,096 environments 537 us, 547 by halves).  A lane owns cell l of the first part and cell LAST0 + l of the second; cell LAST0 lies in both, and has its bytes of the
// other part beside the area, where nobody reads them, so that no byte is tested for its part.
// For the float layout a staged byte v stands for v / 140: 140 is the 1 of a one-hot channel and 7 * level
// the light level / 20.  Multiplying by the float nearest to 1/140 gives exactly those floats.
constexpr float F32_UNIT = 1.0f / 140.0f;
constexpr bool staged_floats_are_exact()
{
    for (int lv = 0; lv <= MAX_LIGHT; ++lv) if ((float)(7 * lv) * F32_UNIT != (float)((double)lv / 20.0)) return false;
    return true;
}
static_assert(staged_floats_are_exact(), "light levels through staged bytes");
template <bool HALVES>
struct Parts {
    static constexpr int HEAD = stage_bytes<HALVES>, LAST0 = HEAD / NCHAN, BEFORE1 = HEAD - LAST0 * NCHAN;     // bytes of the first part, the cell on the border, its bytes there
    static_assert(HEAD % 128 == 0 && STRIDE_U8 - HEAD <= HEAD && LAST0 < 64 && NCELL - LAST0 <= 64 && BEFORE1 <= STAGE_BEFORE && NCHAN - BEFORE1 <= stage_behind<HALVES>, "cells of the two parts");
};
// FLOATS: how they are stored (see floats_kept); where that is STREAM, through says whether this observation is written through
// all the same (the same for the wavefront).  Bytes are streamed.
template <bool F32, cx::Keep FLOATS, bool HALVES>
__device__ __forceinline__ void render_staged(const int l, uint32_t* e, const int wx0, const int wy0, const int m_alive, const int m_x,
                                              const int m_y, const int m_type, const Luts* __restrict__ luts, uint8_t* __restrict__ out,
                                              const RenderAux<64>* aux, const bool through)
{
    const uint32_t* rec = e + L_REC;
    const uint8_t* wb = reinterpret_cast<const uint8_t*>(e + L_WB);
    const uint8_t* wi = reinterpret_cast<const uint8_t*>(e + L_WI);
    uint32_t* cre = e + L_CRE;
    uint8_t* stage = reinterpret_cast<uint8_t*>(e + L_STAGE);
    constexpr uint32_t ONE = F32 ? 140u : 1u, LIGHT = F32 ? 7u : 1u;
    constexpr int STAGE_BYTES = Parts<HALVES>::HEAD, LAST0 = Parts<HALVES>::LAST0, BEFORE1 = Parts<HALVES>::BEFORE1;
    static_assert(!F32 || !HALVES, "a turn of floats is 64 pieces");
    const uint32_t pos = uniu(rec[R_POS]);
    const int px = pos & 0xFF, py = (pos >> 8) & 0xFF;
    const int corner = (py - VROWS / 2 - wy0) * WIN_PITCH + px - VCOLS / 2 - wx0;    // upper left cell of the view in the windows
    // beyond the edge of the map the windows hold B_OOB at full light
    uint32_t il[2], block[2];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const int own = part == 0 ? LAST0 + 1 : NCELL - LAST0, cell = (part == 0 ? 0 : LAST0) + min(l, own - 1), r = cell / VCOLS;
        const int at = CX_IDX(corner + r * WIN_PITCH + cell - r * VCOLS, WIN_ROWS * WIN_PITCH);
        il[part] = wi[at];
        block[part] = wb[at] & 63u;
        if (l >= own) il[part] = 0u;
    }
    // the creature of a cell is the one in its lowest slot, and is seen where there is light
    const int vr = m_y - (py - VROWS / 2), vc = m_x - (px - VCOLS / 2), m_cell = vr * VCOLS + vc;
    const bool in_view = l < NSLOT && m_alive && (unsigned)vr < (unsigned)VROWS && (unsigned)vc < (unsigned)VCOLS;
    uint32_t m_byte = 0xFFFFFFFFu;
    if (in_view) cre[CX_IDX(m_cell, NCELL)] = 0xFFFFFFFFu;
    wave_sync();
    if (in_view) atomicMin(&cre[CX_IDX(m_cell, NCELL)], (uint32_t)l);
    wave_sync();
    if (in_view && cre[CX_IDX(m_cell, NCELL)] == (uint32_t)l && (wi[CX_IDX(corner + vr * WIN_PITCH + vc, WIN_ROWS * WIN_PITCH)] >> 3) != 0)
        m_byte = (uint32_t)(m_cell * NCHAN + creature_channel(l, m_type));
    const float scalar = l >= NVEC ? 0.0f : (aux != nullptr ? scalar_value_fast(l, aux->field[0], rec, aux->lut, aux->day) : scalar_value(l, rec, luts));
    wave_sync();
    // part 0: bytes 0 .. STAGE_BYTES - 1; part 1: the rest
    auto fill = [&](int part) {
        const uint32_t start = part == 0 ? 0u : (uint32_t)STAGE_BYTES, size = part == 0 ? (uint32_t)STAGE_BYTES : (uint32_t)(CELL_BYTES - STAGE_BYTES);
        uint4* clear = reinterpret_cast<uint4*>(stage) + l;
#pragma unroll
        for (int k = 0; k < (STAGE_BYTES + 1023) / 1024; ++k)
            if ((part == 0 || k * 1024 < STRIDE_U8 - STAGE_BYTES) && (64 * k + 64 <= STAGE_BYTES / 16 || l < STAGE_BYTES / 16 - 64 * k)) clear[64 * k] = make_uint4(0u, 0u, 0u, 0u);
        wave_sync();
        // before the cells: an imported creature type may fall on a light channel, which holds the light level all the same
        if (m_byte - start < size) stage[CX_IDX(m_byte - start, STAGE_BYTES)] = (uint8_t)ONE;
        wave_sync();
        if ((il[part] >> 3) != 0u) {                // cells darker than 0.05 stay blank
            uint8_t* cell = stage - STAGE_BEFORE;
            const int at = STAGE_BEFORE + l * NCHAN - (part == 0 ? 0 : BEFORE1);
            constexpr int ROOM = STAGE_BEFORE + STAGE_BYTES + stage_behind<HALVES>;
            cell[CX_IDX(at + (int)block[part], ROOM)] = (uint8_t)ONE;
            cell[CX_IDX(at + 37 + (int)(il[part] & 7u), ROOM)] = (uint8_t)ONE;
            cell[CX_IDX(at + 82, ROOM)] = (uint8_t)(LIGHT * (il[part] >> 3));
        }
    };
    using cx::piece_t;
    if constexpr (!F32) {
        piece_t* dst = reinterpret_cast<piece_t*>(out) + l;
        const piece_t* src = reinterpret_cast<const piece_t*>(stage) + l;
        constexpr int PIECES = STRIDE_U8 / 16, HEAD = STAGE_BYTES / 16;
        // 16-byte streaming stores
        auto store = [&](int first, int pieces) {
#pragma unroll
            for (int k = 0; k < (pieces + 63) / 64; ++k)
                if (64 * k + 64 <= pieces || l < pieces - 64 * k) __builtin_nontemporal_store(src[64 * k], dst + first + 64 * k);
        };
        fill(0);
        wave_sync();
        store(0, HEAD);
        wave_sync();
        fill(1);
        if (l < NVEC) reinterpret_cast<float*>(stage + (VEC_OFFSET - STAGE_BYTES))[l] = scalar;
        wave_sync();
        store(HEAD, PIECES - HEAD);
    } else {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(stage) + l;
        auto floats = [&](int k) {
            const uint32_t four = src[64 * k];
            return __builtin_bit_cast(piece_t, make_float4((float)(four & 0xFFu) * F32_UNIT, (float)((four >> 8) & 0xFFu) * F32_UNIT, (float)((four >> 16) & 0xFFu) * F32_UNIT,
                                                           (float)(four >> 24) * F32_UNIT));
        };
        // 16-byte pieces `first`, first + 64, ..., one per lane and turn, in a loop for each kind of store
        auto store = [&](const int first, auto turns, auto&& piece) {
            constexpr int TURNS = decltype(turns)::value;
            piece_t* dst = reinterpret_cast<piece_t*>(out) + first + l;
            if constexpr (FLOATS == cx::Keep::PLAIN) {
#pragma unroll 5
                for (int k = 0; k < TURNS; ++k) dst[64 * k] = piece(k);
            } else if (FLOATS == cx::Keep::THROUGH || through) {
                const uintptr_t at = reinterpret_cast<uintptr_t>(out);
                uint8_t* base = reinterpret_cast<uint8_t*>(((uintptr_t)uniu((uint32_t)(at >> 32)) << 32) | uniu((uint32_t)at));
#pragma unroll 5
                for (int k = 0; k < TURNS; ++k) cx::store_through(base, STRIDE_F32, 16 * (first + 64 * k + l), piece(k));
            } else {
#pragma unroll 5
                for (int k = 0; k < TURNS; ++k) __builtin_nontemporal_store(piece(k), dst + 64 * k);
            }
        };
        // pieces of four floats; from TAIL on they hold scalars (after one last light level)
        constexpr int PIECES = STRIDE_F32 / 16, HEAD = STAGE_BYTES / 4, TAIL = CELL_BYTES / 4, TAIL_AT = 3328;
        static_assert(HEAD % 64 == 0 && TAIL_AT % 16 == 0 && TAIL_AT >= STRIDE_U8 - STAGE_BYTES && TAIL_AT + 16 * (PIECES - TAIL) <= STAGE_BYTES && CELL_BYTES == 4 * TAIL + 1, "tail of the float layout");
        fill(0);
        wave_sync();
        store(0, std::integral_constant<int, HEAD / 64>(), floats);
        wave_sync();
        fill(1);
        float* tail = reinterpret_cast<float*>(stage + TAIL_AT);
        if (l < NVEC) tail[1 + l] = scalar;
        if (l >= NVEC) tail[1 + l] = 0.0f;
        if (l < 4 * (PIECES - TAIL) - 65) tail[65 + l] = 0.0f;
        if (l == NCELL - 1 - LAST0) tail[0] = (float)(LIGHT * (il[1] >> 3)) * F32_UNIT;
        wave_sync();
        constexpr int TURNS = (TAIL - HEAD) / 64, LEFT = (TAIL - HEAD) % 64;
        store(HEAD, std::integral_constant<int, TURNS>(), floats);
        if (l < LEFT) store(HEAD + 64 * TURNS, std::integral_constant<int, 1>(), [&](int) { return floats(TURNS); });
        if (l < PIECES - TAIL) store(TAIL, std::integral_constant<int, 1>(), [&](int) { return reinterpret_cast<const piece_t*>(tail)[l]; });
    }
}

// How the float observations of n environments are stored, by an instance of the kernel for each kind (a choice at run time: 16 environments
// 9.7 -> 9.9 us, craftax_observe of 1,000 7.3 -> 7.8).  Up to CACHE_SHARE they are written through to the last-level cache, up to FLOATS_KEPT, which
// that cache holds with what else lies there, left in the L2; of a larger buffer those of every fourth block are written through, in its first
// SPLIT_TO bytes, and the others streamed.  us, left in the L2 / through / by every fourth block, one state | three in turn | one that a
// maximum over the observation reads | one that a cast to bfloat16 reads:
//   500 12.1 / 10.9 | 12.4 / 11.0 | 28.3 / 27.4 | 44.2 / 44.5     1,000 13.3 / 11.5 | 13.5 / 11.6 | 35.6 / 36.2 | 71.6 / 72.8     2,688 20.4 / 18.6 | 22.3 / 20.9 | 46.1 / 46.9 | 161 / 162
//   3,333 23.8 / 22.8 / 23.9 | 30.6 / 31.2 / 24.1 | 50.8 / 50.8 / 62.2 | 198 / 200 / 266     4,096 26.1 / 24.7 / 26.4 | 35.4 / 35.9 / 27.1 | 56.1 / 57.1 / 71.3 | 254 / 257 / 326
//   6,000 39.6 / 37.5 / 38.9 | 55.6 / 55.8 / 44.1 | 78.8 / 79.3 / 101 | 469 / 471 / 487     7,200 49.6 / 45.0 / 42.6 | 61.1 / 63.5 / 52.2 | 99.6 / 103 / 116 | 580 / 581 / 581
//   7,800 52.9 / 49.5 / 45.3 | 61.1 / 60.7 / 53.6 | 119 / 122 / 123 | 631 / 626 / 619     8,192 59.4 / 57.3 / 47.8 | 68.6 / 68.2 / 60.0 | 141 / 142 / 129 | 666 / 670 / 659
//   10,000 84.4 / 76.9 / 59.8 | 83.7 / 78.7 / 69.5 | 181 / 178 / 157 | 811 / 813 / 801
// craftax_observe in the same order: 4,096 21.3 / 20.6 | 29.2 / 29.2 | 54.3 / 54.5 | 250 / 244     8,192 43.7 / 37.0 / 41.5 | 58.9 / 59.2 / 44.9 | 122 / 123 / 122 | 648 / 654 / 645
//   12,000 81.3 / 77.1 / 65.0 | 81.2 / 84.0 / 71.7 | 191 / 196 / 178 | 948 / 954 / 944.
// Rollouts write all of them through (plain / streamed / through: 256 514 / 512 / 499, 1,000 558 / 541 / 532, 4,096 1,233 / 1,699 / 1,163; with a cast behind
// each of 8 steps, plain / through: 256 97.0 / 94.2, 4,096 413 / 404, 8,192 983 / 961).  Bytes are streamed: through, 1,024 environments take 9.8 instead
// of 10.2 us and 4,096 15.2 instead of 14.6, 16,384 55.6 instead of 42.7; by a choice at run time, 4,096 lose 1 %.
constexpr long long FLOATS_KEPT = 240ll << 20;
inline cx::Keep floats_kept(int n)
{
    const long long bytes = (long long)n * STRIDE_F32;
    return bytes <= cx::CACHE_SHARE ? cx::Keep::THROUGH : bytes <= FLOATS_KEPT ? cx::Keep::PLAIN : cx::Keep::STREAM;
}
// A step of a few environments leaves its floats in the L2, too, which takes less time to write back than they take to go through one by
// one (1 environment 8.54 us left there, 8.86 written through, 4 9.38 and 9.50, 16 9.82 and 9.90, 32 10.3 either way, 64 10.6 and 10.5).
constexpr int FLOATS_THROUGH_FROM = 32;
// Where that is STREAM: whether the observation of environment env, written by block `block`, is written through.
__device__ inline bool floats_written_through(int env, uint32_t block) { return cx::written_through(block) && (long long)env * STRIDE_F32 < cx::SPLIT_TO; }

// The same by GW < 64 lanes of a wavefront, whose areas have no room for staged bytes (L_ENV_DWORDS): the
// one-hot bytes are staged as single bits (a few LDS atomics per cell) next to a light level per cell;
// every lane then expands 16 bits at a time into one 16-byte piece of the output.
// GW: lanes that render this environment (see Lanes); l: the calling lane's number among them.  FLOATS, through: see render_staged.
template <bool F32, int GW = 64, cx::Keep FLOATS = cx::Keep::THROUGH, bool HALVES = false>
__device__ __forceinline__ void render_env(const int l, uint32_t* e, const int wx0, const int wy0, const int m_alive, const int m_x,
                                  const int m_y, const int m_type, const Luts* __restrict__ luts, uint8_t* __restrict__ out,
                                  const RenderAux<GW>* aux = nullptr, const bool through = false)
{
    if constexpr (GW == 64) { render_staged<F32, FLOATS, HALVES>(l, e, wx0, wy0, m_alive, m_x, m_y, m_type, luts, out, aux, through); return; } else {
    using G = Lanes<GW>;
    const uint32_t* rec = e + L_REC;
    const uint8_t* wb = reinterpret_cast<const uint8_t*>(e + L_WB);
    const uint8_t* wi = reinterpret_cast<const uint8_t*>(e + L_WI);
    uint32_t* cre = e + L_CRE;
    uint32_t* bits = e + L_BITS;
    uint8_t* light = reinterpret_cast<uint8_t*>(e + L_LIGHT);
    float* vec = reinterpret_cast<float*>(e + L_VEC);
    const uint32_t pos = G::uniu(rec[R_POS]);
    const int px = pos & 0xFF, py = (pos >> 8) & 0xFF;
#pragma unroll
    for (int it = 0; it < (260 + GW - 1) / GW; ++it) {
        const int i = l + GW * it;
        if (i < 260) bits[i] = 0u;
    }
#pragma unroll
    for (int it = 0; it < (NCELL + 1 + GW - 1) / GW; ++it) {
        const int i = l + GW * it;
        if (i < NCELL + 1) cre[i] = 0xFFFFFFFFu;
    }
    wave_sync();
    if (l < NSLOT && m_alive) {
        const int vr = m_y - (py - VROWS / 2), vc = m_x - (px - VCOLS / 2);
        if ((unsigned)vr < (unsigned)VROWS && (unsigned)vc < (unsigned)VCOLS)
            atomicMin(&cre[vr * VCOLS + vc], ((uint32_t)l << 8) | (uint32_t)creature_channel(l, m_type));   // lowest slot wins
    }
#pragma unroll
    for (int it = 0; it < (NVEC + 1 + GW - 1) / GW; ++it) {
        const int i = l + GW * it;
        if (i < NVEC + 1) vec[i] = i >= NVEC ? 0.0f : (aux != nullptr ? scalar_value_fast(i, aux->field[it], rec, aux->lut, aux->day) : scalar_value(i, rec, luts));
    }
    wave_sync();
    auto set_bit = [&](int i) { atomicOr(&bits[CX_IDX(i >> 5, 260)], 1u << (i & 31)); };
#pragma unroll
    for (int it = 0; it < (NCELL + GW - 1) / GW; ++it) {
        const int cell = l + GW * it;
        if (cell < NCELL) {
            const int r = cell / VCOLS, c = cell - r * VCOLS;
            const int x = px - VCOLS / 2 + c, y = py - VROWS / 2 + r;
            int lv = 0;
            if (!inb(x, y)) {   // beyond the edge of the map: always visible
                set_bit(cell * NCHAN + B_OOB); set_bit(cell * NCHAN + 37 + IT_NONE); lv = MAX_LIGHT;
            } else {
                const int il = wi[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)];
                lv = il >> 3;
                if (lv != 0) {      // cells darker than 0.05 stay blank
                    set_bit(cell * NCHAN + (wb[CX_IDX((y - wy0) * WIN_PITCH + (x - wx0), WIN_ROWS * WIN_PITCH)] & 63));
                    set_bit(cell * NCHAN + 37 + (il & 7));
                    const uint32_t cr = cre[cell];
                    if (cr != 0xFFFFFFFFu && (cr & 0xFFu) != 82u) set_bit(cell * NCHAN + (int)(cr & 0xFFu));   // channel 82 is the light level, whatever type was imported
                }
            }
            light[cell] = (uint8_t)lv;
        }
    }
    wave_sync();
    // piece j covers bytes [16j, 16j+16) of the cell area; the one light byte inside it (cell c,
    // byte 83c + 82) is patched in
    auto light_in_piece = [&](int j, int* at, int* lv) {
        *at = -1; *lv = 0;
        if (16 * j + 15 >= 82) {
            const int c = (16 * j + 15 - 82) / NCHAN, p = NCHAN * c + 82;
            if (p >= 16 * j && c < NCELL) { *at = p - 16 * j; *lv = light[c]; }
        }
    };
    if (!F32) {
        uint4* dst = reinterpret_cast<uint4*>(out);
#pragma unroll 3
        for (int it = 0; it < (STRIDE_U8 / 16 + GW - 1) / GW; ++it) {
            const int j = l + GW * it;
            if (j < STRIDE_U8 / 16) {
                uint32_t v[4] = { 0u, 0u, 0u, 0u };
                if (j < VEC_OFFSET / 16) {
                    const uint32_t b16 = (bits[j >> 1] >> ((j & 1) * 16)) & 0xFFFFu;
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = spread4((b16 >> (4 * k)) & 15u);
                    int at, lv;
                    light_in_piece(j, &at, &lv);
#pragma unroll
                    for (int k = 0; k < 4; ++k) if ((at >> 2) == k) v[k] |= (uint32_t)lv << (8 * (at & 3));
                } else if (j < VEC_OFFSET / 16 + (NVEC + 3) / 4) {
                    const uint4 f = reinterpret_cast<const uint4*>(e + L_VEC)[j - VEC_OFFSET / 16];
                    v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
                }
                typedef uint32_t piece_t __attribute__((ext_vector_type(4)));
                const piece_t piece = { v[0], v[1], v[2], v[3] };
                __builtin_nontemporal_store(piece, reinterpret_cast<piece_t*>(dst + j));   // one 16-byte streaming store
            }
        }
    } else {
        float4* dst = reinterpret_cast<float4*>(out);
#pragma unroll 1
        for (int j = l; j < STRIDE_F32 / 64; j += GW) {   // 16 floats per piece
            const uint32_t b16 = j < 520 ? (bits[j >> 1] >> ((j & 1) * 16)) & 0xFFFFu : 0u;
            int at, lv;
            light_in_piece(j, &at, &lv);
            const float lf = aux != nullptr ? aux->lut[LUT_LIGHT20 + lv] : luts->light20[lv];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int idx = 16 * j + 4 * q + k;
                    float f = 0.0f;
                    if (idx < CELL_BYTES) f = (4 * q + k == at) ? lf : (float)((b16 >> (4 * q + k)) & 1u);
                    else if (idx < CELL_BYTES + NVEC) f = vec[idx - CELL_BYTES];
                    v[k] = f;
                }
                dst[4 * j + q] = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
    }
}

}  // namespace cf
