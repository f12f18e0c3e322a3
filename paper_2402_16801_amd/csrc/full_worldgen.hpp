// Block-cooperative generation of the nine floors of one full-Craftax world (section "World
// Generation" of the paper's appendix lists the floors: overworld, dungeon, gnomish mines,
// sewers, vault, troll mines, fire realm, ice realm, graveyard).  The paper does not print its
// generators; here every cell of every floor is a pure integer function of (seed, env, episode,
// floor, x, y): noise thresholds for the open floors, eight seeded rooms joined by L-shaped
// corridors for the built ones.  A floor of an environment belongs to a block or to a single wavefront
// (floor_route.hpp), a thread owning a run of 8 cells at a time, so that a reset is nine short pieces of
// work instead of one long one.
#pragma once

#include <type_traits>

#include "full_common.hpp"
#include "worldgen.hpp"

namespace cf {

// A run of 8 cells: the draws of its cells are exactly one Philox block, it lies in one row and in one
// column of lattice cells (of spacing 8 and of spacing 16), and both its maps are stored as 8 bytes.
constexpr int RUN = 8, ROW_RUNS = W / RUN, RUNS = CELLS / RUN;   // 6 runs a row, 288 a floor
// Threads that generate a floor: a single wavefront (five passes over the 288 runs) or a block of five
// wavefronts (one pass); floor_route.hpp says when which.
constexpr int FLOOR_THREADS = 64, GEN_THREADS = 320;
constexpr int LAT0_U16 = 2 * 16 + 4 * 49;                 // overworld lattices: two 4x4 (spacing 16), four 7x7 (spacing 8)
constexpr int LAT0_BLOCKS = (LAT0_U16 + 7) / 8;           // 29
constexpr int LATC_U16 = 2 * 49, LATC_BLOCKS = (LATC_U16 + 7) / 8;   // cave floors: two 7x7 lattices, 13 blocks
constexpr int LAT_TOTAL = LAT0_BLOCKS * 8;                // a block generates one floor: the largest lattice set

// The lattices lie in LDS as in the Classic generator, one number after the other: as floats, for Perlin noise the
// cosines.  The sines of a cave's lattices follow behind them; those of the overworld, which needs no row masks,
// take the masks' place.  The overworld's 4x4 lattices come first.
constexpr int WIDE0 = 2 * 16, LATC_N = LATC_BLOCKS * 8;
constexpr int LAT_WORDS = LAT_TOTAL;
static_assert(2 * LATC_N <= LAT_WORDS, "cosines and sines of a cave");

struct Room { int x, y, w, h, cx, cy; };
struct GenLayout {
    Room room[3][8];          // dungeon (floor 1), sewers (3), vault (4)
    int up[FLOORS][2], down[FLOORS][2];
    uint32_t perm;            // potion colour -> effect, 6 x 3 bits
    // The floor being generated, row by row (bit x = column x).  Built floors (dungeon_row_mask): cells
    // inside rooms 0..3 and 4..7, cells on corridors 0..3 and 4..6, chest cells.  Caves
    // (cave_row_mask): the cells that are open whatever the noise says.  And the single cells of
    // a floor as x | y << 8: fountain, the two enchantment tables, ladder up, ladder down (0xFFFF:
    // this floor has none).
    uint64_t row_mask[5][W];
    uint32_t spot[5];
    __device__ float* overworld_sines() { return reinterpret_cast<float*>(row_mask); }
};
static_assert(sizeof(GenLayout::row_mask) >= LAT_TOTAL * sizeof(float), "sines of the overworld");

__device__ inline int dungeon_index(int f) { return f == 1 ? 0 : (f == 3 ? 1 : 2); }
__device__ inline bool is_dungeon(int f) { return f == 1 || f == 3 || f == 4; }
__device__ inline bool is_cave(int f) { return f == 2 || f == 5 || f == 6 || f == 7; }

constexpr int START_BIAS_R = cx::START_BIAS_R, START_BIAS = cx::START_BIAS, START_CLEAR = cx::START_CLEAR;
static_assert((int)B_GRASS == cx::BK_GRASS && (int)B_WATER == cx::BK_WATER && (int)B_STONE == cx::BK_STONE && (int)B_TREE == cx::BK_TREE &&
              (int)B_PATH == cx::BK_PATH && (int)B_COAL == cx::BK_COAL && (int)B_IRON == cx::BK_IRON && (int)B_DIAMOND == cx::BK_DIAMOND &&
              (int)B_SAND == cx::BK_SAND && (int)B_LAVA == cx::BK_LAVA, "the overworld is the Classic rule (cx::classify)");

// A built floor as bit masks per row, so that a run costs a few shifts and byte masks instead of eight
// room tests, seven corridor tests and nine single-cell tests per cell.  Part p of row y (five parts,
// so that 240 threads share the work): rooms 0..3, rooms 4..7, corridors 0..3, corridors 4..6
// (corridor i: along row cy of room i from its centre to the centre column of room i + 1, then along
// that column), chests (one right and below the centre of rooms 1..6).  The single cells go to L.spot.
constexpr int M_ROOMS_A = 0, M_ROOMS_B = 1, M_PATH_A = 2, M_PATH_B = 3, M_CHEST = 4, MASK_PARTS = 5;
constexpr int SPOT_FOUNTAIN = 0, SPOT_FIRE = 1, SPOT_ICE = 2, SPOT_UP = 3, SPOT_DOWN = 4;
__device__ inline void dungeon_row_mask(GenLayout& L, int f, int y, int part)
{
    const Room* R = L.room[dungeon_index(f)];
    auto span = [](int a, int b) -> uint64_t { return (~0ull >> (63 - (b - a))) << a; };   // bits a..b, 0 <= a <= b < 64
    uint64_t m = 0ull;
    if (part == M_ROOMS_A || part == M_ROOMS_B) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const Room r = R[4 * (part - M_ROOMS_A) + k];
            if ((unsigned)(y - r.y) < (unsigned)r.h) m |= span(r.x, r.x + r.w - 1);
        }
    } else if (part == M_PATH_A || part == M_PATH_B) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = 4 * (part - M_PATH_A) + k;
            if (i < 7) {
                const int x0 = R[i].cx, y0 = R[i].cy, x1 = R[i + 1].cx, y1 = R[i + 1].cy;
                if (y == y0) m |= span(min(x0, x1), max(x0, x1));
                if (y >= min(y0, y1) && y <= max(y0, y1)) m |= 1ull << x1;
            }
        }
    } else {
#pragma unroll
        for (int i = 1; i <= 6; ++i) if (y == R[i].cy + 1) m |= 1ull << (R[i].cx + 1);
    }
    L.row_mask[CX_IDX(part, MASK_PARTS)][CX_IDX(y, W)] = m;
}
__device__ inline void dungeon_spot(GenLayout& L, int f, int k)
{
    const Room* R = L.room[dungeon_index(f)];
    auto at = [](int x, int y) { return (uint32_t)x | ((uint32_t)y << 8); };
    uint32_t v = 0xFFFFu;
    if (k == SPOT_FOUNTAIN && f == 1) v = at(R[2].cx - 1, R[2].cy - 1);
    if (k == SPOT_FIRE && f == 4) v = at(R[3].cx - 1, R[3].cy - 1);
    if (k == SPOT_ICE && f == 4) v = at(R[4].cx - 1, R[4].cy - 1);
    if (k == SPOT_UP) v = at(R[0].cx, R[0].cy);
    if (k == SPOT_DOWN) v = at(R[7].cx, R[7].cy);
    L.spot[k] = v;
}
// Row y of a cave floor as one bit mask (L.row_mask[M_CAVE_OPEN]): the cells that are open whatever the
// noise says, i.e. the 3 x 3 clearings around the two ladders and the L-shaped corridor between
// them (the two ladders are always connected); the ladders themselves go to L.spot.
constexpr int M_CAVE_OPEN = 0;
__device__ inline void cave_row_mask(GenLayout& L, int f, int y)
{
    const int ux = L.up[f][0], uy = L.up[f][1], dx = L.down[f][0], dy = L.down[f][1];
    auto span = [](int a, int b) -> uint64_t { return (~0ull >> (63 - (b - a))) << a; };   // bits a..b, 0 <= a <= b < 64
    uint64_t m = 0ull;
    if (iabs(y - uy) <= 1) m |= span(ux - 1, ux + 1);
    if (iabs(y - dy) <= 1) m |= span(dx - 1, dx + 1);
    if (y == uy) m |= span(min(ux, dx), max(ux, dx));                 // along row uy from ux to dx,
    if (y >= min(uy, dy) && y <= max(uy, dy)) m |= 1ull << dx;        // then along column dx from uy to dy
    L.row_mask[M_CAVE_OPEN][CX_IDX(y, W)] = m;
    if (y == 0) {
        L.spot[SPOT_UP] = (uint32_t)ux | ((uint32_t)uy << 8);
        L.spot[SPOT_DOWN] = (uint32_t)dx | ((uint32_t)dy << 8);
    }
}

// World-generation draws: counter (env, stream, episode, WORLDGEN | block); stream = floor*4 +
// {0 lattices, 1 per-cell u16, 2 layout words}, stream 63 = potion permutation.
__device__ inline U4 wg_block(uint32_t lo, uint32_t hi, uint32_t env, uint32_t episode, uint32_t stream, uint32_t block)
{
    return philox4x32_10(env, stream, episode, (cx::DOM_WORLDGEN << 16) | block, lo, hi);
}

__device__ inline void make_room(GenLayout& L, int f, int i, const U4& r)
{
    Room R;
    R.w = 5 + (int)choice(r.w[0], 5);
    R.h = 5 + (int)choice(r.w[1], 5);
    R.x = 1 + (int)choice(r.w[2], (uint32_t)(46 - R.w));
    R.y = 1 + (int)choice(r.w[3], (uint32_t)(46 - R.h));
    R.cx = R.x + R.w / 2;
    R.cy = R.y + R.h / 2;
    L.room[dungeon_index(f)][i] = R;
    if (i == 0) { L.up[f][0] = R.cx; L.up[f][1] = R.cy; }
    if (i == 7) { L.down[f][0] = R.cx; L.down[f][1] = R.cy; }
}
__device__ inline void make_cave_ladders(GenLayout& L, int f, const U4& r)
{
    L.up[f][0] = 10 + (int)choice(r.w[0], 6); L.up[f][1] = 10 + (int)choice(r.w[1], 6);
    L.down[f][0] = 32 + (int)choice(r.w[2], 6); L.down[f][1] = 32 + (int)choice(r.w[3], 6);
}

// The eight lattice numbers of Philox block `block`; sines: where those go with Perlin noise, of COUNT numbers
template <bool CAN_PERLIN, int COUNT>
__device__ inline void put_lattice(uint32_t* s_lat, float* sines, int block, const U4& r, const uint32_t* __restrict__ perlin_cs, const uint16_t* theta_f)
{
    float* lat = reinterpret_cast<float*>(s_lat);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int i = CX_IDX(block * 8 + j, COUNT);
        uint32_t v = (j & 1) ? (r.w[j >> 1] >> 16) : (r.w[j >> 1] & 0xFFFFu);
        if (CAN_PERLIN && perlin_cs != nullptr) {
            if (theta_f != nullptr) v = (v + ((theta_f[i] & 1023u) << 6)) & 0xFFFFu;
            const uint32_t cs = perlin_cs[v >> 6];
            lat[i] = (float)(int)(int16_t)(cs & 0xFFFFu);
            sines[i] = (float)((int)cs >> 16);
        } else lat[i] = (float)v;
    }
}

// Eight cells, one byte each: cells 0..3 in x, 4..7 in y.
__device__ inline uint2 all_cells(uint32_t v) { return make_uint2(v * 0x01010101u, v * 0x01010101u); }
// the bytes whose bit of `where` (bit 0 = cell 0) is set become v
__device__ inline uint2 cells_where(uint2 c, uint32_t where, uint32_t v)
{
    auto mask = [](uint32_t nibble) { const uint32_t ones = (nibble * 0x00204081u) & 0x01010101u; return (ones << 8) - ones; };
    const uint32_t m0 = mask(where & 15u), m1 = mask((where >> 4) & 15u);
    return make_uint2((c.x & ~m0) | (v * 0x01010101u & m0), (c.y & ~m1) | (v * 0x01010101u & m1));
}
// the single cell `spot` (x | y << 8), if it lies in the run whose first cell is (x0, y)
__device__ inline bool spot_in_run(uint32_t spot, int x0, int y) { return (spot & 0xFFF8u) == ((uint32_t)x0 | ((uint32_t)y << 8)); }

// What a cave floor makes of a cell's fields and draw u.  Open cells (cave field above 31000): a plant
// where u < plant_below, a liquid where the second field is above its threshold, the floor's ground
// elsewhere; rock: ore i where u < below_i for the first such i, stone elsewhere.  What a kind of floor
// lacks is left out of its code: the gnomish mines have no liquid (and no need of the second field),
// the troll mines no plants, the fire and ice realms two ores instead of five.
// A cell is a code 0..7, its place in the floor's table of blocks, so that one byte permutation looks up
// four cells: 0 stone, 1 2 3 4 5 the ores in order, 6 ground, 7 the plant, and the liquid is 7
// where there are no plants and 5 where there are only two ores.
enum CaveKind : int { GNOME_MINES, TROLL_MINES, REALM };
struct CaveRule { uint32_t table_lo, table_hi, below1; };   // blocks of codes 0..3 and 4..7; realms: where the second ore ends, as a draw in the upper half
__device__ inline CaveRule cave_rule(int f)
{
    using cx::four_bytes;
    CaveRule c;
    const bool mines = f == 2 || f == 5;
    c.table_lo = mines ? four_bytes(B_STONE, B_COAL, B_IRON, B_DIAMOND) : f == 6 ? four_bytes(B_STONE, B_RUBY, B_COAL, B_STONE) : four_bytes(B_STONE, B_SAPPHIRE, B_DIAMOND, B_STONE);
    c.table_hi = f == 2 ? four_bytes(B_SAPPHIRE, B_RUBY, B_PATH, B_STALAGMITE) : f == 5 ? four_bytes(B_SAPPHIRE, B_RUBY, B_PATH, B_WATER)
               : f == 6 ? four_bytes(B_STONE, B_LAVA, B_FIRE_GRASS, B_FIRE_TREE) : four_bytes(B_STONE, B_WATER, B_ICE_GRASS, B_ICE_SHRUB);
    c.below1 = (f == 6 ? 6000u : 5000u) << 16;
    return c;
}
__device__ inline uint32_t cave_ground(int f) { return f == 6 ? (uint32_t)B_FIRE_GRASS : (f == 7 ? (uint32_t)B_ICE_GRASS : (uint32_t)B_PATH); }
// thresholds in scalar registers, as in cx::Thresholds: of the fields, of the draws
template <bool PERLIN, int KIND>
struct CaveThresholds {
    template <int T> __device__ static uint32_t draw() { return cx::scalar_const<(uint32_t)T << 16>(); }
    template <int T> __device__ static float field() { return __uint_as_float(cx::scalar_const<cx::f32_bits(cx::first_above<PERLIN>(T))>()); }
    static constexpr bool GNOME = KIND == GNOME_MINES, MINES = KIND != REALM;
    float open = field<31000>(), liquid = field<MINES ? 44000 : 43000>();
    uint32_t plant = draw<GNOME ? 1500 : 3000>(), b0 = draw<MINES ? 5000 : 2500>(), b1 = draw<7500>(), b2 = draw<8000>(), b3 = draw<GNOME ? 8600 : 9000>(), b4 = draw<GNOME ? 9200 : 10000>();
};
// Appends the cell's code to `word`, where a cell takes a byte.  C, F: the fields; u: the draw in the upper half
template <bool PERLIN, int KIND>
__device__ __forceinline__ void classify_cave(uint32_t& word, const CaveThresholds<PERLIN, KIND>& t, uint32_t below1, float C, float F, uint32_t u)
{
    using cx::Mask; using cx::mask_of; using cx::shift_in_or;
    const Mask open = mask_of(C >= t.open), ore0 = mask_of(u < t.b0);
    word <<= 5;
    if (KIND == REALM) {
        const Mask liquid = mask_of(F >= t.liquid);
        cx::shift_in(word, open);
        shift_in_or(word, open & ~liquid, mask_of(u < below1) & ~(ore0 | open));
        shift_in_or(word, open & (liquid | mask_of(u < t.plant)), ore0 & ~open);
    } else {
        const Mask special = KIND == GNOME_MINES ? mask_of(u < t.plant) : mask_of(F >= t.liquid);
        const Mask b2 = mask_of(u < t.b2), b4 = mask_of(u < t.b4);
        shift_in_or(word, open, b4 & ~b2);
        shift_in_or(word, open, b2 & ~ore0);
        shift_in_or(word, open & special, (ore0 | (b2 & ~mask_of(u < t.b1)) | (b4 & ~mask_of(u < t.b3))) & ~open);
    }
}
__device__ inline uint32_t cave_blocks(const CaveRule& k, uint32_t word) { return __builtin_amdgcn_perm(k.table_hi, k.table_lo, word); }

// Generates floor f of one environment with the NT threads of the calling block (NT = 64: with the
// calling wavefront, whatever the other wavefronts of its block do): run t (of 288)
// is the 8 cells [8t, 8t+8) of the floor (row t/6).  The block of floor 0 also derives the
// ladders of every floor and the potion permutation (whole_layout), which the fresh record
// needs, and may drop the cells around the start position into an LDS window (start_wb /
// start_wi, 44 dwords each) for the first observation.  maps: this environment's 41472
// bytes.  s_lat (LAT_WORDS dwords), L: LDS scratch.  All arguments are the same for the whole block.
// Ends with a barrier of those threads.
// perlin_cs (with CAN_PERLIN): the gradient table; the fields of the overworld and of the caves are
// then Perlin noise over the same lattices (appendix "World Generation") instead of value noise.
// A kernel instantiated without CAN_PERLIN carries no code for it.
// theta_f (with CAN_PERLIN; LDS, LAT_TOTAL entries, the same for the whole block): angle offsets in
// 1024ths of a turn added to the upper ten bits of this floor's lattice numbers, the level of the
// noise mutation (section "Craftax-1B: UED").
// Bound by instruction issue, like the Classic generator, and written in the same way (worldgen.hpp): fields in
// 32-bit floating point rounded down, masks on the scalar unit, a code per cell that byte permutations turn into
// blocks.  A run of 8 cells uses all of its Philox block, and the built floors are byte masks over whole
// runs.  Measured: craftax_reset with its observation, fields in 64 bits and in 32: 4,096 environments (8,192 worlds, 340 MB)
// 176 -> 171 us, with Perlin noise 269 -> 218, of 256 with Perlin noise 46.3 -> 43.3.
// LOOPED: the call stands in a loop over worlds; what a thread derives from its index is then derived
// anew in every call instead of being kept (and spilled) across the loop.
template <int NT = GEN_THREADS, bool CAN_PERLIN = false, bool LOOPED = false>
__device__ __forceinline__ void worldgen_floor_block(uint8_t* __restrict__ maps, uint32_t* s_lat, GenLayout& L, uint32_t lo, uint32_t hi,
                                            uint32_t env, uint32_t episode, int f, uint32_t* start_wb = nullptr,
                                            uint32_t* start_wi = nullptr, const uint32_t* __restrict__ perlin_cs = nullptr,
                                            const uint16_t* theta_f = nullptr)
{
    const bool use_perlin = CAN_PERLIN && perlin_cs != nullptr;
    static_assert(NT >= 64, "the layout phase uses the first wavefront");
    // uniform arguments that come from memory: in scalar registers, with the key schedule and the
    // first products of every Philox block
    lo = uniu(lo); hi = uniu(hi); env = uniu(env); episode = uniu(episode); f = uni(f);
    int tid0 = NT == 64 ? (int)(threadIdx.x & 63u) : (int)threadIdx.x;
    if (LOOPED) asm volatile("" : "+v"(tid0));
    auto barrier = []() { if (NT == 64) wave_sync(); else __syncthreads(); };
    // Layout phase, all in the first wavefront and with one Philox call for the whole wave: every
    // lane picks the (stream, block) of its role, then the roles unpack their words.
    if (tid0 < 64) {
        const int tid = tid0;
        if (f == 0) {
            // lanes 0..28 lattice blocks; 29..52 rooms of floors 1, 3, 4; 53..56 ladders of the caves 2, 5, 6, 7;
            // 57 overworld ladder; 58, 59 potion permutation (section "Potions and Enchantments")
            uint32_t stream = 0u, block = (uint32_t)tid;
            int ff = 0;
            if (tid >= 29 && tid < 53) { const int d = (tid - 29) >> 3; ff = d == 0 ? 1 : (d == 1 ? 3 : 4); stream = (uint32_t)ff * 4u + 2u; block = (uint32_t)((tid - 29) & 7); }
            else if (tid >= 53 && tid < 57) { const int c = tid - 53; ff = c == 0 ? 2 : (c == 1 ? 5 : (c == 2 ? 6 : 7)); stream = (uint32_t)ff * 4u + 2u; block = 0u; }
            else if (tid == 57) { stream = 2u; block = 0u; }
            else if (tid >= 58) { stream = 63u; block = tid == 59 ? 1u : 0u; }
            const U4 r = wg_block(lo, hi, env, episode, stream, block);
            const uint32_t fifth = (uint32_t)__shfl((int)r.w[0], 59);
            if (tid < LAT0_BLOCKS) put_lattice<CAN_PERLIN, LAT_TOTAL>(s_lat, L.overworld_sines(), tid, r, perlin_cs, theta_f);
            else if (tid < 53) make_room(L, ff, (tid - 29) & 7, r);
            else if (tid < 57) make_cave_ladders(L, ff, r);
            else if (tid == 57) {
                int dx = (int)choice(r.w[0], 13) - 6;
                const int dy = (int)choice(r.w[1], 13) - 6;
                if (max(iabs(dx), iabs(dy)) < 3) dx = 3;
                L.up[0][0] = 0; L.up[0][1] = 0; L.down[0][0] = W / 2 + dx; L.down[0][1] = W / 2 + dy;
                L.spot[SPOT_DOWN] = (uint32_t)(W / 2 + dx) | ((uint32_t)(W / 2 + dy) << 8);
                L.up[8][0] = 24; L.up[8][1] = 42; L.down[8][0] = 0; L.down[8][1] = 0;
            } else if (tid == 58) {
                // a fresh colour -> effect permutation per episode
                const uint32_t draws[5] = { r.w[0], r.w[1], r.w[2], r.w[3], fifth };
                uint32_t perm = 0u;
#pragma unroll
                for (int i = 0; i < 6; ++i) perm |= (uint32_t)i << (3 * i);
#pragma unroll
                for (int i = 5; i >= 1; --i) {
                    const int j = (int)choice(draws[5 - i], (uint32_t)(i + 1));
                    const uint32_t a = (perm >> (3 * i)) & 7u, b = (perm >> (3 * j)) & 7u;
                    perm &= ~((7u << (3 * i)) | (7u << (3 * j)));
                    perm |= (b << (3 * i)) | (a << (3 * j));
                }
                L.perm = perm;
            }
        } else if (is_dungeon(f)) {
            if (tid < 8) make_room(L, f, tid, wg_block(lo, hi, env, episode, (uint32_t)f * 4u + 2u, (uint32_t)tid));
        } else if (is_cave(f)) {
            // lanes 0..12 lattice blocks, lane 13 the ladders
            if (tid <= LATC_BLOCKS) {
                const U4 r = wg_block(lo, hi, env, episode, (uint32_t)f * 4u + (tid == LATC_BLOCKS ? 2u : 0u), tid == LATC_BLOCKS ? 0u : (uint32_t)tid);
                if (tid < LATC_BLOCKS) put_lattice<CAN_PERLIN, LATC_N>(s_lat, reinterpret_cast<float*>(s_lat) + LATC_N, tid, r, perlin_cs, theta_f);
                else make_cave_ladders(L, f, r);
            }
        }
    }
    barrier();
    if (is_dungeon(f)) {                       // the same floor for the whole block
        for (int i = tid0; i < MASK_PARTS * W; i += NT) dungeon_row_mask(L, f, i % W, i / W);
        if (tid0 < 5) dungeon_spot(L, f, tid0);
        barrier();
    } else if (is_cave(f)) {
        if (tid0 < W) cave_row_mask(L, f, tid0);
        barrier();
    }
    const float* lat = reinterpret_cast<const float*>(s_lat);
    cx::floor_rounding(tid0);
    // A run's number and the number of its strip are even or odd together, and so is the lane's: whether a
    // run is the right half of a spacing-16 lattice cell is the same in every pass.
    static_assert(ROW_RUNS % 2 == 0 && NT % 2 == 0, "parity of the strips");
    // runs of 8 cells, one per thread and pass.  A block that covers the floor in one pass is no loop: the range of tid0 is not known
    // any more here, and in front of a loop the compiler kept the constants of every kind of floor in scalar registers and spilled
    // 14 to 16 of them (craftax_reset of 64 and 256 environments 26.1 and 39.2 us, 25.3 and 35.8 without; level turns over 400 and 500
    // 47.2 and 57.8, 45.6 and 56.4; Perlin resets of 64 29.7 and 27.2, Perlin level turns over 128 57.5 and 54.0).
#pragma unroll 1
    for (int run = tid0; run < RUNS; run += NT) {
    const int y = run / ROW_RUNS, strip = run - y * ROW_RUNS, x0 = strip * RUN;
    U4 r = { { 0u, 0u, 0u, 0u } };                          // the run's draws: eight u16, one per cell
    if (!(f == 1 || f == 4 || f == 8)) r = wg_block(lo, hi, env, episode, (uint32_t)f * 4u + 1u, (uint32_t)run);
    uint2 blocks = make_uint2(0u, 0u), items = all_cells(lit_floor(f) ? (uint32_t)MAX_LIGHT << 3 : 0u);
    // single cells, the last one placed counts (the two ladders of a built floor may fall on one cell)
    auto place = [&](uint32_t spot, uint32_t block, uint32_t item) {
        if (!spot_in_run(spot, x0, y)) return;
        const uint32_t j = spot & 7u, sh = 8u * (j & 3u), keep = ~(0xFFu << sh), light = ~(7u << sh);
        if (j < 4u) { blocks.x = (blocks.x & keep) | (block << sh); items.x = (items.x & light) | (item << sh); }
        else { blocks.y = (blocks.y & keep) | (block << sh); items.y = (items.y & light) | (item << sh); }
    };
    uint32_t word = 0u, second = 0u;                        // the cells under way, from right to left; the finished cells 4..7
    auto draw = [&](auto j) { return (j & 1) ? r.w[j >> 1] : r.w[j >> 1] << 16; };   // draw of cell j, in the upper half
    // the floor is the same for the whole block: one kind of cell function per block
    if (f == 0) {
        // the points above and left of the run in the two lattices of spacing 16 and the four of spacing 8
        const int at16 = CX_IDX((y >> 4) * 4 + (x0 >> 4), 16 - 5), at8 = WIDE0 + CX_IDX((y >> 3) * 7 + strip, 49 - 8);
        const int w16 = at16, m16 = w16 + 16, w8 = at8, m8 = w8 + 49, c8 = m8 + 49, f8 = c8 + 49;
        uint32_t odd = 0u - (uint32_t)(run & 1);            // all ones: right half of a spacing-16 lattice cell
        asm volatile("" : "+v"(odd));                        // or the weights of all passes are computed, and spilled, before the first
        // 4 times the lowering (10 - d) * 2500 of W and M within Chebyshev distance d < 10 of the start
        const int step = 4 * START_BIAS, bias_y = max(0, START_BIAS_R - iabs(y - W / 2)) * step;
        const int bias_l = (START_BIAS_R + x0 - W / 2) * step, bias_r = (START_BIAS_R - x0 + W / 2) * step;
        const bool near_rows = __any(bias_y != 0);          // a pass covers ten or eleven rows
        auto put = [&](const auto& thresholds, auto j, float W4, float M4, float C, float F) {
            uint32_t u = draw(j);
            if (near_rows) cx::near_start(max(0, min(min(bias_l + j * step, bias_r - j * step), bias_y)), W4, M4, u);
            cx::classify(word, thresholds, W4, M4, C, F, u);
            cx::settle(word);
            if (j == 4) second = word;                      // (the next four cells shift it out)
        };
        if (CAN_PERLIN && use_perlin) {
            const int ky16 = y & 15, ky8 = y & 7;
            const float wy16 = (float)cx::perlin_fade<16>(ky16) * (1.0f / 65536.0f), wy8 = (float)cx::perlin_fade<8>(ky8) * (1.0f / 65536.0f);
            // One field after the other for the whole run; the last one with the rule.
            // The empty statement keeps the loads of a field's gradients from being moved before the field at hand.
            auto along = [&](cx::PerlinLine line, auto&& weight, float wy, auto&& cell) {
                cx::for_run([&](auto j) { cell(j, line.field(weight(j), wy)); line.advance(); });
                asm volatile("" ::: "memory");
            };
            const float* sines = L.overworld_sines();
            auto wide = [&](int at) { return cx::perlin_line<16>(lat + at, sines + at, 4, (float)((x0 & 15) + 7), (float)ky16); };
            auto narrow = [&](int at) { return cx::perlin_line<8>(lat + at, sines + at, 7, 7.0f, (float)ky8); };
            auto wx16 = [&](auto j) { return cx::pick<cx::f32_bits(cx::perlin_weight<16>(8 + j)), cx::f32_bits(cx::perlin_weight<16>(j))>(odd); };
            auto wx8 = [&](auto j) { return cx::perlin_weight<8>(j); };
            float W4[RUN], M4[RUN], C[RUN];
            const cx::PerlinScale<16> coarse;
            const cx::PerlinScale<8> fine;
            along(wide(w16), wx16, wy16, [&](int j, float v) { W4[j] = coarse.value(v); cx::settle(W4[j]); });
            along(narrow(w8), wx8, wy8, [&](int j, float v) { W4[j] = cx::perlin_mix31(W4[j], fine.value(v)); cx::settle(W4[j]); });
            along(wide(m16), wx16, wy16, [&](int j, float v) { M4[j] = coarse.value(v); cx::settle(M4[j]); });
            along(narrow(m8), wx8, wy8, [&](int j, float v) { M4[j] = cx::perlin_mix31(M4[j], fine.value(v)); cx::settle(M4[j]); });
            along(narrow(c8), wx8, wy8, [&](int j, float v) { C[j] = v; cx::settle(C[j]); });
            const cx::Thresholds<CAN_PERLIN> thresholds;
            along(narrow(f8), wx8, wy8, [&](auto j, float v) { put(thresholds, j, W4[j], M4[j], C[j], v); });
        } else {
            const float wy16 = (float)cx::smooth16(y & 15) * (1.0f / 256.0f), wy8 = (float)cx::smooth8(y & 7) * (1.0f / 256.0f);
            const cx::Line W16 = cx::line_at(lat + w16, 4, wy16), M16 = cx::line_at(lat + m16, 4, wy16);
            const cx::Line W8 = cx::line_at(lat + w8, 7, wy8), M8 = cx::line_at(lat + m8, 7, wy8), C8 = cx::line_at(lat + c8, 7, wy8), F8 = cx::line_at(lat + f8, 7, wy8);
            const cx::Thresholds<false> thresholds;
            cx::for_run([&](auto j) {
                const float wx16 = cx::pick<cx::f32_bits(cx::weight16(8 + j)), cx::f32_bits(cx::weight16(j))>(odd);
                constexpr float wx8 = cx::weight8(j);
                put(thresholds, j, cx::mix31(W16.at(wx16), W8.at(wx8)), cx::mix31(M16.at(wx16), M8.at(wx8)), C8.at(wx8), F8.at(wx8));
            });
        }
        blocks = make_uint2(cx::blocks_of(word), cx::blocks_of(second));
        place(L.spot[SPOT_DOWN], B_PATH, IT_LADDER_DOWN);
    } else if (is_dungeon(f)) {
        const int yr = CX_IDX(y, W);
        const uint32_t in = (uint32_t)((L.row_mask[M_ROOMS_A][yr] | L.row_mask[M_ROOMS_B][yr]) >> x0),
                       path = (uint32_t)((L.row_mask[M_PATH_A][yr] | L.row_mask[M_PATH_B][yr]) >> x0), chest = (uint32_t)(L.row_mask[M_CHEST][yr] >> x0);
        uint32_t wet = 0u;                                  // the sewers: cells of rooms that hold water
        if (f == 3) {
#pragma unroll
            for (int j = 0; j < 8; ++j) wet |= (((j & 1) ? r.w[j >> 1] >> 16 : r.w[j >> 1] & 0xFFFFu) < 12000u ? 1u : 0u) << j;
        }
        blocks = cells_where(all_cells(f == 3 ? B_WALL_MOSS : B_WALL), in, B_PATH);
        blocks = cells_where(blocks, in & wet, B_WATER);
        blocks = cells_where(blocks, chest, B_CHEST);
        place(L.spot[SPOT_FOUNTAIN], B_FOUNTAIN, 0u);
        place(L.spot[SPOT_FIRE], B_ENCH_FIRE, 0u);
        place(L.spot[SPOT_ICE], B_ENCH_ICE, 0u);
        blocks = cells_where(blocks, path, B_PATH);         // corridors last: room centre 0 (ladder up) always reaches room centre 7 (ladder down)
        place(L.spot[SPOT_UP], B_PATH, IT_LADDER_UP);
        place(L.spot[SPOT_DOWN], B_PATH, IT_LADDER_DOWN_BLOCKED);
    } else if (f == 8) {
        // walled arena, fifteen graves of three kinds in turn, the necromancer and the ladder up
        const bool rim = y == 0 || y == W - 1;
        blocks = all_cells(rim ? B_WALL : B_PATH);
        if (x0 == 0) blocks.x = (blocks.x & ~0xFFu) | B_WALL;
        if (x0 == W - RUN) blocks.y = (blocks.y & 0x00FFFFFFu) | ((uint32_t)B_WALL << 24);
        if (strip >= 1 && strip <= 5 && (y == 12 || y == 24 || y == 36)) blocks.x = (blocks.x & ~0xFFu) | (uint32_t)(B_GRAVE1 + (strip - 1 + y / 12 - 1) % 3);
        place((uint32_t)BOSS_X | ((uint32_t)BOSS_Y << 8), B_NECRO_VULN, 0u);
        place(24u | (42u << 8), B_PATH, IT_LADDER_UP);
    } else {
        const CaveRule rule = cave_rule(f);
        const float* c8 = lat + CX_IDX((y >> 3) * 7 + strip, 49 - 8);
        const float* f8 = c8 + 49;
        auto cave = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
            if (CAN_PERLIN && use_perlin) {
                const int ky8 = y & 7;
                const float wy8 = (float)cx::perlin_fade<8>(ky8) * (1.0f / 65536.0f);
                float C[RUN];
                cx::PerlinLine nC = cx::perlin_line<8>(c8, c8 + LATC_N, 7, 7.0f, (float)ky8);
                cx::for_run([&](auto j) { C[j] = nC.field(cx::perlin_weight<8>(j), wy8); cx::settle(C[j]); nC.advance(); });
                asm volatile("" ::: "memory");
                cx::PerlinLine nF = cx::perlin_line<8>(f8, f8 + LATC_N, 7, 7.0f, (float)ky8);
                const CaveThresholds<CAN_PERLIN, KIND> thresholds;
                cx::for_run([&](auto j) {
                    classify_cave<CAN_PERLIN, KIND>(word, thresholds, rule.below1, C[j], KIND == GNOME_MINES ? 0.0f : nF.field(cx::perlin_weight<8>(j), wy8), draw(j));
                    cx::settle(word);
                    if (j == 4) second = word;
                    nF.advance();
                });
            } else {
                const float wy8 = (float)cx::smooth8(y & 7) * (1.0f / 256.0f);
                const cx::Line C8 = cx::line_at(c8, 7, wy8), F8 = cx::line_at(f8, 7, wy8);
                const CaveThresholds<false, KIND> thresholds;
                cx::for_run([&](auto j) {
                    constexpr float wx8 = cx::weight8(j);
                    classify_cave<false, KIND>(word, thresholds, rule.below1, C8.at(wx8), KIND == GNOME_MINES ? 0.0f : F8.at(wx8), draw(j));
                    cx::settle(word);
                    if (j == 4) second = word;
                });
            }
        };
        if (f == 2) cave(std::integral_constant<int, GNOME_MINES>());
        else if (f == 5) cave(std::integral_constant<int, TROLL_MINES>());
        else cave(std::integral_constant<int, REALM>());
        blocks = make_uint2(cave_blocks(rule, word), cave_blocks(rule, second));
        blocks = cells_where(blocks, (uint32_t)(L.row_mask[M_CAVE_OPEN][CX_IDX(y, W)] >> x0), cave_ground(f));
        place(L.spot[SPOT_UP], B_PATH, IT_LADDER_UP);
        place(L.spot[SPOT_DOWN], B_PATH, IT_LADDER_DOWN_BLOCKED);
    }
    *reinterpret_cast<uint2*>(maps + block_off(f, x0, y)) = blocks;
    *reinterpret_cast<uint2*>(maps + il_off(f, x0, y)) = items;
    if (start_wb != nullptr && f == 0) {
        // window of the start cell (24, 24): rows 19..29, columns 16..31
        const int wr = y - win_y0(W / 2), wc = x0 - win_x0(W / 2);
        static_assert(win_x0(W / 2) % RUN == 0, "a run lies in the window or outside");
        if ((unsigned)wr < (unsigned)WIN_ROWS && (unsigned)wc < (unsigned)WIN_COLS) {
            const int at = CX_IDX(wr * (WIN_PITCH / 4) + wc / 4, WIN_DWORDS - 1);
            start_wb[at] = blocks.x; start_wb[at + 1] = blocks.y;
            start_wi[at] = items.x; start_wi[at + 1] = items.y;
        }
    }
    if (NT >= RUNS) break;
    }
    cx::nearest_rounding();                                  // every run has been stored
    barrier();
}

// The ten dwords that describe a generated world beyond its maps: ladders of the nine floors and
// the potion permutation (valid in the block that generated floor 0).
__device__ inline uint32_t layout_word(const GenLayout& L, int i)
{
    if (i < FLOORS) return (uint32_t)L.up[i][0] | ((uint32_t)L.up[i][1] << 8) | ((uint32_t)L.down[i][0] << 16) | ((uint32_t)L.down[i][1] << 24);
    return L.perm;
}

// Word i (0..63) of the record of a fresh episode: player in the middle of the overworld
// facing down, vitals 9, attributes 1, boss vulnerable, floor 0 visited.
// layout: the ten layout_word values of the world.
__device__ inline uint32_t fresh_record_word(int i, const uint32_t* layout, uint32_t lo, uint32_t hi, uint32_t episode)
{
    if (i >= R_LADDER && i < R_LADDER + FLOORS) return layout[i - R_LADDER];
    switch (i) {
    case R_POS: return (uint32_t)(W / 2) | ((uint32_t)(W / 2) << 8) | (4u << 16);
    case R_FLAGS: return 1u << 17;
    case R_ATTR: return (1u << 20) | (1u << 23) | (1u << 26);
    case R_VIT: return 0x09090909u;
    case R_MANA: return 9u;
    case R_PERM: return layout[FLOORS] | (1u << 18);
    case R_EPISODE: return episode;
    case R_SEED_LO: return lo;
    case R_SEED_HI: return hi;
    default: return 0u;
    }
}

}  // namespace cf
