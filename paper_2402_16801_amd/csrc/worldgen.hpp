// Block-cooperative generation of one 64x64 Craftax-Classic world (appendix "World
// Generation" of the paper: noise thresholds carve grassland, forest, lakes, mountains with
// caves, tunnels, ores and lava).  Two noises feed the same rule: seeded integer value noise
// (the benchmark configurations) and Perlin gradient noise as the paper uses, with the values of
// integer arithmetic; either way every cell is a pure integer function of (seed, env, episode).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "noise_fields.hpp"

namespace cx {

constexpr int LAT16_N = 25;   // 5x5 lattice points at spacing 16
constexpr int LAT8_N = 81;    // 9x9 lattice points at spacing 8
constexpr int LAT_TOTAL = 2 * LAT16_N + 4 * LAT8_N;   // 374 u16 values
constexpr int LAT_BLOCKS = (LAT_TOTAL + 7) / 8;       // Philox blocks holding them (8 u16 each)
constexpr int LAT_N = LAT_BLOCKS * 8;

// terrain thresholds on 0..65535 scales
constexpr int TH_MOUNTAIN = 39500, TH_CAVE_M = 41000, TH_CAVE_C = 43000;
constexpr int TH_LAVA_M = 43000, TH_LAVA_F = 44000, TH_DIAMOND_M = 42000;
constexpr int U_DIAMOND = 500, U_IRON = 3000, TH_IRON_F = 33000, U_COAL = 8000;
constexpr int TH_WATER = 39500, TH_SAND = 37800, TH_FOREST_F = 33500;
constexpr int U_TREE_FOREST = 26000, U_TREE_SPARSE = 1300;

// The generators below are bound by instruction issue (a 64x64 world is 4 KB of stores).  Most vector
// instructions cost their SIMD four cycles: compares, byte permutations, additions with carry, dot products,
// integer products, everything in 64 bits.  32-bit floating-point additions, products and multiply-adds cost
// two, and issue beside one of the others from another wavefront: alternating with a compare or a permutation
// both together take 4.6 to 5.6 cycles.  The scalar unit takes one instruction per SIMD in four.  So:
//  - fields are evaluated in 32-bit floating point, rounded towards minus infinity, with the floors and comparisons
//    of integers (noise_fields.hpp);
//  - the thresholds stay in scalar registers;
//  - the rule's masks are combined on the scalar unit to a code of five bits, each shifted into the run's
//    word by one add with carry, and one byte permutation looks up the blocks of four cells.
// Measured against the same with fields in 64 bits (two to three times the cycles for a field), and that against
// 24-bit integer products: craftax_reset of 16,384 environments (32,768 worlds, 134 MB) 262 -> 224 -> 200 us, with
// Perlin noise 669 -> 435 -> 291.  Sign bits in place of masks (a subtraction per comparison, bit operations on
// vector registers) took 276 us and selects in place of the code of five bits 227, both with the fields in 64 bits.

// f(7) .. f(0), the cells of a run from right to left, with the number as a compile-time constant
template <typename F>
__device__ __forceinline__ void for_run(F&& f)
{
    f(std::integral_constant<int, 7>()); f(std::integral_constant<int, 6>()); f(std::integral_constant<int, 5>()); f(std::integral_constant<int, 4>());
    f(std::integral_constant<int, 3>()); f(std::integral_constant<int, 2>()); f(std::integral_constant<int, 1>()); f(std::integral_constant<int, 0>());
}
// a constant in a scalar register, from where any vector instruction takes it as it is
template <uint32_t V>
__device__ __forceinline__ uint32_t scalar_const() { uint32_t s; asm("s_mov_b32 %0, %1" : "=s"(s) : "i"(V)); return s; }
// which ? A : B, which: all ones or zero, a scalar or by lane
template <uint32_t A, uint32_t B>
__device__ __forceinline__ float pick(uint32_t which) { return __uint_as_float(B ^ (which & (A ^ B))); }

// Computes a value here and now: left alone, the scheduler has the fields of a whole run under way at
// once and spills them.
template <typename T>
__device__ __forceinline__ void settle(T& v) { asm volatile("" : "+v"(v)); }
// Sets the rounding of 32-bit floating point to "towards minus infinity" for what depends on `first`, and
// back to nearest behind what every one of `last` depends on and what has been stored before.  Everything that these kernels compute in
// floating point outside depends on memory that is read outside; the machine's own instruction keeps the rest in its place
// (no floating-point instruction is scheduled across a change of the mode register).
constexpr int MODE_ROUND_32 = 1 | (0 << 6) | ((2 - 1) << 11);   // bits 0 and 1 of the mode register
__device__ inline void floor_rounding(int& first)
{
    __builtin_amdgcn_s_setreg(MODE_ROUND_32, 2u);
    asm volatile("" : "+v"(first));
}
template <typename... Words>
__device__ inline void nearest_rounding(Words&... last)
{
    (settle(last), ...);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_setreg(MODE_ROUND_32, 0u);
}
// one bit per lane
typedef uint64_t Mask;
__device__ __forceinline__ Mask mask_of(bool b) { return __builtin_amdgcn_ballot_w64(b); }
// 2 * word + the calling lane's bit of a mask: of m, of a | b, of a & ~b.  The addition takes the mask from
// a scalar instruction in the same statement.  Straight from a vector instruction (a compare, or the
// v_readlane that brings a spilled mask back) it would read it two wait states too early, and nobody
// else sees to that around inline assembly; a scalar instruction waits for it by itself.
__device__ __forceinline__ void shift_in(uint32_t& word, Mask m)
{
    Mask t;
    asm("s_mov_b64 %1, %2\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(word), "=s"(t) : "s"(m) : "vcc");
}
__device__ __forceinline__ void shift_in_or(uint32_t& word, Mask a, Mask b)
{
    Mask t;
    asm("s_or_b64 %1, %2, %3\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(word), "=s"(t) : "s"(a), "s"(b) : "vcc", "scc");
}
__device__ __forceinline__ void shift_in_andn(uint32_t& word, Mask a, Mask b)
{
    Mask t;
    asm("s_andn2_b64 %1, %2, %3\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(word), "=s"(t) : "s"(a), "s"(b) : "vcc", "scc");
}
__host__ __device__ constexpr uint32_t four_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return a | (b << 8) | (c << 16) | (d << 24); }
// The thresholds in scalar registers (an instruction that writes a mask takes no literal), moved there once
// for a run.
template <bool PERLIN>
struct Thresholds {
    static constexpr uint32_t draw(int t) { return (uint32_t)t << 16; }
    template <int T> __device__ static float mix() { return __uint_as_float(scalar_const<f32_bits(first_mix_above<PERLIN>(T))>()); }
    template <int T> __device__ static float field() { return __uint_as_float(scalar_const<f32_bits(first_above<PERLIN>(T))>()); }
    float sand = mix<TH_SAND>(), water = mix<TH_WATER>(), mountain = mix<TH_MOUNTAIN>(), cave_m = mix<TH_CAVE_M>(), lava_m = mix<TH_LAVA_M>(),
          diamond_m = mix<TH_DIAMOND_M>(), forest_f = field<TH_FOREST_F>(), iron_f = field<TH_IRON_F - 1>(), lava_f = field<TH_LAVA_F>(),
          cave_c = field<TH_CAVE_C>();
    uint32_t diamond = scalar_const<draw(U_DIAMOND)>(), iron = scalar_const<draw(U_IRON)>(), coal = scalar_const<draw(U_COAL)>(),
             sparse = scalar_const<draw(U_TREE_SPARSE)>(), forest = scalar_const<draw(U_TREE_FOREST)>(), tunnel = scalar_const<Tunnel<PERLIN>::WIDTH>();
};

// The overworld's rule for one cell: appends five bits to `word`, where a cell takes a byte.  w, m: the
// water and mountain fields (a mix of two noises, see mix31), lowered near the start; C, F: cave and
// forest field; u: the cell's draw in the upper half (what lies in the lower half does not matter).
// In order of precedence: path, lava, diamond, iron, coal, stone on rock; water, sand, tree, grass elsewhere.
// The bits: plain kind (2: 0 grass, 1 tree, 2 sand, 3 water), rock kind (3: 0 no rock, 1 stone, 2 coal,
// 3 iron, 4 lava, 5 diamond, 6 and 7 path).  No branches: 64 rows of the world nearly always hold some
// mountain, so a branch around the mountain rules would save nothing.
template <bool PERLIN>
__device__ __forceinline__ void classify(uint32_t& word, const Thresholds<PERLIN>& t, float w, float m, float C, float F, uint32_t u)
{
    const Mask shore = mask_of(w >= t.sand), rock = mask_of(m >= t.mountain), u500 = mask_of(u < t.diamond), u3000 = mask_of(u < t.iron);
    const Mask tree = mask_of(u < t.sparse) | (mask_of(F >= t.forest_f) & mask_of(u < t.forest));
    const Mask tunnel = mask_of(__float_as_uint(C) - Tunnel<PERLIN>::FIRST < t.tunnel);
    const Mask path = (mask_of(m >= t.cave_m) & mask_of(C >= t.cave_c)) | (tunnel & rock);
    const Mask lava = mask_of(m >= t.lava_m) & mask_of(F >= t.lava_f), gem = lava | (mask_of(m >= t.diamond_m) & u500);
    const Mask coal = mask_of(u < t.coal) & ~u3000, iron = u3000 & ~(u500 | mask_of(F >= t.iron_f));
    word <<= 3;
    shift_in(word, shore);
    shift_in_or(word, mask_of(w >= t.water), tree & ~shore);
    shift_in_or(word, gem, path);
    shift_in_or(word, path, (coal | iron) & rock & ~gem);
    shift_in_andn(word, rock, coal | lava);
}
// four cells, the first in the lowest byte
__device__ inline uint32_t blocks_of(uint32_t word)
{
    const uint32_t rock = word & 0x07070707u, plain = (word >> 3) & 0x03030303u;
    const uint32_t on_rock = __builtin_amdgcn_perm(four_bytes(BK_LAVA, BK_DIAMOND, BK_PATH, BK_PATH), four_bytes(0, BK_STONE, BK_COAL, BK_IRON), rock);
    const uint32_t no_rock = __builtin_amdgcn_perm(0u, 0xFFu, rock), elsewhere = __builtin_amdgcn_perm(0u, four_bytes(BK_GRASS, BK_TREE, BK_SAND, BK_WATER), plain);
    return on_rock | (elsewhere & no_rock);
}
static_assert(TH_MOUNTAIN < TH_CAVE_M && TH_CAVE_M < TH_DIAMOND_M && TH_DIAMOND_M < TH_LAVA_M, "the mountain thresholds imply rock");

// dwords of the lattices in LDS
template <bool PERLIN>
constexpr int lattice_words = (PERLIN ? 2 : 1) * LAT_N;
constexpr int LAT_WORDS = lattice_words<true>;

// Generates the map of one environment, or a part of it, with the NT threads of the calling block.
// A wavefront owns a strip of 8 columns and all 64 rows, a lane the 8 cells of one row: one
// spacing-8 lattice cell wide (and inside one spacing-16 cell), and the per-cell uniforms are
// exactly Philox block (row * 8 + strip) of stream 1.  The horizontal weights are then constants,
// or the same for the whole wavefront.  NT / 64 strips from first_strip on: a whole world with 512
// threads, half of one with 256 (a world may be split over several blocks).
// s_lat: LDS scratch of lattice_words<PERLIN> dwords.  Ends with a block barrier, after which the cells are
// visible to the whole block.
// start_win (may be null): LDS window (9 rows x 4 dwords) of the start position (32, 32); the
// threads that own those cells drop them there, so the first observation of the new episode
// can be rendered without reading the map back.
// PERLIN: the fields are Perlin noise over the same lattices (perlin_cs: the gradient table).
// SPLIT: the run's code once with and once without what a strip near the start needs, and the world's
// identity in scalar registers, where the kernel has the registers for it.  Steps with four lanes carry the code
// once (in two copies: spills, a step of 65,536 environments 43.0 -> 45.3 us), and rollouts (see generate_half).
// theta (with PERLIN; may be null; LDS or global, LAT_TOTAL values): angle offsets of a mutated level
// (section "Craftax-1B: UED"): every gradient angle, the upper ten bits of its lattice number, is
// turned by theta[i] 1024ths of a turn.
constexpr int WG_THREADS = 512, STRIPS = MAPW / 8;
template <int NT = WG_THREADS, bool PERLIN = false, bool SPLIT = true>
__device__ __forceinline__ void worldgen_block(uint8_t* __restrict__ map, uint32_t* s_lat, uint32_t seed_lo, uint32_t seed_hi,
                                      uint32_t env, uint32_t episode, uint32_t* start_win = nullptr, int first_strip = 0,
                                      const uint32_t* __restrict__ perlin_cs = nullptr, const uint16_t* theta = nullptr)
{
    static_assert(WG_THREADS % NT == 0 && NT >= 64, "block size must divide 512");
    const int tid = threadIdx.x;
    if (SPLIT) {
        env = __builtin_amdgcn_readfirstlane(env); episode = __builtin_amdgcn_readfirstlane(episode);
        seed_lo = __builtin_amdgcn_readfirstlane(seed_lo); seed_hi = __builtin_amdgcn_readfirstlane(seed_hi);
    }
    float* lat = reinterpret_cast<float*>(s_lat);
    if (tid < LAT_BLOCKS) {
        const U4 r = philox4x32_10(env, 0u, episode, (DOM_WORLDGEN << 16) | (uint32_t)tid, seed_lo, seed_hi);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = tid * 8 + j;
            uint32_t v = (j & 1) ? (r.w[j >> 1] >> 16) : (r.w[j >> 1] & 0xFFFFu);
            if (PERLIN) {
                if (theta != nullptr && i < LAT_TOTAL) v = (v + ((theta[i] & 1023u) << 6)) & 0xFFFFu;
                const uint32_t cs = perlin_cs[v >> 6];
                lat[CX_IDX(i, lattice_words<PERLIN>)] = (float)(int)(int16_t)(cs & 0xFFFFu);
                lat[CX_IDX(LAT_N + i, lattice_words<PERLIN>)] = (float)((int)cs >> 16);
            } else lat[CX_IDX(i, lattice_words<PERLIN>)] = (float)v;
        }
    }
    __syncthreads();
    {
    if (SPLIT) asm("" : "+s"(seed_lo), "+s"(seed_hi));     // or the key schedule of the branch above is kept for here, in vector registers
    int y = tid & 63;
    floor_rounding(y);
    const int strip = first_strip + __builtin_amdgcn_readfirstlane(tid >> 6), x0 = strip * 8;
    const U4 r = philox4x32_10(env, 1u, episode, (DOM_WORLDGEN << 16) | (uint32_t)(y * STRIPS + strip), seed_lo, seed_hi);
    // the points above and left of the run in the two lattices of spacing 16 and the four of spacing 8
    const float* w16 = lat + CX_IDX((y >> 4) * 5 + (x0 >> 4), LAT16_N - 6);
    const float* m16 = w16 + LAT16_N;
    const float* w8 = lat + 2 * LAT16_N + CX_IDX((y >> 3) * 9 + strip, LAT8_N - 10);
    const float* m8 = w8 + LAT8_N;
    const float* c8 = m8 + LAT8_N;
    const float* f8 = c8 + LAT8_N;
    const uint32_t odd = 0u - (uint32_t)(strip & 1);   // all ones: right half of a spacing-16 lattice cell
    // 4 times the lowering (10 - d) * 2500 of W and M within Chebyshev distance d < 10 of the start: by
    // rows here, by columns below, and the smaller of the two counts
    const bool near_strip = x0 + 7 > MAPW / 2 - START_BIAS_R && x0 < MAPW / 2 + START_BIAS_R;
    const int bias_y = max(0, START_BIAS_R - iabs(y - MAPW / 2)) * (4 * START_BIAS);
    uint32_t word = 0u, four = 0u;                     // the cells under way, the finished cells 4..7
    const Thresholds<PERLIN> thresholds;
    auto draw = [&](auto j) { return (j & 1) ? r.w[j >> 1] : r.w[j >> 1] << 16; };   // draw of cell j, in the upper half
    auto put = [&](auto near, int j, uint32_t u, float W4, float M4, float C, float F) {
        if (near) near_start(min(bias_y, max(0, START_BIAS_R - iabs(x0 + j - MAPW / 2)) * (4 * START_BIAS)), W4, M4, u);
        classify<PERLIN>(word, thresholds, W4, M4, C, F, u);
        if (PERLIN) settle(word);
    };
    // the run's code with and without what only a strip near the start needs
    auto by_strip = [&](auto&& cells) { if (!SPLIT || near_strip) cells(std::true_type()); else cells(std::false_type()); };
    if (PERLIN) {
        const int ky16 = y & 15, ky8 = y & 7;
        const float wy16 = (float)perlin_fade<16>(ky16) * (1.0f / 65536.0f), wy8 = (float)perlin_fade<8>(ky8) * (1.0f / 65536.0f);
        // One field after the other for the whole run; the last one with the rule.
        // The empty statement keeps the loads of a field's gradients from being moved before the field at hand.
        auto along = [&](PerlinLine line, auto&& weight, float wy, auto&& cell) {
            for_run([&](auto j) { cell(j, line.field(weight(j), wy)); line.advance(); });
            asm volatile("" ::: "memory");
        };
        auto wide = [&](const float* at) { return perlin_line<16>(at, at + LAT_N, 5, (float)((x0 & 15) + 7), (float)ky16); };
        auto narrow = [&](const float* at) { return perlin_line<8>(at, at + LAT_N, 9, 7.0f, (float)ky8); };
        auto wx16 = [&](auto j) { return pick<f32_bits(perlin_weight<16>(8 + j)), f32_bits(perlin_weight<16>(j))>(odd); };
        auto wx8 = [&](auto j) { return perlin_weight<8>(j); };
        float W4[8], M4[8], C[8];
        const PerlinScale<16> coarse;
        const PerlinScale<8> fine;
        along(wide(w16), wx16, wy16, [&](int j, float v) { W4[j] = coarse.value(v); settle(W4[j]); });
        along(narrow(w8), wx8, wy8, [&](int j, float v) { W4[j] = perlin_mix31(W4[j], fine.value(v)); settle(W4[j]); });
        along(wide(m16), wx16, wy16, [&](int j, float v) { M4[j] = coarse.value(v); settle(M4[j]); });
        along(narrow(m8), wx8, wy8, [&](int j, float v) { M4[j] = perlin_mix31(M4[j], fine.value(v)); settle(M4[j]); });
        along(narrow(c8), wx8, wy8, [&](int j, float v) { C[j] = v; settle(C[j]); });
        const PerlinLine forest = narrow(f8);
        by_strip([&](auto near) {
            along(forest, wx8, wy8, [&](auto j, float v) {
                put(near, j, draw(j), W4[j], M4[j], C[j], v);
                if (j == 4) four = word;                       // (the next four cells shift it out)
            });
        });
    } else {
        const float wy16 = (float)smooth16(y & 15) * (1.0f / 256.0f), wy8 = (float)smooth8(y & 7) * (1.0f / 256.0f);
        const Line W16 = line_at(w16, 5, wy16), M16 = line_at(m16, 5, wy16);
        const Line W8 = line_at(w8, 9, wy8), M8 = line_at(m8, 9, wy8), C8 = line_at(c8, 9, wy8), F8 = line_at(f8, 9, wy8);
        by_strip([&](auto near) {
            for_run([&](auto j) {
                const float wx16 = pick<f32_bits(weight16(8 + j)), f32_bits(weight16(j))>(odd);
                constexpr float wx8 = weight8(j);
                put(near, j, draw(j), mix31(W16.at(wx16), W8.at(wx8)), mix31(M16.at(wx16), M8.at(wx8)), C8.at(wx8), F8.at(wx8));
                if (j == 4) { four = word; word = 0u; }        // the other four cells do not wait for these
            });
        });
    }
    nearest_rounding(word, four);
    const uint32_t first = blocks_of(word);
    four = blocks_of(four);
    *reinterpret_cast<uint2*>(map + map_index(x0, y)) = make_uint2(first, four);   // 8 cells inside one tile row
    {
        // window of the start cell: rows 28..36, columns 24..39 (aligned start of 32-5)
        constexpr int WY0 = MAPW / 2 - WIN_ROWS / 2, WX0 = (MAPW / 2 - WIN_COLS / 2) & ~3;
        const int wr = y - WY0, wc = x0 - WX0;
        if (start_win != nullptr && (unsigned)wr < (unsigned)WIN_ROWS && (unsigned)wc < (unsigned)WIN_PITCH) {
            start_win[CX_IDX(wr * (WIN_PITCH / 4) + wc / 4, WIN_DWORDS)] = first;
            start_win[CX_IDX(wr * (WIN_PITCH / 4) + wc / 4 + 1, WIN_DWORDS)] = four;
        }
    }
    }
    __syncthreads();
}

// Word i of a fresh record: full vitals, empty tables, player in the middle facing down.
__device__ inline uint32_t fresh_record_word(int i, uint32_t seed_lo, uint32_t seed_hi, uint32_t episode)
{
    switch (i) {
    case RW_POS: return (uint32_t)(MAPW / 2) | ((uint32_t)(MAPW / 2) << 8) | (4u << 16);
    case RW_VIT: return (uint32_t)MAX_COUNT * 0x1111u;
    case RW_EPISODE: return episode;
    case RW_SEED_LO: return seed_lo;
    case RW_SEED_HI: return seed_hi;
    default: return 0u;
    }
}

}  // namespace cx
