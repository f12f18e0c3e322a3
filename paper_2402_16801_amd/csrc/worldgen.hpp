// Block-cooperative generation of one 64x64 Craftax-Classic world (appendix "World
// Generation" of the paper: noise thresholds carve grassland, forest, lakes, mountains with
// caves, tunnels, ores and lava).  Two noises feed the same rule: seeded integer value noise
// (the benchmark configurations) and Perlin gradient noise as the paper uses, evaluated in
// integers; either way every cell is a pure integer function of (seed, env, episode).
#pragma once

#include "common.hpp"

namespace cx {

constexpr int LAT16_N = 25;   // 5x5 lattice points at spacing 16
constexpr int LAT8_N = 81;    // 9x9 lattice points at spacing 8
constexpr int LAT_TOTAL = 2 * LAT16_N + 4 * LAT8_N;   // 374 u16 values
constexpr int LAT_BLOCKS = (LAT_TOTAL + 7) / 8;       // Philox blocks holding them (8 u16 each)

// terrain thresholds on 0..65535 scales
constexpr int TH_MOUNTAIN = 39500, TH_CAVE_M = 41000, TH_CAVE_C = 43000;
constexpr int TH_TUNNEL_CENTER = 30000, TH_TUNNEL_HALF = 1300;
constexpr int TH_LAVA_M = 43000, TH_LAVA_F = 44000, TH_DIAMOND_M = 42000;
constexpr int U_DIAMOND = 500, U_IRON = 3000, TH_IRON_F = 33000, U_COAL = 8000;
constexpr int TH_WATER = 39500, TH_SAND = 37800, TH_FOREST_F = 33500;
constexpr int U_TREE_FOREST = 26000, U_TREE_SPARSE = 1300;
constexpr int START_CLEAR = 2, START_BIAS_R = 10, START_BIAS = 2500;

// smoothstep(k/S) in 1/256 units for S = 8 and S = 16
__host__ __device__ constexpr uint32_t smooth8(int k) { return (uint32_t)(12 * k * k - k * k * k); }
__host__ __device__ constexpr uint32_t smooth16(int k) { return (uint32_t)((24 * k * k - k * k * k + 4) >> 3); }

// The generators below are bound by vector instruction issue (a 64x64 world is 4 KB of stores against
// 589 instructions for every 64 runs of 8 cells), so they are written for few instructions:
// every product is one that a 24-bit multiply or a 16-bit dot product forms exactly, fields are
// compared with their thresholds before the shift that would bring them to the 0..65535 scale, and
// the rule is compares and selects whose masks combine on the scalar unit.  Measured against a
// generator of 32-bit products and a branching rule: craftax_reset of 16,384 environments (32,768
// worlds, 134 MB) 412 -> 263 us, of 8,192 with Perlin noise (which was in 64-bit integers) 455 -> 338.

// exact products of values below 2^24 (one v_mul_u32_u24 / v_mad_u32_u24)
__device__ inline uint32_t mul24u(uint32_t a, uint32_t b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }
// a.lo * b.lo + a.hi * b.hi over 16-bit halves, unsigned and signed
__device__ inline uint32_t dot16u(uint32_t a, uint32_t b)
{
    typedef unsigned short pair_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_udot2(__builtin_bit_cast(pair_t, a), __builtin_bit_cast(pair_t, b), 0u, false);
}
__device__ inline int dot16s(uint32_t a, uint32_t b)
{
    typedef short pair_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(pair_t, a), __builtin_bit_cast(pair_t, b), 0, false);
}

// Bilinear value noise, evaluated column-first: two lattice rows are blended once per lattice
// column (vertical weight wy), then every cell of a run blends two columns (horizontal weight wx).
// The integer result equals the row-first formula
// ((a(256-wx)+b wx)(256-wy) + (c(256-wx)+d wx) wy) >> 16 because nothing is rounded before
// the final shift and every intermediate fits in 32 bits (a blended column in 24).
// A lattice lies in LDS as one dword per point: the point itself in the low half, the point below
// it in the high half, so that a column is one dot product.
__device__ inline uint32_t vertical_weights(uint32_t wy) { return (256u - wy) | (wy << 16); }
// 2^16 times the field
__device__ inline uint32_t across(uint32_t left, uint32_t right, uint32_t wx) { return mul24u(left, 256u - wx) + mul24u(right, wx); }
// 4 times the mix (3 coarse + fine) / 4 of two fields given as 2^16 times their values
__device__ inline int mix31(uint32_t coarse, uint32_t fine)
{
    return (int)dot16u(__builtin_amdgcn_perm(coarse, fine, 0x07060302u), 1u | (3u << 16));   // (fine, coarse) as halves
}

// Perlin gradient noise (appendix "World Generation"): the lattice numbers are read as one of 1024
// directions (top ten bits); cs[a] holds the unit gradient of direction a in Q14.  S is the
// lattice spacing; offsets from the four corners are in units of 1/S; the fade weight
// 6t^5 - 15t^4 + 10t^3 of t = k/S is (F 65536 + S^5 / 2) / S^5 in Q16 with
// F = k^3 (6 k^2 - 15 k S + 10 S^2); blends are p + floor((q - p) w / 65536), along x then y; the
// value, in units of 1 / (16384 S), lands on the 0..65535 scale of the thresholds as
// 32768 + floor(n * 3900 / (1024 S)), clamped.  All divisors are powers of two: floors are shifts.
// A dot product is at most 16385 sqrt(2) S < 2^18.6, a blend lies between its ends and a weight is
// below 2^16, so 24-bit products are exact and n * 3900 fits 32 bits.
// A lattice lies in LDS as one gradient (cos | sin << 16) per point.
constexpr int PERLIN_GAIN = 3900;
template <int S>
__host__ __device__ constexpr int perlin_fade(int k)
{
    const int F = k * k * k * (6 * k * k - 15 * k * S + 10 * S * S);
    return S == 16 ? (F + 8) >> 4 : 2 * F;
}
__device__ inline int perlin_blend(int p, int q, int w)
{
    const int d = q - p;
    return p + (int)(((int64_t)((d << 8) >> 8) * (int64_t)(w & 0xFFFF)) >> 16);
}
// the four gradients around a run, which lies inside one lattice cell
struct Gradients { uint32_t g[2][2]; };
__device__ inline Gradients gradients_at(const uint32_t* lat, int width, int ix, int iy)
{
    Gradients r;
#pragma unroll
    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) r.g[cy][cx] = lat[CX_IDX((iy + cy) * width + ix + cx, width * width)];
    return r;
}
// n of the cell at offset (kx, ky) from the upper left corner
template <int S>
__device__ inline int perlin_n(const Gradients& r, int kx, int ky, int wx, int wy)
{
    const uint32_t x0 = (uint32_t)kx & 0xFFFFu, x1 = (uint32_t)(kx - S) & 0xFFFFu, y0 = (uint32_t)ky << 16, y1 = (uint32_t)(ky - S) << 16;
    return perlin_blend(perlin_blend(dot16s(r.g[0][0], x0 | y0), dot16s(r.g[0][1], x1 | y0), wx),
                        perlin_blend(dot16s(r.g[1][0], x0 | y1), dot16s(r.g[1][1], x1 | y1), wx), wy);
}
template <int S>
__device__ inline int perlin_value(int n)
{
    const int v = 32768 + ((n * PERLIN_GAIN) >> (S == 16 ? 14 : 13));
    return v < 0 ? 0 : (v > 65535 ? 65535 : v);
}

// A field of spacing 8 as the rule compares it: 2^16 times the value (value noise) or n (Perlin
// noise); field > t and t0 < field < t1 without the steps that lead to the 0..65535 scale.
constexpr int perlin_above(int t)      // smallest n whose value exceeds t: n * GAIN >= (t + 1 - 32768) * 2^13
{
    const long long num = (long long)(t + 1 - 32768) * 8192, q = num / PERLIN_GAIN;
    return (int)(q + (q * PERLIN_GAIN < num ? 1 : 0));
}
template <bool PERLIN>
__device__ inline bool above(uint32_t field, int t)
{
    return PERLIN ? (int)field >= perlin_above(t) : field >= (uint32_t)(t + 1) << 16;
}
template <bool PERLIN>
__device__ inline bool between(uint32_t field, int t0, int t1)
{
    return PERLIN ? ((int)field >= perlin_above(t0)) & ((int)field < perlin_above(t1 - 1)) : field - ((uint32_t)(t0 + 1) << 16) < (uint32_t)(t1 - 1 - t0) << 16;
}
static_assert(perlin_above(32767) == 0 && perlin_above(32768) == 3 && perlin_above(32766) == -2, "floor(n * 3900 / 8192) first exceeds 0 at n = 3, -1 at 0, -2 at -2");

// The overworld's rule for one cell.  w, m: 4 times the water and mountain fields (a mix of two
// noises, see mix31), lowered near the start; C, F: cave and forest field as `above` takes them; u:
// the cell's draw in the upper half (what lies in the lower half does not matter).  x >> 2 > t is
// compared as x > 4t + 3.  The order of precedence is the order of the written-out rule read from the end.
// Compares and selects only: 64 rows of the world nearly always hold some mountain, so a branch
// around the mountain rules would save nothing, and the masks are combined by the scalar unit.
template <bool PERLIN>
__device__ __forceinline__ int classify(int w, int m, uint32_t C, uint32_t F, uint32_t u)
{
    constexpr auto over = [](int t) { return 4 * t + 3; };
    const bool u500 = u < ((uint32_t)U_DIAMOND << 16), u3000 = u < ((uint32_t)U_IRON << 16), u8000 = u < ((uint32_t)U_COAL << 16);
    int b = BK_GRASS;
    auto set = [&](bool where, int block) { b = where ? block : b; };
    set((u < ((uint32_t)U_TREE_SPARSE << 16)) | (above<PERLIN>(F, TH_FOREST_F) & (u < ((uint32_t)U_TREE_FOREST << 16))), BK_TREE);
    set(w > over(TH_SAND), BK_SAND);
    set(w > over(TH_WATER), BK_WATER);
    const bool rock = m > over(TH_MOUNTAIN);
    set(rock, BK_STONE);
    set(rock & u8000 & !u3000, BK_COAL);
    set(rock & u3000 & !u500 & !above<PERLIN>(F, TH_IRON_F - 1), BK_IRON);
    set((m > over(TH_DIAMOND_M)) & u500, BK_DIAMOND);
    set((m > over(TH_LAVA_M)) & above<PERLIN>(F, TH_LAVA_F), BK_LAVA);
    const bool cave = (m > over(TH_CAVE_M)) & above<PERLIN>(C, TH_CAVE_C);
    set(cave | (rock & between<PERLIN>(C, TH_TUNNEL_CENTER - TH_TUNNEL_HALF, TH_TUNNEL_CENTER + TH_TUNNEL_HALF)), BK_PATH);
    return b;
}
static_assert(TH_MOUNTAIN < TH_CAVE_M && TH_CAVE_M < TH_DIAMOND_M && TH_DIAMOND_M < TH_LAVA_M, "the mountain thresholds imply rock");

// Where lattice number i of the stream lies in LDS (dwords) and how far above the point over it: two
// 5x5 lattices, then four 9x9.  The gaps in front of both groups take the high halves that the first
// row of a group would leave above itself; between lattices of one group they fall into the last row
// of the previous one, whose high halves nobody reads.
constexpr int LAT_PAD16 = 5, LAT_PAD8 = 9;
constexpr int LAT_AT16 = LAT_PAD16, LAT_AT8 = LAT_PAD16 + 2 * LAT16_N + LAT_PAD8;
constexpr int LAT_WORDS = LAT_AT8 + (LAT_BLOCKS * 8 - 2 * LAT16_N) + 2;

// Generates the map of one environment, or a part of it, with the NT threads of the calling block.
// A wavefront owns a strip of 8 columns and all 64 rows, a lane the 8 cells of one row: one
// spacing-8 lattice cell wide (and inside one spacing-16 cell), and the per-cell uniforms are
// exactly Philox block (row * 8 + strip) of stream 1.  The horizontal weights are then constants,
// or the same for the whole wavefront.  NT / 64 strips from first_strip on: a whole world with 512
// threads, half of one with 256 (a world may be split over several blocks).
// s_lat: LDS scratch of LAT_WORDS dwords.  Ends with a block barrier, after which the cells are
// visible to the whole block.
// start_win (may be null): LDS window (9 rows x 4 dwords) of the start position (32, 32); the
// threads that own those cells drop them there, so the first observation of the new episode
// can be rendered without reading the map back.
// PERLIN: the fields are Perlin noise over the same lattices (perlin_cs: the gradient table).
// theta (with PERLIN; may be null; LDS or global, LAT_TOTAL values): angle offsets of a mutated level
// (section "Craftax-1B: UED"): every gradient angle, the upper ten bits of its lattice number, is
// turned by theta[i] 1024ths of a turn.
constexpr int WG_THREADS = 512, STRIPS = MAPW / 8;
template <int NT = WG_THREADS, bool PERLIN = false, bool UNROLLED = false>
__device__ __forceinline__ void worldgen_block(uint8_t* __restrict__ map, uint32_t* s_lat, uint32_t seed_lo, uint32_t seed_hi,
                                      uint32_t env, uint32_t episode, uint32_t* start_win = nullptr, int first_strip = 0,
                                      const uint32_t* __restrict__ perlin_cs = nullptr, const uint16_t* theta = nullptr)
{
    static_assert(WG_THREADS % NT == 0 && NT >= 64, "block size must divide 512");
    const int tid = threadIdx.x;
    if (tid < LAT_BLOCKS) {
        const U4 r = philox4x32_10(env, 0u, episode, (DOM_WORLDGEN << 16) | (uint32_t)tid, seed_lo, seed_hi);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = tid * 8 + j;
            uint32_t v = (j & 1) ? (r.w[j >> 1] >> 16) : (r.w[j >> 1] & 0xFFFFu);
            const bool wide = i < 2 * LAT16_N;
            const int at = i + (wide ? LAT_AT16 : LAT_AT8 - 2 * LAT16_N);
            if (PERLIN) {
                if (theta != nullptr && i < LAT_TOTAL) v = (v + ((theta[i] & 1023u) << 6)) & 0xFFFFu;
                s_lat[CX_IDX(at, LAT_WORDS)] = perlin_cs[v >> 6];
            } else {
                uint16_t* half = reinterpret_cast<uint16_t*>(s_lat);
                half[CX_IDX(2 * at, 2 * LAT_WORDS)] = (uint16_t)v;
                half[CX_IDX(2 * (at - (wide ? 5 : 9)) + 1, 2 * LAT_WORDS)] = (uint16_t)v;
            }
        }
    }
    __syncthreads();
    {
    const int strip = first_strip + __builtin_amdgcn_readfirstlane(tid >> 6), y = tid & 63, x0 = strip * 8;
    const U4 r = philox4x32_10(env, 1u, episode, (DOM_WORLDGEN << 16) | (uint32_t)(y * STRIPS + strip), seed_lo, seed_hi);
    const uint32_t* w16 = s_lat + LAT_AT16;
    const uint32_t* m16 = w16 + LAT16_N;
    const uint32_t* w8 = s_lat + LAT_AT8;
    const uint32_t* m8 = w8 + LAT8_N;
    const uint32_t* c8 = m8 + LAT8_N;
    const uint32_t* f8 = c8 + LAT8_N;
    const int iy16 = y >> 4, iy8 = y >> 3, ix16 = x0 >> 4, ix8 = strip, odd8 = x0 & 8;
    // 4 times the lowering (10 - d) * 2500 of W and M within Chebyshev distance d < 10 of the start: by
    // rows here, by columns below, and the smaller of the two counts
    const bool near_strip = x0 + 7 > MAPW / 2 - START_BIAS_R && x0 < MAPW / 2 + START_BIAS_R;
    const int bias_y = max(0, START_BIAS_R - iabs(y - MAPW / 2)) * (4 * START_BIAS);
    uint32_t first = 0u, four = 0u, draw_a = r.w[0], draw_b = r.w[1];   // finished cells 0..3; the cells and draws of the half at hand
    auto put = [&](int j, int W4, int M4, uint32_t C, uint32_t F) {
        const uint32_t pair = (j & 2) ? draw_b : draw_a, u = (j & 1) ? pair : (pair << 16);
        const int bias = min(bias_y, max(0, START_BIAS_R - iabs(x0 + j - MAPW / 2)) * (4 * START_BIAS));
        if (near_strip) { W4 -= bias; M4 -= bias; }
        int b = classify<PERLIN>(W4, M4, C, F, u);
        if (near_strip) b = bias >= (START_BIAS_R - START_CLEAR) * (4 * START_BIAS) ? (int)BK_GRASS : b;
        four |= (uint32_t)b << (8 * (j & 3));
    };
    // The run in two halves of four cells, a loop that is not unrolled: half the code, and few enough
    // registers for the kernels that hold an environment's record meanwhile.  UNROLLED: for blocks that
    // generate one world after the other and last as long as the chain of a run (regeneration_block).
    constexpr int HALVES_UNROLL = UNROLLED ? 2 : 1;
    auto halves = [&](auto&& cell) {
#pragma unroll HALVES_UNROLL
        for (int h = 0; h < 8; h += 4) {
            first = four;
            four = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) cell(h + j);
            draw_a = r.w[2];
            draw_b = r.w[3];
        }
    };
    if (PERLIN) {
        const Gradients gW = gradients_at(w16, 5, ix16, iy16), gM = gradients_at(m16, 5, ix16, iy16);
        const Gradients hW = gradients_at(w8, 9, ix8, iy8), hM = gradients_at(m8, 9, ix8, iy8), hC = gradients_at(c8, 9, ix8, iy8), hF = gradients_at(f8, 9, ix8, iy8);
        const int ky16 = y & 15, ky8 = y & 7, wy16 = perlin_fade<16>(ky16), wy8 = perlin_fade<8>(ky8);
        auto coarse = [&](const Gradients& g, int j, int wx) { return perlin_value<16>(perlin_n<16>(g, odd8 + j, ky16, wx, wy16)); };
        auto fine = [&](const Gradients& g, int j) { return perlin_n<8>(g, j, ky8, perlin_fade<8>(j), wy8); };
        halves([&](int j) {
            const int wx16 = perlin_fade<16>(odd8 + j);
            put(j, 3 * coarse(gW, j, wx16) + perlin_value<8>(fine(hW, j)), 3 * coarse(gM, j, wx16) + perlin_value<8>(fine(hM, j)),
                (uint32_t)fine(hC, j), (uint32_t)fine(hF, j));
        });
    } else {
        const uint32_t v16 = vertical_weights(smooth16(y & 15)), v8 = vertical_weights(smooth8(y & 7));
        struct Ends { uint32_t l, r; };
        auto ends16 = [&](const uint32_t* lat) { const uint32_t* c = lat + CX_IDX(iy16 * 5 + ix16, LAT16_N - 1); return Ends{ dot16u(c[0], v16), dot16u(c[1], v16) }; };
        auto ends8 = [&](const uint32_t* lat) { const uint32_t* c = lat + CX_IDX(iy8 * 9 + ix8, LAT8_N - 1); return Ends{ dot16u(c[0], v8), dot16u(c[1], v8) }; };
        const Ends W16 = ends16(w16), M16 = ends16(m16), W8 = ends8(w8), M8 = ends8(m8), C8 = ends8(c8), F8 = ends8(f8);
        halves([&](int j) {
            const uint32_t wx16 = smooth16(odd8 + j), wx8 = smooth8(j);
            put(j, mix31(across(W16.l, W16.r, wx16), across(W8.l, W8.r, wx8)), mix31(across(M16.l, M16.r, wx16), across(M8.l, M8.r, wx8)),
                across(C8.l, C8.r, wx8), across(F8.l, F8.r, wx8));
        });
    }
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
