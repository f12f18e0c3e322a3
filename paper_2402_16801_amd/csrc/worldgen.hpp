// Block-cooperative generation of one 64x64 Craftax-Classic world (appendix "World
// Generation" of the paper: noise thresholds carve grassland, forest, lakes, mountains with
// caves, tunnels, ores and lava).  Two noises feed the same rule: seeded integer value noise
// (the benchmark configurations) and Perlin gradient noise as the paper uses, evaluated in
// integers; either way every cell is a pure integer function of (seed, env, episode).
#pragma once

#include <type_traits>

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

// The generators below are bound by instruction issue (a 64x64 world is 4 KB of stores): nearly every
// vector instruction costs its SIMD four cycles, among them v_fma_f64, v_add_f64, compares and dot
// products, and the scalar unit takes one instruction per SIMD in the same time.  So they are written for
// few vector instructions, with fewer scalar ones beside them:
//  - fields are evaluated in 64-bit floating point, where every step below is exact and one
//    multiply-add does what takes two (value noise) to five (Perlin noise) integer instructions;
//  - fields are compared with their thresholds before the shift that would bring them to the 0..65535
//    scale, and the thresholds stay in scalar registers;
//  - the rule's masks are combined on the scalar unit to a code of five bits, each shifted into the run's
//    word by one add with carry, and one byte permutation looks up the blocks of four cells.
// Measured against 24-bit integer products, a floor per blend and a select per rule: craftax_reset of 16,384
// environments (32,768 worlds, 134 MB) 262 -> 224 us, with Perlin noise 669 -> 435.  Sign bits in place of
// masks (a subtraction per comparison, bit operations on vector registers) took 276 us, selects in place
// of the code of five bits 227.
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

// f(7) .. f(0), the cells of a run from right to left, with the number as a compile-time constant
template <typename F>
__device__ __forceinline__ void for_run(F&& f)
{
    f(std::integral_constant<int, 7>()); f(std::integral_constant<int, 6>()); f(std::integral_constant<int, 5>()); f(std::integral_constant<int, 4>());
    f(std::integral_constant<int, 3>()); f(std::integral_constant<int, 2>()); f(std::integral_constant<int, 1>()); f(std::integral_constant<int, 0>());
}
// High half of a double whose low half is zero: every weight below is a small whole number or a fraction of
// sixteen bits.  NOT_A_HALF for a value that does not fit, which the functions that put it together refuse.
constexpr uint32_t NOT_A_HALF = 0xFFFFFFFFu;
__host__ __device__ constexpr uint32_t high_half(double v)
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, v);
    return (uint32_t)bits != 0u ? NOT_A_HALF : (uint32_t)(bits >> 32);
}
static_assert(high_half(1.5) == 0x3FF80000u && high_half(1.0 / 3.0) == NOT_A_HALF, "a third has a low half");
// such a constant in scalar registers, from where a multiply-add takes it as it is
template <uint32_t V>
__device__ __forceinline__ uint32_t scalar_const() { uint32_t s; asm("s_mov_b32 %0, %1" : "=s"(s) : "i"(V)); return s; }
template <uint32_t HIGH>
__device__ __forceinline__ double scalar_double() { static_assert(HIGH != NOT_A_HALF, "a constant with a low half"); return __hiloint2double((int)scalar_const<HIGH>(), 0); }
// which ? A : B, which: all ones or zero, a scalar or by lane
template <uint32_t A, uint32_t B>
__device__ __forceinline__ uint32_t half_of(uint32_t which) { return B ^ (which & (A ^ B)); }
template <uint32_t A, uint32_t B>
__device__ __forceinline__ double pick(uint32_t which) { static_assert(A != NOT_A_HALF && B != NOT_A_HALF, "a constant with a low half"); return __hiloint2double((int)half_of<A, B>(which), 0); }

// Bilinear value noise, evaluated column-first: two lattice rows are blended once per lattice
// column (vertical weight wy), then every cell of a run blends two columns (horizontal weight wx).
// The integer result equals the row-first formula
// ((a(256-wx)+b wx)(256-wy) + (c(256-wx)+d wx) wy) >> 16 because nothing is rounded before
// the final shift and every intermediate fits in 32 bits (a blended column in 24).
// A lattice lies in LDS as one dword per point: the point itself in the low half, the point below
// it in the high half, so that a column is one dot product.
__device__ inline uint32_t vertical_weights(uint32_t wy) { return (256u - wy) | (wy << 16); }
// A field along a run: 2^16 times its value is a whole number below 2^32, kept as 2^52 + that number, so
// that the low half of the double is the number itself.  slope: what one unit of weight adds.
struct Line {
    double at, slope;
    __device__ uint32_t field() const { return (uint32_t)__double2loint(at); }
    __device__ void advance(double weight) { at = __builtin_fma(slope, weight, at); }
};
constexpr int TWO52_HI = 0x43300000;   // high half of 2^52
// left, right: the lattice columns at both ends, blended vertically; weight: that of the right one where the line starts
__device__ inline Line line_between(uint32_t left, uint32_t right, double weight)
{
    Line l{__hiloint2double(TWO52_HI, (int)(left << 8)), (double)((int)right - (int)left)};
    l.advance(weight);
    return l;
}
// the weight of a run's last cell, and from cell j to cell j - 1
constexpr double LAST8 = (double)smooth8(7), LAST16 = (double)smooth16(7), LAST16_ODD = (double)smooth16(15);
__host__ __device__ constexpr double step8(int j) { return j == 0 ? 0.0 : (double)smooth8(j - 1) - (double)smooth8(j); }
__host__ __device__ constexpr double step16(int j) { return j == 0 ? 0.0 : (double)smooth16(j - 1) - (double)smooth16(j); }
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
// below 2^16, so in 64-bit floating point every sum and product is exact, and n * 3900 fits 32 bits.
// A lattice lies in LDS as one gradient (cos | sin << 16) per point.
constexpr int PERLIN_GAIN = 3900;
template <int S>
__host__ __device__ constexpr int perlin_fade(int k)
{
    const int F = k * k * k * (6 * k * k - 15 * k * S + 10 * S * S);
    return S == 16 ? (F + 8) >> 4 : 2 * F;
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
// A Perlin field along a run.  Along a row the dot products with the four corners are linear in kx:
// top and bottom are those with the left corners, dtop and dbottom what the right ones are more, g* what
// a cell further to the right adds to each.  top and bottom carry the offset 2^52 + 2^31: a multiply-add onto them,
// rounded towards minus infinity (see floor_rounding), is then the blend with its floor in one
// instruction, and the low half of the last one is n + 2^31.
constexpr uint32_t PERLIN_BIAS = 0x80000000u;
struct PerlinLine {
    double top, dtop, bottom, dbottom, gtop, gdtop, gbottom, gdbottom;
    // weights in units of 1: fade of kx and of ky
    __device__ double field(double wx, double wy) const
    {
        const double t = __builtin_fma(dtop, wx, top), b = __builtin_fma(dbottom, wx, bottom);
        return __builtin_fma(b - t, wy, t);
    }
    __device__ void advance() { top -= gtop; dtop -= gdtop; bottom -= gbottom; dbottom -= gdbottom; }
};
// Computes a value here and now: left alone, the scheduler has the fields of a whole run under way at
// once, each in a pair of registers, and spills them.
template <typename T>
__device__ __forceinline__ void settle(T& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ uint32_t settled(double v) { uint32_t out; asm volatile("v_mov_b32 %0, %1" : "=v"(out) : "v"(__double2loint(v))); return out; }
// starts at offset (kx, ky) from the upper left corner
template <int S>
__device__ inline PerlinLine perlin_line(const Gradients& r, int kx, int ky)
{
    const uint32_t x0 = (uint32_t)kx & 0xFFFFu, x1 = (uint32_t)(kx - S) & 0xFFFFu, y0 = (uint32_t)ky << 16, y1 = (uint32_t)(ky - S) << 16;
    const int t = dot16s(r.g[0][0], x0 | y0), b = dot16s(r.g[1][0], x0 | y1);
    auto cosine = [](uint32_t g) { return (int)(int16_t)(g & 0xFFFFu); };
    PerlinLine l;
    l.top = __hiloint2double(TWO52_HI, (int)((uint32_t)t ^ PERLIN_BIAS));
    l.bottom = __hiloint2double(TWO52_HI, (int)((uint32_t)b ^ PERLIN_BIAS));
    l.dtop = (double)(dot16s(r.g[0][1], x1 | y0) - t);
    l.dbottom = (double)(dot16s(r.g[1][1], x1 | y1) - b);
    l.gtop = (double)cosine(r.g[0][0]); l.gdtop = (double)(cosine(r.g[0][1]) - cosine(r.g[0][0]));
    l.gbottom = (double)cosine(r.g[1][0]); l.gdbottom = (double)(cosine(r.g[1][1]) - cosine(r.g[1][0]));
    return l;
}
template <int S>
__host__ __device__ constexpr double perlin_weight(int k) { return perlin_fade<S>(k) * (1.0 / 65536.0); }
// Sets the rounding of 64-bit floating point to "towards minus infinity" for what depends on `first`, and
// back to nearest behind what `last` depends on.  Nothing else in these kernels computes in 64-bit
// (or 16-bit) floating point; 32-bit has a rounding mode of its own.
__device__ inline void floor_rounding(int& first) { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 2\n\ts_nop 1" : "+v"(first)); }
__device__ inline void nearest_rounding(uint32_t& last) { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0\n\ts_nop 1" : "+v"(last)); }
// the value of a field on the 0..65535 scale: onto 1.5 * 2^52, with its floor, in one multiply-add more
template <int S>
struct PerlinScale {
    static constexpr double GAIN = PERLIN_GAIN / (1024.0 * S);
    static constexpr double OFFSET = 6755399441055744.0 + 32768.0 - (4503599627370496.0 + 2147483648.0) * GAIN;
    static_assert(OFFSET == (double)(long long)OFFSET && OFFSET < 9007199254740992.0, "a whole number below 2^53");
    double gain = scalar_double<high_half(GAIN)>(), offset = OFFSET;
    __device__ int value(double field) const
    {
        const int v = __double2loint(__builtin_fma(field, gain, offset));
        return v < 0 ? 0 : (v > 65535 ? 65535 : v);
    }
};
// A field of spacing 8 as the rule compares it: 2^16 times the value (value noise) or n + 2^31 (Perlin
// noise), without the steps that lead to the 0..65535 scale.
constexpr int perlin_above(int t)      // smallest n whose value exceeds t: n * GAIN >= (t + 1 - 32768) * 2^13
{
    const long long num = (long long)(t + 1 - 32768) * 8192, q = num / PERLIN_GAIN;
    return (int)(q + (q * PERLIN_GAIN < num ? 1 : 0));
}
static_assert(perlin_above(32767) == 0 && perlin_above(32768) == 3 && perlin_above(32766) == -2, "floor(n * 3900 / 8192) first exceeds 0 at n = 3, -1 at 0, -2 at -2");
template <bool PERLIN>
__host__ __device__ constexpr uint32_t first_above(int t)      // smallest field that exceeds t
{
    return PERLIN ? (uint32_t)perlin_above(t) ^ PERLIN_BIAS : (uint32_t)(t + 1) << 16;
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
    static constexpr int TUNNEL0 = TH_TUNNEL_CENTER - TH_TUNNEL_HALF, TUNNEL1 = TH_TUNNEL_CENTER + TH_TUNNEL_HALF;
    static constexpr uint32_t mix(int t) { return (uint32_t)(4 * t + 3); }     // x >> 2 > t is x > 4t + 3
    static constexpr uint32_t draw(int t) { return (uint32_t)t << 16; }
    int sand = (int)scalar_const<mix(TH_SAND)>(), water = (int)scalar_const<mix(TH_WATER)>(), mountain = (int)scalar_const<mix(TH_MOUNTAIN)>(),
        cave_m = (int)scalar_const<mix(TH_CAVE_M)>(), lava_m = (int)scalar_const<mix(TH_LAVA_M)>(), diamond_m = (int)scalar_const<mix(TH_DIAMOND_M)>();
    uint32_t diamond = scalar_const<draw(U_DIAMOND)>(), iron = scalar_const<draw(U_IRON)>(), coal = scalar_const<draw(U_COAL)>(),
             sparse = scalar_const<draw(U_TREE_SPARSE)>(), forest = scalar_const<draw(U_TREE_FOREST)>();
    uint32_t forest_f = scalar_const<first_above<PERLIN>(TH_FOREST_F)>(), iron_f = scalar_const<first_above<PERLIN>(TH_IRON_F - 1)>(),
             lava_f = scalar_const<first_above<PERLIN>(TH_LAVA_F)>(), cave_c = scalar_const<first_above<PERLIN>(TH_CAVE_C)>(),
             tunnel = scalar_const<first_above<PERLIN>(TUNNEL1 - 1) - first_above<PERLIN>(TUNNEL0)>();
};

// The overworld's rule for one cell: appends five bits to `word`, where a cell takes a byte.  w, m: 4 times
// the water and mountain fields (a mix of two noises, see mix31), lowered near the start; C, F: cave and
// forest field; u: the cell's draw in the upper half (what lies in the lower half does not matter).
// In order of precedence: path, lava, diamond, iron, coal, stone on rock; water, sand, tree, grass elsewhere.
// The bits: plain kind (2: 0 grass, 1 tree, 2 sand, 3 water), rock kind (3: 0 no rock, 1 stone, 2 coal,
// 3 iron, 4 lava, 5 diamond, 6 and 7 path).  No branches: 64 rows of the world nearly always hold some
// mountain, so a branch around the mountain rules would save nothing.
template <bool PERLIN>
__device__ __forceinline__ void classify(uint32_t& word, const Thresholds<PERLIN>& t, int w, int m, uint32_t C, uint32_t F, uint32_t u)
{
    const Mask shore = mask_of(w > t.sand), rock = mask_of(m > t.mountain), u500 = mask_of(u < t.diamond), u3000 = mask_of(u < t.iron);
    const Mask tree = mask_of(u < t.sparse) | (mask_of(F >= t.forest_f) & mask_of(u < t.forest));
    const Mask tunnel = mask_of(C - first_above<PERLIN>(Thresholds<PERLIN>::TUNNEL0) < t.tunnel);
    const Mask path = (mask_of(m > t.cave_m) & mask_of(C >= t.cave_c)) | (tunnel & rock);
    const Mask lava = mask_of(m > t.lava_m) & mask_of(F >= t.lava_f), gem = lava | (mask_of(m > t.diamond_m) & u500);
    const Mask coal = mask_of(u < t.coal) & ~u3000, iron = u3000 & ~(u500 | mask_of(F >= t.iron_f));
    word <<= 3;
    shift_in(word, shore);
    shift_in_or(word, mask_of(w > t.water), tree & ~shore);
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
// Near the start the fields W4 and M4 are lowered by `bias`, and where that is as large as it is within
// START_CLEAR cells of it, the cell is grass: lowered below every threshold, its draw above every one.
__device__ inline void near_start(int bias, int& W4, int& M4, uint32_t& u)
{
    constexpr int FLAG = 1 << 20, CLEAR = (START_BIAS_R - START_CLEAR) * (4 * START_BIAS);
    static_assert(CLEAR < FLAG && START_BIAS_R * 4 * START_BIAS < CLEAR + FLAG && 4 * 65536 < FLAG, "the flag is above every field and bias");
    const int flag = (bias + (FLAG - CLEAR)) & FLAG;
    W4 -= bias + flag; M4 -= bias + flag;
    u |= (uint32_t)flag << 11;
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
    if (SPLIT) asm("" : "+s"(seed_lo), "+s"(seed_hi));     // or the key schedule of the branch above is kept for here, in vector registers
    int y = tid & 63;
    if (PERLIN) floor_rounding(y);
    const int strip = first_strip + __builtin_amdgcn_readfirstlane(tid >> 6), x0 = strip * 8;
    const U4 r = philox4x32_10(env, 1u, episode, (DOM_WORLDGEN << 16) | (uint32_t)(y * STRIPS + strip), seed_lo, seed_hi);
    const uint32_t* w16 = s_lat + LAT_AT16;
    const uint32_t* m16 = w16 + LAT16_N;
    const uint32_t* w8 = s_lat + LAT_AT8;
    const uint32_t* m8 = w8 + LAT8_N;
    const uint32_t* c8 = m8 + LAT8_N;
    const uint32_t* f8 = c8 + LAT8_N;
    const int iy16 = y >> 4, iy8 = y >> 3, ix16 = x0 >> 4, ix8 = strip;
    const uint32_t odd = 0u - (uint32_t)(strip & 1);   // all ones: right half of a spacing-16 lattice cell
    // 4 times the lowering (10 - d) * 2500 of W and M within Chebyshev distance d < 10 of the start: by
    // rows here, by columns below, and the smaller of the two counts
    const bool near_strip = x0 + 7 > MAPW / 2 - START_BIAS_R && x0 < MAPW / 2 + START_BIAS_R;
    const int bias_y = max(0, START_BIAS_R - iabs(y - MAPW / 2)) * (4 * START_BIAS);
    uint32_t word = 0u, four = 0u;                     // the cells under way, the finished cells 4..7
    const Thresholds<PERLIN> thresholds;
    auto draw = [&](auto j) { return (j & 1) ? r.w[j >> 1] : r.w[j >> 1] << 16; };   // draw of cell j, in the upper half
    auto put = [&](auto near, int j, uint32_t u, int W4, int M4, uint32_t C, uint32_t F) {
        if (near) near_start(min(bias_y, max(0, START_BIAS_R - iabs(x0 + j - MAPW / 2)) * (4 * START_BIAS)), W4, M4, u);
        classify<PERLIN>(word, thresholds, W4, M4, C, F, u);
        if (PERLIN) settle(word);
    };
    // the run's code with and without what only a strip near the start needs
    auto by_strip = [&](auto&& cells) { if (!SPLIT || near_strip) cells(std::true_type()); else cells(std::false_type()); };
    if (PERLIN) {
        const int ky16 = y & 15, ky8 = y & 7, kx16 = x0 & 15;
        const double wy16 = perlin_fade<16>(ky16) * (1.0 / 65536.0), wy8 = perlin_fade<8>(ky8) * (1.0 / 65536.0);
        // One field after the other for the whole run (a line takes 16 registers); the last one with the rule.
        // The empty statement keeps the loads of a field's gradients from being moved before the field at hand.
        auto along = [&](PerlinLine line, auto&& weight, double wy, auto&& cell) {
            for_run([&](auto j) { cell(j, line.field(weight(j), wy)); line.advance(); });
            asm volatile("" ::: "memory");
        };
        auto wide = [&](const uint32_t* lat) { return perlin_line<16>(gradients_at(lat, 5, ix16, iy16), kx16 + 7, ky16); };
        auto narrow = [&](const uint32_t* lat) { return perlin_line<8>(gradients_at(lat, 9, ix8, iy8), 7, ky8); };
        auto weight16 = [&](auto j) { return pick<high_half(perlin_weight<16>(8 + j)), high_half(perlin_weight<16>(j))>(odd); };
        auto weight8 = [&](auto j) { return scalar_double<high_half(perlin_weight<8>(j))>(); };
        int W4[8], M4[8];
        uint32_t C[8];
        const PerlinScale<16> coarse;
        const PerlinScale<8> fine;
        along(wide(w16), weight16, wy16, [&](int j, double v) { W4[j] = coarse.value(v); settle(W4[j]); });
        along(narrow(w8), weight8, wy8, [&](int j, double v) { W4[j] = 3 * W4[j] + fine.value(v); settle(W4[j]); });
        along(wide(m16), weight16, wy16, [&](int j, double v) { M4[j] = coarse.value(v); settle(M4[j]); });
        along(narrow(m8), weight8, wy8, [&](int j, double v) { M4[j] = 3 * M4[j] + fine.value(v); settle(M4[j]); });
        along(narrow(c8), weight8, wy8, [&](int j, double v) { C[j] = settled(v); });
        const PerlinLine forest = narrow(f8);
        by_strip([&](auto near) {
            along(forest, weight8, wy8, [&](auto j, double v) {
                put(near, j, draw(j), W4[j], M4[j], C[j], (uint32_t)__double2loint(v));
                if (j == 4) four = word;                       // (the next four cells shift it out)
            });
        });
    } else {
        const uint32_t v16 = vertical_weights(smooth16(y & 15)), v8 = vertical_weights(smooth8(y & 7));
        auto column = [&](const uint32_t* lat, int width, int cells, int ix, int iy, uint32_t weights, double start) {
            const uint32_t* c = lat + CX_IDX(iy * width + ix, cells - 1);
            return line_between(dot16u(c[0], weights), dot16u(c[1], weights), start);
        };
        const double last16 = pick<high_half(LAST16_ODD), high_half(LAST16)>(odd);
        Line W16 = column(w16, 5, LAT16_N, ix16, iy16, v16, last16), M16 = column(m16, 5, LAT16_N, ix16, iy16, v16, last16);
        Line W8 = column(w8, 9, LAT8_N, ix8, iy8, v8, LAST8), M8 = column(m8, 9, LAT8_N, ix8, iy8, v8, LAST8);
        Line C8 = column(c8, 9, LAT8_N, ix8, iy8, v8, LAST8), F8 = column(f8, 9, LAT8_N, ix8, iy8, v8, LAST8);
        by_strip([&](auto near) {
            for_run([&](auto j) {
                put(near, j, draw(j), mix31(W16.field(), W8.field()), mix31(M16.field(), M8.field()), C8.field(), F8.field());
                if (j == 4) { four = word; word = 0u; }        // the other four cells do not wait for these
                const double s16 = pick<high_half(step16(8 + j)), high_half(step16(j))>(odd);
                W16.advance(s16); M16.advance(s16);
                for (Line* l : {&W8, &M8, &C8, &F8}) l->advance(step8(j));
            });
        });
    }
    if (PERLIN) nearest_rounding(word);
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
