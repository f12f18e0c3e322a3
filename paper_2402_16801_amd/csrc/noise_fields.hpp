// The noise fields of the world generators, evaluated in 32-bit floating point with rounding towards minus infinity
// (every function here but the constants expects that rounding).  A whole number stays where it is under
// it and what lies between two of them stays between them, so the floor of a rounded value is the floor of
// the exact one, however many bits were lost below it: floors, and comparisons with whole numbers, come
// out as in integers of any width.
// Plain C++ so that this can be compared with the oracle's integers without a GPU.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define FIELD_FN __host__ __device__ __forceinline__
#else
#define FIELD_FN inline
#endif

namespace cx {

// smoothstep(k/S) in 1/256 units for S = 8 and S = 16
FIELD_FN constexpr uint32_t smooth8(int k) { return (uint32_t)(12 * k * k - k * k * k); }
FIELD_FN constexpr uint32_t smooth16(int k) { return (uint32_t)((24 * k * k - k * k * k + 4) >> 3); }

// Bilinear value noise, evaluated column-first: two lattice rows are blended once per lattice
// column (vertical weight wy), then every cell of a run blends two columns (horizontal weight wx).
// Its value equals the row-first formula
// ((a(256-wx)+b wx)(256-wy) + (c(256-wx)+d wx) wy) >> 16: nothing is rounded before the final shift there, and
// here only the last multiply-add is, downwards.  Weights are in units of 1: a blended column is a multiple
// of 2^-8 below 2^16, 24 bits, exact as is the difference of two; the field along the run is
// rounded to 24 bits, its floor is the value.
// Lattices lie in LDS as 32-bit floats, one after the other.
FIELD_FN float column(float upper, float lower, float wy) { return __builtin_fmaf(lower - upper, wy, upper); }
struct Line {
    float left, slope;
    // wx: a compile-time constant or the same for many cells
    FIELD_FN float at(float wx) const { return __builtin_fmaf(slope, wx, left); }
};
// lat: the lattice's point above and left of the run
FIELD_FN Line line_at(const float* lat, int width, float wy)
{
    const float left = column(lat[0], lat[width], wy);
    return Line{left, column(lat[1], lat[width + 1], wy) - left};
}
FIELD_FN constexpr float weight8(int k) { return (float)smooth8(k) / 256.0f; }
FIELD_FN constexpr float weight16(int k) { return (float)smooth16(k) / 256.0f; }
// The mix (3 coarse + fine) / 4 of two fields, as the rule compares it: 4 times it, above a whole number that leaves no bits
// for what the division by four loses.  Value noise: floor(coarse) + 2^23 by one addition, where a unit is
// the last bit; three times that and fine lie between 2^24 and 2^25, where it is two.
constexpr float TWO23 = 8388608.0f, MIX_BASE = 3.0f * TWO23;
FIELD_FN float mix31(float coarse, float fine) { return __builtin_fmaf(coarse + TWO23, 3.0f, fine); }

// Perlin gradient noise (appendix "World Generation"): the lattice numbers are read as one of 1024
// directions (top ten bits); cs[a] holds the unit gradient of direction a in Q14.  S is the
// lattice spacing; offsets from the four corners are in units of 1/S; the fade weight
// 6t^5 - 15t^4 + 10t^3 of t = k/S is (F 65536 + S^5 / 2) / S^5 in Q16 with
// F = k^3 (6 k^2 - 15 k S + 10 S^2); blends are p + floor((q - p) w / 65536), along x then y; the
// value, in units of 1 / (16384 S), lands on the 0..65535 scale of the thresholds as
// 32768 + floor(n * 3900 / (1024 S)), clamped.  All divisors are powers of two: floors are shifts.
// A dot product is at most 16385 sqrt(2) S < 2^18.6 and a blend lies between its ends: whole numbers of 20 bits,
// exact in 32-bit floating point; a blend is one multiply-add onto a number above 2^23, rounded down
// (see PerlinLine).
// A lattice lies in LDS as the cosines of its points and, elsewhere, the sines, as 32-bit floats.
constexpr int PERLIN_GAIN = 3900;
template <int S>
FIELD_FN constexpr int perlin_fade(int k)
{
    const int F = k * k * k * (6 * k * k - 15 * k * S + 10 * S * S);
    return S == 16 ? (F + 8) >> 4 : 2 * F;
}
// A Perlin field along a run.  Along a row the dot products with the four corners are linear in kx:
// top and bottom are those with the left corners, dtop and dbottom what the right ones are more, g* what
// a cell further to the right adds to each.  top and bottom carry the offset PERLIN_BASE, between 2^23 and 2^24, where
// a unit is the last bit: a multiply-add onto them, rounded towards minus infinity, is then the blend with
// its floor in one instruction.
constexpr float PERLIN_BASE = 1.5f * TWO23;
struct PerlinLine {
    float top, dtop, bottom, dbottom, gtop, gdtop, gbottom, gdbottom;
    // n + PERLIN_BASE; weights in units of 1: fade of kx and of ky
    FIELD_FN float field(float wx, float wy) const
    {
        const float t = __builtin_fmaf(dtop, wx, top), b = __builtin_fmaf(dbottom, wx, bottom);
        return __builtin_fmaf(b - t, wy, t);
    }
    FIELD_FN void advance() { top -= gtop; dtop -= gdtop; bottom -= gbottom; dbottom -= gdbottom; }
};
// starts at offset (kx, ky) from the upper left corner; cosine, sine: the lattice's point there
template <int S>
FIELD_FN PerlinLine perlin_line(const float* cosine, const float* sine, int width, float kx, float ky)
{
    const float c00 = cosine[0], c01 = cosine[1], c10 = cosine[width], c11 = cosine[width + 1], rx = kx - (float)S, ry = ky - (float)S;
    PerlinLine l;
    const float t = __builtin_fmaf(c00, kx, sine[0] * ky), b = __builtin_fmaf(c10, kx, sine[width] * ry);
    l.top = t + PERLIN_BASE;
    l.bottom = b + PERLIN_BASE;
    l.dtop = __builtin_fmaf(c01, rx, sine[1] * ky) - t;
    l.dbottom = __builtin_fmaf(c11, rx, sine[width + 1] * ry) - b;
    l.gtop = c00; l.gdtop = c01 - c00;
    l.gbottom = c10; l.gdbottom = c11 - c10;
    return l;
}
template <int S>
FIELD_FN constexpr float perlin_weight(int k) { return (float)perlin_fade<S>(k) / 65536.0f; }
// the value of a field on the 0..65535 scale, above PERLIN_BASE: with its floor in one multiply-add
template <int S>
struct PerlinScale {
    static constexpr float GAIN = (float)PERLIN_GAIN / (1024.0f * S);
    static constexpr double OFFSET = (double)PERLIN_BASE + 32768.0 - (double)PERLIN_BASE * GAIN;
    static_assert((double)GAIN * 1024 * S == PERLIN_GAIN && OFFSET == (double)(int)OFFSET && OFFSET > 0.0 && OFFSET < 16777216.0, "exact in 32 bits");
    FIELD_FN float value(float field) const
    {
        const float v = __builtin_fmaf(field, GAIN, (float)OFFSET);
#ifdef __HIP_DEVICE_COMPILE__
        return __builtin_amdgcn_fmed3f(v, PERLIN_BASE, PERLIN_BASE + 65535.0f);
#else
        return v < PERLIN_BASE ? PERLIN_BASE : (v > PERLIN_BASE + 65535.0f ? PERLIN_BASE + 65535.0f : v);
#endif
    }
};
// 4 times the mix of two such values, a multiple of four above 4 * PERLIN_BASE (between 2^25 and 2^26, where the last bit is four)
FIELD_FN float perlin_mix31(float coarse, float fine) { return __builtin_fmaf(coarse, 3.0f, fine); }
// A field of spacing 8 as the rule compares it: the value with what lies below its units (value noise) or
// n + PERLIN_BASE (Perlin noise), without the steps that lead to the 0..65535 scale.
FIELD_FN constexpr int perlin_above(int t)      // smallest n whose value exceeds t: n * GAIN >= (t + 1 - 32768) * 2^13
{
    const long long num = (long long)(t + 1 - 32768) * 8192, q = num / PERLIN_GAIN;
    return (int)(q + (q * PERLIN_GAIN < num ? 1 : 0));
}
static_assert(perlin_above(32767) == 0 && perlin_above(32768) == 3 && perlin_above(32766) == -2, "floor(n * 3900 / 8192) first exceeds 0 at n = 3, -1 at 0, -2 at -2");
template <bool PERLIN>
FIELD_FN constexpr float first_above(int t)      // smallest field that exceeds t
{
    return PERLIN ? (float)perlin_above(t) + PERLIN_BASE : (float)(t + 1);
}
template <bool PERLIN>
FIELD_FN constexpr float first_mix_above(int t)  // the same of a mix
{
    return (PERLIN ? 4.0f * PERLIN_BASE : MIX_BASE) + (float)(4 * t + 4);
}

constexpr uint32_t f32_bits(float v) { return __builtin_bit_cast(uint32_t, v); }
// A field in a tunnel, |value - TH_TUNNEL_CENTER| < TH_TUNNEL_HALF, is one comparison of bit patterns: bits - FIRST < WIDTH, since those of
// positive floats are in the order of their values.
constexpr int TH_TUNNEL_CENTER = 30000, TH_TUNNEL_HALF = 1300;
template <bool PERLIN>
struct Tunnel {
    static constexpr uint32_t FIRST = f32_bits(first_above<PERLIN>(TH_TUNNEL_CENTER - TH_TUNNEL_HALF)),
                              WIDTH = f32_bits(first_above<PERLIN>(TH_TUNNEL_CENTER + TH_TUNNEL_HALF - 1)) - FIRST;
};
constexpr int START_CLEAR = 2, START_BIAS_R = 10, START_BIAS = 2500;
// Near the start the fields W4 and M4 are lowered by `bias`, and where that is as large as it is within
// START_CLEAR cells of it, the cell is grass: lowered below every threshold, its draw above every one.
FIELD_FN void near_start(int bias, float& W4, float& M4, uint32_t& u)
{
    constexpr int FLAG = 1 << 20, CLEAR = (START_BIAS_R - START_CLEAR) * (4 * START_BIAS);
    static_assert(CLEAR < FLAG && START_BIAS_R * 4 * START_BIAS < CLEAR + FLAG && 4 * 65536 < FLAG, "the flag is above every field and bias");
    static_assert(MIX_BASE - 2.0f * FLAG >= 2.0f * TWO23 && 4.0f * PERLIN_BASE - 2.0f * FLAG >= 4.0f * TWO23 && (4 * START_BIAS) % 4 == 0, "the difference is exact");
    const int flag = (bias + (FLAG - CLEAR)) & FLAG;
    const float lower = (float)(bias + flag);
    W4 -= lower; M4 -= lower;
    u |= (uint32_t)flag << 11;
}

}  // namespace cx
