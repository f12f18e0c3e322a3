// The generators' noise fields in 32-bit floating point rounded down (csrc/noise_fields.hpp) against the oracle's
// integers: values, and every comparison that the rules make of a field or a mix: with thresholds, with the tunnel's two
// ends, and of a mix lowered near the start.  All offsets inside a lattice cell, lattice numbers at their ends and at random.
#include <cfenv>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "../../paper_2402_16801_amd/csrc/noise_fields.hpp"

extern "C" uint32_t orc_value_noise(const uint16_t* lattice, int width, int spacing, int x, int y);
extern "C" uint32_t orc_perlin_noise(const uint16_t* lattice, int width, int spacing, int x, int y);

static uint64_t rng = 12345;
static uint32_t draw() { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(rng >> 33); }
static float cosine[1024], sine[1024];
static long long bad = 0, clamped = 0, in_tunnel = 0;
static void expect(bool ok, const char* what, int x, int y)
{
    if (!ok && bad++ < 10) std::printf("%s at (%d, %d)\n", what, x, y);
}

// one lattice cell of each spacing: the fields at offset (x, y), x < 8 from the start of a run
struct Fields { uint32_t coarse, fine; float f_coarse, f_fine, f_field; };
template <bool PERLIN>
static void compare(const Fields& f, int x, int y)
{
    for (int d = -1; d <= 1; ++d) {
        const int v = (int)f.fine + d, mix = (int)((3u * f.coarse + f.fine) >> 2) + d;
        // a threshold outside the scale has no smallest value above it in Perlin noise, where values are clamped there
        if (v >= 0 && v < 65535) expect((f.f_field >= cx::first_above<PERLIN>(v)) == ((int)f.fine > v), "field", x, y);
        if (mix >= 0) expect(((PERLIN ? cx::perlin_mix31(f.f_coarse, f.f_fine) : cx::mix31(f.f_coarse, f.f_fine)) >= cx::first_mix_above<PERLIN>(mix)) ==
                             ((int)((3u * f.coarse + f.fine) >> 2) > mix), "mix", x, y);
    }
    const bool tunnel = std::abs((int)f.fine - cx::TH_TUNNEL_CENTER) < cx::TH_TUNNEL_HALF;
    expect((cx::f32_bits(f.f_field) - cx::Tunnel<PERLIN>::FIRST < cx::Tunnel<PERLIN>::WIDTH) == tunnel, "tunnel", x, y);
    in_tunnel += tunnel;
    // a cell at distance d from the start: lowered, and below every threshold where it is cleared
    for (int d = 0; d < cx::START_BIAS_R; ++d) {
        float w = PERLIN ? cx::perlin_mix31(f.f_coarse, f.f_fine) : cx::mix31(f.f_coarse, f.f_fine), m = w;
        uint32_t u = 0u;
        cx::near_start((cx::START_BIAS_R - d) * 4 * cx::START_BIAS, w, m, u);
        const int lowered = (int)((3u * f.coarse + f.fine) >> 2) - (cx::START_BIAS_R - d) * cx::START_BIAS;
        expect(w == m && (u == 0x80000000u) == (d <= cx::START_CLEAR) && (u & 0x7FFFFFFFu) == 0u, "cleared", x, y);
        for (int e = -1; e <= 1; ++e)
            if (lowered + e >= 0) expect((w >= cx::first_mix_above<PERLIN>(lowered + e)) == (d > cx::START_CLEAR && e < 0), "near the start", x, y);
    }
}

static void cell(const uint16_t* l16, const uint16_t* l8)
{
    float p16[4], p8[4], c16[4], s16[4], c8[4], s8[4];
    for (int i = 0; i < 4; ++i) {
        p16[i] = l16[i]; p8[i] = l8[i];
        c16[i] = cosine[l16[i] >> 6]; s16[i] = sine[l16[i] >> 6]; c8[i] = cosine[l8[i] >> 6]; s8[i] = sine[l8[i] >> 6];
    }
    for (int y = 0; y < 16; ++y)
        for (int half = 0; half < 2; ++half) {
            const int y8 = y & 7;
            const cx::Line wide = cx::line_at(p16, 2, cx::weight16(y)), narrow = cx::line_at(p8, 2, cx::weight8(y8));
            cx::PerlinLine pw = cx::perlin_line<16>(c16, s16, 2, (float)(8 * half + 7), (float)y), pn = cx::perlin_line<8>(c8, s8, 2, 7.0f, (float)y8);
            for (int j = 7; j >= 0; --j) {
                const int x = 8 * half + j;
                Fields v;
                v.coarse = orc_value_noise(l16, 2, 16, x, y); v.fine = orc_value_noise(l8, 2, 8, j, y8);
                v.f_coarse = wide.at(cx::weight16(x)); v.f_fine = v.f_field = narrow.at(cx::weight8(j));
                expect(std::floor(v.f_coarse) == (float)v.coarse && std::floor(v.f_fine) == (float)v.fine, "value", x, y);
                compare<false>(v, x, y);
                v.coarse = orc_perlin_noise(l16, 2, 16, x, y); v.fine = orc_perlin_noise(l8, 2, 8, j, y8);
                v.f_field = pn.field(cx::perlin_weight<8>(j), cx::perlin_weight<8>(y8));
                v.f_coarse = cx::PerlinScale<16>().value(pw.field(cx::perlin_weight<16>(x), cx::perlin_weight<16>(y)));
                v.f_fine = cx::PerlinScale<8>().value(v.f_field);
                expect(v.f_coarse - cx::PERLIN_BASE == (float)v.coarse && v.f_fine - cx::PERLIN_BASE == (float)v.fine, "Perlin value", x, y);
                clamped += v.coarse == 0 || v.coarse == 65535 || v.fine == 0 || v.fine == 65535;
                compare<true>(v, x, y);
                pw.advance(); pn.advance();
            }
        }
}

int main()
{
    for (int a = 0; a < 1024; ++a) {
        const double turn = 6.283185307179586476925286766559 * (double)a / 1024.0;
        cosine[a] = (float)std::lround(std::cos(turn) * 16384.0); sine[a] = (float)std::lround(std::sin(turn) * 16384.0);
    }
    const uint16_t ends[] = { 0, 1, 255, 256, 32767, 32768, 65279, 65280, 65534, 65535 };
    uint16_t a[4] = { 0, 0, 0, 0 }, b[4];
    (void)orc_perlin_noise(a, 2, 8, 0, 0);           // the oracle's tables, made with the usual rounding
    std::fesetround(FE_DOWNWARD);
    for (int i = 0; i < 10000; ++i) {                // all corners at the ends of the range: 10^4 combinations
        for (int k = 0, n = i; k < 4; ++k, n /= 10) { a[k] = ends[n % 10]; b[3 - k] = ends[n % 10]; }
        cell(a, b);
    }
    for (int i = 0; i < 30000; ++i) {
        for (int k = 0; k < 4; ++k) { a[k] = (uint16_t)draw(); b[k] = (uint16_t)draw(); }
        cell(a, b);
    }
    // gradients that point at the middle of their cell, where Perlin noise leaves the scale
    for (int i = 0; i < 2000; ++i) {
        const int towards[4] = { 128, 384, 896, 640 };       // in 1024ths of a turn, from the corners in reading order
        for (int k = 0; k < 4; ++k) {
            const int away = i & 1 ? 512 : 0;
            a[k] = (uint16_t)(((towards[k] + away + (int)(draw() % 65) - 32) & 1023) << 6); b[k] = (uint16_t)(((towards[k] + away + (int)(draw() % 65) - 32) & 1023) << 6);
        }
        cell(a, b);
    }
    if (in_tunnel < 1000) { std::printf("only %lld values in the tunnel\n", in_tunnel); ++bad; }
    if (clamped < 1000) { std::printf("only %lld clamped values\n", clamped); ++bad; }
    if (bad == 0) std::printf("noise_fields_test: ok\n");
    return bad != 0;
}
