// Kernels and the C ABI of the MI355X Craftax-Classic simulator (see include/craftax.h).
#include "../../include/craftax.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "common.hpp"
#include "full_api.hpp"
#include "launch_limits.hpp"
#include "lookahead.hpp"
#include "regen_units.hpp"
#include "render.hpp"
#include "rollout_route.hpp"
#include "step.hpp"
#include "worldgen.hpp"

namespace cx {

constexpr int BLOCK = 256;

// Copies a 128-byte record between HBM (uint4 granules) and an environment's LDS area.  The load
// comes in two halves so that a kernel can issue it early and park it in LDS later.
template <int G>
struct RecordRegs { uint4 v[((REC_DWORDS / 4) + G - 1) / G]; };
template <int G>
__device__ inline void fetch_record(int l, const uint4* __restrict__ grec, RecordRegs<G>& r)
{
#pragma unroll
    for (int it_c = 0; it_c < ((REC_DWORDS / 4) + G - 1) / G; ++it_c) {
        const int c = l + it_c * G;
        if (c < (REC_DWORDS / 4)) r.v[it_c] = grec[c];
    }
}
template <int G>
__device__ inline void park_record(int l, const RecordRegs<G>& r, uint32_t* e)
{
#pragma unroll
    for (int it_c = 0; it_c < ((REC_DWORDS / 4) + G - 1) / G; ++it_c) {
        const int c = l + it_c * G;
        if (c >= (REC_DWORDS / 4)) break;
        const uint4 v = r.v[it_c];
        uint2* d = reinterpret_cast<uint2*>(e + LDS_REC + 4 * c);
        d[0] = make_uint2(v.x, v.y);
        d[1] = make_uint2(v.z, v.w);
    }
}
template <int G>
__device__ inline void load_record(int l, const uint4* __restrict__ grec, uint32_t* e)
{
    RecordRegs<G> r;
    fetch_record<G>(l, grec, r);
    park_record<G>(l, r, e);
}
// The same the other way round.
template <int G>
__device__ inline void take_record(int l, const uint32_t* e, RecordRegs<G>& r)
{
#pragma unroll
    for (int it_c = 0; it_c < ((REC_DWORDS / 4) + G - 1) / G; ++it_c) {
        const int c = l + it_c * G;
        if (c >= (REC_DWORDS / 4)) break;
        const uint2* d = reinterpret_cast<const uint2*>(e + LDS_REC + 4 * c);
        const uint2 a = d[0], b = d[1];
        r.v[it_c] = make_uint4(a.x, a.y, b.x, b.y);
    }
}
template <int G>
__device__ inline void put_record(int l, uint4* __restrict__ grec, const RecordRegs<G>& r)
{
#pragma unroll
    for (int it_c = 0; it_c < ((REC_DWORDS / 4) + G - 1) / G; ++it_c) {
        const int c = l + it_c * G;
        if (c < (REC_DWORDS / 4)) grec[c] = r.v[it_c];
    }
}
template <int G>
__device__ inline void store_record(int l, uint4* __restrict__ grec, const uint32_t* e)
{
    RecordRegs<G> r;
    take_record<G>(l, e, r);
    put_record<G>(l, grec, r);
}

// ---------------------------------------------------------------------------------------------
// Worlds are generated one episode ahead (see lookahead.hpp).  Two tags per environment, one per
// half of the spare map (a world is regenerated by two blocks).
using la::Lists;
using la::counter;
using la::ENTRY_VOID;
using la::NSUB;

// reset: two blocks per environment, for the worlds of episodes 0 and 1
template <bool PERLIN>
__global__ __launch_bounds__(WG_THREADS, 8) void k_reset(uint4* __restrict__ recs, uint8_t* __restrict__ maps,
                                                 const uint64_t* __restrict__ seeds, Lists ls, const Luts* __restrict__ luts,
                                                 uint32_t* __restrict__ unlocks)
{
    if (blockIdx.x == 0) la::reset_counters(ls);
    __shared__ uint32_t s_lat[lattice_words<PERLIN>];
    const uint32_t env = blockIdx.x >> 1, ep = blockIdx.x & 1u;
    const uint64_t seed = seeds[env];
    const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
    worldgen_block<WG_THREADS, PERLIN>(maps + map_offset(env, ep), s_lat, lo, hi, env, ep, nullptr, 0, luts->perlin_cs);
    if (ep == 0) {
        if (threadIdx.x < REC_DWORDS)
            reinterpret_cast<uint32_t*>(recs + (size_t)env * 8)[threadIdx.x] = fresh_record_word(threadIdx.x, lo, hi, 0u);
        if (threadIdx.x < UNLOCK_STRIDE) unlocks[(size_t)env * UNLOCK_STRIDE + threadIdx.x] = 0u;
    } else if (threadIdx.x < 2) ls.tags[2 * env + threadIdx.x] = make_uint2(1u, 0u);
}

// A regeneration block of the step grid: worlds for the episodes after next of the episodes that
// ended in the previous launch.  The generator's code for strips near the start and far from it apart (SPLIT):
// where many episodes end at once these blocks go through several worlds each and the launch waits for them
// (16,384 environments, episodes of 2 steps 100.7 us with the code once, 95.5 so; of 10 steps 31.4 and 30.5, of 4,096
// and 2 steps 26.3 and 25.1; no difference where few end).
template <bool PERLIN>
__device__ __forceinline__ void regeneration_block(uint8_t* __restrict__ maps, const Lists& ls, uint32_t seq, uint32_t count,
                                                   uint32_t rb, uint32_t nrb, uint32_t* s_lat, const uint32_t* __restrict__ perlin_cs)
{
    const uint4* list = la::consumed_sub_list(ls, seq, rb);
    // two blocks per world, one half (32 columns) each: a regeneration block is then as short as it can be
    // with one run of 8 cells per thread, and the tail it adds to the launch is half as long
    const uint32_t pair = rb / NSUB, half = pair & 1u;
    for (uint32_t i = pair >> 1; i < count; i += nrb / NSUB / 2) {
        const uint4 entry = list[i];
        if (entry.x == ENTRY_VOID) continue;
        worldgen_block<BLOCK, PERLIN>(maps + map_offset(entry.x, entry.w), s_lat, entry.y, entry.z, entry.x, entry.w, nullptr,
                                      (int)half * (STRIPS / 2), perlin_cs);
        if (threadIdx.x == 0) ls.tags[2 * entry.x + half] = make_uint2(entry.w, seq);
    }
}

// Regeneration inside a step launch whose step blocks fill the chip (four lanes per environment),
// shared between the regeneration blocks of the grid and the step blocks.  Sub-list s is seen as
// units u = 2 * entry + half, u < 2 * count.  Its per_sub regeneration blocks (index pr among
// them) take the head, units pr, pr + per_sub, ... (head_rounds of them): they sit in the one
// place per compute unit that the step blocks leave free and work from the start of the launch.
// The tail is dealt out to the step blocks that append to this sub-list (index q among the nq of
// them) and, behind them, to the regeneration blocks again, so that a launch in which very many
// episodes ended is shared by every block of the grid.  A step block generates its share BEFORE it
// steps, while its record is on its way: at the start of a launch every wavefront waits for memory
// and the vector units idle, whereas a regeneration block that is dispatched only when a step
// block has finished competes with the slowest step blocks and ends the launch later.  The step
// blocks with the lowest numbers get the tail: they are served first and finish first anyway.
// helper: the calling block is step block q; else regeneration block pr.
// The walk over the units is in regen_units.hpp (plain arithmetic, unit-tested on the host).
template <bool PERLIN>
__device__ __forceinline__ void regeneration_share(uint8_t* __restrict__ maps, const Lists& ls, uint32_t seq, uint32_t count, uint32_t sub,
                                                   bool helper, uint32_t index, uint32_t per_sub, uint32_t nq, uint32_t rounds, uint32_t* s_lat,
                                                   const uint32_t* __restrict__ perlin_cs)
{
    const uint4* list = la::consumed_sub_list(ls, seq, sub);
    for (UnitWalk w = first_unit(helper, index, per_sub, rounds); w.u < 2u * count; w = next_unit(w, helper, index, per_sub, nq, rounds)) {
        const uint4 entry = list[w.u >> 1];
        const uint32_t half = w.u & 1u;
        if (entry.x != ENTRY_VOID) {
            worldgen_block<BLOCK, PERLIN, false>(maps + map_offset(entry.x, entry.w), s_lat, entry.y, entry.z, entry.x, entry.w, nullptr,
                                          (int)half * (STRIPS / 2), perlin_cs);
            if (threadIdx.x == 0) ls.tags[2 * entry.x + half] = make_uint2(entry.w, seq);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// step: G lanes per environment, 256/G environments per block, followed in the same grid by
// the regeneration blocks for the episodes that ended in the previous launch (with four lanes per
// environment the step blocks take a share of that work before they step: regeneration_share).
constexpr int COMPUTE_UNITS = 256;
// Step blocks that a compute unit holds, by registers (a wavefront of a block on each of the four SIMDs): five with either noise.  With Perlin noise
// four were dealt for while the generator took more registers (steps of 57,344 environments 45.6 us, 44.0 dealt for five, of 65,536 46.1 and
// 43.9; one state alone 33.1 and 31.7).  The bound the compiler is given stays at four there, which it needs no spills for and beats anyway
// (with five 40,000 environments take 29.4 instead of 28.5, 49,152 35.0 instead of 34.0).
constexpr int STEP_BLOCKS_PER_CU = 5;
constexpr int step_bound(bool perlin) { return perlin ? 4 : STEP_BLOCKS_PER_CU; }
// Neighbouring environments whose entries go to the same sub-list of the regeneration list: those of a step block, which
// appends them together, or, with 16 lanes, where an entry is appended by itself, one: a few environments whose episodes
// end together then occupy the regeneration blocks of all sub-lists instead of those of one or two (16 environments,
// episodes of 2 steps 27.1 -> 7.1 us, 64: 11.0 -> 7.4; ordinary episodes the same).
constexpr int envs_per_list_turn(int lanes) { return lanes == 16 ? 1 : BLOCK / lanes; }
// Byte layouts are written through to the last-level cache, from THROUGH_FROM environments on where there are sixteen lanes (see Keep; us,
// left in the L2 / written through, one state stepped over and over | three in turn | one whose observation a cast to bfloat16 reads
// behind every step).  Sixteen lanes: 256 8.1 / 8.3 | 8.3 / 8.3 | -, 1,500 8.7 / 8.6 | 8.7 / 8.6 | 15.7 / 15.9, 4,096 9.2 / 8.8 |
// 9.2 / 8.8 | 23.7 / 23.4, 11,000 12.1 / 10.5 | 12.5 / 11.0 | 44.6 / 42.5.  Eight and four, and streamed past the cache (with four
// lanes three blocks of four, the fourth written through): 13,000 14.3 / 14.4 / 14.0 | 14.8 / 15.0 / 14.5 | 51.3 / 51.0 / 60.7,
// 20,000 17.7 / 16.2 / 16.0 | 18.3 / 17.5 / 17.0 | 69.5 / 68.6 / 85.9, 32,768 21.4 / 19.8 / 19.4 | 23.2 / 22.1 / 20.7 | 102 / 101 / 129,
// 49,152 25.8 / 24.3 / 23.4 | 31.9 / 33.9 / 25.1 | 145 / 145 / 186, 65,536 31.4 / 30.8 / 29.8 | 43.2 / 43.6 / 33.5 | 198 / 199 / 256:
// what streaming saves the step, and more, whoever reads the observation waits for.
constexpr int THROUGH_FROM = 1500;
// DRAW (pixels, 16 lanes): a block holds one environment, whose 16 lanes step it, and all its threads then draw
// the picture, from the record in LDS: one launch instead of two, and the pictures of some blocks hide the steps of others.
template <int G, int OBS_MODE, bool PERLIN, bool DRAW = false>
__global__ __launch_bounds__(BLOCK, step_bound(PERLIN)) void k_step(uint4* __restrict__ recs, uint8_t* __restrict__ maps,
                                                   const Luts* __restrict__ luts, const int32_t* __restrict__ actions,
                                                   uint8_t* __restrict__ obs, float* __restrict__ reward,
                                                   uint8_t* __restrict__ done, Lists ls, Params p, int step_blocks)
{
    static_assert(!DRAW || (G == 16 && OBS_MODE == CRAFTAX_OBS_PIXELS_F32), "pictures are drawn behind a step with 16 lanes");
    constexpr int EPB = DRAW ? 1 : Grp<G>::EPB;
    using LY = StepLayout;
    constexpr int ENV_AT = DRAW ? PIX_STRIP_FLOATS : 0;     // the environments' areas, behind the strips of the picture's pixels
    __shared__ __attribute__((aligned(16))) uint32_t s_env[ENV_AT + EPB * LY::STRIDE];
    __shared__ int s_tile[DRAW ? PIX_CELLS : 1], s_ent[DRAW ? PIX_CELLS : 1];
    __shared__ int s_ndone;
    __shared__ uint32_t s_base;
    __shared__ uint4 s_list[EPB];
    const int tid = threadIdx.x;
    const bool regen_role = (int)blockIdx.x >= step_blocks;
    const uint32_t rb = blockIdx.x - (uint32_t)step_blocks, nrb = gridDim.x - (uint32_t)step_blocks;
    const int g = tid / G, l = tid % G;
    const int env = blockIdx.x * EPB + (DRAW ? 0 : g);
    const bool active = !regen_role && env < p.n && (!DRAW || tid < G);
    // the record and the action are asked for before the launch bookkeeping, which waits for a
    // counter of its own: the two round trips then overlap
    RecordRegs<G> fetched;
    int action = 0;
    // EAGER (16 lanes per environment, a launch of one short chain per wavefront): what an episode that ends
    // needs (the tags of the spare world, the window of its start position) and the tables that the renderer
    // looks scalars up in are fetched in advance, its place on the list is claimed before the rendering,
    // and no wavefront waits for the others of its block once all have the number of the launch.  The launch ends with its slowest
    // wavefront, nearly always one with such an episode, and each of these was a trip to memory of its own
    // at the end of that one's chain (4,096 environments 10.4 -> 9.3 us, 8,192: 12.2 -> 10.9, 500: 9.1 -> 8.2; one
    // alone 7.5 either way).  With fewer lanes the chip is full, and the launch bound by memory and issue.
    constexpr bool EAGER = G == 16, kFloats = OBS_MODE == CRAFTAX_OBS_SYM_U8_F32 || OBS_MODE == CRAFTAX_OBS_SYM_F32;
    uint4 spare_tag = make_uint4(0u, 0u, 0u, 0u);
    float lut_sqrt10 = 0.0f, lut_tenth = 0.0f;
    if (active) {
        fetch_record<G>(l, recs + (size_t)env * 8, fetched);
        action = actions[env];
        if (EAGER) {
            spare_tag = reinterpret_cast<const uint4*>(ls.tags)[env];
            if (kFloats) { lut_sqrt10 = luts->sqrt10[l]; lut_tenth = luts->tenth[l]; }
        }
    }
    // SHARE: every block reads the length of one sub-list of the consumed list, a regeneration block
    // its own, a step block the one it appends to (see regeneration_share)
    constexpr bool SHARE = G == 4;
    static_assert(ENV_AT + EPB * LY::STRIDE >= lattice_words<PERLIN>, "the environments' area, empty until the records are parked, doubles as lattice scratch");
    if (!EAGER && tid == 0) s_ndone = 0;
    const la::Ticket ticket = la::enter_launch(ls, SHARE || regen_role, regen_role ? rb : blockIdx.x);   // holds a block barrier
    const uint32_t seq = ticket.seq, regen_count = ticket.regen_count;
    auto leave = [&]() { la::leave_launch(ls, ticket); };
    const uint32_t sub = (regen_role ? rb : blockIdx.x) % NSUB, per_sub = nrb / NSUB;
    const uint32_t nq = ((uint32_t)step_blocks + NSUB - 1u - sub) / NSUB;   // step blocks that append to this sub-list

    const uint32_t rounds = head_rounds((uint32_t)step_blocks, nrb, COMPUTE_UNITS * STEP_BLOCKS_PER_CU);
    // SHARE: a regeneration block's units, or this step block's share of the worlds owed from the previous
    // launch while its records arrive (one call for both: the generator is in the kernel's code once)
    if (SHARE && (regen_role || first_helper_unit(blockIdx.x / NSUB, per_sub, rounds) < 2u * regen_count))
        regeneration_share<PERLIN>(maps, ls, seq, regen_count, sub, !regen_role, (regen_role ? rb : blockIdx.x) / NSUB, per_sub, nq, rounds, s_env, luts->perlin_cs);
    // The hint is for what the generator costs the step: without it the compiler spills scalar registers for the generator in front
    // of this branch, 22 of them with Perlin noise, and the step fetches them back one by one (steps with Perlin noise of 100
    // environments 8.06 us, 7.92 with the hint, of 500 8.34 and 8.23, flat floats of 4,096 11.34 and 11.14).  A probability near
    // one has the generator put into a function of its own, with a stack.
    if (__builtin_expect_with_probability(regen_role, 0, 0.75)) {
        if (!SHARE && rb / NSUB / 2 < regen_count) regeneration_block<PERLIN>(maps, ls, seq, regen_count, rb, nrb, s_env, luts->perlin_cs);
        leave();
        return;
    }

    bool queued = false;                 // EAGER: this group's episode ended; its place on the list is on its way
    uint32_t list_at = 0u;
    uint4 entry = make_uint4(0u, 0u, 0u, 0u);
    uint32_t* e = s_env + ENV_AT + (DRAW ? 0 : g) * LY::STRIDE;
    constexpr bool kSymbolic = OBS_MODE != CRAFTAX_OBS_PIXELS_F32;
    constexpr bool kBytes = OBS_MODE == CRAFTAX_OBS_SYM_U8_I8 || OBS_MODE == CRAFTAX_OBS_SYM_U8_F32;
    // Records go out behind the observations (the renderer stages the scalars in their place in LDS, so they wait in registers): in front
    // of them, they are what the observations' stores queue up behind (65,536 environments 44.0 us on states in turn and 30.8 on one, 42.8 and
    // 30.4 so).
    constexpr bool RECORD_LAST = !EAGER && kBytes;
    bool staged = false;
    if (active) {
        park_record<G>(l, fetched, e);
        group_sync();
        const uint32_t* rec = e + LDS_REC;
        const uint32_t ep = rec[RW_EPISODE], lo = rec[RW_SEED_LO], hi = rec[RW_SEED_HI];
        // the windows of the current position and of the spare world's start come together
        StartWindow<G> spare;
        if (EAGER) spare.fetch(l, maps + map_offset((uint32_t)env, ep + 1u));
        float day_next = 0.0f, day_fresh = 0.0f;               // daylight of the state that will be rendered
        uint32_t q7_next = 0u, q7_fresh = 0u;
        if (EAGER) {
            uint32_t phase = (rec[RW_VIT] >> 16) + 1u;
            if (phase == p.day_length) phase = 0u;
            if (kFloats) { day_next = luts->daylight[phase]; day_fresh = luts->daylight[0]; }
            else if (kSymbolic) { q7_next = luts->light_q7[phase]; q7_fresh = luts->light_q7[0]; }
        }
        StepOut o = step_env<G>(l, (uint32_t)env, e, maps + map_offset((uint32_t)env, ep), luts, action, p);
        if (l == 0) { reward[env] = o.reward; done[env] = o.done ? 1 : 0; }
        count_unlocks<G>(l, p.unlocks + (size_t)env * UNLOCK_STRIDE, o.unlocked);
        bool write_back = !o.done;
        if (o.done) {
            // the record in LDS is still the episode that just ended
            const uint4 tag = EAGER ? spare_tag : reinterpret_cast<const uint4*>(ls.tags)[env];   // (episode, launch) of the two halves of the spare world
            if (p.reset_mode == CRAFTAX_RESET_EXACT && tag.x == ep + 1u && tag.y < seq && tag.z == ep + 1u && tag.w < seq) {
                // the next world is waiting in the other slot: start the new episode right here
                group_sync();
#pragma unroll
                for (int it = 0; it < (REC_DWORDS + G - 1) / G; ++it) {
                    const int i = l + it * G;
                    if (i < REC_DWORDS) e[LDS_REC + i] = fresh_record_word(i, lo, hi, ep + 1u);
                }
                if (EAGER) spare.park(l, e + LDS_WIN);
                else load_window<G>(l, MAPW / 2, MAPW / 2, maps + map_offset((uint32_t)env, ep + 1u), e + LDS_WIN);
                group_sync();
                o.mvx = 0; o.mvy = 0; o.woff = (MAPW / 2 - WIN_COLS / 2) & 3;
                write_back = true;
                if (l == 0) {
                    entry = make_uint4((uint32_t)env, lo, hi, ep + 2u);
                    if (EAGER) { list_at = la::claim_entry(ls, seq, (uint32_t)env); queued = true; }
                    else s_list[atomicAdd(&s_ndone, 1)] = entry;
                }
            } else if (l == 0) {
                la::append_slow(ls, (uint32_t)p.n, make_uint4((uint32_t)env, lo, hi, ep + 1u));
            }
        }
        if (write_back) {
            if (RECORD_LAST && obs != nullptr) take_record<G>(l, e, fetched);
            else store_record<G>(l, recs + (size_t)env * 8, e);
            if (kSymbolic && obs != nullptr) {
                // staged in LDS here and written by the whole wave below
                const RenderLuts tables{lut_sqrt10, lut_tenth, o.done ? day_fresh : day_next, o.done ? q7_fresh : q7_next};
                render_symbolic<G, OBS_MODE, true, false, LY, EAGER>(l, e, o.mvx, o.mvy, o.woff, luts, obs + (size_t)env * obs_stride(OBS_MODE), &tables);
                staged = true;
            }
        }
    }
    if (kSymbolic && obs != nullptr) {
        if (kBytes && l == 0) e[LY::FLAG] = staged ? 1u : 0u;      // floats are told by a vote
        group_sync();
        const int first = __builtin_amdgcn_readfirstlane((tid & ~63) / G);   // first environment of this wave within the block
        const uint32_t* wave_env = s_env + first * LY::STRIDE;
        uint8_t* wave_obs = obs + (size_t)(blockIdx.x * EPB + first) * obs_stride(OBS_MODE);
        if constexpr (!kBytes) {
            if ((long long)p.n * OBS_STRIDE_F32 <= CACHE_SHARE) flush_wave_floats<G, LY, Keep::THROUGH>(wave_env, wave_obs, __ballot(staged));
            else flush_wave_floats<G, LY, Keep::PLAIN>(wave_env, wave_obs, __ballot(staged));
        }
        else if (G == 16 && p.n < THROUGH_FROM) flush_wave_observations<G, OBS_MODE, LY, Keep::PLAIN>(wave_env, wave_obs);
        else flush_wave_observations<G, OBS_MODE, LY, Keep::THROUGH>(wave_env, wave_obs);
        if (RECORD_LAST && staged) put_record<G>(l, recs + (size_t)env * 8, fetched);
    }
    if (EAGER) {
        // an entry at a time, the place claimed before the rendering: no wavefront waits for the others of its block
        if (queued) la::commit_entry(ls, seq, (uint32_t)env, list_at, entry);
        leave();
        if (DRAW) {
            // the record is in LDS, the step's changes to the map have left for memory.  An episode that ended without a spare
            // world shows the state in memory: step_env leaves the record in LDS alone when an episode ends.
            __syncthreads();
            const uint8_t* map = maps + map_offset((uint32_t)env, e[LDS_REC + RW_EPISODE]);
            uint8_t* out = obs + (size_t)env * OBS_STRIDE_PIXELS;
            float* strip = reinterpret_cast<float*>(s_env);
            if (picture_kept(p.n, env, blockIdx.x)) render_pixels_block<Keep::THROUGH>(e + LDS_REC, map, luts, out, s_tile, s_ent, strip);
            else render_pixels_block<Keep::STREAM>(e + LDS_REC, map, luts, out, s_tile, s_ent, strip);
        }
        return;
    }
    __syncthreads();
    leave();
    const int nd = s_ndone;
    if (nd == 0) return;
    la::append_block_entries(ls, seq, s_list, nd, &s_base, blockIdx.x);
}

// A launch of regeneration blocks only (before and after a rollout): brings every spare world up to date
// and empties the lists, with the bookkeeping of a step launch that has no step blocks.
// Eight blocks per compute unit (value noise, which needs no more registers: five: rollouts of 16,384 environments and 64 steps 662 us, 657
// with eight, of 32,768 1,046 and 1,034; of 600 and one step 17.8 either way).  The Perlin generator spills a vector register for the eighth
// (8 bytes of scratch) and 23 scalar ones; seven blocks, which spill no vector register: 256 environments and 16 steps 110.2 us, 110.8 with eight, 12,000
// 152.1 and 151.3, 32,768 and 64 steps 1,072 and 1,071.
constexpr int DRAIN_BLOCKS_PER_CU = 8;
template <bool PERLIN>
__global__ __launch_bounds__(BLOCK, DRAIN_BLOCKS_PER_CU) void k_drain(uint8_t* __restrict__ maps, const Luts* __restrict__ luts, Lists ls)
{
    __shared__ uint32_t s_lat[lattice_words<PERLIN>];
    const uint32_t rb = blockIdx.x, nrb = gridDim.x;
    const la::Ticket ticket = la::enter_launch(ls, true, rb);
    if (rb / NSUB / 2 < ticket.regen_count) regeneration_block<PERLIN>(maps, ls, ticket.seq, ticket.regen_count, rb, nrb, s_lat, luts->perlin_cs);
    la::leave_launch(ls, ticket);
}

// Half a world by a whole block.  Not inlined: the rollout kernel's loop would pay for the generator's
// registers in spills at every step.  SPLIT: see worldgen_block.  With four lanes per environment, where the blocks
// fill the chip and short episodes make it a matter of throughput (65,536 environments, 32 steps in episodes of 5:
// 4,615 us with the code once, 4,465 split); with sixteen the code once is ahead (4,096: 714 / 732).
template <typename T> using Lds = T __attribute__((address_space(3)));
template <bool PERLIN, bool SPLIT>
__device__ __attribute__((noinline)) void generate_half(uint8_t* map, Lds<uint32_t>* lat, Lds<uint32_t>* start_win, uint32_t lo, uint32_t hi, uint32_t env,
                                                        uint32_t ep, int half, const uint32_t* perlin_cs)
{
    worldgen_block<BLOCK, PERLIN, SPLIT>(map, (uint32_t*)lat, lo, hi, env, ep, (uint32_t*)start_win, half * (STRIPS / 2), perlin_cs);
}

// ---------------------------------------------------------------------------------------------
// rollout: several steps in one launch for callers that have the actions of all those steps at
// hand (a random or scripted policy; appendix "Optimistic Environment Resets" measures such
// rollouts).  A block keeps its environments (64 at 4 lanes each, 16 at 16 lanes) in LDS for the whole launch and walks through
// the steps on its own, so blocks drift apart and the memory traffic of some overlaps the
// arithmetic of others; nothing is exchanged between blocks.  Worlds stay one episode ahead as in
// the step kernel: an environment whose episode ends moves into its spare world.  The world after that
// one is left to the regeneration launch behind this one, which generates all of them with the whole
// chip, or generated by the block itself after step own_from (see rollout_route.hpp);
// the environments that are owed a world at the end go on the regeneration list.  An environment whose
// episode ends without a spare world has the next world generated on the spot.  Before the launch the
// regeneration lists of the step kernel must be empty (the host runs a list-only launch first).
// Measured against blocks that generate all their worlds, by code in the loop (64 steps, value noise /
// Perlin): 12,000 environments 603 / 710 -> 569 / 614 us, 32,768: 1,164 / 1,367 -> 1,065 / 1,157,
// 65,536: 1,801 / 2,051 -> 1,761 / 1,877.
// Blocks per compute unit: four of 64 environments, by LDS.  Of the blocks of 16 with float observations and value noise five, which needs no
// spills (96 registers; unbounded 102, with which from 16,385 environments on the launch waits for a second round of blocks: 16 steps of 16,530
// 342 us on states in turn and 270 on one, with five 303 and 232, of 20,480 392 and 296, now 335 and 264; 4,096 114.3 and 114.9).
constexpr int rollout_bound(int lanes, int obs_mode, bool perlin) { return lanes == 16 && obs_mode == CRAFTAX_OBS_SYM_F32 && !perlin ? 5 : 4; }
template <int G, int OBS_MODE, bool PERLIN>
__global__ __launch_bounds__(BLOCK, rollout_bound(G, OBS_MODE, PERLIN)) void k_rollout(uint4* __restrict__ recs, uint8_t* __restrict__ maps,
                                                      const Luts* __restrict__ luts, const int32_t* __restrict__ actions,
                                                      uint8_t* __restrict__ obs, float* __restrict__ reward,
                                                      uint8_t* __restrict__ done, Lists ls, Params p, int steps, int own_from)
{
    constexpr int EPB = Grp<G>::EPB;
    __shared__ uint32_t s_env[EPB * LDS_ENV_DWORDS];
    __shared__ __attribute__((aligned(16))) uint32_t s_lat[lattice_words<PERLIN>];   // the generator's lattices; at the end the environments that are owed a world
    static_assert(lattice_words<PERLIN> >= EPB * 4, "an entry per environment");
    __shared__ uint8_t s_queue[EPB];        // ring of environments (index in the block) waiting for a new spare world
    __shared__ uint8_t s_urgent[EPB];       // environments whose episode ended without a spare world
    __shared__ uint8_t s_spare_ok[EPB], s_pending[EPB];
    __shared__ int s_qhead, s_qtail, s_nurgent;
    __shared__ uint32_t s_base;
    const int tid = threadIdx.x, g = tid / G, l = tid % G;
    const int env = blockIdx.x * EPB + g;
    const bool active = env < p.n;
    uint32_t* e = s_env + g * LDS_ENV_DWORDS;
    constexpr bool kBytes = OBS_MODE == CRAFTAX_OBS_SYM_U8_I8 || OBS_MODE == CRAFTAX_OBS_SYM_U8_F32;
    if (tid == 0) { s_qhead = 0; s_qtail = 0; s_nurgent = 0; }
    if (tid < EPB) { s_spare_ok[tid] = 0; s_pending[tid] = 0; s_env[tid * LDS_ENV_DWORDS + LDS_WINPOS] = 0u; }
    if (active) load_record<G>(l, recs + (size_t)env * 8, e);
    __syncthreads();
    if (active && l == 0) {
        const uint4 tag = reinterpret_cast<const uint4*>(ls.tags)[env];
        const uint32_t next = e[LDS_REC + RW_EPISODE] + 1u;
        const bool ok = tag.x == next && tag.z == next;
        s_spare_ok[g] = ok ? 1 : 0;
        if (!ok) { s_pending[g] = 1; s_queue[atomicAdd(&s_qtail, 1) % EPB] = (uint8_t)g; }
    }
    __syncthreads();

    // Generates the world of the episode after the one in the record of block-local environment gt
    // into the map slot of that episode (all threads of the block; two halves of 256 runs).
    auto generate = [&](int gt, uint32_t* start_win) __attribute__((always_inline)) {
        const uint32_t* rt = s_env + gt * LDS_ENV_DWORDS + LDS_REC;
        const uint32_t tenv = (uint32_t)(blockIdx.x * EPB + gt), ep = rt[RW_EPISODE] + 1u, lo = rt[RW_SEED_LO], hi = rt[RW_SEED_HI];
#pragma unroll 1
        for (int half = 0; half < 2; ++half)
            generate_half<PERLIN, G == 4>(maps + map_offset(tenv, ep), (Lds<uint32_t>*)s_lat, (Lds<uint32_t>*)start_win, lo, hi, tenv, ep, half, luts->perlin_cs);
    };

#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
        // Everything a lane derives from its index is derived again in every turn: the compiler would
        // otherwise keep dozens of such values alive across the whole loop and spill them.
        int tid_t = threadIdx.x;
        uint8_t* obs_t = obs;
        asm volatile("" : "+v"(tid_t));
        asm volatile("" : "+s"(obs_t));
        const int tid = tid_t, g = tid / G, l = tid % G;
        const int env = blockIdx.x * EPB + g;
        const bool active = env < p.n;
        uint32_t* e = s_env + g * LDS_ENV_DWORDS;
        uint8_t* obs = obs_t;
        bool fresh = false;        // this group starts a new episode in this step
        StepOut o;
        o.done = false; o.mvx = 0; o.mvy = 0; o.woff = 0; o.reward = 0.0f; o.unlocked = 0u;
        if (active) {
            const uint32_t* rec = e + LDS_REC;
            const uint32_t ep = rec[RW_EPISODE], lo = rec[RW_SEED_LO], hi = rec[RW_SEED_HI];
            o = step_env<G, true>(l, (uint32_t)env, e, maps + map_offset((uint32_t)env, ep), luts, actions[(size_t)t * p.n + env], p);
            if (l == 0) { reward[(size_t)t * p.n + env] = o.reward; done[(size_t)t * p.n + env] = o.done ? 1 : 0; }
            count_unlocks<G>(l, p.unlocks + (size_t)env * UNLOCK_STRIDE, o.unlocked);
            if (o.done) {
                if (s_spare_ok[g]) {
                    // the next world is waiting in the other slot: start the new episode right here
                    group_sync();
#pragma unroll
                    for (int it = 0; it < (REC_DWORDS + G - 1) / G; ++it) {
                        const int i = l + it * G;
                        if (i < REC_DWORDS) e[LDS_REC + i] = fresh_record_word(i, lo, hi, ep + 1u);
                    }
                    load_window<G>(l, MAPW / 2, MAPW / 2, maps + map_offset((uint32_t)env, ep + 1u), e + LDS_WIN);
                    group_sync();
                    o.mvx = 0; o.mvy = 0; o.woff = (MAPW / 2 - WIN_COLS / 2) & 3;
                    fresh = true;
                    if (l == 0) {
                        e[LDS_WINPOS] = 0x80000000u | (uint32_t)(MAPW / 2) | ((uint32_t)(MAPW / 2) << 8);
                        s_spare_ok[g] = 0; s_pending[g] = 1; s_queue[atomicAdd(&s_qtail, 1) % EPB] = (uint8_t)g;
                    }
                } else if (l == 0) {
                    s_urgent[atomicAdd(&s_nurgent, 1)] = (uint8_t)g;
                }
            }
        }
        __syncthreads();
        // worlds that have to exist now, then queued spare worlds
        bool own = t >= own_from;
#pragma unroll 1
        while (true) {
            const int nurgent = s_nurgent, qhead = s_qhead, qtail = s_qtail;
            int gt;
            bool urgent;
            if (nurgent > 0) { gt = s_urgent[nurgent - 1]; urgent = true; }
            else if (own && qhead != qtail) { gt = s_queue[qhead % EPB]; urgent = false; own = own_from >= 0; }
            else break;
            __syncthreads();                               // everyone has read the counters
            uint32_t* et = s_env + gt * LDS_ENV_DWORDS;
            generate(gt, urgent ? et + LDS_WIN : nullptr);   // ends with a block barrier
            if (urgent) {
                // the record still holds the episode that ended: replace it by the first state of the next
                const uint32_t ep1 = et[LDS_REC + RW_EPISODE] + 1u, lo = et[LDS_REC + RW_SEED_LO], hi = et[LDS_REC + RW_SEED_HI];
                __syncthreads();
                if (tid < REC_DWORDS) et[LDS_REC + tid] = fresh_record_word(tid, lo, hi, ep1);
                if (tid == 0) {
                    et[LDS_WINPOS] = 0x80000000u | (uint32_t)(MAPW / 2) | ((uint32_t)(MAPW / 2) << 8);   // the generator left the start window
                    s_nurgent = nurgent - 1;
                    if (!s_pending[gt]) { s_pending[gt] = 1; s_queue[s_qtail % EPB] = (uint8_t)gt; s_qtail = s_qtail + 1; }
                }
            } else if (tid == 0) {
                s_spare_ok[gt] = 1; s_pending[gt] = 0; s_qhead = qhead + 1;
            }
            __syncthreads();
        }
        // an environment that went through the urgent path starts its episode at the map centre
        // with the window the generator left in LDS
        if (active && o.done && !fresh) { o.mvx = 0; o.mvy = 0; o.woff = (MAPW / 2 - WIN_COLS / 2) & 3; }
        bool staged = false;
        if (active && obs != nullptr) {
            render_symbolic<G, OBS_MODE, true, false>(l, e, o.mvx, o.mvy, o.woff, luts, obs + (size_t)env * obs_stride(OBS_MODE));
            staged = true;
        }
        if (obs != nullptr) {
            if (kBytes && l == 0) e[LDS_FLAG] = staged ? 1u : 0u;
            group_sync();
            const int first = __builtin_amdgcn_readfirstlane((tid & ~63) / G);
            const uint32_t* wave_env = s_env + first * LDS_ENV_DWORDS;
            uint8_t* wave_obs = obs + (size_t)(blockIdx.x * EPB + first) * obs_stride(OBS_MODE);
            // Floats of sixteen lanes are written through at every size: a rollout goes over one buffer again and again, which the last-level
            // cache holds whole (left in the L2 beyond CACHE_SHARE, 16 steps of 18,000 environments 315 us on states in turn and 262 on one, 317 and
            // 244 so, of 24,575 433 and 359, 435 and 344 so).
            if constexpr (kBytes) flush_wave_observations<G, OBS_MODE>(wave_env, wave_obs);
            else flush_wave_floats<G, KeepLayout, G == 16 ? Keep::THROUGH : Keep::PLAIN>(wave_env, wave_obs, __ballot(staged));
        }
        __syncthreads();
    }
    // the records; the tags of the spare worlds that the block has generated (the others are as they were);
    // the worlds owed, for the regeneration launch (on the list that a step launch before it would fill)
    uint4* s_list = reinterpret_cast<uint4*>(s_lat);
    if (active) {
        store_record<G>(l, recs + (size_t)env * 8, e);
        if (s_spare_ok[g]) { if (own_from < steps && l < 2) ls.tags[2 * env + l] = make_uint2(e[LDS_REC + RW_EPISODE] + 1u, 0u); }
        else if (l == 0) s_list[atomicAdd(&s_nurgent, 1)] = make_uint4((uint32_t)env, e[LDS_REC + RW_SEED_LO], e[LDS_REC + RW_SEED_HI], e[LDS_REC + RW_EPISODE] + 1u);
    }
    __syncthreads();
    const int owed = s_nurgent;
    if (owed != 0) la::append_block_entries(ls, *counter(ls, la::CT_SEQ) - 1u, s_list, owed, &s_base, blockIdx.x);
}

// Serves the slow list: generates the world of the new episode in place (one block each, looping
// if the list is longer than the grid), writes the fresh record, renders the first observation,
// and asks the next step launch to generate the world after it.  Runs after the step kernel (which
// has already advanced the launch number), and only when the episode cap is 1.
template <int OBS_MODE>
__global__ __launch_bounds__(WG_THREADS) void k_reset_list(uint4* __restrict__ recs, uint8_t* __restrict__ maps,
                                                      const Luts* __restrict__ luts, uint8_t* __restrict__ obs,
                                                      const uint8_t* __restrict__ done, Lists ls, Params p, int envs_per_turn)
{
    constexpr int G = 16;
    __shared__ uint32_t s_lat[LAT_WORDS];
    __shared__ uint32_t s_env[LDS_ENV_DWORDS];
    __shared__ uint32_t s_rank[WG_THREADS / 64];
    const int tid = threadIdx.x;
    const uint32_t count = la::slow_count(ls, (uint32_t)p.n);
    if (blockIdx.x >= count) return;
    // Optimistic resets: the worlds come from this step's pool (see CRAFTAX_RESET_POOL).  The step
    // kernel has already advanced the launch number: it is the index of the step just done + 2.
    const bool pool = p.reset_mode == CRAFTAX_RESET_POOL;
    const uint32_t step_index = pool ? *la::counter(ls, la::CT_SEQ) - 2u : 0u;
    const uint32_t pool_lo = pool ? reinterpret_cast<const uint32_t*>(recs)[RW_SEED_LO] : 0u;
    const uint32_t pool_hi = pool ? reinterpret_cast<const uint32_t*>(recs)[RW_SEED_HI] : 0u;
    const uint32_t pool_size = (uint32_t)p.n / POOL_RATIO ? (uint32_t)p.n / POOL_RATIO : 1u;
    // the scalars of a fresh episode are constants: fetch their table entries before anything else
    const float fresh_tenth = luts->tenth[MAX_COUNT], fresh_day = luts->daylight[0];
    const uint32_t fresh_q7 = luts->light_q7[0];
    constexpr bool kSymbolic = OBS_MODE != CRAFTAX_OBS_PIXELS_F32;
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
        const uint4 entry = ls.slow[i];
        if (entry.x == ENTRY_VOID) continue;
        const uint32_t env = entry.x, lo = entry.y, hi = entry.z, ep = entry.w;
        uint32_t wlo = lo, whi = hi, wenv = env, wep = ep;          // the world's identity: the environment's own ...
        if (pool) {
            // ... or the pool's: rank of this environment among the finished ones = finished environments before it
            uint32_t before = 0u;
            if ((reinterpret_cast<uintptr_t>(done) & 3u) == 0u) {   // four flags per load
                const uint32_t* d4 = reinterpret_cast<const uint32_t*>(done);
                for (uint32_t j = (uint32_t)tid; j < env / 4u; j += WG_THREADS) before += (uint32_t)__builtin_popcount(d4[j] & 0x01010101u);
                if ((uint32_t)tid < (env & 3u)) before += done[(env & ~3u) + (uint32_t)tid];
            } else {
                for (uint32_t j = (uint32_t)tid; j < env; j += WG_THREADS) before += done[j];
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) before += (uint32_t)__shfl_xor((int)before, d);
            __syncthreads();                                         // the previous entry's ranks have been read
            if ((tid & 63) == 0) s_rank[tid >> 6] = before;
            __syncthreads();
            uint32_t rank = 0u;
#pragma unroll
            for (int w = 0; w < WG_THREADS / 64; ++w) rank += s_rank[w];
            const U4 sh = philox4x32_10(0xFFFFFFFFu, 2u, step_index, DOM_WORLDGEN << 16, pool_lo, pool_hi);
            wlo = pool_lo; whi = pool_hi; wenv = POOL_ENV | ((choice(sh.w[0], pool_size) + rank) % pool_size); wep = step_index;
        }
        uint32_t* grec = reinterpret_cast<uint32_t*>(recs + (size_t)env * 8);
        if (tid >= 64 && tid < 64 + REC_DWORDS) {              // wave 1 writes the record, wave 0 will render
            const uint32_t w = fresh_record_word(tid - 64, lo, hi, ep);
            grec[tid - 64] = w;
            s_env[LDS_REC + tid - 64] = w;
        }
        if (tid == 96 && !pool) la::append_after_step(ls, env / (uint32_t)envs_per_turn, make_uint4(env, lo, hi, ep + 1u));
        // ends with a block barrier
        if (p.worldgen == CRAFTAX_WORLDGEN_PERLIN)
            worldgen_block<WG_THREADS, true>(maps + map_offset(env, ep), s_lat, wlo, whi, wenv, wep, s_env + LDS_WIN, 0, luts->perlin_cs);
        else worldgen_block(maps + map_offset(env, ep), s_lat, wlo, whi, wenv, wep, s_env + LDS_WIN);
        if (kSymbolic && obs != nullptr && tid < G) {
            // scalars of a fresh episode: empty inventory, vitals 9, facing down, noon, awake
            uint32_t* vec = s_env + LDS_VEC;
            for (int i = tid; i < 24; i += G) {
                uint32_t w = 0;
                if (OBS_MODE == CRAFTAX_OBS_SYM_U8_I8) {
                    if (i == 3) w = 0x09090909u;                       // bytes 12..15: the four vitals
                    if (i == 4) w = 1u << 24;                          // byte 19: facing down
                    if (i == 5) w = fresh_q7;                          // byte 20: daylight
                } else {
                    if (i >= 12 && i < 16) w = __float_as_uint(fresh_tenth);
                    if (i == 19) w = __float_as_uint(1.0f);
                    if (i == 20) w = __float_as_uint(fresh_day);
                }
                vec[i] = w;
            }
            render_symbolic<G, OBS_MODE, false>(tid, s_env, 0, 0, (MAPW / 2 - WIN_COLS / 2) & 3, luts, obs + (size_t)env * obs_stride(OBS_MODE));
        }
        __syncthreads();
    }
    la::finish_slow_list(ls, count);
}

template <int OBS_MODE>
__global__ __launch_bounds__(BLOCK) void k_observe(const uint4* __restrict__ recs, const uint8_t* __restrict__ maps,
                                                   const Luts* __restrict__ luts, uint8_t* __restrict__ obs, Params p)
{
    constexpr int G = 16, EPB = Grp<G>::EPB;
    __shared__ uint32_t s_env[EPB * LDS_ENV_DWORDS];
    const int tid = threadIdx.x, g = tid / G, l = tid % G;
    const int env = blockIdx.x * EPB + g;
    if (env >= p.n) return;
    uint32_t* e = s_env + g * LDS_ENV_DWORDS;
    load_record<G>(l, recs + (size_t)env * 8, e);
    group_sync();
    const uint32_t w_pos = e[LDS_REC + RW_POS];
    const int px = w_pos & 0xFF;
    load_window<G>(l, px, (w_pos >> 8) & 0xFF, maps + map_offset((uint32_t)env, e[LDS_REC + RW_EPISODE]), e + LDS_WIN);
    group_sync();
    render_symbolic<G, OBS_MODE>(l, e, 0, 0, (px - WIN_COLS / 2) & 3, luts, obs + (size_t)env * obs_stride(OBS_MODE));
}

__global__ __launch_bounds__(BLOCK) void k_pixels(const uint4* __restrict__ recs, const uint8_t* __restrict__ maps,
                                                  const Luts* __restrict__ luts, uint8_t* __restrict__ obs, Params p)
{
    __shared__ uint32_t s_rec[REC_DWORDS];
    __shared__ int s_tile[PIX_CELLS], s_ent[PIX_CELLS];
    __shared__ __attribute__((aligned(16))) float s_strip[PIX_STRIP_FLOATS];
    const int env = blockIdx.x;
    if (threadIdx.x < REC_DWORDS) s_rec[threadIdx.x] = reinterpret_cast<const uint32_t*>(recs + (size_t)env * 8)[threadIdx.x];
    __syncthreads();
    const uint8_t* map = maps + map_offset((uint32_t)env, s_rec[RW_EPISODE]);
    uint8_t* out = obs + (size_t)env * OBS_STRIDE_PIXELS;
    if (picture_kept(p.n, env, blockIdx.x)) render_pixels_block<Keep::THROUGH>(s_rec, map, luts, out, s_tile, s_ent, s_strip);
    else render_pixels_block<Keep::STREAM>(s_rec, map, luts, out, s_tile, s_ent, s_strip);
}

// ---------------------------------------------------------------------------------------------
// canonical dumps: one block per environment
__global__ __launch_bounds__(BLOCK) void k_export(const uint4* __restrict__ recs, const uint8_t* __restrict__ maps,
                                                  craftax_env_dump* __restrict__ dumps, int first)
{
    const int env = first + blockIdx.x, tid = threadIdx.x;
    craftax_env_dump* d = dumps + blockIdx.x;
    __shared__ uint32_t r[REC_DWORDS];
    if (tid < REC_DWORDS) r[tid] = reinterpret_cast<const uint32_t*>(recs + (size_t)env * 8)[tid];
    __syncthreads();
    {   // 16-byte piece tid of the tiled map = row (tid & 7) of tile (tid >> 3) -> row-major dump
        const int tile = tid >> 3, y = ((tile >> 2) << 3) + (tid & 7), x = (tile & 3) << 4;
        *reinterpret_cast<uint4*>(d->map + y * MAPW + x) = reinterpret_cast<const uint4*>(maps + map_offset((uint32_t)env, r[RW_EPISODE]))[tid];
    }
    if (tid == 0) {
        d->px = r[RW_POS] & 0xFF; d->py = (r[RW_POS] >> 8) & 0xFF; d->dir = (r[RW_POS] >> 16) & 0xFF; d->sleeping = r[RW_POS] >> 24;
        for (int i = 0; i < 6; ++i) { d->inv[i] = (r[RW_INV] >> (4 * i)) & 15; d->inv[6 + i] = (r[RW_INV] >> (24 + i)) & 1; }
        for (int i = 0; i < 4; ++i) { d->vit[i] = (int8_t)((r[RW_VIT] >> (4 * i)) & 15); d->cnt[i] = (int16_t)(int8_t)(r[RW_CNT] >> (8 * i)); }
        d->ach = r[RW_ACH]; d->t = r[RW_T]; d->episode = r[RW_EPISODE];
        d->seed = (uint64_t)r[RW_SEED_LO] | ((uint64_t)r[RW_SEED_HI] << 32);
        d->env = (uint32_t)env;
    }
    if (tid < NMOB) {
        const Mob m = unpack_mob(r[RW_MOB + tid]);
        craftax_mob o;
        o.alive = m.alive; o.x = m.x; o.y = m.y; o.dir = m.dir; o.hp = (int8_t)m.hp; o.cd = m.cd; o.pad[0] = 0; o.pad[1] = 0;
        d->mob[tid] = o;
    }
    if (tid >= 32 && tid < 32 + NPLANT) {
        const Plant q = unpack_plant(r[RW_PLANT + tid - 32]);
        craftax_plant o;
        o.alive = q.alive; o.x = q.x; o.y = q.y; o.pad = 0; o.age = (uint16_t)q.age;
        d->plant[tid - 32] = o;
    }
}

// Import packs into the record's bit fields: counts and vitals 0..15, counters -128..127, mob hp
// and cooldown 0..15, coordinates 0..63, block ids 1..16 (every state the rules can reach is);
// values outside are brought into range so that no kernel ever indexes beyond its tables or
// buffers: a block id outside the table becomes BK_OOB.
__device__ inline uint32_t sanitise_blocks(uint32_t four)
{
    uint32_t out = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b = (four >> (8 * i)) & 0xFFu;
        out |= (b - 1u < 16u ? b : (uint32_t)BK_OOB) << (8 * i);
    }
    return out;
}
__global__ __launch_bounds__(BLOCK) void k_import(uint4* __restrict__ recs, uint8_t* __restrict__ maps, Lists ls,
                                                  const craftax_env_dump* __restrict__ dumps, int first, Params p)
{
    const int env = first + blockIdx.x, tid = threadIdx.x;
    const craftax_env_dump* d = dumps + blockIdx.x;
    {
        const int tile = tid >> 3, y = ((tile >> 2) << 3) + (tid & 7), x = (tile & 3) << 4;
        const uint4 v = *reinterpret_cast<const uint4*>(d->map + y * MAPW + x);
        reinterpret_cast<uint4*>(maps + map_offset((uint32_t)env, d->episode))[tid] =
            make_uint4(sanitise_blocks(v.x), sanitise_blocks(v.y), sanitise_blocks(v.z), sanitise_blocks(v.w));
    }
    // whatever was queued for this environment belongs to the episode that is being replaced
    la::cancel_entries(ls, (uint32_t)env);
    __shared__ uint32_t r[REC_DWORDS];
    if (tid < REC_DWORDS) r[tid] = 0;
    __syncthreads();
    if (tid == 0) {
        r[RW_POS] = (uint32_t)(d->px & 63) | ((uint32_t)(d->py & 63) << 8) | ((uint32_t)(d->dir & 7) << 16) | ((uint32_t)(d->sleeping & 1) << 24);
        uint32_t wi = 0, wv = 0, wc = 0;
        for (int i = 0; i < 6; ++i) wi |= ((uint32_t)(d->inv[i] & 15) << (4 * i)) | ((uint32_t)(d->inv[6 + i] & 1) << (24 + i));
        for (int i = 0; i < 4; ++i) {
            wv |= (uint32_t)(d->vit[i] & 15) << (4 * i);
            const int c = max(-128, min(127, (int)d->cnt[i]));
            wc |= (uint32_t)(c & 0xFF) << (8 * i);
        }
        r[RW_INV] = wi;
        r[RW_VIT] = wv | ((d->t % p.day_length) << 16);
        r[RW_CNT] = wc;
        r[RW_ACH] = d->ach; r[RW_T] = d->t; r[RW_EPISODE] = d->episode;
        r[RW_SEED_LO] = (uint32_t)d->seed; r[RW_SEED_HI] = (uint32_t)(d->seed >> 32);
    }
    if (tid < NMOB) {
        const craftax_mob s = d->mob[tid];
        Mob m;
        m.alive = s.alive & 1; m.x = s.x & 63; m.y = s.y & 63; m.dir = s.dir & 7; m.hp = s.hp & 15; m.cd = s.cd & 15;
        r[RW_MOB + tid] = pack_mob(m);
    }
    if (tid >= 32 && tid < 32 + NPLANT) {
        const craftax_plant s = d->plant[tid - 32];
        Plant q;
        q.alive = s.alive & 1; q.x = s.x & 63; q.y = s.y & 63; q.age = s.age;
        r[RW_PLANT + tid - 32] = pack_plant(q);
    }
    __syncthreads();
    if (tid < REC_DWORDS) reinterpret_cast<uint32_t*>(recs + (size_t)env * 8)[tid] = r[tid];
}

// after an import: the world of the episode after the imported one, into the spare slot
template <bool PERLIN>
__global__ __launch_bounds__(WG_THREADS, 8) void k_import_spare(const uint4* __restrict__ recs, uint8_t* __restrict__ maps, Lists ls, int first,
                                                                             const Luts* __restrict__ luts)
{
    __shared__ uint32_t s_lat[lattice_words<PERLIN>];
    const uint32_t env = (uint32_t)first + blockIdx.x;
    const uint32_t* r = reinterpret_cast<const uint32_t*>(recs + (size_t)env * 8);
    const uint32_t ep = r[RW_EPISODE] + 1u, lo = r[RW_SEED_LO], hi = r[RW_SEED_HI];
    worldgen_block<WG_THREADS, PERLIN>(maps + map_offset(env, ep), s_lat, lo, hi, env, ep, nullptr, 0, luts->perlin_cs);
    if (threadIdx.x < 2) ls.tags[2 * env + threadIdx.x] = make_uint2(ep, 0u);
}

// Level mutation (section "Craftax-1B: UED"): swaps two tiles of different type, one of them in
// the central 16x16 area; restricted: only stone <-> ores and grass <-> tree.  Up to 32 tries, one lane
// each (a thread that walked through them made a chain of up to 64 trips to memory, on a handful of
// wavefronts: 1,000 levels 11.2 -> 4.8 us); try k draws Philox block (env, round, 0, MUTATE | k) under the
// mutation seed (word 0: the central cell, word 1: any cell), and the first one is carried out whose
// blocks differ, whose cells hold neither the player nor a live mob nor a plant, and, restricted,
// whose blocks are of one group.
__device__ inline int swap_group(int b)
{
    if (b == BK_STONE || b == BK_COAL || b == BK_IRON || b == BK_DIAMOND) return 1;
    if (b == BK_GRASS || b == BK_TREE) return 2;
    return 0;
}
__global__ void k_mutate_swap(const uint4* __restrict__ recs, uint8_t* __restrict__ maps, int first, int count, uint32_t k0,
                              uint32_t k1, uint32_t round, int restricted, int32_t* __restrict__ tries)
{
    const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) / MUTATE_TRIES), k = threadIdx.x % MUTATE_TRIES;
    if (i >= count) return;
    const uint32_t env = (uint32_t)(first + i);
    const uint32_t* r = reinterpret_cast<const uint32_t*>(recs + (size_t)env * 8);
    uint8_t* map = maps + map_offset(env, r[RW_EPISODE]);
    const int px = r[RW_POS] & 0xFF, py = (r[RW_POS] >> 8) & 0xFF;
    auto taken = [&](int x, int y) {
        bool t = x == px && y == py;
        for (int k = 0; k < NMOB; ++k) {
            const Mob m = unpack_mob(r[RW_MOB + k]);
            t |= m.alive && (int)m.x == x && (int)m.y == y;
        }
        return t;
    };
    const U4 d = philox4x32_10(env, round, 0u, (DOM_MUTATE << 16) | (uint32_t)k, k0, k1);
    const int a = (int)choice(d.w[0], MUTATE_AREA * MUTATE_AREA), b = (int)choice(d.w[1], MAPW * MAPW);
    const int c0 = (MAPW - MUTATE_AREA) / 2;
    const int ax = c0 + a % MUTATE_AREA, ay = c0 + a / MUTATE_AREA, bx = b % MAPW, by = b / MAPW;
    const int ba = map[map_index(ax, ay)], bb = map[map_index(bx, by)];
    bool accepted = ba != bb && !taken(ax, ay) && !taken(bx, by);
    accepted = accepted && ba != BK_PLANT && ba != BK_RIPE && bb != BK_PLANT && bb != BK_RIPE;
    accepted = accepted && (!restricted || (swap_group(ba) != 0 && swap_group(ba) == swap_group(bb)));
    const uint32_t good = (uint32_t)(__ballot(accepted) >> (threadIdx.x & 32u));
    const int done = __ffs((int)good);          // number of the first such try, counted from 1, or 0
    if (done == k + 1) {
        map[map_index(ax, ay)] = (uint8_t)bb;
        map[map_index(bx, by)] = (uint8_t)ba;
    }
    if (tries != nullptr && k == 0) tries[i] = done;
}

// Noise mutation (section "Craftax-1B: UED"): one block per environment.  The level is the vector of
// Perlin gradient angles; every element gets a uniform offset in [-amplitude, amplitude] (u16
// number i of stream (round, 1) of the mutation domain), the world of the current episode is
// generated again from the new angles and the episode starts over in it.
__global__ __launch_bounds__(WG_THREADS) void k_mutate_noise(uint4* __restrict__ recs, uint8_t* __restrict__ maps,
                                                            const Luts* __restrict__ luts, uint16_t* __restrict__ theta, int first,
                                                            uint32_t k0, uint32_t k1, uint32_t round, uint32_t amplitude)
{
    __shared__ uint32_t s_lat[LAT_WORDS];
    __shared__ uint16_t s_theta[LAT_BLOCKS * 8];
    const int tid = threadIdx.x;
    const uint32_t env = (uint32_t)first + blockIdx.x;
    uint32_t* r = reinterpret_cast<uint32_t*>(recs + (size_t)env * 8);
    const uint32_t ep = r[RW_EPISODE], lo = r[RW_SEED_LO], hi = r[RW_SEED_HI];
    uint16_t* th = theta + (size_t)blockIdx.x * LAT_TOTAL;
    if (tid < LAT_BLOCKS) {
        const U4 d = philox4x32_10(env, round, 1u, (DOM_MUTATE << 16) | (uint32_t)tid, k0, k1);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = tid * 8 + j;
            if (i < LAT_TOTAL) {
                const uint32_t w = d.w[j >> 1], d16 = (j & 1) ? (w >> 16) : (w & 0xFFFFu);
                const int u = (int)((d16 * (2u * amplitude + 1u)) >> 16) - (int)amplitude;
                const uint16_t v = (uint16_t)(((int)(th[i] & 1023u) + u) & 1023);
                th[i] = v;
                s_theta[i] = v;
            }
        }
    }
    __syncthreads();   // every thread has read the record before the new one is written below
    worldgen_block<WG_THREADS, true>(maps + map_offset(env, ep), s_lat, lo, hi, env, ep, nullptr, 0, luts->perlin_cs, s_theta);
    if (tid < REC_DWORDS) r[tid] = fresh_record_word(tid, lo, hi, ep);
}

// synthetic action stream (input generation for benchmarks; not part of the simulator)
__global__ void k_synth_actions(int32_t* __restrict__ actions, int n, int step0, int steps, uint32_t k0, uint32_t k1, int kind)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)n * (size_t)steps) return;
    const uint32_t s = (uint32_t)(i / (size_t)n), env = (uint32_t)(i % (size_t)n);
    const U4 r = philox4x32_10(env, (uint32_t)step0 + s, 0u, DOM_ACTIONS << 16, k0, k1);
    const uint32_t count = kind >= 2 ? 43u : (uint32_t)AC_COUNT;   // appendix "Action Space": 17 Classic, 43 Craftax
    int a;
    if ((kind & 1) == 0) a = (int)choice(r.w[0], count);
    else a = r.w[0] < 0x80000000u ? 1 + (int)choice(r.w[1], 5) : (int)choice(r.w[1], count);
    actions[i] = a;
}

// ---------------------------------------------------------------------------------------------
// Metrics: a snapshot over the records (both variants; the layout of a record is passed in).  One
// block per 256 environments leaves a partial result (achievement counts, episodes, steps) in a
// scratch buffer; a second, single-block kernel adds the partial results up.  No atomics on global
// memory, so the result is independent of the order in which blocks run.
constexpr int STATS_ENVS_PER_BLOCK = 256;
constexpr int STATS_A = CRAFTAX_STATS_ACHIEVEMENTS;
constexpr int STATS_PARTIAL_WORDS = 256;     // 96 counts of running episodes, 96 unlock counts, episodes and steps as two words each, padding to 1 KiB
static_assert(2 * STATS_A + 4 <= STATS_PARTIAL_WORDS, "a partial result holds both histograms and the two sums");

__global__ __launch_bounds__(STATS_ENVS_PER_BLOCK) void k_stats_partial(cf::host::RecordLayout ly, int n, uint32_t* __restrict__ partial)
{
    __shared__ uint32_t s_hist[2 * STATS_A];
    __shared__ unsigned long long s_sum[2];
    const int tid = threadIdx.x, env = blockIdx.x * STATS_ENVS_PER_BLOCK + tid;
    if (tid < 2 * STATS_A) s_hist[tid] = 0u;
    if (tid < 2) s_sum[tid] = 0ull;
    __syncthreads();
    const bool valid = env < n;
    const uint32_t* r = ly.recs + (size_t)(valid ? env : 0) * ly.stride;
    unsigned long long episodes = valid ? r[ly.episode] : 0u, steps = valid ? r[ly.t] : 0u;
    for (int w = 0; w < ly.ach_words; ++w) {
        const uint32_t a = valid ? r[ly.ach + w] : 0u;
#pragma unroll 4
        for (int b = 0; b < 32; ++b) {
            const uint32_t c = (uint32_t)__popcll(__ballot((a >> b) & 1u));
            if ((tid & 63) == 0 && c) atomicAdd(&s_hist[w * 32 + b], c);
        }
    }
    // the unlock counters of this block's environments lie one after the other: read them in order
    const int first = blockIdx.x * STATS_ENVS_PER_BLOCK, envs = min(STATS_ENVS_PER_BLOCK, n - first);
    const uint32_t* u = ly.unlocks + (size_t)first * ly.unlock_stride;
    for (int i = tid; i < envs * ly.unlock_stride; i += STATS_ENVS_PER_BLOCK) {
        const int k = i % ly.unlock_stride;
        const uint32_t c = u[i];
        if (c && k < STATS_A) atomicAdd(&s_hist[STATS_A + k], c);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        episodes += (unsigned long long)__shfl_xor((long long)episodes, d);
        steps += (unsigned long long)__shfl_xor((long long)steps, d);
    }
    if ((tid & 63) == 0) { atomicAdd(&s_sum[0], episodes); atomicAdd(&s_sum[1], steps); }
    __syncthreads();
    uint32_t* out = partial + (size_t)blockIdx.x * STATS_PARTIAL_WORDS;
    if (tid < 2 * STATS_A) out[tid] = s_hist[tid];
    if (tid >= 2 * STATS_A && tid < 2 * STATS_A + 4) {
        const int j = tid - 2 * STATS_A;
        out[tid] = (uint32_t)(s_sum[j >> 1] >> (32 * (j & 1)));
    }
}

// 1024 threads: thread (g, j) adds word j of the partial results g, g + 4, ... (independent loads, so
// they are all in flight together), then the four part sums of a word meet in LDS.
constexpr int STATS_TOTAL_THREADS = 1024;
__global__ __launch_bounds__(STATS_TOTAL_THREADS) void k_stats_total(const uint32_t* __restrict__ partial, int blocks, int n, craftax_metrics* __restrict__ out)
{
    constexpr int PARTS = STATS_TOTAL_THREADS / STATS_PARTIAL_WORDS;
    __shared__ unsigned long long s_part[PARTS][STATS_PARTIAL_WORDS];
    const int j = threadIdx.x % STATS_PARTIAL_WORDS, g = threadIdx.x / STATS_PARTIAL_WORDS;
    // words 0..191 are 32-bit counts; 192..195 the halves of two 64-bit sums, added as 64-bit numbers by the even word
    unsigned long long c = 0;
    const bool wide = j >= 2 * STATS_A && j < 2 * STATS_A + 4;
    if (j < 2 * STATS_A || (wide && (j & 1) == 0)) {
#pragma unroll 4
        for (int b = g; b < blocks; b += PARTS) {
            const uint32_t* p = partial + (size_t)b * STATS_PARTIAL_WORDS + j;
            c += wide ? ((unsigned long long)p[0] | ((unsigned long long)p[1] << 32)) : (unsigned long long)p[0];
        }
    }
    s_part[g][j] = c;
    __syncthreads();
    if (g != 0) return;
#pragma unroll
    for (int k = 1; k < PARTS; ++k) c += s_part[k][j];
    if (j < STATS_A) out->achievements[j] = (uint32_t)c;
    else if (j < 2 * STATS_A) out->unlocks[j - STATS_A] = c;
    else if (j == 2 * STATS_A) out->episodes = c;
    else if (j == 2 * STATS_A + 2) out->steps = c;
    else if (j == 2 * STATS_A + 4) { out->n = (uint32_t)n; out->pad = 0u; }
}

// Scratch of craftax_stats_static: the partial results of up to STATS_STATIC_BLOCKS blocks, inside the
// library's device image (every GPU the library runs on holds its own copy).  Host code never uses
// this name as an address: it asks the runtime for the device address once per device
// (stats_scratch_address) and passes that pointer to the kernels.
constexpr int STATS_STATIC_BLOCKS = CRAFTAX_STATS_STATIC_MAX_ENVS / STATS_ENVS_PER_BLOCK;
static __device__ __align__(256) uint32_t scratch[(size_t)STATS_STATIC_BLOCKS * STATS_PARTIAL_WORDS];

#ifdef CRAFTAX_DEBUG_BOUNDS
// forms index 5 into a four-element table through the checked path: caught, replaced by 0
__global__ void k_bounds_selftest(uint32_t* out)
{
    const uint32_t table[4] = {11u, 22u, 33u, 44u};
    out[0] = table[CX_IDX((int)threadIdx.x + 5, 4)];
}
#endif

// ---------------------------------------------------------------------------------------------
// host side
struct HostState {
    craftax_config cfg;
    int n;
    int lanes;   // lanes per environment used by the step kernel
    Header hdr;
    bool has_worlds;   // craftax_reset has run (or the blob was attached): records, maps and tags are valid
    bool serve_slow;   // the next step also launches the slow-list kernel (see note_edit)
};

static std::mutex g_mutex;
static std::unordered_map<const void*, HostState> g_states;
static thread_local std::string g_error;

static int fail(int code, const std::string& msg)
{
    g_error = msg;
    return code;
}

static bool config_ok(const craftax_config* c, std::string* why)
{
    if (c->variant == CRAFTAX_VARIANT_CRAFTAX) return cf::host::config_ok(c, why);
    if (c->abi_version != CRAFTAX_ABI_VERSION) { *why = "abi_version mismatch"; return false; }
    if (c->variant != CRAFTAX_VARIANT_CLASSIC) { *why = "unknown variant"; return false; }
    if (c->obs_mode > CRAFTAX_OBS_PIXELS_F32) { *why = "unknown obs_mode"; return false; }
    if (c->worldgen > CRAFTAX_WORLDGEN_PERLIN) { *why = "unknown worldgen"; return false; }
    if (c->reset_mode > CRAFTAX_RESET_POOL) { *why = "unknown reset_mode"; return false; }
    if (c->day_length < 2 || c->day_length > MAX_DAY || (c->day_length & 1)) { *why = "day_length must be even and in 2..1024"; return false; }
    if (c->cap_zombie > 3 || c->cap_cow > 3 || c->cap_skeleton > 3 || c->cap_arrow > 3) { *why = "mob caps must be 0..3"; return false; }
    if (c->cap_plant > NPLANT) { *why = "cap_plant must be 0..10"; return false; }
    if (c->max_episode_steps == 0) { *why = "max_episode_steps must be positive"; return false; }
    if (c->group_lanes != 0 && c->group_lanes != 4 && c->group_lanes != 8 && c->group_lanes != 16) { *why = "group_lanes must be 0, 4, 8 or 16"; return false; }
    if (c->reserved != 0) { *why = "reserved must be 0"; return false; }
    return true;
}

static uint64_t round_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

static uint64_t sub_list_capacity(int n) { return la::sub_list_capacity((uint64_t)n, 64); }   // 64 environments per block at 4 lanes each

static Header make_header(const craftax_config* c, int n)
{
    Header h;
    std::memset(&h, 0, sizeof(h));
    h.magic = MAGIC; h.version = CRAFTAX_ABI_VERSION; h.n = (uint32_t)n;
    h.obs_mode = c->obs_mode; h.max_episode_steps = c->max_episode_steps; h.day_length = c->day_length;
    h.cap_zombie = c->cap_zombie; h.cap_cow = c->cap_cow; h.cap_skeleton = c->cap_skeleton;
    h.cap_arrow = c->cap_arrow; h.cap_plant = c->cap_plant; h.atlas_seed = c->atlas_seed;
    h.variant = c->variant; h.worldgen = c->worldgen; h.reset_mode = c->reset_mode;
    h.off_ctrs = HEADER_BYTES;
    h.off_luts = h.off_ctrs + la::COUNTER_BYTES;
    h.off_recs = round_up(h.off_luts + sizeof(Luts), 256);
    h.off_maps = h.off_recs + (uint64_t)n * (REC_DWORDS * 4);
    h.off_tags = h.off_maps + (uint64_t)n * 2 * (MAPW * MAPW);     // two map slots per environment
    h.off_regen0 = round_up(h.off_tags + (uint64_t)n * 16, 256);
    const uint64_t list_bytes = (uint64_t)NSUB * sub_list_capacity(n) * 16;
    h.off_regen1 = h.off_regen0 + list_bytes;
    h.off_slow = h.off_regen1 + list_bytes;
    h.off_unlocks = round_up(h.off_slow + (uint64_t)n * 16, 256);
    h.total = round_up(h.off_unlocks + (uint64_t)n * UNLOCK_STRIDE * 4, 256);
    return h;
}

// Lookup tables.  Day/night: phase i = t mod L, H = L/2, k = |i - H|, daylight =
// smoothstep(k/H) = k^2 (3H - 2k) / H^3 (noon at t = 0, midnight at t = H): the paper only
// says the observation carries a day/night value in [0,1] (appendix "Observation Space").
static void build_luts(const craftax_config* c, Luts* L)
{
    std::memset(L, 0, sizeof(*L));
    const uint64_t len = c->day_length, half = len / 2, den = half * half * half;
    for (uint64_t i = 0; i < len; ++i) {
        const uint64_t k = i < half ? half - i : i - half;
        const uint64_t num = k * k * (3 * half - 2 * k);
        L->daylight[i] = (float)((double)num / (double)den);
        const uint32_t dark = 255u - (uint32_t)(255u * num / den);
        L->zombie_thr[i] = (40u + 3u * dark) << 20;
        L->light_q7[i] = (uint8_t)(127u * num / den);
    }
    for (int i = 0; i < 16; ++i) {
        L->sqrt10[i] = (float)(std::sqrt((double)i) / 10.0);
        L->tenth[i] = (float)((double)i / 10.0);
    }
    const uint32_t k0 = (uint32_t)c->atlas_seed, k1 = (uint32_t)(c->atlas_seed >> 32);
    auto word = [&](uint32_t stream, uint32_t idx) {
        const U4 r = philox4x32_10(0u, stream, 0u, (DOM_ATLAS << 16) | (idx >> 2), k0, k1);
        return r.w[idx & 3u];
    };
    for (uint32_t i = 0; i < 16 * 147; ++i) L->tile[i] = (float)(word(0, i) >> 8) * (1.0f / 16777216.0f);
    for (uint32_t i = 0; i < 5 * 147; ++i) L->ent[i] = (float)(word(1, i) >> 8) * (1.0f / 16777216.0f);
    for (uint32_t i = 0; i < 5 * 49; ++i) L->ent_mask[i] = (uint8_t)(word(2, i) >> 31);
    // unit gradients of the 1024 Perlin directions in Q14, rounded to nearest
    for (int a = 0; a < 1024; ++a) {
        const double turn = 6.283185307179586476925286766559 * (double)a / 1024.0;
        const int16_t c16 = (int16_t)std::lround(std::cos(turn) * 16384.0), s16 = (int16_t)std::lround(std::sin(turn) * 16384.0);
        L->perlin_cs[a] = (uint32_t)(uint16_t)c16 | ((uint32_t)(uint16_t)s16 << 16);
    }
}

static Params make_params(const void* state, const HostState& s)
{
    Params p;
    p.n = s.n;
    p.unlocks = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(static_cast<const uint8_t*>(state)) + s.hdr.off_unlocks);
    p.max_episode_steps = s.cfg.max_episode_steps; p.day_length = s.cfg.day_length;
    p.cap_zombie = s.cfg.cap_zombie; p.cap_cow = s.cfg.cap_cow; p.cap_skeleton = s.cfg.cap_skeleton;
    p.cap_arrow = s.cfg.cap_arrow; p.cap_plant = s.cfg.cap_plant; p.worldgen = s.cfg.worldgen; p.reset_mode = s.cfg.reset_mode;
    return p;
}

static int lookup(const void* state, int n, bool need_n, HostState* out)
{
    if (state == nullptr) return fail(CRAFTAX_E_NULL, "state is NULL");
    std::lock_guard<std::mutex> lock(g_mutex);
    auto it = g_states.find(state);
    if (it == g_states.end()) return fail(CRAFTAX_E_STATE, "state was not initialised by craftax_state_init or attached by craftax_state_attach");
    if (need_n && n != it->second.n) return fail(CRAFTAX_E_COUNT, "n differs from the n given to craftax_state_init");
    *out = it->second;
    return CRAFTAX_OK;
}
// Checked last among a call's arguments, by every call that reads records or maps: they hold
// nothing before the first craftax_reset.
static int need_worlds(const HostState& s)
{
    return s.has_worlds ? CRAFTAX_OK : fail(CRAFTAX_E_STATE, "the state holds no worlds yet: call craftax_reset first");
}

static void update_state(const void* state, bool has_worlds, bool serve_slow)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    auto it = g_states.find(state);
    if (it == g_states.end()) return;
    it->second.has_worlds = has_worlds;
    it->second.serve_slow = serve_slow;
}
// An episode that ends finds its next world ready unless it ends on its very first step, which a
// fresh episode cannot do by the rules.  An edit between the step that started the episode and its
// first own step can make it (a swap that puts lava next to the start): after every call that edits
// worlds, the next step therefore also launches the kernel that serves such episodes.
static void note_edit(const void* state) { update_state(state, true, true); }

static int check_launch(const char* what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
    return CRAFTAX_OK;
}

struct Ptrs { uint4* recs; uint8_t* maps; const Luts* luts; Lists ls; };
static Ptrs pointers(const void* state, const HostState& s)
{
    uint8_t* base = const_cast<uint8_t*>(static_cast<const uint8_t*>(state));
    Ptrs q;
    q.luts = reinterpret_cast<const Luts*>(base + s.hdr.off_luts);
    q.recs = reinterpret_cast<uint4*>(base + s.hdr.off_recs);
    q.maps = base + s.hdr.off_maps;
    q.ls.ctr = reinterpret_cast<uint32_t*>(base + s.hdr.off_ctrs);
    q.ls.sub_cap = (uint32_t)sub_list_capacity(s.n);
    q.ls.slow_cap = (uint32_t)s.n;
    q.ls.regen[0] = reinterpret_cast<uint4*>(base + s.hdr.off_regen0);
    q.ls.regen[1] = reinterpret_cast<uint4*>(base + s.hdr.off_regen1);
    q.ls.slow = reinterpret_cast<uint4*>(base + s.hdr.off_slow);
    q.ls.tags = reinterpret_cast<uint2*>(base + s.hdr.off_tags);
    return q;
}

// Lanes per environment: few lanes amortise the per-environment scalar work over more
// environments per wave and win once there are enough environments to fill the chip; many
// lanes give more, shorter waves and win for small batches.  cfg->group_lanes = 4, 8 or 16
// overrides the choice (for tuning).  The lanes belong to the state, whatever its calls are, and no line suits all of these (us with 16 / 8 / 4 lanes,
// three states in turn).  Steps without an observation 12,288 9.7 / 10.0 / 11.2, 16,384 11.3 / 10.3 / 11.3, 32,768 17.7 / 14.3 / 14.8, 45,000 22.0 / 17.9 / 16.7;
// floats 12,288 16.7 / 19.0 / 20.6, 14,000 22.0 / 20.4 / 22.1, 32,768 55.2 / 51.0 / 54.5, 65,536 104.8 / 102.2 / 103.7; bytes 8,192
// 9.2 / 12.3 / 14.6, 16,384 13.9 / 15.3 / 15.7, 20,480 16.2 / 17.1 / 19.5, 24,576 18.8 / 18.1 / 20.2, 32,768 26.2 / 20.8 / 22.4, 45,000
// 35.0 / 33.3 / 29.9.  The lower line is that of the first two (bytes alone would stay with sixteen lanes to about 21,000), the upper one that
// of rollouts, which have sixteen lanes or four (a step of a rollout 20,000 13.1 / 13.3, 24,576 14.5 / 13.7, 32,768 18.0 / 14.8; steps alone would stay with eight to about 41,000).
static int group_lanes(const craftax_config* cfg, int n)
{
    const int g = (int)cfg->group_lanes;
    if (g == 4 || g == 8 || g == 16) return g;
    return n >= 24576 ? 4 : (n >= 12288 ? 8 : 16);
}

constexpr int RESET_GRID = 64;    // blocks of k_reset_list (the slow list is nearly always empty); each loops over the list
constexpr int FULL_LIST_GRID = 512;    // the same where every finished episode is on that list (4,096 environments with episodes of one step, 64 blocks 349 us, 512: 129)
constexpr int REGEN_BLOCKS = 1024; // regeneration blocks appended to the step grid (two per world); those beyond the list exit at once
constexpr int OWED_BLOCKS = COMPUTE_UNITS * DRAIN_BLOCKS_PER_CU;   // regeneration blocks behind a rollout: all that the chip holds at once
constexpr int SHARED_REGEN_BLOCKS = 256;   // with four lanes per environment: one per compute unit, beside its four step blocks (see regeneration_share)

template <int OBS_MODE>
static void launch_step(int G, int n, hipStream_t st, const Ptrs& q, const int32_t* actions, uint8_t* o, float* reward,
                        uint8_t* done, const Params& p, bool serve_slow)
{
    const dim3 block(BLOCK);
    const int most = G == 4 ? SHARED_REGEN_BLOCKS : REGEN_BLOCKS;
    const int regen = ((2 * n < most ? 2 * n : most) + 2 * NSUB - 1) / (2 * NSUB) * (2 * NSUB);   // a multiple of twice the sub-list count
    const int sb = (n + 256 / G - 1) / (256 / G);
    const bool perlin = p.worldgen == CRAFTAX_WORLDGEN_PERLIN;
    // with optimistic resets every finished episode is served after the step, because its world depends on who else
    // finished, and with an episode cap of 1 every episode has finished; else the list is nearly always empty, and it is
    // served only where an episode can have ended before its spare world existed: see note_edit
    const bool all = p.reset_mode == CRAFTAX_RESET_POOL || p.max_episode_steps == 1u;
    if (OBS_MODE == CRAFTAX_OBS_PIXELS_F32 && o != nullptr && !all && !serve_slow) {
        // step and picture in one launch, whatever the lanes of a step without
        const int beside = ((2 * n < REGEN_BLOCKS ? 2 * n : REGEN_BLOCKS) + 2 * NSUB - 1) / (2 * NSUB) * (2 * NSUB);
        if (perlin) hipLaunchKernelGGL((k_step<16, CRAFTAX_OBS_PIXELS_F32, true, true>), dim3(n + beside), block, 0, st, q.recs, q.maps, q.luts, actions, o, reward, done, q.ls, p, n);
        else hipLaunchKernelGGL((k_step<16, CRAFTAX_OBS_PIXELS_F32, false, true>), dim3(n + beside), block, 0, st, q.recs, q.maps, q.luts, actions, o, reward, done, q.ls, p, n);
        return;
    }
#define CRAFTAX_LAUNCH_STEP(LANES, NOISE) \
    hipLaunchKernelGGL((k_step<LANES, OBS_MODE, NOISE>), dim3(sb + regen), block, 0, st, q.recs, q.maps, q.luts, actions, o, reward, done, q.ls, p, sb)
    if (G == 4) { if (perlin) CRAFTAX_LAUNCH_STEP(4, true); else CRAFTAX_LAUNCH_STEP(4, false); }
    else if (G == 8) { if (perlin) CRAFTAX_LAUNCH_STEP(8, true); else CRAFTAX_LAUNCH_STEP(8, false); }
    else { if (perlin) CRAFTAX_LAUNCH_STEP(16, true); else CRAFTAX_LAUNCH_STEP(16, false); }
#undef CRAFTAX_LAUNCH_STEP
    const int most_served = all ? FULL_LIST_GRID : RESET_GRID;
    if (all || serve_slow)
        hipLaunchKernelGGL((k_reset_list<OBS_MODE>), dim3(n < most_served ? n : most_served), dim3(WG_THREADS), 0, st, q.recs, q.maps, q.luts, o, done, q.ls, p, envs_per_list_turn(G));
    if (OBS_MODE == CRAFTAX_OBS_PIXELS_F32 && o != nullptr) hipLaunchKernelGGL(k_pixels, dim3(n), block, 0, st, q.recs, q.maps, q.luts, o, p);
}

template <int OBS_MODE>
static void launch_rollout(int lanes, int n, hipStream_t st, const Ptrs& q, const int32_t* actions, int steps, uint8_t* o,
                           float* reward, uint8_t* done, const Params& p)
{
    // launches of regeneration blocks only bring every spare world up to date and empty the lists: before
    // the rollout for what steps left, behind it for the worlds that it owes, unless its blocks generate those
    const int regen = ((2 * n < REGEN_BLOCKS ? 2 * n : REGEN_BLOCKS) + 2 * NSUB - 1) / (2 * NSUB) * (2 * NSUB);
    const int owed = ((2 * n < OWED_BLOCKS ? 2 * n : OWED_BLOCKS) + 2 * NSUB - 1) / (2 * NSUB) * (2 * NSUB);
    // lanes per environment as chosen for single steps: four (64 environments per block) where there
    // are enough environments to fill the chip that way, else sixteen (16 per block)
    const bool wide = lanes != 4;
    const int own_from = (int)rollout_own_from(!wide, p.worldgen == CRAFTAX_WORLDGEN_PERLIN, o != nullptr, n, steps, p.max_episode_steps);
    const int blocks = wide ? (n + 15) / 16 : (n + 63) / 64;
#define CRAFTAX_LAUNCH_ROLLOUT(LANES, NOISE) \
    hipLaunchKernelGGL((k_rollout<LANES, OBS_MODE, NOISE>), dim3(blocks), dim3(BLOCK), 0, st, q.recs, q.maps, q.luts, actions, o, reward, \
                       done, q.ls, p, steps, own_from)
    if (p.worldgen == CRAFTAX_WORLDGEN_PERLIN) {
        hipLaunchKernelGGL(k_drain<true>, dim3(regen), dim3(BLOCK), 0, st, q.maps, q.luts, q.ls);
        if (wide) CRAFTAX_LAUNCH_ROLLOUT(16, true); else CRAFTAX_LAUNCH_ROLLOUT(4, true);
        if (own_from != steps - 1) hipLaunchKernelGGL(k_drain<true>, dim3(owed), dim3(BLOCK), 0, st, q.maps, q.luts, q.ls);
    } else {
        hipLaunchKernelGGL(k_drain<false>, dim3(regen), dim3(BLOCK), 0, st, q.maps, q.luts, q.ls);
        if (wide) CRAFTAX_LAUNCH_ROLLOUT(16, false); else CRAFTAX_LAUNCH_ROLLOUT(4, false);
        if (own_from != steps - 1) hipLaunchKernelGGL(k_drain<false>, dim3(owed), dim3(BLOCK), 0, st, q.maps, q.luts, q.ls);
    }
#undef CRAFTAX_LAUNCH_ROLLOUT
}

}  // namespace cx

using namespace cx;

// Device address of `scratch` on the current device, looked up once per device.
constexpr int MAX_DEVICES = 64;
static uint32_t* g_scratch_ptr[MAX_DEVICES];
static int stats_scratch_address(uint32_t** ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(CRAFTAX_E_HIP, "device number out of range");
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return fail(CRAFTAX_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        }
        g_scratch_ptr[dev] = static_cast<uint32_t*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return CRAFTAX_OK;
}

extern "C" {

void craftax_default_config_for(craftax_config* cfg, uint32_t variant)
{
    if (!cfg) return;
    std::memset(cfg, 0, sizeof(*cfg));
    cfg->abi_version = CRAFTAX_ABI_VERSION;
    cfg->variant = variant;
    cfg->obs_mode = CRAFTAX_OBS_SYM_U8_F32;
    cfg->max_episode_steps = variant == CRAFTAX_VARIANT_CRAFTAX ? 100000 : 10000;
    cfg->day_length = 300;
    cfg->cap_zombie = cfg->cap_cow = cfg->cap_skeleton = cfg->cap_arrow = 3;
    if (variant == CRAFTAX_VARIANT_CRAFTAX) cfg->cap_skeleton = 2;
    cfg->cap_plant = 10;
    cfg->atlas_seed = 0;
    cfg->worldgen = CRAFTAX_WORLDGEN_VALUE;
    cfg->reset_mode = CRAFTAX_RESET_EXACT;
}

void craftax_default_config(craftax_config* cfg) { craftax_default_config_for(cfg, CRAFTAX_VARIANT_CLASSIC); }

size_t craftax_state_bytes(const craftax_config* cfg, int n)
{
    std::string why;
    if (!cfg || n <= 0 || !config_ok(cfg, &why)) return 0;
    if (cfg->variant == CRAFTAX_VARIANT_CRAFTAX) return cf::host::state_bytes(cfg, n);
    return (size_t)make_header(cfg, n).total;
}

size_t craftax_obs_bytes(const craftax_config* cfg)
{
    if (!cfg || cfg->obs_mode > CRAFTAX_OBS_PIXELS_F32) return 0;
    if (cfg->variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string why;
        return cf::host::config_ok(cfg, &why) ? cf::host::obs_bytes(cfg) : 0;
    }
    return (size_t)obs_stride((int)cfg->obs_mode);
}

size_t craftax_env_dump_bytes(void) { return sizeof(craftax_env_dump); }
size_t craftax_env_dump_bytes_for(const craftax_config* cfg)
{
    if (!cfg) return 0;
    return cfg->variant == CRAFTAX_VARIANT_CRAFTAX ? sizeof(craftax_full_env_dump) : sizeof(craftax_env_dump);
}

// LDS and thread needs of the kernels a Classic configuration launches, against the device's limits.
static int check_kernels(const craftax_config* cfg, int lanes, std::string* err)
{
    int dev = 0, lds = 0, threads = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
        hipDeviceGetAttribute(&threads, hipDeviceAttributeMaxThreadsPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        *err = "no usable HIP device";
        return CRAFTAX_E_HIP;
    }
    const DeviceLimits limits{(size_t)lds, threads};
    auto fits = [&](const char* name, const void* fn, int block) {
        hipFuncAttributes a;
        if (hipFuncGetAttributes(&a, fn) != hipSuccess) { (void)hipGetLastError(); *err = std::string("no attributes for ") + name; return false; }
        return kernel_fits(KernelNeeds{name, a.sharedSizeBytes, a.maxThreadsPerBlock, block}, limits, err);
    };
    const bool perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN;
    bool ok = true;
#define CRAFTAX_CHECK_MODE(M) \
    do { \
        if (lanes == 4) ok = ok && (perlin ? fits("k_step", (const void*)k_step<4, M, true>, BLOCK) : fits("k_step", (const void*)k_step<4, M, false>, BLOCK)); \
        else if (lanes == 8) ok = ok && (perlin ? fits("k_step", (const void*)k_step<8, M, true>, BLOCK) : fits("k_step", (const void*)k_step<8, M, false>, BLOCK)); \
        else ok = ok && (perlin ? fits("k_step", (const void*)k_step<16, M, true>, BLOCK) : fits("k_step", (const void*)k_step<16, M, false>, BLOCK)); \
        ok = ok && fits("k_reset_list", (const void*)k_reset_list<M>, WG_THREADS); \
    } while (0)
#define CRAFTAX_CHECK_ROLLOUT(M) \
    do { \
        if (lanes == 4) ok = ok && (perlin ? fits("k_rollout", (const void*)k_rollout<4, M, true>, BLOCK) : fits("k_rollout", (const void*)k_rollout<4, M, false>, BLOCK)); \
        else ok = ok && (perlin ? fits("k_rollout", (const void*)k_rollout<16, M, true>, BLOCK) : fits("k_rollout", (const void*)k_rollout<16, M, false>, BLOCK)); \
        ok = ok && fits("k_observe", (const void*)k_observe<M>, BLOCK); \
    } while (0)
    switch (cfg->obs_mode) {
    case CRAFTAX_OBS_SYM_U8_I8: CRAFTAX_CHECK_MODE(0); CRAFTAX_CHECK_ROLLOUT(0); break;
    case CRAFTAX_OBS_SYM_U8_F32: CRAFTAX_CHECK_MODE(1); CRAFTAX_CHECK_ROLLOUT(1); break;
    case CRAFTAX_OBS_SYM_F32: CRAFTAX_CHECK_MODE(2); CRAFTAX_CHECK_ROLLOUT(2); break;
    default: CRAFTAX_CHECK_MODE(3); ok = ok && fits("k_pixels", (const void*)k_pixels, BLOCK) &&
        (perlin ? fits("k_step with pictures", (const void*)k_step<16, 3, true, true>, BLOCK) : fits("k_step with pictures", (const void*)k_step<16, 3, false, true>, BLOCK)); break;
    }
#undef CRAFTAX_CHECK_MODE
#undef CRAFTAX_CHECK_ROLLOUT
    ok = ok && (perlin ? fits("k_reset", (const void*)k_reset<true>, WG_THREADS) : fits("k_reset", (const void*)k_reset<false>, WG_THREADS)) && (perlin ? fits("k_import_spare", (const void*)k_import_spare<true>, WG_THREADS) : fits("k_import_spare", (const void*)k_import_spare<false>, WG_THREADS)) &&
         fits("k_mutate_noise", (const void*)k_mutate_noise, WG_THREADS) &&
         (perlin ? fits("k_drain", (const void*)k_drain<true>, BLOCK) : fits("k_drain", (const void*)k_drain<false>, BLOCK));
    return ok ? CRAFTAX_OK : CRAFTAX_E_CONFIG;
}

static int check_arguments(void* state, const craftax_config* cfg, int n)
{
    if (!state || !cfg) return fail(CRAFTAX_E_NULL, "state or cfg is NULL");
    if ((uintptr_t)state % 256) return fail(CRAFTAX_E_ALIGN, "state must be 256-byte aligned");
    if (n <= 0) return fail(CRAFTAX_E_COUNT, "n must be positive");
    std::string why;
    if (!config_ok(cfg, &why)) return fail(CRAFTAX_E_CONFIG, why);
    return CRAFTAX_OK;
}

int craftax_state_init(void* state, const craftax_config* cfg, int n, void* stream)
{
    if (int rc = check_arguments(state, cfg, n)) return rc;
    HostState s;
    s.cfg = *cfg; s.n = n; s.has_worlds = false; s.serve_slow = false;
    if (cfg->variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::memset(&s.hdr, 0, sizeof(s.hdr));
        s.lanes = 64;
        std::string err;
        if (int rc = cf::host::check_kernels(cfg, &err)) return fail(rc, err);
        uint32_t* unused = nullptr;
        if (int rc = stats_scratch_address(&unused)) return rc;    // set-up: the library's own scratch on this device
        if (int rc = cf::host::state_init(state, cfg, n, stream, &err)) return fail(rc, err);
        std::lock_guard<std::mutex> lock(g_mutex);
        g_states[state] = s;
        return CRAFTAX_OK;
    }
    s.hdr = make_header(cfg, n); s.lanes = group_lanes(cfg, n);
    {
        std::string err;
        if (int rc = check_kernels(cfg, s.lanes, &err)) return fail(rc, err);
    }
    {
        uint32_t* unused = nullptr;
        if (int rc = stats_scratch_address(&unused)) return rc;    // set-up: the library's own scratch on this device
    }
    std::vector<uint8_t> staging((size_t)s.hdr.off_recs, 0);
    std::memcpy(staging.data(), &s.hdr, sizeof(Header));
    build_luts(cfg, reinterpret_cast<Luts*>(staging.data() + s.hdr.off_luts));
    hipError_t e = hipMemcpyAsync(state, staging.data(), staging.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);   // staging dies with this call
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("state_init copy: ") + hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(g_mutex);
    g_states[state] = s;
    return CRAFTAX_OK;
}

int craftax_state_attach(void* state, const craftax_config* cfg, int n, void* stream)
{
    if (int rc = check_arguments(state, cfg, n)) return rc;
    uint8_t bytes[HEADER_BYTES];
    hipError_t e = hipMemcpyAsync(bytes, state, sizeof(bytes), hipMemcpyDeviceToHost, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("state_attach copy: ") + hipGetErrorString(e));
    HostState s;
    s.cfg = *cfg; s.n = n; s.has_worlds = true;
    s.serve_slow = true;     // the source's pending edit, if any, is not part of the blob: serve the slow list once
    std::string err;
    if (cfg->variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::memset(&s.hdr, 0, sizeof(s.hdr));
        s.lanes = 64;
        if (int rc = cf::host::check_header(bytes, cfg, n, &err)) return fail(rc, err);
        if (int rc = cf::host::check_kernels(cfg, &err)) return fail(rc, err);
    } else {
        s.hdr = make_header(cfg, n); s.lanes = group_lanes(cfg, n);
        Header got;
        std::memcpy(&got, bytes, sizeof(got));
        if (got.magic != MAGIC) return fail(CRAFTAX_E_STATE, "the memory holds no Craftax-Classic state blob");
        if (got.version != CRAFTAX_ABI_VERSION) return fail(CRAFTAX_E_STATE, "the state blob was written by another library version");
        if (got.n != (uint32_t)n) return fail(CRAFTAX_E_COUNT, "the state blob holds another number of environments");
        if (std::memcmp(&got, &s.hdr, sizeof(Header)) != 0) return fail(CRAFTAX_E_CONFIG, "the state blob was initialised with another configuration");
        if (int rc = check_kernels(cfg, s.lanes, &err)) return fail(rc, err);
    }
    {
        uint32_t* unused = nullptr;
        if (int rc = stats_scratch_address(&unused)) return rc;    // set-up: the library's own scratch on this device
    }
    std::lock_guard<std::mutex> lock(g_mutex);
    g_states[state] = s;
    return CRAFTAX_OK;
}

int craftax_state_release(void* state)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    return g_states.erase(state) ? CRAFTAX_OK : fail(CRAFTAX_E_STATE, "unknown state");
}

int craftax_reset(void* state, const uint64_t* seeds, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!seeds) return fail(CRAFTAX_E_NULL, "seeds is NULL");
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::reset(state, &s.cfg, n, seeds, stream, &err);
        if (rc == CRAFTAX_OK) update_state(state, true, false);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(2u * (unsigned)n), dim3(WG_THREADS), 0, (hipStream_t)stream, q.recs, q.maps, seeds, q.ls, q.luts,
                           make_params(state, s).unlocks);
    };
    if (s.cfg.worldgen == CRAFTAX_WORLDGEN_PERLIN) go(k_reset<true>); else go(k_reset<false>);
    const int rc = check_launch("craftax_reset");
    if (rc == CRAFTAX_OK) update_state(state, true, false);
    return rc;
}

int craftax_step(void* state, const int32_t* actions, void* obs, float* reward, uint8_t* done, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!actions || !reward || !done) return fail(CRAFTAX_E_NULL, "actions, reward or done is NULL");
    if ((uintptr_t)obs % 16) return fail(CRAFTAX_E_ALIGN, "obs must be 16-byte aligned");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::step(state, &s.cfg, n, actions, obs, reward, done, s.serve_slow, stream, &err);
        if (rc == CRAFTAX_OK && s.serve_slow) update_state(state, true, false);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    const Params p = make_params(state, s);
    hipStream_t st = (hipStream_t)stream;
    uint8_t* o = static_cast<uint8_t*>(obs);
    const int G = s.lanes;
    switch (s.cfg.obs_mode) {
    case CRAFTAX_OBS_SYM_U8_I8: launch_step<0>(G, n, st, q, actions, o, reward, done, p, s.serve_slow); break;
    case CRAFTAX_OBS_SYM_U8_F32: launch_step<1>(G, n, st, q, actions, o, reward, done, p, s.serve_slow); break;
    case CRAFTAX_OBS_SYM_F32: launch_step<2>(G, n, st, q, actions, o, reward, done, p, s.serve_slow); break;
    default: launch_step<3>(G, n, st, q, actions, o, reward, done, p, s.serve_slow); break;
    }
    if (s.serve_slow) update_state(state, true, false);
    return check_launch("craftax_step");
}

int craftax_rollout(void* state, const int32_t* actions, int steps, void* obs, float* reward, uint8_t* done, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!actions || !reward || !done) return fail(CRAFTAX_E_NULL, "actions, reward or done is NULL");
    if (steps <= 0) return fail(CRAFTAX_E_COUNT, "steps must be positive");
    if (obs && (uintptr_t)obs % 16) return fail(CRAFTAX_E_ALIGN, "obs must be 16-byte aligned");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::rollout(state, &s.cfg, s.n, actions, steps, obs, reward, done, stream, &err);
        return rc ? fail(rc, err) : rc;
    }
    if (s.cfg.obs_mode == CRAFTAX_OBS_PIXELS_F32) return fail(CRAFTAX_E_CONFIG, "craftax_rollout needs a symbolic observation");
    if (s.cfg.reset_mode != CRAFTAX_RESET_EXACT) return fail(CRAFTAX_E_CONFIG, "craftax_rollout needs exact resets");
    const Ptrs q = pointers(state, s);
    const Params p = make_params(state, s);
    uint8_t* o = static_cast<uint8_t*>(obs);
    switch (s.cfg.obs_mode) {
    case CRAFTAX_OBS_SYM_U8_I8: launch_rollout<0>(s.lanes, n, (hipStream_t)stream, q, actions, steps, o, reward, done, p); break;
    case CRAFTAX_OBS_SYM_U8_F32: launch_rollout<1>(s.lanes, n, (hipStream_t)stream, q, actions, steps, o, reward, done, p); break;
    default: launch_rollout<2>(s.lanes, n, (hipStream_t)stream, q, actions, steps, o, reward, done, p); break;
    }
    return check_launch("craftax_rollout");
}

int craftax_observe(void* state, void* obs, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!obs) return fail(CRAFTAX_E_NULL, "obs is NULL");
    if ((uintptr_t)obs % 16) return fail(CRAFTAX_E_ALIGN, "obs must be 16-byte aligned");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::observe(state, &s.cfg, n, obs, stream, &err);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    const Params p = make_params(state, s);
    const dim3 grid((n + 15) / 16), block(BLOCK);
    hipStream_t st = (hipStream_t)stream;
    uint8_t* o = static_cast<uint8_t*>(obs);
    switch (s.cfg.obs_mode) {
    case CRAFTAX_OBS_SYM_U8_I8: hipLaunchKernelGGL(k_observe<0>, grid, block, 0, st, q.recs, q.maps, q.luts, o, p); break;
    case CRAFTAX_OBS_SYM_U8_F32: hipLaunchKernelGGL(k_observe<1>, grid, block, 0, st, q.recs, q.maps, q.luts, o, p); break;
    case CRAFTAX_OBS_SYM_F32: hipLaunchKernelGGL(k_observe<2>, grid, block, 0, st, q.recs, q.maps, q.luts, o, p); break;
    default: hipLaunchKernelGGL(k_pixels, dim3(n), block, 0, st, q.recs, q.maps, q.luts, o, p); break;
    }
    return check_launch("craftax_observe");
}

int craftax_export_envs(const void* state, int first, int count, void* dumps, void* stream)
{
    HostState s;
    if (int rc = lookup(state, 0, false, &s)) return rc;
    if (!dumps) return fail(CRAFTAX_E_NULL, "dumps is NULL");
    if (first < 0 || count <= 0 || first + count > s.n) return fail(CRAFTAX_E_COUNT, "range outside the state");
    if ((uintptr_t)dumps % 16) return fail(CRAFTAX_E_ALIGN, "dumps must be 16-byte aligned");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::export_envs(state, &s.cfg, s.n, first, count, dumps, stream, &err);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    hipLaunchKernelGGL(k_export, dim3(count), dim3(BLOCK), 0, (hipStream_t)stream, q.recs, q.maps,
                       static_cast<craftax_env_dump*>(dumps), first);
    return check_launch("craftax_export_envs");
}

int craftax_import_envs(void* state, int first, int count, const void* dumps, void* stream)
{
    HostState s;
    if (int rc = lookup(state, 0, false, &s)) return rc;
    if (!dumps) return fail(CRAFTAX_E_NULL, "dumps is NULL");
    if (first < 0 || count <= 0 || first + count > s.n) return fail(CRAFTAX_E_COUNT, "range outside the state");
    if ((uintptr_t)dumps % 16) return fail(CRAFTAX_E_ALIGN, "dumps must be 16-byte aligned");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::import_envs(state, &s.cfg, s.n, first, count, dumps, stream, &err);
        if (rc == CRAFTAX_OK) note_edit(state);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    hipLaunchKernelGGL(k_import, dim3(count), dim3(BLOCK), 0, (hipStream_t)stream, q.recs, q.maps, q.ls,
                       static_cast<const craftax_env_dump*>(dumps), first, make_params(state, s));
    if (s.cfg.worldgen == CRAFTAX_WORLDGEN_PERLIN)
        hipLaunchKernelGGL(k_import_spare<true>, dim3(count), dim3(WG_THREADS), 0, (hipStream_t)stream, q.recs, q.maps, q.ls, first, q.luts);
    else hipLaunchKernelGGL(k_import_spare<false>, dim3(count), dim3(WG_THREADS), 0, (hipStream_t)stream, q.recs, q.maps, q.ls, first, q.luts);
    note_edit(state);
    return check_launch("craftax_import_envs");
}

int craftax_mutate_swap(void* state, int first, int count, uint64_t mutation_seed, uint32_t round, int restricted, int32_t* tries,
                        void* stream)
{
    HostState s;
    if (int rc = lookup(state, 0, false, &s)) return rc;
    if (first < 0 || count <= 0 || first + count > s.n) return fail(CRAFTAX_E_COUNT, "range outside the state");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::mutate_swap(state, &s.cfg, s.n, first, count, mutation_seed, round, restricted, tries, stream, &err);
        if (rc == CRAFTAX_OK) note_edit(state);
        return rc ? fail(rc, err) : rc;
    }
    const Ptrs q = pointers(state, s);
    hipLaunchKernelGGL(k_mutate_swap, dim3((unsigned)(((long long)count * MUTATE_TRIES + 255) / 256)), dim3(256), 0, (hipStream_t)stream, q.recs, q.maps, first,
                       count, (uint32_t)mutation_seed, (uint32_t)(mutation_seed >> 32), round, restricted != 0 ? 1 : 0, tries);
    note_edit(state);
    return check_launch("craftax_mutate_swap");
}

int craftax_mutate_noise(void* state, int first, int count, uint16_t* theta, uint64_t mutation_seed, uint32_t round, uint32_t amplitude,
                         void* stream)
{
    HostState s;
    if (int rc = lookup(state, 0, false, &s)) return rc;
    if (!theta) return fail(CRAFTAX_E_NULL, "theta is NULL");
    if ((uintptr_t)theta % 2) return fail(CRAFTAX_E_ALIGN, "theta must be 2-byte aligned");
    if (first < 0 || count <= 0 || first + count > s.n) return fail(CRAFTAX_E_COUNT, "range outside the state");
    if (amplitude > 511u) return fail(CRAFTAX_E_COUNT, "amplitude above half a turn (511)");
    if (s.cfg.worldgen != CRAFTAX_WORLDGEN_PERLIN) return fail(CRAFTAX_E_CONFIG, "the noise mutation needs Perlin world generation");
    if (int rc = need_worlds(s)) return rc;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) {
        std::string err;
        const int rc = cf::host::mutate_noise(state, &s.cfg, s.n, first, count, theta, mutation_seed, round, amplitude, stream, &err);
        if (rc == CRAFTAX_OK) note_edit(state);
        return rc == CRAFTAX_OK ? rc : fail(rc, err);
    }
    const Ptrs q = pointers(state, s);
    hipLaunchKernelGGL(k_mutate_noise, dim3((unsigned)count), dim3(WG_THREADS), 0, (hipStream_t)stream, q.recs, q.maps, q.luts, theta,
                       first, (uint32_t)mutation_seed, (uint32_t)(mutation_seed >> 32), round, amplitude);
    note_edit(state);
    return check_launch("craftax_mutate_noise");
}

int craftax_synth_actions(int32_t* actions, int n, int step0, int steps, uint64_t action_seed, int kind, void* stream)
{
    if (!actions) return fail(CRAFTAX_E_NULL, "actions is NULL");
    if (n <= 0 || steps <= 0 || step0 < 0 || kind < 0 || kind > 3) return fail(CRAFTAX_E_COUNT, "bad n, steps, step0 or kind");
    const size_t total = (size_t)n * (size_t)steps;
    hipLaunchKernelGGL(k_synth_actions, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, actions, n,
                       step0, steps, (uint32_t)action_seed, (uint32_t)(action_seed >> 32), kind);
    return check_launch("craftax_synth_actions");
}

static int stats_blocks(int n) { return (n + STATS_ENVS_PER_BLOCK - 1) / STATS_ENVS_PER_BLOCK; }

// both kernels of the metrics snapshot, partial results in `scratch` (device memory, stats_blocks(n) x 1 KiB)
static int launch_stats(const void* state, const HostState& s, craftax_metrics* out, uint32_t* scratch, int n, hipStream_t st)
{
    cf::host::RecordLayout ly;
    if (s.cfg.variant == CRAFTAX_VARIANT_CRAFTAX) ly = cf::host::record_layout(state, &s.cfg, n);
    else ly = cf::host::RecordLayout{reinterpret_cast<const uint32_t*>(pointers(state, s).recs), REC_DWORDS, RW_ACH, 1, RW_T, RW_EPISODE,
                                     make_params(state, s).unlocks, UNLOCK_STRIDE};
    const int blocks = stats_blocks(n);
    hipLaunchKernelGGL(k_stats_partial, dim3((unsigned)blocks), dim3(STATS_ENVS_PER_BLOCK), 0, st, ly, n, scratch);
    hipLaunchKernelGGL(k_stats_total, dim3(1), dim3(STATS_TOTAL_THREADS), 0, st, scratch, blocks, n, out);
    return check_launch("craftax_stats");
}

int craftax_stats_static(const void* state, craftax_metrics* out, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!out) return fail(CRAFTAX_E_NULL, "out is NULL");
    if ((uintptr_t)out % 8) return fail(CRAFTAX_E_ALIGN, "out must be 8-byte aligned");
    if (n > CRAFTAX_STATS_STATIC_MAX_ENVS) return fail(CRAFTAX_E_COUNT, "craftax_stats_static serves at most CRAFTAX_STATS_STATIC_MAX_ENVS environments: use craftax_stats with a workspace");
    if (int rc = need_worlds(s)) return rc;
    uint32_t* ptr = nullptr;
    if (int rc = stats_scratch_address(&ptr)) return rc;
    // every block of the first kernel overwrites its whole partial result and the second kernel reads
    // only the blocks of this call, so nothing left by an earlier call needs clearing
    return launch_stats(state, s, out, ptr, n, (hipStream_t)stream);
}

size_t craftax_stats_workspace_bytes(int n)
{
    return n <= 0 ? 0 : (size_t)stats_blocks(n) * STATS_PARTIAL_WORDS * 4;
}

int craftax_stats(const void* state, craftax_metrics* out, void* workspace, size_t workspace_bytes, int n, void* stream)
{
    HostState s;
    if (int rc = lookup(state, n, true, &s)) return rc;
    if (!out || !workspace) return fail(CRAFTAX_E_NULL, "out or workspace is NULL");
    if ((uintptr_t)out % 8 || (uintptr_t)workspace % 16) return fail(CRAFTAX_E_ALIGN, "out must be 8-byte aligned, workspace 16-byte aligned");
    if (workspace_bytes < craftax_stats_workspace_bytes(n)) return fail(CRAFTAX_E_COUNT, "workspace smaller than craftax_stats_workspace_bytes(n)");
    if (int rc = need_worlds(s)) return rc;
    return launch_stats(state, s, out, static_cast<uint32_t*>(workspace), n, (hipStream_t)stream);
}

int craftax_debug_bounds(uint32_t report[4])
{
    if (!report) return fail(CRAFTAX_E_NULL, "report is NULL");
    report[0] = report[1] = report[2] = report[3] = 0u;
#ifdef CRAFTAX_DEBUG_BOUNDS
    hipError_t e = hipDeviceSynchronize();
    const uint32_t zero[4] = {0u, 0u, 0u, 0u};
    if (e == hipSuccess) e = hipMemcpyFromSymbol(report, HIP_SYMBOL(cx::g_bounds), 4 * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(cx::g_bounds), zero, sizeof(zero));
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("craftax_debug_bounds: ") + hipGetErrorString(e));
    std::string err;
    if (int rc = cf::host::debug_bounds(report, &err)) return fail(rc, err);
    return 1;
#else
    return 0;
#endif
}

int craftax_debug_bounds_selftest(void)
{
#ifdef CRAFTAX_DEBUG_BOUNDS
    uint32_t report[4];
    if (int rc = craftax_debug_bounds(report); rc < 0) return rc;      // clears what was there
    uint32_t* out = nullptr;
    // the one allocation of the debug library: a word for the self-test kernel to write
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&out), sizeof(uint32_t));
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("selftest: ") + hipGetErrorString(e));
    hipLaunchKernelGGL(k_bounds_selftest, dim3(1), dim3(1), 0, (hipStream_t) nullptr, out);
    uint32_t value = 0;
    e = hipMemcpy(&value, out, sizeof(value), hipMemcpyDeviceToHost);
    (void)hipFree(out);
    if (e != hipSuccess) return fail(CRAFTAX_E_HIP, std::string("selftest: ") + hipGetErrorString(e));
    if (int rc = craftax_debug_bounds(report); rc < 0) return rc;
    return (report[0] == 1u && report[2] == 5u && report[3] == 4u && value == 11u) ? 1 : fail(CRAFTAX_E_STATE, "the bounds record did not show the planted index");
#else
    return 0;
#endif
}

const char* craftax_last_error(void) { return g_error.c_str(); }

}  // extern "C"
