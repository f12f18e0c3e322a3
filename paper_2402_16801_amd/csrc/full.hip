// Kernels and host entry points of the full-Craftax variant (nine floors, 43 actions).
#include "full_api.hpp"
#include "floor_route.hpp"
#include "launch_limits.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "worldgen.hpp"
#include "full_common.hpp"
#include "full_render.hpp"
#include "full_pixels.hpp"
#include "full_step.hpp"
#include "full_worldgen.hpp"

namespace cf {

static_assert(sizeof(craftax_full_env_dump) == 63432, "canonical dump layout");

using la::Lists;
using la::counter;
using la::ENTRY_VOID;
using la::NSUB;

// Up to here a step fetches the spare world's start window in advance (EAGER, see kf_step).  Steps with bytes: while the chip holds all blocks of such a
// launch at once (six per compute unit, regeneration blocks among them, with Perlin noise five); beyond, the instance without, of which it holds
// eight and six, is ahead.  us, with / without: 1,024 10.0 / 10.4, 4,096 13.2 / 13.5, 5,000 14.9 / 15.1, 5,300 17.2 / 15.8, 7,000 20.4 / 18.0,
// 8,192 21.9 / 21.9; Perlin noise 4,096 13.7 / 13.6, 4,500 16.7 / 14.9, 5,800 19.1 / 18.8, 8,000 22.1 / 21.3.
constexpr int EAGER_SPARE_ENVS = 8192;
constexpr int eager_spare_envs(bool bytes, bool perlin, int lanes) { return !bytes || lanes != 64 ? EAGER_SPARE_ENVS : perlin ? 4096 : 5120; }
// The same line for steps with bytes that fetch nothing in advance at any size, because their episodes end without a spare world (optimistic
// resets): beyond it the instance for a full chip, up to it one that is not bounded to as many blocks (us, with that of a full chip / so: 64
// 12.3 / 12.2, 256 16.1 / 15.8, 1,024 18.8 / 18.5, 4,096 25.0 / 24.7, 5,120 28.0 / 27.6, 8,192 37.9 / 38.6; Perlin noise 1,024 20.2 / 20.1, 4,096 26.6 / 26.5).
constexpr bool chip_is_full(int n, bool perlin) { return n > eager_spare_envs(true, perlin, 64); }
constexpr int RESET_SLOTS = 64;    // environments served at once by kf_reset_list (nine blocks each)
constexpr int MAX_ENVS_PER_STEP_BLOCK = 16;   // a step block holds 4 environments (a wavefront each) or 16 (16 lanes each)
constexpr int REGEN_BLOCKS = 256;  // regeneration blocks at the head of the step grid: with 1,024 step blocks (4,096 environments) they fill the chip exactly

// Floors in the order in which the blocks of a launch take them: all worlds' overworlds first (six fields), then the caves (two, two,
// two, one), the floors built from masks last, so that a launch ends with short ones (world by world before: level turns over 1,000
// Perlin worlds 138 us, 113 so, over 400 75 and 63, resets of 420 43.0 and 37.3, of 4,096 170 and 162, with Perlin noise 217 and 199).  A few floors are all on
// the chip from the start; they go world by world, which keeps the long ones apart (level turns over 32 43.8 us, 46.7 by floors, over 64 43.7 and
// 47.3, over 100 49.7 either way; resets of 48 22.6 and 23.6, of 85 25.8 and 24.9).
__device__ inline int floor_in_turn(int turn) { return (int)((0x841325760ull >> (4 * turn)) & 15u); }
constexpr long long FLOORS_BY_TURN_FROM = 1000;
static dim3 floor_grid(unsigned worlds) { return (long long)worlds * FLOORS >= FLOORS_BY_TURN_FROM ? dim3(worlds, FLOORS) : dim3(worlds * FLOORS); }
// which world and floor of such a launch a block takes
struct FloorBlock { int world, floor; };
__device__ inline FloorBlock floor_block()
{
    if (gridDim.y == (unsigned)FLOORS) return FloorBlock{ (int)blockIdx.x, floor_in_turn((int)blockIdx.y) };
    return FloorBlock{ (int)(blockIdx.x / (unsigned)FLOORS), (int)(blockIdx.x % (unsigned)FLOORS) };
}

// What the block that generated floor 0 of a world leaves behind for the environment: as the
// current world (fresh record, empty mob tables) or as the spare world (its ladders and potion map).
// SAME_EPISODE: the record already holds this episode and seed (blocks of other floors may be reading
// them): those three words are left alone.
template <bool SAME_EPISODE = false>
__device__ inline void publish_world(uint32_t* __restrict__ genv, const GenLayout& L, uint32_t lo, uint32_t hi, uint32_t ep,
                                     bool current, uint32_t* s_layout_words)
{
    const int tid = threadIdx.x;
    if (tid < FLOORS + 1) s_layout_words[tid] = layout_word(L, tid);
    __syncthreads();
    if (current) {
        for (int i = tid; i < SPARE_LADDER; i += blockDim.x) {
            const bool identity = i == R_EPISODE || i == R_SEED_LO || i == R_SEED_HI;
            if (!(SAME_EPISODE && identity)) genv[i] = i < REC_DWORDS ? fresh_record_word(i, s_layout_words, lo, hi, ep) : 0u;
        }
    } else if (tid < FLOORS + 1) genv[SPARE_LADDER + tid] = s_layout_words[tid];
}

// ---------------------------------------------------------------------------------------------
// reset of every environment: one block per (environment, episode 0 or 1, floor); see floor_grid
template <bool PERLIN, int NT>
__global__ __launch_bounds__(NT, PERLIN ? PERLIN_WAVES : VALUE_WAVES) void kf_reset(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps,
                                                       const uint64_t* __restrict__ seeds, Lists ls, const uint32_t* __restrict__ perlin_cs,
                                                       int pool, uint32_t* __restrict__ unlocks)
{
    if (blockIdx.x == 0 && blockIdx.y == 0) la::reset_counters(ls);
    __shared__ uint32_t s_lat[LAT_WORDS];
    __shared__ GenLayout s_layout;
    __shared__ uint32_t s_words[FLOORS + 1];
    const FloorBlock block = floor_block();
    const uint32_t env = (uint32_t)block.world >> 1, ep = (uint32_t)block.world & 1u;
    const int f = block.floor;
    const uint64_t seed = seeds[env];
    const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
    worldgen_floor_block<NT, PERLIN>(maps + map_offset(env, ep), s_lat, s_layout, lo, hi, env, ep, f, nullptr, nullptr, perlin_cs);
    if (f == 0) publish_world(envs + (size_t)env * ENV_DWORDS, s_layout, lo, hi, ep, ep == 0u, s_words);
    if (f == 0 && ep == 0u) for (int i = threadIdx.x; i < UNLOCK_STRIDE; i += NT) unlocks[(size_t)env * UNLOCK_STRIDE + i] = 0u;
    // With optimistic resets no spare world is ever valid: tag 0 matches no next episode (they count
    // from 1), so the step kernel hands every finished episode to kf_reset_list.
    if (ep == 1u && threadIdx.x == 0) ls.tags[(size_t)env * NTAG + f] = make_uint2(pool ? 0u : 1u, 0u);
}

// LDS scratch of the threads that generate a world (or a floor of one)
struct WorldScratch { uint32_t lat[LAT_WORDS]; GenLayout layout; uint32_t words[FLOORS + 1]; };
static_assert(sizeof(WorldScratch) % 8 == 0 && offsetof(WorldScratch, layout) % 8 == 0, "row masks are 64-bit words");

// Regeneration blocks (of the step grid, or of a launch of their own): worlds after next for the
// episodes that ended in the previous launch.  The consumed list is one dense queue of work units, one
// floor of one world each; block rb of nrb takes units rb, rb + nrb, ...  In the step grid the blocks
// stand at the head: a step launch holds as many of them as the chip has room for beside the step
// blocks, so every unit starts with the launch and none waits for a block that is scheduled late.
// A unit's turn, sub-list and place come from votes in which a lane holds the end of one turn and of one sub-list, and what
// the entry says is moved to scalar registers: the floor and its seed are the same for the wavefront, which an index divided by a number
// from LDS hides from the compiler (with that division and a walk over the sub-lists, a step's us / so: 2,048 environments 10.6 / 10.2, without
// an observation 10.1 / 9.6; with episodes of at most 20 steps, of every age, 4,096 34.0 / 31.9, 8,192 67.7 / 62.4, 16,384 128 / 118, Perlin noise 135 / 127).
// By turn at every length (see floor_grid; us, world by world / by turn): up to a floor per block either is as fast (64 environments 7.9 / 7.9, 1,000 9.9 / 9.9, 2,048
// 10.2 / 10.3, with Perlin noise 12.5 / 12.5), beyond that the first has blocks that get two overworlds (4,096 with episodes of at most 100 steps 14.5 / 14.0,
// of 20 33.2 / 31.8, Perlin noise 17.7 / 15.6 and 38.2 / 35.5, 16,384 of 20 119 / 118 and 128 / 127).
template <int NT, bool PERLIN>
__device__ __forceinline__ void regeneration_queue(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps, const Lists& ls,
                                                   uint32_t seq, WorldScratch& s, const uint32_t* s_prefix, int regen_blocks,
                                                   const uint32_t* __restrict__ perlin_cs)
{
    const uint32_t lane = threadIdx.x & 63u, total = s_prefix[lane < (uint32_t)NSUB ? lane : 0u];
    const uint32_t worlds = (uint32_t)lane_get((int)total, NSUB - 1), units = worlds * (uint32_t)FLOORS, turn_ends = (lane + 1u) * worlds;
    for (uint32_t u = blockIdx.x; u < units; u += (uint32_t)regen_blocks) {
        __syncthreads();   // the previous unit's scratch has been read by everyone
        const int turn = __popcll(__ballot(u >= turn_ends) & ((1ull << (FLOORS - 1)) - 1ull));
        const uint32_t world = u - (uint32_t)turn * worlds;
        const int sub = __popcll(__ballot(world >= total) & ((1ull << (NSUB - 1)) - 1ull));
        const uint4 found = la::queue_entry(ls, seq, (uint32_t)sub, world - (sub == 0 ? 0u : (uint32_t)lane_get((int)total, sub - 1)));
        const uint4 entry = make_uint4(uniu(found.x), uniu(found.y), uniu(found.z), uniu(found.w));
        const int f = floor_in_turn(turn);
        if (entry.x == ENTRY_VOID) continue;
        worldgen_floor_block<NT, PERLIN, true>(maps + map_offset(entry.x, entry.w), s.lat, s.layout, entry.y, entry.z, entry.x, entry.w, f, nullptr, nullptr,
                                         PERLIN ? perlin_cs : nullptr);
        if (f == 0) publish_world(envs + (size_t)entry.x * ENV_DWORDS, s.layout, entry.y, entry.z, entry.w, false, s.words);
        if (threadIdx.x == 0) ls.tags[(size_t)entry.x * NTAG + f] = make_uint2(entry.w, seq);
    }
}
// where a regeneration block of the step grid keeps its scratch in the step kernel's LDS area (dwords)
constexpr int REGEN_SCRATCH_AT = 0, REGEN_PREFIX_AT = REGEN_SCRATCH_AT + (int)sizeof(WorldScratch) / 4;
static_assert(REGEN_PREFIX_AT + NSUB <= ENVS_PER_BLOCK * L_ENV_DWORDS, "regeneration scratch outgrows the environments' area");

// A launch of regeneration blocks only (before and after a rollout): generates every world on the
// lists and empties them, with the bookkeeping of a step launch that has no step blocks.  A kernel
// of its own, at the occupancy of the generator instead of that of the step kernel.
template <bool PERLIN, int NT>
__global__ __launch_bounds__(NT, PERLIN ? PERLIN_WAVES : VALUE_WAVES) void kf_drain(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps, const Luts* __restrict__ luts, Lists ls)
{
    __shared__ WorldScratch s_gen;
    __shared__ uint32_t s_prefix[NSUB];
    const la::Ticket ticket = la::enter_launch_queue(ls, s_prefix);
    regeneration_queue<NT, PERLIN>(envs, maps, ls, ticket.seq, s_gen, s_prefix, (int)gridDim.x, luts->perlin_cs);
    la::leave_launch(ls, ticket);
}

// ---------------------------------------------------------------------------------------------
// step: one wavefront per environment, four environments per block; the grid starts with the
// regeneration blocks for the episodes that ended in the previous launch.
// EAGER: the window of the spare world's start position is fetched in every step, with the current
// window, so that an episode that ends switches worlds without a further trip to memory.  With a
// few thousand environments the launch ends when its slowest block ends, and that trip would sit
// on exactly those blocks (+0.7 us per launch at 4,096 environments); with tens of thousands the
// kernel is bound by instruction issue and the hundred instructions per step cost more than the
// rare trip (255 -> 216 us per launch at 65,536 environments).
// PERLIN: the regeneration blocks generate Perlin worlds (a kernel of its own, so that the value-noise
// kernel carries none of that code).
// GW: lanes per environment (see Lanes): 64 = one wavefront per environment, four environments per
// block; 16 = four environments per wavefront, sixteen per block.
// DRAW (pixels): a block holds one environment, which its first wavefront steps, and all its wavefronts then draw the picture, from the
// record and mobs in LDS.
// FLOATS: see floats_kept.
// FULL (bytes; see chip_is_full): every further block on a compute unit hides waits, and the compiler is bounded to as many: eight,
// the most that registers and LDS allow where worlds are of value noise (32,768 environments, bytes: 79.1 us with six, 76.3 with seven, 74.7
// with eight).  Below that the launch waits for its slowest wavefronts, which spill fewer scalars with more registers (4,096: 13.4 us, 13.6).
constexpr int step_bound(bool bytes, bool full, bool perlin, int lanes) { return lanes != 64 ? 2 : !full || !bytes ? 5 : perlin ? 6 : 8; }
template <bool F32, bool EAGER, bool PERLIN, int GW, bool DRAW = false, cx::Keep FLOATS = cx::Keep::THROUGH, bool FULL = !EAGER>
__global__ __launch_bounds__(BLOCK, step_bound(!F32 && !DRAW, FULL, PERLIN, GW)) void kf_step(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps,
                                                const Luts* __restrict__ luts, const int32_t* __restrict__ actions,
                                                uint8_t* __restrict__ obs, float* __restrict__ reward,
                                                uint8_t* __restrict__ done, Lists ls, Params p, int regen_blocks)
{
    using G = Lanes<GW>;
    static_assert(!DRAW || (GW == 64 && !F32), "pictures are drawn behind a step by a wavefront");
    constexpr int EPB = DRAW ? 1 : BLOCK / GW;               // environments per block
    constexpr bool HALVES = !F32 && !DRAW && FULL && GW == 64;
    constexpr int REC_IT = REC_DWORDS / GW > 0 ? REC_DWORDS / GW : 1;
    static_assert(REC_DWORDS % GW == 0 || GW > REC_DWORDS, "the record is moved in whole turns of the group");
    static_assert(GW >= MOBTAB_DWORDS && GW >= NTAG && GW >= FLOORS + 1, "a group holds a mob table, the tags and the header in one turn");
    constexpr int ENV_DWORDS_LDS = GW == 64 ? staged_dwords<HALVES> : L_ENV_DWORDS;
    constexpr int REGEN_DWORDS = REGEN_PREFIX_AT + NSUB;
    __shared__ __attribute__((aligned(16))) uint32_t s_env[EPB * ENV_DWORDS_LDS > REGEN_DWORDS ? EPB * ENV_DWORDS_LDS : REGEN_DWORDS];
    __shared__ float s_lut[LUT_FLOATS];
    using Picture = std::conditional_t<DRAW, PictureScratch, uint32_t>;
    __shared__ __attribute__((aligned(16))) Picture s_picture;
    __shared__ uint32_t s_mob[DRAW ? NSLOT : 1];
    const int tid = threadIdx.x, w = tid / GW, l = tid % GW;
    if ((int)blockIdx.x < regen_blocks) {
        const la::Ticket ticket = la::enter_launch_queue(ls, s_env + REGEN_PREFIX_AT);
        regeneration_queue<BLOCK, PERLIN>(envs, maps, ls, ticket.seq, *reinterpret_cast<WorldScratch*>(s_env + REGEN_SCRATCH_AT), s_env + REGEN_PREFIX_AT,
                                          regen_blocks, luts->perlin_cs);
        la::leave_launch(ls, ticket);
        return;
    }
    const uint32_t step_block = blockIdx.x - (uint32_t)regen_blocks;
    const int env = (int)step_block * EPB + (DRAW ? 0 : w);
    const bool active = env < p.n && (!DRAW || w == 0);
    uint32_t* genv = envs + (size_t)(active ? env : 0) * ENV_DWORDS;
    // Everything that depends on the environment's number alone is fetched before the launch
    // bookkeeping, whose own trip to memory then costs nothing extra: the record, the action, and
    // what a finished episode needs from the spare world (its tags, its ladders and potion map).
    uint32_t rec_word[REC_IT], hdr = 0u;
    int action_raw = 0;
    uint2 tag = make_uint2(0u, 0u);
#pragma unroll
    for (int it = 0; it < REC_IT; ++it) rec_word[it] = 0u;
    // what the renderer looks up in tables: asked for now, used at the end of the step
    RenderAux<GW> aux;
    fetch_scalar_fields<GW>(l, aux);
    aux.lut = s_lut;
    if (tid < LUT_FLOATS) s_lut[tid] = lut_entry(tid, luts);
    if (active) {
#pragma unroll
        for (int it = 0; it < REC_IT; ++it) if (l + GW * it < REC_DWORDS) rec_word[it] = genv[l + GW * it];
        action_raw = actions[env];
        if (l < NTAG) tag = ls.tags[(size_t)env * NTAG + l];
        if (l < FLOORS + 1) hdr = genv[SPARE_LADDER + l];
    }
    if constexpr (DRAW) prepare_picture(s_picture, luts);
    const la::Ticket ticket = la::enter_launch(ls, false, 0u);   // holds a block barrier: the conversion tables are in LDS
    const uint32_t seq = ticket.seq;
    if (active) {
        uint32_t* e = s_env + (DRAW ? 0 : w) * ENV_DWORDS_LDS;
#pragma unroll
        for (int it = 0; it < REC_IT; ++it) if (l + GW * it < REC_DWORDS) e[L_REC + l + GW * it] = rec_word[it];
        const int action = G::uni(action_raw);
        wave_sync();
        const RecordWords<GW> old{ e + L_REC, rec_word[0] };
        const uint32_t ep = old[R_EPISODE], lo = old[R_SEED_LO], hi = old[R_SEED_HI];
        const uint32_t table = day_table<GW>(l, old[R_MANA] >> 16, p.day_length, luts);
        MobRegs m;
        uint32_t qw, kept = 0u;
        Player P;
        // the window of the spare world's start position comes with the current window
        const uint8_t* spare = maps + map_offset((uint32_t)env, ep + 1u);
        Window<GW> spare_window;
        if (EAGER) spare_window.fetch(l, spare, 0, W / 2, W / 2);
        auto park = [&]() {
            if (l < NTAG) { e[L_SPARE_TAG + 2 * l] = tag.x; e[L_SPARE_TAG + 2 * l + 1] = tag.y; }
            if (l < FLOORS + 1) e[L_SPARE_HDR + l] = hdr;
            if (EAGER) spare_window.park(l, e + L_SPARE_WB, e + L_SPARE_WI);
        };
        StepOut o = step_env<GW>(l, (uint32_t)env, e, old, genv, maps + map_offset((uint32_t)env, ep), action, table, p, m, qw, P, kept, park);
        if (l == 0) { reward[env] = o.reward; done[env] = o.done ? 1 : 0; }
#pragma unroll
        for (int aw = 0; aw < 3; ++aw) count_unlocks<GW>(l, p.unlocks + (size_t)env * UNLOCK_STRIDE, aw, o.unlocked[aw]);
        bool write_back = !o.done, queued = false;
        uint32_t list_at = 0u;
        int floor_now = P.floor;
        if (!o.done) {
            if (l == 0) pack_player(e + L_REC, P, o.t);
            if (l < NPLANT) e[L_REC + R_PLANT + l] = qw;
            wave_sync();
        } else {
            // every part of the next world must have been written by an earlier launch
            constexpr uint32_t ALL = (1u << NTAG) - 1u;
            const bool ready = (G::ballot(l < NTAG && e[L_SPARE_TAG + 2 * (l < NTAG ? l : 0)] == ep + 1u &&
                                          e[L_SPARE_TAG + 2 * (l < NTAG ? l : 0) + 1] < seq) & ALL) == ALL;
            if (ready) {
                // start the new episode right here: fresh record from the spare world's ladders and
                // potion map, all mob tables empty, window of the start position from the other slot
                wave_sync();
#pragma unroll
                for (int it = 0; it < REC_IT; ++it)
                    if (l + GW * it < REC_DWORDS) e[L_REC + l + GW * it] = fresh_record_word(l + GW * it, e + L_SPARE_HDR, lo, hi, ep + 1u);
                if (EAGER) {
#pragma unroll
                    for (int it = 0; it < (WIN_DWORDS + GW - 1) / GW; ++it) {
                        const int i = l + GW * it;
                        if (i < WIN_DWORDS) { e[L_WB + i] = e[L_SPARE_WB + i]; e[L_WI + i] = e[L_SPARE_WI + i]; }
                    }
                } else {
                    load_window<GW>(l, spare, 0, W / 2, W / 2, e);
                }
#pragma unroll
                for (int it = 0; it < (FLOORS * MOBTAB_DWORDS + GW - 1) / GW; ++it) {
                    const int i = l + GW * it;
                    if (i < FLOORS * MOBTAB_DWORDS) genv[REC_DWORDS + i] = 0u;
                }
                clear_mob(m);
                floor_now = 0;
                o.wx0 = win_x0(W / 2); o.wy0 = win_y0(W / 2);
                wave_sync();
                write_back = true;
                if (l == 0) list_at = la::claim_entry(ls, seq, step_block);   // the place on the list; the entry follows after the rendering
                queued = true;
            } else if (l == 0) {
                la::append_slow(ls, (uint32_t)p.n, make_uint4((uint32_t)env, lo, hi, ep + 1u));
            }
        }
        if (write_back) {
#pragma unroll
            for (int it = 0; it < REC_IT; ++it) if (l + GW * it < REC_DWORDS) genv[l + GW * it] = e[L_REC + l + GW * it];
            if (l < MOBTAB_DWORDS) genv[REC_DWORDS + floor_now * MOBTAB_DWORDS + l] = l < NSLOT ? m.w : 0u;
            if (!DRAW && obs != nullptr) {
                aux.day = day_of<GW>(table, o.done);
                render_env<F32, GW, FLOATS, HALVES>(l, e, o.wx0, o.wy0, m.alive(), m.x(), m.y(), m.type(), luts, obs + (size_t)env * (F32 ? STRIDE_F32 : STRIDE_U8), &aux,
                                            FLOATS == cx::Keep::STREAM && floats_written_through(env, blockIdx.x));
            }
        }
        if (DRAW) {
            // an episode that ended without a spare world is not started anew here: its picture is that of the state in memory,
            // record and mobs, whatever the step has changed of the copies
            if (!write_back) {
#pragma unroll
                for (int it = 0; it < REC_IT; ++it) if (l + GW * it < REC_DWORDS) e[L_REC + l + GW * it] = genv[l + GW * it];
                wave_sync();
            }
            if (l < NSLOT) s_mob[l] = write_back ? m.w : genv[REC_DWORDS + ((e[L_REC + R_POS] >> 24) & 0xFu) * MOBTAB_DWORDS + l];
        }
        if (queued && l == 0) la::commit_entry(ls, seq, step_block, list_at, make_uint4((uint32_t)env, lo, hi, ep + 2u));
    }
    la::leave_launch(ls, ticket);
    if constexpr (DRAW) {
        __syncthreads();                    // record and mobs are in LDS, the step's changes to the map have left for memory
        const uint32_t* rec = s_env + L_REC;
        const uint8_t* map = maps + map_offset((uint32_t)env, rec[R_EPISODE]);
        uint8_t* out = obs + (size_t)env * STRIDE_PIXELS;
        if (cx::picture_kept(p.n, env, blockIdx.x, STRIDE_PIXELS)) draw_picture<cx::Keep::THROUGH>(s_picture, rec, s_mob, map, luts, out);
        else draw_picture<cx::Keep::STREAM>(s_picture, rec, s_mob, map, luts, out);
    }
}

// ---------------------------------------------------------------------------------------------
// A whole world by the calling wavefront alone, into its map slot; leaves the ten layout words in
// s->words and drops the cells around the start position into the windows.  Not inlined: it runs for
// few environments of a rollout, whose loop would otherwise pay for its registers in spills.
template <typename T> using Lds = T __attribute__((address_space(3)));
template <bool PERLIN>
__device__ __attribute__((noinline)) void generate_world(uint8_t* slot, Lds<WorldScratch>* scratch, Lds<uint32_t>* win_blocks, Lds<uint32_t>* win_items,
                                                         uint32_t lo, uint32_t hi, uint32_t env, uint32_t ep, const uint32_t* perlin_cs)
{
    WorldScratch& s = *(WorldScratch*)scratch;
    const int l = threadIdx.x & 63;
#pragma unroll 1
    for (int f = 0; f < FLOORS; ++f) {
        worldgen_floor_block<64, PERLIN, true>(slot, s.lat, s.layout, lo, hi, env, ep, f, (uint32_t*)win_blocks, (uint32_t*)win_items, perlin_cs);
        if (f == 0) {                             // the layout of floor 0 describes the whole world
            if (l < FLOORS + 1) s.words[l] = layout_word(s.layout, l);
            wave_sync();
        }
    }
}

// rollout: several steps in one launch (see craftax_rollout).  A wavefront keeps the record of its
// environment in LDS for the whole launch and walks it through the steps; nothing is exchanged
// between wavefronts, so they drift apart and the memory traffic of some overlaps the arithmetic
// of others.  Worlds stay one episode ahead as in the step kernel: an environment whose episode ends
// moves into the spare world in its other map slot (ladders and potion map from the header, the start
// window from the map).  The world after that one is not generated here: at the end of the launch
// the environment goes on the regeneration list, and the regeneration launch behind this one
// generates all of them with the whole chip.  Only an environment whose episode ends a second time in
// one launch has no spare world; its wavefront generates the next world on the spot.  Generated by the
// block at every end of an episode, worlds stalled whole blocks, and a launch lasted as long as the
// block with the most of them (64 steps: 4,096 environments 1,072 -> 900 us, 1,024: 780 -> 580, 100
// environments and 16 steps: 230 -> 150; with packed state, staged bytes and kept windows 660, 442, 117;
// the first 646 with the present generator).
// Before the launch the regeneration lists of the step kernel must be empty (the host runs a
// list-only launch first).
template <bool F32, bool PERLIN>
__global__ __launch_bounds__(BLOCK, 4) void kf_rollout(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps,
                                                       const Luts* __restrict__ luts, const int32_t* __restrict__ actions,
                                                       uint8_t* __restrict__ obs, float* __restrict__ reward,
                                                       uint8_t* __restrict__ done, Lists ls, Params p, int steps)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_env[ENVS_PER_BLOCK * staged_dwords<false>];
    __shared__ WorldScratch s_gen[ENVS_PER_BLOCK];
    __shared__ float s_lut[LUT_FLOATS];
    __shared__ uint32_t s_field[64];
    if (threadIdx.x < LUT_FLOATS) s_lut[threadIdx.x] = lut_entry((int)threadIdx.x, luts);
    if (threadIdx.x < 64) s_field[threadIdx.x] = SCALARS.fields[min((int)threadIdx.x, NVEC - 1)];
    __syncthreads();
    bool spare_ok;           // the world of the next episode is complete in the other map slot
    MobRegs m;               // the mob table of the current floor; in memory it is brought up to date when the player leaves the floor and at the end
    int action;              // fetched a step ahead
    uint32_t kept = 0u;      // window_key of the windows in LDS
    {
        const int w = threadIdx.x >> 6, l = threadIdx.x & 63, env = blockIdx.x * ENVS_PER_BLOCK + w;
        if (env >= p.n) return;
        uint32_t* e = s_env + w * staged_dwords<false>;
        const uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
        e[L_REC + l] = genv[l];
        wave_sync();
        const uint32_t ep = uniu(e[L_REC + R_EPISODE]);
        m.w = l < NSLOT ? genv[REC_DWORDS + (uniu(e[L_REC + R_POS]) >> 24) * MOBTAB_DWORDS + l] : 0u;
        action = uni(actions[env]);
        constexpr uint64_t ALL = (1ull << NTAG) - 1ull;
        spare_ok = (__ballot(l < NTAG && ls.tags[(size_t)env * NTAG + (l < NTAG ? l : 0)].x == ep + 1u) & ALL) == ALL;
    }
#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
        // Everything a lane derives from its index is derived again in every turn: the compiler would
        // otherwise keep dozens of such values alive across the whole loop and spill them.
        int tid_t = threadIdx.x;
        uint8_t* obs_t = obs;
        asm volatile("" : "+v"(tid_t));
        asm volatile("" : "+s"(obs_t));
        const int w = uni(tid_t >> 6), l = tid_t & 63;
        const int env = blockIdx.x * ENVS_PER_BLOCK + w;
        uint32_t* e = s_env + w * staged_dwords<false>;
        uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
        // The next action, asked for through a lane: a load to a scalar register would be waited for with the next access to LDS.
        int action_lane = 0;
        if (t + 1 < steps) action_lane = actions[(size_t)(t + 1) * p.n + blockIdx.x * ENVS_PER_BLOCK + (tid_t >> 6)];
        const RecordWords<64> old{ e + L_REC, e[L_REC + l] };
        const uint32_t ep = old[R_EPISODE];
        const uint32_t table = day_table<64>(l, old[R_MANA] >> 16, p.day_length, luts);
        uint32_t qw;
        Player P;
        StepOut o = step_env<64, true>(l, (uint32_t)env, e, old, genv, maps + map_offset((uint32_t)env, ep), action, table, p, m, qw, P, kept, []() {});
        action = uni(action_lane);          // arrived with what the step has read
        if (l == 0) { reward[(size_t)t * p.n + env] = o.reward; done[(size_t)t * p.n + env] = o.done ? 1 : 0; }
#pragma unroll
        for (int aw = 0; aw < 3; ++aw) count_unlocks<64>(l, p.unlocks + (size_t)env * UNLOCK_STRIDE, aw, o.unlocked[aw]);
        if (!o.done) {
            if (l == 0) pack_player(e + L_REC, P, o.t);
            if (l < NPLANT) e[L_REC + R_PLANT + l] = qw;
            wave_sync();
        } else {
            const uint32_t lo = old[R_SEED_LO], hi = old[R_SEED_HI];
            uint8_t* next = maps + map_offset((uint32_t)env, ep + 1u);
            uint32_t* words = e + L_SPARE_HDR;
            if (spare_ok) {
                if (l < FLOORS + 1) words[l] = genv[SPARE_LADDER + l];
                load_window(l, next, 0, W / 2, W / 2, e);
                spare_ok = false;
            } else {
                generate_world<PERLIN>(next, (Lds<WorldScratch>*)(s_gen + w), (Lds<uint32_t>*)(e + L_WB), (Lds<uint32_t>*)(e + L_WI), lo, hi, (uint32_t)env,
                                       ep + 1u, PERLIN ? luts->perlin_cs : nullptr);
                if (l < FLOORS + 1) words[l] = s_gen[w].words[l];
            }
            wave_sync();
            // fresh record, empty mob tables
            e[L_REC + l] = fresh_record_word(l, words, lo, hi, ep + 1u);
            for (int i = l; i < FLOORS * MOBTAB_DWORDS; i += 64) genv[REC_DWORDS + i] = 0u;
            wave_sync();
            clear_mob(m);
            kept = window_key(0, W / 2, W / 2);
            o.wx0 = win_x0(W / 2); o.wy0 = win_y0(W / 2);
        }
        if (obs != nullptr) {
            RenderAux<64> aux;
            aux.field[0] = s_field[l];
            aux.lut = s_lut;
            aux.day = day_of<64>(table, o.done);
            render_env<F32>(l, e, o.wx0, o.wy0, m.alive(), m.x(), m.y(), m.type(), luts, obs_t + (size_t)env * (F32 ? STRIDE_F32 : STRIDE_U8), &aux);
        }
        wave_sync();
    }
    // the record back; the world after this episode, if it is owed, for the regeneration launch
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, env = blockIdx.x * ENVS_PER_BLOCK + w;
    const uint32_t* e = s_env + w * staged_dwords<false>;
    uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
    genv[l] = e[L_REC + l];
    if (l < MOBTAB_DWORDS) genv[REC_DWORDS + (uniu(e[L_REC + R_POS]) >> 24) * MOBTAB_DWORDS + l] = l < NSLOT ? m.w : 0u;
    if (!spare_ok && l == 0)
        la::append_after_step(ls, (uint32_t)env / ENVS_PER_BLOCK, make_uint4((uint32_t)env, e[L_REC + R_SEED_LO], e[L_REC + R_SEED_HI], e[L_REC + R_EPISODE] + 1u));
}

// Serves the slow list: generates the world of the new episode in place (nine blocks each, looping
// if the list is longer than the grid); the block of floor 0 writes the fresh record, renders the
// first observation and asks the next step launch for the world after it.  Runs after the step
// kernel, and only when the episode cap is 1.
template <bool F32>
__global__ __launch_bounds__(GEN_THREADS) void kf_reset_list(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps,
                                                            const Luts* __restrict__ luts, uint8_t* __restrict__ obs, Lists ls, int perlin,
                                                            const uint8_t* __restrict__ done, int n, int pool)
{
    __shared__ uint32_t s_lat[LAT_WORDS];
    __shared__ GenLayout s_layout;
    __shared__ uint32_t s_words[FLOORS + 1];
    __shared__ __attribute__((aligned(16))) uint32_t s_env[staged_dwords<false>];
    __shared__ uint32_t s_rank[(GEN_THREADS + 63) / 64];
    // Optimistic resets (pool != 0): the world comes from this step's pool.  The step kernel has
    // already advanced the launch number: it is the index of the step just done + 2.  The pool is
    // keyed by the seed of environment 0 (whoever rewrites that record writes the same seed back).
    const uint32_t step_index = pool ? *counter(ls, la::CT_SEQ) - 2u : 0u;
    const uint32_t pool_lo = pool ? envs[R_SEED_LO] : 0u, pool_hi = pool ? envs[R_SEED_HI] : 0u;
    const uint32_t pool_size = (uint32_t)n / cx::POOL_RATIO ? (uint32_t)n / cx::POOL_RATIO : 1u;
    const uint32_t count = la::slow_count(ls, ls.slow_cap);
    const uint32_t slot = blockIdx.x / FLOORS, slots = gridDim.x / FLOORS;
    const int f = blockIdx.x % FLOORS;
    if (slot >= count) return;
    const int tid = threadIdx.x;
    for (uint32_t i = slot; i < count; i += slots) {
        const uint4 entry = ls.slow[i];
        if (entry.x == ENTRY_VOID) continue;
        const uint32_t env = entry.x, lo = entry.y, hi = entry.z, ep = entry.w;
        uint32_t wlo = lo, whi = hi, wenv = env, wep = ep;   // the world's identity: the environment's own ...
        if (pool) {
            // ... or the pool's: rank of this environment among the finished ones = finished environments before it
            uint32_t before = 0u;
            for (uint32_t j = (uint32_t)tid; j < env; j += GEN_THREADS) before += done[j];
            for (int o = 32; o > 0; o >>= 1) before += __shfl_down(before, o);
            __syncthreads();                                  // the previous entry's ranks have been read
            if ((tid & 63) == 0) s_rank[tid >> 6] = before;
            __syncthreads();
            uint32_t rank = 0u;
#pragma unroll
            for (int w = 0; w < (GEN_THREADS + 63) / 64; ++w) rank += s_rank[w];
            const cx::U4 sh = cx::philox4x32_10(0xFFFFFFFFu, 2u, step_index, cx::DOM_WORLDGEN << 16, pool_lo, pool_hi);
            wlo = pool_lo; whi = pool_hi; wenv = cx::POOL_ENV | ((cx::choice(sh.w[0], pool_size) + rank) % pool_size); wep = step_index;
        }
        worldgen_floor_block<GEN_THREADS, true>(maps + map_offset(env, ep), s_lat, s_layout, wlo, whi, wenv, wep, f,
                                                s_env + L_WB, s_env + L_WI,
                                                perlin ? luts->perlin_cs : nullptr);
        if (f == 0) {
            publish_world(envs + (size_t)env * ENV_DWORDS, s_layout, lo, hi, ep, true, s_words);
            if (tid < REC_DWORDS) s_env[L_REC + tid] = fresh_record_word(tid, s_words, lo, hi, ep);
            if (tid == 96 && !pool) la::append_after_step(ls, env / ENVS_PER_BLOCK, make_uint4(env, lo, hi, ep + 1u));
            __syncthreads();
            if (obs != nullptr && tid < 64)
                render_env<F32>(tid, s_env, win_x0(W / 2), win_y0(W / 2), 0, 0, 0, 0, luts,
                                obs + (size_t)env * (F32 ? STRIDE_F32 : STRIDE_U8));
        }
        __syncthreads();
    }
    // the last working block empties the list (nine blocks per served slot)
    if (tid == 0) {
        const uint32_t workers = (count < slots ? count : slots) * FLOORS;
        if (atomicAdd(counter(ls, la::CT_SLOW_FINISHED), 1u) == workers - 1u) { *counter(ls, la::CT_SLOW) = 0u; *counter(ls, la::CT_SLOW_FINISHED) = 0u; }
    }
}

template <bool F32, cx::Keep FLOATS = cx::Keep::THROUGH>
__global__ __launch_bounds__(BLOCK) void kf_observe(const uint32_t* __restrict__ envs, const uint8_t* __restrict__ maps,
                                                   const Luts* __restrict__ luts, uint8_t* __restrict__ obs, int n)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_env[ENVS_PER_BLOCK * staged_dwords<false>];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int env = blockIdx.x * ENVS_PER_BLOCK + w;
    if (env >= n) return;
    uint32_t* e = s_env + w * staged_dwords<false>;
    const uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
    e[L_REC + l] = genv[l];
    wave_sync();
    const uint32_t pos = uniu(e[L_REC + R_POS]), ep = uniu(e[L_REC + R_EPISODE]);
    const int px = pos & 0xFF, py = (pos >> 8) & 0xFF, f = (pos >> 24) & 0xF;
    const Mob u = unpack_mob(l < NSLOT ? genv[REC_DWORDS + f * MOBTAB_DWORDS + l] : 0u);
    load_window(l, maps + map_offset((uint32_t)env, ep), f, px, py, e);
    wave_sync();
    render_env<F32, 64, FLOATS>(l, e, win_x0(px), win_y0(py), u.alive, u.x, u.y, u.type, luts,
                                obs + (size_t)env * (F32 ? STRIDE_F32 : STRIDE_U8), nullptr, FLOATS == cx::Keep::STREAM && floats_written_through(env, blockIdx.x));
}

// Noise mutation (section "Craftax-1B: UED"): one block per (environment, floor).  The level is the
// vector of the Perlin angles of every noise lattice: the overworld's 228, then 98 for each of the
// cave floors 2, 5, 6, 7.  The block of a floor adds to its own segment a uniform offset in
// [-amplitude, amplitude] per element (u16 number i of stream (round, 1) of the mutation domain, i
// counted over the whole vector) and generates the floor of the current episode again from the
// turned lattice; the block of floor 0 also starts the episode over.  It writes every word of the
// record but the episode and the seed, which the other blocks read and which stay as they are, so one
// launch does it all (1,000 levels, floor 0 in a launch of its own behind the others: 131 us, one launch 92 then; now 49 by blocks
// and 31 by single wavefronts).
__device__ inline int theta_offset(int f)
{
    return f == 0 ? 0 : LAT0_U16 + LATC_U16 * (f == 2 ? 0 : (f == 5 ? 1 : (f == 6 ? 2 : 3)));
}
template <int NT>
__global__ __launch_bounds__(NT, PERLIN_WAVES) void kf_mutate_noise(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps, const Luts* __restrict__ luts,
                                                                uint16_t* __restrict__ theta, int first, uint32_t k0, uint32_t k1,
                                                                uint32_t round, uint32_t amplitude)
{
    __shared__ uint32_t s_lat[LAT_WORDS];
    __shared__ uint16_t s_theta[LAT_TOTAL];
    __shared__ GenLayout s_layout;
    __shared__ uint32_t s_words[FLOORS + 1];
    const FloorBlock block = floor_block();
    const int tid = threadIdx.x, slot = block.world, f = block.floor;
    const uint32_t env = (uint32_t)first + (uint32_t)slot;
    uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
    const uint32_t ep = genv[R_EPISODE], lo = genv[R_SEED_LO], hi = genv[R_SEED_HI];
    const bool noisy = f == 0 || is_cave(f);
    for (int k = tid; k < LAT_TOTAL; k += NT) {
        uint16_t v = 0;
        const int len = f == 0 ? LAT0_U16 : LATC_U16;
        if (noisy && k < len) {
            const int i = theta_offset(f) + k;
            uint16_t* th = theta + (size_t)slot * CRAFTAX_FULL_THETA_LEN + i;
            const cx::U4 d = cx::philox4x32_10(env, round, 1u, (cx::DOM_MUTATE << 16) | (uint32_t)(i >> 3), k0, k1);
            const uint32_t w = d.w[(i >> 1) & 3], d16 = (i & 1) ? (w >> 16) : (w & 0xFFFFu);
            const int u = (int)((d16 * (2u * amplitude + 1u)) >> 16) - (int)amplitude;
            v = (uint16_t)(((int)(*th & 1023u) + u) & 1023);
            *th = v;
        }
        s_theta[k] = v;
    }
    __syncthreads();
    worldgen_floor_block<NT, true>(maps + map_offset(env, ep), s_lat, s_layout, lo, hi, env, ep, f, nullptr, nullptr,
                                            luts->perlin_cs, noisy ? s_theta : nullptr);
    if (f == 0) publish_world<true>(genv, s_layout, lo, hi, ep, true, s_words);
}

// ---------------------------------------------------------------------------------------------
// canonical dumps: one block per (environment, floor), a thread moving runs of 8 cells of all three maps of
// the dump (63 KB, so a copy with some arithmetic: byte by byte, one block per environment, 1,000
// dumps took 34 us, now 16.5, 6.3 TB/s of the dumps and maps); the block of floor 0 also unpacks the
// record.  A dump is a multiple of 8 bytes long; the pieces are moved without assuming more than byte
// alignment of the caller's array.
__device__ inline uint2 load8(const uint8_t* p) { uint2 v; __builtin_memcpy(&v, p, 8); return v; }
__device__ inline void store8(uint8_t* p, uint2 v) { __builtin_memcpy(p, &v, 8); }
__global__ __launch_bounds__(GEN_THREADS) void kf_export(const uint32_t* __restrict__ envs, const uint8_t* __restrict__ maps,
                                                  craftax_full_env_dump* __restrict__ dumps, int first)
{
    const int slot = blockIdx.x / FLOORS, floor = blockIdx.x % FLOORS, env = first + slot, tid = threadIdx.x;
    craftax_full_env_dump* d = dumps + slot;
    const uint32_t* r = envs + (size_t)env * ENV_DWORDS;
    if (tid < RUNS) {
        const uint8_t* em = maps + map_offset((uint32_t)env, r[R_EPISODE]) + (size_t)floor * 2 * CELLS + tid * RUN;
        const uint2 b = *reinterpret_cast<const uint2*>(em), il = *reinterpret_cast<const uint2*>(em + CELLS);
        store8(d->block[floor] + tid * RUN, b);
        store8(d->item[floor] + tid * RUN, make_uint2(il.x & 0x07070707u, il.y & 0x07070707u));
        store8(d->light[floor] + tid * RUN, make_uint2((il.x >> 3) & 0x1F1F1F1Fu, (il.y >> 3) & 0x1F1F1F1Fu));
    }
    if (floor != 0) return;
    if (tid == 0) {
        d->px = r[R_POS] & 0xFF; d->py = (r[R_POS] >> 8) & 0xFF; d->dir = (r[R_POS] >> 16) & 0xFF; d->floor = (r[R_POS] >> 24) & 0xF;
        const uint32_t fl = r[R_FLAGS], at = r[R_ATTR];
        d->sleeping = fl & 1; d->resting = (fl >> 1) & 1; d->learned_fireball = (fl >> 2) & 1; d->learned_iceball = (fl >> 3) & 1;
        d->book = (fl >> 4) & 3; d->pickaxe = (fl >> 6) & 7; d->sword = (fl >> 9) & 7; d->sword_ench = (fl >> 12) & 3;
        d->bow = (fl >> 14) & 1; d->bow_ench = (fl >> 15) & 3; d->boss_vulnerable = (fl >> 17) & 1; d->boss_hits = (fl >> 18) & 15;
        for (int i = 0; i < 4; ++i) { d->armour[i] = (at >> (2 * i)) & 3; d->armour_ench[i] = (at >> (8 + 2 * i)) & 3; }
        d->xp = (at >> 16) & 15; d->dex = (at >> 20) & 7; d->str = (at >> 23) & 7; d->intel = (at >> 26) & 7;
        for (int i = 0; i < 10; ++i) d->inv[i] = (r[R_INV + (i >> 2)] >> (8 * (i & 3))) & 0xFF;
        for (int i = 0; i < 6; ++i) { const int b = 10 + i; d->potion[i] = (r[R_INV + (b >> 2)] >> (8 * (b & 3))) & 0xFF; }
        for (int i = 0; i < 4; ++i) { d->vit[i] = (int8_t)((r[R_VIT] >> (8 * i)) & 0xFF); d->cnt[i] = (int16_t)(int8_t)(r[R_CNT] >> (8 * i)); }
        d->vit[4] = (int8_t)(r[R_MANA] & 0xFF); d->cnt[4] = (int16_t)(int8_t)(r[R_MANA] >> 8);
        for (int i = 0; i < 6; ++i) d->potion_effect[i] = (r[R_PERM] >> (3 * i)) & 7;
        d->visited = (uint16_t)((r[R_PERM] >> 18) & 0x1FF);
        for (int i = 0; i < FLOORS; ++i) {
            d->kills[i] = (r[R_KILLS + (i >> 2)] >> (8 * (i & 3))) & 0xFF;
            const uint32_t lw = r[R_LADDER + i];
            d->ladder_up[i][0] = lw & 0xFF; d->ladder_up[i][1] = (lw >> 8) & 0xFF;
            d->ladder_down[i][0] = (lw >> 16) & 0xFF; d->ladder_down[i][1] = (lw >> 24) & 0xFF;
        }
        d->pad_a = 0; d->pad_b = 0; d->pad_c[0] = d->pad_c[1] = 0; d->pad0 = 0;
        for (int i = 0; i < 4; ++i) d->pad1[i] = 0;
        for (int i = 0; i < 3; ++i) d->ach[i] = r[R_ACH + i];
        d->t = r[R_T]; d->episode = r[R_EPISODE]; d->env = (uint32_t)env;
        d->seed = (uint64_t)r[R_SEED_LO] | ((uint64_t)r[R_SEED_HI] << 32);
    }
    if (tid < FLOORS * NSLOT) {
        const int f = tid / NSLOT, k = tid - f * NSLOT;
        const Mob m = unpack_mob(r[REC_DWORDS + f * MOBTAB_DWORDS + k]);
        craftax_full_mob o;
        o.alive = m.alive; o.x = m.x; o.y = m.y; o.dir = m.dir; o.hp = (int8_t)m.hp; o.cd = m.cd; o.type = m.type; o.pad = 0;
        d->mob[f][k] = o;
    }
    if (tid >= 128 && tid < 128 + NPLANT) {
        const uint32_t q = r[R_PLANT + tid - 128];
        craftax_plant o;
        o.alive = q & 1u; o.x = (q >> 1) & 63u; o.y = (q >> 7) & 63u; o.pad = 0; o.age = (uint16_t)(q >> 16);
        d->plant[tid - 128] = o;
    }
}

// The record of an import (all threads of the block call).
template <int NT>
__device__ inline void import_record(uint32_t* __restrict__ r, const Lists& ls, uint32_t env, const craftax_full_env_dump* __restrict__ d, const Params& p)
{
    __shared__ uint32_t s[ENV_DWORDS];
    const int tid = threadIdx.x;
    la::cancel_entries(ls, env);   // whatever was queued for this environment belongs to the episode that is being replaced
    for (int i = tid; i < ENV_DWORDS; i += NT) s[i] = 0u;
    __syncthreads();
    if (tid == 0) {
        s[R_POS] = (uint32_t)min((int)d->px, W - 1) | ((uint32_t)min((int)d->py, W - 1) << 8) | ((uint32_t)(d->dir & 7) << 16) |
                   ((uint32_t)min((int)d->floor, FLOORS - 1) << 24);
        s[R_FLAGS] = (uint32_t)(d->sleeping & 1) | ((uint32_t)(d->resting & 1) << 1) | ((uint32_t)(d->learned_fireball & 1) << 2) |
                     ((uint32_t)(d->learned_iceball & 1) << 3) | ((uint32_t)(d->book & 3) << 4) | ((uint32_t)(d->pickaxe & 7) << 6) |
                     ((uint32_t)(d->sword & 7) << 9) | ((uint32_t)(d->sword_ench & 3) << 12) | ((uint32_t)(d->bow & 1) << 14) |
                     ((uint32_t)(d->bow_ench & 3) << 15) | ((uint32_t)(d->boss_vulnerable & 1) << 17) | ((uint32_t)(d->boss_hits & 15) << 18);
        uint32_t at = ((uint32_t)(d->xp & 15) << 16) | ((uint32_t)(d->dex & 7) << 20) | ((uint32_t)(d->str & 7) << 23) | ((uint32_t)(d->intel & 7) << 26);
        for (int i = 0; i < 4; ++i) at |= ((uint32_t)(d->armour[i] & 3) << (2 * i)) | ((uint32_t)(d->armour_ench[i] & 3) << (8 + 2 * i));
        s[R_ATTR] = at;
        for (int i = 0; i < 10; ++i) s[R_INV + (i >> 2)] |= (uint32_t)min((int)d->inv[i], 99) << (8 * (i & 3));
        for (int i = 0; i < 6; ++i) { const int b = 10 + i; s[R_INV + (b >> 2)] |= (uint32_t)min((int)d->potion[i], 99) << (8 * (b & 3)); }
        uint32_t wv = 0, wc = 0;
        for (int i = 0; i < 4; ++i) {
            wv |= (uint32_t)max(0, min(31, (int)d->vit[i])) << (8 * i);
            wc |= (uint32_t)(max(-128, min(127, (int)d->cnt[i])) & 0xFF) << (8 * i);
        }
        s[R_VIT] = wv; s[R_CNT] = wc;
        s[R_MANA] = (uint32_t)max(0, min(31, (int)d->vit[4])) | ((uint32_t)(max(-128, min(127, (int)d->cnt[4])) & 0xFF) << 8) |
                    ((d->t % p.day_length) << 16);
        uint32_t pm = (uint32_t)(d->visited & 0x1FF) << 18;
        for (int i = 0; i < 6; ++i) pm |= (uint32_t)(d->potion_effect[i] & 7) << (3 * i);
        s[R_PERM] = pm;
        for (int i = 0; i < FLOORS; ++i) {
            s[R_KILLS + (i >> 2)] |= (uint32_t)d->kills[i] << (8 * (i & 3));
            s[R_LADDER + i] = (uint32_t)min((int)d->ladder_up[i][0], W - 1) | ((uint32_t)min((int)d->ladder_up[i][1], W - 1) << 8) |
                              ((uint32_t)min((int)d->ladder_down[i][0], W - 1) << 16) | ((uint32_t)min((int)d->ladder_down[i][1], W - 1) << 24);
        }
        for (int i = 0; i < 3; ++i) s[R_ACH + i] = d->ach[i];
        s[R_T] = d->t; s[R_EPISODE] = d->episode;
        s[R_SEED_LO] = (uint32_t)d->seed; s[R_SEED_HI] = (uint32_t)(d->seed >> 32);
    }
    for (int i = tid; i < FLOORS * NSLOT; i += NT) {
        const int f = i / NSLOT, k = i - f * NSLOT;
        const craftax_full_mob u = d->mob[f][k];
        Mob m;
        m.alive = u.alive & 1; m.x = min((int)u.x, W - 1); m.y = min((int)u.y, W - 1); m.dir = u.dir & 7; m.hp = max(0, min(31, (int)u.hp)); m.cd = min(15, (int)u.cd);
        m.type = min((int)u.type, 18);
        s[REC_DWORDS + f * MOBTAB_DWORDS + k] = pack_mob(m);
    }
    if (tid < NPLANT) {
        const craftax_plant u = d->plant[tid];
        s[R_PLANT + tid] = (u.alive & 1) ? (1u | ((uint32_t)min((int)u.x, W - 1) << 1) | ((uint32_t)min((int)u.y, W - 1) << 7) | ((uint32_t)u.age << 16)) : 0u;
    }
    __syncthreads();
    for (int i = tid; i < SPARE_LADDER; i += NT) r[i] = s[i];   // the spare world's description follows
}

// Import packs into the record's bit fields: counts 0..99, vitals 0..31, counters -128..127, mob
// hp 0..31, cooldown 0..15, creature type 0..18, experience 0..15, coordinates 0..47, floor 0..8,
// block ids 1..36, items 0..4, light 0..20 (every state the rules can reach is); values outside
// are brought into range so that no kernel ever indexes beyond its tables or buffers.
// One block per (environment, floor): it takes the floor in, and generates the same floor of the world
// of the next episode into the spare slot, so that the copy of some blocks overlaps the arithmetic of
// others; the block of floor 0 also packs the record.  (A copy byte by byte and a second launch for
// the spare worlds: 50 + 87 us for 1,000 Perlin worlds, one launch 101 then; now 44 by blocks and 39 by single wavefronts.)
template <bool PERLIN, int NT>
__global__ __launch_bounds__(NT, PERLIN ? PERLIN_WAVES : VALUE_WAVES) void kf_import(uint32_t* __restrict__ envs, uint8_t* __restrict__ maps, Lists ls,
                                                                        const craftax_full_env_dump* __restrict__ dumps, int first, Params p,
                                                                        const uint32_t* __restrict__ perlin_cs, int pool)
{
    __shared__ WorldScratch s_gen;
    const FloorBlock block = floor_block();
    const int slot = block.world, floor = block.floor, env = first + slot, tid = threadIdx.x;
    const craftax_full_env_dump* d = dumps + slot;
    const uint32_t lo = (uint32_t)d->seed, hi = (uint32_t)(d->seed >> 32), ep = d->episode;
    uint32_t* r = envs + (size_t)env * ENV_DWORDS;
#pragma unroll 2
    for (int run = tid; run < RUNS; run += NT) {
        const uint2 b = load8(d->block[floor] + run * RUN), it = load8(d->item[floor] + run * RUN), light = load8(d->light[floor] + run * RUN);
        auto blocks = [](uint32_t four) {
            uint32_t out = 0u;
#pragma unroll
            for (int i = 0; i < 32; i += 8) { const uint32_t v = (four >> i) & 0xFFu; out |= (v - 1u < (uint32_t)(B_COUNT - 1) ? v : (uint32_t)B_OOB) << i; }
            return out;
        };
        auto items = [](uint32_t four_items, uint32_t four_lights) {
            uint32_t out = 0u;
#pragma unroll
            for (int i = 0; i < 32; i += 8) {
                const uint32_t v = (four_items >> i) & 0xFFu;
                out |= ((v <= 4u ? v : 0u) | (min((four_lights >> i) & 0xFFu, 20u) << 3)) << i;
            }
            return out;
        };
        uint8_t* em = maps + map_offset((uint32_t)env, ep) + (size_t)floor * 2 * CELLS + run * RUN;
        *reinterpret_cast<uint2*>(em) = make_uint2(blocks(b.x), blocks(b.y));
        *reinterpret_cast<uint2*>(em + CELLS) = make_uint2(items(it.x, light.x), items(it.y, light.y));
    }
    if (floor == 0) import_record<NT>(r, ls, (uint32_t)env, d, p);
    worldgen_floor_block<NT, PERLIN>(maps + map_offset((uint32_t)env, ep + 1u), s_gen.lat, s_gen.layout, lo, hi, (uint32_t)env, ep + 1u, floor, nullptr,
                                              nullptr, perlin_cs);
    if (floor == 0) publish_world(r, s_gen.layout, lo, hi, ep + 1u, false, s_gen.words);
    if (tid == 0) ls.tags[(size_t)env * NTAG + floor] = make_uint2(pool ? 0u : ep + 1u, 0u);
}

// Level mutation of the overworld (section "Craftax-1B: UED"), as for Classic: up to 32 tries, try
// k drawing Philox block (env, round, 0, MUTATE | k) under the mutation seed; refused if the blocks
// are equal, a cell holds the player (when on floor 0), a live mob of floor 0 or an item, a block
// is a plant, or, restricted, the blocks are not of one group (stone and ores, gems included;
// grass and tree).  One lane per try, as for Classic (1,000 levels: 16.6 -> 4.8 us).
__device__ inline int swap_group(int b)
{
    if (b == B_STONE || b == B_COAL || b == B_IRON || b == B_DIAMOND || b == B_SAPPHIRE || b == B_RUBY) return 1;
    if (b == B_GRASS || b == B_TREE) return 2;
    return 0;
}
constexpr int MUTATE_SWAP_THREADS = 256;
__global__ void kf_mutate_swap(const uint32_t* __restrict__ envs, uint8_t* __restrict__ maps, int first, int count, uint32_t k0,
                               uint32_t k1, uint32_t round, int restricted, int32_t* __restrict__ tries)
{
    const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) / cx::MUTATE_TRIES), k = threadIdx.x % cx::MUTATE_TRIES;
    if (i >= count) return;
    const uint32_t env = (uint32_t)(first + i);
    const uint32_t* genv = envs + (size_t)env * ENV_DWORDS;
    uint8_t* m = maps + map_offset(env, genv[R_EPISODE]);
    const uint32_t pos = genv[R_POS];
    const int px = pos & 0xFF, py = (pos >> 8) & 0xFF, floor = (pos >> 24) & 0xF;
    auto taken = [&](int x, int y) {
        bool t = floor == 0 && x == px && y == py;
        for (int k = 0; k < NSLOT; ++k) {
            const Mob u = unpack_mob(genv[REC_DWORDS + k]);
            t |= u.alive && (int)u.x == x && (int)u.y == y;
        }
        return t || (m[il_off(0, x, y)] & 7) != IT_NONE;
    };
    const cx::U4 d = cx::philox4x32_10(env, round, 0u, (cx::DOM_MUTATE << 16) | (uint32_t)k, k0, k1);
    const int a = (int)cx::choice(d.w[0], cx::MUTATE_AREA * cx::MUTATE_AREA), b = (int)cx::choice(d.w[1], CELLS);
    const int c0 = (W - cx::MUTATE_AREA) / 2;
    const int ax = c0 + a % cx::MUTATE_AREA, ay = c0 + a / cx::MUTATE_AREA, bx = b % W, by = b / W;
    const int ba = m[block_off(0, ax, ay)], bb = m[block_off(0, bx, by)];
    bool accepted = ba != bb && !taken(ax, ay) && !taken(bx, by);
    accepted = accepted && ba != B_PLANT && ba != B_RIPE && bb != B_PLANT && bb != B_RIPE;
    accepted = accepted && (!restricted || (swap_group(ba) != 0 && swap_group(ba) == swap_group(bb)));
    const uint32_t good = (uint32_t)(__ballot(accepted) >> (threadIdx.x & 32u));
    const int done = __ffs((int)good);          // number of the first such try, counted from 1, or 0
    if (done == k + 1) {
        m[block_off(0, ax, ay)] = (uint8_t)bb;
        m[block_off(0, bx, by)] = (uint8_t)ba;
    }
    if (tries != nullptr && k == 0) tries[i] = done;
}

// ---------------------------------------------------------------------------------------------
namespace host {

static uint64_t round_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

bool config_ok(const craftax_config* c, std::string* why)
{
    if (c->abi_version != CRAFTAX_ABI_VERSION) { *why = "abi_version mismatch"; return false; }
    if (c->obs_mode != CRAFTAX_OBS_SYM_U8_F32 && c->obs_mode != CRAFTAX_OBS_SYM_F32 && c->obs_mode != CRAFTAX_OBS_PIXELS_F32) {
        *why = "the Craftax variant renders SYM_U8_F32, SYM_F32 or PIXELS_F32"; return false;
    }
    if (c->day_length < 2 || c->day_length > (uint32_t)MAX_DAY || (c->day_length & 1)) { *why = "day_length must be even and in 2..1024"; return false; }
    if (c->cap_zombie > 3 || c->cap_cow > 3 || c->cap_skeleton > 2) { *why = "caps: melee 0..3, passive 0..3, ranged 0..2"; return false; }
    if (c->cap_plant > (uint32_t)NPLANT) { *why = "cap_plant must be 0..10"; return false; }
    if (c->max_episode_steps == 0) { *why = "max_episode_steps must be positive"; return false; }
    if (c->reset_mode > CRAFTAX_RESET_POOL) { *why = "unknown reset_mode"; return false; }
    if (c->worldgen > CRAFTAX_WORLDGEN_PERLIN) { *why = "unknown worldgen"; return false; }
    if (c->reserved != 0) { *why = "reserved must be 0"; return false; }
    if (c->group_lanes != 0 && c->group_lanes != 16 && c->group_lanes != 64) { *why = "group_lanes must be 0, 16 or 64"; return false; }
    return true;
}

static Header make_header(const craftax_config* c, int n)
{
    Header h;
    std::memset(&h, 0, sizeof(h));
    h.magic = MAGIC; h.version = CRAFTAX_ABI_VERSION; h.n = (uint32_t)n; h.variant = c->variant;
    h.obs_mode = c->obs_mode; h.max_episode_steps = c->max_episode_steps; h.day_length = c->day_length;
    h.cap_melee = c->cap_zombie; h.cap_ranged = c->cap_skeleton; h.cap_passive = c->cap_cow; h.cap_plant = c->cap_plant;
    h.atlas_seed = c->atlas_seed; h.worldgen = c->worldgen; h.reset_mode = c->reset_mode;
    h.off_ctrs = cx::HEADER_BYTES;
    h.off_luts = h.off_ctrs + la::COUNTER_BYTES;
    h.off_envs = round_up(h.off_luts + sizeof(Luts), 256);
    h.off_maps = h.off_envs + (uint64_t)n * (ENV_DWORDS * 4);
    h.off_tags = round_up(h.off_maps + (uint64_t)n * 2 * MAP_BYTES, 256);     // two map slots per environment
    h.off_regen0 = round_up(h.off_tags + (uint64_t)n * NTAG * 8, 256);
    const uint64_t list_bytes = (uint64_t)NSUB * la::sub_list_capacity((uint64_t)n, MAX_ENVS_PER_STEP_BLOCK) * 16;
    h.off_regen1 = h.off_regen0 + list_bytes;
    h.off_slow = h.off_regen1 + list_bytes;
    h.off_unlocks = round_up(h.off_slow + (uint64_t)n * 16, 256);
    h.total = round_up(h.off_unlocks + (uint64_t)n * UNLOCK_STRIDE * 4, 256);
    return h;
}

// Day/night: phase i = t mod L, H = L/2, k = |i - H|, daylight = k^2 (3H - 2k) / H^3 (noon at
// t = 0); the paper only says the observation carries a day/night value in [0,1].
static void build_luts(const craftax_config* c, Luts* L)
{
    std::memset(L, 0, sizeof(*L));
    const uint64_t len = c->day_length, half = len / 2, den = half * half * half;
    for (uint64_t i = 0; i < len; ++i) {
        const uint64_t k = i < half ? half - i : i - half;
        const uint64_t num = k * k * (3 * half - 2 * k);
        L->daylight[i] = (float)((double)num / (double)den);
        L->zombie_thr[i] = (40u + 3u * (255u - (uint32_t)(255u * num / den))) << 20;
    }
    for (int i = 0; i < 100; ++i) L->sqrt10[i] = (float)(std::sqrt((double)i) / 10.0);
    for (int i = 0; i < 32; ++i) L->tenth[i] = (float)((double)i / 10.0);
    for (int i = 0; i < 32; ++i) L->light20[i] = (float)((double)i / 20.0);
    // unit gradients of the 1024 Perlin directions in Q14, rounded to nearest
    for (int a = 0; a < 1024; ++a) {
        const double turn = 6.283185307179586476925286766559 * (double)a / 1024.0;
        const int16_t c16 = (int16_t)std::lround(std::cos(turn) * 16384.0), s16 = (int16_t)std::lround(std::sin(turn) * 16384.0);
        L->perlin_cs[a] = (uint32_t)(uint16_t)c16 | ((uint32_t)(uint16_t)s16 << 16);
    }
    if (c->obs_mode != CRAFTAX_OBS_PIXELS_F32) return;
    // tile atlas: word idx of stream s is word idx % 4 of Philox block (0, s, 0, ATLAS | idx / 4)
    // under the atlas seed; streams 8 blocks, 9 items, 10 creatures, 11 player, 12 icons, 13 masks
    const uint32_t k0 = (uint32_t)c->atlas_seed, k1 = (uint32_t)(c->atlas_seed >> 32);
    auto fill = [&](uint32_t stream, uint32_t count, float* dst) {
        for (uint32_t i = 0; i < count; i += 4) {
            const cx::U4 r = cx::philox4x32_10(0u, stream, 0u, (cx::DOM_ATLAS << 16) | (i >> 2), k0, k1);
            for (uint32_t k = 0; k < 4 && i + k < count; ++k) dst[i + k] = (float)(r.w[k] >> 8) * (1.0f / 16777216.0f);
        }
    };
    fill(8, 37 * 300, L->atlas);
    fill(9, 5 * 300, L->atlas + AT_ITEM * 300);
    fill(10, 40 * 300, L->atlas + AT_CRE * 300);
    fill(11, 300, L->atlas + AT_PLAYER * 300);
    fill(12, 44 * 300, L->atlas + AT_ICON * 300);
    for (uint32_t i = 0; i < 46 * 100; i += 4) {
        const cx::U4 r = cx::philox4x32_10(0u, 13u, 0u, (cx::DOM_ATLAS << 16) | (i >> 2), k0, k1);
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t t = (i + k) / 100, pix = (i + k) % 100;
            if (r.w[k] >> 31) L->mask[t][pix / 10] |= (uint16_t)(1u << (pix % 10));
        }
    }
}

struct Ptrs { uint32_t* envs; uint8_t* maps; const Luts* luts; Lists ls; };
static Ptrs pointers(const void* state, const Header& h)
{
    uint8_t* base = const_cast<uint8_t*>(static_cast<const uint8_t*>(state));
    Ptrs q;
    q.luts = reinterpret_cast<const Luts*>(base + h.off_luts);
    q.envs = reinterpret_cast<uint32_t*>(base + h.off_envs);
    q.maps = base + h.off_maps;
    q.ls.ctr = reinterpret_cast<uint32_t*>(base + h.off_ctrs);
    q.ls.regen[0] = reinterpret_cast<uint4*>(base + h.off_regen0);
    q.ls.regen[1] = reinterpret_cast<uint4*>(base + h.off_regen1);
    q.ls.slow = reinterpret_cast<uint4*>(base + h.off_slow);
    q.ls.tags = reinterpret_cast<uint2*>(base + h.off_tags);
    q.ls.sub_cap = (uint32_t)la::sub_list_capacity((uint64_t)h.n, MAX_ENVS_PER_STEP_BLOCK);
    q.ls.slow_cap = h.n;
    return q;
}
static Params make_params(const void* state, const craftax_config* c, int n)
{
    Params p;
    p.unlocks = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(static_cast<const uint8_t*>(state)) + make_header(c, n).off_unlocks);
    p.n = n; p.max_episode_steps = c->max_episode_steps; p.day_length = c->day_length;
    p.cap_melee = c->cap_zombie; p.cap_ranged = c->cap_skeleton; p.cap_passive = c->cap_cow; p.cap_plant = c->cap_plant;
    p.worldgen = c->worldgen;
    return p;
}
// the gradient table for the kernels that choose the noise at run time: null = value noise
static const uint32_t* gradients(const craftax_config* c, const Ptrs& q)
{
    return c->worldgen == CRAFTAX_WORLDGEN_PERLIN ? q.luts->perlin_cs : nullptr;
}
static int check_launch(const char* what, std::string* err)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { *err = std::string(what) + ": " + hipGetErrorString(e); return CRAFTAX_E_HIP; }
    return CRAFTAX_OK;
}

size_t state_bytes(const craftax_config* cfg, int n) { return (size_t)make_header(cfg, n).total; }
size_t obs_bytes(const craftax_config* cfg)
{
    return cfg->obs_mode == CRAFTAX_OBS_PIXELS_F32 ? STRIDE_PIXELS : cfg->obs_mode == CRAFTAX_OBS_SYM_F32 ? STRIDE_F32 : STRIDE_U8;
}

int state_init(void* state, const craftax_config* cfg, int n, void* stream, std::string* err)
{
    const Header h = make_header(cfg, n);
    std::vector<uint8_t> staging((size_t)h.off_envs, 0);
    std::memcpy(staging.data(), &h, sizeof(Header));
    build_luts(cfg, reinterpret_cast<Luts*>(staging.data() + h.off_luts));
    hipError_t e = hipMemcpyAsync(state, staging.data(), staging.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);   // staging dies with this call
    if (e != hipSuccess) { *err = std::string("state_init copy: ") + hipGetErrorString(e); return CRAFTAX_E_HIP; }
    return CRAFTAX_OK;
}

int check_header(const void* header_bytes, const craftax_config* cfg, int n, std::string* err)
{
    Header got;
    std::memcpy(&got, header_bytes, sizeof(got));
    if (got.magic != MAGIC) { *err = "the memory holds no Craftax state blob"; return CRAFTAX_E_STATE; }
    if (got.version != CRAFTAX_ABI_VERSION) { *err = "the state blob was written by another library version"; return CRAFTAX_E_STATE; }
    if (got.n != (uint32_t)n) { *err = "the state blob holds another number of environments"; return CRAFTAX_E_COUNT; }
    const Header want = make_header(cfg, n);
    if (std::memcmp(&got, &want, sizeof(Header)) != 0) { *err = "the state blob was initialised with another configuration"; return CRAFTAX_E_CONFIG; }
    return CRAFTAX_OK;
}

int debug_bounds(uint32_t report[4], std::string* err)
{
#ifdef CRAFTAX_DEBUG_BOUNDS
    uint32_t mine[4] = {0u, 0u, 0u, 0u};
    const uint32_t zero[4] = {0u, 0u, 0u, 0u};
    hipError_t e = hipMemcpyFromSymbol(mine, HIP_SYMBOL(cx::g_bounds), sizeof(mine));
    if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(cx::g_bounds), zero, sizeof(zero));
    if (e != hipSuccess) { *err = std::string("debug_bounds: ") + hipGetErrorString(e); return CRAFTAX_E_HIP; }
    if (report[0] == 0u && mine[0] != 0u) { report[1] = mine[1]; report[2] = mine[2]; report[3] = mine[3]; }
    report[0] += mine[0];
#else
    (void)report; (void)err;
#endif
    return CRAFTAX_OK;
}

RecordLayout record_layout(const void* state, const craftax_config* cfg, int n)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    return RecordLayout{q.envs, ENV_DWORDS, R_ACH, 3, R_T, R_EPISODE, make_params(state, cfg, n).unlocks, UNLOCK_STRIDE};
}

// Every kernel that is launched for a layout and a noise, with the block sizes it is launched with.
template <bool F32, bool PERLIN, typename Fits>
static bool kernels_fit(const Fits& fits)
{
    auto step = [&](const char* name, const void* eager, const void* plain) { return fits(name, eager, BLOCK) && fits(name, plain, BLOCK); };
    auto floors = [&](const char* name, const void* blocks, const void* wavefronts) { return fits(name, blocks, GEN_THREADS) && fits(name, wavefronts, FLOOR_THREADS); };
    return step("kf_step", (const void*)kf_step<F32, true, PERLIN, 64>, (const void*)kf_step<F32, false, PERLIN, 64>) &&
           (F32 || fits("kf_step of small pooled batches", (const void*)kf_step<false, false, PERLIN, 64, false, cx::Keep::THROUGH, false>, BLOCK)) &&
           (!F32 || step("kf_step of large float buffers", (const void*)kf_step<true, true, PERLIN, 64, false, cx::Keep::PLAIN>, (const void*)kf_step<true, false, PERLIN, 64, false, cx::Keep::STREAM>)) &&
           (!F32 || (fits("kf_observe of large float buffers", (const void*)kf_observe<true, cx::Keep::PLAIN>, BLOCK) && fits("kf_observe of larger ones", (const void*)kf_observe<true, cx::Keep::STREAM>, BLOCK))) &&
           step("kf_step with pictures", (const void*)kf_step<false, true, PERLIN, 64, true>, (const void*)kf_step<false, false, PERLIN, 64, true>) &&
           step("kf_step (16 lanes)", (const void*)kf_step<F32, true, PERLIN, 16>, (const void*)kf_step<F32, false, PERLIN, 16>) &&
           fits("kf_rollout", (const void*)kf_rollout<F32, PERLIN>, BLOCK) && fits("kf_reset_list", (const void*)kf_reset_list<F32>, GEN_THREADS) &&
           fits("kf_observe", (const void*)kf_observe<F32>, BLOCK) && fits("kf_pixels", (const void*)kf_pixels, BLOCK) &&
           floors("kf_reset", (const void*)kf_reset<PERLIN, GEN_THREADS>, (const void*)kf_reset<PERLIN, FLOOR_THREADS>) &&
           floors("kf_drain", (const void*)kf_drain<PERLIN, GEN_THREADS>, (const void*)kf_drain<PERLIN, FLOOR_THREADS>) &&
           floors("kf_import", (const void*)kf_import<PERLIN, GEN_THREADS>, (const void*)kf_import<PERLIN, FLOOR_THREADS>) &&
           (!PERLIN || floors("kf_mutate_noise", (const void*)kf_mutate_noise<GEN_THREADS>, (const void*)kf_mutate_noise<FLOOR_THREADS>)) &&
           fits("kf_export", (const void*)kf_export, GEN_THREADS) && fits("kf_mutate_swap", (const void*)kf_mutate_swap, MUTATE_SWAP_THREADS);
}

int check_kernels(const craftax_config* cfg, std::string* err)
{
    int dev = 0, lds = 0, threads = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
        hipDeviceGetAttribute(&threads, hipDeviceAttributeMaxThreadsPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        *err = "no usable HIP device";
        return CRAFTAX_E_HIP;
    }
    const cx::DeviceLimits limits{(size_t)lds, threads};
    auto fits = [&](const char* name, const void* fn, int block) {
        hipFuncAttributes a;
        if (hipFuncGetAttributes(&a, fn) != hipSuccess) { (void)hipGetLastError(); *err = std::string("no attributes for ") + name; return false; }
        return cx::kernel_fits(cx::KernelNeeds{name, a.sharedSizeBytes, a.maxThreadsPerBlock, block}, limits, err);
    };
    const bool perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN;
    const bool ok = cfg->obs_mode == CRAFTAX_OBS_SYM_F32 ? (perlin ? kernels_fit<true, true>(fits) : kernels_fit<true, false>(fits))
                                                         : (perlin ? kernels_fit<false, true>(fits) : kernels_fit<false, false>(fits));
    return ok ? CRAFTAX_OK : CRAFTAX_E_CONFIG;
}

int reset(void* state, const craftax_config* cfg, int n, const uint64_t* seeds, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, floor_grid(2u * (unsigned)n), dim3((unsigned)threads), 0, (hipStream_t)stream, q.envs, q.maps, seeds, q.ls, gradients(cfg, q),
                           cfg->reset_mode == CRAFTAX_RESET_POOL ? 1 : 0, make_params(state, cfg, n).unlocks);
    };
    const bool perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN, blocks = floors_by_blocks(FloorWork::RESET, perlin, 2ll * n * FLOORS);
    if (perlin) { if (blocks) go(kf_reset<true, GEN_THREADS>, GEN_THREADS); else go(kf_reset<true, FLOOR_THREADS>, FLOOR_THREADS); }
    else { if (blocks) go(kf_reset<false, GEN_THREADS>, GEN_THREADS); else go(kf_reset<false, FLOOR_THREADS>, FLOOR_THREADS); }
    return check_launch("craftax_reset", err);
}

// Lanes per environment of the step kernel.  A whole wavefront (the default at every batch size)
// keeps the player's state and the 43-action code on the scalar unit, which works beside the vector
// unit.  Sixteen lanes put four environments in a wavefront and fill 14 of 16 lanes with mob slots
// instead of 14 of 64, but the player's code then runs on the vector unit, the kernel needs 48 KB
// of LDS (three wavefronts per SIMD instead of six to eight), and a wavefront
// renders four observations one after the other.  us per step, 16 / 64 lanes: 16.8 / 9.9 at 1,024
// environments, 17.4 / 12.8 at 4,096, 43.4 / 34.0 at 16,384, 138 / 118 at 65,536.  It is selectable
// (cfg->group_lanes = 16) and tested like the default.
static int group_lanes(const craftax_config* cfg, int n)
{
    (void)n;
    return cfg->group_lanes == 16 ? 16 : 64;
}

// one launch of the step kernel: the instance for this spare-world policy, this noise and this group width
template <bool F32>
static void launch_step(int gw, bool eager, bool perlin, dim3 grid, hipStream_t st, const Ptrs& q, const int32_t* actions, uint8_t* o, float* reward,
                        uint8_t* done, const Params& p, int rb)
{
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), 0, st, q.envs, q.maps, q.luts, actions, o, reward, done, q.ls, p, rb); };
    if (gw == 16) {
        if (perlin) { if (eager) go(kf_step<F32, true, true, 16>); else go(kf_step<F32, false, true, 16>); }
        else { if (eager) go(kf_step<F32, true, false, 16>); else go(kf_step<F32, false, false, 16>); }
    } else if (F32 && floats_kept(p.n) == cx::Keep::STREAM) {      // above EAGER_SPARE_ENVS but for a few hundred environments
        if (perlin) go(kf_step<true, false, true, 64, false, cx::Keep::STREAM>); else go(kf_step<true, false, false, 64, false, cx::Keep::STREAM>);
    } else if (F32 && eager && (p.n < FLOATS_THROUGH_FROM || floats_kept(p.n) == cx::Keep::PLAIN)) {
        if (perlin) go(kf_step<true, true, true, 64, false, cx::Keep::PLAIN>); else go(kf_step<true, true, false, 64, false, cx::Keep::PLAIN>);
    } else if (!F32 && !eager && !chip_is_full(p.n, perlin)) {
        if (perlin) go(kf_step<false, false, true, 64, false, cx::Keep::THROUGH, false>); else go(kf_step<false, false, false, 64, false, cx::Keep::THROUGH, false>);
    } else {
        if (perlin) { if (eager) go(kf_step<F32, true, true, 64>); else go(kf_step<F32, false, true, 64>); }
        else { if (eager) go(kf_step<F32, true, false, 64>); else go(kf_step<F32, false, false, 64>); }
    }
}

int step(void* state, const craftax_config* cfg, int n, const int32_t* actions, void* obs, float* reward, uint8_t* done,
         bool serve_slow, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    const Params p = make_params(state, cfg, n);
    hipStream_t st = (hipStream_t)stream;
    uint8_t* o = static_cast<uint8_t*>(obs);
    const int gw = group_lanes(cfg, n), epb = BLOCK / gw;
    const int sb = (n + epb - 1) / epb;
    const int rb = FLOORS * n < REGEN_BLOCKS ? FLOORS * n : REGEN_BLOCKS;    // persistent blocks serving a queue: any number works
    const dim3 grid((unsigned)(rb + sb)), rgrid((unsigned)(n < RESET_SLOTS ? n : RESET_SLOTS) * FLOORS);
    const int pool = cfg->reset_mode == CRAFTAX_RESET_POOL ? 1 : 0;
    // kf_reset_list serves the episodes that end before their spare world exists: with exact resets
    // only one-step episodes can, or a fresh episode whose world was edited before its first step
    // (serve_slow: the caller mutated or imported since the last step); with optimistic resets there
    // are no spare worlds and every finished episode is served there, its world depending on who
    // else finished
    const bool slow = p.max_episode_steps == 1u || pool != 0 || serve_slow;
    const int perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN ? 1 : 0;
    const bool bytes = cfg->obs_mode != CRAFTAX_OBS_SYM_F32 && cfg->obs_mode != CRAFTAX_OBS_PIXELS_F32;
    const bool eager = n <= eager_spare_envs(bytes, perlin != 0, gw) && pool == 0;
    if (cfg->obs_mode == CRAFTAX_OBS_PIXELS_F32) {
        if (o != nullptr && !slow) {
            // step and picture in one launch, whatever the lanes of a step without
            auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)(rb + n)), dim3(BLOCK), 0, st, q.envs, q.maps, q.luts, actions, o, reward, done, q.ls, p, rb); };
            if (perlin) { if (eager) go(kf_step<false, true, true, 64, true>); else go(kf_step<false, false, true, 64, true>); }
            else { if (eager) go(kf_step<false, true, false, 64, true>); else go(kf_step<false, false, false, 64, true>); }
            return check_launch("craftax_step", err);
        }
        // episodes are served behind the step: it runs without rendering, and the picture is drawn from the state both leave
        launch_step<false>(gw, eager, perlin != 0, grid, st, q, actions, nullptr, reward, done, p, rb);
        if (slow) hipLaunchKernelGGL(kf_reset_list<false>, rgrid, dim3(GEN_THREADS), 0, st, q.envs, q.maps, q.luts, (uint8_t*)nullptr, q.ls, perlin, done, n, pool);
        if (o != nullptr) hipLaunchKernelGGL(kf_pixels, dim3((unsigned)n), dim3(BLOCK), 0, st, q.envs, q.maps, q.luts, o);
    } else if (cfg->obs_mode == CRAFTAX_OBS_SYM_F32) {
        launch_step<true>(gw, eager, perlin != 0, grid, st, q, actions, o, reward, done, p, rb);
        if (slow) hipLaunchKernelGGL(kf_reset_list<true>, rgrid, dim3(GEN_THREADS), 0, st, q.envs, q.maps, q.luts, o, q.ls, perlin, done, n, pool);
    } else {
        launch_step<false>(gw, eager, perlin != 0, grid, st, q, actions, o, reward, done, p, rb);
        if (slow) hipLaunchKernelGGL(kf_reset_list<false>, rgrid, dim3(GEN_THREADS), 0, st, q.envs, q.maps, q.luts, o, q.ls, perlin, done, n, pool);
    }
    return check_launch("craftax_step", err);
}

int rollout(void* state, const craftax_config* cfg, int n, const int32_t* actions, int steps, void* obs, float* reward, uint8_t* done,
            void* stream, std::string* err)
{
    if (cfg->obs_mode == CRAFTAX_OBS_PIXELS_F32) { *err = "craftax_rollout needs a symbolic observation"; return CRAFTAX_E_CONFIG; }
    if (cfg->reset_mode != CRAFTAX_RESET_EXACT) { *err = "craftax_rollout needs exact resets"; return CRAFTAX_E_CONFIG; }
    const Ptrs q = pointers(state, make_header(cfg, n));
    const Params p = make_params(state, cfg, n);
    hipStream_t st = (hipStream_t)stream;
    uint8_t* o = static_cast<uint8_t*>(obs);
    const dim3 grid((unsigned)((n + ENVS_PER_BLOCK - 1) / ENVS_PER_BLOCK));
    const bool perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN;
    auto launch_drain = [&](auto kernel, int threads, long long blocks) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(blocks, (long long)FLOORS * n)), dim3((unsigned)threads), 0, st, q.envs, q.maps, q.luts, q.ls);
    };
    // by six blocks on each of 256 compute units or by sixteen single wavefronts.  Both launches in the form
    // that suits the second: the first one has little to do, and a launch of the other form before the
    // rollout made the one behind it slower (4,096 x 64, Perlin noise: 90 -> 102 us).
    const bool by_blocks = floors_by_blocks(FloorWork::OWED, perlin, worlds_owed(n, steps, p.max_episode_steps) * FLOORS);
    auto drain = [&]() {
        if (by_blocks) { if (perlin) launch_drain(kf_drain<true, GEN_THREADS>, GEN_THREADS, 1536); else launch_drain(kf_drain<false, GEN_THREADS>, GEN_THREADS, 1536); }
        else { if (perlin) launch_drain(kf_drain<true, FLOOR_THREADS>, FLOOR_THREADS, 4096); else launch_drain(kf_drain<false, FLOOR_THREADS>, FLOOR_THREADS, 4096); }
    };
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), 0, st, q.envs, q.maps, q.luts, actions, o, reward, done, q.ls, p, steps); };
    // launches of regeneration blocks only: the worlds still owed by the step kernel, and afterwards
    // those of the episodes that ended in the rollout
    drain();
    if (cfg->obs_mode == CRAFTAX_OBS_SYM_F32) { if (perlin) go(kf_rollout<true, true>); else go(kf_rollout<true, false>); }
    else { if (perlin) go(kf_rollout<false, true>); else go(kf_rollout<false, false>); }
    drain();
    return check_launch("craftax_rollout", err);
}

int observe(void* state, const craftax_config* cfg, int n, void* obs, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    const dim3 grid((n + ENVS_PER_BLOCK - 1) / ENVS_PER_BLOCK);
    uint8_t* o = static_cast<uint8_t*>(obs);
    if (cfg->obs_mode == CRAFTAX_OBS_PIXELS_F32) hipLaunchKernelGGL(kf_pixels, dim3((unsigned)n), dim3(BLOCK), 0, (hipStream_t)stream, q.envs, q.maps, q.luts, o);
    else if (cfg->obs_mode == CRAFTAX_OBS_SYM_F32) {
        auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), 0, (hipStream_t)stream, q.envs, q.maps, q.luts, o, n); };
        switch (floats_kept(n)) {
        case cx::Keep::THROUGH: go(kf_observe<true>); break;
        case cx::Keep::PLAIN: go(kf_observe<true, cx::Keep::PLAIN>); break;
        case cx::Keep::STREAM: go(kf_observe<true, cx::Keep::STREAM>); break;
        }
    }
    else hipLaunchKernelGGL(kf_observe<false>, grid, dim3(BLOCK), 0, (hipStream_t)stream, q.envs, q.maps, q.luts, o, n);
    return check_launch("craftax_observe", err);
}

int export_envs(const void* state, const craftax_config* cfg, int n, int first, int count, void* dumps, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    hipLaunchKernelGGL(kf_export, dim3((unsigned)count * FLOORS), dim3(GEN_THREADS), 0, (hipStream_t)stream, q.envs, q.maps,
                       static_cast<craftax_full_env_dump*>(dumps), first);
    return check_launch("craftax_export_envs", err);
}

int import_envs(void* state, const craftax_config* cfg, int n, int first, int count, const void* dumps, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, floor_grid((unsigned)count), dim3((unsigned)threads), 0, (hipStream_t)stream, q.envs, q.maps, q.ls,
                           static_cast<const craftax_full_env_dump*>(dumps), first, make_params(state, cfg, n), gradients(cfg, q),
                           cfg->reset_mode == CRAFTAX_RESET_POOL ? 1 : 0);
    };
    const bool perlin = cfg->worldgen == CRAFTAX_WORLDGEN_PERLIN, blocks = floors_by_blocks(FloorWork::IMPORT, perlin, (long long)count * FLOORS);
    if (perlin) { if (blocks) go(kf_import<true, GEN_THREADS>, GEN_THREADS); else go(kf_import<true, FLOOR_THREADS>, FLOOR_THREADS); }
    else { if (blocks) go(kf_import<false, GEN_THREADS>, GEN_THREADS); else go(kf_import<false, FLOOR_THREADS>, FLOOR_THREADS); }
    return check_launch("craftax_import_envs", err);
}

int mutate_swap(void* state, const craftax_config* cfg, int n, int first, int count, uint64_t mutation_seed, uint32_t round,
                int restricted, int32_t* tries, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    hipLaunchKernelGGL(kf_mutate_swap, dim3((unsigned)(((long long)count * cx::MUTATE_TRIES + MUTATE_SWAP_THREADS - 1) / MUTATE_SWAP_THREADS)), dim3(MUTATE_SWAP_THREADS), 0, (hipStream_t)stream, q.envs, q.maps, first,
                       count, (uint32_t)mutation_seed, (uint32_t)(mutation_seed >> 32), round, restricted != 0 ? 1 : 0, tries);
    return check_launch("craftax_mutate_swap", err);
}

int mutate_noise(void* state, const craftax_config* cfg, int n, int first, int count, uint16_t* theta, uint64_t mutation_seed, uint32_t round,
                 uint32_t amplitude, void* stream, std::string* err)
{
    const Ptrs q = pointers(state, make_header(cfg, n));
    const uint32_t k0 = (uint32_t)mutation_seed, k1 = (uint32_t)(mutation_seed >> 32);
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, floor_grid((unsigned)count), dim3((unsigned)threads), 0, (hipStream_t)stream, q.envs, q.maps, q.luts, theta, first, k0, k1,
                           round, amplitude);
    };
    if (floors_by_blocks(FloorWork::MUTATE, true, (long long)count * FLOORS)) go(kf_mutate_noise<GEN_THREADS>, GEN_THREADS); else go(kf_mutate_noise<FLOOR_THREADS>, FLOOR_THREADS);
    return check_launch("craftax_mutate_noise", err);
}

}  // namespace host
}  // namespace cf
