// The launch bookkeeping of csrc/lookahead.hpp under hostile orders: whatever wavefront of whatever
// block is served last, every wavefront of a launch sees the same launch number and list lengths, and
// every entry lands on the list that the next launch consumes.  Wavefronts are fibers (a lane each where
// one is enough); a block's barrier is the only thing that makes one wait for another, as on the GPU.
#include <ucontext.h>

#include <cstdio>
#include <functional>
#include <memory>
#include <vector>

#include "../../paper_2402_16801_amd/csrc/lookahead.hpp"

dim threadIdx, blockIdx, blockDim, gridDim;

struct Fiber {
    uint32_t block, thread;
    int barriers = 0, exchanges = 0;             // how many it has arrived at
    int exchanged = 0;
    bool done = false;
    std::function<void()> body;
    ucontext_t context;
    std::vector<char> stack;
};
static std::vector<std::unique_ptr<Fiber>> fibers;
static Fiber* current;
static ucontext_t scheduler;

static void wait_turn() { swapcontext(&current->context, &scheduler); }
void __syncthreads() { ++current->barriers; wait_turn(); }
uint32_t atomicAdd(uint32_t* at, uint32_t value) { const uint32_t old = *at; *at += value; return old; }
int __shfl_up(int value, int delta, int)
{
    Fiber* me = current;
    me->exchanged = value;
    ++me->exchanges;
    wait_turn();
    int got = value;
    for (auto& f : fibers) if (f->block == me->block && (int)f->thread == (int)me->thread - delta) got = f->exchanged;
    ++me->exchanges;
    wait_turn();
    return got;
}
// A fiber may go on once all fibers of its block have arrived where it waits (finished ones never wait again).
static bool may_run(const Fiber& f)
{
    if (f.done) return false;
    for (auto& o : fibers) {
        if (o->block != f.block || o->done) continue;
        if (o->barriers < f.barriers) return false;
        if (f.thread < 16u && o->thread < 16u && o->barriers == f.barriers && o->exchanges < f.exchanges) return false;
    }
    return true;
}
static void entry() { current->body(); current->done = true; swapcontext(&current->context, &scheduler); }

static int failures = 0;
static void expect(bool cond, const char* what, int kernel, int late_block, int late_wave)
{
    if (!cond && failures < 10) std::printf("FAILED: %s (kernel %d, served last: wavefront %d of block %d)\n", what, kernel, late_wave, late_block);
    if (!cond) ++failures;
}

static void start(uint32_t block, uint32_t thread, const std::function<void()>& kernel)
{
    auto f = std::make_unique<Fiber>();
    f->block = block;
    f->thread = thread;
    f->body = kernel;
    f->stack.resize(1 << 16);
    getcontext(&f->context);
    f->context.uc_stack.ss_sp = f->stack.data();
    f->context.uc_stack.ss_size = f->stack.size();
    f->context.uc_link = nullptr;
    makecontext(&f->context, entry, 0);
    fibers.push_back(std::move(f));
}
// One launch of `blocks` blocks of four wavefronts; the wavefront (late_block, late_wave) runs only when nothing else can.
static void launch(int blocks, int late_block, int late_wave, const std::function<void()>& kernel)
{
    fibers.clear();
    gridDim.x = (uint32_t)blocks;
    blockDim.x = 256;
    for (uint32_t b = 0; b < gridDim.x; ++b) {
        for (uint32_t t = 0; t < 16; ++t) start(b, t, kernel);       // the lanes that exchange list lengths
        for (uint32_t t = 64; t < 256; t += 64) start(b, t, kernel);
    }
    auto late = [&](const Fiber& f) { return (int)f.block == late_block && (int)(f.thread / 64) == late_wave; };
    for (bool ran = true; ran;) {
        ran = false;
        for (int pass = 0; pass < 2 && !ran; ++pass)
            for (auto& f : fibers) {
                if (late(*f) != (pass == 1) || !may_run(*f)) continue;
                current = f.get();
                threadIdx.x = f->thread;
                blockIdx.x = f->block;
                swapcontext(&scheduler, &f->context);
                ran = true;
            }
    }
}

int main()
{
    using namespace la;
    constexpr int BLOCKS = 70;                               // more blocks than groups: some groups have two members
    constexpr uint32_t CAP = 64, COUNT = 5;
    long orders = 0;
    for (int kernel = 0; kernel < 2; ++kernel)               // 0: enter_launch, 1: enter_launch_queue
        for (int late_block = 0; late_block < BLOCKS; late_block += 23)
            for (int late_wave = 0; late_wave < 4; ++late_wave)
                for (uint32_t seq = 6; seq < 8; ++seq) {
                    std::vector<uint32_t> ctr((size_t)CT_COUNT * CTR_STRIDE, 0u);
                    std::vector<uint4> lists[2];
                    for (auto& l : lists) l.assign((size_t)NSUB * CAP, uint4{ENTRY_VOID, 0u, 0u, 0u});
                    Lists ls{ctr.data(), {lists[0].data(), lists[1].data()}, nullptr, nullptr, CAP, 0u};
                    *counter(ls, CT_SEQ) = seq;
                    for (int s = 0; s < NSUB; ++s) *counter(ls, CT_REGEN + (int)((seq & 1u) ^ 1u) * NSUB + s) = COUNT;
                    std::vector<uint32_t> prefix((size_t)BLOCKS * NSUB, 0u);
                    bool same = true;
                    uint32_t ended = 0;
                    launch(BLOCKS, late_block, late_wave, [&]() {
                        uint32_t* s_prefix = prefix.data() + (size_t)blockIdx.x * NSUB;
                        const Ticket t = kernel == 0 ? enter_launch(ls, true, blockIdx.x) : enter_launch_queue(ls, s_prefix);
                        same = same && t.seq == seq && (kernel == 0 ? t.regen_count == COUNT : s_prefix[NSUB - 1] == NSUB * COUNT);
                        if (threadIdx.x % 64u == 0u) {           // an episode ends in every wavefront
                            ++ended;
                            commit_entry(ls, t.seq, blockIdx.x, claim_entry(ls, t.seq, blockIdx.x), uint4{blockIdx.x * 4u + threadIdx.x / 64u, 0u, 0u, 0u});
                        }
                        leave_launch(ls, t);
                    });
                    for (auto& f : fibers) same = same && f->done;
                    uint32_t listed = 0, left = 0;
                    for (int s = 0; s < NSUB; ++s) {
                        listed += *counter(ls, CT_REGEN + (int)(seq & 1u) * NSUB + s);
                        left += *counter(ls, CT_REGEN + (int)((seq & 1u) ^ 1u) * NSUB + s);
                    }
                    expect(same, "every wavefront sees this launch's number and list lengths", kernel, late_block, late_wave);
                    expect(ended == 4u * BLOCKS && listed == ended, "every entry is on the list that the next launch consumes", kernel, late_block, late_wave);
                    expect(left == 0u && *counter(ls, CT_SEQ) == seq + 1u, "the launch ends with its list empty and the number advanced once", kernel, late_block, late_wave);
                    ++orders;
                }
    for (uint64_t n = 1; n < 300000; n += n < 5000 ? 1 : 977)
        for (uint64_t most : { 16, 64 })
            if (sub_list_capacity(n, most) < (n + NSUB - 1) / NSUB) expect(false, "a sub-list holds every NSUB-th environment", (int)n, (int)most, 0);
    if (failures) std::printf("launch_order_test: %d failures\n", failures);
    else std::printf("launch_order_test: ok (%ld orders)\n", orders);
    return failures ? 1 : 0;
}
