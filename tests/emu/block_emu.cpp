// Runs one block of device code on the CPU: a context per work-item, block
// barriers and wavefront operations as points where it waits for the others.
// The compiler's thread-sanitizer calls record every access, and two
// wavefronts that touch a word between the same two barriers, one of them
// writing, are reported.  (Built without the sanitizer itself.)
#include "block_emu.h"

#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <unordered_map>
#include <vector>

#include "hip/hip_runtime.h"

namespace emu {
dim3 thread_idx, block_idx, block_dim, grid_dim;

namespace {
enum State { READY, AT_BARRIER, AT_WAVE, DONE };
constexpr size_t STACK = 128 << 10;
struct Item {
    ucontext_t ctx;
    State state = READY;
    const char *file = "";
    int line = 0;
    unsigned long long word = 0;
};
struct Word {
    unsigned long long interval = ~0ull, readers = 0, writers = 0;   // wavefronts, a bit each
};
std::vector<Item> items;
std::vector<char> stacks;
ucontext_t scheduler;
int current = -1;              // the running work-item, -1 outside the block
const std::function<void()> *body;
unsigned long long snap[64][64];   // per wavefront: the words of its last exchange
unsigned long long interval = 0;
std::unordered_map<uintptr_t, Word> shadow;
std::set<std::string> found;

void pause(State s) {
    Item &it = items[current];
    it.state = s;
    swapcontext(&it.ctx, &scheduler);
}
void entry() {
    (*body)();
    items[current].state = DONE;
    swapcontext(&items[current].ctx, &scheduler);
}
}  // namespace

void barrier(const char *file, int line) {
    items[current].file = file;
    items[current].line = line;
    pause(AT_BARRIER);
}
const unsigned long long *exchange(unsigned long long word) {
    items[current].word = word;
    const int w = current >> 6;
    pause(AT_WAVE);
    return snap[w];
}

// one access of the running work-item (its calls into the standard library may
// be the instrumented copies: not recorded)
void access(const void *p, size_t n, bool write) {
    if (current < 0) return;
    const int item = current;
    current = -1;
    const uintptr_t a = (uintptr_t)p, s0 = (uintptr_t)stacks.data();
    const bool own = a >= s0 && a < s0 + stacks.size();   // a work-item's own variables
    if (!own && p != &thread_idx) {
        const unsigned long long bit = 1ull << (item >> 6);
        for (uintptr_t w = a & ~(uintptr_t)3; w < a + n; w += 4) {
            Word &x = shadow[w];
            if (x.interval != interval) x = Word{interval, 0, 0};
            (write ? x.writers : x.readers) |= bit;
            if (write ? ((x.readers | x.writers) & ~bit) : (x.writers & ~bit))
                found.insert("a word two wavefronts touch without a barrier between");
        }
    }
    current = item;
}

std::string run_block(int nt, const int *waves, const std::function<void()> &kernel) {
    items.assign(nt, Item{});
    stacks.assign((size_t)nt * STACK, 0);
    shadow.clear();
    found.clear();
    body = &kernel;
    block_dim = dim3(nt);
    block_idx = dim3(0, 0, 0);
    for (int t = 0; t < nt; ++t) {
        getcontext(&items[t].ctx);
        items[t].ctx.uc_stack.ss_sp = stacks.data() + (size_t)t * STACK;
        items[t].ctx.uc_stack.ss_size = STACK;
        items[t].ctx.uc_link = &scheduler;
        makecontext(&items[t].ctx, entry, 0);
    }
    const int nw = nt / 64;
    for (;;) {
        bool ran = false;
        for (int k = 0; k < nw && !ran; ++k) {
            const int w = waves[k];
            int ready = 0, wait = 0, bar = 0;
            for (int t = 64 * w; t < 64 * w + 64; ++t) {
                ready += items[t].state == READY;
                wait += items[t].state == AT_WAVE;
                bar += items[t].state == AT_BARRIER;
            }
            if (!ready && wait) {   // every live lane has handed in its word
                if (bar) found.insert("lanes of a wavefront at a barrier and at an exchange");
                for (int i = 0; i < 64; ++i) {
                    Item &it = items[64 * w + i];
                    snap[w][i] = it.state == AT_WAVE ? it.word : 0;
                    if (it.state == AT_WAVE) it.state = READY;
                }
                ready = wait;
            }
            if (!ready) continue;
            ran = true;
            for (int t = 64 * w + 63; t >= 64 * w; --t)   // lane 0 last: what it alone writes comes after the others' reads
                if (items[t].state == READY) {
                    current = t;
                    thread_idx = dim3(t, 0, 0);
                    swapcontext(&scheduler, &items[t].ctx);
                    current = -1;
                }
        }
        if (ran) continue;
        std::set<std::pair<std::string, int>> at;
        for (Item &it : items)
            if (it.state == AT_BARRIER) {
                at.insert({it.file, it.line});
                it.state = READY;
            }
        if (at.empty()) break;
        if (at.size() > 1) found.insert("wavefronts at different barriers");
        ++interval;
    }
    std::string r;
    for (const std::string &f : found) r += f + "\n";
    return r;
}
}  // namespace emu

extern "C" {
void __tsan_init() {}
void __tsan_func_entry(void *) {}
void __tsan_func_exit() {}
#define ACCESS(n)                                                                        \
    void __tsan_read##n(void *p) { emu::access(p, n, false); }                           \
    void __tsan_write##n(void *p) { emu::access(p, n, true); }                           \
    void __tsan_unaligned_read##n(void *p) { emu::access(p, n, false); }                 \
    void __tsan_unaligned_write##n(void *p) { emu::access(p, n, true); }
ACCESS(1) ACCESS(2) ACCESS(4) ACCESS(8) ACCESS(16)
void __tsan_read_range(void *p, unsigned long n) { emu::access(p, n, false); }
void __tsan_write_range(void *p, unsigned long n) { emu::access(p, n, true); }
void __tsan_vptr_update(void **, void *) {}
void __tsan_vptr_read(void **) {}
}
