// The scheduler and the access records behind simt.h.  Compiled without instrumentation.
#include "simt.h"

#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <map>
#include <set>
#include <vector>

#include "simt_run.h"

simt_dim threadIdx, blockIdx, blockDim;
long simt_word_adds;

namespace {
const int STACK = 128 << 10;
enum State { RUN, LANES, BARRIER, DONE };
struct Fiber {
    ucontext_t at;
    State state;
    int line, phase;
    std::vector<char> stack;
};
std::vector<Fiber> fibers;
ucontext_t scheduler;
uint64_t slots[16][2][64], live_lanes[16];
int current, epoch;
const std::function<void()> *body;

struct Word { int epoch = -1; uint32_t by[3] = {0, 0, 0}; };   // the waves that have read, written, worked atomically since the last barrier
std::map<uintptr_t, Word> words;
std::set<std::string> races;
extern "C" char __data_start, _end;

void enter() {
    (*body)();
    fibers[current].state = DONE;
    swapcontext(&fibers[current].at, &scheduler);
}
void yield(State s) {
    fibers[current].state = s;
    swapcontext(&fibers[current].at, &scheduler);
}
}   // namespace

void simt_barrier(int line) {
    fibers[current].line = line;
    yield(BARRIER);
}
const uint64_t *simt_exchange(uint64_t mine, uint64_t *live) {
    Fiber &f = fibers[current];
    const int wave = current / 64, phase = f.phase++ & 1;
    slots[wave][phase][current % 64] = mine;
    yield(LANES);
    *live = live_lanes[wave];
    return slots[wave][phase];
}
void simt_access(const void *p, int bytes, int kind) {
    if ((const char *)p < &__data_start || (const char *)p >= &_end) return;   // LDS is what the kernels' file has as static data
    const uint32_t me = 1u << (current / 64);
    for (uintptr_t a = (uintptr_t)p / 4; a <= ((uintptr_t)p + bytes - 1) / 4; ++a) {
        Word &w = words[a];
        if (w.epoch != epoch) {
            w = Word();
            w.epoch = epoch;
        }
        w.by[kind] |= me;
        const uint32_t other = ~me;
        if (((w.by[SIMT_WRITE] & me) && ((w.by[0] | w.by[1] | w.by[2]) & other)) || ((w.by[SIMT_WRITE] & other) && ((w.by[0] | w.by[1] | w.by[2]) & me)) ||
            ((w.by[SIMT_READ] & me) && (w.by[SIMT_ATOMIC] & other)) || ((w.by[SIMT_READ] & other) && (w.by[SIMT_ATOMIC] & me))) {
            char what[96];
            snprintf(what, sizeof what, "race behind barrier of line %d, access kind %d", fibers[current].line, kind);
            races.insert(what);
        }
    }
}

int simt_run(int threads, int order, const std::function<void()> &kernel, std::string *report) {
    fibers.clear();
    fibers.resize(threads);
    words.clear();
    races.clear();
    body = &kernel;
    epoch = 0;
    blockDim.x = threads;
    for (Fiber &f : fibers) {
        f.stack.resize(STACK);
        f.state = RUN;
        f.line = f.phase = 0;
        getcontext(&f.at);
        f.at.uc_stack.ss_sp = f.stack.data();
        f.at.uc_stack.ss_size = STACK;
        f.at.uc_link = nullptr;
        makecontext(&f.at, enter, 0);
    }
    const int waves = threads / 64;
    for (;;) {
        std::set<int> lines;
        for (int k = 0; k < waves; ++k) {
            const int w = order == 0 ? k : order == 1 ? waves - 1 - k : (k * 7 + order + epoch) % waves;
            for (;;) {   // this wave up to the next barrier
                int count[4] = {0, 0, 0, 0};
                for (int t = 64 * w; t < 64 * w + 64; ++t) {
                    if (fibers[t].state != RUN) continue;
                    current = threadIdx.x = t;
                    swapcontext(&scheduler, &fibers[t].at);
                }
                live_lanes[w] = 0;
                for (int t = 64 * w; t < 64 * w + 64; ++t) {
                    ++count[fibers[t].state];
                    if (fibers[t].state == LANES) live_lanes[w] |= 1ull << (t % 64);
                }
                if (count[LANES] && count[BARRIER]) {
                    *report = "lanes of a wave part between a lane operation and a barrier";
                    return 1;
                }
                if (!count[LANES]) break;
                for (int t = 64 * w; t < 64 * w + 64; ++t)
                    if (fibers[t].state == LANES) fibers[t].state = RUN;
            }
            for (int t = 64 * w; t < 64 * w + 64; ++t)
                if (fibers[t].state == BARRIER) lines.insert(fibers[t].line);
        }
        if (lines.size() > 1) {
            *report = "waves at different barriers: lines";
            for (int l : lines) *report += " " + std::to_string(l);
            return 1;
        }
        if (lines.empty()) break;
        ++epoch;
        for (Fiber &f : fibers)
            if (f.state == BARRIER) f.state = RUN;
    }
    report->clear();
    for (const std::string &r : races) *report += r + "; ";
    return races.empty() ? 0 : 1;
}

extern "C" {
void __tsan_init() {}
void __tsan_func_entry(void *) {}
void __tsan_func_exit() {}
#define SIMT_HOOK(N)                                                         \
    void __tsan_read##N(void *p) { simt_access(p, N, SIMT_READ); }           \
    void __tsan_write##N(void *p) { simt_access(p, N, SIMT_WRITE); }         \
    void __tsan_unaligned_read##N(void *p) { simt_access(p, N, SIMT_READ); } \
    void __tsan_unaligned_write##N(void *p) { simt_access(p, N, SIMT_WRITE); }
SIMT_HOOK(1) SIMT_HOOK(2) SIMT_HOOK(4) SIMT_HOOK(8) SIMT_HOOK(16)
void __tsan_read_range(void *p, unsigned long n) { simt_access(p, (int)n, SIMT_READ); }
void __tsan_write_range(void *p, unsigned long n) { simt_access(p, (int)n, SIMT_WRITE); }
void __tsan_vptr_update(void **, void *) {}
}
