// Fibers, rendezvous, barriers and LDS copies of the CPU stand-in for the
// device (hip/hip_runtime.h).  One thread; wavefronts run to their next barrier
// in ascending or descending order.
#include "hip/hip_runtime.h"

#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <deque>
#include <random>
#include <set>
#include <vector>

extern "C" void sim_switch(void **save, void *to);
asm(R"(
.text
.globl sim_switch
sim_switch:
    push %rbp; push %rbx; push %r12; push %r13; push %r14; push %r15
    mov %rsp, (%rdi)
    mov %rsi, %rsp
    pop %r15; pop %r14; pop %r13; pop %r12; pop %rbx; pop %rbp
    ret
)");
// float -> bf16, round to nearest even (no library call for it on this host)
extern "C" __bf16 __truncsfbf2(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7fffffffu) > 0x7f800000u)
        u = (u >> 16) | 0x40u;
    else
        u = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    return __builtin_bit_cast(__bf16, (uint16_t)u);
}

namespace sim {

Lane *cur;
dim3 block, blocks, threads;
bool compute = true;

namespace {

constexpr size_t STACK = 512 * 1024, VALUE = 64;
constexpr int MAXT = 1024;
bool early = false, reversed = false;  // copies land at once; order of the wavefronts
long sample = 0;                       // > 0: about so many work-groups of a launch
struct Copy {
    char *dst;
    std::vector<char> bytes;
};
struct Wave {
    long gen;
    int arrived, alive;
    alignas(64) char in[2][64][VALUE];
    std::deque<Copy> copies;
};
char *stacks;
Lane lanes[MAXT];
Wave waves[MAXT / 64];
int nthreads, at_barrier, alive;
void *sched_sp;
const std::function<void()> *body;
std::set<void *> lds_seen;
size_t lds_bytes, dyn_bytes;
std::vector<unsigned char> dyn;
std::mt19937 rng(1);
const char *kernel = "";

void die(const char *what) {
    fprintf(stderr, "devsim: %s in %.120s, block (%u, %u, %u) of (%u, %u, %u), wave %d lane %d\n", what,
            kernel, block.x, block.y, block.z, blocks.x, blocks.y, blocks.z, cur ? cur->wave : -1,
            cur ? cur->lane : -1);
    abort();
}

void retire(Wave &w, size_t left) {
    while (w.copies.size() > left) {
        Copy &c = w.copies.front();
        memcpy(c.dst, c.bytes.data(), c.bytes.size());
        w.copies.pop_front();
    }
}

void yield() { sim_switch(&cur->sp, sched_sp); }

void entry() {
    (*body)();
    Wave &w = waves[cur->wave];
    cur->state = 3;
    --alive;
    if (--w.alive == 0 && !w.copies.empty())
        die("wavefront ends with LDS copies outstanding");
    yield();
    abort();
}

void start(int i) {
    Lane &l = lanes[i];
    char *top = stacks + (size_t)(i + 1) * STACK;
    void **sp = (void **)((uintptr_t)top & ~(uintptr_t)63);
    *--sp = nullptr;         // alignment: entry() sees rsp = 16 n + 8
    *--sp = (void *)entry;
    sp -= 6;
    memset(sp, 0, 6 * sizeof(void *));
    l.sp = sp;
    l.wave = i / 64;
    l.lane = i & 63;
    l.gen = 0;
    l.state = 0;
    l.tid = dim3(i % threads.x, i / threads.x, 0);
}

bool runnable(const Lane &l) {
    return l.state == 0 || (l.state == 1 && waves[l.wave].gen > l.gen);
}

void run_block() {
    lds_seen.clear();
    lds_bytes = dyn_bytes;
    if (dyn_bytes)
        dyn.assign(dyn_bytes, 0xc5);
    const int nw = nthreads / 64;
    for (int i = 0; i < nthreads; ++i)
        start(i);
    for (int w = 0; w < nw; ++w) {
        waves[w].gen = 0;
        waves[w].arrived = 0;
        waves[w].alive = 64;
        waves[w].copies.clear();
    }
    alive = nthreads;
    at_barrier = 0;
    while (alive > 0) {
        bool progress = false;
        for (int q = 0; q < nw; ++q) {
            const int w = reversed ? nw - 1 - q : q;
            for (bool again = true; again;) {
                again = false;
                for (int i = w * 64; i < w * 64 + 64; ++i)
                    if (runnable(lanes[i])) {
                        cur = &lanes[i];
                        cur->state = 0;
                        sim_switch(&sched_sp, cur->sp);
                        again = progress = true;
                    }
            }
        }
        if (alive > 0 && at_barrier == alive) {
            at_barrier = 0;
            for (int i = 0; i < nthreads; ++i)
                if (lanes[i].state == 2)
                    lanes[i].state = 0;
            progress = true;
        }
        if (!progress)
            die("deadlock (a rendezvous or barrier that not every lane reaches)");
    }
    cur = nullptr;
}

} // namespace

void lds(void *p, size_t bytes) {
    if (!lds_seen.insert(p).second)
        return;
    lds_bytes += bytes;
    if (lds_bytes > 160 * 1024)
        die("more than 160 KB of LDS");
    memset(p, 0xc5, bytes);
}

unsigned char *dynamic_lds() { return dyn.data(); }

char *meet(const void *v, size_t bytes) {
    Wave &w = waves[cur->wave];
    if (bytes > VALUE)
        die("rendezvous value too large");
    const int b = w.gen & 1;
    // values side by side, as the reader indexes them
    memcpy(&w.in[b][0][0] + cur->lane * bytes, v, bytes);
    cur->gen = w.gen;
    if (++w.arrived == w.alive) {
        if (w.alive != 64)
            die("rendezvous of a wavefront with finished lanes");
        w.arrived = 0;
        ++w.gen;
    } else {
        cur->state = 1;
        yield();
    }
    return &w.in[b][0][0];
}

void barrier() {
    cur->state = 2;
    ++at_barrier;
    yield();
}

void wait(int vm) {
    wave_sync();
    if (cur->lane == 0)
        retire(waves[cur->wave], vm);
    wave_sync();
}

void copy(const void *src, void *dst, int bytes) {
    struct Req { const void *s; void *d; };
    const auto r = all(Req{src, dst});
    if (cur->lane == 0) {
        Copy c;
        c.dst = (char *)r[0].d;
        c.bytes.resize(64 * bytes);
        for (int i = 0; i < 64; ++i) {
            if ((uintptr_t)r[i].s % (bytes == 16 ? 16 : 4))
                die("misaligned LDS copy");
            for (int e = 0; e < bytes; ++e)  // (checked loads)
                c.bytes[i * bytes + e] = ((const volatile char *)r[i].s)[e];
        }
        volatile char first = c.dst[0], last = c.dst[64 * bytes - 1];  // (checked)
        (void)first;
        (void)last;
        Wave &w = waves[cur->wave];
        w.copies.push_back(std::move(c));
        if (early)
            retire(w, 0);
    }
    wave_sync();
}

void launch(dim3 grid, dim3 blk, size_t lds, const std::function<void()> &f, const char *name) {
    if (!stacks)
        stacks = (char *)mmap(nullptr, STACK * MAXT, PROT_READ | PROT_WRITE,
                              MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    blocks = grid;
    threads = blk;
    kernel = name;
    nthreads = blk.x * blk.y * blk.z;
    dyn_bytes = lds;
    body = &f;
    if (nthreads % 64 || nthreads > MAXT || !nthreads || grid.x == 0 || grid.y == 0 || grid.z == 0 ||
        grid.y > 65535 || grid.z > 65535)
        die("launch configuration");
    const bool product = strstr(name, "gemm1") || strstr(name, "wgrad");
    const double n = (double)grid.x * grid.y * grid.z;
    const double p = sample > 0 && product ? sample / n : 1.0;
    std::uniform_real_distribution<double> u(0, 1);
    for (unsigned z = 0; z < grid.z; ++z)
        for (unsigned y = 0; y < grid.y; ++y)
            for (unsigned x = 0; x < grid.x; ++x) {
                // the work-groups that write the index, the last ones and some others
                const bool corner = strstr(name, "gemm1") && x == 0 && y == 0 && grid.z <= 64;
                const bool last = x == grid.x - 1 && y == grid.y - 1 && (z == grid.z - 1 || grid.z <= 4);
                if (p >= 1 || corner || last || u(rng) < p) {
                    block = dim3(x, y, z);
                    run_block();
                }
            }
}

} // namespace sim

extern "C" void devsim_config(int compute, int early, int reversed, long sample, unsigned seed) {
    sim::compute = compute;
    sim::early = early;
    sim::reversed = reversed;
    sim::sample = sample;
    sim::rng.seed(seed);
}
