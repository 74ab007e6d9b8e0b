// hip_runtime.h -- runs the library's device code on the CPU, for tests of what a
// kernel does with its memory.  It takes the place of <hip/hip_runtime.h> when a
// .hip file is compiled as C++.
//
// A workgroup is a host thread, each of its work-items a fiber of that thread.  A
// wave's fibers meet at every cross-lane operation and a workgroup's at every
// barrier; there, after one atomic in eight and at a wave's fences, the scheduler goes
// on with a wave chosen at random, so that a seed is an interleaving.  Cross-lane
// operations and wave barriers have to be reached by all 64 lanes (checked); a fence
// holds those that reach it until the wave's next turn.  Memory is sequentially
// consistent.
#pragma once

#include <setjmp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <atomic>
#include <functional>
#include <random>
#include <thread>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ thread_local
#define __HIP_MEMORY_SCOPE_WORKGROUP 1
#define __HIP_MEMORY_SCOPE_AGENT 2

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace lanes {

constexpr int WAVE_LANES = 64;
constexpr size_t STACK = 128 * 1024;

struct Meet { // where n fibers wait for one another
    int n = 0, here = 0;
    unsigned epoch = 0;
};

struct Wave {
    Meet meet;
    uint64_t val[2][WAVE_LANES]; // the operation's operands, two operations in turn
    int op[2][WAVE_LANES];
};

struct Lane {
    int tid = 0;
    unsigned ops = 0; // cross-lane operations so far
    bool started = false, done = false;
    const Meet *waits = nullptr;
    unsigned epoch = 0;
    ucontext_t ctx;
    jmp_buf at;
};

struct Group {
    dim3 block, grid, index;
    std::vector<Lane> lanes;
    std::vector<Wave> waves;
    Meet barrier;
    std::mt19937 rng;
    jmp_buf scheduler;
    ucontext_t entry;
    Lane *cur = nullptr;
    std::function<void()> kernel;
};

inline unsigned &seed()
{
    static unsigned s = 1;
    return s;
}
inline std::function<long long()> &clock_step()
{
    static std::function<long long()> f = [] { return 1ll; };
    return f;
}
inline thread_local Group *group = nullptr;
inline thread_local dim3 lane_index;

inline void fail(const char *what)
{
    fprintf(stderr, "lanes: %s\n", what);
    abort();
}

__attribute__((noinline)) inline void yield()
{
    Group *g = group;
    Lane *l = g->cur;
    if (_setjmp(l->at) == 0)
        _longjmp(g->scheduler, 1);
}

inline void meet(Meet &m)
{
    Lane *l = group->cur;
    l->waits = &m;
    l->epoch = m.epoch;
    if (++m.here == m.n) {
        m.here = 0;
        ++m.epoch; // the lanes after this one go on in this turn, the others in the next
    }
    yield();
}

// The operands of this operation, of all lanes of the wave.
inline const uint64_t *collect(int op, uint64_t x)
{
    Group *g = group;
    Lane *l = g->cur;
    Wave &w = g->waves[l->tid / WAVE_LANES];
    const unsigned par = l->ops++ & 1u;
    w.val[par][l->tid % WAVE_LANES] = x;
    w.op[par][l->tid % WAVE_LANES] = op;
    meet(w.meet);
    for (int i = 0; i < WAVE_LANES; ++i)
        if (w.op[par][i] != op)
            fail("the lanes of a wave are at different cross-lane operations");
    return w.val[par];
}

inline int lane() { return group->cur->tid % WAVE_LANES; }

template <class T> uint64_t bits(T x)
{
    static_assert(sizeof(T) <= 8, "one register pair");
    uint64_t b = 0;
    memcpy(&b, &x, sizeof x);
    return b;
}

template <class T> T from_bits(uint64_t b)
{
    T x;
    memcpy(&x, &b, sizeof x);
    return x;
}

inline void shuffle_waves()
{
    if (group && (group->rng() & 7u) == 0)
        yield();
}

inline void fiber_main()
{
    group->kernel();
    group->cur->done = true;
    for (;;)
        yield();
}

inline void run_group(Group &g)
{
    group = &g;
    const int n = (int)(g.block.x * g.block.y * g.block.z);
    if (n % WAVE_LANES)
        fail("whole waves only");
    char *stacks = (char *)mmap(nullptr, STACK * n, PROT_READ | PROT_WRITE,
                                MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (stacks == MAP_FAILED)
        fail("no memory for stacks");
    g.lanes = std::vector<Lane>(n);
    g.waves = std::vector<Wave>(n / WAVE_LANES);
    for (auto &w : g.waves)
        w.meet.n = WAVE_LANES;
    g.barrier.n = n;
    int left = n;
    for (int i = 0; i < n; ++i)
        g.lanes[i].tid = i;
    volatile int idle = 0;
    while (left > 0) {
        const int w = (int)(g.rng() % g.waves.size());
        for (volatile int i = w * WAVE_LANES; i < (w + 1) * WAVE_LANES; i = i + 1) {
            Lane &l = g.lanes[i];
            if (l.done || (l.waits && l.waits->epoch == l.epoch))
                continue;
            l.waits = nullptr;
            g.cur = &l;
            lane_index = dim3((unsigned)l.tid, 0, 0);
            idle = 0;
            if (_setjmp(g.scheduler) == 0) {
                if (l.started)
                    _longjmp(l.at, 1);
                l.started = true;
                getcontext(&l.ctx);
                l.ctx.uc_stack.ss_sp = stacks + STACK * i;
                l.ctx.uc_stack.ss_size = STACK;
                l.ctx.uc_link = nullptr;
                makecontext(&l.ctx, fiber_main, 0);
                setcontext(&l.ctx);
            }
            if (g.lanes[i].done)
                --left;
        }
        idle = idle + 1;
        if (idle > (1 << 20))
            fail("no lane can go on (a barrier or cross-lane operation that some never reach)");
    }
    munmap(stacks, STACK * n);
    group = nullptr;
}

// Every workgroup of the grid, up to 64 at a time.
inline void launch(std::function<void()> kernel, dim3 grid, dim3 block)
{
    const unsigned n = grid.x * grid.y * grid.z;
    for (unsigned b0 = 0; b0 < n; b0 += 64) {
        std::vector<std::thread> threads;
        for (unsigned b = b0; b < n && b < b0 + 64; ++b)
            threads.emplace_back([=] {
                Group g;
                g.kernel = kernel;
                g.block = block;
                g.grid = grid;
                g.index = dim3(b % grid.x, b / grid.x % grid.y, b / grid.x / grid.y);
                g.rng.seed(seed() * 7919u + b);
                run_group(g);
            });
        for (auto &t : threads)
            t.join();
    }
}

template <class T, class F> T update(T *p, F f) // atomic; the old value
{
    T was, now;
    __atomic_load(p, &was, __ATOMIC_SEQ_CST);
    do {
        now = f(was);
    } while (!__atomic_compare_exchange(p, &was, &now, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST));
    shuffle_waves();
    return was;
}

template <class T, class V> T add(T *p, V v) { return update(p, [=](T x) { return (T)(x + (T)v); }); }
template <class T, class V> T least(T *p, V v)
{
    return update(p, [=](T x) { return x < (T)v ? x : (T)v; });
}
template <class T, class V> T most(T *p, V v)
{
    return update(p, [=](T x) { return x > (T)v ? x : (T)v; });
}
template <class T, class V> T bit_or(T *p, V v) { return update(p, [=](T x) { return (T)(x | (T)v); }); }
template <class T, class V> T bit_and(T *p, V v) { return update(p, [=](T x) { return (T)(x & (T)v); }); }
template <class T, class V> T exchange(T *p, V v) { return update(p, [=](T) { return (T)v; }); }
template <class T> T load(const T *p)
{
    T x;
    __atomic_load(const_cast<T *>(p), &x, __ATOMIC_SEQ_CST);
    return x;
}
template <class T, class V> void store(T *p, V v)
{
    T x = (T)v;
    __atomic_store(p, &x, __ATOMIC_SEQ_CST);
}

inline int dpp(int old, int src, int ctrl, int rows)
{
    const uint64_t *v = collect(100 + ctrl, bits(src));
    const int l = lane(), row = l / 16;
    if (!((rows >> row) & 1))
        return old;
    int from = -1;
    if (ctrl >= 0x111 && ctrl <= 0x11f) // row_shr
        from = l % 16 >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    else if (ctrl == 0x142) // row_bcast:15
        from = row > 0 ? row * 16 - 1 : -1;
    else if (ctrl == 0x143) // row_bcast:31
        from = row > 1 ? 31 : -1;
    else
        fail("dpp control");
    return from < 0 ? old : from_bits<int>(v[from]);
}

inline int permute(int addr, int src)
{
    const uint64_t *v = collect(2, (uint64_t)(uint32_t)addr << 32 | (uint32_t)src);
    int r = 0;
    for (int i = 0; i < WAVE_LANES; ++i)
        if ((int)(v[i] >> 34) % WAVE_LANES == lane())
            r = (int)(uint32_t)v[i];
    return r;
}

} // namespace lanes

#define threadIdx lanes::lane_index
#define blockIdx lanes::group->index
#define blockDim lanes::group->block
#define gridDim lanes::group->grid

inline void __syncthreads() { lanes::meet(lanes::group->barrier); }
inline void __threadfence() { std::atomic_thread_fence(std::memory_order_seq_cst); }
inline unsigned __lane_id() { return (unsigned)lanes::lane(); }
inline uint64_t __ballot(int p)
{
    const uint64_t *v = lanes::collect(1, p != 0);
    uint64_t m = 0;
    for (int i = 0; i < lanes::WAVE_LANES; ++i)
        m |= v[i] << i;
    return m;
}
template <class T> T __shfl(T x, int from)
{
    return lanes::from_bits<T>(lanes::collect(3, lanes::bits(x))[from & 63]);
}
template <class T> T __shfl_xor(T x, int mask)
{
    return lanes::from_bits<T>(lanes::collect(4, lanes::bits(x))[lanes::lane() ^ mask]);
}
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __ffsll(unsigned long long x) { return __builtin_ffsll((long long)x); }
// ticks of a clock that only goes on when it is read, in steps of lanes::clock_step()
inline long long wall_clock64()
{
    static std::atomic<long long> t{0};
    return t += lanes::clock_step()();
}

inline int __builtin_amdgcn_readlane(int x, int from)
{
    return lanes::from_bits<int>(lanes::collect(5, lanes::bits(x))[from & 63]);
}
inline int __builtin_amdgcn_readfirstlane(int x) { return __builtin_amdgcn_readlane(x, 0); }
inline int __builtin_amdgcn_ds_permute(int addr, int src) { return lanes::permute(addr, src); }
#define __builtin_amdgcn_update_dpp(old, src, ctrl, rows, banks, bound) \
    lanes::dpp(old, src, ctrl, rows)
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t add)
{
    const int l = lanes::lane();
    return add + (uint32_t)__builtin_popcount(l >= 32 ? m : m & ((1u << l) - 1u));
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t add)
{
    const int l = lanes::lane();
    return add + (l <= 32 ? 0u : (uint32_t)__builtin_popcount(m & ((1u << (l - 32)) - 1u)));
}
inline void __builtin_amdgcn_wave_barrier() { lanes::collect(6, 0); }
inline void __builtin_amdgcn_fence(int, const char *) { lanes::yield(); }
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline void __builtin_amdgcn_s_sleep(int)
{
    std::this_thread::yield();
    lanes::yield();
}

#define __hip_atomic_load(p, o, s) lanes::load(p)
#define __hip_atomic_store(p, v, o, s) lanes::store(p, v)
#define __hip_atomic_fetch_add(p, v, o, s) lanes::add(p, v)
#define __hip_atomic_fetch_min(p, v, o, s) lanes::least(p, v)
#define __hip_atomic_fetch_or(p, v, o, s) lanes::bit_or(p, v)
#define __hip_atomic_fetch_and(p, v, o, s) lanes::bit_and(p, v)
#define __hip_atomic_exchange(p, v, o, s) lanes::exchange(p, v)
#define __hip_atomic_compare_exchange_strong(p, e, v, o1, o2, s) \
    __atomic_compare_exchange_n(p, e, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)
template <class T, class V> T atomicAdd(T *p, V v) { return lanes::add(p, v); }
template <class T, class V> T atomicMin(T *p, V v) { return lanes::least(p, v); }
template <class T, class V> T atomicMax(T *p, V v) { return lanes::most(p, v); }
template <class T, class V> T atomicOr(T *p, V v) { return lanes::bit_or(p, v); }
template <class T, class V> T unsafeAtomicAdd(T *p, V v) { return lanes::add(p, v); }

typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum { hipFuncAttributeMaxDynamicSharedMemorySize };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void *, int, int) { return hipSuccess; }
template <class F>
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, F, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, st, ...) \
    lanes::launch([=] { kernel(__VA_ARGS__); }, grid, block)
