// The label-tree kernel's own source (csrc/routing.hpp, given as KERNELS with its LDS arrays made statics) on the
// CPU: every thread of the workgroup is a coroutine that runs until a barrier, in the order asked for, so that one
// thread is as far ahead of the next as the barriers allow.  Threads that wait at different barriers, or at one while
// others have ended, end the run with their source lines.
#include <ucontext.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

namespace emu {
struct Dim { unsigned x, y, z; };
struct Thread {
    ucontext_t ctx;
    std::vector<char> stack;
    int line;        // barrier it waits at; quads wait at -line; 0: ended
    int value;       // what it gives its quad
};
Dim threadIdx, blockIdx, blockDim, gridDim;
std::vector<Thread> threads;
ucontext_t scheduler;
int jumps;           // times the threshold started again from the smallest waiting label

void wait(int line) {
    Thread& t = threads[threadIdx.x];
    t.line = line;
    const unsigned me = threadIdx.x;
    swapcontext(&t.ctx, &scheduler);
    threadIdx.x = me;
}
int quad(int x, int lane, int line) {
    const unsigned me = threadIdx.x;
    threads[me].value = x;
    wait(-line);
    const int r = threads[(me & ~3u) + lane].value;
    wait(-line);                    // every lane has read before one gives again
    return r;
}
}  // namespace emu

using emu::blockDim;
using emu::blockIdx;
using emu::gridDim;
using emu::threadIdx;
struct uint4 { unsigned x, y, z, w; };
#define __global__
#define __device__
#define __launch_bounds__(x)
#define __align__(x) alignas(x)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
#define __builtin_amdgcn_s_waitcnt(x) (void)0
#define __builtin_amdgcn_mov_dpp(x, ctl, row, bank, bound) emu::quad(x, (ctl) / 0x55, __LINE__)
#define __syncthreads() emu::wait(__LINE__)
template <class T, class O> T change(T* p, O&& f) { const T old = *p; *p = f(old); return old; }
template <class T> T atomicAdd(T* p, T v) { return change(p, [&](T o) { return o + v; }); }
template <class T> T atomicOr(T* p, T v) { return change(p, [&](T o) { return o | v; }); }
template <class T> T atomicExch(T* p, T v) { return change(p, [&](T) { return v; }); }
template <class T> T atomicMin(T* p, T v) { return change(p, [&](T o) { return o < v ? o : v; }); }
template <class D, class S> D bits(S s) { D d; memcpy(&d, &s, 4); return d; }
inline float __uint_as_float(unsigned x) { return bits<float>(x); }
inline float __int_as_float(int x) { return bits<float>(x); }
inline unsigned __float_as_uint(float x) { return bits<unsigned>(x); }
inline int __float_as_int(float x) { return bits<int>(x); }
inline int min(int a, int b) { return a < b ? a : b; }
inline unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }
// (the kernel takes a maximum in one place: where the threshold starts again from the smallest waiting label)
inline unsigned max(unsigned a, unsigned b) {
    emu::jumps += threadIdx.x == 0;
    return a < b ? b : a;
}
namespace manta { alignas(16) unsigned lab[1 << 16]; }

#include KERNELS

namespace {
struct Args {
    int V, list, *tab, *len;
    const manta::RouteIn* in;
    const manta::RouteOut* out;
    const int *out_off, *dests, *qoff, *qord, *origin;
    float step;
} g;

void entry() {
    manta::k_route_tree(g.V, g.in, g.out_off, g.out, g.dests, g.list, g.step, g.tab, g.qoff, g.qord, g.origin, g.len);
    emu::threads[threadIdx.x].line = 0;
    swapcontext(&emu::threads[threadIdx.x].ctx, &emu::scheduler);
}
}  // namespace

extern "C" float route_tree_step(const float* cost, int n) { return manta::route_tree_step(cost, n); }

// order: 1 the lowest thread first, -1 the highest.  0, or -1 with the two source lines that threads wait at.
extern "C" int route_tree(int nt, int order, int nd, int V, const void* in, const int* out_off, const void* out,
                          const int* dests, int list, float step, int* tab, const int* qoff, const int* qord,
                          const int* origin, int* len, int* jumps, int* lines) {
    g = Args{V, list, tab, len, (const manta::RouteIn*)in, (const manta::RouteOut*)out, out_off, dests, qoff, qord,
             origin, step};
    blockDim.x = (unsigned)nt;
    emu::threads.assign(nt, emu::Thread{});
    emu::jumps = 0;
    for (int q = 0; q < nd; ++q) {
        blockIdx.x = (unsigned)q;
        memset(manta::lab, 0xA5, sizeof manta::lab);   // LDS is not cleared
        for (int i = 0; i < nt; ++i) {
            emu::Thread& t = emu::threads[i];
            t.stack.resize(64 << 10);
            t.line = INT_MAX;
            getcontext(&t.ctx);
            t.ctx.uc_stack.ss_sp = t.stack.data();
            t.ctx.uc_stack.ss_size = t.stack.size();
            t.ctx.uc_link = nullptr;
            makecontext(&t.ctx, entry, 0);
        }
        auto run = [&](int i) {
            threadIdx.x = (unsigned)i;
            swapcontext(&emu::scheduler, &emu::threads[i].ctx);
        };
        for (bool live = true; live;) {
            for (int k = 0; k < nt; ++k) run(order > 0 ? k : nt - 1 - k);
            for (bool quads = true; quads;) {          // quads meet until every thread is at a barrier
                quads = false;
                for (int k = 0; k < nt; k += 4) {
                    const int a = emu::threads[k].line;
                    for (int j = 1; j < 4; ++j)
                        if ((a < 0 || emu::threads[k + j].line < 0) && emu::threads[k + j].line != a) {
                            lines[0] = std::abs(a);
                            lines[1] = std::abs(emu::threads[k + j].line);
                            return -1;
                        }
                    if (a >= 0) continue;
                    quads = true;
                    for (int j = 0; j < 4; ++j) run(order > 0 ? k + j : k + 3 - j);
                }
            }
            live = emu::threads[0].line != 0;
            for (int k = 1; k < nt; ++k)
                if (emu::threads[k].line != emu::threads[0].line) {
                    lines[0] = emu::threads[0].line;
                    lines[1] = emu::threads[k].line;
                    return -1;
                }
        }
    }
    *jumps = emu::jumps;
    return 0;
}
