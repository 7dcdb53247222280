// Kernels of the library as host code, for tests of the order in which the waves of a workgroup may run.
//
// Every workgroup is a thread of the operating system, every lane a fiber of it.  Lanes run one at a time up to their next
// operation of the whole wave (matrix product, vote, lane exchange) or barrier, and of the lanes that could go on, one of the wave
// that comes first in `host::order` does: {2, 3, 0, 1} lets waves 2 and 3 be as far ahead of waves 0 and 1 as barriers allow.
// Memory answers at once.  Only what lstm.hip uses is here.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <type_traits>
#include <vector>
#include <stdarg.h>

typedef int   hipError_t;
typedef void* hipStream_t;
constexpr int hipSuccess = 0, hipDeviceAttributeMultiprocessorCount = 0;
inline int hipGetLastError() { return 0; }
inline int hipGetDevice(int* d) { return *d = 0; }
inline int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, 0; }
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace host {
extern int              order[4];    // waves by precedence
extern std::atomic<int> worked[8];   // workgroups by XCD (ids go round them) that did not return at once
constexpr int LANES = 64, THREADS = 256, STACK = 256 << 10;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float    f4 __attribute__((ext_vector_type(4)));
typedef short    s4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

enum State { READY, WAVE, BARRIER, DONE };
struct Lane {
    ucontext_t        ctx;
    State             state = READY;
    const void*       give;   // operand of a wave's operation ...
    void*             take;   // ... and where its result goes
    dim3              thread;
    std::unique_ptr<char[]> stack;
};
struct Group {
    dim3                  block, grid;
    std::vector<Lane>     lanes{THREADS};
    ucontext_t            scheduler;
    std::function<void()> body;
    int                   now = 0, waiting = 0, in_wave[4] = {0, 0, 0, 0};
    bool                  barriers = false;

    void yield() { swapcontext(&lanes[now].ctx, &scheduler); }
    static void enter();
    void run() {
        for (int i = 0; i < THREADS; ++i) {
            lanes[i].stack.reset(new char[STACK]);   // (not cleared: most of it is never touched)
            lanes[i].thread = dim3(i, 0, 0);
            getcontext(&lanes[i].ctx);
            lanes[i].ctx.uc_stack.ss_sp   = lanes[i].stack.get();
            lanes[i].ctx.uc_stack.ss_size = STACK;
            lanes[i].ctx.uc_link          = &scheduler;
            makecontext(&lanes[i].ctx, &Group::enter, 0);
        }
        for (;;) {
            int next = -1, left = 0;
            for (int w = 0; w < 4 && next < 0; ++w)
                for (int l = 0; l < LANES && next < 0; ++l)
                    if (lanes[order[w] * LANES + l].state == READY) next = order[w] * LANES + l;
            for (const Lane& l : lanes) left += l.state != DONE;
            if (left == 0) return;
            if (next < 0) {
                fprintf(stderr, "workgroup %u: %d lanes wait for each other\n", block.x, left);
                abort();
            }
            now = next;
            swapcontext(&scheduler, &lanes[now].ctx);
        }
    }
    void barrier() {
        if (++waiting == THREADS) {
            waiting  = 0;
            barriers = true;
            for (Lane& l : lanes)
                if (l.state == BARRIER) l.state = READY;
            return;
        }
        lanes[now].state = BARRIER;
        yield();
    }
    // all 64 lanes give an operand; the last one runs op(lanes of the wave), which fills in every lane's result
    template <typename OP>
    void together(const void* give, void* take, OP&& op) {
        const int w = now / LANES;
        lanes[now].give = give;
        lanes[now].take = take;
        if (++in_wave[w] < LANES) {
            lanes[now].state = WAVE;
            yield();
            return;
        }
        in_wave[w] = 0;
        op(&lanes[w * LANES]);
        for (int l = 0; l < LANES; ++l)
            if (lanes[w * LANES + l].state == WAVE) lanes[w * LANES + l].state = READY;
    }
};
extern thread_local Group* group;
inline void Group::enter() {
    group->body();
    group->lanes[group->now].state = DONE;
}
template <typename F>
void launch(dim3 grid, const F& body) {
    std::vector<std::thread> wgs;
    for (unsigned b = 0; b < grid.x; ++b)
        wgs.emplace_back([=] {
            auto g   = std::make_unique<Group>();
            g->block = dim3(b, 0, 0);
            g->grid  = grid;
            g->body  = body;
            group    = g.get();
            g->run();
            worked[b & 7] += g->barriers;
        });
    for (std::thread& t : wgs) t.join();
}

inline void asm_text(const char* s) {
    if (strstr(s, "s_barrier")) group->barrier();
}
inline bool any(bool b) {
    bool r;
    group->together(&b, &r, [](Lane* l) {
        bool v = false;
        for (int i = 0; i < LANES; ++i) v |= *static_cast<const bool*>(l[i].give);
        for (int i = 0; i < LANES; ++i) *static_cast<bool*>(l[i].take) = v;
    });
    return r;
}
// lane i of a row of 16: the value of lane i + (ctrl & 15), 0 behind the row's end (the only control used: row shift left)
inline int row_shift(int v, int ctrl) {
    struct Give { int v, ctrl; } g{v, ctrl};
    int r;
    group->together(&g, &r, [](Lane* l) {
        for (int i = 0; i < LANES; ++i) {
            const Give* own = static_cast<const Give*>(l[i].give);
            const int   by = own->ctrl & 15;
            if (own->ctrl >> 4 != 0x10) abort();
            *static_cast<int*>(l[i].take) = (i & 15) + by < 16 ? static_cast<const Give*>(l[i + by].give)->v : 0;
        }
    });
    return r;
}
// D = A B + C, 16 x 16 over 32: lane l has row (A) or column (B) l % 16, k = 8 (l / 16) ... + 7, and of C, D rows 4 (l / 16) ... + 3, column l % 16
inline f4 mfma(h8 a, h8 b, f4 c) {
    struct Give { h8 a, b; } g{a, b};
    f4 r = c;
    group->together(&g, &r, [](Lane* l) {
        for (int i = 0; i < LANES; ++i) {
            f4& d = *static_cast<f4*>(l[i].take);
            for (int e = 0; e < 4; ++e) {
                double s = d[e];
                for (int k = 0; k < 32; ++k)
                    s += (double)static_cast<const Give*>(l[16 * (k / 8) + 4 * (i / 16) + e].give)->a[k % 8] *
                         (double)static_cast<const Give*>(l[16 * (k / 8) + i % 16].give)->b[k % 8];
                d[e] = (float)s;
            }
        }
    });
    return r;
}
// transposing LDS read: element e of lane n of 16 is half n % 4 of the 8 bytes that lane 4 e + n / 4 addresses
inline s4 read_tr(const void* p) {
    s4 r;
    group->together(p, &r, [](Lane* l) {
        for (int i = 0; i < LANES; ++i) {
            s4 v;
            for (int e = 0; e < 4; ++e) v[e] = static_cast<const short*>(l[(i & ~15) + 4 * e + (i & 15) / 4].give)[i & 3];
            *static_cast<s4*>(l[i].take) = v;
        }
    });
    return r;
}
struct Rsrc {
    char*    base;
    unsigned bytes;
    char* at(unsigned off, unsigned n) const {
        if (off + n > bytes) {
            fprintf(stderr, "buffer access of %u bytes at %u of %u\n", n, off, bytes);
            abort();
        }
        return base + off;
    }
};
inline u4 load128(Rsrc r, unsigned off) {
    u4 v;
    const volatile uint64_t* p = reinterpret_cast<const volatile uint64_t*>(r.at(off, 16));
    const uint64_t           q[2] = {p[0], p[1]};
    memcpy(&v, q, 16);
    return v;
}
inline void store128(u4 v, Rsrc r, unsigned off) {
    uint64_t q[2];
    memcpy(q, &v, 16);
    volatile uint64_t* p = reinterpret_cast<volatile uint64_t*>(r.at(off, 16));
    p[0] = q[0];
    p[1] = q[1];
}
inline long long ticks() {   // 100 MHz
    return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count() / 10;
}
}  // namespace host

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...) unused
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static thread_local   // (a workgroup is a thread)
#define __restrict__
#define threadIdx (host::group->lanes[host::group->now].thread)
#define blockIdx (host::group->block)
#define gridDim (host::group->grid)
#define hipLaunchKernelGGL(kernel, grid, threads, lds, stream, args) host::launch(grid, [=] { kernel(args); })
#define asm
#define volatile(...) host::asm_text(#__VA_ARGS__)

#define __any(x) host::any(x)
#define __syncthreads() host::group->barrier()
#define __expf(x) expf(x)
#define __float_as_int(x) __builtin_bit_cast(int, (float)(x))
#define __int_as_float(x) __builtin_bit_cast(float, (int)(x))
#define __float_as_uint(x) __builtin_bit_cast(unsigned, (float)(x))
#define __uint_as_float(x) __builtin_bit_cast(float, (unsigned)(x))
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define atomicOr(p, v) __atomic_fetch_or(p, v, __ATOMIC_RELAXED)
#define wall_clock64() host::ticks()
using std::max;
using std::min;
#define __amdgpu_buffer_rsrc_t host::Rsrc
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, bytes, flags) (host::Rsrc{reinterpret_cast<char*>(p), bytes})
#define __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, aux) host::load128(r, off)
#define __builtin_amdgcn_raw_buffer_store_b128(v, r, off, soff, aux) host::store128(v, r, off)
#define __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, aux) __atomic_load_n(reinterpret_cast<unsigned*>((r).at(off, 4)), __ATOMIC_RELAXED)
#define __builtin_amdgcn_raw_buffer_store_b32(v, r, off, soff, aux) __atomic_store_n(reinterpret_cast<unsigned*>((r).at(off, 4)), v, __ATOMIC_RELAXED)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) host::row_shift(v, ctrl)
#define __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, x, y, z) host::mfma(a, b, c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(p) host::read_tr((const void*)(p))
#define __builtin_amdgcn_s_getreg(r) (host::group->block.x & 7u)   // (the XCD)
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __builtin_amdgcn_sched_barrier(n) ((void)0)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) (host::u4{a, b, 0, 0})   // (reductions of whole waves: not in these kernels)
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) (host::u4{a, b, 0, 0})
