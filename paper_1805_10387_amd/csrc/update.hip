// Optimizer wrapper and loss-scale policy kernels (paper Sections 3.1 item 1, 3.2, 3.3).
//
// Both kernels of mp_unscale_check_update are pure streaming kernels bound by HBM:
//   inspect : reads 2 B/parameter  (fp16 gradient bit test, one ballot per wave)
//   update  : Adam reads g16 + w32 + m + v (14 B) and writes w32 + m + v + w16 (14 B) = 28 B/param,
//             SGD reads 6 B and writes 6 B = 12 B/param,
// with 16-byte accesses per lane, consecutive lanes on consecutive addresses.
#include "mean.hpp"

#include <mutex>
#include <string.h>
#include <vector>

namespace mp {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}
int hip_fail(hipError_t e, const char* what) {
    set_error("%s: %s", what, hipGetErrorString(e));
    return MP_E_HIP;
}

// ------------------------------------------------------------------ scale state
__global__ void scale_state_init_kernel(mp_scale_state* st, int mode, float s, int interval, float smin,
                                        float smax) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < MP_HISTORY) {
        st->hist_scale[i]     = 0.f;
        st->hist_found_inf[i] = 0;
    }
    if (i == 0) {
        st->scale = s;
        st->inv_scale = 1.0f / s;
        st->min_scale = smin;
        st->max_scale = smax;
        st->mode = mode;
        st->growth_interval = interval;
        st->good_steps = 0;
        st->found_inf = 0;
        st->opt_step = 0;
        st->total_steps = 0;
        st->skipped_steps = 0;
        st->reserved = 0;
    }
}

__device__ __forceinline__ void loss_scale_update(mp_scale_state* st) {
    const int   found = st->found_inf != 0;
    float       s     = st->scale;
    const int   slot  = st->total_steps % MP_HISTORY;
    st->hist_scale[slot]     = s;
    st->hist_found_inf[slot] = found;
    st->total_steps += 1;
    if (found) {
        st->skipped_steps += 1;
        st->good_steps = 0;
        if (st->mode == MP_SCALE_BACKOFF) s = fmaxf(s * 0.5f, st->min_scale);
    } else {
        st->opt_step += 1;
        int good = st->good_steps + 1;
        if (st->mode == MP_SCALE_BACKOFF && good >= st->growth_interval) {
            s = fminf(s * 2.0f, st->max_scale);
            good = 0;
        }
        st->good_steps = good;
    }
    st->scale     = s;
    st->inv_scale = 1.0f / s;
    st->found_inf = 0;
}
__global__ void loss_scale_update_kernel(mp_scale_state* st) {
    if (threadIdx.x == 0) loss_scale_update(st);
}
// The end of an iteration: the loss out of its partial sums as well, so that it needs no launch between loss and backward (1.6 us of
// a captured chain of small kernels, up to 4.7 behind one that has written much).
template <int LOADS>
__global__ __launch_bounds__(MEAN_THREADS) void loss_scale_update_mean_kernel(mp_scale_state* st, const float* __restrict__ part, int n,
                                                                              double denom, float* __restrict__ loss) {
    if (threadIdx.x == MEAN_THREADS - 1) loss_scale_update(st);
    mean_of_parts<LOADS>(part, n, denom, loss);
}

// ------------------------------------------------------------------ multi-tensor update
constexpr int UPD_THREADS     = 256;
constexpr int UPD_VEC         = 4;                                  // elements per lane per access
constexpr int UPD_PIECE       = UPD_THREADS * UPD_VEC;              // elements a workgroup takes per iteration
constexpr int UPD_MAX_ITERS   = 8;
constexpr int INS_VEC         = 8;                                  // the inspection pass reads fp16 only: 16 B per lane
constexpr int UPD_MAX_TENSORS = 32;                                 // descriptors per launch

// Iterations per workgroup (1, 2, 4 or 8): the fewest with which the list makes no more than about one full chip of
// workgroups (8 of 256 threads per compute unit).  A workgroup's iterations are a serial chain of memory round trips, so
// a small model must not be packed into few workgroups; a large one amortises the start of a workgroup over more work.
// Iteration times with 8 iterations for all -> with this rule and the early loads: 0.22 M parameters 76.0 -> 65.4 us,
// 0.77 M 56.6 -> 48.7, 3.2 M 280 -> 264, 6.4 M 682 -> 663; from 16 M on the split is the same.
static int upd_iters(long long total) {
    int it = 1;
    while (it < UPD_MAX_ITERS && total > 2048ll * UPD_PIECE * it) it *= 2;
    return it;
}

struct UpdBatch {
    const uint16_t*    g16[UPD_MAX_TENSORS];
    float*             w32[UPD_MAX_TENSORS];
    uint16_t*          w16[UPD_MAX_TENSORS];
    float*             m[UPD_MAX_TENSORS];
    float*             v[UPD_MAX_TENSORS];
    unsigned long long n[UPD_MAX_TENSORS];
    int                chunk_start[UPD_MAX_TENSORS + 1];  // first workgroup of each tensor
    unsigned           vec_ok;                            // bit i: tensor i's pointers are 16-byte aligned
    int                ntensors;
};

struct UpdScalars {
    float  lr, beta1, beta2, eps, wd, omb1, omb2;
    double beta1d, beta2d;
    int    kind;
};

// (entries past the last tensor hold the workgroup count: no branch, the whole table comes with a few scalar loads)
__device__ __forceinline__ int find_tensor(const UpdBatch& b, int bid) {
    int t = 0;
#pragma unroll
    for (int i = 1; i < UPD_MAX_TENSORS; ++i) t += bid >= b.chunk_start[i];
    return t;
}

template <int ITERS>
__global__ __launch_bounds__(UPD_THREADS) void inspect_kernel(UpdBatch b, mp_scale_state* st) {
    const int                 t   = find_tensor(b, blockIdx.x);
    const unsigned long long  n   = b.n[t];
    const unsigned long long  off = (unsigned long long)(blockIdx.x - b.chunk_start[t]) * (UPD_PIECE * ITERS);
    const uint16_t*           g   = b.g16[t];
    const bool                vec = (b.vec_ok >> t) & 1u;
    bool                      bad = false;
#pragma unroll
    for (int it = 0; it < (ITERS + 1) / 2; ++it) {
        if (ITERS == 1 && threadIdx.x >= UPD_PIECE / INS_VEC) break;
        const unsigned long long i = off + (unsigned long long)(it * UPD_THREADS + threadIdx.x) * INS_VEC;
        if (vec && i + INS_VEC <= n) {
            const uint4 q = *reinterpret_cast<const uint4*>(g + i);
            // both halves of each 32-bit word: exponent field 0x7C00 all ones
            const unsigned w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                bad |= ((w[k] & 0x7C00u) == 0x7C00u) | ((w[k] & 0x7C000000u) == 0x7C000000u);
            }
        } else {
            for (unsigned long long j = i; j < n && j < i + INS_VEC; ++j) bad |= half_nonfinite(g[j]);
        }
    }
    if (__any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(&st->found_inf, 1);
    }
}

// (1 - beta^t) in double by repeated squaring, rounded to fp32.
__device__ __forceinline__ float bias_correction(double beta, int t) {
    double r = 1.0, p = beta;
    for (int e = t; e > 0; e >>= 1) {
        if (e & 1) r *= p;
        p *= p;
    }
    return (float)(1.0 - r);
}

template <int KIND>
__device__ __forceinline__ void update_one(float g16v, float& w, float& m, float& v, const UpdScalars& s,
                                           float inv_scale, float bc1, float bc2) {
    float g = g16v * inv_scale;
    if (s.wd != 0.f) g = g + s.wd * w;
    if (KIND == MP_OPT_SGD) {
        w = w - s.lr * g;
    } else {
        m = s.beta1 * m + s.omb1 * g;
        v = s.beta2 * v + s.omb2 * (g * g);
        const float mhat = m / bc1;
        const float vhat = v / bc2;
        w = w - s.lr * mhat / (sqrtf(vhat) + s.eps);
    }
}

typedef float    f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x2v __attribute__((ext_vector_type(2)));

// One workgroup's share.  The loads of an iteration do not wait for the scale state: the flag is looked at once they are
// on their way, so a small model's update is one memory round trip long, not two.
// Later iterations load behind their bounds test, in one branch with the arithmetic: with the loads under a test of their own
// large Adam updates took 3 % longer (33.5 M parameters 161 -> 167 us; this way 162).
template <int KIND, int ITERS>
__device__ __forceinline__ void update_share(const UpdBatch& b, const UpdScalars& s, const mp_scale_state* st) {
    const int                t   = find_tensor(b, blockIdx.x);
    const unsigned long long n   = b.n[t];
    const unsigned long long off = (unsigned long long)(blockIdx.x - b.chunk_start[t]) * (UPD_PIECE * ITERS);
    const uint16_t* __restrict__ g16 = b.g16[t];
    float* __restrict__          w32 = b.w32[t];
    uint16_t* __restrict__       w16 = b.w16[t];
    float* __restrict__          mm  = b.m[t];
    float* __restrict__          vv  = b.v[t];
    const bool                   vec = (b.vec_ok >> t) & 1u;

    // pieces of an iteration: streaming data, touched once per step, so non-temporal accesses keep it from displacing
    // cache contents.  Every access instruction of a wave covers one contiguous run (64 lanes x 16 B of fp32, 64 x 8 B of
    // fp16), so each 128-byte line is touched by exactly one load and one store per array
    u32x2v gq;
    f32x4v w0, m0, v0;
    auto   fetch = [&](unsigned long long i) {
        gq = __builtin_nontemporal_load(reinterpret_cast<const u32x2v*>(g16 + i));
        w0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(w32 + i));
        if (KIND == MP_OPT_ADAM) {
            m0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(mm + i));
            v0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(vv + i));
        }
    };
    m0 = v0 = f32x4v{0.f, 0.f, 0.f, 0.f};
    if (vec && off + threadIdx.x * UPD_VEC + UPD_VEC <= n) fetch(off + threadIdx.x * UPD_VEC);
    __builtin_amdgcn_sched_barrier(0);
    if (st->found_inf != 0) return;  // overflow somewhere in this iteration: the whole step is skipped
    const float inv_scale = st->inv_scale;
    float       bc1 = 1.f, bc2 = 1.f;
    if (KIND == MP_OPT_ADAM) {
        const int k = st->opt_step + 1;
        bc1 = bias_correction(s.beta1d, k);
        bc2 = bias_correction(s.beta2d, k);
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const unsigned long long i = off + (unsigned long long)(it * UPD_THREADS + threadIdx.x) * UPD_VEC;
        if (vec && i + UPD_VEC <= n) {
            if (it > 0) fetch(i);
            const float gh[4] = {h2f((uint16_t)(gq.x & 0xFFFFu)), h2f((uint16_t)(gq.x >> 16)),
                                 h2f((uint16_t)(gq.y & 0xFFFFu)), h2f((uint16_t)(gq.y >> 16))};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float w = w0[k], m = m0[k], v = v0[k];
                update_one<KIND>(gh[k], w, m, v, s, inv_scale, bc1, bc2);
                w0[k] = w;
                m0[k] = m;
                v0[k] = v;
            }
            __builtin_nontemporal_store(w0, reinterpret_cast<f32x4v*>(w32 + i));
            if (KIND == MP_OPT_ADAM) {
                __builtin_nontemporal_store(m0, reinterpret_cast<f32x4v*>(mm + i));
                __builtin_nontemporal_store(v0, reinterpret_cast<f32x4v*>(vv + i));
            }
            u32x2v hq;
            hq.x = (unsigned)f2h(w0.x) | ((unsigned)f2h(w0.y) << 16);
            hq.y = (unsigned)f2h(w0.z) | ((unsigned)f2h(w0.w) << 16);
            *reinterpret_cast<u32x2v*>(w16 + i) = hq;  // read again by the next forward pass: ordinary store
        } else {
            for (unsigned long long j = i; j < n && j < i + UPD_VEC; ++j) {
                float w = w32[j], m1 = 0.f, v1 = 0.f;
                if (KIND == MP_OPT_ADAM) {
                    m1 = mm[j];
                    v1 = vv[j];
                }
                update_one<KIND>(h2f(g16[j]), w, m1, v1, s, inv_scale, bc1, bc2);
                w32[j] = w;
                if (KIND == MP_OPT_ADAM) {
                    mm[j] = m1;
                    vv[j] = v1;
                }
                w16[j] = f2h(w);
            }
        }
    }
}

template <int KIND, int ITERS>
__global__ __launch_bounds__(UPD_THREADS) void update_kernel(UpdBatch b, UpdScalars s, const mp_scale_state* st) {
    update_share<KIND, ITERS>(b, s, st);
}

// The update whose last workgroup to arrive also ends the iteration: nobody reads the state any more by then.  Arrivals are
// counted in two levels (9 ns each at one address: 500 workgroups on one counter take 4.4 us): UPD_END_GROUPS counters a cache
// line apart, then one for the groups; whoever completes a counter clears it for the next call.  us of inspection, update
// and scale update in a captured chain, apart / this way: 0.05 M parameters 7.8 / 8.0, 0.5 M 9.3 / 9.1, 1 M 10.3 / 10.2, 2 M 14.9 / 15.1;
// called one by one a launch is 4.4 us of the host's time, which is what a small model's iteration waits for (64 x 256 network 41.8
// -> 36.5, ragged 192-wide layer 108 -> 102, LSTM of 2 x 128 71.5 -> 65.5, the host's other savings with it).
constexpr int UPD_END_WGS = 1024, UPD_END_GROUPS = 32, UPD_END_LINE = 32;
struct UpdEnd {
    mp_mean_parts parts;
    float*        loss;
    int*          counters;   // [UPD_END_GROUPS + 1][UPD_END_LINE]
};
template <int KIND, int ITERS>
__global__ __launch_bounds__(UPD_THREADS) void update_end_kernel(UpdBatch b, UpdScalars s, mp_scale_state* st, UpdEnd end) {
    static_assert(UPD_THREADS == MEAN_THREADS, "one workgroup size");
    __shared__ int last;
    update_share<KIND, ITERS>(b, s, st);
    __syncthreads();   // (every wave has read the state)
    if (threadIdx.x == 0) {
        const int wgs = gridDim.x, group = blockIdx.x % UPD_END_GROUPS, members = (wgs - group + UPD_END_GROUPS - 1) / UPD_END_GROUPS;
        int* const mine = end.counters + group * UPD_END_LINE;
        int* const all  = end.counters + UPD_END_GROUPS * UPD_END_LINE;
        last = 0;
        if (atomicAdd(mine, 1) == members - 1) {
            *mine = 0;
            if (atomicAdd(all, 1) == min(wgs, UPD_END_GROUPS) - 1) {
                *all = 0;
                last = 1;
            }
        }
    }
    __syncthreads();
    if (!last) return;
    if (threadIdx.x == UPD_THREADS - 1) loss_scale_update(st);
    if (end.parts.part) mean_of_parts<MEAN_LOADS>(end.parts.part, end.parts.n, end.parts.denom, end.loss);
}

// *ended: in: whether to end the iteration too, out: whether that was done (`end`)
template <int ITERS>
static int launch_update(const std::vector<UpdBatch>& batches, const UpdScalars& s, mp_scale_state* st, bool inspect, const UpdEnd& end, bool* ended,
                         hipStream_t hs) {
    const bool with_end = *ended && !batches.empty() && batches.back().chunk_start[batches.back().ntensors] <= UPD_END_WGS;
    *ended = with_end;
    if (inspect) {
        for (const UpdBatch& b : batches) {
            hipLaunchKernelGGL(inspect_kernel<ITERS>, dim3(b.chunk_start[b.ntensors]), dim3(UPD_THREADS), 0, hs, b, st);
            MP_LAUNCH_CHECK("mp_unscale_check_update(inspect)");
        }
    }
    for (const UpdBatch& b : batches) {
        if (with_end && &b == &batches.back()) {
            if (s.kind == MP_OPT_ADAM)
                hipLaunchKernelGGL((update_end_kernel<MP_OPT_ADAM, ITERS>), dim3(b.chunk_start[b.ntensors]), dim3(UPD_THREADS), 0, hs, b, s, st, end);
            else
                hipLaunchKernelGGL((update_end_kernel<MP_OPT_SGD, ITERS>), dim3(b.chunk_start[b.ntensors]), dim3(UPD_THREADS), 0, hs, b, s, st, end);
        } else if (s.kind == MP_OPT_ADAM)
            hipLaunchKernelGGL((update_kernel<MP_OPT_ADAM, ITERS>), dim3(b.chunk_start[b.ntensors]), dim3(UPD_THREADS), 0, hs, b, s, st);
        else
            hipLaunchKernelGGL((update_kernel<MP_OPT_SGD, ITERS>), dim3(b.chunk_start[b.ntensors]), dim3(UPD_THREADS), 0, hs, b, s, st);
        MP_LAUNCH_CHECK("mp_unscale_check_update(update)");
    }
    return MP_OK;
}

}  // namespace mp

using namespace mp;

extern "C" const char* mp_last_error(void) { return g_err; }
extern "C" int         mp_version(void) { return MP_VERSION; }

extern "C" int mp_scale_state_init(mp_scale_state* st, int mode, float init_scale, int growth_interval,
                                   float min_scale, float max_scale, mp_stream stream) {
    MP_REQUIRE(st != nullptr, "mp_scale_state_init: st is NULL");
    MP_REQUIRE(mode == MP_SCALE_STATIC || mode == MP_SCALE_BACKOFF, "mp_scale_state_init: bad mode %d", mode);
    MP_REQUIRE(growth_interval >= 1, "mp_scale_state_init: growth_interval %d < 1", growth_interval);
    MP_REQUIRE(init_scale > 0.f && min_scale > 0.f && min_scale <= init_scale && init_scale <= max_scale,
               "mp_scale_state_init: need 0 < min_scale <= init_scale <= max_scale (got %g %g %g)",
               (double)min_scale, (double)init_scale, (double)max_scale);
    hipLaunchKernelGGL(scale_state_init_kernel, dim3((MP_HISTORY + 255) / 256), dim3(256), 0, as_stream(stream),
                       st, mode, init_scale, growth_interval, min_scale, max_scale);
    MP_LAUNCH_CHECK("mp_scale_state_init");
    return MP_OK;
}

extern "C" int mp_loss_scale_update(mp_scale_state* st, mp_stream stream) {
    MP_REQUIRE(st != nullptr, "mp_loss_scale_update: st is NULL");
    hipLaunchKernelGGL(loss_scale_update_kernel, dim3(1), dim3(64), 0, as_stream(stream), st);
    MP_LAUNCH_CHECK("mp_loss_scale_update");
    return MP_OK;
}

extern "C" int mp_loss_scale_update_mean(mp_scale_state* st, const mp_mean_parts* parts, float* loss, mp_stream stream) {
    MP_REQUIRE(st && parts && loss, "mp_loss_scale_update_mean: NULL argument");
    MP_REQUIRE(parts->part && parts->n > 0, "mp_loss_scale_update_mean: no partial sums");
    hipStream_t hs = as_stream(stream);
    if (parts->n <= MEAN_THREADS)
        hipLaunchKernelGGL(loss_scale_update_mean_kernel<1>, dim3(1), dim3(MEAN_THREADS), 0, hs, st, parts->part, parts->n, parts->denom, loss);
    else
        hipLaunchKernelGGL(loss_scale_update_mean_kernel<MEAN_LOADS>, dim3(1), dim3(MEAN_THREADS), 0, hs, st, parts->part, parts->n, parts->denom, loss);
    MP_LAUNCH_CHECK("mp_loss_scale_update_mean");
    return MP_OK;
}

// *ended: see launch_update
static int unscale_check_update(const mp_tensor_desc* tensors, int ntensors, const mp_opt_cfg* cfg, mp_scale_state* st, int flags,
                                const UpdEnd& end, bool* ended, mp_stream stream) {
    MP_REQUIRE(st != nullptr && cfg != nullptr, "mp_unscale_check_update: st / cfg is NULL");
    MP_REQUIRE(ntensors >= 0 && (ntensors == 0 || tensors != nullptr), "mp_unscale_check_update: bad tensor list");
    MP_REQUIRE(cfg->kind == MP_OPT_SGD || cfg->kind == MP_OPT_ADAM, "mp_unscale_check_update: bad optimizer kind %d",
               cfg->kind);
    MP_REQUIRE((flags & ~MP_UPDATE_PRECHECKED) == 0, "mp_unscale_check_update: unknown flags 0x%x", flags);
    for (int i = 0; i < ntensors; ++i) {
        const mp_tensor_desc& d = tensors[i];
        if (d.n == 0) continue;
        MP_REQUIRE(d.g16 && d.w32 && d.w16, "mp_unscale_check_update: tensor %d has a NULL g16/w32/w16", i);
        MP_REQUIRE(cfg->kind != MP_OPT_ADAM || (d.m && d.v), "mp_unscale_check_update: tensor %d lacks Adam moments", i);
        MP_REQUIRE((reinterpret_cast<uintptr_t>(d.g16) & 1) == 0 && (reinterpret_cast<uintptr_t>(d.w16) & 1) == 0 &&
                       (reinterpret_cast<uintptr_t>(d.w32) & 3) == 0,
                   "mp_unscale_check_update: tensor %d is not element-aligned", i);
        MP_REQUIRE(d.n < (1ull << 40), "mp_unscale_check_update: tensor %d too large", i);
    }

    UpdScalars s;
    s.kind   = cfg->kind;
    s.lr     = (float)cfg->lr;
    s.beta1  = (float)cfg->beta1;
    s.beta2  = (float)cfg->beta2;
    s.eps    = (float)cfg->eps;
    s.wd     = (float)cfg->weight_decay;
    s.omb1   = (float)(1.0 - cfg->beta1);
    s.omb2   = (float)(1.0 - cfg->beta2);
    s.beta1d = cfg->beta1;
    s.beta2d = cfg->beta2;

    long long total = 0;
    for (int i = 0; i < ntensors; ++i) total += (long long)tensors[i].n;
    const int             iters = upd_iters(total);
    const long long       chunk = (long long)UPD_PIECE * iters;
    std::vector<UpdBatch> batches;
    UpdBatch              cur;
    cur = UpdBatch{};
    long long chunks = 0;
    auto      flush  = [&]() {
        if (cur.ntensors > 0) {
            for (int k = cur.ntensors; k <= UPD_MAX_TENSORS; ++k) cur.chunk_start[k] = (int)chunks;
            batches.push_back(cur);
        }
        cur = UpdBatch{};
        chunks = 0;
    };
    for (int i = 0; i < ntensors; ++i) {
        const mp_tensor_desc& d = tensors[i];
        if (d.n == 0) continue;
        const long long c = ((long long)d.n + chunk - 1) / chunk;
        if (cur.ntensors == UPD_MAX_TENSORS || chunks + c > 0x3FFFFFFF) flush();
        const int k = cur.ntensors++;
        cur.g16[k]  = d.g16;
        cur.w32[k]  = d.w32;
        cur.w16[k]  = d.w16;
        cur.m[k]    = d.m;
        cur.v[k]    = d.v;
        cur.n[k]    = d.n;
        cur.chunk_start[k] = (int)chunks;
        const bool ok = aligned16(d.g16) && aligned16(d.w32) && aligned16(d.w16) &&
                        (cfg->kind != MP_OPT_ADAM || (aligned16(d.m) && aligned16(d.v)));
        if (ok) cur.vec_ok |= (1u << k);
        chunks += c;
    }
    flush();

    const bool inspect = !(flags & MP_UPDATE_PRECHECKED);
    switch (iters) {
        case 1: return launch_update<1>(batches, s, st, inspect, end, ended, as_stream(stream));
        case 2: return launch_update<2>(batches, s, st, inspect, end, ended, as_stream(stream));
        case 4: return launch_update<4>(batches, s, st, inspect, end, ended, as_stream(stream));
        default: return launch_update<8>(batches, s, st, inspect, end, ended, as_stream(stream));
    }
}

extern "C" int mp_unscale_check_update(const mp_tensor_desc* tensors, int ntensors, const mp_opt_cfg* cfg,
                                       mp_scale_state* st, int flags, mp_stream stream) {
    bool ended = false;
    return unscale_check_update(tensors, ntensors, cfg, st, flags, UpdEnd{}, &ended, stream);
}

extern "C" size_t mp_update_counters_bytes(void) { return (UPD_END_GROUPS + 1) * UPD_END_LINE * sizeof(int); }

extern "C" int mp_unscale_check_update_end(const mp_tensor_desc* tensors, int ntensors, const mp_opt_cfg* cfg, mp_scale_state* st,
                                           int flags, const mp_mean_parts* parts, float* loss, int32_t* counters, mp_stream stream) {
    MP_REQUIRE(counters != nullptr && (reinterpret_cast<uintptr_t>(counters) & 3) == 0, "mp_unscale_check_update_end: counters NULL or not 4-byte aligned");
    MP_REQUIRE(parts == nullptr || (parts->part && parts->n > 0 && loss), "mp_unscale_check_update_end: parts without partial sums or loss");
    const UpdEnd end{parts ? *parts : mp_mean_parts{}, loss, counters};
    bool      ended = true;
    const int rc    = unscale_check_update(tensors, ntensors, cfg, st, flags, end, &ended, stream);
    if (rc != MP_OK || ended) return rc;
    return parts ? mp_loss_scale_update_mean(st, parts, loss, stream) : mp_loss_scale_update(st, stream);
}
