// Persistent recurrent-layer kernels: every time step of one LSTM layer in ONE launch per direction (the GNMT-like
// encoder of the paper's Section 2 configuration listing and Section 5.1; arithmetic of Sections 3.1 / 3.2: fp16
// operands, fp32 sums, fp16 storage points, fp32 cell state).
//
// A layer unrolled over time is a chain of small dependent products (batch rows x [4H, H]): launched one by one a time
// step costs its launches and first-load latencies, not its bytes.  Here each workgroup owns RL_UNITS hidden units of
// RL_ROWS batch rows for the whole sequence (batch rows never mix in the recurrence, so each block of rows is a group
// of workgroups of its own that never waits for another):
//   forward : its 4 x RL_UNITS rows of the recurrent weight block W_h live in registers as matrix-core fragments for
//             all T steps; per step it takes h_{t-1} (all units) from the exchange ring, forms its gate sums, adds the
//             input half x_t W_x^T (computed for all steps at once by one large product beforehand, kept fp32, so the
//             gate sum is still rounded once), updates its cells (c in registers, fp32) and publishes its slice of h_t.
//   backward: its RL_UNITS columns of W_h (as W_h^T fragments) live in registers; per step it runs the cell backward
//             for its units (the recurrent gradient of its own units and the cell-state gradient never leave the
//             workgroup), publishes its slice of dgates_t, and contracts the whole dgates_t (rows x 4H) with its columns
//             to get the recurrent gradient of its units for step t - 1.
//
// What bounds a time step is the trip of a small tensor from every workgroup to every other through the memory system.
// There is no barrier and no flag: the data announce themselves.  The exchanged slice of a step goes to a slot of a
// ring of RL_RING slots that is filled with a bit pattern no published value has (RL_EMPTY), with device-scope stores,
// and a reader loads the whole slice with device-scope loads until none of it is empty.  One trip per step instead of
// three (data acknowledged - flag raised - flag seen - data fetched), no cache write-back or invalidation, and a wave
// waits for exactly the values it multiplies.  Slots lie in the order the matrix cores take them (one coalesced 1 KB
// load per fragment pair), and a publisher writes whole 128-byte lines.
//   Reuse: P_n (the slice of step n) is published by a workgroup after a workgroup barrier behind which all its waves
//   have read P_(n-1).  So once a workgroup has seen P_(n-1) from everybody, everybody has read P_(n-2), and after
//   publishing P_n it empties its part of P_(n-2); that is acknowledged ahead of its P_(n+1), and only
//   who has seen P_(n+1) from everybody looks for P_(n+2), which takes the slot over.
//   8 batch rows per workgroup, not the matrix core's 16: a group then reads half as much (64 KB per workgroup and
//   backward step, 0.4 us at the vector cache's 64 bytes a clock) and 32 rows x 1024 units occupy 256 workgroups.  The 16
//   columns of an operand hold 8 rows of two successive k-steps; each is multiplied with both k-steps' weights into
//   separate sums, and the half of each result that pairs the right ones is kept.
//   Distance: a slice takes 0.57 us between two XCDs and 0.45 inside one when it is stored to the whole device, 0.28 inside
//   one when the store stays in the L2 that reader and writer share (both ways in turn between two workgroups).  So the
//   placed calls put a group of up to 32 workgroups on one XCD, which stores to its L2 once every member has told that it runs
//   there (RlXcds); wider layers have groups that no XCD holds with one workgroup per compute unit, and keep the order of the ids.
//   So do the other calls unless the groups come out even over the XCDs: three one-group launches that fit the device may not fit
//   one XCD.  (us per time step, forward / backward, spread and placed: 512 x 8 1.58 / 1.71 and 1.20 / 1.45, 256 x 32 1.49 / 1.53
//   and 1.06 / 1.06, 128 x 8 1.45 / 1.41 and 0.98 / 0.94.)
//   What else an owner of cells does between two slices counts in full, so it does nothing else: inputs and results go through
//   waves 2 and 3 (RlCellIn), the backward activations are made while the slices are on their way, and the status word
//   is looked at after 16 looks in vain, not after the first.
// us per time step, forward / backward, 50 steps, one launch of the placed calls: units x batch 1024 x 32 2.04 / 2.51 before these four and 1.76 /
// 2.29 with them, 768 x 40 1.86 / 2.31 -> 1.66 / 2.05, 512 x 64 1.68 / 2.06 -> 1.20 / 1.44, 256 x 32 1.53 / 1.79 -> 1.05 / 1.02, 128 x 8
// 1.50 / 1.65 -> 0.96 / 0.92 (one flag per workgroup behind a device-scope release and acquire, 1024 x 32: 6.7 / 10.0).
// All workgroups must be co-resident: the register use allows two per compute unit and the host refuses larger grids.
// Every wait is bounded in wall-clock time; a wave that gives up raises *status and stops waiting, which makes every other
// wave give up too, and all of them walk the remaining steps without waiting: the grid always drains.
#include "cell_math.hpp"
#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace mp {

constexpr int RL_THREADS = 256;  // 4 waves: each takes a quarter of the contraction
constexpr int RL_UNITS   = 16;   // hidden units per workgroup = one 16-row matrix-core block per gate
constexpr int RL_ROWS    = 8;    // batch rows per workgroup; more rows: more groups of workgroups
constexpr int RL_CELLS   = RL_UNITS * RL_ROWS;
constexpr int RL_MAX_H   = 1024; // register budget of the fragment arrays below
constexpr int RL_MAX_B   = 32;
constexpr int RL_RING    = 4;    // slots of the exchange ring
constexpr int RL_EAGER   = 4;    // fragment pairs per wave up to which a group on one XCD looks at once
constexpr int RL_XCD_WGS = 32;   // workgroups of an XCD, one per compute unit
constexpr int RL_VMCNT0 = 0x0F70;  // operand of s_waitcnt: all vector memory operations done, nothing else waited for
constexpr uint16_t RL_EMPTY = 0xFFFF;  // a NaN; published NaNs of this pattern lose one payload bit on the way
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef short    s16x4 __attribute__((ext_vector_type(4)));

struct RlSync {
    char*     ring;         // [groups][RL_RING][slot bytes], all RL_EMPTY at launch
    int*      status;       // 0 on entry; set nonzero by a wave whose wait ran out
    int       never;        // tests: behave as if part of every slice never arrived
    long long limit_ticks;  // bound of one wait, in ticks of the constant 100 MHz clock
    u32x4*    next;         // the ring of the launch behind this one, which this one fills with RL_EMPTY ...
    unsigned  next_pieces;  // ... in 16-byte pieces (0: none)
    char*     xcds;         // where workgroups tell their XCD: RL_XCD_WGS words per group, RL_EMPTY at launch (NULL: they need not)
    int       per_xcd;      // > 0: every group on one XCD, which has so many workgroups (see rl_per_xcd)
    int       first_xcd;    // ... and that of group 0
};
// Which workgroup this is: its group, and which of the group's units.  Ids go round the 8 XCDs; with per_xcd the grid is 8 times
// that, and places behind the last group have nothing to do.
struct RlPlace {
    int group, unit_block;
};
__device__ __forceinline__ RlPlace rl_place(const RlSync& s, const int units) {
    const int id = blockIdx.x;
    const int v  = s.per_xcd > 0 ? ((id - s.first_xcd) & 7) * s.per_xcd + (id >> 3) : id;
    return {v / units, v % units};
}
// A launch's ring has to be empty before it starts: a fill launch (5 us of a captured chain, of the 46 to 130 us that the
// recurrent kernels take) unless the launch ahead has done it, one or a few stores per thread that nothing waits for.
__device__ __forceinline__ void rl_empty_next(const RlSync& s) {
    for (unsigned i = blockIdx.x * RL_THREADS + threadIdx.x; i < s.next_pieces; i += gridDim.x * RL_THREADS)
        s.next[i] = u32x4{~0u, ~0u, ~0u, ~0u};
}

constexpr int RL_DEVICE_SCOPE = 16;  // cache-policy bit (sc1) of the buffer intrinsics: coherent across the device
constexpr int RL_XCD_SCOPE    = 0;   // of a store that only workgroups of the same XCD read past their vector caches: it stays in the L2
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rl_ring(char* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}

// After look number `it` in vain: give up when the wait has lasted too long or another wave has given up.  (Not after the first
// looks: the status takes as long to read as a slice.)
__device__ __forceinline__ void rl_check_wait(const int it, long long& t0, const RlSync& s, bool& dead) {
    if ((it & 15) != 15) return;
    const long long now = wall_clock64();
    if (it == 15) t0 = now;
    const int give_up = (now - t0 > s.limit_ticks) || __hip_atomic_load(s.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    if (__any(give_up)) {  // (lanes read the clock a few ticks apart: the wave decides as one)
        dead = true;
        if ((threadIdx.x & 63) == 0) atomicOr(s.status, 1);
    }
}

// publish(store) with the stores of the scope that reaches every workgroup of the group
template <typename PUBLISH>
__device__ __forceinline__ void rl_publish(__amdgpu_buffer_rsrc_t ring, const bool local, PUBLISH&& publish) {
    if (local) publish([&](const u32x4& v, unsigned at) { __builtin_amdgcn_raw_buffer_store_b128(v, ring, at, 0, RL_XCD_SCOPE); });
    else publish([&](const u32x4& v, unsigned at) { __builtin_amdgcn_raw_buffer_store_b128(v, ring, at, 0, RL_DEVICE_SCOPE); });
}

// The NP fragment pairs (1 KB apart) of a published slice, loaded until nothing in them is empty.  GUARD_LAST: lanes
// without last_ok never get anything in the last pair (it reads as zero there).  Waves decide alone; `dead` (wave-uniform) is set when this
// or another wave gave up, and ends all waiting.
template <int NP, bool GUARD_LAST, typename MEANWHILE>
__device__ __forceinline__ void rl_take(__amdgpu_buffer_rsrc_t ring, unsigned off, bool last_ok, u32x4 (&f)[NP],
                                        const RlSync& s, bool& dead, MEANWHILE&& meanwhile) {
    constexpr int CH = 4, NC = (NP + CH - 1) / CH;
    unsigned  absent = (1u << NC) - 1;  // the parts of CH pairs that are not whole yet
    long long t0     = 0;
    for (int it = 0;; ++it) {
        asm volatile("" ::: "memory");  // (every round loads anew)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (!(absent >> c & 1u)) continue;
#pragma unroll
            for (int p = c * CH; p < NP && p < (c + 1) * CH; ++p) f[p] = __builtin_amdgcn_raw_buffer_load_b128(ring, off + p * 1024, 0, RL_DEVICE_SCOPE);
        }
        if (it == 0) {
            __builtin_amdgcn_sched_barrier(0);
            meanwhile();
            __builtin_amdgcn_sched_barrier(0);
        }
        if (GUARD_LAST && !last_ok) f[NP - 1] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            u16x2 m = {0, 0};  // the largest half seen: RL_EMPTY is the largest pattern there is
#pragma unroll
            for (int p = c * CH; p < NP && p < (c + 1) * CH; ++p) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const unsigned x = f[p][w];
                    m                = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, x));
                }
            }
            if (!__any(m[0] == RL_EMPTY || m[1] == RL_EMPTY || s.never != 0)) absent &= ~(1u << c);
        }
        if (dead || absent == 0) return;
        rl_check_wait(it, t0, s, dead);
    }
}

// Whether all workgroups of a group run on one XCD.  Each tells its XCD at the start of the launch, ahead of its P_0, and asks
// once it has requested P_0 from the others.  An answer that is not there yet counts as no: a workgroup that publishes to the
// whole device is right whatever the others do.
__device__ __forceinline__ unsigned rl_xcd() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)); }  // hardware register XCC_ID, 4 bits
template <int UNITS>
struct RlXcds {
    __amdgpu_buffer_rsrc_t told;
    unsigned               answer;
    bool                   on;
    __device__ __forceinline__ RlXcds(const RlSync& s, const RlPlace& p, int T) {
        on = UNITS <= RL_XCD_WGS && s.xcds != nullptr && T > 1;
        if (!on) return;
        told = rl_ring(s.xcds + p.group * 4 * RL_XCD_WGS, 4 * UNITS);
        if (threadIdx.x == 0) __builtin_amdgcn_raw_buffer_store_b32(rl_xcd(), told, 4 * p.unit_block, 0, RL_DEVICE_SCOPE);
    }
    __device__ __forceinline__ void ask() {
        const unsigned lane = threadIdx.x & 63;
        if (on) answer = lane < UNITS ? __builtin_amdgcn_raw_buffer_load_b32(told, 4 * lane, 0, RL_DEVICE_SCOPE) : rl_xcd();
    }
    __device__ __forceinline__ bool all_here() const { return on && !__any(answer != rl_xcd()); }
};

// x of this lane (lanes 0-7 of each 16) plus y of the lane 8 further on
__device__ __forceinline__ float rl_add_upper(float x, float y) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), 0x108, 0xF, 0xF, true));
}

// Inputs of a cell-backward step.  In both kernels waves 0 and 1 own a cell per thread, and waves 2 and 3, which would only wait
// while the cells are worked on and the slice is on its way, fetch the cells' inputs from memory and store their results; both
// go through LDS.  (Accesses complete in order: in an owner's queue a load from memory holds up the slice's acknowledgement or
// the slices that it waits for.)
struct RlCellIn {
    unsigned g[4];    // stored gate sums i, f, g, o (a word each: packing them would wait for the loads)
    float    cp, cn;  // cell state before and after the step
    unsigned da;      // gradient from the layer above
};

// The 8 values of lanes 8 j .. 8 j + 7, packed, in lane 8 j (row shifts within 16 lanes), none of them RL_EMPTY.
__device__ __forceinline__ u32x4 rl_gather8(uint16_t h) {
    const int      v  = h == RL_EMPTY ? RL_EMPTY - 1 : h;
    const unsigned w  = (unsigned)v | ((unsigned)__builtin_amdgcn_update_dpp(0, v, 0x101, 0xF, 0xF, true) << 16);
    return u32x4{w, (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x102, 0xF, 0xF, true),
                 (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x104, 0xF, 0xF, true),
                 (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x106, 0xF, 0xF, true)};
}
__device__ __forceinline__ f16x8 as_frag(const u32x4& v) { return __builtin_bit_cast(f16x8, v); }

// ------------------------------------------------------------------------------------------------ forward
struct LstmFwdArgs {
    int             T, B, I, H;
    long long       step_rows;  // rows from one time step to the next in all tensors (>= B)
    const float*    gx;     // [T*step_rows, 4H] fp32: x_t W_x^T
    const uint16_t* w;      // [4H, ldw]; recurrent block = columns I .. I+H
    int             ldw;
    const uint16_t* bias;   // [4H]
    uint16_t*       gates;  // [T*step_rows, 4H] out
    float*          c;      // [(T+1)*step_rows, H]: rows of step 0 given, steps 1..T out
    uint16_t*       xh;     // [T*step_rows, ldxh]: h_0 is read from columns I.. of step 0, h_t written to step t+1
    int             ldxh;
    uint16_t*       h_up;   // [T*step_rows, ld_up] or NULL: h_t also goes here
    int             ld_up;
    RlSync          sync;
};
// The contraction over h is cut into k-steps of 32, dealt to the 4 waves in runs that differ by at most one.  Most
// k-steps of a wave, fragment pairs per wave, and bytes of one slot:
__host__ __device__ constexpr int      rl_fwd_steps(int H) { return (H / 32 + 3) / 4; }
__host__ __device__ constexpr int      rl_fwd_pairs(int H) { return (rl_fwd_steps(H) + 1) / 2; }
__host__ __device__ constexpr unsigned rl_fwd_slot(int H) { return 4u * 1024u * rl_fwd_pairs(H); }

template <int HQ>  // H = 64 HQ
__global__ __launch_bounds__(RL_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_layer_fwd_kernel(LstmFwdArgs a) {
    __shared__ f32x4 in[2][RL_CELLS];   // per step parity: input half of a cell's gate sums ...
    __shared__ u32x4 out[2][RL_CELLS];  // ... and what it leaves: gate sums (4 halves), h (a half), c (fp32)
    __shared__ f32x4 red[2][4][RL_ROWS][RL_UNITS + 1];  // per step parity and wave: partial gate sums, all four of a cell together
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    constexpr int H = 64 * HQ;
    const int I = a.I, T = a.T;
    rl_empty_next(a.sync);
    const RlPlace place = rl_place(a.sync, H / RL_UNITS);
    const int j0  = place.unit_block * RL_UNITS;   // this workgroup's hidden units
    const int b0  = place.group * RL_ROWS;         // ... and batch rows
    if (b0 >= a.B) return;
    const int nb  = min(RL_ROWS, a.B - b0);
    constexpr int nks = rl_fwd_steps(H), np = rl_fwd_pairs(H);
    constexpr int each = H / 32 / 4, more = H / 32 % 4;    // k-steps of every wave; that many waves have one more
    const int mine = each + (wave < more ? 1 : 0);
    const int k0   = 32 * (wave * each + min(wave, more)) + 8 * lq;  // first k of this lane's 8 consecutive values, + 32 ks
    const bool last_ok = 2 * (np - 1) + (lr >> 3) < mine;            // this lane's k-step of the last pair exists
    constexpr unsigned slot = rl_fwd_slot(H);
    const __amdgpu_buffer_rsrc_t ring = rl_ring(a.sync.ring + (size_t)place.group * RL_RING * slot, RL_RING * slot);
    bool dead = false, local = false;
    RlXcds<H / RL_UNITS> xcds(a.sync, place, T);

    // W_h fragments, resident for the whole sequence: gate g, unit lr, 8 consecutive k
    u32x4 wf[4][nks];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int ks = 0; ks < nks; ++ks) {
            wf[g][ks] = u32x4{0u, 0u, 0u, 0u};
            if (more == 0 || ks < mine) wf[g][ks] = *reinterpret_cast<const u32x4*>(a.w + (long long)(g * H + j0 + lr) * a.ldw + I + k0 + 32 * ks);
        }

    // cells: batch row b0 + cr, unit j0 + cu.  Waves 0 and 1 own them; waves 2 and 3 fetch their inputs and store their results
    // (see RlCellIn).  Rows beyond the batch repeat the last one (their values are published but never stored), so that no load
    // hangs on a condition.
    const int  ct = tid & (RL_CELLS - 1), cr = ct >> 4, cu = ct & 15;
    const bool owner = tid < RL_CELLS, cell = cr < nb;
    const long long brow = b0 + min(cr, nb - 1);
    float cst = 0.f, bia[4] = {0.f, 0.f, 0.f, 0.f};
    f32x4 gx;  // waves 2 and 3: input half of the next step's gate sums
    auto  load_gx = [&](int t) {
#pragma unroll
        for (int g = 0; g < 4; ++g) gx[g] = a.gx[(t * a.step_rows + brow) * 4 * H + g * H + j0 + cu];
    };
    if (owner) {
#pragma unroll
        for (int g = 0; g < 4; ++g) bia[g] = h2f(a.bias[g * H + j0 + cu]);
        cst = a.c[brow * H + j0 + cu];
    } else {
        load_gx(0);
    }
    auto store_step = [&](int t) {  // what step t leaves in memory
        const u32x4     r   = out[t & 1][ct];
        const long long row = t * a.step_rows + brow;
        uint16_t* const g   = a.gates + row * 4 * H + j0 + cu;
        const uint16_t  h16 = (uint16_t)r[2];
        g[0]     = (uint16_t)r[0];
        g[H]     = (uint16_t)(r[0] >> 16);
        g[2 * H] = (uint16_t)r[1];
        g[3 * H] = (uint16_t)(r[1] >> 16);
        a.c[(row + a.step_rows) * H + j0 + cu] = __uint_as_float(r[3]);
        if (t + 1 < T) a.xh[(row + a.step_rows) * a.ldxh + I + j0 + cu] = h16;
        if (a.h_up != nullptr) a.h_up[row * a.ld_up + j0 + cu] = h16;
    };
    // where this workgroup's units lie in a slot: fragment pair, k-step of the pair, and the lane rows of its two 8-unit pieces
    const int      jks = j0 >> 5, jw = jks < more * (each + 1) ? jks / (each + 1) : (each > 0 ? (jks - more) / (each > 0 ? each : 1) : 0);
    const int      pks = jks - (jw * each + min(jw, more)), plq = ((j0 & 31) >> 3) + (cu >> 3);
    const unsigned pub = (jw * np + (pks >> 1)) * 1024 + (plq * 16 + (pks & 1) * 8 + cr) * 16;

    // A slice is published ahead of everything else of its step, and the workgroup looks for the others' when its own is
    // acknowledged: looks queue ahead of stores on their way out and keep invalidated lines moving between the caches (1024 units
    // without that wait: 2.3 us a step instead of 1.8).  Inside one XCD a look costs little where a wave takes few pairs, and the
    // wait is left out (128 units: 0.1 us a step; 512 units backward, 8 pairs, are 0.05 slower without it).
    for (int t = 0; t < T; ++t) {
        // lane lr < 8: row lr, k-step 2 p of pair p; lr >= 8: row lr - 8, k-step 2 p + 1
        u32x4 f[np];
        if (t == 0) {
#pragma unroll
            for (int p = 0; p < np; ++p) {
                f[p] = u32x4{0u, 0u, 0u, 0u};
                if (2 * p + (lr >> 3) < mine && (lr & 7) < nb)
                    f[p] = *reinterpret_cast<const u32x4*>(a.xh + (long long)(b0 + (lr & 7)) * a.ldxh + I + k0 + 32 * (2 * p + (lr >> 3)));
            }
        } else {
            rl_take<np, (more != 0 || (nks & 1) != 0)>(ring, ((t - 1) % RL_RING) * slot + wave * np * 1024 + lane * 16, last_ok, f, a.sync, dead, [&] {
                if (t == 1) xcds.ask();
            });
            __builtin_amdgcn_s_waitcnt(RL_VMCNT0);  // what this wave emptied is empty for everybody, ahead of its next slice
            if (t == 1) local = xcds.all_here();
        }
        f32x4 acc[2][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[0][g] = acc[1][g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < nks; ++ks) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
                acc[ks & 1][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_frag(wf[g][ks]), as_frag(f[ks >> 1]), acc[ks & 1][g], 0, 0, 0);
        }
        // acc[.][g][r] = partial sum of gate g, unit 4 lq + r, column lr; columns 0-7 are right for even k-steps, 8-15 for odd
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 v;
#pragma unroll
            for (int g = 0; g < 4; ++g) v[g] = rl_add_upper(acc[0][g][r], acc[1][g][r]);
            if (lr < 8) red[t & 1][wave][lr][4 * lq + r] = v;
        }
        if (!owner) in[t & 1][ct] = gx;
        lds_barrier();
        if (owner) {
            const f32x4 gi = in[t & 1][ct];
            f32x4       sum = red[t & 1][0][cr][cu];
#pragma unroll
            for (int q = 1; q < 4; ++q) sum += red[t & 1][q][cr][cu];
            float       gs[4];
            uint16_t    g16[4], h16;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                g16[g] = f2h((sum[g] + gi[g]) + bia[g]);  // the gate sum's one rounding to storage
                gs[g]  = h2f(g16[g]);
            }
            cst = lstm_cell_forward(gs[0], gs[1], gs[2], gs[3], cst, &h16);
            if (t + 1 < T) {
                const u32x4 piece = rl_gather8(h16);
                if ((cu & 7) == 0) {
                    rl_publish(ring, local, [&](auto store) {
                        store(piece, (t % RL_RING) * slot + pub);
                        if (t >= 2) store(u32x4{~0u, ~0u, ~0u, ~0u}, ((t - 2) % RL_RING) * slot + pub);
                    });
                }
            }
            out[t & 1][ct] = u32x4{(unsigned)g16[0] | ((unsigned)g16[1] << 16), (unsigned)g16[2] | ((unsigned)g16[3] << 16), h16, __float_as_uint(cst)};
            if (!local || np > RL_EAGER) __builtin_amdgcn_s_waitcnt(RL_VMCNT0);
        } else {
            if (t > 0 && cell) store_step(t - 1);
            if (t + 1 < T) load_gx(t + 1);
        }
        // (what lies in LDS under this parity is written again two steps on, behind this barrier)
        lds_barrier();
    }
    if (!owner && cell) store_step(T - 1);
}

// ------------------------------------------------------------------------------------------------ backward
struct LstmBwdArgs {
    int             T, B, I, H;
    long long       step_rows;
    const uint16_t* w;         // [4H, ldw]
    int             ldw;
    const uint16_t* gates;     // [T*step_rows, 4H]
    const float*    c;         // [(T+1)*step_rows, H]
    const uint16_t* dh_above;  // [T*step_rows, ld_above]: gradient reaching h_t from the layer above (or the loss)
    int             ld_above;
    uint16_t*       dgates;    // [T*step_rows, 4H] out
    RlSync          sync;
};
__host__ __device__ constexpr unsigned rl_bwd_slot(int H) { return 4u * 1024u * (H / 64); }

template <int HQ>
__global__ __launch_bounds__(RL_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_layer_bwd_kernel(LstmBwdArgs a) {
    __shared__ __align__(16) float red[2][4][RL_ROWS][16];  // per step parity and wave: partial recurrent gradients [row][unit]
    __shared__ __align__(16) char stage[4][1024];
    __shared__ RlCellIn in[RL_CELLS];
    __shared__ u32x2    out[2][RL_CELLS];  // per step parity: a cell's gate gradients (4 halves)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    constexpr int H = 64 * HQ;
    const int I = a.I, T = a.T;
    rl_empty_next(a.sync);
    const RlPlace place = rl_place(a.sync, H / RL_UNITS);
    const int j0  = place.unit_block * RL_UNITS;
    const int b0  = place.group * RL_ROWS;
    if (b0 >= a.B) return;
    const int nb  = min(RL_ROWS, a.B - b0);
    constexpr int nks = H / 32;            // this wave contracts over the H rows of gate block `wave`, 32 at a time
    constexpr int np  = nks / 2;
    constexpr unsigned slot = rl_bwd_slot(H);
    const __amdgpu_buffer_rsrc_t ring = rl_ring(a.sync.ring + (size_t)place.group * RL_RING * slot, RL_RING * slot);
    bool dead = false, local = false;
    RlXcds<H / RL_UNITS> xcds(a.sync, place, T);

    // W_h^T fragments: unit lr, 8 consecutive gate rows n = wave H + 32 ks + 8 lq ...: W[n][I + j0 + lr].  Read as row
    // pieces of 8 units, turned by the transposing LDS read (see gemm_dtl.hpp for its lane mapping): 32 rows at a time
    // through 1 KB of this wave's own LDS.
    u32x4 wt[nks];
#pragma unroll
    for (int ks = 0; ks < nks; ++ks)
        wt[ks] = *reinterpret_cast<const u32x4*>(a.w + (long long)(wave * H + 32 * ks + (lane >> 1)) * a.ldw + I + j0 + 8 * (lane & 1));
#pragma unroll
    for (int ks = 0; ks < nks; ++ks) {
        char* st = stage[wave];
        *reinterpret_cast<u32x4*>(st + (lane >> 1) * 32 + (lane & 1) * 16) = wt[ks];
        const char* rd = st + (8 * lq + (lr >> 2)) * 32 + (lr & 3) * 8;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)rd);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(rd + 4 * 32));
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        wt[ks]        = __builtin_bit_cast(u32x4, v);
    }

    const int  ct = tid & (RL_CELLS - 1), cr = ct >> 4, cu = ct & 15;  // (as in the forward kernel)
    const bool owner = tid < RL_CELLS, cell = cr < nb;
    const long long brow = b0 + min(cr, nb - 1);
    float      dc = 0.f, dhrec = 0.f;
    const int      pks = j0 >> 5, plq = ((j0 & 31) >> 3) + (cu >> 3);
    const unsigned pub = (pks >> 1) * 1024 + (plq * 16 + (pks & 1) * 8 + cr) * 16;  // + gate * np * 1024

    // waves 2 and 3: the inputs of a cell, two steps ahead
    RlCellIn next;
    auto     load_cell = [&](int t) {
        const long long row = t * a.step_rows + brow;
#pragma unroll
        for (int g = 0; g < 4; ++g) next.g[g] = a.gates[row * 4 * H + g * H + j0 + cu];
        next.cp = a.c[row * H + j0 + cu];
        next.cn = a.c[(row + a.step_rows) * H + j0 + cu];
        next.da = a.dh_above[row * a.ld_above + j0 + cu];
    };
    auto store_step = [&](int t) {
        const u32x2     r = out[t & 1][ct];
        uint16_t* const o = a.dgates + (t * a.step_rows + brow) * 4 * H + j0 + cu;
        o[0]     = (uint16_t)r[0];
        o[H]     = (uint16_t)(r[0] >> 16);
        o[2 * H] = (uint16_t)r[1];
        o[3 * H] = (uint16_t)(r[1] >> 16);
    };
    // waves 0 and 1: the activations of the next step's cell, which do not depend on the recurrence
    LstmCellAct act{};
    float       cp = 0.f, da = 0.f;
    auto        activate = [&] {
        const RlCellIn q = in[ct];
        act = lstm_cell_act(h2f((uint16_t)q.g[0]), h2f((uint16_t)q.g[1]), h2f((uint16_t)q.g[2]), h2f((uint16_t)q.g[3]), q.cn);
        cp  = q.cp;
        da  = h2f((uint16_t)q.da);
    };
    if (!owner) {
        load_cell(T - 1);
        in[ct] = next;
        if (T > 1) load_cell(T - 2);
    }
    lds_barrier();
    if (owner) activate();
    lds_barrier();  // (`in` is written again in the first step, ahead of its first barrier; in later steps the barrier behind `red` is between)

    for (int t = T - 1; t >= 0; --t) {
        const int n = T - 1 - t;  // number of the slice
        if (owner) {
            uint16_t d4[4];
            dc = lstm_cell_backward(act, cp, da + dhrec, dc, d4);
            if (t > 0) {
                u32x4 piece[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) piece[g] = rl_gather8(d4[g]);
                if ((cu & 7) == 0) {
                    rl_publish(ring, local, [&](auto store) {
#pragma unroll
                        for (int g = 0; g < 4; ++g) store(piece[g], (n % RL_RING) * slot + g * np * 1024 + pub);
                        if (n >= 2) {
#pragma unroll
                            for (int g = 0; g < 4; ++g) store(u32x4{~0u, ~0u, ~0u, ~0u}, ((n - 2) % RL_RING) * slot + g * np * 1024 + pub);
                        }
                    });
                }
            }
            out[t & 1][ct] = u32x2{(unsigned)d4[0] | ((unsigned)d4[1] << 16), (unsigned)d4[2] | ((unsigned)d4[3] << 16)};
            if (!local || np > RL_EAGER) __builtin_amdgcn_s_waitcnt(RL_VMCNT0);  // (as in the forward kernel)
        } else {
            if (t > 0) in[ct] = next;
            if (n > 0 && cell) store_step(t + 1);
            if (t >= 2) load_cell(t - 2);
        }
        lds_barrier();  // (nobody looks before the own slice is on its way, as in the forward kernel)
        if (t == 0) break;
        // recurrent gradient of this workgroup's units: dgates_t[rows, 4H] W_h[:, j0 .. j0+16)
        u32x4 f[np];
        rl_take<np, false>(ring, (n % RL_RING) * slot + wave * np * 1024 + lane * 16, true, f, a.sync, dead, [&] {
            if (n == 0) xcds.ask();
            if (owner) activate();
        });
        __builtin_amdgcn_s_waitcnt(RL_VMCNT0);  // (as in the forward kernel)
        if (n == 0) local = xcds.all_here();
        f32x4 acc[4];  // k-step ks into chain ks % 4
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < nks; ++ks)
            acc[ks & 3] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_frag(wt[ks]), as_frag(f[ks >> 1]), acc[ks & 3], 0, 0, 0);
        // acc[.][r] = partial sum for unit 4 lq + r, column lr; columns 0-7 are right for even k-steps, 8-15 for odd
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = rl_add_upper(acc[0][r] + acc[2][r], acc[1][r] + acc[3][r]);
        if (lr < 8) *reinterpret_cast<f32x4*>(&red[t & 1][wave][lr][4 * lq]) = v;
        lds_barrier();
        if (owner) {
            float s = red[t & 1][0][cr][cu];
#pragma unroll
            for (int q = 1; q < 4; ++q) s += red[t & 1][q][cr][cu];
            dhrec = round16(s);              // the recurrent gradient is a stored (fp16) tensor
        }
        // (`red` of this parity is written again two steps on, behind the next barriers)
    }
    if (!owner && cell) store_step(0);
}

}  // namespace mp

using namespace mp;

// f(std::integral_constant<int, H / 64>)
template <int HQ = 1, typename F>
static void rl_with_width(int H, F f) {
    if constexpr (HQ < RL_MAX_H / 64) {
        if (H > 64 * HQ) return rl_with_width<HQ + 1>(H, f);
    }
    f(std::integral_constant<int, HQ>{});
}

static int rl_groups(int B) { return (B + RL_ROWS - 1) / RL_ROWS; }

static int rl_check(const mp_lstm_layer_desc* d, const char* who, int* nwg) {
    MP_REQUIRE(d != nullptr, "%s: desc is NULL", who);
    MP_REQUIRE(d->T >= 1 && d->B >= 1 && d->I >= 0 && d->H >= 1, "%s: bad sizes T=%d B=%d I=%d H=%d", who, d->T, d->B, d->I, d->H);
    MP_REQUIRE(d->ldw >= d->I + d->H && d->ldxh >= d->I + d->H, "%s: leading dimension smaller than I + H", who);
    MP_REQUIRE(d->wait_limit_us >= 0 && d->debug_extra_participants >= 0 && d->debug_extra_participants <= 64,
               "%s: bad wait limit / debug participants", who);
    // (a caller that gives step_rows has asked mp_lstm_layer_desc_workspace_bytes for its workspace)
    const int rows = d->step_rows > 0 ? 0x7FFFFFFF : RL_MAX_B, unit = d->step_rows > 0 ? 64 : 128;
    if (d->B > rows || d->H % unit != 0 || d->H > RL_MAX_H || d->I % 8 != 0 || d->ldw % 8 != 0 || d->ldxh % 8 != 0) {
        set_error("%s: the persistent kernel needs H a multiple of %d up to %d, and I / ldw / ldxh multiples of 8, and without "
                  "step_rows B <= %d (got B=%d H=%d I=%d ldw=%d ldxh=%d); run the layer step by step instead", who, unit, RL_MAX_H,
                  RL_MAX_B, d->B, d->H, d->I, d->ldw, d->ldxh);
        return MP_E_UNSUPPORTED;
    }
    MP_REQUIRE(d->step_rows == 0 || d->step_rows >= d->B, "%s: step_rows=%d smaller than B=%d", who, d->step_rows, d->B);
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, who);
    *nwg = d->H / RL_UNITS;
    const int groups = rl_groups(d->B);
    if (*nwg * groups > 2 * cus) {  // every workgroup must be resident at once (two fit a compute unit), or no wait can end
        set_error("%s: %d workgroups needed, the device has %d compute units for two each", who, *nwg * groups, cus);
        return MP_E_UNSUPPORTED;
    }
    return MP_OK;
}

// Workgroups per XCD where every group goes on one XCD, as few groups on each as come out; 0 where one XCD does not hold them
// with a workgroup per compute unit (32).
static int rl_per_xcd(int units, int groups) {
    const int n = units * ((groups + 7) / 8);
    return n <= RL_XCD_WGS ? n : 0;
}
static dim3 rl_grid(const RlSync& s, int units, int groups) { return dim3(s.per_xcd > 0 ? 8 * s.per_xcd : units * groups); }

// the exchange rings: one per block of batch rows, backward slices being the larger ones
// (16 bytes more than they hold, so that a workspace at any 4-byte boundary has room for them at a 16-byte one)
static size_t rl_xcds_bytes(int units, int groups) { return rl_per_xcd(units, groups) > 0 ? (size_t)groups * 4 * RL_XCD_WGS : 0; }
static size_t rl_rings(int B, int H) { return (size_t)rl_groups(B) * RL_RING * rl_bwd_slot(H) + 16; }
extern "C" size_t mp_lstm_layer_workspace_bytes(void) { return rl_rings(RL_MAX_B, RL_MAX_H); }
extern "C" size_t mp_lstm_layer_desc_workspace_bytes(const mp_lstm_layer_desc* d) {
    return d && d->B > 0 && d->H > 0 && d->H % 64 == 0 && d->H <= RL_MAX_H ? rl_rings(d->B, d->H) + rl_xcds_bytes(d->H / RL_UNITS, rl_groups(d->B)) : 0;
}

static uintptr_t align_up16(const void* p) { return (reinterpret_cast<uintptr_t>(p) + 15) & ~(uintptr_t)15; }

// place: groups on one XCD each where one holds them (see the *_placed calls in mp.h for what that asks of the caller).  Where the
// groups come out even over the 8 XCDs that asks for nothing: each has as many workgroups as if the ids went round them.
static int rl_sync(const mp_lstm_layer_desc* d, unsigned slot, int32_t* status, void* ws, size_t ws_bytes, int ws_is_empty,
                   void* next_ws, size_t next_ws_bytes, bool place, mp_stream stream, const char* who, RlSync* out) {
    MP_REQUIRE(status != nullptr, "%s: status is NULL", who);
    const size_t need = d->step_rows > 0 ? rl_rings(d->B, d->H) : mp_lstm_layer_workspace_bytes();
    if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 3u)) {
        set_error("%s: 4-byte aligned workspace of %zu bytes needed, %zu given", who, need, ws_bytes);
        return MP_E_WORKSPACE;
    }
    if (next_ws != nullptr) {
        const char *a = static_cast<const char*>(ws), *b = static_cast<const char*>(next_ws);
        MP_REQUIRE((reinterpret_cast<uintptr_t>(next_ws) & 3u) == 0 && next_ws_bytes >= 16 && next_ws_bytes < (1ull << 32) &&
                       (b + next_ws_bytes <= a || a + ws_bytes <= b),
                   "%s: next_ws has to be a 4-byte aligned workspace apart from ws", who);
        out->next        = reinterpret_cast<u32x4*>(align_up16(next_ws));
        out->next_pieces = (unsigned)((next_ws_bytes - (align_up16(next_ws) - reinterpret_cast<uintptr_t>(next_ws))) / 16);
    }
    char* const  ring = reinterpret_cast<char*>(align_up16(ws));
    const int    units = d->H / RL_UNITS, groups = rl_groups(d->B);
    if (groups % 8 == 0) place = true;
    const size_t used = (size_t)groups * RL_RING * slot, xcds = place ? rl_xcds_bytes(units, groups) : 0;
    out->per_xcd   = place ? rl_per_xcd(units, groups) : 0;
    out->first_xcd = (int)(((unsigned)(reinterpret_cast<uintptr_t>(ring) >> 8) * 0x9E3779B1u) >> 29);  // (several models of one group: not all on XCD 0)
    // (a workspace that holds the rings alone will do: the group's stores then go to the whole device)
    out->xcds = xcds > 0 && ws_bytes - (size_t)(ring - static_cast<char*>(ws)) >= used + xcds ? ring + used : nullptr;
    if (!ws_is_empty) {
        const int rc = mp_fill_u32((used + (out->xcds ? xcds : 0)) / 4, ~0u, ring, stream);  // everything starts empty (a kernel: capturable)
        if (rc != MP_OK) return rc;
    }
    out->ring        = ring;
    out->status      = status;
    out->never       = d->debug_extra_participants > 0;
    out->limit_ticks = (d->wait_limit_us > 0 ? (long long)d->wait_limit_us : 2000000ll) * 100;  // 100 MHz clock
    return MP_OK;
}

static int rl_fwd(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias, mp_half* gates, float* c,
                  mp_half* xh, mp_half* h_up, int32_t* status, void* ws, size_t ws_bytes, int ws_is_empty, void* next_ws,
                  size_t next_ws_bytes, bool place, mp_stream stream) {
    int nwg = 0;
    int rc  = rl_check(d, "mp_lstm_layer_fwd", &nwg);
    if (rc) return rc;
    MP_REQUIRE(gx && w && bias && gates && c && xh, "mp_lstm_layer_fwd: NULL argument");
    MP_REQUIRE(h_up == nullptr || (d->ld_up >= d->H && d->ld_up % 2 == 0), "mp_lstm_layer_fwd: ld_up=%d must be even and >= H", d->ld_up);
    MP_REQUIRE(aligned16(w) && aligned16(xh) && aligned16(gx) && aligned16(gates) && aligned16(c) && (h_up == nullptr || aligned16(h_up)),
               "mp_lstm_layer_fwd: pointers must be 16-byte aligned");
    LstmFwdArgs a{};
    rc = rl_sync(d, rl_fwd_slot(d->H), status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, place, stream, "mp_lstm_layer_fwd", &a.sync);
    if (rc) return rc;
    a.T = d->T; a.B = d->B; a.I = d->I; a.H = d->H; a.step_rows = d->step_rows > 0 ? d->step_rows : d->B;
    a.gx = gx; a.w = w; a.ldw = d->ldw; a.bias = bias; a.gates = gates; a.c = c; a.xh = xh; a.ldxh = d->ldxh;
    a.h_up = h_up; a.ld_up = d->ld_up;
    rl_with_width(d->H, [&](auto hb) {
        hipLaunchKernelGGL(lstm_layer_fwd_kernel<decltype(hb)::value>, rl_grid(a.sync, nwg, rl_groups(d->B)), dim3(RL_THREADS), 0, as_stream(stream), a);
    });
    MP_LAUNCH_CHECK("mp_lstm_layer_fwd");
    return MP_OK;
}

static int rl_bwd(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c, const mp_half* dh_above,
                  mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes, int ws_is_empty, void* next_ws,
                  size_t next_ws_bytes, bool place, mp_stream stream) {
    int nwg = 0;
    int rc  = rl_check(d, "mp_lstm_layer_bwd", &nwg);
    if (rc) return rc;
    MP_REQUIRE(w && gates && c && dh_above && dgates, "mp_lstm_layer_bwd: NULL argument");
    MP_REQUIRE(d->ld_up >= d->H && d->ld_up % 2 == 0, "mp_lstm_layer_bwd: ld_up=%d (leading dimension of dh_above) must be even and >= H", d->ld_up);
    MP_REQUIRE(aligned16(w) && aligned16(gates) && aligned16(c) && aligned16(dh_above) && aligned16(dgates),
               "mp_lstm_layer_bwd: pointers must be 16-byte aligned");
    LstmBwdArgs a{};
    rc = rl_sync(d, rl_bwd_slot(d->H), status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, place, stream, "mp_lstm_layer_bwd", &a.sync);
    if (rc) return rc;
    a.T = d->T; a.B = d->B; a.I = d->I; a.H = d->H; a.step_rows = d->step_rows > 0 ? d->step_rows : d->B;
    a.w = w; a.ldw = d->ldw; a.gates = gates; a.c = c; a.dh_above = dh_above; a.ld_above = d->ld_up; a.dgates = dgates;
    rl_with_width(d->H, [&](auto hb) {
        hipLaunchKernelGGL(lstm_layer_bwd_kernel<decltype(hb)::value>, rl_grid(a.sync, nwg, rl_groups(d->B)), dim3(RL_THREADS), 0, as_stream(stream), a);
    });
    MP_LAUNCH_CHECK("mp_lstm_layer_bwd");
    return MP_OK;
}

extern "C" int mp_lstm_layer_fwd(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias,
                                 mp_half* gates, float* c, mp_half* xh, mp_half* h_up, int32_t* status, void* ws,
                                 size_t ws_bytes, mp_stream stream) {
    return rl_fwd(d, gx, w, bias, gates, c, xh, h_up, status, ws, ws_bytes, 0, nullptr, 0, false, stream);
}

extern "C" int mp_lstm_layer_fwd_chain(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias,
                                       mp_half* gates, float* c, mp_half* xh, mp_half* h_up, int32_t* status, void* ws,
                                       size_t ws_bytes, int ws_is_empty, void* next_ws, size_t next_ws_bytes,
                                       mp_stream stream) {
    return rl_fwd(d, gx, w, bias, gates, c, xh, h_up, status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, false, stream);
}

extern "C" int mp_lstm_layer_fwd_placed(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias,
                                        mp_half* gates, float* c, mp_half* xh, mp_half* h_up, int32_t* status, void* ws,
                                        size_t ws_bytes, int ws_is_empty, void* next_ws, size_t next_ws_bytes,
                                        mp_stream stream) {
    return rl_fwd(d, gx, w, bias, gates, c, xh, h_up, status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, true, stream);
}

extern "C" int mp_lstm_layer_bwd(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c,
                                 const mp_half* dh_above, mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes,
                                 mp_stream stream) {
    return rl_bwd(d, w, gates, c, dh_above, dgates, status, ws, ws_bytes, 0, nullptr, 0, false, stream);
}

extern "C" int mp_lstm_layer_bwd_chain(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c,
                                       const mp_half* dh_above, mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes,
                                       int ws_is_empty, void* next_ws, size_t next_ws_bytes, mp_stream stream) {
    return rl_bwd(d, w, gates, c, dh_above, dgates, status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, false, stream);
}

extern "C" int mp_lstm_layer_bwd_placed(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c,
                                        const mp_half* dh_above, mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes,
                                        int ws_is_empty, void* next_ws, size_t next_ws_bytes, mp_stream stream) {
    return rl_bwd(d, w, gates, c, dh_above, dgates, status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, true, stream);
}
