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
// (4 layers x 50 steps, 1024 units, batch 32, us per time step: one flag per workgroup behind a device-scope release and
// acquire, 16 rows per workgroup: 6.7 forward, 10.0 backward; now 2.2 and 2.8.)
// All workgroups must be co-resident: the register use allows two per compute unit and the host refuses larger grids.
// Every wait is bounded in wall-clock time; a wave that gives up raises *status and stops waiting, which makes every other
// wave give up too, and all of them walk the remaining steps without waiting: the grid always drains.
#include "cell_math.hpp"
#include "common.hpp"

#include <type_traits>

namespace mp {

constexpr int RL_THREADS = 256;  // 4 waves: each takes a quarter of the contraction
constexpr int RL_UNITS   = 16;   // hidden units per workgroup = one 16-row matrix-core block per gate
constexpr int RL_ROWS    = 8;    // batch rows per workgroup; more rows: more workgroups (grid y)
constexpr int RL_MAX_H   = 1024; // register budget of the fragment arrays below
constexpr int RL_MAX_B   = 32;
constexpr int RL_RING    = 4;    // slots of the exchange ring
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
};
// A launch's ring has to be empty before it starts: a fill launch (5 us of a captured chain, of the 46 to 130 us that the
// recurrent kernels take) unless the launch ahead has done it, one or a few stores per thread that nothing waits for.
__device__ __forceinline__ void rl_empty_next(const RlSync& s) {
    for (unsigned i = (blockIdx.y * gridDim.x + blockIdx.x) * RL_THREADS + threadIdx.x; i < s.next_pieces;
         i += gridDim.x * gridDim.y * RL_THREADS)
        s.next[i] = u32x4{~0u, ~0u, ~0u, ~0u};
}

constexpr int RL_DEVICE_SCOPE = 16;  // cache-policy bit (sc1) of the buffer intrinsics: coherent across the device
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rl_ring(char* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}

// The NP fragment pairs (1 KB apart) of a published slice, loaded until nothing in them is empty.  GUARD_LAST: lanes
// without last_ok never get anything in the last pair (it reads as zero there).  Waves decide alone; `dead` (wave-uniform) is set when this
// or another wave gave up, and ends all waiting.
template <int NP, bool GUARD_LAST>
__device__ __forceinline__ void rl_take(__amdgpu_buffer_rsrc_t ring, unsigned off, bool last_ok, u32x4 (&f)[NP],
                                        const RlSync& s, bool& dead) {
    long long  t0    = 0;
    for (int it = 0;; ++it) {
        asm volatile("" ::: "memory");  // (every round loads anew)
#pragma unroll
        for (int p = 0; p < NP; ++p) f[p] = __builtin_amdgcn_raw_buffer_load_b128(ring, off + p * 1024, 0, RL_DEVICE_SCOPE);
        if (GUARD_LAST && !last_ok) f[NP - 1] = u32x4{0u, 0u, 0u, 0u};
        u16x2 m = {0, 0};  // the largest half seen: RL_EMPTY is the largest pattern there is
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned x = f[p][w];
                m                = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, x));
            }
        }
        const bool missing = m[0] == RL_EMPTY || m[1] == RL_EMPTY || s.never != 0;
        if (dead || !__any(missing)) return;
        if ((it & 15) == 0) {
            const long long now = wall_clock64();
            if (it == 0) t0 = now;
            const int give_up = (now - t0 > s.limit_ticks) ||
                                __hip_atomic_load(s.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            if (__any(give_up)) {  // (lanes read the clock a few ticks apart: the wave decides as one)
                dead = true;
                if ((threadIdx.x & 63) == 0) atomicOr(s.status, 1);
            }
        }
    }
}

// x of this lane (lanes 0-7 of each 16) plus y of the lane 8 further on
__device__ __forceinline__ float rl_add_upper(float x, float y) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), 0x108, 0xF, 0xF, true));
}

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
    __shared__ __align__(16) float red[2][4][RL_ROWS][80];  // per step parity and wave: partial gate sums [row][16 g + unit] (row stride: 64 banks + 16)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    constexpr int H = 64 * HQ;
    const int I = a.I, T = a.T;
    const int j0  = blockIdx.x * RL_UNITS;   // this workgroup's hidden units
    const int b0  = blockIdx.y * RL_ROWS;    // ... and batch rows
    const int nb  = min(RL_ROWS, a.B - b0);
    constexpr int nks = rl_fwd_steps(H), np = rl_fwd_pairs(H);
    constexpr int each = H / 32 / 4, more = H / 32 % 4;    // k-steps of every wave; that many waves have one more
    const int mine = each + (wave < more ? 1 : 0);
    const int k0   = 32 * (wave * each + min(wave, more)) + 8 * lq;  // first k of this lane's 8 consecutive values, + 32 ks
    const bool last_ok = 2 * (np - 1) + (lr >> 3) < mine;            // this lane's k-step of the last pair exists
    constexpr unsigned slot = rl_fwd_slot(H);
    const __amdgpu_buffer_rsrc_t ring = rl_ring(a.sync.ring + (size_t)blockIdx.y * RL_RING * slot, RL_RING * slot);
    bool dead = false;
    rl_empty_next(a.sync);

    // W_h fragments, resident for the whole sequence: gate g, unit lr, 8 consecutive k
    u32x4 wf[4][nks];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int ks = 0; ks < nks; ++ks) {
            wf[g][ks] = u32x4{0u, 0u, 0u, 0u};
            if (more == 0 || ks < mine) wf[g][ks] = *reinterpret_cast<const u32x4*>(a.w + (long long)(g * H + j0 + lr) * a.ldw + I + k0 + 32 * ks);
        }

    // cell ownership (waves 0 and 1): thread -> batch row b0 + cr, unit j0 + cu.  Rows beyond the batch repeat the last one
    // (their values are published but never stored), so that no load hangs on a condition.
    const int  cr = tid >> 4, cu = tid & 15;
    const bool owner = cr < RL_ROWS, cell = cr < nb;
    const long long brow = b0 + min(cr, nb - 1);
    float    cst = 0.f, bia[4] = {0.f, 0.f, 0.f, 0.f}, gx0[4], gx1[4];
    uint16_t g16[4] = {0, 0, 0, 0}, h16 = 0;
    auto     load_gx = [&](int t, float (&gx)[4]) {
#pragma unroll
        for (int g = 0; g < 4; ++g) gx[g] = a.gx[(t * a.step_rows + brow) * 4 * H + g * H + j0 + cu];
    };
    if (owner) {
#pragma unroll
        for (int g = 0; g < 4; ++g) bia[g] = h2f(a.bias[g * H + j0 + cu]);
        cst = a.c[brow * H + j0 + cu];
        load_gx(0, gx0);
    }
    auto store_step = [&](int t) {  // what step t leaves in memory
        const long long row = t * a.step_rows + brow;
#pragma unroll
        for (int g = 0; g < 4; ++g) a.gates[row * 4 * H + g * H + j0 + cu] = g16[g];
        a.c[(row + a.step_rows) * H + j0 + cu] = cst;
        if (t + 1 < T) a.xh[(row + a.step_rows) * a.ldxh + I + j0 + cu] = h16;
        if (a.h_up != nullptr) a.h_up[row * a.ld_up + j0 + cu] = h16;
    };
    // where this workgroup's units lie in a slot: fragment pair, k-step of the pair, and the lane rows of its two 8-unit pieces
    const int      jks = j0 >> 5, jw = jks < more * (each + 1) ? jks / (each + 1) : (each > 0 ? (jks - more) / (each > 0 ? each : 1) : 0);
    const int      pks = jks - (jw * each + min(jw, more)), plq = ((j0 & 31) >> 3) + (cu >> 3);
    const unsigned pub = (jw * np + (pks >> 1)) * 1024 + (plq * 16 + (pks & 1) * 8 + cr) * 16;

    // gx: the input half of this step's gate sums, gxn: of the next step's.
    // Order of the memory instructions: a slice is published ahead of everything else of its step, and the workgroup looks
    // for the others' only when its own is acknowledged: polling loads queue ahead of stores on their way out and keep
    // invalidated lines moving between the caches (both kernels 25-30 % slower with waves that poll from the start).
    // Results and the next inputs follow, and their latency runs under the flight of the slices.
    auto step = [&](const int t, const float (&gx)[4], float (&gxn)[4]) {
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
            rl_take<np, (more != 0 || (nks & 1) != 0)>(ring, ((t - 1) % RL_RING) * slot + wave * np * 1024 + lane * 16, last_ok, f, a.sync, dead);
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
        for (int g = 0; g < 4; ++g) {
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = rl_add_upper(acc[0][g][r], acc[1][g][r]);
            if (lr < 8) *reinterpret_cast<f32x4*>(&red[t & 1][wave][lr][16 * g + 4 * lq]) = v;
        }
        lds_barrier();
        if (owner) {
            float gs[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = 16 * g + cu;
                float     s = red[t & 1][0][cr][n];
#pragma unroll
                for (int q = 1; q < 4; ++q) s += red[t & 1][q][cr][n];
                g16[g] = f2h((s + gx[g]) + bia[g]);  // the gate sum's one rounding to storage
                gs[g]  = h2f(g16[g]);
            }
            cst = lstm_cell_forward(gs[0], gs[1], gs[2], gs[3], cst, &h16);
            if (t + 1 < T) {
                const u32x4 piece = rl_gather8(h16);
                if ((cu & 7) == 0) {
                    __builtin_amdgcn_raw_buffer_store_b128(piece, ring, (t % RL_RING) * slot + pub, 0, RL_DEVICE_SCOPE);
                    if (t >= 2)
                        __builtin_amdgcn_raw_buffer_store_b128(u32x4{~0u, ~0u, ~0u, ~0u}, ring, ((t - 2) % RL_RING) * slot + pub, 0,
                                                               RL_DEVICE_SCOPE);
                }
            }
            // acknowledged: also what was emptied is empty for everybody, ahead of this workgroup's next slice
            __builtin_amdgcn_s_waitcnt(RL_VMCNT0);
        }
        // (`red` of this parity is written again two steps on, behind this barrier)
        lds_barrier();
        if (cell) store_step(t);
        if (owner && t + 1 < T) load_gx(t + 1, gxn);
    };
    for (int t = 0; t < T; t += 2) {
        step(t, gx0, gx1);
        if (t + 1 < T) step(t + 1, gx1, gx0);
    }
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
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    constexpr int H = 64 * HQ;
    const int I = a.I, T = a.T;
    const int j0  = blockIdx.x * RL_UNITS;
    const int b0  = blockIdx.y * RL_ROWS;
    const int nb  = min(RL_ROWS, a.B - b0);
    constexpr int nks = H / 32;            // this wave contracts over the H rows of gate block `wave`, 32 at a time
    constexpr int np  = nks / 2;
    constexpr unsigned slot = rl_bwd_slot(H);
    const __amdgpu_buffer_rsrc_t ring = rl_ring(a.sync.ring + (size_t)blockIdx.y * RL_RING * slot, RL_RING * slot);
    bool dead = false;
    rl_empty_next(a.sync);

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

    const int  cr = tid >> 4, cu = tid & 15;  // (as in the forward kernel)
    const bool owner = cr < RL_ROWS, cell = cr < nb;
    const long long brow = b0 + min(cr, nb - 1);
    float      dc = 0.f, dhrec = 0.f;
    const int      pks = j0 >> 5, plq = ((j0 & 31) >> 3) + (cu >> 3);
    const unsigned pub = (pks >> 1) * 1024 + (plq * 16 + (pks & 1) * 8 + cr) * 16;  // + gate * np * 1024

    // inputs of one cell-backward step for this thread's cell (they do not depend on the recurrence: requested two steps
    // ahead)
    struct CellIn {
        uint16_t gp[4], da;
        float    cp, cn;
    };
    auto load_cell = [&](int t, CellIn& q) {
        const long long row = t * a.step_rows + brow;
#pragma unroll
        for (int g = 0; g < 4; ++g) q.gp[g] = a.gates[row * 4 * H + g * H + j0 + cu];
        q.cp = a.c[row * H + j0 + cu];
        q.cn = a.c[(row + a.step_rows) * H + j0 + cu];
        q.da = a.dh_above[row * a.ld_above + j0 + cu];
    };
    CellIn in0, in1;
    if (owner) {
        load_cell(T - 1, in0);
        if (T > 1) load_cell(T - 2, in1);
    }

    auto step = [&](const int t, CellIn& in) {
        const int n = T - 1 - t;  // number of the slice
        uint16_t  d4[4] = {0, 0, 0, 0};
        auto      store_step = [&] {
            uint16_t* o = a.dgates + (t * a.step_rows + brow) * 4 * H + j0 + cu;
#pragma unroll
            for (int g = 0; g < 4; ++g) o[g * H] = d4[g];
        };
        if (owner) {
            dc = lstm_cell_backward(h2f(in.gp[0]), h2f(in.gp[1]), h2f(in.gp[2]), h2f(in.gp[3]), in.cp, in.cn, h2f(in.da) + dhrec, dc, d4);
            if (t > 0) {
                u32x4 piece[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) piece[g] = rl_gather8(d4[g]);
                if ((cu & 7) == 0) {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        __builtin_amdgcn_raw_buffer_store_b128(piece[g], ring, (n % RL_RING) * slot + g * np * 1024 + pub, 0, RL_DEVICE_SCOPE);
                    if (n >= 2) {
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            __builtin_amdgcn_raw_buffer_store_b128(u32x4{~0u, ~0u, ~0u, ~0u}, ring,
                                                                   ((n - 2) % RL_RING) * slot + g * np * 1024 + pub, 0, RL_DEVICE_SCOPE);
                    }
                }
            }
        }
        if (t == 0) {
            if (cell) store_step();
            return;
        }
        if (owner) __builtin_amdgcn_s_waitcnt(RL_VMCNT0);  // (as in the forward kernel)
        lds_barrier();  // (nobody looks before the own slice is on its way, as in the forward kernel)
        if (cell) store_step();
        if (owner && t >= 2) load_cell(t - 2, in);
        // recurrent gradient of this workgroup's units: dgates_t[rows, 4H] W_h[:, j0 .. j0+16)
        u32x4 f[np];
        rl_take<np, false>(ring, (n % RL_RING) * slot + wave * np * 1024 + lane * 16, true, f, a.sync, dead);
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
    };
    for (int t = T - 1; t >= 0; t -= 2) {
        step(t, in0);
        if (t >= 1) step(t - 1, in1);
    }
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
    const int groups = (d->B + RL_ROWS - 1) / RL_ROWS;
    if (*nwg * groups > 2 * cus) {  // every workgroup must be resident at once (two fit a compute unit), or no wait can end
        set_error("%s: %d workgroups needed, the device has %d compute units for two each", who, *nwg * groups, cus);
        return MP_E_UNSUPPORTED;
    }
    return MP_OK;
}

// the exchange rings: one per block of batch rows, backward slices being the larger ones
// (16 bytes more than they hold, so that a workspace at any 4-byte boundary has room for them at a 16-byte one)
static size_t rl_rings(int B, int H) { return (size_t)((B + RL_ROWS - 1) / RL_ROWS) * RL_RING * rl_bwd_slot(H) + 16; }
extern "C" size_t mp_lstm_layer_workspace_bytes(void) { return rl_rings(RL_MAX_B, RL_MAX_H); }
extern "C" size_t mp_lstm_layer_desc_workspace_bytes(const mp_lstm_layer_desc* d) {
    return d && d->B > 0 && d->H > 0 && d->H % 64 == 0 && d->H <= RL_MAX_H ? rl_rings(d->B, d->H) : 0;
}

static uintptr_t align_up16(const void* p) { return (reinterpret_cast<uintptr_t>(p) + 15) & ~(uintptr_t)15; }

static int rl_sync(const mp_lstm_layer_desc* d, unsigned slot, int32_t* status, void* ws, size_t ws_bytes, int ws_is_empty,
                   void* next_ws, size_t next_ws_bytes, mp_stream stream, const char* who, RlSync* out) {
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
    const size_t used = (size_t)((d->B + RL_ROWS - 1) / RL_ROWS) * RL_RING * slot;
    if (!ws_is_empty) {
        const int rc = mp_fill_u32(used / 4, ~0u, ring, stream);  // everything starts empty (a kernel: capturable)
        if (rc != MP_OK) return rc;
    }
    out->ring        = ring;
    out->status      = status;
    out->never       = d->debug_extra_participants > 0;
    out->limit_ticks = (d->wait_limit_us > 0 ? (long long)d->wait_limit_us : 2000000ll) * 100;  // 100 MHz clock
    return MP_OK;
}

extern "C" int mp_lstm_layer_fwd(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias,
                                 mp_half* gates, float* c, mp_half* xh, mp_half* h_up, int32_t* status, void* ws,
                                 size_t ws_bytes, mp_stream stream) {
    return mp_lstm_layer_fwd_chain(d, gx, w, bias, gates, c, xh, h_up, status, ws, ws_bytes, 0, nullptr, 0, stream);
}

extern "C" int mp_lstm_layer_fwd_chain(const mp_lstm_layer_desc* d, const float* gx, const mp_half* w, const mp_half* bias,
                                       mp_half* gates, float* c, mp_half* xh, mp_half* h_up, int32_t* status, void* ws,
                                       size_t ws_bytes, int ws_is_empty, void* next_ws, size_t next_ws_bytes,
                                       mp_stream stream) {
    int nwg = 0;
    int rc  = rl_check(d, "mp_lstm_layer_fwd", &nwg);
    if (rc) return rc;
    MP_REQUIRE(gx && w && bias && gates && c && xh, "mp_lstm_layer_fwd: NULL argument");
    MP_REQUIRE(h_up == nullptr || (d->ld_up >= d->H && d->ld_up % 2 == 0), "mp_lstm_layer_fwd: ld_up=%d must be even and >= H", d->ld_up);
    MP_REQUIRE(aligned16(w) && aligned16(xh) && aligned16(gx) && aligned16(gates) && aligned16(c) && (h_up == nullptr || aligned16(h_up)),
               "mp_lstm_layer_fwd: pointers must be 16-byte aligned");
    LstmFwdArgs a{};
    rc = rl_sync(d, rl_fwd_slot(d->H), status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, stream, "mp_lstm_layer_fwd", &a.sync);
    if (rc) return rc;
    a.T = d->T; a.B = d->B; a.I = d->I; a.H = d->H; a.step_rows = d->step_rows > 0 ? d->step_rows : d->B;
    a.gx = gx; a.w = w; a.ldw = d->ldw; a.bias = bias; a.gates = gates; a.c = c; a.xh = xh; a.ldxh = d->ldxh;
    a.h_up = h_up; a.ld_up = d->ld_up;
    rl_with_width(d->H, [&](auto hb) {
        hipLaunchKernelGGL(lstm_layer_fwd_kernel<decltype(hb)::value>, dim3(nwg, (d->B + RL_ROWS - 1) / RL_ROWS), dim3(RL_THREADS), 0, as_stream(stream), a);
    });
    MP_LAUNCH_CHECK("mp_lstm_layer_fwd");
    return MP_OK;
}

extern "C" int mp_lstm_layer_bwd(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c,
                                 const mp_half* dh_above, mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes,
                                 mp_stream stream) {
    return mp_lstm_layer_bwd_chain(d, w, gates, c, dh_above, dgates, status, ws, ws_bytes, 0, nullptr, 0, stream);
}

extern "C" int mp_lstm_layer_bwd_chain(const mp_lstm_layer_desc* d, const mp_half* w, const mp_half* gates, const float* c,
                                       const mp_half* dh_above, mp_half* dgates, int32_t* status, void* ws, size_t ws_bytes,
                                       int ws_is_empty, void* next_ws, size_t next_ws_bytes, mp_stream stream) {
    int nwg = 0;
    int rc  = rl_check(d, "mp_lstm_layer_bwd", &nwg);
    if (rc) return rc;
    MP_REQUIRE(w && gates && c && dh_above && dgates, "mp_lstm_layer_bwd: NULL argument");
    MP_REQUIRE(d->ld_up >= d->H && d->ld_up % 2 == 0, "mp_lstm_layer_bwd: ld_up=%d (leading dimension of dh_above) must be even and >= H", d->ld_up);
    MP_REQUIRE(aligned16(w) && aligned16(gates) && aligned16(c) && aligned16(dh_above) && aligned16(dgates),
               "mp_lstm_layer_bwd: pointers must be 16-byte aligned");
    LstmBwdArgs a{};
    rc = rl_sync(d, rl_bwd_slot(d->H), status, ws, ws_bytes, ws_is_empty, next_ws, next_ws_bytes, stream, "mp_lstm_layer_bwd", &a.sync);
    if (rc) return rc;
    a.T = d->T; a.B = d->B; a.I = d->I; a.H = d->H; a.step_rows = d->step_rows > 0 ? d->step_rows : d->B;
    a.w = w; a.ldw = d->ldw; a.gates = gates; a.c = c; a.dh_above = dh_above; a.ld_above = d->ld_up; a.dgates = dgates;
    rl_with_width(d->H, [&](auto hb) {
        hipLaunchKernelGGL(lstm_layer_bwd_kernel<decltype(hb)::value>, dim3(nwg, (d->B + RL_ROWS - 1) / RL_ROWS), dim3(RL_THREADS), 0, as_stream(stream), a);
    });
    MP_LAUNCH_CHECK("mp_lstm_layer_bwd");
    return MP_OK;
}
