// Contraction kernel whose operand tiles go from global memory straight into LDS (`buffer_load ... lds`: no staging
// registers, no LDS store instructions), for products whose rows are 16-byte aligned and whose contraction is a multiple of 8
// (any, where both operands are output-contiguous).  Same arithmetic as gemm_kernels.hpp (paper Section 3.1: fp16 operands,
// fp32 sums, one rounding); what differs is how the operands reach the matrix cores and how the results leave them.
//
// What bounds it.  Under a full-chip load the matrix cores' clock follows the power that the operands draw, so both the
// issue slots and the energy per flop count:
//   * v_mfma_f32_16x16x32_f16 and not 32x32x16: with N(0,1) operands in registers and nothing else the chip sustains 1.90
//     PFLOP/s with the former and 1.65 with the latter (the wide one reads and writes twice the accumulator data per flop).
//   * a wave owns its SIMD (128 x 128 of a 256 x 256 tile in 256 accumulators), so every other instruction has to fit between
//     two matrix-core instructions, which leave three issue slots each.  A load is one scalar add that sets M0 (the LDS
//     destination) and, one matrix-core instruction later, the load; the loads are spread evenly over a k-tile.  Issued in
//     clumps of four instructions they cost 11 % (8192^3, all-zero operands: 604 us, spread 545, no loads at all 485).
//   * loads need time: each has at least 96 of a k-tile's 128 matrix-core instructions (about 1 us) to arrive.  A k-tile is
//     worked on in two PHASES, the upper and then the lower half of every wave's rows, and not in two slices of the
//     contraction: the second operand's and the upper rows' LDS space is then free a quarter into the k-tile and takes the
//     loads of the k-tile after next, the lower rows' space half a k-tile later.  Two stages of 64 KB behave like three that
//     way (two stages worked on slice by slice, which free their space half a k-tile late: 730 us on zeros, 545 this way;
//     five stages of 32 k, whose rows are half a cache line: 648).
//   us, this kernel / the register-staged one / the vendor library, N(0,1) operands on one card: 8192^3 764 / 868 / 739;
//   8192 x 4096 over 1024 62 / 71 / 60; 8192 x 1024 over 4096 58.7 / 68 / 65; input gradient 8192 x 1024 over 3072 45.6 / 56 / 52.
//
// LDS layout.  A wave load deposits 64 lanes x 16 bytes contiguously, so the layout is chosen by choosing which piece each
// lane fetches:
//   contraction-contiguous operand ([row][k]): rows of 64 k = 128 bytes = 8 pieces, a whole cache line; piece s of row r sits
//     in slot s ^ ((r >> 1) & 7), which spreads the 16 rows of a fragment read over all banks;
//   output-contiguous operand ([k][row]): LDS keeps the global orientation; the 16-byte piece p (8 rows) of k-row k sits at
//     piece p ^ k_slot(k).  Fragments come out of it with the transposing LDS read (`ds_read_b64_tr_b16`): within 16
//     lanes, lane i receives element i % 4 of the 8-byte chunks addressed by lanes i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4, so
//     four lanes that address the same k and four consecutive 4-row groups hand every lane of the 16 its own row at 4
//     consecutive k.  Two such reads make the 8-k fragment of an instruction.
// The first operand's rows come in two units, the upper halves of both wave rows and then the lower ones.
#pragma once
#include "gemm_kernels.hpp"

namespace mp {

#define MP_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int    dtl_stage(int bm, int bn) { return (bm + bn) * 128; }            // LDS bytes of one k-tile
constexpr int    dtl_out_pitch(int wn) { return wn > 64 ? 256 : 128; }            // bytes of an output row on its way out
constexpr int    dtl_out_bytes(int wn) { return 16 * dtl_out_pitch(wn); }         // of one wave
constexpr size_t dtl_lds(int bm, int bn) { return 2 * (size_t)dtl_stage(bm, bn) + 4 * dtl_out_bytes(bn / 2); }

// One operand (R tile rows, WR of them per wave).  SPLIT: LDS rows come in two units, the first WR/2 rows of every wave's
// block and then the others.  GUARD: rows may lie outside the matrix (see rsrc below).
template <int R, int WR, bool KC, bool SPLIT, bool GUARD>
struct DtlOperand {
    static_assert(R % 64 == 0 && (KC || R == 64 || R == 128 || R == 256), "tile edge");
    static constexpr int BYTES = R * 128;             // one k-tile: R rows x 64 k x 2 bytes
    static constexpr int NL    = R / 32;              // loads per wave and k-tile (1 KB each)
    static constexpr int UR    = SPLIT ? R / 2 : R;   // rows of a unit
    static constexpr int KR    = KC ? 1 : 512 / UR;   // output-contiguous: k-rows per load ...
    static constexpr int RB    = 2 * UR;              // ... and bytes of a k-row
    unsigned voff[GUARD ? NL : 1];                    // this lane's byte offset from the k-tile's origin, load q (INTERIOR: load 0)
    unsigned ld;
    int      piece;                                   // contraction-contiguous: which piece of a k-tile's row this lane fetches
    int      foff[KC ? 1 : 4];                        // fragment read offsets

    // output-contiguous: what a k-row's piece numbers are XOR-ed with, so that the 4 k-rows x 32 bytes of a transposing read
    // fall on different banks (a k-row of 64 rows is half of the banks' 256 bytes)
    static __device__ __forceinline__ int k_slot(int k) { return UR == 64 ? (k & 2) << 1 : (k & 3) << 2; }
    // bytes from load 0 to load Q
    template <int Q>
    __device__ __forceinline__ unsigned q_off() const {
        if constexpr (KC) {
            constexpr int p = 32 * Q;  // LDS row of the load
            constexpr int row = SPLIT ? (p % UR) / (WR / 2) * WR + (p / UR) * (WR / 2) + p % (WR / 2) : p;
            return row * 2u * ld;
        } else if constexpr (SPLIT) {
            constexpr int u = Q / (NL / 2), k = (Q % (NL / 2)) * 4 * KR;
            return k * 2u * ld + u * WR;  // (WR / 2 rows of 2 bytes)
        } else {
            return Q * 8u * KR * ld;
        }
    }
    __device__ __forceinline__ void init(int ld_, int wave, int lane, int wrow) {  // wrow: index of this wave's row block
        ld = (unsigned)ld_;
        const int row0 = SPLIT ? wrow * (WR / 2) : wrow * WR;  // inside a unit
        if constexpr (KC) {
            const int row = 8 * wave + (lane >> 3), r = lane & 15, h = lane >> 4;
            voff[0] = (unsigned)row * ld * 2u + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
            foff[0] = (row0 + r) * 128 + ((h ^ ((r >> 1) & 7)) << 4);
        } else {
            const int k = wave * KR + lane / (UR / 8), gp = (lane % (UR / 8)) ^ k_slot(k);
            const int row = SPLIT ? (gp * 8) / (WR / 2) * WR + (gp * 8) % (WR / 2) : gp * 8;
            voff[0] = (unsigned)k * ld * 2u + row * 2;
            const int h = lane >> 4, i16 = lane & 15, kq = i16 >> 2;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                foff[i] = (8 * h + kq) * RB + (((((row0 + 32 * i) >> 3) ^ k_slot(kq)) + ((i16 & 3) >> 1)) << 4) + (i16 & 1) * 8;
        }
        if constexpr (GUARD) {
            static_for<NL - 1>([&](auto qc) { voff[decltype(qc)::value + 1] = voff[0] + q_off<decltype(qc)::value + 1>(); });
        }
        piece = (lane & 7) ^ ((8 * wave + (lane >> 3)) >> 1 & 7);   // (contraction-contiguous: the same for every load)
    }
    // Contraction-contiguous rows whose last k-tile holds only k_last (a multiple of 8) of the contraction: while the load
    // stream stands at it, the lanes whose piece lies beyond fetch from outside the buffer, which gives zeros.
    __device__ __forceinline__ void tail_on(int k_last) {
        if constexpr (KC && GUARD) {
#pragma unroll
            for (int q = 0; q < NL; ++q) voff[q] |= 8 * piece >= k_last ? BUF_OUT : 0u;
        }
    }
    __device__ __forceinline__ void tail_off() {
        if constexpr (KC && GUARD) {
#pragma unroll
            for (int q = 0; q < NL; ++q) voff[q] &= ~BUF_OUT;
        }
    }
    // Load Q of a k-tile, in two instructions of their own: its LDS destination (base: this wave's part of the stage) and, no
    // sooner than one instruction later, the load.  Assembly on purpose: the compiler orders every LDS read behind an
    // LDS-writing load it knows of by waiting for ALL loads in flight (it cannot tell the stages apart).  The counted waits
    // in front of the barriers are what orders these loads against the reads.  (Nothing else here uses M0.)
    template <int Q>
    static __device__ __forceinline__ void target(unsigned base) { asm volatile("s_add_u32 m0, %0, %1" ::"s"(base), "n"(Q * 4096) : "scc"); }
    template <int Q>
    __device__ __forceinline__ void issue(const u32x4 rsrc) const {
        // (the buffer's bounds are checked without the scalar offset, so rows that may lie outside go by the vector one alone)
        if constexpr (GUARD) asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff[Q]), "s"(rsrc) : "memory");
        else asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff[0]), "s"(rsrc), "s"(q_off<Q>()) : "memory");
    }
    // matrix-core fragment of slice KK (32 k): k = 8 (lane / 16) ... + 7 for row (lane % 16) of 16-row tile I of unit U
    template <int KK, int U, int I>
    __device__ __forceinline__ f16x8 frag(const char* stage) const {
        if constexpr (KC) return *reinterpret_cast<const f16x8*>(stage + (foff[0] ^ (KK * 64)) + U * (UR * 128) + I * 2048);
        else return frag_at<KK>(stage + frag_offset<U, I>());
    }
    // ... output-contiguous: in two steps
    template <int U, int I>
    __device__ __forceinline__ unsigned frag_offset() const {
        return KC ? 0u : foff[KC ? 0 : I >> 1] + (I & 1) * 32 + U * (UR * 128);
    }
    template <int KK>
    static __device__ __forceinline__ f16x8 frag_at(const char* p) {
        if constexpr (KC) {
            return f16x8{};
        } else {
            p += KK * 32 * RB;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)MP_LDS_PTR(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)MP_LDS_PTR(p + 4 * RB));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            return __builtin_bit_cast(f16x8, v);
        }
    }
    // Bytes a tile's buffer spans from the origin of its k-tile, `left` of its rows and `k_left` of its k being inside the
    // matrix.  Loads beyond it give zeros.  Output-contiguous: k-rows beyond the contraction, and columns beyond `left` (whole
    // words: a piece may straddle) of the last k-row; those of the other k-rows are elements behind the row's end or of the row
    // that follows, and no stored result depends on them.
    static __device__ __forceinline__ unsigned span(int left, int ld, int k_left) {
        return KC ? (left - 1) * (unsigned)ld * 2u + 2u * BK : (unsigned)(min(k_left, BK) - 1) * (unsigned)ld * 2u + ((2u * left + 3u) & ~3u);
    }
    static __device__ __forceinline__ long long origin(int row, int ld) { return KC ? (long long)row * ld * 2 : 2ll * row; }  // bytes
};

// Epilogue of one wave tile (TM x TN matrix-core tiles of 16 x 16; rows mw ..., columns nw ...).  Of tile (i, j) lane
// (er = lane % 16, eh = lane / 16) holds row er and the 4 consecutive columns 4 eh ...  16 rows at a time go through a
// wave-private piece of LDS (`stg`, 16-byte slots ^ row) and come back as 8 consecutive columns per lane with consecutive
// lanes along a row, so that stores and residual / ReLU-source loads cover whole cache lines.  Straight from the
// matrix-core layout every 16 bytes of a wave's store lie in another line, and the stores of a tile take 5 us longer to drain
// (8192 x 32768 over 1024: 538 us that way, 489 this way).
// Returns after STORES = TM * NI store instructions of this wave if every lane's element exists (fp16 output).
template <int TN>
constexpr int dtl_out_accesses() { return 16 / (16 * TN > 64 ? 4 : 8); }   // stores per 16-row block
template <int TM, int TN, int MODE>
__device__ __forceinline__ void dtl_epilogue(const GemmArgs& g, f32x4 (&acc)[TM][TN], const int mw, const int nw, const bool split,
                                             const bool fold_bias, char* const stg, bool& bad) {
    const int lane = threadIdx.x & 63, er = lane & 15, eh = lane >> 4;
    asm volatile("s_nop 15\n\ts_nop 15");  // the last matrix-core results have landed before the explicit accumulator reads
    constexpr bool GUARD = MODE != INTERIOR;
    if (g.C32) {  // raw accumulator out: split-K partial, or fp32 result with alpha and addend
        static_for<TM * TN>([&](auto tc) {
            constexpr int t = decltype(tc)::value, i = t / TN, j = t % TN;
            const int m = mw + er + 16 * i, n = nw + 16 * j + 4 * eh;
            if (GUARD && (m >= g.M || n >= g.N)) return;
            f32x4 v = {acc_get(acc[i][j][0]), acc_get(acc[i][j][1]), acc_get(acc[i][j][2]), acc_get(acc[i][j][3])};
            const long long mn = (long long)m * g.N + n;
            if (!split) {
                v *= g.alpha;
                if (g.acc_in) v += *reinterpret_cast<const f32x4_u*>(g.acc_in + mn);
            }
            *reinterpret_cast<f32x4_u*>(g.C32 + mn) = v;
        });
        return;
    }
    typedef float    f32x2 __attribute__((ext_vector_type(2)));
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    // the uncommon terms first, in fp32: scale factor, fp32 addend, a bias that could not start the accumulators
    if (g.alpha != 1.f || g.acc_in || (g.bias && !fold_bias)) {
        static_for<TM * TN>([&](auto tc) {
            constexpr int t = decltype(tc)::value, i = t / TN, j = t % TN;
            const int m = mw + er + 16 * i, n = nw + 16 * j + 4 * eh;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = !GUARD || (m < g.M && n + (MODE == TAIL ? e : 0) < g.N);
                float x = acc_get(acc[i][j][e]) * g.alpha;
                if (g.acc_in && in) x += g.acc_in[(long long)m * g.N + n + e];
                if (g.bias && !fold_bias && in) x += h2f(g.bias[n + e]);
                acc[i][j][e] = acc_put(x);
            }
        });
    }
    constexpr int WN = 16 * TN, PITCH = dtl_out_pitch(WN), SLOTS = PITCH / 16;  // 16-byte slots of a row in LDS
    constexpr int RPA = 64 / SLOTS, NI = dtl_out_accesses<TN>();               // rows per access, accesses per 16-row block
    static_assert(16 / RPA == NI, "accesses of a block");
    auto slot = [](int row) { return SLOTS == 16 ? row & 15 : (row >> 1) & 7; };
    const int       orow = lane / SLOTS, op = lane % SLOTS;   // row inside an access, 8-column piece
    const int       n    = nw + 8 * op;
    const bool      act  = op < WN / 8 && (!GUARD || n < g.N);
    const uint16_t* aux  = g.relu_src ? g.relu_src : g.add;
    u16x2           mag  = {0, 0};  // running maximum of the magnitude bits of everything stored (non-finite: >= 0x7C00)
    constexpr int   AD   = 3;       // residual / ReLU-source blocks on their way
    u32x4           av[AD][NI], out[2][NI];
    auto row_of   = [&](const int i, const int t) { return mw + 16 * i + RPA * t + orow; };
    auto aux_load = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        static_for<NI>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            av[i % AD][t]   = u32x4{0u, 0u, 0u, 0u};
            const int m     = row_of(i, t);
            const uint16_t* const a = aux + (long long)m * g.ld_aux + n;
            if (act && (!GUARD || m < g.M)) av[i % AD][t] = MODE == TAIL ? load8_guard(a, g.N - n) : *reinterpret_cast<const u32x4*>(a);
        });
    };
    auto finish = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        static_for<NI>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const int     m = row_of(i, t);
            if (!act || (GUARD && m >= g.M)) return;
            u32x4 o = out[i & 1][t];
            if (aux) {
                const u32x4 a = av[i % AD][t];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const unsigned ow = o[w], aw = a[w];  // (bit_cast wants whole objects, not vector elements)
                    const f16x2    hv = __builtin_bit_cast(f16x2, ow), tv = __builtin_bit_cast(f16x2, aw);
                    f16x2          rv;
                    if (g.relu_src) {
                        rv[0] = (tv[0] > (_Float16)0) ? hv[0] : (_Float16)0;
                        rv[1] = (tv[1] > (_Float16)0) ? hv[1] : (_Float16)0;
                    } else {
                        rv = __builtin_convertvector(__builtin_convertvector(hv, f32x2) + __builtin_convertvector(tv, f32x2), f16x2);
                    }
                    o[w] = __builtin_bit_cast(unsigned, rv);
                }
            }
            if (g.found_inf) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    unsigned mw_ = o[w] & 0x7FFF7FFFu;
                    if (MODE == TAIL) {  // columns beyond N do not count (they may hold inf * 0)
                        if (n + 2 * w >= g.N) mw_ = 0u;
                        else if (n + 2 * w + 1 >= g.N) mw_ &= 0xFFFFu;
                    }
                    mag = __builtin_elementwise_max(mag, __builtin_bit_cast(u16x2, mw_));
                }
            }
            uint16_t* const c = g.C + (long long)m * g.ldc + n;
            if (MODE != TAIL) *reinterpret_cast<u32x4*>(c) = o;
            else if (n + 8 <= g.N) *reinterpret_cast<u32x4_u*>(c) = o;
            else store8_tail(c, o, g.N - n);
        });
    };
    if (aux) static_for<(AD - 1 < TM ? AD - 1 : TM)>([&](auto ic) { aux_load(ic); });
    __builtin_amdgcn_sched_barrier(0);
    static_for<TM + 1>([&](auto ic) {  // block i through LDS, then block i - 1 out
        constexpr int i = decltype(ic)::value;
        if constexpr (i < TM) {
            static_for<TN>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                float         v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc_get(acc[i][j][e]);
                if (g.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (v[e] < 0.f) ? 0.f : v[e];  // max(v, 0) that keeps a NaN (the comparison is false for it)
                }
                const f16x2 lo = __builtin_convertvector(f32x2{v[0], v[1]}, f16x2), hi = __builtin_convertvector(f32x2{v[2], v[3]}, f16x2);
                *reinterpret_cast<u32x2g*>(stg + er * PITCH + (((2 * j + (eh >> 1)) ^ slot(er)) << 4) + (eh & 1) * 8) =
                    u32x2g{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
            });
            static_for<NI>([&](auto tc) {
                constexpr int t   = decltype(tc)::value;
                const int     row = RPA * t + orow;
                out[i & 1][t]     = *reinterpret_cast<const u32x4*>(stg + row * PITCH + ((op ^ slot(row)) << 4));
            });
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (i > 0) finish(std::integral_constant<int, i - 1>{});
        if constexpr (i + AD - 1 < TM) {
            if (aux) aux_load(std::integral_constant<int, i + AD - 1>{});  // (into the registers of block i - 1)
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    bad |= mag[0] >= 0x7C00 || mag[1] >= 0x7C00;
}

// tile numbering: XCD-contiguous runs, bands of 4 tile rows (as gemm_kernel)
__device__ __forceinline__ int dtl_tile_of(const int vb, const int ntiles) {
    const int q = ntiles >> 3, rem = ntiles & 7, x = vb & 7, local = vb >> 3;
    return x * q + min(x, rem) + local;
}
template <int BM, int BN>
__device__ __forceinline__ void dtl_tile_origin(const GemmArgs& g, const int p, int& mm, int& nn) {
    constexpr int GROUP = 4;
    const int     band  = p / (GROUP * g.tiles_n);
    const int     first = band * GROUP;
    const int     gsz   = min(GROUP, g.tiles_m - first);
    const int     inb   = p - band * GROUP * g.tiles_n;
    mm                  = (first + inb % gsz) * BM;
    nn                  = (inb / gsz) * BN;
}
// buffer descriptors (words 0 and 1: address, word 2: size)
__device__ __forceinline__ void buffer_move(u32x4& r, const long long d) {
    const unsigned long long a = (((unsigned long long)r[1] << 32) | r[0]) + d;
    r[0] = (unsigned)a;
    r[1] = (unsigned)(a >> 32);
}
__device__ __forceinline__ u32x4 buffer_at(const uint16_t* p, const long long bytes, const unsigned size) {
    u32x4 r = {0u, 0u, size, 0x00020000u};
    buffer_move(r, (long long)reinterpret_cast<unsigned long long>(p) + bytes);
    return r;
}

// bias of the 4 columns n ...
template <int MODE>
__device__ __forceinline__ u32x2g dtl_bias(const GemmArgs& g, const int n) {
    if (MODE == INTERIOR) return *reinterpret_cast<const u32x2g*>(g.bias + n);
    if (n + 4 <= g.N) return *reinterpret_cast<const u32x2_u*>(g.bias + n);
    if (MODE != TAIL || n >= g.N) return u32x2g{0u, 0u};
    unsigned b0 = g.bias[n], b1 = 0u;
    if (n + 1 < g.N) b0 |= (unsigned)g.bias[n + 1] << 16;
    if (n + 2 < g.N) b1 = g.bias[n + 2];
    return u32x2g{b0, b1};
}

// Sums of the first operand over the contraction: the bias gradient that goes with a weight gradient, of which this kernel has
// every element in LDS anyway.  The tiles beside each other and the two wave columns of each share the row tiles of 16 out among
// them (`slot`), one to a wave, which reads that row tile's fragments once more.  (Picking them out of the registers by the
// wave's number costs a chain of branches: 5 us of a product of 28.)  DOT: summed with 8 two-element dot products per k-tile,
// for the kernels whose accumulators fill the matrix cores' half of the registers, where a conditional matrix instruction costs
// 8 copies each way (8192 x 3072 x 1024 74.0 us that way, 67.6 this way, 63.4 without sums); else with 2 matrix instructions
// against a fragment of ones (2048 x 1024 x 1024 14.9 / 14.3).
template <typename OPA, int TM, int UNIT, bool ON, bool DOT>   // UNIT: row tiles of a unit of OPA's rows
struct DtlSums {
    int      mine;      // row tile of this wave, or none
    unsigned off;       // where its fragments lie in a stage
    f16x8    f[2];      // of slice 0 and 1
    float    dot[2];
    f32x4    mfma[2];
    __device__ __forceinline__ void start(const GemmArgs& g, const OPA& oa, const int slot) {
        if constexpr (ON) {
            mine = __builtin_amdgcn_readfirstlane(slot < TM ? slot : -1);
            off  = 0;
            static_for<TM>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (mine == i) off = oa.template frag_offset<i / UNIT, i % UNIT>();
            });
            dot[0] = dot[1] = 0.f;
            mfma[0] = mfma[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __device__ __forceinline__ bool upper() const { return ON && mine >= 0 && mine < UNIT; }
    __device__ __forceinline__ bool lower() const { return ON && mine >= UNIT; }
    __device__ __forceinline__ void read(const char* stage) {
        if constexpr (ON) {
            f[0] = OPA::template frag_at<0>(stage + off);
            f[1] = OPA::template frag_at<1>(stage + off);
        }
    }
    __device__ __forceinline__ void add() {
        if constexpr (ON) {
            const f16   one  = (f16)1.f;
            const f16x2 ones = {one, one};
            if (mine >= 0) {
                if constexpr (DOT) {
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
#pragma unroll
                        for (int q = 0; q < 2; ++q) dot[q] = __builtin_amdgcn_fdot2(f16x2{f[q][e], f[q][e + 1]}, ones, dot[q], false);
                    }
                } else {
                    const f16x8 ones8 = {one, one, one, one, one, one, one, one};
#pragma unroll
                    for (int q = 0; q < 2; ++q) mfma[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones8, f[q], mfma[q], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // mw: first row of the wave
    __device__ __forceinline__ void store(const GemmArgs& g, const int mw, const bool split, bool& bad) const {
        if constexpr (ON) {
            if (mine < 0) return;
            const int lane = threadIdx.x & 63, m = mw + 16 * mine + lane;
            float     s    = DOT ? dot[0] + dot[1] : mfma[0][0] + mfma[1][0];
            if constexpr (DOT) {   // (lanes r, r + 16, r + 32 and r + 48 have row r over k of their own)
                s += __shfl_xor(s, 16, 64);
                s += __shfl_xor(s, 32, 64);
            }
            if (lane >= 16 || m >= g.M) return;
            if (split) {
                g.db_part[m] = s;
            } else {
                const uint16_t h = f2h(s);
                g.db[m]          = h;
                bad |= half_nonfinite(h);
            }
        }
    }
};

// The output tiles vb0, vb0 + vb_step, ... (< tiles_m * tiles_n) of problem g, one after the other, with the load stream
// running on from tile to tile.  remap: number the tiles so that each XCD gets a contiguous run (a launch of one problem);
// otherwise vb is the tile number itself (the caller has placed the tiles).  split: g describes one part of a split contraction.
template <int BM, int BN, bool A_KC, bool B_KC, int MODE, bool SUMS>
__device__ __forceinline__ void dtl_tiles(const GemmArgs& g, const int vb0, const int vb_step, const bool remap, const bool split,
                                          char* smem, bool& bad) {
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16, TH = TM / 2;
    typedef DtlOperand<BM, WM, A_KC, true, MODE != INTERIOR>  OpA;
    typedef DtlOperand<BN, WN, B_KC, false, MODE != INTERIOR> OpB;
    constexpr int STAGE = dtl_stage(BM, BN);
    constexpr int MS = TH * TN * 2;   // matrix-core instructions per phase ...
    constexpr int PB = TH * 2;        // ... of which in front of its barrier: one column of tiles
    // Loads: phase 0 the upper rows of the first operand and half of the second (their space is free behind phase 0's
    // barrier), phase 1 the rest of the second operand and the lower rows.
    constexpr int NA = OpA::NL, NB = OpB::NL, NL = NA + NB, NAH = NA / 2, NBH = NB / 2;
    constexpr int L0 = NAH + NBH, L1 = NL - L0;
    constexpr int PI0 = (MS - PB) / L0, PI1 = (MS - PB) / L1;   // matrix-core instructions per load
    // Loads in flight that a barrier does not wait for: those issued behind the ones it needs.  Phase 0's needs the lower
    // rows of this k-tile (the last loads of the k-tile before last), phase 1's the next k-tile but for its lower rows.
    constexpr int FLY0 = NL, FLY1 = NAH + L0;
    // ... and a tile's output stores behind them (see `behind`)
    constexpr int NS = MODE == INTERIOR ? TM * dtl_out_accesses<TN>() : 0;
    static_assert(FLY0 + NS <= 63 && FLY1 + L1 <= 63 && PI0 >= 2 && PI1 >= 2, "loads in flight must fit the counter");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lds_a = (unsigned)(size_t)MP_LDS_PTR(smem) + wave * 1024, lds_b = lds_a + OpA::BYTES;
    const int wm = wave >> 1, wn = wave & 1;
    const int eh = lane >> 4;
    const int nkt    = (g.K + BK - 1) / BK;
    const int ntiles = g.tiles_m * g.tiles_n;

    auto tile_origin = [&](const int vb, int& mm, int& nn) { dtl_tile_origin<BM, BN>(g, remap ? dtl_tile_of(vb, ntiles) : vb, mm, nn); };

    OpA oa;
    OpB ob;
    oa.init(g.lda, wave, lane, wm);
    ob.init(g.ldb, wave, lane, wn);
    const long long step_a = A_KC ? 2 * BK : 2ll * BK * g.lda;   // bytes from one k-tile to the next
    const long long step_b = B_KC ? 2 * BK : 2ll * BK * g.ldb;

    // ---- the load stream: k-tile after k-tile, output tile after output tile, two k-tiles ahead of the matrix cores
    int m0, n0;
    tile_origin(vb0, m0, n0);
    u32x4 ra = buffer_at(g.A, OpA::origin(m0, g.lda), OpA::span(min(g.M - m0, BM), g.lda, BK));
    u32x4 rb = buffer_at(g.B, OpB::origin(n0, g.ldb), OpB::span(min(g.N - n0, BN), g.ldb, BK));
    auto  size_to = [&](const int m, const int n, const int k_left) {
        ra[2] = OpA::span(min(g.M - m, BM), g.lda, k_left);
        rb[2] = OpB::span(min(g.N - n, BN), g.ldb, k_left);
    };
    const int k_last  = g.K - (nkt - 1) * BK;   // k of a tile's last k-tile
    int       l_m = m0, l_n = n0;               // its tile (with three k-tiles to a tile the stream is a whole tile ahead by then)
    auto      to_last = [&] {
        size_to(l_m, l_n, k_last);
        oa.tail_on(k_last);
        ob.tail_on(k_last);
    };
    int      left = nkt;      // k-tiles of its output tile from where the stream stands
    unsigned l_st = 0;        // LDS offset of the stage it writes
    // load q of a phase: its LDS destination (SET), or the load itself
    auto load0 = [&](auto qc, auto setc) {
        constexpr int  q   = decltype(qc)::value;
        constexpr bool set = decltype(setc)::value;
        if constexpr (q < NAH) {
            if constexpr (set) OpA::template target<q>(lds_a + l_st);
            else oa.template issue<q>(ra);
        } else {
            if constexpr (set) OpB::template target<q - NAH>(lds_b + l_st);
            else ob.template issue<q - NAH>(rb);
        }
    };
    auto load1 = [&](auto qc, auto setc) {
        constexpr int  q   = decltype(qc)::value;
        constexpr bool set = decltype(setc)::value;
        if constexpr (q < NB - NBH) {
            if constexpr (set) OpB::template target<q + NBH>(lds_b + l_st);
            else ob.template issue<q + NBH>(rb);
        } else {
            if constexpr (set) OpA::template target<q - (NB - NBH) + NAH>(lds_a + l_st);
            else oa.template issue<q - (NB - NBH) + NAH>(ra);
        }
    };
    typedef std::true_type  Set;
    typedef std::false_type Load;

    f16x8 alo[2][TH], ahi[2][TH], bf[2][TN];  // fragments [slice][tile]
    auto  read_alo = [&](const char* st, auto fc) { constexpr int f = decltype(fc)::value; alo[f / TH][f % TH] = oa.template frag<f / TH, 0, f % TH>(st); };
    auto  read_ahi = [&](const char* st, auto fc) { constexpr int f = decltype(fc)::value; ahi[f / TH][f % TH] = oa.template frag<f / TH, 1, f % TH>(st); };
    auto  read_b   = [&](const char* st, auto fc) { constexpr int f = decltype(fc)::value; bf[f % 2][f / 2] = ob.template frag<f % 2, 0, f / 2>(st + OpA::BYTES); };

    // prologue: both stages requested, in the order the loop requests them; the first k-tile but for its lower rows landed
    static_for<2>([&](auto sc) {
        static_for<L0>([&](auto qc) { load0(qc, Set{}); asm volatile("s_nop 0"); load0(qc, Load{}); });
        static_for<L1>([&](auto qc) { load1(qc, Set{}); asm volatile("s_nop 0"); load1(qc, Load{}); });
        l_st = STAGE - l_st;
        --left;
        buffer_move(ra, step_a);
        buffer_move(rb, step_b);
    });
    if (MODE != INTERIOR && left == 1) to_last();
    // the bias starts the accumulators; a tile's values are requested ahead of the previous tile's output stores (a wait for
    // a load behind them would be a wait for the stores)
    u32x2g     braw[TN];
    const bool fold_bias = g.bias != nullptr && g.C32 == nullptr && g.alpha == 1.f;
    auto load_bias = [&](const int nn) {
        static_for<TN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int     n = nn + wn * WN + 16 * j + 4 * eh;
            braw[j] = dtl_bias<MODE>(g, n);
        });
    };
    if (fold_bias) load_bias(n0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLY1 + L1) : "memory");
    __syncthreads();
    unsigned c_st = 0;   // LDS offset of the stage the matrix cores work on
    static_for<2 * TH>([&](auto fc) { read_alo(smem, fc); });
    static_for<2 * TN - 2>([&](auto fc) { read_b(smem, fc); });

    for (int vb = vb0; vb < ntiles; vb += vb_step) {
        // from the last k-tile of this tile to the first of the next (or back to this tile's own first: those loads go to
        // stages nobody reads any more, are in bounds, and keep the count of loads in flight uniform)
        int m1 = m0, n1 = n0;
        if (vb + vb_step < ntiles) tile_origin(vb + vb_step, m1, n1);
        const long long jump_a = OpA::origin(m1, g.lda) - OpA::origin(m0, g.lda) - (nkt - 1) * step_a;
        const long long jump_b = OpB::origin(n1, g.ldb) - OpB::origin(n0, g.ldb) - (nkt - 1) * step_b;
        f32x4 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (fold_bias) {
            static_for<TN>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float b = h2f((uint16_t)((e & 1) ? (braw[j][e >> 1] >> 16) : (braw[j][e >> 1] & 0xFFFFu)));
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][j][e] = acc_put(b);
                }
            });
        }
        DtlSums<OpA, TM, TH, SUMS, true> sums;
        sums.start(g, oa, 2 * (n0 / BN) + wn);
        // The previous tile's output stores are younger than the loads that the first three barriers of a tile need, which
        // therefore need not wait for them: `behind` counts those barriers (three, or none for the first tile).
        int behind = NS > 0 && vb != vb0 ? 3 : 0;
        auto barrier = [&](auto flyc) {
            constexpr int fly = decltype(flyc)::value;
            if (NS > 0 && behind > 0) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(fly + NS) : "memory");
                --behind;
            } else {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(fly) : "memory");
            }
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int kt = 0; kt < nkt; ++kt) {
            const char* st = smem + c_st;
            __builtin_amdgcn_sched_barrier(0);
            // Phase 0: upper rows.  Instruction m: column m / (2 TH), slice (m / TH) % 2, row tile m % TH.  In front of the
            // barrier: the last column's fragments (their registers were in use until now).  Behind it: this k-tile's lower
            // rows, and loads of the k-tile after next into the space of this k-tile's upper rows and second operand.
            static_for<MS>([&](auto mc) {
                constexpr int m = decltype(mc)::value, j = m / (2 * TH), s = m / TH % 2, i = m % TH;
                // (rows to be summed are read once more: upper ones while they are there, lower ones once they are)
                if constexpr (m == 0) {
                    if (sums.upper()) sums.read(st);
                }
                if constexpr (m == PB) {
                    barrier(std::integral_constant<int, FLY0>{});
                    if (sums.lower()) sums.read(st);
                }
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[s][j], alo[s][i], acc[i][j], 0, 0, 0);
                if constexpr (m < 2) read_b(st, std::integral_constant<int, 2 * TN - 2 + m>{});
                if constexpr (m >= PB) {
                    constexpr int x = m - PB;
                    if constexpr (x % 2 == 0 && x / 2 < 2 * TH) read_ahi(st, std::integral_constant<int, x / 2>{});
                    if constexpr (x / PI0 < L0 && x % PI0 == PI0 - 2) load0(std::integral_constant<int, x / PI0>{}, Set{});
                    if constexpr (x / PI0 < L0 && x % PI0 == PI0 - 1) load0(std::integral_constant<int, x / PI0>{}, Load{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            sums.add();
            c_st = STAGE - c_st;
            st   = smem + c_st;
            // Phase 1: lower rows.  Behind the barrier: the next k-tile's upper rows, and its column c once this k-tile's
            // instructions of column c are out; loads of the k-tile after next.
            static_for<MS>([&](auto mc) {
                constexpr int m = decltype(mc)::value, j = m / (2 * TH), s = m / TH % 2, i = m % TH;
                if constexpr (m == PB) barrier(std::integral_constant<int, FLY1>{});
                acc[TH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[s][j], ahi[s][i], acc[TH + i][j], 0, 0, 0);
                if constexpr (m >= PB) {
                    constexpr int x = m - PB, y = x % (2 * TH), c = x / (2 * TH);
                    constexpr int AR = TH == 4 ? 3 : 2;   // fragments of the upper rows per column
                    if constexpr (y < 2) read_b(st, std::integral_constant<int, 2 * c + y>{});
                    else if constexpr (y < 2 + AR && AR * c + y - 2 < 2 * TH) read_alo(st, std::integral_constant<int, AR * c + y - 2>{});
                    if constexpr (x / PI1 < L1 && x % PI1 == PI1 - 2) load1(std::integral_constant<int, x / PI1>{}, Set{});
                    if constexpr (x / PI1 < L1 && x % PI1 == PI1 - 1) load1(std::integral_constant<int, x / PI1>{}, Load{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            static_assert((TN - 1) * (TH == 4 ? 3 : 2) >= 2 * TH, "columns to read the upper rows in");
            l_st = STAGE - l_st;
            const bool last = left == 1;
            left = last ? nkt : left - 1;
            buffer_move(ra, last ? jump_a : step_a);
            buffer_move(rb, last ? jump_b : step_b);
            if (MODE != INTERIOR && last) {
                l_m = m1;
                l_n = n1;
                size_to(l_m, l_n, BK);
                oa.tail_off();
                ob.tail_off();
            }
            if (MODE != INTERIOR && left == 1) to_last();
        }
        if (fold_bias) load_bias(n1);
        sums.store(g, m0 + wm * WM, split, bad);
        dtl_epilogue<TM, TN, MODE>(g, acc, m0 + wm * WM, n0 + wn * WN, split, fold_bias, smem + 2 * STAGE + wave * dtl_out_bytes(WN), bad);
        m0 = m1;
        n0 = n1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last (unused) loads have landed before the LDS is reused
    __syncthreads();
}

// The same for tiles of 128 x 64 and 64 x 128, which have a quarter of the matrix-core work per k-tile: a k-tile's loads need
// several k-tiles of lead, so the stages form a ring (six, all of a compute unit's LDS) and each is worked on as a whole; a
// stage is free once its fragments are in registers, one k-tile ahead of its use.  One barrier per k-tile.  What bounds a
// k-tile is that chain and no unit's rate (counters over a layer of d_model 512, 4096 tokens, in the compute units' busy cycles: LDS
// instructions 19 %, with a transposed operand 31 % of which 12 are bank conflicts, matrix cores 23 %; waves wait 35 %): 0.27 us, the
// register-staged kernel 0.38 (4096 x 512 over 2048: 16.4 -> 13.5 us; input gradient 1600 x 1024 over 4096: 29.5 -> 23.2).
constexpr int    DEEP_STAGES = 6;
constexpr size_t deep_lds(int bm, int bn) { return DEEP_STAGES * (size_t)dtl_stage(bm, bn) + 4 * dtl_out_bytes(bn / 2); }
template <int BM, int BN, bool A_KC, bool B_KC, int MODE, bool SUMS>
__device__ __forceinline__ void deep_tiles(const GemmArgs& g, const int vb0, const int vb_step, const bool split, char* smem, bool& bad) {
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16;
    typedef DtlOperand<BM, WM, A_KC, false, MODE != INTERIOR> OpA;
    typedef DtlOperand<BN, WN, B_KC, false, MODE != INTERIOR> OpB;
    constexpr int STAGE = dtl_stage(BM, BN), MS = TM * TN * 2, NA = OpA::NL, NL = NA + OpB::NL, NR = 2 * (TM + TN);
    constexpr int PI = MS / NL;   // matrix-core instructions per load
    static_assert(PI >= 2 && (DEEP_STAGES - 1) * NL <= 63, "loads in flight must fit the counter");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lds_a = (unsigned)(size_t)MP_LDS_PTR(smem) + wave * 1024, lds_b = lds_a + OpA::BYTES;
    const int wm = wave >> 1, wn = wave & 1;
    const int eh = lane >> 4;
    const int nkt    = (g.K + BK - 1) / BK;
    const int ntiles = g.tiles_m * g.tiles_n;
    auto tile_origin = [&](const int vb, int& mm, int& nn) { dtl_tile_origin<BM, BN>(g, dtl_tile_of(vb, ntiles), mm, nn); };

    OpA oa;
    OpB ob;
    oa.init(g.lda, wave, lane, wm);
    ob.init(g.ldb, wave, lane, wn);
    const long long step_a = A_KC ? 2 * BK : 2ll * BK * g.lda, step_b = B_KC ? 2 * BK : 2ll * BK * g.ldb;

    // the load stream: k-tile after k-tile, output tile after output tile (past the last k-tile of all it starts that tile
    // again: in bounds, into stages nobody reads any more)
    u32x4    ra, rb;
    int      l_vb = vb0, left = nkt;
    unsigned l_st = 0;
    auto stand = [&] {
        int m, n;
        tile_origin(l_vb, m, n);
        ra = buffer_at(g.A, OpA::origin(m, g.lda), OpA::span(min(g.M - m, BM), g.lda, g.K));
        rb = buffer_at(g.B, OpB::origin(n, g.ldb), OpB::span(min(g.N - n, BN), g.ldb, g.K));
    };
    stand();
    auto load = [&](auto qc, auto setc) {
        constexpr int  q   = decltype(qc)::value;
        constexpr bool set = decltype(setc)::value;
        if constexpr (q < NA) {
            if constexpr (set) OpA::template target<q>(lds_a + l_st);
            else oa.template issue<q>(ra);
        } else {
            if constexpr (set) OpB::template target<q - NA>(lds_b + l_st);
            else ob.template issue<q - NA>(rb);
        }
    };
    auto advance = [&] {
        l_st = l_st + STAGE == DEEP_STAGES * STAGE ? 0 : l_st + STAGE;
        if (__builtin_expect(--left > 0, 1)) {
            buffer_move(ra, step_a);
            buffer_move(rb, step_b);
            if (MODE != INTERIOR && left == 1) {   // the last k-tile may be short
                const int k_last = g.K - (nkt - 1) * BK;
                int       m, n;
                tile_origin(l_vb, m, n);
                ra[2] = OpA::span(min(g.M - m, BM), g.lda, k_last);
                rb[2] = OpB::span(min(g.N - n, BN), g.ldb, k_last);
                oa.tail_on(k_last);
                ob.tail_on(k_last);
            }
        } else {
            oa.tail_off();
            ob.tail_off();
            if (l_vb + vb_step < ntiles) l_vb += vb_step;
            left = nkt;
            stand();
        }
    };
    typedef std::true_type  Set;
    typedef std::false_type Load;
    f16x8 af[2][2][TM], bf[2][2][TN];  // fragments [k-tile parity][slice][tile]
    auto  read = [&](const char* st, auto pc, auto fc) {
        constexpr int p = decltype(pc)::value, f = decltype(fc)::value, s = f / (TM + TN), t = f % (TM + TN);
        if constexpr (t < TN) bf[p][s][t] = ob.template frag<s, 0, t>(st + OpA::BYTES);
        else af[p][s][t - TN] = oa.template frag<s, 0, t - TN>(st);
    };
    u32x2g     braw[TN];
    const bool fold_bias = g.bias != nullptr && g.C32 == nullptr && g.alpha == 1.f;
    auto load_bias = [&](const int nn) {
        static_for<TN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int     n = nn + wn * WN + 16 * j + 4 * eh;
            braw[j] = dtl_bias<MODE>(g, n);
        });
    };
    int m0, n0;
    tile_origin(vb0, m0, n0);
    if (fold_bias) load_bias(n0);
    static_for<DEEP_STAGES>([&](auto) {
        static_for<NL>([&](auto qc) { load(qc, Set{}); asm volatile("s_nop 0"); load(qc, Load{}); });
        advance();
    });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEEP_STAGES - 1) * NL) : "memory");
    __syncthreads();
    unsigned c_st = 0;
    static_for<NR>([&](auto fc) { read(smem, std::integral_constant<int, 0>{}, fc); });
    DtlSums<OpA, TM, TM, SUMS, false> sums;   // of the k-tile that is being read, one ahead of the matrix cores
    sums.start(g, oa, 2 * (n0 / BN) + wn);
    if (sums.upper()) sums.read(smem);
    sums.add();

    for (int vb = vb0; vb < ntiles; vb += vb_step) {
        int m1 = m0, n1 = n0;
        if (vb + vb_step < ntiles) tile_origin(vb + vb_step, m1, n1);
        f32x4 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (fold_bias) {
            static_for<TN>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float b = h2f((uint16_t)((e & 1) ? (braw[j][e >> 1] >> 16) : (braw[j][e >> 1] & 0xFFFFu)));
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][j][e] = acc_put(b);
                }
            });
        }
        DtlSums<OpA, TM, TM, SUMS, false> tile_sums;
        auto ktile = [&](auto pc, const bool last) {
            constexpr int p = decltype(pc)::value;
            c_st = c_st + STAGE == DEEP_STAGES * STAGE ? 0 : c_st + STAGE;
            const char* st = smem + c_st;   // of the next k-tile
            __builtin_amdgcn_sched_barrier(0);
            // the next k-tile has landed, and every wave has this one's fragments in registers
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((DEEP_STAGES - 2) * NL) : "memory");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            if (SUMS && last) {   // (the k-tile read here is the next tile's first)
                tile_sums = sums;
                sums.start(g, oa, 2 * (n1 / BN) + wn);
            }
            if (sums.upper()) sums.read(st);
            static_for<MS>([&](auto mc) {
                constexpr int m = decltype(mc)::value, s = m / (TM * TN), i = m / TN % TM, j = m % TN;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[p][s][j], af[p][s][i], acc[i][j], 0, 0, 0);
                constexpr int f0 = m * NR / (MS - 2), f1 = (m + 1) * NR / (MS - 2);
                static_for<(f1 < NR ? f1 : NR) - (f0 < NR ? f0 : NR)>([&](auto fc) { read(st, std::integral_constant<int, 1 - p>{}, std::integral_constant<int, f0 + decltype(fc)::value>{}); });
                if constexpr (m / PI < NL && m % PI == 0) load(std::integral_constant<int, m / PI>{}, Set{});
                if constexpr (m / PI < NL && m % PI == 1) load(std::integral_constant<int, m / PI>{}, Load{});
                __builtin_amdgcn_sched_barrier(0);
            });
            sums.add();
            advance();
        };
        typedef std::integral_constant<int, 0> P0;
        typedef std::integral_constant<int, 1> P1;
        int kt = 0;
        for (; kt + 1 < nkt; kt += 2) {
            ktile(P0{}, false);
            ktile(P1{}, kt + 2 == nkt);
        }
        if (kt < nkt) {
            ktile(P0{}, true);
#pragma unroll
            for (int s = 0; s < 2; ++s) {   // (a tile starts with its first fragments in set 0)
#pragma unroll
                for (int i = 0; i < TM; ++i) af[0][s][i] = af[1][s][i];
#pragma unroll
                for (int j = 0; j < TN; ++j) bf[0][s][j] = bf[1][s][j];
            }
        }
        if (fold_bias) load_bias(n1);
        tile_sums.store(g, m0 + wm * WM, split, bad);
        dtl_epilogue<TM, TN, MODE>(g, acc, m0 + wm * WM, n0 + wn * WN, split, fold_bias, smem + DEEP_STAGES * STAGE + wave * dtl_out_bytes(WN), bad);
        m0 = m1;
        n0 = n1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// grid: (workgroups, 1, splits of the contraction); g.k_per_split is a multiple of BK.  SUMS: with g.db (see DtlSums; a kernel of
// its own, since the branches cost a product without sums 3 to 10 %)
template <int BM, int BN, bool A_KC, bool B_KC, int MODE, bool SUMS = false>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_dtl_kernel(GemmArgs g) {
    extern __shared__ __align__(16) char smem[];
    bool       bad   = false;
    const bool split = gridDim.z > 1;
    if (split) {
        const long long k0 = (long long)blockIdx.z * g.k_per_split;
        g.A += A_KC ? k0 : k0 * g.lda;
        g.B += B_KC ? k0 : k0 * g.ldb;
        g.C32 += (long long)blockIdx.z * g.M * g.N;
        if (SUMS) g.db_part += (long long)blockIdx.z * g.M;
        g.K = min(g.k_per_split, g.K - (int)k0);
    }
    if constexpr (BM * BN < 128 * 128) deep_tiles<BM, BN, A_KC, B_KC, MODE, SUMS>(g, blockIdx.x, gridDim.x, split, smem, bad);
    else dtl_tiles<BM, BN, A_KC, B_KC, MODE, SUMS>(g, blockIdx.x, gridDim.x, true, split, smem, bad);
    if (g.found_inf && __any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(g.found_inf, 1);
    }
}

// Several independent weight-gradient problems (both operands output-contiguous) in one launch, tiles numbered one
// problem after the other as in gemm_grouped_kernel; every tile runs its own load stream (no chaining across problems).
template <int BM, int BN>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_dtl_grouped_kernel(GroupArgs ga) {
    extern __shared__ __align__(16) char smem[];
    bool bad_any = false;
    int* flag    = ga.found_inf;
    group_run(ga, smem, bad_any, [&](const int vb) {
        int            first;
        const GemmArgs g = group_problem(ga, vb, first);
        bool           bad = false;
        dtl_tiles<BM, BN, false, false, INTERIOR, false>(g, vb - first, 1 << 30, false, false, smem, bad);
        bad_any |= bad;
    });
    if (flag && __any(bad_any)) {
        if ((threadIdx.x & 63) == 0) atomicOr(flag, 1);
    }
}

template <int BM, int BN>
int launch_dtl_grouped(const GroupArgs& ga, hipStream_t hs) {
    constexpr size_t  lds = dtl_lds(BM, BN);
    static std::once_flag once;
    static hipError_t     attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_dtl_grouped_kernel<BM, BN>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    if (attr_err != hipSuccess) return hip_fail(attr_err, "gemm: hipFuncSetAttribute(LDS size)");
    hipLaunchKernelGGL((gemm_dtl_grouped_kernel<BM, BN>), dim3(ga.share.wgs), dim3(GEMM_THREADS), lds, hs, ga);
    MP_LAUNCH_CHECK("grouped gemm launch (direct-to-LDS)");
    return MP_OK;
}

// Launch (host): the caller has checked dtl_ok.
template <int BM, int BN, bool AKC, bool BKC, int MODE, bool SUMS = false>
int launch_dtl_mode(const GemmArgs& g, dim3 grid, hipStream_t hs) {
    constexpr size_t  lds = BM * BN < 128 * 128 ? deep_lds(BM, BN) : dtl_lds(BM, BN);
    static std::once_flag once;
    static hipError_t     attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_dtl_kernel<BM, BN, AKC, BKC, MODE, SUMS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    if (attr_err != hipSuccess) return hip_fail(attr_err, "gemm: hipFuncSetAttribute(LDS size)");
    hipLaunchKernelGGL((gemm_dtl_kernel<BM, BN, AKC, BKC, MODE, SUMS>), grid, dim3(GEMM_THREADS), lds, hs, g);
    MP_LAUNCH_CHECK("gemm launch (direct-to-LDS)");
    return MP_OK;
}
template <int BM, int BN, bool AKC, bool BKC>
int launch_dtl(const GemmArgs& g, dim3 grid, hipStream_t hs) {
    // an output (bias, residual) of any alignment and width: the forward product of a vocabulary as a tokenizer leaves it
    // (1021 x 12001 over 512: 32.9 us with the register-staged kernel, 23.8 here)
    if constexpr (AKC && BKC) {
        if (!g.aligned) return launch_dtl_mode<BM, BN, AKC, BKC, TAIL>(g, grid, hs);
    }
    return g.M % BM || g.N % BN || g.K % BK ? launch_dtl_mode<BM, BN, AKC, BKC, EDGE>(g, grid, hs) : launch_dtl_mode<BM, BN, AKC, BKC, INTERIOR>(g, grid, hs);
}

// weight gradients with sums (tile: as sums_ride has it)
template <int BM, int BN>
int launch_dtl_sums(const GemmArgs& g, dim3 grid, hipStream_t hs) {
    return g.M % BM || g.N % BN || g.K % BK ? launch_dtl_mode<BM, BN, false, false, EDGE, true>(g, grid, hs)
                                            : launch_dtl_mode<BM, BN, false, false, INTERIOR, true>(g, grid, hs);
}
int launch_dtl_sums_tile(int t, const GemmArgs& g, dim3 grid, hipStream_t hs);

// tile index as in the planner's table; returns MP_E_UNSUPPORTED for shapes this kernel is not built for
template <bool AKC, bool BKC>
int launch_dtl_tile(int t, const GemmArgs& g, dim3 grid, hipStream_t hs) {
    switch (t) {
        case 0: return launch_dtl<256, 256, AKC, BKC>(g, grid, hs);
        case 1: return launch_dtl<256, 128, AKC, BKC>(g, grid, hs);
        case 2: return launch_dtl<128, 256, AKC, BKC>(g, grid, hs);
        case 3: return launch_dtl<128, 128, AKC, BKC>(g, grid, hs);
        case 4: return launch_dtl<128, 64, AKC, BKC>(g, grid, hs);
        case 5: return launch_dtl<64, 128, AKC, BKC>(g, grid, hs);
        case 8:
            if constexpr (AKC && BKC) return launch_dtl<256, 192, AKC, BKC>(g, grid, hs);
            [[fallthrough]];
        default: return MP_E_UNSUPPORTED;
    }
}

}  // namespace mp
