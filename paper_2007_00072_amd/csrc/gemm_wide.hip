// Wide contraction kernels for the large 16-bit contractions, alone or
// several in one grid.
//
// A block of four waves (one per SIMD) computes a 256 x BN tile, BN = 256 or
// 192, each wave 128 x BN/2 with v_mfma_f32_16x16x32 and every accumulator
// in the AGPR file (256 registers at BN = 256).  What bounds it, and why it
// is laid out this way (MI355X, 4096 x 4096 fp16, k-loop time per 1024 of K
// from sweeps over K; the same kernel with parts left out):
//   MFMAs alone on random data 17.2 us (the shader clock settles near
//   2 GHz), global -> LDS copies alone 10.5, LDS fragment reads alone 4.6,
//   MFMAs + reads 18.4, MFMAs + copies 20.8, all of it 22.4
//   (the 8-wave ping-pong kernel, cfg 23: 28-29).
// * 128-wide wave tiles read a fragment from LDS once per 8 MFMAs; 128x64
//   ones (8 waves) need 1.5 times the LDS bytes.
// * 64-wide k-steps: a row of a k-contiguous operand is then one whole
//   128-byte line per step; with 32-wide steps each line left L2 twice.
// * One wave per SIMD hides nothing behind another wave, so the k-loop is
//   free of branches (a scalar branch per copy cost 3 %), fragment reads are
//   one slice (32 of k) ahead, spread over the MFMAs, and copies go out one
//   per 7-8 MFMAs (issued together they hold up the wave).
// * Five 32 KB LDS slots (160 KB) hold A and B chunks of 64 k in turn: chunk
//   c (A of step c/2, or B for odd c) sits in slot c % 5.  The one barrier
//   of step s, early in its second slice, frees the slots of A(s) and B(s)
//   and publishes step s+1; B(s+2) is copied into A(s)'s slot right after
//   it, A(s+2) during the first slice, into the slot B(s-1) left.  So a copy
//   has about a step (1.3 us) to land.
// * Copies are buffer_load ... lds with a scalar base and step offset: no
//   vector address arithmetic in the loop.
// * The MFMAs are written in assembly with the accumulator tied in place:
//   with all 256 AGPRs in use the compiler otherwise rotates accumulators
//   through copies (1.5 instructions per MFMA).
// The result is computed transposed (B fragment as the MFMA's first
// operand), so a lane holds four consecutive columns of one row: float
// outputs are stored as 16-byte pieces straight from the accumulators,
// 16-bit ones staged through LDS with 8-byte writes (instead of 2-byte
// ones) and stored as whole 256-byte row runs.
#include <stddef.h>

#include <algorithm>

#include "gemm.hpp"
#include "internal.hpp"

namespace dm {
namespace {

constexpr int WK = 64;             // k per step
constexpr int SLOT = 32768;        // bytes of one LDS slot
constexpr int WBM = 256;           // rows of a block tile

template <typename P>
__device__ __forceinline__ P pick(P const (&p)[3], int seg) {
    return seg == 0 ? p[0] : (seg == 1 ? p[1] : p[2]);
}

// c += a b on 16x16x32 blocks, c in place.  (Operands come from LDS reads,
// whose waits the compiler inserts; the accumulators are only read after
// wide_settle.)
template <typename T> struct WMfma;
template <> struct WMfma<half_t> {
    typedef half8 frag;
    __device__ __forceinline__ static void run(floatx4& c, frag a, frag b) {
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
    __device__ __forceinline__ static frag ones() {
        const half_t o = (half_t)1.0f;
        return frag{o, o, o, o, o, o, o, o};
    }
};
template <> struct WMfma<bf16_t> {
    typedef bf16x8 frag;
    __device__ __forceinline__ static void run(floatx4& c, frag a, frag b) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
    __device__ __forceinline__ static frag ones() {
        const bf16_t o = (bf16_t)1.0f;
        return frag{o, o, o, o, o, o, o, o};
    }
};
// Row sums of a fragment: c += ones a, in VGPRs (its own wait states: the
// sums of one slice are 8 independent MFMAs, read next at the kernel's end).
__device__ __forceinline__ void rowsum_mfma(floatx4& c, half8 o, half8 a) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(o), "v"(a));
}
__device__ __forceinline__ void rowsum_mfma(floatx4& c, bf16x8 o, bf16x8 a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(o), "v"(a));
}

// 16 bytes per lane from the buffer's base + voff + soff to LDS at m0 + 16
// lane.  m0 is set one MFMA ahead of the copy (set_m0, then copy16 after the
// next MFMA): one wave issues an instruction every 4 cycles, so with its 16
// an MFMA covers three others, and a copy with all of its scalar work in
// one place held up the MFMAs (k-loop 26.0 against 22.5 us per 1024 of k
// with outer-contiguous operands).  Neither statement tells the compiler of
// m0, and before none of the assembly here does it insert wait states:
// tests/test_wide_asm_cpu.py checks both in the assembly that it makes.
__device__ __forceinline__ void set_m0(uint32_t slot, uint32_t ofs) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(slot), "i"(ofs) : "scc", "memory");
}
__device__ __forceinline__ void copy16(u32x4 rsrc, uint32_t voff, uint32_t soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ u32x4 buffer_at(uint64_t base, uint32_t records) {
    return u32x4{(uint32_t)base, (uint32_t)(base >> 32) & 0xffffu, records, 0x00020000u};
}
template <int N>
__device__ __forceinline__ void wait_copies() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v) |
           ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32);
}

// Each operand: init, then per k-step `Step` (scalar state: at(first step),
// advanced by next()), and copy(step, i) of its NV copies.
//
// k-contiguous operand, R rows: LDS row r holds 8 chunks of 16 bytes,
// logical chunk c at c ^ ((r >> 1) & 7) (the 16 rows of one fragment read
// cover all 64 banks once).  Copy i of wave w brings rows 32 i + 8 w .. + 7,
// which any row map with a lowest radix that is a multiple of 8 keeps evenly
// spaced and in one segment.  A single-segment operand (A) has one scalar
// base and a lane offset per copy; one of several segments (B: stacked
// weights) a base per copy and one lane offset.  (Bases per copy for both
// did not fit the scalar registers: they spilled, and a base read back just
// before the copy that uses it needs wait states that the compiler does not
// insert before assembly.)
template <typename T, int R, bool KC, bool SEG>
struct WideOp;
template <typename T, int R>
struct WideOp<T, R, true, false> {
    static constexpr int NV = R / 32;
    uint64_t base;
    uint32_t vo[NV];
    __device__ __forceinline__ void init(const Operand& op, int kb, int, int o0, int omax, int w, int lane) {
        base = (uint64_t)(reinterpret_cast<const T*>(op.ptr[0]) + kb);
        const uint32_t vl =
            (uint32_t)((lane >> 3) * op.row.s0 * 2) + (uint32_t)(((lane & 7) ^ ((w * 4 + (lane >> 4)) & 7)) * 16);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = min(o0 + i * 32 + w * 8, omax - 8);  // (rows past the end: any valid ones)
            int seg = 0;
            vo[i] = vl + (uint32_t)(map_off(op.row, (uint32_t)row, 1, &seg) * 2);
        }
    }
    struct Step { uint32_t soff; };
    __device__ __forceinline__ Step first(const Operand&) const { return Step{0u}; }
    __device__ __forceinline__ void next(const Operand&, Step& t) const { t.soff += WK * 2; }
    __device__ __forceinline__ void copy(const Step& t, int i) const {
        copy16(buffer_at(base, 0xffffffffu), vo[i], t.soff);
    }
    __device__ __forceinline__ static u32x4 frag(const unsigned char* lds, int ob, int q, int lane) {
        return WideOp<T, R, true, true>::frag(lds, ob, q, lane);
    }
};
template <typename T, int R>
struct WideOp<T, R, true, true> {
    static constexpr int NV = R / 32;
    uint64_t base[NV];
    uint32_t vo;
    __device__ __forceinline__ void init(const Operand& op, int kb, int, int o0, int omax, int w, int lane) {
        vo = (uint32_t)((lane >> 3) * op.row.s0 * 2) + (uint32_t)(((lane & 7) ^ ((w * 4 + (lane >> 4)) & 7)) * 16);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = min(o0 + i * 32 + w * 8, omax - 8);
            int seg = 0;
            const int64_t off = map_off(op.row, (uint32_t)row, op.nseg, &seg);
            base[i] = uniform64((uint64_t)(reinterpret_cast<const T*>(pick(op.ptr, seg)) + off + kb)) & 0xffffffffffffull;
        }
    }
    struct Step { uint32_t soff; };
    __device__ __forceinline__ Step first(const Operand&) const { return Step{0u}; }
    __device__ __forceinline__ void next(const Operand&, Step& t) const { t.soff += WK * 2; }
    __device__ __forceinline__ void copy(const Step& t, int i) const {
        copy16(u32x4{(uint32_t)base[i], (uint32_t)(base[i] >> 32), 0xffffffffu, 0x00020000u}, vo, t.soff);
    }
    // lane l: row ob + l % 16, k = 32 q + 8 (l / 16) .. + 7
    __device__ __forceinline__ static u32x4 frag(const unsigned char* lds, int ob, int q, int lane) {
        const int r = ob + (lane & 15), c = q * 4 + (lane >> 4);
        return *reinterpret_cast<const u32x4*>(lds + r * 128 + ((c ^ ((r >> 1) & 7)) * 16));
    }
};
// outer-contiguous operand: LDS keeps [k][outer] rows of 2 R bytes,
// 16-byte chunk c of k-row r at c ^ swz(r); fragments are read with the
// transposing ds_read_b64_tr_b16 (within 16 lanes, lane i receives element
// i % 4 of the 8-byte pieces addressed by lanes i / 4 + 4 j), whose eight
// 4-row groups of two lane groups then fall on different banks.  The buffer of a step ends with its
// last valid k-row, and what lies past a buffer's end is read as zeros.
template <typename T, int R, bool SEG>
struct WideOp<T, R, false, SEG> {
    static_assert(R == 256 || R == 128, "k-rows of 32 or 16 chunks");
    static constexpr int CPR = R / 8, KPC = 256 / CPR, NV = WK / KPC;  // chunks a k-row, k-rows a copy
    uint32_t vo[NV];
    int k0, ke, o0;
    uint32_t pitch;  // bytes of a k-row
    bool plain;      // one stride for every k-row
    __device__ __forceinline__ static int swz(int r) { return 2 * (r & 3) + 8 * ((r >> 3) & 1); }
    __device__ __forceinline__ void init(const Operand& op, int kb, int ke_, int o0_, int omax, int w, int lane) {
        k0 = kb; ke = ke_; o0 = o0_;
        pitch = (uint32_t)(op.row.s0 * 2);
        plain = op.row.r0 == 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int kr = i * KPC + w * (KPC / 4) + lane / CPR, c = (lane % CPR) ^ swz(kr);
            const int o = o0 + c * 8 < omax ? c * 8 : 0;  // (columns past the end: any valid ones)
            vo[i] = (uint32_t)kr * pitch + (uint32_t)(o * 2);
        }
    }
    struct Step { uint64_t base; int k; };
    __device__ __forceinline__ uint64_t base_of(const Operand& op, int k) const {
        int seg = 0;
        const int64_t off = map_off(op.row, (uint32_t)k, op.nseg, &seg);
        return uniform64((uint64_t)(reinterpret_cast<const T*>(pick(op.ptr, seg)) + off + o0));
    }
    __device__ __forceinline__ Step first(const Operand& op) const { return Step{base_of(op, k0), k0}; }
    __device__ __forceinline__ void next(const Operand& op, Step& t) const {
        t.k += WK;
        if (plain) t.base += (uint64_t)pitch * WK;
        else if (t.k < ke) t.base = base_of(op, t.k);
    }
    __device__ __forceinline__ void copy(const Step& t, int i) const {
        // (a step that is copied has at least 8 valid rows)
        copy16(buffer_at(t.base, (uint32_t)min(ke - t.k, WK) * pitch), vo[i], 0u);
    }
    __device__ __forceinline__ static u32x4 frag(const unsigned char* lds, int ob, int q, int lane) {
        typedef short s4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s4 lds_s4;
        const int g = lane >> 4, sl = lane & 15;
        const int r = q * 32 + 8 * g + (sl >> 2);
        const int c = (ob >> 3) + ((sl & 3) >> 1);
        const unsigned char* p = lds + r * (R * 2) + ((c ^ (2 * (sl >> 2) + 8 * (g & 1))) * 16) + (sl & 1) * 8;
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p));
        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + 8 * R)));
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
};

template <bool V> struct Flag { static constexpr bool value = V; };

// RSUM (A outer-contiguous): partial sums of A's rows over k, for
// Epilogue::rsum.  The 2 tiles_n waves that read the same rows share the
// 32-wide slices u = 0, 1, .. round robin; a wave whose turn it is adds its
// A fragments up with MFMAs against ones.
template <typename T, int FM, bool RSUM>
struct RowSums {
    typedef typename WMfma<T>::frag frag;
    floatx4 rs[RSUM ? FM : 1];
    frag ones;
    int next, stride;
    bool on;
    __device__ __forceinline__ RowSums(const GemmArgs& g, int tn, int wn) {
        if constexpr (RSUM) {
            on = g.c.rsum != nullptr;
            stride = g.tiles_n * 2;
            next = tn * 2 + wn;
#pragma unroll
            for (int i = 0; i < FM; ++i) rs[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            // (kept in registers: formed again next to an MFMA it would need
            // wait states that the compiler does not insert before assembly)
            ones = WMfma<T>::ones();
            asm volatile("" : "+v"(ones));
        }
    }
    __device__ __forceinline__ void add(const frag (&a)[FM], int u) {
        if constexpr (RSUM) {
            if (on && u == next) {
                asm volatile("s_nop 3" ::: "memory");
#pragma unroll
                for (int i = 0; i < FM; ++i) rowsum_mfma(rs[i], ones, a[i]);
                next += stride;
            }
        }
    }
    // after the k-loop's last MFMAs have settled
    __device__ __forceinline__ void store(const GemmArgs& g, int mw, int sidx, int tn, int wn, int lane) {
        if constexpr (RSUM) {
#pragma unroll
            for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(rs[i])::"memory");
            if (!on) return;
            float* prow = g.c.rsum + (int64_t)(sidx * stride + tn * 2 + wn) * g.c.rsum_ld;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int m = mw + i * 16 + lane;
                if (lane < 16 && m < g.M) prow[m] = rs[i][0];
            }
        }
    }
};

// The k-loop of one block tile: acc[i][j] of lane l = element (row
// 16 i + l % 16, columns 16 j + 4 (l / 16) .. + 3) of the wave's tile.
template <typename T, int BN, bool AKC, bool BKC, bool RSUM>
__device__ __forceinline__ void wide_loop(const GemmArgs& g, unsigned char* smem, int tm, int tn, int sidx,
                                          floatx4 (&acc)[8][BN / 32]) {
    constexpr int FM = 8, FN = BN / 32, NM = FM * FN, NR = FM + FN;
    typedef WideOp<T, WBM, AKC, false> OA;
    typedef WideOp<T, BN, BKC, true> OB;
    typedef typename WMfma<T>::frag frag;
    // positions: MFMAs of the second slice before the barrier; MFMAs per
    // fragment read in the first and in the second slice; per copy of A
    // (first slice) and of B (second slice)
    constexpr int BP = 8, R0 = NM / NR < 3 ? NM / NR : 3, R1 = (NM - BP) / NR < 3 ? (NM - BP) / NR : 3;
    constexpr int CA = NM / OA::NV, CB = (NM - BP) / OB::NV;
    static_assert(CA > 2 && CB > 2 && R0 * NR <= NM && R1 * NR <= NM - BP && 2 + (OB::NV - 1) * CB < NM - BP, "schedule");

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w >> 1, wn = w & 1;
    const int m0 = tm * WBM, n0 = tn * BN;
    const int kb = sidx * g.kper, ke = min(g.K, kb + g.kper);
    OA da;
    OB db;
    da.init(g.a, kb, ke, m0, g.M, w, lane);
    db.init(g.b, kb, ke, n0, g.N, w, lane);
    const uint32_t base = lds_offset(smem) + (uint32_t)w * 1024u;  // of the wave's part of a copy
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    RowSums<T, FM, RSUM> rs(g, tn, wn);

    const int nk = (ke - kb + WK - 1) / WK;
    frag a[2][FM], b[2][FN];
    // read j of a slice, in the order the MFMAs need them
    auto read = [&](int buf, const unsigned char* A, const unsigned char* B, int q, int j) {
        if (j == 0) a[buf][0] = __builtin_bit_cast(frag, OA::frag(A, wm * 128, q, lane));
        else if (j <= FN) b[buf][j - 1] = __builtin_bit_cast(frag, OB::frag(B, wn * (BN / 2) + (j - 1) * 16, q, lane));
        else a[buf][j - FN] = __builtin_bit_cast(frag, OA::frag(A, wm * 128 + (j - FN) * 16, q, lane));
    };
    auto mma = [&](int buf, int t) { WMfma<T>::run(acc[t / FN][t % FN], b[buf][t % FN], a[buf][t / FN]); };
    // steps 0 and 1 (slots 0..3)
    auto ta = da.first(g.a);
    auto tb = db.first(g.b);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < OA::NV; ++i) {
                set_m0(base + (uint32_t)(2 * s) * SLOT, (uint32_t)i * 4096u);
                asm volatile("s_nop 0" ::: "memory");
                da.copy(ta, i);
            }
#pragma unroll
            for (int i = 0; i < OB::NV; ++i) {
                set_m0(base + (uint32_t)(2 * s + 1) * SLOT, (uint32_t)i * 4096u);
                asm volatile("s_nop 0" ::: "memory");
                db.copy(tb, i);
            }
        }
        da.next(g.a, ta);
        db.next(g.b, tb);
    }
    if (nk >= 2) wait_copies<OA::NV + OB::NV>();
    else wait_copies<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < NR; ++j) read(0, smem, smem + SLOT, 0, j);
    asm volatile("s_nop 7" ::: "memory");  // (accumulator initialisation before the first MFMA)

    uint32_t sA = 0;  // slot of A(s)
    auto adv = [](uint32_t x, int n) { x += n * SLOT; return x >= 5u * SLOT ? x - 5u * SLOT : x; };
    auto step = [&](int s, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;  // step s + 2 exists
        const uint32_t sB = adv(sA, 1), sA1 = adv(sA, 2), sB1 = adv(sA, 3), sA2 = adv(sA, 4);
        const unsigned char *A = smem + sA, *B = smem + sB, *A1 = smem + sA1, *B1 = smem + sB1;
        const uint32_t toA = base + sA2, toB = base + sA;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            mma(0, t);
            if (t % R0 == 0 && t / R0 < NR) read(1, A, B, 1, t / R0);
            if (MORE && t % CA == 1 && t / CA < OA::NV) set_m0(toA, (uint32_t)(t / CA) * 4096u);
            if (MORE && t % CA == 2 && t / CA < OA::NV) da.copy(ta, t / CA);
            __builtin_amdgcn_sched_barrier(0);
        }
        rs.add(a[0], 2 * s);
#pragma unroll
        for (int t = 0; t < BP; ++t) {
            mma(1, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        // step s+1 has landed (of the copies in flight only A(s+2) is
        // younger) and this wave's reads of step s are complete
        if (MORE) wait_copies<OA::NV>();
        else wait_copies<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (MORE) da.next(g.a, ta);
        __builtin_amdgcn_sched_barrier(0);
        // (after the last step the reads are of a stale slot, unused)
#pragma unroll
        for (int t = BP; t < NM; ++t) {
            mma(1, t);
            const int u = t - BP;
            if (u % R1 == 0 && u / R1 < NR) read(0, A1, B1, 0, u / R1);
            if (MORE && u >= 1 && (u - 1) % CB == 0 && (u - 1) / CB < OB::NV) set_m0(toB, (uint32_t)((u - 1) / CB) * 4096u);
            if (MORE && u >= 2 && (u - 2) % CB == 0 && (u - 2) / CB < OB::NV) db.copy(tb, (u - 2) / CB);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (MORE) db.next(g.b, tb);
        rs.add(a[1], 2 * s + 1);
        sA = sA1;
    };
    int s = 0;
#pragma unroll 1
    for (; s + 2 < nk; ++s) step(s, Flag<true>{});
#pragma unroll 1
    for (; s < nk; ++s) step(s, Flag<false>{});
    // the last MFMAs' results are written before anything reads them, and
    // every wave is done with the slots before the epilogue reuses them
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j])::"memory");
    rs.store(g, m0 + wm * 128, sidx, tn, wn, lane);
}

// Float outputs (split partials, or fp32 C through a row map): 16-byte
// pieces, four lanes covering 64 contiguous bytes of a row.
template <int FM, int FN>
__device__ __forceinline__ void wide_store_f32(const GemmArgs& g, const floatx4 (&acc)[FM][FN], int mw, int nw,
                                               int sidx) {
    const int lane = threadIdx.x & 63;
    const int nb = nw + 4 * (lane >> 4);
    const bool part = g.splits > 1;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = mw + i * 16 + (lane & 15);
        if (m >= g.M) continue;
        float* row;
        if (part) {
            row = g.split_ws + ((int64_t)sidx * g.M + m) * g.N;
        } else {
            int seg = 0;
            const int64_t off = map_off(g.c.mmap, (uint32_t)m, g.c.seg_on_m ? g.c.nseg : 1, &seg);
            row = reinterpret_cast<float*>(pick(g.c.ptr, seg)) + off;
        }
#pragma unroll
        for (int j = 0; j < FN; ++j)
            if (nb + j * 16 < g.N) *reinterpret_cast<floatx4*>(row + nb + j * 16) = acc[i][j];
    }
}

// Outputs in the storage type with a residual: 16 rows at a time staged in
// fp32 through the wave's own LDS (a wave's LDS accesses run in order, so no
// barrier), read back as row pieces, the residual added before rounding.
template <typename T, int FM, int FN>
__device__ __forceinline__ void wide_store_resid(const GemmArgs& g, const floatx4 (&acc)[FM][FN], int mw, int nw,
                                                 unsigned char* region) {
    constexpr int WN = FN * 16, PITCH = WN * 4 + 16;
    constexpr int VPR = WN / 8, RPI = 64 / VPR, NPASS = (16 + RPI - 1) / RPI;
    const int lane = threadIdx.x & 63;
    const Epilogue& e = g.c;
    const int rr0 = lane / VPR, vc = (lane % VPR) * 8, n = nw + vc;
    const bool lane_on = lane < RPI * VPR && n < g.N;
    int d = 0;
    const int64_t noff = map_off(e.nmap, (uint32_t)(n < g.N ? n : 0), 1, &d);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int mb = mw + i * 16;
        if (mb >= g.M) break;
#pragma unroll
        for (int j = 0; j < FN; ++j)
            *reinterpret_cast<floatx4*>(region + (lane & 15) * PITCH + (lane >> 4) * 16 + j * 64) = acc[i][j];
        u32x4 hv[NPASS];
        int64_t off[NPASS];
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
            const int rr = p * RPI + rr0, m = mb + rr;
            hv[p] = u32x4{0u, 0u, 0u, 0u};
            off[p] = noff + map_off(e.mmap, (uint32_t)m, 1, &d);
            if (lane_on && rr < 16 && m < g.M)
                hv[p] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(e.resid) + off[p]);
        }
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
            const int rr = p * RPI + rr0;
            if (!lane_on || rr >= 16 || mb + rr >= g.M) continue;
            float a[8], b[8];
            V8<float>::load(reinterpret_cast<const float*>(region + rr * PITCH + vc * 4), a);
            V8<T>::unpack(hv[p], b);
#pragma unroll
            for (int q = 0; q < 8; ++q) a[q] += b[q];
            V8<T>::store(reinterpret_cast<T*>(e.ptr[0]) + off[p], a);
        }
    }
}

// Outputs in the storage type: the wave's whole tile goes to its own LDS
// (8-byte writes of four columns; pitch 16 bytes over the row, so 16 rows
// start on different bank groups) and is read back as 16-byte row pieces in
// one rolled loop.  ACT 1 / 2: the activation operators of
// Epilogue::act_mode on each piece (one wave per SIMD has nothing to hide a
// load behind but its own later pieces: mode 2 keeps the pre-activations of
// two groups of pieces in flight).
template <typename T, int FM, int FN, int ACT>
__device__ __forceinline__ void wide_store(const GemmArgs& g, const floatx4 (&acc)[FM][FN], int mw, int nw,
                                           unsigned char* region) {
    constexpr int WN = FN * 16, PITCH = WN * 2 + 16;
    constexpr int VPR = WN / 8, RPI = 64 / VPR, WM = FM * 16, NP = (WM + RPI - 1) / RPI, U = 4;
    const int lane = threadIdx.x & 63;
    const Epilogue& e = g.c;
    const int rr0 = lane / VPR, vc = (lane % VPR) * 8, n = nw + vc;
    const bool lane_on = lane < RPI * VPR && n < g.N;
    const int rows = min(WM, g.M - mw);  // rows of the tile inside the output
    // pre-activations of pieces p .. p + U - 1
    const T* hp = nullptr;
    u32x4 h0[ACT == 2 ? U : 1], h1[ACT == 2 ? U : 1];
    auto request = [&](u32x4 (&h)[ACT == 2 ? U : 1], int p) {
        if constexpr (ACT == 2) {
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int rr = (p + t) * RPI + rr0;
                h[t] = u32x4{0u, 0u, 0u, 0u};
                if (lane_on && rr < rows) h[t] = *reinterpret_cast<const u32x4*>(hp + (int64_t)(p + t) * RPI * g.ldc);
            }
        }
    };
    if constexpr (ACT == 2) {
        hp = reinterpret_cast<const T*>(e.act_in) + (int64_t)(mw + rr0) * g.ldc + n;
        request(h0, 0);
    }
    u32x4 bias_raw = {0u, 0u, 0u, 0u};
    if constexpr (ACT != 0)
        if (lane_on) bias_raw = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(e.act_bias) + n);
    const bool biased = ACT == 0 && e.bias[0] != nullptr && !e.bias_on_m;
    // a bias along m: the lane's row of each 16-row block
    float bm[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        bm[i] = 0.f;
        if (ACT == 0 && e.bias[0] != nullptr && e.bias_on_m) {
            const int m = mw + i * 16 + (lane & 15);
            int sg = 0;
            const int64_t bo = map_off(e.bias_map, (uint32_t)(m < g.M ? m : 0), e.bias_nseg, &sg);
            bm[i] = to_f(reinterpret_cast<const T*>(pick(e.bias, sg))[bo]);
        }
    }
    unsigned char* wr = region + (lane & 15) * PITCH + (lane >> 4) * 8;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        // bias of the lane's four columns (consecutive indices stay inside
        // one digit: the bias map's lowest radix is a multiple of 8)
        float bn[4] = {0.f, 0.f, 0.f, 0.f};
        if (biased) {
            const int c = nw + j * 16 + 4 * (lane >> 4);
            int sg = 0;
            const int64_t bo = map_off(e.bias_map, (uint32_t)(c < g.N ? c : 0), e.bias_nseg, &sg);
            const T* bp = reinterpret_cast<const T*>(pick(e.bias, sg)) + bo;
#pragma unroll
            for (int r = 0; r < 4; ++r) bn[r] = to_f(bp[r * e.bias_map.s0]);
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            T v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = from_f<T>(ACT == 0 ? acc[i][j][r] + (bn[r] + bm[i]) : acc[i][j][r]);
            *reinterpret_cast<u32x2*>(wr + i * 16 * PITCH + j * 32) = __builtin_bit_cast(u32x2, v);
        }
    }
    const unsigned char* rd = region + rr0 * PITCH + vc * 2;
    if (!g.affine) {
        // through index maps: the column part of an address is the lane's
        // for the whole tile, the row part is taken per row
        int nsg = 0;
        const int64_t noff = map_off(e.nmap, (uint32_t)(n < g.N ? n : 0), e.seg_on_m ? 1 : e.nseg, &nsg);
#pragma unroll 4
        for (int p = 0; p < NP; ++p) {
            const int rr = p * RPI + rr0;
            if (!lane_on || rr >= rows) continue;
            int msg = 0;
            const int64_t off = map_off(e.mmap, (uint32_t)(mw + rr), e.seg_on_m ? e.nseg : 1, &msg) + noff;
            *reinterpret_cast<u32x4*>(reinterpret_cast<T*>(pick(e.ptr, e.seg_on_m ? msg : nsg)) + off) =
                *reinterpret_cast<const u32x4*>(rd + p * RPI * PITCH);
        }
        return;
    }
    const int64_t ix0 = (int64_t)(mw + rr0) * g.ldc + n;  // element index of piece 0
    T* out = reinterpret_cast<T*>(e.ptr[0]) + ix0;
    if constexpr (ACT == 0) {
#pragma unroll 4
        for (int p = 0; p < NP; ++p)
            if (lane_on && p * RPI + rr0 < rows)
                *reinterpret_cast<u32x4*>(out + (int64_t)p * RPI * g.ldc) =
                    *reinterpret_cast<const u32x4*>(rd + p * RPI * PITCH);
    } else {
        float bb[8], cs[8];
        V8<T>::unpack(bias_raw, bb);
#pragma unroll
        for (int q = 0; q < 8; ++q) cs[q] = 0.f;
        T* act = ACT == 1 ? reinterpret_cast<T*>(e.act_out) + ix0 : nullptr;
        auto piece = [&](int p, u32x4 h) {
            if (!lane_on || p * RPI + rr0 >= rows) return;
            const int64_t step = (int64_t)p * RPI * g.ldc;
            const u32x4 v = *reinterpret_cast<const u32x4*>(rd + p * RPI * PITCH);
            float a[8];
            V8<T>::unpack(v, a);
            if constexpr (ACT == 1) {
                // the stored values, then their activation (the bias +
                // activation operator's arithmetic)
                *reinterpret_cast<u32x4*>(out + step) = v;
                act_fwd8(a, bb, e.act);
                dropout8(e.act_dp, (uint64_t)(ix0 + step), a);
                V8<T>::store(act + step, a);
            } else {
                // the activation backward of the (rounded) gradient
                float u[8];
                V8<T>::unpack(h, u);
                dropout8(e.act_dp, (uint64_t)(ix0 + step), a);
                act_grad8(a, u, bb, e.act);
                store_rounded8<T>(out + step, a);
#pragma unroll
                for (int q = 0; q < 8; ++q) cs[q] += a[q];
            }
        };
        if constexpr (ACT == 1) {
#pragma unroll 2
            for (int p = 0; p < NP; ++p) piece(p, u32x4{0u, 0u, 0u, 0u});
        } else {
            static_assert(NP % (2 * U) == 0, "whole double groups of pieces");
#pragma unroll 1
            for (int p = 0; p < NP; p += 2 * U) {
                request(h1, p + U);
#pragma unroll
                for (int t = 0; t < U; ++t) piece(p + t, h0[t]);
                request(h0, p + 2 * U);  // (past the tile: no rows, no loads)
#pragma unroll
                for (int t = 0; t < U; ++t) piece(p + U + t, h1[t]);
            }
            // lanes with the same 8 columns differ by multiples of VPR
            static_assert((VPR & (VPR - 1)) == 0, "column groups of a power-of-two lane count");
#pragma unroll
            for (int d = VPR; d < 64; d <<= 1)
#pragma unroll
                for (int q = 0; q < 8; ++q) cs[q] += __shfl_xor(cs[q], d, 64);
            if (lane < VPR && n < g.N) V8<float>::store(e.act_part + (int64_t)(mw / WM) * g.N + n, cs);
        }
    }
}

// Tile order: groups of 4 tile rows, column-major inside a group.
__device__ __forceinline__ void wide_tile(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int per_group = 4 * tiles_n, grp = t / per_group, first = grp * 4;
    const int gm = min(tiles_m - first, 4), r = t - grp * per_group;
    tm = first + r % gm;
    tn = r / gm;
}

// EP: 0 storage type (bias), 1 / 2 with the activation step, 3 with a residual, 4 float
template <typename T, int BN, bool AKC, bool BKC, bool RSUM, int EP>
__device__ __forceinline__ void wide_block(const GemmArgs& g, unsigned char* smem, int tm, int tn, int sidx) {
    constexpr int FN = BN / 32;
    floatx4 acc[8][FN];
    wide_loop<T, BN, AKC, BKC, RSUM>(g, smem, tm, tn, sidx, acc);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mw = tm * WBM + (w >> 1) * 128, nw = tn * BN + (w & 1) * (BN / 2);
    static_assert(4 * 128 * (FN * 32 + 16) <= 5 * SLOT && 16 * (FN * 64 + 16) <= SLOT, "staging regions");
    if constexpr (EP == 4) wide_store_f32<8, FN>(g, acc, mw, nw, sidx);
    else if constexpr (EP == 3) wide_store_resid<T, 8, FN>(g, acc, mw, nw, smem + w * SLOT);
    else wide_store<T, 8, FN, EP>(g, acc, mw, nw, smem + w * 128 * (FN * 32 + 16));
}

template <typename T, int BN, bool AKC, bool BKC, int EP>
__global__ __launch_bounds__(256) void gemm_wide(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[5 * SLOT];
    const int nt = g.tiles_m * g.tiles_n, total = nt * (g.splits > 1 ? g.splits : 1);
    const int b = (int)blockIdx.x;
    // (blocks reach the 8 XCDs round-robin: each takes one contiguous run)
    const int lid = (total & 7) == 0 ? (b & 7) * (total >> 3) + (b >> 3) : b;
    const int sidx = lid / nt;
    int tm, tn;
    wide_tile(lid - sidx * nt, g.tiles_m, g.tiles_n, tm, tn);
    wide_block<T, BN, AKC, BKC, false, EP>(g, smem, tm, tn, sidx);
}

// The same on a 128x128 tile (waves of 64x64), for outputs with too few
// 256x256 tiles: what bounds it there is the copies (32 KB a step of 512
// MFMA cycles a wave; copies alone reach about 47 bytes a cycle and CU), so
// the five 32 KB slots hold whole steps and copies run four steps ahead.
// The barrier of step s, in its second slice, frees slot s % 5 and publishes
// step s + 1; step s + 5 is copied into the freed slot, three of its eight
// copies right after the barrier, the others during the next step's first
// slice.  (4096 x 1024 x 4096 fp16: the lean 128x128 kernel 45 us.)
template <typename T, bool AKC, bool BKC, int EP, bool RSUM>
__device__ __forceinline__ void mid_block(const GemmArgs& g, unsigned char* smem, int tm, int tn, int sidx) {
    constexpr int BT = 128, FM = 4, FN = 4, NM = FM * FN, NR = FM + FN, BP = 4, ST = 5, HALF = SLOT / 2;
    typedef WideOp<T, BT, AKC, false> OA;
    typedef WideOp<T, BT, BKC, true> OB;
    typedef typename WMfma<T>::frag frag;
    constexpr int NV = OA::NV + OB::NV, EARLY = 3;
    static_assert(NV == 8 && EARLY * 4 + 1 <= NM - BP + 1 && (NV - EARLY - 1) * 4 + 2 < NM + BP, "schedule");
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w >> 1, wn = w & 1;
    const int m0 = tm * BT, n0 = tn * BT;
    const int kb = sidx * g.kper, ke = min(g.K, kb + g.kper);
    OA da;
    OB db;
    da.init(g.a, kb, ke, m0, g.M, w, lane);
    db.init(g.b, kb, ke, n0, g.N, w, lane);
    const uint32_t base = lds_offset(smem) + (uint32_t)w * 1024u;
    floatx4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int nk = (ke - kb + WK - 1) / WK;
    frag a[2][FM], b[2][FN];
    auto read = [&](int buf, const unsigned char* st, int q, int j) {
        if (j == 0) a[buf][0] = __builtin_bit_cast(frag, OA::frag(st, wm * 64, q, lane));
        else if (j <= FN) b[buf][j - 1] = __builtin_bit_cast(frag, OB::frag(st + HALF, wn * 64 + (j - 1) * 16, q, lane));
        else a[buf][j - FN] = __builtin_bit_cast(frag, OA::frag(st, wm * 64 + (j - FN) * 16, q, lane));
    };
    auto mma = [&](int buf, int t) { WMfma<T>::run(acc[t / FN][t % FN], b[buf][t % FN], a[buf][t / FN]); };
    RowSums<T, FM, RSUM> rs(g, tn, wn);
    auto ta = da.first(g.a);
    auto tb = db.first(g.b);
    auto aim = [&](uint32_t slot, int c) {
        set_m0(slot, c < OA::NV ? (uint32_t)c * 4096u : (uint32_t)HALF + (uint32_t)(c - OA::NV) * 4096u);
    };
    auto copy = [&](int c) {
        if (c < OA::NV) da.copy(ta, c);
        else db.copy(tb, c - OA::NV);
    };
    // steps 0 .. 3 and the first copies of step 4
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        if (s < nk) {
#pragma unroll
            for (int c = 0; c < (s < ST - 1 ? NV : EARLY); ++c) {
                aim(base + (uint32_t)s * SLOT, c);
                asm volatile("s_nop 0" ::: "memory");
                copy(c);
            }
        }
        if (s < ST - 1) {
            da.next(g.a, ta);
            db.next(g.b, tb);
        }
    }
    if (nk >= ST) wait_copies<3 * NV + EARLY>();
    else wait_copies<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < NR; ++j) read(0, smem, 0, j);
    asm volatile("s_nop 7" ::: "memory");
    uint32_t at = 0, last = (ST - 1) * SLOT;  // slots of step s and of step s - 1 (s + 4)
    auto step = [&](int s, auto old_c, auto new_c) {
        // OLD: step s + 4 exists (its later copies go out now); NEW: step s + 5
        constexpr bool OLD = decltype(old_c)::value, NEW = decltype(new_c)::value;
        const uint32_t nxt = at + SLOT == ST * SLOT ? 0u : at + SLOT;
        const uint32_t to_old = base + last, to_new = base + at;
        const unsigned char *S0 = smem + at, *S1 = smem + nxt;
        // copy c >= EARLY at MFMA 4 (c - EARLY) + 2 of the step
        auto old_copy = [&](int f) {
            if (OLD && f % 4 == 1 && f / 4 + EARLY < NV) aim(to_old, f / 4 + EARLY);
            if (OLD && f % 4 == 2 && f / 4 + EARLY < NV) copy(f / 4 + EARLY);
        };
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            mma(0, t);
            if (t < NR) read(1, S0, 1, t);
            old_copy(t);
            __builtin_amdgcn_sched_barrier(0);
        }
        rs.add(a[0], 2 * s);
#pragma unroll
        for (int t = 0; t < BP; ++t) {
            mma(1, t);
            old_copy(NM + t);
            __builtin_amdgcn_sched_barrier(0);
        }
        // step s + 1 has landed; steps s + 2 .. s + 4 may still fly
        if (OLD) wait_copies<3 * NV>();
        else if (nk - 2 - s == 2) wait_copies<2 * NV>();
        else if (nk - 2 - s == 1) wait_copies<NV>();
        else wait_copies<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (NEW) {
            da.next(g.a, ta);
            db.next(g.b, tb);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = BP; t < NM; ++t) {
            mma(1, t);
            const int u = t - BP;
            if (u < NR) read(0, S1, 0, u);
            if (NEW && u % 4 == 0 && u / 4 < EARLY) aim(to_new, u / 4);
            if (NEW && u % 4 == 1 && u / 4 < EARLY) copy(u / 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        rs.add(a[1], 2 * s + 1);
        last = at;
        at = nxt;
    };
    int s = 0;
#pragma unroll 1
    for (; s + ST < nk; ++s) step(s, Flag<true>{}, Flag<true>{});
    if (s + ST - 1 < nk) {
        step(s, Flag<true>{}, Flag<false>{});
        ++s;
    }
#pragma unroll 1
    for (; s < nk; ++s) step(s, Flag<false>{}, Flag<false>{});
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j])::"memory");
    rs.store(g, m0 + wm * 64, sidx, tn, wn, lane);
    const int mw = m0 + wm * 64, nw = n0 + wn * 64;
    if constexpr (EP == 4) wide_store_f32<FM, FN>(g, acc, mw, nw, sidx);
    else if constexpr (EP == 3) wide_store_resid<T, FM, FN>(g, acc, mw, nw, smem + w * SLOT);
    else wide_store<T, FM, FN, EP>(g, acc, mw, nw, smem + w * SLOT);
}

template <typename T, bool AKC, bool BKC, int EP, bool RSUM = false>
__global__ __launch_bounds__(256) void gemm_mid(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[5 * SLOT];
    const int nt = g.tiles_m * g.tiles_n, total = nt * (g.splits > 1 ? g.splits : 1);
    const int b = (int)blockIdx.x;
    const int lid = (total & 7) == 0 ? (b & 7) * (total >> 3) + (b >> 3) : b;
    const int sidx = lid / nt;
    int tm, tn;
    wide_tile(lid - sidx * nt, g.tiles_m, g.tiles_n, tm, tn);
    mid_block<T, AKC, BKC, EP, RSUM>(g, smem, tm, tn, sidx);
}

static_assert(offsetof(GemmGroup, g) == 0, "contraction p at p * sizeof(GemmArgs) of the kernel arguments");

// Several contractions: weight gradients (both operands outer-contiguous,
// float output) and input gradients (A k-contiguous, B outer-contiguous,
// residual).
template <typename T>
__global__ __launch_bounds__(256) void gemm_wide_group(GemmGroup grp) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[5 * SLOT];
    const int x = (int)blockIdx.x & 7;
    int ix = (int)blockIdx.x >> 3;  // index among the XCD's blocks
    int t = -1, o = 0;  // o: place in the order of the contractions
    auto at = [&](int i) { return grp.first_last ? (i == 0 ? grp.n - 1 : i - 1) : i; };
    if (grp.spread) {
        // an eighth of every contraction's tiles, contraction by contraction
        for (; o < grp.n; ++o) {
            const int nb = grp.blocks[at(o)], lo = nb * x / 8, hi = nb * (x + 1) / 8;
            if (ix < hi - lo) { t = lo + ix; break; }
            ix -= hi - lo;
        }
    } else {
        // one contiguous run of all tiles
        int total = 0;
        for (int i = 0; i < grp.n; ++i) total += grp.blocks[i];
        const int lo = total * x / 8, hi = total * (x + 1) / 8;
        if (ix < hi - lo) {
            t = lo + ix;
            for (; o < grp.n; ++o) {
                const int nb = grp.blocks[at(o)];
                if (t < nb) break;
                t -= nb;
            }
        }
    }
    if (t < 0 || o >= grp.n) return;
    const int p = __builtin_amdgcn_readfirstlane(at(o));
    t = __builtin_amdgcn_readfirstlane(t);
    // (the contraction's arguments straight from the kernel-argument segment:
    // indexing the by-value argument would copy it to scratch memory)
    typedef const __attribute__((address_space(4))) char* kernarg;
    GemmArgs g;
    __builtin_memcpy(&g, (const void*)((kernarg)__builtin_amdgcn_kernarg_segment_ptr() + (size_t)p * sizeof(GemmArgs)),
                     sizeof(GemmArgs));
    const int nt = g.tiles_m * g.tiles_n, sidx = t / nt;
    int tm, tn;
    wide_tile(t - sidx * nt, g.tiles_m, g.tiles_n, tm, tn);
    if (!g.a.kcontig) wide_block<T, 256, false, false, true, 4>(g, smem, tm, tn, sidx);
    else wide_block<T, 256, true, false, false, 3>(g, smem, tm, tn, sidx);
}

// Split partials of the group's contractions added in split order (float
// outputs): block y takes contraction y.
__global__ __launch_bounds__(256) void wide_group_reduce(GemmGroup grp) {
    const GemmArgs& g = grp.g[blockIdx.y];
    if (g.splits <= 1) return;
    const int64_t plane = (int64_t)g.M * g.N, nv = g.N / 4;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < plane / 4; v += (int64_t)gridDim.x * 256) {
        const int m = (int)(v / nv), n = (int)(v - m * nv) * 4;
        floatx4 a = *reinterpret_cast<const floatx4*>(g.split_ws + v * 4);
        for (int s = 1; s < g.splits; ++s) a += *reinterpret_cast<const floatx4*>(g.split_ws + s * plane + v * 4);
        int seg = 0;
        const int64_t off = map_off(g.c.mmap, (uint32_t)m, g.c.seg_on_m ? g.c.nseg : 1, &seg);
        *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(pick(g.c.ptr, seg)) + off + n) = a;
    }
}

template <typename T, int BN, bool AKC, bool BKC>
void launch_ep(const GemmArgs& g, hipStream_t st) {
    const dim3 grid(g.tiles_m * g.tiles_n * (g.splits > 1 ? g.splits : 1)), block(256);
    const int ep = g.splits > 1 || g.c.out_f32 ? 4 : g.c.act_mode ? g.c.act_mode : g.c.resid ? 3 : 0;
    if (ep == 4) hipLaunchKernelGGL((gemm_wide<T, BN, AKC, BKC, 4>), grid, block, 0, st, g);
    else if (ep == 3) hipLaunchKernelGGL((gemm_wide<T, BN, AKC, BKC, 3>), grid, block, 0, st, g);
    else if (ep == 0) hipLaunchKernelGGL((gemm_wide<T, BN, AKC, BKC, 0>), grid, block, 0, st, g);
    // (activation steps come with one operand layout each)
    if constexpr (AKC && BKC)
        if (ep == 1) hipLaunchKernelGGL((gemm_wide<T, BN, true, true, 1>), grid, block, 0, st, g);
    if constexpr (AKC && !BKC && BN == 256)
        if (ep == 2) hipLaunchKernelGGL((gemm_wide<T, BN, true, false, 2>), grid, block, 0, st, g);
}

template <typename T, bool AKC, bool BKC>
void launch_mid_ep(const GemmArgs& g, hipStream_t st) {
    const dim3 grid(g.tiles_m * g.tiles_n * (g.splits > 1 ? g.splits : 1)), block(256);
    const int ep = g.splits > 1 || g.c.out_f32 ? 4 : g.c.act_mode ? g.c.act_mode : g.c.resid ? 3 : 0;
    if constexpr (!AKC)
        if (ep == 4 && g.c.rsum) {
            hipLaunchKernelGGL((gemm_mid<T, false, BKC, 4, true>), grid, block, 0, st, g);
            return;
        }
    if (ep == 4) hipLaunchKernelGGL((gemm_mid<T, AKC, BKC, 4>), grid, block, 0, st, g);
    else if (ep == 3) hipLaunchKernelGGL((gemm_mid<T, AKC, BKC, 3>), grid, block, 0, st, g);
    else if (ep == 0) hipLaunchKernelGGL((gemm_mid<T, AKC, BKC, 0>), grid, block, 0, st, g);
    if constexpr (AKC && BKC)
        if (ep == 1) hipLaunchKernelGGL((gemm_mid<T, true, true, 1>), grid, block, 0, st, g);
    if constexpr (AKC && !BKC)
        if (ep == 2) hipLaunchKernelGGL((gemm_mid<T, true, false, 2>), grid, block, 0, st, g);
}

template <typename T>
void launch_layout(const GemmArgs& g, int bn, hipStream_t st) {
    if (bn == 128) {
        if (g.a.kcontig && g.b.kcontig) launch_mid_ep<T, true, true>(g, st);
        else if (g.a.kcontig) launch_mid_ep<T, true, false>(g, st);
        else if (g.b.kcontig) launch_mid_ep<T, false, true>(g, st);
        else launch_mid_ep<T, false, false>(g, st);
    } else if (bn == 192) {
        if (g.a.kcontig) launch_ep<T, 192, true, true>(g, st);
        else launch_ep<T, 192, false, true>(g, st);
    } else if (g.a.kcontig && g.b.kcontig) launch_ep<T, 256, true, true>(g, st);
    else if (g.a.kcontig) launch_ep<T, 256, true, false>(g, st);
    else if (g.b.kcontig) launch_ep<T, 256, false, true>(g, st);
    else launch_ep<T, 256, false, false>(g, st);
}

bool operand_ok(const Operand& o, int64_t outer, int64_t K) {
    // byte offsets of a copy fit 32 bits, rows are 16-byte aligned
    if (o.row.s0 < 0 || o.row.s0 >= (1 << 24) || o.row.s0 % 8 || o.row.s1 % 8 || o.row.s2 % 8) return false;
    for (int i = 0; i < (o.nseg > 0 ? o.nseg : 1); ++i)
        if ((uintptr_t)o.ptr[i] % 16) return false;
    if (!o.kcontig) return o.row.r0 % WK == 0;  // (64 k-rows: s0 < 2^24)
    // (the offset of the last row of a segment, in bytes)
    const uint64_t r0 = o.row.r0, r1 = o.row.r1, n = (uint64_t)outer;
    const uint64_t d0 = r0 ? std::min(r0, n) : n, d1 = r0 ? (r1 ? std::min(r1, (n + r0 - 1) / r0) : (n + r0 - 1) / r0) : 1;
    const uint64_t d2 = r0 && r1 && o.nseg <= 1 ? (n + r0 * r1 - 1) / (r0 * r1) : 1;
    const uint64_t last = (d0 - 1) * o.row.s0 + (d1 - 1) * o.row.s1 + (d2 - 1) * o.row.s2;
    return o.row.s1 >= 0 && o.row.s2 >= 0 && o.row.r0 % 8 == 0 && (last + K) * 2 < ((uint64_t)1 << 32);
}

}  // namespace

// Sizes are multiples of 8 (checked by the caller).  Row sums: the 128x128
// tile (and the grouped launch) only.  k in whole steps
// unless both operands are outer-contiguous (their k-rows past the end are
// read as zeros).
bool gemm_wide_ok(const GemmArgs& g, int bn) {
    const Epilogue& e = g.c;
    if (g.batch != 1 || e.alpha != 1.0f || (e.rsum && (bn != 128 || g.a.kcontig || !e.out_f32)) || (g.a.kcontig && g.a.nseg > 1) || !operand_ok(g.a, g.M, g.K) ||
        !operand_ok(g.b, g.N, g.K)) return false;
    if ((g.a.kcontig || g.b.kcontig) && g.K % WK) return false;
    if (bn == 192 && !g.b.kcontig) return false;
    if (g.splits > 1 && (g.kper % WK || (uintptr_t)g.split_ws % 16)) return false;
    auto m8 = [](const IdxMap& m) { return m.s0 % 8 == 0 && m.s1 % 8 == 0 && m.s2 % 8 == 0; };
    if (g.splits > 1) return true;  // (the reduction launch writes the output)
    if (!e.contig_n || e.nmap.s0 != 1 || !m8(e.mmap)) return false;
    for (int i = 0; i < (e.nseg > 0 ? e.nseg : 1); ++i)
        if (!e.ptr[i] || (uintptr_t)e.ptr[i] % 16) return false;
    if (e.out_f32) return e.nmap.r0 == 0 && (e.nseg <= 1 || e.seg_on_m) && !e.resid && !e.bias[0];
    if (e.nmap.r0 % 8 || e.nmap.s1 % 8 || e.nmap.s2 % 8) return false;
    if (e.bias[0] && (e.resid || (!e.bias_on_m && e.bias_map.r0 % 8))) return false;
    if (e.resid && (e.nseg != 1 || (uintptr_t)e.resid % 16)) return false;
    return true;
}

void launch_wide(int dtype, const GemmArgs& args, int bn, hipStream_t st) {
    GemmArgs g = args;
    if (g.splits <= 1) { g.splits = 1; g.kper = g.K; }
    if (dtype == G_F16) launch_layout<half_t>(g, bn, st);
    else launch_layout<bf16_t>(g, bn, st);
}

void launch_wide_group(int dtype, const GemmGroup& group, hipStream_t st) {
    GemmGroup grp = group;
    // blocks of the XCD that takes most
    int most = 0, total = 0;
    for (int i = 0; i < grp.n; ++i) {
        const GemmArgs& g = grp.g[i];
        grp.blocks[i] = g.tiles_m * g.tiles_n * std::max(1, g.splits);
        total += grp.blocks[i];
        if (g.splits <= 1) { grp.g[i].splits = 1; grp.g[i].kper = g.K; }
    }
    for (int x = 0; x < 8; ++x) {
        int c = 0;
        if (grp.spread)
            for (int i = 0; i < grp.n; ++i) c += grp.blocks[i] * (x + 1) / 8 - grp.blocks[i] * x / 8;
        else
            c = total * (x + 1) / 8 - total * x / 8;
        most = std::max(most, c);
    }
    const dim3 grid(8 * most), block(256);
    if (dtype == G_F16) hipLaunchKernelGGL((gemm_wide_group<half_t>), grid, block, 0, st, grp);
    else hipLaunchKernelGGL((gemm_wide_group<bf16_t>), grid, block, 0, st, grp);
}

void launch_wide_reduce(const GemmGroup& grp, hipStream_t st) {
    hipLaunchKernelGGL(wide_group_reduce, dim3(512, grp.n), dim3(256), 0, st, grp);
}

}  // namespace dm
