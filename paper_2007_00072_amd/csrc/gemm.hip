// Contractions, host side: validation, plan and configuration choice of
// every launch, and the float32 kernel.  The 16-bit kernels are in
// gemm_kernels.hpp, compiled for each storage type by gemm_f16.hip and
// gemm_bf16.hip, and in gemm_wide.hip.
#include <algorithm>
#include <mutex>
#include <string.h>
#include <vector>

#include "gemm.hpp"
#include "internal.hpp"

namespace dm {

IdxMap make_map(uint32_t r0, uint32_t r1, int64_t s0, int64_t s1, int64_t s2) {
    IdxMap m{};
    m.r0 = r0; m.r1 = r1; m.s0 = s0; m.s1 = s1; m.s2 = s2;
    auto magic = [](uint32_t d, uint32_t& mul, uint32_t& shr) {
        if (d == 0) { mul = 0; shr = 0; return; }
        uint32_t l = 0;
        while ((1ull << l) < d) ++l;
        mul = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
        shr = l;
    };
    magic(r0, m.mul0, m.shr0);
    magic(r1, m.mul1, m.shr1);
    return m;
}
namespace {

// Pointer of segment `seg` (compile-time indices only, see gemm_kernels.hpp).
template <typename P>
__device__ __forceinline__ P seg_ptr(P const (&p)[3], int seg) {
    return seg == 0 ? p[0] : (seg == 1 ? p[1] : p[2]);
}
constexpr int BK = 64;  // k per step of the 64-wide kernels; split ranges are multiples of it

// True when map m is affine over every aligned block of 32 indices (its
// lowest radix is unbounded or a multiple of 32), so offset(x + d) =
// offset(x) + d * s0 and the segment stay fixed for x % 32 == 0, d < 32.
inline bool block32_linear(const IdxMap& m) { return m.r0 == 0 || m.r0 % 32 == 0; }

// True when a lean kernel with k-steps of bks takes this contraction.
bool lean_ok(const GemmArgs& g, int bks) {
    const Epilogue& e = g.c;
    if (g.K % bks || (g.splits > 1 && g.kper % bks)) return false;
    // outer-contiguous operands: row map affine over every k-step
    if (!g.a.kcontig && g.a.row.r0 % bks) return false;
    if (!g.b.kcontig && g.b.row.r0 % bks) return false;
    if (!g.blk32 || (e.bias[0] && e.bias_on_m)) return false;
    // a residual operand: only on the 128x128 tile (small wave tiles), along
    // n, in the input dtype, through a single pointer
    if (e.resid && (bks != 64 || !e.contig_n || e.out_f32 || e.nseg != 1)) return false;
    return true;
}
// ------------------------------------------------------------ fp32 path
// Float32 contractions on v_mfma_f32_16x16x4f32: a 32x32 block tile of four
// 16x16 waves.  The float32 layers are small (a 64-token layer's largest
// contraction is 64 x 128 x 128), so what counts is the chain of latencies
// in one block, not throughput: k goes in steps of 64, whose operands are
// requested a step ahead as 16-byte pieces along whichever index is
// contiguous (one map evaluation per piece), so a 128-long contraction waits
// for memory once; small tiles give more blocks, and 16x16x4 MFMAs a quarter
// of the serial chain of 32x32x2 ones.  (A 64x64 tile with 16-wide steps
// gathered element by element took 8-25 us for the contractions of that
// layer; this kernel 2-4.)
// LDS holds [outer][k] rows (pitch 68 floats: 16 rows at one 16-byte piece
// cover all banks once); lane l supplies row l % 16 and, over four MFMAs,
// k = 16 j + 4 (l / 16) .. + 3: the order of the sum over k is free as
// long as both operands take the same.  Any map, ragged sizes (zeros past
// M, N, K); the epilogue stores through the output maps.
constexpr int F32_T = 32, F32_K = 64, F32_P = F32_K + 4;
constexpr uint32_t F32_ROW = 1 << 22;  // most tiles in a row of the grid

// Piece p (of 512) of a 32 x 64 operand step: 4 elements along k of row p /
// 16 (k-contiguous), or 4 rows of k-row p / 8 (outer-contiguous).
__device__ __forceinline__ floatx4 f32_piece(const Operand& op, int64_t boff, int p, int o0, int omax, int k0, int kmax) {
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    const int o = op.kcontig ? o0 + (p >> 4) : o0 + (p & 7) * 4;
    const int k = op.kcontig ? k0 + (p & 15) * 4 : k0 + (p >> 3);
    if (o >= omax || k >= kmax) return v;
    int seg = 0;
    const int64_t off = boff + map_off(op.row, (uint32_t)(op.kcontig ? o : k), op.nseg, &seg) + (op.kcontig ? k : o);
    const float* src = reinterpret_cast<const float*>(seg_ptr(op.ptr, seg)) + off;
    const int left = op.kcontig ? kmax - k : omax - o;
    if (left >= 4 && ((uintptr_t)src & 15u) == 0) return *reinterpret_cast<const floatx4*>(src);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t < left) v[t] = src[t];
    return v;
}
__device__ __forceinline__ void f32_put(float* lds, bool kcontig, int p, floatx4 v) {
    if (kcontig) {
        *reinterpret_cast<floatx4*>(lds + (p >> 4) * F32_P + (p & 15) * 4) = v;
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) lds[((p & 7) * 4 + t) * F32_P + (p >> 3)] = v[t];
    }
}

__global__ __launch_bounds__(256) void gemm_f32(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) float sa[F32_T * F32_P];
    __shared__ __attribute__((aligned(16))) float sb[F32_T * F32_P];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    // (tiles past the last one, in a grid of several rows, lie past N: nothing
    // is loaded or stored there; a branch around them cost 0.7 us a launch, a
    // row length from the arguments 0.4)
    const uint32_t tile = blockIdx.z * F32_ROW + blockIdx.x;
    const int m0 = (int)(tile % g.tiles_m) * F32_T, n0 = (int)(tile / g.tiles_m) * F32_T;
    const uint32_t z = blockIdx.y;
    int dummy = 0;
    const int64_t aoff = map_off(g.a.batch, z, 1, &dummy);
    const int64_t boff = map_off(g.b.batch, z, 1, &dummy);
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    floatx4 ra[2], rb[2];
    auto request = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            ra[u] = f32_piece(g.a, aoff, u * 256 + tid, m0, g.M, k0, g.K);
            rb[u] = f32_piece(g.b, boff, u * 256 + tid, n0, g.N, k0, g.K);
        }
    };
    request(0);
    for (int k0 = 0; k0 < g.K; k0 += F32_K) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f32_put(sa, g.a.kcontig, u * 256 + tid, ra[u]);
            f32_put(sb, g.b.kcontig, u * 256 + tid, rb[u]);
        }
        __syncthreads();
        if (k0 + F32_K < g.K) request(k0 + F32_K);
        const float* pa = sa + (wm * 16 + (lane & 15)) * F32_P + (lane >> 4) * 4;
        const float* pb = sb + (wn * 16 + (lane & 15)) * F32_P + (lane >> 4) * 4;
#pragma unroll
        for (int j = 0; j < F32_K / 16; ++j) {
            const floatx4 av = *reinterpret_cast<const floatx4*>(pa + j * 16);
            const floatx4 bv = *reinterpret_cast<const floatx4*>(pb + j * 16);
            // (first operand: columns, so that a lane holds 4 consecutive
            // columns 4 (l / 16) .. + 3 of row l % 16)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[t], av[t], acc, 0, 0, 0);
        }
        __syncthreads();
    }
    const Epilogue& e = g.c;
    const int m = m0 + wm * 16 + (lane & 15), nb = n0 + wn * 16 + 4 * (lane >> 4);
    if (m >= g.M) return;
    int sm = 0;
    const int64_t moff = map_off(e.batch, z, 1, &dummy) + map_off(e.mmap, (uint32_t)m, e.seg_on_m ? e.nseg : 1, &sm);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = nb + r;
        if (n >= g.N) continue;
        float v = acc[r] * e.alpha;
        if (e.bias[0]) {
            int bseg = 0;
            const int64_t bo = map_off(e.bias_map, (uint32_t)(e.bias_on_m ? m : n), e.bias_nseg, &bseg);
            v += reinterpret_cast<const float*>(seg_ptr(e.bias, bseg))[bo];
        }
        int sn = 0;
        const int64_t off = moff + map_off(e.nmap, (uint32_t)n, e.seg_on_m ? 1 : e.nseg, &sn);
        const int seg = e.seg_on_m ? sm : sn;
        if (e.resid) v += reinterpret_cast<const float*>(e.resid)[off];
        reinterpret_cast<float*>(seg_ptr(e.ptr, seg))[off] = v;
    }
}

// Tile configurations: (BM, BN, waves along m, waves along n).
struct TileCfg {
    int bm, bn, wgm, wgn;
};
// 0-4: register-staged kernel; 5-8: asynchronous (global -> LDS) kernel;
// 9-12: asynchronous kernel on 32x32x16 MFMAs; 13: lean 256x256 kernel
// (8 waves of 128x64, four stages of 32-wide k-steps); 14: the general
// 256x256 kernel with the same waves; 15: lean 128x128 kernel (8 waves of
// 64x32, four stages of 64-wide k-steps); 16: lean 128x128 kernel with two
// k groups of 4 waves of 64x64.  Contractions a lean kernel does not take
// run on 14 (for 13) or 11 (for 15, 16).  17: lean 256x256 kernel with 4
// waves of 128x128 (one per SIMD); 18: lean 128x128 kernel with 4 waves of
// 64x64 (one per SIMD): each SIMD's wave then reads every fragment of its
// region once per k-step, where two waves per SIMD read the shared operand
// twice.  Contractions they do not take run on 14 (17) or 11 (18).
// 19: lean 256x192 kernel (4 waves of 128x96) for outputs whose width is a
// multiple of 192 but leaves 256x256 tiles short of the CU count (3072
// columns: 16 x 16 tiles instead of 16 x 12); the 192-wide operand must be
// contiguous along k (else run as 13).  20, 21, 22: the tiles of 17, 19
// and 18 with the interleaved schedule (each MFMA issued next to its share
// of the fragment reads and copies); contractions they do not take run as
// 17, 19 and 18 would.  23, 24: the tile and waves of 13 with the
// ping-pong schedule (the two wave rows alternate between reading a
// k-step's fragments and multiplying them), four and five stages (copies
// two and three k-steps ahead); contractions they do not take run as 13
// would.  25: the ping-pong schedule on a 256x192 tile of 8 waves of 64x96
// (4 wave rows, 2 columns), for a B operand contiguous along k (otherwise
// run as 23): 3072-wide outputs get 16 x 16 tiles, every CU one.  26, 27,
// 28: the wide kernels (gemm_wide.hip), 256x256, 256x192 and 128x128; the
// library's own choices and plan entries' only; contractions they do not take
// run as 23, 25 and 15 would.
constexpr TileCfg CFGS[] = {{256, 256, 2, 4}, {256, 128, 2, 2}, {128, 128, 2, 2}, {256, 64, 4, 1}, {128, 64, 2, 2},
                            {256, 128, 2, 2}, {128, 128, 2, 2}, {256, 64, 4, 1}, {128, 64, 2, 2},
                            {256, 256, 2, 4}, {256, 128, 2, 2}, {128, 128, 2, 2}, {256, 128, 4, 2},
                            {256, 256, 2, 4}, {256, 256, 2, 4}, {128, 128, 2, 4}, {128, 128, 2, 2},
                            {256, 256, 2, 2}, {128, 128, 2, 2}, {256, 192, 2, 2}, {256, 256, 2, 2}, {256, 192, 2, 2}, {128, 128, 2, 2},
                            {256, 256, 2, 4}, {256, 256, 2, 4}, {256, 192, 4, 2},
                            {256, 256, 2, 2}, {256, 192, 2, 2}, {128, 128, 2, 2}};
static_assert(sizeof(CFGS) / sizeof(CFGS[0]) == GEMM_CFG_MID + 1, "configuration table");
constexpr int NCFG = sizeof(CFGS) / sizeof(CFGS[0]);
int64_t ntiles(const TileCfg& c, const GemmArgs& g) {
    return (int64_t)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn) * g.batch;
}

// Tile and split choice, from measurements of the layer's contraction
// shapes on MI355X (every configuration x split 1/2/4): 256x256 tiles when
// they alone give (nearly) every CU a block, otherwise 128x128 tiles, split
// along k for long-k contractions with few output tiles (up to four ways,
// towards one block per CU), each on the wide kernel where that takes the
// contraction and on the lean one otherwise; narrow outputs
// (n <= 64) on the asynchronous 128x64 tile.  A lean kernel hands
// contractions it does not take to its general counterpart.  Explicit
// choices (cfg >= 0, splits > 0) are kept.
void choose(GemmArgs& g) {
    constexpr int64_t CUS = 256;
    const bool split_ok = g.split_ws != nullptr && g.batch == 1;
    int want_split = 1, min_k = 256;
    if (g.cfg < 0 || g.cfg >= NCFG) {
        if (g.N <= 64) {
            g.cfg = 8;
        } else if (ntiles(CFGS[13], g) * 4 >= CUS * 3) {
            // (the 256x192 tiles of cfg 19, which give 3072-wide outputs
            // every CU where 256x256 leaves a quarter idle, measured slower
            // than cfg 13 with its two waves per SIMD; a plan may still pick
            // them).  The ping-pong schedule (cfg 23) runs the k-loop about
            // 10 % faster than cfg 13 at the same fixed cost; row sums are
            // produced by cfg 13 only.
            // The wide kernels, where they take the contraction: 20 % faster
            // k-loop again at the same fixed cost.
            g.cfg = g.c.rsum ? 13 : 23;
            // a 192-wide tile where 256-wide ones leave CUs idle and 192-wide
            // ones still fit in one round (3072-wide outputs: 256 against
            // 192 tiles)
            if (!g.c.rsum && g.c.act_mode != 2 && g.b.kcontig && g.N % 192 == 0 && ntiles(CFGS[23], g) < CUS &&
                ntiles(CFGS[25], g) <= CUS)
                g.cfg = 25;
            if (g.splits <= 1 && g.cfg >= 23 && gemm_wide_ok(g, g.cfg == 25 ? 192 : 256))
                g.cfg = g.cfg == 25 ? GEMM_CFG_WIDE192 : GEMM_CFG_WIDE;
        } else {
            g.cfg = 15;
            const int64_t t = ntiles(CFGS[15], g);
            if (split_ok && g.K >= 2048 && t < CUS * 3 / 4) want_split = (int)std::min<int64_t>(4, std::max<int64_t>(1, CUS / t));
            // Partials that the next kernel sums cost no launch: split any k
            // into pieces of three steps or more, up to four ways (eight
            // pieces of two steps where all partials together stay below
            // 2 MB).  64 x 768 forward 60.1 us with the rule above, 55.0
            // with four, 53.8 with eight; 1024 x 768 71.3, 69.6, 73.3.
            if (split_ok && g.defer && t < CUS * 3 / 4) {
                const bool small = (int64_t)g.M * g.N * 8 * 4 <= 2 << 20;
                want_split = (int)std::min<int64_t>(small ? 8 : 4, CUS / t);
                min_k = small ? 128 : 192;
            }
            // the wide kernels' 128x128 tile from k = 512 on (eight 64-wide
            // steps; its LDS slots hold five); split, a piece may have as few
            // as two steps
            if (g.splits <= 1 && g.K >= 512 && gemm_wide_ok(g, 128)) g.cfg = GEMM_CFG_MID;
        }
    }
    if (g.splits <= 0) {
        int s = split_ok ? want_split : 1;
        while (s > 1 && (g.K / s < min_k || (int64_t)s * g.batch * g.M * g.N > g.split_cap)) --s;
        g.splits = s;
    }
    if (g.splits > 1) {
        const int ksteps = (g.K + BK - 1) / BK;
        g.kper = (ksteps + g.splits - 1) / g.splits * BK;
        g.splits = (g.K + g.kper - 1) / g.kper;
    }
    // a wide kernel that a plan names for what it does not take
    if (g.cfg >= GEMM_CFG_WIDE && !gemm_wide_ok(g, CFGS[g.cfg].bn))
        g.cfg = g.cfg == GEMM_CFG_WIDE ? 23 : g.cfg == GEMM_CFG_WIDE192 ? 25 : 15;
    // the 32x32x16 kernels' epilogues take no bias along m and only output
    // maps affine over 32-wide blocks; of them only the lean 128x128 kernel
    // takes a residual operand
    if (((g.c.bias[0] && g.c.bias_on_m) || !g.blk32) && g.cfg >= 9 && g.cfg < GEMM_CFG_WIDE) g.cfg = 8;
    if (g.c.resid && g.cfg >= 9 && g.cfg < GEMM_CFG_WIDE && g.cfg != 15 && g.cfg != 16 && g.cfg != 18 && g.cfg != 22) g.cfg = 8;
    if (g.cfg == 19 && !g.b.kcontig) g.cfg = 13;
    if (g.cfg == 21 && !g.b.kcontig) g.cfg = 20;
    if (g.cfg == 25 && !g.b.kcontig) g.cfg = 23;
    if ((g.cfg == 13 || g.cfg == 17 || g.cfg == 19 || g.cfg == 20 || g.cfg == 21 || g.cfg == 23 || g.cfg == 24 ||
         g.cfg == 25) &&
        !lean_ok(g, 32))
        g.cfg = 14;
    if ((g.cfg == 15 || g.cfg == 16 || g.cfg == 18 || g.cfg == 22) && !lean_ok(g, 64)) g.cfg = g.c.resid ? 8 : 11;
    // tile counts of the configuration that runs (the fallback from 15 to 8
    // changes the tile width)
    const TileCfg& c = CFGS[g.cfg];
    g.tiles_m = (g.M + c.bm - 1) / c.bm;
    g.tiles_n = (g.N + c.bn - 1) / c.bn;
}

// Classifies the output addressing for the fast store pass.
void set_affine(GemmArgs& g) {
    const Epilogue& e = g.c;
    const bool cn = e.contig_n != 0;
    g.blk32 = block32_linear(e.mmap) && block32_linear(e.nmap);
    g.affine = 0;
    g.bias_mode = 0;
    g.ldc = 0;
    if (e.nseg != 1 || e.mmap.r0 != 0 || e.nmap.r0 != 0) return;
    if (cn ? e.nmap.s0 != 1 : e.mmap.s0 != 1) return;
    if (e.bias[0]) {
        if (e.bias_nseg != 1 || e.bias_map.r0 != 0 || e.bias_map.s0 != 1) return;
        g.bias_mode = (e.bias_on_m != 0) == !cn ? 1 : 2;
    }
    g.ldc = cn ? e.mmap.s0 : e.nmap.s0;
    g.affine = 1;
}

// Whether the lean kernels may stage the output (and split partials)
// through LDS: row-major single-pointer output without a residual, 16-byte
// aligned rows of whole 8-element pieces.
void set_ep_stage(GemmArgs& g) {
    const Epilogue& e = g.c;
    g.ep_stage = 0;
    if (g.N % 8) return;
    if ((uintptr_t)g.split_ws % 16 == 0) g.ep_stage |= 2;
    const bool bias_ok = !e.bias[0] || g.bias_mode == 1;
    if (g.affine && e.contig_n && !e.resid && bias_ok && g.ldc % 8 == 0 && (g.batch == 1 || e.batch.s0 % 8 == 0) &&
        e.batch.r0 == 0 && ((uintptr_t)e.ptr[0] % 16) == 0) {
        g.ep_stage |= 1;
        return;
    }
    // an output through index maps (head permutation, segments): staged
    // when every aligned 8-column piece of a row is 8 contiguous elements
    // at a 16-byte aligned address
    auto mult8 = [](int64_t v) { return v % 8 == 0; };
    bool ok = e.contig_n && !e.resid && !(e.bias[0] && e.bias_on_m) && e.nmap.s0 == 1 &&
              (e.nmap.r0 == 0 || e.nmap.r0 % 8 == 0) && mult8(e.nmap.s1) && mult8(e.nmap.s2) &&
              mult8(e.mmap.s0) && mult8(e.mmap.s1) && mult8(e.mmap.s2) && mult8(e.batch.s0) &&
              mult8(e.batch.s1) && mult8(e.batch.s2);
    for (int i = 0; i < (e.nseg > 0 ? e.nseg : 1); ++i) ok = ok && e.ptr[i] && ((uintptr_t)e.ptr[i] % 16) == 0;
    if (ok) g.ep_stage |= 4;
}

// The plan of the running call (entries keyed by sizes, dtype and operand
// contiguity) and this thread's launch record.
thread_local const dm_plan* t_plan = nullptr;
thread_local bool t_log_on = false;
thread_local std::vector<dm_contract_choice> t_log;

bool same_contraction(const dm_contract_choice& e, const GemmArgs& g, int dtype) {
    return e.M == g.M && e.N == g.N && e.K == g.K && e.batch == g.batch && e.dtype == dtype &&
           e.a_kcontig == (g.a.kcontig ? 1 : 0) && e.b_kcontig == (g.b.kcontig ? 1 : 0);
}

// The running plan's entry for this contraction (the first), if any.
const dm_contract_choice* plan_entry(const GemmArgs& g, int dtype) {
    if (!t_plan) return nullptr;
    for (const dm_contract_choice& e : t_plan->entries)
        if (same_contraction(e, g, dtype)) return &e;
    return nullptr;
}

// A plan entry's tile and split factor for an automatically configured
// contraction; the split factor is cut to what the scratch holds and to
// pieces of 256 of k (128 where the next kernel sums the partials: what
// choose() itself goes down to there).
void apply_plan(GemmArgs& g, int dtype) {
    const dm_contract_choice* e = plan_entry(g, dtype);
    if (!e) return;
    g.cfg = e->tile_cfg;
    int s = e->splits > 1 ? e->splits : 1;
    if (!g.split_ws || g.batch != 1) s = 1;
    while (s > 1 && (g.K / s < (g.defer ? 128 : 256) || (int64_t)s * g.batch * g.M * g.N > g.split_cap)) --s;
    g.splits = s;
}

// Keeps the activation step only where the staged epilogue takes it:
// unsplit lean 256x256 or 128x128 kernel of 8 waves (2 wave rows: cfg 13,
// 15 and the ping-pong forms of 13, 23 and 24; mode 1 also on the 256x192
// ping-pong tile, cfg 25), staged
// row-major output, 16-bit storage, no alpha scaling or bias; mode 1 with A
// and B contiguous along k, mode 2 with A contiguous along k and B along
// n, its partial rows (2 per tile row) within act_part_cap.  Returns the
// partial rows mode 2 writes (1 for mode 1), 0 when not taken.
int settle_act(GemmArgs& g, int dtype) {
    const Epilogue& e = g.c;
    // (cfg 25, 4 wave rows and 96-column waves, takes mode 1 only: mode 2's
    // partial rows assume 2 wave rows and its column groups a power-of-two
    // lane count)
    const bool tile_ok = g.cfg == 13 || g.cfg == 15 || g.cfg == 23 || g.cfg == 24 || g.cfg == GEMM_CFG_WIDE ||
                         g.cfg == GEMM_CFG_MID ||
                         ((g.cfg == 25 || g.cfg == GEMM_CFG_WIDE192) && e.act_mode == 1);
    bool ok = e.act_mode && dtype != G_F32 && tile_ok && !e.rsum && g.splits <= 1 &&
              (g.ep_stage & 1) && !e.out_f32 && !e.bias[0] && e.alpha == 1.0f && e.act_bias && g.batch == 1;
    int parts = 1;
    if (ok && e.act_mode == 1) ok = g.a.kcontig && g.b.kcontig && e.act_out && ((uintptr_t)e.act_out % 16) == 0;
    else if (ok && e.act_mode == 2) {
        parts = g.tiles_m * 2;
        ok = g.a.kcontig && !g.b.kcontig && e.act_in && e.act_part && parts <= e.act_part_cap &&
             ((uintptr_t)e.act_in % 16) == 0 && ((uintptr_t)e.act_part % 16) == 0;
    } else {
        ok = false;
    }
    if (!ok) g.c.act_mode = 0;
    return ok ? parts : 0;
}

thread_local int t_act_parts = 0;

thread_local int t_rsum_parts = 0;
thread_local int t_deferred = 0;

// Keeps the row-sum request only where the kernel that runs produces it
// (the lean 256x256 and 128x128 tiles, both 4 wave tiles wide, and the wide
// 128x128 one, unsplit, A outer-contiguous) and its partial rows fit.
void settle_rowsums(GemmArgs& g) {
    // (partial rows: one per wave along n and tile column)
    const int nw = g.tiles_n * (g.cfg == GEMM_CFG_MID ? 2 : 4);
    const bool ok = g.c.rsum != nullptr && (g.cfg == 13 || g.cfg == 15 || g.cfg == GEMM_CFG_MID) && g.splits <= 1 && !g.a.kcontig && g.batch == 1 &&
                    nw <= g.c.rsum_cap && g.c.rsum_ld >= g.M;
    t_rsum_parts = ok ? nw : 0;
    if (!ok) g.c.rsum = nullptr;
}

// x: the contraction as asked for (g may run its transpose)
void log_launch(const GemmArgs& g, int dtype, const GemmArgs* x = nullptr) {
    if (!t_log_on) return;
    if (!x) x = &g;
    dm_contract_choice r{};
    r.M = x->M; r.N = x->N; r.K = x->K; r.batch = x->batch; r.dtype = dtype;
    r.a_kcontig = x->a.kcontig ? 1 : 0; r.b_kcontig = x->b.kcontig ? 1 : 0;
    r.tile_cfg = g.cfg; r.splits = g.splits > 1 ? g.splits : 1;
    strncpy(r.label, trace_current_label(), sizeof(r.label) - 1);
    t_log.push_back(r);
}

}  // namespace

const dm_plan* current_plan() { return t_plan; }
int gemm_deferred_splits() { return t_deferred; }
int gemm_rowsum_parts() { return t_rsum_parts; }

static int prepare(GemmArgs& g, int dtype, bool pair);

bool gemm_act_fusable(int dtype, const GemmArgs& args) {
    if (dtype == G_F32 || args.M <= 0 || args.N <= 0 || args.K <= 0 || args.batch != 1) return false;
    GemmArgs g = args;
    if (prepare(g, dtype, false)) return false;
    return settle_act(g, dtype) > 0;
}

int gemm_act_parts() { return t_act_parts; }
PlanScope::PlanScope(const dm_plan* p) : prev(t_plan) { t_plan = p; }
PlanScope::~PlanScope() { t_plan = prev; }
int current_attn_path() { return t_plan ? t_plan->attn_path : 0; }

FusedLayout fused_layout(int dtype, int64_t T, int I, int F) {
    (void)F;
    FusedLayout f{};
    const dm_layout_choice c = t_plan ? t_plan->layout : dm_layout_choice{-1, -1, -1, -1};
    f.ln_form = c.ln_bwd_form > 0 ? c.ln_bwd_form : 0;
    f.ln_lanes = c.ln_lanes > 0 ? c.ln_lanes : 0;
    f.dO_t = !ln_bwd_uses_split(I, dtype, f.ln_form) ? 0 : c.dO_transposed < 0 ? 2 : c.dO_transposed;
    f.dH_t = dtype != DM_F32 && T % 8 == 0 && c.dH_transposed == 1;
    return f;
}

void plan_log_set(bool on) {
    t_log_on = on;
    if (on) t_log.clear();
}

int plan_log_copy(dm_contract_choice* out, int cap) {
    for (int i = 0; i < cap && i < (int)t_log.size(); ++i) out[i] = t_log[i];
    return (int)t_log.size();
}

// The same contraction with its outputs transposed (C^T = B^T A^T): the
// operands and the output indexes trade places.
static GemmArgs transposed(const GemmArgs& x) {
    GemmArgs g = x;
    std::swap(g.M, g.N);
    std::swap(g.a, g.b);
    Epilogue& e = g.c;
    std::swap(e.mmap, e.nmap);
    e.contig_n = !e.contig_n;
    e.seg_on_m = e.nseg > 1 ? !e.seg_on_m : e.seg_on_m;
    e.bias_on_m = e.bias[0] ? !e.bias_on_m : e.bias_on_m;
    return g;
}

// Validation, plan and configuration of a 16-bit contraction; `pair`: when
// no plan entry fixes the configuration, ask for the lean 128x128 kernel
// unsplit (what a paired launch runs).
static int prepare(GemmArgs& g, int dtype, bool pair) {
    if (g.K % 8 || g.M % 8 || g.N % 8)
        return set_error(DM_ERR_UNSUPPORTED, "contraction sizes must be multiples of 8");
    if (g.c.bias[0] && ((g.c.bias_on_m != 0) == (g.c.contig_n == 0)) && g.c.bias_map.r0 % 8 != 0)
        return set_error(DM_ERR_UNSUPPORTED, "bias map radix along the output vector must be a multiple of 8");
    if (!g.split_ws) g.splits = 1;
    set_affine(g);
    set_ep_stage(g);
    g.defer = g.defer && !pair && g.batch == 1 && g.affine && g.c.contig_n && g.ldc == g.N && !g.c.bias[0] &&
              !g.c.resid && !g.c.rsum && !g.c.act_mode && !g.c.out_f32 && g.c.alpha == 1.f;
    if (g.cfg < 0) apply_plan(g, dtype);
    // an output contiguous along m (the paper's [i][b][j] order) as its
    // transpose, where the wide kernels then take it: they store along n
    if ((g.cfg < 0 || g.cfg >= GEMM_CFG_WIDE) && !pair && !g.c.contig_n && !g.c.rsum && !g.c.act_mode && g.batch == 1 && g.K >= 512 && g.M > 64) {
        GemmArgs t = transposed(g);
        set_affine(t);
        set_ep_stage(t);
        if (gemm_wide_ok(t, 128)) g = t;
    }
    if (pair && g.cfg < 0) { g.cfg = 15; g.splits = 1; }
    choose(g);
    g.defer = g.defer && g.splits > 1;
    if (g.splits > 1 && (int64_t)g.splits * g.batch * g.M * g.N > g.split_cap)
        return set_error(DM_ERR_WORKSPACE, "split-k scratch too small");
    if ((int64_t)g.batch * g.splits > 65535) return set_error(DM_ERR_UNSUPPORTED, "contraction grid too large");
    return 0;
}

int launch_gemm(int dtype, const GemmArgs& args, hipStream_t st) {
    t_rsum_parts = 0;
    t_deferred = 0;
    t_act_parts = 0;
    GemmArgs g = args;
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return 0;
    if (g.K <= 0) return set_error(DM_ERR_ARG, "contraction with K <= 0");
    if (g.batch > 65535) return set_error(DM_ERR_UNSUPPORTED, "contraction batch above 65535");
    if (dtype == G_F32) {
        g.tiles_m = (g.M + F32_T - 1) / F32_T;
        g.tiles_n = (g.N + F32_T - 1) / F32_T;
        if ((int64_t)((g.M + 63) / 64) * g.batch > 65535)
            return set_error(DM_ERR_UNSUPPORTED, "fp32 contraction grid too large");
        // (a grid holds less than 2^32 threads along x, 68 GB of output: more
        // tiles go in several rows; the indexes past the last tile fit too)
        const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n, rows = (tiles + F32_ROW - 1) / F32_ROW;
        if (rows > 512 || (rows * F32_ROW / g.tiles_m + 1) * F32_T > INT32_MAX)
            return set_error(DM_ERR_UNSUPPORTED, "fp32 contraction grid too large");
        dim3 grid((unsigned)std::min<int64_t>(tiles, F32_ROW), g.batch, (unsigned)rows);
        hipLaunchKernelGGL(gemm_f32, grid, dim3(256), 0, st, g);
        g.cfg = -1;
        log_launch(g, dtype);
    } else {
        if (int rc = prepare(g, dtype, false)) return rc;
        settle_rowsums(g);
        const int ap = settle_act(g, dtype);
        t_act_parts = g.c.act_mode == 2 ? ap : 0;
        if (g.cfg >= GEMM_CFG_WIDE) {
            launch_wide(dtype, g, CFGS[g.cfg].bn, st);
            if (g.splits > 1 && !g.defer) {
                if (dtype == G_F16) launch_reduce_f16(g, st);
                else launch_reduce_bf16(g, st);
            }
        } else if (dtype == G_F16) launch_tiles_f16(g, st);
        else launch_tiles_bf16(g, st);
        if (g.defer) t_deferred = g.splits;
        log_launch(g, dtype, &args);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return set_error(DM_ERR_DEVICE, "contraction launch: %s", hipGetErrorString(err));
    return 0;
}

// ------------------------------------------------------------ groups
// Expected times (us).  A wide 256x256 tile takes 1.4 us per 64-wide k-step
// and 9 us for its prologue and stores (one round of a group in the encoder
// backward, 1024 wide, 64 to 1024 tokens: 17.6 to 38.7 us, 1.41 a step and 16
// fixed; 4096 tokens, every CU busy: 118); the 128x128 kernels 0.57 us per
// step and round of 256 tiles and 7 us (the wide one there, 512 to 8192
// tokens: 11.9 to 81.3 us, 0.54 a step and 7.6 fixed); a launch costs about
// 3 us on top, and split partials are written and read back at about 4 TB/s.
// Against the times measured (backward us, separate launches less the group,
// 48 widths and token counts from 512 x 8192 to 2048 x 2048): where the model
// expects more than 12 us from the group, it gives 14 to 250; below that its
// sign is not to be trusted (expected 10.0 / 7.0 / 11.1 / 1.7 / 7.7 / 6.9 at
// 896 x 1024, 960 x 512, 1088 x 768, 1088 x 1024, 1152 x 1536, 1280 x 1024:
// measured -8 / -9 / -4 / -4 / +6 / +5), so separate launches keep those,
// unless the token count is ragged (960 x 400: the general kernels that
// separate launches then run are 40 us slower).  Which of the splits, and
// whether the input gradient goes along, the same constants pick well (other
// fits that describe each kernel better lost up to 12 % there).
namespace {
constexpr double WIDE_STEP = 1.4, WIDE_FIX = 9.0, LEAN_STEP = 0.57, LEAN_FIX = 7.0, LAUNCH = 3.0, GROUP_MARGIN = 12.0;

double ceil_div(double a, double b) { return (double)(int64_t)((a + b - 1) / b); }

double expect_single(const GemmArgs& x) {
    const double t256 = ceil_div(x.M, 256) * ceil_div(x.N, 256), steps = ceil_div(x.K, 64);
    if (t256 * 4 >= 256 * 3 && !x.c.rsum) return LAUNCH + ceil_div(t256, 256) * (WIDE_STEP * steps + WIDE_FIX);
    const double t128 = ceil_div(x.M, 128) * ceil_div(x.N, 128);
    double s = 1, red = 0;
    if (x.K >= 2048 && t128 < 192) {
        s = std::min(4.0, std::max(1.0, (double)(int64_t)(256 / t128)));
        if (s > 1) red = LAUNCH + 2 * s * x.M * x.N * 4.0 / 4e6;
    }
    return LAUNCH + red + ceil_div(t128 * s, 256) * (LEAN_STEP * ceil_div(steps, s) + LEAN_FIX);
}

// Time until `nw` blocks of tw each and then `nb` blocks of tb each are done
// on 256 CUs, longest first.
double makespan(int64_t nw, double tw, int64_t nb, double tb) {
    constexpr int64_t CUS = 256;
    const int64_t full = nw / CUS, rest = nw % CUS;  // CUs with full + 1 long blocks, and with full
    if (nb == 0) return (full + (rest ? 1 : 0)) * tw;
    double best = 1e30;
    // the last block is short: try every count of short blocks on the CUs
    // with fewer long ones
    for (int64_t k = 0; k <= (nb + CUS - rest - 1) / (CUS - rest); ++k) {
        const double t = std::max(full * tw + k * tb, (full + (rest ? 1 : 0)) * tw);
        int64_t done = (CUS - rest) * (int64_t)((t - full * tw + 1e-9) / tb);
        if (rest) done += rest * (int64_t)((t - (full + 1) * tw + 1e-9) / tb);
        if (done >= nb) { best = t; break; }
    }
    return best;
}
}  // namespace

int plan_gemm_group(int dtype, const GemmArgs* gs, int n, GemmGroup* grp) {
    if (dtype == G_F32 || n < 2 || n > GEMM_GROUP_MAX) return 0;
    double separate = 0, expect_input = 0;
    int64_t nw = 0, nb = 0;
    int kw = 0, kb = 0, weights = 0;
    int want = 0;  // split factor that the plan names for the weight gradients
    for (int i = 0; i < n; ++i) {
        GemmArgs& g = grp->g[i];
        g = gs[i];
        if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.M % 8 || g.N % 8 || g.K % 8) return 0;
        // (entries may name what a grouped launch reports; one that gives the
        // input gradient another kernel leaves only that one out)
        bool own_launch = false;
        if (const dm_contract_choice* e = plan_entry(g, dtype)) {
            own_launch = e->tile_cfg != GEMM_CFG_WIDE || (g.a.kcontig ? e->splits > 1 : want && want != e->splits);
            if (own_launch && !g.a.kcontig) return 0;
            if (!g.a.kcontig) want = e->splits;
        }
        set_affine(g);
        set_ep_stage(g);
        g.splits = 1;
        g.kper = g.K;
        g.cfg = GEMM_CFG_WIDE;
        GemmArgs t = g;
        t.c.rsum = nullptr;
        if (!gemm_wide_ok(t, 256)) return 0;
        g.tiles_m = (g.M + 255) / 256;
        g.tiles_n = (g.N + 255) / 256;
        const double single = expect_single(g);
        if (!g.a.kcontig) {
            if (g.b.kcontig || !g.c.out_f32 || (i > 0 && (gs[i].K != gs[0].K || gs[i].c.rsum))) return 0;
            nw += (int64_t)g.tiles_m * g.tiles_n;
            kw = g.K;
            ++weights;
        } else {
            if (i != n - 1 || g.b.kcontig || g.c.out_f32 || !g.c.resid) return 0;
            nb = own_launch ? 0 : (int64_t)g.tiles_m * g.tiles_n;
            kb = g.K;
            expect_input = single;
        }
        separate += single;
    }
    if (weights == 0) return 0;
    // split factor of the weight gradients (the same for all), with and
    // without the input gradient in the grid
    const double tb = WIDE_STEP * ((kb + 63) / 64) + WIDE_FIX;
    double best = separate - (kw % 64 == 0 ? GROUP_MARGIN : 0.0);
    int best_s = 0, best_n = 0;
    for (int s = 1; s <= 4; ++s) {
        int64_t floats = 0, outs = 0;
        const int kper = ((kw + 63) / 64 + s - 1) / s * 64;
        if (s > 1 && (kper < 512 || !gs[0].split_ws)) break;
        for (int i = 0; i < weights; ++i) outs += (int64_t)gs[i].M * gs[i].N;
        floats = s * outs;
        if (s > 1 && floats > gs[0].split_cap) break;
        if (want && s != want) continue;
        const double tw = WIDE_STEP * (kper / 64) + WIDE_FIX;
        const double red = s > 1 ? LAUNCH + 2.0 * floats * 4 / 4e6 : 0;
        // (a grid that leaves more than a quarter of the CUs idle is left to
        // the 128x128 kernels and their paired launch)
        const double alone = LAUNCH + makespan(nw * s, tw, 0, 0) + red + expect_input;
        if (nw * s >= 192 && alone < best) { best = alone; best_s = s; best_n = weights; }
        if (nb && nw * s + nb >= 192) {
            const double together = LAUNCH + (tw >= tb ? makespan(nw * s, tw, nb, tb) : makespan(nb, tb, nw * s, tw)) + red;
            if (together < best) { best = together; best_s = s; best_n = n; }
        }
    }
    if (!best_s) return 0;
    int64_t at = 0, total = 0;
    for (int i = 0; i < best_n; ++i) {
        GemmArgs& g = grp->g[i];
        if (i < weights && best_s > 1) {
            g.kper = ((kw + 63) / 64 + best_s - 1) / best_s * 64;
            g.splits = (g.K + g.kper - 1) / g.kper;
            g.split_ws = gs[0].split_ws + at;
            at += (int64_t)g.splits * g.M * g.N;
        }
        total += (int64_t)g.tiles_m * g.tiles_n * g.splits;
    }
    grp->n = best_n;
    // longer blocks first
    if (best_n > weights && (kb + 63) / 64 > (grp->g[0].kper + 63) / 64) grp->first_last = 1;
    else grp->first_last = 0;
    grp->spread = total > 256;
    // row sums of the first contraction, where its partial rows fit
    GemmArgs& g0 = grp->g[0];
    if (g0.c.rsum && (g0.splits * g0.tiles_n * 2 > g0.c.rsum_cap || g0.c.rsum_ld < g0.M)) g0.c.rsum = nullptr;
    return best_n;
}

int launch_gemm_group(int dtype, const GemmGroup& grp, hipStream_t st) {
    t_rsum_parts = grp.g[0].c.rsum ? grp.g[0].splits * grp.g[0].tiles_n * 2 : 0;
    t_act_parts = 0;
    launch_wide_group(dtype, grp, st);
    bool split = false;
    for (int i = 0; i < grp.n; ++i) {
        log_launch(grp.g[i], dtype);
        split = split || grp.g[i].splits > 1;
    }
    if (split) {
        trace_next("reduce");
        launch_wide_reduce(grp, st);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return set_error(DM_ERR_DEVICE, "contraction launch: %s", hipGetErrorString(err));
    return 0;
}

int launch_gemm_pair(int dtype, const GemmArgs& x0, const GemmArgs& x1, hipStream_t st) {
    constexpr int64_t CUS = 256;
    t_rsum_parts = 0;
    if (dtype != G_F32 && x0.batch == 1 && x1.batch == 1 && x0.M > 0 && x0.N > 0 && x0.K > 0 && x1.M > 0 &&
        x1.N > 0 && x1.K > 0 && x0.a.kcontig == x1.a.kcontig && x0.b.kcontig == x1.b.kcontig) {
        GemmArgs g0 = x0, g1 = x1;
        if (int rc = prepare(g0, dtype, true)) return rc;
        if (int rc = prepare(g1, dtype, true)) return rc;
        // together the two fill the chip with one block per CU (fewer tiles
        // would leave CUs idle for the whole reduction, where separate
        // launches split it)
        const int64_t tiles = (int64_t)g0.tiles_m * g0.tiles_n + (int64_t)g1.tiles_m * g1.tiles_n;
        if (g0.cfg == 15 && g1.cfg == 15 && g0.splits == 1 && g1.splits == 1 && tiles >= CUS * 3 / 4 &&
            tiles <= CUS) {
            // the pair runs lean 128x128 tiles unsplit: row sums of either
            // operand A are produced (the first contraction's are reported)
            settle_rowsums(g1);
            settle_rowsums(g0);
            if (dtype == G_F16) launch_pair_f16(g0, g1, st);
            else launch_pair_bf16(g0, g1, st);
            log_launch(g0, dtype);
            log_launch(g1, dtype);
            hipError_t err = hipGetLastError();
            if (err != hipSuccess) return set_error(DM_ERR_DEVICE, "contraction launch: %s", hipGetErrorString(err));
            return 0;
        }
    }
    if (int rc = launch_gemm(dtype, x0, st)) return rc;
    const int first_parts = t_rsum_parts;
    trace_next("2");
    const int rc = launch_gemm(dtype, x1, st);
    t_rsum_parts = first_parts;
    return rc;
}

}  // namespace dm
