// conv_triple.hip -- the float convolution layer on the bf16 matrix
// instructions: every float operand as the exact sum of three bf16 terms.
//
// Why.  The float matrix instructions do 157 TFLOP/s and the float GEMMs of
// this library reach 70-80% of it; the bf16 ones do sixteen times as much.  A
// float has 24 significant bits and a bf16 eight, so x = x0 + x1 + x2 with
// x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1 (each rounded to nearest
// even) is exact (see kScale for the smallest floats), and
//   x * y = x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0) + rest,
// the rest at most 2^-24 of the product (2^-26.5 in the mean square), is six
// bf16 products, each exact in the float accumulator, at sixteen times the
// rate.  The accumulator of the first products is rounded once per 16 reduction
// elements (32x32x16) instead of once per 2, the small products have one of
// their own, and the sums come out closer to the 64-bit ones than the float
// instructions' (conv2 at N = 256: forward 2.1e-7 of the norm against
// 6.4e-7, data gradient 2.7e-7 / 6.6e-7, weight gradient 4.3e-7 / 5.1e-7).
//
// Measured at N = 256 (GEMM launches alone, us, float path -> here): conv2
// forward 890 -> 544, data gradient 937 -> 647, weight gradient 944 -> 525;
// conv3 628 -> 321, 620 -> 311, 630 -> 330; conv4 491 -> 266, 496 -> 256, 492 ->
// 282; conv5 318 -> 171, 341 -> 181, 323 -> 182.  That is 1.06-1.48 PFLOP/s of
// bf16 products.  The matrix units are 47-72% busy (counters), at a clock that
// falls as they get busier: conv2's data gradient 47% at 2.30 GHz, conv3's
// forward 72% at 1.83, where the float kernels hold 2.4 GHz at 70%.  A busier
// pipeline so gains less than its share.
//
// Operand staging.  Each operand is first rewritten in the workspace as
// channel-contiguous units of 8 channels x 3 terms (48 bytes):
//   X3[n][hp][wp][c / 8][term][c % 8]
// on a zero-bordered grid, each group's channels padded with zeros to a
// multiple of 8 (Cgp), as the bf16 path stages its single term.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace caffe_hip {

typedef uint16_t bf16_t;

namespace {

constexpr int kUnit = 48;    // bytes of one unit: 8 channels x 3 terms x 2
constexpr int kStageU = 4;   // units per operand row and stage (32 channels)
constexpr int kRowC = 12;    // 16-byte chunks per operand row and stage

// Slot of unit j within its term's four chunks of LDS row r: j ^ row_swz(r).
__device__ __forceinline__ int row_swz(int r) { return (-(r >> 2)) & 3; }

// Terms are those of 2^16 x: a float's last bit is 2^-149 or more and bf16's
// smallest value 2^-133, so every float down to the subnormals is the exact sum
// of its terms (unscaled, the third term was lost below 2^-110: an error of
// 2^-16 at 2^-118, all of it at 2^-136).  The sums are divided by 2^32 at the
// end.
constexpr float kScale = 65536.f;
constexpr float kUnscale = 1.f / (65536.f * 65536.f);

// A float that its first term can't stand for -- infinity, NaN, from 2^112 (less
// half a bf16 step) on -- is staged as this NaN and its own upper and lower 16
// bits.  The NaN reaches every output that the value enters, and such
// outputs are formed again in float arithmetic (x3_float, the end of both
// kernels).
constexpr uint32_t kMark = 0x7fc0;

// The three bf16 terms of a pair of floats, packed (x low, y high).
__device__ __forceinline__ void split_pair(float x, float y, uint32_t t[3])
{
    const uint32_t ux = __builtin_bit_cast(uint32_t, x), uy = __builtin_bit_cast(uint32_t, y);
    x *= kScale;
    y *= kScale;
    t[0] = f32x2_to_bf16x2_rne(x, y);
    const float rx = x - __builtin_bit_cast(float, t[0] << 16);
    const float ry = y - __builtin_bit_cast(float, t[0] & 0xffff0000u);
    t[1] = f32x2_to_bf16x2_rne(rx, ry);
    t[2] = f32x2_to_bf16x2_rne(rx - __builtin_bit_cast(float, t[1] << 16),
                               ry - __builtin_bit_cast(float, t[1] & 0xffff0000u));
    const uint32_t ax = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
    const uint32_t ay = __builtin_bit_cast(uint32_t, y) & 0x7fffffffu;
    if (__builtin_expect((ax > ay ? ax : ay) >= 0x7f7f8000u, 0)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t u = h ? uy : ux;
            if ((h ? ay : ax) < 0x7f7f8000u)
                continue;
            const uint32_t keep = h ? 0x0000ffffu : 0xffff0000u;
            const int sh = 16 * h;
            t[0] = (t[0] & keep) | (kMark << sh);
            t[1] = (t[1] & keep) | ((u >> 16) << sh);
            t[2] = (t[2] & keep) | ((u & 0xffffu) << sh);
        }
    }
}

// The float that three terms (16 bits each) stand for.
__device__ __forceinline__ float x3_float(uint32_t t0, uint32_t t1, uint32_t t2)
{
    const float sum = (__builtin_bit_cast(float, t0 << 16) + __builtin_bit_cast(float, t1 << 16)) +
                      __builtin_bit_cast(float, t2 << 16);
    return t0 == kMark ? __builtin_bit_cast(float, (t1 << 16) | t2) : sum * (1 / kScale);
}

// The three terms of eight floats, a 16-byte chunk each.
__device__ __forceinline__ void unit_terms(const float v[8], u32x4 o[3])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t t[3];
        split_pair(v[2 * k], v[2 * k + 1], t);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            o[p][k] = t[p];
    }
}

// Eight floats -> one unit (three 16-byte chunks at dst).
__device__ __forceinline__ void store_unit(const float v[8], bf16_t* dst)
{
    u32x4 o[3];
    unit_terms(v, o);
#pragma unroll
    for (int p = 0; p < 3; ++p)
        ((u32x4*)dst)[p] = o[p];
}

// The twelve chunks of four neighbouring lanes' units (lane u = lane % 4 holds
// unit u, all four active) in place: lane u stores chunks u, 4 + u, 8 + u of the
// 192 bytes at dst, so that a store's lanes are contiguous; chunk j, term j % 3
// of unit j / 3, comes across the quad.  Units from `units` on aren't stored.
__device__ __forceinline__ void store_quad(const u32x4 o[3], int u, int units, bf16_t* dst)
{
    constexpr int kPerm[3] = {0x40, 0xA5, 0xFE};  // lane (4 s + u) / 3 for lane u
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int j = 4 * s + u;
        const int unit = (j * 11) >> 5;  // j / 3
        const int term = j - 3 * unit;
        u32x4 c;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t t[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const int x = (int)o[p][k];
                t[p] = s == 0   ? __builtin_amdgcn_mov_dpp(x, kPerm[0], 0xf, 0xf, true)
                       : s == 1 ? __builtin_amdgcn_mov_dpp(x, kPerm[1], 0xf, 0xf, true)
                                : __builtin_amdgcn_mov_dpp(x, kPerm[2], 0xf, 0xf, true);
            }
            c[k] = term == 0 ? t[0] : term == 1 ? t[1] : t[2];
        }
        if (unit < units)
            ((u32x4*)dst)[j] = c;
    }
}

template <int MT>
struct MfmaX3;

template <>
struct MfmaX3<32> {
    static constexpr int kK = 16;
    static constexpr int kRegs = 16;
    typedef floatx16 acc_t;
    static __device__ __forceinline__ acc_t run(bf16x8 a, bf16x8 b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int q, int lane)
    {
        return 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
    }
};

template <>
struct MfmaX3<16> {
    static constexpr int kK = 32;
    static constexpr int kRegs = 4;
    typedef floatx4 acc_t;
    static __device__ __forceinline__ acc_t run(bf16x8 a, bf16x8 b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int q, int lane) { return 4 * (lane >> 4) + q; }
};

__device__ __forceinline__ void copy16(__amdgpu_buffer_rsrc_t r, u32x4* dst, uint32_t voff,
                                       uint32_t soff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, voff, soff, 0, 0);
}

// Barrier between pipeline stages: each wave has waited for its own copies
// (vmcnt) and fragment reads (lgkmcnt) before it; the empty asm statements
// keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void x3_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// s_waitcnt vmcnt(0) lgkmcnt(0), expcnt at its maximum
constexpr int kWaitVmLgkm0 = 0x0070;

}  // namespace

// ------------------------------------------------------------ forward / dgrad
// One workgroup of 8 waves per TM x 256 tile, 32 reduction channels per stage
// (192 bytes of each operand row: 4 units), double-buffered in LDS.  Both
// operands are copied global -> LDS by 16-byte DMA; a wave's three copies move
// 16 rows x 192 bytes, lane i of copy c taking chunk (64c + i) % 12 of row
// (64c + i) / 12, so that its lanes cover whole contiguous runs.  Inside a
// row, term p of unit j sits at slot 4p + (j ^ row_swz(row)).  The LDS serves
// a 16-byte read in groups of 16 lanes, lanes 0-3, 12-15, 20-23, 24-27 and
// 4-7, 8-11, 16-19, 28-31 of each half wave: with this order the rows and
// units of a group, in the 32- and the 16-row form, cover all 64 banks once
// (counters: no conflict; with (row / 4) % 4 in its place the 16-row form lost
// half its LDS cycles to conflicts).
//
// A step (one instruction depth) runs six groups of MI x NI instructions, one
// per pair of terms; each group reads the one operand term it adds two groups
// ahead.  The stage barrier stands before the last two groups of a stage:
// they cover the latency of the next stage's first reads, and the copies of
// the stage after it start there, into the buffer just freed.
template <int MT, int WM, int WN, int MI, int NI, int EPI, bool MASK, int ORD>
__global__ void __launch_bounds__(64 * WM * WN, 2)
conv_gemm_x3_kernel(const GemmX3Params p)
{
    typedef MfmaX3<MT> Op;
    constexpr int NW = WM * WN;
    constexpr int TM = WM * MI * MT;
    constexpr int TN = WN * NI * MT;
    constexpr int KL = 64 / MT;        // lane groups along k of one instruction
    constexpr int KS = 32 / Op::kK;    // steps per stage
    constexpr int GA = TM / 16, GB = TN / 16;  // 16-row copy groups
    constexpr int QA = (GA + NW - 1) / NW, QB = GB / NW;
    constexpr bool UNI = ORD == 2;
    static_assert(TM % 16 == 0 && GB % NW == 0, "copy groups");
    static_assert(KL * KS == kStageU, "units per stage");

    __shared__ u32x4 A0[TM * kRowC], A1[TM * kRowC];
    __shared__ u32x4 B0[TN * kRowC], B1[TN * kRowC];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM;
    const int wn = wave / WM;
    // XCD-contiguous tile order, row tiles fastest; split-K and tail-split
    // work items as in the float kernel (conv_gemm.hip)
    const int n_mt = (p.M + TM - 1) / TM;
    const int n_ct = (p.Ncol + TN - 1) / TN;
    const int n_tiles = n_mt * n_ct * p.G;
    const bool has_tail = EPI < 2 && p.tail_splits > 1;
    int T;
    {
        const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
        if (has_tail) {
            const int n_items = (n_tiles - p.tail_T) * p.tail_splits;
            const int fq = (p.tail_T + 7) >> 3, tq = (n_items + 7) >> 3;
            if (i < fq) {
                const int f = x * fq + i;
                T = f < p.tail_T ? f : INT_MAX;
            } else {
                const int j = x * tq + (i - fq);
                T = j < n_items ? p.tail_T + j : INT_MAX;
            }
        } else {
            T = x * (int)(gridDim.x >> 3) + i;
        }
    }
    int tile = T, split = 0;
    bool tail = false;
    if constexpr (EPI >= 2) {
        if (T >= n_tiles * p.splits)
            return;
        tile = T % n_tiles;
        split = T / n_tiles;
    } else {
        if (has_tail && T >= p.tail_T && T != INT_MAX) {
            const int j = T - p.tail_T;
            const int jt = j / p.tail_splits;
            tile = p.tail_T + jt;
            split = j - jt * p.tail_splits;
            tail = true;
        }
        if (tile >= n_tiles)
            return;
    }
    const int mt = tile % n_mt;
    const int ct = (tile / n_mt) % n_ct;
    const int g = tile / (n_mt * n_ct);
    const int m0 = mt * TM;
    const int n0 = ct * TN;
    const int M = p.M;
    const int OHW = p.OH * p.OW;

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.A, p.A_bytes);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.X, p.X_bytes);

    // this lane's chunk of copy c: row cr[c] of a 16-row group, unit cj[c]
    uint32_t a_voff[QA][3], b_pix[QB][3];
    int cj[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int idx = 64 * c + lane;
        const int row = idx / kRowC;
        const int slot = idx - row * kRowC;
        const int j = (slot & 3) ^ row_swz(row);
        const uint32_t in_row = (uint32_t)((slot >> 2) * 16);
        cj[c] = j;
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int m = m0 + 16 * (wave + NW * q) + row;
            a_voff[q][c] = m < M ? (uint32_t)((g * M + m) * p.Ru + j) * (uint32_t)kUnit + in_row
                                 : kOob;
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const int col = min(n0 + 16 * (wave + NW * q) + row, p.Ncol - 1);
            const int n = (int)fdiv((uint32_t)col, p.div_ohw);
            const int pix = col - n * OHW;
            const int i = (int)fdiv((uint32_t)pix, p.div_ow);
            const int jj = pix - i * p.OW;
            b_pix[q][c] =
                (uint32_t)(((n * p.IHp + i * p.sh + p.oh0) * p.IWp + jj * p.sw + p.ow0) * p.Ctot +
                           g * p.Cgp) * 6u + in_row +
                (ORD == 2 ? (uint32_t)(j * kUnit) : ORD == 1 ? (uint32_t)((j & 1) * kUnit) : 0u);
        }
    }
    // Byte offsets of stage t's units from a column's pixel.  ORD 2 (Cgp a
    // multiple of 32): the stage is 32 channels of one tap, one scalar offset
    // (the lane's unit is in b_pix).  ORD 1 (a multiple of 16): two units
    // share a tap, two scalars and a select by lane.  ORD 0: per lane, out of
    // range past the last unit.
    struct Delta {
        uint32_t v[UNI ? 1 : 3];
    };
    auto b_delta = [&](int t) -> Delta {
        Delta d;
        if constexpr (ORD == 2) {
            // stage t: 32-channel block t / ntap of tap t % ntap
            const int cb = (int)fdiv((uint32_t)t, p.div_ntap);
            const int tap = t - cb * p.ntap;
            const int u = (int)fdiv((uint32_t)tap, p.div_kw);
            const int v = tap - u * p.kw;
            d.v[0] = (uint32_t)((u * p.IWp + v) * p.Ctot + 32 * cb) * 6u;
        } else if constexpr (ORD == 1) {
            uint32_t o[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kc = t * kStageU + 2 * h;
                const int tap = (int)fdiv((uint32_t)kc, p.div_cg8);
                const int u = (int)fdiv((uint32_t)tap, p.div_kw);
                const int v = tap - u * p.kw;
                o[h] = kc < p.KC
                           ? (uint32_t)((u * p.IWp + v) * p.Ctot + 8 * (kc - tap * p.Cg8)) * 6u
                           : kOob;
            }
#pragma unroll
            for (int c = 0; c < 3; ++c)
                d.v[c] = cj[c] >= 2 ? o[1] : o[0];
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int kc = t * kStageU + cj[c];
                const int tap = (int)fdiv((uint32_t)kc, p.div_cg8);
                const int c8 = kc - tap * p.Cg8;
                const int u = (int)fdiv((uint32_t)tap, p.div_kw);
                const int v = tap - u * p.kw;
                const uint32_t o = (uint32_t)((u * p.IWp + v) * p.Ctot + 8 * c8) * 6u;
                d.v[c] = kc < p.KC ? o : kOob;
            }
        }
        return d;
    };
    // a stage's copies, 3 (QA + QB) per wave, in parts
    constexpr int NCP = 3 * (QA + QB);
    constexpr int PARTS = 5;
    constexpr int CPP = (NCP + PARTS - 1) / PARTS;
    auto issue_part = [&](int t, u32x4* As, u32x4* Bs, int part, const Delta& d) {
#pragma unroll
        for (int i = part * CPP; i < (part + 1) * CPP && i < NCP; ++i) {
            const int q = i / 3, c = i % 3;
            if (q < QB) {
                u32x4* dst = &Bs[(wave + NW * q) * 16 * kRowC + 64 * c];
                if constexpr (UNI)
                    copy16(rx, dst, b_pix[q][c], d.v[0]);
                else
                    copy16(rx, dst, b_pix[q][c] + d.v[c], 0u);
            } else {
                const int qa = q - QB;
                if (GA % NW == 0 || wave + NW * qa < GA)
                    copy16(ra, &As[(wave + NW * qa) * 16 * kRowC + 64 * c], a_voff[qa][c],
                           (uint32_t)(t * kStageU * kUnit));
            }
        }
    };

    // Forward: accumulators start at the bias of their row (a tail split's
    // partials leave the bias to the reduce).
    // The products of the two first terms add up in acc, the other five, 2^-8
    // of them and less, in lo: acc is rounded once per instruction depth, not
    // six times.
    typename Op::acc_t acc[MI][NI], lo[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        typename Op::acc_t init{};
        if constexpr (EPI == 0) {
            const __amdgpu_buffer_rsrc_t rbias =
                make_rsrc(p.bias, p.bias && !tail ? (uint32_t)(p.G * M) * 4u : 0u);
#pragma unroll
            for (int q = 0; q < Op::kRegs; ++q) {
                const int m = m0 + wm * MI * MT + mi * MT + Op::row(q, lane);
                init[q] = buf_ld_f32(rbias, m < M ? (uint32_t)(g * M + m) * 4u : kOob) / kUnscale;
            }
        }
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            acc[mi][ni] = init;
            lo[mi][ni] = typename Op::acc_t{};
        }
    }

    // fragment slots (term p adds 4 slots, a row block MT * 12)
    int fa[KS], fb[KS];
    {
        const int ra0 = wm * MI * MT + lane % MT;
        const int rb0 = wn * NI * MT + lane % MT;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            fa[ks] = ra0 * kRowC + ((ks * KL + lane / MT) ^ row_swz(ra0));
            fb[ks] = rb0 * kRowC + ((ks * KL + lane / MT) ^ row_swz(rb0));
        }
    }
    // fragments, two sets used by alternate steps
    bf16x8 xa[2][3][MI], xb[2][3][NI];
    auto read_a = [&](const u32x4* As, int ks, int set, int t) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            xa[set][t][mi] = __builtin_bit_cast(bf16x8, As[fa[ks] + 4 * t + mi * MT * kRowC]);
    };
    auto read_b = [&](const u32x4* Bs, int ks, int set, int t) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            xb[set][t][ni] = __builtin_bit_cast(bf16x8, Bs[fb[ks] + 4 * t + ni * MT * kRowC]);
    };
    auto mul = [&](int set, int ta, int tb) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                auto& a = ta + tb == 0 ? acc[mi][ni] : lo[mi][ni];
                a = Op::run(xa[set][ta][mi], xb[set][tb][ni], a);
            }
        __builtin_amdgcn_sched_barrier(0);
    };

    const int nst_all = (p.KC + kStageU - 1) / kStageU;
    const bool splitk = EPI >= 2 || tail;
    const int sps = EPI >= 2 ? p.stages_per_split : p.tail_sps;
    const int s_begin = splitk ? split * sps : 0;
    const int nst = splitk ? min(nst_all, s_begin + sps) : nst_all;

    if (s_begin < nst) {
        const Delta d = b_delta(s_begin);
#pragma unroll
        for (int part = 0; part < PARTS; ++part)
            issue_part(s_begin, A0, B0, part, d);
    }
    // (the last two groups of the stage before the first: zeros)
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        constexpr int set = 1;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            xa[set][t][mi] = bf16x8{};
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            xb[set][t][ni] = bf16x8{};
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
    x3_barrier();
    for (int s0 = s_begin; s0 < nst; s0 += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int s = s0 + h;
            if (s >= nst)
                break;
            // stage s has landed in Ac / Bc, the other buffers are read out
            const u32x4* Ac = h ? A1 : A0;
            const u32x4* Bc = h ? B1 : B0;
            u32x4* An = h ? A0 : A1;
            u32x4* Bn = h ? B0 : B1;
            const bool more = s + 1 < nst;
            const int first = KS == 2 ? 0 : h;
            read_a(Ac, 0, first, 0);
            read_b(Bc, 0, first, 0);
            read_b(Bc, 0, first, 1);
            const Delta d = b_delta(s + 1);
            mul(first ^ 1, 0, 2);
            if (more)
                issue_part(s + 1, An, Bn, 0, d);
            mul(first ^ 1, 2, 0);
            if (more)
                issue_part(s + 1, An, Bn, 1, d);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int set = KS == 2 ? ks : h;
                const bool last = ks == KS - 1;
                read_a(Ac, ks, set, 1);
                mul(set, 0, 0);
                if (ks == 0 && more)
                    issue_part(s + 1, An, Bn, 2, d);
                read_b(Bc, ks, set, 2);
                mul(set, 0, 1);
                if (ks == 0 && more)
                    issue_part(s + 1, An, Bn, 3, d);
                read_a(Ac, ks, set, 2);
                mul(set, 1, 0);
                if (ks == 0 && more)
                    issue_part(s + 1, An, Bn, 4, d);
                if (!last) {
                    read_a(Ac, ks + 1, set ^ 1, 0);
                    read_b(Bc, ks + 1, set ^ 1, 0);
                }
                mul(set, 1, 1);
                if (!last) {
                    read_b(Bc, ks + 1, set ^ 1, 1);
                    mul(set, 0, 2);
                    mul(set, 2, 0);
                }
            }
            __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
            x3_barrier();
        }
    }
    if (KS == 2 || ((nst - s_begin) & 1) == 0) {
        mul(1, 0, 2);
        mul(1, 2, 0);
    } else {
        mul(0, 0, 2);
        mul(0, 2, 0);
    }
    float odd = 0.f;  // (NaN once a sum is infinite or NaN)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            acc[mi][ni] = (acc[mi][ni] + lo[mi][ni]) * kUnscale;
#pragma unroll
            for (int q = 0; q < Op::kRegs; ++q)
                odd = fmaf(acc[mi][ni][q], 0.f, odd);
        }
    // the lane's outputs to form again, a bit each
    static_assert(MI * NI * Op::kRegs <= 64, "one bit per output");
    uint64_t again = 0;
    if (__builtin_expect(odd != odd, 0)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int q = 0; q < Op::kRegs; ++q)
                    again |= (uint64_t)!__builtin_isfinite(acc[mi][ni][q])
                             << ((mi * NI + ni) * Op::kRegs + q);
    }

    // ---- epilogue (branch-free: masked lanes store to an out-of-range offset)
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.Y, p.Y_bytes);
    // (the row and column indices are formed here and not kept from the bias
    // loads on: live through the main loop they made it spill)
    int le = lane;
    asm volatile("" : "+v"(le));
    const int brow = wn * NI * MT + le % MT;
    if (EPI >= 2 || tail) {
        // split partial P[split][g][m][col], or the tail region's
        // Pt[split][m][col - tail_c0] (the last group's)
        const __amdgpu_buffer_rsrc_t rp = EPI >= 2 ? ry : make_rsrc(p.Pt, p.Pt_bytes);
        const int c0 = EPI >= 2 ? 0 : p.tail_c0;
        const int Nc = p.Ncol - c0;
        const int r0 = (EPI >= 2 ? split * p.G + g : split) * M;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int col = n0 + brow + ni * MT;
                const uint32_t cbad = (uint32_t)(col >= p.Ncol) << 31;
#pragma unroll
                for (int q = 0; q < Op::kRegs; ++q) {
                    const int m = m0 + wm * MI * MT + mi * MT + Op::row(q, le);
                    const uint32_t off = ((uint32_t)((r0 + m) * Nc + col - c0) * 4u) | cbad |
                                         ((uint32_t)(m >= M) << 31);
                    buf_st_f32(acc[mi][ni][q], rp, off);
                }
            }
    } else if constexpr (EPI == 0) {
        int cbase[NI];
        uint32_t cbad[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int col = n0 + brow + ni * MT;
            const int n = (int)fdiv((uint32_t)col, p.div_ohw);
            const int pix = col - n * OHW;
            cbase[ni] = n * p.Cout * OHW + pix;
            cbad[ni] = (uint32_t)(col >= p.Ncol) << 31;
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int q = 0; q < Op::kRegs; ++q) {
                    const int m = m0 + wm * MI * MT + mi * MT + Op::row(q, le);
                    const float z = acc[mi][ni][q];
                    const float v = z > 0.f ? z : (p.relu ? 0.f : z);
                    const uint32_t off = ((uint32_t)(cbase[ni] + (g * M + m) * OHW) * 4u) |
                                         cbad[ni] | ((uint32_t)(m >= M) << 31);
                    buf_st_f32(v, ry, off);
                }
    } else if constexpr (EPI == 1) {
        const int pss = p.psh * p.psw;
        const int OutHW = p.OutH * p.OutW;
        const __amdgpu_buffer_rsrc_t rom = make_rsrc(MASK ? p.Omask : p.Y, p.Y_bytes);
        int cb[NI], hb[NI], wb[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int col = n0 + brow + ni * MT;
            const bool cok = col < p.Ncol;
            const int n = cok ? (int)fdiv((uint32_t)col, p.div_ohw) : 0;
            const int pix = col - n * OHW;
            const int a = (int)fdiv((uint32_t)pix, p.div_ow);
            const int b = pix - a * p.OW;
            hb[ni] = cok ? p.psh * (a + p.a0h) - p.oph : -(1 << 28);
            wb[ni] = p.psw * (b + p.a0w) - p.opw;
            cb[ni] = (n * p.Cout + g * p.Cg_out) * OutHW;
        }
        // per row block: every position (and mask value) first, then the
        // stores, half a 32-row block at a time
        constexpr int QC = Op::kRegs > 8 ? 8 : Op::kRegs;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int q0 = 0; q0 < Op::kRegs; q0 += QC) {
                uint32_t off[QC][NI];
                float y[QC][NI];
#pragma unroll
                for (int qq = 0; qq < QC; ++qq) {
                    const int m = m0 + wm * MI * MT + mi * MT + Op::row(q0 + qq, le);
                    int c = m, fh = 0, fw = 0;
                    if (pss != 1) {
                        c = (int)fdiv((uint32_t)m, p.div_pss);
                        const int fr = m - c * pss;
                        fh = (int)fdiv((uint32_t)fr, p.div_psw);
                        fw = fr - fh * p.psw;
                    }
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const int hh = hb[ni] + fh;
                        const int ww = wb[ni] + fw;
                        const uint32_t bad = ((uint32_t)(m >= M) |
                                              (uint32_t)((unsigned)hh >= (unsigned)p.OutH) |
                                              (uint32_t)((unsigned)ww >= (unsigned)p.OutW))
                                             << 31;
                        const uint32_t idx = (uint32_t)(cb[ni] + c * OutHW + hh * p.OutW + ww);
                        off[qq][ni] = (idx * 4u) | bad;
                        if constexpr (MASK)
                            y[qq][ni] = buf_ld_f32(rom, off[qq][ni]);
                    }
                }
#pragma unroll
                for (int qq = 0; qq < QC; ++qq)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        float v = acc[mi][ni][q0 + qq];
                        if constexpr (MASK)
                            v = y[qq][ni] > 0.f ? v : 0.f;
                        buf_st_f32(v, ry, off[qq][ni]);
                    }
            }
    }

    // ---- sums that came out infinite or NaN, formed again in float
    // arithmetic and stored over: an operand is no ordinary float, or a sum of
    // 2^32 x y overflows, from x y about 2^96 on (the small products, of any sign, then overflow as well and
    // would make NaN of infinity).  A lane forms its outputs one after the
    // other, each until it is NaN: a path for blobs that are diverging (conv2's
    // forward at N = 64: 0.28 ms, with one infinity 3.5, all infinite 10, all
    // NaN 2.2; backward 0.5, 12, 30 and 1.1).
    if (__builtin_expect(again == 0, 1))
        return;
    __builtin_amdgcn_s_waitcnt(kVmcnt0);
    const int first_s = ORD == 2 ? p.ntap / 2 : (nst - s_begin) / 2;
    do {
        const int bit = __builtin_ctzll(again);
        again &= again - 1;
        const int blk = bit / Op::kRegs;
        const int m = m0 + wm * MI * MT + blk / NI * MT + Op::row(bit % Op::kRegs, le);
        const int col = n0 + brow + blk % NI * MT;
        if (m >= M || col >= p.Ncol)
            continue;
        const int n = (int)fdiv((uint32_t)col, p.div_ohw);
        const int pix = col - n * OHW;
        const int i = (int)fdiv((uint32_t)pix, p.div_ow);
        const int j = pix - i * p.OW;
        const uint32_t at = (uint32_t)(((n * p.IHp + i * p.sh + p.oh0) * p.IWp + j * p.sw + p.ow0) *
                                           p.Ctot + g * p.Cgp) * 6u;
        float sum = EPI == 0 && !tail && p.bias ? p.bias[g * M + m] : 0.f;
        for (int e0 = 0; e0 < nst - s_begin && sum == sum; ++e0) {
            // from the window's centre on: the one place that is never padding
            const int s = s_begin + (e0 + first_s) % (nst - s_begin);
            u32x4 a[kStageU][3], b[kStageU][3];
#pragma unroll
            for (int e = 0; e < kStageU; ++e) {
                const int kc = s * kStageU + e;
                int tap, c8;
                if constexpr (ORD == 2) {
                    const int cb = (int)fdiv((uint32_t)s, p.div_ntap);
                    tap = s - cb * p.ntap;
                    c8 = cb * kStageU + e;
                } else {
                    tap = (int)fdiv((uint32_t)kc, p.div_cg8);
                    c8 = kc - tap * p.Cg8;
                }
                const int u = (int)fdiv((uint32_t)tap, p.div_kw);
                const int v = tap - u * p.kw;
                const uint32_t oa = (uint32_t)((g * M + m) * p.Ru + kc) * (uint32_t)kUnit;
                const uint32_t ob = at + (uint32_t)((u * p.IWp + v) * p.Ctot + 8 * c8) * 6u;
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    a[e][t] = buf_ld_b128(ra, kc < p.KC ? oa + 16 * t : kOob);
                    b[e][t] = buf_ld_b128(rx, kc < p.KC ? ob + 16 * t : kOob);
                }
            }
            float part[kStageU] = {};  // (short chains of additions)
#pragma unroll
            for (int e = 0; e < kStageU; ++e)
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int w = k / 2, sh = k % 2 * 16;
                    const float va = x3_float(a[e][0][w] >> sh & 0xffffu, a[e][1][w] >> sh & 0xffffu,
                                              a[e][2][w] >> sh & 0xffffu);
                    const float vb = x3_float(b[e][0][w] >> sh & 0xffffu, b[e][1][w] >> sh & 0xffffu,
                                              b[e][2][w] >> sh & 0xffffu);
                    part[e] = fmaf(va, vb, part[e]);
                }
            sum += (part[0] + part[1]) + (part[2] + part[3]);
        }
        if (EPI >= 2 || tail) {
            const int c0 = EPI >= 2 ? 0 : p.tail_c0;
            const int r0 = (EPI >= 2 ? split * p.G + g : split) * M;
            buf_st_f32(sum, EPI >= 2 ? ry : make_rsrc(p.Pt, p.Pt_bytes),
                       (uint32_t)((r0 + m) * (p.Ncol - c0) + col - c0) * 4u);
        } else if constexpr (EPI == 0) {
            buf_st_f32(sum > 0.f ? sum : (p.relu ? 0.f : sum), ry,
                       (uint32_t)((n * p.Cout + g * M + m) * OHW + pix) * 4u);
        } else if constexpr (EPI == 1) {
            const int c = (int)fdiv((uint32_t)m, p.div_pss);
            const int fr = m - c * p.psh * p.psw;
            const int fh = (int)fdiv((uint32_t)fr, p.div_psw);
            const int h = p.psh * (i + p.a0h) - p.oph + fh;
            const int w = p.psw * (j + p.a0w) - p.opw + fr - fh * p.psw;
            if ((unsigned)h >= (unsigned)p.OutH || (unsigned)w >= (unsigned)p.OutW)
                continue;
            const uint32_t off =
                (uint32_t)(((n * p.Cout + g * p.Cg_out + c) * p.OutH + h) * p.OutW + w) * 4u;
            if (MASK && !(p.Omask[off / 4] > 0.f))
                sum = 0.f;
            buf_st_f32(sum, ry, off);
        }
    } while (again);
}

// ----------------------------------------------------------- weight gradient
// Split-K over the output pixels, 32 per stage, both operands read from their
// staging as [pixel][channel] rows: a 64-channel line of one pixel is 8 units,
// 384 contiguous bytes; a wave's three copies of a line move 8 pixels of it.
// LDS holds a line's 24 chunks per pixel in the order term * 8 + (unit ^ 4
// (pixel / 2 % 2)), so that the transposed reads of four pixels and 32
// channels cover all 64 banks once.  ds_read_b64_tr_b16 hands each lane the
// four consecutive pixels of a channel that the instructions want (as in the
// bf16 kernel, conv_bf16.hip).  Pipeline as in conv_gemm_x3_kernel.
typedef short short4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short4v x3_read_tr16(const void* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) short4v*)p);
}

template <int WM, int WN, int MI, int NI>
__global__ void __launch_bounds__(64 * WM * WN, 2)
conv_wgrad_x3_kernel(const WgradX3Params p)
{
    constexpr int MT = 32;
    constexpr int TM = WM * MI * MT;
    constexpr int TN = WN * NI * MT;
    constexpr int TKP = 32;              // pixels per stage
    constexpr int KS = TKP / 16;
    constexpr int NLA = (TM + 63) / 64;  // 64-channel lines per pixel
    constexpr int NLB = TN / 64;
    constexpr int LC = 8 * 24;           // chunks of 8 pixels of a line
    static_assert(WM * WN == 8 && NLB == 4 && NLA <= 2, "copy mapping: wave = (pixels, half)");

    __shared__ u32x4 A0[4 * NLA * LC], A1[4 * NLA * LC];
    __shared__ u32x4 B0[4 * NLB * LC], B1[4 * NLB * LC];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM;
    const int wn = wave / WM;
    const int n_rt = (p.Rw + TN - 1) / TN;
    const int n_mt = (p.Kg + TM - 1) / TM;
    // each XCD takes a contiguous run of tiles, the row and column tiles of a
    // (group, split) unit, which read the same slabs, next to each other
    const int T = (blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    if (T >= n_rt * n_mt * p.G * p.splits)
        return;
    const int rt = T % n_rt;
    const int mt = (T / n_rt) % n_mt;
    const int g = (T / (n_rt * n_mt)) % p.G;
    const int split = T / (n_rt * n_mt * p.G);
    const int m0 = mt * TM;
    const int r0 = rt * TN;
    const int OHW = p.OH * p.OW;
    const int col_begin = split * p.cols_per_split;
    const int col_end = min(p.Ncol, col_begin + p.cols_per_split);

    const __amdgpu_buffer_rsrc_t rd = make_rsrc(p.D, p.D_bytes);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.X, p.X_bytes);

    // wave w copies pixels 8 (w / 2) .. + 7 of a stage: line w % 2 of D and
    // lines 2 (w % 2), + 1 of X.  Rows past Kg and columns past Rw are read
    // (inside the buffer or as zeros past its end) but feed only results that
    // are never stored.
    const int rg = wave >> 1, hf = wave & 1;
    int cpx[3];
    uint32_t a_off[3], b_off[2][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int idx = 64 * c + lane;
        const int px = idx / 24;
        const int slot = idx - px * 24;
        const int c8 = (slot & 7) ^ (((px >> 1) & 1) << 2);
        const uint32_t term = (uint32_t)((slot >> 3) * 16);
        cpx[c] = 8 * rg + px;
        a_off[c] = (uint32_t)(g * p.Kgp + m0 + 64 * hf + 8 * c8) * 6u + term;
#pragma unroll
        for (int L = 0; L < 2; ++L) {
            const int r = r0 + 64 * (2 * hf + L) + 8 * c8;  // 8 channels of one tap
            const int t = r / p.Cgp;
            const int cc = r - t * p.Cgp;
            const int u = t / p.kw;
            const int v = t - u * p.kw;
            b_off[L][c] = (uint32_t)((u * p.IWp + v) * p.Ctot + g * p.Cgp + cc) * 6u + term;
        }
    }
    // byte offsets of the lane's pixels in stage t (kOob past the split's
    // end: with the channel offset added they stay out of range)
    struct Pix {
        uint32_t d[3], x[3];
    };
    auto pixels = [&](int t) -> Pix {
        Pix q;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int col = col_begin + t * TKP + cpx[c];
            const int n = (int)fdiv((uint32_t)col, p.div_ohw);
            const int pix = col - n * OHW;
            const int i = (int)fdiv((uint32_t)pix, p.div_ow);
            const int j = pix - i * p.OW;
            const bool ok = col < col_end;
            q.d[c] = ok ? (uint32_t)(((n * p.DHp + i + p.dtb) * p.DWp + j + p.dlb) * p.Ktot) * 6u
                        : kOob;
            q.x[c] = ok ? (uint32_t)(((n * p.IHp + i * p.sh) * p.IWp + j * p.sw) * p.Ctot) * 6u
                        : kOob;
        }
        return q;
    };
    constexpr int NCP = 9, PARTS = 5, CPP = 2;
    auto issue_part = [&](u32x4* As, u32x4* Bs, int part, const Pix& q) {
#pragma unroll
        for (int i = part * CPP; i < (part + 1) * CPP && i < NCP; ++i) {
            const int L = i / 3, c = i % 3;
            if (L < 2)
                copy16(rx, &Bs[(rg * NLB + 2 * hf + L) * LC + 64 * c], q.x[c] + b_off[L][c], 0u);
            else if (NLA == 2 || hf == 0)
                copy16(rd, &As[(rg * NLA + hf) * LC + 64 * c], q.d[c] + a_off[c], 0u);
        }
    };

    // (first terms' products in acc, the small ones in lo, as in the GEMM)
    floatx16 acc[MI][NI], lo[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            acc[mi][ni] = lo[mi][ni] = floatx16{};

    // transposed-read addresses (bytes): lane as a source points at pixel
    // 8 (lane / 32) + 4h + (lane % 16) / 4 of the step, channel
    // 16 (lane / 16 % 2) + 4 (lane % 4) of its 32-row block; a step adds two
    // 8-pixel groups, a term 8 chunks
    const int prow = (lane & 15) >> 2;
    const int csrc = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    auto tile_off = [&](int c, int h, int NL) {
        return (((lane >> 5) * NL + (c >> 6)) * LC + (4 * h + prow) * 24 +
                (((c & 63) >> 3) ^ (((prow >> 1) & 1) << 2))) * 16 + (c & 7) * 2;
    };
    int fa[MI][2], fb[NI][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            fa[mi][h] = tile_off(wm * MI * MT + mi * MT + csrc, h, NLA);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            fb[ni][h] = tile_off(wn * NI * MT + ni * MT + csrc, h, NLB);
    }
    bf16x8 xa[2][3][MI], xb[2][3][NI];
    auto frag = [&](const u32x4* base, const int off[2], int imm) {
        const short4v k0 = x3_read_tr16((const char*)base + off[0] + imm);
        const short4v k4 = x3_read_tr16((const char*)base + off[1] + imm);
        return __builtin_bit_cast(bf16x8,
                                  __builtin_shufflevector(k0, k4, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_a = [&](const u32x4* As, int ks, int t) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            xa[ks][t][mi] = frag(As, fa[mi], ks * 2 * NLA * LC * 16 + t * 128);
    };
    auto read_b = [&](const u32x4* Bs, int ks, int t) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            xb[ks][t][ni] = frag(Bs, fb[ni], ks * 2 * NLB * LC * 16 + t * 128);
    };
    auto mul = [&](int ks, int ta, int tb) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                floatx16& a = ta + tb == 0 ? acc[mi][ni] : lo[mi][ni];
                a = MfmaX3<32>::run(xa[ks][ta][mi], xb[ks][tb][ni], a);
            }
        __builtin_amdgcn_sched_barrier(0);
    };

    const int nst = col_end > col_begin ? (col_end - col_begin + TKP - 1) / TKP : 0;
    if (nst > 0) {
        const Pix q = pixels(0);
#pragma unroll
        for (int part = 0; part < PARTS; ++part)
            issue_part(A0, B0, part, q);
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            xa[1][t][mi] = bf16x8{};
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            xb[1][t][ni] = bf16x8{};
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
    x3_barrier();
    for (int s0 = 0; s0 < nst; s0 += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int s = s0 + h;
            if (s >= nst)
                break;
            const u32x4* Ac = h ? A1 : A0;
            const u32x4* Bc = h ? B1 : B0;
            u32x4* An = h ? A0 : A1;
            u32x4* Bn = h ? B0 : B1;
            const bool more = s + 1 < nst;
            read_a(Ac, 0, 0);
            read_b(Bc, 0, 0);
            read_b(Bc, 0, 1);
            const Pix q = pixels(s + 1);
            mul(1, 0, 2);
            if (more)
                issue_part(An, Bn, 0, q);
            mul(1, 2, 0);
            if (more)
                issue_part(An, Bn, 1, q);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bool last = ks == KS - 1;
                read_a(Ac, ks, 1);
                mul(ks, 0, 0);
                if (ks == 0 && more)
                    issue_part(An, Bn, 2, q);
                read_b(Bc, ks, 2);
                mul(ks, 0, 1);
                if (ks == 0 && more)
                    issue_part(An, Bn, 3, q);
                read_a(Ac, ks, 2);
                mul(ks, 1, 0);
                if (ks == 0 && more)
                    issue_part(An, Bn, 4, q);
                if (!last) {
                    read_a(Ac, ks + 1, 0);
                    read_b(Bc, ks + 1, 0);
                }
                mul(ks, 1, 1);
                if (!last) {
                    read_b(Bc, ks + 1, 1);
                    mul(ks, 0, 2);
                    mul(ks, 2, 0);
                }
            }
            __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
            x3_barrier();
        }
    }
    mul(1, 0, 2);
    mul(1, 2, 0);
    float odd = 0.f;  // (NaN once a sum is infinite or NaN)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            acc[mi][ni] = (acc[mi][ni] + lo[mi][ni]) * kUnscale;
#pragma unroll
            for (int q = 0; q < 16; ++q)
                odd = fmaf(acc[mi][ni][q], 0.f, odd);
        }
    static_assert(MI * NI * 16 <= 64, "one bit per output");
    uint64_t again = 0;
    if (__builtin_expect(odd != odd, 0)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    again |= (uint64_t)!__builtin_isfinite(acc[mi][ni][q])
                             << ((mi * NI + ni) * 16 + q);
    }

    // partial result P[split][g*Kg + m][r], lanes along r
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(p.P, p.P_bytes);
    const int pbase = split * p.K * p.Rw;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int r = r0 + wn * NI * MT + ni * MT + (lane & 31);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int m = m0 + wm * MI * MT + mi * MT + MfmaX3<32>::row(q, lane);
                const uint32_t bad = ((uint32_t)(m >= p.Kg) | (uint32_t)(r >= p.Rw)) << 31;
                buf_st_f32(acc[mi][ni][q], rp,
                           ((uint32_t)(pbase + (g * p.Kg + m) * p.Rw + r) * 4u) | bad);
            }
    }

    // sums that came out infinite or NaN, formed again in float arithmetic (see
    // conv_gemm_x3_kernel)
    if (__builtin_expect(again == 0, 1))
        return;
    __builtin_amdgcn_s_waitcnt(kVmcnt0);
    do {
        const int bit = __builtin_ctzll(again);
        again &= again - 1;
        const int blk = bit / 16;
        const int m = m0 + wm * MI * MT + blk / NI * MT + MfmaX3<32>::row(bit % 16, lane);
        const int r = r0 + wn * NI * MT + blk % NI * MT + (lane & 31);
        if (m >= p.Kg || r >= p.Rw)
            continue;
        const int t = r / p.Cgp;
        const int u = t / p.kw;
        const int cd = g * p.Kgp + m, cx = g * p.Cgp + r - t * p.Cgp;
        const uint32_t od = (uint32_t)(cd / 8 * kUnit + cd % 8 * 2);
        const uint32_t ox = (uint32_t)((u * p.IWp + t - u * p.kw) * p.Ctot) * 6u +
                            (uint32_t)(cx / 8 * kUnit + cx % 8 * 2);
        float sum = 0.f;
        for (int c = col_begin; c < col_end && sum == sum; c += 16) {
            uint16_t d[16][3], x[16][3];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int n = (int)fdiv((uint32_t)(c + e), p.div_ohw);
                const int pix = c + e - n * OHW;
                const int i = (int)fdiv((uint32_t)pix, p.div_ow);
                const int j = pix - i * p.OW;
                const uint32_t ad =
                    (uint32_t)(((n * p.DHp + i + p.dtb) * p.DWp + j + p.dlb) * p.Ktot) * 6u + od;
                const uint32_t ax =
                    (uint32_t)(((n * p.IHp + i * p.sh) * p.IWp + j * p.sw) * p.Ctot) * 6u + ox;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    d[e][k] = buf_ld_u16(rd, c + e < col_end ? ad + 16 * k : kOob);
                    x[e][k] = buf_ld_u16(rx, c + e < col_end ? ax + 16 * k : kOob);
                }
            }
            float part[2] = {};
#pragma unroll
            for (int e = 0; e < 16; ++e)
                part[e & 1] = fmaf(x3_float(d[e][0], d[e][1], d[e][2]),
                                   x3_float(x[e][0], x[e][1], x[e][2]), part[e & 1]);
            sum += part[0] + part[1];
        }
        buf_st_f32(sum, rp, (uint32_t)(pbase + (g * p.Kg + m) * p.Rw + r) * 4u);
    } while (again);
}

// ------------------------------------------------------------------ staging
// X3[n][hp][wp][g*Cgp/8 + c/8][term][c%8] from X[n][g*Cg + c][hp - tb][wp - lb]
// inside the H x W image (c < Cg), else 0; with RELU, X [Y > 0] in its place
// (Y laid out like X).  A block takes 32 staged channels of one image's
// bordered rows r0 .. r0 + RH - 1: the real rows among them are one contiguous
// run of at most 256 pixels per channel plane, one pixel per thread with all
// 32 channels' loads in flight; the floats cross LDS and each thread writes
// whole units, the four units of a pixel across a quad.  Streams: bound by HBM.
// (Blocks linear and three 16-byte stores 48 bytes apart a lane -> this, 256
// images: 96 x 27 x 27 for conv2 69 us -> 54, its masked top gradient 182 -> 158;
// the eight of a training step 570 -> 446.)  sums (may be null): the block's sum of
// each channel's (masked) floats, sums[(g*Kg + c) * T + n * rchunks + chunk]
// (T = N * rchunks), for the bias gradient.
constexpr int kX3Ch = 32;
constexpr int kX3Pix = 256;

template <bool RELU>
__global__ void __launch_bounds__(256)
stage_x3_kernel(const float* __restrict__ X, const float* __restrict__ Y, bf16_t* __restrict__ Xp,
                float* __restrict__ sums, int N, int C, int H, int W, int Cg, int Cgp, int Ctot,
                int Hp, int Wp, int tb, int lb, int RH, int rchunks, int ctiles)
{
    __shared__ float tile[kX3Ch][kX3Pix + 2];
    // each XCD takes a contiguous run of blocks: the channel tiles of a pixel,
    // whose 192-byte runs share lines, meet in one L2
    const int b = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    const int n = b / (rchunks * ctiles);
    if (n >= N)
        return;
    const int rem = b - n * rchunks * ctiles;
    const int rc = rem / ctiles;
    const int c0 = (rem - rc * ctiles) * kX3Ch;
    const int r0 = rc * RH;
    const int r1 = min(Hp, r0 + RH);
    const int h0 = max(0, r0 - tb);
    const int h1 = min(H, r1 - tb);
    const int RP = h1 > h0 ? (h1 - h0) * W : 0;
    const int tid = threadIdx.x;
    const uint32_t plane = (uint32_t)(H * W) * 4u;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + (size_t)n * C * H * W, (uint32_t)C * plane);
    const __amdgpu_buffer_rsrc_t ry =
        make_rsrc(RELU ? Y + (size_t)n * C * H * W : X, RELU ? (uint32_t)C * plane : 0u);
    {
        // threads past the run read out of range (0)
        const uint32_t voff = tid < RP ? (uint32_t)(h0 * W + tid) * 4u : kOob;
        float v[kX3Ch], y[RELU ? kX3Ch : 1];
        int g = c0 / Cgp, cl = c0 - g * Cgp;  // (uniform)
        uint32_t so[kX3Ch];
#pragma unroll
        for (int c = 0; c < kX3Ch; ++c) {
            // a padded channel, or one past the last, is out of range
            so[c] = cl < Cg && c0 + c < Ctot ? (uint32_t)(g * Cg + cl) * plane : kOob;
            if (++cl == Cgp) {
                cl = 0;
                ++g;
            }
        }
#pragma unroll
        for (int c = 0; c < kX3Ch; ++c)
            v[c] = buf_ld_f32(rx, so[c] == kOob ? kOob : voff + so[c]);
        if constexpr (RELU) {
#pragma unroll
            for (int c = 0; c < kX3Ch; ++c)
                y[c] = buf_ld_f32(ry, so[c] == kOob ? kOob : voff + so[c]);
        }
#pragma unroll
        for (int c = 0; c < kX3Ch; ++c)
            tile[c][tid] = !RELU || y[RELU ? c : 0] > 0.f ? v[c] : 0.f;
    }
    __syncthreads();
    if (sums) {
        // 8 threads per channel: strided partial sums, then a fixed tree
        const int c = tid >> 3;
        float s = 0.f;
        for (int i = tid & 7; i < RP; i += 8)
            s += tile[c][i];
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        s += __shfl_xor(s, 4, 64);
        const int cp = c0 + c;
        const int g = cp / Cgp, cl = cp - g * Cgp;
        if ((tid & 7) == 0 && cp < Ctot && cl < Cg)
            sums[(size_t)(g * Cg + cl) * ((size_t)N * rchunks) + (size_t)n * rchunks + rc] = s;
    }
    const int npix = (r1 - r0) * Wp;
    constexpr int U = kX3Ch / 8;
    static_assert(U == 4, "a quad stores a pixel's units");
    for (int id = tid; id < npix * U; id += 256) {
        // (a quad's four units are of one pixel: its lanes run alike)
        const int u = id % U;
        const int pl = id / U;
        const int pr = pl / Wp;
        const int hp = r0 + pr;
        const int wp = pl - pr * Wp;
        const int h = hp - tb;
        const int w = wp - lb;
        u32x4 o[3] = {};
        if ((unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W) {
            const int q = (h - h0) * W + w;
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                v[k] = tile[8 * u + k][q];
            unit_terms(v, o);
        }
        store_quad(o, u, (Ctot - c0) / 8,
                   &Xp[((((size_t)n * Hp + hp) * Wp + wp) * Ctot + c0) * 3]);
    }
}

int stage_x3_chunks(int W, int Hp)
{
    const int RH = kX3Pix / W;
    return (Hp + RH - 1) / RH;
}

hipError_t launch_stage_x3(const float* X, const float* Y, uint16_t* Xp, float* sums, int N, int C,
                           int H, int W, int Cg, int Cgp, int Ctot, int Hp, int Wp, int tb, int lb,
                           hipStream_t s)
{
    if (N == 0)
        return hipSuccess;
    if (W > kX3Pix || Cgp % 8 != 0 || Ctot % Cgp != 0 || (Ctot / Cgp) * Cg != C)
        return hipErrorInvalidValue;
    const int RH = kX3Pix / W;
    const int rchunks = stage_x3_chunks(W, Hp);
    const int ctiles = (Ctot + kX3Ch - 1) / kX3Ch;
    const dim3 grid((unsigned)(((int64_t)N * rchunks * ctiles + 7) / 8 * 8));
    if (Y)
        hipLaunchKernelGGL(stage_x3_kernel<true>, grid, dim3(256), 0, s, X, Y, Xp, sums, N, C, H,
                           W, Cg, Cgp, Ctot, Hp, Wp, tb, lb, RH, rchunks, ctiles);
    else
        hipLaunchKernelGGL(stage_x3_kernel<false>, grid, dim3(256), 0, s, X, Y, Xp, sums, N, C, H,
                           W, Cg, Cgp, Ctot, Hp, Wp, tb, lb, RH, rchunks, ctiles);
    return hipGetLastError();
}

// Forward weights, one unit per thread: unit kc of row o holds the terms of
// W[o][8*c8 ..][u][v] (zero for channels past Cg and units past the last),
// kc = (u*kw + v)*Cg8 + c8, or with `blocked` ((c8 / 4)*khw + u*kw + v)*4 + c8 % 4.
__global__ void __launch_bounds__(256)
pack_weights_x3_kernel(const float* __restrict__ W, bf16_t* __restrict__ Wp, int K, int Cg,
                       int Cg8, int khw, int Ru, int blocked)
{
    const int total = K * Ru;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
        const int o = e / Ru;
        const int kc = e - o * Ru;
        int t, c8;
        if (blocked) {
            const int b = kc / (khw * 4);
            const int rem = kc - b * khw * 4;
            t = rem >> 2;
            c8 = b * 4 + (rem & 3);
        } else {
            t = kc / Cg8;
            c8 = kc - t * Cg8;
        }
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = 8 * c8 + i;
            v[i] = t < khw && c < Cg ? W[((size_t)o * Cg + c) * khw + t] : 0.f;
        }
        store_unit(v, &Wp[(size_t)e * 24]);
    }
}

hipError_t launch_pack_weights_x3(const float* W, uint16_t* Wp, int K, int Cg, int Cgp, int khw,
                                  int Ru, int blocked, hipStream_t s)
{
    const int64_t total = (int64_t)K * Ru;
    if (total == 0)
        return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(pack_weights_x3_kernel, dim3(blocks), dim3(256), 0, s, W, Wp, K, Cg,
                       Cgp / 8, khw, Ru, blocked);
    return hipGetLastError();
}

// Phase-stacked data-gradient weights (see dgrad_weight_transform_kernel), one
// unit of 8 output channels k per thread, units ordered over (tap, k / 8) as
// the forward weights' over (tap, c / 8).
__global__ void __launch_bounds__(256)
dgrad_weights_x3_kernel(const float* __restrict__ W, bf16_t* __restrict__ Wt, int G, int Kg,
                        int Kg8, int Cg, int kh, int kw, int sh, int sw, int Th, int Tw, int Ru,
                        int blocked)
{
    const int Mt = Cg * sh * sw;
    const int ntap = Th * Tw;
    const int64_t total = (int64_t)G * Mt * Ru;
    for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * 256) {
        const int gm = (int)(e / Ru);
        const int kc = (int)(e - (int64_t)gm * Ru);
        const int g = gm / Mt;
        const int m = gm - g * Mt;
        int t, k8;
        if (blocked) {
            const int b = kc / (ntap * 4);
            const int rem = kc - b * ntap * 4;
            t = rem >> 2;
            k8 = b * 4 + (rem & 3);
        } else {
            t = kc / Kg8;
            k8 = kc - t * Kg8;
        }
        const int th = t / Tw, tw = t - th * Tw;
        const int c = m / (sh * sw);
        const int f = m - c * sh * sw;
        const int fh = f / sw, fw = f - fh * sw;
        const int u = fh + sh * (Th - 1 - th);
        const int v2 = fw + sw * (Tw - 1 - tw);
        const bool ok = t < ntap && u < kh && v2 < kw;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 8 * k8 + i;
            v[i] = ok && k < Kg ? W[(((size_t)(g * Kg + k) * Cg + c) * kh + u) * kw + v2] : 0.f;
        }
        store_unit(v, &Wt[(size_t)e * 24]);
    }
}

hipError_t launch_dgrad_weights_x3(const float* W, uint16_t* Wt, int G, int Kg, int Kgp, int Cg,
                                   int kh, int kw, int sh, int sw, int Th, int Tw, int Ru,
                                   int blocked, hipStream_t s)
{
    const int64_t total = (int64_t)G * Cg * sh * sw * Ru;
    if (total == 0)
        return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(dgrad_weights_x3_kernel, dim3(blocks), dim3(256), 0, s, W, Wt, G, Kg,
                       Kgp / 8, Cg, kh, kw, sh, sw, Th, Tw, Ru, blocked);
    return hipGetLastError();
}

// ------------------------------------------------------------------- launch
namespace {

template <int MT, int WM, int WN, int MI, int NI, int EPI, bool MASK>
hipError_t launch_x3(const GemmX3Params& p, hipStream_t s)
{
    constexpr int TM = WM * MI * MT, TN = WN * NI * MT;
    const int64_t tiles = (int64_t)((p.M + TM - 1) / TM) * ((p.Ncol + TN - 1) / TN) * p.G;
    int64_t blocks;
    if (EPI >= 2)
        blocks = (tiles * p.splits + 7) / 8 * 8;
    else if (p.tail_splits > 1)
        blocks = 8 * ((p.tail_T + 7) / 8 + ((tiles - p.tail_T) * p.tail_splits + 7) / 8);
    else
        blocks = (tiles + 7) / 8 * 8;
    if (blocks > INT_MAX / 2)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(64 * WM * WN);
    if (p.Cgp % 32 == 0)
        hipLaunchKernelGGL((conv_gemm_x3_kernel<MT, WM, WN, MI, NI, EPI, MASK, 2>), grid, block, 0,
                           s, p);
    else if (p.Cgp % 16 == 0)
        hipLaunchKernelGGL((conv_gemm_x3_kernel<MT, WM, WN, MI, NI, EPI, MASK, 1>), grid, block, 0,
                           s, p);
    else
        hipLaunchKernelGGL((conv_gemm_x3_kernel<MT, WM, WN, MI, NI, EPI, MASK, 0>), grid, block, 0,
                           s, p);
    return hipGetLastError();
}

template <int EPI, bool MASK>
hipError_t launch_x3_tile(const GemmX3Params& p, int tile, hipStream_t s)
{
    switch (tile) {
    case X3TILE_128x256:
        return launch_x3<32, 2, 4, 2, 2, EPI, MASK>(p, s);
    case X3TILE_96x256:
        return launch_x3<32, 1, 8, 3, 1, EPI, MASK>(p, s);
    case X3TILE_64x256:
        return launch_x3<32, 1, 8, 2, 1, EPI, MASK>(p, s);
    case X3TILE_48x128:
        return launch_x3<16, 1, 4, 3, 2, EPI, MASK>(p, s);
    default:
        return hipErrorInvalidValue;
    }
}

template <int WM, int WN, int MI, int NI>
hipError_t launch_x3_wgrad(const WgradX3Params& p, hipStream_t s)
{
    constexpr int TM = WM * MI * 32, TN = WN * NI * 32;
    const int64_t tiles = (int64_t)((p.Rw + TN - 1) / TN) * ((p.Kg + TM - 1) / TM) * p.G *
                          p.splits;
    const int64_t blocks = (tiles + 7) / 8 * 8;
    if (blocks > INT_MAX / 2)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((conv_wgrad_x3_kernel<WM, WN, MI, NI>), dim3((unsigned)blocks), dim3(512), 0,
                       s, p);
    return hipGetLastError();
}

}  // namespace

int x3_wgrad_tile_m(int tile) { return tile == X3WTILE_64x256 ? 64 : tile == X3WTILE_96x256 ? 96 : 128; }

hipError_t launch_conv_wgrad_x3(const WgradX3Params& p, int tile, hipStream_t s)
{
    if (p.Cgp % 8 != 0 || p.Kgp % 8 != 0 || p.Rw != p.kh * p.kw * p.Cgp ||
        p.cols_per_split % kX3TK != 0)
        return hipErrorInvalidValue;
    switch (tile) {
    case X3WTILE_128x256:
        return launch_x3_wgrad<2, 4, 2, 2>(p, s);
    case X3WTILE_96x256:
        return launch_x3_wgrad<1, 8, 3, 1>(p, s);
    case X3WTILE_64x256:
        return launch_x3_wgrad<1, 8, 2, 1>(p, s);
    default:
        return hipErrorInvalidValue;
    }
}

int x3_tile_m(int tile)
{
    switch (tile) {
    case X3TILE_128x256:
        return 128;
    case X3TILE_96x256:
        return 96;
    case X3TILE_64x256:
        return 64;
    case X3TILE_48x128:
        return 48;
    default:
        return 0;
    }
}

int x3_tile_n(int tile) { return tile == X3TILE_48x128 ? 128 : 256; }

hipError_t launch_conv_gemm_x3(const GemmX3Params& p, int epi, int tile, hipStream_t s)
{
    if (p.Ncol == 0 || p.M == 0)
        return hipSuccess;
    // units of 8 channels; a row of A holds whole stages; 32-channel blocks
    // of a tap (Cgp % 32 == 0) imply the blocked order
    if (p.Cgp % 8 != 0 || p.Cg8 * 8 != p.Cgp || p.Ctot % 8 != 0 || p.Ru % kStageU != 0 ||
        p.KC > p.Ru || p.KC != p.ntap * p.Cg8 || p.ntap != p.kh * p.kw)
        return hipErrorInvalidValue;
    if (epi == 0)
        return launch_x3_tile<0, false>(p, tile, s);
    if (epi == 1)
        return p.Omask ? launch_x3_tile<1, true>(p, tile, s) : launch_x3_tile<1, false>(p, tile, s);
    if (epi == 3)
        return launch_x3_tile<3, false>(p, tile, s);
    return hipErrorInvalidValue;
}

}  // namespace caffe_hip
