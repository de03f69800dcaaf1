// Convolution weight gradient over input windows held in LDS (bf16, kernels of 2 x 2, 3 x 3, 5 x 5
// and 7 x 7, stride 1 or 2, any channel count).
//
// The implicit GEMM writes every input element to LDS once per tap, and its 128 x 128 tile reads
// eight fragments for 16 products.  Here a block takes 64 (or 32) output channels and, per wave, NG
// kernel rows of 16 input channels (3 x 3: all nine taps), and walks 128-position tiles of one
// shard: the tile's dy and its input window are staged once, both with positions as rows, and the
// transposing LDS reads feed every tap at an offset from the position's window origin.  A wave's
// 9 x 4 fragments of sums take 26 reads (512 bytes each) for 36 products, half the LDS traffic of
// the GEMM; the next tile's loads are in flight in registers meanwhile.  The four consecutive rows
// of a result fragment are input channels, so that a lane holds 4 * K * K consecutive values of the
// logical weight order and stores them as they are; the splits' rows are then added by a streaming
// pass (the GEMM's reduction scattered 4-byte stores: AlexNet's four 13 x 13 / 27 x 27 layers
// 37 + 46 + 35 + 23 us -> 12 + 19 + 18 + 12 us).
//
// What bounds it: latency.  The plan launches about one block per compute unit (two would fit: a wave's
// sums take 144 registers, but they double the partial rows, see choose_splits), so each SIMD has one
// wave, and the staging between the tiles shows: matrix cores busy 17 to 28% on the CIFAR, residual
// and AlexNet layers (first layers 10%), LDS 10 to 20%, waves waiting a third of their cycles.  Measured per launch, without the
// reductions: 27 x 27, 5 x 5, 2 groups of 48 -> 128, batch 256 in 8 shards 176 -> 139 us (6 splits; 4:
// 169); 13 x 13, 256 -> 384 118 -> 108 us, 2 groups of 192 -> 192 115 -> 84 us; 32 x 32, 64 -> 64, batch
// 512 114 -> 71 us; 16 x 16, 128 -> 128 75 -> 67 us; 2 groups of 20 -> 36 channels (narrow loads)
// 86 -> 55 us.
#include <algorithm>
#include <cmath>

#include "halo.h"

namespace mtx {

struct HaloWArgs {
    const bf16_t* x;   // [R * N][H][W][C]
    const bf16_t* dy;  // [R * N][OH][OW][OC]
    float* out;        // gradient rows (one split) or partial rows
    long long row_ld, row_off;
    unsigned x_bytes, dy_bytes;
    int N, C, H, W, OC, OH, OW, S, PD, G;
    int cg, og, Q, R;
    int ckg, stride, Hp, Wp, ngroups, cot, ubs, splits, tps, tiles, dy_off, pt_off, gt_off, vx, vdy, vec;
    int KT, row, ru, Cp;  // kernel size; RUN: elements per padded row, groups per window row, channels of a pixel
    long long w_len;
    FastDiv fd_ohw, fd_ow, fd_hp, fd_wp, fd_ckg;
};

// LDS bytes of a position's 16 * fa values of dy (fa even): an odd multiple of 32
constexpr int halo_w_dys(int fa) { return fa * 32 + 32; }

// window granules per thread loaded ahead, as registers allow
constexpr int halo_w_nx(int accs) { return accs > 36 ? 5 : 7; }

// V8: both operands are loaded 16 bytes at a time.  RUN: the padded first-layer input
// (conv_wgrad_run): a group is 16 elements of one window row (K = 1 here; a.ru of them per row).
template <int K, int NG, int FA, bool V8, bool RUN>
__global__ __launch_bounds__(256, 2) void conv_halo_wgrad_kernel(const HaloWArgs a)
{
    constexpr int U = K * NG, BQ = 128, CO = 16 * FA, DYS = halo_w_dys(FA), DG = CO / 8;
    constexpr int ND = BQ * DG / 256, NX = halo_w_nx(U * FA);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* const sdy = lds + a.dy_off;
    int* const pt = reinterpret_cast<int*>(lds + a.pt_off);

    // Blocks that read the same positions (all channel tiles of one shard's split) are
    // consecutive on one XCD.
    const unsigned nb = gridDim.x, hw = blockIdx.x;
    const unsigned xq = nb / 8, xr = nb % 8, xc = hw % 8;
    unsigned l = xc * xq + min(xc, xr) + hw / 8;
    const int ub = (int)(l % (unsigned)a.ubs);
    l /= (unsigned)a.ubs;
    const int co0 = (int)(l % (unsigned)a.cot) * CO;
    l /= (unsigned)a.cot;
    const int grp = (int)(l % (unsigned)a.G);
    l /= (unsigned)a.G;
    const int sp = (int)(l % (unsigned)a.splits), r = (int)(l / (unsigned)a.splits);
    const int t0 = sp * a.tps, t1 = min(t0 + a.tps, a.tiles);

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // the wave's kernel-row groups: group = ci16 * K + u; the block's window holds the channels
    // from its first group's on
    const int g0 = (ub * 4 + wave) * NG, c16 = RUN ? 0 : ub * 4 * NG / K;
    int goff[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const int g = min(g0 + i, a.ngroups - 1);
        if constexpr (RUN) {
            const int u = g / a.ru;
            goff[i] = u * a.row * 2 + (g - u * a.ru) * 32;
        } else {
            const int ci = g / K, u = g - ci * K;
            goff[i] = u * a.Wp * a.stride + (ci - c16) * 32;
        }
    }
    const int cbase = c16 * 16;  // first input channel (in the group) of the window

    const __amdgpu_buffer_rsrc_t bx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.x), (short)0, (int)a.x_bytes, (int)kRsrcWord3);
    const __amdgpu_buffer_rsrc_t bd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.dy), (short)0, (int)a.dy_bytes, (int)kRsrcWord3);

    // a tile of BQ positions of the shard: window rows row0 .., ngran granules
    struct Tile { int q0, q1, row0, ngran; };
    auto tile_of = [&](int t) {
        Tile w;
        w.q0 = t * BQ;
        w.q1 = min(w.q0 + BQ, a.Q) - 1;
        const unsigned n0 = fdiv(a.fd_ohw, (unsigned)w.q0), n1 = fdiv(a.fd_ohw, (unsigned)w.q1);
        const unsigned h0 = fdiv(a.fd_ow, (unsigned)w.q0 - n0 * (unsigned)(a.OH * a.OW));
        const unsigned h1 = fdiv(a.fd_ow, (unsigned)w.q1 - n1 * (unsigned)(a.OH * a.OW));
        w.row0 = (int)n0 * a.Hp + (int)h0 * a.S;
        const int rows = (int)n1 * a.Hp + (int)h1 * a.S + a.KT - w.row0;
        // (RUN: the last window of a row may read past it, into values that are not stored)
        w.ngran = RUN ? rows * (a.row / 8) + a.ru * 2 : rows * a.Wp * a.ckg;
        return w;
    };
    // Granule t of a window: padded row pr, input offset within a row (kOOB: in the padding or
    // past the group's channels), LDS byte.  They do not depend on the tile.
    auto granule = [&](int t, int& pr, int& src, int& dst, int& c8) {
        const unsigned pos = fdiv(a.fd_ckg, (unsigned)t), g = (unsigned)t - pos * (unsigned)a.ckg;
        const unsigned p = fdiv(a.fd_wp, pos), pw = pos - p * (unsigned)a.Wp;
        const int iw = (int)pw - a.PD;
        c8 = cbase + (int)g * 8;
        pr = (int)p;
        src = (unsigned)iw < (unsigned)a.W && c8 < a.cg ? iw * a.C + grp * a.cg + c8 : (int)kOOB;
        dst = (int)(pos * (unsigned)a.stride + g * 16);
    };
    // element offset of row pr of the tile's window, kOOB in the padding
    auto row_base = [&](const Tile& w, int pr) {
        const unsigned ar = (unsigned)(w.row0 + pr);
        const unsigned n = fdiv(a.fd_hp, ar);
        const int ih = (int)(ar - n * (unsigned)a.Hp) - a.PD;
        return (unsigned)ih < (unsigned)a.H ? ((r * a.N + (int)n) * a.H + ih) * a.W * a.C : (int)kOOB;
    };
    u32x4 px[NX], pd[ND];
    // (kept in LDS for the prefetched granules: src, and dst / 16 | pr << 16)
    int2* const gt = reinterpret_cast<int2*>(lds + a.gt_off);
#pragma unroll
    for (int s = 0; s < NX && !RUN; ++s) {
        int pr, src, dst, c8;
        granule(tid + s * 256, pr, src, dst, c8);
        gt[tid + s * 256] = make_int2(src, dst >> 4 | pr << 16);
    }
    // (each thread reads back its own entries only)
    auto load_by = [&](auto vx, const Tile& w) {
        constexpr int VX = decltype(vx)::value;
#pragma unroll
        for (int s = 0; s < NX; ++s) {
            if constexpr (RUN) {  // the window is contiguous
                const int t = tid + s * 256, off = (r * a.N * a.Hp + w.row0) * a.row + t * 8;
                px[s] = __builtin_amdgcn_raw_buffer_load_b128(bx, t < w.ngran ? off * 2 : (int)kOOB, 0, 0);
                continue;
            }
            const int2 m = gt[tid + s * 256];
            const int rb = row_base(w, m.y >> 16);
            const bool ok = (tid + s * 256 < w.ngran) & (rb != (int)kOOB) & (m.x != (int)kOOB);
            if constexpr (VX == 8) {
                px[s] = __builtin_amdgcn_raw_buffer_load_b128(bx, ok ? (rb + m.x) * 2 : (int)kOOB, 0, 0);
            } else {
                int pr, src, dst, c8;
                granule(tid + s * 256, pr, src, dst, c8);
                px[s] = halo_granule<VX>(bx, ok, rb + src, a.cg - c8);
            }
        }
    };
    auto load_dy = [&](auto vd, const Tile& w) {
#pragma unroll
        for (int s = 0; s < ND; ++s) {
            const int t = tid + s * 256, pos = t / DG, c = co0 + (t % DG) * 8;
            pd[s] = halo_granule<decltype(vd)::value>(
                bd, w.q0 + pos <= w.q1, (r * a.Q + w.q0 + pos) * a.OC + grp * a.og + c, a.og - c);
        }
    };
    typedef std::integral_constant<int, 8> L8;
    typedef std::integral_constant<int, 4> L4;
    typedef std::integral_constant<int, 1> L1;
    auto load = [&](const Tile& w) {
        if constexpr (V8) {
            load_dy(L8{}, w);
            load_by(L8{}, w);
        } else {
            if (a.vdy == 4) load_dy(L4{}, w);
            else load_dy(L1{}, w);
            if (a.vx == 4) load_by(L4{}, w);
            else load_by(L1{}, w);
        }
    };
    // window granules beyond the prefetched ones
    auto stage_rest = [&](const Tile& w) {
        for (int t = NX * 256 + tid; t < w.ngran; t += 256) {
            if constexpr (RUN) {
                const int off = (r * a.N * a.Hp + w.row0) * a.row + t * 8;
                *reinterpret_cast<u32x4*>(lds + t * 16) =
                    __builtin_amdgcn_raw_buffer_load_b128(bx, off * 2, 0, 0);
                continue;
            }
            int pr, src, dst, c8;
            granule(t, pr, src, dst, c8);
            const int rb = row_base(w, pr);
            const bool ok = (rb != (int)kOOB) & (src != (int)kOOB);
            *reinterpret_cast<u32x4*>(lds + dst) =
                V8 ? halo_granule<8>(bx, ok, rb + src, a.cg - c8)
                   : a.vx == 4 ? halo_granule<4>(bx, ok, rb + src, a.cg - c8)
                               : halo_granule<1>(bx, ok, rb + src, a.cg - c8);
        }
    };

    f32x4 acc[U][FA];
    // bias gradient: the wave's fragments of dy (every fourth), this lane's positions
    constexpr int NB = (FA + 3) / 4;
    float accb[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) accb[b] = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < FA; ++j) acc[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool bias = ub == 0;

    typedef __attribute__((address_space(3))) s16x4* P3;
    auto tr = [&](const char* p) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((P3)(__attribute__((address_space(3))) char*)p);
    };
    const int krow = lg * 4 + (lr >> 2);  // position of this lane's first transposing read
    const char* const dyl = sdy + krow * DYS + (lr & 3) * 8;

    Tile w = tile_of(t0);
    load(w);
    for (int t = t0; t < t1; ++t) {
        if (t > t0) __syncthreads();
#pragma unroll
        for (int s = 0; s < ND; ++s) {
            const int i = tid + s * 256;
            *reinterpret_cast<u32x4*>(sdy + (i / DG) * DYS + (i % DG) * 16) = pd[s];
        }
#pragma unroll
        for (int s = 0; s < NX; ++s)
            if (tid + s * 256 < w.ngran)
                *reinterpret_cast<u32x4*>(lds + (RUN ? (tid + s * 256) << 4 : (gt[tid + s * 256].y & 0xffff) << 4)) = px[s];
        stage_rest(w);
        if (tid < BQ) {  // window origin of every position (past the end: the last one's, dy is 0)
            const unsigned q = (unsigned)min(w.q0 + tid, w.q1);
            const unsigned n = fdiv(a.fd_ohw, q), p = q - n * (unsigned)(a.OH * a.OW);
            const unsigned h = fdiv(a.fd_ow, p), ow = p - h * (unsigned)a.OW;
            pt[tid] = RUN ? (((int)n * a.Hp + (int)h * a.S - w.row0) * a.row + (int)ow * a.S * a.Cp) * 2
                          : (((int)n * a.Hp + (int)h * a.S - w.row0) * a.Wp + (int)ow * a.S) * a.stride;
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        if (t + 1 < t1) {
            w = tile_of(t + 1);
            load(w);
        }
        __syncthreads();
#pragma unroll 1
        for (int ks = 0; ks < BQ / 32; ++ks) {
            const char* const xlo = lds + pt[ks * 32 + krow] + (lr & 3) * 8;
            const char* const xhi = lds + pt[ks * 32 + 16 + krow] + (lr & 3) * 8;
            const char* const dk = dyl + ks * 32 * DYS;
            s16x8 fd[FA];
#pragma unroll
            for (int j = 0; j < FA; ++j)
                fd[j] = __builtin_shufflevector(tr(dk + j * 32), tr(dk + 16 * DYS + j * 32), 0, 1, 2, 3, 4, 5, 6, 7);
            auto xfrag = [&](int u) {
                const int o = goff[u / K] + (u % K) * a.stride;
                return __builtin_shufflevector(tr(xlo + o), tr(xhi + o), 0, 1, 2, 3, 4, 5, 6, 7);
            };
            s16x8 fx[2];
            fx[0] = xfrag(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u + 1 < U) fx[(u + 1) & 1] = xfrag(u + 1);
#pragma unroll
                for (int j = 0; j < FA; ++j) Mma<bf16_t>::run(acc[u][j], fx[u & 1], fd[j]);
            }
            // Scheduling order: dy's fragments and the first two input fragments, then after the
            // products of each input fragment the reads of the one after the next.
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * FA + 5, 0);  // LDS reads
#pragma unroll
            for (int u = 0; u < U; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x008, FA, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            if (bias) {
#pragma unroll
                for (int j = 0; j < FA; ++j)
                    if (wave == (j & 3))
#pragma unroll
                        for (int e = 0; e < 8; ++e) accb[j >> 2] += bf16_to_f32((bf16_t)fd[j][e]);
            }
        }
    }

    // lane: output channel co0 + j*16 + lr, input channels ci*16 + 4*lg .. +3, taps (u, v)
    float* const row = a.out + (a.splits > 1 ? (long long)(sp * a.R + r) * a.row_ld
                                             : (long long)r * a.row_ld + a.row_off);
    constexpr int KK = K * K;
#pragma unroll
    for (int j = 0; j < FA; ++j) {
        const int co = co0 + j * 16 + lr;
        if (co >= a.og) continue;
        float* const wrow = row + (long long)(grp * a.og + co) * a.cg * KK;
        if constexpr (RUN) {
            // element j = v * Cp + ci of window row u
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                const int g = g0 + i, u = g / a.ru, jb = (g - u * a.ru) * 16 + lg * 4;
                if (g >= a.ngroups) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = (jb + e) / a.Cp, ci = jb + e - v * a.Cp;
                    if (v < a.KT && ci < a.cg)
                        row[((long long)co * a.cg + ci) * a.KT * a.KT + u * a.KT + v] = acc[i][j][e];
                }
            }
            continue;
        }
        if constexpr (NG == K && !RUN) {
            // every tap of 4 input channels: 4*K*K consecutive values
            const int ci = g0 / K * 16 + lg * 4;
            if (g0 < a.ngroups && a.vec && ci < a.cg) {
#pragma unroll
                for (int e = 0; e < KK; ++e) {
                    f32x4 v;
#pragma unroll
                    for (int b = 0; b < 4; ++b) v[b] = acc[(e * 4 + b) % KK][j][(e * 4 + b) / KK];
                    *reinterpret_cast<f32x4*>(wrow + (long long)ci * KK + e * 4) = v;
                }
                continue;
            }
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int g = g0 + i, c = g / K, u = g - c * K;
            if (g >= a.ngroups) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ci = c * 16 + lg * 4 + e;
                if (ci >= a.cg) continue;
#pragma unroll
                for (int v = 0; v < K; ++v) wrow[(long long)ci * KK + u * K + v] = acc[i * K + v][j][e];
            }
        }
    }
    if (bias) {  // the four lane groups hold different positions
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float v = accb[b];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            const int j = b * 4 + wave, co = co0 + j * 16 + lr;
            if (lg == 0 && j < FA && co < a.og) row[a.w_len + grp * a.og + co] = v;
        }
    }
}

// The splits' partial rows [split][R][ld] added in ascending order into the gradient rows.
__global__ __launch_bounds__(256) void halo_wgrad_reduce(const float* __restrict__ part, int splits, int R,
                                                         long long ld, long long n,
                                                         float* __restrict__ grads, long long gld,
                                                         long long off)
{
    const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
    const int r = blockIdx.y;
    if (i >= n) return;
    const float* src = part + (long long)r * ld + i;
    f32x4 s = *reinterpret_cast<const f32x4*>(src);
#pragma unroll 8
    for (int k = 1; k < splits; ++k)
        s += *reinterpret_cast<const f32x4*>(src + (long long)k * R * ld);
    float* g = grads + (long long)r * gld + off + i;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (i + e < n) g[e] = s[e];
}

// ---- plan -------------------------------------------------------------------------------------
namespace {
// Largest estimated time over the implicit GEMM's for which a layer takes the windows.  Beside the
// data-gradient chain, one block per compute unit leaves that chain more of the GPU than the implicit
// GEMM's many: over 70 drawn networks whose streams overlap, the steps took 0.918 of their time
// without windows at 0.95, 0.912 at 1.1 and 1.2, 0.909 at 1.35, 0.910 at 1.6 and without a limit.
constexpr double kAlone = 0.95, kBeside = 1.35;

// Reduction splits of a planned launch: as few as give every compute unit a block, of at least three
// tiles (with two, 88 channels of a small layer took 16 to 18 us against the implicit GEMM's 14.6):
// the partial rows that a second block per unit would write and read back cost more than it gains
// (two per unit: CIFAR step 828 -> 863 us, residual block 558 -> 580, AlexNet 2370 -> 2427), and the
// data-gradient chain on the other stream runs beside one.
void choose_splits(HaloWPlan& h, int R, int G)
{
    const long long base = (long long)R * G * h.cot * h.ubs;
    h.ld = (h.n + 3) / 4 * 4;
    long long splits = (256 + base - 1) / base;
    splits = std::min<long long>(splits, std::max(1, h.tiles / 3));
    while (splits > 1 && splits * R * h.ld > (64ll << 20)) --splits;
    h.tps = halo_cdiv(h.tiles, (int)splits);
    h.splits = halo_cdiv(h.tiles, h.tps);
    if (base * h.splits < 192) h.ok = false;
}
}  // namespace

HaloWPlan conv_halo_wgrad_plan(int dt, const ConvGeom& g, int R, bool beside)
{
    HaloWPlan h{};
    const int cg = g.C / g.G, og = g.OC / g.G;
    if (dt != DT_BF16 || (g.K != 2 && g.K != 3 && g.K != 5 && g.K != 7) || g.S > 2 || cg < 8) return h;
    // (element-wise loads only for grouped layers, whose operand rows are short in the implicit GEMM
    // too: a step with 2 groups of 10 -> 18 channels 585 -> 564 us; ungrouped, 19 -> 13 channels took
    // 38 us against the implicit GEMM's 33, and 225 -> 153 43 against 34)
    if (g.G == 1 && (cg % 4 || og % 4)) return h;
    const long long Q = (long long)g.N * g.OH * g.OW;
    if (Q > (1ll << 30)) return h;
    h.Hp = (g.OH - 1) * g.S + g.K;
    h.Wp = (g.OW - 1) * g.S + g.K;
    h.tiles = (int)((Q + 127) / 128);
    h.fa = og <= 32 ? 2 : 4;
    h.cot = halo_cdiv(og, 16 * h.fa);
    h.ngroups = halo_cdiv(cg, 16) * g.K;
    int rows = 0;
    // (tiles repeat their place in an image)
    const long long period = (long long)g.OH * g.OW / std::__gcd(128, g.OH * g.OW) * 128;
    for (long long q0 = 0; q0 < std::min(Q, period); q0 += 128) {
        const long long q1 = std::min<long long>(q0 + 128, Q) - 1;
        const long long r0 = q0 / (g.OH * g.OW) * h.Hp + q0 % (g.OH * g.OW) / g.OW * g.S;
        const long long r1 = q1 / (g.OH * g.OW) * h.Hp + q1 % (g.OH * g.OW) / g.OW * g.S;
        rows = std::max(rows, (int)(r1 - r0) + g.K);
    }
    // kernel-row groups per wave: the fewest idle ones, then the most per wave
    static const int kNg[][4] = {{0}, {0}, {4, 2, 0}, {3, 2, 1, 0}, {0}, {2, 1, 0}, {0}, {1, 0}};
    double best = 0;
    for (int i = 0; kNg[g.K][i]; ++i) {
        const int ng = kNg[g.K][i], ubs = halo_cdiv(h.ngroups, 4 * ng);
        // channels the widest block's groups span
        int span = 0;
        for (int u = 0; u < ubs; ++u) {
            const int lo = u * 4 * ng / g.K, hi = std::min((u + 1) * 4 * ng, h.ngroups) - 1;
            span = std::max(span, hi / g.K - lo + 1);
        }
        int stride = span * 32;
        while (stride % 64 != 32) stride += 16;
        const long long xl = (long long)rows * h.Wp * stride;
        if (xl + 128 * halo_w_dys(h.fa) + 512 + halo_w_nx(g.K * ng * h.fa) * 2048 > kHaloMaxLds) continue;
        // (a wave with fewer groups reads its dy fragments for fewer products)
        const double score = (double)h.ngroups / (ubs * 4 * ng) * (1.0 - 0.3 / (ng * g.K));
        if (score > best) {
            best = score;
            h.ok = true;
            h.ng = ng; h.ubs = ubs; h.ckg = span * 2; h.stride = stride; h.xlds = (int)xl;
        }
    }
    if (!h.ok) return h;
    h.n = (long long)g.OC * cg * g.K * g.K + g.OC;
    choose_splits(h, R, g.G);
    // Estimated time of both (see gemm_us).  Here, per tile of the busiest compute unit: its products or
    // the latency of its loads, the fragment reads, window granules past the prefetched ones, narrow
    // loads; then the splits' rows.  The implicit GEMM pays for narrow loads too, and for its scattered
    // gradient stores.  Channel counts that fill the 64 x 16 fragments badly, wide windows (64 -> 32
    // channels, 52 x 52, unpadded: 201 us against 148) and few products per tile (416 -> 4 channels: 296
    // against 173) are left to it: of 720 drawn layers 239 were slower here, with this rule 29 (49.1
    // -> 48.8 ms in sum; 55.6 all on the implicit GEMM, 51.2 without the rule).
    const int accs = g.K * h.ng * h.fa, odd = cg % 4 || og % 4 ? 2 : cg % 8 || og % 8 ? 1 : 0;
    const double n = std::ceil((double)R * g.G * h.cot * h.ubs * h.splits / 256);
    const double gran = (double)h.xlds / h.stride * h.ckg / 256;
    const double tile = std::max(0.0417 * accs * n, 1.86 * std::ceil(n / 2)) +
                        n * (0.048 * (g.K * h.ng + h.fa) + 0.106 * std::max(0.0, gran - halo_w_nx(accs)) +
                             (odd == 2 ? 0.124 : odd ? 0.0165 : 0.0) * (gran + h.fa));
    const double us = 14 + h.tps * tile + 2.8e-7 * R * h.ld * (h.splits > 1 ? h.splits * 8 : 4);
    const GemmDims d = conv_wgrad_dims(dt, g, R);
    const GemmPlan p = plan_for(dt, d);
    const double narrow = gemm_us(d, p, 0, 0, 1) / (p.FP + p.FQ) *  // (k steps)
                          (0.072 * p.FQ * (cg % 8 > 0) + 0.034 * p.FP * (og % 8 > 0));
    const double out = 4.0 * d.P * d.Q * d.Z;
    const double other = gemm_us(d, p, 17.5, 0.0114, 0.0255) + narrow +
                         out * (6.9e-7 + (p.splits > 1 ? 4.7e-7 * p.splits : 0.0));
    if (us > (beside ? kBeside : kAlone) * other) h.ok = false;
    return h;
}

HaloWPlan conv_halo_wgrad_run_plan(int dt, const ConvGeom& g, const RunGeom& r, int R)
{
    HaloWPlan h{};
    const long long Q = (long long)g.N * g.OH * g.OW;
    if (dt != DT_BF16 || g.G != 1 || g.OC % 4 || Q > (1ll << 30)) return h;
    h.Hp = r.Hp;
    h.tiles = (int)((Q + 127) / 128);
    h.fa = g.OC <= 32 ? 2 : 4;
    h.cot = halo_cdiv(g.OC, 16 * h.fa);
    h.ru = halo_cdiv(r.RUN, 16);
    h.ngroups = g.K * h.ru;
    int rows = 0;
    // (tiles repeat their place in an image)
    const long long period = (long long)g.OH * g.OW / std::__gcd(128, g.OH * g.OW) * 128;
    for (long long q0 = 0; q0 < std::min(Q, period); q0 += 128) {
        const long long q1 = std::min<long long>(q0 + 128, Q) - 1;
        auto row = [&](long long q) { return q / (g.OH * g.OW) * r.Hp + q % (g.OH * g.OW) / g.OW * g.S; };
        rows = std::max(rows, (int)(row(q1) - row(q0)) + g.K);
    }
    h.xlds = (rows * r.Wp * r.Cp + h.ru * 16) * 2;
    // Window rows of at most two groups, that is small kernels; with more, the sums of a wave leave one
    // wave per SIMD and a quarter of its groups idle (11 x 11, stride 4, 96 channels: 190 us against the
    // implicit GEMM's 179).
    h.ng = 2;
    h.ubs = halo_cdiv(h.ngroups, 4 * h.ng);
    h.ok = h.ru <= 2 && h.xlds + 128 * halo_w_dys(h.fa) + 512 <= kHaloMaxLds;
    if (!h.ok) return h;
    h.n = (long long)g.OC * g.C * g.K * g.K + g.OC;
    h.run = true;
    choose_splits(h, R, 1);
    // Estimated time of both (see gemm_us): tiles of few products wait for their loads, so that a
    // small layer in one block per unit gains (32 x 32, 3 -> 64 channels, 3 x 3, batch 512: 43 -> 41 us
    // alone, CIFAR step 830 -> 808), one of several channel tiles does not (3 -> 256, batch 256: 56 -> 65
    // us).  Of 52 drawn layers 37 were slower here (2245 -> 2579 us in sum), with this rule 2 (by 6 us).
    const double n = std::ceil((double)R * h.cot * h.ubs * h.splits / 256);
    const double us = 16 + h.tps * (std::max(0.047 * h.fa * n, 1.05 * std::ceil(n / 2)) + 0.08 * n * (2 + h.fa));
    const GemmDims d = conv_wgrad_run_dims(dt, g, r, R);
    if (us > kAlone * gemm_us(d, plan_for(dt, d), 17.2, 0.018, 0.028)) h.ok = false;
    return h;
}

size_t conv_halo_wgrad_partial(const HaloWPlan& h, int R)
{
    return h.ok && h.splits > 1 ? (size_t)h.splits * R * h.ld : 0;
}

template <int K, int NG, int FA, bool RUN = false>
static void launch_wgrad(const HaloWArgs& a, const HaloWPlan& h, hipStream_t s)
{
    const dim3 grid((unsigned)(a.R * a.splits * a.G * a.cot * a.ubs));
    const size_t lds = (size_t)h.xlds + 128 * halo_w_dys(FA) + 512 + (RUN ? 0 : halo_w_nx(K * NG * FA) * 2048);
    note_gemm(16 * FA, 64 * NG * K, 32, a.splits, kGemmHalo | kGemmInterleaved);
    if (a.vx == 8 && a.vdy == 8)
        hipLaunchKernelGGL((conv_halo_wgrad_kernel<K, NG, FA, true, RUN>), grid, dim3(256), lds, s, a);
    else
        hipLaunchKernelGGL((conv_halo_wgrad_kernel<K, NG, FA, false, RUN>), grid, dim3(256), lds, s, a);
}

// fields that both launchers set, the launch and the reduction
static hipError_t run_wgrad(HaloWArgs& a, const ConvGeom& g, const HaloWPlan& h, int R, const void* x,
                            const void* dy, float* grads, long long ld, long long w_off, float* partial,
                            hipStream_t s)
{
    if (!h.ok || (h.splits > 1 && !partial)) return hipErrorInvalidValue;
    a.x = static_cast<const bf16_t*>(x); a.dy = static_cast<const bf16_t*>(dy);
    a.dy_bytes = (unsigned)((size_t)R * g.N * g.OC * g.OH * g.OW * 2);
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.OC = g.OC; a.OH = g.OH; a.OW = g.OW;
    a.S = g.S; a.PD = g.PD; a.G = g.G; a.KT = g.K;
    a.cg = g.C / g.G; a.og = g.OC / g.G; a.Q = g.N * g.OH * g.OW; a.R = R;
    a.ckg = h.ckg; a.stride = h.stride; a.Hp = h.Hp; a.Wp = h.Wp; a.ngroups = h.ngroups;
    a.cot = h.cot; a.ubs = h.ubs; a.splits = h.splits; a.tps = h.tps; a.tiles = h.tiles;
    a.dy_off = h.xlds;
    a.pt_off = h.xlds + 128 * halo_w_dys(h.fa);
    a.gt_off = a.pt_off + 512;
    a.vx = h.run || a.cg % 8 == 0 ? 8 : a.cg % 4 == 0 ? 4 : 1;
    a.vdy = a.og % 8 == 0 ? 8 : a.og % 4 == 0 ? 4 : 1;
    if (a.vx != 8 || a.vdy != 8) {  // one kernel variant for every narrower load
        a.vx = std::min(a.vx, 4);
        a.vdy = std::min(a.vdy, 4);
    }
    a.w_len = h.n - g.OC;
    a.out = h.splits > 1 ? partial : grads;
    a.row_ld = h.splits > 1 ? h.ld : ld;
    a.row_off = h.splits > 1 ? 0 : w_off;
    a.vec = a.cg % 4 == 0 && (h.splits > 1 || (w_off % 4 == 0 && ld % 4 == 0));
    a.fd_ohw = make_fastdiv((unsigned)(g.OH * g.OW));
    a.fd_ow = make_fastdiv((unsigned)g.OW);
    a.fd_hp = make_fastdiv((unsigned)h.Hp);
    a.fd_wp = make_fastdiv((unsigned)h.Wp);
    a.fd_ckg = make_fastdiv((unsigned)h.ckg);
    const int id = (h.run ? 0 : g.K) * 100 + h.ng * 10 + h.fa;
    switch (id) {
    case 24: launch_wgrad<1, 2, 4, true>(a, h, s); break;
    case 22: launch_wgrad<1, 2, 2, true>(a, h, s); break;
    case 244: launch_wgrad<2, 4, 4>(a, h, s); break;
    case 242: launch_wgrad<2, 4, 2>(a, h, s); break;
    case 224: launch_wgrad<2, 2, 4>(a, h, s); break;
    case 222: launch_wgrad<2, 2, 2>(a, h, s); break;
    case 334: launch_wgrad<3, 3, 4>(a, h, s); break;
    case 332: launch_wgrad<3, 3, 2>(a, h, s); break;
    case 324: launch_wgrad<3, 2, 4>(a, h, s); break;
    case 322: launch_wgrad<3, 2, 2>(a, h, s); break;
    case 314: launch_wgrad<3, 1, 4>(a, h, s); break;
    case 312: launch_wgrad<3, 1, 2>(a, h, s); break;
    case 524: launch_wgrad<5, 2, 4>(a, h, s); break;
    case 522: launch_wgrad<5, 2, 2>(a, h, s); break;
    case 514: launch_wgrad<5, 1, 4>(a, h, s); break;
    case 512: launch_wgrad<5, 1, 2>(a, h, s); break;
    case 714: launch_wgrad<7, 1, 4>(a, h, s); break;
    case 712: launch_wgrad<7, 1, 2>(a, h, s); break;
    default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || h.splits <= 1) return e;
    timing_split(s, "reduce");
    hipLaunchKernelGGL(halo_wgrad_reduce, dim3((unsigned)((h.ld / 4 + 255) / 256), R), dim3(256), 0, s,
                       partial, h.splits, R, h.ld, h.n, grads, ld, w_off);
    return hipGetLastError();
}

hipError_t conv_halo_wgrad(const ConvGeom& g, const HaloWPlan& h, int R, const void* x, const void* dy,
                           float* grads, long long ld, long long w_off, float* partial, hipStream_t s)
{
    HaloWArgs a{};
    a.x_bytes = (unsigned)((size_t)R * g.N * g.C * g.H * g.W * 2);
    return run_wgrad(a, g, h, R, x, dy, grads, ld, w_off, partial, s);
}

hipError_t conv_halo_wgrad_run(const ConvGeom& g, const RunGeom& rg, const HaloWPlan& h, int R,
                               const void* xp, const void* dy, float* grads, long long ld,
                               long long w_off, float* partial, hipStream_t s)
{
    HaloWArgs a{};
    a.x_bytes = (unsigned)((size_t)R * g.N * rg.Hp * rg.Wp * rg.Cp * 2);
    a.row = rg.Wp * rg.Cp; a.ru = h.ru; a.Cp = rg.Cp;
    return run_wgrad(a, g, h, R, xp, dy, grads, ld, w_off, partial, s);
}

}  // namespace mtx
