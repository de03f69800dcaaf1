// Convolution forward and data gradient (bf16, stride 1, K x K kernels up to 7 x 7) over
// an input window held in LDS.
//
// The implicit GEMM (igemm.h) stages every k tile of its activation operand through LDS, so an
// input element crosses the load path, the LDS write port and the index arithmetic once per tap
// (9 times for 3 x 3), and the LDS traffic, not the matrix core, bounds its loop (20-33% of the
// bf16 peak).  Here a block loads the input rows that its output tile needs once - they are
// contiguous positions of the NHWC tensor - keeps them in LDS for the whole launch, and every
// tap reads its fragments at an offset from the same origins.  Weights do not pass through LDS:
// they are prepared fragment by fragment (1 KB per 16 rows and k step, in lane order), so that a
// wave loads them straight into registers at the full 64 bytes per clock, one k step ahead.  The
// main loop has no barrier.  What bounds it now is latency (weights from L2, fragments from LDS)
// rather than a port: on the CIFAR and AlexNet layers the matrix cores are busy 24 to 45% of a launch
// (CIFAR's first layer 13%), LDS 15 to 32% (with 0.2 to 0.37 bank conflict cycles for an active one),
// and a wave waits 34 to 67% of its cycles.  Other waves cover it: 16 waves per compute unit (two blocks of 8) beat 8 to 12 with twice
// the products per read (CIFAR 64-channel layers 56 -> 53 us), and images of 13 x 13, whose rows fill
// 11 column fragments, take a whole image per block.
//
// Every output's products are added in the order of the implicit GEMM (taps ascending, channels
// ascending, 32 per matrix instruction, in the same lanes), so the results are the same bits;
// reductions that the implicit GEMM splits keep it.  Data gradients of unpadded layers, where the
// alternative is the col product (a sum per tap, then the taps), are this one chain here: the same
// error against 64 bits (3e-5 of the values round the other way on either).
//
// Measured per launch, implicit GEMM -> this kernel: 27 x 27 images, 5 x 5, 2 groups of 48 -> 128
// channels, batch 256 (115 GFLOP) 152 -> 110 us forward, 193 -> 158 us data gradient; 13 x 13,
// 256 -> 384 93 -> 70 and 95 -> 82 us, 2 groups of 192 -> 192 83 -> 58 and 88 -> 60 us; 32 x 32,
// 64 -> 64, batch 512 68 -> 53 and 87 -> 57 us; 8 x 8, 256 -> 256 56 -> 41 and 58 -> 40 us.
// A padded first layer (conv_fwd_run) takes the same kernel at any stride: its window is whole rows
// of the padded input and a reduction granule lies at a fixed offset from an output's origin.
// AlexNet step (11 x 11, stride 4) 2370 -> 2338 us, CIFAR 828 -> 814, residual block 558 -> 550.
// Other strided layers keep the implicit GEMM (16 x 16 outputs, 3 x 3 stride 2, 128 channels: 39 us
// against 41 here, whose window holds four times the positions), and so do channel counts that
// are not whole 16-byte granules (their reduction steps would hold other products).
#include <algorithm>

#include "halo.h"

namespace mtx {

struct HaloArgs {
    const bf16_t* x;     // input [N][H][W][C] (forward: activations, data gradient: dy)
    const bf16_t* w;     // fragment-major weights (PREP_HALO_F / PREP_HALO_D)
    const float* bias;   // forward
    const bf16_t* mask;  // data gradient: stored output of the layer below (its ReLU), or null
    bf16_t* y;           // output [N][OH][OW][OC]
    unsigned x_bytes, w_bytes, y_bytes;
    int N, C, H, W, OC, OH, OW, K, PD, G;
    int cg, P, Q, relu;
    int tile;            // outputs of a block (at most its columns)
    int ckg, ks, stride, PT, PB, zero_off, tab_off, vout;
    int S, Hp, row;      // padded first-layer input: stride, rows per image, elements per row
    FastDiv fd_ohw, fd_ow, fd_ckg;
};

// BWD: y = data gradient, input rows h + PD - u instead of h - PD + u.  NW waves, WP of
// them along the output channels.  MODE: M_C64: channels per group a multiple of 64, so that a
// tap is an even number of whole k steps; M_RUN: the padded first-layer input (conv_fwd_run),
// whose reduction runs along window rows.
enum { M_ANY = 0, M_C64 = 1, M_RUN = 2 };
template <int NW, int FP, int WP, int FQ, bool BWD, int MODE>
__global__ __launch_bounds__(64 * NW, FP * FQ <= 16 ? 4 : 2) void conv_halo_kernel(const HaloArgs a)
{
    constexpr bool C64 = MODE == M_C64, RUN = MODE == M_RUN;
    constexpr int NT = 64 * NW, WQ = NW / WP, BP = 16 * FP * WP, BQ = 16 * FQ * WQ;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    int2* tab = reinterpret_cast<int2*>(lds + a.tab_off);

    // Consecutive output tiles read overlapping input rows, and the channel tiles and groups of
    // one output tile the same input: an XCD takes a contiguous range of them, channel tiles
    // fastest.
    const unsigned nb = gridDim.x, hw = blockIdx.x;
    const unsigned xq = nb / 8, xr = nb % 8, xc = hw % 8;
    const unsigned l = xc * xq + min(xc, xr) + hw / 8;
    const unsigned pg = (unsigned)(a.PT * a.G);
    const int qt = (int)(l / pg), pgi = (int)(l % pg), grp = pgi / a.PT, p0 = (pgi % a.PT) * BP;

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wp = wave % WP, wq = wave / WP;
    const int q0 = qt * a.tile, q1 = min(q0 + a.tile, a.Q) - 1;

    // The window: the input rows (n, h) from the first output's first one to the last output's
    // last one, which are contiguous positions of x.
    auto row_lo = [&](int h) { return BWD ? h + a.PD - (a.K - 1) : h - a.PD; };
    const unsigned n0 = fdiv(a.fd_ohw, (unsigned)q0), n1 = fdiv(a.fd_ohw, (unsigned)q1);
    const unsigned h0 = fdiv(a.fd_ow, (unsigned)q0 - n0 * (unsigned)(a.OH * a.OW));
    const unsigned h1 = fdiv(a.fd_ow, (unsigned)q1 - n1 * (unsigned)(a.OH * a.OW));
    int r0, r1;
    if constexpr (RUN) {
        r0 = (int)n0 * a.Hp + (int)h0 * a.S;
        r1 = (int)n1 * a.Hp + (int)h1 * a.S + a.K - 1;
    } else {
        r0 = (int)n0 * a.H + min(max(row_lo((int)h0), 0), a.H - 1);
        r1 = (int)n1 * a.H + min(max(row_lo((int)h1) + a.K - 1, 0), a.H - 1);
    }
    // (a padded row's last window may read past the row, against zero weights: one more run)
    const int pos0 = r0 * a.W;
    const int ngran = RUN ? (r1 - r0 + 1) * (a.row / 8) + a.ckg : (r1 - r0 + 1) * a.W * a.ckg;

    const __amdgpu_buffer_rsrc_t bx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.x), (short)0, (int)a.x_bytes, (int)kRsrcWord3);
    const __amdgpu_buffer_rsrc_t bw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.w), (short)0, (int)a.w_bytes, (int)kRsrcWord3);
    const __amdgpu_buffer_rsrc_t bm = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.mask), (short)0, (int)a.y_bytes, (int)kRsrcWord3);

    // all loads of a batch are issued before its LDS writes
    constexpr int NS = 8;
    for (int t0 = tid; t0 < ngran; t0 += NT * NS) {
        u32x4 v[NS];
        int dst[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int t = t0 + s * NT;
            const unsigned pos = fdiv(a.fd_ckg, (unsigned)t), g = (unsigned)t - pos * (unsigned)a.ckg;
            const int off = RUN ? r0 * a.row + t * 8 : (pos0 + (int)pos) * a.C + grp * a.cg + (int)g * 8;
            v[s] = __builtin_amdgcn_raw_buffer_load_b128(bx, t < ngran ? off * 2 : (int)kOOB, 0, 0);
            dst[s] = RUN ? t * 16 : (int)(pos * (unsigned)a.stride + g * 16);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (t0 + s * NT < ngran) *reinterpret_cast<u32x4*>(lds + dst[s]) = v[s];
    }
    // the zero position that taps in the padding read (it may have more granules than the block has
    // threads)
    for (int i = tid; i < (RUN ? 1 : a.ckg); i += NT)
        *reinterpret_cast<u32x4*>(lds + a.zero_off + i * 16) = u32x4{0u, 0u, 0u, 0u};
    // table of the reduction granules i = (u, v, c8) in ascending order: LDS byte offset from an
    // output's origin, and the two validity bits the tap needs
    const int ngr = (RUN ? a.K : a.K * a.K) * a.ckg;
    for (int i = tid; !C64 && i < (a.ks + 2) * 4; i += NT) {
        const int tap = (int)fdiv(a.fd_ckg, (unsigned)i), c8 = i - tap * a.ckg, u = tap / a.K, v = tap - u * a.K;
        if constexpr (RUN) {  // i = (u, c8): window row u, run granule c8
            tab[i] = i < ngr ? make_int2(tap * a.row * 2 + c8 * 16, 0) : make_int2(0, (int)0x80000000u);
            continue;
        }
        const int o = (u * a.W + v) * a.stride;
        // (granules past the last tap: no output has bit 31, so they read zeros)
        tab[i] = i < ngr ? make_int2((BWD ? -o : o) + c8 * 16, 1 << u | 1 << (8 + v))
                         : make_int2(0, (int)0x80000000u);
    }
    // this lane's output columns: origin, valid rows u (bits 0..) and columns v (bits 8..)
    int base[FQ], ok[FQ];
#pragma unroll
    for (int j = 0; j < FQ; ++j) {
        const int q = q0 + (wq * FQ + j) * 16 + lr;
        const unsigned qq = q <= q1 ? q : q0;
        const unsigned n = fdiv(a.fd_ohw, qq), r = qq - n * (unsigned)(a.OH * a.OW);
        const unsigned oh = fdiv(a.fd_ow, r), ow = r - oh * (unsigned)a.OW;
        if constexpr (RUN) {
            base[j] = (((int)n * a.Hp + (int)oh * a.S - r0) * a.row + (int)ow * a.S * a.C) * 2;
            ok[j] = 0;
            continue;
        }
        const int h = BWD ? (int)oh + a.PD : (int)oh - a.PD;
        const int w = BWD ? (int)ow + a.PD : (int)ow - a.PD;
        base[j] = (((int)n * a.H + h) * a.W + w - pos0) * a.stride;
        int m = 0;
        for (int u = 0; u < a.K; ++u) {
            const int hu = BWD ? h - u : h + u, wu = BWD ? w - u : w + u;
            m |= ((unsigned)hu < (unsigned)a.H) << u | ((unsigned)wu < (unsigned)a.W) << (8 + u);
        }
        ok[j] = m;
    }

    f32x4 acc[FP][FQ];
#pragma unroll
    for (int i = 0; i < FP; ++i)
#pragma unroll
        for (int j = 0; j < FQ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // weight fragments: 1 KB per (16 rows, k step), the k steps contiguous
    int wb[FP];
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int pb = p0 / 16 + wp * FP + i;
        wb[i] = pb < a.PB ? (grp * a.PB + pb) * a.ks * 1024 + lane * 16 : (int)kOOB;
    }
    auto wload = [&](u32x4 (&f)[FP], int k) {
#pragma unroll
        for (int i = 0; i < FP; ++i)
            f[i] = __builtin_amdgcn_raw_buffer_load_b128(bw, wb[i], k * 1024, 0);
    };
    auto products = [&](u32x4 (&fa)[FP], const s16x8 (&fb)[FQ], int k) {
#pragma unroll
        for (int j = 0; j < FQ; ++j)
#pragma unroll
            for (int i = 0; i < FP; ++i)
                Mma<bf16_t>::run(acc[i][j], __builtin_bit_cast(s16x8, fa[i]), fb[j]);
        // (at the end the last step's again, not used: the buffer's bound covers the per-lane offset
        // only, so the scalar one must stay inside the weights)
        wload(fa, min(k + 2, a.ks - 1));
    };
    // two register sets of weight fragments: a set's next fragments are loaded as soon as its
    // products are issued, one k step ahead of their use (an even number of k steps)
    u32x4 fa0[FP], fa1[FP];
    wload(fa0, 0);
    wload(fa1, 1);
    // (with the window's loads known to be done, the loop waits for its own loads only)
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    if constexpr (C64) {
        // one tap at a time: its origins (or the zero position) once, then its channels
        int k = 0;
        for (int u = 0; u < a.K; ++u)
            for (int v = 0; v < a.K; ++v) {
                const int need = 1 << u | 1 << (8 + v), o = (u * a.W + v) * a.stride;
                int at[FQ];
#pragma unroll
                for (int j = 0; j < FQ; ++j)
                    at[j] = ((ok[j] & need) == need ? base[j] + (BWD ? -o : o) : a.zero_off) + lg * 16;
                for (int c = 0; c < a.ckg; c += 8, k += 2) {
                    s16x8 fb[FQ];
#pragma unroll
                    for (int j = 0; j < FQ; ++j) fb[j] = *reinterpret_cast<const s16x8*>(lds + at[j]);
                    products(fa0, fb, k);
#pragma unroll
                    for (int j = 0; j < FQ; ++j) {
                        fb[j] = *reinterpret_cast<const s16x8*>(lds + at[j] + 64);
                        at[j] += 128;
                    }
                    products(fa1, fb, k + 1);
                }
            }
    } else {
        // input fragments under table entry e
        auto iread = [&](s16x8 (&fb)[FQ], int2 e) {
#pragma unroll
            for (int j = 0; j < FQ; ++j) {
                const int at = (ok[j] & e.y) == e.y ? base[j] + e.x : a.zero_off;
                fb[j] = *reinterpret_cast<const s16x8*>(lds + at);
            }
        };
        int2 e0 = tab[lg], e1 = tab[4 + lg];  // table entries of the next two k steps
        for (int k = 0; k < a.ks; k += 2) {
            s16x8 fb[FQ];
            iread(fb, e0);
            e0 = tab[(k + 2) * 4 + lg];
            products(fa0, fb, k);
            iread(fb, e1);
            e1 = tab[(k + 3) * 4 + lg];
            products(fa1, fb, k + 1);
        }
    }

    // Epilogue: bias and ReLU in fp32, the tile rounded into LDS as [q][p], then whole rows of
    // channels with 16-byte stores (8-byte ones where the channels are a multiple of 4 only); the
    // data gradient's mask is read with them.
    constexpr int OSTR = BP + 8, GP = BP / 8, NO = (BQ * GP + NT - 1) / NT;
    typedef std::integral_constant<int, 8> W8;
    typedef std::integral_constant<int, 4> W4;
    typedef std::integral_constant<int, 1> W1;
    const int pn = min(BP, a.P - p0);
    u32x4 mk[BWD ? NO : 1];
    if constexpr (BWD) {
        // the mask's latency passes while the tile goes to LDS
        auto mask_rows = [&](auto width) {
#pragma unroll
            for (int t = 0; t < NO; ++t) {
                const int q = (tid + t * NT) / GP, g = (tid + t * NT) % GP;
                const int idx = (q0 + q) * a.OC + grp * a.P + p0 + g * 8;
                mk[t] = halo_row_load<decltype(width)::value>(bm, q0 + q <= q1, idx, pn - g * 8);
            }
        };
        if (a.mask && a.vout == 8) mask_rows(W8{});
        else if (a.mask && a.vout == 4) mask_rows(W4{});
    }
    __syncthreads();
    bf16_t* ot = reinterpret_cast<bf16_t*>(lds);
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int pl = (wp * FP + i) * 16 + lg * 4;
        f32x4 b = {0.f, 0.f, 0.f, 0.f};
        if constexpr (!BWD) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p0 + pl + e < a.P) b[e] = a.bias[grp * a.P + p0 + pl + e];
        }
#pragma unroll
        for (int j = 0; j < FQ; ++j) {
            f32x4 v = acc[i][j];
            if constexpr (!BWD) {
                v = v + b;
                if (a.relu)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
            }
            const unsigned lo = (unsigned)f32_to_bf16(v[0]) | ((unsigned)f32_to_bf16(v[1]) << 16);
            const unsigned hi = (unsigned)f32_to_bf16(v[2]) | ((unsigned)f32_to_bf16(v[3]) << 16);
            *reinterpret_cast<u32x2*>(ot + ((wq * FQ + j) * 16 + lr) * OSTR + pl) = u32x2{lo, hi};
        }
    }
    __syncthreads();
    auto store_rows = [&](auto width) {
        constexpr int W = decltype(width)::value;
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            const int q = (tid + t * NT) / GP, g = (tid + t * NT) % GP;
            if (q0 + q > q1 || q >= a.tile || g * 8 >= pn) continue;
            u32x4 v = *reinterpret_cast<const u32x4*>(ot + q * OSTR + g * 8);
            const long long idx = (long long)(q0 + q) * a.OC + grp * a.P + p0 + g * 8;
            if constexpr (W > 1) {
                if (BWD && a.mask) v = halo_masked(v, mk[BWD ? t : 0]);
                halo_row_store<W>(a.y + idx, v, pn - g * 8);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (g * 8 + e >= pn) break;
                    bf16_t b = (bf16_t)(v[e / 2] >> (16 * (e & 1)));
                    if (BWD && a.mask && !(bf16_to_f32(a.mask[idx + e]) > 0.f)) b = 0;
                    a.y[idx + e] = b;
                }
            }
        }
    };
    if (a.vout == 8) store_rows(W8{});
    else if (a.vout == 4) store_rows(W4{});
    else store_rows(W1{});
}

// ---- plan -------------------------------------------------------------------------------------
namespace {

// nw waves, fp x fq fragments per wave, wp waves along the output channels, blocks per compute
// unit that the registers allow; weight: relative time of a product on this shape (measured on
// the AlexNet and CIFAR layers, with the occupancy factors of the plan divided out)
struct Shape { int nw, fp, wp, fq, res; double weight; };
constexpr Shape kShapes[] = {{8, 1, 2, 4, 2, 1.6},  {8, 2, 2, 4, 2, 1.15},  {8, 3, 2, 4, 2, 0.95},
                             {8, 2, 4, 4, 2, 1.0},  {8, 3, 4, 4, 2, 0.79},  {8, 4, 2, 4, 2, 0.91},
                             {4, 3, 4, 11, 2, 0.78}, {8, 2, 8, 11, 1, 0.86}, {8, 3, 8, 11, 1, 0.76}};
constexpr int kCuLds = 160 * 1024, kLdsUnit = 1280;

// Chooses the block shape of a convolution of N images with img outputs each (OW per row), P
// output channels in each of G groups and ks k steps: rows(q0, q1) gives the window of a range
// of outputs in rows of rowb LDS bytes, extra more bytes belong to it, tab bytes follow it.
template <class Rows>
void choose_shape(HaloPlan& h, long long Q, int img, int P, int G, long long rowb, long long extra,
                  long long tab, Rows&& rows_of)
{
    double best = 0;
    for (int i = 0; i < (int)(sizeof kShapes / sizeof kShapes[0]); ++i) {
        const Shape& s = kShapes[i];
        const int BP = 16 * s.fp * s.wp, BQ = 16 * s.fq * (s.nw / s.wp);
        // (rows at least half used: 24 channels on 128 rows took 12 us against 8 of the implicit GEMM's
        // 32-row tiles)
        if (BP > 32 && halo_cdiv(P, 16) * 32 <= BP) continue;
        // whole images where they fit and fill the columns, else BQ outputs in a row
        const int whole = BQ / img * img, tile = whole * 10 >= BQ * 9 ? whole : BQ;
        // the largest input window of any output tile (tiles repeat their place in an image)
        long long rows = 0;
        const long long period = (long long)img / std::__gcd(tile, img) * tile;
        for (long long q0 = 0; q0 < std::min(Q, period); q0 += tile)
            rows = std::max<long long>(rows, rows_of(q0, std::min<long long>(q0 + tile, Q) - 1));
        const long long win = rows * rowb + extra;
        const long long body = std::max(win, (long long)BQ * (BP + 8) * 2), lds = body + tab;
        if (lds > kCuLds) continue;
        const long long blocks = (Q + tile - 1) / tile * halo_cdiv(P, BP) * G;
        // (fewer blocks than this leave a quarter of the compute units idle, where the implicit
        // GEMM's smaller tiles do not)
        if (blocks < 192) continue;
        // products per SIMD on the busiest compute unit; the fewer waves a SIMD has, the more of
        // the fragment reads' latency shows, and one block per unit overlaps no staging
        const int res = std::min<int>(s.res, (int)(kCuLds / ((lds + kLdsUnit - 1) / kLdsUnit * kLdsUnit)));
        const long long n = (blocks + 255) / 256;
        const int waves = (int)std::min<long long>(res, n) * s.nw / 4;
        const double cost = (double)n * s.nw / 4 * s.fp * s.fq * s.weight *
                            (waves < 2 ? 1.35 : waves < 3 ? 1.07 : 1.0) * (n == 1 ? 1.05 : 1.0);
        if (best == 0 || cost < best) {
            best = cost;
            h.shape = i;
            h.tile = tile;
            h.zero_off = (int)(win - extra);
            h.lds = (int)((body + 15) / 16 * 16);
            h.ok = true;
        }
    }
    h.PB = halo_cdiv(P, 16);
    h.w_elems = (long long)G * h.PB * h.ks * 512;
    if (h.w_elems * 2 > (1ll << 30)) h.ok = false;
}

// Estimated time of a launch in microseconds (see gemm_us): for every block on the busiest compute unit
// its products, its window's 16-byte pieces per thread, which cost three times as much where the
// window leaves room for one block, and its output rows.
double halo_us(const HaloPlan& h, long long Q, int P, int G)
{
    const Shape& s = kShapes[h.shape];
    const int BP = 16 * s.fp * s.wp;
    const long long blocks = (Q + h.tile - 1) / h.tile * halo_cdiv(P, BP) * G;
    const bool alone = s.res == 1 || halo_cdiv(h.lds, kLdsUnit) * kLdsUnit * 2 > kCuLds;
    const double pieces = h.zero_off / 16.0 / (64 * s.nw), kb = h.tile * std::min(BP, P) * 2e-3;
    return 6.8 + (double)((blocks + 255) / 256) *
                     (h.ks * (0.05 + s.fp * s.fq * s.nw / 4 * (alone ? 0.011 : 0.0085)) +
                      pieces * (alone ? 0.235 : 0.07) + 0.72 + kb * (P % 4 ? 0.196 : 0.049));
}

// The same of an implicit GEMM that writes bf16 rows (bwd: and reads their mask).
double direct_us(int dt, const GemmDims& d, bool bwd)
{
    return gemm_us(d, plan_for(dt, d), 7.8, kGemmProduct, kGemmOperand) +
           2.0 * d.P * d.Q * d.Z * (bwd ? 4.4e-7 : 2.1e-7) * (d.P % 4 ? 3.5 : 1.0);
}

// The convolution as the kernel sees it: the data gradient reads dy and writes the input's shape.
ConvGeom halo_geom(const ConvGeom& g, bool bwd)
{
    if (!bwd) return g;
    return ConvGeom{g.N, g.OC, g.OH, g.OW, g.C, g.H, g.W, g.K, 1, g.PD, g.G};
}

}  // namespace

HaloPlan conv_halo_plan(int dt, const ConvGeom& geom, bool bwd)
{
    HaloPlan h{};
    if (dt != DT_BF16 || geom.K > 7 || geom.S != 1) return h;
    const ConvGeom g = halo_geom(geom, bwd);
    const int cg = g.C / g.G, P = g.OC / g.G, img = g.OH * g.OW;
    const long long Q = (long long)g.N * img;
    if (cg % 8 || Q > (1ll << 30)) return h;
    // (the implicit GEMM splits this reduction: too few outputs, or too long)
    if (plan_for(dt, bwd ? conv_dgrad_dims(dt, geom) : conv_fwd_dims(dt, geom)).splits > 1) return h;
    h.ckg = cg / 8;
    h.ks = halo_cdiv(g.K * g.K * h.ckg, 8) * 2;
    h.stride = cg * 2;  // an odd multiple of 32 bytes: neighbouring positions start in other banks
    while (h.stride % 64 != 32) h.stride += 16;
    auto lo = [&](long long q) {
        const int oh = (int)(q % img / g.OW);
        return bwd ? oh + g.PD - (g.K - 1) : oh - g.PD;
    };
    auto clamp = [&](int r) { return std::min(std::max(r, 0), g.H - 1); };
    choose_shape(h, Q, img, P, g.G, (long long)g.W * h.stride, h.stride,
                 cg % 64 ? (h.ks + 2) * 32 : 0, [&](long long q0, long long q1) {
                     return (q1 / img - q0 / img) * g.H + clamp(lo(q1) + g.K - 1) - clamp(lo(q0)) + 1;
                 });
    // A 1 x 1 kernel reads its input once either way.  The implicit GEMM's masked output is its slow
    // part: data gradient of 256 -> 128 channels, 32 x 32, batch 256: 124 -> 68 us here (a copy of
    // its bytes: 66).  Not where a window leaves room for one block per unit (512 -> 128, 16 x 16: 22
    // us against 29 here), and not forward (256 -> 128 51 against 61, 128 -> 512 29 against 31).
    if (geom.K == 1 && (!bwd || h.lds > kHaloMaxLds)) h.ok = false;
    // Small blocks, padded rows and wide windows leave the implicit GEMM ahead: of 651 drawn layers the
    // kernel was slower in 76 forward and 7 data gradients, with this rule in 28 and 4 (most by a
    // few percent; 22.42 -> 22.27 ms in sum, the implicit GEMM 26.51).  An unpadded layer's data gradient
    // multiplies the padding around dy, which the col product does not: the kernel gains up to
    // about four products for a useful one (256 -> 256 channels, 8 x 8, 5 x 5: 55 us, col 61), for
    // narrow layers more, and loses beyond (7 x 7 closing 7 x 7 images, 256 -> 256: 133 us, col 38).
    const GemmDims d = bwd ? conv_dgrad_dims(dt, geom) : conv_fwd_dims(dt, geom);
    const double other = bwd && conv_dgrad_use_col(geom) ? conv_dgrad_col_us(dt, geom)
                                                         : 1.1 * direct_us(dt, d, bwd);
    if (h.ok && halo_us(h, Q, P, g.G) > other) h.ok = false;
    return h;
}

HaloPlan conv_halo_run_plan(int dt, const ConvGeom& g, const RunGeom& r)
{
    HaloPlan h{};
    const int img = g.OH * g.OW;
    const long long Q = (long long)g.N * img;
    if (dt != DT_BF16 || g.K < 2 || g.G != 1 || Q > (1ll << 30)) return h;
    if (plan_for(dt, conv_fwd_run_dims(dt, g, r)).splits > 1) return h;
    h.ckg = r.RUN / 8;
    h.ks = halo_cdiv(g.K * h.ckg, 8) * 2;
    choose_shape(h, Q, img, g.OC, 1, (long long)r.Wp * r.Cp * 2, r.RUN * 2 + 16, (h.ks + 2) * 32,
                 [&](long long q0, long long q1) {
                     auto row = [&](long long q) { return q / img * r.Hp + q % img / g.OW * g.S; };
                     return row(q1) + g.K - row(q0);
                 });
    h.zero_off += r.RUN * 2;  // behind the run that the last row may read past its end
    if (h.ok && halo_us(h, Q, g.OC, 1) > 1.1 * direct_us(dt, conv_fwd_run_dims(dt, g, r), false)) h.ok = false;
    return h;
}

template <int NW, int FP, int WP, int FQ>
static void launch_halo(HaloArgs& a, const HaloPlan& h, bool bwd, hipStream_t s)
{
    constexpr int BP = 16 * FP * WP, BQ = 16 * FQ * (NW / WP);
    a.PT = halo_cdiv(a.P, BP);
    const dim3 grid((unsigned)(halo_cdiv(a.Q, a.tile) * a.PT * a.G)), block(64 * NW);
    const size_t lds = (size_t)h.lds + (a.cg % 64 || a.row ? (size_t)(h.ks + 2) * 32 : 0);
    note_gemm(BP, BQ, 32, 1, kGemmHalo);
    auto go = [&](auto bwd_, auto mode) {
        hipLaunchKernelGGL((conv_halo_kernel<NW, FP, WP, FQ, decltype(bwd_)::value, decltype(mode)::value>),
                           grid, block, lds, s, a);
    };
    typedef std::integral_constant<int, M_ANY> Any;
    typedef std::integral_constant<int, M_C64> C64;
    typedef std::integral_constant<int, M_RUN> Run;
    const bool c64 = a.cg % 64 == 0;
    if (a.row) go(std::false_type{}, Run{});
    else if (bwd && c64) go(std::true_type{}, C64{});
    else if (bwd) go(std::true_type{}, Any{});
    else if (c64) go(std::false_type{}, C64{});
    else go(std::false_type{}, Any{});
}

static hipError_t launch_shape(HaloArgs& a, const HaloPlan& h, const ConvGeom& g, bool bwd, hipStream_t s)
{
    a.tile = h.tile; a.ckg = h.ckg; a.ks = h.ks; a.stride = h.stride; a.PB = h.PB;
    a.zero_off = h.zero_off; a.tab_off = h.lds;
    a.vout = halo_row_width(a.P);
    a.fd_ohw = make_fastdiv((unsigned)(g.OH * g.OW));
    a.fd_ow = make_fastdiv((unsigned)g.OW);
    a.fd_ckg = make_fastdiv((unsigned)h.ckg);
    switch (h.shape) {
    case 0: launch_halo<8, 1, 2, 4>(a, h, bwd, s); break;
    case 1: launch_halo<8, 2, 2, 4>(a, h, bwd, s); break;
    case 2: launch_halo<8, 3, 2, 4>(a, h, bwd, s); break;
    case 3: launch_halo<8, 2, 4, 4>(a, h, bwd, s); break;
    case 4: launch_halo<8, 3, 4, 4>(a, h, bwd, s); break;
    case 5: launch_halo<8, 4, 2, 4>(a, h, bwd, s); break;
    case 6: launch_halo<4, 3, 4, 11>(a, h, bwd, s); break;
    case 7: launch_halo<8, 2, 8, 11>(a, h, bwd, s); break;
    case 8: launch_halo<8, 3, 8, 11>(a, h, bwd, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t conv_halo(const ConvGeom& geom, const HaloPlan& h, bool bwd, const void* x, const void* w,
                     const float* bias, bool relu, const void* mask, void* y, hipStream_t s)
{
    if (!h.ok) return hipErrorInvalidValue;
    const ConvGeom g = halo_geom(geom, bwd);
    HaloArgs a{};
    a.x = static_cast<const bf16_t*>(x); a.w = static_cast<const bf16_t*>(w);
    a.bias = bias; a.mask = static_cast<const bf16_t*>(mask); a.y = static_cast<bf16_t*>(y);
    a.x_bytes = (unsigned)((size_t)g.N * g.C * g.H * g.W * 2);
    a.w_bytes = (unsigned)(h.w_elems * 2);
    a.y_bytes = (unsigned)((size_t)g.N * g.OC * g.OH * g.OW * 2);
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.OC = g.OC; a.OH = g.OH; a.OW = g.OW;
    a.K = g.K; a.PD = g.PD; a.G = g.G;
    a.cg = g.C / g.G; a.P = g.OC / g.G; a.Q = g.N * g.OH * g.OW; a.relu = relu;
    return launch_shape(a, h, g, bwd, s);
}

hipError_t conv_halo_run(const ConvGeom& g, const RunGeom& r, const HaloPlan& h, const void* xp,
                         const void* w, const float* bias, bool relu, void* y, hipStream_t s)
{
    if (!h.ok || g.G != 1) return hipErrorInvalidValue;
    HaloArgs a{};
    a.x = static_cast<const bf16_t*>(xp); a.w = static_cast<const bf16_t*>(w);
    a.bias = bias; a.y = static_cast<bf16_t*>(y);
    a.x_bytes = (unsigned)((size_t)g.N * r.Hp * r.Wp * r.Cp * 2);
    a.w_bytes = (unsigned)(h.w_elems * 2);
    a.y_bytes = (unsigned)((size_t)g.N * g.OC * g.OH * g.OW * 2);
    a.N = g.N; a.C = r.Cp; a.H = g.H; a.W = g.W; a.OC = g.OC; a.OH = g.OH; a.OW = g.OW;
    a.K = g.K; a.PD = 0; a.G = 1; a.S = g.S; a.Hp = r.Hp; a.row = r.Wp * r.Cp;
    a.cg = r.Cp; a.P = g.OC; a.Q = g.N * g.OH * g.OW; a.relu = relu;
    return launch_shape(a, h, g, false, s);
}

}  // namespace mtx
