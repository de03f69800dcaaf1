// Data gradient of a stride-2 convolution (bf16, K x K kernels from 2 x 2 to 7 x 7, output channels
// per group a multiple of 64), without the fp32 col buffer.
//
// An input position (h, w) takes the taps u = (h + PD) mod 2, + 2, ... (likewise v), so the
// positions of one parity class (h mod 2, w mod 2) are a stride-1 convolution of dy with every
// second tap: 4, 2, 2 and 1 taps of a 3 x 3 kernel, no product wasted.  A block computes 128
// positions of one class from a window of dy held in LDS, as conv_halo.hip does.  The col route
// this replaces stored every tap's sum over the output channels in fp32 (302 MB for 32 x 32 x 128
// at batch 256) and added them in a second pass in tap order; here a tap's sum is formed in the
// same order from zero and added to the position's total in the same order, so the results are
// the same bits.  Its bytes are dy, the mask and dx (151 MB at the size below, 30 us at a copy's rate);
// the rest is the start of every block, whose window must be there before its few products (4 k
// steps of a tap) begin.  32 x 32, 3 x 3, 128 -> 128, batch 256: col 73 + 105 us -> 54 us.
#include <algorithm>

#include "halo.h"

namespace mtx {

struct HaloS2Args {
    const bf16_t* dy;    // [N][OH][OW][OC]
    const bf16_t* w;     // fragment-major weights (PREP_HALO_D)
    const bf16_t* mask;  // stored output of the layer below (its ReLU), or null
    bf16_t* dx;          // [N][H][W][C]
    unsigned dy_bytes, w_bytes, dx_bytes;
    int N, C, H, W, OC, OH, OW, K, PD, G;
    int cg, og, ks, stride, PT, PB, zero_off, vout;
    int ch[4], cw[4], tiles[4], q[4];  // per class: rows, columns, blocks, positions
    FastDiv fd_hw[4], fd_w[4];
};

template <int FP, int WP, int FQ>
__global__ __launch_bounds__(512, 4) void conv_dgrad_s2_kernel(const HaloS2Args a)
{
    constexpr int NT = 512, WQ = 8 / WP, BP = 16 * FP * WP, BQ = 16 * FQ * WQ;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    // the four classes of a place are neighbours: they read the same rows of dy, and every die gets
    // as many of each (a class with a quarter of another's taps ends early)
    const unsigned nb = gridDim.x, hwb = blockIdx.x;
    const unsigned xq = nb / 8, xr = nb % 8, xc = hwb % 8;
    const unsigned l = xc * xq + min(xc, xr) + hwb / 8;
    const unsigned pg = (unsigned)(a.PT * a.G);
    const int cls = (int)(l / pg) & 3, qt = (int)(l / pg) >> 2;
    const int pgi = (int)(l % pg), grp = pgi / a.PT, p0 = (pgi % a.PT) * BP;
    if (qt >= a.tiles[cls]) return;
    const int ph = cls >> 1, pw = cls & 1;
    const int CH = a.ch[cls], CW = a.cw[cls], Q = a.q[cls];
    const FastDiv fhw = a.fd_hw[cls], fw = a.fd_w[cls];

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wp = wave % WP, wq = wave / WP;
    const int q0 = qt * BQ, q1 = min(q0 + BQ, Q) - 1;

    // taps u0, u0 + 2, ... of a row, dy row of the first one at class row i: i + dh
    const int u0 = (ph + a.PD) & 1, v0 = (pw + a.PD) & 1;
    const int dh = (ph + a.PD - u0) / 2, dw = (pw + a.PD - v0) / 2;
    const int TU = (a.K - u0 + 1) / 2, TV = (a.K - v0 + 1) / 2;

    const unsigned n0 = fdiv(fhw, (unsigned)q0), n1 = fdiv(fhw, (unsigned)q1);
    const int i0 = (int)fdiv(fw, (unsigned)q0 - n0 * (unsigned)(CH * CW));
    const int i1 = (int)fdiv(fw, (unsigned)q1 - n1 * (unsigned)(CH * CW));
    const int r0 = (int)n0 * a.OH + min(max(i0 + dh - (TU - 1), 0), a.OH - 1);
    const int r1 = (int)n1 * a.OH + min(max(i1 + dh, 0), a.OH - 1);
    const int ckg = a.og / 8, pos0 = r0 * a.OW, ngran = (r1 - r0 + 1) * a.OW * ckg;

    const __amdgpu_buffer_rsrc_t bx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.dy), (short)0, (int)a.dy_bytes, (int)kRsrcWord3);
    const __amdgpu_buffer_rsrc_t bw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.w), (short)0, (int)a.w_bytes, (int)kRsrcWord3);
    const __amdgpu_buffer_rsrc_t bm = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.mask), (short)0, (int)a.dx_bytes, (int)kRsrcWord3);

    constexpr int NS = 8;
    for (int t0 = tid; t0 < ngran; t0 += NT * NS) {
        u32x4 v[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int t = t0 + s * NT, pos = t / ckg, g = t - pos * ckg;
            const int off = (pos0 + pos) * a.OC + grp * a.og + g * 8;
            v[s] = __builtin_amdgcn_raw_buffer_load_b128(bx, t < ngran ? off * 2 : (int)kOOB, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int t = t0 + s * NT, pos = t / ckg, g = t - pos * ckg;
            if (t < ngran) *reinterpret_cast<u32x4*>(lds + pos * a.stride + g * 16) = v[s];
        }
    }
    for (int i = tid; i < ckg; i += NT)
        *reinterpret_cast<u32x4*>(lds + a.zero_off + i * 16) = u32x4{0u, 0u, 0u, 0u};

    int base[FQ], ok[FQ];  // origin (tap u0, v0), valid taps t (bits 0.. rows, 8.. columns)
#pragma unroll
    for (int j = 0; j < FQ; ++j) {
        const int q = q0 + (wq * FQ + j) * 16 + lr;
        const unsigned qq = q <= q1 ? q : q0;
        const unsigned n = fdiv(fhw, qq), r = qq - n * (unsigned)(CH * CW);
        const unsigned ci = fdiv(fw, r), cj = r - ci * (unsigned)CW;
        const int h = (int)ci + dh, w = (int)cj + dw;
        base[j] = (((int)n * a.OH + h) * a.OW + w - pos0) * a.stride;
        int m = 0;
        for (int t = 0; t < 4; ++t)
            m |= ((unsigned)(h - t) < (unsigned)a.OH) << t | ((unsigned)(w - t) < (unsigned)a.OW) << (8 + t);
        ok[j] = m;
    }

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
    f32x4 tot[FP][FQ];
#pragma unroll
    for (int i = 0; i < FP; ++i)
#pragma unroll
        for (int j = 0; j < FQ; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kt = ckg / 4;  // k steps of a tap (even)
    auto kstep = [&](int t) { return ((u0 + 2 * (t / TV)) * a.K + v0 + 2 * (t % TV)) * kt; };
    const int T = TU * TV;
    u32x4 fa0[FP], fa1[FP];
    int k = kstep(0);
    wload(fa0, k);
    wload(fa1, k + 1);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    for (int t = 0; t < T; ++t) {
        const int tu = t / TV, tv = t - tu * TV, need = 1 << tu | 1 << (8 + tv);
        const int o = (tu * a.OW + tv) * a.stride, knext = t + 1 < T ? kstep(t + 1) : k;
        int at[FQ];
#pragma unroll
        for (int j = 0; j < FQ; ++j)
            at[j] = ((ok[j] & need) == need ? base[j] - o : a.zero_off) + lg * 16;
        f32x4 acc[FP][FQ];
#pragma unroll
        for (int i = 0; i < FP; ++i)
#pragma unroll
            for (int j = 0; j < FQ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < kt; c += 2) {
            const int kn = c + 2 < kt ? k + c + 2 : knext;  // the k step after the next
            s16x8 fb[FQ];
#pragma unroll
            for (int j = 0; j < FQ; ++j) fb[j] = *reinterpret_cast<const s16x8*>(lds + at[j]);
#pragma unroll
            for (int j = 0; j < FQ; ++j)
#pragma unroll
                for (int i = 0; i < FP; ++i)
                    Mma<bf16_t>::run(acc[i][j], __builtin_bit_cast(s16x8, fa0[i]), fb[j]);
            wload(fa0, kn);
#pragma unroll
            for (int j = 0; j < FQ; ++j) {
                fb[j] = *reinterpret_cast<const s16x8*>(lds + at[j] + 64);
                at[j] += 128;
            }
#pragma unroll
            for (int j = 0; j < FQ; ++j)
#pragma unroll
                for (int i = 0; i < FP; ++i)
                    Mma<bf16_t>::run(acc[i][j], __builtin_bit_cast(s16x8, fa1[i]), fb[j]);
            wload(fa1, kn + 1);
        }
        k = knext;
        // (a tap outside dy adds nothing, whatever its weights)
#pragma unroll
        for (int j = 0; j < FQ; ++j)
            if ((ok[j] & need) == need)
#pragma unroll
                for (int i = 0; i < FP; ++i) tot[i][j] += acc[i][j];
    }

    constexpr int OSTR = BP + 8, GP = BP / 8, NO = (BQ * GP + NT - 1) / NT;
    const int pn = min(BP, a.cg - p0);
    // dx element of class position q, channel p0
    auto out_at = [&](int q) {
        const unsigned n = fdiv(fhw, (unsigned)q), r = (unsigned)q - n * (unsigned)(CH * CW);
        const unsigned ci = fdiv(fw, r), cj = r - ci * (unsigned)CW;
        return (((int)n * a.H + 2 * (int)ci + ph) * a.W + 2 * (int)cj + pw) * a.C + grp * a.cg + p0;
    };
    __syncthreads();
    bf16_t* ot = reinterpret_cast<bf16_t*>(lds);
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int pl = (wp * FP + i) * 16 + lg * 4;
#pragma unroll
        for (int j = 0; j < FQ; ++j) {
            const f32x4 v = tot[i][j];
            const unsigned lo = (unsigned)f32_to_bf16(v[0]) | ((unsigned)f32_to_bf16(v[1]) << 16);
            const unsigned hi = (unsigned)f32_to_bf16(v[2]) | ((unsigned)f32_to_bf16(v[3]) << 16);
            *reinterpret_cast<u32x2*>(ot + ((wq * FQ + j) * 16 + lr) * OSTR + pl) = u32x2{lo, hi};
        }
    }
    u32x4 mk[NO];
    int idx[NO];
    auto mask_rows = [&](auto width) {
        constexpr int W = decltype(width)::value;
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            const int q = (tid + t * NT) / GP, g = (tid + t * NT) % GP;
            idx[t] = q0 + q <= q1 && g * 8 < pn ? out_at(q0 + q) + g * 8 : -1;
            if constexpr (W > 1)
                if (a.mask) mk[t] = halo_row_load<W>(bm, idx[t] >= 0, idx[t], pn - g * 8);
        }
    };
    auto store_rows = [&](auto width) {
        constexpr int W = decltype(width)::value;
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            if (idx[t] < 0) continue;
            const int q = (tid + t * NT) / GP, g = (tid + t * NT) % GP;
            u32x4 v = *reinterpret_cast<const u32x4*>(ot + q * OSTR + g * 8);
            if constexpr (W > 1) {
                if (a.mask) v = halo_masked(v, mk[t]);
                halo_row_store<W>(a.dx + idx[t], v, pn - g * 8);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (g * 8 + e >= pn) break;
                    bf16_t b = (bf16_t)(v[e / 2] >> (16 * (e & 1)));
                    if (a.mask && !(bf16_to_f32(a.mask[idx[t] + e]) > 0.f)) b = 0;
                    a.dx[idx[t] + e] = b;
                }
            }
        }
    };
    auto finish = [&](auto width) {
        mask_rows(width);
        __syncthreads();
        store_rows(width);
    };
    if (a.vout == 8) finish(std::integral_constant<int, 8>{});
    else if (a.vout == 4) finish(std::integral_constant<int, 4>{});
    else finish(std::integral_constant<int, 1>{});
}

// ---- plan -------------------------------------------------------------------------------------
namespace {
struct ClassGeom { int ch, cw, u0, dh, TU; };
ClassGeom class_of(const ConvGeom& g, int cls)
{
    const int ph = cls >> 1, pw = cls & 1, u0 = (ph + g.PD) & 1;
    return ClassGeom{(g.H - ph + 1) / 2, (g.W - pw + 1) / 2, u0, (ph + g.PD - u0) / 2, (g.K - u0 + 1) / 2};
}
}  // namespace

HaloPlan conv_dgrad_s2_plan(int dt, const ConvGeom& g)
{
    HaloPlan h{};
    const int cg = g.C / g.G, og = g.OC / g.G;
    if (dt != DT_BF16 || g.S != 2 || g.K < 2 || g.K > 7 || og % 64 || g.H < 2 || g.W < 2) return h;
    // (the products of the col route, which must not be split)
    if (!conv_dgrad_use_col(g) || plan_for(dt, conv_dgrad_col_dims(dt, g)).splits > 1) return h;
    h.ckg = og / 8;
    h.ks = g.K * g.K * (og / 32);
    h.stride = og * 2 + 32;  // an odd multiple of 32 bytes
    h.shape = cg <= 64 ? 0 : 1;
    const int BP = h.shape ? 128 : 64, BQ = h.shape ? 128 : 256;
    auto clamp = [&](int r) { return std::min(std::max(r, 0), g.OH - 1); };
    long long rows = 0, blocks = 0, taps = 0;  // (taps: of all blocks)
    for (int cls = 0; cls < 4; ++cls) {
        const ClassGeom c = class_of(g, cls);
        const long long img = (long long)c.ch * c.cw, Q = img * g.N;
        if (Q > (1ll << 30)) return h;
        const int v0 = ((cls & 1) + g.PD) & 1, TV = (g.K - v0 + 1) / 2;
        blocks += (Q + BQ - 1) / BQ;
        taps += (Q + BQ - 1) / BQ * c.TU * TV;
        const long long period = img / std::__gcd<long long>(BQ, img) * BQ;
        for (long long q0 = 0; q0 < std::min(Q, period); q0 += BQ) {
            const long long q1 = std::min(q0 + BQ, Q) - 1;
            const int i0 = (int)(q0 % img / c.cw), i1 = (int)(q1 % img / c.cw);
            rows = std::max(rows, (q1 / img - q0 / img) * g.OH + clamp(i1 + c.dh) -
                                      clamp(i0 + c.dh - (c.TU - 1)) + 1);
        }
    }
    const long long win = rows * g.OW * h.stride + h.stride;
    const long long body = std::max(win, (long long)BQ * (BP + 8) * 2);
    if (body > 160 * 1024 || blocks * halo_cdiv(cg, BP) * g.G < 192) return h;
    h.zero_off = (int)(win - h.stride);
    h.lds = (int)body;
    h.PB = halo_cdiv(cg, 16);
    h.w_elems = (long long)g.G * h.PB * h.ks * 512;
    // Estimated time (see gemm_us): products and window pieces of the blocks on a compute unit.  Few
    // input channels fill a block's 64 rows badly: 8 <- 192 channels, 22 x 22, 3 x 3, 1920 images took
    // 169 us here, the col product 71 (23 drawn layers: 3 were slower, with this rule 1, by 5%).
    const double per_cu = halo_cdiv(cg, BP) * g.G / 256.0;
    const double us = 10.3 + per_cu * ((double)taps * (og / 32) * 16 * 0.014 +
                                       (double)blocks * (2.4 + h.zero_off / 16.0 / 512 *
                                                                   (h.lds > kHaloMaxLds ? 0.39 : 0.19)));
    h.ok = h.w_elems * 2 <= (1ll << 30) && us <= conv_dgrad_col_us(dt, g);
    return h;
}

hipError_t conv_dgrad_s2(const ConvGeom& g, const HaloPlan& h, const void* dy, const void* w,
                         const void* mask, void* dx, hipStream_t s)
{
    if (!h.ok) return hipErrorInvalidValue;
    HaloS2Args a{};
    a.dy = static_cast<const bf16_t*>(dy); a.w = static_cast<const bf16_t*>(w);
    a.mask = static_cast<const bf16_t*>(mask); a.dx = static_cast<bf16_t*>(dx);
    a.dy_bytes = (unsigned)((size_t)g.N * g.OC * g.OH * g.OW * 2);
    a.w_bytes = (unsigned)(h.w_elems * 2);
    a.dx_bytes = (unsigned)((size_t)g.N * g.C * g.H * g.W * 2);
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.OC = g.OC; a.OH = g.OH; a.OW = g.OW;
    a.K = g.K; a.PD = g.PD; a.G = g.G; a.cg = g.C / g.G; a.og = g.OC / g.G;
    a.ks = h.ks; a.stride = h.stride; a.PB = h.PB; a.zero_off = h.zero_off;
    a.vout = halo_row_width(a.cg);
    const int BP = h.shape ? 128 : 64, BQ = h.shape ? 128 : 256;
    int tiles = 0;
    for (int cls = 0; cls < 4; ++cls) {
        const ClassGeom c = class_of(g, cls);
        a.ch[cls] = c.ch; a.cw[cls] = c.cw; a.q[cls] = g.N * c.ch * c.cw;
        a.tiles[cls] = halo_cdiv(a.q[cls], BQ);
        tiles = std::max(tiles, a.tiles[cls] * 4);
        a.fd_hw[cls] = make_fastdiv((unsigned)(c.ch * c.cw));
        a.fd_w[cls] = make_fastdiv((unsigned)c.cw);
    }
    a.PT = halo_cdiv(a.cg, BP);
    const dim3 grid((unsigned)(tiles * a.PT * a.G));
    note_gemm(BP, BQ, 32, 1, kGemmHalo);
    if (h.shape) hipLaunchKernelGGL((conv_dgrad_s2_kernel<2, 4, 4>), grid, dim3(512), (size_t)h.lds, s, a);
    else hipLaunchKernelGGL((conv_dgrad_s2_kernel<2, 2, 4>), grid, dim3(512), (size_t)h.lds, s, a);
    return hipGetLastError();
}

}  // namespace mtx
