// adjoint.hip -- one reverse round of the unpooled mean-field on lane groups:
// the adjoint message of round t, the parameter sums, and the adjoints of the
// softmax, unary addition and compatibility of round t - 1, for k = 3, 5, 7.
//
// Compiled once per window side k (-DCRF_ADJ_K=k).  Four lanes share four
// horizontally adjacent pixels and split the window (rows four apart for the
// two 16-lane rows of each half-wavefront, as group.hip explains); each holds
// the weights of its taps and, beside them, the sums dk(x, x + d) over the
// classes, while Q^t and dL/dM^t stream through LDS two classes at a time.
// All classes pass through one work-group, so that a pixel's weights are
// computed once and the pointwise adjoints, which need every class, follow
// from registers: dL/dQ^t is never written.
//
// Bound by the issue of vector instructions: three FMAs a tap and class, and
// the weights twice (their parts are taken again for the parameter sums, which
// is less than holding them); of a work-group's 66 k clocks the chunks take 31,
// the weights and the sums 11, the product of matrices 8, the epilogue 7, and two
// work-groups share a CU.  1 x 21 x 512 x 512, k = 7, Potts, per round: the
// message, a pointwise kernel and the dL/dQ between them 96 us, this kernel 69;
// the whole backward pass of five rounds 582 -> 449 us.  With two learned
// features and compatibility (2 x 21 x 240 x 320) 699 -> 575 us.
#include "crf_internal.h"
#include "lane_group.h"
#include "lds_dma.h"

#ifndef CRF_ADJ_K
#error "compile with -DCRF_ADJ_K=<3, 5 or 7>"
#endif

namespace convcrf {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// The window over four lanes: NF full rows each and NT taps of the centre row
// (k = 5), or rows alone (k = 3 and 7, whose last part repeats one, weighing
// zero).
template <int K>
struct AdjSplit {
    static constexpr bool PART = K == 5;
    static constexpr int NF = K == 7 ? 2 : 1, NT = PART ? 1 : 0;
    static constexpr int NS = NF + NT, NTAP = NF * K + NT;
    static constexpr unsigned rows(int j) {
        return K == 3 ? 0x1120u : K == 5 ? 0x3140u : j == 0 ? 0x5140u : 0x3362u;
    }
    __device__ static int row(int g, int j) { return (int)(rows(j) >> (4 * g)) & 15; }
    static constexpr bool spare(int j) { return !PART && j == NF - 1; }
    __device__ static int ct(int g) { return g + (g >= 2 ? 1 : 0); }
};

// CM: class planes the registers hold (even, >= a.C).  FD: feature planes
// staged (0, 2 or 4).  WM: the compatibility derivative too.  A16: staged with
// 16-byte loads.
template <int K, int CM, int FD, bool WM, bool A16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void adj_kernel(const AdjArgs a) {
    using S = AdjSplit<K>;
    constexpr int R = (K - 1) / 2, NF = S::NF, NS = S::NS, CH = kAdjCH, PLANE = kAdjPlane;
    constexpr int TW = kAdjTW, TH = kAdjTH, LS = 80, XO = 4, SH = XO - R, LH = TH + 2 * R;
    constexpr int NWAVE = 4, VF = A16 ? 4 : 1, NV = PLANE / (64 * VF * NWAVE);
    constexpr int SLOT = 2 * CH * PLANE, L = 2 * CH * NV;
    constexpr int NCH = CM / CH, NPR = (SH + K + 3 + 3) / 4, SP = 257;
    static_assert(CM % CH == 0 && LH * LS <= PLANE && LS >= XO + TW + R, "the tile fits its plane");
    extern __shared__ float4 smem4[];
    float* const smem = reinterpret_cast<float*>(smem4);
    float* const Qs = smem;                        // [kAdjSlots][Q planes, dL/dM planes]
    float* const Cs = Qs + kAdjSlots * SLOT;       // [3][PLANE]
    float* const Fs = Cs + 3 * PLANE;              // [FD][PLANE]
    float* const Tb = Fs + FD * PLANE;             // the tap table
    float* const Mt = Tb + kGroupTab;              // compatibility transposed [CM][CM4]
    constexpr int CM4 = (CM + 3) / 4 * 4;
    __shared__ float red[5][NWAVE];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) float*)smem;
    auto lds_addr = [&](const float* p) { return lds0 + (unsigned)((p - smem) * 4); };

    const int C = a.C, H = a.H, W = a.W;
    const int tile = xcd_tile(blockIdx.x, a.ntiles);
    const int b = tile / a.tiles_per_img;
    const int trem = tile - b * a.tiles_per_img;
    const int tyi = trem / a.tiles_x;
    const int y0 = tyi * TH, x0 = (trem - tyi * a.tiles_x) * TW;
    const size_t HW = (size_t)H * W;
    const int hw4 = (int)(HW * 4);
    const int nch = (C + CH - 1) / CH;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane >> 4, cq = 4 * (lane & 15), ty = wave;
    const int y = y0 + ty, xo = x0 + cq + g;       // the pixel this lane finishes
    const bool in = y < H && xo < W;

    // ---- every load straight into LDS (as group_kernel): table, compatibility,
    // colours, features, then the first chunks
    {
        const char* const args = (const char*)__builtin_amdgcn_kernarg_segment_ptr();
        const rsrc_t rt = buffer_rsrc((const float*)(args + offsetof(AdjArgs, a_log2)),
                                      (unsigned)(2 * (kMaxN + 1) * sizeof(float)));
        lds_dma(rt, (wave * 64 + lane) * 4, 0, lds_addr(Tb + wave * 64));
        if (a.mu) {
            const rsrc_t rm = buffer_rsrc(a.mu, (unsigned)(C * C * 4));
            for (int j = wave; j < (CM * CM4 + 63) / 64; j += NWAVE) {
                const int i = j * 64 + lane, lp = i / CM4, l = i - (i / CM4) * CM4;
                lds_dma(rm, l < C && lp < C ? (unsigned)((l * C + lp) * 4) : kDmaOob, 0,
                        lds_addr(Mt + j * 64));
            }
        }
    }
    unsigned voff[NV];
#pragma unroll
    for (int s = 0; s < NV; ++s) {
        const int f = ((wave + NWAVE * s) * 64 + lane) * VF;
        const int r = f / LS, col = f - (f / LS) * LS;
        const int gy = y0 - R + r, gx = x0 - XO + col;
        const bool ok = f < LH * LS && gy >= 0 && gy < H && gx >= 0 && gx < W;
        voff[s] = ok ? (unsigned)((gy * W + gx) * 4) : kDmaOob;
    }
    const unsigned lw = lds0 + (unsigned)(wave * 64 * VF * 4);
    // plane p of a tensor (zeros unless ok) to float offset `to`
    auto stage = [&](rsrc_t r, int p, bool ok, unsigned to) {
#pragma unroll
        for (int s = 0; s < NV; ++s) {
            const unsigned at = lw + (to + (unsigned)(s * NWAVE * 64 * VF)) * 4;
            const unsigned vo = ok ? voff[s] : kDmaOob;
            if constexpr (A16) lds_dma16(r, vo, ok ? p * hw4 : 0, at);
            else lds_dma(r, vo, ok ? p * hw4 : 0, at);
        }
    };
    const rsrc_t rf = buffer_rsrc(a.image + (size_t)b * 3 * HW, (unsigned)(3 * HW * 4));
    const rsrc_t rq = buffer_rsrc(a.q + (size_t)b * C * HW, (unsigned)(C * HW * 4));
    const rsrc_t rm = buffer_rsrc(a.dm + (size_t)b * C * HW, (unsigned)(C * HW * 4));
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) stage(rf, ch, true, (unsigned)(Cs - smem) + ch * PLANE);
    if constexpr (FD > 0) {
        const rsrc_t rs = buffer_rsrc(a.sfeat + (size_t)b * a.D * HW, (unsigned)(a.D * HW * 4));
#pragma unroll
        for (int ch = 0; ch < FD; ++ch)
            stage(rs, ch, ch < a.D, (unsigned)(Fs - smem) + ch * PLANE);
    }
    auto issue_chunk = [&](int k) {
        const unsigned to = (unsigned)((k % kAdjSlots) * SLOT);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            stage(rq, k * CH + i, k * CH + i < C, to + i * PLANE);
            stage(rm, k * CH + i, k * CH + i < C, to + (CH + i) * PLANE);
        }
    };
#pragma unroll
    for (int k = 0; k < kAdjSlots; ++k)
        if (k < nch) issue_chunk(k);

    // ---- colours landed: the weights of the lane's taps
    if (nch >= 3) __builtin_amdgcn_s_waitcnt(vm_wait(3 * L));
    else if (nch == 2) __builtin_amdgcn_s_waitcnt(vm_wait(2 * L));
    else __builtin_amdgcn_s_waitcnt(vm_wait(L));
    __syncthreads();
    unsigned base[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        base[j] = (unsigned)((ty + S::row(g, j)) * LS + cq);
        asm volatile("" : "+v"(base[j]));
    }
    unsigned hbase = (unsigned)((ty + R) * LS + cq + SH + (S::PART ? S::ct(g) : 0));
    unsigned obase = (unsigned)((ty + R) * LS + cq + XO);
    asm volatile("" : "+v"(hbase), "+v"(obase));

    // The taps of step j, one pixel quad against one staged row: f(t, i, e) for
    // tap t of the lane, pixel i, element e of the row's pieces.  A whole row
    // starts SH into its pieces, the centre row's taps (j = NF) at its start.
    auto each = [&](auto jc, auto&& f) {
        constexpr int j = decltype(jc)::value;
        constexpr int n = j == NF ? S::NT : K, o = j == NF ? 0 : SH;
#pragma unroll
        for (int d = 0; d < n; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) f(j * K + d, d, i, o + i + d);
    };
    auto read_step = [&](auto jc, const float* plane, f32x4 (&v)[NPR]) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j < NF) {
            read_row(plane + base[j], v);
        } else {
#pragma unroll
            for (int e = 0; e < S::NT + 3; ++e) v[e / 4][e % 4] = plane[hbase + e];
        }
    };
    auto use_step = [&](auto jc, f32x4 (&v)[NPR]) {
        if constexpr (decltype(jc)::value < NF)
#pragma unroll
            for (int p = 0; p < NPR; ++p) use(v[p]);
    };
    // offset of step j's tap d from the centre, and whether the lane has it
    auto tap_dy = [&](auto jc) { return decltype(jc)::value < NF ? S::row(g, decltype(jc)::value) - R : 0; };
    auto tap_dx = [&](auto jc, int d) {
        return decltype(jc)::value < NF ? d - R : (S::PART ? S::ct(g) : 0) + d - R;
    };
    // One step's kernel parts.  Per tap: av, sv = the Gaussians of Eq. 4
    // without their weights (zero for the centre and a repeated row), cd2 =
    // the squared colour distance, sd2 = the squared distance sv is taken on;
    // handed to f(t, d, i, av, sv, cd2, sd2).
    auto parts = [&](auto jc, auto&& f) {
        constexpr int j = decltype(jc)::value;
        constexpr int n = j == NF ? S::NT : K;
        const int dy = tap_dy(jc);
        const bool keep = j == NF || !S::spare(j) || g < 3;
        float fd2[FD > 0 ? n : 1][4];
        if constexpr (FD > 0) {
#pragma unroll
            for (int d = 0; d < n; ++d)
#pragma unroll
                for (int i = 0; i < 4; ++i) fd2[d][i] = 0.f;
#pragma unroll
            for (int ch = 0; ch < FD; ++ch) {
                f32x4 v[NPR];
                read_step(jc, Fs + ch * PLANE, v);
                const f32x4 fo = *reinterpret_cast<const f32x4*>(Fs + ch * PLANE + obase);
                use_step(jc, v);
                each(jc, [&](int, int d, int i, int e) {
                    const float x = fo[i] - v[e / 4][e % 4];
                    fd2[d][i] = fmaf(x, x, fd2[d][i]);
                });
            }
        }
        f32x4 nc[3][NPR], own[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            read_step(jc, Cs + ch * PLANE, nc[ch]);
            own[ch] = *reinterpret_cast<const f32x4*>(Cs + ch * PLANE + obase);
        }
        float al[n], s0[n], nn[n];
#pragma unroll
        for (int d = 0; d < n; ++d) {
            const int dx = tap_dx(jc, d), m = dy * dy + dx * dx;
            const bool none = !keep || (!S::PART && m == 0);
            al[d] = none ? -INFINITY : Tb[m];
            s0[d] = none ? 0.f : FD > 0 ? 1.f : Tb[kMaxN + 1 + m];
            nn[d] = (float)m;
        }
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) use_step(jc, nc[ch]);
        each(jc, [&](int t, int d, int i, int e) {
            const float er = own[0][i] - nc[0][e / 4][e % 4];
            const float eg = own[1][i] - nc[1][e / 4][e % 4];
            const float eb = own[2][i] - nc[2][e / 4][e % 4];
            const float cd2 = fmaf(er, er, fmaf(eg, eg, eb * eb));
            const float av = __builtin_amdgcn_exp2f(fmaf(a.neg_beta, cd2, al[d]));
            const float sd2 = FD > 0 ? fd2[d][i] : nn[d];
            const float sv = FD > 0 ? s0[d] * __builtin_amdgcn_exp2f(a.neg_gamma * fd2[d][i]) : s0[d];
            f(t, d, i, av, sv, cd2, sd2, nn[d]);
        });
    };
    using Steps = std::make_integer_sequence<int, NS>;

    float w[4][S::NTAP], dk[4][S::NTAP];
    static_for([&](auto jc) {
        parts(jc, [&](int t, int, int i, float av, float sv, float, float, float) {
            w[i][t] = fmaf(a.w_app, av, a.w_smooth * sv);
            asm volatile("" : "+v"(w[i][t]));
        });
        __builtin_amdgcn_sched_barrier(0);
    }, Steps{});
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < S::NTAP; ++t) dk[i][t] = 0.f;
    __builtin_amdgcn_sched_barrier(0);

    // ---- the classes: dq = sum_d K(x, x + d) dM_{x+d} (the transpose of the
    // message, by K's symmetry), the forward message M likewise from Q, and
    // dk(x, x + d) = sum_l dM_x(l) Q_{x+d}(l) (with features plus its mirror
    // sum_l dM_{x+d}(l) Q_x(l): the parameter terms are symmetric in the pair,
    // so half of both is either summed over the image, and dL/dF needs both)
    float dq[CM], mf[WM ? CM : 1], dkc = 0.f;
#pragma unroll
    for (int c = 0; c < CM; ++c) dq[c] = 0.f;
    if constexpr (WM)
#pragma unroll
        for (int c = 0; c < CM; ++c) mf[c] = 0.f;
    static_for([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if (k >= nch) return;
        const int after = k == 0 ? (nch >= 3 ? 2 : nch - 1) : (k + 1 < nch ? 1 : 0);
        if (after == 2) __builtin_amdgcn_s_waitcnt(vm_wait(2 * L));
        else if (after == 1) __builtin_amdgcn_s_waitcnt(vm_wait(L));
        else __builtin_amdgcn_s_waitcnt(vm_wait(0));
        __syncthreads();
        if (k >= 1 && k + 2 < nch) issue_chunk(k + 2);
        const float* const qk = Qs + (k % kAdjSlots) * SLOT;
        // rows of step t = class t / NS, window step t % NS, one step ahead
        f32x4 qr[2][NPR], mr[2][NPR], dmo[CH], qo[FD > 0 ? CH : 1];
        constexpr int nsteps = CH * NS;
        auto rd = [&](auto tc) {
            constexpr int t = decltype(tc)::value, c = t / NS, j = t % NS;
            constexpr std::integral_constant<int, j> jc{};
            if constexpr (j == 0) {
                dmo[c] = *reinterpret_cast<const f32x4*>(qk + (CH + c) * PLANE + obase);
                if constexpr (FD > 0) qo[c] = *reinterpret_cast<const f32x4*>(qk + c * PLANE + obase);
            }
            read_step(jc, qk + c * PLANE, qr[t & 1]);
            read_step(jc, qk + (CH + c) * PLANE, mr[t & 1]);
        };
        rd(std::integral_constant<int, 0>{});
        float da[4], ma[4];
        static_for([&](auto tc) {
            constexpr int t = decltype(tc)::value, c = t / NS, j = t % NS;
            constexpr std::integral_constant<int, j> jc{};
            if constexpr (t + 1 < nsteps) rd(std::integral_constant<int, t + 1>{});
            if constexpr (j == 0)
#pragma unroll
                for (int i = 0; i < 4; ++i) da[i] = ma[i] = 0.f;
            use_step(jc, qr[t & 1]);
            use_step(jc, mr[t & 1]);
            each(jc, [&](int tp, int, int i, int e) {
                const float q = qr[t & 1][e / 4][e % 4], m = mr[t & 1][e / 4][e % 4];
                dk[i][tp] = fmaf(dmo[c][i], q, dk[i][tp]);
                if constexpr (FD > 0) dk[i][tp] = fmaf(qo[c][i], m, dk[i][tp]);
                da[i] = fmaf(w[i][tp], m, da[i]);
                if constexpr (WM) ma[i] = fmaf(w[i][tp], q, ma[i]);
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j == NS - 1) {
                constexpr int cc = k * CH + c;
                dq[cc] = add_rows(add_halves(da[0], da[2]), add_halves(da[1], da[3]));
                if constexpr (WM)
                    mf[cc] = add_rows(add_halves(ma[0], ma[2]), add_halves(ma[1], ma[3]));
                if (a.include_center) {
                    const float qc = qk[c * PLANE + obase + g], mc = qk[(CH + c) * PLANE + obase + g];
                    dq[cc] = fmaf(a.center_w, mc, dq[cc]);
                    if constexpr (WM) mf[cc] = fmaf(a.center_w, qc, mf[cc]);
                    dkc = fmaf(mc, qc, dkc);
                }
                asm volatile("" : "+v"(dq[cc]));
                if constexpr (WM) asm volatile("" : "+v"(mf[cc]));
            }
        }, std::make_integer_sequence<int, nsteps>{});
    }, std::make_integer_sequence<int, NCH>{});

    const int po = in ? (int)((unsigned)(y * W + xo) * 4u) : (int)kDmaOob;
    auto buf = [&](const float* p, int planes) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(p + (size_t)b * planes * HW), (short)0,
                                                 (int)(planes * HW * 4), 0x00020000);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t r, int c) {
        return __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(r, po, c * hw4, 0));
    };
    auto store = [&](__amdgpu_buffer_rsrc_t r, int c, float v) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, po, c * hw4, 0);
    };
    // What the product of matrices below takes of this pixel: under way during the
    // sums, where the registers reach for it.
    const bool potts = a.dm_sum_scale != 0.f;
    float pv[WM ? CM : 1];
    auto load_dp = [&] {
        if constexpr (WM) {
            const auto rp = buf(potts ? a.dm : a.dp, C);
#pragma unroll
            for (int c = 0; c < CM; ++c) pv[c] = load(rp, c < C ? c : C - 1);
        }
    };
    if constexpr (FD == 0) load_dp();

    // ---- the five parameter sums (the parts taken again) and dL/dF
    float gs[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    float df[FD > 0 ? FD : 1][4];
    if constexpr (FD > 0)
#pragma unroll
        for (int ch = 0; ch < FD; ++ch)
#pragma unroll
            for (int i = 0; i < 4; ++i) df[ch][i] = 0.f;
    static_for([&](auto jc) {
        parts(jc, [&](int t, int, int i, float av, float sv, float cd2, float sd2, float nn) {
            const float da = dk[i][t] * av, ds = dk[i][t] * sv;
            gs[0] += da;
            gs[1] = fmaf(da, nn, gs[1]);
            gs[2] = fmaf(da, cd2, gs[2]);
            gs[3] += ds;
            gs[4] = fmaf(ds, sd2, gs[4]);
            if constexpr (FD > 0) {
                dk[i][t] = -ds * a.w_smooth * a.inv_gamma2;
                asm volatile("" : "+v"(dk[i][t]));
            }
        });
#pragma unroll
        for (int e = 0; e < 5; ++e) asm volatile("" : "+v"(gs[e]));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FD > 0) {
#pragma unroll
            for (int ch = 0; ch < FD; ++ch) {
                f32x4 v[NPR];
                read_step(jc, Fs + ch * PLANE, v);
                const f32x4 fo = *reinterpret_cast<const f32x4*>(Fs + ch * PLANE + obase);
                use_step(jc, v);
                each(jc, [&](int t, int, int i, int e) {
                    df[ch][i] = fmaf(dk[i][t], fo[i] - v[e / 4][e % 4], df[ch][i]);
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }, Steps{});
    if constexpr (FD > 0)
#pragma unroll
        for (int e = 0; e < 5; ++e) gs[e] *= 0.5f;
    gs[0] += dkc;                                  // the centre: both Gaussians are 1
    gs[3] += dkc;
#pragma unroll
    for (int e = 0; e < 5; ++e)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) gs[e] += __shfl_xor(gs[e], off, 64);
    if (lane == 0)
#pragma unroll
        for (int e = 0; e < 5; ++e) red[e][wave] = gs[e];

    if constexpr (FD > 0) {
        const auto rd = buf(a.dfeat, a.D);
#pragma unroll
        for (int ch = 0; ch < FD; ++ch) {
            const float v = add_rows(add_halves(df[ch][0], df[ch][2]), add_halves(df[ch][1], df[ch][3]));
            if (ch < a.D) store(rd, ch, a.accumulate ? load(rd, ch) + v : v);
        }
    }
    __syncthreads();                               // the staged planes have been read
    if (tid < 5) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NWAVE; ++i) s += red[tid][i];
        float* o = a.kpart + (size_t)tile * 5 + tid;
        *o = a.accumulate ? *o + s : s;
    }

    // Q and dL/dU of this pixel, for the pointwise adjoints at the end
    float qv[CM], uo[CM];
    const auto r1 = buf(a.q, C), r2 = buf(a.du, C);
    auto load_own = [&] {
#pragma unroll
        for (int c = 0; c < CM; ++c) {
            qv[c] = load(r1, c < C ? c : C - 1);
            uo[c] = load(r2, c < C ? c : C - 1);
        }
    };

    // ---- the tile's sum of -dZ_x(l) M_x(l') over its pixels, a product of
    // matrices over 256 pixels: 64 on each wavefront's matrix core, two a step
    if constexpr (WM) {
        float* const gp = smem;                    // [CM][SP] -dZ
        float* const gm = smem + CM * SP;          // [CM][SP] M
        if constexpr (FD > 0) load_dp();
        float psum = 0.f;
#pragma unroll
        for (int c = 0; c < CM; ++c) psum += c < C ? pv[c] : 0.f;
        const float sh = psum * a.dm_sum_scale;
#pragma unroll
        for (int c = 0; c < CM; ++c) {
            // Potts: dZ(l) = dM(l) + sum_l' dM(l') / (1 - C)
            const float p = potts ? -(pv[c] + sh) : pv[c];
            gp[c * SP + tid] = in && c < C ? p : 0.f;
            gm[c * SP + tid] = in && c < C ? mf[c] : 0.f;
        }
        load_own();
        // the sums so far (at most three entries a thread, C * C <= 576)
        float old[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const int i = tid + 256 * e;
            old[e] = a.accumulate && i < C * C ? a.gpart[(size_t)tile * C * C + i] : 0.f;
        }
        __syncthreads();
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        const int cl = (lane & 31) < CM ? lane & 31 : CM - 1;
        const int px = wave * 64 + (lane >> 5);
#pragma unroll 8
        for (int p = 0; p < 64; p += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(gp[cl * SP + px + p], gm[cl * SP + px + p],
                                                       acc, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e)
            smem[wave * 1024 + (8 * (e / 4) + e % 4 + 4 * (lane >> 5)) * 32 + (lane & 31)] = acc[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const int i = tid + 256 * e;
            if (i >= C * C) continue;
            const int l = i / C, at = l * 32 + i - l * C;
            a.gpart[(size_t)tile * C * C + i] =
                old[e] + ((smem[at] + smem[1024 + at]) + (smem[2048 + at] + smem[3072 + at]));
        }
    }

    // ---- the pointwise adjoints of round t - 1 (Q^t = softmax(Z)):
    // dZ = Q (dQ - <Q, dQ>), dU += dZ, dM(l') = -sum_l mu[l][l'] dZ(l)
    if constexpr (!WM) load_own();
    float dot = 0.f, sum = 0.f;
#pragma unroll
    for (int c = 0; c < CM; ++c) dot = c < C ? fmaf(qv[c], dq[c], dot) : dot;
#pragma unroll
    for (int c = 0; c < CM; ++c) {
        dq[c] = c < C ? qv[c] * (dq[c] - dot) : 0.f;
        sum += dq[c];
    }
#pragma unroll
    for (int c = 0; c < CM; ++c)
        if (c < C) store(r2, c, uo[c] + dq[c]);
    if (!a.dm_out) return;
    const auto r3 = buf(a.dm_out, C);
    if (a.mu) {
        if (a.dp_out) {
            const auto r4 = buf(a.dp_out, C);
#pragma unroll
            for (int c = 0; c < CM; ++c)
                if (c < C) store(r4, c, -dq[c]);
        }
#pragma unroll
        for (int lp = 0; lp < CM; ++lp) {
            if (lp >= C) continue;
            float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int l = 0; l < CM; l += 4) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(Mt + lp * CM4 + l);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (l + e < CM) t[e] = fmaf(v[e], -dq[l + e], t[e]);
            }
            store(r3, lp, (t[0] + t[1]) + (t[2] + t[3]));
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // Potts, mu[l][l'] = [l != l']: dm(l') = dZ(l') - sum_l dZ(l)
#pragma unroll
        for (int c = 0; c < CM; ++c)
            if (c < C) store(r3, c, dq[c] - sum);
    }
}

template <int K, int CM, int FD, bool WM, bool A16>
hipError_t launch_adj_one(const AdjArgs& a, hipStream_t stream) {
    auto fn = adj_kernel<K, CM, FD, WM, A16>;
    static unsigned long long done = 0;            // devices opted into 160 KB of LDS
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(done & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
        if (e != hipSuccess) return e;
        done |= bit;
    }
    hipLaunchKernelGGL(fn, dim3(a.ntiles), dim3(256), adj_lds_bytes(CM, FD, a.mu != nullptr), stream, a);
    return hipGetLastError();
}

template <int K, int CM, int FD>
hipError_t launch_adj_fd(const AdjArgs& a, hipStream_t stream) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a.q) | reinterpret_cast<uintptr_t>(a.dm) |
                        reinterpret_cast<uintptr_t>(a.image) |
                        (FD > 0 ? reinterpret_cast<uintptr_t>(a.sfeat) : 0);
    const bool a16 = a.W % 4 == 0 && p % 16 == 0;
    if (a.gpart)
        return a16 ? launch_adj_one<K, CM, FD, true, true>(a, stream)
                   : launch_adj_one<K, CM, FD, true, false>(a, stream);
    return a16 ? launch_adj_one<K, CM, FD, false, true>(a, stream)
               : launch_adj_one<K, CM, FD, false, false>(a, stream);
}

template <int K, int CM>
hipError_t launch_adj_cm(const AdjArgs& a, hipStream_t stream) {
    if (!a.sfeat) return launch_adj_fd<K, CM, 0>(a, stream);
    return a.D <= 2 ? launch_adj_fd<K, CM, 2>(a, stream) : launch_adj_fd<K, CM, 4>(a, stream);
}

}  // namespace

#define CRF_CAT2(a, b) a##b
#define CRF_CAT(a, b) CRF_CAT2(a, b)
hipError_t CRF_CAT(launch_adj_k, CRF_ADJ_K)(AdjArgs a, hipStream_t stream) {
    if (a.C < 1 || a.C > kMaxC || (a.sfeat && (a.D < 1 || a.D > kMaxFeat)))
        return hipErrorNotSupported;
    a.tiles_x = (a.W + kAdjTW - 1) / kAdjTW;
    a.tiles_per_img = a.tiles_x * ((a.H + kAdjTH - 1) / kAdjTH);
    a.ntiles = a.tiles_per_img * a.B;
    return a.C <= 12 ? launch_adj_cm<CRF_ADJ_K, 12>(a, stream)
                     : a.C <= 22 ? launch_adj_cm<CRF_ADJ_K, 22>(a, stream)
                                 : launch_adj_cm<CRF_ADJ_K, 24>(a, stream);
}

}  // namespace convcrf
