// group.hip -- one mean-field round on lane groups: any class count up to
// kMaxC, any width and alignment, Potts or a general compatibility, with or
// without learnable smoothness features (Sec. 4.2), for k = 3 .. 15.
//
// Compiled once per window side k (-DCRF_GROUP_K=k).  A group of G lanes
// shares four horizontally adjacent pixels and splits the window between its
// lanes, so that every weight of the tile (Eq. 4) is computed once and held in
// registers while the classes stream through LDS in chunks, and a lane reads
// k + 3 staged values of a window row for 4 k FMAs.  The lanes of a group lie
// 64 / G apart: the sixteen lanes that read LDS together read consecutive
// 16-byte pieces of one row, and the partial messages are added by
// half-wavefront and row swaps, two values per instruction, without selects.
//
// Bound by the issue of the two wavefronts a SIMD holds (one instruction per
// four clocks each; 25 .. 30 thousand clocks a tile at k = 7, of which the
// message takes 15, the weights 7, softmax and stores 3.5, the loads' issue 5;
// the classes' loads are waited for less than 200 clocks a chunk).  What it
// measured against the kernels that ran these shapes before (us a round):
// 1 x 21 x 512 x 512, k = 11: 96 -> 43; 4 x 12 x 240 x 320, k = 5, general
// compatibility: 42 -> 15.5; 1 x 21 x 500 x 375, k = 7: 25 -> 20.5; 1 x 21 x
// 512 x 512, k = 7: 19.8 -> 18.5, with two feature planes 23 -> 22.5.
// Loads of 16 bytes a lane instead of 4 and rows that LDS serves at full rate
// (Split below) were worth 9% and 5% of that; four parts instead of two at
// k = 7 (three wavefronts a SIMD, a sixth more FMAs) lost 20%.
#include "crf_internal.h"
#include "lane_group.h"
#include "lds_dma.h"

#ifndef CRF_GROUP_K
#error "compile with -DCRF_GROUP_K=<odd window side>"
#endif

namespace convcrf {
namespace {

// x + x of the lane eight away in the 16-lane row
[[maybe_unused]] __device__ __forceinline__ float add_eights(float x) {
    return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xF, 0xF, false));
}

// The split of a k x k window over the G lanes of a group: part g takes NF
// full rows and, where k - 1 divides by G, NT taps of the centre row from
// column ct(g) on (the centre itself is nobody's).  Which rows a part takes
// follows from how LDS serves 16-byte reads: lanes 0..15 and 16..31 of each
// half-wavefront are served together, 256 bytes a clock if what they read lies
// a multiple of 64 floats apart and 146 otherwise (measured).  With rows 80
// floats apart (48 at k = 15) that is a multiple of four rows, so the two
// 16-lane rows of a half take window rows (G >= 4) or tile rows (G = 2) four
// apart; at k = 11 and 13 one pair is left that is not.
template <int K>
struct Split : GroupShape<K> {
    using S = GroupShape<K>;
    static constexpr bool PART = S::NT > 0;
    static constexpr int NS = S::NF + (PART ? 1 : 0);      // steps per class
    static constexpr int NTAP = S::NF * K + S::NT;         // taps of a lane
    // the centre row's taps start at columns 0 and 4: whole pieces from there
    static constexpr bool WHOLE = PART && S::G == 2 && S::NT == 3;
    // window row of part g at step j; 4 bits a part, part 0 lowest
    static constexpr unsigned rows(int j) {
        constexpr unsigned t3[] = {0x20}, t5[] = {0x30, 0x41}, t7[] = {0x40, 0x51, 0x62};
        constexpr unsigned t9[] = {0x7351, 0x8062}, t11[] = {0x7340, 0x9851, 0x2a62};
        constexpr unsigned t13[] = {0xc840, 0xa251, 0xb973}, t15[] = {0xeac86240, 0x7bd97351};
        return K == 3 ? t3[j] : K == 5 ? t5[j] : K == 7 ? t7[j] : K == 9 ? t9[j]
             : K == 11 ? t11[j] : K == 13 ? t13[j] : t15[j];
    }
    __device__ static int row(int g, int j) { return (int)(rows(j) >> (4 * g)) & 15; }
    // k = 11 and 15 have a row less than their parts take: the last part's
    // last step repeats one, weighing zero
    static constexpr bool spare(int j) { return (K == 11 || K == 15) && j == S::NF - 1; }
    __device__ static int ct(int g) { return S::NT * g + (g >= S::G / 2 ? 1 : 0); }
};

// CM: class planes the registers hold (a multiple of kGroupCH, >= a.C).
// FD: feature planes staged (0, 2 or 4, >= a.D; the surplus reads zero).
// A16: staged with 16-byte loads (W a multiple of 4, 16-byte aligned planes).
template <int K, int CM, int FD, bool A16>
__global__ __launch_bounds__(64 * GroupShape<K>::NWAVE)
__attribute__((amdgpu_waves_per_eu(K <= 5 ? 3 : 2, 4)))
void group_kernel(const GroupArgs a) {
    using S = Split<K>;
    constexpr int R = (K - 1) / 2, G = S::G, NF = S::NF, NT = S::NT, NS = S::NS, CH = kGroupCH;
    constexpr int TW = S::TW, TH = S::TH, NWAVE = S::NWAVE;
    constexpr int LH = TH + 2 * R, LS = S::LS, PLANE = S::PLANE, XO = S::XO, SH = XO - R;
    constexpr int VF = A16 ? 4 : 1;                // floats per lane of a load
    constexpr int NI = PLANE / (64 * VF);          // loads per plane
    constexpr int L = (CH * NI + NWAVE - 1) / NWAVE;   // per wave and chunk
    constexpr int NV = NI % NWAVE == 0 ? NI / NWAVE : L;   // distinct offsets among them
    constexpr int NCH = CM / CH;
    constexpr int NWA = (SH + K + 3 + 3) / 4 * 4;  // staged values read per full row
    constexpr int PX = 4 / G > 0 ? 4 / G : 1;      // pixels a lane finishes
    constexpr int QPR = TW / 4;                    // pixel quads per tile row
    constexpr int SLOT = S::slot(A16);
    static_assert(CM % CH == 0 && PLANE % 256 == 0 && LS % 4 == 0, "whole chunks and loads");
    static_assert(SLOT >= L * NWAVE * 64 * VF, "a chunk's loads stay in its slot");
    extern __shared__ float4 smem4[];
    float* const smem = reinterpret_cast<float*>(smem4);
    float* const Qs = smem;                        // [kGroupSlots][SLOT]
    float* const Cs = Qs + kGroupSlots * SLOT;     // the colours, one chunk
    float* const Fs = Cs + SLOT;                   // [FD][PLANE]
    float* const Tb = Fs + FD * PLANE;             // the tap table
    constexpr int MR = (CM + 3) / 4 * 4;           // row of the compatibility
    float* const Ms = Tb + kGroupTab;              // [CM][MR] when given, zero past C
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
    const int nch = (C + CH - 1) / CH;             // chunks of this call

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane / (64 / G);                 // part of the window
    const int li = lane % (64 / G);                // quad of the wavefront
    const int cq = 4 * (li % QPR);                 // first tile column of the quad
    // groups of two: the half's 16-lane rows hold tile rows NWAVE apart
    const int ty = wave + NWAVE * (li / QPR);
    const int y = y0 + ty;
    // the pixels this lane finishes: xo .. xo + PX - 1
    const int xo = x0 + cq + (G == 1 ? 0 : G == 2 ? 2 * g : lane / 16);
    const bool row_ok = y < H;

    // ---- every load straight into LDS: the tap table (from the kernel's own
    // arguments) and the compatibility, then the colours and the features,
    // then the first chunks of Q_t.  A wave's loads complete in order, so it
    // can use the first ones while the last are in flight.
    {
        const char* const args = (const char*)__builtin_amdgcn_kernarg_segment_ptr();
        const rsrc_t rt = buffer_rsrc((const float*)(args + offsetof(GroupArgs, taps)),
                                      (unsigned)sizeof(TapTable));
        if (wave < kGroupTab / 64) lds_dma(rt, (wave * 64 + lane) * 4, 0, lds_addr(Tb + wave * 64));
        if (a.mu) {
            const rsrc_t rm = buffer_rsrc(a.mu, (unsigned)(C * C * 4));
            for (int j = wave; j < (CM * MR + 63) / 64; j += NWAVE) {
                const int i = j * 64 + lane, l = i / MR, m = i - (i / MR) * MR;
                lds_dma(rm, l < C && m < C ? (unsigned)((l * C + m) * 4) : kDmaOob, 0,
                        lds_addr(Ms + j * 64));
            }
        }
    }
    // load s of a chunk: piece j = wave + NWAVE s of its planes, piece j % NI
    // of plane j / NI (past the chunk's planes: zeros into the slot's padding)
    unsigned voff[NV];
#pragma unroll
    for (int s = 0; s < NV; ++s) {
        const int f = ((wave + NWAVE * s) % NI * 64 + lane) * VF;
        const int r = f / LS, col = f - (f / LS) * LS;
        const int gy = y0 - R + r, gx = x0 - XO + col;
        const bool in = f < LH * LS && gy >= 0 && gy < H && gx >= 0 && gx < W;
        voff[s] = in ? (unsigned)((gy * W + gx) * 4) : kDmaOob;
    }
    const unsigned lw = lds0 + (unsigned)(wave * 64 * VF * 4);
    // planes p0 .. p0 + n - 1 (n <= CH) of a tensor into the slot at float
    // offset `to`, zeros for the chunk's remaining planes
    auto stage = [&](rsrc_t r, int p0, int n, unsigned to) {
#pragma unroll
        for (int s = 0; s < L; ++s) {
            const int j = wave + NWAVE * s, pl = j / NI;
            const unsigned at = lw + (to + (unsigned)(s * NWAVE * 64 * VF)) * 4;
            const bool ok = pl < n;
            const unsigned vo = ok ? voff[s % NV] : kDmaOob;
            const int so = ok ? (p0 + pl) * hw4 : 0;
            if constexpr (A16) lds_dma16(r, vo, so, at);
            else lds_dma(r, vo, so, at);
        }
    };
    const rsrc_t rf = buffer_rsrc(a.image + (size_t)b * 3 * HW, (unsigned)(3 * HW * 4));
    const rsrc_t rq = buffer_rsrc(a.src + (size_t)b * C * HW, (unsigned)(C * HW * 4));
    stage(rf, 0, 3, (unsigned)(Cs - smem));
    if constexpr (FD > 0) {
        const rsrc_t rs = buffer_rsrc(a.sfeat + (size_t)b * a.D * HW, (unsigned)(a.D * HW * 4));
        for (int j = wave; j < FD * NI; j += NWAVE) {
            const int pl = j / NI;
            const int f = ((j - pl * NI) * 64 + lane) * VF;
            const int r = f / LS, col = f - (f / LS) * LS;
            const int gy = y0 - R + r, gx = x0 - XO + col;
            const bool in = pl < a.D && f < LH * LS && gy >= 0 && gy < H && gx >= 0 && gx < W;
            const unsigned vo = in ? (unsigned)((gy * W + gx) * 4) : kDmaOob;
            const unsigned at = lds_addr(Fs + j * 64 * VF);
            if constexpr (A16) lds_dma16(rs, vo, pl < a.D ? pl * hw4 : 0, at);
            else lds_dma(rs, vo, pl < a.D ? pl * hw4 : 0, at);
        }
    }
    // chunk k goes to slot k % kGroupSlots
    auto issue_chunk = [&](int k) {
        const int n = C - k * CH < CH ? C - k * CH : CH;
        stage(rq, k * CH, n, (unsigned)((k % kGroupSlots) * SLOT));
    };
#pragma unroll
    for (int k = 0; k < kGroupSlots; ++k)
        if (k < nch) issue_chunk(k);

    // ---- colours landed (all but the chunks' loads): the lane's weights
    if (nch >= 3) __builtin_amdgcn_s_waitcnt(vm_wait(3 * L));
    else if (nch == 2) __builtin_amdgcn_s_waitcnt(vm_wait(2 * L));
    else __builtin_amdgcn_s_waitcnt(vm_wait(L));
    __syncthreads();
    // byte-free offsets into a staged plane: step j's row of this lane (whole
    // pieces; the window starts SH into them), its taps of the centre row, and
    // the quad itself.  Opaque, so that classes and slots stay in the reads'
    // immediate offsets.
    unsigned base[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) base[j] = (unsigned)((ty + S::row(g, j)) * LS + cq);
    unsigned hbase = (unsigned)((ty + R) * LS + cq + (S::WHOLE ? 0 : SH) + (S::PART ? S::ct(g) : 0));
    const unsigned obase = (unsigned)((ty + R) * LS + cq + XO);
    // the weights, a row at a time, the colours of the next row on their way
    // while one is computed; finished (opaque values, which keep their order)
    // before the one after is read: all rows at once would not fit
    float w[4][S::NTAP];
    {
        constexpr int NPR = NWA / 4, NPH = S::PART ? ((S::WHOLE ? SH : 0) + NT + 6) / 4 : 1;
        float own[3][4];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(Cs + ch * PLANE + obase);
#pragma unroll
            for (int i = 0; i < 4; ++i) own[ch][i] = t[i];
        }
        // (log2 appearance, smoothness) of squared distance n
        auto tab = [&](int n) { return make_float2(Tb[n], Tb[kMaxN + 1 + n]); };
        // staged values of the plane at q: a whole row, or the centre row's taps
        auto read_half = [&](const float* q, f32x4 (&v)[NPH]) {
            if constexpr (S::WHOLE) {
                read_row(q, v);
            } else {
#pragma unroll
                for (int j = 0; j < NT + 3; ++j) v[j / 4][j % 4] = q[j];
            }
        };
        // weights of the N taps from w[.][t0] on: colours nc (the window O
        // into them), constants cs, smoothness weight ws (features, whose
        // squared distances w holds already); ctr: the row holds the centre
        auto weigh = [&](auto ntap, auto off, int t0, auto& nc, const auto& cs, float ws, bool ctr) {
            constexpr int N = decltype(ntap)::value, O = decltype(off)::value;
#pragma unroll
            for (int d = 0; d < N; ++d) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = O + i + d;
                    const float d0 = own[0][i] - nc[0][e / 4][e % 4];
                    const float d1 = own[1][i] - nc[1][e / 4][e % 4];
                    const float d2 = own[2][i] - nc[2][e / 4][e % 4];
                    const float col2 = fmaf(d2, d2, fmaf(d1, d1, d0 * d0));
                    const float smo =
                        FD > 0 ? ws * __builtin_amdgcn_exp2f(a.neg_gamma * w[i][t0 + d]) : cs[d].y;
                    const float v = __builtin_amdgcn_exp2f(fmaf(col2, a.neg_beta, cs[d].x)) + smo;
                    // the centre tap is left out here (added below when included)
                    w[i][t0 + d] = N == K && d == R && ctr ? 0.f : v;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int d = 0; d < N; ++d) asm volatile("" : "+v"(w[i][t0 + d]));
        };
        // the squared feature distances of N taps, one plane at a time
        auto distances = [&](auto ntap, auto off, int t0, unsigned at0) {
            constexpr int N = decltype(ntap)::value, O = decltype(off)::value;
            constexpr bool ROW = N == K;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int d = 0; d < N; ++d) w[i][t0 + d] = 0.f;
            f32x4 nf[2][ROW ? NPR : NPH], fo[2];
            auto read = [&](int ch) {              // plane ch into buffer ch % 2
                unsigned at = at0 + ch * PLANE, oat = obase + ch * PLANE;
                asm volatile("" : "+v"(at), "+v"(oat));
                if constexpr (ROW) read_row(Fs + at, nf[ch & 1]);
                else read_half(Fs + at, nf[ch & 1]);
                fo[ch & 1] = *reinterpret_cast<const f32x4*>(Fs + oat);
            };
            read(0);
#pragma unroll
            for (int ch = 0; ch < FD; ++ch) {
                if (ch + 1 < FD) read(ch + 1);
                auto& v = nf[ch & 1];
                if constexpr (ROW || S::WHOLE)
#pragma unroll
                    for (auto& x : v) use(x);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int d = 0; d < N; ++d) {
                        const float e = fo[ch & 1][i] - v[(O + i + d) / 4][(O + i + d) % 4];
                        w[i][t0 + d] = fmaf(e, e, w[i][t0 + d]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int d = 0; d < N; ++d) asm volatile("" : "+v"(w[i][t0 + d]));
            }
        };
        constexpr std::integral_constant<int, K> kRow{};
        constexpr std::integral_constant<int, NT> kHalf{};
        constexpr std::integral_constant<int, SH> kRowOff{};
        constexpr std::integral_constant<int, S::WHOLE ? SH : 0> kHalfOff{};
        f32x4 nc[2][3][NPR], hc[3][NPH];
        auto read_colours = [&](int j, f32x4 (&v)[3][NPR]) {
            asm volatile("" : "+v"(base[j]));
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) read_row(Cs + ch * PLANE + base[j], v[ch]);
        };
        read_colours(0, nc[0]);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            if (j + 1 < NF) {
                read_colours(j + 1, nc[(j + 1) & 1]);
            } else if (S::PART) {
                asm volatile("" : "+v"(hbase));
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) read_half(Cs + ch * PLANE + hbase, hc[ch]);
            }
            const int dy = S::row(g, j) - R;
            const bool keep = !S::spare(j) || g < G - 1;
            float2 cs[K];
#pragma unroll
            for (int d = 0; d < K; ++d) {
                cs[d] = tab(dy * dy + (d - R) * (d - R));
                if (S::spare(j)) {
                    cs[d].x = keep ? cs[d].x : -INFINITY;
                    cs[d].y = keep ? cs[d].y : 0.f;
                }
            }
            if constexpr (FD > 0) distances(kRow, kRowOff, j * K, base[j]);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
#pragma unroll
                for (int p = 0; p < NPR; ++p) use(nc[j & 1][ch][p]);
            weigh(kRow, kRowOff, j * K, nc[j & 1], cs, keep ? a.w_smooth : 0.f, !S::PART && dy == 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (S::PART) {
            float2 cs[NT];
            const int c0 = S::ct(g) - R;
#pragma unroll
            for (int d = 0; d < NT; ++d) cs[d] = tab((c0 + d) * (c0 + d));
            if constexpr (FD > 0) distances(kHalf, kHalfOff, NF * K, hbase);
            if constexpr (S::WHOLE)
#pragma unroll
                for (int ch = 0; ch < 3; ++ch)
#pragma unroll
                    for (int p = 0; p < NPH; ++p) use(hc[ch][p]);
            weigh(kHalf, kHalfOff, NF * K, hc, cs, a.w_smooth, false);
        }
    }
    // keep the weights' arithmetic above the chunk loop
    __builtin_amdgcn_sched_barrier(0);

    // ---- the message, chunk by chunk
    float fin[PX][CM], u[PX][CM];
#pragma unroll
    for (int i = 0; i < PX; ++i)
#pragma unroll
        for (int c = 0; c < CM; ++c) fin[i][c] = u[i][c] = 0.f;
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.unary + (size_t)b * C * HW), (short)0, (int)(C * HW * 4), 0x00020000);
    // buffer offset of the lane's pixels (whole dwords are all that a buffer
    // access of several dwords asks for; pixels past the row's end read what
    // follows it and are dropped)
    const int uoff = row_ok && xo < W ? (int)((unsigned)(y * W + xo) * 4u) : (int)kDmaOob;
    // the unary of the classes of chunks 0 .. k
    auto load_unary = [&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
    for (int c = 0; c < CM; ++c) {
        if (c / CH > k) continue;
        const int so = (int)((c < C ? c : C - 1) * HW * 4);
        if constexpr (PX == 4) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(ru, uoff, so, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) u[i][c] = __int_as_float((int)t[i]);
        } else if constexpr (PX == 2) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(ru, uoff, so, 0);
            u[0][c] = __int_as_float((int)t[0]);
            u[1][c] = __int_as_float((int)t[1]);
        } else {
            u[0][c] = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(ru, uoff, so, 0));
        }
    }
    };
    static_for([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if (k >= nch) return;
        // chunk k landed; issued after it: the other slots' chunks at the
        // start (k = 0), later only chunk k + 1
        const int after = k == 0 ? (nch >= 3 ? 2 : nch - 1) : (k + 1 < nch ? 1 : 0);
        if (after == 2) __builtin_amdgcn_s_waitcnt(vm_wait(2 * L));
        else if (after == 1) __builtin_amdgcn_s_waitcnt(vm_wait(L));
        else __builtin_amdgcn_s_waitcnt(vm_wait(0));
        __syncthreads();
        // every wave is past chunk k - 1: its slot takes chunk k + 2
        if (k >= 1 && k + 2 < nch) issue_chunk(k + 2);
        if (!S::LATE_U && k == nch - 1) load_unary(kc);   // once no chunk is left to load
        const float* const qk = Qs + (k % kGroupSlots) * SLOT;
        float acc[4][CH];
        // step t: row t % NS of class t / NS, read kDepth - 1 steps ahead of
        // the one applied (a rolling pipeline, one scheduling region a step)
        constexpr int kDepth = S::DEPTH, nsteps = CH * NS;
        f32x4 qr[kDepth][NWA / 4];
        auto rd = [&](int t, f32x4 (&v)[NWA / 4]) {
            if (S::WHOLE && t % NS == NF) {
#pragma unroll
                for (int j = 0; j < (SH + NT + 6) / 4; ++j)
                    v[j] = *reinterpret_cast<const f32x4*>(qk + (t / NS) * PLANE + hbase + 4 * j);
            } else if (S::PART && t % NS == NF) {
#pragma unroll
                for (int j = 0; j < NT + 3; ++j) v[j / 4][j % 4] = qk[(t / NS) * PLANE + hbase + j];
            } else {
                read_row(qk + (t / NS) * PLANE + base[t % NS], v);
            }
        };
#pragma unroll
        for (int t = 0; t < kDepth - 1; ++t)
            if (t < nsteps) rd(t, qr[t]);
#pragma unroll
        for (int t = 0; t < nsteps; ++t) {
            const int nx = t + kDepth - 1;
            if (nx < nsteps) rd(nx, qr[nx % kDepth]);
            const int c = t / NS, j = t % NS;
            const bool part = S::PART && j == NF;
            const int nt = part ? NT : K, o = part && !S::WHOLE ? 0 : SH;
            const int np = part ? (S::WHOLE ? (SH + NT + 6) / 4 : 0) : NWA / 4;
#pragma unroll
            for (int p = 0; p < np; ++p) use(qr[t % kDepth][p]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int d = 0; d < nt; ++d) {
                    const float q = qr[t % kDepth][(o + i + d) / 4][(o + i + d) % 4];
                    acc[i][c] = j + d == 0 ? w[i][0] * q : fmaf(w[i][j * K + d], q, acc[i][c]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        // the group's partial messages added, each lane keeping its pixels
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if constexpr (G == 1) {
#pragma unroll
                for (int i = 0; i < 4; ++i) fin[i][k * CH + c] = acc[i][c];
            } else {
                float v0 = add_halves(acc[0][c], acc[2][c]);
                float v1 = add_halves(acc[1][c], acc[3][c]);
                if constexpr (G == 2) {
                    fin[0][k * CH + c] = v0;
                    fin[PX - 1][k * CH + c] = v1;
                } else {
                    v0 = add_rows(v0, v1);
                    if constexpr (G == 8) v0 = add_eights(v0);
                    fin[0][k * CH + c] = v0;
                }
            }
        }
        if (a.include_center) {
            const float* const p = qk + (ty + R) * LS + (xo - x0) + XO;
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int i = 0; i < PX; ++i)
                    fin[i][k * CH + c] = fmaf(a.center_w, p[c * PLANE + i], fin[i][k * CH + c]);
        }
        // materialised here: sunk to the epilogue, the sums would keep their
        // operands live through the remaining chunks
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int i = 0; i < PX; ++i) asm volatile("" : "+v"(fin[i][k * CH + c]));
        if (S::LATE_U && k == nch - 1) load_unary(kc);    // its registers held weights
    }, std::make_integer_sequence<int, NCH>{});
    __builtin_amdgcn_s_waitcnt(vm_wait(0));        // the unary
    if (!row_ok || xo >= W || (G == 8 && (lane & 8))) return;

    // ---- compatibility, unary, softmax (Alg. 1), store Q_{t+1}; classes past
    // C take minus infinity and add nothing to the normalisation
    if (a.mu) {
        float z[PX][CM];
#pragma unroll
        for (int l = 0; l < CM; ++l) {
            if (l < C) {
                // four sums, shorter chains and smaller roundings than one
                float t[PX][4];
#pragma unroll
                for (int i = 0; i < PX; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[i][e] = 0.f;
#pragma unroll
                for (int m = 0; m < CM; m += 4) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(Ms + l * MR + m);
#pragma unroll
                    for (int i = 0; i < PX; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (m + e < CM) t[i][e] = fmaf(v[e], fin[i][m + e], t[i][e]);
                }
#pragma unroll
                for (int i = 0; i < PX; ++i)
                    z[i][l] = u[i][l] - ((t[i][0] + t[i][1]) + (t[i][2] + t[i][3]));
            } else {
#pragma unroll
                for (int i = 0; i < PX; ++i) z[i][l] = -INFINITY;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < PX; ++i)
#pragma unroll
            for (int c = 0; c < CM; ++c) fin[i][c] = z[i][c];
    } else {
        // Potts: softmax(U + M)
#pragma unroll
        for (int i = 0; i < PX; ++i)
#pragma unroll
            for (int c = 0; c < CM; ++c) fin[i][c] = c < C ? fin[i][c] + u[i][c] : -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < PX; ++i) softmax_regs<CM, true>(fin[i], CM);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.dst + (size_t)b * C * HW), (short)0, (int)(C * HW * 4), 0x00020000);
    if (xo + PX <= W) {
#pragma unroll
        for (int c = 0; c < CM; ++c) {
            if (c >= C) continue;
            const int so = (int)(c * HW * 4);
            if constexpr (PX == 4) {
                typedef unsigned u4 __attribute__((ext_vector_type(4)));
                const u4 t = {__float_as_uint(fin[0][c]), __float_as_uint(fin[1][c]),
                              __float_as_uint(fin[2][c]), __float_as_uint(fin[3][c])};
                __builtin_amdgcn_raw_buffer_store_b128(t, rd, uoff, so, 0);
            } else if constexpr (PX == 2) {
                typedef unsigned u2 __attribute__((ext_vector_type(2)));
                const u2 t = {__float_as_uint(fin[0][c]), __float_as_uint(fin[1][c])};
                __builtin_amdgcn_raw_buffer_store_b64(t, rd, uoff, so, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fin[0][c]), rd, uoff, so, 0);
            }
        }
    } else {
        // the row ends inside the lane's pixels
#pragma unroll
        for (int c = 0; c < CM; ++c) {
            if (c >= C) continue;
#pragma unroll
            for (int i = 0; i < PX - 1; ++i)
                if (xo + i < W)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fin[i][c]), rd,
                                                          uoff + 4 * i, (int)(c * HW * 4), 0);
        }
    }
}

template <int K, int CM, int FD, bool A16>
hipError_t launch_group_one(const GroupArgs& a, hipStream_t stream) {
    auto fn = group_kernel<K, CM, FD, A16>;
    static unsigned long long done = 0;            // devices opted into 160 KB of LDS
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(done & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        done |= bit;
    }
    hipLaunchKernelGGL(fn, dim3(a.ntiles), dim3(64 * GroupShape<K>::NWAVE),
                       group_lds_bytes<K>(CM, FD, A16, a.mu != nullptr), stream, a);
    return hipGetLastError();
}

template <int K, int CM, int FD>
hipError_t launch_group_a16(const GroupArgs& a, hipStream_t stream) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a.src) | reinterpret_cast<uintptr_t>(a.image) |
                        (FD > 0 ? reinterpret_cast<uintptr_t>(a.sfeat) : 0);
    return a.W % 4 == 0 && p % 16 == 0 ? launch_group_one<K, CM, FD, true>(a, stream)
                                       : launch_group_one<K, CM, FD, false>(a, stream);
}

template <int K, int CM>
hipError_t launch_group_fd(const GroupArgs& a, hipStream_t stream) {
    if (!a.sfeat) return launch_group_a16<K, CM, 0>(a, stream);
    return a.D <= 2 ? launch_group_a16<K, CM, 2>(a, stream) : launch_group_a16<K, CM, 4>(a, stream);
}

}  // namespace

#define CRF_CAT2(a, b) a##b
#define CRF_CAT(a, b) CRF_CAT2(a, b)
hipError_t CRF_CAT(launch_group_k, CRF_GROUP_K)(GroupArgs a, hipStream_t stream) {
    using S = GroupShape<CRF_GROUP_K>;
    if (a.C < 1 || a.C > kMaxC || (a.sfeat && (a.D < 1 || a.D > kMaxFeat)) ||
        (size_t)a.C * a.H * a.W * 4 >= (1ull << 31) || (size_t)3 * a.H * a.W * 4 >= (1ull << 31) ||
        (size_t)kMaxFeat * a.H * a.W * 4 >= (1ull << 31))
        return hipErrorNotSupported;
    a.tiles_x = (a.W + S::TW - 1) / S::TW;
    a.tiles_per_img = a.tiles_x * ((a.H + S::TH - 1) / S::TH);
    a.ntiles = a.tiles_per_img * a.B;
    if (a.C <= 12) return launch_group_fd<CRF_GROUP_K, 12>(a, stream);
    return a.C <= 21 ? launch_group_fd<CRF_GROUP_K, 21>(a, stream)
                     : launch_group_fd<CRF_GROUP_K, 24>(a, stream);
}

}  // namespace convcrf
