// The gradient kernel of the factored backward: one workgroup per head and per run of
// NBK = grad_blocks() 16-token blocks, all in parallel, from what the scans recorded (GradLayout):
// the state S entering the run, dL/dS leaving it (G), and every block's Delta and G_F.
//
// Relations, with KG = conj(K) G, QG = conj(Q) G, KI = K / G per token and channel (g the running
// decay from the block's start, g_C at its end), Y' = KI diag(g_C), G_R = conj(dL/do):
//   S_out = diag(g_C) S + Y'^T Delta,   dL/dS_in = diag(conj(g_C)) G + QG^H G_R - KG^H D_beta G_F
//   (the walk from the run's ends to each block's S and G);
//   G_A = tril(G_R Delta^*),   G_L' = -D_beta strict_tril(G_F Delta^*)
//   G_Qg = G_R S^* + G_A conj(KI),   G_Kg = -D_beta G_F S^* + G_L' conj(KI)
//   G_Ki = conj(Delta) G^T diag(conj(g_C)) + G_L'^T conj(KG) + G_A^T conj(QG)
//   G_gC = rowsum(G * conj(S)) + colsum(conj(Delta) G^T * conj(KI))
//   dbeta_t = Re[ conj(G_F) (conj(V) - KG S - L' Delta) ]_t, summed over the value columns
//           = Re[ sum_v conj(G_F) conj(V) - sum_i KG conj(G_F S^*) - sum_j L' conj(G_F Delta^*) ]_t,
//             which needs no product beyond those above but L' itself (KG KI^T)
// and elementwise per token and channel:
//   dq = g conj(G_Qg),   dk = g conj(G_Kg) + conj(1/g) G_Ki,
//   dL/dz = conj(g) (q G_Qg + k G_Kg) - conj(k / g) G_Ki  (+ conj(g_C) G_gC at the block's last token),
//   dalpha = suffix sum(Re dL/dz) / alpha,   dtheta = suffix sum(Im).
// G_A's diagonal takes part in dq and dk in fp32, elementwise; in dL/dz its terms cancel exactly
// and are left out.
//
// Layout: wave w holds channel block w, lane (c, g) channel c of it, everything over tokens or value
// columns 4g .. 4g + 3 -- the accumulator layout, in which S and G come from the records, every
// product over the value columns or over tokens takes its right operand from registers, and the
// elementwise stage finds G_Qg, G_Kg, G_Ki, q, k and g on one lane.  Only the rows (Delta, G_F, G_R:
// shared by the channel blocks) and the four 16 x 16 products pass through LDS.
//
// Bound by memory (bf16): B8 H16 T4096 reads 2.62 GB and writes 0.40 in 600-620 us, 5 TB/s where a
// device copy runs at 5.17; fp32 by the matrix instructions (332 of 32 cycles a block): B4 H8 T2048
// 175-185 us; B2 H6 T509 bf16 11 us.  The pass over the 16-token chunks' records (staging S and G
// themselves through LDS) takes 1190, 241 and 19 us.
#include <type_traits>

#include "sfda_factored.h"
#include "sfda_frag.h"

namespace sfda {
namespace fac {

struct GradArgs {
    const void *q, *k, *v, *alpha, *theta, *beta, *dO;
    const char *S, *G, *D, *F;
    void *dq, *dk, *dalpha, *dtheta, *dbeta;
    int T, m, n;
    GradLayout lay;
};

// The rows' tiles (16 tokens x 16 columns): as row fragments, and (bf16, NBK > 1) as column
// fragments for the walk.  Row fragments, bf16: lane order, 16 bytes more after every 16 lanes
// (the writers hold one column: 64 different words); fp32: rows of 144 bytes.
template <int P, int NBK> struct GradTiles {
    static constexpr int NT = 3 * NBK;
    static constexpr bool COL = P == PREC_BF16 && NBK > 1;
    static constexpr int ROWB = P == PREC_BF16 ? 1024 + 64 : 16 * 144;
    char row[NT][ROWB];
    char col[COL ? NT : 1][COL ? 1024 : 16];
};
template <int P, int NBK> struct GradSmem {
    union {
        GradTiles<P, NBK> tile[2];
        f32x4 mat[NBK][4][2][64];        // the 16 x 16 products [block][product][re, im][lane]
    };
    static constexpr int XP = P == PREC_BF16 ? 80 : 144;     // row bytes of 16 entries, padded
    char xp[4][2][16 * XP];              // per wave: KG, KI by rows
    float vsum[NBK][16], dsum[4][NBK][16];
};

// sums over 16 lanes (one row of the wave): lanes ^ 1, ^ 2, then the other quad and half, mirrored
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum(float x) {
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x141>(x);
    x += dpp<0x140>(x);
    return x;
}
// value of another lane; `at` is four times its index
__device__ __forceinline__ float lane_at(int at, float x) { return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(x))); }
__device__ __forceinline__ u32 lane_at(int at, u32 x) { return static_cast<u32>(__builtin_amdgcn_ds_bpermute(at, static_cast<int>(x))); }
template <typename T> __device__ __forceinline__ float ld_real_at(rsrc_t r, u32 off, int s) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, s, 0));
    else return __uint_as_float(static_cast<u32>(__builtin_amdgcn_raw_buffer_load_b16(r, off, s, 0)) << 16);
}
// four complex elements as loaded, converted where they are used
template <typename T> struct Raw4;
template <> struct Raw4<float> {
    float2 x[4];
    __device__ __forceinline__ void load(int r, rsrc_t rs, u32 off, int s) { x[r] = ldv2(rs, off, s); }
    __device__ __forceinline__ float2 get(int r) const { return x[r]; }
};
template <> struct Raw4<uint16_t> {
    u32 w[4];
    __device__ __forceinline__ void load(int r, rsrc_t rs, u32 off, int s) { w[r] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, s, 0); }
    __device__ __forceinline__ float2 get(int r) const { return make_float2(bf_lo(w[r]), bf_hi(w[r])); }
};
// a gradient's element in the inputs' type
template <typename T> __device__ __forceinline__ void st_cplx(rsrc_t r, u32 off, int s, float2 x) {
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(x.x), __float_as_uint(x.y)}, r, off, s, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(x.x, x.y), r, off, s, 0);
}

template <int P, typename TIN, typename TOUT, int NBK>
__global__ __launch_bounds__(256, 2) void grad_steps_kernel(GradArgs A)
{
    constexpr int ES = P == PREC_BF16 ? 4 : 8;
    constexpr int NT = 3 * NBK, TU = (NT + 3) / 4;
    __shared__ __align__(16) GradSmem<P, NBK> sm;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = A.T, m = A.m, n = A.n, ncb = A.lay.ncb;
    const long bh = blockIdx.x / static_cast<unsigned>(A.lay.recs);
    const int rec = static_cast<int>(blockIdx.x - bh * A.lay.recs);
    const int t0 = rec * NBK * 16;
    const bool live = w < A.lay.nkb;
    const int ch = w * 16 + c;                   // this lane's channel
    const int rows_in = max(min(T - t0, NBK * 16), 0);
#ifdef SFDA_LDS_POISON
    lds_poison(&sm, sizeof(sm), tid, 256);
    __syncthreads();
#endif

    // ---- per token and channel
    struct Raw { float a[4], th[4]; float2 q[4], k[4]; };
    // (a row's offset is scalar: rows past T and channels past m lie past the ranges)
    constexpr int EI = static_cast<int>(sizeof(TIN));
    const long e_m = (bh * T + t0) * static_cast<long>(m);
    const int by_m = live ? rows_in * m * EI : 0;
    const rsrc_t r_a = rsrc(static_cast<const TIN*>(A.alpha) + e_m, by_m), r_t = rsrc(static_cast<const TIN*>(A.theta) + e_m, by_m);
    const rsrc_t r_q = rsrc(static_cast<const TIN*>(A.q) + 2 * e_m, 2 * by_m), r_k = rsrc(static_cast<const TIN*>(A.k) + 2 * e_m, 2 * by_m);
    const rsrc_t r_b = rsrc(static_cast<const TIN*>(A.beta) + bh * T + t0, rows_in * EI);
    const u32 o_m = ch < m ? static_cast<u32>((4 * g * m + ch) * EI) : OOR, o_m2 = ch < m ? static_cast<u32>((4 * g * m + ch) * 2 * EI) : OOR;
    auto row_m = [&](int b, int r) { return (b * 16 + r) * m * EI; };
    auto load_raw = [&](int b, Raw& x) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = row_m(b, r);
            x.a[r] = ld_real_at<TIN>(r_a, o_m, s);
            x.th[r] = ld_real_at<TIN>(r_t, o_m, s);
            x.q[r] = ld_cplx<TIN>(r_q, o_m2, 2 * s);
            x.k[r] = ld_cplx<TIN>(r_k, o_m2, 2 * s);
        }
    };
    auto load_beta = [&](int b, float (&bt)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bt[r] = ld_real<TIN>(r_b, static_cast<u32>(b * 16 + 4 * g + r) * static_cast<u32>(sizeof(TIN)));
    };
    // running decay g from the block's start, 1 / g, g_C: products and phase sums (in 2^-32
    // revolutions: exact, wrapping by themselves) over the lane's tokens, then over the lanes;
    // NaN where the block's decay is below 2^-126 or an angle is not finite
    struct Decay { float2 g[4], gi[4], gc; };
    const int up1 = ((lane + 48) & 63) * 4, up2 = ((lane + 32) & 63) * 4, dn1 = ((lane + 16) & 63) * 4, last = (c + 48) * 4;
    auto decay_of = [&](int b, const Raw& x, Decay& d) __attribute__((always_inline)) {
        float p[4], al[4], pr = 1.f, finite = 0.f;
        u32 ph[4], ps = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = t0 + b * 16 + 4 * g + r < T && ch < m;
            al[r] = ok ? x.a[r] : 1.f;
            pr *= al[r];
            finite = __builtin_fmaf(x.th[r], 0.f, finite);
            ps += static_cast<u32>(__builtin_amdgcn_fractf(x.th[r] * 0.15915494309189535f) * 4294967296.f);
            p[r] = pr;
            ph[r] = ps;
        }
        float im = pr + finite;                          // (0, or NaN)
        u32 ip = ps;
        float fy = lane_at(up1, im);
        u32 uy = lane_at(up1, ip);
        im *= g >= 1 ? fy : 1.f;
        ip += g >= 1 ? uy : 0u;
        fy = lane_at(up2, im);
        uy = lane_at(up2, ip);
        im *= g >= 2 ? fy : 1.f;
        ip += g >= 2 ? uy : 0u;
        const float em0 = lane_at(up1, im);
        const u32 ep0 = lane_at(up1, ip);
        float em = g ? em0 : 1.f;
        const u32 ep = g ? ep0 : 0u;
        float D = lane_at(last, im);
        const u32 tot = lane_at(last, ip);
        if (!(D >= 1.17549435e-38f)) D = em = __builtin_nanf("");
        constexpr float REV = 1.f / 4294967296.f;
        float Pi = 1.f / (em * p[3]);
#pragma unroll
        for (int r = 3; r >= 0; --r) {
            const float f = static_cast<float>(ep + ph[r]) * REV, cs = __builtin_amdgcn_cosf(f), sn = __builtin_amdgcn_sinf(f);
            const float P0 = em * p[r];
            d.g[r] = make_float2(P0 * cs, P0 * sn);
            d.gi[r] = make_float2(Pi * cs, -Pi * sn);
            Pi *= al[r];                                 // 1 / g of the token before
        }
        const float f = static_cast<float>(tot) * REV;
        d.gc = make_float2(D * __builtin_amdgcn_cosf(f), D * __builtin_amdgcn_sinf(f));
    };
    auto mul = [](float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); };
    auto cmul = [](float2 a, float2 b) { return make_float2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x); };   // conj(a) b
    auto conj = [](float2 a) { return make_float2(a.x, -a.y); };

    // ---- the walk's operands of every block: Y' and conj(QG), -beta conj(KG); g_C
    Raw first;                                           // NBK == 1: kept for the elementwise stage
    [[maybe_unused]] Frag<P> wy[NBK], wq[NBK], wk[NBK];
    [[maybe_unused]] float2 wg[NBK];
    if constexpr (NBK == 1) {
        load_raw(0, first);
    } else if (live) {
#pragma unroll
        for (int b = 0; b < NBK; ++b) {
            Raw x;
            Decay d;
            float bt[4];
            load_raw(b, x);
            load_beta(b, bt);
            decay_of(b, x, d);
            float2 y[4], qg[4], kg[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y[r] = mul(mul(x.k[r], d.gi[r]), d.gc);
                qg[r] = conj(cmul(x.q[r], d.g[r]));
                kg[r] = cmul(x.k[r], d.g[r]);
                kg[r] = make_float2(-bt[r] * kg[r].x, bt[r] * kg[r].y);
            }
            wy[b] = frag4<P>(y);
            wq[b] = frag4<P>(qg);
            wk[b] = frag4<P>(kg);
            wg[b] = d.gc;
        }
    }

    // ---- the rows' tiles: tile kind * NBK + b, kind 0 Delta, 1 G_F (with V, for dbeta), 2 G_R
    // (bf16 rows stay the pairs they are: G_R's conjugate flips a sign bit)
    constexpr bool RAW_O = P == PREC_BF16 && sizeof(TOUT) == 2;
    struct Tile { float2 x[4]; Raw4<TIN> v; };      // (a pair that stays as loaded: in x[].x)
    auto tile_of = [&](int u, int& kind, int& b) __attribute__((always_inline)) {
        kind = (w + 4 * u) / NBK;
        b = (w + 4 * u) % NBK;
        return w + 4 * u < NT;
    };
    const long e_n = 2 * (bh * T + t0) * static_cast<long>(n);
    const rsrc_t r_o = rsrc(static_cast<const TOUT*>(A.dO) + e_n, rows_in * n * 2 * static_cast<int>(sizeof(TOUT)));
    const rsrc_t r_v = rsrc(static_cast<const TIN*>(A.v) + e_n, rows_in * n * 2 * static_cast<int>(sizeof(TIN)));
    const long row0 = (bh * A.lay.blocks + rec * NBK) * A.lay.rows;
    const rsrc_t r_d = rsrc(A.D + row0, NBK * A.lay.rows), r_f = rsrc(A.F + row0, NBK * A.lay.rows);
    auto load_tile = [&](int kind, int b, int cb, Tile& x) __attribute__((always_inline)) {
        const int j = cb * 16 + c;                       // (past n: past the last column block too)
        const u32 o_n = j < n ? static_cast<u32>((4 * g * n + j) * 2) : OOR;      // (times an element's bytes)
        if (kind < 2) {
            const rsrc_t rr = kind ? r_f : r_d;
            if constexpr (P == PREC_BF16) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const f32x4 y = ldv4(rr, lane * 16 + e * 1024, b * A.lay.rows + cb * 2048);
                    x.x[2 * e] = make_float2(y[0], y[1]);
                    x.x[2 * e + 1] = make_float2(y[2], y[3]);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    x.x[r] = ldv2(rr, j < n ? static_cast<u32>((4 * g + r) * ncb * 16 + j) * 8 : OOR, b * A.lay.rows);
            }
        } else if constexpr (RAW_O) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                x.x[r] = make_float2(__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_o, j < n ? o_n * 2u : OOR, (b * 16 + r) * n * 4, 0)), 0.f);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) x.x[r] = ld_cplx<TOUT>(r_o, j < n ? o_n * static_cast<u32>(sizeof(TOUT)) : OOR, (b * 16 + r) * n * 2 * static_cast<int>(sizeof(TOUT)));
        }
        if (kind == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) x.v.load(r, r_v, j < n ? o_n * EI : OOR, (b * 16 + r) * n * 2 * EI);
        }
    };
    float vd[TU][4];                                     // Re(conj(G_F) conj(V)), this lane's columns
#pragma unroll
    for (int u = 0; u < TU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) vd[u][r] = 0.f;
    auto put_tile = [&](int kind, int b, const Tile& x, GradTiles<P, NBK>& t, float (&acc)[4]) __attribute__((always_inline)) {
        Frag<P> f;
        if (kind == 2 && RAW_O) {
            if constexpr (RAW_O) {
#pragma unroll
                for (int r = 0; r < 4; ++r) f.w[r] = __float_as_uint(x.x[r].x) ^ 0x80000000u;
            }
        } else if (kind == 2) {
            float2 y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = conj(x.x[r]);
            f = frag4<P>(y);
        } else {
            f = frag4<P>(x.x);
        }
        if (kind == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 y = x.x[r];
                const float2 v = x.v.get(r);
                acc[r] = __builtin_fmaf(y.x, v.x, __builtin_fmaf(-y.y, v.y, acc[r]));
            }
        }
        const int i = kind * NBK + b;
        if constexpr (GradTiles<P, NBK>::COL) *reinterpret_cast<u32x4*>(t.col[i] + lane * 16) = f.w;
#pragma unroll
        for (int r = 0; r < 4; ++r) {                    // entry (token 4g + r, column c); Delta conjugated
            if constexpr (P == PREC_BF16)
                *reinterpret_cast<u32*>(t.row[i] + (4 * g + r) * 16 + (c >> 2) * 272 + (c & 3) * 4) = kind == 0 ? f.w[r] ^ 0x80000000u : f.w[r];
            else
                *reinterpret_cast<float2*>(t.row[i] + (4 * g + r) * 144 + c * 8) = kind == 0 ? conj(f.x[r]) : f.x[r];
        }
    };
    auto row_frag = [&](const char* t) __attribute__((always_inline)) {
        Frag<P> f;
        if constexpr (P == PREC_BF16) {
            f.w = *reinterpret_cast<const u32x4*>(t + lane * 16 + g * 16);
        } else {
            const float4 a = *reinterpret_cast<const float4*>(t + c * 144 + g * 32), b = *reinterpret_cast<const float4*>(t + c * 144 + g * 32 + 16);
            f.x[0] = make_float2(a.x, a.y); f.x[1] = make_float2(a.z, a.w);
            f.x[2] = make_float2(b.x, b.y); f.x[3] = make_float2(b.z, b.w);
        }
        return f;
    };
    auto col_frag = [&](const GradTiles<P, NBK>& t, int i) __attribute__((always_inline)) {
        Frag<P> f;
        if constexpr (GradTiles<P, NBK>::COL) {
            f.w = *reinterpret_cast<const u32x4*>(t.col[i] + lane * 16);
        } else {                                         // (Delta's row copy is conjugated)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 y = *reinterpret_cast<const float2*>(t.row[i] + (4 * g + r) * 144 + c * 8);
                if constexpr (P == PREC_F32) f.x[r] = i < NBK ? conj(y) : y;
            }
        }
        return f;
    };
    // S and G of one column block
    const long st0 = (bh * A.lay.recs + rec) * A.lay.state;
    const u32 st_off = !live ? OOR : static_cast<u32>(P == PREC_F32 ? ch * ncb * 128 + g * 32 : w * ncb * 2048 + lane * 32);
    // (fp32 scans run 8 columns a workgroup: past the last of them the record holds nothing)
    const int n_rec = P == PREC_F32 ? (n + 7) / 8 * 8 : ncb * 16;
    struct Pair { f32x4 a, b; };
    auto load_state = [&](const char* p, int cb, Pair& x) __attribute__((always_inline)) {
        const rsrc_t r = rsrc(p + st0, A.lay.state);
        const u32 o = cb * 16 + 4 * g < n_rec ? st_off : OOR;
        x.a = ldv4(r, o, cb * (P == PREC_F32 ? 128 : 2048));
        x.b = ldv4(r, o + 16, cb * (P == PREC_F32 ? 128 : 2048));
    };
    auto cacc = [](const Pair& x) {
        CAcc z;
        z.re = f32x4{x.a[0], x.a[2], x.b[0], x.b[2]};
        z.im = f32x4{x.a[1], x.a[3], x.b[1], x.b[3]};
        return z;
    };
    auto scale = [](CAcc& z, float2 s) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = z.re[r], y = z.im[r];
            z.re[r] = __builtin_fmaf(s.x, x, -s.y * y);
            z.im[r] = __builtin_fmaf(s.x, y, s.y * x);
        }
    };

    CAcc gqg[NBK], gkg[NBK], gki[NBK], mat[NBK];
    float2 phi[NBK];                                     // rowsum(G * conj(S))
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
        czero(gqg[b]); czero(gkg[b]); czero(gki[b]); czero(mat[b]);
        phi[b] = make_float2(0.f, 0.f);
    }
    Pair ns, ng;
    Tile nt[TU];
    auto load = [&](int cb) __attribute__((always_inline)) {
        load_state(A.S, cb, ns);
        load_state(A.G, cb, ng);
#pragma unroll
        for (int u = 0; u < TU; ++u) {
            int kind, b;
            if (tile_of(u, kind, b)) load_tile(kind, b, cb, nt[u]);
        }
    };
    auto put = [&](GradTiles<P, NBK>& t) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < TU; ++u) {
            int kind, b;
            if (tile_of(u, kind, b)) put_tile(kind, b, nt[u], t, vd[u]);
        }
    };
    load(0);
    put(sm.tile[0]);
    __syncthreads();
    for (int cb = 0; cb < ncb; ++cb) {
        GradTiles<P, NBK>& t = sm.tile[cb & 1];
        CAcc S = cacc(ns), G = cacc(ng);
        if (cb + 1 < ncb) load(cb + 1);
        CAcc Sb[NBK];
        if (live) {
#pragma unroll
            for (int b = 0; b < NBK; ++b) {
                Sb[b] = S;
                if (b + 1 < NBK) {
                    scale(S, wg[b]);
                    cmma<P>(S, col_frag(t, b), right<P>(wy[b]));
                }
            }
        }
#pragma unroll
        for (int b = NBK - 1; b >= 0; --b) {
            const Frag<P> rd = row_frag(t.row[b]), rf = row_frag(t.row[NBK + b]), rr = row_frag(t.row[2 * NBK + b]);
            // products 0, 1: G_R Delta^* and 2, 3: G_F Delta^*, by columns (even: rows j on the
            // accumulator) and by rows (odd)
            if (w == 0) cmma<P>(mat[b], rd, right<P>(rr));
            else if (w == 1) cmma<P>(mat[b], rr, right<P>(rd));
            else if (w == 2) cmma<P>(mat[b], rd, right<P>(rf));
            else cmma<P>(mat[b], rf, right<P>(rd));
            if (live) {
                const CAcc& s = Sb[b];
                CAcc cs;
                cs.re = s.re;
                cs.im = -s.im;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    phi[b].x = __builtin_fmaf(G.re[r], s.re[r], __builtin_fmaf(G.im[r], s.im[r], phi[b].x));
                    phi[b].y = __builtin_fmaf(G.im[r], s.re[r], __builtin_fmaf(-G.re[r], s.im[r], phi[b].y));
                }
                const Right<P> sr = right_acc<P>(cs);
                cmma<P>(gqg[b], rr, sr);
                cmma<P>(gkg[b], rf, sr);
                cmma<P>(gki[b], rd, right_acc<P>(G));
                if (b > 0) {
                    scale(G, conj(wg[b]));
                    cmma<P>(G, col_frag(t, 2 * NBK + b), right<P>(wq[b]));
                    cmma<P>(G, col_frag(t, NBK + b), right<P>(wk[b]));
                }
            }
        }
        if (cb + 1 < ncb) put(sm.tile[(cb + 1) & 1]);
        __syncthreads();
    }

    // ---- the 16 x 16 products, dbeta's part over V
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
        sm.mat[b][w][0][lane] = mat[b].re;
        sm.mat[b][w][1][lane] = mat[b].im;
    }
#pragma unroll
    for (int u = 0; u < TU; ++u) {
        int kind, b;
        if (tile_of(u, kind, b) && kind == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = row_sum(vd[u][r]);
                if (c == 0) sm.vsum[b][4 * g + r] = x;
            }
        }
    }
    __syncthreads();
    if (live) {
        const rsrc_t r_dq = rsrc(static_cast<const TIN*>(A.dq) + 2 * e_m, 2 * by_m), r_dk = rsrc(static_cast<const TIN*>(A.dk) + 2 * e_m, 2 * by_m);
        const rsrc_t r_da = rsrc(static_cast<const TIN*>(A.dalpha) + e_m, by_m), r_dt = rsrc(static_cast<const TIN*>(A.dtheta) + e_m, by_m);
#pragma unroll 1
        for (int b = 0; b < NBK; ++b) {
            Raw x;
            Decay d;
            float bt[4];
            if constexpr (NBK == 1) x = first;
            else load_raw(b, x);
            load_beta(b, bt);
            const float btc = ld_real<TIN>(r_b, static_cast<u32>(b * 16 + c) * static_cast<u32>(sizeof(TIN)));
            decay_of(b, x, d);
            // KG, KI, QG of this lane's tokens; L' = KG KI^T over this wave's channels
            float2 kg[4], ki[4], qg[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                kg[r] = cmul(x.k[r], d.g[r]);
                ki[r] = mul(x.k[r], d.gi[r]);
                qg[r] = cmul(x.q[r], d.g[r]);
            }
            char *xk = sm.xp[w][0], *xi = sm.xp[w][1];
            constexpr int XP = GradSmem<P, NBK>::XP;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = (4 * g + r) * XP + c * ES;
                if constexpr (P == PREC_BF16) {
                    *reinterpret_cast<u32*>(xk + o) = pack_bf16(kg[r].x, kg[r].y);
                    *reinterpret_cast<u32*>(xi + o) = pack_bf16(ki[r].x, ki[r].y);
                } else {
                    *reinterpret_cast<float2*>(xk + o) = kg[r];
                    *reinterpret_cast<float2*>(xi + o) = ki[r];
                }
            }
            wave_order();
            auto xp_frag = [&](const char* p) __attribute__((always_inline)) {
                Frag<P> f;
                const char* o = p + c * XP + 4 * g * ES;
                if constexpr (P == PREC_BF16) {
                    f.w = *reinterpret_cast<const u32x4*>(o);
                } else {
                    const float4 a = *reinterpret_cast<const float4*>(o), e = *reinterpret_cast<const float4*>(o + 16);
                    f.x[0] = make_float2(a.x, a.y); f.x[1] = make_float2(a.z, a.w);
                    f.x[2] = make_float2(e.x, e.y); f.x[3] = make_float2(e.z, e.w);
                }
                return f;
            };
            CAcc lp;
            czero(lp);
            cmma<P>(lp, xp_frag(xk), right<P>(xp_frag(xi)));         // L'[4g + r][c]
            wave_order();
            CAcc z[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                z[i].re = sm.mat[b][i][0][lane];
                z[i].im = sm.mat[b][i][1][lane];
            }
            // strict triangles: [t = c][j = 4g + r] below, [j = c][t = 4g + r] above the diagonal
            float2 ar[4], ac[4], lr[4], lc[4], dg[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool lo = 4 * g + r < c, hi = 4 * g + r > c;
                ar[r] = lo ? make_float2(z[0].re[r], z[0].im[r]) : make_float2(0.f, 0.f);
                ac[r] = hi ? make_float2(z[1].re[r], z[1].im[r]) : make_float2(0.f, 0.f);
                lr[r] = lo ? make_float2(-btc * z[2].re[r], -btc * z[2].im[r]) : make_float2(0.f, 0.f);
                lc[r] = hi ? make_float2(-bt[r] * z[3].re[r], -bt[r] * z[3].im[r]) : make_float2(0.f, 0.f);
                // G_A's diagonal, entry (4g + r, 4g + r): lane (4g + r, g), register r
                const f32x4* md = &sm.mat[b][1][0][0];
                dg[r] = make_float2(reinterpret_cast<const float*>(&md[4 * g + r + 16 * g])[r],
                                    reinterpret_cast<const float*>(&md[64 + 4 * g + r + 16 * g])[r]);
            }
            // dbeta's parts over the channels and over the earlier tokens
            CAcc &zq = gqg[0], &zk = gkg[0], &zi = gki[0];      // block b's (they move down, below)
            float db[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float e = kg[r].x * zk.re[r] + kg[r].y * zk.im[r];
                if (c < 4 * g + r) e += lp.re[r] * z[3].re[r] + lp.im[r] * z[3].im[r];
                db[r] = row_sum(e);
            }
            if (c == 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) sm.dsum[w][b][4 * g + r] = db[r];
            }
            // dL/dg_C: + colsum(G_Yp * conj(KI)); G_Yp diag(conj(g_C)); -D_beta G_F S^*
            float2 gg = phi[0];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 y = make_float2(zi.re[r], zi.im[r]), p = cmul(ki[r], y);
                gg.x += p.x;
                gg.y += p.y;
                const float2 s = cmul(d.gc, y);
                zi.re[r] = s.x;
                zi.im[r] = s.y;
                zk.re[r] *= -bt[r];
                zk.im[r] *= -bt[r];
            }
            gg.x += lane_at(dn1, gg.x);
            gg.y += lane_at(dn1, gg.y);
            gg.x += lane_at(up2, gg.x);
            gg.y += lane_at(up2, gg.y);
            float2 y[4];
            auto cright = [&](const float2 (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = conj(v[r]);
                return right<P>(frag4<P>(y));
            };
            {
                const Right<P> kr = cright(ki);
                cmma<P>(zq, frag4<P>(ar), kr);
                cmma<P>(zk, frag4<P>(lr), kr);
            }
            cmma<P>(zi, frag4<P>(lc), cright(kg));
            cmma<P>(zi, frag4<P>(ac), cright(qg));
            // elementwise, suffix sums
            float sl[4], sp[4], al = 0.f, ap = 0.f;
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const float2 gqv = make_float2(zq.re[r], zq.im[r]), gkv = make_float2(zk.re[r], zk.im[r]);
                const float2 gkiv = make_float2(zi.re[r], zi.im[r]);
                const float2 gqf0 = cmul(ki[r], dg[r]), gkf0 = mul(dg[r], conj(qg[r]));     // (q conj(g) is conj(QG))
                const float2 gqf = make_float2(gqv.x + gqf0.x, gqv.y + gqf0.y);
                const float2 gkf = make_float2(gkiv.x + gkf0.x, gkiv.y + gkf0.y);
                const float2 k1 = mul(d.g[r], conj(gkv)), k2 = cmul(d.gi[r], gkf);
                const int s = row_m(b, r);
                st_cplx<TIN>(r_dq, o_m2, 2 * s, mul(d.g[r], conj(gqf)));
                st_cplx<TIN>(r_dk, o_m2, 2 * s, make_float2(k1.x + k2.x, k1.y + k2.y));
                const float2 p1 = cmul(qg[r], gqv), p2 = cmul(kg[r], gkv), p3 = cmul(ki[r], gkiv);
                float2 dz = make_float2(p1.x + p2.x - p3.x, p1.y + p2.y - p3.y);
                if (r == 3) {                            // the block's last token
                    const float2 e = cmul(d.gc, gg);
                    dz.x += g == 3 ? e.x : 0.f;
                    dz.y += g == 3 ? e.y : 0.f;
                }
                al += dz.x;
                ap += dz.y;
                sl[r] = al;
                sp[r] = ap;
            }
            float xl = al, xs = ap;
            float yl = lane_at(dn1, xl), ys = lane_at(dn1, xs);
            xl += g < 3 ? yl : 0.f;
            xs += g < 3 ? ys : 0.f;
            yl = lane_at(up2, xl);
            ys = lane_at(up2, xs);
            xl += g < 2 ? yl : 0.f;
            xs += g < 2 ? ys : 0.f;
            yl = lane_at(dn1, xl);
            ys = lane_at(dn1, xs);
            const float ol = g < 3 ? yl : 0.f, op = g < 3 ? ys : 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int s = row_m(b, r);
                const float da = sl[r] + ol;
                st_real<TIN>(r_da, o_m, s, da / x.a[r]);
                st_real<TIN>(r_dt, o_m, s, sp[r] + op);
            }
#pragma unroll
            for (int i = 0; i + 1 < NBK; ++i) {              // (an index would put them in scratch)
                gqg[i] = gqg[i + 1];
                gkg[i] = gkg[i + 1];
                gki[i] = gki[i + 1];
                phi[i] = phi[i + 1];
            }
        }
    }
    __syncthreads();
    if (tid < NBK * 16 && t0 + tid < T) {
        float s = sm.vsum[tid >> 4][tid & 15];
        for (int i = 0; i < A.lay.nkb; ++i) s -= sm.dsum[i][tid >> 4][tid & 15];
        Elem<TIN>::store(static_cast<TIN*>(A.dbeta), bh * static_cast<long>(T) + t0 + tid, s);
    }
}

}  // namespace fac

template <int P, typename TIN, typename TOUT>
static hipError_t launch_grad_t(const GradLaunch& L, const GradRecords& rec, hipStream_t st)
{
    constexpr int NBK = fac::grad_blocks(P == PREC_BF16);
    const fac::GradArgs a{L.q, L.k, L.v, L.alpha, L.theta, L.beta, L.dO, rec.S, rec.G, rec.D, rec.F,
                          L.dq, L.dk, L.dalpha, L.dtheta, L.dbeta, L.T, L.m, L.n, fac::GradLayout(L.T, L.m, L.n, P == PREC_BF16)};
    const long heads = static_cast<long>(L.B) * L.H;
    hipLaunchKernelGGL((fac::grad_steps_kernel<P, TIN, TOUT, NBK>), dim3(static_cast<unsigned>(heads * a.lay.recs)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_grad_steps(const GradLaunch& L, const GradRecords& rec, hipStream_t st)
{
    if (bf16_operands(L.in_bf16, L.m))
        return L.out_bf16 ? launch_grad_t<PREC_BF16, uint16_t, uint16_t>(L, rec, st) : launch_grad_t<PREC_BF16, uint16_t, float>(L, rec, st);
    if (L.in_bf16)          // a few key channels: fp32 operands
        return L.out_bf16 ? launch_grad_t<PREC_F32, uint16_t, uint16_t>(L, rec, st) : launch_grad_t<PREC_F32, uint16_t, float>(L, rec, st);
    return L.out_bf16 ? launch_grad_t<PREC_F32, float, uint16_t>(L, rec, st) : launch_grad_t<PREC_F32, float, float>(L, rec, st);
}

}  // namespace sfda
