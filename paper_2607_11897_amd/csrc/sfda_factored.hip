// The factored chunk evaluation (sfda_factored.h has the relations and the operand records):
// the preparing kernel and the scans.
#include <algorithm>
#include <type_traits>

#include "sfda_factored.h"
#include "sfda_frag.h"

namespace sfda {
namespace fac {

// ------------------------------------------------------------------ preparing kernel
// One wave per 16-token block: everything after the phase totals stays inside the wave, so the
// workgroup meets one barrier.  LDS per wave is two 16 x 64 operand areas that the operands pass
// through one after another (held together they would leave one workgroup per compute unit):
// their rows are padded by 16 bytes, so a row fragment (16 rows x one 16-byte chunk) and a
// column fragment (4 rows x 16 consecutive entries) both read distinct banks.
struct PrepArgs {
    const void *q, *k, *alpha, *theta, *beta, *r, *wbeta;
    char* fac;
    int T, m, step0, nsteps;             // steps of this piece
    RecLayout lay;
    BwdLayout bwd;                       // the records' layout for the backward
};

template <int P> struct Op {             // operand areas of one wave
    static constexpr int ES = P == PREC_BF16 ? 4 : 8;
    static constexpr int PITCH = MP * ES + 16;
    static constexpr int AREA = 16 * PITCH;
};

template <int P> __device__ __forceinline__ Frag<P> lds_row(const char* a, int row, int kb, int g) {
    Frag<P> f;
    const char* p = a + row * Op<P>::PITCH + (kb * 16 + 4 * g) * Op<P>::ES;
    if constexpr (P == PREC_BF16) {
        f.w = *reinterpret_cast<const u32x4*>(p);
    } else {
        const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 16);
        f.x[0] = make_float2(lo.x, lo.y); f.x[1] = make_float2(lo.z, lo.w);
        f.x[2] = make_float2(hi.x, hi.y); f.x[3] = make_float2(hi.z, hi.w);
    }
    return f;
}
template <int P> __device__ __forceinline__ Frag<P> lds_col(const char* a, int col, int g) {
    Frag<P> f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const char* p = a + (4 * g + r) * Op<P>::PITCH + col * Op<P>::ES;
        if constexpr (P == PREC_BF16) f.w[r] = *reinterpret_cast<const u32*>(p);
        else f.x[r] = *reinterpret_cast<const float2*>(p);
    }
    return f;
}
// 4 consecutive entries, at lane word `at` (in entries) of a row-padded area or of a fragment
template <int P> __device__ __forceinline__ void put4(char* p, const float2 (&x)[4]) {
    if constexpr (P == PREC_BF16) {
        u32x4 w;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = pack_bf16(x[r].x, x[r].y);
        *reinterpret_cast<u32x4*>(p) = w;
    } else {
        *reinterpret_cast<float4*>(p) = make_float4(x[0].x, x[0].y, x[1].x, x[1].y);
        *reinterpret_cast<float4*>(p + 16) = make_float4(x[2].x, x[2].y, x[3].x, x[3].y);
    }
}
template <typename TIN, bool WIDE>
__device__ __forceinline__ void load4r(rsrc_t rs, u32 e, int left, float (&x)[4])
{
    if constexpr (WIDE && sizeof(TIN) == 2) {
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, left > 0 ? e * 2 : OOR, 0, 0);
        x[0] = bf_lo(w.x); x[1] = bf_hi(w.x); x[2] = bf_lo(w.y); x[3] = bf_hi(w.y);
    } else if constexpr (WIDE) {
        const u32x4 w = ld128(rs, left > 0 ? e * 4 : OOR);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = __uint_as_float(w[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = ld_real<TIN>(rs, k < left ? (e + k) * static_cast<u32>(sizeof(TIN)) : OOR);
    }
}
template <typename TIN, bool WIDE>
__device__ __forceinline__ void load4c(rsrc_t rs, u32 e, int left, float2 (&x)[4])
{
    if constexpr (WIDE && sizeof(TIN) == 2) {
        const u32x4 w = ld128(rs, left > 0 ? e * 4 : OOR);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = make_float2(bf_lo(w[k]), bf_hi(w[k]));
    } else if constexpr (WIDE) {
        const u32x4 a = ld128(rs, left > 0 ? e * 8 : OOR), b = ld128(rs, left > 0 ? e * 8 + 16 : OOR);
        x[0] = make_float2(__uint_as_float(a[0]), __uint_as_float(a[1]));
        x[1] = make_float2(__uint_as_float(a[2]), __uint_as_float(a[3]));
        x[2] = make_float2(__uint_as_float(b[0]), __uint_as_float(b[1]));
        x[3] = make_float2(__uint_as_float(b[2]), __uint_as_float(b[3]));
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = ld_cplx<TIN>(rs, k < left ? (e + k) * 2 * static_cast<u32>(sizeof(TIN)) : OOR);
    }
}

template <int S, typename X> __device__ __forceinline__ X quad_lane(X x) {   // DPP quad permutation
    return __builtin_bit_cast(X, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), S, 0xF, 0xF, false));
}

template <int P> struct PrepSmem {
    struct Wave { char r0[Op<P>::AREA], r1[Op<P>::AREA]; float beta[16], wb[16]; };
    Wave w[NB];
    u32 tph[NB][MP];                     // theta / 2 pi summed over each block, in 2^-32 revolutions
    static_assert(Op<P>::AREA >= 16 * 18 * 8, "the inverse's scratch fits an operand area");
};

template <int P, typename TIN, int KIND>
__device__ __forceinline__ void prep(PrepSmem<P>& sm, const PrepArgs& A, unsigned wg)
{
    constexpr int ES = Op<P>::ES, PITCH = Op<P>::PITCH;
    constexpr bool DEC = KIND == Kind::DEC, BWD = KIND == Kind::BWD;
    auto& sw = sm.w;
    auto& tph = sm.tph;

    const int tid = threadIdx.x, lane = tid & 63;
    const int pw = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const long bh = wg / static_cast<unsigned>(A.nsteps);
    const int st = static_cast<int>(wg - bh * A.nsteps);
    const int T = A.T, m = A.m;
    const int t0 = (A.step0 + st) * CP + pw * 16;      // the block's first token
    const int tsg = lane & 3, cg = lane >> 2;          // tokens 4 tsg .. + 3, channels 4 cg .. + 3
    const int pc0 = cg * 4;
    auto& w = sw[pw];
#ifdef SFDA_LDS_POISON
    lds_poison(&sm, sizeof(sm), tid, 256);
    __syncthreads();
#endif

    // ---- loads: every one in flight together; past T or past m they read as zero
    float av[4][4], th[4][4];
    float2 kq[4][4], qq[4][4], rq[4][4];
    {
        const int rows = min(max(T - t0, 0), 16);
        const long e0 = (bh * T + t0) * static_cast<long>(m);
        const int rb = rows * m * static_cast<int>(sizeof(TIN));
        const TIN *gq = static_cast<const TIN*>(A.q), *gk = static_cast<const TIN*>(A.k);
        const TIN *ga = static_cast<const TIN*>(A.alpha), *gt = static_cast<const TIN*>(A.theta);
        const rsrc_t ra = rsrc(ga + e0, rb), rt = rsrc(gt + e0, rb);
        const rsrc_t rqq = rsrc(gq + 2 * e0, 2 * rb), rk = rsrc(gk + 2 * e0, 2 * rb);
        const rsrc_t rr = DEC ? rsrc(static_cast<const TIN*>(A.r) + 2 * e0, 2 * rb) : rk;
        auto load = [&](auto wide_c) __attribute__((always_inline)) {
            constexpr bool W = decltype(wide_c)::value;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const u32 e = static_cast<u32>((tsg * 4 + u) * m + pc0);
                load4r<TIN, W>(ra, e, m - pc0, av[u]);
                load4r<TIN, W>(rt, e, m - pc0, th[u]);
                load4c<TIN, W>(rk, e, m - pc0, kq[u]);
                load4c<TIN, W>(rqq, e, m - pc0, qq[u]);
                if constexpr (DEC) load4c<TIN, W>(rr, e, m - pc0, rq[u]);
            }
        };
        if ((m & 3) == 0) load(std::true_type{});
        else load(std::false_type{});
        if (lane < 16) {
            const rsrc_t rbt = rsrc(static_cast<const TIN*>(A.beta) + bh * T + t0, rows * static_cast<int>(sizeof(TIN)));
            w.beta[lane] = ld_real<TIN>(rbt, lane * static_cast<u32>(sizeof(TIN)));
            if constexpr (DEC) {
                const rsrc_t rw = rsrc(static_cast<const TIN*>(A.wbeta) + bh * T + t0, rows * static_cast<int>(sizeof(TIN)));
                w.wb[lane] = ld_real<TIN>(rw, lane * static_cast<u32>(sizeof(TIN)));
            }
        }
    }

    // ---- scans of the block per channel: prefix products P, suffix products Q, phase sums.
    // Phases are kept in units of 2^-32 revolutions: the sums are exact and wrap by themselves
    // (summed as fp32 revolutions they put float32 results at 9.6e-7 instead of 6e-7 of the
    // 64-bit ones)
    float Pf[4][4], Qb[4][4], dtot[4], invd[4];              // [token u][channel k]
    u32 ph[4][4];
    {
        const bool s0 = tsg == 0, s01 = tsg < 2, s3 = tsg == 3, s23 = tsg >= 2;
        u32 tpk[4];
        bool low = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float a[4], finite = 0.f;                     // finite: NaN once a theta is not
            u32 lp[4], rp = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = t0 + tsg * 4 + u < T && pc0 + k < m;
                a[u] = ok ? av[u][k] : 1.f;               // the identity token's alpha
                finite = __builtin_fmaf(th[u][k], 0.f, finite);
                rp += static_cast<u32>(__builtin_amdgcn_fractf(th[u][k] * 0.15915494309189535f) * 4294967296.f);
                lp[u] = rp;
            }
            const float m0 = a[0], m1 = m0 * a[1], m2 = m1 * a[2], m3 = m2 * a[3];
            const float x2 = a[3], x1 = a[2] * a[3], x0 = a[1] * x1;
            float im = m3, is = m3;
            u32 ip = rp;
            float y = quad_lane<0x90>(im);                                 // [0, 0, 1, 2]
            u32 yp = quad_lane<0x90>(ip);
            im *= s0 ? 1.f : y;
            ip += s0 ? 0u : yp;
            y = quad_lane<0x40>(im); yp = quad_lane<0x40>(ip);             // [0, 0, 0, 1]
            im *= s01 ? 1.f : y;
            ip += s01 ? 0u : yp;
            float ys = quad_lane<0xF9>(is);                                // [1, 2, 3, 3]
            is *= s3 ? 1.f : ys;
            ys = quad_lane<0xFE>(is);                                      // [2, 3, 3, 3]
            is *= s23 ? 1.f : ys;
            const float pm = quad_lane<0x90>(im), ps = quad_lane<0xF9>(is), D = quad_lane<0xFF>(im);   // [3, 3, 3, 3]
            const u32 pp = quad_lane<0x90>(ip);
            const float em = s0 ? 1.f : pm, es = s3 ? 1.f : ps;
            const u32 ep = s0 ? 0u : pp;
            tpk[k] = quad_lane<0xFF>(ip);
            Pf[0][k] = em * m0; Pf[1][k] = em * m1; Pf[2][k] = em * m2; Pf[3][k] = em * m3;
            Qb[0][k] = es * x0; Qb[1][k] = es * x1; Qb[2][k] = es * x2; Qb[3][k] = es;
#pragma unroll
            for (int u = 0; u < 4; ++u) ph[u][k] = ep + lp[u];
            dtot[k] = D;
            low = low || !(D >= 1.17549435e-38f) || finite != finite;      // below the normal range (or NaN)
        }
        const bool bad = __builtin_amdgcn_ballot_w64(low) != 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (bad) dtot[k] = __builtin_nanf("");
            invd[k] = 1.f / dtot[k];
        }
        if (s0) *reinterpret_cast<u32x4*>(&tph[pw][pc0]) = u32x4{tpk[0], tpk[1], tpk[2], tpk[3]};
    }
    __syncthreads();
    char* const rec = A.fac + ((bh * A.nsteps + st) * static_cast<long>(NB) + pw) * (BWD ? A.bwd.block : A.lay.block);
    const int nkb = A.lay.nkb, frag = A.lay.frag;
    constexpr float REV = 1.f / 4294967296.f;
    u32 off[4] = {0, 0, 0, 0};
    float2 turn_end[4];                   // e^{i phi} at the end of the frame (step, or block: BWD)
    {
        u32 tot[4] = {0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const u32x4 t = *reinterpret_cast<const u32x4*>(&tph[b][pc0]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!BWD && b < pw) off[k] += t[k];
                if (!BWD || b == pw) tot[k] += t[k];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float p = static_cast<float>(tot[k]) * REV;
            turn_end[k] = make_float2(__builtin_amdgcn_cosf(p), __builtin_amdgcn_sinf(p));
        }
        if (BWD && tsg == 0) {
            float2 z[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) z[k] = make_float2(dtot[k] * turn_end[k].x, dtot[k] * turn_end[k].y);
            put4<PREC_F32>(rec + A.bwd.gc + pc0 * 8, z);
        } else if (tsg == 0) {
            const float2 (&z)[4] = turn_end;
            *reinterpret_cast<float4*>(rec + A.lay.dm + pc0 * 4) = make_float4(dtot[0], dtot[1], dtot[2], dtot[3]);
            put4<PREC_F32>(rec + A.lay.rot + pc0 * 8, z);
        }
    }
    // conj(q) e^{i phi}, conj(k) e^{i phi} (and conj(r) e^{i phi}); x e^{-i phi} is the conjugate
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float Ph = static_cast<float>(off[k] + ph[u][k]) * REV;
            const float sn = __builtin_amdgcn_sinf(Ph), cs = __builtin_amdgcn_cosf(Ph);
            auto turn = [&](float2 x) { return make_float2(__builtin_fmaf(x.x, cs, x.y * sn), __builtin_fmaf(x.x, sn, -x.y * cs)); };
            qq[u][k] = turn(qq[u][k]);
            kq[u][k] = turn(kq[u][k]);
            if constexpr (DEC) rq[u][k] = turn(rq[u][k]);
        }

    // ---- K Q (and R Q D_beta) to the record, through the wave's area so that the stores are
    // whole lines
    [[maybe_unused]] float2 kq_end[4][4];           // BWD: K Q turned to the block's end
    auto out_cols = [&](const float2 (&x)[4][4], int at, const float* wt) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float2 y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float s = Qb[u][k];
                if constexpr (DEC) if (wt) s *= wt[tsg * 4 + u];
                y[u] = make_float2(x[u][k].x * s, -x[u][k].y * s);
                if constexpr (BWD) {
                    const float2 e = turn_end[k];
                    y[u] = make_float2(y[u].x * e.x - y[u].y * e.y, y[u].x * e.y + y[u].y * e.x);
                    kq_end[u][k] = y[u];
                }
            }
            const int l2 = (cg & 3) * 4 + k + 16 * tsg;       // the fragment's lane
            put_frag<P>(w.r1 + (cg >> 2) * frag, l2, frag4<P>(y));
        }
        wave_order();
        for (int i = 0; i < nkb * frag; i += 1024)
            *reinterpret_cast<u32x4*>(rec + at + i + lane * 16) = *reinterpret_cast<const u32x4*>(w.r1 + i + lane * 16);
        wave_order();
    };
    out_cols(kq, BWD ? A.bwd.kq : A.lay.kq, nullptr);
    if constexpr (DEC) out_cols(rq, A.lay.rq, w.wb);

    // ---- row operands: conj(Q) G, conj(K) G (kept in area 0), K / G
    auto out_rows = [&](char* area, const float2 (&x)[4][4], auto scale, float sy) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float2 y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float s = scale(u, k);
                y[k] = make_float2(x[u][k].x * s, sy * x[u][k].y * s);
            }
            put4<P>(area + (tsg * 4 + u) * PITCH + pc0 * ES, y);
        }
        wave_order();
    };
    Frag<P> qf[4], kf[4];
    // BWD with bf16 operands: W, Z and A N are rounded once, as operands of the scans; what their
    // own operands' rounding leaves over takes part in forming them (formed from rounded operands
    // they put dS0 at 2.5e-3 of the 64-bit result, with the rest 1.9e-3)
    constexpr bool FINE = BWD && P == PREC_BF16;
    auto rest_rows = [&](const float2 (&x)[4][4]) __attribute__((always_inline)) {   // of x G, to area 1
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float2 y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) y[k] = rest(make_float2(x[u][k].x * Pf[u][k], x[u][k].y * Pf[u][k]));
            put4<P>(w.r1 + (tsg * 4 + u) * PITCH + pc0 * ES, y);
        }
        wave_order();
    };
    [[maybe_unused]] Frag<P> ql[FINE ? 4 : 1], kl[FINE ? 4 : 1];
    if constexpr (BWD) {                  // conj(K Q), rows tokens
        out_rows(w.r1, kq_end, [&](int, int) { return 1.f; }, -1.f);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            if (kb >= nkb) break;
            put_frag<P>(rec + A.bwd.kr + kb * frag, lane, lds_row<P>(w.r1, c, kb, g));
        }
        wave_order();
    }
    out_rows(w.r1, qq, [&](int u, int k) { return Pf[u][k]; }, 1.f);
    // BWD: by columns (conj(Q) G is then formed on as rows tokens, by channel on the lanes)
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) qf[kb] = lds_row<P>(w.r1, c, kb, g);
    [[maybe_unused]] Frag<P> qc[BWD ? 4 : 1];
    if constexpr (BWD) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) qc[kb] = lds_col<P>(w.r1, kb * 16 + c, g);
    }
    wave_order();
    if constexpr (FINE) {
        rest_rows(qq);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) ql[kb] = lds_col<P>(w.r1, kb * 16 + c, g);
        wave_order();
        rest_rows(kq);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) kl[kb] = lds_col<P>(w.r1, kb * 16 + c, g);
        wave_order();
    }
    out_rows(w.r0, kq, [&](int u, int k) { return Pf[u][k]; }, 1.f);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kf[kb] = lds_row<P>(w.r0, c, kb, g);
    out_rows(w.r1, kq, [&](int u, int k) { return Qb[u][k] * invd[k]; }, -1.f);

    // ---- Grams: L (rows t, columns j) and A^T (rows j, columns t), so that A comes out as the
    // right operand it is used as
    CAcc zl, za, zlr, zar;
    czero(zl); czero(za); czero(zlr); czero(zar);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        if (kb >= nkb) break;
        const Frag<P> d = lds_row<P>(w.r1, c, kb, g);
        cmma<P>(zl, kf[kb], right<P>(d));
        cmma<P>(za, d, right<P>(qf[kb]));
    }
    wave_order();
    if constexpr (DEC) {
        out_rows(w.r1, rq, [&](int u, int k) { return Qb[u][k] * invd[k]; }, -1.f);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            if (kb >= nkb) break;
            const Frag<P> d = lds_row<P>(w.r1, c, kb, g);
            cmma<P>(zlr, kf[kb], right<P>(d));
            cmma<P>(zar, d, right<P>(qf[kb]));
        }
        wave_order();
    }

    // ---- T = (I + D_beta L)^{-1} D_beta, row c on the lanes (c, .)
    float2* const xs = reinterpret_cast<float2*>(w.r1);     // [16][18]
    {
        const float4 bt = *reinterpret_cast<const float4*>(&w.beta[4 * g]);
        const float btr[4] = {bt.x, bt.y, bt.z, bt.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool lo = c < 4 * g + r;
            xs[(4 * g + r) * 18 + c] = make_float2(lo ? -btr[r] * zl.re[r] : 0.f, lo ? -btr[r] * zl.im[r] : 0.f);
        }
        wave_order();
        float2 xrow[16];
#pragma unroll
        for (int s2 = 0; s2 < 16; s2 += 2) {
            const float4 x2 = *reinterpret_cast<const float4*>(&xs[c * 18 + s2]);
            xrow[s2] = make_float2(x2.x, x2.y);
            xrow[s2 + 1] = make_float2(x2.z, x2.w);
        }
        float nr[4], ni[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) { nr[k] = c == 4 * k + g ? 1.f : 0.f; ni[k] = 0.f; }
        subst_steps(nr, ni, xrow, std::make_integer_sequence<int, 15>{});
        wave_order();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float b = BWD ? 1.f : w.beta[4 * k + g];      // T = N D_beta (BWD: N)
            xs[c * 18 + 4 * k + g] = make_float2(nr[k] * b, ni[k] * b);
        }
        wave_order();
    }
    Frag<P> tf, af;                    // T[c][4g + r]; A[c][4g + r]
    [[maybe_unused]] Frag<P> tl, al;
    {
        float2 x[4], y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[r] = xs[c * 18 + 4 * g + r];
            if constexpr (BWD) {
                const float b = w.beta[4 * g + r];
                x[r] = make_float2(x[r].x * b, x[r].y * b);
            }
            const bool keep = 4 * g + r <= c;
            y[r] = make_float2(keep ? za.re[r] : 0.f, keep ? za.im[r] : 0.f);
        }
        tf = frag4<P>(x);
        af = frag4<P>(y);
        if constexpr (FINE) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[r] = rest(x[r]);
                y[r] = rest(y[r]);
            }
            tl = frag4<P>(x);
            al = frag4<P>(y);
        }
    }
    const Right<P> tr = right<P>(tf), ar = right<P>(af);

    if constexpr (BWD) {
        auto conj_frag = [&](const CAcc& z, float s) __attribute__((always_inline)) {    // s conj(z)
            float2 x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = make_float2(s * z.re[r], -s * z.im[r]);
            return frag4<P>(x);
        };
        // x += (a + al) (b + bl), the rests' own product left out
        auto fine = [&](CAcc& x, const Frag<P>& a, const Frag<P>& ar_, const Right<P>& b, const Right<P>& br_) __attribute__((always_inline)) {
            cmma<P>(x, a, b);
            if constexpr (FINE) {
                cmma<P>(x, a, br_);
                cmma<P>(x, ar_, b);
            }
        };
        // T, N^* (bf16: without its diagonal of ones, which the scan adds in fp32), (A N)^*
        float2 x[4], xc[4], xl[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[r] = xs[(4 * g + r) * 18 + c];                                    // N[4g + r][c]
            xc[r] = FINE && c == 4 * g + r ? make_float2(0.f, 0.f) : make_float2(x[r].x, -x[r].y);
            xl[r] = rest(x[r]);
        }
        CAcc an;
        czero(an);
        fine(an, af, al, right<P>(frag4<P>(x)), right<P>(frag4<P>(xl)));
        put_frag<P>(rec + A.bwd.x, lane, tf);
        put_frag<P>(rec + A.bwd.ns, lane, frag4<P>(xc));
        put_frag<P>(rec + A.bwd.an, lane, conj_frag(an, 1.f));
        // -W, -W^*, Z^*
        const Right<P> tlr = right<P>(FINE ? tl : tf);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            if (kb >= nkb) break;
            const Frag<P> kt = lds_col<P>(w.r0, kb * 16 + c, g), ktl = kl[FINE ? kb : 0];
            CAcc a, b, z;
            czero(a); czero(b);
            fine(a, tf, tl, right<P>(kt), right<P>(ktl));                       // W (rows tokens)
            fine(b, kt, ktl, tr, tlr);                                          // W^T
            put_frag<P>(rec + kb * frag, lane, frag_acc<P>(b, -1.f));
            put_frag<P>(rec + A.bwd.ws + kb * frag, lane, conj_frag(a, -1.f));
            CAcc nw, nl;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float2 q = frag_get<P>(qc[kb], r);
                if constexpr (FINE) {
                    const float2 y = frag_get<P>(ql[kb], r), l = rest(make_float2(-a.re[r], -a.im[r]));
                    q = make_float2(q.x + y.x, q.y + y.y);
                    nl.re[r] = l.x;
                    nl.im[r] = l.y;
                }
                z.re[r] = q.x;
                z.im[r] = q.y;
                nw.re[r] = -a.re[r];
                nw.im[r] = -a.im[r];
            }
            if constexpr (!FINE) nl = nw;
            fine(z, af, al, right_acc<P>(nw), right_acc<P>(nl));                // Z = conj(Q) G - A W (rows tokens)
            put_frag<P>(rec + A.bwd.zs + kb * frag, lane, conj_frag(z, 1.f));
        }
        return;
    }

    // ---- X and Y
    {
        CAcc y;
        if constexpr (!DEC) {
            float2 x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = xs[(4 * g + r) * 18 + c];        // T^T, row c
            put_frag<P>(rec + A.lay.x, lane, tf);
            czero(y);
            cmma<P>(y, frag4<P>(x), ar);                                        // Y^T = T^T A^T
        } else {
            float2 x[4];
            const float bj = w.wb[c];
            const float4 b4 = *reinterpret_cast<const float4*>(&w.wb[4 * g]);
            const float br[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool lo = c < 4 * g + r, keep = 4 * g + r <= c;
                x[r] = make_float2(lo ? zlr.re[r] * bj : 0.f, lo ? zlr.im[r] * bj : 0.f);   // (L_r D_beta)[4g + r][c]
                y.re[r] = keep ? zar.re[r] * br[r] : 0.f;                       // (A_r D_beta)^T
                y.im[r] = keep ? zar.im[r] * br[r] : 0.f;
            }
            const Frag<P> lb = frag4<P>(x);
            CAcc xa, xt;
            czero(xa); czero(xt);
            cmma<P>(xa, tf, right<P>(lb));                                      // T L_r D_beta
            cmma<P>(xt, lb, tr);                                                // its transpose
            put_frag<P>(rec + A.lay.x, lane, frag_acc<P>(xt, -1.f));
            cmma<P>(y, frag_acc<P>(xa, -1.f), ar);                              // + X^T A^T
        }
        put_frag<P>(rec + A.lay.y, lane, frag_acc<P>(y));
    }

    // ---- -W and Z, channel block by channel block
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        if (kb >= nkb) break;
        const Frag<P> kt = lds_col<P>(w.r0, kb * 16 + c, g);                    // (conj(K) G)[4g + r][kb * 16 + c]
        CAcc a, b, z;
        czero(a); czero(b);
        cmma<P>(a, tf, right<P>(kt));                                           // W (rows tokens)
        cmma<P>(b, kt, tr);                                                     // W^T
        put_frag<P>(rec + kb * A.lay.frag, lane, frag_acc<P>(b, -1.f));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 x = frag_get<P>(qf[kb], r);
            z.re[r] = x.x;
            z.im[r] = x.y;
        }
        cmma<P>(z, frag_acc<P>(a, -1.f), ar);                                   // Z^T = (conj(Q) G)^T - W^T A^T
        put_frag<P>(rec + A.lay.z + kb * A.lay.frag, lane, frag_acc<P>(z));
    }
}

template <int P, typename TIN, int KIND>
__global__ __launch_bounds__(256, 2) void prep_kernel(PrepArgs A)
{
    __shared__ __align__(16) PrepSmem<P> sm;
    prep<P, TIN, KIND>(sm, A, blockIdx.x);
}

// ------------------------------------------------------------------ forward scans
struct ScanArgs {
    const char* fac;
    const void* v;
    void* o;
    const float* Sin;      // entering state (may be null: zero); Sout may be the same buffer
    float* Sout;           // may be null
    long heads;
    int T, m, n, n_slices;
    int step0, nsteps;
    RecLayout lay;
};

// Workgroup w of a scan: the slices of a head read the same records, so they go to one XCD (the
// dispatcher hands workgroups to the 8 XCDs round-robin by index): indices 8 S j + 8 s + x for
// head 8 j + x, the grid padded to whole groups of 8 heads.  Below 8 heads the plain order
// spreads the slices over the XCDs.
__device__ __forceinline__ bool scan_place(unsigned w, int S, long heads, long& bh, int& sl) {
    if (heads >= 8) {
        const unsigned x = w & 7u, q = w >> 3, j = q / static_cast<unsigned>(S);
        sl = static_cast<int>(q - j * static_cast<unsigned>(S));
        bh = 8L * j + x;
    } else {
        bh = w / static_cast<unsigned>(S);
        sl = static_cast<int>(w - bh * S);
    }
    return bh < heads;
}
static long scan_grid(long heads, int S) { return (heads >= 8 ? (heads + 7) / 8 * 8 : heads) * S; }

// What the scans share: the piece's tokens, and one step's resources.  A block's offset in them is
// scalar, and a step past the end is an empty range (loads read zero, stores drop).  Every step
// has four blocks: those past the end of the sequence hold identity tokens (no change of the
// state, no output), so the scans have no ragged tail.
struct Span {
    int tb, te, nsteps;
    long base_tn, base_mn;
    const char* fac;
    __device__ __forceinline__ Span(const ScanArgs& A, long bh) {
        tb = A.step0 * CP;
        te = static_cast<int>(min(static_cast<unsigned>(A.T), static_cast<unsigned>(tb) + static_cast<unsigned>(A.nsteps) * CP));
        nsteps = (te - tb + CP - 1) / CP;
        base_tn = (bh * A.T + tb) * static_cast<long>(A.n);
        base_mn = bh * static_cast<long>(A.m) * A.n;
        fac = A.fac + bh * A.nsteps * static_cast<long>(NB) * A.lay.block;
    }
    __device__ __forceinline__ int bytes(const ScanArgs& A, int st) const { return st < nsteps ? NB * A.lay.block : 0; }
    __device__ __forceinline__ int rows(int st) const { return max(min(te - tb - st * CP, CP), 0); }
    __device__ __forceinline__ const char* rec(const ScanArgs& A, int st) const { return fac + static_cast<long>(st) * (NB * A.lay.block); }
    __device__ __forceinline__ long elem(const ScanArgs& A, int st) const { return 2 * (base_tn + static_cast<long>(st) * CP * A.n); }
};
// fp32 operands.  Workgroup: 8 value columns on four waves; wave w holds channel block w of them
// (16 x 8 complex, interleaved columns: lane (c, g) part c & 1 of column c / 2), so a block's
// chain is 10 matrix instructions for its share of Delta, one exchange of the shares through LDS,
// and 8 for the update -- with the state on one wave it would be four times that, and with 16
// columns per workgroup half as many compute units would work.  The products of the output wait
// behind the exchange (they fill its 330 cycles); their shares are summed after the next block's
// barrier.  An fp32 matrix instruction takes 32 cycles and the SIMD issues no vector instruction
// beside it, so the chain is the sum of the two, about 1400 of the 2060 cycles a block takes;
// separate waves for the outputs changed nothing (113 us against 111 us for B4 H8 T2048).  Each
// wave reads only its own channel block of the records, four blocks ahead, straight into
// registers; waves past the channels read an empty range, so their state stays zero without a
// branch.
constexpr int FCOLS = 8;
struct ScanF32Smem { f32x4 red[2][2][4][64]; };        // [parity][Delta, O][wave][lane]
template <typename TV, typename TOUT, bool DEC>
__device__ __forceinline__ void scan_f32(ScanF32Smem& sm, const ScanArgs& A, unsigned wg)
{
    auto& red = sm.red;
    long bh;
    int sl;
    if (!scan_place(wg, A.n_slices, A.heads, bh, sl)) return;
    poison_area(red, 256);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, qp = lane & 1;
    const int n = A.n, m = A.m;
    const int j = sl * FCOLS + (c >> 1);
    const bool live = wave < A.lay.nkb;                // this wave's channels exist
    const Span sp(A, bh);
    const TV* const gv = static_cast<const TV*>(A.v);
    TOUT* const go = static_cast<TOUT*>(A.o);

    f32x4 S;
    {
        const rsrc_t rs = rsrc(A.Sin ? A.Sin + 2 * sp.base_mn : A.Sin, A.Sin && live ? m * n * 8 : 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = wave * 16 + 4 * g + r;
            S[r] = ld_f32(rs, j < n ? static_cast<u32>(((i * n + j) * 2 + qp) * 4) : OOR);
        }
    }

    struct Pre { f32x4 w0, w1, z0, z1, k0, k1, r0, r1, d; float2 x, y, v, u0, u1, u2, u3; };
    Pre pre[NB];
    const int so = wave * A.lay.frag;
    const u32 l16 = lane * 16;
    const u32 lx = (wave >> 1) * 1024 + lane * 16 + (wave & 1) * 8;           // K index 4g + wave of X, Y
    const int row_v = n * 2 * static_cast<int>(sizeof(TV)), row_o = n * 2 * static_cast<int>(sizeof(TOUT));
    auto voff = [&](int r) { return j < n ? static_cast<u32>((4 * g + r) * n + j) * 2 * static_cast<u32>(sizeof(TV)) : OOR; };
    const u32 lv = voff(wave);
    struct Step { rsrc_t own, all, v, o; };
    auto step_of = [&](int st) __attribute__((always_inline)) {
        const int bytes = sp.bytes(A, st), rows = sp.rows(st);
        const char* rec = sp.rec(A, st);
        const long e = sp.elem(A, st);
        return Step{rsrc(rec, live ? bytes : 0), rsrc(rec, bytes), rsrc(gv + e, rows * row_v), rsrc(go + e, go ? rows * row_o : 0)};
    };
    // a block's operands in three parts, each requested again as soon as its products have
    // issued: eleven loads in a row hold up the wave behind the load unit (120 us against 111)
    auto fetch_w = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block;
        p.w0 = ldv4(q.own, l16, at + so);
        p.w1 = ldv4(q.own, l16 + 1024, at + so);
        p.x = ldv2(q.all, lx, at + A.lay.x);
        LOAD_ORDER();
    };
    auto fetch_z = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block;
        p.z0 = ldv4(q.own, l16, at + so + A.lay.z);
        p.z1 = ldv4(q.own, l16 + 1024, at + so + A.lay.z);
        p.y = ldv2(q.all, lx, at + A.lay.y);
        LOAD_ORDER();
    };
    auto fetch_k = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block;
        p.k0 = ldv4(q.own, l16, at + so + A.lay.kq);
        p.k1 = ldv4(q.own, l16 + 1024, at + so + A.lay.kq);
        p.d = ldv4(q.own, g * 16, at + A.lay.dm + wave * 64);
        if constexpr (DEC) {
            p.r0 = ldv4(q.own, l16, at + so + A.lay.rq);
            p.r1 = ldv4(q.own, l16 + 1024, at + so + A.lay.rq);
            p.u0 = ld_cplx<TV>(q.v, voff(0), b * 16 * row_v);
            p.u1 = ld_cplx<TV>(q.v, voff(1), b * 16 * row_v);
            p.u2 = ld_cplx<TV>(q.v, voff(2), b * 16 * row_v);
            p.u3 = ld_cplx<TV>(q.v, voff(3), b * 16 * row_v);
        }
        p.v = ld_cplx<TV>(q.v, lv, b * 16 * row_v);
        LOAD_ORDER();
    };
    auto mma1 = [&](f32x4& acc, float a, float b) __attribute__((always_inline)) {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    };
    auto mma8 = [&](f32x4& acc, f32x4 a, f32x4 b, const Frag8& y) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 8; ++s) mma1(acc, s < 4 ? a[s & 3] : b[s & 3], y.v[s]);
    };
    const u32 eo = j < n ? static_cast<u32>(((4 * g + wave) * n + j) * 2 + qp) * static_cast<u32>(sizeof(TOUT)) : OOR;
    // o of block b of a step, whose shares lie in red[b & 1][1]: wave w sums and stores the rows
    // 4g + w
    auto store_o = [&](rsrc_t ro, int b) __attribute__((always_inline)) {
        float o = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) o += reinterpret_cast<const float*>(&red[b & 1][1][w2][lane])[wave];
        st_real<TOUT>(ro, eo, b * 16 * row_o, qp ? -o : o);
    };
    // block b of a step; prev, next: the resources that hold the block before it and the one four
    // further
    auto block = [&](int b, Pre& p, const Step& prev, const Step& next) __attribute__((always_inline)) {
        const Frag8 sb = bfrag_from_acc(S, qp);
        f32x4 pw = zero4(), pz = zero4();
        const float v0 = qp ? -p.v.y : p.v.x, v1 = qp ? p.v.x : p.v.y;       // conj(v) = (x, -y)
        mma1(pw, p.x.x, v0);
        mma1(pw, p.x.y, v1);
        mma8(pw, p.w0, p.w1, sb);
        fetch_w(next, b, p);
        red[b & 1][0][wave][lane] = pw;
        __syncthreads();
        poison_slot(red[(b & 1) ^ 1][0][wave][lane]);
        poison_slot(red[b & 1][1][wave][lane]);
        f32x4 d[4];
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) d[w2] = red[b & 1][0][w2][lane];
        mma1(pz, p.y.x, v0);
        mma1(pz, p.y.y, v1);
        mma8(pz, p.z0, p.z1, sb);
        fetch_z(next, b, p);
        store_o(prev.o, (b + NB - 1) % NB);
        S *= p.d;
        mma8(S, p.k0, p.k1, bfrag_from_acc((d[0] + d[1]) + (d[2] + d[3]), qp));
        if constexpr (DEC) {
            Frag8 vb;
            bpair(vb, 0, p.u0.x, -p.u0.y, qp);
            bpair(vb, 1, p.u1.x, -p.u1.y, qp);
            bpair(vb, 2, p.u2.x, -p.u2.y, qp);
            bpair(vb, 3, p.u3.x, -p.u3.y, qp);
            mma8(S, p.r0, p.r1, vb);
        }
        red[b & 1][1][wave][lane] = pz;
        fetch_k(next, b, p);
    };
    // back from the step's frame
    auto turn = [&](f32x4 r0, f32x4 r1) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float cs = r < 2 ? r0[2 * r] : r1[2 * r - 4], sn = r < 2 ? r0[2 * r + 1] : r1[2 * r - 3];
            const float own = S[r], oth = partner(own);
            S[r] = qp ? __builtin_fmaf(cs, own, sn * oth) : __builtin_fmaf(cs, own, -sn * oth);
        }
    };
    Step cur = step_of(0), prev = cur;
    prev.o = rsrc(go, 0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        fetch_w(cur, b, pre[b]);
        fetch_z(cur, b, pre[b]);
        fetch_k(cur, b, pre[b]);
    }
    for (int st = 0; st < sp.nsteps; ++st) {
        const Step next = step_of(st + 1);
        const f32x4 r0 = ldv4(cur.own, g * 32, A.lay.rot + wave * 128), r1 = ldv4(cur.own, g * 32 + 16, A.lay.rot + wave * 128);
#pragma unroll
        for (int b = 0; b < NB; ++b) block(b, pre[b], b ? cur : prev, next);
        turn(r0, r1);
        prev = cur;
        cur = next;
    }
    __syncthreads();
    store_o(prev.o, NB - 1);
    if (A.Sout != nullptr && live && j < n) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = wave * 16 + 4 * g + r;
            if (i < m) A.Sout[2 * (sp.base_mn + static_cast<long>(i) * n + j) + qp] = S[r];
        }
    }
}
template <typename TV, typename TOUT, bool DEC>
__global__ __launch_bounds__(256, 2) void scan_f32_kernel(ScanArgs A)
{
    __shared__ ScanF32Smem sm;
    scan_f32<TV, TOUT, DEC>(sm, A, blockIdx.x);
}

// The scan of one piece beside the preparation of the next, in one launch (the first nscan
// workgroups scan).  For a scan that leaves half of the compute units or more idle: a few heads
// over a long sequence.  The two roles' LDS together keeps one workgroup per compute unit, so that
// a scan shares its matrix cores with nobody.
template <typename TIN, typename TOUT>
__global__ __launch_bounds__(256, 1) void scan_prep_f32_kernel(ScanArgs S, PrepArgs N, unsigned nscan)
{
    __shared__ __align__(16) struct { ScanF32Smem scan; PrepSmem<PREC_F32> prep; } sm;
    if (blockIdx.x < nscan) scan_f32<TIN, TOUT, false>(sm.scan, S, blockIdx.x);
    else prep<PREC_F32, TIN, Kind::FWD>(sm.prep, N, blockIdx.x - nscan);
}

// bf16 operands.  Workgroup: 32 value columns.  The state's chain and the outputs on different
// waves, two on each SIMD: in one wave everything adds up -- matrix instructions (17 cycles),
// vector instructions (6.5 each), the 330 cycles of an exchange through LDS -- while another
// wave's vector instructions issue beside a bf16 matrix instruction (dec. forward B8 H16 T4096: scan
// 244 us, 256-266 us with the outputs on the state's waves).  The state waves put the operand
// words of the entering state, which they form anyway, into LDS before the block's one barrier;
// an output wave takes every second block whole.  State wave (cw, h) holds 16 of them (cw) with
// channel blocks 2h, 2h + 1: half the channels per wave halves a wave's instructions, at the price
// of one exchange of the halves of Delta.  Output wave (cw, p) takes the blocks of parity p.
// What a wave has no use for (channels past m; X on the second half, whose share of Delta has
// none) it reads from an empty range, without a branch.
constexpr int BCOLS = 32;
template <typename TOUT, bool DEC>
__global__ __launch_bounds__(512, 1) void scan_bf16_kernel(ScanArgs A)
{
    constexpr int P = PREC_BF16;
    __shared__ f32x4 red[2][4][2][64];                 // [parity][state wave][re, im][lane]: shares of Delta
    __shared__ u32x4 ent[2][2][4][2][64];              // [parity][cw][channel block][re, im words][lane]: entering state
    long bh;
    int sl;
    if (!scan_place(blockIdx.x, A.n_slices, A.heads, bh, sl)) return;
    poison_area(red, 512);
    poison_area(ent, 512);
    const int lane = threadIdx.x & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave8 & 3;
    const int c = lane & 15, g = lane >> 4, h = wave & 1, cw = wave >> 1;
    const int n = A.n, m = A.m;
    const int j = sl * BCOLS + cw * 16 + c;
    const Span sp(A, bh);
    const uint16_t* const gv = static_cast<const uint16_t*>(A.v);
    TOUT* const go = static_cast<TOUT*>(A.o);
    const u32 l16 = lane * 16;
    const int row_v = n * 4, row_o = n * 2 * static_cast<int>(sizeof(TOUT));
    u32 voff[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) voff[r] = j < n ? static_cast<u32>((4 * g + r) * n + j) * 4u : OOR;
    auto ldf = [&](rsrc_t r, u32 off, int s) __attribute__((always_inline)) {
        Frag<P> f;
        f.w = __builtin_amdgcn_raw_buffer_load_b128(r, off, s, 0);
        return f;
    };
    auto conj_v = [&](const u32 (&v)[4]) __attribute__((always_inline)) {
        Frag<P> f;
#pragma unroll
        for (int r = 0; r < 4; ++r) f.w[r] = v[r] ^ 0x80000000u;
        return right<P>(f);
    };

    if (wave8 < 4) {
        // ================================================ state waves
        const bool live0 = 2 * h < A.lay.nkb, live1 = 2 * h + 1 < A.lay.nkb;
        CAcc S[2];
        {
            const rsrc_t rs = rsrc(A.Sin ? A.Sin + 2 * sp.base_mn : A.Sin, A.Sin ? m * n * 8 : 0);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = (2 * h + kb) * 16 + 4 * g + r;
                    const float2 x = ld_c64(rs, j < n && i < m ? static_cast<u32>(i * n + j) * 8u : OOR);
                    S[kb].re[r] = x.x;
                    S[kb].im[r] = x.y;
                }
        }
        struct Pre { Frag<P> w[2], k[2], r[2], x; f32x4 d[2]; u32 v[4]; };
        Pre pre[NB];
        const int so = 2 * h * 1024;
        struct Step { rsrc_t own[2], x, v; };
        auto step_of = [&](int st) __attribute__((always_inline)) {
            const int bytes = sp.bytes(A, st);
            const char* rec = sp.rec(A, st);
            return Step{{rsrc(rec, live0 ? bytes : 0), rsrc(rec, live1 ? bytes : 0)}, rsrc(rec, h ? 0 : bytes),
                        rsrc(gv + sp.elem(A, st), sp.rows(st) * row_v)};
        };
        auto fetch_w = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
            const int at = b * A.lay.block;
            p.x = ldf(q.x, l16, at + A.lay.x);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) p.w[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so);
            LOAD_ORDER();
        };
        auto fetch_k = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
            const int at = b * A.lay.block;
#pragma unroll
            for (int r = 0; r < 4; ++r) p.v[r] = __builtin_amdgcn_raw_buffer_load_b32(q.v, voff[r], b * 16 * row_v, 0);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                p.d[kb] = ldv4(q.own[kb], g * 16 + kb * 64, at + A.lay.dm + h * 128);
                if constexpr (DEC) p.r[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so + A.lay.rq);
                p.k[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so + A.lay.kq);
            }
            LOAD_ORDER();
        };
        // block b of a step; next: the resources that hold the block four further
        auto block = [&](int b, Pre& p, const Step& next) __attribute__((always_inline)) {
            const Right<P> vb = conj_v(p.v);
            CAcc d;
            czero(d);
            cmma<P>(d, p.x, vb);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const Right<P> sb = right_acc<P>(S[kb]);
                ent[b & 1][cw][2 * h + kb][0][lane] = sb.re;
                ent[b & 1][cw][2 * h + kb][1][lane] = sb.im;
                cmma<P>(d, p.w[kb], sb);
            }
            red[b & 1][wave][0][lane] = d.re;
            red[b & 1][wave][1][lane] = d.im;
            fetch_w(next, b, p);
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                poison_slot(red[(b & 1) ^ 1][wave][e][lane]);
                poison_slot(ent[(b & 1) ^ 1][cw][2 * h][e][lane]);
                poison_slot(ent[(b & 1) ^ 1][cw][2 * h + 1][e][lane]);
            }
            const f32x4 ore = red[b & 1][wave ^ 1][0][lane], oim = red[b & 1][wave ^ 1][1][lane];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                S[kb].re *= p.d[kb];
                S[kb].im *= p.d[kb];
                if constexpr (DEC) cmma<P>(S[kb], p.r[kb], vb);
            }
            d.re += ore;
            d.im += oim;
            const Right<P> db = right_acc<P>(d);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) cmma<P>(S[kb], p.k[kb], db);
            fetch_k(next, b, p);
        };
        // back from the step's frame
        struct Rot { f32x4 x[2][2]; };
        auto load_rot = [&](const Step& q) __attribute__((always_inline)) {
            Rot z;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int u = 0; u < 2; ++u) z.x[kb][u] = ldv4(q.own[kb], g * 32 + kb * 128 + u * 16, A.lay.rot + h * 256);
            return z;
        };
        auto turn = [&](const Rot& z) __attribute__((always_inline)) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float cs = z.x[kb][r >> 1][2 * (r & 1)], sn = z.x[kb][r >> 1][2 * (r & 1) + 1];
                    const float x = S[kb].re[r], y = S[kb].im[r];
                    S[kb].re[r] = __builtin_fmaf(cs, x, -sn * y);
                    S[kb].im[r] = __builtin_fmaf(cs, y, sn * x);
                }
        };
        Step cur = step_of(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            fetch_w(cur, b, pre[b]);
            fetch_k(cur, b, pre[b]);
        }
        for (int st = 0; st < sp.nsteps; ++st) {
            const Step next = step_of(st + 1);
            const Rot z = load_rot(cur);
#pragma unroll
            for (int b = 0; b < NB; ++b) block(b, pre[b], next);
            turn(z);
            cur = next;
        }
        if (A.Sout != nullptr) {
            const rsrc_t rs = rsrc(A.Sout + 2 * sp.base_mn, m * n * 8);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = (2 * h + kb) * 16 + 4 * g + r;
                    const u32x2 x = {__float_as_uint(S[kb].re[r]), __float_as_uint(S[kb].im[r])};
                    __builtin_amdgcn_raw_buffer_store_b64(x, rs, j < n && i < m ? static_cast<u32>(i * n + j) * 8u : OOR, 0, 0);
                }
        }
    } else {
        // ================================================ output waves: blocks 2 i + h
        const int nkb = A.lay.nkb;
        u32 ooff[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) ooff[r] = j < n ? static_cast<u32>((4 * g + r) * n + j) * 2u * static_cast<u32>(sizeof(TOUT)) : OOR;
        struct Pre { Frag<P> z[4], y; u32 v[4]; };
        Pre pre[2];                                    // blocks h and 2 + h of a step
        auto fetch = [&](int st, int b, Pre& p) __attribute__((always_inline)) {
            const rsrc_t q = rsrc(sp.rec(A, st), sp.bytes(A, st));
            const rsrc_t qv = rsrc(gv + sp.elem(A, st), sp.rows(st) * row_v);
            const int at = b * A.lay.block;
            p.y = ldf(q, l16, at + A.lay.y);
#pragma unroll
            for (int r = 0; r < 4; ++r) p.v[r] = __builtin_amdgcn_raw_buffer_load_b32(qv, voff[r], b * 16 * row_v, 0);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) p.z[kb] = ldf(q, l16, at + A.lay.z + kb * 1024);   // (past nkb not used)
            LOAD_ORDER();
        };
        fetch(0, h, pre[0]);
        fetch(0, 2 + h, pre[1]);
        for (int st = 0; st < sp.nsteps; ++st) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                __syncthreads();
                if ((b & 1) != h) continue;
                Pre& p = pre[b >> 1];
                CAcc o;
                czero(o);
                cmma<P>(o, p.y, conj_v(p.v));
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    if (kb >= nkb) break;
                    cmma<P>(o, p.z[kb], Right<P>{ent[b & 1][cw][kb][0][lane], ent[b & 1][cw][kb][1][lane]});
                }
                const rsrc_t ro = rsrc(go + sp.elem(A, st), go ? sp.rows(st) * row_o : 0);
                fetch(st + 1, b, p);
#pragma unroll
                for (int r = 0; r < 4; ++r) {                // o = conj(O^*)
                    if constexpr (sizeof(TOUT) == 2)
                        __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(o.re[r], -o.im[r]), ro, ooff[r], b * 16 * row_o, 0);
                    else
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(o.re[r]), __float_as_uint(-o.im[r])}, ro, ooff[r],
                                                              b * 16 * row_o, 0);
                }
            }
        }
    }
}

// ------------------------------------------------------------------ backward scans
// The forward scan recording the state entering every run of blocks and Delta, and the adjoint scan
// (blocks in reverse) recording dL/dS leaving every run and G_F and writing dv and dS0; both in
// one launch (they read the same records and are independent).  fp32 is bound by the SIMDs' issue
// (both scans' workgroups share them: 330 us for B4 H8 T2048, 128 blocks at 2.6 us), bf16 at many
// heads by what it writes and reads (B8 H16 T4096: 1.07 GB of states, 0.54 GB of rows and 0.14 GB of
// dv written, 1.08 GB read, 780 us: 3.6 TB/s, two rounds of workgroups in a chain of blocks; with rows
// of 16 bits 740 us, then with the states of every block 1150 us, of every fourth 615 us, but see
// grad_blocks).  The scans in place take 1112 and 1290 us.
struct BwdArgs {
    const char* fac;
    const void *v, *dO, *beta;
    const float *S0, *dS_T;              // may be null (zero)
    float* dS0;                          // may be null
    char *S_rec, *G_rec, *D_rows, *F_rows;
    void* dv;
    long heads;
    int T, m, n, n_slices, nsteps;
    BwdLayout lay;
    GradLayout grad;
};

// One scan's walk over its steps: resources of a step's inputs (operands four blocks ahead; steps
// outside the sequence are empty ranges), of the outputs' blocks.  Blocks past the end of the
// sequence, in the last step, are identities and write their records like any other.
struct Walk {
    int nsteps;
    long tok, mn8, head;
    const char* fac;
    __device__ __forceinline__ Walk(const BwdArgs& A, long bh) {
        nsteps = A.nsteps;
        head = bh;
        tok = bh * A.T;
        mn8 = static_cast<long>(A.m) * A.n * 8;
        fac = A.fac + bh * A.nsteps * static_cast<long>(NB) * A.lay.block;
    }
    __device__ __forceinline__ bool in(int st) const { return st >= 0 && st < nsteps; }
    __device__ __forceinline__ rsrc_t rec(const BwdArgs& A, int st, bool on) const {
        return rsrc(fac + static_cast<long>(st) * (NB * A.lay.block), on && in(st) ? NB * A.lay.block : 0);
    }
    // rows of a [T][n] complex array of `es`-byte parts, from step st on
    __device__ __forceinline__ rsrc_t rows(const BwdArgs& A, const void* p, int es, int st) const {
        const int left = in(st) ? min(A.T - st * CP, CP) : 0;
        return rsrc(static_cast<const char*>(p) + (tok + static_cast<long>(st) * CP) * A.n * 2 * es, left * A.n * 2 * es);
    }
    __device__ __forceinline__ rsrc_t state(const BwdArgs& A, const char* p, int rec) const {
        return rsrc(p + (head * A.grad.recs + rec) * A.grad.state, A.grad.state);
    }
    __device__ __forceinline__ rsrc_t block_rows(const BwdArgs& A, const char* p, int ch, bool on = true) const {
        return rsrc(p + (head * A.grad.blocks + ch) * A.grad.rows, on ? A.grad.rows : 0);
    }
};

// fp32 operands: the forward scan's layout of work (8 value columns, one channel block per wave).
struct BwdF32Smem { f32x4 red[2][2][4][64]; };
template <typename TV, typename TO>
__device__ __forceinline__ void bwd_f32(BwdF32Smem& sm, const BwdArgs& A, unsigned wg, bool adj)
{
    auto& red = sm.red;
    long bh;
    int sl;
    if (!scan_place(wg, A.n_slices, A.heads, bh, sl)) return;
    poison_area(red, 256);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, qp = lane & 1;
    const int n = A.n, m = A.m;
    const int j = sl * FCOLS + (c >> 1);
    const bool live = wave < A.lay.nkb;
    const Walk wk(A, bh);
    const u32 l16 = lane * 16;
    const int so = wave * A.lay.frag;
    const u32 lx = (wave >> 1) * 1024 + lane * 16 + (wave & 1) * 8;           // K index 4g + wave
    auto mma1 = [&](f32x4& acc, float a, float b) __attribute__((always_inline)) {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    };
    auto mma8 = [&](f32x4& acc, f32x4 a, f32x4 b, const Frag8& y) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 8; ++s) mma1(acc, s < 4 ? a[s & 3] : b[s & 3], y.v[s]);
    };
    // this wave's part of a state [m][n]: rows wave * 16 + 4g + r (past m they lie past the
    // range), column j, part qp
    u32 soff[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        soff[r] = j < n && live ? static_cast<u32>((((wave * 16 + 4 * g + r) * n + j) * 2 + qp) * 4) : OOR;
    f32x4 S;
    {
        const float* init = adj ? A.dS_T : A.S0;
        const rsrc_t rs = rsrc(init ? reinterpret_cast<const char*>(init) + bh * wk.mn8 : nullptr, init ? static_cast<int>(wk.mn8) : 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) S[r] = ld_f32(rs, soff[r]);
    }
    constexpr int GB = grad_blocks(false);
    const bool in_rec = live && (j >> 4) < A.grad.ncb;
    const int row_rec = A.grad.ncb * 128;
    const u32 so_rec = in_rec ? static_cast<u32>((wave * 16 + 4 * g) * row_rec + j * 8 + qp * 4) : OOR;
    auto put_state = [&](rsrc_t rs) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(S[r]), rs, so_rec, r * row_rec, 0);
    };
    // row 4g + wave of a block's rows
    const u32 roff = (j >> 4) < A.grad.ncb ? static_cast<u32>((((4 * g + wave) * A.grad.ncb * 16 + j) * 2 + qp) * 4) : OOR;
    // S <- g S (adjoint: conj(g) S)
    auto decay = [&](f32x4 g0, f32x4 g1, float s) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = r < 2 ? g0[2 * r] : g1[2 * r - 4], y = s * (r < 2 ? g0[2 * r + 1] : g1[2 * r - 3]);
            const float own = S[r], oth = partner(own);
            S[r] = qp ? __builtin_fmaf(x, own, y * oth) : __builtin_fmaf(x, own, -y * oth);
        }
    };

    if (!adj) {
        const int row_v = n * 2 * static_cast<int>(sizeof(TV));
        const u32 lv = j < n ? static_cast<u32>((4 * g + wave) * n + j) * 2 * static_cast<u32>(sizeof(TV)) : OOR;
        struct Pre { f32x4 w0, w1, k0, k1, g0, g1; float2 x, v; };
        Pre pre[NB];
        struct Step { rsrc_t own, all, v; };
        auto step_of = [&](int st) __attribute__((always_inline)) {
            return Step{wk.rec(A, st, live), wk.rec(A, st, true), wk.rows(A, A.v, sizeof(TV), st)};
        };
        auto fetch_w = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
            const int at = b * A.lay.block;
            p.w0 = ldv4(q.own, l16, at + so);
            p.w1 = ldv4(q.own, l16 + 1024, at + so);
            p.x = ldv2(q.all, lx, at + A.lay.x);
            p.v = ld_cplx<TV>(q.v, lv, b * 16 * row_v);
            LOAD_ORDER();
        };
        auto fetch_k = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
            const int at = b * A.lay.block;
            p.g0 = ldv4(q.own, g * 32, at + A.lay.gc + wave * 128);
            p.g1 = ldv4(q.own, g * 32 + 16, at + A.lay.gc + wave * 128);
            p.k0 = ldv4(q.own, l16, at + so + A.lay.kq);
            p.k1 = ldv4(q.own, l16 + 1024, at + so + A.lay.kq);
            LOAD_ORDER();
        };
        Step cur = step_of(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) { fetch_w(cur, b, pre[b]); fetch_k(cur, b, pre[b]); }
        for (int st = 0; st < A.nsteps; ++st) {
            const Step next = step_of(st + 1);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                Pre& p = pre[b];
                const int ch = st * NB + b;
                if (b % GB == 0) put_state(wk.state(A, A.S_rec, ch / GB));
                f32x4 pw = zero4();
                mma1(pw, p.x.x, qp ? -p.v.y : p.v.x);        // conj(v) = (x, -y)
                mma1(pw, p.x.y, qp ? p.v.x : p.v.y);
                mma8(pw, p.w0, p.w1, bfrag_from_acc(S, qp));
                fetch_w(next, b, p);
                red[b & 1][0][wave][lane] = pw;
                __syncthreads();
                poison_slot(red[(b & 1) ^ 1][0][wave][lane]);
                f32x4 d[4];
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) d[w2] = red[b & 1][0][w2][lane];
                decay(p.g0, p.g1, 1.f);
                const f32x4 dd = (d[0] + d[1]) + (d[2] + d[3]);
                mma8(S, p.k0, p.k1, bfrag_from_acc(dd, qp));
                fetch_k(next, b, p);
                const float mine = wave == 0 ? dd[0] : wave == 1 ? dd[1] : wave == 2 ? dd[2] : dd[3];
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(mine), wk.block_rows(A, A.D_rows, ch), roff, 0, 0);
            }
        }
        return;
    }

    const int row_o = n * 2 * static_cast<int>(sizeof(TO));
    auto ooff = [&](int r) { return j < n ? static_cast<u32>((4 * g + r) * n + j) * 2 * static_cast<u32>(sizeof(TO)) : OOR; };
    struct Pre { f32x4 k0, k1, w0, w1, z0, z1, g0, g1; float2 ns, an, gw, u0, u1, u2, u3; };
    Pre pre[NB];
    struct Step { rsrc_t own, all, o; };
    auto step_of = [&](int st) __attribute__((always_inline)) {
        return Step{wk.rec(A, st, live), wk.rec(A, st, true), wk.rows(A, A.dO, sizeof(TO), st)};
    };
    auto fetch_k = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block;
        p.k0 = ldv4(q.own, l16, at + so + A.lay.kr);
        p.k1 = ldv4(q.own, l16 + 1024, at + so + A.lay.kr);
        LOAD_ORDER();
    };
    auto fetch_z = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block, t = b * 16 * row_o;
        p.g0 = ldv4(q.own, g * 32, at + A.lay.gc + wave * 128);
        p.g1 = ldv4(q.own, g * 32 + 16, at + A.lay.gc + wave * 128);
        p.u0 = ld_cplx<TO>(q.o, ooff(0), t);
        p.u1 = ld_cplx<TO>(q.o, ooff(1), t);
        p.u2 = ld_cplx<TO>(q.o, ooff(2), t);
        p.u3 = ld_cplx<TO>(q.o, ooff(3), t);
        p.z0 = ldv4(q.own, l16, at + so + A.lay.zs);
        p.z1 = ldv4(q.own, l16 + 1024, at + so + A.lay.zs);
        LOAD_ORDER();
    };
    auto fetch_w = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
        const int at = b * A.lay.block;
        p.w0 = ldv4(q.own, l16, at + so + A.lay.ws);
        p.w1 = ldv4(q.own, l16 + 1024, at + so + A.lay.ws);
        p.ns = ldv2(q.all, lx, at + A.lay.ns);
        p.an = ldv2(q.all, lx, at + A.lay.an);
        p.gw = ld_cplx<TO>(q.o, ooff(wave), b * 16 * row_o);
        LOAD_ORDER();
    };
    // G_F of block ch, whose shares lie in red[b & 1][1]: wave w sums rows 4g + w, records them
    // and writes dv = conj(beta G_F)
    const TV* const gb = static_cast<const TV*>(A.beta);
    TV* const gdv = static_cast<TV*>(A.dv);
    auto finish = [&](int b, int ch, bool some) __attribute__((always_inline)) {
        float f = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) f += reinterpret_cast<const float*>(&red[b & 1][1][w2][lane])[wave];
        const int rows = some ? max(min(A.T - ch * 16, 16), 0) : 0;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f), wk.block_rows(A, A.F_rows, ch, some), roff, 0, 0);
        const float bt = ld_real<TV>(rsrc(gb + wk.tok + ch * 16, rows * static_cast<int>(sizeof(TV))), (4 * g + wave) * static_cast<u32>(sizeof(TV)));
        const rsrc_t rv = rsrc(gdv + 2 * (wk.tok + ch * 16) * n, rows * n * 2 * static_cast<int>(sizeof(TV)));
        const float x = qp ? -bt * f : bt * f;
        st_real<TV>(rv, j < n ? static_cast<u32>(((4 * g + wave) * n + j) * 2 + qp) * static_cast<u32>(sizeof(TV)) : OOR, 0, x);
    };
    Step cur = step_of(A.nsteps - 1);
#pragma unroll
    for (int b = NB - 1; b >= 0; --b) { fetch_k(cur, b, pre[b]); fetch_z(cur, b, pre[b]); fetch_w(cur, b, pre[b]); }
    for (int st = A.nsteps - 1; st >= 0; --st) {
        const Step next = step_of(st - 1);
#pragma unroll
        for (int b = NB - 1; b >= 0; --b) {
            Pre& p = pre[b];
            const int ch = st * NB + b;
            if (b % GB == GB - 1) put_state(wk.state(A, A.G_rec, ch / GB));
            f32x4 px = zero4();                              // share of X' = conj(K Q) G
            mma8(px, p.k0, p.k1, bfrag_from_acc(S, qp));
            fetch_k(next, b, p);
            red[b & 1][0][wave][lane] = px;
            __syncthreads();
            poison_slot(red[(b & 1) ^ 1][0][wave][lane]);
            poison_slot(red[b & 1][1][wave][lane]);
            f32x4 d[4];
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) d[w2] = red[b & 1][0][w2][lane];
            decay(p.g0, p.g1, -1.f);
            {
                Frag8 gr;                                    // G_R = conj(dL/do)
                bpair(gr, 0, p.u0.x, -p.u0.y, qp);
                bpair(gr, 1, p.u1.x, -p.u1.y, qp);
                bpair(gr, 2, p.u2.x, -p.u2.y, qp);
                bpair(gr, 3, p.u3.x, -p.u3.y, qp);
                mma8(S, p.z0, p.z1, gr);
            }
            fetch_z(next, b, p);
            const Frag8 xb = bfrag_from_acc((d[0] + d[1]) + (d[2] + d[3]), qp);
            mma8(S, p.w0, p.w1, xb);
            f32x4 pf = zero4();                              // share of G_F: K index 4g + wave
            const float x0 = wave == 0 ? xb.v[0] : wave == 1 ? xb.v[2] : wave == 2 ? xb.v[4] : xb.v[6];
            const float x1 = wave == 0 ? xb.v[1] : wave == 1 ? xb.v[3] : wave == 2 ? xb.v[5] : xb.v[7];
            mma1(pf, p.ns.x, x0);
            mma1(pf, p.ns.y, x1);
            mma1(pf, p.an.x, qp ? -p.gw.y : p.gw.x);
            mma1(pf, p.an.y, qp ? p.gw.x : p.gw.y);
            finish((b + 1) % NB, ch + 1, ch + 1 < A.nsteps * NB);       // the block before this one in the walk
            red[b & 1][1][wave][lane] = pf;
            fetch_w(next, b, p);
        }
    }
    __syncthreads();
    finish(0, 0, true);
    if (A.dS0 != nullptr) {
        const rsrc_t rs = rsrc(reinterpret_cast<const char*>(A.dS0) + bh * wk.mn8, static_cast<int>(wk.mn8));
#pragma unroll
        for (int r = 0; r < 4; ++r) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(S[r]), rs, soff[r], 0, 0);
    }
}
template <typename TV, typename TO>
__global__ __launch_bounds__(256, 2) void bwd_f32_kernel(BwdArgs A, unsigned nfwd)
{
    __shared__ BwdF32Smem sm;
    const bool adj = blockIdx.x >= nfwd;
    bwd_f32<TV, TO>(sm, A, adj ? blockIdx.x - nfwd : blockIdx.x, adj);
}

// bf16 operands: the forward scan's layout of work (32 value columns; state waves with half the
// channels each, row waves that take Delta or X' from the exchange and write the rows).
template <typename TO>
__global__ __launch_bounds__(512, 1) void bwd_bf16_kernel(BwdArgs A, unsigned nfwd)
{
    constexpr int P = PREC_BF16;
    constexpr int GB = grad_blocks(true);
    static_assert(GB % 2 == 0, "the states to record wait in LDS for one block");
    __shared__ f32x4 red[2][4][2][64];                 // [parity][state wave][re, im][lane]
    __shared__ __align__(16) char st_out[4][2][16 * 144];     // states to record [state wave][half's block]: 16 channels x 16 columns, padded rows
    const bool adj = blockIdx.x >= nfwd;
    long bh;
    int sl;
    if (!scan_place(adj ? blockIdx.x - nfwd : blockIdx.x, A.n_slices, A.heads, bh, sl)) return;
    poison_area(red, 512);
    poison_area(st_out, 512);
    const int lane = threadIdx.x & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave8 & 3;
    const int c = lane & 15, g = lane >> 4, h = wave & 1, cw = wave >> 1;
    const int n = A.n, m = A.m;
    const int j = sl * BCOLS + cw * 16 + c;
    const Walk wk(A, bh);
    const u32 l16 = lane * 16;
    auto ldf = [&](rsrc_t r, u32 off, int s) __attribute__((always_inline)) {
        Frag<P> f;
        f.w = __builtin_amdgcn_raw_buffer_load_b128(r, off, s, 0);
        return f;
    };
    // rows 4g + r of a block, complex bf16 (v, dL/do as bf16) or fp32 (records, dL/do as fp32)
    u32 off4[4], off8[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        off4[r] = j < n ? static_cast<u32>((4 * g + r) * n + j) * 4u : OOR;
        off8[r] = j < n ? static_cast<u32>((4 * g + r) * n + j) * 8u : OOR;
    }
    auto rows_frag = [&](rsrc_t q, int es, int b) __attribute__((always_inline)) {   // conj of a block's rows
        Frag<P> f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (es == 2) {
                f.w[r] = __builtin_amdgcn_raw_buffer_load_b32(q, off4[r], b * 16 * n * 4, 0);
            } else {
                const float2 x = ldv2(q, off8[r], b * 16 * n * 8);
                f.w[r] = pack_bf16(x.x, x.y);
            }
        }
        return f;
    };
    auto conj_right = [&](Frag<P> f) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) f.w[r] ^= 0x80000000u;
        return right<P>(f);
    };
    const int st0 = adj ? A.nsteps - 1 : 0, dst = adj ? -1 : 1;

    if (wave8 < 4) {
        // ================================================ state waves
        const bool live0 = 2 * h < A.lay.nkb, live1 = 2 * h + 1 < A.lay.nkb;
        auto soff = [&](int g4, int kb, int r) {             // [m][n]
            const int i = (2 * h + kb) * 16 + g4 + r;
            return j < n && i < m ? static_cast<u32>(i * n + j) * 8u : OOR;
        };
        CAcc S[2];
        {
            const float* init = adj ? A.dS_T : A.S0;
            const rsrc_t rs = rsrc(init ? reinterpret_cast<const char*>(init) + bh * wk.mn8 : nullptr, init ? static_cast<int>(wk.mn8) : 0);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float2 x = ld_c64(rs, soff(4 * g, kb, r));
                    S[kb].re[r] = x.x;
                    S[kb].im[r] = x.y;
                }
        }
        auto put_state = [&]() __attribute__((always_inline)) {     // for the row waves to record
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<float2*>(st_out[wave][kb] + (4 * g + r) * 144 + c * 8) = make_float2(S[kb].re[r], S[kb].im[r]);
        };
        // a: the operand of the first product (-W; adjoint: conj(K Q)); k: of the second (K Q;
        // adjoint: -W^*); z, rows: the term known beforehand (T conj(V); adjoint: Z^* G_R)
        struct Pre { Frag<P> a[2], k[2], z[2], u; f32x4 g[2][2]; };
        Pre pre[NB];
        const int so = 2 * h * 1024, oa = adj ? A.lay.kr : 0, ok = adj ? A.lay.ws : A.lay.kq;
        struct Step { rsrc_t own[2], x, u; };
        auto step_of = [&](int st) __attribute__((always_inline)) {
            return Step{{wk.rec(A, st, live0), wk.rec(A, st, live1)}, wk.rec(A, st, h == 0),
                        adj ? wk.rows(A, A.dO, sizeof(TO), st) : wk.rows(A, A.v, 2, st)};
        };
        auto fetch_a = [&](const Step& q, int b, Pre& p) __attribute__((always_inline)) {
            const int at = b * A.lay.block;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) p.a[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so + oa);
            LOAD_ORDER();
        };
        auto fetch_k = [&](const Step& q, int b, Pre& p, auto adj_c) __attribute__((always_inline)) {
            constexpr bool ADJ = decltype(adj_c)::value;
            const int at = b * A.lay.block;
            p.u = rows_frag(q.u, ADJ ? static_cast<int>(sizeof(TO)) : 2, b);
            if constexpr (!ADJ) p.z[0] = ldf(q.x, l16, at + A.lay.x);      // T, on the first half's wave
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                for (int e = 0; e < 2; ++e) p.g[kb][e] = ldv4(q.own[kb], g * 32 + kb * 128 + e * 16, at + A.lay.gc + h * 256);
                if constexpr (ADJ) p.z[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so + A.lay.zs);
                p.k[kb] = ldf(q.own[kb], l16 + kb * 1024, at + so + ok);
            }
            LOAD_ORDER();
        };
        auto walk = [&](auto adj_c) __attribute__((always_inline)) {
            constexpr bool ADJ = decltype(adj_c)::value;
            auto block = [&](int b, int ch, Pre& p, const Step& next) __attribute__((always_inline)) {
                if (b % GB == (ADJ ? GB - 1 : 0)) put_state();
                const Right<P> ub = conj_right(p.u);
                CAcc d;
                czero(d);
                if constexpr (!ADJ) cmma<P>(d, p.z[0], ub);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) cmma<P>(d, p.a[kb], right_acc<P>(S[kb]));
                red[b & 1][wave][0][lane] = d.re;
                red[b & 1][wave][1][lane] = d.im;
                fetch_a(next, b, p);
                __syncthreads();
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    poison_slot(red[(b & 1) ^ 1][wave][e][lane]);
                    if (b % GB == (ADJ ? GB - 1 : 0)) continue;      // (read behind this barrier)
#pragma unroll
                    for (int r = 0; r < 4; ++r) poison_slot(*reinterpret_cast<float2*>(st_out[wave][e] + (4 * g + r) * 144 + c * 8));
                }
                const f32x4 ore = red[b & 1][wave ^ 1][0][lane], oim = red[b & 1][wave ^ 1][1][lane];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {             // S <- g S (adjoint: conj(g) S)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float x = p.g[kb][r >> 1][2 * (r & 1)], y0 = p.g[kb][r >> 1][2 * (r & 1) + 1], y = ADJ ? -y0 : y0;
                        const float a = S[kb].re[r], i = S[kb].im[r];
                        S[kb].re[r] = __builtin_fmaf(x, a, -y * i);
                        S[kb].im[r] = __builtin_fmaf(x, i, y * a);
                    }
                    if constexpr (ADJ) cmma<P>(S[kb], p.z[kb], ub);
                }
                d.re += ore;
                d.im += oim;
                const Right<P> db = right_acc<P>(d);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) cmma<P>(S[kb], p.k[kb], db);
                fetch_k(next, b, p, adj_c);
            };
            Step cur = step_of(st0);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = ADJ ? NB - 1 - i : i;
                fetch_a(cur, b, pre[b]);
                fetch_k(cur, b, pre[b], adj_c);
            }
            for (int s = 0, st = st0; s < A.nsteps; ++s, st += dst) {
                const Step next = step_of(st + dst);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int b = ADJ ? NB - 1 - i : i;
                    block(b, st * NB + b, pre[b], next);
                }
            }
        };
        if (adj) walk(std::true_type{});
        else walk(std::false_type{});
        if (adj && A.dS0 != nullptr) {
            const rsrc_t rs = rsrc(reinterpret_cast<const char*>(A.dS0) + bh * wk.mn8, static_cast<int>(wk.mn8));
            int g4 = 4 * g;                                  // (formed again: not held through the walk)
            asm volatile("" : "+v"(g4));
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(S[kb].re[r]), __float_as_uint(S[kb].im[r])}, rs, soff(g4, kb, r), 0, 0);
        }
    } else {
        // ================================================ row waves: blocks of parity h
        const char* const rowrec = adj ? A.F_rows : A.D_rows;
        const u32 rec_off = sl * 2 + cw < A.grad.ncb ? static_cast<u32>((sl * 2 + cw) * 2048) + l16 : OOR;
        const u32 st_off = sl * 2 + cw < A.grad.ncb ? static_cast<u32>((sl * 2 + cw) * 2048 + lane * 32) : OOR;
        struct Pre { Frag<P> ns, an, u; float b[4]; };
        Pre pre[2];
        const uint16_t* const gb = static_cast<const uint16_t*>(A.beta);
        uint16_t* const gdv = static_cast<uint16_t*>(A.dv);
        auto fetch = [&](int st, int b, Pre& p) __attribute__((always_inline)) {
            const rsrc_t q = wk.rec(A, st, true);
            const int at = b * A.lay.block;
            p.ns = ldf(q, l16, at + A.lay.ns);
            p.an = ldf(q, l16, at + A.lay.an);
            p.u = rows_frag(wk.rows(A, A.dO, sizeof(TO), st), sizeof(TO), b);
            const int rows = wk.in(st) ? max(min(A.T - (st * NB + b) * 16, 16), 0) : 0;
            const rsrc_t qb = rsrc(gb + wk.tok + (st * NB + b) * 16, rows * 2);
#pragma unroll
            for (int r = 0; r < 4; ++r) p.b[r] = ld_real<uint16_t>(qb, (4 * g + r) * 2);
            LOAD_ORDER();
        };
        if (adj) {
            fetch(st0, NB - 2 + h, pre[1]);
            fetch(st0, h, pre[0]);
        }
        for (int s = 0, st = st0; s < A.nsteps; ++s, st += dst) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                __syncthreads();
                // (the walks meet parity b & 1 = i & 1 forwards and 1 - (i & 1) backwards)
                const int par = adj ? 1 - (i & 1) : i & 1;
                const int ch = st * NB + (adj ? NB - 1 - i : i);
                if (par != h) {
                    // the state of a run's start (adjoint: end) to the records, by whole lines
                    if (i % GB != 0) continue;
                    const rsrc_t rs = wk.state(A, adj ? A.G_rec : A.S_rec, ch / GB);
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) {
                        const char* p = st_out[2 * cw + (kb >> 1)][kb & 1] + c * 144 + g * 32;
#pragma unroll
                        for (int e = 0; e < 2; ++e)
                            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(p + e * 16), rs, st_off + e * 16, kb * A.grad.ncb * 2048, 0);
                    }
                    continue;
                }
                CAcc d;
                d.re = red[par][2 * cw][0][lane] + red[par][2 * cw + 1][0][lane];
                d.im = red[par][2 * cw][1][lane] + red[par][2 * cw + 1][1][lane];
                if (adj) {
                    Pre& p = pre[(NB - 1 - i) >> 1];
                    cmma<P>(d, p.ns, right_acc<P>(d));           // (N^* without its ones)
                    cmma<P>(d, p.an, conj_right(p.u));
                    const rsrc_t rv = rsrc(gdv + 2 * (wk.tok + ch * 16) * n, max(min(A.T - ch * 16, 16), 0) * n * 4);
#pragma unroll
                    for (int r = 0; r < 4; ++r)              // dv = conj(beta G_F)
                        __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(p.b[r] * d.re[r], -p.b[r] * d.im[r]), rv, off4[r], 0, 0);
                    fetch(st - 1, ch - st * NB, p);
                }
                const rsrc_t rr = wk.block_rows(A, rowrec, ch);
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(d.re[2 * e]), __float_as_uint(d.im[2 * e]),
                                                                 __float_as_uint(d.re[2 * e + 1]), __float_as_uint(d.im[2 * e + 1])},
                                                           rr, rec_off + e * 1024, 0, 0);
            }
        }
    }
}

// ------------------------------------------------------------------ launches

template <int P, typename TIN, int KIND>
static hipError_t prep_t(const PrepArgs& a, long heads, hipStream_t st)
{
    hipLaunchKernelGGL((prep_kernel<P, TIN, KIND>), dim3(static_cast<unsigned>(heads * a.nsteps)), dim3(256), 0, st, a);
    return hipGetLastError();
}
template <int KIND>
static hipError_t prepare(const PrepArgs& a, long heads, bool bf, bool in_bf16, hipStream_t st)
{
    if (bf) return prep_t<PREC_BF16, uint16_t, KIND>(a, heads, st);
    return in_bf16 ? prep_t<PREC_F32, uint16_t, KIND>(a, heads, st) : prep_t<PREC_F32, float, KIND>(a, heads, st);
}

template <bool DEC>
static hipError_t scan_t(const ChunkLaunch& L, bool bf, const ScanArgs& a, hipStream_t st)
{
    const dim3 grid(static_cast<unsigned>(scan_grid(a.heads, a.n_slices)));
    if (bf) {
        if (L.out_bf16) hipLaunchKernelGGL((scan_bf16_kernel<uint16_t, DEC>), grid, dim3(512), 0, st, a);
        else hipLaunchKernelGGL((scan_bf16_kernel<float, DEC>), grid, dim3(512), 0, st, a);
    } else if (L.in_bf16) {
        if (L.out_bf16) hipLaunchKernelGGL((scan_f32_kernel<uint16_t, uint16_t, DEC>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((scan_f32_kernel<uint16_t, float, DEC>), grid, dim3(256), 0, st, a);
    } else {
        if (L.out_bf16) hipLaunchKernelGGL((scan_f32_kernel<float, uint16_t, DEC>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((scan_f32_kernel<float, float, DEC>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace fac

// Records of one 64-token step of every head, and the state carried between pieces
static long fac_step_bytes(long heads, int m, bool bf, bool dec)
{
    return heads * fac::NB * fac::RecLayout(m, bf, dec).block;
}

size_t factored_bytes(long heads, int T, int m, int n, bool in_bf16, bool dec, size_t cap)
{
    const long steps = (static_cast<long>(T) + fac::CP - 1) / fac::CP;
    const long one = fac_step_bytes(heads, m, bf16_operands(in_bf16, m), dec);
    long piece = one > 0 ? static_cast<long>(cap) / one : steps;
    piece = piece < 1 ? 1 : piece > steps ? steps : piece;
    return static_cast<size_t>(piece) * one + (piece < steps ? static_cast<size_t>(heads) * m * n * 8 : 0);
}

FactoredPlan factored_plan(long heads, int T, int m, int n, bool in_bf16, bool dec, size_t bytes, long cus)
{
    using namespace fac;
    const bool bf = bf16_operands(in_bf16, m);
    const long steps = (static_cast<long>(T) + CP - 1) / CP, one = fac_step_bytes(heads, m, bf, dec);
    const long carry_bytes = heads * m * static_cast<long>(n) * 8;
    const bool whole = static_cast<size_t>(steps) * one <= bytes;
    FactoredPlan p{whole ? steps : (static_cast<long>(bytes) - carry_bytes) / one, false};
    if (p.piece < 1) return FactoredPlan{0, false};
    const long most = ((1L << 32) / 256 - 1) / heads;   // workgroups of a launch (less than 2^32 threads)
    if (p.piece > most) p.piece = most;
    // float32 scans on at most half of the compute units: each piece's scan with the next one's
    // preparation beside it, the records in two halves of the workspace (H16 T65536: 3.86 ms
    // one after the other)
    const int cols = bf ? BCOLS : FCOLS;
    if (!dec && !in_bf16 && 2 * scan_grid(heads, (n + cols - 1) / cols) <= cus && steps >= 8) {
        const long half = whole ? (steps + 3) / 4 : p.piece / 2;
        if (half >= 1 && static_cast<size_t>(2 * half * one + carry_bytes) <= bytes) p = FactoredPlan{half, true};
    }
    return p;
}

hipError_t launch_factored(const ChunkLaunch& L, void* ws, size_t bytes, int cus, hipStream_t st)
{
    using namespace fac;
    const bool dec = L.r != nullptr, bf = bf16_operands(L.in_bf16, L.m);
    const long heads = static_cast<long>(L.B) * L.H;
    const int steps = static_cast<int>((static_cast<long>(L.T) + CP - 1) / CP);
    const long one = fac_step_bytes(heads, L.m, bf, dec);
    const long carry_bytes = heads * L.m * static_cast<long>(L.n) * 8;
    const FactoredPlan plan = factored_plan(heads, L.T, L.m, L.n, L.in_bf16, dec, bytes, cus);
    const long piece = plan.piece;
    const bool beside = plan.beside;
    if (piece < 1) return hipErrorInvalidValue;
    // the state between pieces: S_T where the caller wants it, else the end of the workspace
    float* carry = L.S_T ? L.S_T : reinterpret_cast<float*>(static_cast<char*>(ws) + bytes - carry_bytes);

    ScanArgs sa{static_cast<const char*>(ws), L.v, L.o, L.S0, nullptr, heads, L.T, L.m, L.n, 0, 0, 0, RecLayout(L.m, bf, dec)};
    const int cols = bf ? BCOLS : FCOLS;
    sa.n_slices = (L.n + cols - 1) / cols;
    PrepArgs pa{L.q, L.k, L.alpha, L.theta, L.beta, L.r, L.wbeta, static_cast<char*>(ws), L.T, L.m, 0, 0, sa.lay, BwdLayout(L.m, bf)};
    const long nscan = scan_grid(heads, sa.n_slices);
    for (int s = 0, half = 0; s < steps; s += static_cast<int>(piece), half ^= beside) {
        const int here = steps - s < piece ? steps - s : static_cast<int>(piece);
        const int after = steps - s - here < piece ? steps - s - here : static_cast<int>(piece);
        char* const at = static_cast<char*>(ws) + half * piece * one;
        pa.step0 = sa.step0 = s;
        pa.nsteps = sa.nsteps = here;
        pa.fac = at;
        sa.fac = at;
        sa.Sout = s + here < steps ? carry : L.S_T;
        hipError_t e = hipSuccess;
        if (!beside || s == 0)
            e = dec ? prepare<Kind::DEC>(pa, heads, bf, L.in_bf16, st) : prepare<Kind::FWD>(pa, heads, bf, L.in_bf16, st);
        if (e != hipSuccess) return e;
        if (beside && after > 0) {
            pa.step0 = s + here;
            pa.nsteps = after;
            pa.fac = static_cast<char*>(ws) + (half ^ 1) * piece * one;
            const dim3 grid(static_cast<unsigned>(nscan + heads * after));
            if (L.out_bf16) hipLaunchKernelGGL((scan_prep_f32_kernel<float, uint16_t>), grid, dim3(256), 0, st, sa, pa, static_cast<unsigned>(nscan));
            else hipLaunchKernelGGL((scan_prep_f32_kernel<float, float>), grid, dim3(256), 0, st, sa, pa, static_cast<unsigned>(nscan));
            e = hipGetLastError();
        } else {
            e = dec ? scan_t<true>(L, bf, sa, st) : scan_t<false>(L, bf, sa, st);
        }
        if (e != hipSuccess) return e;
        sa.Sin = carry;
    }
    return hipSuccess;
}

// ------------------------------------------------------------------ backward

// (n: a state record's bytes and a step's rows are 32-bit offsets; the gradient kernel's and both scans'
// launches, 256 threads per run of blocks, 256 per 8 or 512 per 32 columns, have less than 2^32 threads)
bool bwd_factored_fits(long heads, int T, int n)
{
    const long scans = std::max(256 * ((n + 7L) / 8), 512 * ((n + 31L) / 32));
    return heads * (T / 16L + fac::NB) * 256 < (1L << 32) && n <= (1 << 20) && 2 * (heads + 7) * scans < (1L << 32);
}

size_t bwd_factored_bytes(long heads, int T, int m, int n, bool in_bf16)
{
    const bool bf = bf16_operands(in_bf16, m);
    const fac::GradLayout g(T, m, n, bf);
    return g.bytes(heads) + static_cast<size_t>(heads) * g.blocks * fac::BwdLayout(m, bf).block;
}

// F: the forward's inputs; L: dL/do, dL/dS_T (S0), dS0 (S_T) and dv; Gl: the gradients' pointers
hipError_t launch_bwd_factored(const ChunkLaunch& F, const ChunkLaunch& L, const GradLaunch& Gl, void* ws, hipStream_t st)
{
    using namespace fac;
    const bool bf = bf16_operands(F.in_bf16, F.m);
    const long heads = static_cast<long>(F.B) * F.H;
    const int steps = static_cast<int>((static_cast<long>(F.T) + CP - 1) / CP);
    const GradLayout gl(F.T, F.m, F.n, bf);
    char* const rec = static_cast<char*>(ws) + heads * gl.blocks * BwdLayout(F.m, bf).block;
    const size_t states = static_cast<size_t>(heads) * gl.recs * gl.state, rows = static_cast<size_t>(heads) * gl.blocks * gl.rows;
    BwdArgs a{static_cast<const char*>(ws), F.v, L.dO, F.beta, F.S0, L.S0, L.S_T, rec, rec + states, rec + 2 * states,
              rec + 2 * states + rows, L.dv, heads, F.T, F.m, F.n, 0, steps, BwdLayout(F.m, bf), gl};
    const int cols = bf ? BCOLS : FCOLS;
    a.n_slices = (F.n + cols - 1) / cols;
    const PrepArgs pa{F.q, F.k, F.alpha, F.theta, F.beta, nullptr, nullptr, static_cast<char*>(ws), F.T, F.m, 0, steps,
                      RecLayout(F.m, bf, false), a.lay};
    hipError_t e = prepare<Kind::BWD>(pa, heads, bf, F.in_bf16, st);
    if (e != hipSuccess) return e;
    const unsigned nfwd = static_cast<unsigned>(scan_grid(heads, a.n_slices));
    const dim3 grid(2 * nfwd);
    if (bf) {
        if (F.out_bf16) hipLaunchKernelGGL((bwd_bf16_kernel<uint16_t>), grid, dim3(512), 0, st, a, nfwd);
        else hipLaunchKernelGGL((bwd_bf16_kernel<float>), grid, dim3(512), 0, st, a, nfwd);
    } else if (F.in_bf16) {
        if (F.out_bf16) hipLaunchKernelGGL((bwd_f32_kernel<uint16_t, uint16_t>), grid, dim3(256), 0, st, a, nfwd);
        else hipLaunchKernelGGL((bwd_f32_kernel<uint16_t, float>), grid, dim3(256), 0, st, a, nfwd);
    } else {
        if (F.out_bf16) hipLaunchKernelGGL((bwd_f32_kernel<float, uint16_t>), grid, dim3(256), 0, st, a, nfwd);
        else hipLaunchKernelGGL((bwd_f32_kernel<float, float>), grid, dim3(256), 0, st, a, nfwd);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_grad_steps(Gl, {a.S_rec, a.G_rec, a.D_rows, a.F_rows}, st);
}

}  // namespace sfda
