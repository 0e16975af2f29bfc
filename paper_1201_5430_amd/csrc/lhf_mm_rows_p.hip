// lhf_mm_rows_p.hip -- M2M and L2L by quarter turns, each coefficient vector split over the four 16-lane
// rows of a wavefront as in lhf_m2l_rows_p.hip, for one type and order (LHF_TURN_T, LHF_TURN_P on the
// compiler's command line).
//
// Eight shifts per wavefront: a parent's eight children (M2M), or eight consecutive children of a level
// (L2L).  Z(pi - a) Y Z(-b) Y C Y Z(b) Y Z(a) as for the M2L, C the (S|S) or (R|R) shift by the distance
// of child and parent with the conversion of eq. rcr1, one triangle per column m with (-1)^m, the powers
// of two between the box sizes and the distance folded in.  Orders 2k, 2k + 1 of both potentials are one
// stretch of a box's expansion: it passes through LDS (16 stretches per wavefront, 4 lanes each), the next
// one requested before the current one is turned; M2M sums the children there, in one order.
//
// What bounded the kernels before: table reads, one 16-byte load per two multiplications (the classes'
// tables in LDS or, from p = 20 on, in the caches), and for other orders a serial per-box kernel.
// M2M before and now: ring of 4.2 million at FP64 p = 23 15.4 -> 4.1 ms (L2L with the M2L's source copy 13.2 ->
// 5.0), 65,537 elements at p = 18 1.27 -> 0.06 ms.  What bounds it there: waits for memory and LDS, 64% of a
// wavefront's cycles (one per SIMD; 796 and 816 bytes of scratch a lane); the vector unit issues 20% of the time.
#include <algorithm>

#include "lhf_m2l_turn.h"
#include "lhf_rows.h"

namespace lhf {

template <typename T, int P, int KIND>
__global__ void __launch_bounds__(256 * (tm::waves<T, P>()), (tm::waves<T, P>())) k_mm_rows(
    int64_t off, int64_t nb, const int32_t *__restrict__ bchild0, const int32_t *__restrict__ bnchild,
    const int32_t *__restrict__ bparent, const uint64_t *__restrict__ bkey, const T *__restrict__ src_exp,
    T *__restrict__ dst_exp, const T *__restrict__ tab, const T *__restrict__ trig, const tn::Dir *__restrict__ dirs)
{
    static_assert(KIND == 0 || KIND == 2, "M2M or L2L");
    using tn::sfor;
    using tr::S;
    using tr::hoff;
    constexpr int P2 = P * P, K = (P + 1) / 2, NV = hoff(2 * K);
    constexpr int NW = 4 * tm::waves<T, P>(), NTH = 64 * NW;
    constexpr int TY = tr::ytab<T>(P), TH = tm::htab<T>(P), BS = tm::stretch(P);
    constexpr int E = 16 / (int)sizeof(T), CE = 16 * E;
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    typedef T V2 __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    T *wl = (T *)smem;                           // [4][TY] turns, [2][TH] shift
    V2 *trl = (V2 *)(wl + 4 * TY + 2 * TH);      // [octant][azimuth, polar][P] (cos, sin), one more for odd P
    T *sci = (T *)(trl + tm::trig_pairs(P)), *sco = sci + P2;
    // the last entry that trigs() reads: slot j = K - 1 of a lane with odd m, in the last octant
    static_assert(15 * P + 2 * (K - 1) + 1 < tm::trig_pairs(P), "angle table");
    T *buf = sco + P2 + wave * 16 * BS;          // the wavefront's stretches: [shift][potential][BS]
    {
        const V *ty = (const V *)tab, *th = (const V *)(tab + 4 * TY + KIND * TH);
        for (int i = tid; i < 4 * TY / E; i += NTH) ((V *)wl)[i] = ty[i];
        for (int i = tid; i < 2 * TH / E; i += NTH) ((V *)(wl + 4 * TY))[i] = th[i];
        const T *sc = tab + 4 * TY + 4 * TH + KIND * P2;
        for (int i = tid; i < 2 * P2; i += NTH) sci[i] = sc[i];
        for (int i = tid; i < 16 * P; i += NTH) {
            const int oct = i / (2 * P), r = i % (2 * P);
            // M2M: parent - child, L2L: child - parent
            const int sg = KIND == 0 ? -1 : 1;
            const int dx = oct & 1 ? sg : -sg, dy = oct & 2 ? sg : -sg, dz = oct & 4 ? sg : -sg;
            const tn::Dir dd = dirs[dx + 3 + 7 * (dy + 3) + 49 * (dz + 3)];
            trl[i] = ((const V2 *)trig)[(size_t)(r < P ? dd.ia : dd.ib) * P + r % P];
        }
        if ((P & 1) && tid == 0) trl[16 * P] = V2{0, 0};
    }
    __syncthreads();
    const int row = lane >> 4, r0 = row & 1, r1 = row >> 1, part = r1 ^ r0, pot = lane & 1, t = (lane & 15) >> 1;
    const int pin = part ? 1 - r0 : r0;
    using L = const volatile __attribute__((address_space(3))) V;
    L *wl3 = (L *)(const volatile __attribute__((address_space(3))) char *)wl + (lane & 15);
    L *wy1 = wl3 + (2 * part + pin) * (TY / E), *wh = wl3 + 4 * (TY / E) + pin * (TH / E);
    L *wy2[2] = {wl3 + (2 * part + r0) * (TY / E), wl3 + (2 * part + 1 - r0) * (TY / E)};
    const unsigned sga = r1 ? 0x80000000u : 0u, sgb = r0 ? 0x80000000u : 0u;
    const int st = lane >> 3, sp = (lane >> 2) & 1, se = lane & 3;  // a stretch's lanes: shift, potential, first entry
    const T *bin = buf + (2 * t + pot) * BS;

    const int64_t nwork = KIND == 0 ? nb : (nb + 7) / 8;
    for (int64_t w = (int64_t)blockIdx.x * NW + wave; w < nwork; w += (int64_t)gridDim.x * NW) {
        // the boxes of this lane's shift (its octant) and of its stretch (source, and target of L2L)
        int oct = t, src = -1, dst = 0;
        if constexpr (KIND == 0) {
            const int64_t b = off + w;
            const int nc = bnchild[b];
            if (nc == 0) continue;  // a leaf keeps its own multipole
            const int c0 = bchild0[b];
            for (int k = 0; k < nc; k++)
                if ((int)(bkey[c0 + k] & 7u) == st) src = c0 + k;
        } else {
            const int64_t c = off + 8 * w;
            const int nc = (int)min((int64_t)8, off + nb - c);
            oct = (int)(bkey[c + (t < nc ? t : 0)] & 7u);
            if (st < nc) {
                dst = (int)(c + st);
                src = bparent[dst];
            }
        }
        const bool act = src >= 0;
        const T *gsrc = src_exp + (size_t)(act ? src : 0) * 2 * P2 + sp * P2 + se;
        // opaque: what follows from it is cheaper formed again than held over the shifts
        int par = pin;
        asm volatile("" : "+v"(par));
        const V2 *ta = trl + oct * 2 * P + r1, *tb = trl + oct * 2 * P + P + (r0 ^ r1);
        V cur, nxt;
        auto request = [&](V &x, L *p, int chunk) __attribute__((always_inline)) {
            x = p[chunk * 16];
            __builtin_amdgcn_sched_barrier(0);
        };
        // the asm multiplications write registers unseen by the compiler's hazard checks: two wait states
        // before a cross-lane instruction reads them
        auto settle = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 1");
            __builtin_amdgcn_sched_barrier(0);
        };
        // what other lanes of the wavefront wrote to its stretches
        auto exchange = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        auto zrot = [&](auto kk, T *f, T *g, const V2 *cs, unsigned sg) __attribute__((always_inline)) {
            sfor<0, decltype(kk)::value + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                const T c = cs[j][0], s = tr::flip(cs[j][1], sg);
                const T x = f[j], y = g[j];
                f[j] = x * c - y * s;
                g[j] = y * c + x * s;
            });
        };
        // (cos, sin) of m = 2j + the row's parity; beyond the last order the entry is not used
        auto trigs = [&](auto kk, V2 *cs, const V2 *p) __attribute__((always_inline)) {
            sfor<0, decltype(kk)::value + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                cs[j] = p[2 * j];
            });
        };
        auto turn = [&](auto nn, T *x, L *p, L *np, int nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nn)::value, s = S(n), e0 = tr::yoff(n), e1 = e0 + s * s;
            T o[s];
            sfor<0, s>([&](auto ii) { o[decltype(ii)::value] = 0; });
            sfor<e0 / CE, (e1 + CE - 1) / CE>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                if constexpr ((c + 1) * CE < e1) request(nxt, p, c + 1);
                else request(nxt, np, nc);
                sfor<0, CE>([&](auto ii) {
                    constexpr int i = decltype(ii)::value, k = c * CE + i - e0;
                    if constexpr (k >= 0 && k < s * s) tr::fmab<i / E>(o[k % s], cur[i % E], x[k / s]);
                });
                __builtin_amdgcn_sched_barrier(0);
                cur = nxt;
            });
            sfor<0, s>([&](auto ii) { x[decltype(ii)::value] = o[decltype(ii)::value]; });
        };
        // a lane's part of the stretch of orders 2k, 2k + 1: entries se, se + 4, ..
        T pre[2 * K - 1];
        auto fetch = [&](auto kk, const T *p) __attribute__((always_inline)) {
            constexpr int k = decltype(kk)::value, cnt = tm::count(P, k), b0 = 4 * k * k;
            sfor<0, (cnt + 3) / 4>([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                if constexpr (4 * i + 3 < cnt) pre[i] = p[b0 + 4 * i];
                else pre[i] = p[se + 4 * i < cnt ? b0 + 4 * i : 0];
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        T v[NV];
        fetch(std::integral_constant<int, 0>{}, gsrc);
        request(cur, wy1, 0);
        sfor<0, K>([&](auto kk) {
            constexpr int k = decltype(kk)::value, n0 = 2 * k, n1 = n0 + 1, cnt = tm::count(P, k), b0 = 4 * k * k;
            constexpr bool two = n1 < P;
            using N0 = std::integral_constant<int, n0>;
            using N1 = std::integral_constant<int, n1>;
            T f[k + 1], g[k + 1];
            exchange();
            sfor<0, (cnt + 3) / 4>([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                const int e = se + 4 * i;
                if (4 * i + 3 < cnt || e < cnt)
                    buf[(2 * st + sp) * BS + e] = act ? pre[i] * sci[b0 + e] : (T)0;
            });
            exchange();
            if constexpr (k + 1 < K) fetch(std::integral_constant<int, k + 1>{}, gsrc);
            // order n0 + r0, m = 2j + r1: (Re, Im) in rows 0, 1, (Im, Re) in rows 2, 3
            const int re = (r0 ? 2 * n0 + 1 : 0) + r1, im = re + n0 + r0;
            const bool has = two || r0 == 0;
            const int first = r1 ? im : re, second = r1 ? re : im;
            sfor<0, k + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                const bool in = has && (j < k || r1 <= r0);  // m <= n
                const bool i1 = in && (j > 0 || r1);         // and m > 0, for the entry that can be Im of m = 0
                const T x = bin[in ? first + 2 * j : 0], y = bin[i1 ? second + 2 * j : 0];
                f[j] = in ? x : (T)0;
                g[j] = i1 ? y : (T)0;
            });
            V2 cs[k + 1];
            trigs(kk, cs, ta);
            zrot(kk, f, g, cs, sga);
            settle();
            sfor<0, k + 1>([&](auto jj) { tr::swap<16>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            constexpr int c0 = tr::yoff(n0) / CE, c1 = tr::yoff(n1) / CE, c2 = tr::yoff(n1 + 1) / CE;
            if constexpr (two) {
                turn(N0{}, f, wy1, wy1, c1);
                turn(N1{}, g, wy1, wy2[0], c0);
            } else {
                turn(N0{}, f, wy1, wy2[0], c0);
            }
            trigs(kk, cs, tb);
            settle();
            sfor<0, k + 1>([&](auto jj) { tr::swap<32>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            zrot(kk, f, g, cs, sgb);
            sfor<0, k + 1>([&](auto jj) { tr::swap<32>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            L *np = k + 1 < K ? wy1 : wh;
            if constexpr (two) {
                turn(N0{}, f, wy2[0], wy2[1], c1);
                turn(N1{}, g, wy2[1], np, k + 1 < K ? c2 : 0);
            } else {
                turn(N0{}, f, wy2[0], np, 0);
            }
            sfor<0, k + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                v[hoff(n0) + j] = f[j];
                v[hoff(n1) + j] = two ? g[j] : (T)0;
            });
        });
        // shift and conversion, slot j of every order (m = 2j + pin): the triangle by diagonals, then the
        // factors of the neighbouring order's chi
        sfor<0, K>([&](auto jj) {
            constexpr int j = decltype(jj)::value, n0 = 2 * j, R = P - n0;
            constexpr int e0 = tm::hoff_tab(P, j), q1 = R * (R + 1) / 2, e1 = e0 + q1 + R;
            T o[R], oth[R];
            const T s0 = pot == (KIND == 0 ? 0 : 1) ? (T)0.5 : (T)1, wchi = pot ? (T)1 : (T)0;
            sfor<0, R>([&](auto ii) { o[decltype(ii)::value] = 0; });
            sfor<e0 / CE, (e1 + CE - 1) / CE>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                if constexpr ((c + 1) * CE < e1) request(nxt, wh, c + 1);
                else if constexpr (j + 1 < K) request(nxt, wh, tm::hoff_tab(P, j + 1) / CE);
                else request(nxt, wy1, 0);
                sfor<0, CE>([&](auto ii) {
                    constexpr int i = decltype(ii)::value, k = c * CE + i - e0;
                    if constexpr (k >= 0 && k < q1) {
                        constexpr tr::Sym y = tr::sym(R, k);  // (r, r + d)
                        if constexpr (KIND == 0) tr::fmab<i / E>(o[y.c], cur[i % E], v[hoff(n0 + y.r) + j]);
                        else tr::fmab<i / E>(o[y.r], cur[i % E], v[hoff(n0 + y.c) + j]);
                    } else if constexpr (k >= q1 && k < q1 + R) {
                        if constexpr (k == q1) {
                            sfor<0, R>([&](auto aa) { o[decltype(aa)::value] *= s0; });
                            settle();
                            sfor<0, R>([&](auto aa) { oth[decltype(aa)::value] = swz_xor<17>(o[decltype(aa)::value]); });
                        }
                        // chi_n + (tau / n) chi_{n-1}, the highest order first, or chi_n - (tau / (n+1)) chi_{n+1}
                        constexpr int r = KIND == 0 ? R - 1 - (k - q1) : k - q1, q = KIND == 0 ? r - 1 : r + 1;
                        if constexpr (q >= 0 && q < R) tr::fmab<i / E>(o[r], cur[i % E], wchi * o[q]);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
                cur = nxt;
            });
            // phi -+ i tau m / (n + 1 | n) chi
            const T tau = (T)(KIND == 0 ? 0.4330127018922193 : 0.8660254037844386);  // sqrt(3) / 4, sqrt(3) / 2
            const T mw = (pot ? (T)0 : tau) * (part == (KIND == 0 ? 1 : 0) ? (T)-1 : (T)1) * (T)(2 * j + par);
            sfor<0, R>([&](auto ii) {
                constexpr int r = decltype(ii)::value, n = n0 + r, d = KIND == 0 ? n + 1 : n;
                T a = o[r];
                if constexpr (d > 0) a += mw * (T)(1.0 / (double)d) * oth[r];
                v[hoff(n) + j] = a;
            });
        });
        T *gdst = nullptr;
        if constexpr (KIND == 0) gdst = dst_exp + (size_t)(off + w) * 2 * P2;
        else gdst = dst_exp + (size_t)dst * 2 * P2 + sp * P2 + se;
        sfor<0, K>([&](auto kk) {
            constexpr int k = decltype(kk)::value, n0 = 2 * k, n1 = n0 + 1, cnt = tm::count(P, k), b0 = 4 * k * k;
            constexpr bool two = n1 < P;
            using N0 = std::integral_constant<int, n0>;
            using N1 = std::integral_constant<int, n1>;
            T f[k + 1], g[k + 1];
            if constexpr (KIND == 2) fetch(kk, gdst);  // L2L adds to what the M2L wrote
            sfor<0, k + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                f[j] = v[hoff(n0) + j];
                g[j] = two ? v[hoff(n1) + j] : (T)0;
            });
            V2 cs[k + 1];
            constexpr int c0 = tr::yoff(n0) / CE, c1 = tr::yoff(n1) / CE, c2 = tr::yoff(n1 + 1) / CE;
            if constexpr (two) {
                turn(N0{}, f, wy1, wy1, c1);
                turn(N1{}, g, wy1, wy2[0], c0);
            } else {
                turn(N0{}, f, wy1, wy2[0], c0);
            }
            trigs(kk, cs, tb);
            settle();
            sfor<0, k + 1>([&](auto jj) { tr::swap<32>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            zrot(kk, f, g, cs, sgb ^ 0x80000000u);
            sfor<0, k + 1>([&](auto jj) { tr::swap<32>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            if constexpr (two) {
                turn(N0{}, f, wy2[0], wy2[1], c1);
                turn(N1{}, g, wy2[1], wy1, k + 1 < K ? c2 : 0);
            } else {
                turn(N0{}, f, wy2[0], wy1, 0);
            }
            trigs(kk, cs, ta);
            settle();
            sfor<0, k + 1>([&](auto jj) { tr::swap<16>(f[decltype(jj)::value], g[decltype(jj)::value]); });
            zrot(kk, f, g, cs, sga ^ 0x80000000u);
            exchange();
            {
                const int re = (r0 ? 2 * n0 + 1 : 0) + r1, im = re + n0 + r0;
                const bool has = two || r0 == 0;
                const int first = r1 ? im : re, second = r1 ? re : im;
                T *bo = buf + (2 * t + pot) * BS;
                sfor<0, k + 1>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    const bool in = has && (j < k || r1 <= r0);
                    if (in) bo[first + 2 * j] = f[j];
                    if (in && (j > 0 || r1)) bo[second + 2 * j] = g[j];
                });
            }
            exchange();
            if constexpr (KIND == 0) {
                const int po = lane >> 5;
                sfor<0, (cnt + 31) / 32>([&](auto ii) {
                    const int e = (lane & 31) + 32 * decltype(ii)::value;
                    if (e < cnt) {
                        T a = 0;
                        for (int c = 0; c < 8; c++) a += buf[(2 * c + po) * BS + e];
                        gdst[po * P2 + b0 + e] = a * sco[b0 + e];
                    }
                });
            } else if (act) {
                sfor<0, (cnt + 3) / 4>([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    const int e = se + 4 * i;
                    if (4 * i + 3 < cnt || e < cnt) {
                        const T a = buf[(2 * st + sp) * BS + e] * sco[b0 + e];
                        gdst[b0 + 4 * i] = pre[i] + a;
                    }
                });
            }
        });
    }
}

template <typename T, int P, int KIND>
static void launch(const lhf_plan *Pl, int l, hipStream_t st)
{
    constexpr int NW = 4 * tm::waves<T, P>();
    const int64_t nb = Pl->lev[l].nb, nwork = KIND == 0 ? nb : (nb + 7) / 8;
    if (nb == 0) return;
    // one pass over the tables per workgroup: as many as the chip (CUS compute units of LDS_CU bytes) holds
    const unsigned grid = (unsigned)std::min<int64_t>((nwork + NW - 1) / NW, CUS * (LDS_CU / tm::bytes<T, P>()));
    k_mm_rows<T, P, KIND><<<dim3(grid), dim3(64 * NW), tm::bytes<T, P>(), st>>>(
        Pl->lev[l].off, nb, Pl->bchild0, Pl->bnchild, Pl->bparent, Pl->bkey,
        (const T *)(KIND == 0 ? Pl->M : Pl->Lc), (T *)(KIND == 0 ? Pl->M : Pl->Lc), (const T *)Pl->mmtab,
        (const T *)Pl->ttrig, (const tn::Dir *)Pl->tdir);
}

template <typename T, int P>
hipError_t mm_rows_attr()
{
    static_assert(tm::bytes<T, P>() <= LDS_CU, "tables and stretches exceed the LDS");
    const hipError_t e = hipFuncSetAttribute((const void *)k_mm_rows<T, P, 0>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)tm::bytes<T, P>());
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_mm_rows<T, P, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)tm::bytes<T, P>());
}

// M2M into the boxes of level l, or L2L into them from level l - 1 (l >= 3), added to what they hold
template <typename T, int P>
void mm_rows_launch(const lhf_plan *Pl, bool down, int l, hipStream_t st)
{
    if (down) launch<T, P, 2>(Pl, l, st);
    else launch<T, P, 0>(Pl, l, st);
}

template hipError_t mm_rows_attr<LHF_TURN_T, LHF_TURN_P>();
template void mm_rows_launch<LHF_TURN_T, LHF_TURN_P>(const lhf_plan *, bool, int, hipStream_t);

}  // namespace lhf
