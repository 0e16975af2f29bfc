// lhf_m2l_rows_p.hip -- the M2L by quarter turns with each coefficient vector split over the four
// 16-lane rows of a wavefront, for one type and order (LHF_TURN_T, LHF_TURN_P on the compiler's
// command line).
//
// A quarter turn does not mix four classes of coefficients: Re or Im, and the parity of m.  Row r of a
// wavefront holds one class (r0 = r & 1, r1 = r >> 1: parity r0 for Re, 1 - r0 for Im, Re where
// r1 == r0), lane 2t + pot of a row translation t of the batch (8 per wavefront).  In
// between two turns the class is (Re or Im, parity (r0 + n) & 1).  What mixes classes is exchanged
// between rows:
//   * z-rotations (Re with Im of one m): orders 2k and 2k + 1 are paired; a row swap gives each lane both
//     parts of one m of one of the two orders (swap of rows r, r ^ 1 outside the turns, r, r ^ 2 between
//     them).  The sources are loaded and the targets accumulated in that form, so the outer rotations
//     need one swap only;
//   * the conversion's other potential (row r ^ 1, lane ^ 1) comes by ds_swizzle.
// The turn's and the shift's matrix entries are the same for all 16 lanes of a row: a row's next 16 or
// 32 entries are one LDS load, and the multiplications broadcast them from the loaded register
// (row_newbcast), so LDS returns 1/16 of what a broadcast read for each multiplication would.
// What bounds it (4M ring at p = 23, one wavefront per SIMD, 256 VGPRs + 256 AGPRs, no scratch; counters in
// profiles/): vector instructions are in flight 58% of a wavefront's cycles, 66% of them FMAs; it waits 19% of them,
// 8% on LDS, where accumulations and angles conflict.  HBM 102 GB in 237 ms, 5% of the peak.  p = 13 (two
// wavefronts): vector issue 53% of the time, waits 32%, LDS 12%.
#include <algorithm>

#include "lhf_m2l_turn.h"
#include "lhf_rows.h"

namespace lhf {

template <typename T, int P, bool SC>
__global__ void __launch_bounds__(256 * (tr::waves<T, P>()), (tr::waves<T, P>())) k_m2l_rows(
    tn::Levels lv, const uint64_t *__restrict__ bkey, const T *__restrict__ Ms, T *__restrict__ Lc,
    const T *__restrict__ tab, const T *__restrict__ trig, const T *__restrict__ oscale,
    const tn::Dir *__restrict__ dirs)
{
    using tn::sfor;
    using tr::S;
    using tr::hoff;
    constexpr int NPOT = SC ? 1 : 2, NTB = 16 / NPOT;
    constexpr int P2 = P * P, K = (P + 1) / 2, NS = tr::nslot(P), NV = hoff(2 * K);
    constexpr int SS = tr::acc_stride(P, NPOT), TS = tn::trig_stride(P), NTH = 256 * tr::waves<T, P>();
    constexpr int TY = tr::ytab<T>(P), TH = tr::htab<T>(P);
    constexpr int E = 16 / (int)sizeof(T), CE = 16 * E;  // entries of a lane's load, of a chunk
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    typedef T V2 __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t per = (lv.ntiles + 7) / 8;
    const int64_t tile = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (tile >= lv.ntiles) return;
    int q = 0;
    while (q + 1 < lv.n && tile >= lv.l[q + 1].tile0) q++;
    const int level = lv.level[q], ns = lv.l[q].ns, side = 1 << level;
    const int32_t *dmap = lv.l[q].dmap;
    const int64_t b0 = lv.l[q].off + (tile - lv.l[q].tile0) * ns;
    const int nt = (int)min((int64_t)ns, lv.l[q].off + lv.l[q].nb - b0);

    T *wl = (T *)smem;                                   // [4][TY] turns, [2][TH] shift
    T *trl = wl + 4 * TY + 2 * TH;                       // [NROW][TS] (cos, sin), one more for odd P
    double *acc = (double *)(trl + 2 * tn::trig_pairs(P));  // [ns + 1][SS] (last slot absorbs)
    // the last entry that trigs() reads: slot j = K - 1 of a lane with odd m, in the last row
    static_assert((tn::NROW - 1) * TS + 2 * (K - 1) + 1 < tn::trig_pairs(P), "angle table");
    int *esrc = (int *)(acc + (size_t)(ns + 1) * SS);
    int *sxyz = esrc + VMAX * ns, *ssys = sxyz + ns;
    int *cnt = ssys + ns;
    uint16_t *ecode = (uint16_t *)(cnt + 1);

    for (int i = tid; i < (4 * TY + 2 * TH) / E; i += NTH) ((V *)wl)[i] = ((const V *)tab)[i];
    for (int i = tid; i < tn::NROW * P; i += NTH) ((V2 *)trl)[i / P * TS + i % P] = ((const V2 *)trig)[i];
    if ((P & 1) && tid == 0) ((V2 *)trl)[tn::NROW * TS] = V2{0, 0};
    for (int i = tid; i < (ns + 1) * SS; i += NTH) acc[i] = 0.0;
    tn::targets(b0, nt, level, bkey, sxyz, ssys, cnt, tid);
    __syncthreads();
    tn::translations<NTH>(nt, side, dmap, sxyz, ssys, cnt, esrc, ecode, tid, lane);
    __syncthreads();
    const int ne = *cnt;
    const int row = lane >> 4, r0 = row & 1, r1 = row >> 1, part = r1 ^ r0, pot = SC ? 0 : lane & 1;
    // table of a class: [part][parity of the input]
    const int pin = part ? 1 - r0 : r0;                   // outside the turns; between them (r0 + n) & 1
    using L = const volatile __attribute__((address_space(3))) V;
    L *wl3 = (L *)(const volatile __attribute__((address_space(3))) char *)wl + (lane & 15);
    L *wy1 = wl3 + (2 * part + pin) * (TY / E), *wh = wl3 + 4 * (TY / E) + pin * (TH / E);
    L *wy2[2] = {wl3 + (2 * part + r0) * (TY / E), wl3 + (2 * part + 1 - r0) * (TY / E)};
    const unsigned sga = r1 ? 0x80000000u : 0u, sgb = r0 ? 0x80000000u : 0u;

    for (int bt = wave * NTB; bt < ne; bt += NTB * (NTH / 64)) {
        const int e = bt + (lane & 15) / NPOT;
        const bool act = e < ne;
        const int code = ecode[act ? e : bt], src = esrc[act ? e : bt];
        const int slot = act ? (code & 63) : ns;
        const tn::Dir dd = dirs[code >> 6];
        const T itau = (T)dd.itau, tau = (T)dd.tau;
        // opaque: what follows from it is cheaper formed again than held over the batches
        int par = pin;
        asm volatile("" : "+v"(par));
        const V2 *ta = (const V2 *)trl + dd.ia * TS + r1, *tb = (const V2 *)trl + dd.ib * TS + (r0 ^ r1);
        // source: (first, second) of order 2k + r0, m = 2j + r1, first = Re in rows 0, 1 and Im in rows 2, 3
        V2 sv[NS];
        {
            const V2 *sp = (const V2 *)Ms + ((size_t)src * NS * 4 + row) * NPOT + pot;
            sfor<0, NS>([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                sv[i] = sp[i * 4 * NPOT];
            });
        }
        // chunks of the row's table entries: the next one is requested before the current one is used
        V cur, nxt;
        auto request = [&](V &w, L *p, int chunk) __attribute__((always_inline)) {
            w = p[chunk * 16];
            __builtin_amdgcn_sched_barrier(0);
        };
        // out-of-line effects of the asm multiplications on cross-lane instructions that follow: the
        // compiler does not see that they wrote the registers by the vector unit (two wait states)
        auto settle = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 1");
            __builtin_amdgcn_sched_barrier(0);
        };
        auto zrot = [&](auto kk, T *f, T *g, const V2 *cs, unsigned sg) __attribute__((always_inline)) {
            constexpr int k = decltype(kk)::value;
            sfor<0, k + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                const T c = cs[j][0], s = tr::flip(cs[j][1], sg);
                const T x = f[j], y = g[j];
                f[j] = x * c - y * s;
                g[j] = y * c + x * s;
            });
        };
        auto trigs = [&](auto kk, V2 *cs, const V2 *t) __attribute__((always_inline)) {
            sfor<0, decltype(kk)::value + 1>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                cs[j] = t[2 * j];
            });
        };
        // x <- Y x for order n with the table p; the chunk after the last: 'nc' of the table 'np'
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
        T v[NV];
        request(cur, wy1, 0);
        {
            T t0 = (T)1;
            sfor<0, K>([&](auto kk) {
                constexpr int k = decltype(kk)::value, n0 = 2 * k, n1 = n0 + 1;
                constexpr bool two = n1 < P;
                using N0 = std::integral_constant<int, n0>;
                using N1 = std::integral_constant<int, n1>;
                T f[k + 1], g[k + 1];
                sfor<0, k + 1>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    f[j] = sv[tr::nslot(2 * k) + j][0];
                    g[j] = sv[tr::nslot(2 * k) + j][1];
                });
                V2 cs[k + 1];
                trigs(kk, cs, ta);
                zrot(kk, f, g, cs, sga);
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
                    v[hoff(n0) + j] = f[j] * t0;
                    v[hoff(n1) + j] = two ? g[j] * (t0 * itau) : (T)0;
                });
                t0 *= itau * itau;
            });
        }
        {
            // coaxial shift and R-conversion, slot j of every order (m = 2j + pin): the shift's symmetric
            // block, its order-p row and the conversion's factors kappa follow each other in the table
            const T wphi = (pot ? (T)0 : tau) * (part ? (T)1 : (T)-1), wchi = pot ? (T)-1 : (T)0;
            sfor<0, K>([&](auto jj) {
                constexpr int j = decltype(jj)::value, n0 = 2 * j, R = P - n0;  // orders n0 .. P - 1 (and P)
                constexpr int e0 = tr::hoff_tab(P, j), q1 = R * (R + 1) / 2, e1 = e0 + q1 + 2 * R;
                T o[R + 1];
                sfor<0, R + 1>([&](auto ii) { o[decltype(ii)::value] = 0; });
                T oth[R];
                sfor<e0 / CE, (e1 + CE - 1) / CE>([&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    if constexpr ((c + 1) * CE < e1) request(nxt, wh, c + 1);
                    else if constexpr (j + 1 < K) request(nxt, wh, tr::hoff_tab(P, j + 1) / CE);
                    else request(nxt, wy1, 0);
                    sfor<0, CE>([&](auto ii) {
                        constexpr int i = decltype(ii)::value, k = c * CE + i - e0;
                        if constexpr (k >= 0 && k < q1) {
                            // diagonal d of the block (entries (r, r + d)): neighbours write different sums
                            constexpr tr::Sym y = tr::sym(R, k);
                            tr::fmab<i / E>(o[y.r], cur[i % E], v[hoff(n0 + y.c) + j]);
                            if constexpr (y.r != y.c) tr::fmab<i / E>(o[y.c], cur[i % E], v[hoff(n0 + y.r) + j]);
                        } else if constexpr (!SC && k >= q1 && k < q1 + R) {
                            tr::fmab<i / E>(o[R], cur[i % E], v[hoff(n0 + k - q1) + j]);
                        } else if constexpr (!SC && k >= q1 + R && k < q1 + 2 * R) {
                            constexpr int r = k - q1 - R;
                            if constexpr (r == 0) {
                                settle();
                                // phi: + i |d| m / n chi (the same m of the other potential)
                                sfor<0, R>([&](auto aa) { oth[decltype(aa)::value] = swz_xor<17>(o[decltype(aa)::value]); });
                            }
                            // chi_n - kappa chi_{n+1}
                            tr::fmab<i / E>(o[r], cur[i % E], wchi * o[r + 1]);
                        }
                    });
                    __builtin_amdgcn_sched_barrier(0);
                    cur = nxt;
                });
                const T mw = wphi * (T)(2 * j + par);
                sfor<0, R>([&](auto ii) {
                    constexpr int r = decltype(ii)::value, n = n0 + r;
                    T a = o[r];
                    if constexpr (!SC && n > 0) a += mw * (T)(1.0 / (double)n) * oth[r];
                    v[hoff(n) + j] = a;
                });
            });
        }
        {
            double *ap = acc + (size_t)slot * SS + row * NPOT + pot;
            T t0 = itau;
            sfor<0, K>([&](auto kk) {
                constexpr int k = decltype(kk)::value, n0 = 2 * k, n1 = n0 + 1;
                constexpr bool two = n1 < P;
                using N0 = std::integral_constant<int, n0>;
                using N1 = std::integral_constant<int, n1>;
                T f[k + 1], g[k + 1];
                sfor<0, k + 1>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    f[j] = v[hoff(n0) + j] * t0;
                    g[j] = two ? v[hoff(n1) + j] * (t0 * itau) : (T)0;
                });
                t0 *= itau * itau;
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
                sfor<0, k + 1>([&](auto jj) {
                    constexpr int j = decltype(jj)::value, i = tr::nslot(2 * k) + j;
                    unsafeAtomicAdd(ap + i * 8 * NPOT, (double)f[j]);
                    unsafeAtomicAdd(ap + i * 8 * NPOT + 4 * NPOT, (double)g[j]);
                });
            });
        }
    }
    __syncthreads();
    for (int i = tid; i < nt * 2 * P2; i += NTH) {
        const int sl = i / (2 * P2), kk = i % (2 * P2), po = kk / P2, r = kk % P2;
        int n = (int)sqrtf((float)r);
        if ((n + 1) * (n + 1) <= r) n++;
        if (n * n > r) n--;
        const int c = r - n * n, pt = c > n, m = pt ? c - n : c;
        const int k = n >> 1, s = k * (k + 1) / 2 + (m >> 1), rw = 2 * (m & 1) + (n & 1);
        const double a = po < NPOT ? acc[(size_t)sl * SS + s * 8 * NPOT + (pt ^ (m & 1)) * 4 * NPOT + rw * NPOT + po] : 0.0;
        Lc[(size_t)b0 * 2 * P2 + i] = (T)(a * (double)oscale[r]);
    }
}

template <typename T, int P, bool SC>
static void launch(const lhf_plan *Pl, hipStream_t st)
{
    constexpr int NPOT = SC ? 1 : 2, NTH = 256 * tr::waves<T, P>();
    const size_t fixed = tr::fixed_bytes<T>(P, NPOT), each = tr::slot_bytes(P, NPOT);
    const int mx = tr::max_ns<T>(P, NPOT), ns = tr::own_ns(Pl, mx);
    const tn::Levels lv = tn::levels(Pl, ns, mx);
    if (lv.ntiles == 0) return;
    k_m2l_rows<T, P, SC><<<dim3((unsigned)((lv.ntiles + 7) / 8 * 8)), dim3(NTH), fixed + tn::max_ns(lv) * each, st>>>(
        lv, Pl->bkey, (const T *)Pl->l2pv, (T *)Pl->Lc, (const T *)Pl->ttab, (const T *)Pl->ttrig,
        (const T *)Pl->tscale + P * P, (const tn::Dir *)Pl->tdir);
}

template <typename T, int P>
hipError_t rows_attr()
{
    const hipError_t e = hipFuncSetAttribute((const void *)k_m2l_rows<T, P, false>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CU);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_m2l_rows<T, P, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CU);
}

template <typename T, int P>
void rows_launch(const lhf_plan *Pl, bool scalar, hipStream_t st)
{
    if (scalar) launch<T, P, true>(Pl, st);
    else launch<T, P, false>(Pl, st);
}

template hipError_t rows_attr<LHF_TURN_T, LHF_TURN_P>();
template void rows_launch<LHF_TURN_T, LHF_TURN_P>(const lhf_plan *, bool, hipStream_t);

}  // namespace lhf
