// lhf_m2l_turn_p.hip -- the M2L by quarter turns with whole coefficient vectors per lane, for one type
// and order (LHF_TURN_T, LHF_TURN_P on the compiler's command line).
//
// A lane holds both parts of one potential of one translation (p^2 values), so rotations, shift and
// conversion stay in the lane; only the other potential of the conversion comes from the neighbour lane
// (DPP).  32 translations per wavefront.  All lanes multiply by the same table entry: the entries are
// scalar loads (two of 64 bytes at a time) and a scalar operand of the multiplication.  Scalar loads
// return out of order, so a wait is for all of them: the next chunk is requested before the current
// chunk's multiplications and waited for after them (volatile loads: as plain ones the compiler places
// them behind the multiplications; FP64 p = 12 on the 2^20 cube 47.6 -> 41 ms with the request ahead, and
// 33 ms with outputs as the inner loop, which keeps neighbouring multiplications independent).
// What bounds it (FP64 p = 12, 2^20 cube, one wavefront per SIMD: 256 VGPRs + 256 AGPRs, 100 bytes of scratch a
// lane; counters in profiles/): the vector unit issues 52% of the time, 58% of that FMAs; a wavefront waits 18%
// of its cycles for scalar loads, LDS and sources, and 12% to issue.  FP32 and FP64 p = 8 (two or more
// wavefronts): also the source loads (64 lines an instruction) and LDS (angles, accumulation).
#include <algorithm>

#include "lhf_m2l_turn.h"

namespace lhf {

template <typename T, int P, bool SC>
__global__ void __launch_bounds__(tn::NTHR, (tn::waves<T, P>())) k_m2l_turn(tn::Levels lv, const uint64_t *__restrict__ bkey,
                                                           const T *__restrict__ Ms, T *__restrict__ Lc,
                                                           const T *__restrict__ tab, const T *__restrict__ trig,
                                                           const T *__restrict__ oscale,
                                                           const tn::Dir *__restrict__ dirs)
{
    using tn::sfor;
    constexpr int NPOT = SC ? 1 : 2, NTB = 64 / NPOT;  // potentials, translations of a batch
    constexpr int P2 = P * P, SS = tn::acc_stride(P, NPOT), TS = tn::trig_stride(P), SP = tn::src_stride<T>(P);
    using Chunk = tn::Chunk<T>;
    using Half = typename Chunk::H;
    using CHalf = const volatile __attribute__((address_space(4))) Half;
    constexpr int CH = tn::chunk<T>();
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // consecutive tiles stay on one XCD (shared L2)
    const int64_t per = (lv.ntiles + 7) / 8;
    const int64_t tile = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (tile >= lv.ntiles) return;
    int q = 0;
    while (q + 1 < lv.n && tile >= lv.l[q + 1].tile0) q++;
    const int level = lv.level[q], ns = lv.l[q].ns, side = 1 << level;
    const int32_t *dmap = lv.l[q].dmap;
    const int64_t b0 = lv.l[q].off + (tile - lv.l[q].tile0) * ns;
    const int nt = (int)min((int64_t)ns, lv.l[q].off + lv.l[q].nb - b0);

    const tn::Lds at = tn::lds<T, P, NPOT>(ns);
    T *trl = (T *)(smem + at.trl);                      // [NROW][TS] (cos, sin)
    double *acc = (double *)(smem + at.acc);            // [ns + 1][SS] (last slot absorbs)
    int *esrc = (int *)(smem + at.esrc);
    int *sxyz = (int *)(smem + at.sxyz), *ssys = (int *)(smem + at.ssys);
    int *cnt = (int *)(smem + at.cnt);
    uint16_t *ecode = (uint16_t *)(smem + at.ecode);

    for (int i = tid; i < 2 * tn::NROW * P; i += tn::NTHR) {
        const int r = i / (2 * P);
        trl[r * 2 * TS + i % (2 * P)] = trig[i];
    }
    for (int i = tid; i < (ns + 1) * SS; i += tn::NTHR) acc[i] = 0.0;
    tn::targets(b0, nt, level, bkey, sxyz, ssys, cnt, tid);
    __syncthreads();
    tn::translations<tn::NTHR>(nt, side, dmap, sxyz, ssys, cnt, esrc, ecode, tid, lane);
    __syncthreads();
    const int ne = *cnt;
    const int pot = SC ? 0 : lane & 1;

    for (int bt = wave * NTB; bt < ne; bt += 4 * NTB) {
        const int e = bt + lane / NPOT;
        const bool act = e < ne;
        const int code = act ? ecode[e] : 0, src = esrc[act ? e : bt];
        const int slot = act ? (code & 63) : ns;
        const int dir = act ? (code >> 6) : (ecode[bt] >> 6);
        const tn::Dir dd = dirs[dir];
        const T itau = (T)dd.itau, tau = (T)dd.tau;
        const T *ta = trl + dd.ia * 2 * TS, *tb = trl + dd.ib * 2 * TS;
        using V2 = T __attribute__((ext_vector_type(2)));
        T v[P2];
        {
            constexpr int E = 16 / sizeof(T);
            typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
            const V *sp = (const V *)(Ms + ((size_t)src * NPOT + pot) * SP);
            sfor<0, SP / E>([&](auto qq) {
                constexpr int k0 = decltype(qq)::value;
                const V x = sp[k0];
                sfor<0, E>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    if constexpr (k0 * E + j < P2) v[k0 * E + j] = x[j];
                });
            });
        }
        // the table's chunks: the next one is requested before the current one's multiplications, and
        // waited for after them (scalar loads return in any order: a wait is for all of them)
        Chunk cur, nxt;
        auto request = [&](Chunk &w, int off) __attribute__((always_inline)) {
            const T *p = tab;
            asm volatile("" : "+s"(p));  // the entries are loop-invariant and must not be hoisted
            const Half *q = (const Half *)(p + off);
            w.a = *(CHalf *)q;
            w.b = *(CHalf *)(q + 1);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto wait = [&](Chunk &w) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+s"(w.a), "+s"(w.b));
        };
        // (cos, sin)(m a) of order n's m from LDS
        auto trigs = [&](auto nn, T *cs, const T *t) __attribute__((always_inline)) {
            constexpr int n = decltype(nn)::value;
            sfor<1, n + 1>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                const V2 x = *(const V2 *)(t + 2 * m);
                cs[2 * m] = x[0];
                cs[2 * m + 1] = x[1];
            });
        };
        // Re' = Re c - Im s, Im' = Im c + Re s (s = sgn sin)
        auto zrot = [&](auto nn, T *x, const T *cs, T sg) __attribute__((always_inline)) {
            constexpr int n = decltype(nn)::value;
            sfor<1, n + 1>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                const T c = cs[2 * m], s = cs[2 * m + 1] * sg;
                const T re = x[m], im = x[n + m];
                x[m] = re * c - im * s;
                x[n + m] = im * c + re * s;
            });
        };
        // x <- Y x of order n with the chunk 'cur' in hand; 'next': offset of the chunk that follows;
        // 'ahead' issues the loads of what follows
        auto turn = [&](auto nn, T *x, int next, auto &&ahead) __attribute__((always_inline)) {
            constexpr int n = decltype(nn)::value;
            constexpr int NY = tn::ysize(n), NC = (NY + CH - 1) / CH, Y0 = tn::yoff(n, CH);
            T o[2 * n + 1];
            sfor<0, NC>([&](auto kk) {
                constexpr int k = decltype(kk)::value;
                if constexpr (k == 0) ahead();
                request(nxt, k + 1 < NC ? Y0 + (k + 1) * CH : next);
                sfor<0, CH>([&](auto ii) {
                    constexpr int i = decltype(ii)::value, e = k * CH + i;
                    if constexpr (e < NY) {
                        constexpr tn::YEnt y = tn::yent(n, e);
                        const T w = cur.template at<i>();
                        if constexpr (y.first) o[y.out] = w * x[y.in];
                        else o[y.out] += w * x[y.in];
                    }
                });
                wait(nxt);
                cur = nxt;
            });
            sfor<0, 2 * n + 1>([&](auto ii) { x[decltype(ii)::value] = o[decltype(ii)::value]; });
        };
        request(cur, tn::yoff(0, CH));
        wait(cur);
        {
            T tn_ = (T)1;
            T ca[2 * P], cb[2 * P];
            sfor<0, P>([&](auto nn) {
                constexpr int n = decltype(nn)::value;
                constexpr int Y0 = tn::yoff(n, CH), Y1 = n + 1 < P ? tn::yoff(n + 1, CH) : tn::hoff(P, 0, CH);
                T *x = v + n * n;
                if constexpr (n == 0) trigs(nn, ca, ta);
                zrot(nn, x, ca, (T)1);
                turn(nn, x, Y0, [&]() __attribute__((always_inline)) { trigs(nn, cb, tb); });
                zrot(nn, x, cb, (T)1);
                turn(nn, x, Y1, [&]() __attribute__((always_inline)) {
                    if constexpr (n + 1 < P) trigs(std::integral_constant<int, n + 1>{}, ca, ta);
                });
                sfor<0, 2 * n + 1>([&](auto ii) { x[decltype(ii)::value] *= tn_; });
                tn_ *= itau;
            });
        }
        {
            [[maybe_unused]] const T tphi = pot ? (T)0 : tau, wchi = pot ? (T)-1 : (T)0;
            sfor<0, P>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                constexpr int K = P - m, R = K + 1, NH = tn::hsize(P, m), NC = (NH + CH - 1) / CH;
                constexpr int H0 = tn::hoff(P, m, CH), H1 = m + 1 < P ? tn::hoff(P, m + 1, CH) : tn::yoff(0, CH);
                T ore[R], oim[R];
                sfor<0, NC>([&](auto kk) {
                    constexpr int k = decltype(kk)::value;
                    request(nxt, k + 1 < NC ? H0 + (k + 1) * CH : H1);
                    sfor<0, CH>([&](auto ii) {
                        constexpr int i = decltype(ii)::value, e = k * CH + i, c = e / R, r = e % R, n2 = m + c;
                        if constexpr (e < NH && !(SC && r == K)) {
                            const T w = cur.template at<i>();
                            if constexpr (c == 0) ore[r] = w * v[n2 * n2 + m];
                            else ore[r] += w * v[n2 * n2 + m];
                            if constexpr (m > 0) {
                                if constexpr (c == 0) oim[r] = w * v[n2 * n2 + n2 + m];
                                else oim[r] += w * v[n2 * n2 + n2 + m];
                            }
                        }
                    });
                    wait(nxt);
                    cur = nxt;
                });
                // R-conversion: phi~ = phi + i |d| m/n chi, chi~_n = chi_n - |d| kappa/(n+1) chi_{n+1}; the
                // powers |d|^-(n+1) of out_n come with the back-rotation, so out_{n+1}'s extra one cancels |d|
                sfor<0, K>([&](auto rr) {
                    constexpr int r = decltype(rr)::value, n = m + r;
                    constexpr double kap = tn::csqrt((double)((n + 1) * (n + 1) - m * m)) / (double)(n + 1);
                    T a = ore[r];
                    if constexpr (!SC) a += wchi * (T)kap * ore[r + 1];
                    if constexpr (m > 0) {
                        T b = oim[r];
                        if constexpr (!SC) {
                            b += wchi * (T)kap * oim[r + 1];
                            const T fphi = tphi * (T)((double)m / (double)n);
                            a -= fphi * dpp_f<DPP_XOR1>(oim[r]);
                            b += fphi * dpp_f<DPP_XOR1>(ore[r]);
                        }
                        v[n * n + n + m] = b;
                    }
                    v[n * n + m] = a;
                });
            });
        }
        {
            double *ap = acc + (size_t)slot * SS + pot;
            T tn_ = itau;
            T ca[2 * P], cb[2 * P];
            sfor<0, P>([&](auto nn) {
                constexpr int n = decltype(nn)::value;
                constexpr int Y0 = tn::yoff(n, CH), Y1 = n + 1 < P ? tn::yoff(n + 1, CH) : 0;
                T *x = v + n * n;
                sfor<0, 2 * n + 1>([&](auto ii) { x[decltype(ii)::value] *= tn_; });
                tn_ *= itau;
                turn(nn, x, Y0, [&]() __attribute__((always_inline)) { trigs(nn, cb, tb); });
                zrot(nn, x, cb, (T)-1);
                turn(nn, x, Y1, [&]() __attribute__((always_inline)) { trigs(nn, ca, ta); });
                zrot(nn, x, ca, (T)-1);
                sfor<0, 2 * n + 1>([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    unsafeAtomicAdd(ap + NPOT * (n * n + i), (double)x[i]);
                });
            });
        }
    }
    __syncthreads();
    for (int i = tid; i < nt * 2 * P2; i += tn::NTHR) {
        const int sl = i / (2 * P2), k = i % (2 * P2), po = k / P2, r = k % P2;
        Lc[(size_t)b0 * 2 * P2 + i] = po < NPOT ? (T)(acc[(size_t)sl * SS + NPOT * r + po] * (double)oscale[r]) : (T)0;
    }
}

// targets per tile: as many as the LDS takes (one workgroup per compute unit and wavefront of a SIMD),
// fewer where that would leave compute units without a tile
template <typename T, int P, bool SC>
static void launch(const lhf_plan *Pl, hipStream_t st)
{
    constexpr int NPOT = SC ? 1 : 2, WGS = tn::waves<T, P>();  // workgroups per compute unit
    constexpr size_t fixed = tn::fixed_bytes<T, P, NPOT>(), each = tn::slot_bytes<T, P, NPOT>();
    const int mx = (int)std::min<size_t>(60, (LDS_CU / WGS - fixed) / each);
    int64_t nb = 0;
    for (int l = 2; l <= Pl->depth; l++) nb += Pl->lev[l].nb;
    const int ns = (int)std::max<int64_t>(1, std::min<int64_t>(mx, nb / (512 * WGS)));
    const tn::Levels lv = tn::levels(Pl, ns, mx);
    if (lv.ntiles == 0) return;
    k_m2l_turn<T, P, SC><<<dim3((unsigned)((lv.ntiles + 7) / 8 * 8)), dim3(tn::NTHR), fixed + tn::max_ns(lv) * each, st>>>(
        lv, Pl->bkey, (const T *)Pl->l2pv, (T *)Pl->Lc, (const T *)Pl->ttab, (const T *)Pl->ttrig,
        (const T *)Pl->tscale + P * P, (const tn::Dir *)Pl->tdir);
}

template <typename T, int P>
hipError_t turn_attr()
{
    const int lds = LDS_CU / tn::waves<T, P>();
    const hipError_t e = hipFuncSetAttribute((const void *)k_m2l_turn<T, P, false>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_m2l_turn<T, P, true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

template <typename T, int P>
void turn_launch(const lhf_plan *Pl, bool scalar, hipStream_t st)
{
    if (scalar) launch<T, P, true>(Pl, st);
    else launch<T, P, false>(Pl, st);
}

template hipError_t turn_attr<LHF_TURN_T, LHF_TURN_P>();
template void turn_launch<LHF_TURN_T, LHF_TURN_P>(const lhf_plan *, bool, hipStream_t);

}  // namespace lhf
