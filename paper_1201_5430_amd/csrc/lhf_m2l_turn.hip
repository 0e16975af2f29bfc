// lhf_m2l_turn.hip -- tables, source layout and dispatch of the M2L by quarter turns (its kernels: lhf_m2l_turn_p.hip).
#include "lhf_m2l_turn.h"

namespace lhf {

namespace {

// Y: exact integer sums over binomials.  With U = exp(-pi/2 G) and e(k) = (-1)^k for k > 0, else 1,
// U_mm' = e(m) e(m') d^n_m'm(pi/2),
// d^n_m'm = 2^-n sqrt((n+m')! (n-m')! / ((n+m)! (n-m)!)) sum_s (-1)^(m'-m+s) C(n+m, s) C(n-m, m'-m+s)
__device__ double binom(int n, int k)
{
    if (k < 0 || k > n) return 0.0;
    double b = 1.0;
    for (int i = 1; i <= k; i++) b = b * (double)(n - k + i) / (double)i;  // exact: every product is an integer
    return b;
}
__device__ double fact(int k)
{
    double f = 1.0;
    for (int i = 2; i <= k; i++) f *= (double)i;
    return f;
}
__device__ double quarter(int n, int mp, int m)
{
    double s = 0.0;
    for (int k = max(0, m - mp); k <= min(n + m, n - mp); k++) {
        const double t = binom(n + m, k) * binom(n - m, mp - m + k);
        s += ((mp - m + k) & 1) ? -t : t;
    }
    const double r = sqrt(fact(n + mp) / fact(n + m) * (fact(n - mp) / fact(n - m)));
    return ((m + mp) & 1 ? -1.0 : 1.0) * ldexp(s, -n) * r;
}

__device__ double yval(int n, bool im, int mp, int m)
{
    return (im ? 2.0 : m ? (mp ? 2.0 : sqrt(2.0)) : (mp ? sqrt(2.0) : 1.0)) * quarter(n, mp, m);
}
// (n + n')! / (N_nm N_n'm)
__device__ double hval(int n1, int n2, int m) { return sqrt(binom(n1 + n2, n1 - m)) * sqrt(binom(n1 + n2, n1 + m)); }

// entry t of the table for whole vectors (blocks of the orders' Y, then the columns of the coaxial shift,
// each padded to whole chunks of ch)
__device__ double turn_entry(int p, int ch, int t)
{
    int n = 0, o = t;
    while (n < p && o >= tn::pad(tn::ysize(n), ch)) o -= tn::pad(tn::ysize(n++), ch);
    if (n < p) {
        if (o >= tn::ysize(n)) return 0.0;
        const tn::YEnt y = tn::yent(n, o);
        const bool im = y.in > n;
        return yval(n, im, im ? y.out - n : y.out, im ? y.in - n : y.in);
    }
    int m = 0;
    while (o >= tn::pad(tn::hsize(p, m), ch)) o -= tn::pad(tn::hsize(p, m++), ch);
    if (o >= tn::hsize(p, m)) return 0.0;
    return hval(m + o % (p - m + 1), m + o / (p - m + 1), m);
}

// entry t of the tables for rows: [part][parity of the input] turns of ty entries, [parity] shifts of th
__device__ double rows_entry(int p, int ty, int th, int t)
{
    if (t < 4 * ty) {
        const int part = t / ty >> 1, pin = t / ty & 1;
        int n = 0, o = t % ty;
        while (n < p && o >= tr::S(n) * tr::S(n)) {
            o -= tr::S(n) * tr::S(n);
            n++;
        }
        if (n == p) return 0.0;
        const int m = 2 * (o / tr::S(n)) + pin, mp = 2 * (o % tr::S(n)) + ((pin + n + part) & 1);
        return (m > n || mp > n || (part && (m == 0 || mp == 0))) ? 0.0 : yval(n, part, mp, m);
    }
    const int par = (t - 4 * ty) / th;
    int o = (t - 4 * ty) % th, j = 0;
    for (; 2 * j < p; j++) {
        const int R = p - 2 * j, sz = R * (R + 1) / 2 + 2 * R;
        if (o < sz) break;
        o -= sz;
    }
    if (2 * j >= p) return 0.0;
    const int n0 = 2 * j, R = p - n0, m = n0 + par, q1 = R * (R + 1) / 2;
    if (o < q1) {
        const tr::Sym y = tr::sym(R, o);
        return n0 + y.r < m ? 0.0 : hval(n0 + y.r, n0 + y.c, m);  // r <= c
    }
    o -= q1;
    if (o < R) return n0 + o < m ? 0.0 : hval(p, n0 + o, m);
    const double n1 = (double)(n0 + o - R + 1);
    return sqrt(n1 * n1 - (double)m * m) / n1;
}

// the tables and the scales of the sources and of the targets
template <typename T>
__global__ void k_turn_tab(int p, bool rows, int size, T *__restrict__ tab, T *__restrict__ scale)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < size)
        tab[t] = (T)(rows ? rows_entry(p, tr::ytab<T>(p), tr::htab<T>(p), t) : turn_entry(p, tn::chunk<T>(), t));
    if (t < p * p) {
        int n = (int)sqrtf((float)t);
        while ((n + 1) * (n + 1) <= t) n++;
        while (n * n > t) n--;
        const int i = t - n * n, m = i > n ? i - n : i;
        const double N = sqrt(fact(n - m)) * sqrt(fact(n + m)), c = m ? sqrt(2.0) : 1.0, sg = (m & 1) ? -1.0 : 1.0;
        scale[t] = (T)(sg * c * N);
        scale[p * p + t] = (T)(sg * N / c);
    }
}
// entry t of the M2M and L2L tables (lhf_mm_rows_p.hip): the turns of rows_entry, [M2M, L2L][parity] shifts
// of th entries, [M2M, L2L][into, out of the orthonormal basis] scales.  The distance of child and parent is
// sqrt(3) / 4 of the parent's size, sqrt(3) / 2 of the child's; (-tau)^k / k! are the shift's coefficients
// in the stored basis and 2^-n the ratio of the sizes.
__device__ double mm_entry(int p, int ty, int th, int t)
{
    if (t < 4 * ty) return rows_entry(p, ty, 0, t);
    t -= 4 * ty;
    const double taup = 0.4330127018922193;
    if (t >= 4 * th) {
        t -= 4 * th;
        const int kind = t / (2 * p * p), dir = t / (p * p) & 1, i = t % (p * p);
        int n = (int)sqrtf((float)i);
        while ((n + 1) * (n + 1) <= i) n++;
        while (n * n > i) n--;
        const int r = i - n * n, m = r > n ? r - n : r;
        const double N = sqrt(fact(n - m)) * sqrt(fact(n + m)), c = m ? sqrt(2.0) : 1.0, sg = (m & 1) ? -1.0 : 1.0;
        return kind == 0 ? (dir ? 1.0 / (c * N) : sg * c * N) : (dir ? sg * N / c : c / N);
    }
    const int kind = t / (2 * th), par = t / th & 1;
    int o = t % th, j = 0;
    for (; 2 * j < p; j++) {
        const int R = p - 2 * j, sz = R * (R + 1) / 2 + R;
        if (o < sz) break;
        o -= sz;
    }
    if (2 * j >= p) return 0.0;
    const int n0 = 2 * j, R = p - n0, m = n0 + par, q1 = R * (R + 1) / 2;
    if (o < q1) {
        const tr::Sym y = tr::sym(R, o);
        const int lo = n0 + y.r, hi = n0 + y.c;
        if (lo < m) return 0.0;
        double cf = 1.0;
        for (int k = 1; k <= hi - lo; k++) cf *= -taup / (double)k;
        const double q = sqrt(fact(hi - m) / fact(lo - m)) * sqrt(fact(hi + m) / fact(lo + m));
        return ((m & 1) ? -1.0 : 1.0) * ldexp(cf * q, -lo);
    }
    o -= q1;
    const int n = kind == 0 ? n0 + R - 1 - o : n0 + o + 1;
    if (n < 1 || n < m) return 0.0;
    return (kind == 0 ? taup : -2.0 * taup) * sqrt((double)n * n - (double)m * m) / (double)n;
}
template <typename T>
__global__ void k_mm_tab(int p, int size, T *__restrict__ tab)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < size) tab[t] = (T)mm_entry(p, tr::ytab<T>(p), tm::htab<T>(p), t);
}

// a direction of every row of the angle table (azimuths, then polar angles) and the rows of every
// direction
struct Rows {
    int16_t rep[tn::NROW];
    uint8_t ia[343], ib[343];
};
Rows make_rows()
{
    Rows R;
    int na = 0, nb = 0;
    for (int d = 0; d < 343; d++) {
        const int x = d % 7 - 3, y = (d / 7) % 7 - 3, z = d / 49 - 3, q = x * x + y * y;
        R.ia[d] = R.ib[d] = 0;
        if (q == 0 && z == 0) continue;
        // equal azimuths: parallel (x, y) of one sense (the z axis takes azimuth 0)
        int k = 0;
        for (; k < na; k++) {
            const int e = R.rep[k], ex = e % 7 - 3, ey = (e / 7) % 7 - 3;
            if (q == 0 ? (ey == 0 && ex > 0) : (x * ey == y * ex && x * ex + y * ey > 0)) break;
        }
        if (k == na && q) R.rep[na++] = (int16_t)d;
        R.ia[d] = (uint8_t)k;
        // equal polar angles: one sign of z and one ratio z^2 : x^2 + y^2
        for (k = 0; k < nb; k++) {
            const int e = R.rep[tn::NPHI + k], ex = e % 7 - 3, ey = (e / 7) % 7 - 3, ez = e / 49 - 3;
            if ((z > 0) - (z < 0) == (ez > 0) - (ez < 0) && z * z * (ex * ex + ey * ey) == ez * ez * q) break;
        }
        if (k == nb) R.rep[tn::NPHI + nb++] = (int16_t)d;
        R.ib[d] = (uint8_t)(tn::NPHI + k);
    }
    // the z axis' directions seen before azimuth 0 had its row
    for (int d = 0; d < 343; d++)
        if (d % 7 == 3 && (d / 7) % 7 == 3)
            for (int k = 0; k < na; k++) {
                const int e = R.rep[k], ex = e % 7 - 3, ey = (e / 7) % 7 - 3;
                if (ey == 0 && ex > 0) R.ia[d] = (uint8_t)k;
            }
    return R;
}

// rows of (cos, sin)(m a), m < p: a = phi + pi/2 of the azimuths, a = theta + pi of the polar angles.
// The powers of dx + i dy and dz + i rho are integers (times rho in the imaginary part), so each entry is
// one rounded quotient.
template <typename T>
__global__ void k_turn_trig(int p, Rows R, T *__restrict__ trig, tn::Dir *__restrict__ dirs)
{
    const int r = blockIdx.x, lane = threadIdx.x;
    for (int d = r * 64 + lane; d < 343; d += tn::NROW * 64) {
        const int ex = d % 7 - 3, ey = (d / 7) % 7 - 3, ez = d / 49 - 3;
        const double tau = sqrt((double)(ex * ex + ey * ey + ez * ez));
        dirs[d].tau = tau;
        dirs[d].itau = tau > 0.0 ? 1.0 / tau : 0.0;
        dirs[d].ia = R.ia[d];
        dirs[d].ib = R.ib[d];
    }
    const int rep = R.rep[r], dx = rep % 7 - 3, dy = (rep / 7) % 7 - 3, dz = rep / 49 - 3;
    const int x = r < tn::NPHI ? dx : dz, y = dy, y2 = dx * dx + dy * dy;
    if (lane >= p) return;
    const int m = lane;
    const double xx = x, im2 = r < tn::NPHI ? (double)(y * y) : (double)y2, im1 = r < tn::NPHI ? (double)y : 1.0;
    // (x + i w)^m = A + i w' B with w'^2 = im2 / im1^2
    double A = 1.0, B = 0.0;
    for (int k = 0; k < m; k++) {
        const double a = xx * A - (r < tn::NPHI ? im1 * B : im2 * B), b = (r < tn::NPHI ? im1 * A : A) + xx * B;
        A = a;
        B = b;
    }
    const double n2 = xx * xx + im2;
    double den = 1.0;
    for (int k = 0; k < m / 2; k++) den *= n2;
    double c = A / den, s = (r < tn::NPHI ? B : B * sqrt(im2)) / den;
    if (m & 1) {
        const double q = sqrt(n2);
        c /= q;
        s /= q;
    }
    double co, si;
    if (r < tn::NPHI) {  // times i^m
        const int q = m & 3;
        co = q == 0 ? c : q == 1 ? -s : q == 2 ? -c : s;
        si = q == 0 ? s : q == 1 ? c : q == 2 ? -s : -c;
    } else {  // times (-1)^m
        co = (m & 1) ? -c : c;
        si = (m & 1) ? -s : s;
    }
    trig[(size_t)r * 2 * p + 2 * m] = (T)co;
    trig[(size_t)r * 2 * p + 2 * m + 1] = (T)si;
}

// multipoles of the boxes of levels >= 2 in the orthonormal basis, one potential every sp values
// ... in the row layout: [pair][row][potential](first, second), pair k (k + 1) / 2 + j, row r0 + 2 r1: order
// n = 2k + r0, m = 2j + r1, first = Re and second = Im where r1 = 0, the other way round where r1 = 1
template <typename T, int NPOT>
__global__ void k_rows_src(int64_t off, int64_t nb, int p, int ns, const T *__restrict__ M, const T *__restrict__ scale,
                           T *__restrict__ Ms)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int per = ns * 8 * NPOT;
    if (i >= nb * per) return;
    const int64_t b = off + i / per;
    const int e = (int)(i % per), c = e & 1, po = (e >> 1) % NPOT, row = e / (2 * NPOT) & 3, s = e / (8 * NPOT);
    int k = (int)((sqrtf(8.0f * (float)s + 1.0f) - 1.0f) * 0.5f);
    if ((k + 1) * (k + 2) / 2 <= s) k++;
    if (k * (k + 1) / 2 > s) k--;
    const int n = 2 * k + (row & 1), r1 = row >> 1, m = 2 * (s - k * (k + 1) / 2) + r1, part = c ^ r1;
    const bool ok = n < p && m <= n && !(part && m == 0);
    const int q = ok ? n * n + (part ? n : 0) + m : 0;
    Ms[off * per + i] = ok ? M[(size_t)b * 2 * p * p + po * p * p + q] * scale[q] : (T)0;
}

template <typename T, int NPOT>
__global__ void k_turn_src(int64_t off, int64_t nb, int P2, int sp, const T *__restrict__ M,
                           const T *__restrict__ scale, T *__restrict__ Ms)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nb * NPOT * sp) return;
    const int k = (int)(i % sp);
    const int64_t bp = i / sp;  // box and potential
    const int64_t b = off + bp / NPOT;
    const int po = (int)(bp % NPOT);
    Ms[off * NPOT * sp + i] = k < P2 ? M[(size_t)b * 2 * P2 + po * P2 + k] * scale[k] : (T)0;
}

template <typename T>
bool build_t(lhf_plan *Pl, hipStream_t st)
{
    const int p = Pl->p;
    const int size = Pl->turn_rows ? tr::tab_size<T>(p) : tn::tab_size(p, tn::chunk<T>());
    if (dev_malloc(&Pl->ttab, sizeof(T) * size) != hipSuccess) return false;
    if (dev_malloc(&Pl->tscale, sizeof(T) * 2 * p * p) != hipSuccess) return false;
    if (dev_malloc(&Pl->ttrig, sizeof(T) * 2 * p * tn::NROW) != hipSuccess) return false;
    if (dev_malloc(&Pl->tdir, sizeof(tn::Dir) * 343) != hipSuccess) return false;
    k_turn_tab<T><<<dim3((size + 255) / 256), dim3(256), 0, st>>>(p, Pl->turn_rows, size, (T *)Pl->ttab, (T *)Pl->tscale);
    static const Rows rows = make_rows();
    k_turn_trig<T><<<dim3(tn::NROW), dim3(64), 0, st>>>(p, rows, (T *)Pl->ttrig, (tn::Dir *)Pl->tdir);
    if (Pl->use_mmrows) {
        const int mm = tm::tab_size<T>(p);
        if (dev_malloc(&Pl->mmtab, sizeof(T) * mm) != hipSuccess) return false;
        k_mm_tab<T><<<dim3((mm + 63) / 64), dim3(64), 0, st>>>(p, mm, (T *)Pl->mmtab);
    }
    return true;
}

template <typename T, int NPOT>
void stage_t(const lhf_plan *Pl, hipStream_t st)
{
    const int P2 = Pl->p * Pl->p, e = 16 / (int)sizeof(T), sp = (P2 + e - 1) / e * e;
    const int64_t off = Pl->lev[2].off, nb = Pl->nbox - off;
    if (nb <= 0) return;
    if (Pl->turn_rows) {
        const int ns = tr::nslot(Pl->p);
        k_rows_src<T, NPOT><<<dim3((unsigned)((nb * ns * 8 * NPOT + 255) / 256)), dim3(256), 0, st>>>(
            off, nb, Pl->p, ns, (const T *)Pl->M, (const T *)Pl->tscale, (T *)Pl->l2pv);
        return;
    }
    const int64_t cnt = nb * NPOT * sp;
    k_turn_src<T, NPOT><<<dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st>>>(off, nb, P2, sp, (const T *)Pl->M,
                                                                             (const T *)Pl->tscale, (T *)Pl->l2pv);
}

}  // namespace

// values of the source copy, of the plan's type (it shares the L2P's coefficient buffer)
size_t turn_src_values(const lhf_plan *Pl)
{
    const int P2 = Pl->p * Pl->p, e = 16 / (int)Pl->tsize;
    if (Pl->turn_rows) return (size_t)Pl->nbox * 16 * tr::nslot(Pl->p);
    return (size_t)Pl->nbox * 2 * ((P2 + e - 1) / e * e);
}

// orders built (each a compilation of lhf_m2l_turn_p.hip or lhf_m2l_rows_p.hip: the lists of the build
// script).  Whole vectors per lane as long as they fit a lane's 512 registers: M2L of 5.8 M translations
// (131,101 elements uniform, depth 5) whole against rows, FP64 p = 9 2.3 / 3.8 ms, p = 11 3.5 / 5.4 ms,
// p = 12 4.5 / 5.8 ms, p = 13 (part of the vector in scratch) 8.4 / 6.9 ms; FP32 p = 10 1.5 / 3.4 ms,
// p = 16 6.6 / 8.4 ms.  Below p = 7 the ownership tile keeps its fixed order of sums.
#define LHF_TURN_FP64(F) F(7) F(8) F(9) F(10) F(11) F(12)
#define LHF_ROWS_FP64(F) F(13) F(14) F(15) F(16) F(17) F(18) F(19) F(20) F(21) F(22) F(23) F(24)
#define LHF_TURN_FP32(F) F(7) F(8) F(9) F(10) F(11) F(12) F(13) F(14) F(15) F(16)

// 1: whole vectors, 2: rows, 0: not built
int turn_kind(int precision, int p)
{
#define F(N) \
    if (p == N) return 1;
#define G(N) \
    if (p == N) return 2;
    if (precision == LHF_FP64) {
        LHF_TURN_FP64(F) LHF_ROWS_FP64(G)
    } else {
        LHF_TURN_FP32(F)
    }
#undef F
#undef G
    return 0;
}

bool turn_build(lhf_plan *Pl, hipStream_t st)
{
#define F(N) \
    if (Pl->p == N) return build_t<T>(Pl, st) && turn_attr<T, N>() == hipSuccess && mm_rows_attr<T, N>() == hipSuccess;
#define G(N) \
    if (Pl->p == N) return build_t<T>(Pl, st) && rows_attr<T, N>() == hipSuccess && mm_rows_attr<T, N>() == hipSuccess;
    if (Pl->precision == LHF_FP64) {
        using T = double;
        LHF_TURN_FP64(F) LHF_ROWS_FP64(G)
    } else {
        using T = float;
        LHF_TURN_FP32(F)
    }
#undef F
#undef G
    return false;
}

void turn_stage(const lhf_plan *Pl, bool scalar, hipStream_t st)
{
    if (Pl->precision == LHF_FP64) scalar ? stage_t<double, 1>(Pl, st) : stage_t<double, 2>(Pl, st);
    else scalar ? stage_t<float, 1>(Pl, st) : stage_t<float, 2>(Pl, st);
}

void m2l_turn_launch(const lhf_plan *Pl, bool scalar, hipStream_t st)
{
#define F(N) \
    if (Pl->p == N) return turn_launch<T, N>(Pl, scalar, st);
#define G(N) \
    if (Pl->p == N) return rows_launch<T, N>(Pl, scalar, st);
    if (Pl->precision == LHF_FP64) {
        using T = double;
        LHF_TURN_FP64(F) LHF_ROWS_FP64(G)
    } else {
        using T = float;
        LHF_TURN_FP32(F)
    }
#undef F
#undef G
}

// targets per tile of the rows kernel: the most that it holds, and what it takes unless told otherwise
int turn_max_ns(const lhf_plan *Pl)
{
    return Pl->precision == LHF_FP64 ? tr::max_ns<double>(Pl->p, 2) : tr::max_ns<float>(Pl->p, 2);
}
int turn_own_ns(const lhf_plan *Pl) { return tr::own_ns(Pl, turn_max_ns(Pl)); }

// M2M into the boxes of level l (down: L2L into them, added to what they hold)
void mm_rows(const lhf_plan *Pl, bool down, int l, hipStream_t st)
{
#define F(N) \
    if (Pl->p == N) return mm_rows_launch<T, N>(Pl, down, l, st);
    if (Pl->precision == LHF_FP64) {
        using T = double;
        LHF_TURN_FP64(F) LHF_ROWS_FP64(F)
    } else {
        using T = float;
        LHF_TURN_FP32(F)
    }
#undef F
}

}  // namespace lhf
