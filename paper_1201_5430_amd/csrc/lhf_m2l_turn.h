// lhf_m2l_turn.h -- batched M2L by quarter turns (internal): the kernel and its tables.
//
// The translation along d is rotation / coaxial shift / back-rotation (Sec. 4.4).  The rotation about
// y by the direction's polar angle is taken apart into quarter turns,
//   B(theta) = Z(pi/2) Y Z(pi + theta) Y Z(pi/2),   Y = B(pi/2),
// in an orthonormal real basis (the stored coefficients times c_m (-1)^m N_nm for the S basis, c_m / N_nm
// for the R basis; c_0 = 1, c_m = sqrt 2, N_nm = sqrt((n - m)! (n + m)!)), in which S- and R-basis
// rotations are the same orthogonal matrix.  With a = phi + pi/2 and b = theta + pi the translation is
//   Z(pi - a) Y Z(-b) Y  C  Y Z(b) Y Z(a),
// C the coaxial shift H_nn' = (n + n')! / (N_nm N_n'm) between powers of |d|, column by column in m
// (Z(pi/2) on both sides of the axisymmetric C only leaves (-1)^m, which cancels the S basis' sign).
// Y is one constant matrix per order for every direction, and half of it is zero (Re: m + m' + n odd,
// Im: even), so the two turns that replace a dense rotation cost the same multiplications.  What is
// gained: no table per polar angle, no class order, no barrier between classes, any translation beside
// any other in a batch, and matrix entries that all lanes (or all 16 lanes of a row) use at the same
// time, which therefore need no LDS read per multiplication.  The M2L of every level is one launch.
//
// M2L per execute on MI355X, before (half- and quarter-vector kernels, per-box kernel at other orders)
// and now: 2^20 cube FP64 p = 12 48.0 -> 33.0 ms, FP32 p = 10 23.5 -> 10.2 ms; 4M ring FP64 p = 23
// 381 -> 237 ms, FP64 p = 16 114 -> 76 ms, FP32 p = 16 101 -> 46 ms; 131,101 elements at depth 5, FP64
// p = 13 143 -> 7.4 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "lhf_internal.h"
#include "lhf_m2l_common.h"

namespace lhf {

constexpr int CUS = 256;           // compute units
constexpr size_t LDS_CU = 163840;  // bytes of LDS of one

namespace tn {

// f(I), f(I + 1), .., f(N - 1) with the index as a type: arrays indexed by it stay in registers
template <int I, int N, typename F>
__device__ __attribute__((always_inline)) inline void sfor(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        sfor<I + 1, N>(f);
    }
}

// The non-zero entries of order n's Y, input by input (consecutive entries add into different outputs):
// Re: input m = 0 .. n, outputs m' of the parity of m + n; then Im: input m = 1 .. n, outputs of the other
struct YEnt {
    int out, in;   // places in the order's block [Re 0 .. n | Im 1 .. n]
    bool first;    // first entry of its output
};
__host__ __device__ constexpr int ysize(int n)
{
    int s = 0;
    for (int m = 0; m <= n; m++) s += (n - ((m + n) & 1)) / 2 + 1;
    for (int m = 1; m <= n; m++) {
        const int f = ((m + n + 1) & 1) ? 1 : 2;
        if (f <= n) s += (n - f) / 2 + 1;
    }
    return s;
}
__host__ __device__ constexpr YEnt yent(int n, int e)
{
    for (int m = 0; m <= n; m++) {
        const int f = (m + n) & 1, c = (n - f) / 2 + 1;
        if (e < c) return YEnt{f + 2 * e, m, m < 2};
        e -= c;
    }
    for (int m = 1; m <= n; m++) {
        const int f = ((m + n + 1) & 1) ? 1 : 2, c = f <= n ? (n - f) / 2 + 1 : 0;
        if (e < c) return YEnt{n + f + 2 * e, n + m, m < 3};
        e -= c;
    }
    return YEnt{0, 0, false};
}
// Tables are read in chunks of 128 bytes (two scalar loads); every order's block and every column of the
// coaxial shift starts a chunk
template <typename T>
__host__ __device__ constexpr int chunk() { return 128 / (int)sizeof(T); }
__host__ __device__ constexpr int pad(int k, int c) { return (k + c - 1) / c * c; }
__host__ __device__ constexpr int yoff(int n, int c)
{
    int o = 0;
    for (int k = 0; k < n; k++) o += pad(ysize(k), c);
    return o;
}
// column m of the coaxial shift: inputs n' = m .. p - 1, for each the outputs n = m .. p (order p for the
// conversion of chi)
__host__ __device__ constexpr int hsize(int p, int m) { return (p - m + 1) * (p - m); }
__host__ __device__ constexpr int hoff(int p, int m, int c)
{
    int o = yoff(p, c);
    for (int k = 0; k < m; k++) o += pad(hsize(p, k), c);
    return o;
}
__host__ __device__ constexpr int tab_size(int p, int c) { return hoff(p, p, c); }

constexpr double csqrt(double x)
{
    double r = x > 1.0 ? x : 1.0;
    for (int i = 0; i < 200; i++) {
        const double q = 0.5 * (r + x / r);
        if (q == r) break;
        r = q;
    }
    return r;
}

// a lane's source: p^2 values, padded to whole 16-byte vectors
template <typename T>
__host__ __device__ constexpr int src_stride(int p)
{
    return (p * p + 16 / (int)sizeof(T) - 1) / (16 / (int)sizeof(T)) * (16 / (int)sizeof(T));
}

constexpr int NPHI = 32, NROW = NPHI + 49;  // rows of the angle table: azimuths, then polar angles
__host__ __device__ constexpr int trig_stride(int p) { return p | 1; }
// (cos, sin) pairs of the table where vectors are split over rows: the last pair of orders of an odd p reads
// m = p as well (and multiplies a zero by it), behind the last row's own entries
__host__ __device__ constexpr int trig_pairs(int p) { return NROW * trig_stride(p) + (p & 1); }

// target accumulators: entry k of both potentials side by side, one target every acc_stride entries,
// 2 (1 with a single potential) modulo 32: the lanes of a batch spread over the banks
__host__ __device__ constexpr int acc_stride(int p, int npot) { return (npot * p * p + 31 - npot) / 32 * 32 + npot; }

struct Level {
    int64_t tile0;         // first tile of the level
    int64_t off;           // first box
    int64_t nb;            // boxes
    const int32_t *dmap;   // dense box map
    int ns;                // targets per tile
};
struct Levels {
    Level l[MAXDEPTH + 1];  // in tile order
    int level[MAXDEPTH + 1];
    int n;
    int64_t ntiles;
};

// per direction code: |d|, 1/|d|, the rows of its azimuth and of its polar angle
struct Dir {
    double tau, itau;
    int ia, ib;
};

// one chunk of the table in scalar registers
template <typename T>
struct Chunk {
    typedef T H __attribute__((ext_vector_type(64 / sizeof(T))));
    H a, b;
    template <int I>
    __device__ __attribute__((always_inline)) T at() const
    {
        constexpr int n = 64 / sizeof(T);
        if constexpr (I < n) return a[I];
        else return b[I - n];
    }
};

constexpr int NTHR = 256;

// wavefronts per SIMD the register allocation aims at: a lane holds p^2 values of its translation
template <typename T, int P>
constexpr int waves()
{
    return sizeof(T) == 8 ? (P <= 8 ? 2 : 1) : (P <= 8 ? 4 : P <= 12 ? 2 : 1);
}

// bytes of LDS: the angle table and the spare slot, and what each target adds
template <typename T, int P, int NPOT>
__host__ __device__ constexpr size_t fixed_bytes()
{
    return sizeof(double) * acc_stride(P, NPOT) + sizeof(T) * 2 * NROW * trig_stride(P) + 16;
}
template <typename T, int P, int NPOT>
__host__ __device__ constexpr size_t slot_bytes()
{
    return sizeof(double) * acc_stride(P, NPOT) + VMAX * 6 + 8;
}
// where the arrays of a tile of ns targets begin.  The angle table is read by 16-byte (FP32: 8-byte) vectors,
// so it comes first: behind the accumulators of one potential, an odd number of doubles each, it would begin
// off their alignment
struct Lds {
    size_t trl, acc, esrc, sxyz, ssys, cnt, ecode, end;
};
template <typename T, int P, int NPOT>
__host__ __device__ constexpr Lds lds(int ns)
{
    Lds o{};
    o.trl = 0;
    o.acc = o.trl + sizeof(T) * 2 * NROW * trig_stride(P);
    o.esrc = o.acc + sizeof(double) * (size_t)(ns + 1) * acc_stride(P, NPOT);
    o.sxyz = o.esrc + sizeof(int) * (size_t)VMAX * ns;
    o.ssys = o.sxyz + sizeof(int) * (size_t)ns;
    o.cnt = o.ssys + sizeof(int) * (size_t)ns;
    o.ecode = o.cnt + sizeof(int);
    o.end = o.ecode + sizeof(uint16_t) * (size_t)VMAX * ns;
    return o;
}

// packed coordinates and system of the tile's nt targets
__device__ inline void targets(int64_t b0, int nt, int level, const uint64_t *__restrict__ bkey, int *sxyz, int *ssys,
                               int *cnt, int tid)
{
    if (tid < nt) {
        const uint64_t key = bkey[b0 + tid];
        uint32_t ix = 0, iy = 0, iz = 0;
        for (int b = 0; b < level; b++) {
            ix |= (uint32_t)((key >> (3 * b)) & 1u) << b;
            iy |= (uint32_t)((key >> (3 * b + 1)) & 1u) << b;
            iz |= (uint32_t)((key >> (3 * b + 2)) & 1u) << b;
        }
        sxyz[tid] = (int)(ix | (iy << 10) | (iz << 20));
        ssys[tid] = (int)(key >> (3 * level));
    }
    if (tid == 0) *cnt = 0;
}

// the tile's translations, direction-major: source box and (direction, slot); their number in *cnt
template <int NTH>
__device__ inline void translations(int nt, int side, const int32_t *__restrict__ dmap, const int *sxyz, const int *ssys,
                                    int *cnt, int *esrc, uint16_t *ecode, int tid, int lane)
{
    for (int i0 = 0; i0 < 343 * nt; i0 += NTH) {
        const int i = i0 + tid, dir = i / nt, slot = i % nt;
        int src = -1;
        if (i < 343 * nt) {
            const int dx = dir % 7 - 3, dy = (dir / 7) % 7 - 3, dz = dir / 49 - 3;
            const int xyz = sxyz[slot];
            const int x = xyz & 1023, y = (xyz >> 10) & 1023, z = xyz >> 20;
            const int sx = x - dx, sy = y - dy, sz = z - dz;
            const bool far = dx < -1 || dx > 1 || dy < -1 || dy > 1 || dz < -1 || dz > 1;
            const bool in = sx >= 0 && sy >= 0 && sz >= 0 && sx < side && sy < side && sz < side;
            const int px = (sx >> 1) - (x >> 1), py = (sy >> 1) - (y >> 1), pz = (sz >> 1) - (z >> 1);
            if (far && in && px * px <= 1 && py * py <= 1 && pz * pz <= 1)
                src = dmap[(((size_t)ssys[slot] * side + sz) * side + sy) * side + sx];
        }
        const unsigned long long m = __ballot(src >= 0);
        if (m) {
            int base = 0;
            if (lane == 0) base = atomicAdd(cnt, __popcll(m));
            base = __builtin_amdgcn_readfirstlane(base);
            if (src >= 0) {
                const int k = base + __popcll(m & ((1ull << lane) - 1));
                esrc[k] = src;
                ecode[k] = (uint16_t)(dir * 64 + slot);
            }
        }
    }
}

// tiles of ns consecutive boxes over the levels, the deepest first; a tuned number of targets of a level (at
// most mx) goes before ns
inline Levels levels(const lhf_plan *Pl, int ns, int mx)
{
    Levels lv;
    lv.n = 0;
    lv.ntiles = 0;
    for (int l = Pl->depth; l >= 2; l--) {
        if (Pl->lev[l].nb == 0) continue;
        const int k = Pl->m2l_ns[l] > 0 ? std::min(Pl->m2l_ns[l], mx) : ns;
        lv.l[lv.n] = {lv.ntiles, Pl->lev[l].off, Pl->lev[l].nb, Pl->dmap[l], k};
        lv.level[lv.n++] = l;
        lv.ntiles += (Pl->lev[l].nb + k - 1) / k;
    }
    return lv;
}
inline int max_ns(const Levels &lv)
{
    int m = 0;
    for (int k = 0; k < lv.n; k++) m = std::max(m, lv.l[k].ns);
    return m;
}
}  // namespace tn

// layout of the kernel that splits a vector over the four rows of a wavefront (lhf_m2l_rows_p.hip)
namespace tr {
// entries of order n in one row's class: m = 2j or 2j + 1, j < S(n)
__host__ __device__ constexpr int S(int n) { return n / 2 + 1; }
__host__ __device__ constexpr int hoff(int n)
{
    int o = 0;
    for (int k = 0; k < n; k++) o += S(k);
    return o;
}
// pairs (first, second) of a row: orders 2k, 2k + 1 share k + 1 of them
__host__ __device__ constexpr int nslot(int p) { return ((p + 1) / 2) * ((p + 1) / 2 + 1) / 2; }
// turn tables: order n's S^2 entries, input by input
__host__ __device__ constexpr int yoff(int n)
{
    int o = 0;
    for (int k = 0; k < n; k++) o += S(k) * S(k);
    return o;
}
// column j of the shift: R = p - 2j orders: the symmetric block's diagonals, row p, the factors kappa
__host__ __device__ constexpr int hoff_tab(int p, int j)
{
    int o = 0;
    for (int k = 0; k < j; k++) o += (p - 2 * k) * (p - 2 * k + 1) / 2 + 2 * (p - 2 * k);
    return o;
}
struct Sym {
    int r, c;
};
__host__ __device__ constexpr Sym sym(int R, int k)
{
    int d = 0;
    while (k >= R - d) k -= R - d++;
    return Sym{k, k + d};
}
// entries of one chunk (a 16-byte load of each lane of a row) and table lengths
template <typename T>
__host__ __device__ constexpr int chunk() { return 256 / (int)sizeof(T); }
template <typename T>
__host__ __device__ constexpr int ytab(int p) { return tn::pad(yoff(p), chunk<T>()); }
template <typename T>
__host__ __device__ constexpr int htab(int p) { return tn::pad(hoff_tab(p, (p + 1) / 2), chunk<T>()); }
template <typename T>
__host__ __device__ constexpr int tab_size(int p) { return 4 * ytab<T>(p) + 2 * htab<T>(p); }
// target accumulators: [slot][first, second][row][potential], one target every acc_stride entries
__host__ __device__ constexpr int acc_stride(int p, int npot)
{
    return tn::pad(8 * npot * nslot(p) - 4 * npot, 32) + 4 * npot;
}
// wavefronts per SIMD
template <typename T, int P>
constexpr int waves()
{
    return sizeof(T) == 8 ? (P <= 12 ? 3 : P <= 20 ? 2 : 1) : (P <= 12 ? 4 : 3);
}
template <typename T>
inline size_t fixed_bytes(int p, int npot)
{
    return sizeof(T) * (tab_size<T>(p) + 2 * tn::trig_pairs(p)) + sizeof(double) * acc_stride(p, npot) + 16;
}
inline size_t slot_bytes(int p, int npot) { return sizeof(double) * acc_stride(p, npot) + VMAX * 6 + 8; }
// targets per tile: as many as the LDS holds, fewer where that would leave compute units without a tile
template <typename T>
inline int max_ns(int p, int npot)
{
    return (int)std::min<size_t>(60, (LDS_CU - fixed_bytes<T>(p, npot)) / slot_bytes(p, npot));
}
inline int own_ns(const lhf_plan *Pl, int mx)
{
    int64_t nb = 0;
    for (int l = 2; l <= Pl->depth; l++) nb += Pl->lev[l].nb;
    return (int)std::max<int64_t>(1, std::min<int64_t>(mx, nb / 512));
}
}  // namespace tr

// M2M and L2L in the same split (lhf_mm_rows_p.hip)
namespace tm {
// column j of the shift: R = p - 2j orders: the triangle's diagonals, then a factor per order
__host__ __device__ constexpr int hoff_tab(int p, int j)
{
    int o = 0;
    for (int k = 0; k < j; k++) o += (p - 2 * k) * (p - 2 * k + 1) / 2 + (p - 2 * k);
    return o;
}
template <typename T>
__host__ __device__ constexpr int htab(int p) { return tn::pad(hoff_tab(p, (p + 1) / 2), tr::chunk<T>()); }
// turns, shifts of M2M and of L2L, then the scales into and out of the orthonormal basis for each
template <typename T>
__host__ __device__ constexpr int tab_size(int p) { return 4 * tr::ytab<T>(p) + 4 * htab<T>(p) + 4 * p * p; }
// entries of orders 2k, 2k + 1 (one potential), and the length of a stretch in LDS (odd)
__host__ __device__ constexpr int count(int p, int k) { return 2 * k + 1 < p ? 8 * k + 4 : 4 * k + 1; }
__host__ __device__ constexpr int stretch(int p) { return (8 * ((p + 1) / 2) - 4) | 1; }
// (cos, sin) pairs of the eight octants, m = p of the last one included (as tn::trig_pairs)
__host__ __device__ constexpr int trig_pairs(int p) { return 16 * p + (p & 1); }
// wavefronts per SIMD
template <typename T, int P>
constexpr int waves()
{
    return sizeof(T) == 8 ? (P <= 16 ? 2 : 1) : 2;
}
template <typename T, int P>
__host__ __device__ constexpr size_t bytes()
{
    return sizeof(T) * (4 * tr::ytab<T>(P) + 2 * htab<T>(P) + 2 * trig_pairs(P) + 2 * P * P +
                        4 * (size_t)waves<T, P>() * 16 * stretch(P));
}
}  // namespace tm

// one translation unit per (T, P): the kernels with both potentials and with the scalar one
template <typename T, int P>
hipError_t turn_attr();
template <typename T, int P>
void turn_launch(const lhf_plan *Pl, bool scalar, hipStream_t st);
template <typename T, int P>
hipError_t rows_attr();
template <typename T, int P>
void rows_launch(const lhf_plan *Pl, bool scalar, hipStream_t st);
template <typename T, int P>
hipError_t mm_rows_attr();
template <typename T, int P>
void mm_rows_launch(const lhf_plan *Pl, bool down, int l, hipStream_t st);

}  // namespace lhf
