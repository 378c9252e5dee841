// Four Jacobi steps per pass over memory.
//
// Tiles are boxes of the whole grid, not of one chare: a workgroup's lanes
// cover EX x EY cells of the xy-plane, a ring of four cells included, and
// march z.  Every lane holds kRows rows of one 16-byte vector and computes
// every level (step) on all its cells; the outer cells of the ring go stale
// by one cell a level, and only the cells whose four steps are right are
// written.  A lane finds its cells' chare when it enters a chare along z
// (`locate`), so tiles cross chares freely, at any overdecomposition.
//
// Levels are skewed by one plane: iteration j loads plane j of level 0 and
// finishes plane j - s of level s from
//     S(s-1) = ((((x- + x+) + y-) + y+) + z-)   of plane j - s, kept from the
//                                               iteration before, and
//     z+      = level s-1, plane j - s + 1,     finished just before it.
// After one barrier, S of every level's newest plane is summed: x neighbours
// come from the lanes beside (a row's lanes lie in one wave), y neighbours
// from the lane's own rows, or for a strip's outer rows from LDS, which holds
// only those (two of four rows), twice: one barrier per iteration orders every
// write and read.  Each value is the expression of a single sweep in its
// order, so the result is the same bits.
//
// Bound: a pair of steps per pass is bound by HBM (9.45 bytes per update at
// 512^3 fp64, 5.2 TB/s), so the passes got longer: 4.4 bytes per update here,
// counters included.  64 x 64 cells are what a CU can hold: 128 VGPRs of
// levels per lane at two waves per SIMD in fp64, and 128 KB of LDS for the outer
// rows; fp32 holds two such tiles.  The lanes' overlap computes 1.3 times the
// cells at 512^3.  The pass is now bound by issue (VALU 60-75 % busy) and by
// the latency of the plane loaded ahead; with every load hitting the cache it
// runs 115-120 us per iteration at 512^3 fp64, with the stores too.
//
// Measured, us per iteration, this pass against pairs at the default tile:
// 512^3 fp64 ODF 4096 153 / 270, fp32 76 / 156; 256^3 fp64 22.6 / 39.3; 64^3
// fp64 7.3 / 16.8; 1024^3 fp64 1077 / 2221; 768^3 octree fp64 469 / 1021.  No
// size that the rule (deep_tiles) admits ran slower: (512,512,16) fp32, the
// worst of those tried, 9.8 / 11.0.
#pragma once

#include <hip/hip_runtime.h>

#include "deep.hpp"

namespace od {

constexpr int kRows = 4;      // rows of a lane's strip
constexpr int kEX = 64;       // cells of a row: 32 lanes (fp64) or 16 (fp32)
constexpr int kRing = kDeepSteps + 1;   // planes of boundary values kept in LDS: one per level, one written ahead

template <typename T>
struct DV;
template <>
struct DV<double> {
    typedef double __attribute__((ext_vector_type(2))) t;
    static constexpr int N = 2;
};
template <>
struct DV<float> {
    typedef float __attribute__((ext_vector_type(4))) t;
    static constexpr int N = 4;
};

// s / 6, correctly rounded, in a multiplication and an fma: 1/6 = hi + lo with
// hi the value below 1/6, so fma(s, hi, s * lo) rounds a number within
// 2^-52 ulp of s / 6, and s / 6 is never closer than 1/6 ulp to a rounding
// boundary (s is a multiple of 4 ulps of the quotient, a boundary times 6 an
// odd multiple of 3).  Needs s * lo not to underflow: |s| >= kTiny; smaller sums
// (0 among them) take the division.  Infinities and NaN pass through.
template <typename T>
struct Sixth;
template <>
struct Sixth<double> {
    static constexpr double hi = 0x1.5555555555555p-3, lo = 0x1.5555555555555p-57;
    static constexpr float tiny = 0x1.ep-120f;   // high word of 2^-960
};
template <>
struct Sixth<float> {
    static constexpr float hi = 0x1.555554p-3f, lo = 0x1.555556p-27f, tiny = 0x1p-90f;
};

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
// Smallest of m, |a| and |b| in one instruction; doubles by their high words,
// which order like the doubles when read as floats.  A NaN (a float's, or the
// high word of a double from 2^1017 on) may make the result NaN.
__device__ __forceinline__ float min3_abs(float m, float a, float b) {
    float r;
    asm("v_min3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "v"(m));
    return r;
}
__device__ __forceinline__ float min3_abs(float m, double a, double b) {
    return min3_abs(m, __int_as_float(__double2hiint(a)), __int_as_float(__double2hiint(b)));
}
// larger of m and |v| (a NaN v leaves m)
__device__ __forceinline__ double max_abs(double m, double v) { return __builtin_fmax(m, __builtin_fabs(v)); }
__device__ __forceinline__ float max_abs(float m, float v) { return __builtin_fmaxf(m, __builtin_fabsf(v)); }

// A lane's value from the lane before / after it in the wave (0 shifted in at
// the wave's ends; the ends of a row hold ring or boundary cells).
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kShr1 = 0x138, kShl1 = 0x130;   // whole-wave shift by one lane

// fp64: the same with `alt` in the lanes of `mask`, in the shift's own instruction
// (v_cndmask takes the shift on its first operand).  s_nop: a shift reads its
// operand's lanes two wait states after a VALU write at the earliest; the mask has to be in vcc.
// (512^3 154 against 158 us per iteration with a shift and a select.  In fp32,
// where the addition does the shift, it measured 3 % slower.)
template <int CTRL>
__device__ __forceinline__ double lane_shift_or(double v, double alt, unsigned long long mask) {
    int lo, hi;
    if constexpr (CTRL == kShr1)
        asm("s_mov_b64 vcc, %6\n\ts_nop 1\n\tv_cndmask_b32_dpp %0, %2, %4, vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_cndmask_b32_dpp %1, %3, %5, vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
            : "=&v"(lo), "=v"(hi)
            : "v"(__double2loint(v)), "v"(__double2hiint(v)), "v"(__double2loint(alt)), "v"(__double2hiint(alt)),
              "s"(mask) : "vcc");
    else
        asm("s_mov_b64 vcc, %6\n\ts_nop 1\n\tv_cndmask_b32_dpp %0, %2, %4, vcc wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_cndmask_b32_dpp %1, %3, %5, vcc wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
            : "=&v"(lo), "=v"(hi)
            : "v"(__double2loint(v)), "v"(__double2hiint(v)), "v"(__double2loint(alt)), "v"(__double2hiint(alt)),
              "s"(mask) : "vcc");
    return __hiloint2double(hi, lo);
}

// Chare of a global interior cell from the per-axis index tables.
__device__ __forceinline__ int32_t deep_owner(const DeepMap& m, int ix, int iy, int iz) {
    const int32_t e = (iz * m.k[1] + iy) * m.k[0] + ix;
    return m.owner ? m.owner[e] : e;
}

template <typename T, int NW>
struct Deep {
    using V = typename DV<T>::t;
    static constexpr int VX = DV<T>::N;
    static constexpr int NT = NW * 64;
    static constexpr int EX = kEX, LX = EX / VX;
    static constexpr int NS = NT / LX;            // strips
    static constexpr int EY = NS * kRows;
    static constexpr int SH = 2 * EY + 2 * EX;    // boundary cells of a plane: x-, x+ rows, y-, y+ columns
    static_assert(SH <= NT, "one lane per boundary cell");
    struct Lds {
        T edge[2][kDeepSteps][NS][2][EX];         // [buffer][level][strip][first row, last row]
        T shell[kRing][SH];
        uint32_t dst[NT][kRows], dst_pz[NT][kRows];   // each lane's rows of the plane written next
        T red[NW];
    };
};

// XF: the tile touches the grid's x- face (bit 0), its x+ face (bit 1).
template <typename T, int NW, int XF>
__device__ __forceinline__ T deep_tile(const DeepMap& g, const DeepTile& t, const int parity,
                                       typename Deep<T, NW>::Lds& L, const int hints, const bool want_res) {
    using D = Deep<T, NW>;
    using V = typename D::V;
    constexpr int VX = D::VX, EX = D::EX, EY = D::EY;
    const int tid = threadIdx.x, lx = tid & (D::LX - 1), strip = tid / D::LX;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int xs = t.xs, ys = t.ys, z0 = t.z0, z1 = t.z1;
    const int x = xs + lx * VX, y = ys + strip * kRows;
    constexpr bool xm_face = (XF & 1) != 0, xp_face = (XF & 2) != 0;
    const bool ym_face = ys == 0, yp_face = ys + EY >= ny;
    char* const ab = reinterpret_cast<char*>(g.arena);
    // positions in units of 16 bytes (rows start on 64-byte boundaries and a
    // lane's vector on a multiple of VX cells): 32 bits reach 64 GiB
    auto vec = [&](uint32_t o) -> V* { return reinterpret_cast<V*>(ab + ((uint64_t)o << 4)); };

    // boundary cell of this lane (one of the tile's SH, where the tile
    // touches that face; else a cell of its own is read again)
    int bf = -1, bx = x, by = y;
    if (tid < EY) {
        if (xm_face) bf = 0;
        bx = 0;
        by = ys + tid;
    } else if (tid < 2 * EY) {
        if (xp_face) bf = 1;
        bx = nx - 1;
        by = ys + tid - EY;
    } else if (tid < 2 * EY + EX) {
        if (ym_face) bf = 2;
        bx = xs + tid - 2 * EY;
        by = 0;
    } else if (tid < D::SH) {
        if (yp_face) bf = 3;
        bx = xs + tid - 2 * EY - EX;
        by = ny - 1;
    }

    typedef uint32_t __attribute__((ext_vector_type(4))) U4;
    static_assert(kRows == 4, "a lane's row positions are one vector");
    U4& l_dst = *reinterpret_cast<U4*>(&L.dst[tid][0]);
    U4& l_dst_pz = *reinterpret_cast<U4*>(&L.dst_pz[tid][0]);
    // Positions of the lane's rows in plane q of parity par, and the steps to
    // the next plane, into the lane's l_dst and l_dst_pz.  Entered once per
    // chare along z; one row at a time and through LDS, so that it takes few
    // registers from the loop around it.
    auto locate = [&](int q, int par) {
        const int zc = q < 0 ? 0 : (q >= nz ? nz - 1 : q);
        const int ix = g.ix[x], iz = g.iz[zc];
        const bool in = q >= 0 && q < nz;
#pragma unroll 1
        for (int r = 0; r < kRows; ++r) {
            const int32_t c = deep_owner(g, ix, g.iy[y + r], iz);
            const int32_t* o = g.corigin + 3 * c;
            const BlockDev* B = g.blocks + (in ? c : g.dir_pb[6 * c + (q < 0 ? 4 : 5)]);
            L.dst[tid][r] = (uint32_t)((B->off[par] + (x - o[0]) + (int64_t)(y + r - o[1]) * B->py +
                                        (in ? (int64_t)(q - o[2]) * B->pz : 0)) / VX);
            L.dst_pz[tid][r] = in ? (uint32_t)(B->pz / VX) : 0u;
        }
    };
    U4 src, src_pz;       // the plane loaded next
    const T* bsrc;        // its boundary cell
    uint32_t b_pz;
    auto locate_src = [&](int q) {
        const U4 d = l_dst, d_pz = l_dst_pz;
        locate(q, parity);
        src = l_dst;
        src_pz = l_dst_pz;
        l_dst = d;
        l_dst_pz = d_pz;
        bsrc = reinterpret_cast<const T*>(vec(src[0]));
        b_pz = src_pz[0] * VX;
        if (bf >= 0) {
            const int zc = q < 0 ? 0 : (q >= nz ? nz - 1 : q);
            const int32_t c = deep_owner(g, g.ix[bx], g.iy[by], g.iz[zc]);
            const int32_t* o = g.corigin + 3 * c;
            const BlockDev* B = g.blocks + g.dir_pb[6 * c + bf];
            bsrc = reinterpret_cast<const T*>(ab) + (B->off[parity] + (bf < 2 ? 0 : bx - o[0]) +
                                                     (int64_t)(bf < 2 ? by - o[1] : 0) * B->py +
                                                     (int64_t)(zc - o[2]) * B->pz);
            b_pz = q >= 0 && q < nz ? (uint32_t)B->pz : 0u;
        }
    };
    // first plane behind q's chares (uniform)
    auto next_of = [&](int q) -> int { return q < 0 ? 0 : (q >= nz ? INT32_MAX : g.zn[q]); };
    const bool st_x = x >= t.xo0 && x < t.xo1;
    const int r0 = st_x ? t.yo0 - y : kRows, r1 = t.yo1 - y;   // rows r0 <= r < r1 are written
    const bool x_first = lx == 0, x_last = x + VX == nx;
    const unsigned long long m_first = __ballot(x_first), m_last = __ballot(x_last);

    const int jlo = max(z0 - kDeepSteps, -1), jhi = z1 - 1 + kDeepSteps;
    const int lmax = min(jhi, nz);
    int lq = jlo, lnext = next_of(jlo), dnext = next_of(z0);
    l_dst = l_dst_pz = (U4)0u;
    locate_src(jlo);
    locate(z0, parity ^ 1);

    V F[kRows];   // the plane loaded ahead
    T bv;
    auto load = [&]() {
#pragma unroll
        for (int r = 0; r < kRows; ++r) F[r] = *vec(src[r]);
        bv = *bsrc;
        if (lq < lmax) {
            ++lq;
            if (__builtin_expect(lq == lnext, 0)) {
                lnext = next_of(lq);
                locate_src(lq);
            } else {
                src += src_pz;
                bsrc += b_pz;
            }
        }
    };
    load();

    V U[kDeepSteps][kRows], S[kDeepSteps][kRows];
#pragma unroll
    for (int s = 0; s < kDeepSteps; ++s)
#pragma unroll
        for (int r = 0; r < kRows; ++r) U[s][r] = S[s][r] = (V)(T)1;
    T res = 0;
    const int bslot = tid < D::SH ? tid : 0;

    int slot0 = 0;   // slot of plane j's boundary values
#pragma unroll 1
    for (int j = jlo; j <= jhi; ++j, slot0 = slot0 + 1 == kRing ? 0 : slot0 + 1) {
        const int b = j & 1;
        // finish each level's plane and stage the strips' outer rows
        V N[kDeepSteps + 1][kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) N[0][r] = F[r];
        if (tid < D::SH) L.shell[slot0][bslot] = bv;
        __builtin_amdgcn_sched_barrier(0);
        load();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < kDeepSteps; ++s) {
            *reinterpret_cast<V*>(&L.edge[b][s][strip][0][lx * VX]) = N[s][0];
            *reinterpret_cast<V*>(&L.edge[b][s][strip][1][lx * VX]) = N[s][kRows - 1];
            const int p = j - 1 - s;
            __builtin_amdgcn_sched_barrier(0);
            if (p == -1 || p == nz) {
                // a boundary plane keeps its values
#pragma unroll
                for (int r = 0; r < kRows; ++r) N[s + 1][r] = U[s][r];
            } else {
                V q[kRows];
                float m = __builtin_huge_valf();
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    q[r] = S[s][r] + N[s][r];
#pragma unroll
                    for (int i = 0; i < VX; i += 2) m = min3_abs(m, (T)q[r][i], (T)q[r][i + 1]);
                }
                auto quick = [&]() {
#pragma unroll
                    for (int r = 0; r < kRows; ++r)
#pragma unroll
                        for (int i = 0; i < VX; ++i)
                            N[s + 1][r][i] = fma_((T)q[r][i], Sixth<T>::hi, (T)q[r][i] * Sixth<T>::lo);
                };
                const bool divide = __any(!(m >= Sixth<T>::tiny));
                // (written so that either path leaves its result in place: the other
                // order costs fp64 eight moves a level and fp32 registers)
                if constexpr (sizeof(T) == 8) quick();
                if (__builtin_expect(divide, 0)) {
#pragma unroll
                    for (int r = 0; r < kRows; ++r)
#pragma unroll
                        for (int i = 0; i < VX; ++i) N[s + 1][r][i] = q[r][i] / (T)6;
                } else if constexpr (sizeof(T) == 4) {
                    quick();
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // write the fourth step
        const int p4 = j - kDeepSteps;
        if (p4 >= z0) {
            const U4 d = l_dst;
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                if (r >= r0 && r < r1) {
                    V* o = vec(d[r]);
                    if (hints & 1)
                        __builtin_nontemporal_store(N[kDeepSteps][r], o);
                    else
                        *o = N[kDeepSteps][r];
                }
            if (want_res) {
#pragma unroll
                for (int r = 0; r < kRows; ++r)
                    if (r >= r0 && r < r1) {
#pragma unroll
                        for (int i = 0; i < VX; ++i)
                            res = max_abs(res, (T)(N[kDeepSteps][r][i] - U[kDeepSteps - 1][r][i]));
                    }
            }
            if (p4 + 1 < z1) {
                if (__builtin_expect(p4 + 1 == dnext, 0)) {
                    dnext = next_of(dnext);
                    locate(p4 + 1, parity ^ 1);
                } else {
                    l_dst = d + l_dst_pz;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();

        // S of every level's new plane
#pragma unroll
        for (int s = kDeepSteps - 1; s >= 0; --s) {
            const int slot = slot0 >= s ? slot0 - s : slot0 - s + kRing;
            __builtin_amdgcn_sched_barrier(0);
            const T* ymp = &L.edge[b][s][strip > 0 ? strip - 1 : 0][1][lx * VX];
            const T* ypp = &L.edge[b][s][strip < D::NS - 1 ? strip + 1 : strip][0][lx * VX];
            if (ym_face && strip == 0) ymp = &L.shell[slot][2 * EY + lx * VX];
            if (yp_face && strip == D::NS - 1) ypp = &L.shell[slot][2 * EY + EX + lx * VX];
            const V yme = *reinterpret_cast<const V*>(ymp);
            const V ype = *reinterpret_cast<const V*>(ypp);
            // boundary values beside the row's ends, for the strip's rows
            V bm[kRows / VX], bp[kRows / VX];
#pragma unroll
            for (int q = 0; q < kRows / VX; ++q) {
                // (pinned: read by every lane, with no branch around the read)
                if constexpr (xm_face) {
                    bm[q] = *reinterpret_cast<const V*>(&L.shell[slot][strip * kRows + q * VX]);
                    asm volatile("" : "+v"(bm[q]));
                }
                if constexpr (xp_face) {
                    bp[q] = *reinterpret_cast<const V*>(&L.shell[slot][EY + strip * kRows + q * VX]);
                    asm volatile("" : "+v"(bp[q]));
                }
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const V c = N[s][r];
                T left, right;
                if constexpr (xm_face && sizeof(T) == 8) {
                    left = lane_shift_or<kShr1>(c[VX - 1], bm[r / VX][r % VX], m_first);
                } else {
                    left = lane_shift<kShr1>((T)c[VX - 1]);
                    if constexpr (xm_face) left = x_first ? (T)bm[r / VX][r % VX] : left;
                }
                if constexpr (xp_face && sizeof(T) == 8) {
                    right = lane_shift_or<kShl1>(c[0], bp[r / VX][r % VX], m_last);
                } else {
                    right = lane_shift<kShl1>((T)c[0]);
                    if constexpr (xp_face) right = x_last ? (T)bp[r / VX][r % VX] : right;
                }
                const V ym = r > 0 ? N[s][r > 0 ? r - 1 : 0] : yme;
                const V yp = r < kRows - 1 ? N[s][r < kRows - 1 ? r + 1 : r] : ype;
                V a;
#pragma unroll
                for (int i = 0; i < VX; ++i) {
                    const T xm = i > 0 ? c[i > 0 ? i - 1 : 0] : left;
                    const T xp = i < VX - 1 ? c[i < VX - 1 ? i + 1 : i] : right;
                    T w = xm + xp;
                    w = w + ym[i];
                    w = w + yp[i];
                    w = w + U[s][r][i];
                    a[i] = w;
                }
                S[s][r] = a;
                U[s][r] = c;
            }
        }
    }
    return res;
}

// Waves of a workgroup: 64 x 64 cells either way.  One fp64 workgroup fills a
// CU's registers and LDS, two fp32 ones do.
constexpr int deep_waves(int dtype_bytes) { return dtype_bytes == 8 ? 8 : 4; }
constexpr int deep_per_cu(int dtype_bytes) { return dtype_bytes == 8 ? 1 : 2; }

template <typename T, int NW>
__device__ __forceinline__ T deep_box(const DeepMap& g, const DeepTile& t, int parity, typename Deep<T, NW>::Lds& L,
                                      int hints, bool want_res) {
    const bool m = t.xs == 0, p = t.xs + Deep<T, NW>::EX >= g.n[0];
    return m ? (p ? deep_tile<T, NW, 3>(g, t, parity, L, hints, want_res)
                  : deep_tile<T, NW, 1>(g, t, parity, L, hints, want_res))
             : (p ? deep_tile<T, NW, 2>(g, t, parity, L, hints, want_res)
                  : deep_tile<T, NW, 0>(g, t, parity, L, hints, want_res));
}

}  // namespace od
