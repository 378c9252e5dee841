// Four Jacobi steps per pass over memory.
//
// Tiles are boxes of the whole grid, not of one chare: a workgroup's lanes
// cover EX x EY cells of the xy-plane, a ring of four cells included, and
// march z.  Every lane holds R rows of one 16-byte vector and computes
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
// 512^3 fp64, 5.2 TB/s), so the passes got longer: 4.5 bytes per update here,
// counters included.  64 x 64 cells are what a CU can hold: 128 VGPRs of
// levels per lane at two waves per SIMD in fp64, and 128 KB of LDS for the outer
// rows; fp32 holds two such tiles.  The lanes' overlap computes 1.3 times the
// cells at 512^3.  The pass is now bound by issue (VALU active in 57 % of the busy
// cycles in fp64, 76 % in fp32; 19 and 15 VALU instructions per update) and by the
// latency of the plane loaded ahead (waves wait 35 % of theirs, two to a SIMD).
// Four rows spill 16-24 bytes of scratch per lane in fp64 and 68-100 in fp32
// (the cooperative forms 136-236, whose loops around the pass hold more), one
// row none (message-driven 12-20).
//
// Sums too small for the quick division (Sixth, below), zeros among them, send a
// wave's level through true divisions.  A field of zeros with one hot face, 512^3, us
// per iteration against U[0,1) and against pairs from the same start: fp64 182 /
// 155 / 263, fp32 118 / 80 / 165.
//
// One row a strip (R = 1) makes a box of 16 rows whose iterations are shorter:
// what small grids, which wait for one box's planes, are quicker with.
//
// Measured, us per iteration, this pass against pairs at the default tile:
// 512^3 fp64 ODF 4096 153 / 270, fp32 76 / 156; 256^3 fp64 22.6 / 39.3; 64^3
// fp64 5.1 / 16.8; 1024^3 fp64 1077 / 2221; 768^3 octree fp64 469 / 1021;
// 211 x 163 x 157 fp32 in 27 chares, whose rows end inside vectors, 10.1 / 28.
// (512,512,16) fp32 9.8 / 11.0.  Thin grids, whose lanes lie mostly outside the
// grid, can be slower: where that is estimated the grid runs by tiles (deep.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "deep.hpp"

namespace od {

constexpr int deep_waves(int dtype_bytes) { return dtype_bytes == 8 ? 8 : 4; }   // of a workgroup
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
// which order like the doubles when read as floats.  The high word of a double
// from 2^1017 on reads as a NaN, signalling up to 2^1021: v_min3 would make that
// a quiet one and then drop it with the value beside it, however small that is,
// so doubles take v_minimum3, whose result stays a NaN (and the wave divides).
// Sums of floats hold quiet NaNs only, which v_min3 leaves out.
__device__ __forceinline__ float min3_abs(float m, float a, float b) {
    float r;
    asm("v_min3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "v"(m));
    return r;
}
__device__ __forceinline__ float min3_abs(float m, double a, double b) {
    float r;
    asm("v_minimum3_f32 %0, |%1|, |%2|, %3"
        : "=v"(r) : "v"(__int_as_float(__double2hiint(a))), "v"(__int_as_float(__double2hiint(b))), "v"(m));
    return r;
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

// A strip's R boundary values; pinned: read by every lane, with no branch
// around the read.
template <typename T, int R>
__device__ __forceinline__ void shell_rows(T (&v)[R], const T* p) {
    using V = typename DV<T>::t;
    constexpr int VX = DV<T>::N;
    if constexpr (R % VX == 0) {
#pragma unroll
        for (int q = 0; q < R / VX; ++q) {
            V t = *reinterpret_cast<const V*>(p + q * VX);
            asm volatile("" : "+v"(t));
#pragma unroll
            for (int i = 0; i < VX; ++i) v[q * VX + i] = t[i];
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = p[r];
            asm volatile("" : "+v"(v[r]));
        }
    }
}

// Chare of a global interior cell from the per-axis index tables.
__device__ __forceinline__ int32_t deep_owner(const DeepMap& m, int ix, int iy, int iz) {
    const int32_t e = (iz * m.k[1] + iy) * m.k[0] + ix;
    return m.owner ? m.owner[e] : e;
}

// R rows a strip, W waves a workgroup.
template <typename T, int R, int W = deep_waves((int)sizeof(T))>
struct Deep {
    using V = typename DV<T>::t;
    static constexpr int VX = DV<T>::N;
    static constexpr int NW = W, NT = NW * 64;
    static constexpr int EX = kEX, LX = EX / VX;
    static constexpr int NS = NT / LX;            // strips of R rows
    static constexpr int EY = NS * R;
    static constexpr int RE = R > 1 ? 2 : 1;      // outer rows of a strip
    static constexpr int SH = 2 * EY + 2 * EX;    // boundary cells of a plane: x-, x+ rows, y-, y+ columns
    static_assert(SH <= NT, "one lane per boundary cell");
    struct Lds {
        T edge[2][kDeepSteps][NS][RE][EX];        // [buffer][level][strip][first row, last row]
        T shell[kRing][SH];
        uint32_t dst[NT][R], dst_pz[NT][R];       // each lane's rows of the plane written next
        T red[NW];
    };
};

// R: rows of a lane's strip.  XF: the tile touches the grid's x- face (bit 0),
// its x+ face (bit 1).  RAG: some vectors are not full (a chare's row, or the
// grid's, ends inside them): the cells beside their end come from the lane after.
// ST: steps of the pass (one of four at most).  skip (uniform): that many fewer;
// the first levels copy, so that the last step is still the last level's.
template <typename T, int R, int XF, bool RAG, int W, int ST = kDeepSteps>
__device__ __forceinline__ T deep_tile(const DeepMap& g, const DeepTile& t, const int parity,
                                       typename Deep<T, R, W>::Lds& L, const int hints, const bool want_res,
                                       const int skip) {
    using D = Deep<T, R, W>;
    using V = typename D::V;
    constexpr int VX = D::VX, EX = D::EX, EY = D::EY;
    const int tid = threadIdx.x, lx = tid & (D::LX - 1), strip = tid / D::LX;
    const int nv_all = g.nv, ny = g.ny, nz = g.nz;
    const int ws = t.ws, ys = t.ys, z0 = t.z0, z1 = t.z1;
    // lanes behind the row's last vector read that again and write nothing
    const int w = ws + lx, wc = min(w, nv_all - 1), x = g.vx[wc], y = ys + strip * R;
    const int nv = RAG ? g.vx[wc + 1] - x : VX;   // cells of the lane's vector
    constexpr bool xm_face = (XF & 1) != 0, xp_face = (XF & 2) != 0;
    const bool ym_face = ys == 0, yp_face = ys + EY >= ny;
    char* const ab = reinterpret_cast<char*>(g.arena);
    // positions in units of 16 bytes (rows start on 64-byte boundaries and a
    // lane's vector on a multiple of VX cells): 32 bits reach 64 GiB
    auto vec = [&](uint32_t o) -> V* { return reinterpret_cast<V*>(ab + ((uint64_t)o << 4)); };

    // boundary cell of this lane (one of the tile's SH, where the tile
    // touches that face; else a cell of its own is read again)
    int bf = -1, bw = wc, bi = 0, by = min(y, ny - 1);   // face, vector, cell in it, row
    if (tid < EY) {
        if (xm_face) bf = 0;
        bw = 0;
        by = min(ys + tid, ny - 1);
    } else if (tid < 2 * EY) {
        if (xp_face) bf = 1;
        bw = nv_all - 1;
        by = min(ys + tid - EY, ny - 1);
    } else if (tid < D::SH) {
        const int k = tid - 2 * EY, c = k < EX ? k : k - EX;
        if (k < EX ? ym_face : yp_face) bf = k < EX ? 2 : 3;
        bw = min(ws + c / VX, nv_all - 1);
        bi = min(c % VX, g.vx[bw + 1] - g.vx[bw] - 1);
        by = k < EX ? 0 : ny - 1;
    }

    // Positions of the lane's rows in plane q of parity par, and the steps to
    // the next plane, into the lane's L.dst and L.dst_pz.  Entered once per
    // chare along z; one row at a time and through LDS, so that it takes few
    // registers from the loop around it.
    auto locate = [&](int q, int par) {
        const int zc = q < 0 ? 0 : (q >= nz ? nz - 1 : q);
        const int ix = g.vi[wc], iz = g.iz[zc];
        const bool in = q >= 0 && q < nz;
#pragma unroll 1
        for (int r = 0; r < R; ++r) {
            const int yr = min(y + r, ny - 1);
            const int32_t c = deep_owner(g, ix, g.iy[yr], iz);
            const int32_t* o = g.corigin + 3 * c;
            const BlockDev* B = g.blocks + (in ? c : g.dir_pb[6 * c + (q < 0 ? 4 : 5)]);
            L.dst[tid][r] = (uint32_t)((B->off[par] + (x - o[0]) + (int64_t)(yr - o[1]) * B->py +
                                        (in ? (int64_t)(q - o[2]) * B->pz : 0)) / VX);
            L.dst_pz[tid][r] = in ? (uint32_t)(B->pz / VX) : 0u;
        }
    };
    uint32_t src[R], src_pz[R];   // the plane loaded next
    const T* bsrc;                // its boundary cell
    uint32_t b_pz;
    auto locate_src = [&](int q) {
        uint32_t d[R], d_pz[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            d[r] = L.dst[tid][r];
            d_pz[r] = L.dst_pz[tid][r];
        }
        locate(q, parity);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            src[r] = L.dst[tid][r];
            src_pz[r] = L.dst_pz[tid][r];
            L.dst[tid][r] = d[r];
            L.dst_pz[tid][r] = d_pz[r];
        }
        bsrc = reinterpret_cast<const T*>(vec(src[0]));
        b_pz = src_pz[0] * VX;
        if (bf >= 0) {
            const int zc = q < 0 ? 0 : (q >= nz ? nz - 1 : q);
            const int bx = g.vx[bw] + bi;
            const int32_t c = deep_owner(g, g.vi[bw], g.iy[by], g.iz[zc]);
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
    const bool st_x = w >= t.wo0 && w < t.wo1;
    const int r0 = st_x ? t.yo0 - y : R, r1 = t.yo1 - y;   // rows r0 <= r < r1 are written
    const bool x_first = w == 0, x_last = w == nv_all - 1, y_first = ym_face && strip == 0, y_last = y + R == ny;
    const unsigned long long m_first = __ballot(x_first), m_last = __ballot(x_last);

    const int jlo = max(z0 - ST, -1), jhi = z1 - 1 + ST;
    const int lmax = min(jhi, nz);
    int lq = jlo, lnext = next_of(jlo), dnext = next_of(z0);
#pragma unroll
    for (int r = 0; r < R; ++r) L.dst[tid][r] = L.dst_pz[tid][r] = 0u;
    locate_src(jlo);
    locate(z0, parity ^ 1);

    V F[R];   // the plane loaded ahead
    T bv;
    auto load = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r) F[r] = *vec(src[r]);
        bv = *bsrc;
        if (lq < lmax) {
            ++lq;
            if (__builtin_expect(lq == lnext, 0)) {
                lnext = next_of(lq);
                locate_src(lq);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) src[r] += src_pz[r];
                bsrc += b_pz;
            }
        }
    };
    load();

    V U[ST][R], S[ST][R];
#pragma unroll
    for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) U[s][r] = S[s][r] = (V)(T)1;
    T res = 0;
    const int bslot = tid < D::SH ? tid : 0;

    int slot0 = 0;   // slot of plane j's boundary values
#pragma unroll 1
    for (int j = jlo; j <= jhi; ++j, slot0 = slot0 + 1 == kRing ? 0 : slot0 + 1) {
        const int b = j & 1;
        // finish each level's plane and stage the strips' outer rows
        V N[ST + 1][R];
#pragma unroll
        for (int r = 0; r < R; ++r) N[0][r] = F[r];
        if (tid < D::SH) L.shell[slot0][bslot] = bv;
        __builtin_amdgcn_sched_barrier(0);
        load();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            *reinterpret_cast<V*>(&L.edge[b][s][strip][0][lx * VX]) = N[s][0];
            if constexpr (R > 1) *reinterpret_cast<V*>(&L.edge[b][s][strip][1][lx * VX]) = N[s][R - 1];
            const int p = j - 1 - s;
            __builtin_amdgcn_sched_barrier(0);
            if (p == -1 || p == nz || s < skip) {
                // a boundary plane keeps its values
#pragma unroll
                for (int r = 0; r < R; ++r) N[s + 1][r] = U[s][r];
            } else {
                V q[R];
                float m = __builtin_huge_valf();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    q[r] = S[s][r] + N[s][r];
#pragma unroll
                    for (int i = 0; i < VX; i += 2) m = min3_abs(m, (T)q[r][i], (T)q[r][i + 1]);
                }
                auto quick = [&]() {
#pragma unroll
                    for (int r = 0; r < R; ++r)
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
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int i = 0; i < VX; ++i) N[s + 1][r][i] = q[r][i] / (T)6;
                } else if constexpr (sizeof(T) == 4) {
                    quick();
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // write the fourth step
        const int p4 = j - ST;
        if (p4 >= z0) {
            uint32_t d[R];
#pragma unroll
            for (int r = 0; r < R; ++r) d[r] = L.dst[tid][r];
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r >= r0 && r < r1) {
                    V* o = vec(d[r]);
                    if (hints & 1)
                        __builtin_nontemporal_store(N[ST][r], o);
                    else
                        *o = N[ST][r];
                }
            if (want_res) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r >= r0 && r < r1) {
#pragma unroll
                        for (int i = 0; i < VX; ++i)
                            if (!RAG || i < nv) res = max_abs(res, (T)(N[ST][r][i] - U[ST - 1][r][i]));
                    }
            }
            if (p4 + 1 < z1) {
                if (__builtin_expect(p4 + 1 == dnext, 0)) {
                    dnext = next_of(dnext);
                    locate(p4 + 1, parity ^ 1);
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) L.dst[tid][r] = d[r] + L.dst_pz[tid][r];
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();

        // S of every level's new plane
#pragma unroll
        for (int s = ST - 1; s >= 0; --s) {
            const int slot = slot0 >= s ? slot0 - s : slot0 - s + kRing;
            __builtin_amdgcn_sched_barrier(0);
            const T* ymp = &L.edge[b][s][strip > 0 ? strip - 1 : 0][D::RE - 1][lx * VX];
            const T* ypp = &L.edge[b][s][strip < D::NS - 1 ? strip + 1 : strip][0][lx * VX];
            if (y_first) ymp = &L.shell[slot][2 * EY + lx * VX];
            if (y_last) ypp = &L.shell[slot][2 * EY + EX + lx * VX];
            const V yme = *reinterpret_cast<const V*>(ymp);
            const V ype = *reinterpret_cast<const V*>(ypp);
            // boundary values beside the row's ends, for the strip's rows
            T bm[R], bp[R];
            if constexpr (xm_face) shell_rows(bm, &L.shell[slot][strip * R]);
            if constexpr (xp_face) shell_rows(bp, &L.shell[slot][EY + strip * R]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const V c = N[s][r];
                // the row's last cell in this lane, what the lane after reads
                T tail = c[VX - 1];
                if constexpr (RAG) {
#pragma unroll
                    for (int i = 0; i < VX - 1; ++i) tail = nv == i + 1 ? (T)c[i] : tail;
                }
                T left, right;
                if constexpr (xm_face && sizeof(T) == 8) {
                    left = lane_shift_or<kShr1>(tail, bm[r], m_first);
                } else {
                    left = lane_shift<kShr1>(tail);
                    if constexpr (xm_face) left = x_first ? bm[r] : left;
                }
                if constexpr (xp_face && sizeof(T) == 8) {
                    right = lane_shift_or<kShl1>(c[0], bp[r], m_last);
                } else {
                    right = lane_shift<kShl1>((T)c[0]);
                    if constexpr (xp_face) right = x_last ? bp[r] : right;
                }
                const V ym = r > 0 ? N[s][r > 0 ? r - 1 : 0] : yme;
                const V yp = r < R - 1 ? N[s][r < R - 1 ? r + 1 : r] : ype;
                V a;
#pragma unroll
                for (int i = 0; i < VX; ++i) {
                    const T xm = i > 0 ? c[i > 0 ? i - 1 : 0] : left;
                    T xp = i < VX - 1 ? c[i < VX - 1 ? i + 1 : i] : right;
                    if constexpr (RAG) xp = i < VX - 1 && i + 1 >= nv ? right : xp;
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

// Occupancy the kernels are compiled for: the levels of four rows take half of
// a SIMD's registers per wave, of one row a quarter of that.
#define OD_DEEP_OCC(R) __attribute__((amdgpu_waves_per_eu(R == 1 ? 4 : 2, R == 1 ? 4 : 2)))
#define OD_DEEP_VARIANTS(X)                                                                  \
    X(double, 4, false) X(double, 4, true) X(double, 1, false) X(double, 1, true)            \
    X(float, 4, false) X(float, 4, true) X(float, 1, false) X(float, 1, true)

template <typename T, int R, bool RAG, int W = deep_waves((int)sizeof(T))>
__device__ __forceinline__ T deep_box(const DeepMap& g, const DeepTile& t, int parity,
                                      typename Deep<T, R, W>::Lds& L, int hints, bool want_res, int skip = 0) {
    const bool m = t.ws == 0, p = t.ws + Deep<T, R, W>::LX >= g.nv;
    return m ? (p ? deep_tile<T, R, 3, RAG, W>(g, t, parity, L, hints, want_res, skip)
                  : deep_tile<T, R, 1, RAG, W>(g, t, parity, L, hints, want_res, skip))
             : (p ? deep_tile<T, R, 2, RAG, W>(g, t, parity, L, hints, want_res, skip)
                  : deep_tile<T, R, 0, RAG, W>(g, t, parity, L, hints, want_res, skip));
}

}  // namespace od
