// Eight Jacobi steps per pass of the 2D 5-point stencil (rows of the (x, z)
// plane of an (nx, 1, nz) grid).
//
// One wave per box, and nothing between waves: a lane holds 32 bytes of a row
// (4 cells fp64, 8 fp32), the wave a stretch of 64 lanes with a ring of eight
// cells at either end, and marches the rows.  Levels (steps) are skewed by one
// row as in deep_dev.hpp: iteration j loads row j and finishes row j - s of
// level s from S = (x- + x+) + z- of that row, kept from the iteration before,
// and z+ finished just before it.  x neighbours come from the lanes beside by
// lane shifts: no LDS, no barrier.  s / 4 is the same bits as s * 0.25.
//
// Bound: HBM, as pairs were (8192^2 fp64: 109-128 us per iteration at 8 bytes per
// update); eight steps move 2 bytes per update.  Sixteen would take 256 VGPRs of
// levels.  Rows are loaded three ahead, into registers of their own (the loop is
// written out three times), as two waves per SIMD are what the levels leave
// room for.
//
// Measured, us per iteration, against pairs with a tuned tile: 8192^2 fp64 ODF 64
// 32.5 / 109 (4.3 TB/s), fp32 18.3 / 66, 32768^2 fp64 531 / 1749, 1000^2 ODF 16
// 4.4 / 7.6, 256^2 2.1 / 4.3.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "deep_dev.hpp"

namespace od {

namespace {

constexpr int kSteps = kDeep2dSteps, kAhead = 3;

template <typename T>
struct Row {
    static constexpr int N = 32 / (int)sizeof(T);
    T v[N];
};

// XF: the box touches the grid's x- or x+ face: lanes before the first and
// behind the last group hold the face's value and keep it.  RAG: some groups
// are not full.
template <typename T, bool XF, bool RAG>
__device__ __forceinline__ T deep2d_box(const DeepMap& g, const DeepTile& t, const int parity, const int hints,
                                        const bool want_res) {
    using V = typename DV<T>::t;
    constexpr int VX = DV<T>::N, N = Row<T>::N;
    const int lane = threadIdx.x, nz = g.nz, z0 = t.z0, z1 = t.z1;
    // (ws is -1 in a box at the x- face: its first lane is that face)
    const int w = t.ws + lane, wc = min(max(w, 0), g.nv - 1), x = g.vx[wc];
    const int nv = RAG ? g.vx[wc + 1] - x : N;
    const bool fixed = XF && (w < 0 || w >= g.nv);
    T* const arena = reinterpret_cast<T*>(g.arena);
    const T* src;
    const T* bsrc;
    int64_t src_pz, b_pz;
    auto chare = [&](int q) { return deep_owner(g, g.vi[wc], g.iy[0], g.iz[q < 0 ? 0 : (q >= nz ? nz - 1 : q)]); };
    auto locate_src = [&](int q) {
        const int32_t c = chare(q);
        const int32_t* o = g.corigin + 3 * c;
        const bool in = q >= 0 && q < nz;
        const BlockDev* B = g.blocks + (in ? c : g.dir_pb[6 * c + (q < 0 ? 4 : 5)]);
        src = arena + B->off[parity] + (x - o[0]) + (in ? (int64_t)(q - o[2]) * B->pz : 0);
        src_pz = in ? B->pz : 0;
        bsrc = src;
        b_pz = src_pz;
        if (fixed) {
            const BlockDev* F = g.blocks + g.dir_pb[6 * c + (w < 0 ? 0 : 1)];
            bsrc = arena + F->off[parity] + (in ? (int64_t)(q - o[2]) * F->pz : 0);
            b_pz = in ? F->pz : 0;
        }
    };
    T* dst;
    int64_t dst_pz;
    auto locate_dst = [&](int q) {
        const int32_t c = chare(q);
        const int32_t* o = g.corigin + 3 * c;
        const BlockDev* B = g.blocks + c;
        dst = arena + B->off[parity ^ 1] + (x - o[0]) + (int64_t)(q - o[2]) * B->pz;
        dst_pz = B->pz;
    };
    auto next_of = [&](int q) -> int { return q < 0 ? 0 : (q >= nz ? INT32_MAX : g.zn[q]); };
    const bool st = w >= t.wo0 && w < t.wo1;
    const int jlo = max(z0 - kSteps, -1), jhi = z1 - 1 + kSteps, lmax = min(jhi, nz);
    int lq = jlo, lnext = next_of(jlo), dnext = next_of(z0);
    locate_src(jlo);
    locate_dst(z0);

    struct Ahead {
        V a, b;
        T f;
    };
    auto load = [&](Ahead& F) {
        F.a = *reinterpret_cast<const V*>(src);
        F.b = *reinterpret_cast<const V*>(src + VX);
        if constexpr (XF) F.f = *bsrc;
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
    Row<T> U[kSteps], S[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
        for (int i = 0; i < N; ++i) U[s].v[i] = S[s].v[i] = 0;
    T res = 0;
    auto step = [&](int j, Ahead& F) {
        Row<T> L[kSteps + 1];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            L[0].v[i] = i < VX ? F.a[i < VX ? i : 0] : F.b[i < VX ? 0 : i - VX];
            if constexpr (XF) L[0].v[i] = fixed ? F.f : L[0].v[i];
        }
        load(F);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int p = j - 1 - s;
            if (p == -1 || p == nz) {   // a boundary row keeps its values
                L[s + 1] = U[s];
            } else {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const T v = (S[s].v[i] + L[s].v[i]) * (T)0.25;
                    L[s + 1].v[i] = XF && fixed ? U[s].v[i] : v;
                }
            }
        }
        const int p = j - kSteps;
        if (p >= z0 && p < z1) {
            if (st) {
                V a, b;
#pragma unroll
                for (int i = 0; i < VX; ++i) {
                    a[i] = L[kSteps].v[i];
                    b[i] = L[kSteps].v[VX + i];
                }
                V* o = reinterpret_cast<V*>(dst);
                if (hints & 1) {
                    __builtin_nontemporal_store(a, o);
                    if (!RAG || nv > VX) __builtin_nontemporal_store(b, o + 1);
                } else {
                    o[0] = a;
                    if (!RAG || nv > VX) o[1] = b;
                }
                if (want_res)
#pragma unroll
                    for (int i = 0; i < N; ++i)
                        if (!RAG || i < nv) res = max_abs(res, L[kSteps].v[i] - U[kSteps - 1].v[i]);
            }
            if (p + 1 < z1) {
                if (__builtin_expect(p + 1 == dnext, 0)) {
                    dnext = next_of(dnext);
                    locate_dst(p + 1);
                } else {
                    dst += dst_pz;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            T tail = L[s].v[N - 1];
            if constexpr (RAG) {
#pragma unroll
                for (int i = 0; i < N - 1; ++i) tail = nv == i + 1 ? L[s].v[i] : tail;
            }
            const T left = lane_shift<kShr1>(tail), right = lane_shift<kShl1>(L[s].v[0]);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const T xm = i > 0 ? L[s].v[i > 0 ? i - 1 : 0] : left;
                T xp = i < N - 1 ? L[s].v[i < N - 1 ? i + 1 : i] : right;
                if constexpr (RAG) xp = i < N - 1 && i + 1 >= nv ? right : xp;
                T a = xm + xp;
                a = a + U[s].v[i];
                S[s].v[i] = a;
            }
            U[s] = L[s];
        }
    };
    static_assert(kAhead == 3, "the loop is written out for three rows ahead");
    Ahead F0, F1, F2;
    load(F0);
    load(F1);
    load(F2);
#pragma unroll 1
    for (int j = jlo; j <= jhi; j += kAhead) {
        step(j, F0);
        step(j + 1, F1);   // (up to two rows past jhi: nothing is written there)
        step(j + 2, F2);
    }
    return res;
}

template <typename T, bool RAG>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_deep2d(DeepMap g, const DeepTile* __restrict__ tiles, int parity, unsigned long long* __restrict__ res, int zero_lo,
         int zero_hi, int hints, int want_res) {
    if (blockIdx.x == 0)
        for (int s = zero_lo + (int)threadIdx.x; s < zero_hi; s += 64) res[2 * s + parity] = 0ull;
    const DeepTile& t = tiles[blockIdx.x];
    T r = t.ws < 0 || t.ws + 64 > g.nv ? deep2d_box<T, true, RAG>(g, t, parity, hints, want_res != 0)
                                       : deep2d_box<T, false, RAG>(g, t, parity, hints, want_res != 0);
    if (!want_res) return;
    for (int off = 32; off > 0; off >>= 1) {
        const T o = __shfl_xor(r, off, 64);
        r = o > r ? o : r;
    }
    if (threadIdx.x == 0) atomicMax(&res[parity ^ 1], (unsigned long long)__double_as_longlong((double)r));
}

}  // namespace

DeepPlan deep_plan2d(const Plan& p, int dtype_bytes) {
    DeepPlan d;
    const int32_t N = 32 / dtype_bytes;
    if (!p.regular) return d;
    for (int32_t i = 0; i < p.k[0]; ++i)
        for (int32_t x = p.split[0][(size_t)i]; x < p.split[0][(size_t)i + 1]; x += N) {
            d.ragged = d.ragged || x + N > p.split[0][(size_t)i + 1];
            d.vx.push_back(x);
            d.vi.push_back(i);
        }
    const int32_t nv = (int32_t)d.vx.size();
    d.vx.push_back((int32_t)p.n[0]);
    d.rows = 0;
    // stretches of 64 groups: a box begins far enough before what it writes that
    // eight cells lie between, or at the face (lane 0 is the face then)
    struct Cut {
        int32_t s, o0, o1;
    };
    std::vector<Cut> cx;
    auto cells = [&](int32_t w) { return d.vx[(size_t)w]; };
    for (int32_t o = 0; o < nv;) {
        int32_t s = o;
        while (s > 0 && cells(o) - cells(s) < kSteps) --s;
        if (s == 0) s = -1;
        int32_t e = std::min(nv, s + 64);
        if (s + 64 <= nv)   // the last lane is not the x+ face
            while (e > o && cells(s + 64) - cells(e) < kSteps) --e;
        if (e <= o) return DeepPlan{};
        cx.push_back({s, o, e});
        o = e;
    }
    // z: as few row iterations as fill two waves a SIMD, a piece of l rows taking l + 16
    int64_t best = INT64_MAX, zc = 1;
    const int64_t xs = (int64_t)cx.size(), slots = 256 * 4 * 2;
    for (int64_t k = 1; k <= std::min<int64_t>(p.n[2], 4 * slots); ++k) {
        const int64_t len = (p.n[2] + k - 1) / k, cost = ((xs * k + slots - 1) / slots) * (len + 2 * kSteps);
        if (cost < best) {
            best = cost;
            zc = k;
        }
    }
    std::vector<DeepTile> list;
    for (int64_t k = 0; k < zc; ++k)
        for (const Cut& a : cx)
            list.push_back({a.s, 0, a.o0, a.o1, 0, 1, (int32_t)(p.n[2] * k / zc), (int32_t)(p.n[2] * (k + 1) / zc)});
    d.tiles = xcd_runs(list);
    return d;
}

hipError_t launch_deep2d(int dtype_bytes, const DeepPlan& d, hipStream_t st, const DeepMap& g, const DeepTile* tiles,
                         int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                         bool want_res) {
    if (d.tiles.empty()) return hipErrorInvalidValue;
    const unsigned n = (unsigned)d.tiles.size();
#define OD_LAUNCH(T, RAG)                                                                                       \
    if (dtype_bytes == (int)sizeof(T) && d.ragged == RAG) {                                                     \
        hipLaunchKernelGGL((k_deep2d<T, RAG>), dim3(n), dim3(64), 0, st, g, tiles, parity, res, zero_lo,        \
                           zero_hi, hints, want_res ? 1 : 0);                                                   \
        return hipGetLastError();                                                                               \
    }
    OD_LAUNCH(double, false)
    OD_LAUNCH(double, true)
    OD_LAUNCH(float, false)
    OD_LAUNCH(float, true)
#undef OD_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace od
