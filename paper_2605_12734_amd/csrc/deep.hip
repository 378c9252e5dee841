// The four-step pass as a launch of its own (deep_dev.hpp has the pass), its
// boxes, and the rule that admits a grid.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <map>

#include "deep_dev.hpp"

namespace od {

namespace {

template <typename T, int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_deep(DeepMap g, const DeepTile* __restrict__ tiles, int parity, unsigned long long* __restrict__ res, int zero_lo,
       int zero_hi, int hints, int want_res) {
    using D = Deep<T, NW>;
    __shared__ __align__(16) typename D::Lds L;
    if (blockIdx.x == 0)
        for (int s = zero_lo + (int)threadIdx.x; s < zero_hi; s += D::NT) res[2 * s + parity] = 0ull;
    const DeepTile& t = tiles[blockIdx.x];
    T r = deep_box<T, NW>(g, t, parity, L, hints, want_res != 0);
    if (!want_res) return;
    for (int off = 32; off > 0; off >>= 1) {
        const T o = __shfl_xor(r, off, 64);
        r = o > r ? o : r;
    }
    if ((threadIdx.x & 63) == 0) L.red[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        T m = L.red[0];
        for (int w = 1; w < NW; ++w) m = L.red[w] > m ? L.red[w] : m;
        atomicMax(&res[parity ^ 1], (unsigned long long)__double_as_longlong((double)m));
    }
}

struct Cut {
    int32_t start, o0, o1;
};

// Tiles of one axis of n cells: lanes cover e cells from `start`, a multiple
// of vx, and write [o0, o1).  At the grid's faces no ring is needed.
std::vector<Cut> cut_axis(int64_t n, int32_t e, int32_t vx, int32_t align) {
    std::vector<Cut> out;
    const int64_t first = e - kDeepSteps, mid = e - 2 * kDeepSteps;
    if (n < e) return out;
    if (n == e) {
        out.push_back({0, 0, (int32_t)n});
        return out;
    }
    int64_t m = 2;
    if (n > 2 * first) m = 2 + (n - 2 * first + mid - 1) / mid;
    std::vector<int64_t> o((size_t)m + 1, 0);
    o[(size_t)m] = n;
    for (int64_t i = 1; i < m; ++i) {
        // what the tiles before can reach, and what those behind must cover
        const int64_t hi = i == 1 ? first : o[(size_t)i - 1] + mid;
        int64_t lo = n - first - (m - 1 - i) * mid;
        lo = (std::max<int64_t>(lo, o[(size_t)i - 1] + 1) + vx - 1) / vx * vx;
        int64_t v = n * i / m / align * align;
        if (v < lo || v > hi) v = std::min(std::max(v, lo), hi) / align * align;
        if (v < lo || v > hi) v = hi / vx * vx;
        if (v < lo || v > hi) return {};
        o[(size_t)i] = v;
    }
    for (int64_t i = 0; i < m; ++i) {
        int64_t s = i == 0 ? 0 : o[(size_t)i] - kDeepSteps;
        const int64_t top = (n - e + vx - 1) / vx * vx;
        s = i == m - 1 ? top : std::min(std::max<int64_t>(s, 0), top);
        out.push_back({(int32_t)s, (int32_t)o[(size_t)i], (int32_t)o[(size_t)i + 1]});
    }
    return out;
}

}  // namespace

void deep_shape(int dtype_bytes, int* ex, int* ey) {
    *ex = kEX;
    *ey = deep_waves(dtype_bytes) * 64 / (kEX * dtype_bytes / 16) * kRows;
}

std::vector<DeepTile> deep_tiles(const Plan& p, int dtype_bytes) {
    std::vector<DeepTile> out;
    int ex, ey;
    deep_shape(dtype_bytes, &ex, &ey);
    const int32_t vx = 16 / dtype_bytes;
    if (p.multires || p.n[0] < ex || p.n[0] % vx != 0 || p.n[1] < ey || p.n[2] < 1) return out;
    for (const Chare& c : p.chares) {
        if (c.u[0] % vx != 0) return out;   // a lane's vector lies in one chare
        // plane steps are 32-bit byte counts
        if ((int64_t)(c.e[0] + 16) * c.e[1] * dtype_bytes > INT32_MAX) return out;
    }
    const std::vector<Cut> cx = cut_axis(p.n[0], ex, vx, 64 / dtype_bytes), cy = cut_axis(p.n[1], ey, 1, 1);
    if (cx.empty() || cy.empty()) return out;
    // z: as many pieces as fill the chip's 256 CUs in the fewest plane
    // iterations, a piece of l planes taking l + 8
    const int64_t xy = (int64_t)cx.size() * (int64_t)cy.size(), slots = 256 * deep_per_cu(dtype_bytes);
    int64_t best = INT64_MAX, zc = 1;
    for (int64_t k = 1; k <= p.n[2]; ++k) {
        const int64_t len = (p.n[2] + k - 1) / k, cost = ((xy * k + slots - 1) / slots) * (len + 2 * kDeepSteps);
        if (cost < best) {
            best = cost;
            zc = k;
        }
    }
    std::vector<DeepTile> list;
    for (int64_t k = 0; k < zc; ++k)
        for (const Cut& b : cy)
            for (const Cut& a : cx)
                list.push_back({a.start, b.start, a.o0, a.o1, b.o0, b.o1, (int32_t)(p.n[2] * k / zc),
                                (int32_t)(p.n[2] * (k + 1) / zc)});
    // workgroup w runs on XCD w % 8: give each XCD a contiguous run
    const size_t N = list.size();
    out.reserve(N);
    std::vector<size_t> at(kNumXcd), end(kNumXcd);
    for (size_t g = 0, o = 0; g < (size_t)kNumXcd; ++g) {
        const size_t cnt = N / kNumXcd + (g < N % kNumXcd ? 1 : 0);
        at[g] = o;
        end[g] = o += cnt;
    }
    for (size_t i = 0; out.size() < N; ++i) {
        const size_t g = i % kNumXcd;
        if (at[g] < end[g]) out.push_back(list[at[g]++]);
    }
    return out;
}

void deep_deps(const std::vector<DeepTile>& t, int dtype_bytes, std::vector<int32_t>& ptr, std::vector<int32_t>& idx) {
    int ex, ey;
    deep_shape(dtype_bytes, &ex, &ey);
    auto reads = [&](const DeepTile& a, const DeepTile& b) {
        return b.xo0 < a.xs + ex && a.xs < b.xo1 && b.yo0 < a.ys + ey && a.ys < b.yo1 && b.z0 < a.z1 + kDeepSteps &&
               a.z0 - kDeepSteps < b.z1;
    };
    // boxes by their place on each axis; along an axis only cuts whose lanes and
    // written cells together meet can be related
    struct Span {
        int32_t lo, hi;
    };
    std::array<std::map<int32_t, Span>, 3> cuts;   // first written cell -> reach
    auto first = [](const DeepTile& b, int d) { return d == 0 ? b.xo0 : (d == 1 ? b.yo0 : b.z0); };
    std::map<std::array<int32_t, 3>, int32_t> at;
    for (size_t i = 0; i < t.size(); ++i) {
        const DeepTile& b = t[i];
        cuts[0][b.xo0] = {std::min(b.xs, b.xo0), std::max(b.xs + ex, b.xo1)};
        cuts[1][b.yo0] = {std::min(b.ys, b.yo0), std::max(b.ys + ey, b.yo1)};
        cuts[2][b.z0] = {b.z0 - kDeepSteps, b.z1 + kDeepSteps};
        at[{b.xo0, b.yo0, b.z0}] = (int32_t)i;
    }
    std::array<std::map<int32_t, std::vector<int32_t>>, 3> near;
    for (size_t d = 0; d < 3; ++d)
        for (const auto& a : cuts[d])
            for (const auto& b : cuts[d])
                if (a.second.lo < b.second.hi && b.second.lo < a.second.hi) near[d][a.first].push_back(b.first);
    ptr.assign(t.size() + 1, 0);
    idx.clear();
    for (size_t i = 0; i < t.size(); ++i) {
        const size_t lo = idx.size();
        for (int32_t z : near[2][first(t[i], 2)])
            for (int32_t y : near[1][first(t[i], 1)])
                for (int32_t x : near[0][first(t[i], 0)]) {
                    const int32_t k = at[{x, y, z}];
                    if (k != (int32_t)i && (reads(t[i], t[(size_t)k]) || reads(t[(size_t)k], t[i]))) idx.push_back(k);
                }
        std::sort(idx.begin() + (std::ptrdiff_t)lo, idx.end());
        ptr[i + 1] = (int32_t)idx.size();
    }
}

hipError_t launch_deep(int dtype_bytes, hipStream_t st, const DeepMap& g, const DeepTile* tiles, int32_t ntiles,
                       int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                       bool want_res) {
    if (ntiles <= 0) return hipErrorInvalidValue;
    if (dtype_bytes == 8)
        hipLaunchKernelGGL((k_deep<double, deep_waves(8)>), dim3((unsigned)ntiles), dim3(deep_waves(8) * 64), 0, st, g,
                           tiles, parity, res, zero_lo, zero_hi, hints, want_res ? 1 : 0);
    else
        hipLaunchKernelGGL((k_deep<float, deep_waves(4)>), dim3((unsigned)ntiles), dim3(deep_waves(4) * 64), 0, st, g,
                           tiles, parity, res, zero_lo, zero_hi, hints, want_res ? 1 : 0);
    return hipGetLastError();
}

}  // namespace od
