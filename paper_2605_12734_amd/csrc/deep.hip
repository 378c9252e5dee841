// The four-step pass as a launch of its own (deep_dev.hpp has the pass), its
// boxes, and the rule that admits a grid.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <map>

#include "deep_dev.hpp"

namespace od {

namespace {

// A plane iteration of a full chip, in units of 10 ns: measured over cubes from
// 64^3 to 512^3 as 2.5 (four rows) and 1.55 us (one) in fp64, 3.2 and 1.65 us in
// fp32, whose CUs hold twice the workgroups.  us per iteration with four / one
// rows: fp64 64^3 7.4 / 5.1, 128^3 9.9 / 9.0, 160^3 10.5 / 11.6, 256^3 22.6 / 34.7;
// fp32 64^3 6.4 / 3.6, 192^3 11.1 / 10.5, 224^3 11.8 / 13.0, 512^3 89 / 115.
int64_t plane_cost(int dtype_bytes, int rows) {
    return dtype_bytes == 8 ? (rows == 1 ? 155 : 250) : (rows == 1 ? 165 : 325);
}

// What a task of the message-driven scheduler adds to its pass, in the same
// units: queueing it and counting its finish for up to 26 others goes through
// few words per XCD; and a box of four rows a strip starts more slowly.  us per
// iteration with nothing added and so: fp32 300 x 300 x 4 11.8 / 5.2 (888 and 222
// boxes; pairs 8.1), 250 x 250 x 12 13.9 / 8.6 (pairs 11.9), 225 x 391 x 6 9.3 / 7.5
// (pairs 8.3), 128^3 14.0 / 12.2, 64^3 7.1 / 5.7; fp64 64^3 7.7 / 6.0, 512^3 the same
// boxes.  Twice as much in fp64 took 237 x 747 x 6 from 11.2 to 14.3, a start-up of
// 6 us for four rows 140^3 from 11.6 (252 boxes) to 12.1 (510 of one row).
int64_t task_cost(int dtype_bytes) { return dtype_bytes == 8 ? 1 : 2; }
constexpr int64_t kTaskRows = 200;

template <typename T, int R, bool RAG>
__global__ void __launch_bounds__(deep_waves((int)sizeof(T)) * 64) OD_DEEP_OCC(R)
k_deep(DeepMap g, const DeepTile* __restrict__ tiles, int parity, unsigned long long* __restrict__ res, int zero_lo,
       int zero_hi, int hints, int want_res) {
    using D = Deep<T, R>;
    __shared__ __align__(16) typename D::Lds L;
    if (blockIdx.x == 0)
        for (int s = zero_lo + (int)threadIdx.x; s < zero_hi; s += D::NT) res[2 * s + parity] = 0ull;
    T r = deep_box<T, R, RAG>(g, tiles[blockIdx.x], parity, L, hints, want_res != 0);
    if (!want_res) return;
    for (int off = 32; off > 0; off >>= 1) {
        const T o = __shfl_xor(r, off, 64);
        r = o > r ? o : r;
    }
    if ((threadIdx.x & 63) == 0) L.red[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        T m = L.red[0];
        for (int w = 1; w < D::NW; ++w) m = L.red[w] > m ? L.red[w] : m;
        atomicMax(&res[parity ^ 1], (unsigned long long)__double_as_longlong((double)m));
    }
}

// Workgroups a CU holds: registers and LDS at four rows a strip (128 VGPRs of
// levels), LDS at one.
int per_cu(int dtype_bytes, int rows) { return (dtype_bytes == 8 ? 1 : 2) * (rows == 1 ? 2 : 1); }

// Planes a box reads beyond what it writes, on either side: passes of more than
// one step march as four do (the levels not needed copy).
int32_t pass_planes(int32_t ring) { return ring == 1 ? 1 : kDeepSteps; }

// Planes of a served solve's box at least: fewer make a solve alone quicker and
// leave less of a shared chip to the others, each box computing eight more.  ms
// for 600 iterations checked every 10, without a least / 8 / 12 / 16 planes: 16
// solves of 32-48 cells an edge 42 / 11.7 / 12.0 / 13.8, of 32-256 120 / 80 / 75 / 70;
// fp64 64^3 alone 7.2 / 10.7 / 13.4 / 14.6, 128^3 10.4 / 10.9 / 12.4 / 14.5.
// A solve checked at every one to three iterations has passes of as many steps,
// whose boxes need a ring of no more cells; with one step they may also be cut finer
// in a tiny solve.  ms for 200 iterations checked at each, by tiles / with a ring of
// four and 8 planes / so: 64 solves of 32-64 cells an edge 37 / 43 / 37, of 48-100 79 / 88 /
// 78, 32 of 64-256 198 / 192 / 179; fp64 alone 8^3 2.5 / 3.9 / 3.3, 16^3 3.1 / 3.9 / 3.3,
// 64^3 6.9 / 6.0 / 6.7, 200^3 14.1 / 10.4 / 10.4.  At every second: 64 of 32-48 30.9 /
// 29.0 / 25.3, of 48-100 64.1 / 67.9 / 66.8, 8^3 alone 2.4 / 3.0 / 3.1.
int64_t serve_planes(int32_t ring, int64_t n) {
    return ring > 1 ? 8 : (n <= 24 ? std::max<int64_t>(4, n / 4) : 10);
}

struct Cut {
    int32_t start, o0, o1;
};

// Boxes along an axis of n items (vectors, or rows) of which the lanes cover L:
// item i holds cells(i + 1) - cells(i) cells.  A box writes [o0, o1) from the
// lanes [start, start + L); between what it writes and lanes with more grid
// behind them lie at least `ring` cells.
template <typename Cells>
std::vector<Cut> cut_axis(int32_t n, int32_t L, int32_t ring, Cells cells) {
    auto left = [&](int32_t o) {   // first lane needed to write from o on
        int32_t s = o;
        while (s > 0 && cells(o) - cells(s) < ring) --s;
        return s;
    };
    auto right = [&](int32_t s) {   // items a box that starts at s can write up to
        if (s + L >= n) return n;
        int32_t o = s + L;
        while (o > s && cells(s + L) - cells(o) < ring) --o;
        return o;
    };
    auto build = [&](int32_t most) {   // boxes of at most `most` items each
        std::vector<Cut> out;
        for (int32_t o = 0; o < n;) {
            int32_t s = left(o);
            int32_t e = std::min(right(s), std::min(n, o + most));
            if (e <= o) return std::vector<Cut>{};
            if (e == n) s = std::max(0, std::min(s, n - L));
            out.push_back({s, o, e});
            o = e;
        }
        return out;
    };
    std::vector<Cut> out = build(n);
    if (out.size() < 2) return out;
    // as many boxes, as even as their reach allows
    const size_t m = out.size();
    for (int32_t most = (n + (int32_t)m - 1) / (int32_t)m; most < n; ++most) {
        std::vector<Cut> even = build(most);
        if (even.size() == m) return even;
    }
    return out;
}

}  // namespace

void deep_shape(int dtype_bytes, const DeepPlan& d, int* lx, int* ey) {
    *lx = kEX * dtype_bytes / 16;
    *ey = d.waves * 64 / *lx * d.rows;
}

std::vector<DeepTile> xcd_runs(const std::vector<DeepTile>& list) {
    std::vector<DeepTile> out;
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

namespace {

DeepPlan plan_boxes(const Plan& p, int dtype_bytes, bool serve, bool tasks, int32_t ring, int64_t* pass_cost) {
    DeepPlan out;
    const int32_t VX = 16 / dtype_bytes;
    if (p.multires || p.chares.empty()) return out;
    for (const Chare& c : p.chares)   // plane steps are 32-bit byte counts
        if ((int64_t)(c.e[0] + 16) * c.e[1] * dtype_bytes > INT32_MAX) return out;
    // vectors along x: every chare's row begins one (explicit blocks begin on
    // multiples of a vector)
    DeepPlan d;
    if (p.regular) {
        for (int32_t i = 0; i < p.k[0]; ++i)
            for (int32_t x = p.split[0][(size_t)i]; x < p.split[0][(size_t)i + 1]; x += VX) {
                d.ragged = d.ragged || x + VX > p.split[0][(size_t)i + 1];
                d.vx.push_back(x);
                d.vi.push_back(i);
            }
    } else {
        for (int32_t x = 0; x < p.n[0]; x += VX) {
            d.ragged = d.ragged || x + VX > p.n[0];
            d.vx.push_back(x);
            d.vi.push_back(x / p.gran);
        }
    }
    const int32_t nv = (int32_t)d.vx.size();
    d.vx.push_back((int32_t)p.n[0]);
    std::vector<Cut> cx, cy;
    int64_t best = INT64_MAX, zc = 1;
    d.waves = serve ? kServeWaves : deep_waves(dtype_bytes);
    for (int rows : {serve && dtype_bytes == 4 ? 2 : 4, 1}) {
        if (serve && best != INT64_MAX) continue;   // solves share the chip: the boxes of least work
        int lx, ey;
        DeepPlan shape;
        shape.rows = rows;
        shape.waves = d.waves;
        deep_shape(dtype_bytes, shape, &lx, &ey);
        if (rows > 1 && p.n[1] < ey) continue;   // the last row ends a strip
        const std::vector<Cut> ax = cut_axis(nv, lx, ring, [&](int32_t i) { return d.vx[(size_t)i]; }),
                               ay = cut_axis((int32_t)p.n[1], ey, ring, [](int32_t i) { return i; });
        if (ax.empty() || ay.empty()) continue;
        // z: as many pieces as fill the chip's 256 CUs in the fewest plane
        // iterations, a piece of l planes taking l + 8
        const int64_t xy = (int64_t)ax.size() * (int64_t)ay.size(),
                      slots = 256 * (serve ? 1 : per_cu(dtype_bytes, rows));
        for (int64_t k = 1; k <= p.n[2] && (!serve || xy * k <= kServeBoxes); ++k) {
            const int64_t len = (p.n[2] + k - 1) / k;
            if (serve && k > 1 && len < serve_planes(ring, p.n[2])) break;
            const int64_t cost = ((xy * k + slots - 1) / slots) * (len + 2 * pass_planes(ring)) * plane_cost(dtype_bytes, rows) +
                                 (tasks ? xy * k * task_cost(dtype_bytes) + (rows > 1 ? kTaskRows : 0) : 0);
            if (cost < best) {
                best = cost;
                zc = k;
                d.rows = rows;
                cx = ax;
                cy = ay;
            }
        }
    }
    if (best == INT64_MAX) return out;
    std::vector<DeepTile> list;
    for (int64_t k = 0; k < zc; ++k)
        for (const Cut& b : cy)
            for (const Cut& a : cx)
                list.push_back({a.start, b.start, a.o0, a.o1, b.o0, b.o1, (int32_t)(p.n[2] * k / zc),
                                (int32_t)(p.n[2] * (k + 1) / zc)});
    d.tiles = xcd_runs(list);
    if (pass_cost) *pass_cost = best;
    return d;
}

// Thin grids, whose boxes are mostly lanes outside the grid (three quarters at
// least): four steps by passes of the planned tiles, `steps` steps a pass, are
// estimated to take no longer than a pass over the boxes (`cost`, in units of
// 10 ns).  tile_time: a tile's march of tz planes takes lat * (tz + 2) and a start-up; a full
// chip's tiles go through at `rate` per plane, start-up counted as ten planes,
// more the more of a tile's row is cells (measured over 1 to 8000 cells an axis).
// us per iteration by boxes / by tiles, fused: fp64 (1,2000,2000) 223 / 170,
// (16,2000,2000) 195 / 184 but (32,2000,2000) 195 / 230 and (8,300,300) 12.2 / 17.4;
// (8000,1,8000) 716 / 415 but (1000,1,1000) 18 / 52, whose 64 tiles leave most of the
// chip idle; (1,1,100000) 85 / 67; fp32 (8000,1,8000) 397 / 212, (4,8000,2000)
// 423 / 384.  Of 600 random grids with an axis of 1 to 40, in all forms, boxes cost
// 13 more than 5 % and half a microsecond without the rule, 1 with it.
double tile_time(const Plan& p, int dtype_bytes, od_exec exec, double full) {
    int32_t ex = 1, ez = 1;
    for (const Chare& c : p.chares) {
        ex = std::max(ex, c.e[0]);
        ez = std::max(ez, c.e[2]);
    }
    const double f = std::min(1.0, (double)ex / p.tile[0]), tz = std::min(p.tile[2], ez), n = (double)p.tiles.size() / 256;
    const bool f64 = dtype_bytes == 8, row = p.tile[1] == 1;
    const double lat = row ? (f64 ? 0.8 : 1.13) * (tz + 6) : 4.8 + (f64 ? 1.0 : 1.25) * (tz + 2);
    const double rate = row ? (f64 ? 0.15 + 0.33 * f : 0.19 + 0.18 * f) : (f64 ? 0.24 : 0.29) + full * f;
    // (the cooperative forms' barrier or queue, per pass over the tiles)
    const double coop = row ? (exec == OD_FUSED || exec == OD_GRAPH ? 1.0 : 1.08)
                            : (exec == OD_PERSISTENT ? 1.13 : (exec == OD_MSGDRIVEN ? (f64 ? 1.25 : 1.5) : 1.0));
    return coop * std::max(lat, n * (tz + 10) * rate);
}

bool tiles_quicker(const Plan& p, int dtype_bytes, const DeepPlan& d, int64_t cost, od_exec exec, int steps) {
    int lx, ey;
    deep_shape(dtype_bytes, d, &lx, &ey);
    if (cost < 4000) return false;   // 40 us a pass: either is mostly start-up
    if (4 * std::min<int64_t>(p.n[0], kEX) * std::min<int64_t>(p.n[1], ey) > (int64_t)kEX * ey) return false;
    // (rows of one cache line or less: the boxes were 5-25 % over the estimate)
    const double boxes = (double)cost * (p.n[0] * dtype_bytes <= 64 ? 1.1 : 1.0);
    return 100.0 * kDeepSteps / steps * tile_time(p, dtype_bytes, exec, dtype_bytes == 8 ? 0.11 : 0.12) <= boxes;
}

}  // namespace

DeepPlan deep_plan(const Plan& p, int dtype_bytes, od_exec exec, int tile_steps) {
    int64_t cost = 0;
    DeepPlan d = plan_boxes(p, dtype_bytes, false, exec == OD_MSGDRIVEN, kDeepSteps, &cost);
    if (d.tiles.empty()) return d;
    d.by_tiles = tiles_quicker(p, dtype_bytes, d, cost, exec, tile_steps);
    if (exec == OD_MSGDRIVEN) {
        // Short counts.  us of od_iterate(n) and the residual, by pairs / by boxes
        // and pairs for the rest: fp64 128^3 (495 boxes) n = 4 157 / 198, 8 236 / 244, 12
        // 317 / 286, 6 197 / 291, 10 277 / 338; 64^3 (224) 4 140 / 113, 6 176 / 196, 10 250 /
        // 220; 256^3 (250), whose launches of tiles start slowly, 4 407 / 209, 6 501 /
        // 496; fp32 128^3 (720) 4 164 / 220, 8 255 / 260, 12 349 / 304; 256^3 4 265 / 220, 6
        // 325 / 403, 10 440 / 481.
        // A launch of tiles takes about 60 us and 0.16 for each of up to 1250 tiles to
        // start, one of boxes 55 and 0.18.
        const double pass = tile_time(p, dtype_bytes, OD_FUSED, dtype_bytes == 8 ? 0.34 : 0.41);
        const double slow = std::min(0.16 * (double)p.tiles.size(), 200.0);
        d.gain = std::max(1.0, pass * kDeepSteps / tile_steps - 0.01 * (double)(cost - (d.rows > 1 ? kTaskRows : 0)));
        d.start = 0.18 * (double)d.tiles.size() - 5 - slow;
        d.rest = 45 + slow;
    }
    return d;
}
DeepPlan deep_plan_serve(const Plan& p, int dtype_bytes, int ring) {
    return plan_boxes(p, dtype_bytes, true, false, ring, nullptr);
}

std::vector<int32_t> deep_tables(const Plan& p, const DeepPlan& d, size_t at[5]) {
    std::vector<int32_t> tab(d.vx);
    at[0] = 0;
    at[1] = tab.size();
    tab.insert(tab.end(), d.vi.begin(), d.vi.end());
    for (int q = 1; q < 3; ++q) {
        at[q + 1] = tab.size();
        for (int64_t v = 0, i = 0; v < p.n[q]; ++v) {
            if (p.regular)
                while (v >= p.split[q][(size_t)i + 1]) ++i;
            tab.push_back((int32_t)(p.regular ? i : v / p.gran));
        }
    }
    at[4] = tab.size();
    tab.resize(at[4] + (size_t)p.n[2]);
    for (int64_t v = p.n[2] - 1; v >= 0; --v) {
        const bool same = v + 1 < p.n[2] && tab[at[3] + (size_t)v + 1] == tab[at[3] + (size_t)v];
        tab[at[4] + (size_t)v] = same ? tab[at[4] + (size_t)v + 1] : (int32_t)(v + 1);
    }
    return tab;
}

void deep_deps(const DeepPlan& d, int dtype_bytes, std::vector<int32_t>& ptr, std::vector<int32_t>& idx, int ring) {
    const int32_t steps = pass_planes(ring);
    const std::vector<DeepTile>& t = d.tiles;
    int ex, ey;
    deep_shape(dtype_bytes, d, &ex, &ey);
    auto reads = [&](const DeepTile& a, const DeepTile& b) {
        return b.wo0 < a.ws + ex && a.ws < b.wo1 && b.yo0 < a.ys + ey && a.ys < b.yo1 && b.z0 < a.z1 + steps &&
               a.z0 - steps < b.z1;
    };
    // boxes by their place on each axis; along an axis only cuts whose lanes and
    // written cells together meet can be related
    struct Span {
        int32_t lo, hi;
    };
    std::array<std::map<int32_t, Span>, 3> cuts;   // first written cell -> reach
    auto first = [](const DeepTile& b, int q) { return q == 0 ? b.wo0 : (q == 1 ? b.yo0 : b.z0); };
    std::map<std::array<int32_t, 3>, int32_t> at;
    for (size_t i = 0; i < t.size(); ++i) {
        const DeepTile& b = t[i];
        cuts[0][b.wo0] = {std::min(b.ws, b.wo0), std::max(b.ws + ex, b.wo1)};
        cuts[1][b.yo0] = {std::min(b.ys, b.yo0), std::max(b.ys + ey, b.yo1)};
        cuts[2][b.z0] = {b.z0 - steps, b.z1 + steps};
        at[{b.wo0, b.yo0, b.z0}] = (int32_t)i;
    }
    std::array<std::map<int32_t, std::vector<int32_t>>, 3> near;
    for (size_t q = 0; q < 3; ++q)
        for (const auto& a : cuts[q])
            for (const auto& b : cuts[q])
                if (a.second.lo < b.second.hi && b.second.lo < a.second.hi) near[q][a.first].push_back(b.first);
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

hipError_t launch_deep(int dtype_bytes, const DeepPlan& d, hipStream_t st, const DeepMap& g, const DeepTile* tiles,
                       int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                       bool want_res) {
    if (d.tiles.empty()) return hipErrorInvalidValue;
    const unsigned n = (unsigned)d.tiles.size();
#define OD_LAUNCH(T, R, RAG)                                                                                       \
    if (dtype_bytes == (int)sizeof(T) && d.rows == R && d.ragged == RAG) {                                         \
        hipLaunchKernelGGL((k_deep<T, R, RAG>), dim3(n), dim3(Deep<T, R>::NT), 0, st, g, tiles, parity, res,       \
                           zero_lo, zero_hi, hints, want_res ? 1 : 0);                                             \
        return hipGetLastError();                                                                                  \
    }
    OD_DEEP_VARIANTS(OD_LAUNCH)
#undef OD_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace od
