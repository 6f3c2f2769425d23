// Builder of the patch layout (host_patch.hpp).
#include "host_patch.hpp"

#include <algorithm>
#include <atomic>
#include <climits>
#include <exception>
#include <map>
#include <new>
#include <thread>
#include <unordered_map>

#include "../../include/nimble_plan.h"
#include "../../include/nimble_plan_debug.h"
#include "host_topo.hpp"

namespace nimble {

namespace {

constexpr int32_t kZero = -1, kInf = -2;      // offsets that are no link

// One slot with global link ids: 9 offsets (product) or 20 (plain, candidate-major).
struct Slot {
    int32_t at[20];
    int32_t base, shift, n;
};

struct Path {
    const int32_t *p;
    int32_t n;
};

// a0 a2 b0 b2 c d0 d1 e0 e1
enum { A0, A2, B0, B2, C, D0, D1, E0, E1 };

bool same(const int32_t *p, const int32_t *q, int32_t n) { return std::equal(p, p + n, q); }

// puts `n` links (at most two) into two places, zeros first
void put2(int32_t &u, int32_t &v, const int32_t *p, int32_t n)
{
    u = n > 1 ? p[0] : kZero;
    v = n > 1 ? p[1] : n > 0 ? p[0] : kZero;
}

// the same with the zero last: after the shared middle the order inside a tail stays free too
void put2_front(int32_t &u, int32_t &v, const int32_t *p, int32_t n)
{
    u = n > 0 ? p[0] : kZero;
    v = n > 1 ? p[1] : kZero;
}

// Four candidates that are one middle link reached two ways and left two ways.
bool full_slot(const Path (&c)[4], Slot &s)
{
    for (int32_t m0 = 0; m0 < c[0].n && m0 <= 2; ++m0) {
        const int32_t mid = c[0].p[m0];
        int32_t m[4];
        bool ok = true;
        for (int32_t i = 0; i < 4 && ok; ++i) {
            m[i] = -1;
            for (int32_t j = 0; j < c[i].n && j <= 2; ++j)
                if (c[i].p[j] == mid) m[i] = j;
            ok = m[i] >= 0 && c[i].n - m[i] - 1 <= 2;
        }
        if (!ok) continue;
        auto tail = [&](int32_t i) { return c[i].p + m[i] + 1; };
        auto tail_n = [&](int32_t i) { return c[i].n - m[i] - 1; };
        if (m[0] != m[1] || m[2] != m[3] || tail_n(0) != tail_n(2) || tail_n(1) != tail_n(3))
            continue;
        if (!same(c[0].p, c[1].p, m[0]) || !same(c[2].p, c[3].p, m[2]) ||
            !same(tail(0), tail(2), tail_n(0)) || !same(tail(1), tail(3), tail_n(1)))
            continue;
        put2(s.at[A0], s.at[B0], c[0].p, m[0]);
        put2(s.at[A2], s.at[B2], c[2].p, m[2]);
        s.at[C] = mid;
        put2_front(s.at[D0], s.at[E0], tail(0), tail_n(0));
        put2_front(s.at[D1], s.at[E1], tail(1), tail_n(1));
        s.shift = 0;
        s.n = 4;
        return true;
    }
    return false;
}

// Two paths with a common tail of at most three links after at most two links each.
bool half_slot(const Path &x, const Path &y, Slot &s)
{
    int32_t t = 0;
    while (t < 3 && t < x.n && t < y.n && x.p[x.n - 1 - t] == y.p[y.n - 1 - t]) ++t;
    if (x.n - t > 2 || y.n - t > 2) return false;
    put2(s.at[A0], s.at[B0], x.p, x.n - t);
    put2(s.at[A2], s.at[B2], y.p, y.n - t);
    const int32_t *tail = x.p + x.n - t;
    s.at[C] = t > 0 ? tail[0] : kZero;
    s.at[D0] = t > 1 ? tail[1] : kZero;
    s.at[E0] = t > 2 ? tail[2] : kZero;
    s.at[D1] = kInf;
    s.at[E1] = kZero;
    s.shift = 1;
    s.n = 2;
    return true;
}

void single_slot(const Path &x, Slot &s)
{
    const int32_t h = x.n < 2 ? x.n : 2;
    put2(s.at[A0], s.at[B0], x.p, h);
    s.at[C] = x.n > 2 ? x.p[2] : kZero;
    s.at[D0] = x.n > 3 ? x.p[3] : kZero;
    s.at[E0] = x.n > 4 ? x.p[4] : kZero;
    s.at[A2] = kInf;
    s.at[B2] = kZero;
    s.at[D1] = kInf;
    s.at[E1] = kZero;
    s.shift = 2;
    s.n = 1;
}

// The slots of one commodity, in candidate order; `out` holds at most 127 of them.
int32_t slots_of(int32_t n_cand, int32_t p0, const int32_t *path_link_ptr,
                 const int32_t *path_links, bool product, Slot *out)
{
    auto path = [&](int32_t j) {
        Path p;
        p.p = path_links + path_link_ptr[p0 + j];
        p.n = path_link_ptr[p0 + j + 1] - path_link_ptr[p0 + j];
        return p;
    };
    int32_t n = 0;
    if (!product) {
        for (int32_t j = 0; j < n_cand; j += 4) {
            Slot &s = out[n++];
            s.base = j;
            s.shift = 0;
            s.n = std::min(4, n_cand - j);
            for (int32_t c = 0; c < 4; ++c) {
                int32_t *at = s.at + 5 * c;
                for (int32_t i = 0; i < 5; ++i) at[i] = i == 0 ? kInf : kZero;
                if (c < s.n) {
                    const Path p = path(j + c);
                    for (int32_t i = 0; i < 5; ++i) at[i] = i < p.n ? p.p[i] : kZero;
                }
            }
        }
        return n;
    }
    for (int32_t j = 0; j < n_cand;) {
        Slot &s = out[n++];
        s.base = j;
        if (n_cand - j >= 4) {
            const Path four[4] = {path(j), path(j + 1), path(j + 2), path(j + 3)};
            if (full_slot(four, s)) {
                j += 4;
                continue;
            }
        }
        if (n_cand - j >= 2 && half_slot(path(j), path(j + 1), s)) {
            j += 2;
            continue;
        }
        single_slot(path(j), s);
        j += 1;
    }
    return n;
}

// the parts of a group are read eight users at a time
int32_t padded_parts(int32_t users) { return (users + 7) / 8 * 8; }

// Test hook: 1 the next range of a calling thread, 2 of a worker runs out of memory, 3 no worker
// can be started.
std::atomic<int32_t> g_fault{0};

void fault_point(int32_t where)
{
    int32_t want = where;
    if (g_fault.load() == where && g_fault.compare_exchange_strong(want, 0)) throw std::bad_alloc();
}

// f(begin, end) over ranges that cover 0..n-1, on up to eight threads.  Ranges whose thread cannot
// be started run in the calling one; an exception of any range is thrown again here, once all
// threads have ended.
template <typename F>
void parallel_ranges(int64_t n, F f, int64_t grain = 1)
{
    int64_t want = std::max<int64_t>(1, std::min<int64_t>(8, std::thread::hardware_concurrency()));
    want = std::min(want, std::max<int64_t>(1, n / grain));
    if (want <= 1) {
        fault_point(1);
        f(int64_t(0), n);
        return;
    }
    std::vector<std::exception_ptr> thrown(static_cast<size_t>(want));
    std::vector<std::thread> pool;
    pool.reserve(static_cast<size_t>(want));
    auto run = [&](int64_t w) {
        try {
            fault_point(w > 0 ? 2 : 1);
            f(n * w / want, n * (w + 1) / want);
        } catch (...) {
            thrown[static_cast<size_t>(w)] = std::current_exception();
        }
    };
    int64_t started = 1;
    for (; started < want; ++started) {
        try {
            const int64_t w = started;
            if (g_fault.load() == 3) throw std::bad_alloc();
            pool.emplace_back([&run, w] { run(w); });
        } catch (...) {
            break;
        }
    }
    run(0);
    for (int64_t w = started; w < want; ++w) run(w);
    for (auto &t : pool) t.join();
    for (const std::exception_ptr &e : thrown)
        if (e) std::rethrow_exception(e);
}

}  // namespace

void scan_patches(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                  const int32_t *pl, PatchScan &out)
{
    out = PatchScan();
    int32_t pmax = 0, lmax = 0;
    for (int32_t k = 0; k < n_comm; ++k) pmax = std::max(pmax, cp[k + 1] - cp[k]);
    for (int32_t p = 0; p < cp[n_comm]; ++p) lmax = std::max(lmax, lp[p + 1] - lp[p]);
    if (lmax > 5 || pmax > 32) return;
    // slots either way
    std::atomic<int64_t> sum[2] = {{0}, {0}};
    std::atomic<int32_t> most[2] = {{0}, {0}};
    std::vector<int32_t> cx(n_comm), cy(n_comm);
    const int64_t n_blocks = (static_cast<int64_t>(n_comm) + PatchScan::kBlock - 1) / PatchScan::kBlock;
    out.links.resize(static_cast<size_t>(n_blocks));
    out.link_ptr.resize(static_cast<size_t>(n_comm));
    parallel_ranges(n_blocks, [&](int64_t b0, int64_t b1) {
        Slot tmp[32];
        int64_t s[2] = {0, 0};
        int32_t m[2] = {0, 0};
        std::vector<int32_t> stamp(n_links, -1);
        const int64_t k1 = std::min<int64_t>(n_comm, b1 * PatchScan::kBlock);
        for (int64_t k = b0 * PatchScan::kBlock; k < k1; ++k) {
            std::vector<int32_t> &mine = out.links[static_cast<size_t>(k / PatchScan::kBlock)];
            out.link_ptr[k] = static_cast<int32_t>(mine.size());
            for (int32_t q = lp[cp[k]]; q < lp[cp[k + 1]]; ++q)
                if (stamp[pl[q]] != k) {
                    stamp[pl[q]] = static_cast<int32_t>(k);
                    mine.push_back(pl[q]);
                }
            const int32_t n = cp[k + 1] - cp[k];
            const int32_t ns[2] = {slots_of(n, cp[k], lp, pl, true, tmp), (n + 3) / 4};
            for (int32_t form = 0; form < 2; ++form) {
                s[form] += ns[form];
                m[form] = std::max(m[form], ns[form]);
            }
            int32_t first = INT32_MAX, last = INT32_MAX;
            for (int32_t p = cp[k]; p < cp[k + 1]; ++p) {
                first = std::min(first, pl[lp[p]]);
                last = std::min(last, pl[lp[p + 1] - 1]);
            }
            cx[k] = first;
            cy[k] = last;
        }
        for (int32_t i = 0; i < 2; ++i) {
            sum[i] += s[i];
            int32_t seen = most[i].load();
            while (seen < m[i] && !most[i].compare_exchange_weak(seen, m[i])) {
            }
        }
    }, 4);
    // price reads: nine per product slot, twenty per plain slot
    const bool product_fits = most[0] <= 8, plain_fits = most[1] <= 8;
    if (!product_fits && !plain_fits) return;
    out.product = product_fits && (!plain_fits || 9 * sum[0].load() <= 20 * sum[1].load()) ? 1 : 0;
    out.slots = most[out.product ? 0 : 1];
    // Coordinates as ranks, and for every rank how many links a cut after it divides.  For the
    // source coordinate the first two links of the paths count, for the destination coordinate
    // the last two: a cut between two nodes divides none of the node's own links.
    auto ranks = [&](const std::vector<int32_t> &c, bool head, std::vector<int32_t> &rank,
                     std::vector<int32_t> &cross, std::vector<int64_t> &count) {
        std::vector<int32_t> v(c);
        std::sort(v.begin(), v.end());
        v.erase(std::unique(v.begin(), v.end()), v.end());
        rank.resize(n_comm);
        count.assign(v.size(), 0);
        std::vector<int32_t> lo(n_links, INT32_MAX), hi(n_links, -1);
        for (int32_t k = 0; k < n_comm; ++k) {
            const int32_t r = static_cast<int32_t>(std::lower_bound(v.begin(), v.end(), c[k]) -
                                                   v.begin());
            rank[k] = r;
            count[r] += 1;
            for (int32_t p = cp[k]; p < cp[k + 1]; ++p) {
                const int32_t a = lp[p], b = lp[p + 1];
                for (int32_t i = 0; i < 2 && i < b - a; ++i) {
                    const int32_t e = pl[head ? a + i : b - 1 - i];
                    lo[e] = std::min(lo[e], r);
                    hi[e] = std::max(hi[e], r);
                }
            }
        }
        cross.assign(v.size() + 1, 0);
        for (int32_t e = 0; e < n_links; ++e)
            if (hi[e] > lo[e]) {
                cross[lo[e]] += 1;
                cross[hi[e]] -= 1;
            }
        for (size_t r = 1; r < cross.size(); ++r) cross[r] += cross[r - 1];
        for (size_t r = 1; r < count.size(); ++r) count[r] += count[r - 1];
    };
    parallel_ranges(2, [&](int64_t c0, int64_t c1) {
        for (int64_t c = c0; c < c1; ++c)
            if (c == 0) ranks(cx, true, out.x, out.x_cross, out.x_count);
            else ranks(cy, false, out.y, out.y_cross, out.y_count);
    }, n_comm < 8192 ? 2 : 1);
    out.fits = true;
}

namespace {

// Strip of every rank: `strips` runs of ranks with about equally many commodities, each cut
// moved (by at most 30 % of a strip) to where it divides the fewest links.
std::vector<int32_t> cut(const std::vector<int64_t> &count, const std::vector<int32_t> &cross,
                         int32_t strips)
{
    const int32_t n = static_cast<int32_t>(count.size());
    std::vector<int32_t> strip(n, 0);
    const int64_t total = n > 0 ? count[n - 1] : 0;
    const double width = static_cast<double>(total) / strips;
    int32_t from = 0;
    for (int32_t s = 1; s < strips; ++s) {
        const double want = width * s;
        int32_t best = -1;
        for (int32_t r = from; r < n - 1; ++r) {
            const double off = std::abs(static_cast<double>(count[r]) - want);
            if (off > 0.3 * width) continue;
            if (best < 0 || cross[r] < cross[best] ||
                (cross[r] == cross[best] &&
                 off < std::abs(static_cast<double>(count[best]) - want)))
                best = r;
        }
        if (best < 0) continue;                  // no boundary near: this strip joins the next
        for (int32_t r = best + 1; r < n; ++r) strip[r] = s;
        from = best + 1;
    }
    return strip;
}

}  // namespace

void cut_patches(int32_t n_comm, const PatchScan &scan, int32_t strips, PatchCut &out)
{
    out = PatchCut();
    out.strips = strips;
    std::vector<std::vector<int32_t>> grid(static_cast<size_t>(strips) * strips);
    if (strips == 1) {
        grid[0].resize(n_comm);
        for (int32_t k = 0; k < n_comm; ++k) grid[0][k] = k;
    } else {
        const std::vector<int32_t> sx = cut(scan.x_count, scan.x_cross, strips);
        const std::vector<int32_t> sy = cut(scan.y_count, scan.y_cross, strips);
        for (int32_t k = 0; k < n_comm; ++k)
            grid[static_cast<size_t>(sx[scan.x[k]]) * strips + sy[scan.y[k]]].push_back(k);
    }
    for (auto &m : grid)
        if (!m.empty()) {
            out.most = std::max<int64_t>(out.most, static_cast<int64_t>(m.size()));
            out.members.push_back(std::move(m));
        }
}

double patch_scan_us(const PatchShape &s)
{
    // cycles the LDS is busy (four per price read of a wave, more per atomic the more lanes add)
    // and cycles of vector issue; a wave's own chain of reads and additions on top
    const double waves = s.threads / 64.0;
    const double lds = waves * (s.quads * (s.product ? 36.0 : 80.0) + 50.0 + 80.0 / s.lanes);
    const double valu = waves * (s.quads * (s.product ? 28.0 : 50.0) + (s.lanes > 1 ? 85.0 : 70.0));
    // (fabrics of one patch, 240 to 992 pairs: 0.85, 1.28, 1.56, 1.99 and 2.16 us measured where this
    // says 0.85, 1.43, 1.15, 2.09 and 2.07)
    return 0.88 * (0.3 + 0.06 * s.quads + std::max(lds, valu) / 2400.0);
}

double patch_iteration_us(const PatchShape &s, int32_t patches, int32_t groups, int32_t parts)
{
    if (patches < 2 || groups == 0) return patch_scan_us(s);
    // Fitted to 269 measured layouts: 18 fabrics of 2 to 64 nodes and 11 irregular ones, every
    // grid they can be cut into.  The fabrics' estimates are within 11 % of the measured time for
    // 90 % of the grids and within 15 % for all (irregular ones: 18 %), and the grid with the
    // lowest estimate is the fastest or within 2 % of it.  A trip of a word from patch to patch
    // and the fixed steps are 1.8 us; a wave reads its bundles of four groups one after the
    // other, 0.7 us each; then what a thread has to publish and take up, the parts a compute unit
    // reads, and the parts all of them read from the memory side.
    const int32_t waves = s.threads / 64, bundles = (groups + 3) / 4;
    const double trips = (bundles + waves - 1) / waves;
    return kPatchTripUs + waves * (s.quads * (s.product ? 0.0196 : 0.0444) + 0.0128) + 0.72 * (trips - 1.0) +
           0.727 * (groups * kPatchGroup) / s.threads + 8.6e-4 * parts +
           3.4e-7 * parts * static_cast<double>(patches);
}

bool patch_shape(const PatchScan &scan, int64_t most, int32_t lanes, PatchShape &out)
{
    out = PatchShape();
    double best = 0.0;
    auto offer = [&](int32_t product, int32_t L, int32_t QL) {
        if (product != scan.product || (lanes > 0 && L != lanes)) return;
        if (L * QL < scan.slots || (L > 1 && L * (QL - 1) >= scan.slots)) return;
        if (most * L > kPatchThreads) return;
        PatchShape s;
        s.product = product;
        s.lanes = L;
        s.quads = QL;
        s.threads = static_cast<int32_t>((most * L + 63) / 64 * 64);
        const double us = patch_scan_us(s);
        if (out.threads == 0 || us < best) {
            best = us;
            out = s;
        }
    };
#define NIMBLE_PATCH_OFFER(PR, LL, QQ) offer(PR, LL, QQ);
    NIMBLE_PATCH_SHAPES(NIMBLE_PATCH_OFFER)
#undef NIMBLE_PATCH_OFFER
    return out.threads > 0;
}

namespace {

// the links of a patch's commodities, each once; `stamp` is a thread's own, b another number each time
void links_of_patch(const PatchScan &scan, const std::vector<int32_t> &members, int32_t b,
                    std::vector<int32_t> &stamp, std::vector<int32_t> &out)
{
    out.clear();
    const int32_t n_comm = static_cast<int32_t>(scan.link_ptr.size());
    for (int32_t k : members) {
        const std::vector<int32_t> &block = scan.links[static_cast<size_t>(k / PatchScan::kBlock)];
        const size_t end = k + 1 < n_comm && (k + 1) % PatchScan::kBlock != 0
                               ? static_cast<size_t>(scan.link_ptr[k + 1])
                               : block.size();
        for (size_t q = static_cast<size_t>(scan.link_ptr[k]); q < end; ++q)
            if (stamp[block[q]] != b) {
                stamp[block[q]] = b;
                out.push_back(block[q]);
            }
    }
}

}  // namespace

PatchSizes measure_cut(int32_t n_links, const PatchScan &scan, const PatchCut &cut,
                       const PatchShape &shape)
{
    PatchSizes m;
    const int32_t B = static_cast<int32_t>(cut.members.size());
    std::vector<std::vector<int32_t>> links(B);
    std::vector<int32_t> stamp(n_links, -1);
    for (int32_t b = 0; b < B; ++b) links_of_patch(scan, cut.members[b], b, stamp, links[b]);
    // links with the same users: a number for every set of users (two sets with one number would
    // only spoil an estimate), how many users it has and how many groups its links fill
    std::vector<uint64_t> sig(n_links, 0u);
    std::vector<int32_t> users(n_links, 0);
    for (int32_t b = 0; b < B; ++b) {
        uint64_t z = (static_cast<uint64_t>(b) + 1u) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z ^= z >> 27;
        for (int32_t e : links[b]) {
            sig[e] += z;
            users[e] += 1;
        }
    }
    std::unordered_map<uint64_t, std::pair<int32_t, int32_t>> sets;      // first link, links
    for (int32_t e = 0; e < n_links; ++e)
        if (users[e] > 1) {
            auto &s = sets[sig[e]];
            if (s.second++ == 0) s.first = e;
        }
    std::vector<int32_t> groups_of_first(n_links, 0);
    for (const auto &s : sets)
        groups_of_first[s.second.first] = (s.second.second + kPatchGroup - 1) / kPatchGroup;
    for (int32_t b = 0; b < B; ++b) {
        int32_t groups = 0, parts = 0, own = 0;
        for (int32_t e : links[b]) {
            own += users[e] == 1 ? 1 : 0;
            groups += groups_of_first[e];
            parts += groups_of_first[e] * padded_parts(users[e]);
        }
        m.max_groups = std::max(m.max_groups, groups);
        m.max_parts = std::max(m.max_parts, parts);
        m.max_local = std::max(m.max_local, groups * kPatchGroup + own);
    }
    m.patches = B;
    m.max_comm = static_cast<int32_t>(cut.most);
    // (prices, link states, groups and counts: lds_layout in patch_kernel.hpp)
    const int64_t links_lds = 48ll * m.max_local + 16ll * m.max_groups + 512;
    const int64_t slots = static_cast<int64_t>(m.max_comm) * shape.lanes * shape.quads;
    m.fits = m.max_local <= kPatchMaxLocal && links_lds + 8 * slots <= 160 * 1024;
    m.fits_adaptive = m.fits && links_lds + 32 * slots <= 160 * 1024;
    return m;
}

PatchChoice choose_cuts(int32_t n_links, int32_t n_comm, const PatchScan &scan,
                        int32_t most_patches, int32_t forced, int32_t lanes)
{
    int32_t most_strips = 1;
    while ((most_strips + 1) * (most_strips + 1) <= most_patches) ++most_strips;
    struct Tried {
        PatchSizes sizes;
        double us;
    };
    std::vector<Tried> tried(static_cast<size_t>(most_strips) + 1);
    auto try_strips = [&](int32_t strips) {
        // (most grids are ruled out by their size alone)
        if (forced > 0 && strips != forced) return;
        if (n_comm > static_cast<int64_t>(strips) * strips * kPatchThreads) return;
        Tried &t = tried[static_cast<size_t>(strips)];
        PatchCut cut;
        PatchShape shape;
        cut_patches(n_comm, scan, strips, cut);
        if (!patch_shape(scan, cut.most, lanes, shape)) return;
        t.sizes = measure_cut(n_links, scan, cut, shape);
        t.us = patch_iteration_us(shape, t.sizes.patches, t.sizes.max_groups, t.sizes.max_parts);
    };
    PatchChoice c;
    auto offer = [&](int32_t strips) {
        const Tried &t = tried[static_cast<size_t>(strips)];
        if (!t.sizes.fits || t.sizes.patches > most_patches) return;
        if (c.fewest == 0) c.fewest = strips;
        if (c.best == 0 || t.us < tried[static_cast<size_t>(c.best)].us) c.best = strips;
    };
    // one patch that is done before words could go from patch to patch needs no comparison
    try_strips(1);
    offer(1);
    if (c.best == 1 && tried[1].us < kPatchTripUs && tried[1].sizes.fits_adaptive) return c;
    parallel_ranges(most_strips - 1, [&](int64_t s0, int64_t s1) {
        for (int64_t s = s0; s < s1; ++s) try_strips(static_cast<int32_t>(s) + 2);
    }, n_comm < 2048 ? 16 : 1);
    for (int32_t s = 2; s <= most_strips; ++s) offer(s);
    auto patches = [&](int32_t strips) { return tried[static_cast<size_t>(strips)].sizes.patches; };
    if (c.best == 0) return c;
    if (patches(c.best) == patches(c.fewest)) c.fewest = c.best;
    if (!tried[static_cast<size_t>(c.best)].sizes.fits_adaptive &&
        !tried[static_cast<size_t>(c.fewest)].sizes.fits_adaptive)
        for (int32_t s = 1; s <= most_strips; ++s) {
            const Tried &t = tried[static_cast<size_t>(s)];
            if (t.sizes.fits_adaptive && t.sizes.patches <= most_patches &&
                (c.adaptive == 0 || t.us < tried[static_cast<size_t>(c.adaptive)].us))
                c.adaptive = s;
        }
    return c;
}

bool build_patches(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                   const int32_t *pl, const PatchScan &scan, PatchCut &cut,
                   const PatchShape &shape, PatchLayout &out)
{
    out = PatchLayout();
    out.shape = shape;
    const bool product = shape.product != 0;
    const int32_t L = shape.lanes, QL = shape.quads, NT = shape.threads;
    const int32_t NW = product ? kPatchWordsProduct : kPatchWordsPlain;
    std::vector<std::vector<int32_t>> &members = cut.members;
    const int32_t B = static_cast<int32_t>(members.size());
    if (cut.most * L > NT) return false;
    // Lanes that work side by side should hold commodities of different sources and different
    // destinations: their loads then fall on different links.  So a patch's commodities are taken
    // diagonal by diagonal of its source x destination table.
    parallel_ranges(B, [&](int64_t b0, int64_t b1) {
        std::vector<int32_t> xs, ys;
        std::vector<std::pair<int64_t, int32_t>> key;
        for (int64_t b = b0; b < b1; ++b) {
            xs.clear();
            ys.clear();
            for (int32_t k : members[b]) {
                xs.push_back(scan.x[k]);
                ys.push_back(scan.y[k]);
            }
            for (auto *v : {&xs, &ys}) {
                std::sort(v->begin(), v->end());
                v->erase(std::unique(v->begin(), v->end()), v->end());
            }
            const int64_t n = static_cast<int64_t>(std::max(xs.size(), ys.size()));
            key.clear();
            for (int32_t k : members[b]) {
                const int64_t x = std::lower_bound(xs.begin(), xs.end(), scan.x[k]) - xs.begin();
                const int64_t y = std::lower_bound(ys.begin(), ys.end(), scan.y[k]) - ys.begin();
                key.emplace_back(((y - x + n) % n) * n + x, k);
            }
            std::sort(key.begin(), key.end());
            for (size_t i = 0; i < key.size(); ++i) members[b][i] = key[i].second;
        }
    });

    // the links of every patch and the patches of every link
    std::vector<std::vector<int32_t>> links(B);
    parallel_ranges(B, [&](int64_t b0, int64_t b1) {
        std::vector<int32_t> stamp(n_links, -1);
        for (int32_t b = static_cast<int32_t>(b0); b < b1; ++b) {
            links_of_patch(scan, members[b], b, stamp, links[b]);
            std::sort(links[b].begin(), links[b].end());
        }
    });
    std::vector<std::vector<int32_t>> users(n_links);
    for (int32_t b = 0; b < B; ++b)
        for (int32_t e : links[b]) users[e].push_back(b);
    // groups of shared links with the same users, in order of first appearance
    struct Group {
        std::vector<int32_t> links;
        const std::vector<int32_t> *users;
        int64_t first_part;
    };
    std::vector<Group> groups;
    std::vector<std::vector<int32_t>> groups_of(B);
    {
        std::map<std::vector<int32_t>, int32_t> open;      // users -> group with room
        for (int32_t e = 0; e < n_links; ++e) {
            if (users[e].size() < 2) continue;
            auto it = open.find(users[e]);
            if (it == open.end() ||
                static_cast<int32_t>(groups[it->second].links.size()) == kPatchGroup) {
                const int32_t g = static_cast<int32_t>(groups.size());
                groups.push_back(Group{{}, &users[e], out.n_parts});
                out.n_parts += padded_parts(static_cast<int32_t>(users[e].size())) * kPatchGroup;
                out.max_users = std::max(out.max_users, static_cast<int32_t>(users[e].size()));
                for (int32_t b : users[e]) groups_of[b].push_back(g);
                if (it == open.end()) it = open.emplace(users[e], g).first;
                else it->second = g;
            }
            groups[it->second].links.push_back(e);
        }
    }
    if (out.n_parts > (int64_t(1) << 28)) return false;
    // local numbering: the groups (padded), then the private links
    out.desc.assign(static_cast<size_t>(kPatchDescInts) * B, 0);
    std::vector<int32_t> first_local(B + 1, 0), first_group(B + 1, 0);
    std::vector<int32_t> first_comm(B + 1, 0);
    for (int32_t b = 0; b < B; ++b) {
        int32_t n_private = 0, parts = 0;
        for (int32_t e : links[b]) n_private += users[e].size() == 1 ? 1 : 0;
        for (int32_t g : groups_of[b]) parts += padded_parts(static_cast<int32_t>(groups[g].users->size()));
        const int32_t ng = static_cast<int32_t>(groups_of[b].size());
        const int32_t n_local = ng * kPatchGroup + n_private;
        if (n_local > kPatchMaxLocal) return false;
        first_local[b + 1] = first_local[b] + n_local;
        first_group[b + 1] = first_group[b] + ng;
        out.max_local = std::max(out.max_local, n_local);
        out.max_groups = std::max(out.max_groups, ng);
        out.max_parts = std::max(out.max_parts, parts);
        int32_t *d = &out.desc[static_cast<size_t>(kPatchDescInts) * b];
        d[0] = first_local[b];
        d[1] = n_local;
        d[2] = ng * kPatchGroup;
        d[3] = first_group[b];
        d[4] = ng;
        d[5] = first_comm[b];
        d[6] = static_cast<int32_t>(members[b].size());
        first_comm[b + 1] = first_comm[b] + d[6];
        out.max_comm = std::max(out.max_comm, d[6]);
    }
    out.loc_link.assign(first_local[B], -1);
    out.group.assign(static_cast<size_t>(4) * first_group[B], 0);
    out.comm.assign(n_comm, -1);
    out.words.assign(static_cast<size_t>(B) * QL * NW * NT, 0u);
    out.first.assign(static_cast<size_t>(B) * QL * NT, 0u);
    parallel_ranges(B, [&](int64_t b0, int64_t b1) {
        std::vector<int32_t> local(n_links, 0), seen(n_links, -1);
        Slot slot[32];
        for (int32_t b = static_cast<int32_t>(b0); b < b1; ++b) {
            int32_t at = 0;
            for (size_t gi = 0; gi < groups_of[b].size(); ++gi) {
                const Group &g = groups[groups_of[b][gi]];
                int32_t *gd = &out.group[static_cast<size_t>(4) * (first_group[b] + gi)];
                gd[0] = static_cast<int32_t>(g.first_part);
                gd[1] = padded_parts(static_cast<int32_t>(g.users->size()));
                gd[3] = static_cast<int32_t>(g.users->size());
                gd[2] = static_cast<int32_t>(
                    std::lower_bound(g.users->begin(), g.users->end(), b) - g.users->begin());
                for (int32_t q = 0; q < kPatchGroup; ++q, ++at)
                    if (q < static_cast<int32_t>(g.links.size())) {
                        const int32_t e = g.links[q];
                        out.loc_link[first_local[b] + at] = e | (gd[2] == 0 ? kPatchExport : 0);
                        local[e] = at;
                    }
            }
            for (int32_t e : links[b])
                if (users[e].size() == 1) {
                    out.loc_link[first_local[b] + at] = e | kPatchExport;
                    local[e] = at++;
                }
            const uint32_t zero = 8u * static_cast<uint32_t>(at), inf = zero + 8u;
            auto offset = [&](int32_t e) -> uint32_t {
                return e == kZero ? zero : e == kInf ? inf : 8u * static_cast<uint32_t>(local[e]);
            };
            uint32_t *words = &out.words[static_cast<size_t>(b) * QL * NW * NT];
            uint32_t *first = &out.first[static_cast<size_t>(b) * QL * NT];
            std::copy(members[b].begin(), members[b].end(), out.comm.begin() + first_comm[b]);
            for (int32_t g = 0; g < NT / L; ++g) {
                const int32_t k =
                    g < static_cast<int32_t>(members[b].size()) ? members[b][g] : -1;
                const int32_t n =
                    k < 0 ? 0 : slots_of(cp[k + 1] - cp[k], cp[k], lp, pl, product, slot);
                // lane j scans the slots j, j + L, ...: candidates ascend
                for (int32_t q = 0; q < QL; ++q)
                    for (int32_t j = 0; j < L; ++j) {
                        const int32_t si = q * L + j;
                        const size_t t = static_cast<size_t>(g) * L + j;
                        uint32_t o[20], meta = 0u, once = 0u;
                        const int32_t n_off = product ? 9 : 20;
                        for (int32_t x = 0; x < n_off; ++x) o[x] = inf;
                        if (si < n) {
                            const Slot &s = slot[si];
                            meta = static_cast<uint32_t>(s.base | s.shift << 7 | s.n << 9);
                            for (int32_t x = 0; x < n_off; ++x) {
                                o[x] = offset(s.at[x]);
                                if (s.at[x] >= 0 && seen[s.at[x]] != k) {
                                    seen[s.at[x]] = k;
                                    once |= 1u << x;
                                }
                            }
                        }
                        uint32_t w[kPatchWordsPlain];
                        if (product) {
                            w[0] = o[A0] | o[A2] << 16;
                            w[1] = o[B0] | o[B2] << 16;
                            w[2] = o[C] | meta << 16;
                            w[3] = o[D0] | o[D1] << 16;
                            w[4] = o[E0] | o[E1] << 16;
                        } else {
                            for (int32_t c = 0; c < 4; ++c) {
                                w[2 * c] = o[5 * c] | o[5 * c + 1] << 16;
                                w[2 * c + 1] = o[5 * c + 2] | o[5 * c + 3] << 16;
                            }
                            w[8] = o[4] | o[9] << 16;
                            w[9] = o[14] | o[19] << 16;
                            w[10] = meta << 16;
                        }
                        for (int32_t x = 0; x < NW; ++x)
                            words[(static_cast<size_t>(q) * NW + x) * NT + t] = w[x];
                        first[static_cast<size_t>(q) * NT + t] = once;
                    }
            }
        }
    });
    out.n_patches = B;
    return true;
}

int check_patches(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                  const int32_t *pl, const PatchLayout &t)
{
    const int32_t L = t.shape.lanes, QL = t.shape.quads, NT = t.shape.threads;
    const bool product = t.shape.product != 0;
    const int32_t NW = product ? kPatchWordsProduct : kPatchWordsPlain;
    if (NT < 64 || NT > kPatchThreads || NT % 64 || t.max_local > kPatchMaxLocal) return 1;
    std::vector<int32_t> comm_seen(n_comm, 0), exported(n_links, 0);
    std::vector<uint8_t> part_owner(static_cast<size_t>(t.n_parts / kPatchGroup), 0);
    std::vector<std::vector<int32_t>> group_links(static_cast<size_t>(t.n_parts / kPatchGroup));
    for (int32_t b = 0; b < t.n_patches; ++b) {
        const int32_t *d = &t.desc[static_cast<size_t>(kPatchDescInts) * b];
        const int32_t n_local = d[1];
        const int32_t *ll = &t.loc_link[d[0]];
        if (d[2] != kPatchGroup * d[4] || d[2] > n_local) return 2;
        for (int32_t i = 0; i < n_local; ++i) {
            if (ll[i] == -1 && i >= d[2]) return 3;
            if (ll[i] == -1) continue;
            const int32_t e = ll[i] & ~kPatchExport;
            if (e < 0 || e >= n_links) return 4;
            if (ll[i] & kPatchExport) exported[e] += 1;
        }
        for (int32_t g = 0; g < d[4]; ++g) {
            const int32_t *gd = &t.group[static_cast<size_t>(4) * (d[3] + g)];
            if (gd[0] < 0 || gd[0] % (8 * kPatchGroup) || gd[3] < 2 || gd[1] != padded_parts(gd[3]) ||
                gd[2] < 0 || gd[2] >= gd[3] ||
                gd[0] + static_cast<int64_t>(kPatchGroup) * gd[1] > t.n_parts)
                return 5;
            // every part has one writer, and the users of a group agree on its links
            for (int32_t c = gd[2]; c < gd[1]; c += gd[3])
                if (part_owner[gd[0] / kPatchGroup + c]++) return 6;
            std::vector<int32_t> mine(kPatchGroup);
            for (int32_t i = 0; i < kPatchGroup; ++i) {
                const int32_t v = ll[g * kPatchGroup + i];
                mine[i] = v == -1 ? -1 : v & ~kPatchExport;
            }
            std::vector<int32_t> &ref = group_links[gd[0] / kPatchGroup];
            if (ref.empty()) ref = mine;
            else if (ref != mine) return 7;
        }
        if (d[6] > NT / L) return 18;
        for (int32_t g = 0; g < NT / L; ++g) {
            const int32_t k = g < d[6] ? t.comm[d[5] + g] : -1;
            std::vector<int32_t> used;
            int32_t next = 0;
            for (int32_t q = 0; q < QL; ++q)
                for (int32_t j = 0; j < L; ++j) {
                    const size_t th = static_cast<size_t>(g) * L + j;
                    auto word = [&](int32_t x) {
                        return t.words[((static_cast<size_t>(b) * QL + q) * NW + x) * NT + th];
                    };
                    const uint32_t once = t.first[(static_cast<size_t>(b) * QL + q) * NT + th];
                    uint32_t o[20], meta;
                    const int32_t n_off = product ? 9 : 20;
                    if (product) {
                        const uint32_t w[5] = {word(0), word(1), word(2), word(3), word(4)};
                        o[A0] = w[0] & 0xFFFFu, o[A2] = w[0] >> 16;
                        o[B0] = w[1] & 0xFFFFu, o[B2] = w[1] >> 16;
                        o[C] = w[2] & 0xFFFFu, meta = w[2] >> 16;
                        o[D0] = w[3] & 0xFFFFu, o[D1] = w[3] >> 16;
                        o[E0] = w[4] & 0xFFFFu, o[E1] = w[4] >> 16;
                    } else {
                        for (int32_t c = 0; c < 4; ++c) {
                            o[5 * c] = word(2 * c) & 0xFFFFu;
                            o[5 * c + 1] = word(2 * c) >> 16;
                            o[5 * c + 2] = word(2 * c + 1) & 0xFFFFu;
                            o[5 * c + 3] = word(2 * c + 1) >> 16;
                            o[5 * c + 4] = (word(8 + c / 2) >> (16 * (c % 2))) & 0xFFFFu;
                        }
                        meta = word(10) >> 16;
                    }
                    const uint32_t zero = 8u * n_local, inf = zero + 8u;
                    for (int32_t x = 0; x < n_off; ++x)
                        if (o[x] % 8 || o[x] > inf) return 8;
                    const int32_t base = meta & 127, shift = (meta >> 7) & 3;
                    const int32_t n = (meta >> 9) & 7;
                    if (k < 0 && (n != 0 || once != 0u)) return 20;
                    for (int32_t x = 0; x < n_off; ++x)
                        if ((once >> x) & 1u) {
                            if (o[x] >= zero) return 9;
                            used.push_back(ll[o[x] / 8] & ~kPatchExport);
                        }
                    if (n == 0) continue;
                    if (k < 0 || base != next) return 10;
                    next += n;
                    for (int32_t c = 0; c < n; ++c) {
                        const int32_t pos = c << shift;
                        std::vector<int32_t> path;
                        auto add = [&](uint32_t off) {
                            if (off < zero) path.push_back(ll[off / 8] & ~kPatchExport);
                            return off != inf;
                        };
                        bool ok = true;
                        if (product) {
                            const int32_t h = pos >> 1, l = pos & 1;
                            for (int32_t x : {A0 + h, B0 + h, int32_t(C), D0 + l, E0 + l})
                                ok = add(o[x]) && ok;
                        } else {
                            for (int32_t x = 0; x < 5; ++x) ok = add(o[5 * pos + x]) && ok;
                        }
                        const int32_t p = cp[k] + base + c;
                        if (!ok || p >= cp[k + 1] ||
                            path != std::vector<int32_t>(pl + lp[p], pl + lp[p + 1]))
                            return 11;
                    }
                    // what the slot does not hold must never be chosen
                    for (int32_t pos = 0; pos < 4; ++pos) {
                        if ((pos & ((1 << shift) - 1)) == 0 && (pos >> shift) < n) continue;
                        bool absent = false;
                        if (product) {
                            const int32_t h = pos >> 1, l = pos & 1;
                            for (int32_t x : {A0 + h, B0 + h, int32_t(C), D0 + l, E0 + l})
                                absent = absent || o[x] == inf;
                        } else {
                            absent = o[5 * pos] == inf;
                        }
                        if (!absent) return 12;
                    }
                }
            if (k < 0) continue;
            comm_seen[k] += 1;
            if (next != cp[k + 1] - cp[k]) return 13;
            std::vector<int32_t> all(pl + lp[cp[k]], pl + lp[cp[k + 1]]);
            std::sort(all.begin(), all.end());
            all.erase(std::unique(all.begin(), all.end()), all.end());
            std::sort(used.begin(), used.end());
            if (used != all) return 14;
        }
    }
    for (int32_t k = 0; k < n_comm; ++k)
        if (comm_seen[k] != 1) return 15;
    for (uint8_t o : part_owner)
        if (o != 1) return 16;
    std::vector<uint8_t> in_use(n_links, 0);
    for (int32_t q = 0; q < lp[cp[n_comm]]; ++q) in_use[pl[q]] = 1;
    for (int32_t e = 0; e < n_links; ++e)
        if (exported[e] != in_use[e]) return 17;
    return 0;
}

}  // namespace nimble

extern "C" void nimble_debug_fail_patch_build(int32_t where) { nimble::g_fault.store(where); }

extern "C" nimble_status_t nimble_host_patch_check(int32_t n_links, int32_t n_comm,
                                                   const int32_t *comm_path_ptr, int32_t n_paths,
                                                   const int32_t *path_link_ptr,
                                                   const int32_t *path_links, int32_t strips,
                                                   int32_t lanes, int64_t *out)
{
    try {
        std::string why;
        nimble_status_t st = nimble::validate_csr(n_links, nullptr, n_comm, comm_path_ptr, n_paths,
                                                  path_link_ptr, path_links, why);
        if (st != NIMBLE_OK) return st;
        if (!out || strips < 1 || strips > 64 || lanes < 0) return NIMBLE_ERR_INVALID;
        nimble::PatchScan scan;
        nimble::PatchLayout t;
        nimble::scan_patches(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links, scan);
        nimble::PatchCut cut;
        nimble::PatchShape shape;
        if (scan.fits) nimble::cut_patches(n_comm, scan, strips, cut);
        nimble::PatchSizes m;
        if (scan.fits && nimble::patch_shape(scan, cut.most, lanes, shape)) {
            m = nimble::measure_cut(n_links, scan, cut, shape);
            nimble::build_patches(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links, scan, cut,
                                  shape, t);
        }
        out[0] = t.n_patches;
        out[1] = t.n_patches > 0 ? nimble::check_patches(n_links, n_comm, comm_path_ptr, path_link_ptr,
                                                         path_links, t)
                                 : 0;
        // what is found without building a layout is what it has
        if (t.n_patches > 0 && out[1] == 0 &&
            (m.patches != t.n_patches || m.max_comm != t.max_comm || m.max_local != t.max_local ||
             m.max_groups != t.max_groups || m.max_parts != t.max_parts))
            out[1] = 19;
        out[2] = t.shape.product;
        out[3] = t.shape.lanes;
        out[4] = t.shape.quads;
        out[5] = t.shape.threads;
        out[6] = t.max_local;
        out[7] = t.max_groups;
        out[8] = t.max_users;
        out[9] = t.max_parts;
        out[10] = t.n_parts;
        return NIMBLE_OK;
    } catch (const std::exception &) {           // out of memory, in whatever thread
        return NIMBLE_ERR_ALLOC;
    }
}
