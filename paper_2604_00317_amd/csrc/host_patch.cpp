// Builder of the patch layout (host_patch.hpp).
#include "host_patch.hpp"

#include <algorithm>
#include <atomic>
#include <climits>
#include <exception>
#include <map>
#include <new>
#include <thread>
#include <tuple>
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

// The same with the links in the places they have in the paths of five links, where a link of the
// path has one: so that the tails of a destination's paths are equal whatever their heads leave out.
void placed_slot(const Path &x, const int8_t *place, Slot &s)
{
    int32_t shift = -1;
    for (int32_t i = 0; i < x.n && shift < 0; ++i)
        if (place[x.p[i]] >= i && place[x.p[i]] - i + x.n <= 5) shift = place[x.p[i]] - i;
    single_slot(x, s);
    if (shift < 0) return;
    for (int32_t i = 0; i < 5; ++i) {
        const int32_t e = i >= shift && i < shift + x.n ? x.p[i - shift] : kZero;
        s.at[i == 0 ? A0 : i == 1 ? B0 : i == 2 ? C : i == 3 ? D0 : E0] = e;
    }
}

// The slots of one commodity, in candidate order; `out` holds at most 127 of them.  `place`: links
// are put into their places (blocks), null: single paths begin in the first one.
int32_t slots_of(int32_t n_cand, int32_t p0, const int32_t *path_link_ptr,
                 const int32_t *path_links, bool product, Slot *out, const int8_t *place = nullptr)
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
        if (place != nullptr) placed_slot(path(j), place, s);
        else single_slot(path(j), s);
        j += 1;
    }
    return n;
}

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

namespace {

uint64_t mixed(uint64_t h, uint64_t v)
{
    h = (h ^ v) * 0x9E3779B97F4A7C15ull;
    return h ^ (h >> 29);
}

// the links of a slot's head (a0 a2 b0 b2 c) and tail (d0 d1 e0 e1), and numbers for them (never 0)
constexpr int32_t kHeadAt[5] = {A0, A2, B0, B2, C}, kTailAt[4] = {D0, D1, E0, E1};
uint64_t head_number(const Slot &s)
{
    uint64_t h = 1;
    for (int32_t x : kHeadAt) h = mixed(h, static_cast<uint32_t>(s.at[x]));
    return h | 1u;
}
uint64_t tail_number(const Slot &s)
{
    uint64_t h = 2;
    for (int32_t x : kTailAt) h = mixed(h, static_cast<uint32_t>(s.at[x]));
    return h | 1u;
}

void scan_blocks(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                 const int32_t *pl, int32_t most_slots, PatchScan &out)
{
    const int32_t L = most_slots <= 2 ? 2 : most_slots <= 4 ? 4 : 8;
    const int64_t n_blocks = static_cast<int64_t>(out.links.size());
    // places of the links in paths of five links
    out.place.assign(static_cast<size_t>(n_links), -1);
    std::vector<std::atomic<uint8_t>> seen(static_cast<size_t>(n_links));      // a bit per place
    auto range = [&](int64_t b0, int64_t b1, auto f) {
        const int64_t k1 = std::min<int64_t>(n_comm, b1 * PatchScan::kBlock);
        for (int64_t k = b0 * PatchScan::kBlock; k < k1; ++k) f(static_cast<int32_t>(k));
    };
    parallel_ranges(n_blocks, [&](int64_t b0, int64_t b1) {
        range(b0, b1, [&](int32_t k) {
            for (int32_t p = cp[k]; p < cp[k + 1]; ++p)
                for (int32_t i = 0; i < 5 && lp[p + 1] - lp[p] == 5; ++i) {
                    std::atomic<uint8_t> &w = seen[static_cast<size_t>(pl[lp[p] + i])];
                    const uint8_t bit = static_cast<uint8_t>(1u << i);
                    if (!(w.load(std::memory_order_relaxed) & bit)) w.fetch_or(bit);
                }
        });
    }, 4);
    for (int32_t e = 0; e < n_links; ++e) {
        const uint8_t w = seen[static_cast<size_t>(e)].load();
        for (int32_t i = 0; i < 5; ++i)
            if ((w >> i) & 1u) out.place[e] = w == 1u << i ? static_cast<int8_t>(i) : int8_t(-2);
    }
    out.head.assign(static_cast<size_t>(n_comm) * L, 0u);
    out.tail.assign(static_cast<size_t>(n_comm) * L, 0u);
    std::atomic<int32_t> two{0};
    parallel_ranges(n_blocks, [&](int64_t b0, int64_t b1) {
        Slot tmp[32];
        bool ways = false;
        range(b0, b1, [&](int32_t k) {
            const int32_t n = slots_of(cp[k + 1] - cp[k], cp[k], lp, pl, true, tmp, out.place.data());
            for (int32_t j = 0; j < n; ++j) {
                out.head[static_cast<size_t>(k) * L + j] = head_number(tmp[j]);
                out.tail[static_cast<size_t>(k) * L + j] = tail_number(tmp[j]);
                ways = ways || tmp[j].at[D1] != kInf;
            }
        });
        if (ways) two.store(1);
    }, 4);
    out.block_lanes = L;
    out.block_product = two.load();
}

}  // namespace

void find_blocks(const PatchScan &scan, const std::vector<int32_t> &members, PatchBlocks &out)
{
    const int32_t L = scan.block_lanes;
    out = PatchBlocks();
    // Commodities with the same tails, of the same L sources, make a block; where a source comes
    // twice (pairs inside a node have no tails) they fill blocks one after the other.
    std::vector<int32_t> xs;
    xs.reserve(members.size());
    for (int32_t k : members) xs.push_back(scan.x[k]);
    std::sort(xs.begin(), xs.end());
    xs.erase(std::unique(xs.begin(), xs.end()), xs.end());
    struct Place {
        uint64_t tails;
        int32_t x, y, k;
    };
    std::vector<Place> at;
    at.reserve(members.size());
    for (int32_t k : members) {
        uint64_t h = 3;
        for (int32_t j = 0; j < L; ++j) h = mixed(h, scan.tail[static_cast<size_t>(k) * L + j]);
        const int32_t x = static_cast<int32_t>(std::lower_bound(xs.begin(), xs.end(), scan.x[k]) -
                                               xs.begin());
        at.push_back(Place{h, x, scan.y[k], k});
    }
    std::sort(at.begin(), at.end(), [&](const Place &a, const Place &b) {
        if (a.tails != b.tails) return a.tails < b.tails;
        if (a.x != b.x) return a.x < b.x;
        return a.y != b.y ? a.y < b.y : a.k < b.k;
    });
    struct Block {
        int32_t chunk, y;
        std::vector<int32_t> comm;
    };
    std::vector<Block> blocks;
    for (size_t i = 0; i < at.size();) {
        const int32_t chunk = at[i].x / L;
        size_t end = i;
        bool twice = false;
        while (end < at.size() && at[end].tails == at[i].tails && at[end].x / L == chunk) {
            twice = twice || (end > i && at[end].x == at[end - 1].x);
            ++end;
        }
        for (size_t q = i; q < end; ++q) {
            const bool open = q == i || (twice && blocks.back().comm.back() >= 0);
            if (open) {
                blocks.push_back(Block{chunk, at[q].y, std::vector<int32_t>(L, -1)});
            }
            std::vector<int32_t> &c = blocks.back().comm;
            if (twice) *std::find(c.begin(), c.end(), -1) = at[q].k;
            else c[at[q].x % L] = at[q].k;
        }
        i = end;
    }
    // Blocks side by side in a wave should be of different sources and different destinations: their
    // loads then fall on different links (scan and scatter of a wave with the same four sources in all
    // its blocks took 2600 cycles, 1600 this way: 16 nodes on one XCD).  So they are taken diagonal by
    // diagonal of the sources x destinations.
    std::vector<int32_t> ys;
    for (const Block &b : blocks) ys.push_back(b.y);
    std::sort(ys.begin(), ys.end());
    ys.erase(std::unique(ys.begin(), ys.end()), ys.end());
    const int32_t chunks = static_cast<int32_t>((xs.size() + L - 1) / L);
    const int32_t across = std::max<int32_t>(chunks, static_cast<int32_t>(ys.size()));
    auto key = [&](const Block &b) {
        const int32_t y = static_cast<int32_t>(std::lower_bound(ys.begin(), ys.end(), b.y) - ys.begin());
        const int32_t diagonal = (y - b.chunk + across) % across;
        return std::make_tuple(diagonal % chunks, diagonal / chunks, b.chunk);
    };
    std::sort(blocks.begin(), blocks.end(), [&](const Block &a, const Block &b) {
        const auto ka = key(a), kb = key(b);
        return ka != kb ? ka < kb : a.comm < b.comm;
    });
    std::unordered_map<uint64_t, int32_t> heads, tails;
    auto number = [](std::unordered_map<uint64_t, int32_t> &all, uint64_t h, size_t where,
                     std::vector<int32_t> &first) {
        const auto it = all.emplace(h, static_cast<int32_t>(all.size()));
        if (it.second) first.push_back(static_cast<int32_t>(where));
        return it.first->second;
    };
    for (size_t b = 0; b < blocks.size(); ++b) {
        out.comm.insert(out.comm.end(), blocks[b].comm.begin(), blocks[b].comm.end());
        for (int32_t j = 0; j < L; ++j) {
            uint64_t h = 4, tail = 0;
            for (int32_t k : blocks[b].comm) {
                h = mixed(h, k < 0 ? 0u : scan.head[static_cast<size_t>(k) * L + j]);
                if (k >= 0) tail = scan.tail[static_cast<size_t>(k) * L + j];
            }
            out.head.push_back(number(heads, h, b * L + j, out.head_at));
            out.tail.push_back(number(tails, tail, b * L + j, out.tail_at));
        }
    }
}

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
    if (product_fits && most[0] > 1) scan_blocks(n_links, n_comm, cp, lp, pl, most[0], out);
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

void cut_patches(int32_t n_comm, const PatchScan &scan, PatchGrid strips, PatchCut &out)
{
    out = PatchCut();
    std::vector<std::vector<int32_t>> grid(static_cast<size_t>(strips.x) * strips.y);
    if (strips.x * strips.y == 1) {
        grid[0].resize(n_comm);
        for (int32_t k = 0; k < n_comm; ++k) grid[0][k] = k;
    } else {
        const std::vector<int32_t> sx = cut(scan.x_count, scan.x_cross, strips.x);
        const std::vector<int32_t> sy = cut(scan.y_count, scan.y_cross, strips.y);
        for (int32_t k = 0; k < n_comm; ++k)
            grid[static_cast<size_t>(sx[scan.x[k]]) * strips.y + sy[scan.y[k]]].push_back(k);
    }
    // Patch p runs on XCD p modulo kPatchXcds.  A quarter of the columns and half of the rows of the
    // grid go to each: of the patches that share links most are then on few XCDs (64 nodes of 8 in
    // 16 x 16 patches 7.20 -> 6.96 us per iteration, 16 nodes 2.28 -> 2.25 against XCDs that have
    // whole columns, which is what the grid's own order comes to).
    std::vector<std::pair<int32_t, size_t>> order;
    for (size_t q = 0; q < grid.size(); ++q) {
        const int32_t r = static_cast<int32_t>(q) / strips.y, c = static_cast<int32_t>(q) % strips.y;
        if (!grid[q].empty()) order.emplace_back(4 * (2 * r / strips.x) + 4 * c / strips.y, q);
    }
    std::sort(order.begin(), order.end());
    std::vector<size_t> dealt(order.size());
    size_t next = 0;
    for (size_t x = 0; x < kPatchXcds; ++x)
        for (size_t p = x; p < dealt.size(); p += kPatchXcds) dealt[p] = order[next++].second;
    for (size_t q : dealt) {
        out.most = std::max<int64_t>(out.most, static_cast<int64_t>(grid[q].size()));
        out.members.push_back(std::move(grid[q]));
    }
}

double patch_scan_us(const PatchShape &s)
{
    // cycles the LDS is busy (four per price read of a wave, more per atomic the more lanes add)
    // and cycles of vector issue; a wave's own chain of reads and additions on top
    const double waves = s.threads / 64.0;
    const double lds = waves * (s.quads * (s.product ? 36.0 : 80.0) + 50.0 + 80.0 / s.lanes);
    const double valu = waves * (s.quads * (s.product ? 28.0 : 50.0) + (s.lanes > 1 ? 85.0 : 70.0));
    // (Fabrics of one patch, 240 to 992 pairs, us measured and by this: 2 nodes of 8 0.83 and 0.84, with two
    // NICs in reach of a GPU 1.23 and 1.15, 4 nodes of 6 1.27 and 1.21, 3 of 8 1.45 and 1.38, 8 of 4 with a NIC
    // per GPU 1.72 and 1.55, 3 of 8 with two in reach 2.23 and 2.07.)
    return 0.88 * (0.3 + 0.06 * s.quads + std::max(lds, valu) / 2400.0);
}

double patch_iteration_us(const PatchShape &s, const PatchSizes &m, bool near)
{
    if (m.patches < 2 || m.max_groups == 0) return patch_scan_us(s);
    // Fitted to 2352 measured layouts: 51 fabrics of 2 to 64 nodes in every square grid and in those
    // rectangular ones that fit an XCD, as slots and as blocks.  Within 9 to 11 % of the measured
    // time for nine of ten layouts (27 % for all); the grid with the lowest estimate takes 1.6 % longer
    // than the fastest on average (the worst, 8 x 8 for 8 nodes of 8, 19 %).  Terms: the words of a
    // link's users, asked for four, eight or sixteen at a time, round after round of links; the links
    // a patch publishes; the words it reads; then what the commodities take.
    const double waves = s.threads / 64.0;
    const int32_t lanes = patch_link_lanes(s.threads, patch_row(m.max_groups));
    const int32_t per_round = s.threads / lanes;
    const double rounds = (m.max_groups * kPatchGroup + per_round - 1) / per_round;
    const int32_t words = (m.max_users + lanes - 1) / lanes;
    const double asked = words <= 4 ? 4.0 : words <= 8 ? 8.0 : 16.0 * ((words + 15) / 16);
    const double links = m.max_groups * kPatchGroup / 64.0, at = m.max_at / 100.0;
    if (!s.blocks) {
        const double slots = waves * s.quads;
        return near ? 1.056 + slots * (s.product ? 0.0157 : 0.0441) + 0.129 * s.quads + 0.0534 * rounds * asked +
                          0.0209 * links + 0.0461 * at
                    : 1.083 + slots * (s.product ? 0.0207 : 0.0582) + 0.143 * s.quads + 0.0543 * rounds * asked +
                          0.0598 * links + 0.0179 * at;
    }
    const double comm = m.max_comm / 64.0, scans = comm * s.lanes * (s.product ? 2.0 : 1.0);
    const double folds = (m.max_heads * s.lanes + s.threads - 1) / s.threads;
    return near ? 0.812 + 0.0088 * comm + 0.0047 * scans + 0.045 * waves + 0.195 * folds +
                      0.0642 * rounds * asked + 0.0669 * at + 6.8e-6 * m.max_at * m.patches
                : 1.201 + 0.0185 * comm + 0.005 * scans + 0.0021 * waves + 0.402 * folds +
                      0.0538 * rounds * asked + 0.0469 * links + 0.0694 * at;
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
        int32_t groups = 0, own = 0, at = 0;
        for (int32_t e : links[b]) {
            own += users[e] == 1 ? 1 : 0;
            m.max_users = std::max(m.max_users, users[e]);
            groups += groups_of_first[e];
            at += groups_of_first[e] * users[e];
        }
        m.max_groups = std::max(m.max_groups, groups);
        m.max_at = std::max(m.max_at, at);
        m.max_private = std::max(m.max_private, own);
        m.max_local = std::max(m.max_local, groups * kPatchGroup + own);
    }
    m.patches = B;
    m.max_comm = static_cast<int32_t>(cut.most);
    // (prices, link states, groups and counts: lds_layout in patch_kernel.hpp)
    const int64_t links_lds = 48ll * m.max_local + 2ll * m.max_at + 4ll * m.max_groups + 512;
    const int64_t slots = static_cast<int64_t>(m.max_comm) * shape.lanes * shape.quads;
    m.fits = m.max_local <= kPatchMaxLocal && links_lds + 8 * slots <= kPatchLdsBytes &&
             static_cast<int64_t>(B) * patch_row(m.max_groups) <= kPatchMaxUnits;
    m.fits_adaptive = m.fits && links_lds + 32 * slots <= kPatchLdsBytes;
    return m;
}

bool measure_blocks(const PatchScan &scan, const PatchCut &cut, PatchSizes &m, PatchShape &shape)
{
    const int32_t L = scan.block_lanes;
    if (L == 0 || m.max_local > kPatchMaxLocal || m.max_groups == 0 ||
        static_cast<int64_t>(m.patches) * patch_row(m.max_groups) > kPatchMaxUnits)
        return false;
    std::atomic<size_t> most_comm{0}, most_heads{0}, most_tails{0};
    auto raise = [](std::atomic<size_t> &m, size_t v) {
        size_t old = m.load();
        while (old < v && !m.compare_exchange_weak(old, v)) {
        }
    };
    parallel_ranges(static_cast<int64_t>(cut.members.size()), [&](int64_t b0, int64_t b1) {
        PatchBlocks pb;
        for (int64_t b = b0; b < b1 && most_comm.load() <= static_cast<size_t>(kPatchThreads); ++b) {
            find_blocks(scan, cut.members[static_cast<size_t>(b)], pb);
            raise(most_comm, pb.comm.size());
            raise(most_heads, pb.head_at.size());
            raise(most_tails, pb.tail_at.size());
        }
    }, std::max<int64_t>(1, 4096 / std::max<int64_t>(1, cut.most)));
    const size_t comm = most_comm.load(), heads = most_heads.load(), tails = most_tails.load();
    if (comm > static_cast<size_t>(kPatchThreads)) return false;
    shape = PatchShape();
    shape.blocks = 1;
    shape.product = scan.block_product;
    shape.lanes = L;
    shape.quads = 1;
    m.max_comm = static_cast<int32_t>(comm);
    m.max_heads = static_cast<int32_t>(heads);
    m.max_tails = static_cast<int32_t>(tails);
    // a thread per lane of a block, per shared link, per other link and per head, as far as there are
    const int32_t want = std::max({m.max_comm, m.max_groups * kPatchGroup, m.max_private,
                                  std::min(kPatchThreads, m.max_heads * L)});
    shape.threads = (want + 63) / 64 * 64;
    if (shape.threads > kPatchThreads) return false;
    const int64_t fixed = block_lds(m.max_local, m.max_heads, m.max_tails, 0, m.max_at, shape, 0).bytes;
    const int64_t slots = static_cast<int64_t>(m.max_comm) * L;
    m.fits = fixed + 8 * slots <= kPatchLdsBytes;
    m.fits_adaptive = false;                                 // (there are no such kernels)
    return m.fits;
}

std::vector<PatchOption> choose_cuts(int32_t n_links, int32_t n_comm, const PatchScan &scan,
                                     int32_t cus, int32_t xcds, const PatchForced &forced)
{
    xcds = std::max(1, xcds);
    const int32_t cus_of_xcd = cus / xcds;
    auto estimate = [&](PatchOption &o) {
        o.spread_us = patch_iteration_us(o.shape, o.sizes, false);
        o.us = o.sizes.patches <= cus_of_xcd ? patch_iteration_us(o.shape, o.sizes, true) : o.spread_us;
    };
    std::vector<PatchGrid> grids;
    if (forced.grid.x > 0) {
        grids.push_back(forced.grid);
    } else {
        for (int32_t s = 1; s * s <= cus; ++s) grids.push_back(PatchGrid{s, s});
        // and some that fit an XCD (a list, not a rule: 4 x 7 is what 7 nodes of 6 run on, 3 x 6, its like for
        // six nodes, is not here)
        for (const PatchGrid &g : {PatchGrid{2, 3}, PatchGrid{2, 4}, PatchGrid{3, 4}, PatchGrid{3, 5},
                                   PatchGrid{4, 5}, PatchGrid{4, 7}, PatchGrid{4, 8}, PatchGrid{5, 6},
                                   PatchGrid{8, 4}})
            if (g.x * g.y <= cus_of_xcd) grids.push_back(g);
    }
    // (most grids are ruled out by their size alone)
    grids.erase(std::remove_if(grids.begin(), grids.end(), [&](const PatchGrid &g) {
        return n_comm > static_cast<int64_t>(g.x) * g.y * kPatchThreads;
    }), grids.end());
    std::vector<PatchOption> tried(2 * grids.size());       // slots, blocks
    std::vector<PatchCut> cuts(grids.size());
    auto try_slots = [&](size_t i) {
        cut_patches(n_comm, scan, grids[i], cuts[i]);
        if (static_cast<int64_t>(cuts[i].members.size()) > cus) return;
        PatchOption &o = tried[2 * i];
        o.grid = grids[i];
        const bool fits = patch_shape(scan, cuts[i].most, forced.lanes, o.shape);
        o.sizes = measure_cut(n_links, scan, cuts[i], o.shape);
        tried[2 * i + 1].sizes = o.sizes;
        tried[2 * i + 1].sizes.fits = tried[2 * i + 1].sizes.fits_adaptive = false;
        if (!fits || forced.blocks == 1) o.sizes.fits = o.sizes.fits_adaptive = false;
        if (o.sizes.fits) estimate(o);
    };
    // microseconds of an iteration of as many plans as there is room for, per plan; near teams where they
    // fit an XCD (rated by the spread ones where more of those fit, layouts of 25 patches took the place of
    // 28 to 32 on 13 of 275 fabrics: 1.4 to 1.7 times as fast for 9 and 10 plans, 0.86 to 0.98 for 2
    // to 8, 12, 16, 24, 32 and 64)
    auto shared_us = [&](const PatchOption &o) {
        const PatchTeams t = patch_teams(o.sizes.patches, cus, xcds);
        return t.near > 0 ? o.us / t.near : o.spread_us / t.spread;
    };
    double best_us = 1e30, best_shared = 1e30;
    // what the blocks of a cut come to at best is known without looking for them
    auto least_of = [&](size_t i) {
        PatchOption least = tried[2 * i + 1];
        least.sizes.max_comm = static_cast<int32_t>(cuts[i].most);
        least.shape.blocks = 1;
        least.shape.lanes = scan.block_lanes;
        least.shape.product = scan.block_product;
        least.shape.threads = std::max(64, (std::max(least.sizes.max_comm,
                                                     kPatchGroup * least.sizes.max_groups) + 63) / 64 * 64);
        estimate(least);
        return least;
    };
    auto try_blocks = [&](size_t i, const PatchOption &least) {
        PatchOption &o = tried[2 * i + 1];
        o.grid = grids[i];
        if ((forced.blocks < 0 && least.us >= best_us && shared_us(least) >= best_shared) ||
            !measure_blocks(scan, cuts[i], o.sizes, o.shape)) {
            o.sizes.fits = false;
            return;
        }
        estimate(o);
        best_us = std::min(best_us, o.us);
        best_shared = std::min(best_shared, shared_us(o));
    };
    // One patch that is done before words could go from patch to patch needs no comparison.  (Eight fabrics of
    // 240 to 756 pairs for which the estimate says so: all are fastest on one patch, 0.8 to 1.3 us an iteration,
    // 1.5 to 1.9 on 4 to 16 patches.)
    size_t from = 0;
    if (!grids.empty() && grids[0] == PatchGrid{1, 1}) {
        try_slots(from++);
        if (tried[0].sizes.fits_adaptive && tried[0].us < kPatchTripUs) return {tried[0]};
    }
    const int64_t rest = static_cast<int64_t>(grids.size() - from), grain = n_comm < 1024 ? 16 : 1;
    parallel_ranges(rest, [&](int64_t g0, int64_t g1) {
        for (int64_t g = g0; g < g1; ++g) try_slots(from + static_cast<size_t>(g));
    }, grain);
    for (const PatchOption &o : tried)
        if (o.sizes.fits && o.shape.blocks == 0 && o.us > 0.0) {
            best_us = std::min(best_us, o.us);
            best_shared = std::min(best_shared, shared_us(o));
        }
    if (scan.block_lanes > 0 && forced.blocks != 0 && (forced.lanes == 0 || forced.blocks > 0)) {
        // the most promising first: most of the others need no look then
        std::vector<std::pair<size_t, PatchOption>> least;
        for (size_t i = from; i < grids.size(); ++i)
            if (tried[2 * i + 1].sizes.patches > 1) least.emplace_back(i, least_of(i));
        std::sort(least.begin(), least.end(), [](const auto &a, const auto &b) {
            return a.second.us != b.second.us ? a.second.us < b.second.us : a.first < b.first;
        });
        for (const auto &c : least) try_blocks(c.first, c.second);
    }
    const PatchOption *best = nullptr, *most = nullptr, *adaptive = nullptr;
    for (const PatchOption &o : tried) {
        if (!o.sizes.fits) continue;
        if (best == nullptr || o.us < best->us) best = &o;
        if (most == nullptr || shared_us(o) < shared_us(*most)) most = &o;
        if (o.sizes.fits_adaptive &&
            (adaptive == nullptr || variable_step_us(o.sizes.patches, o.us) <
                                        variable_step_us(adaptive->sizes.patches, adaptive->us)))
            adaptive = &o;
    }
    std::vector<PatchOption> out;
    if (best == nullptr) return out;
    out.push_back(*best);
    if (most != best) out.push_back(*most);
    if (adaptive != nullptr && adaptive != best && adaptive != most) {
        out.push_back(*adaptive);
        out.back().variable_only = true;
    }
    return out;
}

bool build_patches(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                   const int32_t *pl, const PatchScan &scan, PatchCut &cut,
                   const PatchShape &shape, PatchLayout &out)
{
    out = PatchLayout();
    out.shape = shape;
    const bool product = shape.product != 0, blocks = shape.blocks != 0;
    const int32_t L = shape.lanes, QL = shape.quads, NT = shape.threads;
    const int32_t NW = product ? kPatchWordsProduct : kPatchWordsPlain;
    std::vector<std::vector<int32_t>> &members = cut.members;
    const int32_t B = static_cast<int32_t>(members.size());
    if (!blocks && cut.most * L > NT) return false;
    // Lanes that work side by side should hold commodities of different sources and different
    // destinations: their loads then fall on different links.  So a patch's commodities are taken
    // diagonal by diagonal of its source x destination table.
    parallel_ranges(blocks ? 0 : B, [&](int64_t b0, int64_t b1) {
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
        std::vector<int32_t> local;              // its number among the groups of each user
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
                groups.push_back(Group{{}, &users[e], {}});
                out.max_users = std::max(out.max_users, static_cast<int32_t>(users[e].size()));
                for (int32_t b : users[e]) {
                    groups.back().local.push_back(static_cast<int32_t>(groups_of[b].size()));
                    groups_of[b].push_back(g);
                }
                if (it == open.end()) it = open.emplace(users[e], g).first;
                else it->second = g;
            }
            groups[it->second].links.push_back(e);
        }
    }
    std::vector<PatchBlocks> pb(blocks ? B : 0);
    if (blocks)
        parallel_ranges(B, [&](int64_t b0, int64_t b1) {
            for (int64_t q = b0; q < b1; ++q) find_blocks(scan, members[q], pb[q]);
        });
    // local numbering: the groups (padded), then the private links
    out.desc.assign(static_cast<size_t>(kPatchDescInts) * B, 0);
    std::vector<int32_t> first_local(B + 1, 0), first_group(B + 1, 0);
    std::vector<int32_t> first_comm(B + 1, 0), first_head(B + 1, 0), first_tail(B + 1, 0);
    for (int32_t b = 0; b < B; ++b) {
        int32_t n_private = 0, n_at = 0;
        for (int32_t e : links[b]) n_private += users[e].size() == 1 ? 1 : 0;
        for (int32_t g : groups_of[b]) n_at += static_cast<int32_t>(groups[g].users->size());
        const int32_t ng = static_cast<int32_t>(groups_of[b].size());
        const int32_t n_local = ng * kPatchGroup + n_private;
        if (n_local > kPatchMaxLocal) return false;
        first_local[b + 1] = first_local[b] + n_local;
        first_group[b + 1] = first_group[b] + ng;
        out.max_local = std::max(out.max_local, n_local);
        out.max_groups = std::max(out.max_groups, ng);
        out.max_at = std::max(out.max_at, n_at);
        int32_t *d = &out.desc[static_cast<size_t>(kPatchDescInts) * b];
        d[0] = first_local[b];
        d[1] = n_local;
        d[2] = ng * kPatchGroup;
        d[3] = first_group[b] + b;               // (one entry more per patch)
        d[4] = ng;
        d[5] = first_comm[b];
        d[6] = static_cast<int32_t>(blocks ? pb[b].comm.size() : members[b].size());
        first_comm[b + 1] = first_comm[b] + d[6];
        if (blocks) {
            d[8] = first_head[b];
            d[9] = static_cast<int32_t>(pb[b].head_at.size());
            d[10] = first_tail[b];
            d[11] = static_cast<int32_t>(pb[b].tail_at.size());
            first_head[b + 1] = d[8] + d[9];
            first_tail[b + 1] = d[10] + d[11];
            out.max_heads = std::max(out.max_heads, d[9]);
            out.max_tails = std::max(out.max_tails, d[11]);
            if (d[6] > NT || ng * kPatchGroup > NT || n_private > NT) return false;
        }
        out.max_comm = std::max(out.max_comm, d[6]);
    }
    out.row = patch_row(out.max_groups);
    if (static_cast<int64_t>(B) * out.row > kPatchMaxUnits) return false;
    out.n_parts = static_cast<int64_t>(B) * out.row * kPatchGroup;
    out.loc_link.assign(first_local[B], -1);
    for (int32_t b = 0; b < B; ++b) {
        out.desc[static_cast<size_t>(kPatchDescInts) * b + 7] = static_cast<int32_t>(out.at.size());
        int32_t n = 0;
        for (int32_t g : groups_of[b]) {
            out.group.push_back(n);
            n += static_cast<int32_t>(groups[g].users->size());
            for (size_t u = 0; u < groups[g].users->size(); ++u)
                out.at.push_back(static_cast<uint16_t>((*groups[g].users)[u] * out.row + groups[g].local[u]));
        }
        out.group.push_back(n);
    }
    out.comm.assign(first_comm[B], -1);
    out.words.assign(static_cast<size_t>(B) * (blocks ? 1 : QL * NW) * NT, 0u);
    out.first.assign(static_cast<size_t>(B) * (blocks ? L : QL) * NT, 0u);
    out.heads.assign(static_cast<size_t>(first_head[B]) * L * 4, 0u);
    out.tails.assign(static_cast<size_t>(first_tail[B]) * 2, 0u);
    std::atomic<bool> alike{true};               // what has one number is one head or tail
    parallel_ranges(B, [&](int64_t b0, int64_t b1) {
        std::vector<int32_t> local(n_links, 0), seen(n_links, -1);
        Slot slot[32];
        for (int32_t b = static_cast<int32_t>(b0); b < b1; ++b) {
            int32_t at = 0;
            for (size_t gi = 0; gi < groups_of[b].size(); ++gi) {
                const Group &g = groups[groups_of[b][gi]];
                const bool exports = g.users->front() == b;
                for (int32_t q = 0; q < kPatchGroup; ++q, ++at)
                    if (q < static_cast<int32_t>(g.links.size())) {
                        const int32_t e = g.links[q];
                        out.loc_link[first_local[b] + at] = e | (exports ? kPatchExport : 0);
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
            if (blocks) {
                const PatchBlocks &p = pb[b];
                const size_t n_lanes = p.head.size();
                std::copy(p.comm.begin(), p.comm.end(), out.comm.begin() + first_comm[b]);
                // the slots of every place, [block * lanes + place][slot]
                std::vector<Slot> all(n_lanes * L);
                for (size_t c = 0; c < n_lanes; ++c) {
                    const int32_t k = p.comm[c];
                    const int32_t n = k < 0 ? 0 : slots_of(cp[k + 1] - cp[k], cp[k], lp, pl, true, slot,
                                                           scan.place.data());
                    for (int32_t j = 0; j < L; ++j) {
                        Slot &s = all[c * L + j];
                        if (j < n) {
                            s = slot[j];
                            continue;
                        }
                        for (int32_t x = 0; x < 9; ++x) s.at[x] = x == A0 || x == A2 ? kInf : kZero;
                        s.at[D0] = s.at[D1] = kInf;
                        s.base = s.shift = s.n = 0;
                    }
                }
                auto at = [&](size_t lane, int32_t place) -> const Slot & {
                    return all[(lane / L * L + place) * L + lane % L];
                };
                // the thread that holds lane j of a block: its commodities' lanes lie a stride of 16,
                // 32 and 8 lanes apart (patch_blocks.hpp)
                auto thread_of = [&](size_t lane) { return block_thread(static_cast<int32_t>(lane / L),
                                                                        static_cast<int32_t>(lane % L), L); };
                for (size_t c = 0; c < n_lanes; ++c)
                    for (int32_t j = 0; j < L; ++j) {
                        const Slot &s = all[c * L + j];
                        uint32_t once = 0u;
                        for (int32_t x = 0; x < 9 && s.n > 0; ++x)
                            if (s.at[x] >= 0 && seen[s.at[x]] != p.comm[c]) {
                                seen[s.at[x]] = p.comm[c];
                                once |= 1u << x;
                            }
                        out.first[(static_cast<size_t>(b) * L + c % L) * NT + thread_of(c / L * L + j)] =
                            static_cast<uint32_t>(s.base | s.shift << 7 | s.n << 9) | once << 12;
                    }
                auto tail_of = [&](size_t lane) -> const Slot & {      // of any commodity there is
                    for (int32_t i = 0; i < L; ++i)
                        if (p.comm[lane / L * L + i] >= 0) return at(lane, i);
                    return at(lane, 0);
                };
                for (size_t lane = 0; lane < n_lanes; ++lane) {
                    const size_t h0 = static_cast<size_t>(p.head_at[p.head[lane]]);
                    const size_t t0 = static_cast<size_t>(p.tail_at[p.tail[lane]]);
                    const Slot &way = tail_of(t0);
                    for (int32_t i = 0; i < L; ++i) {
                        const Slot &s = at(lane, i), &f = at(h0, i);
                        bool same_as = true;
                        for (int32_t x : kHeadAt) same_as = same_as && s.at[x] == f.at[x];
                        if (p.comm[lane / L * L + i] >= 0)
                            for (int32_t x : kTailAt) same_as = same_as && s.at[x] == way.at[x];
                        if (!same_as) alike.store(false);
                        if (h0 == lane) {
                            uint32_t *w = &out.heads[(static_cast<size_t>(first_head[b] + p.head[lane]) *
                                                          L + i) * 4];
                            w[0] = offset(s.at[A0]) | offset(s.at[A2]) << 16;
                            w[1] = offset(s.at[B0]) | offset(s.at[B2]) << 16;
                            w[2] = offset(s.at[C]);
                        }
                    }
                    out.words[static_cast<size_t>(b) * NT + thread_of(lane)] =
                        static_cast<uint32_t>(p.head[lane] | p.tail[lane] << kBlockIdBits |
                                              static_cast<int32_t>(lane % L) << 2 * kBlockIdBits);
                    if (t0 == lane) {
                        uint32_t *w = &out.tails[static_cast<size_t>(first_tail[b] + p.tail[lane]) * 2];
                        w[0] = offset(way.at[D0]) | offset(way.at[D1]) << 16;
                        w[1] = offset(way.at[E0]) | offset(way.at[E1]) << 16;
                    }
                }
                continue;
            }
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
    if (!alike.load()) return false;
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
    std::vector<int32_t> uses(n_links, 0);
    std::vector<std::vector<int32_t>> shared_by(n_links);
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
            // every user of the group is listed once, in ascending order, this patch among them, and has
            // the group where it says, with the same links
            const int32_t from = t.group[d[3] + g], to = t.group[d[3] + g + 1];
            if (from < 0 || to - from < 2 || to - from > t.max_users || to > t.max_at) return 5;
            std::vector<int32_t> mine(kPatchGroup);
            for (int32_t i = 0; i < kPatchGroup; ++i) {
                const int32_t v = ll[g * kPatchGroup + i];
                mine[i] = v == -1 ? -1 : v & ~kPatchExport;
                if (mine[i] >= 0) shared_by[mine[i]].push_back(b);
            }
            bool own = false;
            for (int32_t u = from, last = -1; u < to; ++u) {
                const int32_t who = t.at[d[7] + u] / t.row, where = t.at[d[7] + u] % t.row;
                if (who <= last || who >= t.n_patches) return 6;
                last = who;
                own = own || (who == b && where == g);
                const int32_t *od = &t.desc[static_cast<size_t>(kPatchDescInts) * who];
                if (where >= od[4] || t.group[od[3] + where + 1] - t.group[od[3] + where] != to - from) return 6;
                for (int32_t i = 0; i < kPatchGroup; ++i) {
                    const int32_t v = t.loc_link[od[0] + where * kPatchGroup + i];
                    if ((v == -1 ? -1 : v & ~kPatchExport) != mine[i]) return 7;
                }
            }
            if (!own) return 6;
        }
        for (int32_t i = 0; i < n_local; ++i)
            if (ll[i] >= 0) uses[ll[i] & ~kPatchExport] += 1;
        if (t.shape.blocks) {
            const int32_t zero = 8 * n_local, inf = zero + 8;
            if (d[6] % L || d[6] > NT) return 18;
            for (int32_t c = 0; c < d[6]; ++c) {
                const int32_t k = t.comm[d[5] + c];
                std::vector<int32_t> used;
                int32_t next = 0;
                for (int32_t j = 0; j < L; ++j) {
                    const int32_t th = block_thread(c / L, j, L);
                    if (th >= NT) return 18;
                    const uint32_t id = t.words[static_cast<size_t>(b) * NT + th];
                    const uint32_t mask = (1u << kBlockIdBits) - 1u;
                    const int32_t head = static_cast<int32_t>(id & mask);
                    const int32_t tail = static_cast<int32_t>(id >> kBlockIdBits & mask);
                    if (static_cast<int32_t>(id >> 2 * kBlockIdBits) != j || head >= d[9] || tail >= d[11])
                        return 21;
                    const uint32_t *hw = &t.heads[(static_cast<size_t>(d[8] + head) * L + c % L) * 4];
                    const uint32_t *tw = &t.tails[static_cast<size_t>(d[10] + tail) * 2];
                    const uint32_t o[9] = {hw[0] & 0xFFFFu, hw[0] >> 16, hw[1] & 0xFFFFu, hw[1] >> 16,
                                           hw[2], tw[0] & 0xFFFFu, tw[0] >> 16, tw[1] & 0xFFFFu,
                                           tw[1] >> 16};
                    for (uint32_t x : o)
                        if (x % 8 || x > static_cast<uint32_t>(inf)) return 8;
                    const uint32_t first =
                        t.first[(static_cast<size_t>(b) * L + c % L) * NT + th];
                    const int32_t base = first & 127, shift = (first >> 7) & 3, n = (first >> 9) & 7;
                    if (k < 0 && first != 0u) return 20;
                    for (int32_t x = 0; x < 9; ++x)
                        if ((first >> (12 + x)) & 1u) {
                            if (o[x] >= static_cast<uint32_t>(zero)) return 9;
                            used.push_back(ll[o[x] / 8] & ~kPatchExport);
                        }
                    if (n > 0 && (k < 0 || base != next)) return 10;
                    next += n;
                    for (int32_t pos = 0; pos < 4; ++pos) {
                        const int32_t h = pos >> 1, l = pos & 1, q = pos >> shift;
                        std::vector<int32_t> path;
                        bool ok = t.shape.product != 0 || l == 0;
                        for (int32_t x : {A0 + h, B0 + h, int32_t(C), D0 + l, E0 + l}) {
                            if (o[x] < static_cast<uint32_t>(zero)) path.push_back(ll[o[x] / 8] & ~kPatchExport);
                            ok = ok && o[x] != static_cast<uint32_t>(inf);
                        }
                        const bool there = n > 0 && (pos & ((1 << shift) - 1)) == 0 && q < n;
                        if (ok != there) return 12;
                        if (!there) continue;
                        const int32_t p = cp[k] + base + q;
                        if (p >= cp[k + 1] || path != std::vector<int32_t>(pl + lp[p], pl + lp[p + 1]))
                            return 11;
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
            continue;
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
    // a link in several patches is shared by all of them, and by as many as its group says
    for (int32_t e = 0; e < n_links; ++e)
        if (uses[e] > 1 ? static_cast<int32_t>(shared_by[e].size()) != uses[e] : !shared_by[e].empty())
            return 16;
    std::vector<uint8_t> in_use(n_links, 0);
    for (int32_t q = 0; q < lp[cp[n_comm]]; ++q) in_use[pl[q]] = 1;
    for (int32_t e = 0; e < n_links; ++e)
        if (exported[e] != in_use[e]) return 17;
    return 0;
}

namespace {

// `out` of nimble_host_patch_check and, `more`, what nimble_host_grid_check adds
nimble_status_t host_check(int32_t n_links, int32_t n_comm, const int32_t *cp, const int32_t *lp,
                           const int32_t *pl, PatchGrid grid, int32_t lanes, bool blocks, bool more,
                           int64_t *out)
{
    PatchScan scan;
    PatchLayout t;
    PatchCut cut;
    PatchShape shape;
    PatchSizes m;
    scan_patches(n_links, n_comm, cp, lp, pl, scan);
    if (scan.fits) cut_patches(n_comm, scan, grid, cut);
    bool fits = scan.fits;
    if (fits && blocks) {
        m = measure_cut(n_links, scan, cut, shape);
        fits = measure_blocks(scan, cut, m, shape);
    } else if (fits) {
        fits = patch_shape(scan, cut.most, lanes, shape);
        if (fits) m = measure_cut(n_links, scan, cut, shape);
    }
    if (fits) build_patches(n_links, n_comm, cp, lp, pl, scan, cut, shape, t);
    out[0] = t.n_patches;
    out[1] = t.n_patches > 0 ? check_patches(n_links, n_comm, cp, lp, pl, t) : 0;
    // what is found without building a layout is what it has
    if (t.n_patches > 0 && out[1] == 0 &&
        (m.patches != t.n_patches || m.max_comm != t.max_comm || m.max_local != t.max_local ||
         m.max_groups != t.max_groups || m.max_heads != t.max_heads ||
         m.max_tails != t.max_tails || m.max_at != t.max_at))
        out[1] = 19;
    out[2] = t.shape.product;
    out[3] = t.shape.lanes;
    out[4] = t.shape.quads;
    out[5] = t.shape.threads;
    out[6] = t.max_local;
    out[7] = t.max_groups;
    out[8] = t.max_users;
    out[9] = t.max_at;
    out[10] = t.n_parts;
    if (more) {
        out[11] = t.max_comm;
        out[12] = t.max_heads;
        out[13] = t.max_tails;
        out[14] = m.max_private;
    }
    return NIMBLE_OK;
}

}  // namespace

}  // namespace nimble

extern "C" nimble_status_t nimble_host_patch_choice(int32_t n_links, int32_t n_comm,
                                                     const int32_t *comm_path_ptr, int32_t n_paths,
                                                     const int32_t *path_link_ptr,
                                                     const int32_t *path_links, int32_t cus, int32_t xcds,
                                                     int32_t strips_x, int32_t strips_y, int32_t lanes,
                                                     int32_t blocks, int64_t *out, int32_t *n_out)
{
    try {
        std::string why;
        const nimble_status_t st = nimble::validate_csr(n_links, nullptr, n_comm, comm_path_ptr, n_paths,
                                                        path_link_ptr, path_links, why);
        if (st != NIMBLE_OK) return st;
        if (!out || !n_out || cus < 1 || xcds < 1 || lanes < 0) return NIMBLE_ERR_INVALID;
        nimble::PatchForced forced;
        forced.grid = nimble::PatchGrid{strips_x, strips_y};
        forced.lanes = lanes;
        forced.blocks = blocks;
        *n_out = 0;
        nimble::PatchScan scan;
        nimble::scan_patches(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links, scan);
        if (!scan.fits) return NIMBLE_OK;
        for (const nimble::PatchOption &o :
             nimble::choose_cuts(n_links, n_comm, scan, cus, xcds, forced)) {
            nimble::PatchCut cut;
            nimble::PatchLayout built;
            nimble::cut_patches(n_comm, scan, o.grid, cut);
            int64_t *row = out + 8 * (*n_out)++;
            row[0] = o.grid.x;
            row[1] = o.grid.y;
            row[2] = o.sizes.patches;
            row[3] = o.sizes.max_groups;
            row[4] = o.shape.blocks;
            row[5] = o.shape.lanes;
            row[6] = o.variable_only ? 1 : 0;
            row[7] = -1;
            if (nimble::build_patches(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links, scan, cut,
                                      o.shape, built))
                row[7] = nimble::check_patches(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links,
                                               built);
        }
        return NIMBLE_OK;
    } catch (const std::exception &) {
        return NIMBLE_ERR_ALLOC;
    }
}

extern "C" nimble_status_t nimble_host_patch_teams(int32_t patches, int32_t cus, int32_t xcds,
                                                    int32_t plans, double near_us, double spread_us,
                                                    int32_t *near, int32_t *teams, double *us)
{
    if (!near || !teams || !us || patches < 1 || xcds < 1 || cus < patches || plans < 1)
        return NIMBLE_ERR_INVALID;
    const nimble::PatchTeams t = nimble::patch_teams(patches, cus, xcds);
    *near = nimble::teams_keep_near(t, plans) ? 1 : 0;
    *teams = std::min(plans, *near ? t.near : t.spread);
    *us = nimble::plans_iteration_us(t, plans, near_us, spread_us);
    return NIMBLE_OK;
}

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
        return nimble::host_check(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links,
                                  nimble::PatchGrid{strips, strips}, lanes, false, false, out);
    } catch (const std::exception &) {           // out of memory, in whatever thread
        return NIMBLE_ERR_ALLOC;
    }
}

extern "C" nimble_status_t nimble_host_grid_check(int32_t n_links, int32_t n_comm,
                                                   const int32_t *comm_path_ptr, int32_t n_paths,
                                                   const int32_t *path_link_ptr,
                                                   const int32_t *path_links, int32_t strips_x,
                                                   int32_t strips_y, int32_t blocks, int64_t *out)
{
    try {
        std::string why;
        nimble_status_t st = nimble::validate_csr(n_links, nullptr, n_comm, comm_path_ptr, n_paths,
                                                  path_link_ptr, path_links, why);
        if (st != NIMBLE_OK) return st;
        if (!out || strips_x < 1 || strips_x > 64 || strips_y < 1 || strips_y > 64)
            return NIMBLE_ERR_INVALID;
        return nimble::host_check(n_links, n_comm, comm_path_ptr, path_link_ptr, path_links,
                                  nimble::PatchGrid{strips_x, strips_y}, 0, blocks != 0, true, out);
    } catch (const std::exception &) {
        return NIMBLE_ERR_ALLOC;
    }
}
