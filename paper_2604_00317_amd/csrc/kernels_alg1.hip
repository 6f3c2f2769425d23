// The sequential planner of Algorithm 1 ("Link Load Balancing w. Iterative Approximation"),
// batched, all problems on the same topology.  Two kernels compute the same numbers: a group of
// G lanes per problem whose lanes cost the candidates of a pair side by side (k_alg1_group, up
// to 64 candidates per pair), and one thread per problem (k_alg1) for anything else and for batches
// that fill the chip several times over with groups.
//
// The algorithm is a Gauss-Seidel sweep -- every routed chunk changes the link costs the next
// pair sees -- so one problem offers no parallelism beyond its candidate scan; a batch of
// problems does.  A thread keeps the link loads L_e and the remainders r_k of its problem in
// LDS (entry-major, one column per thread: conflict-free; 64 problems per workgroup, fewer when
// the topology is larger), reads the candidate CSR through
// wave-uniform loads (all threads walk the same pairs, candidates and links), and sweeps the
// pairs as Algorithm 1 does: bottleneck cost max_e c_e with c_e = F(L_e) = L_e / cap_e, strict
// `<` in candidate order, f = r if r < chi else chi * floor(r * phi / chi) (one chunk when that
// is zero), immediate update of L_e, until no remainder is left.  Every floating-point
// statement is one IEEE binary64 operation.  Both kernels are tested against the hand-worked
// examples of the algorithm directly (tests/test_gpu_alg1.py), not only against the CPU oracle.
#include <hip/hip_runtime.h>

#include <cmath>

#include "kernels.hpp"
#include "wave_ops.hpp"

namespace nimble {

namespace {

constexpr int kAlg1Threads = 64;          // most problems per workgroup
constexpr int kAlg1MinThreads = 8;        // fewest: larger topologies leave less LDS per problem
constexpr size_t kAlg1LdsBudget = 150 * 1024;
constexpr size_t kAlg1LdsPlain = 64 * 1024;      // no opt-in needed below this

__global__ __launch_bounds__(kAlg1Threads) void k_alg1(int E, int K, int P, int batch,
                                                        const int32_t *__restrict__ cp,
                                                        const int32_t *__restrict__ lp,
                                                        const int32_t *__restrict__ pl,
                                                        const double *__restrict__ invcap,
                                                        const double *__restrict__ demand,
                                                        double phi, double chi, int max_sweeps,
                                                        double *__restrict__ flows,
                                                        double *__restrict__ lambda,
                                                        int32_t *__restrict__ sweeps_out)
{
    extern __shared__ double s_state[];              // L[E][T], then r[K][T], T = blockDim.x
    const int t = threadIdx.x;
    const int T = blockDim.x;
    const int b = blockIdx.x * T + t;
    const bool live = b < batch;
    double *L = s_state + t;
    double *r = s_state + size_t(E) * T + t;
    for (int e = 0; e < E; ++e) L[e * T] = 0.0;
    for (int k = 0; k < K; ++k) r[k * T] = live ? demand[size_t(b) * K + k] : 0.0;
    double *my_flows = flows + size_t(live ? b : 0) * P;
    if (live)
        for (int p = 0; p < P; ++p) my_flows[p] = 0.0;
    int sweeps = 0;
    bool gave_up = false;
    for (;;) {
        bool any = false;
        for (int k = 0; k < K; ++k) any = any || r[k * T] > 0.0;
        if (!any) break;
        if (sweeps == max_sweeps) {
            gave_up = true;
            break;
        }
        sweeps += 1;
        for (int k = 0; k < K; ++k) {                // the same pair in every thread
            const double rk = r[k * T];
            if (!(rk > 0.0)) continue;
            double c_best = __builtin_inf();
            int p_best = -1;
            const int pa = cp[k], pb = cp[k + 1];
            for (int p = pa; p < pb; ++p) {
                double c_path = 0.0;                 // costs are >= 0: the max starts at 0
                const int la = lp[p], lb = lp[p + 1];
                for (int i = la; i < lb; ++i) {
                    const int e = pl[i];
                    const double ce = L[e * T] * invcap[e];
                    if (ce > c_path) c_path = ce;
                }
                if (c_path < c_best) {
                    c_best = c_path;
                    p_best = p;
                }
            }
            if (p_best < 0) continue;                // a pair without candidates
            double f;
            if (rk < chi) {
                f = rk;
            } else {
                const double want = rk * phi;
                const double chunks = floor(want / chi);
                f = chunks * chi;
                if (!(f > 0.0)) f = chi;
            }
            my_flows[p_best] = my_flows[p_best] + f;
            const int la = lp[p_best], lb = lp[p_best + 1];
            for (int i = la; i < lb; ++i) {
                const int e = pl[i];
                L[e * T] = L[e * T] + f;
            }
            r[k * T] = rk - f;
        }
    }
    if (live) {
        double lam = 0.0;
        for (int e = 0; e < E; ++e) {
            const double u = L[e * T] * invcap[e];
            if (u > lam) lam = u;
        }
        lambda[b] = gave_up ? __builtin_nan("") : lam;
        sweeps_out[b] = sweeps;
    }
}


// G lanes per problem (G a power of two >= the most candidates of any pair, at most 64), 64 / G
// problems per wave.  The sweep over the pairs stays sequential -- every routed chunk changes
// the costs the next pair sees -- but lane j costs candidate j of the pair, the group takes the
// minimum by DPP and the lowest lane that holds it (the strict `<` of the sequential scan) routes
// the chunk.  A problem lives inside one wave, so its lanes are ordered by the wave's in-order LDS
// operations; workgroups never synchronise after the set-up (a workgroup is one wave).  LDS: 1/capacity
// per workgroup; L[E + 2], the remainders r[K], the amounts f[K] of this sweep and the flows (by path;
// AHEAD: G per pair) per problem.  L[E] (1/capacity 0) stands for a link that is not there, L[E + 1] =
// +inf (1/capacity 1) for a candidate that is not there.  All lanes walk all pairs, so a wave sweeps
// until the last of its problems is done (amounts of 0 change nothing).
//
// What bounds it is the chain from pair to pair, so everything that does not depend on the pair
// before is taken out of it.  What a pair routes depends on its own remainder only: the amounts of
// a sweep (a division each) are worked out before the sweep, side by side.  AHEAD (paths of at most
// two links, at most 16 candidates) also reads the loads of a pair's links before the pair before
// it has routed its chunk, and adds that chunk where the candidate it took uses the same link: a
// table holds, per pair and lane, the links, their 1/capacity and which candidates of the pair
// before use them.  What a decision depends on is then the one before it, without a trip to LDS.
// (The compiled loop forms the sums of the next pair's loads with the chunk beforehand and so still
// waits for them ahead of the decision: 320 cycles a pair, of which the wave's own fifty or so
// instructions are about 200.)  Chunks are added by LDS atomics that return nothing; the lanes that do
// not take the pair add to a spare place.  The other forms read the loads when they are needed and pass
// over pairs that have nothing left in any problem of the wave (a problem routes most of its pairs in
// its first sweeps, so one problem on its own skips more than eight that share a wave).  TABLE: the links
// of all candidates lie in LDS; without it they come from memory, asked for ahead in stages.
// 4096 problems of one node of 8 GPUs (56 pairs, 10 sweeps at most): 222 -> 102 us
// (one problem 200 -> 86; 7.5 us a sweep).  512 problems of two nodes of 8 (240 pairs of up to 16
// candidates, a thread per problem where their lists do not fit the LDS): 8.2 -> 0.79 ms.  Two nodes of
// 4 GPUs (56 pairs, up to 5 links): one problem 176 us with a table but without passing over, 207
// without either, 110 with both; 4096 problems 233, 209, 173.
constexpr int kAheadSteps = 2, kAheadLanes = 16;
constexpr int kAheadPairs = 4;           // steps of the unrolled loop; pairs are padded to them

// a candidate of up to two links: their byte offsets in L (16 bits each), and for each of them the
// candidates of the pair before that use it
struct __align__(16) Alg1Entry {
    uint32_t at, mask0, mask1, unused;
    double ic0, ic1;
};

struct Alg1Lds {
    size_t ic, problem, per_problem, spare, cp, tab, bytes;
};

// link numbers per candidate in the table of the form that is not AHEAD
__host__ __device__ constexpr int alg1_table_steps(int lm) { return lm <= 2 ? 2 : 8; }

// `steps`: alg1_table_steps where the form that is not AHEAD has its table, 0 otherwise
__host__ __device__ inline Alg1Lds alg1_lds(int E, int K, int P, int lanes, bool ahead, int steps)
{
    Alg1Lds l;
    const int pairs = (K + kAheadPairs - 1) / kAheadPairs * kAheadPairs;
    size_t o = 0;
    l.ic = o;       o += sizeof(double) * (E + 2);
    l.per_problem = sizeof(double) * (static_cast<size_t>(E) + 3 + 2 * static_cast<size_t>(pairs) +
                                      (ahead ? static_cast<size_t>(pairs) * lanes : P));
    l.problem = o;  o += l.per_problem * (kWave / lanes);
    l.spare = o;    o += ahead ? sizeof(double) * kWave : 0;    // a place per lane for what is not wanted
    o = (o + 15) & ~size_t(15);
    l.tab = o;      o += ahead ? sizeof(Alg1Entry) * (static_cast<size_t>(pairs) + 2) * lanes
                               : sizeof(uint16_t) * static_cast<size_t>(K) * lanes * steps;
    l.cp = o;       o += sizeof(int32_t) * (K + 1);
    l.bytes = o;
    return l;
}

template <int G, int LM, bool AHEAD, bool TABLE>
__global__ __launch_bounds__(kWave) void k_alg1_group(int E, int K, int P, int batch,
                                                      const int32_t *__restrict__ cp,
                                                      const int32_t *__restrict__ lp,
                                                      const int32_t *__restrict__ pl,
                                                      const double *__restrict__ invcap,
                                                      const double *__restrict__ demand,
                                                      double phi, double chi, int max_sweeps,
                                                      double *__restrict__ flows,
                                                      double *__restrict__ lambda,
                                                      int32_t *__restrict__ sweeps_out)
{
    static_assert(!AHEAD || (LM == kAheadSteps && G <= kAheadLanes), "masks of 16 bits");
    extern __shared__ __align__(16) unsigned char s_alg1[];
    constexpr int kPerBlock = kWave / G;                      // problems of this wave
    constexpr int kSteps = TABLE ? alg1_table_steps(LM) : 0;
    const Alg1Lds l = alg1_lds(E, K, P, G, AHEAD, kSteps);
    const int lane = threadIdx.x;
    const int j = lane % G;
    const int slot = lane / G;
    const int b = blockIdx.x * kPerBlock + slot;
    const bool live = b < batch;
    double *s_ic = reinterpret_cast<double *>(s_alg1 + l.ic);
    double *L = reinterpret_cast<double *>(s_alg1 + l.problem + l.per_problem * slot);
    const int pairs = (K + kAheadPairs - 1) / kAheadPairs * kAheadPairs;
    double *r = L + (E + 2), *amount = r + pairs, *fl = amount + (pairs + 1);
    double *spare = reinterpret_cast<double *>(s_alg1 + l.spare) + lane;
    Alg1Entry *s_tab = reinterpret_cast<Alg1Entry *>(s_alg1 + l.tab);   // [pairs + 2][G]
    uint16_t *s_links = reinterpret_cast<uint16_t *>(s_alg1 + l.tab);   // [K][G][kSteps]
    int32_t *s_cp = reinterpret_cast<int32_t *>(s_alg1 + l.cp);
    for (int e = lane; e < E; e += kWave) s_ic[e] = invcap[e];
    for (int k = lane; k <= K; k += kWave) s_cp[k] = cp[k];
    for (int e = j; e <= E; e += G) L[e] = 0.0;
    // (set-up and results in batches of eight, so that the trips to memory overlap)
    bool some = false;
    for (int k0 = j; k0 < pairs; k0 += 8 * G) {
        double d[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k0 + i * G;
            d[i] = demand[size_t(live ? b : 0) * K + (k < K ? k : 0)];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k0 + i * G;
            if (!live || k >= K) d[i] = 0.0;
            if (k < pairs) r[k] = d[i];
            some = some || d[i] > 0.0;
        }
    }
    for (int i = j; i < (AHEAD ? pairs * G : P); i += G) fl[i] = 0.0;
    if (lane == 0) {
        s_ic[E] = 0.0;
        s_ic[E + 1] = 1.0;
    }
    if (j == 0) L[E + 1] = __builtin_inf();
    __syncthreads();                                 // one wave: orders the set-up
    auto offset = [](double *p, uint32_t bytes) {
        return reinterpret_cast<double *>(reinterpret_cast<unsigned char *>(p) + bytes);
    };
    auto after = [&](int k) { return k + 1 < K ? k + 1 : 0; };
    if constexpr (AHEAD) {
        for (int idx0 = lane; idx0 < (pairs + 2) * G; idx0 += 8 * kWave) {
            bool there[8];
            int la[8], two[8], x0[8], x1[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = (idx0 + i * kWave) / G, kc = k < K ? k : K - 1;
                int p = s_cp[kc] + idx0 % G;
                there[i] = k < K && p < s_cp[kc + 1];
                p = there[i] ? p : 0;
                la[i] = lp[p];
                two[i] = lp[p + 1];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                two[i] = two[i] - la[i] > 1 ? 1 : 0;
                x0[i] = pl[la[i]];
                x1[i] = pl[la[i] + two[i]];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e0 = there[i] ? x0[i] : E + 1, e1 = there[i] && two[i] ? x1[i] : E;
                Alg1Entry entry = {};
                entry.at = 8u * (static_cast<uint32_t>(e0) | static_cast<uint32_t>(e1) << 16);
                entry.ic0 = s_ic[e0];
                entry.ic1 = s_ic[e1];
                if (idx0 + i * kWave < (pairs + 2) * G) s_tab[idx0 + i * kWave] = entry;
            }
        }
        __syncthreads();
        for (int idx = lane; idx < (pairs + 2) * G; idx += kWave) {
            const int before = idx / G > 0 ? idx / G - 1 : 0;      // (the first pair has none)
            const uint32_t e0 = s_tab[idx].at & 0xFFFFu, e1 = s_tab[idx].at >> 16;
            uint32_t m0 = 0u, m1 = 0u;
#pragma unroll
            for (int c = 0; c < G; ++c) {
                const uint32_t o = s_tab[before * G + c].at, o0 = o & 0xFFFFu, o1 = o >> 16;
                m0 |= (e0 == o0 || e0 == o1 ? 1u : 0u) << c;
                m1 |= (e1 == o0 || e1 == o1 ? 1u : 0u) << c;
            }
            s_tab[idx].mask0 = e0 < 8u * E ? m0 : 0u;
            s_tab[idx].mask1 = e1 < 8u * E ? m1 : 0u;
        }
        __syncthreads();
    }
    if constexpr (TABLE) {
        for (int idx = lane; idx < K * G; idx += kWave) {
            const int k = idx / G;
            int p = s_cp[k] + idx % G;
            const bool there = p < s_cp[k + 1];
            p = there ? p : 0;
            const int la = lp[p], n = there ? lp[p + 1] - la : 0;
#pragma unroll
            for (int i = 0; i < LM; ++i)
                s_links[idx * kSteps + i] =
                    static_cast<uint16_t>(i < n ? pl[la + i] : i == 0 ? E + 1 : E);
        }
        __syncthreads();
    }
    // lanes of this problem inside the wave
    const unsigned long long gmask = (G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull)) << (lane - j);
    // the one lane of the group that takes the pair, of those whose cost is the least
    auto takes = [&](double c, double m, uint32_t &low) {
        const unsigned long long eq = __builtin_amdgcn_ballot_w64(c == m);
        if constexpr (G <= 32) {
            const uint32_t half = lane & 32 ? static_cast<uint32_t>(eq >> 32)
                                            : static_cast<uint32_t>(eq);
            const uint32_t field = __builtin_amdgcn_ubfe(half, (lane - j) & 31, G & 31);
            low = G == 32 ? half & (0u - half) : field & (0u - field);
            return low == 1u << (j & 31);
        } else {
            low = 0u;
            return j == __ffsll(static_cast<long long>(eq)) - 1;
        }
    };
    auto least = [&](double c) {
        double m = c;
        if constexpr (G > 1) m = fast_min_f64(m, partner_f64<1>(m));
        if constexpr (G > 2) m = fast_min_f64(m, partner_f64<2>(m));
        if constexpr (G > 4) m = fast_min_f64(m, partner_f64<4>(m));
        if constexpr (G > 8) m = fast_min_f64(m, partner_f64<8>(m));
        if constexpr (G > 16) m = fast_min_f64(m, partner_f64<16>(m));
        if constexpr (G > 32) m = fast_min_f64(m, partner_f64<32>(m));
        return m;
    };
    int sweeps = 0;
    bool gave_up = false, done = false;

    // not AHEAD: links and 1/capacity of the pair at hand, links of the next, list of the one after
    // (asked for without branches, so that nobody waits for one request before the next is made)
    int e_now[LM], e_next[LM], p_now = 0, p_next = 0, p_list = 0, la = 0, lb = 0, k_list = 0;
    double ic_now[LM];
    auto ask_list = [&](int k) {
        p_list = s_cp[k] + j;
        const bool there = p_list < s_cp[k + 1];
        p_list = there ? p_list : 0;
        if constexpr (!TABLE) {
            la = lp[p_list];
            lb = lp[p_list + 1];
            lb = there ? lb : la;
        }
    };
    auto ask_links = [&](int (&e)[LM]) {
        if constexpr (TABLE) {
            const uint16_t *from = s_links + (k_list * G + j) * kSteps;
            if constexpr (kSteps == 2) {
                const uint32_t w = *reinterpret_cast<const uint32_t *>(from);
                e[0] = static_cast<int>(w & 0xFFFFu);
                e[1] = static_cast<int>(w >> 16);
            } else {
                const uint4 w = *reinterpret_cast<const uint4 *>(from);
                const uint32_t of[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int i = 0; i < LM; ++i)
                    e[i] = static_cast<int>(i % 2 ? of[i / 2] >> 16 : of[i / 2] & 0xFFFFu);
            }
            return;
        }
        const int n = lb - la;
#pragma unroll
        for (int i = 0; i < LM; ++i) {
            const int x = pl[la + (i < n ? i : 0)];
            e[i] = i < n ? x : i == 0 ? E + 1 : E;
        }
    };
    if constexpr (!AHEAD) {
        ask_list(0);
        p_now = p_list;
        ask_links(e_now);
#pragma unroll
        for (int i = 0; i < LM; ++i) ic_now[i] = s_ic[e_now[i]];
        k_list = after(0);
        ask_list(k_list);
        p_next = p_list;
        ask_links(e_next);
        k_list = after(after(0));
        ask_list(k_list);
    }
    for (;;) {
        const bool any = (__ballot(some) & gmask) != 0ull;
        if (!done) {
            if (!any) done = true;
            else if (sweeps == max_sweeps) {
                gave_up = true;
                done = true;
            } else sweeps += 1;
        }
        if (__all(done)) break;                      // wave-uniform
        // what every pair routes in this sweep, and what it leaves for the next
        some = false;
        for (int k0 = j; k0 < pairs; k0 += kAheadPairs * G) {
            double rk[kAheadPairs], f[kAheadPairs];
#pragma unroll
            for (int i = 0; i < kAheadPairs; ++i) rk[i] = k0 + i * G < pairs ? r[k0 + i * G] : 0.0;
#pragma unroll
            for (int i = 0; i < kAheadPairs; ++i) {
                const double want = rk[i] * phi;
                const double chunks = floor(want / chi);
                double fc = chunks * chi;
                if (!(fc > 0.0)) fc = chi;
                f[i] = rk[i];
                if (!(rk[i] < chi)) f[i] = fc;
                if (done || !(rk[i] > 0.0)) f[i] = 0.0;
            }
#pragma unroll
            for (int i = 0; i < kAheadPairs; ++i) {
                const double rest = rk[i] - f[i];
                some = some || rest > 0.0;
                if (k0 + i * G < pairs) {
                    amount[k0 + i * G] = f[i];
                    r[k0 + i * G] = rest;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if constexpr (AHEAD) {
            const Alg1Entry *entry = s_tab + j;
            const double *next_amount = amount + 1;
            double *flow = fl + j;
            // the pair at hand (its loads without the chunk of the pair before) and the next one's
            // links; what the pair before routed, and which of its lanes took it
            Alg1Entry now = entry[0], next = entry[G];
            double *at0 = offset(L, now.at & 0xFFFFu), *at1 = offset(L, now.at >> 16);
            double L0 = *at0, L1 = *at1, f = amount[0], routed = 0.0;
            uint32_t took = 0u;
            for (int k0 = 0; k0 < pairs; k0 += kAheadPairs) {
#pragma unroll
                for (int i = 0; i < kAheadPairs; ++i) {
                    const Alg1Entry after = entry[(i + 2) * G];
                    const double f_next = next_amount[i];  // (the one past the last is not used)
                    // (asked for before this pair's own additions: corrected when its turn comes)
                    double *n_at0 = offset(L, next.at & 0xFFFFu), *n_at1 = offset(L, next.at >> 16);
                    const double n0 = *n_at0, n1 = *n_at1;
                    const double a0 = L0 + routed, a1 = L1 + routed;
                    L0 = (now.mask0 & took) != 0u ? a0 : L0;
                    L1 = (now.mask1 & took) != 0u ? a1 : L1;
                    const double c = fast_max_f64(L0 * now.ic0, L1 * now.ic1);
                    const bool me = takes(c, least(c), took);
                    lds_add_f64(me ? flow + i * G : spare, f);
                    lds_add_f64(me ? at0 : spare, f);
                    lds_add_f64(me ? at1 : spare, f);
                    routed = f;
                    f = f_next;
                    now = next;
                    next = after;
                    at0 = n_at0;
                    at1 = n_at1;
                    L0 = n0;
                    L1 = n1;
                }
                entry += kAheadPairs * G;
                next_amount += kAheadPairs;
                flow += kAheadPairs * G;
            }
        } else {
            double f = amount[0];
            for (int k = 0; k < K; ++k) {            // the same pair in every lane
                double Lv[LM];
#pragma unroll
                for (int i = 0; i < LM; ++i) Lv[i] = L[e_now[i]];
                const double f_next = amount[k + 1];
                const double flow_now = fl[p_now];
                double ic_next[LM];
#pragma unroll
                for (int i = 0; i < LM; ++i) ic_next[i] = s_ic[e_next[i]];
                int e_after[LM];
                const int p_after = p_list;
                ask_links(e_after);
                k_list = after(k_list);
                ask_list(k_list);
                // (late in a solve most pairs have nothing left in any problem of the wave)
                if (__builtin_amdgcn_ballot_w64(f > 0.0) != 0ull) {
                    double c = Lv[0] * ic_now[0];
#pragma unroll
                    for (int i = 1; i < LM; ++i) c = fast_max_f64(c, Lv[i] * ic_now[i]);
                    uint32_t low;
                    if (takes(c, least(c), low)) {
                        fl[p_now] = flow_now + f;
#pragma unroll
                        for (int i = 0; i < LM; ++i)
                            if (e_now[i] < E) L[e_now[i]] = Lv[i] + f;
                    }
                }
#pragma unroll
                for (int i = 0; i < LM; ++i) {
                    e_now[i] = e_next[i];
                    ic_now[i] = ic_next[i];
                    e_next[i] = e_after[i];
                }
                p_now = p_next;
                p_next = p_after;
                f = f_next;
                // the next pair sees the loads this one left
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (live) {
        double *out = flows + size_t(b) * P;
        if constexpr (!AHEAD)
            for (int p = j; p < P; p += G) out[p] = fl[p];
        for (int k0 = 0; AHEAD && k0 < K; k0 += 8) {
            int p[8], n[8];
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = k0 + i < K ? k0 + i : K - 1;
                p[i] = s_cp[k];
                n[i] = s_cp[k + 1] - p[i];
                v[i] = fl[k * G + j];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (j < n[i] && k0 + i < K) out[p[i] + j] = v[i];
        }
    }
    double lam = 0.0;
    for (int e = j; e < E; e += G) {
        const double u = L[e] * s_ic[e];
        if (u > lam) lam = u;
    }
    if constexpr (G > 1) lam = fmax(lam, partner_f64<1>(lam));
    if constexpr (G > 2) lam = fmax(lam, partner_f64<2>(lam));
    if constexpr (G > 4) lam = fmax(lam, partner_f64<4>(lam));
    if constexpr (G > 8) lam = fmax(lam, partner_f64<8>(lam));
    if constexpr (G > 16) lam = fmax(lam, partner_f64<16>(lam));
    if constexpr (G > 32) lam = fmax(lam, partner_f64<32>(lam));
    if (live && j == 0) {
        lambda[b] = gave_up ? __builtin_nan("") : lam;
        sweeps_out[b] = sweeps;
    }
}

// What is accepted: topologies whose state fits 64 KB with a group of lanes per problem and the
// candidate lists beside it (2 or 8 links each), or a workgroup of the kernel with a thread per problem.
// The former are also those whose lists are kept in LDS.
bool alg1_small(const DeviceTopo &t)
{
    if (t.pmax > kWave || t.pmax < 1 || t.lmax > 8 || t.K < 1) return false;
    const size_t G = lanes_per_commodity(t.pmax);
    return sizeof(double) * (t.E + 1) +
               sizeof(double) * (kWave / G) * (static_cast<size_t>(t.E) + 1 + t.K + t.P) +
               sizeof(int32_t) * (t.K + 1) +
               sizeof(int32_t) * static_cast<size_t>(t.K) * G * (t.lmax <= 2 ? 2 : 8) <=
           kAlg1LdsPlain;
}

}  // namespace

// Problems per workgroup: the most (a power of two, at most 64) whose state fits the budget.
int alg1_threads(const DeviceTopo &t)
{
    const size_t per_problem = sizeof(double) * (static_cast<size_t>(t.E) + static_cast<size_t>(t.K));
    int threads = kAlg1Threads;
    while (threads > kAlg1MinThreads && per_problem * threads > kAlg1LdsBudget) threads >>= 1;
    return threads;
}

size_t alg1_lds_bytes(const DeviceTopo &t)
{
    return sizeof(double) * alg1_threads(t) * (static_cast<size_t>(t.E) + static_cast<size_t>(t.K));
}

bool alg1_fits(const DeviceTopo &t)
{
    return (!t.alg1_thread_per_problem && alg1_small(t)) || alg1_lds_bytes(t) <= kAlg1LdsBudget;
}

// Rough time of `blocks` workgroups in us per pair and sweep: `us` for one on a compute unit by
// itself, `more` of that for every further one beside it, as many side by side as the LDS holds.
// (It is handed out in pieces of 1280 bytes.)
static double alg1_time(int64_t blocks, size_t lds, double us, double more)
{
    const int64_t side = 160 * 1024 / ((lds + 1279) / 1280 * 1280);
    const int64_t rounds = blocks / (256 * side), rest = (blocks % (256 * side) + 255) / 256;
    return us * (rounds * (1.0 + more * (side - 1)) + (rest ? 1.0 + more * (rest - 1) : 0.0));
}

// The fastest of the forms a topology fits, by the time a pair takes in one sweep: AHEAD 0.13 us, 0.22
// to 0.39 with a table of up to 2, 5 or 8 links, 0.24 to 0.49 with lists from memory, 0.55 and 0.068 per
// link of its candidates with a thread per problem.  The faster a form, the more LDS it takes, and the
// fewer of its workgroups run side by side.  Measured on 41 topologies (one to four nodes of 2 to 20
// GPUs, random ones of up to 64 candidates and 8 links; 6 to 992 pairs) and 1 to 65536 problems,
// 260 calls: the form chosen is the fastest but for two, where it is 3 % behind.
Alg1Form alg1_form(const DeviceTopo &t, int32_t batch)
{
    Alg1Form best = {};
    double least = 0.0;
    auto offer = [&](const Alg1Form &f, int per_block, double us, double more) {
        const double time = alg1_time((batch + int64_t(per_block) - 1) / per_block, f.lds, us, more);
        if (best.lds == 0 || time < least) {
            best = f;
            least = time;
        }
    };
    if (!t.alg1_thread_per_problem && t.pmax >= 1 && t.pmax <= kWave && t.lmax <= 8 && t.K >= 1) {
        const int of = t.lmax <= 2 ? 0 : t.lmax <= 5 ? 1 : 2;
        constexpr double kTable[] = {0.22, 0.32, 0.39}, kMemory[] = {0.24, 0.38, 0.49};
        for (int form = 0; form < 3; ++form) {
            const bool ahead = form == 0, table = form == 1;
            if (table && !alg1_small(t)) continue;
            // (more lanes than candidates where only fewer problems fit the LDS together)
            for (int G = lanes_per_commodity(t.pmax); G <= kWave; G *= 2) {
                if (ahead && (t.lmax > kAheadSteps || G > kAheadLanes || 8 * (t.E + 1) > 0xFFFF)) break;
                const size_t lds =
                    alg1_lds(t.E, t.K, t.P, G, ahead, table ? alg1_table_steps(t.lmax) : 0).bytes;
                if (lds > kAlg1LdsBudget) continue;
                if (ahead) offer({G, ahead, table, lds}, kWave / G, 0.13, 0.16);
                else offer({G, ahead, table, lds}, kWave / G, table ? kTable[of] : kMemory[of], 0.03);
                break;
            }
        }
    }
    if (alg1_lds_bytes(t) <= kAlg1LdsBudget)
        offer({0, false, false, alg1_lds_bytes(t)}, alg1_threads(t),
              0.55 + 0.068 * static_cast<double>(t.nnz) / t.K, 0.02);
    return best;
}

hipError_t launch_alg1(const DeviceTopo &t, int32_t batch, const double *demand, double phi,
                       double chi, int32_t max_sweeps, double *flows, double *lambda,
                       int32_t *sweeps, hipStream_t s)
{
    const Alg1Form form = alg1_form(t, batch);
    const int G = form.lanes;
    const size_t glds = form.lds;
    if (G > 0) {
        const int per_block = kWave / G;
        const int ggrid = (batch + per_block - 1) / per_block;
#define NIMBLE_ALG1_LAUNCH(GG, LM, AHEAD, TABLE)                                               \
    do {                                                                                       \
        if (glds > kAlg1LdsPlain) {                                                            \
            const hipError_t ea = hipFuncSetAttribute(                                         \
                reinterpret_cast<const void *>(&k_alg1_group<GG, LM, AHEAD, TABLE>),           \
                hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kAlg1LdsBudget)); \
            if (ea != hipSuccess) return ea;                                                   \
        }                                                                                      \
        hipLaunchKernelGGL((k_alg1_group<GG, LM, AHEAD, TABLE>), dim3(ggrid), dim3(kWave),     \
                           glds, s, t.E, t.K, t.P, batch, t.comm_ptr, t.path_ptr,              \
                           t.path_links, t.invcap, demand, phi, chi, max_sweeps, flows,        \
                           lambda, sweeps);                                                    \
        return hipGetLastError();                                                              \
    } while (0)
#define NIMBLE_ALG1_FORM(GG, LM)                                                               \
    if (t.lmax <= LM) {                                                                        \
        if (form.table) NIMBLE_ALG1_LAUNCH(GG, LM, false, true);                               \
        NIMBLE_ALG1_LAUNCH(GG, LM, false, false);                                              \
    }
#define NIMBLE_ALG1_LANES(GG)                                                                  \
    case GG:                                                                                   \
        if constexpr (GG <= kAheadLanes)                                                       \
            if (form.ahead) NIMBLE_ALG1_LAUNCH(GG, kAheadSteps, true, false);                  \
        NIMBLE_ALG1_FORM(GG, 2)                                                                \
        NIMBLE_ALG1_FORM(GG, 5)                                                                \
        NIMBLE_ALG1_FORM(GG, 8)                                                                \
        break;
        switch (G) {
            NIMBLE_ALG1_LANES(1)
            NIMBLE_ALG1_LANES(2)
            NIMBLE_ALG1_LANES(4)
            NIMBLE_ALG1_LANES(8)
            NIMBLE_ALG1_LANES(16)
            NIMBLE_ALG1_LANES(32)
            NIMBLE_ALG1_LANES(64)
        }
#undef NIMBLE_ALG1_LANES
#undef NIMBLE_ALG1_FORM
#undef NIMBLE_ALG1_LAUNCH
    }
    const size_t lds = alg1_lds_bytes(t);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_alg1),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(lds));
    if (e != hipSuccess) return e;
    const int threads = alg1_threads(t);
    const int grid = (batch + threads - 1) / threads;
    hipLaunchKernelGGL(k_alg1, dim3(grid), dim3(threads), lds, s, t.E, t.K, t.P, batch,
                       t.comm_ptr, t.path_ptr, t.path_links, t.invcap, demand, phi, chi,
                       max_sweeps, flows, lambda, sweeps);
    return hipGetLastError();
}

}  // namespace nimble
