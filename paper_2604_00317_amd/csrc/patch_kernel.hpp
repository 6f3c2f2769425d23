// The patch kernels: a whole solve in one launch, the commodities of a fabric cut into patches
// (host_patch.hpp), a workgroup per patch.  A patch keeps the candidate lists of its commodities
// in registers and the prices, lengths and congestion sums of its links in LDS from the first
// iteration to the last; per iteration
//   scan     L lanes per commodity add up the prices of their candidates (LDS reads: 9 per four
//            candidates of a product slot) and agree on the cheapest, lowest index first;
//   scatter  the lane that holds it adds the commodity's demand to the loads of the candidate's
//            links (LDS atomics: five per commodity, where a walk of the reverse rows looks at
//            every commodity of every link -- 50 per commodity on the 64-node fabric);
//   update   one thread per link applies  S += u, len *= 1 + eps u / rho, price = len / cap.
// Fabrics of several patches (MULTI) exchange the loads of shared links between scatter and
// update: a patch publishes its part of a link's load and sums the parts of all users, in the
// same order in every patch, so that all hold the same length and price.
//
// Exchange without barriers or fences: a part is one 8-byte word, loaded at agent scope (past the
// L1 caches) and stored at agent scope (past the L2 caches, which are not coherent between the XCDs)
// or, where all its readers are on the writer's XCD, into that XCD's L2 alone (put_word).  Its sign bit
// says which exchange it belongs to -- loads are never negative.  Exchange n uses buffer n & 1 and the sign
// (n >> 1) & 1; all words start with the sign set.  A patch overwrites its part of exchange n
// with that of n + 2 only after it has read all parts of n + 1 of the groups it shares, which
// their writers published after reading n: nobody misses a word.  The words of a patch lie side by
// side, so that it writes whole cache lines: 256 patches that exchange 72 groups of 8 links with 15
// others each and do nothing else take 7820 cycles per exchange where every part of a group is half a
// line of its own, 5900 to 6400 this way; with 16 groups 4860 and 3700.  (Accumulators on the memory side that all users
// add to, a patch per group that adds up the parts for the others, and one per XCD took 8400 to 13200.)
// Every wait is bounded; when one
// expires the team gives up, lambda becomes NaN, and whatever follows in the stream (launch_alone;
// the host, after a solve of variable step) solves the plan without patches.  A limit of zero
// means that nobody waits at all.
//
// Sums of loads do not depend on the order of the atomics: they are sums of integers.  Where the
// demands of a patch lie on a power-of-two grid with a total below 2^53 units (byte counts) those
// are the units, and the sum is what exact additions give; elsewhere a demand is split into
// 2^-61 of the patch's total and 2^-105 of it, which holds every demand that is not below 2^-52 of
// the total to the last bit; both sums are exact, each is rounded to binary64, and so is what they
// add up to (and, with several patches, what the parts of a link add up to).
// Demands that lie further apart, or whose total overflows, are on no such grid: one patch adds
// them as binary64 numbers one after the other, in code of its own (solve_wide: a branch in the
// ordinary loop cost plans of one patch 4 to 15 %); several patches mark the plan as given up.
//
// What bounds it and what it measured, us per iteration (in brackets: two launches per iteration and,
// on 2 nodes, a gather over the reverse rows in one workgroup): 2 nodes of 8 GPUs 0.84 (2.64): one
// patch, the chain scan, barrier, scatter, update; the LDS is busy for half of it; 7 nodes of 6 1.7 to
// 2.0 (7.1) and 16 nodes 2.25 (7.3): the trip of a word from patch to patch, some 3000 cycles with
// the reading of the words; 64 nodes 7.5 (18.5), 6.9 in blocks (patch_blocks.hpp): the words of up to
// 31 users of every shared link, 127 KB per patch and iteration, then vector issue and LDS of the scan.
#pragma once
#include <hip/hip_runtime.h>

#include "host_patch.hpp"
#include "kernels.hpp"
#include "wave_ops.hpp"

namespace nimble {

namespace patch {

constexpr unsigned long long kSign = 1ull << 63;
constexpr int kNone = 0x7FFFFFFF;
constexpr int kSumBits = 61, kLowBits = 44;
constexpr int kXccId = 20 | (31 << 11);          // hardware register XCC_ID

// LDS of a patch, byte offsets.  The prices come first: a slot's offsets are LDS addresses.  The
// state of a link is one record; the choices of a candidate are counted in 16 bits, those of slot
// s (of all the lanes' slots) of the patch's commodity c at count + (c * slots + s) * 8.  A solve
// of variable step sums its steps instead, a double per candidate (slot_bytes 32).
struct LinkState {
    unsigned long long load, low;      // load so far, see Grid
    double len, S, invcap;
};
struct Lds {
    int link, red, group, at, count, bytes;
};

__host__ __device__ inline Lds lds_layout(int n_local, int n_groups, int n_at, int n_comm, int slots,
                                          int slot_bytes)
{
    Lds l;
    int o = 8 * (n_local + 2);                  // [n_local] +0.0, [n_local + 1] +inf
    l.link = o;    o += static_cast<int>(sizeof(LinkState)) * n_local;
    l.red = o;     o += 8 * 40;
    l.group = o;   o += 4 * (n_groups + 1);
    l.at = o;      o += 2 * n_at;
    o = (o + 15) & ~15;
    l.count = o;   o += slot_bytes * n_comm * slots;
    l.bytes = o;
    return l;
}

// The dynamic LDS starts at LDS address 0 (there is no other), so a slot's offsets are addresses.
extern __shared__ __align__(16) unsigned char s_lds[];

__device__ __forceinline__ double lds_f64(uint32_t off)
{
    return *reinterpret_cast<const double *>(s_lds + off);
}
__device__ __forceinline__ double *lds_ptr(uint32_t off)
{
    return reinterpret_cast<double *>(s_lds + off);
}
__device__ __forceinline__ double lds_lo(uint32_t w) { return lds_f64(w & 0xFFFFu); }
__device__ __forceinline__ double lds_hi(uint32_t w) { return lds_f64(w >> 16); }

// The cost of a path so far and the next price.  (The largest of numbers is one instruction; a comparison
// and a selection, three, took 2 nodes of 8 536 us for 500 iterations against 466, 3 nodes 1082 and 841, 7 of
// 6 995 and 940, 24 of 8 with two NICs in reach 2311 and 2191, 64 4169 and 3830.)
template <bool MAXC>
__device__ __forceinline__ double join(double acc, double p)
{
    if constexpr (MAXC) return fast_max_f64(acc, p);
    else return acc + p;
}

__device__ __forceinline__ int select(bool c, int a, int b)
{
    int r;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(c);
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(m));
    return r;
}
__device__ __forceinline__ uint32_t select(bool c, uint32_t a, uint32_t b)
{
    return static_cast<uint32_t>(select(c, static_cast<int>(a), static_cast<int>(b)));
}

// What is derived from these values is worked out where it is used: taken out of the loop over
// the iterations (they never change) it would fill more registers than there are.
__device__ __forceinline__ void keep_in_loop(uint32_t &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_in_loop(double &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_uniform(int &v) { asm volatile("" : "+s"(v)); }

// How the loads of a patch are summed: as whole numbers of units of 2^unit, and where the demands
// are no such whole numbers also of 2^(unit - kLowBits).  (That not even those hold them is noted
// in LDS: looked at hardly ever, it is not worth a register.)
struct Grid {
    bool exact;
    int unit;
};
struct Demand {
    unsigned long long units, low;
};

template <int LOW = kLowBits>
__device__ __forceinline__ Demand on_grid(double d, const Grid &gr)
{
    const double h = trunc(ldexp(d, -gr.unit));
    const double r = d - ldexp(h, gr.unit);
    Demand n;
    n.units = static_cast<unsigned long long>(static_cast<long long>(h));
    n.low = static_cast<unsigned long long>(
        static_cast<long long>(trunc(ldexp(r, LOW - gr.unit))));
    return n;
}

__device__ __forceinline__ void lds_add(unsigned long long *p, unsigned long long v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// adds d to the loads of the links at off[0..N-1] (offsets from `pad` on are no links)
template <int N>
__device__ __forceinline__ void add_loads(LinkState *links, uint32_t pad, const uint32_t (&off)[N],
                                          const Grid &gr, const Demand &d)
{
    static_assert(sizeof(LinkState) == 40, "five times the 8 bytes of a price");
    unsigned char *base = reinterpret_cast<unsigned char *>(links);
#pragma unroll
    for (int x = 0; x < N; ++x)
        if (off[x] < pad)
            lds_add(&reinterpret_cast<LinkState *>(base + off[x] * 5u)->load, d.units);
    if (gr.exact) return;                                               // wave-uniform
#pragma unroll
    for (int x = 0; x < N; ++x)
        if (off[x] < pad) lds_add(&reinterpret_cast<LinkState *>(base + off[x] * 5u)->low, d.low);
}

// the same where the loads of the links lie side by side
template <int N>
__device__ __forceinline__ void add_loads(unsigned long long *load, unsigned long long *low, uint32_t pad,
                                          const uint32_t (&off)[N], const Grid &gr, const Demand &d)
{
    unsigned char *base = reinterpret_cast<unsigned char *>(load);
#pragma unroll
    for (int x = 0; x < N; ++x)
        if (off[x] < pad) lds_add(reinterpret_cast<unsigned long long *>(base + off[x]), d.units);
    if (gr.exact) return;                                               // wave-uniform
    base = reinterpret_cast<unsigned char *>(low);
#pragma unroll
    for (int x = 0; x < N; ++x)
        if (off[x] < pad) lds_add(reinterpret_cast<unsigned long long *>(base + off[x]), d.low);
}

// the load of a link, which starts at zero again
template <int LOW = kLowBits>
__device__ __forceinline__ double take_load(unsigned long long &load, unsigned long long &low,
                                            const Grid &gr)
{
    const double hi = ldexp(static_cast<double>(static_cast<long long>(load)), gr.unit);
    load = 0ull;
    if (gr.exact) return hi;
    const double lo = ldexp(static_cast<double>(static_cast<long long>(low)), gr.unit - LOW);
    low = 0ull;
    return hi + lo;
}
__device__ __forceinline__ double take_load(LinkState &s, const Grid &gr)
{
    return take_load(s.load, s.low, gr);
}

// `near`: all who read the word run on this XCD and find it in its L2; the store need not go on to
// the memory side.  A word is with its reader 255 ns after the store, 412 ns if it goes on all the
// same, 570 to 640 ns on another XCD (two waves that answer each other).  `near` is wave-uniform.
// Such a word is stored at workgroup scope though other workgroups read it, which the language does not
// allow for: it holds because of what this target makes of it.  The L1 of a compute unit is written through,
// so the store (sc0) goes to the L2 all compute units of the XCD share, where the readers' agent-scope
// loads (sc1) look; and atomic stores are neither dropped nor combined.  (Should a word not arrive all
// the same, the wait for it ends and the plan is solved without patches.)
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "words stored at workgroup scope are in the L2 of the XCD on gfx950; look again for another target"
#endif
__device__ __forceinline__ void put_word(double *p, double v, unsigned phase, bool near = false)
{
    const unsigned long long b = (static_cast<unsigned long long>(__double_as_longlong(v)) & ~kSign) |
                                 (static_cast<unsigned long long>(phase) << 63);
    unsigned long long *q = reinterpret_cast<unsigned long long *>(p);
    if (near) __hip_atomic_store(q, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(q, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long get_word(const double *p)
{
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double word_value(unsigned long long b)
{
    return __builtin_fabs(__longlong_as_double(static_cast<long long>(b)));
}

// one more fruitless poll; false when it is time to give up
__device__ __forceinline__ bool keep_waiting(unsigned &polls, unsigned limit, unsigned *abort_word)
{
    if (++polls > limit) {
        __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    if ((polls & 63u) == 0u)
        return __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    return true;
}

// v of the lane 16 (or 32) further, added to the own one in the same order by both
__device__ __forceinline__ double add_across16(double v)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double add_across32(double v)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Loads of shared links.  Every link has `lanes` lanes (1, 2 or 4, the same in all patches: as many as
// there are threads for): lane `sub` of them adds up the parts of users sub, sub + lanes, ... in order,
// then the partial sums are added in a fixed tree, so that all patches get the same bits.  NX words of a
// lane are asked for together, and again as long as some have not arrived.  `at`: LDS address of where
// the users of the link's group have their words; `link`: the link's place in its group; `most`: the
// largest number of users.
template <int NX>
__device__ __forceinline__ double parts_of_link(const double *words, uint32_t at, int users, int most,
                                                int sub, int lanes, uint32_t link, unsigned phase,
                                                unsigned limit, unsigned *abort_word, int &dead)
{
    double sum = 0.0;
    // (what follows from these is worked out here: kept over the iterations it would fill more
    // registers than there are)
    uint32_t n = static_cast<uint32_t>(users > sub ? users - sub : 0);     // of the users from `sub` on
    keep_in_loop(n);
    keep_in_loop(at);
    keep_uniform(lanes);
    at += 2 * static_cast<uint32_t>(n > 0 ? sub : 0);
    for (int c = 0; c < most; c += NX * lanes) {                    // wave-uniform, as all below
        unsigned long long v[NX];
        unsigned polls = 0;
        for (;;) {
            unsigned any = 0u, all = ~0u;
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const uint32_t u = c + x * lanes;        // (users there are not: the first one again)
                const uint32_t unit = *reinterpret_cast<const uint16_t *>(s_lds + at + 2 * (u < n ? u : 0u));
                v[x] = get_word(reinterpret_cast<const double *>(
                    reinterpret_cast<const unsigned char *>(words) + (unit * (8u * kPatchGroup) + 8u * link)));
            }
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                any |= static_cast<unsigned>(v[x] >> 32);
                all &= static_cast<unsigned>(v[x] >> 32);
            }
            const unsigned long long wrong =
                phase ? __builtin_amdgcn_ballot_w64((all >> 31) == 0u)
                      : __builtin_amdgcn_ballot_w64((any >> 31) != 0u);
            if (wrong == 0ull || dead) break;
            ++polls;
            if (polls > limit) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                dead = 1;
            } else if ((polls & 63u) == 0u) {
                dead = __builtin_amdgcn_readfirstlane(static_cast<int>(__hip_atomic_load(
                    abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
            }
        }
#pragma unroll
        for (int x = 0; x < NX; ++x)
            sum = sum + (static_cast<uint32_t>(c + x * lanes) < n ? word_value(v[x]) : 0.0);
    }
    if (lanes > 1) sum = add_across32(sum);
    if (lanes > 2) sum = add_across16(sum);
    return sum;
}
// (the words of four, eight or sixteen users at a time)
__device__ __forceinline__ double load_of_link(const double *words, uint32_t at, int users, int most,
                                               int sub, int lanes, int link, unsigned phase,
                                               unsigned limit, unsigned *abort_word, int &dead)
{
    if (most <= 4 * lanes)
        return parts_of_link<4>(words, at, users, most, sub, lanes, link, phase, limit, abort_word, dead);
    if (most <= 8 * lanes)
        return parts_of_link<8>(words, at, users, most, sub, lanes, link, phase, limit, abort_word, dead);
    return parts_of_link<16>(words, at, users, most, sub, lanes, link, phase, limit, abort_word, dead);
}

__device__ __forceinline__ double wave_sum(double v)
{
    v = v + partner_f64<1>(v);
    v = v + partner_f64<2>(v);
    v = v + partner_f64<4>(v);
    v = v + partner_f64<8>(v);
    v = v + partner_f64<16>(v);
    v = v + partner_f64<32>(v);
    return v;
}

// keep, or the words of slot q where `better`
template <int NW>
__device__ __forceinline__ void take_words(uint32_t (&keep)[NW], const uint32_t (&w)[NW], bool better)
{
#pragma unroll
    for (int x = 0; x < NW; ++x) keep[x] = select(better, w[x], keep[x]);
}

// x[0] + x[1] + ... + x[n-1] in that order, of words other patches (or this one) publish.  256
// words are asked for together; the additions are one dependent chain whatever is done, so every
// lane makes all of them, the terms broadcast lane by lane.
__device__ __forceinline__ double sum_in_order(const double *x, int n, unsigned phase,
                                               unsigned limit, unsigned *abort_word, int &dead,
                                               int lane)
{
    double s = 0.0;
    for (int b = 0; b < n; b += 4 * kWave) {                          // wave-uniform, as all below
        unsigned long long v[4];
        unsigned polls = 0;
        for (;;) {
            bool wrong = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = b + q * kWave + lane;
                v[q] = static_cast<unsigned long long>(phase) << 63;
                if (i < n) v[q] = get_word(x + i);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) wrong = wrong || static_cast<unsigned>(v[q] >> 63) != phase;
            if (__builtin_amdgcn_ballot_w64(wrong) == 0ull || dead) break;
            int late = keep_waiting(polls, limit, abort_word) ? 0 : 1;
            dead = __builtin_amdgcn_readfirstlane(late);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double w = word_value(v[q]);
            const int lo = __double2loint(w), hi = __double2hiint(w);
            const int m = n - b - q * kWave;
            if (m >= kWave) {
#pragma unroll 8
                for (int i = 0; i < kWave; ++i)
                    s = s + __hiloint2double(__builtin_amdgcn_readlane(hi, i),
                                             __builtin_amdgcn_readlane(lo, i));
            } else {
                for (int i = 0; i < m; ++i)
                    s = s + __hiloint2double(__builtin_amdgcn_readlane(hi, i),
                                             __builtin_amdgcn_readlane(lo, i));
            }
        }
    }
    return s;
}

// How the demands of a patch are summed: d is this thread's (0: none).  Noted beside: they lie on no
// grid.  (Called by all threads; ends with a barrier behind it to come.)
__device__ __forceinline__ Grid find_grid(double d, double *red, int *s_wide, int n_waves, int wave,
                                          int lane)
{
    // total and finest grid of the patch's demands
    double sum = d;
    int fine = 4096;
    if (d != 0.0) {
        const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(d));
        const int ex = static_cast<int>((b >> 52) & 2047u);
        const unsigned long long man = (b & ((1ull << 52) - 1ull)) | (ex ? 1ull << 52 : 0ull);
        fine = (ex ? ex : 1) - 1075 + __ffsll(static_cast<long long>(man)) - 1;
    }
    sum = wave_sum(sum);
    for (int o = 32; o > 0; o >>= 1) fine = min(fine, __shfl_xor(fine, o, kWave));
    if (lane == 0) {
        red[wave] = sum;
        reinterpret_cast<int *>(red + 16)[wave] = fine;
    }
    __syncthreads();
    double total = 0.0;
    for (int q = 0; q < n_waves; ++q) {
        total = total + red[q];
        fine = min(fine, reinterpret_cast<const int *>(red + 16)[q]);
    }
    const bool some = total > 0.0 && total < __builtin_inf();
    const int top = some ? ilogb(total) + 1 : 0;            // the total is below 2^top
    Grid gr;
    gr.exact = __builtin_amdgcn_readfirstlane(!some || top - fine <= 53 ? 1 : 0) != 0;
    gr.unit = __builtin_amdgcn_readfirstlane(!some ? 0 : gr.exact ? fine : top - kSumBits);
    if (threadIdx.x == 0)
        *s_wide = total == __builtin_inf() || (some && top - fine > kSumBits + kLowBits);
    return gr;
}

// Whether the patches p, p + every, p - every ... of the team are on this XCD.
__device__ __forceinline__ bool on_one_xcd(double *maxima, const PatchArgs &a, int p, int every, double *red,
                                           int &dead)
{
    double *ids = maxima + (kPatchMeetings - 1) * a.n_patches;
    int *all = reinterpret_cast<int *>(red + 38);
    const int id = __builtin_amdgcn_s_getreg(kXccId) & 15;
    if (threadIdx.x == 0) {
        *all = 1;
        put_word(ids + p, static_cast<double>(id), 0u);
    }
    bool other = false;
    for (int b = threadIdx.x; b < a.n_patches; b += blockDim.x) {
        unsigned polls = 0;
        unsigned long long v;
        for (;;) {
            v = get_word(ids + b);
            if ((v >> 63) == 0ull || dead) break;
            if (!keep_waiting(polls, a.spin_limit, a.abort_word)) dead = 1;
        }
        other = other || dead || (b % every == p % every && word_value(v) != static_cast<double>(id));
    }
    dead = __builtin_amdgcn_ballot_w64(dead != 0) != 0ull ? 1 : 0;
    __syncthreads();
    if (other) *all = 0;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*all) != 0;
}

// The largest v of all patches of the team (v: the patch's, in all threads).
__device__ __forceinline__ double max_of_team(double v, double *maxima, unsigned &meeting,
                                              const PatchArgs &a, int p, bool near, double *red,
                                              int *s_flag, int &dead, int n_waves, int wave, int lane)
{
    double *mx = maxima + (meeting & 1u) * (kPatchCopies * a.n_patches);
    const unsigned phase = (meeting >> 1) & 1u;
    if (threadIdx.x == 0) put_word(mx + p, v, phase, near);
    for (int b = threadIdx.x; b < a.n_patches; b += blockDim.x) {
        unsigned polls = 0;
        unsigned long long x;
        for (;;) {
            x = get_word(mx + b);
            if (static_cast<unsigned>(x >> 63) == phase || dead) break;
            if (!keep_waiting(polls, a.spin_limit, a.abort_word)) dead = 1;
        }
        v = fmax(v, word_value(x));
    }
    meeting += 1u;
    dead = __builtin_amdgcn_ballot_w64(dead != 0) != 0ull ? 1 : 0;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    if (dead) *s_flag = 1;
    __syncthreads();
    for (int q = 0; q < n_waves; ++q) v = fmax(v, red[q]);
    return v;
}

// By one thread of a patch: lambda as this patch has it.
template <bool MULTI, bool ADAPT>
__device__ __forceinline__ void report_lambda(double lam, const PatchArgs &a, int plan, const int *s_flag,
                                              const int *s_wide)
{
    if constexpr (MULTI) {
        // (the largest of non-negative numbers is the largest of their bit patterns, and a quiet NaN is
        // above them all)
        if ((*s_flag & 1) || *s_wide != 0) lam = __longlong_as_double(0x7FF8000000000000ll);
        if (!ADAPT && *s_wide != 0)
            __hip_atomic_store(a.abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        (void)__hip_atomic_fetch_max(reinterpret_cast<unsigned long long *>(a.lambda + plan),
                                     static_cast<unsigned long long>(__double_as_longlong(lam)),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        a.lambda[plan] = lam;
    }
}

// a team that gave up leaves its other plans undone
__device__ __forceinline__ void give_up_rest(const PatchArgs &a, int plan, int t)
{
    if (t == 0)
        for (int rest = plan + a.teams; rest < a.plans; rest += a.teams)
            (void)__hip_atomic_fetch_max(reinterpret_cast<unsigned long long *>(a.lambda + rest),
                                         0x7FF8000000000000ull, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
}

// One plan of a fabric of one patch whose demands no grid holds: the thread of a commodity scans
// its slots where they lie in memory, and loads are added as binary64 numbers thread after thread,
// so always in the same order.  Prices, lengths and counts stand at their start.
template <bool PRODUCT, int L, int QL, bool MAXC>
__device__ __forceinline__ void solve_wide(const PatchArgs &a, int plan, int n_comm, int n_local,
                                           const int32_t *loc_link, int count, LinkState *links,
                                           double *red)
{
    constexpr int NW = PRODUCT ? kPatchWordsProduct : kPatchWordsPlain;
    const int t = threadIdx.x, NT = blockDim.x, lane = t & (kWave - 1), wave = t >> 6;
    const int n_waves = NT >> 6;
    const uint32_t pad = 8u * static_cast<uint32_t>(n_local);
    double *price = lds_ptr(0);
    const int k = t < n_comm ? a.comm[t] : -1;
    const double d = k >= 0 ? a.demand[static_cast<size_t>(plan) * a.K + k] : 0.0;
    auto half = [&](int si, int x, int h) {
        const uint32_t w = a.words[(static_cast<size_t>(si / L) * NW + x) * NT + t * L + si % L];
        return (w >> (16 * h)) & 0xFFFFu;
    };
    // offset x of slot si, in the order of the first-use bits (see host_patch.hpp)
    auto offset = [&](int si, int x) {
        if constexpr (PRODUCT)
            return x < 4 ? half(si, x / 2, x & 1)
                         : x == 4 ? half(si, 2, 0) : half(si, (x + 1) / 2, 1 - (x & 1));
        else
            return x % 5 == 4 ? half(si, 8 + x / 10, x / 5 & 1)
                              : half(si, 2 * (x / 5) + x % 5 / 2, x % 5 & 1);
    };
    // link i of the path in place `pos` of slot si
    auto step = [&](int si, int pos, int i) {
        if constexpr (PRODUCT)
            return offset(si, i < 2 ? 2 * i + (pos >> 1) : i == 2 ? 4 : 2 * i - 1 + (pos & 1));
        else
            return offset(si, 5 * pos + i);
    };
    auto add = [&](uint32_t off) {
        if (off >= pad) return;
        LinkState &s = links[off / 8u];
        s.load = static_cast<unsigned long long>(
            __double_as_longlong(__longlong_as_double(static_cast<long long>(s.load)) + d));
    };
    auto in_turn = [&](auto f) {
#pragma unroll 1
        for (int turn = 0; turn < n_waves; ++turn) {
            if (turn == wave)
#pragma unroll 1
                for (int i = 0; i < kWave; ++i) {
                    if (i == lane && k >= 0) f();
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                    __builtin_amdgcn_wave_barrier();
                }
            __syncthreads();
        }
    };
    auto take = [&](int i) {
        const double v = __longlong_as_double(static_cast<long long>(links[i].load));
        links[i].load = 0ull;
        return v;
    };
    auto largest = [&](double v) {
        v = wave_max(v);
        __syncthreads();
        if (lane == 0) red[wave] = v;
        __syncthreads();
        for (int q = 0; q < n_waves; ++q) v = fmax(v, red[q]);
        return v;
    };
    for (int i = t; i < n_local; i += NT) links[i].load = 0ull;
    __syncthreads();
    in_turn([&] {
#pragma unroll 1
        for (int si = 0; si < L * QL; ++si) {
            const uint32_t once = a.first[static_cast<size_t>(si / L) * NT + t * L + si % L];
#pragma unroll 1
            for (int x = 0; x < (PRODUCT ? 9 : 20); ++x)
                if ((once >> x) & 1u) add(offset(si, x));
        }
    });
    double wmax = 0.0;
    for (int i = t; i < n_local; i += NT) wmax = fmax(wmax, take(i) * links[i].invcap);
    wmax = largest(wmax);
    const double invrho = wmax > 0.0 ? 1.0 / wmax : 0.0;
#pragma unroll 1
    for (int it = 0; it < a.iters; ++it) {
        double best = 0.0;
        int at = -1;                             // 4 * slot + place of the cheapest, first in order
#pragma unroll 1
        for (int si = 0; k >= 0 && si < L * QL; ++si) {
            const uint32_t meta = half(si, PRODUCT ? 2 : NW - 1, 1);
#pragma unroll 1
            for (int c = 0; c < static_cast<int>(meta >> 9); ++c) {
                const int pos = c << ((meta >> 7) & 3u);
                double cost = lds_f64(step(si, pos, 0));
#pragma unroll 1
                for (int i = 1; i < 5; ++i) cost = join<MAXC>(cost, lds_f64(step(si, pos, i)));
                if (at < 0 || cost < best) {
                    best = cost;
                    at = 4 * si + pos;
                }
            }
        }
        if (at >= 0)                             // (no other thread counts in this word)
            *reinterpret_cast<uint32_t *>(lds_ptr(count + 8 * (t * (L * QL) + at / 4) +
                                                  4 * ((at >> 1) & 1))) += 1u << (16 * (at & 1));
        in_turn([&] {
#pragma unroll 1
            for (int i = 0; i < 5; ++i) add(step(at / 4, at & 3, i));
        });
        for (int i = t; i < n_local; i += NT) {
            LinkState &s = links[i];
            const double u = take(i) * s.invcap;
            s.S = s.S + u;
            const double gn = u * invrho;
            const double t1 = a.eps * gn;
            const double t2 = 1.0 + t1;
            const double ln = s.len * t2;
            s.len = ln;
            price[i] = link_price<MAXC>(ln, s.invcap);
        }
        __syncthreads();
    }
    const double T = static_cast<double>(a.iters);
    double *out = k >= 0 ? a.splits + static_cast<size_t>(plan) * a.P + a.comm_ptr[k] : nullptr;
#pragma unroll 1
    for (int si = 0; k >= 0 && si < L * QL; ++si) {
        const uint32_t meta = half(si, PRODUCT ? 2 : NW - 1, 1);
#pragma unroll 1
        for (int c = 0; c < static_cast<int>(meta >> 9); ++c) {
            const int pos = c << ((meta >> 7) & 3u);
            const uint32_t two = *reinterpret_cast<const uint32_t *>(
                lds_ptr(count + 8 * (t * (L * QL) + si) + 4 * (pos >> 1)));
            out[(meta & 127u) + c] = static_cast<double>((two >> (16 * (pos & 1))) & 0xFFFFu) / T;
        }
    }
    double smax = 0.0;
    for (int i = t; i < n_local; i += NT) {
        smax = fmax(smax, links[i].S);
        if (a.len_out != nullptr && (loc_link[i] & kPatchExport) && loc_link[i] >= 0)
            a.len_out[loc_link[i] & ~kPatchExport] = links[i].len;
    }
    smax = largest(smax);
    if (t == 0) a.lambda[plan] = smax / T;
}

// ADAPT: the solve of variable step (one plan, path cost = the sum of the prices).
template <bool PRODUCT, int L, int QL, bool MAXC, bool MULTI, bool ADAPT>
__global__ __launch_bounds__(kPatchThreads) void k_patch(PatchArgs a)
{
    constexpr int NW = PRODUCT ? kPatchWordsProduct : kPatchWordsPlain;
    const int t = threadIdx.x, NT = blockDim.x;
    const int lane = t & (kWave - 1), n_waves = NT >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // Workgroups go to the XCDs in turn.  Teams that fit one XCD are laid out in one each.  (Whether
    // it came to that is seen below.)
    int team = blockIdx.x, p = 0;
    if constexpr (MULTI) {
        const int x = blockIdx.x % a.near_xcds, i = blockIdx.x / a.near_xcds;
        team = x + a.near_xcds * (i / a.n_patches);
        p = i % a.n_patches;
        if (team >= a.teams) return;                                       // workgroup-uniform
    }
    const int32_t *dsc = a.desc + kPatchDescInts * p;
    const int n_local = dsc[1], n_shared = MULTI ? dsc[2] : 0, n_groups = MULTI ? dsc[4] : 0;
    const int n_comm = dsc[6];
    const int n_at = MULTI ? a.group[dsc[3] + n_groups] : 0;
    const int32_t *comm = a.comm + dsc[5];
    const int32_t *loc_link = a.loc_link + dsc[0];
    constexpr int kSlotBytes = ADAPT ? 32 : 8;
    const Lds l = lds_layout(n_local, n_groups, n_at, n_comm, L * QL, kSlotBytes);
    const uint32_t pad = 8u * static_cast<uint32_t>(n_local);
    double *price = lds_ptr(0), *red = lds_ptr(l.red);
    LinkState *links = reinterpret_cast<LinkState *>(lds_ptr(l.link));
    int *s_flag = reinterpret_cast<int *>(red + 39), *s_wide = s_flag + 1;
    int *groups = reinterpret_cast<int *>(s_lds + l.group);          // users of group q: from groups[q] on

    // this lane's share of the lists, for the whole solve
    const int j = t % L, g = t / L;
    uint32_t w[QL][NW];
#pragma unroll
    for (int q = 0; q < QL; ++q)
#pragma unroll
        for (int x = 0; x < NW; ++x)
            w[q][x] = a.words[((static_cast<size_t>(p) * QL + q) * NW + x) * NT + t];
    const bool busy = (wave * kWave) / L < n_comm;         // this wave has commodities
    if constexpr (MULTI)
    {
        for (int q = t; q <= n_groups; q += NT) groups[q] = a.group[dsc[3] + q];
        for (int q = t; q < n_at; q += NT)
            reinterpret_cast<uint16_t *>(s_lds + l.at)[q] = a.at[dsc[7] + q];
    }

    unsigned exchange = 0u;          // exchanges made so far, the same in all patches of a team
    unsigned meeting = 0u;           // maxima folded over all patches so far
    int dead = a.spin_limit == 0u ? 1 : 0;       // this wave has given up waiting
    double *parts_of_team = nullptr, *maxima_of_team = nullptr;
    if constexpr (MULTI) {
        parts_of_team = a.parts + static_cast<size_t>(team) * 2 * a.n_parts;
        maxima_of_team = a.maxima + static_cast<size_t>(team) * patch_meeting_words(a.n_patches);
    }
    bool near = false;               // the whole team is on this XCD
    if constexpr (MULTI)
        if (a.near_xcds > 1) near = on_one_xcd(maxima_of_team, a, p, 1, red, dead);
    // ADAPT, a team that is spread: patches meet XCD by XCD
    const bool by_xcd = MULTI && ADAPT && a.near_xcds == 1 && a.by_xcd != 0;
    bool by_xcd_near = false;
    if constexpr (MULTI && ADAPT)
        if (by_xcd) by_xcd_near = on_one_xcd(maxima_of_team, a, p, kPatchXcds, red, dead);

    for (int plan = team; plan < a.plans; plan += MULTI ? a.teams : a.plans) {
        const double *demand = a.demand + static_cast<size_t>(plan) * a.K;
        double *splits = a.splits + static_cast<size_t>(plan) * a.P;
        const double d = g < n_comm ? demand[comm[g]] : 0.0;
        __syncthreads();                 // (the plan before is done with LDS)
        for (int i = t; i < n_local; i += NT) {
            const int e = loc_link[i];
            const double ic = e >= 0 ? a.invcap[e & ~kPatchExport] : 0.0;
            const double l0 = a.len_in && e >= 0 ? a.len_in[e & ~kPatchExport] : 1.0;
            links[i].load = 0ull;
            links[i].low = 0ull;
            links[i].len = l0;
            links[i].S = 0.0;
            links[i].invcap = ic;
            price[i] = link_price<MAXC>(l0, ic);
        }
        for (int i = t; i < n_comm * L * QL * (kSlotBytes / 8); i += NT) lds_ptr(l.count)[i] = 0.0;
        if (t == 0) {
            price[n_local] = 0.0;
            price[n_local + 1] = __builtin_inf();
            *s_flag = 0;
        }
        const Grid gr = find_grid(j == 0 ? d : 0.0, red, s_wide, n_waves, wave, lane);
        const Demand units = on_grid(d, gr);
        // width rho: every commodity that can reach a link counts once
        if constexpr (!ADAPT) {
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                const uint32_t once = a.first[(static_cast<size_t>(p) * QL + q) * NT + t];
                constexpr int n_off = PRODUCT ? 9 : 20;
                uint32_t off[n_off];
#pragma unroll
                for (int x = 0; x < n_off; ++x) {
                    // where offset x of a slot is kept (see host_patch.hpp)
                    const uint32_t word = PRODUCT ? w[q][x < 4 ? x / 2 : x == 4 ? 2 : (x + 1) / 2]
                                                  : w[q][x % 5 == 4 ? 8 + x / 10 : 2 * (x / 5) + (x % 5) / 2];
                    const bool high = PRODUCT ? (x < 4 ? x & 1 : x != 4 && !(x & 1))
                                              : (x % 5 == 4 ? (x / 5) & 1 : (x % 5) & 1);
                    off[x] = high ? word >> 16 : word & 0xFFFFu;
                    if (!((once >> x) & 1u)) off[x] = pad;
                }
                add_loads<n_off>(links, pad, off, gr, units);
            }
        }
        __syncthreads();
        if constexpr (!MULTI && !ADAPT)
            if (__builtin_amdgcn_readfirstlane(*s_wide) != 0) {              // workgroup-uniform
                solve_wide<PRODUCT, L, QL, MAXC>(a, plan, n_comm, n_local, loc_link, l.count, links,
                                                 red);
                return;
            }
        double wmax = 0.0;
        auto publish = [&](double v, int i) {
            put_word(parts_of_team + (exchange & 1u) * a.n_parts + p * a.row * kPatchGroup + i, v,
                     (exchange >> 1) & 1u, near);
        };
        if constexpr (!ADAPT)
            for (int i = t; i < n_local; i += NT) {
                const double reach = take_load(links[i], gr);
                if (MULTI && i < n_shared) publish(reach, i);
                else wmax = fmax(wmax, reach * links[i].invcap);
            }
        // f(local link, load) for the shared links
        const int lanes = MULTI ? patch_link_lanes(NT, a.row) : 1;
        const int per_wave = kWave / lanes;
        auto for_shared = [&](auto f) {
            for (int i0 = wave * per_wave; i0 < n_shared; i0 += n_waves * per_wave) {
                const int i = i0 + (lane & (per_wave - 1));
                const int q = i < n_shared ? i / kPatchGroup : 0, from = groups[q];
                const double load = load_of_link(
                    parts_of_team + (exchange & 1u) * a.n_parts, l.at + 2 * from, groups[q + 1] - from,
                    a.max_users, lane / per_wave, lanes, i & (kPatchGroup - 1), (exchange >> 1) & 1u,
                    a.spin_limit, a.abort_word, dead);
                if (lane < per_wave && i < n_shared) f(i, load);
            }
        };
        if constexpr (MULTI && !ADAPT) {
            for_shared([&](int i, double reach) { wmax = fmax(wmax, reach * links[i].invcap); });
            exchange += 1u;
        }
        if constexpr (!ADAPT) {
            wmax = wave_max(wmax);
            __syncthreads();
            if (lane == 0) red[wave] = wmax;
            __syncthreads();
            for (int q = 0; q < n_waves; ++q) wmax = fmax(wmax, red[q]);
            if constexpr (MULTI) {
                wmax = max_of_team(wmax, maxima_of_team, meeting, a, p, near, red, s_flag, dead, n_waves,
                                   wave, lane);
            }
        }
        const double invrho = wmax > 0.0 ? 1.0 / wmax : 0.0;

        auto update = [&](int i, double load) {
            LinkState &s = links[i];
            const double ic = s.invcap;
            const double u = load * ic;
            s.S = s.S + u;
            const double gn = u * invrho;
            const double t1 = a.eps * gn;
            const double t2 = 1.0 + t1;
            const double ln = s.len * t2;
            s.len = ln;
            price[i] = link_price<MAXC>(ln, ic);
        };
        // Scan and scatter of an iteration.  ADAPT: `mark` receives the LDS offset of the chosen
        // candidate's weight (0: not this lane's to keep), and where `terms` is given the
        // commodity's term of the bound, demand times cheapest cost, is published there.
        auto pass = [&](double *terms, unsigned term_phase, uint32_t &mark) {
            // Two slots a lane: every slot's candidates one by one.  That spares the second look at the
            // best slot's prices, one trip to the LDS of the five in the chain of an iteration (2 nodes
            // of 8 0.902 -> 0.835 us, with two NICs in reach 1.355 -> 1.230, 8 such nodes 2.27 -> 2.06).
            // The largest price gains as well (2 nodes of 8 482 -> 462 us for 500 iterations, 20 nodes 1836 ->
            // 1664).  With one slot the prices are at hand anyway: a variable step is 1 % faster this way (16
            // nodes 5.54 -> 5.48), the largest price neither way (eleven fabrics, -0.7 to 0.5 %), the sum 0.5 %
            // slower (16 nodes 2.217 -> 2.229).  From three slots on the additions cost more than the trip (one
            // patch of 24 GPUs 1.454 -> 1.492 with four, of 30 2.44 -> 2.60 with six).
            constexpr bool kEach = PRODUCT && (QL == 2 || (QL == 1 && ADAPT));
            double best = 0.0;
            uint32_t wb[NW];             // the slot that holds the best candidate so far
            int sb = 0, pos = 0;
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                if constexpr (QL > 1 || !PRODUCT)
#pragma unroll
                    for (int x = 0; x < NW; ++x) keep_in_loop(w[q][x]);
                const uint32_t *ws = w[q];
                double m;
                int at = 0;
                if constexpr (PRODUCT) {
                    const double mid = lds_lo(ws[2]);
                    const double t0 = join<MAXC>(join<MAXC>(lds_lo(ws[0]), lds_lo(ws[1])), mid);
                    const double t2 = join<MAXC>(join<MAXC>(lds_hi(ws[0]), lds_hi(ws[1])), mid);
                    if constexpr (kEach) {
                        const double d0 = lds_lo(ws[3]), d1 = lds_hi(ws[3]);
                        const double e0 = lds_lo(ws[4]), e1 = lds_hi(ws[4]);
                        const double c0 = join<MAXC>(join<MAXC>(t0, d0), e0);
                        const double c1 = join<MAXC>(join<MAXC>(t0, d1), e1);
                        const double c2 = join<MAXC>(join<MAXC>(t2, d0), e0);
                        m = fast_min_f64(fast_min_f64(c0, c1),
                                         fast_min_f64(c2, join<MAXC>(join<MAXC>(t2, d1), e1)));
                        at = select(c2 == m, 2, 3);
                        at = select(c1 == m, 1, at);
                        at = select(c0 == m, 0, at);
                    } else {
                        // Of the two ways to reach the middle link the cheaper one is the cheaper
                        // one for every way on: rounded additions keep the order.  (Which of equally
                        // cheap candidates comes first is settled below.)
                        const double tm = fast_min_f64(t0, t2);
                        m = fast_min_f64(join<MAXC>(join<MAXC>(tm, lds_lo(ws[3])), lds_lo(ws[4])),
                                         join<MAXC>(join<MAXC>(tm, lds_hi(ws[3])), lds_hi(ws[4])));
                    }
                } else {
                    double c[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        c[x] = join<MAXC>(
                            join<MAXC>(join<MAXC>(lds_lo(ws[2 * x]), lds_hi(ws[2 * x])),
                                       lds_lo(ws[2 * x + 1])),
                            lds_hi(ws[2 * x + 1]));
                        c[x] = join<MAXC>(c[x], x & 1 ? lds_hi(ws[8 + x / 2])
                                                      : lds_lo(ws[8 + x / 2]));
                    }
                    m = fast_min_f64(fast_min_f64(c[0], c[1]), fast_min_f64(c[2], c[3]));
                    at = select(c[2] == m, 2, 3);
                    at = select(c[1] == m, 1, at);
                    at = select(c[0] == m, 0, at);
                }
                if (q == 0) {
                    best = m;
                    pos = at;
#pragma unroll
                    for (int x = 0; x < NW; ++x) wb[x] = ws[x];
                } else {
                    // the strict `<` of a scan in candidate order
                    const bool better = m < best;
                    best = fast_min_f64(best, m);
                    sb = select(better, q, sb);
                    if constexpr (!PRODUCT || kEach) pos = select(better, at, pos);
                    take_words<NW>(wb, w[q], better);
                }
            }
            uint32_t off[5];
            if constexpr (PRODUCT && !kEach) {
                // the candidates of the best slot, exactly: the first that costs `best`
                const double mid = lds_lo(wb[2]);
                const double t0 = join<MAXC>(join<MAXC>(lds_lo(wb[0]), lds_lo(wb[1])), mid);
                const double t2 = join<MAXC>(join<MAXC>(lds_hi(wb[0]), lds_hi(wb[1])), mid);
                const double d0 = lds_lo(wb[3]), d1 = lds_hi(wb[3]);
                const double e0 = lds_lo(wb[4]), e1 = lds_hi(wb[4]);
                pos = select(join<MAXC>(join<MAXC>(t2, d0), e0) == best, 2, 3);
                pos = select(join<MAXC>(join<MAXC>(t0, d1), e1) == best, 1, pos);
                pos = select(join<MAXC>(join<MAXC>(t0, d0), e0) == best, 0, pos);
            }
            // (a commodity whose candidates all cost +inf resolves to its first)
            pos = select(best < __builtin_inf(), pos, 0);
            const uint32_t meta = (PRODUCT ? wb[2] : wb[NW - 1]) >> 16;
            bool mine = (meta >> 9) != 0u;
            if constexpr (L > 1) {
                const int cand = select(
                    mine, static_cast<int>(meta & 127u) + (pos >> ((meta >> 7) & 3u)), kNone);
                mine = group_argmin_two_pass<L>(best, cand) == cand && mine;
            }
            if constexpr (PRODUCT) {
                const int hs = (pos & 2) << 3, ls = (pos & 1) << 4;
                off[0] = (wb[0] >> hs) & 0xFFFFu;
                off[1] = (wb[1] >> hs) & 0xFFFFu;
                off[2] = wb[2] & 0xFFFFu;
                off[3] = (wb[3] >> ls) & 0xFFFFu;
                off[4] = (wb[4] >> ls) & 0xFFFFu;
            } else {
                const bool hi = pos & 2, odd = pos & 1;
                const uint32_t x = select(hi, select(odd, wb[6], wb[4]), select(odd, wb[2], wb[0]));
                const uint32_t y = select(hi, select(odd, wb[7], wb[5]), select(odd, wb[3], wb[1]));
                const uint32_t z = select(hi, wb[9], wb[8]);
                off[0] = x & 0xFFFFu;
                off[1] = x >> 16;
                off[2] = y & 0xFFFFu;
                off[3] = y >> 16;
                off[4] = (z >> (odd ? 16 : 0)) & 0xFFFFu;
            }
            if (mine) {
                add_loads<5>(links, pad, off, gr, units);
                const int slot = l.count + kSlotBytes * (g * (L * QL) + sb * L + j);
                if constexpr (ADAPT) {
                    mark = static_cast<uint32_t>(slot + 8 * pos);
                    if (terms != nullptr) put_word(terms + comm[g], d * best, term_phase, near);
                } else {
                    (void)__hip_atomic_fetch_add(
                        reinterpret_cast<uint32_t *>(lds_ptr(slot + 4 * (pos >> 1))),
                        1u << (16 * (pos & 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        };

        double W = 0.0;                  // ADAPT: sum of the steps, their number
        int done = 0;
        if constexpr (ADAPT) {
            // Iteration t steps by sigma = 1 / (largest normalised load of any link), so all
            // patches meet once more per iteration.  Every check_every iterations the bound
            // (sum of demand * cheapest cost) / (sum of lengths) is taken with sums in index
            // order: patches publish the terms, the chunks of 256 terms are dealt to the waves of
            // all patches, and the first wave of every patch adds the chunk sums and decides --
            // all alike, so nobody has to be told.
            const int n_alpha = (a.K + 255) / 256, n_d = (a.E + 255) / 256;
            const int64_t n_words = static_cast<int64_t>(a.K) + a.E + n_alpha + n_d;
            const double gap = (1.0 + a.eps) * (1.0 + a.eps);
            double lb_best = 0.0;
            int until_check = a.check_every;
            unsigned checks = 0u;
            // The largest v of all patches; `row` alternates between calls.  The first wave leaves
            // its patch's maximum in every copy of the list and waits for the others' in its own
            // copy: one list polled by every wave of every patch made the few cache lines it
            // lies in the bottleneck.
            auto meet = [&](double v, int row) {
                double *r = red + 16 * row;
                v = wave_max(v);
                if (lane == 0) r[wave] = v;
                __syncthreads();
                if (MULTI ? wave == 0 : true)
                    for (int q = 0; q < n_waves; ++q) v = fmax(v, r[q]);
                if constexpr (MULTI) {
                    if (wave == 0 && by_xcd) {
                        // through the leader of the XCD (its first patch), so that every list is
                        // read on one XCD or has eight words
                        const unsigned phase = (meeting >> 1) & 1u;
                        const int x = p % kPatchXcds;
                        double *here = maxima_of_team + kPatchMeetings * a.n_patches +
                                       (meeting & 1u) * kPatchTree / 2;
                        double *all = here + kPatchXcds * kPatchXcdPatches;
                        here += x * kPatchXcdPatches;
                        if (lane == 0) put_word(here + p / kPatchXcds, v, phase, by_xcd_near);
                        auto await_max = [&](const double *w, bool mine) {
                            unsigned polls = 0;
                            unsigned long long b = static_cast<unsigned long long>(phase) << 63;
                            for (;;) {
                                if (mine) b = get_word(w);
                                if (__builtin_amdgcn_ballot_w64(static_cast<unsigned>(b >> 63) != phase) == 0ull ||
                                    dead)
                                    break;
                                const int late = keep_waiting(polls, a.spin_limit, a.abort_word) ? 0 : 1;
                                dead = __builtin_amdgcn_readfirstlane(late);
                            }
                            return word_value(b);
                        };
                        if (p < kPatchXcds) {
                            const double m = wave_max(await_max(
                                here + lane, lane < (a.n_patches - p + kPatchXcds - 1) / kPatchXcds));
                            if (lane == 0) put_word(all + x * kPatchLine, m, phase);
                        }
                        v = await_max(all + lane * kPatchLine, lane < kPatchXcds);
                        v = wave_max(v);
                        if (lane == 0) r[0] = v;
                    } else if (wave == 0) {
                        double *mx = maxima_of_team + (meeting & 1u) * (kPatchCopies * a.n_patches);
                        const unsigned phase = (meeting >> 1) & 1u;
                        if (lane < kPatchCopies)
                            put_word(mx + lane * a.n_patches + p, v, phase, near);
                        mx += (p & (kPatchCopies - 1)) * a.n_patches;
                        for (int b = lane; b < a.n_patches; b += kWave) {
                            unsigned polls = 0;
                            unsigned long long x;
                            for (;;) {
                                x = get_word(mx + b);
                                if (static_cast<unsigned>(x >> 63) == phase || dead) break;
                                if (!keep_waiting(polls, a.spin_limit, a.abort_word)) dead = 1;
                            }
                            v = fmax(v, word_value(x));
                        }
                        dead = __builtin_amdgcn_ballot_w64(dead != 0) != 0ull ? 1 : 0;
                        v = wave_max(v);
                        if (lane == 0) r[0] = v;
                    }
                    meeting += 1u;
                    __syncthreads();
                    v = r[0];
                }
                return v;
            };
            for (;;) {
                until_check -= 1;
                const bool check = until_check == 0;                         // uniform
                double *terms = a.terms + (checks & 1u) * n_words;
                const unsigned phase = (checks >> 1) & 1u;
                uint32_t mark = 0u;
                if (busy) pass(check ? terms : nullptr, phase, mark);        // wave-uniform
                __syncthreads();
                double m = 0.0;
                // the normalised load of a link waits for the step where its price was
                auto put_u = [&](int i, double load) {
                    const double u = load * links[i].invcap;
                    price[i] = u;
                    m = fmax(m, u);
                };
                if constexpr (MULTI)
                    for (int i = t; i < n_shared; i += NT) publish(take_load(links[i], gr), i);
                for (int i = n_shared + t; i < n_local; i += NT) put_u(i, take_load(links[i], gr));
                if (check) {
                    for (int i = t; i < n_local; i += NT) {
                        const int e = loc_link[i];
                        if (e >= 0 && (e & kPatchExport))
                            put_word(terms + a.K + (e & ~kPatchExport), links[i].len, phase, near);
                    }
                    if (p == 0)                      // links no candidate uses keep length 1
                        for (int i = t; i < a.n_idle; i += NT)
                            put_word(terms + a.K + a.idle[i], 1.0, phase, near);
                }
                if constexpr (MULTI) {
                    for_shared(put_u);
                    exchange += 1u;
                }
                const double umax = meet(m, 0);
                double smax = 0.0;
                const bool traffic = umax > 0.0;
                if (traffic) {
                    const double sigma = 1.0 / umax;
                    W = W + sigma;
                    for (int i = t; i < n_local; i += NT) {
                        LinkState &s = links[i];
                        const double su = sigma * price[i];
                        const double S = s.S + su;
                        s.S = S;
                        smax = fmax(smax, S);
                        const double t1 = a.eps * su;
                        const double t2 = 1.0 + t1;
                        const double ln = s.len * t2;
                        s.len = ln;
                        price[i] = link_price<MAXC>(ln, s.invcap);
                    }
                    if (mark != 0u) *lds_ptr(mark) = *lds_ptr(mark) + sigma;
                    done += 1;
                }
                bool stop = !traffic || done == a.iters;
                if (check) {
                    double *sums = terms + a.K + a.E;
                    for (int c = p * n_waves + wave; c < n_alpha + n_d; c += a.n_patches * n_waves) {
                        const bool alpha = c < n_alpha;
                        const int at = 256 * (alpha ? c : c - n_alpha);
                        const int n = (alpha ? a.K : a.E) - at;
                        const double v = sum_in_order(terms + (alpha ? 0 : a.K) + at,
                                                      n < 256 ? n : 256, phase, a.spin_limit,
                                                      a.abort_word, dead, lane);
                        if (lane == 0) put_word(sums + c, v, phase, near);
                    }
                    smax = meet(smax, 1);
                    if (wave == 0 && traffic) {
                        const double alpha = sum_in_order(sums, n_alpha, phase, a.spin_limit,
                                                          a.abort_word, dead, lane);
                        const double D = sum_in_order(sums + n_alpha, n_d, phase, a.spin_limit,
                                                      a.abort_word, dead, lane);
                        const double lb = alpha / D;
                        if (lb > lb_best) lb_best = lb;
                        const double lam = smax / W;
                        const double bound = gap * lb_best;
                        if (lam <= bound) stop = true;
                    }
                    until_check = a.check_every;
                    checks += 1u;
                }
                if (dead) atomicOr(s_flag, 1);
                // (`stop` may be set in the first wave only: the flag is what counts)
                else if (stop && wave == 0 && lane == 0) atomicOr(s_flag, 2);
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(*s_flag) != 0) break;     // workgroup-uniform
            }
            if (t == 0) {
                if ((*s_flag & 1) || *s_wide != 0) a.ad_flags[0] = 2;
                if (p == 0) {
                    a.ad_flags[1] = done;
                    a.ad_scalars[2] = lb_best;
                }
            }
        }
        for (int it = 0; !ADAPT && it < a.iters; ++it) {
            uint32_t mark;
            if (busy) pass(nullptr, 0u, mark);                               // wave-uniform
            __syncthreads();
            if constexpr (MULTI) {
                for (int i = t; i < n_shared; i += NT) publish(take_load(links[i], gr), i);
                for (int i = n_shared + t; i < n_local; i += NT) update(i, take_load(links[i], gr));
                for_shared(update);
                exchange += 1u;
                if (dead) *s_flag = 1;
            } else {
                for (int i = t; i < n_local; i += NT) update(i, take_load(links[i], gr));
            }
            __syncthreads();
            // (looked at now and then only: whoever has given up waits no more)
            if constexpr (MULTI)
                if ((it & 31) == 31 && __builtin_amdgcn_readfirstlane(*s_flag) != 0) break;    // uniform
        }
        const double T = ADAPT ? W : static_cast<double>(a.iters);
        if (g < n_comm) {
            double *out0 = splits + a.comm_ptr[comm[g]];
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                const uint32_t meta = (PRODUCT ? w[q][2] : w[q][NW - 1]) >> 16;
                const int n = static_cast<int>(meta >> 9);
                const int shift = static_cast<int>((meta >> 7) & 3u);
                if (n == 0) continue;
                double *out = out0 + (meta & 127u);
                const int slot = l.count + kSlotBytes * (g * (L * QL) + q * L + j);
                if constexpr (ADAPT) {
                    const int first = static_cast<int>(meta & 127u);
#pragma unroll
                    for (int pos = 0; pos < 4; ++pos)
                        if ((pos & ((1 << shift) - 1)) == 0 && (pos >> shift) < n)
                            out[pos >> shift] = T > 0.0 ? lds_ptr(slot)[pos] / T
                                                        : (first + (pos >> shift) == 0 ? 1.0 : 0.0);
                    continue;
                }
                const uint2 c = *reinterpret_cast<const uint2 *>(lds_ptr(slot));
                const uint32_t n4[4] = {c.x & 0xFFFFu, c.x >> 16, c.y & 0xFFFFu, c.y >> 16};
#pragma unroll
                for (int pos = 0; pos < 4; ++pos)
                    if ((pos & ((1 << shift) - 1)) == 0 && (pos >> shift) < n)
                        out[pos >> shift] = static_cast<double>(n4[pos]) / T;
            }
        }
        double smax = 0.0;
        for (int i = t; i < n_local; i += NT) {
            smax = fmax(smax, links[i].S);
            if (a.len_out != nullptr && (loc_link[i] & kPatchExport) && loc_link[i] >= 0)
                a.len_out[loc_link[i] & ~kPatchExport] = links[i].len;
        }
        smax = wave_max(smax);
        __syncthreads();
        if (lane == 0) red[wave] = smax;
        __syncthreads();
        if (t == 0) {
            for (int q = 0; q < n_waves; ++q) smax = fmax(smax, red[q]);
            // (ADAPT, steps of zero where the largest load over a capacity is infinite: 0 / 0, no number)
            report_lambda<MULTI, ADAPT>(ADAPT && done == 0 ? 0.0 : smax / T, a, plan, s_flag, s_wide);
        }
        if constexpr (MULTI)
            if (!ADAPT && *s_flag != 0) {
                give_up_rest(a, plan, t);
                break;
            }
    }
}

using PatchKernel = void (*)(PatchArgs);

template <bool MAXC, bool MULTI, bool ADAPT>
PatchKernel kernel_for(const PatchShape &s)
{
#define NIMBLE_PATCH(PR, LL, QQ)                                                               \
    if (s.product == PR && s.lanes == LL && s.quads == QQ)                                     \
        return k_patch<PR != 0, LL, QQ, MAXC, MULTI, ADAPT>;
    NIMBLE_PATCH_SHAPES(NIMBLE_PATCH)
#undef NIMBLE_PATCH
    return nullptr;
}

}  // namespace patch

}  // namespace nimble
