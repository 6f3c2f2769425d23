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
// Exchange without barriers or fences: a part is one 8-byte word, stored and loaded at agent
// scope (past the caches that are not coherent between the XCDs), whose sign bit says which
// exchange it belongs to -- loads are never negative.  Exchange n uses buffer n & 1 and the sign
// (n >> 1) & 1; all words start with the sign set.  A patch overwrites its part of exchange n
// with that of n + 2 only after it has read all parts of n + 1 of the groups it shares, which
// their writers published after reading n: nobody misses a word.  Every wait is bounded; when one
// expires the team gives up and lambda becomes NaN.
//
// Sums of loads do not depend on the order of the atomics.  Where the demands of a patch lie on
// a power-of-two grid with a total below 2^53 units (byte counts) binary64 additions are exact;
// elsewhere a demand is split into two 64-bit integers, units of 2^-61 and 2^-105 of the patch's
// total, and integer additions are (the sum is rounded once at the end).
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

// LDS of a patch, byte offsets.  The prices come first: a slot's offsets are LDS addresses.
struct Lds {
    int acc, low, len, S, invcap, group, count, red, bytes;
};

__host__ __device__ inline Lds lds_layout(int n_local, int n_groups, int slots, int threads)
{
    Lds l;
    int o = 8 * (n_local + 2);                  // [n_local] +0.0, [n_local + 1] +inf
    l.acc = o;     o += 8 * (n_local + 2);
    l.low = o;     o += 8 * (n_local + 2);
    l.len = o;     o += 8 * n_local;
    l.S = o;       o += 8 * n_local;
    l.invcap = o;  o += 8 * n_local;
    l.red = o;     o += 8 * 40;
    l.group = o;   o += 16 * n_groups;
    l.count = o;   o += 8 * slots * threads;   // 16 bits per candidate of a slot
    l.bytes = o;
    return l;
}

// The largest of the dynamic LDS arrays has to start at LDS address 0 for the offsets to be
// addresses, so this kernel has no static LDS.
extern __shared__ __align__(16) unsigned char s_lds[];

__device__ __forceinline__ double lds_f64(uint32_t off)
{
    return *reinterpret_cast<const double *>(s_lds + off);
}
__device__ __forceinline__ double *lds_ptr(uint32_t off)
{
    return reinterpret_cast<double *>(s_lds + off);
}

template <bool MAXC>
__device__ __forceinline__ double join(double acc, double p)
{
    if constexpr (MAXC) return (p > acc) ? p : acc;
    else return acc + p;
}

// lowest cost of a slot and the position (0..3) that holds it, lowest first
template <bool PRODUCT, bool MAXC>
__device__ __forceinline__ void scan_slot(const uint32_t *w, double &m, int &pos)
{
    double c[4];
    if constexpr (PRODUCT) {
        const double a0 = lds_f64(w[0] & 0xFFFFu), a2 = lds_f64(w[0] >> 16);
        const double b0 = lds_f64(w[1] & 0xFFFFu), b2 = lds_f64(w[1] >> 16);
        const double mid = lds_f64(w[2] & 0xFFFFu);
        const double d0 = lds_f64(w[3] & 0xFFFFu), d1 = lds_f64(w[3] >> 16);
        const double e0 = lds_f64(w[4] & 0xFFFFu), e1 = lds_f64(w[4] >> 16);
        const double t0 = join<MAXC>(join<MAXC>(a0, b0), mid);
        const double t2 = join<MAXC>(join<MAXC>(a2, b2), mid);
        c[0] = join<MAXC>(join<MAXC>(t0, d0), e0);
        c[1] = join<MAXC>(join<MAXC>(t0, d1), e1);
        c[2] = join<MAXC>(join<MAXC>(t2, d0), e0);
        c[3] = join<MAXC>(join<MAXC>(t2, d1), e1);
    } else {
        double p[4][5];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p[q][0] = lds_f64(w[2 * q] & 0xFFFFu);
            p[q][1] = lds_f64(w[2 * q] >> 16);
            p[q][2] = lds_f64(w[2 * q + 1] & 0xFFFFu);
            p[q][3] = lds_f64(w[2 * q + 1] >> 16);
            p[q][4] = lds_f64((w[8 + q / 2] >> (16 * (q & 1))) & 0xFFFFu);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = p[q][0];
#pragma unroll
            for (int i = 1; i < 5; ++i) c[q] = join<MAXC>(c[q], p[q][i]);
        }
    }
    m = fast_min_f64(fast_min_f64(c[0], c[1]), fast_min_f64(c[2], c[3]));
    pos = c[0] == m ? 0 : (c[1] == m ? 1 : (c[2] == m ? 2 : 3));
}

template <bool PRODUCT>
__device__ __forceinline__ uint32_t meta_of(const uint32_t *w)
{
    return (PRODUCT ? w[2] : w[10]) >> 16;
}

// offsets of the five links of the candidate at position `pos` of a slot
template <bool PRODUCT>
__device__ __forceinline__ void links_of(const uint32_t *w, int pos, uint32_t (&off)[5])
{
    if constexpr (PRODUCT) {
        const int h = (pos & 2) << 3, l = (pos & 1) << 4;
        off[0] = (w[0] >> h) & 0xFFFFu;
        off[1] = (w[1] >> h) & 0xFFFFu;
        off[2] = w[2] & 0xFFFFu;
        off[3] = (w[3] >> l) & 0xFFFFu;
        off[4] = (w[4] >> l) & 0xFFFFu;
    } else {
        const bool hi = pos & 2, odd = pos & 1;
        const uint32_t u0 = odd ? w[2] : w[0], u1 = odd ? w[3] : w[1];
        const uint32_t v0 = odd ? w[6] : w[4], v1 = odd ? w[7] : w[5];
        const uint32_t x = hi ? v0 : u0, y = hi ? v1 : u1, z = hi ? w[9] : w[8];
        off[0] = x & 0xFFFFu;
        off[1] = x >> 16;
        off[2] = y & 0xFFFFu;
        off[3] = y >> 16;
        off[4] = (z >> (odd ? 16 : 0)) & 0xFFFFu;
    }
}

// How the loads of a patch are summed: exact in binary64, or as two integers.
struct Grid {
    bool exact;
    int scale;          // the patch's total is below 2^scale
};

// What is derived from these values is worked out where it is used: taken out of the loop over
// the iterations (they never change) it would fill more registers than there are.
__device__ __forceinline__ void keep_in_loop(uint32_t &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_in_loop(double &v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ void add_load(uint32_t acc, uint32_t low, const Grid &gr, double d)
{
    if (gr.exact) {
        (void)__builtin_amdgcn_ds_atomic_fadd_f64(
            (__attribute__((address_space(3))) double *)(lds_ptr(acc)), d);
        return;
    }
    keep_in_loop(d);
    const double h = trunc(ldexp(d, kSumBits - gr.scale));
    const double r = d - ldexp(h, gr.scale - kSumBits);
    const double l = trunc(ldexp(r, kSumBits + kLowBits - gr.scale));
    (void)__hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(lds_ptr(acc)),
                                 static_cast<unsigned long long>(static_cast<long long>(h)),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    (void)__hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(lds_ptr(low)),
                                 static_cast<unsigned long long>(static_cast<long long>(l)),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// the load of local link i, which starts at zero again
__device__ __forceinline__ double take_load(const Lds &l, int i, const Grid &gr)
{
    double *a = lds_ptr(l.acc) + i;
    const double v = *a;
    *a = 0.0;
    if (gr.exact) return v;
    double *b = lds_ptr(l.low) + i;
    const double hi = static_cast<double>(__double_as_longlong(v));
    const double lo = static_cast<double>(__double_as_longlong(*b));
    *b = 0.0;
    return ldexp(hi, gr.scale - kSumBits) + ldexp(lo, gr.scale - kSumBits - kLowBits);
}

__device__ __forceinline__ void put_word(double *p, double v, unsigned phase)
{
    const unsigned long long b = (static_cast<unsigned long long>(__double_as_longlong(v)) & ~kSign) |
                                 (static_cast<unsigned long long>(phase) << 63);
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), b, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
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

// Loads of shared links, kGroupsAtOnce groups side by side: for every group lane 8j + i adds the
// parts j, j + 8, ... of link i in order, then the eight partial sums are added in a fixed tree.
// All words are asked for together and those that have not arrived asked for again, so that the
// trips to memory of all groups overlap.  (The parts of a group are padded to a multiple of eight;
// its users write the padding too, as zeros.)  Lane 8q + i returns the load of link i of group q
// (q < kGroupsAtOnce).  `at` and `users`: first part and users of the groups (0 users: none).
constexpr int kGroupsAtOnce = 4;
constexpr int kPartsAtOnce = 4;
__device__ __forceinline__ double group_loads(const double *parts, const int (&at)[kGroupsAtOnce],
                                              const int (&users)[kGroupsAtOnce], unsigned phase,
                                              unsigned limit, unsigned *abort_word, bool &dead,
                                              int lane)
{
    const int j = lane >> 3;
    double sum[kGroupsAtOnce];
    int most = 0;
#pragma unroll
    for (int q = 0; q < kGroupsAtOnce; ++q) {
        sum[q] = 0.0;
        most = most > users[q] ? most : users[q];
    }
    for (int c0 = 0; c0 < most; c0 += 8 * kPartsAtOnce) {           // wave-uniform
        unsigned long long v[kGroupsAtOnce][kPartsAtOnce];
        unsigned polls = 0;
        for (;;) {
            unsigned any = 0u, all = ~0u;
#pragma unroll
            for (int q = 0; q < kGroupsAtOnce; ++q) {
                const double *src = parts + at[q] + c0 * kPatchGroup;         // wave-uniform
#pragma unroll
                for (int x = 0; x < kPartsAtOnce; ++x) {
                    v[q][x] = static_cast<unsigned long long>(phase) << 63;
                    if (c0 + 8 * x < users[q])                                // wave-uniform
                        v[q][x] = get_word(src + static_cast<unsigned>(lane) +
                                           x * (8 * kPatchGroup));
                }
            }
#pragma unroll
            for (int q = 0; q < kGroupsAtOnce; ++q)
#pragma unroll
                for (int x = 0; x < kPartsAtOnce; ++x) {
                    any |= static_cast<unsigned>(v[q][x] >> 32);
                    all &= static_cast<unsigned>(v[q][x] >> 32);
                }
            const bool ok = phase ? (all >> 31) != 0u : (any >> 31) == 0u;
            if (__all(ok) || dead) break;
            if (!keep_waiting(polls, limit, abort_word)) dead = true;
        }
#pragma unroll
        for (int q = 0; q < kGroupsAtOnce; ++q)
#pragma unroll
            for (int x = 0; x < kPartsAtOnce; ++x) sum[q] = sum[q] + word_value(v[q][x]);
    }
    double mine = 0.0;
#pragma unroll
    for (int q = 0; q < kGroupsAtOnce; ++q) {
        double t = sum[q] + dpp_f64<0x128>(sum[q]);     // row_ror:8, lane ^ 8
        t = add_across16(t);
        t = add_across32(t);
        mine = j == q ? t : mine;
    }
    return mine;
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

template <bool PRODUCT, int L, int QL, int R, bool MAXC, bool MULTI>
__global__ __launch_bounds__(kPatchThreads) void k_patch(PatchArgs a)
{
    constexpr int QT = QL * R;
    constexpr int NW = PRODUCT ? kPatchWordsProduct : kPatchWordsPlain;
    const int t = threadIdx.x, NT = blockDim.x;
    const int lane = t & (kWave - 1), wave = t >> 6, n_waves = NT >> 6;
    const int team = MULTI ? blockIdx.x / a.n_patches : blockIdx.x;
    const int p = MULTI ? blockIdx.x - team * a.n_patches : 0;
    const int32_t *dsc = a.desc + kPatchDescInts * p;
    const int n_local = dsc[1], n_shared = MULTI ? dsc[2] : 0, n_groups = MULTI ? dsc[4] : 0;
    const int n_comm = dsc[5];
    const int32_t *loc_link = a.loc_link + dsc[0];
    const Lds l = lds_layout(n_local, n_groups, QT, NT);
    double *price = lds_ptr(0), *len = lds_ptr(l.len), *S = lds_ptr(l.S);
    double *invcap = lds_ptr(l.invcap), *red = lds_ptr(l.red);
    int *s_flag = reinterpret_cast<int *>(red + 39);
    int4 *groups = reinterpret_cast<int4 *>(s_lds + l.group);
    // choices of slot s, candidate position pos: half pos & 1 of word (2 s + (pos >> 1)) * NT + t
    uint32_t *tally = reinterpret_cast<uint32_t *>(s_lds + l.count) + t;

    // this lane's share of the lists, for the whole solve
    uint32_t w[QT][NW];
#pragma unroll
    for (int s = 0; s < QT; ++s)
#pragma unroll
        for (int x = 0; x < NW; ++x)
            w[s][x] = a.words[((static_cast<size_t>(p) * QT + s) * NW + x) * NT + t];
    const int per = NT / L, g = t / L, j = t % L;
    if constexpr (MULTI)
        for (int q = t; q < n_groups; q += NT)
            groups[q] = reinterpret_cast<const int4 *>(a.group)[dsc[3] + q];

    unsigned exchange = 0u;          // exchanges made so far, the same in all patches of a team
    unsigned meeting = 0u;           // maxima folded over all patches so far
    bool dead = false;
    double *parts_of_team = nullptr, *maxima_of_team = nullptr;
    if constexpr (MULTI) {
        parts_of_team = a.parts + static_cast<size_t>(team) * 2 * a.n_parts;
        maxima_of_team = a.maxima + static_cast<size_t>(team) * 2 * a.n_patches;
    }

    for (int plan = team; plan < a.plans; plan += MULTI ? a.teams : a.plans) {
        const double *demand = a.demand + static_cast<size_t>(plan) * a.K;
        double *splits = a.splits + static_cast<size_t>(plan) * a.P;
        double d[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int k = a.comm[static_cast<size_t>(p) * a.n_comm_slots + r * per + g];
            d[r] = k >= 0 ? demand[k] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 2 * QT; ++s) tally[s * NT] = 0u;
        __syncthreads();                 // (the plan before is done with LDS)
        for (int i = t; i < n_local; i += NT) {
            const int e = loc_link[i];
            const double ic = e >= 0 ? a.invcap[e & ~kPatchExport] : 0.0;
            const double l0 = a.len_in && e >= 0 ? a.len_in[e & ~kPatchExport] : 1.0;
            invcap[i] = ic;
            len[i] = l0;
            price[i] = MAXC ? l0 : l0 * ic;
            S[i] = 0.0;
            lds_ptr(l.acc)[i] = 0.0;
            lds_ptr(l.low)[i] = 0.0;
        }
        if (t == 0) {
            price[n_local] = 0.0;
            price[n_local + 1] = __builtin_inf();
            *s_flag = 0;
        }
        // total and finest grid of the patch's demands
        Grid gr;
        {
            double sum = 0.0;
            int fine = 4096;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (j != 0 || d[r] == 0.0) continue;
                sum = sum + d[r];
                const unsigned long long b =
                    static_cast<unsigned long long>(__double_as_longlong(d[r]));
                const int ex = static_cast<int>((b >> 52) & 2047u);
                const unsigned long long man =
                    (b & ((1ull << 52) - 1ull)) | (ex ? 1ull << 52 : 0ull);
                fine = min(fine, (ex ? ex : 1) - 1075 + __ffsll(static_cast<long long>(man)) - 1);
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
            gr.exact = !(total > 0.0) || !(total < __builtin_inf());
            gr.scale = gr.exact ? 0 : ilogb(total) + 1;
            gr.exact = gr.exact || gr.scale - fine <= 53;
            gr.exact = __builtin_amdgcn_readfirstlane(gr.exact ? 1 : 0) != 0;
            gr.scale = __builtin_amdgcn_readfirstlane(gr.scale);
        }
        // width rho: every commodity that can reach a link counts once
#pragma unroll
        for (int s = 0; s < QT; ++s) {
            const uint32_t once = a.first[(static_cast<size_t>(p) * QT + s) * NT + t];
            constexpr int n_off = PRODUCT ? 9 : 20;
#pragma unroll
            for (int x = 0; x < n_off; ++x) {
                // where offset x of a slot is kept (see host_patch.hpp)
                const uint32_t word =
                    PRODUCT ? w[s][x < 4 ? x / 2 : x == 4 ? 2 : (x + 1) / 2]
                            : w[s][x % 5 == 4 ? 8 + x / 10 : 2 * (x / 5) + (x % 5) / 2];
                const bool high = PRODUCT ? (x < 4 ? x & 1 : x == 4 ? false : !(x & 1))
                                          : (x % 5 == 4 ? (x / 5) & 1 : (x % 5) & 1);
                if ((once >> x) & 1u) {
                    const uint32_t off = high ? word >> 16 : word & 0xFFFFu;
                    add_load(l.acc + off, l.low + off, gr, d[s / QL]);
                }
            }
        }
        __syncthreads();
        double wmax = 0.0;
        auto publish = [&](double v, int i) {
            const int4 gd = groups[i / kPatchGroup];       // first part, parts, own part, users
            double *dst = parts_of_team + (exchange & 1u) * a.n_parts + gd.x + i % kPatchGroup;
            for (int c = gd.z; c < gd.y; c += gd.w)
                put_word(dst + c * kPatchGroup, c == gd.z ? v : 0.0, (exchange >> 1) & 1u);
        };
        for (int i = t; i < n_local; i += NT) {
            const double reach = take_load(l, i, gr);
            if (MULTI && i < n_shared) publish(reach, i);
            else wmax = fmax(wmax, reach * invcap[i]);
        }
        // f(local link, load) for the shared links, a lane each; the groups of a patch are dealt
        // to its waves in bundles
        auto for_shared = [&](auto f) {
            for (int q0 = wave * kGroupsAtOnce; q0 < n_groups; q0 += n_waves * kGroupsAtOnce) {
                int at[kGroupsAtOnce], users[kGroupsAtOnce];
#pragma unroll
                for (int q = 0; q < kGroupsAtOnce; ++q) {
                    const int4 gd = groups[q0 + q < n_groups ? q0 + q : q0];
                    at[q] = __builtin_amdgcn_readfirstlane(gd.x);
                    users[q] = __builtin_amdgcn_readfirstlane(q0 + q < n_groups ? gd.y : 0);
                }
                const double load =
                    group_loads(parts_of_team + (exchange & 1u) * a.n_parts, at, users,
                                (exchange >> 1) & 1u, a.spin_limit, a.abort_word, dead, lane);
                if (lane < kGroupsAtOnce * kPatchGroup && q0 + (lane >> 3) < n_groups)
                    f(q0 * kPatchGroup + lane, load);
            }
        };
        if constexpr (MULTI) {
            for_shared([&](int i, double reach) { wmax = fmax(wmax, reach * invcap[i]); });
            exchange += 1u;
        }
        wmax = wave_max(wmax);
        __syncthreads();
        if (lane == 0) red[wave] = wmax;
        __syncthreads();
        for (int q = 0; q < n_waves; ++q) wmax = fmax(wmax, red[q]);
        if constexpr (MULTI) {
            // the maximum over all patches of the team
            double *mx = maxima_of_team + (meeting & 1u) * a.n_patches;
            const unsigned phase = (meeting >> 1) & 1u;
            if (t == 0) put_word(mx + p, wmax, phase);
            for (int b = t; b < a.n_patches; b += NT) {
                unsigned polls = 0;
                unsigned long long v;
                for (;;) {
                    v = get_word(mx + b);
                    if (static_cast<unsigned>(v >> 63) == phase || dead) break;
                    if (!keep_waiting(polls, a.spin_limit, a.abort_word)) dead = true;
                }
                wmax = fmax(wmax, word_value(v));
            }
            meeting += 1u;
            wmax = wave_max(wmax);
            __syncthreads();
            if (lane == 0) red[wave] = wmax;
            if (dead) *s_flag = 1;
            __syncthreads();
            for (int q = 0; q < n_waves; ++q) wmax = fmax(wmax, red[q]);
        }
        const double invrho = wmax > 0.0 ? 1.0 / wmax : 0.0;

        auto update = [&](int i, double load) {
            const double ic = invcap[i];
            const double u = load * ic;
            S[i] = S[i] + u;
            const double gn = u * invrho;
            const double t1 = a.eps * gn;
            const double t2 = 1.0 + t1;
            const double ln = len[i] * t2;
            len[i] = ln;
            price[i] = MAXC ? ln : ln * ic;
        };
        for (int it = 0; it < a.iters; ++it) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // (a wave without commodities in this round has nothing to scan)
                if (r * per + (wave * kWave) / L >= n_comm) break;           // wave-uniform
                double best = __builtin_inf();
                int pos = 0;
                uint32_t wb[NW];            // the slot that holds the best candidate so far
                int sb = r * QL;
#pragma unroll
                for (int q = 0; q < QL; ++q) {
                    uint32_t *ws = w[r * QL + q];
                    if constexpr (QT > 1 || !PRODUCT)
#pragma unroll
                        for (int x = 0; x < NW; ++x) keep_in_loop(ws[x]);
                    double m;
                    int at;
                    scan_slot<PRODUCT, MAXC>(ws, m, at);
                    // the strict `<` of a scan in candidate order; a commodity whose candidates
                    // all cost +inf resolves to its first
                    const bool better = q == 0 || m < best;
                    best = better ? m : best;
                    pos = better ? at : pos;
                    sb = better ? r * QL + q : sb;
#pragma unroll
                    for (int x = 0; x < NW; ++x) wb[x] = better ? ws[x] : wb[x];
                }
                const uint32_t meta = meta_of<PRODUCT>(wb);
                bool mine = (meta >> 9) != 0u;
                if constexpr (L > 1) {
                    const int cand = mine ? static_cast<int>(meta & 127u) +
                                                (pos >> ((meta >> 7) & 3u))
                                          : kNone;
                    const int chosen = group_argmin_two_pass<L>(best, cand);   // (all lanes)
                    mine = mine && chosen == cand;
                }
                if (mine) {
                    uint32_t off[5];
                    links_of<PRODUCT>(wb, pos, off);
                    const uint32_t pad = 8u * static_cast<uint32_t>(n_local);
#pragma unroll
                    for (int x = 0; x < 5; ++x)
                        if (off[x] < pad) add_load(l.acc + off[x], l.low + off[x], gr, d[r]);
                    (void)__hip_atomic_fetch_add(tally + (2 * sb + (pos >> 1)) * NT,
                                                 1u << (16 * (pos & 1)), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            __syncthreads();
            if constexpr (MULTI) {
                for (int i = t; i < n_shared; i += NT) publish(take_load(l, i, gr), i);
                for (int i = n_shared + t; i < n_local; i += NT) update(i, take_load(l, i, gr));
                for_shared(update);
                exchange += 1u;
                if (dead) *s_flag = 1;
            } else {
                for (int i = t; i < n_local; i += NT) update(i, take_load(l, i, gr));
            }
            __syncthreads();
            if constexpr (MULTI)
                if (*s_flag != 0) break;                         // workgroup-uniform
        }
        const double T = static_cast<double>(a.iters);
#pragma unroll
        for (int s = 0; s < QT; ++s) {
            const int k = a.comm[static_cast<size_t>(p) * a.n_comm_slots + (s / QL) * per + g];
            const uint32_t meta = meta_of<PRODUCT>(w[s]);
            const int n = static_cast<int>(meta >> 9), shift = static_cast<int>((meta >> 7) & 3u);
            if (k < 0 || n == 0) continue;
            double *out = splits + a.comm_ptr[k] + (meta & 127u);
            const uint32_t c0 = tally[2 * s * NT], c1 = tally[(2 * s + 1) * NT];
            const uint32_t n4[4] = {c0 & 0xFFFFu, c0 >> 16, c1 & 0xFFFFu, c1 >> 16};
#pragma unroll
            for (int pos = 0; pos < 4; ++pos)
                if ((pos & ((1 << shift) - 1)) == 0 && (pos >> shift) < n)
                    out[pos >> shift] = static_cast<double>(n4[pos]) / T;
        }
        double smax = 0.0;
        for (int i = t; i < n_local; i += NT) {
            smax = fmax(smax, S[i]);
            if (a.len_out != nullptr && (loc_link[i] & kPatchExport) && loc_link[i] >= 0)
                a.len_out[loc_link[i] & ~kPatchExport] = len[i];
        }
        smax = wave_max(smax);
        __syncthreads();
        if (lane == 0) red[wave] = smax;
        __syncthreads();
        if (t == 0) {
            for (int q = 0; q < n_waves; ++q) smax = fmax(smax, red[q]);
            double lam = smax / T;
            if constexpr (MULTI) {
                // (the largest of non-negative numbers is the largest of their bit patterns, and
                // a quiet NaN is above them all)
                if (*s_flag != 0) lam = __longlong_as_double(0x7FF8000000000000ll);
                (void)__hip_atomic_fetch_max(
                    reinterpret_cast<unsigned long long *>(a.lambda + plan),
                    static_cast<unsigned long long>(__double_as_longlong(lam)), __ATOMIC_RELAXED,
                    __HIP_MEMORY_SCOPE_AGENT);
            } else {
                a.lambda[plan] = lam;
            }
        }
        if constexpr (MULTI) {
            if (*s_flag != 0) {
                // a team that gave up leaves its other plans undone
                if (t == 0)
                    for (int rest = plan + a.teams; rest < a.plans; rest += a.teams)
                        (void)__hip_atomic_fetch_max(
                            reinterpret_cast<unsigned long long *>(a.lambda + rest),
                            0x7FF8000000000000ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
    }
}

using PatchKernel = void (*)(PatchArgs);

template <bool MAXC, bool MULTI>
PatchKernel kernel_for(const PatchShape &s)
{
#define NIMBLE_PATCH(PR, LL, QQ, RR)                                                           \
    if (s.product == PR && s.lanes == LL && s.quads == QQ && s.rounds == RR)                   \
        return k_patch<PR != 0, LL, QQ, RR, MAXC, MULTI>;
    NIMBLE_PATCH_SHAPES(NIMBLE_PATCH)
#undef NIMBLE_PATCH
    return nullptr;
}

}  // namespace patch

}  // namespace nimble
