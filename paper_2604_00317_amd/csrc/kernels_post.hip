// Plan post-processing: split fractions -> bytes per candidate path in whole chunks.
//
// The dataplane consumes, per pair, a list of paths with a byte amount each (the Paths / Flows
// lists of Algorithm 1); messages must not be fragmented below the chunk granularity and small
// messages stay off the multi-hop paths (Sec. V-A switches forwarding off for messages of 1 MB
// or less).  A pair at or below the threshold keeps everything on its first candidate;
// otherwise its N = floor(d / chi) whole chunks are apportioned to the candidates by largest
// remainder (quota floor(N * c_j / T), the left-over chunks to the largest remainders
// N * c_j mod T, ties to the lower index) and the residual d - N * chi joins the candidate with
// the largest count.  Chunk numbers are exact 64-bit integers.  Two kernels compute the same
// numbers: a group of L lanes per pair, one candidate per lane (pairs of up to 64 candidates:
// coalesced reads and writes, one quotient per candidate, ranks by rotating the remainders
// round the group), and one thread per pair for anything wider.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "wave_ops.hpp"

namespace nimble {

namespace {

constexpr int kPostBlock = 256;
constexpr int kPairsAtOnce = 4;          // of a group of lanes, where there are many pairs

__global__ __launch_bounds__(kPostBlock) void k_quantize(int K, const int32_t *__restrict__ cp,
                                                         const double *__restrict__ demand,
                                                         const double *__restrict__ splits,
                                                         int iters, long long chi, double theta,
                                                         double *__restrict__ flows)
{
    const int k = blockIdx.x * kPostBlock + threadIdx.x;
    if (k >= K) return;
    const int a = cp[k], n = cp[k + 1] - a;
    if (n == 0) return;
    const double dk = demand[k];
    if (dk <= theta) {                                   // small message: first candidate only
        flows[a] = dk;
        for (int j = 1; j < n; ++j) flows[a + j] = 0.0;
        return;
    }
    const double T = static_cast<double>(iters);
    const double chi_d = static_cast<double>(chi);
    const double whole = floor(dk / chi_d);
    if (!(whole < 2147483648.0)) {                       // N * c_j would leave 64 bits
        for (int j = 0; j < n; ++j) flows[a + j] = __builtin_nan("");
        return;
    }
    const long long N = static_cast<long long>(whole);
    const double res = dk - static_cast<double>(N * chi);
    long long sum_q = 0, c_max = -1;
    int j_max = 0;
    for (int j = 0; j < n; ++j) {
        const long long c = llrint(splits[a + j] * T);
        sum_q += (N * c) / iters;
        if (c > c_max) {
            c_max = c;
            j_max = j;
        }
    }
    const long long R = N - sum_q;                       // chunks left over, fewer than n
    for (int j = 0; j < n; ++j) {
        const long long c = llrint(splits[a + j] * T);
        const long long q = (N * c) / iters;
        const long long rem = (N * c) % iters;
        long long rank = 0;                              // candidates ahead of j for a left-over
        for (int i = 0; i < n; ++i) {
            const long long ci = llrint(splits[a + i] * T);
            const long long ri = (N * ci) % iters;
            rank += (ri > rem || (ri == rem && i < j)) ? 1 : 0;
        }
        double f = static_cast<double>(chi * (q + (rank < R ? 1 : 0)));
        if (j == j_max) f = f + res;
        flows[a + j] = f;
    }
}

// The values of v in both rows of a pair of rows (of both halves of the wave): own and other, in an
// order that is the same in all of them.  One vector instruction, where a shuffle goes through the LDS.
struct TwoI32 {
    int a, b;
};
__device__ __forceinline__ TwoI32 both_rows(int v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return {static_cast<int>(r[0]), static_cast<int>(r[1])};
}
__device__ __forceinline__ TwoI32 both_halves(int v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return {static_cast<int>(r[0]), static_cast<int>(r[1])};
}

template <int L>
__device__ __forceinline__ int group_sum_i32(int v)
{
    if constexpr (L > 1) v += partner_i32<1>(v);
    if constexpr (L > 2) v += partner_i32<2>(v);
    if constexpr (L > 4) v += partner_i32<4>(v);
    if constexpr (L > 8) v += partner_i32<8>(v);
    if constexpr (L > 16) {
        const TwoI32 r = both_rows(v);
        v = r.a + r.b;
    }
    if constexpr (L > 32) {
        const TwoI32 h = both_halves(v);
        v = h.a + h.b;
    }
    return v;
}

template <int L>
__device__ __forceinline__ int group_max_i32(int v)
{
    if constexpr (L > 1) v = max(v, partner_i32<1>(v));
    if constexpr (L > 2) v = max(v, partner_i32<2>(v));
    if constexpr (L > 4) v = max(v, partner_i32<4>(v));
    if constexpr (L > 8) v = max(v, partner_i32<8>(v));
    if constexpr (L > 16) {
        const TwoI32 r = both_rows(v);
        v = max(r.a, r.b);
    }
    if constexpr (L > 32) {
        const TwoI32 h = both_halves(v);
        v = max(h.a, h.b);
    }
    return v;
}

// One comparison of the rank count.  Every candidate carries a key that orders the claims on
// the left-over chunks: the remainder in the high bits and 63 - lane below, so a larger key is
// a larger remainder, or the same remainder at a lower index (lanes of a group are in index
// order).  Groups narrower than a DPP row also see keys of their neighbours in the row, which
// do not count.
template <int L>
__device__ __forceinline__ void rank_one(long long ko, int il, long long key, int lane, int &rank)
{
    bool ahead = ko > key;
    if constexpr (L < 16) ahead = ahead && (((il ^ lane) & ~(L - 1)) == 0);
    rank += ahead ? 1 : 0;
}
template <int L>
__device__ __forceinline__ void rank_one(int ko, int il, int key, int lane, int &rank)
{
    bool ahead = ko > key;
    if constexpr (L < 16) ahead = ahead && (((il ^ lane) & ~(L - 1)) == 0);
    rank += ahead ? 1 : 0;
}

template <int CTRL>
__device__ __forceinline__ long long dpp_key(long long v)
{
    const int lo = dpp_i32<CTRL>(static_cast<int>(v));
    const int hi = dpp_i32<CTRL>(static_cast<int>(v >> 32));
    return (static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo);
}
template <int CTRL>
__device__ __forceinline__ int dpp_key(int v)
{
    return dpp_i32<CTRL>(v);
}

// The same against the keys of a 16-lane row rotated by 1..S lanes (DPP row_ror: lane p of a
// row receives from lane (p - S) mod 16 of the same row).
template <int L, int S>
struct RankRow {
    template <typename KEY>
    static __device__ __forceinline__ void add(KEY v, int row_lane0, KEY key, int lane, int &rank)
    {
        RankRow<L, S - 1>::add(v, row_lane0, key, lane, rank);
        const int il = row_lane0 | ((lane - S) & 15);
        rank_one<L>(dpp_key<0x120 + S>(v), il, key, lane, rank);
    }
};
template <int L>
struct RankRow<L, 0> {
    template <typename KEY>
    static __device__ __forceinline__ void add(KEY, int, KEY, int, int &) {}
};

template <int L, typename KEY>
__device__ __forceinline__ int group_rank(KEY key, int lane)
{
    int rank = 0;
    RankRow<L, 15>::add(key, lane & ~15, key, lane, rank);
    if constexpr (L > 16) {
        const KEY k1 = __shfl_xor(key, 16, kWave);
        rank_one<L>(k1, lane ^ 16, key, lane, rank);
        RankRow<L, 15>::add(k1, (lane ^ 16) & ~15, key, lane, rank);
    }
    if constexpr (L > 32) {
        const KEY k2 = __shfl_xor(key, 32, kWave);
        rank_one<L>(k2, lane ^ 32, key, lane, rank);
        RankRow<L, 15>::add(k2, (lane ^ 32) & ~15, key, lane, rank);
        const KEY k3 = __shfl_xor(key, 48, kWave);
        rank_one<L>(k3, lane ^ 48, key, lane, rank);
        RankRow<L, 15>::add(k3, (lane ^ 48) & ~15, key, lane, rank);
    }
    return rank;
}

// The rank counted as above, for 32-bit keys of groups that fill whole DPP rows, without a
// carry from one comparison to the next.  Keys lie in [-1, 2^30) and those of candidates differ, so the
// sign of ko - key says whether ko is behind, and all but the own one are ahead or behind; the
// signs are shifted into a word (32 comparisons at most per word) and counted at the end.
template <int S>
__device__ __forceinline__ void collect_signs(int v, int key, unsigned &signs)
{
    signs = __builtin_amdgcn_alignbit(signs, static_cast<unsigned>(dpp_less_i32<0x120 + S>(v, key)), 31);
    if constexpr (S > 1) collect_signs<S - 1>(v, key, signs);
}
// how many of the sixteen lanes of a row are behind
__device__ __forceinline__ int row_behind(int v, int key)
{
    unsigned signs = static_cast<unsigned>(v - key) >> 31;
    collect_signs<15>(v, key, signs);
    return __popc(signs);
}
template <int L>
__device__ __forceinline__ int group_rank_narrow(int key)
{
    if constexpr (L <= 16) return L - 1 - row_behind(key, key);   // (nobody is behind oneself)
    const TwoI32 r = both_rows(key);
    if constexpr (L <= 32) return L - 1 - row_behind(r.a, key) - row_behind(r.b, key);
    const TwoI32 a = both_halves(r.a), b = both_halves(r.b);
    return L - 1 - row_behind(a.a, key) - row_behind(a.b, key) - row_behind(b.a, key) -
           row_behind(b.b, key);
}

// L lanes per pair (L a power of two, every pair has at most L candidates); the lanes of a
// group take the same branches, so the cross-lane steps are reached by whole groups.
// The two trips to memory a wave makes one after the other (list, then fractions) bound one pair at a
// time: a group takes U pairs, whose lists and fractions are asked for together, and with four of them
// vector issue does (88 % of the cycles where everything comes from the cache).  NARROW (iters < 2^24)
// keeps all whole numbers but the flows in 32 bits: remainders are below iters, so the low halves of
// N * c and q * iters give them, and the product with 1 / iters is as good for the quotient as the
// division.  Measured on 261 632
// pairs of 32 candidates: 59.0 us with 64-bit whole numbers throughout, 49.6 us (2.8 TB/s) in 32 bits,
// 52.0 us with a third fewer instructions (reciprocals passed in, subtractions in the moves across
// lanes), 43.7 us with those and two pairs at a time, 36.2 us (3.8 TB/s) with four whose fractions are
// asked for together too.  These are calls that find their 136 MB in the cache: from memory 59.7 us
// before and 41.6 now.
template <int L, bool NARROW, int U>
__global__ __launch_bounds__(kPostBlock) void k_quantize_group(int K,
                                                               const int32_t *__restrict__ cp,
                                                               const double *__restrict__ demand,
                                                               const double *__restrict__ splits,
                                                               int iters, double inv_iters,
                                                               long long chi, int chi_is_pow2,
                                                               double inv_chi, double theta,
                                                               double *__restrict__ flows)
{
    const int j = static_cast<int>(threadIdx.x % L);
    const int lane = threadIdx.x & (kWave - 1);
    // the lists of all pairs are asked for together, then their fractions
    int at[U], count[U];
    double demand_of[U], split_of[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long kk = (static_cast<long long>(blockIdx.x) * U + u) * (kPostBlock / L) +
                             threadIdx.x / L;
        const int k = kk < K ? static_cast<int>(kk) : K - 1;
        at[u] = cp[k];
        count[u] = kk < K ? cp[k + 1] : 0;
        demand_of[u] = demand[k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        count[u] -= at[u];                               // (not positive: no pair)
        split_of[u] = splits[at[u] + (j < count[u] ? j : 0)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int a = at[u];
        const double dk = demand_of[u], split = split_of[u];
        const bool mine = j < count[u];
        const double chi_d = static_cast<double>(chi);
        // (a product with an exact reciprocal rounds like the quotient)
        const double whole = floor(chi_is_pow2 ? dk * inv_chi : dk / chi_d);
        const bool small = dk <= theta;
        const bool wide = !(whole < 2147483648.0);           // N * c_j would leave 64 bits
        const double Nd = (small || wide) ? 0.0 : whole;
        const double res = dk - Nd * chi_d;                  // (chi <= 2^40: the product is N * chi)
        int c = -1, q = 0, rem = -1;                         // absent candidates rank behind all
        if (mine) {
            const double T = static_cast<double>(iters);
            // floor(N * c / T): the quotient is below 2^31, so the quotient in double (N * c / T, or
            // N * c times 1 / T, three roundings of 2^-53 each) is within one of it and one exact
            // correction step either way settles it
            if constexpr (NARROW) {
                const double cd = rint(split * T);
                c = static_cast<int>(cd);
                q = static_cast<int>((Nd * cd) * inv_iters);
                rem = static_cast<int>(static_cast<unsigned>(static_cast<int>(Nd)) *
                                           static_cast<unsigned>(c) -
                                       static_cast<unsigned>(q) * static_cast<unsigned>(iters));
                const int low = rem < 0 ? 1 : 0, high = rem >= iters ? 1 : 0;
                q += high - low;
                rem += low ? iters : high ? -iters : 0;
            } else {
                const long long N = static_cast<long long>(Nd);
                const long long cl = llrint(split * T);
                const long long nc = N * cl;
                long long ql = static_cast<long long>(static_cast<double>(nc) / T);
                long long r = nc - ql * iters;
                if (r < 0) {
                    ql -= 1;
                    r += iters;
                } else if (r >= iters) {
                    ql += 1;
                    r -= iters;
                }
                c = static_cast<int>(cl);                    // c <= iters < 2^31
                q = static_cast<int>(ql);
                rem = static_cast<int>(r);
            }
        }
        // left-over chunks of the pair: fewer than n (every quota is below 2^31, and so is the sum)
        const int R = static_cast<int>(Nd) - group_sum_i32<L>(q);
        // the candidate with the largest count, the lowest index among equals; then the candidates
        // ahead of j for a left-over chunk
        bool most;
        int rank;
        if constexpr (NARROW) {
            const int claim = mine ? ((c << 6) | (63 - lane)) : -1;
            most = group_max_i32<L>(claim) == claim;
            const int key = mine ? ((rem << 6) | (63 - lane)) : -1;
            if constexpr (L >= 16) rank = group_rank_narrow<L>(key);
            else rank = group_rank<L, int>(key, lane);
            // (wanted by some lanes only, but moved to where they alone are active the subtractions
            // part from the moves across lanes, which have to stay here: an instruction more for each)
            asm volatile("" : "+v"(rank));
        } else {
            const int c_max = group_max_i32<L>(c);
            int j_max = (c == c_max) ? j : 0x7FFFFFFF;
            if constexpr (L > 1) j_max = min(j_max, partner_i32<1>(j_max));
            if constexpr (L > 2) j_max = min(j_max, partner_i32<2>(j_max));
            if constexpr (L > 4) j_max = min(j_max, partner_i32<4>(j_max));
            if constexpr (L > 8) j_max = min(j_max, partner_i32<8>(j_max));
            if constexpr (L > 16) j_max = min(j_max, partner_i32<16>(j_max));
            if constexpr (L > 32) j_max = min(j_max, partner_i32<32>(j_max));
            most = j == j_max;
            const long long key = mine ? ((static_cast<long long>(rem) << 6) | (63 - lane)) : -1;
            rank = group_rank<L, long long>(key, lane);
        }
        if (!mine) continue;
        double f;
        if (small) f = (j == 0) ? dk : 0.0;                  // small message: first candidate only
        else if (wide) f = __builtin_nan("");
        else {
            // (the product of two whole numbers that doubles hold is rounded once, like the conversion
            // of the exact product)
            f = chi_d * static_cast<double>(q + (rank < R ? 1 : 0));
            if (most) f = f + res;
        }
        flows[a + j] = f;
    }
}

}  // namespace

hipError_t launch_quantize(const DeviceTopo &t, const double *demand, const double *splits,
                           int32_t iters, int64_t chi, double theta, double *flows,
                           hipStream_t s)
{
    if (t.pmax <= kWave) {
        const int L = lanes_per_commodity(t.pmax);
        const int64_t threads = static_cast<int64_t>(t.K) * L;
        // (Four pairs at a time pay where that many lanes are more than the chip's 256 compute units
        // hold anyway, 2048 each.  One pair against four, buffers from memory, 8 lanes a pair: 2^19
        // lanes 7.8 and 8.4 us, 2^20 11.6 and 10.9, 2^21 18.5 and 14.9, 2^23 61 and 39; 64 lanes: 9.1
        // and 10.1, 13.9 and 14.0, 22.2 and 20.3, 74 and 56.  Widths between them cross there too.)
        const bool many = iters < (1 << 24) && threads >= (1 << 20);
        const int64_t per_block = many ? kPostBlock * kPairsAtOnce : kPostBlock;
        const int g = static_cast<int>((threads + per_block - 1) / per_block);
        const double inv_iters = 1.0 / static_cast<double>(iters);
        const double inv_chi = 1.0 / static_cast<double>(chi);
        const int chi_is_pow2 = (chi & (chi - 1)) == 0 ? 1 : 0;
#define NIMBLE_QUANT_ARGS                                                                      \
    dim3(g), dim3(kPostBlock), 0, s, t.K, t.comm_ptr, demand, splits, iters, inv_iters,        \
        static_cast<long long>(chi), chi_is_pow2, inv_chi, theta, flows
#define NIMBLE_QUANT_LAUNCH(LL)                                                                \
    case LL:                                                                                   \
        if (many) hipLaunchKernelGGL((k_quantize_group<LL, true, kPairsAtOnce>), NIMBLE_QUANT_ARGS); \
        else if (iters < (1 << 24))   /* counts and remainders above a 6-bit index fit 30 bits */ \
            hipLaunchKernelGGL((k_quantize_group<LL, true, 1>), NIMBLE_QUANT_ARGS);            \
        else hipLaunchKernelGGL((k_quantize_group<LL, false, 1>), NIMBLE_QUANT_ARGS);          \
        return hipGetLastError();
        switch (L) {
            NIMBLE_QUANT_LAUNCH(1)
            NIMBLE_QUANT_LAUNCH(2)
            NIMBLE_QUANT_LAUNCH(4)
            NIMBLE_QUANT_LAUNCH(8)
            NIMBLE_QUANT_LAUNCH(16)
            NIMBLE_QUANT_LAUNCH(32)
            NIMBLE_QUANT_LAUNCH(64)
        }
#undef NIMBLE_QUANT_LAUNCH
#undef NIMBLE_QUANT_ARGS
    }
    const int grid = (t.K + kPostBlock - 1) / kPostBlock;
    hipLaunchKernelGGL(k_quantize, dim3(grid), dim3(kPostBlock), 0, s, t.K, t.comm_ptr, demand,
                       splits, iters, static_cast<long long>(chi), theta, flows);
    return hipGetLastError();
}

}  // namespace nimble
