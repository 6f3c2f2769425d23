// The patch kernels over blocks (host_patch.hpp): the solve of patch_kernel.hpp for several patches --
// same exchange, same arithmetic, same bits -- for fabrics whose commodities share heads and tails.  Per
// iteration
//   fold     a thread per head adds up its two ways to the middle link, a thread per tail fetches the
//            prices of its ways on: LDS to LDS, so that whoever scans them reads 16 bytes at a time;
//   scan     lane j of a block has slot j of L commodities with one tail in registers: one read per
//            commodity and slot, where a commodity that scans its own slots makes nine;
//   choose   the L lanes exchange costs so that lane j ends with the cheapest slot of commodity j:
//            L - 1 exchanges for L commodities, most of them v_permlane swaps of whole half-waves;
//   scatter  lane j finds the candidate within that slot and adds its demand to the loads of its links;
//   update   as in patch_kernel.hpp, but length and congestion of a link in registers of the lane that
//            sums up its parts.
// What bounds it: the exchange (60 % of an iteration of the 64-node fabric), then the LDS in scan and
// scatter (5200 of 16400 cycles, half of them bank conflicts of atomics and of gathers) and vector issue
// (some 200 instructions of a wave outside the exchange, 400 with slots).  Against slots, us per
// iteration: 64 nodes of 8, eight slots a commodity, 7.5 -> 6.9, 32 nodes 4.2 -> 3.8, 24 nodes 4.1 -> 3.7;
// with four slots and fewer, or few commodities in a patch, slots are the faster form (16 nodes 2.7
// against 2.25): the fold is one more trip through the LDS with a barrier behind it.
#pragma once
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

struct __align__(16) Pair {
    double a, b;
};
__device__ __forceinline__ Pair lds_pair(uint32_t off)
{
    return *reinterpret_cast<const Pair *>(s_lds + off);
}

typedef unsigned int Words2 __attribute__((ext_vector_type(2)));

// x and y of lanes 16 (32) apart change places: x becomes what the lower lane had of the lane's own
// value (lower lane: x, upper lane: y), y what the upper one had.
__device__ __forceinline__ void swap16(uint32_t &x, uint32_t &y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}
__device__ __forceinline__ void swap32(uint32_t &x, uint32_t &y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}
template <int BY>
__device__ __forceinline__ void swap_f64(double &x, double &y)
{
    uint32_t xl = static_cast<uint32_t>(__double2loint(x)), xh = static_cast<uint32_t>(__double2hiint(x));
    uint32_t yl = static_cast<uint32_t>(__double2loint(y)), yh = static_cast<uint32_t>(__double2hiint(y));
    if constexpr (BY == 16) {
        swap16(xl, yl);
        swap16(xh, yh);
    } else {
        swap32(xl, yl);
        swap32(xh, yh);
    }
    x = __hiloint2double(static_cast<int>(xh), static_cast<int>(xl));
    y = __hiloint2double(static_cast<int>(yh), static_cast<int>(yl));
}
__device__ __forceinline__ double select(bool c, double a, double b)
{
    return __hiloint2double(select(c, __double2hiint(a), __double2hiint(b)),
                            select(c, __double2loint(a), __double2loint(b)));
}

// The cheapest of L slots for L commodities: v[i] is the cost of this lane's slot for commodity i, `id`
// the lane's word, `low` and `high` those of the lanes of the pair 16 apart.  The lane of commodity i
// (block_thread) ends with its least cost in v[0] and the word of the first slot that has it.
// Costs are compared slot by slot in their order: first neighbours, then pairs of them.
template <int L>
__device__ __forceinline__ uint32_t cheapest(double (&v)[L], uint32_t low, uint32_t high, int lane)
{
    uint32_t id[L / 2];
#pragma unroll
    for (int k = 0; k < L / 2; ++k) {
        swap_f64<16>(v[2 * k], v[2 * k + 1]);
        id[k] = select(v[2 * k + 1] < v[2 * k], high, low);
        v[k] = fast_min_f64(v[2 * k], v[2 * k + 1]);
    }
    if constexpr (L >= 4) {
#pragma unroll
        for (int k = 0; k < L / 4; ++k) {
            swap_f64<32>(v[2 * k], v[2 * k + 1]);
            swap32(id[2 * k], id[2 * k + 1]);
            id[k] = select(v[2 * k + 1] < v[2 * k], id[2 * k + 1], id[2 * k]);
            v[k] = fast_min_f64(v[2 * k], v[2 * k + 1]);
        }
    }
    if constexpr (L >= 8) {
        const bool up = (lane & 8) != 0;
        const double keep = select(up, v[1], v[0]), give = select(up, v[0], v[1]);
        const uint32_t ik = select(up, id[1], id[0]), ig = select(up, id[0], id[1]);
        const double other = dpp_f64<0x128>(give);                     // row_ror:8, lane ^ 8
        const uint32_t io = static_cast<uint32_t>(dpp_i32<0x128>(static_cast<int>(ig)));
        const double lo = select(up, other, keep), hi = select(up, keep, other);
        id[0] = select(hi < lo, select(up, ik, io), select(up, io, ik));
        v[0] = fast_min_f64(lo, hi);
    }
    return id[0];
}

// TWO: some head leads on two ways.  (For several patches only: one patch alone took 2 to 30 % longer than
// with slots, but for 2 nodes with two NICs in reach of a GPU, 1.35 -> 1.27 us per iteration.)
template <bool TWO, int L, bool MAXC>
__global__ __launch_bounds__(kPatchThreads) void k_blocks(PatchArgs a)
{
    constexpr PatchShape kShape = {TWO ? 1 : 0, L, 1, 0, 1};
    const int t = threadIdx.x, NT = blockDim.x;
    const int lane = t & (kWave - 1), n_waves = NT >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int team = blockIdx.x % a.near_xcds + a.near_xcds * (blockIdx.x / a.near_xcds / a.n_patches);
    const int p = blockIdx.x / a.near_xcds % a.n_patches;
    if (team >= a.teams) return;                                           // workgroup-uniform
    const int32_t *dsc = a.desc + kPatchDescInts * p;
    const int n_local = dsc[1], n_shared = dsc[2], n_groups = dsc[4];
    const int n_private = n_local - n_shared, n_comm = dsc[6], n_heads = dsc[9], n_tails = dsc[11];
    const int32_t *comm = a.comm + dsc[5];
    const int32_t *loc_link = a.loc_link + dsc[0];
    const int n_at = a.group[dsc[3] + n_groups];
    constexpr int kSlotBytes = 8;
    const BlockLds l = block_lds(n_local, n_heads, n_tails, n_comm, n_at, kShape, kSlotBytes);
    const uint32_t pad = 8u * static_cast<uint32_t>(n_local);
    double *price = lds_ptr(0), *red = lds_ptr(l.red);
    unsigned long long *load = reinterpret_cast<unsigned long long *>(lds_ptr(l.load));
    unsigned long long *low = reinterpret_cast<unsigned long long *>(lds_ptr(l.low));
    int *s_flag = reinterpret_cast<int *>(red + 39), *s_wide = s_flag + 1;

    // this lane's share of the lists, for the whole solve
    const int j = L == 8 ? (lane >> 4 & 3) | (lane >> 1 & 4) : L == 4 ? lane >> 4 : (lane >> 4) & 1;
    const int block = wave * (kWave / L) +
                      (L == 8 ? lane & 7 : L == 4 ? lane & 15 : (lane & 15) | (lane & 32) >> 1);
    const int c0 = block * L, own = c0 + j;          // commodities of the block, the lane's own
    const bool busy = wave * (kWave / L) * L < n_comm;                     // this wave has some
    const int k_own = own < n_comm ? comm[own] : -1;
    const uint32_t id = a.words[static_cast<size_t>(p) * NT + t];
    constexpr uint32_t kIdMask = (1u << kBlockIdBits) - 1u;
    // words of the lanes of the pair that compares first (slots 2n and 2n + 1)
    uint32_t id_low = id, id_high = id;
    swap16(id_low, id_high);
    const uint32_t *first = a.first + static_cast<size_t>(p) * L * NT + t;
    uint4 my_head = {0u, 0u, 0u, 0u};            // the first head and the first tail this thread folds
    uint2 my_tail = {0u, 0u};
    {
        const uint4 *h = reinterpret_cast<const uint4 *>(a.heads) + static_cast<size_t>(dsc[8]) * L;
        uint4 *to = reinterpret_cast<uint4 *>(s_lds + l.head);
        for (int i = t; i < n_heads * L; i += NT) to[i] = h[i];
        if (t < n_heads * L) my_head = h[t];
        const uint2 *w = reinterpret_cast<const uint2 *>(a.tails) + dsc[10];
        uint2 *tw = reinterpret_cast<uint2 *>(s_lds + l.tail);
        for (int i = t; i < n_tails; i += NT) tw[i] = w[i];
        if (NT - 1 - t < n_tails) my_tail = w[NT - 1 - t];
        for (int i = t; i < n_at; i += NT) reinterpret_cast<uint16_t *>(s_lds + l.at)[i] = a.at[dsc[7] + i];
    }
    const uint32_t my_pairs = l.pair + 16 * block_pair_at(id & kIdMask, L);
    const uint32_t my_ways = l.ways + 16 * block_ways_at((id >> kBlockIdBits) & kIdMask, L, TWO);

    unsigned exchange = 0u;          // exchanges made so far, the same in all patches of a team
    unsigned meeting = 0u;           // maxima folded over all patches so far
    int dead = a.spin_limit == 0u ? 1 : 0;       // this wave has given up waiting
    double *parts_of_team = a.parts + static_cast<size_t>(team) * 2 * a.n_parts;
    double *maxima_of_team = a.maxima + static_cast<size_t>(team) * patch_meeting_words(a.n_patches);
    // (the whole team is on this XCD)
    const bool near = a.near_xcds > 1 && on_one_xcd(maxima_of_team, a, p, 1, red, dead);
    // Shared links: `lanes` lanes add up the parts of a link, the first of them has its state.
    const int lanes = patch_link_lanes(NT, a.row);
    const int per_wave = kWave / lanes, sub = lane / per_wave;
    const int r_link = wave * per_wave + (lane & (per_wave - 1));          // the link whose parts it reads
    const bool reads = wave * per_wave < n_shared;                // this wave reads some
    const int s_link = sub == 0 && r_link < n_shared ? r_link : -1;
    uint32_t users_at = l.at;
    int users = 0;
    if (reads) {
        const int q = r_link < n_shared ? r_link / kPatchGroup : 0, from = a.group[dsc[3] + q];
        users_at = l.at + 2 * from;
        users = a.group[dsc[3] + q + 1] - from;
    }
    const int p_link = t < n_private ? n_shared + t : -1;

    for (int plan = team; plan < a.plans; plan += a.teams) {
        const double *demand = a.demand + static_cast<size_t>(plan) * a.K;
        double *splits = a.splits + static_cast<size_t>(plan) * a.P;
        const double d = k_own >= 0 ? demand[k_own] : 0.0;
        __syncthreads();                 // (the plan before is done with LDS)
        for (int i = t; i < n_local; i += NT) {
            load[i] = 0ull;
            low[i] = 0ull;
        }
        for (int i = t; i < n_comm * L; i += NT) lds_ptr(l.count)[i] = 0.0;
        if (t == 0) {
            price[n_local] = 0.0;
            price[n_local + 1] = __builtin_inf();
            *s_flag = 0;
        }
        // state of the lane's links
        struct State {
            double len, S, invcap;
        } shared = {0.0, 0.0, 0.0}, mine = {0.0, 0.0, 0.0};
        auto start = [&](State &s, int i) {
            if (i < 0) return;
            const int e = loc_link[i];
            s.invcap = e >= 0 ? a.invcap[e & ~kPatchExport] : 0.0;
            s.len = a.len_in && e >= 0 ? a.len_in[e & ~kPatchExport] : 1.0;
            s.S = 0.0;
            price[i] = MAXC ? s.len : s.len * s.invcap;
        };
        start(shared, s_link);
        start(mine, p_link);
        const Grid gr = find_grid(d, red, s_wide, n_waves, wave, lane);
        const Demand units = on_grid(d, gr);
        // the loads of the links if every commodity used all it can reach, once each: their largest
        // part of a capacity is the width rho
        auto reach = [&] {
            const uint2 tw = reinterpret_cast<const uint2 *>(s_lds + l.tail)[(id >> kBlockIdBits) & kIdMask];
#pragma unroll 1
            for (int i = 0; i < L; ++i) {
                // (the lane of commodity i of this block)
                const int src = L == 8 ? (lane & 7) | (i & 1) << 4 | (i & 2) << 4 | (i & 4) << 1
                                       : L == 4 ? (lane & 15) | i << 4 : (lane & 47) | i << 4;
                Demand n;
                n.units = __shfl(units.units, src, kWave);
                n.low = __shfl(units.low, src, kWave);
                const uint32_t once = first[static_cast<size_t>(i) * NT] >> 12;
                const uint4 hw = reinterpret_cast<const uint4 *>(s_lds + l.head)[(id & kIdMask) * L + i];
                uint32_t off[9] = {hw.x & 0xFFFFu, hw.x >> 16, hw.y & 0xFFFFu, hw.y >> 16, hw.z,
                                   tw.x & 0xFFFFu, tw.x >> 16, tw.y & 0xFFFFu, tw.y >> 16};
#pragma unroll
                for (int x = 0; x < 9; ++x)
                    if (!((once >> x) & 1u)) off[x] = pad;
                add_loads<9>(load, low, pad, off, gr, n);
            }
        };
        auto take = [&](int i) { return take_load(load[i], low[i], gr); };
        double invrho = 0.0;

        // Prices that are no numbers (see link_price) become numbers here: in the update, which has the loads
        // of a link's users in registers, that cost 24 nodes 1.3 % and 64 nodes 0.7 %; here nothing measurable.
        auto number = [](double v) {
            return MAXC ? fast_max_f64(v, 0.0) : fast_min_f64(v, __builtin_inf());
        };
        auto fold = [&] {
            auto head = [&](int h, uint32_t x, uint32_t y, uint32_t z) {
                const double mid = lds_f64(z);
                Pair c;
                if constexpr (MAXC) {                // (of the three those that are numbers)
                    c.a = fast_max_f64(fast_max_f64(number(lds_lo(x)), lds_lo(y)), mid);
                    c.b = fast_max_f64(fast_max_f64(number(lds_hi(x)), lds_hi(y)), mid);
                } else {
                    c.a = number(lds_lo(x) + lds_lo(y) + mid);
                    c.b = number(lds_hi(x) + lds_hi(y) + mid);
                }
                *reinterpret_cast<Pair *>(s_lds + l.pair + 16 * (block_pair_at(h / L, L) + h % L)) = c;
            };
            auto tail = [&](int i, uint32_t x, uint32_t y) {
                Pair *to = reinterpret_cast<Pair *>(s_lds + l.ways + 16 * block_ways_at(i, L, TWO));
                to[0] = Pair{number(lds_lo(x)), number(lds_lo(y))};
                if constexpr (TWO) to[1] = Pair{number(lds_hi(x)), number(lds_hi(y))};
            };
            if (t < n_heads * L) head(t, my_head.x, my_head.y, my_head.z);
            // (tails from the last thread on: the first ones have the heads left over)
            if (NT - 1 - t < n_tails) tail(NT - 1 - t, my_tail.x, my_tail.y);
#pragma unroll 1
            for (int h = t + NT; h < n_heads * L; h += NT) {
                const uint4 w = reinterpret_cast<const uint4 *>(s_lds + l.head)[h];
                head(h, w.x, w.y, w.z);
            }
#pragma unroll 1
            for (int i = 2 * NT - 1 - t; i < n_tails; i += NT) {
                const uint2 w = reinterpret_cast<const uint2 *>(s_lds + l.tail)[i];
                tail(i, w.x, w.y);
            }
        };
        // Scan and scatter of an iteration.
        auto pass = [&] {
            double v[L];
            {
                const Pair w0 = lds_pair(my_ways), w1 = TWO ? lds_pair(my_ways + 16) : Pair{0.0, 0.0};
#pragma unroll
                for (int i = 0; i < L; ++i) {
                    // Of the two ways to reach the middle link the cheaper one is the cheaper one
                    // for every way on: rounded additions keep the order.  (Which of equally cheap
                    // candidates comes first is settled below.)
                    const Pair c = lds_pair(my_pairs + 16 * i);
                    const double m = fast_min_f64(c.a, c.b);
                    v[i] = join<MAXC>(join<MAXC>(m, w0.a), w0.b);
                    if constexpr (TWO)
                        v[i] = fast_min_f64(v[i], join<MAXC>(join<MAXC>(m, w1.a), w1.b));
                }
            }
            const uint32_t best_id = cheapest<L>(v, id_low, id_high, lane);
            const double best = v[0];
            // the candidates of the best slot, exactly: the first that costs `best`
            const uint32_t bh = best_id & kIdMask, bt = (best_id >> kBlockIdBits) & kIdMask;
            const Pair c = lds_pair(l.pair + 16 * (block_pair_at(bh, L) + j));
            const uint32_t ways = l.ways + 16 * block_ways_at(bt, L, TWO);
            const uint4 hw = *reinterpret_cast<const uint4 *>(s_lds + l.head + (bh * L + j) * 16u);
            const Pair w0 = lds_pair(ways);
            const uint2 tw = *reinterpret_cast<const uint2 *>(s_lds + l.tail + bt * 8u);
            int pos = select(join<MAXC>(join<MAXC>(c.b, w0.a), w0.b) == best, 2, 3);
            if constexpr (TWO) {
                const Pair w1 = lds_pair(ways + 16);
                pos = select(join<MAXC>(join<MAXC>(c.a, w1.a), w1.b) == best, 1, pos);
            }
            pos = select(join<MAXC>(join<MAXC>(c.a, w0.a), w0.b) == best, 0, pos);
            // (a commodity whose candidates all cost +inf resolves to its first)
            pos = select(best < __builtin_inf(), pos, 0);
            const int hs = (pos & 2) << 3, ls = TWO ? (pos & 1) << 4 : 0;
            const uint32_t off[5] = {(hw.x >> hs) & 0xFFFFu, (hw.y >> hs) & 0xFFFFu, hw.z,
                                     (tw.x >> ls) & 0xFFFFu, (tw.y >> ls) & 0xFFFFu};
            if (k_own >= 0) {
                add_loads<5>(load, low, pad, off, gr, units);
                const int slot = l.count +
                                 kSlotBytes * (own * L + static_cast<int>(best_id >> 2 * kBlockIdBits));
                (void)__hip_atomic_fetch_add(
                    reinterpret_cast<uint32_t *>(lds_ptr(slot + 4 * (pos >> 1))),
                    1u << (16 * (pos & 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        auto update = [&](State &s, int i, double ld) {
            if (i < 0) return;
            const double u = ld * s.invcap;
            s.S = s.S + u;
            const double gn = u * invrho;
            const double t1 = a.eps * gn;
            const double t2 = 1.0 + t1;
            s.len = s.len * t2;
            price[i] = MAXC ? s.len : s.len * s.invcap;
        };

        // (the first round finds the width)
        for (int it = -1; it < a.iters; ++it) {
            if (it >= 0) {
                fold();
                __syncthreads();
                if (busy) pass();                                            // wave-uniform
            } else if (busy) {
                reach();
            }
            __syncthreads();
            double *words = parts_of_team + (exchange & 1u) * a.n_parts;
            const unsigned phase = (exchange >> 1) & 1u;
            if (t < n_shared) put_word(words + p * a.row * kPatchGroup + t, take(t), phase, near);
            const double own_load = p_link >= 0 ? take(p_link) : 0.0;
            if (it >= 0) update(mine, p_link, own_load);
            double all = 0.0;
            if (reads)                                                           // wave-uniform
                all = load_of_link(words, users_at, users, a.max_users, sub, lanes,
                                   r_link & (kPatchGroup - 1), phase, a.spin_limit, a.abort_word, dead);
            exchange += 1u;
            if (it >= 0) update(shared, s_link, all);
            if (it < 0) {
                double wmax = fmax(own_load * mine.invcap, all * shared.invcap);
                wmax = wave_max(wmax);
                __syncthreads();
                if (lane == 0) red[wave] = wmax;
                __syncthreads();
                for (int q = 0; q < n_waves; ++q) wmax = fmax(wmax, red[q]);
                wmax = max_of_team(wmax, maxima_of_team, meeting, a, p, near, red, s_flag, dead,
                                       n_waves, wave, lane);
                invrho = wmax > 0.0 ? 1.0 / wmax : 0.0;
            }
            __syncthreads();
        }
        // (a team that has given up goes through its remaining iterations, in which nobody waits any more:
        // little beside what the one workgroup that solves the plan after it takes)
        if (dead) *s_flag = 1;
        __syncthreads();
        const double T = static_cast<double>(a.iters);
#pragma unroll 1
        for (int i = 0; i < L; ++i) {
            const int k = c0 + i < n_comm ? comm[c0 + i] : -1;
            const uint32_t meta = first[static_cast<size_t>(i) * NT];
            const int n = static_cast<int>((meta >> 9) & 7u);
            if (k < 0 || n == 0) continue;
            const int at = static_cast<int>(meta & 127u), shift = static_cast<int>((meta >> 7) & 3u);
            double *out = splits + a.comm_ptr[k] + at;
            const int slot = l.count + kSlotBytes * ((c0 + i) * L + j);
            const uint2 c = *reinterpret_cast<const uint2 *>(lds_ptr(slot));
            const uint32_t n4[4] = {c.x & 0xFFFFu, c.x >> 16, c.y & 0xFFFFu, c.y >> 16};
#pragma unroll
            for (int pos = 0; pos < 4; ++pos)
                if ((pos & ((1 << shift) - 1)) == 0 && (pos >> shift) < n)
                    out[pos >> shift] = static_cast<double>(n4[pos]) / T;
        }
        double smax = 0.0;
        auto finish = [&](const State &s, int i) {
            if (i < 0) return;
            smax = fmax(smax, s.S);
            const int e = loc_link[i];
            if (a.len_out != nullptr && (e & kPatchExport) && e >= 0)
                a.len_out[e & ~kPatchExport] = s.len;
        };
        finish(shared, s_link);
        finish(mine, p_link);
        smax = wave_max(smax);
        __syncthreads();
        if (lane == 0) red[wave] = smax;
        __syncthreads();
        if (t == 0) {
            for (int q = 0; q < n_waves; ++q) smax = fmax(smax, red[q]);
            report_lambda<true, false>(smax / T, a, plan, s_flag, s_wide);
        }
        if (*s_flag != 0) {
            give_up_rest(a, plan, t);
            break;
        }
    }
}

template <bool MAXC>
PatchKernel block_kernel_for(const PatchShape &s)
{
#define NIMBLE_BLOCK(TT, LL)                                                                   \
    if (s.product == TT && s.lanes == LL) return k_blocks<TT != 0, LL, MAXC>;
    NIMBLE_BLOCK_SHAPES(NIMBLE_BLOCK)
#undef NIMBLE_BLOCK
    return nullptr;
}

}  // namespace patch

}  // namespace nimble
