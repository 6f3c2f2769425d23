// Patch layout: the commodities of a fabric cut into patches, one per workgroup, that keep their
// candidate lists in registers and their links in LDS for a whole solve.  No HIP calls here.
//
// A patch is a set of commodities together with the links their candidates use (its LOCAL
// links).  Commodities are cut by two coordinates -- where their paths leave from (the lowest
// first link of any candidate) and where they arrive (the lowest last link) -- into a grid of
// source strips x destination strips, so that on an all-to-all fabric a patch of S sources and D
// destinations touches the links around S + D endpoints, not S * D.  Links used by one patch only
// are PRIVATE: nobody else ever needs their load or their price.  The others are SHARED: every
// patch that uses one leaves its part of the load in an exchange buffer, reads the parts of the
// other users and applies the length update to its own copy -- same parts, same order, same bits
// in every patch.  Shared links with the same users are bundled into groups of up to
// kPatchGroup links, whose parts lie side by side; all groups of a writer lie side by side, so that
// it writes whole cache lines.
//
// The candidates of a commodity are stored in SLOTS of up to four: byte offsets of local links in
// the price array (16 bits each), padded with the offset of a place that holds +0.0 (adding +0.0
// is exact wherever it happens in the left-to-right sum of a path) and, where a candidate is
// absent, of one that holds +inf.  Two forms, one per layout:
//   product  nine offsets a0 a2 b0 b2 c d0 d1 e0 e1; candidate (h, l) of the slot, h and l from
//            {0, 1}, is the path  a_h b_h c d_l e_l.  Four consecutive candidates of a product
//            rule (egress x ingress of one rail) fill a slot; any two paths that differ in at
//            most two links before a common tail of at most three fill one as (0, 0) and (1, 0);
//            any path of at most five links fits one as (0, 0).
//   plain    four candidates of five offsets each.
// Words of a product slot: a0 | a2 << 16, b0 | b2 << 16, c | meta << 16, d0 | d1 << 16,
// e0 | e1 << 16; of a plain slot: for every candidate p0 | p1 << 16, p2 | p3 << 16, then
// p4 of candidates 0, 1 and 2, 3, then meta << 16.
// meta: bits 0..6 first candidate of the slot, bits 7..8 shift (candidate = first + (2h + l >>
// shift)), bits 9..11 candidates in the slot (0: empty slot).
//
// BLOCKS are another form of the product slots, for fabrics whose commodities share much of them.
// A slot is a HEAD (a0 a2 b0 b2 c: two ways to a middle link) and a TAIL (d0 d1 e0 e1: two ways on).
// A block is L commodities (L: the most slots of a commodity, 2, 4 or 8) that have the same tail in
// every slot -- L sources and one destination -- and takes L lanes: lane j holds slot j of all L
// commodities.  The heads of a lane are L entries side by side (a HEAD BLOCK); blocks of other
// destinations behind the same middle links have the same head blocks, and those are kept once, as
// are equal tails.  A place of a block without a commodity has heads that cost +inf.
#pragma once
#include <cstdint>
#include <vector>

namespace nimble {

constexpr int32_t kPatchGroup = 8;
constexpr int32_t kPatchThreads = 1024;
constexpr int32_t kPatchMaxLocal = 2900;      // local links whose state fits the LDS
constexpr int32_t kPatchMaxUnits = 65536;     // groups' places in an exchange buffer, numbered in 16 bits
constexpr int32_t kPatchExport = 1 << 30;     // in loc_link: this patch writes the link's results
constexpr int32_t kPatchDescInts = 12;
constexpr int32_t kPatchCopies = 8;           // of the list of maxima the patches meet over
constexpr int32_t kPatchMeetings = 2 * kPatchCopies + 1;   // words of a patch: those lists, two of
                                              // each, and the XCD it runs on
// Patches that meet XCD by XCD: XCDs, patches of a team on one at most (patch p runs on XCD p modulo
// kPatchXcds), doubles of a cache line, and words of both lists, two of each.
constexpr int32_t kPatchXcds = 8, kPatchXcdPatches = 32, kPatchLine = 16;
constexpr int32_t kPatchTree = 2 * kPatchXcds * (kPatchXcdPatches + kPatchLine);
constexpr int32_t patch_meeting_words(int32_t patches) { return kPatchMeetings * patches + kPatchTree; }
constexpr int32_t kPatchWordsProduct = 5;
constexpr int32_t kPatchWordsPlain = 11;

// Lane j of block b is thread block_thread(b, j) of the patch: the lanes of a block lie 16 lanes of
// the wave apart (bit 0 of j), 32 (bit 1) and 8 (bit 2), where values change places cheaply.
inline constexpr int32_t block_thread(int32_t b, int32_t j, int32_t lanes)
{
    const int32_t per = 64 / lanes, in = b % per;
    const int32_t lane = lanes == 8 ? in | (j & 1) << 4 | (j & 2) << 4 | (j & 4) << 1
                                    : lanes == 4 ? in | j << 4 : (in & 15) | (in & 16) << 1 | j << 4;
    return b / per * 64 + lane;
}

struct PatchShape {              // what one kernel instantiation is made for
    int32_t product = 0;         // 1: product slots, 0: plain slots
    int32_t lanes = 0;           // lanes per commodity: 1, 2 or 4
    int32_t quads = 0;           // slots per lane
    int32_t threads = 0;         // workgroup size
    int32_t blocks = 0;          // 1: blocks of `lanes` commodities (product: heads lead on two ways,
                                 // quads: 1)
};
// The shapes there are kernels for: X(product, lanes, quads).
#define NIMBLE_PATCH_SHAPES(X)                                                                  \
    X(1, 1, 1) X(1, 1, 2) X(1, 1, 3) X(1, 1, 4) X(1, 1, 6) X(1, 1, 8)                           \
    X(1, 2, 1) X(1, 2, 2) X(1, 2, 3) X(1, 2, 4) X(1, 4, 1) X(1, 4, 2)                           \
    X(0, 1, 1) X(0, 1, 2) X(0, 1, 4) X(0, 2, 1) X(0, 2, 2) X(0, 2, 4) X(0, 4, 1) X(0, 4, 2)
// The same for blocks: X(product, lanes).
#define NIMBLE_BLOCK_SHAPES(X) X(0, 2) X(0, 4) X(0, 8) X(1, 2) X(1, 4) X(1, 8)
// Bits of a lane's word: its head block, its tail, its slot.
constexpr int32_t kBlockIdBits = 11;

constexpr int32_t kPatchLdsBytes = 160 * 1024;    // of a compute unit

// LDS of a patch of blocks, byte offsets.  The prices come first; `pair`: of every head the costs of
// its two ways, 16 bytes; `ways`: of every tail the prices of its ways on, 16 bytes each; `at`: where
// the users of the groups have their words; `count`: `slot_bytes` for every slot of every commodity.
struct BlockLds {
    int32_t load, low, red, pair, head, ways, tail, at, count, bytes;
};
// Where a head block and a tail begin, in units of 16 bytes: what the lanes of a quarter wave read at
// once (head blocks or tails of neighbouring blocks) starts in different banks.
inline constexpr int32_t block_pair_at(int32_t head, int32_t lanes)
{
    return head * (lanes == 8 ? 10 : lanes) + head / lanes;
}
inline constexpr int32_t block_ways_at(int32_t tail, int32_t lanes, bool two)
{
    return tail * (two ? 2 : 1) + tail / lanes;
}
inline constexpr BlockLds block_lds(int32_t n_local, int32_t n_heads, int32_t n_tails,
                                    int32_t n_comm, int32_t n_at, const PatchShape &s,
                                    int32_t slot_bytes)
{
    BlockLds l = {};
    int32_t o = 8 * (n_local + 2);                // [n_local] +0.0, [n_local + 1] +inf
    l.load = o;   o += 8 * n_local;
    l.low = o;    o += 8 * n_local;
    l.red = o;    o += 8 * 40;
    o = (o + 15) & ~15;
    l.pair = o;   o += 16 * block_pair_at(n_heads, s.lanes);
    l.head = o;   o += 16 * s.lanes * n_heads;
    l.ways = o;   o += 16 * block_ways_at(n_tails, s.lanes, s.product != 0);
    l.tail = o;   o += 8 * n_tails;
    l.at = o;     o += (2 * n_at + 7) & ~7;
    l.count = o;  o += slot_bytes * n_comm * s.lanes;
    l.bytes = o;
    return l;
}

struct PatchLayout {
    PatchShape shape;
    int32_t n_patches = 0;       // 0: the fabric does not fit
    int32_t max_comm = 0;        // most commodities of a patch
    int32_t max_local = 0;       // most local links (groups padded) of a patch
    int32_t max_groups = 0;      // most groups of a patch
    int32_t max_users = 0;       // most users of a group
    int32_t max_at = 0;          // most users (summed over its groups) of a patch
    int32_t max_heads = 0;       // blocks: most head blocks of a patch
    int32_t max_tails = 0;       // blocks: most tails of a patch
    int64_t n_parts = 0;         // words of one exchange buffer
    std::vector<int32_t> desc;      // [kPatchDescInts * n_patches] first local link, local links,
                                    // links in groups (padded), first group, groups, first
                                    // commodity (in comm), commodities, first user; blocks: first head block,
                                    // head blocks, first tail, tails
    std::vector<int32_t> loc_link;  // link id | kPatchExport; -1: padding of a group
    std::vector<int32_t> comm;      // [n_comm] commodities, patch after patch; blocks: -1 for places
                                    // without one, a multiple of `lanes` in every patch
    std::vector<uint32_t> words;    // [patch][slot][word][thread]
    std::vector<uint32_t> first;    // [patch][slot][thread] bit i: offset i of the slot is the
                                    // commodity's first use of that link (width); offsets in the
                                    // order a0 a2 b0 b2 c d0 d1 e0 e1, or candidate by candidate
    // Blocks: `words` [patch][thread] is the lane's word (kBlockIdBits), `first` [patch][commodity of
    // the block][thread] the slot's meta | first-use bits << 12.
    std::vector<uint32_t> heads;    // [head block][lanes][4] words a0 | a2 << 16, b0 | b2 << 16, c, 0
    std::vector<uint32_t> tails;    // [tail][2] words d0 | d1 << 16, e0 | e1 << 16
    std::vector<int32_t> group;     // [groups] start of its users in `at`
    // Users of the groups of a patch, group after group: where the group's words lie in the exchange
    // buffer, in units of kPatchGroup words.  The words of patch b are `row` of them from b * row on,
    // its groups in their local order.  A patch's run of `at` starts at desc[7]; its run of `group` has one
    // entry more than groups, so that group q has the users from group[q] to group[q + 1].
    std::vector<uint16_t> at;
    int32_t row = 0;                // of units per patch
};
// (an even number of units: rows begin with a cache line)
constexpr int32_t patch_row(int32_t max_groups) { return (max_groups + 1) / 2 * 2; }

// What a fabric's commodities need, found once and used for every grid that is tried.
struct PatchScan {
    bool fits = false;              // paths and candidate lists suit the slots
    int32_t product = 0;            // 1: product slots, 0: plain slots
    int32_t slots = 0;              // most slots of a commodity
    // links of commodity k, each once: links[k / kBlock] from link_ptr[k] to link_ptr[k + 1] or
    // the end of that block
    static constexpr int32_t kBlock = 1024;
    std::vector<std::vector<int32_t>> links;
    std::vector<int32_t> link_ptr;
    std::vector<int32_t> x, y;      // [n_comm] rank of the commodity's coordinates
    std::vector<int32_t> x_cross, y_cross;   // links a cut after rank r would divide
    std::vector<int64_t> x_count, y_count;   // commodities up to and including rank r
    // Blocks (block_lanes 0: the fabric has none): a number for the links of every slot's head and
    // tail, [n_comm * block_lanes], 0 where there is no slot.
    int32_t block_lanes = 0;
    int32_t block_product = 0;      // 1: some head leads on two ways
    std::vector<uint64_t> head, tail;
    std::vector<int8_t> place;      // place of a link in the paths of five links: 0..4, -1 none, -2
                                    // several
};

// The commodities of a patch as blocks.
struct PatchBlocks {
    std::vector<int32_t> comm;              // [blocks * lanes] or -1
    std::vector<int32_t> head, tail;        // [blocks * lanes] number of the lane's head block and tail
    std::vector<int32_t> head_at, tail_at;  // block * lanes + lane that had the number first
};
void find_blocks(const PatchScan &scan, const std::vector<int32_t> &members, PatchBlocks &out);

void scan_patches(int32_t n_links, int32_t n_comm, const int32_t *comm_path_ptr,
                  const int32_t *path_link_ptr, const int32_t *path_links, PatchScan &out);

// The cut of a fabric into a grid of `x` x `y` patches (1 x 1: one patch).
struct PatchGrid {
    int32_t x = 0, y = 0;
    bool operator==(const PatchGrid &o) const { return x == o.x && y == o.y; }
};
struct PatchCut {
    int64_t most = 0;                            // most commodities of a patch
    std::vector<std::vector<int32_t>> members;   // commodities of every patch
};
void cut_patches(int32_t n_comm, const PatchScan &scan, PatchGrid grid, PatchCut &out);

// The shape with `lanes` lanes per commodity (0: whichever is estimated fastest) for patches of
// at most `most` commodities; false when there is none.
bool patch_shape(const PatchScan &scan, int64_t most, int32_t lanes, PatchShape &out);

// What a cut needs, found without building its layout.
struct PatchSizes {
    bool fits = false;              // its patches keep to their limits, LDS among them
    bool fits_adaptive = false;     // also for a solve of variable step (32 bytes a slot, not 8)
    int32_t patches = 0;
    int32_t max_comm = 0, max_local = 0, max_groups = 0;      // as in PatchLayout
    int32_t max_heads = 0, max_tails = 0, max_at = 0;
    int32_t max_private = 0;        // most links of a patch that no other patch uses
    int32_t max_users = 0;          // most patches that share a link
};
PatchSizes measure_cut(int32_t n_links, const PatchScan &scan, const PatchCut &cut,
                       const PatchShape &shape);
// The same cut as blocks: takes the sizes of its links from `m`, sets the others and the shape.
// False: its blocks do not suit the kernels.
bool measure_blocks(const PatchScan &scan, const PatchCut &cut, PatchSizes &m, PatchShape &shape);

// Estimated times in microseconds of an iteration: the scan, scatter and update of one patch, and
// the same with the exchange between several.
// (`near`: a team within one XCD).
double patch_scan_us(const PatchShape &s);
double patch_iteration_us(const PatchShape &s, const PatchSizes &m, bool near);
constexpr double kPatchTripUs = 1.3;      // no iteration of several patches is shorter
// Teams of patches that are resident at once, a patch per compute unit.
struct PatchTeams {
    int32_t spread = 0;          // each over all XCDs
    int32_t near = 0;            // each within one (0: they do not fit one)
};
constexpr PatchTeams patch_teams(int32_t patches, int32_t cus, int32_t xcds)
{
    return PatchTeams{cus / patches, xcds * (cus / xcds / patches)};
}
// Teams keep to one XCD where they fit one and `plans` plans take no more rounds that way: an iteration is
// 4 to 25 % shorter then, and a round more costs more than that (teams of 12, 20, 28 and 30 patches, 1 to 32
// plans: 20 patches of 10 nodes, 12 plans in one round of spread teams 1071 us, in two of near ones 1687;
// 32 plans in three and four 3073 and 3339; 16 plans, two rounds either way, 2027 and 1703).
constexpr bool teams_keep_near(const PatchTeams &t, int32_t plans)
{
    return t.near > 0 && (plans + t.near - 1) / t.near <= (plans + t.spread - 1) / t.spread;
}
// Microseconds of an iteration of `plans` plans, from those of one of a near and of a spread team.
constexpr double plans_iteration_us(const PatchTeams &t, int32_t plans, double near_us, double spread_us)
{
    return (teams_keep_near(t, plans) ? near_us : spread_us) * ((plans + t.spread - 1) / t.spread);
}
// What a step of variable size takes longer than one of fixed size: 0.9 us with one patch (2 nodes: 1.8
// against 0.9), 3.2 with several (16 nodes: 5.3 against 2.2).
constexpr double kVariableOneUs = 0.9, kVariableMoreUs = 3.2;
constexpr double variable_step_us(int32_t patches, double us)
{
    return us + (patches > 1 ? kVariableMoreUs : kVariableOneUs);
}
// Lanes that add up the parts of a shared link: as many as there are threads for.
constexpr int32_t patch_link_lanes(int32_t threads, int32_t row)
{
    return threads >= 4 * kPatchGroup * row ? 4 : threads >= 2 * kPatchGroup * row ? 2 : 1;
}

// What switches ask for (0, -1: nothing).
struct PatchForced {
    PatchGrid grid;
    int32_t lanes = 0, blocks = -1;
};

// A cut worth building.
struct PatchOption {
    PatchGrid grid;
    PatchShape shape;
    PatchSizes sizes;
    double us = 0.0;             // estimate of an iteration of one plan
    double spread_us = 0.0;      // the same with its patches spread over the XCDs
    bool variable_only = false;  // made for solves of variable step alone
};

// The cut that solves the most plans in a time (by the estimates, `cus` compute units in `xcds`
// XCDs) and the one with the lowest estimate for one plan, of those whose patches keep to their limits;
// one of the two if they are the same.  If neither has the lowest estimate of a variable step of those
// that fit one (layouts of blocks have no such kernels), that one as well.
std::vector<PatchOption> choose_cuts(int32_t n_links, int32_t n_comm, const PatchScan &scan,
                                     int32_t cus, int32_t xcds, const PatchForced &forced);

// The layout of a cut.  Returns false, with out.n_patches = 0, when a patch exceeds its limits.
bool build_patches(int32_t n_links, int32_t n_comm, const int32_t *comm_path_ptr,
                   const int32_t *path_link_ptr, const int32_t *path_links,
                   const PatchScan &scan, PatchCut &cut, const PatchShape &shape,
                   PatchLayout &out);

// Reads every commodity's candidates back from the slots and checks them, the exchange groups and
// the first-use bits against the CSR; 0 when all agree, else the number of the failed check.
int check_patches(int32_t n_links, int32_t n_comm, const int32_t *comm_path_ptr,
                  const int32_t *path_link_ptr, const int32_t *path_links,
                  const PatchLayout &layout);

}  // namespace nimble
