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
// kPatchGroup links, so that the parts of a group are contiguous for writer and reader.
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
#pragma once
#include <cstdint>
#include <vector>

namespace nimble {

constexpr int32_t kPatchGroup = 8;
constexpr int32_t kPatchThreads = 1024;
constexpr int32_t kPatchMaxLocal = 2900;      // local links whose state fits the LDS
constexpr int32_t kPatchExport = 1 << 30;     // in loc_link: this patch writes the link's results
constexpr int32_t kPatchDescInts = 8;
constexpr int32_t kPatchCopies = 8;           // of the list of maxima the patches meet over
constexpr int32_t kPatchMeetings = 2 * kPatchCopies + 1;   // words of a patch: those lists, two of
                                              // each, and the XCD it runs on
constexpr int32_t kPatchWordsProduct = 5;
constexpr int32_t kPatchWordsPlain = 11;

struct PatchShape {              // what one kernel instantiation is made for
    int32_t product = 0;         // 1: product slots, 0: plain slots
    int32_t lanes = 0;           // lanes per commodity: 1, 2 or 4
    int32_t quads = 0;           // slots per lane
    int32_t threads = 0;         // workgroup size
};
// The shapes there are kernels for: X(product, lanes, quads).
#define NIMBLE_PATCH_SHAPES(X)                                                                  \
    X(1, 1, 1) X(1, 1, 2) X(1, 1, 3) X(1, 1, 4) X(1, 1, 6) X(1, 1, 8)                           \
    X(1, 2, 1) X(1, 2, 2) X(1, 2, 3) X(1, 2, 4) X(1, 4, 1) X(1, 4, 2)                           \
    X(0, 1, 1) X(0, 1, 2) X(0, 1, 4) X(0, 2, 1) X(0, 2, 2) X(0, 2, 4) X(0, 4, 1) X(0, 4, 2)

struct PatchLayout {
    PatchShape shape;
    int32_t n_patches = 0;       // 0: the fabric does not fit
    int32_t max_comm = 0;        // most commodities of a patch
    int32_t max_local = 0;       // most local links (groups padded) of a patch
    int32_t max_groups = 0;      // most groups of a patch
    int32_t max_users = 0;       // most users of a group
    int32_t max_parts = 0;       // most parts (summed over its groups) of a patch
    int64_t n_parts = 0;         // doubles of one exchange buffer
    std::vector<int32_t> desc;      // [kPatchDescInts * n_patches] first local link, local links,
                                    // links in groups (padded), first group, groups, first
                                    // commodity (in comm), commodities
    std::vector<int32_t> loc_link;  // link id | kPatchExport; -1: padding of a group
    std::vector<int32_t> comm;      // [n_comm] commodities, patch after patch
    std::vector<uint32_t> words;    // [patch][slot][word][thread]
    std::vector<uint32_t> first;    // [patch][slot][thread] bit i: offset i of the slot is the
                                    // commodity's first use of that link (width); offsets in the
                                    // order a0 a2 b0 b2 c d0 d1 e0 e1, or candidate by candidate
    std::vector<int32_t> group;     // [4 * groups] first part, parts (users rounded up to eight),
                                    // own number among the users, users
};

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
};

void scan_patches(int32_t n_links, int32_t n_comm, const int32_t *comm_path_ptr,
                  const int32_t *path_link_ptr, const int32_t *path_links, PatchScan &out);

// The cut of a fabric into a grid of `strips` x `strips` patches (1: one patch).
struct PatchCut {
    int32_t strips = 0;
    int64_t most = 0;                            // most commodities of a patch
    std::vector<std::vector<int32_t>> members;   // commodities of every patch
};
void cut_patches(int32_t n_comm, const PatchScan &scan, int32_t strips, PatchCut &out);

// The shape with `lanes` lanes per commodity (0: whichever is estimated fastest) for patches of
// at most `most` commodities; false when there is none.
bool patch_shape(const PatchScan &scan, int64_t most, int32_t lanes, PatchShape &out);

// What a cut needs, found without building its layout.
struct PatchSizes {
    bool fits = false;              // its patches keep to their limits, LDS among them
    bool fits_adaptive = false;     // also for a solve of variable step (32 bytes a slot, not 8)
    int32_t patches = 0;
    int32_t max_comm = 0, max_local = 0, max_groups = 0, max_parts = 0;      // as in PatchLayout
};
PatchSizes measure_cut(int32_t n_links, const PatchScan &scan, const PatchCut &cut,
                       const PatchShape &shape);

// Estimated times in microseconds of an iteration: the scan, scatter and update of one patch, and
// the same with the exchange between several (its largest numbers of groups and of 64-byte parts).
double patch_scan_us(const PatchShape &s);
double patch_iteration_us(const PatchShape &s, int32_t patches, int32_t groups, int32_t parts);
constexpr double kPatchTripUs = 1.76;     // a trip of a word from patch to patch and the fixed steps

// The grids (strips) with the fewest patches and with the lowest estimate for one plan, of those
// whose patches keep to their limits and are at most `most_patches`; 0: there is none.  The same if
// they have equally many patches.  `adaptive`: the one with the lowest estimate that a solve of
// variable step fits, if neither of these does.
struct PatchChoice {
    int32_t fewest = 0, best = 0, adaptive = 0;
};
PatchChoice choose_cuts(int32_t n_links, int32_t n_comm, const PatchScan &scan, int32_t most_patches,
                        int32_t forced, int32_t lanes);

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
