// Driver for the sanitizer run of the host-side layout code (tests/test_host_sanitizers.py builds
// it with -fsanitize=address,undefined together with csrc/host_topo.cpp and csrc/host_patch.cpp; no
// HIP involved).
// Reads a topology from four binary files in a directory (cap.bin float64, cp.bin / lp.bin /
// pl.bin int32), runs every host-only helper of the library on it and checks the round trips:
// the streaming layout decodes to the plain reverse CSR, every incidence reads back through
// the forward records, and patch layouts of several grids, in slots and in blocks, and those that are
// chosen read back to the CSR, also after a build that ran out of memory.  Exit status 0 and a line "OK ..." on success.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../include/nimble_plan_debug.h"

template <class T>
static std::vector<T> read_all(const std::string &path)
{
    std::vector<T> v;
    FILE *f = std::fopen(path.c_str(), "rb");
    if (!f) {
        std::fprintf(stderr, "cannot open %s\n", path.c_str());
        std::exit(2);
    }
    std::fseek(f, 0, SEEK_END);
    const long n = std::ftell(f);
    std::fseek(f, 0, SEEK_SET);
    v.resize(static_cast<size_t>(n) / sizeof(T));
    if (n > 0 && std::fread(v.data(), 1, static_cast<size_t>(n), f) != static_cast<size_t>(n)) {
        std::fprintf(stderr, "short read on %s\n", path.c_str());
        std::exit(2);
    }
    std::fclose(f);
    return v;
}

int main(int argc, char **argv)
{
    if (argc < 2) return 2;
    const std::string dir = argv[1];
    const std::vector<double> cap = read_all<double>(dir + "/cap.bin");
    const std::vector<int32_t> cp = read_all<int32_t>(dir + "/cp.bin");
    const std::vector<int32_t> lp = read_all<int32_t>(dir + "/lp.bin");
    const std::vector<int32_t> pl = read_all<int32_t>(dir + "/pl.bin");
    const int32_t E = static_cast<int32_t>(cap.size());
    const int32_t K = static_cast<int32_t>(cp.size()) - 1;
    const int32_t P = static_cast<int32_t>(lp.size()) - 1;
    const size_t nnz = pl.size();

    std::vector<int32_t> rp1(E + 1), rc1(nnz + 1), rq1(nnz + 1), rp2(E + 1), rc2(nnz + 1),
        rq2(nnz + 1);
    if (nimble_host_build_reverse(E, K, cp.data(), P, lp.data(), pl.data(), rp1.data(), rc1.data(),
                                  rq1.data()) != NIMBLE_OK)
        return 3;
    if (nimble_host_build_reverse_streaming(E, K, cp.data(), P, lp.data(), pl.data(), rp2.data(),
                                            rc2.data(), rq2.data()) != NIMBLE_OK)
        return 4;
    if (rp1 != rp2 || std::memcmp(rc1.data(), rc2.data(), nnz * 4) != 0 ||
        std::memcmp(rq1.data(), rq2.data(), nnz * 4) != 0) {
        std::fprintf(stderr, "the streaming layout does not decode to the reverse CSR\n");
        return 5;
    }
    std::vector<int32_t> links(nnz + 1, -1), path_rec(static_cast<size_t>(P) + 1, -1);
    int32_t n_rec = -1;
    if (nimble_host_records_roundtrip(E, K, cp.data(), P, lp.data(), pl.data(), links.data(),
                                      path_rec.data(), &n_rec) != NIMBLE_OK)
        return 6;
    if (n_rec > 0 && std::memcmp(links.data(), pl.data(), nnz * 4) != 0) {
        std::fprintf(stderr, "the forward records do not read back the incidences\n");
        return 7;
    }
    int64_t stats[22] = {0};
    if (nimble_host_layout_stats(E, K, cp.data(), P, lp.data(), pl.data(), stats) != NIMBLE_OK)
        return 8;
    int64_t patch[12] = {0};
    const bool with_patches = argc > 2 && std::string(argv[2]) == "patches";
    for (int32_t strips : {1, 2, 3, 5, 8, 16})
        for (int32_t lanes : {0, 1, 4}) {
            if (!with_patches || (lanes != 0 && strips != 3)) continue;
            if (nimble_host_patch_check(E, K, cp.data(), P, lp.data(), pl.data(), strips, lanes,
                                        patch) != NIMBLE_OK ||
                patch[1] != 0) {
                std::fprintf(stderr, "patch layout %d/%d: check %lld\n", strips, lanes,
                             static_cast<long long>(patch[1]));
                return 9;
            }
        }
    const bool large = K > 5000;                 // (a few of these only)
    const int32_t grids[][2] = {{2, 2}, {3, 2}, {1, 5}, {4, 8}, {16, 16}};
    for (const auto &g : grids)
        for (int32_t blocks : {0, 1}) {
            int64_t grid[15] = {0};
            if (!with_patches || (large && g[0] != 4)) continue;
            if (nimble_host_grid_check(E, K, cp.data(), P, lp.data(), pl.data(), g[0], g[1], blocks,
                                       grid) != NIMBLE_OK ||
                grid[1] != 0) {
                std::fprintf(stderr, "grid %d x %d, blocks %d: check %lld\n", g[0], g[1], blocks,
                             static_cast<long long>(grid[1]));
                return 11;
            }
        }
    // what is chosen, with nothing asked for (compute units, XCDs) and with a grid, some of them none
    const int32_t asked[][4] = {{256, 8, 0, 0}, {64, 2, 0, 0}, {20, 1, 0, 0}, {256, 8, 3, 5},
                                {256, 8, 3, 0}, {256, 8, 3, -1}, {256, 8, 1, 300}};
    for (const auto &w : asked)
        for (int32_t blocks : {-1, 1}) {
            int64_t chosen[24] = {0};
            int32_t n = -1;
            if (!with_patches || (large && (w[0] != 256 || w[2] != 0 || blocks == 1))) continue;
            if (nimble_host_patch_choice(E, K, cp.data(), P, lp.data(), pl.data(), w[0], w[1], w[2], w[3], 0,
                                         blocks, chosen, &n) != NIMBLE_OK ||
                n < 0 || n > 3)
                return 12;
            for (int32_t i = 0; i < n; ++i)
                if (chosen[8 * i + 7] != 0 || chosen[8 * i + 2] > w[0]) {
                    std::fprintf(stderr, "choice %d of %d x %d on %d: check %lld\n", i, w[2], w[3], w[0],
                                 static_cast<long long>(chosen[8 * i + 7]));
                    return 13;
                }
        }
    for (int32_t fault : {1, 2, 3, 0})
        for (int32_t what : {0, 1, 2}) {
            if (!with_patches || (large && what == 2)) break;
            int64_t grid[24] = {0};
            int32_t n = 0;
            nimble_debug_fail_patch_build(fault);
            const nimble_status_t st =
                what == 0 ? nimble_host_patch_check(E, K, cp.data(), P, lp.data(), pl.data(), 3, 0, patch)
                : what == 1
                    ? nimble_host_grid_check(E, K, cp.data(), P, lp.data(), pl.data(), 4, 5, 1, grid)
                    : nimble_host_patch_choice(E, K, cp.data(), P, lp.data(), pl.data(), 256, 8, 0, 0, 0, -1,
                                               grid, &n);
            // (few commodities need no worker that could fail)
            if (st != NIMBLE_OK && !(st == NIMBLE_ERR_ALLOC && (fault == 1 || fault == 2))) return 10;
        }
    nimble_debug_fail_patch_build(0);
    std::printf("OK records %d pairs %lld octets %lld pieces %lld blocks %lld bodies %lld groups %lld\n", n_rec,
                static_cast<long long>(stats[0]), static_cast<long long>(stats[1]),
                static_cast<long long>(stats[10]), static_cast<long long>(stats[8]),
                static_cast<long long>(stats[17]), static_cast<long long>(stats[18]));
    return 0;
}
