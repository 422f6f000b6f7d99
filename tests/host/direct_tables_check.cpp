// Host check of the edge lists of the two-launch CG iteration
// (build_direct_tables): the copies listed for every shared edge or corner
// node, summed in the update's order, must give bitwise the ascending-order
// sum of all copies of its global point (pairs only where the table-free
// gather applies; Dirichlet nodes are masked).
//
// usage: direct_tables_check E N glob_id.bin dirichlet.bin seed
// Prints "direct=<0|1> checked=<slots> generic=<slots listed in egen>" and
// exits 0, or names the first failing point and exits 1.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../paper_2108_12188_amd/csrc/sem_vec_body.h"

namespace sem {
void set_error(const std::string &) {}
[[noreturn]] void fail(sem_status code, const std::string &msg) {
    throw std::runtime_error("status " + std::to_string((int)code) + ": " + msg);
}
void check_hip(hipError_t, const char *) {}
}  // namespace sem

template <typename T>
static std::vector<T> read_all(const char *path, size_t count) {
    std::vector<T> v(count);
    FILE *f = std::fopen(path, "rb");
    if (!f || std::fread(v.data(), sizeof(T), count, f) != count) std::exit(2);
    std::fclose(f);
    return v;
}

int main(int argc, char **argv) {
    if (argc != 6) return 2;
    const int64_t E = std::atoll(argv[1]);
    const int N = std::atoi(argv[2]), P = N + 1, P3 = P * P * P, MS = sem::edge_slots(N);
    const int64_t n = E * P3;
    const std::vector<int64_t> gid = read_all<int64_t>(argv[3], (size_t)n);
    const std::vector<uint8_t> dir = read_all<uint8_t>(argv[4], (size_t)n);
    sem::HostTables t;
    sem::build_tables(E, N, gid.data(), dir.data(), t);
    sem::build_direct_tables(E, N, t);
    int64_t checked = 0, generic = 0;
    if (t.direct) {
        std::map<int64_t, std::vector<int64_t>> copies;
        for (int64_t l = 0; l < n; ++l) copies[gid[l]].push_back(l);
        std::mt19937_64 rng(std::strtoull(argv[5], nullptr, 10));
        std::uniform_real_distribution<float> U(-1.f, 1.f);
        std::vector<float> w(n), wedge((size_t)(E * MS), 0.f);
        std::vector<int64_t> point((size_t)(E * MS), -1);
        for (int64_t l = 0; l < n; ++l) {
            w[l] = U(rng);
            const int loc = (int)(l % P3);
            const int s = sem::edge_slot(N, loc % P, (loc / P) % P, loc / (P * P));
            if (s < 0) continue;
            wedge[(size_t)(l / P3 * MS + s)] = w[l];
            point[(size_t)(l / P3 * MS + s)] = l;
        }
        for (int64_t l = 0; l < n; ++l) {
            const int m = t.mcode[l] & sem::kMultMask;
            const int loc = (int)(l % P3);
            const int s = sem::edge_slot(N, loc % P, (loc / P) % P, loc / (P * P));
            const int64_t g = l / P3 * MS + s;
            const int32_t src = t.gsrc_direct[l];
            if (m > 2 ? src != g : src != t.gsrc[l]) {
                std::printf("FAIL l=%lld: gather source %d\n", (long long)l, src);
                return 1;
            }
            if (s < 0) continue;
            const std::vector<int64_t> &cp = copies[gid[l]];
            bool all = true;
            for (int64_t c : cp) {
                const int lc = (int)(c % P3);
                all &= sem::edge_slot(N, lc % P, (lc / P) % P, lc / (P * P)) >= 0;
            }
            if (m > 2 && !all) {
                std::printf("FAIL l=%lld: group with a copy off the edges\n", (long long)l);
                return 1;
            }
            // pairs are read by their partner's index unless the table-free
            // gather applies, masked groups not at all
            if (!all || (!t.gs_struct && m == 2) || (t.mcode[l] & sem::kDirichletBit)) continue;
            const int4 lo = t.elist[(size_t)g];
            const int cn = sem::corner_of_slot(N, s);
            int4 hi = make_int4(-1, -1, -1, -1);
            if (cn >= 0) hi = t.elist_hi[(size_t)(8 * (l / P3) + cn)];
            const int ix[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            float v = 0.f;
            int count = 0;
            if (lo.x == -2) {
                ++generic;
                for (int q = 0; q < lo.z; ++q) {
                    const int p = t.egen[(size_t)(lo.y + q)];
                    v = q ? v + wedge[(size_t)p] : wedge[(size_t)p];
                    ++count;
                }
            } else {
                for (int q = 0; q < 8; ++q) {
                    if (ix[q] >= E * MS) count = -1000;
                    if (ix[q] < 0) continue;
                    v = count ? v + wedge[(size_t)ix[q]] : wedge[(size_t)ix[q]];
                    ++count;
                }
            }
            float want = w[cp[0]];
            for (size_t q = 1; q < cp.size(); ++q) want += w[cp[q]];
            if (count != m || std::memcmp(&v, &want, 4) != 0) {
                std::printf("FAIL l=%lld: %d of %d copies, %a, expected %a\n", (long long)l, count,
                            m, v, want);
                return 1;
            }
            ++checked;
        }
    }
    // the update's divisions by multiply and shift
    for (int k = 0; k < 1024; ++k)
        if ((int)(((uint32_t)k * ((1u << 20) / (uint32_t)MS + 1)) >> 20) != k / MS) {
            std::printf("FAIL division %d / %d\n", k, MS);
            return 1;
        }
    for (int k = 0; k < MS; ++k)
        if (sem::vecb::corner_of_slot_fast(P, k) != sem::corner_of_slot(N, k)) {
            std::printf("FAIL corner of slot %d\n", k);
            return 1;
        }
    std::printf("direct=%d checked=%lld generic=%lld\n", t.direct ? 1 : 0, (long long)checked,
                (long long)generic);
    return 0;
}
