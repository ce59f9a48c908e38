// Reads "norb nel" pairs and runs every 32-column tile of the strings' single
// excitations through the scatter programs on the host: for the programs that
// hold a tile, the sums they form (partial rounds, then rounds, lane by lane)
// against the plain sum of signed W elements per target, in integers.  Prints the
// first program that holds every tile, or a line starting with FAIL.
#include <cstdio>
#include <map>
#include <set>

#include "../paper_1707_04346_amd/csrc/scatter_prog.h"

using namespace cis;

int main() {
    int n, ne;
    while (std::scanf("%d %d", &n, &ne) == 2) {
        std::vector<uint32_t> str;
        std::map<uint32_t, int> index;
        for (uint32_t m = 0; m < (1u << n); ++m)
            if (__builtin_popcount(m) == ne) { index[m] = int(str.size()); str.push_back(m); }
        const int ld = (int(str.size()) + 63) / 64 * 64, mp = (n * (n + 1) / 2 + 15) / 16 * 16;
        ProgLayout L{32, uint32_t(mp) * 36, uint32_t(ld), 4, 1, 1};
        const int wsize = mp * 36 + 2 * kProgWaves * kProgLanes;
        bool every[kNumProgs];
        std::fill(every, every + kNumProgs, true);
        for (int t = 0; t * 32 < int(str.size()); ++t) {
            std::vector<ProgItem> items;
            for (int c = 0; c < 32 && t * 32 + c < int(str.size()); ++c) {
                const uint32_t J = str[t * 32 + c];
                for (int k = 0; k < n; ++k) {
                    if (!((J >> k) & 1u)) continue;
                    items.push_back({uint32_t(t * 32 + c), uint32_t((k * (k + 1) / 2 + k) * 36 + c), 0u});
                    for (int l = 0; l < n; ++l) {
                        if ((J >> l) & 1u) continue;
                        const int hi = std::max(k, l), lo = std::min(k, l);
                        items.push_back({uint32_t(index[(J & ~(1u << k)) | (1u << l)]),
                                         uint32_t((hi * (hi + 1) / 2 + lo) * 36 + c), uint32_t((k + l + c) & 1)});
                    }
                }
            }
            std::stable_sort(items.begin(), items.end(),
                             [](const ProgItem &a, const ProgItem &b) { return a.slot < b.slot; });
            std::vector<long long> W(wsize, 0), want(ld + 64, 0);
            unsigned long long rnd = 12345 + t;
            for (int r = 0; r < mp; ++r)
                for (int c = 0; c < 32; ++c) {
                    rnd = rnd * 6364136223846793005ull + 1442695040888963407ull;
                    W[r * 36 + c] = (long long)(rnd >> 40) - (1ll << 23);
                }
            for (const ProgItem &it : items) want[it.slot] += it.neg ? -W[it.w] : W[it.w];
            for (int g = 0; g < kNumProgs; ++g) {
                const ScatterProg &P = kProgs[g];
                std::vector<uint32_t> words;
                if (!prog_pack(P, L, items, words)) { every[g] = false; continue; }
                std::vector<long long> w2(W), got(ld + 64, 0);
                std::set<int> written;
                for (int wv = 0; wv < kProgWaves; ++wv) {
                    auto field = [&](int f, int lane) {
                        return (words[(size_t(wv) * P.words() + f / 2) * kProgLanes + lane] >> (16 * (f & 1))) & 0xffffu;
                    };
                    auto ref = [&](int f, int lane) {
                        const uint32_t x = field(f, lane);
                        const size_t e = (x & 0x7fffu) / 4;
                        if (e >= size_t(wsize)) { std::printf("FAIL reference out of range\n"); std::exit(1); }
                        return (x >> 15) ? -w2[e] : w2[e];
                    };
                    for (int p = 0; p < P.np; ++p)
                        for (int lane = 0; lane < kProgLanes; ++lane) {
                            long long s = 0;
                            for (int e = 0; e < P.ps; ++e) s += ref(p * P.ps + e, lane);
                            w2[mp * 36 + (wv * P.np + p) * kProgLanes + lane] = s;
                        }
                    int f = P.np * P.ps;
                    for (int r = 0; r < P.nr; ++r) {
                        for (int lane = 0; lane < kProgLanes; ++lane) {
                            long long s = 0;
                            for (int e = 0; e < P.r[r]; ++e) s += ref(f + 1 + e, lane);
                            const int slot = int(field(f, lane) / 4);
                            if (slot >= ld + 64) { std::printf("FAIL slot out of range\n"); return 1; }
                            if (slot >= ld && s != 0) { std::printf("FAIL discarded sum\n"); return 1; }
                            if (slot < ld && !written.insert(slot).second) { std::printf("FAIL target twice\n"); return 1; }
                            got[slot] += s;
                        }
                        f += 1 + P.r[r];
                    }
                }
                for (int i = 0; i < ld; ++i)
                    if (got[i] != want[i]) { std::printf("FAIL n %d e %d tile %d program %d\n", n, ne, t, g); return 1; }
            }
        }
        int first = 0;
        while (first < kNumProgs && !every[first]) ++first;
        std::printf("%d %d %d\n", n, ne, first < kNumProgs ? first : -1);
    }
    return 0;
}
