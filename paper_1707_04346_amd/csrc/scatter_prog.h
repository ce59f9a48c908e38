// scatter_prog.h -- the beta-side scatter of the one-block sigma_3 kernel as a
// fixed program of rounds, and the host packer that fits a tile's contributions
// into it.
//
// A 32-column source tile adds to each target beta string Ib a sum of W elements
// (the target's "group": (W element, sign) pairs; 1 to ~30 of them, most groups 1
// or 2, the tile's own strings the long ones).  The four scattering waves of a
// workgroup take disjoint sets of groups and run the same program:
//
//   partial rounds   each lane sums PS W elements into its own scratch element;
//   rounds i = 0..   each lane sums R[i] elements (W elements, or scratch elements
//                    of its own wave) and adds the sum to one sigma slot.
//
// A group longer than the rounds' sizes first sums parts of itself in partial
// lanes of its wave.  Every group ends in exactly one lane of one round, so a
// target is read and written once per tile, by one lane: no atomics, no
// conflicts, a fixed order.  Lanes without a group add zeros to a discard slot.
// Compared with cutting the sorted list into equal runs per lane (a
// read-modify-write per contribution, segmented sums across lanes) this takes
// about half the LDS accesses and a third of the vector instructions.
//
// Words per lane (16-bit fields, two per word, low half first): PS references per
// partial round, then per round the slot and R[i] references.  Reference: bits
// 0..14 the element's offset in `unit` bytes from the start of W, bit 15 the sign.  Slot:
// the sigma element in `sunit` bytes.  (One 32-bit word a field, which takes fewer
// vector instructions, doubles the plan's traffic: FP64 sigma_3 of CAS(16,16) 61.7
// instead of 54.8 ms, FP32 19.6 instead of 18.9, both when taken.)
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace cis {

constexpr int kProgLanes = 64, kProgWaves = 4;

struct ScatterProg {
    int np, ps;          // partial rounds and references in each
    int nr, r[6];        // rounds, references in each (descending)
    constexpr int fields() const {
        int f = np * ps;
        for (int i = 0; i < nr; ++i) f += 1 + r[i];
        return f;
    }
    constexpr int words() const { return (fields() + 1) / 2; }
};

// Cheapest first.
constexpr int kNumProgs = 5;
constexpr ScatterProg kProgs[kNumProgs] = {   // (at most 8 references a round)
    {1, 4, 1, {5}},
    {1, 4, 2, {6, 1}},
    {1, 4, 3, {6, 2, 1}},
    {1, 4, 5, {6, 3, 2, 1, 1}},
    {1, 6, 5, {8, 4, 2, 1, 1}},
};

struct ProgItem { uint32_t slot, w, neg; };   // sigma slot, W element, sign

// Where the references point and how they are written.
struct ProgLayout {
    uint32_t zero;       // W element that is always zero
    uint32_t scratch;    // first scratch element (counted from the start of W): [wave][partial round][lane]
    uint32_t spare;      // first of 64 discard slots
    uint32_t bytes;      // bytes per element
    uint32_t unit;       // bytes per reference unit
    uint32_t sunit;      // bytes per slot unit
};

// Fits the items of one tile, sorted by slot, into program g; appends
// kProgWaves * g.words() * kProgLanes words to out ([wave][word][lane]).  False
// (nothing appended) when they do not fit.
inline bool prog_pack(const ScatterProg &g, const ProgLayout &L, const std::vector<ProgItem> &items,
                      std::vector<uint32_t> &out) {
    struct Group { int first, size; };
    std::vector<Group> groups;             // longest first, equal lengths by slot
    {
        std::vector<Group> seen;
        int longest = 0;
        for (size_t i = 0; i < items.size();) {
            size_t j = i + 1;
            while (j < items.size() && items[j].slot == items[i].slot) ++j;
            seen.push_back({int(i), int(j - i)});
            longest = std::max(longest, int(j - i));
            i = j;
        }
        std::vector<int> at(size_t(longest) + 2, 0);
        for (const Group &x : seen) ++at[size_t(longest - x.size) + 1];
        for (int i = 0; i <= longest; ++i) at[size_t(i) + 1] += at[size_t(i)];
        groups.resize(seen.size());
        for (const Group &x : seen) groups[size_t(at[size_t(longest - x.size)]++)] = x;
    }
    const int nf = g.fields(), nw = g.words();
    const uint32_t scale = L.bytes / L.unit, sscale = L.bytes / L.sunit;
    std::vector<uint16_t> f(size_t(kProgWaves) * nf * kProgLanes);
    auto at = [&](int wv, int field, int lane) -> uint16_t & {
        return f[(size_t(wv) * nf + field) * kProgLanes + lane];
    };
    int round_field[6];
    {
        int x = g.np * g.ps;
        for (int i = 0; i < g.nr; ++i) { round_field[i] = x; x += 1 + g.r[i]; }
    }
    for (int wv = 0; wv < kProgWaves; ++wv)
        for (int lane = 0; lane < kProgLanes; ++lane) {
            for (int q = 0; q < nf; ++q) at(wv, q, lane) = uint16_t(L.zero * scale);
            for (int i = 0; i < g.nr; ++i) at(wv, round_field[i], lane) = uint16_t((L.spare + lane) * sscale);
        }
    auto ref = [&](const ProgItem &it) { return uint16_t(it.w * scale | (it.neg << 15)); };
    // LDS accesses are served half a wave at a time: within a half, elements of one
    // bank (of 64 four-byte ones) queue up.  hits counts them per field and half.
    constexpr int H = 2, HL = kProgLanes / H, NB = 64;
    std::vector<uint8_t> hits(size_t(kProgWaves) * nf * H * NB, 0);
    auto hit = [&](int wv, int field, int half, uint32_t elem) -> uint8_t & {
        return hits[((size_t(wv) * nf + field) * H + half) * NB + elem % NB];
    };
    int used[kProgWaves][6][H] = {}, pused[kProgWaves][2][H] = {};
    // next lane of a round (or partial round) with n free lanes per half: the half
    // where `elem` meets fewer others in `field`
    auto pick = [&](const int (&u)[H], int wv, int field, uint32_t elem) {
        int best = -1;
        for (int h = 0; h < H; ++h)
            if (u[h] < HL && (best < 0 || hit(wv, field, h, elem) < hit(wv, field, best, elem))) best = h;
        return best;
    };
    // items [q, q + n) into fields field.. of a lane, each field taking the item whose
    // bank is least hit there
    auto fill = [&](int wv, int field, int lane, int q, int n) {
        int left[8];
        for (int i = 0; i < n; ++i) left[i] = q + i;
        for (; n > 0; --n, ++field) {
            uint8_t *row = &hit(wv, field, lane / HL, 0);
            int best = 0;
            for (int i = 1; i < n && row[items[left[best]].w % NB] > 0; ++i)
                if (row[items[left[i]].w % NB] < row[items[left[best]].w % NB]) best = i;
            at(wv, field, lane) = ref(items[left[best]]);
            ++row[items[left[best]].w % NB];
            left[best] = left[n - 1];
        }
    };
    // one group into one wave: the smallest round that holds it, else the largest
    // round with room and the part that is too long in partial lanes
    auto place = [&](int wv, const Group &gr) {
        auto room = [&](const int (&u)[H]) { return kProgLanes - u[0] - u[1]; };
        int round = -1, parts = 0, proom = 0;
        for (int i = 0; i < g.np; ++i) proom += room(pused[wv][i]);
        for (int i = g.nr - 1; i >= 0 && round < 0; --i)
            if (g.r[i] >= gr.size && room(used[wv][i]) > 0) round = i;
        for (int i = 0; i < g.nr && round < 0; ++i) {
            if (room(used[wv][i]) == 0 || g.ps < 2) continue;
            const int need = (gr.size - g.r[i] + g.ps - 2) / (g.ps - 1);
            if (need <= g.r[i] && need <= proom) { round = i; parts = need; }
        }
        if (round < 0) return false;
        int q = gr.first, field = round_field[round], left = gr.size;
        const uint32_t slot = items[q].slot;
        const int half = pick(used[wv][round], wv, field, slot);
        const int lane = half * HL + used[wv][round][half]++;
        ++hit(wv, field, half, slot);
        at(wv, field++, lane) = uint16_t(slot * sscale);
        const int direct = g.r[round] - parts;     // items that stay out of the parts
        for (int k = 0; k < parts; ++k) {
            int pr = 0;
            while (room(pused[wv][pr]) == 0) ++pr;
            const int ph = pick(pused[wv][pr], wv, pr * g.ps, items[q].w);
            const int pl = ph * HL + pused[wv][pr][ph]++;
            const int n = std::min(g.ps, left - direct > 0 ? left - direct : 0);
            fill(wv, pr * g.ps, pl, q, n);
            q += n;
            left -= n;
            const uint32_t se = L.scratch + (wv * g.np + pr) * kProgLanes + pl;
            at(wv, field, lane) = uint16_t(se * scale);
            ++hit(wv, field++, half, se);
        }
        fill(wv, field, lane, q, left);
        return true;
    };
    // longest groups first, dealt to the waves in turn; a wave without room passes
    int turn = 0;
    for (const Group &gr : groups) {
        bool done = false;
        for (int k = 0; k < kProgWaves && !done; ++k) done = place((turn + k) % kProgWaves, gr);
        if (!done) return false;
        ++turn;
    }
    const size_t base = out.size();
    out.resize(base + size_t(kProgWaves) * nw * kProgLanes);
    for (int wv = 0; wv < kProgWaves; ++wv)
        for (int w = 0; w < nw; ++w)
            for (int lane = 0; lane < kProgLanes; ++lane) {
                const uint32_t lo = at(wv, 2 * w, lane);
                const uint32_t hi = 2 * w + 1 < nf ? at(wv, 2 * w + 1, lane) : 0u;
                out[base + (size_t(wv) * nw + w) * kProgLanes + lane] = lo | (hi << 16);
            }
    return true;
}

}  // namespace cis
