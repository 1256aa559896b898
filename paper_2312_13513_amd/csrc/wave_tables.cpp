// Host builder of the wave-per-cell integrator's tables (wave_tables.h).

#include "wave_tables.h"

#include <algorithm>
#include <cstring>

namespace chem {
namespace {

constexpr int kLanes = 64;

// Appends v to the block, 16-byte aligned; returns its offset.
template <typename T>
size_t place(std::vector<char> &blk, const std::vector<T> &v)
{
    const size_t off = (blk.size() + 15) & ~size_t(15);
    blk.resize(off + std::max<size_t>(v.size(), 1) * sizeof(T), 0);
    if (!v.empty()) std::memcpy(blk.data() + off, v.data(), v.size() * sizeof(T));
    return off;
}

}  // namespace

std::vector<char> build_wave_tables(int K, const std::vector<DevRxn> &rx, int R,
                                    const std::vector<std::vector<std::pair<int, int>>> &inc,
                                    const std::vector<double> &species, const std::vector<double> &W,
                                    const std::vector<double> &aux, const char *base, Wave64Tables &t)
{
    std::vector<char> blk;
    t = Wave64Tables{};
    t.rounds = std::max(4, (R + kLanes - 1) / kLanes);
    // ---- reactions ----
    std::vector<double2> rxa((size_t)t.rounds * 2 * kLanes);
    std::vector<uint32_t> rw((size_t)t.rounds * kLanes);
    for (int i = 0; i < t.rounds; i++)
        for (int l = 0; l < kLanes; l++) {
            const int r = i * kLanes + l;
            double2 a{-1e300, 0.0}, b{0.0, 0.0};   // padded: both rate constants are exp(-1e300) = 0
            uint32_t w = (uint32_t)(K | K << 6 | K << 12 | K << 18) | kRxnWordIrrev;
            if (r < R) {
                const DevRxn &x = rx[r];
                a = double2{x.lnA, x.b};
                b = double2{x.Ea_R, (double)x.dnu};
                w = (uint32_t)(x.r0 | x.r1 << 6 | x.p0 << 12 | x.p1 << 18 | (x.kind & 7) << 24) |
                    ((x.kind & kRxnIrrev) ? kRxnWordIrrev : 0u);
            }
            rxa[(size_t)(2 * i) * kLanes + l] = a;
            rxa[(size_t)(2 * i + 1) * kLanes + l] = b;
            rw[(size_t)i * kLanes + l] = w;
        }
    // ---- production sums: the shortest segment length with which the extra
    // segments fit the lanes from K on, but at least 24 entries: up to there a
    // species is summed by one lane in reaction order (fast forward and
    // reverse rates nearly cancel, so another order moves the last digits of
    // the result the most), and the kernel's code for a few quads is straight ----
    std::vector<std::vector<uint32_t>> ent(K);
    size_t longest = 1;
    for (int k = 0; k < K; k++) {
        for (const auto &e : inc[k])
            for (int c = 0; c < std::abs(e.second); c++)
                ent[k].push_back(8u * (uint32_t)(1 + e.first + (e.second < 0 ? R : 0)));
        longest = std::max(longest, ent[k].size());
    }
    auto extra = [&](size_t seg, int k) { return ent[k].empty() ? size_t(0) : (ent[k].size() - 1) / seg; };
    size_t seg = std::min<size_t>(24, (longest + 3) & ~size_t(3));
    for (; seg < longest; seg += 4) {
        size_t x = 0;
        for (int k = 0; k < K; k++) x += extra(seg, k);
        if (x <= (size_t)(kLanes - K)) break;
    }
    t.gather4 = (int32_t)(seg / 4);
    std::vector<uint32_t> gat((size_t)t.gather4 * kLanes * 4, 0u);   // offset 0: the zero slot
    std::vector<int32_t> xseg(kLanes, 0);
    auto put = [&](int lane, size_t j, uint32_t v) { gat[((j / 4) * kLanes + lane) * 4 + j % 4] = v; };
    int next = K;
    for (int k = 0; k < K; k++) {
        xseg[k] = next;
        for (size_t j = 0; j < ent[k].size(); j++) {
            if (j < seg)
                put(k, j, ent[k][j]);
            else
                put(next + (int)(j / seg) - 1, j % seg, ent[k][j]);
        }
        const int x = (int)extra(seg, k);
        xseg[k] |= x << 8;
        next += x;
        t.extras = std::max(t.extras, x);
    }
    // ---- Jacobian entries ----
    struct Entry {
        int row, col;
        std::vector<uint32_t> con;
    };
    std::vector<Entry> je;
    for (int k = 0; k < K; k++) {
        std::vector<std::vector<uint32_t>> cols(K);
        std::vector<char> listed(K, 0);   // columns of listed third-body efficiencies: the kernel adds to them
        for (const auto &e : inc[k]) {
            const DevRxn &x = rx[e.first];
            if ((x.kind & 7) != kRxnElem)
                for (int j = 0; j < x.neff; j++) listed[(int)aux[x.aux + kAuxHead + 2 * j]] = 1;
            const int sl[4] = {x.r0, x.r1, x.p0, x.p1};
            for (int s = 0; s < 4; s++)
                if (sl[s] < K)
                    for (int c = 0; c < std::abs(e.second); c++)
                        cols[sl[s]].push_back(8u * (uint32_t)(1 + 4 * e.first + s) |
                                              (e.second < 0 ? 0x80000000u : 0u));
        }
        for (int c = 0; c < K; c++)
            if (!cols[c].empty() || listed[c]) je.push_back(Entry{k, c, std::move(cols[c])});
    }
    std::stable_sort(je.begin(), je.end(), [](const Entry &a, const Entry &b) { return a.con.size() > b.con.size(); });
    t.jrounds = (int32_t)((je.size() + kLanes - 1) / kLanes);
    std::vector<int2> jcnt;
    std::vector<uint32_t> jrc((size_t)t.jrounds * kLanes, 0xFFFFu), jcon;
    for (int i = 0; i < t.jrounds; i++) {
        const size_t n = std::max<size_t>(4, (je[(size_t)i * kLanes].con.size() + 3) & ~size_t(3));
        jcnt.push_back(int2{(int)(jcon.size() / kLanes), (int)n});
        const size_t at = jcon.size();
        jcon.resize(at + n * kLanes, 0u);
        for (int l = 0; l < kLanes && (size_t)(i * kLanes + l) < je.size(); l++) {
            const Entry &e = je[(size_t)i * kLanes + l];
            jrc[(size_t)i * kLanes + l] = (uint32_t)(e.row | e.col << 8);
            for (size_t j = 0; j < e.con.size(); j++) jcon[at + j * kLanes + l] = e.con[j];
        }
    }
    // ---- thermo ----
    std::vector<double2> th((size_t)2 * 7 * kLanes, double2{0.0, 0.0});
    std::vector<double> tmid(kLanes, 0.0), invw(kLanes, 0.0);
    for (int k = 0; k < K; k++) {
        const double *s = &species[(size_t)k * kSpeciesLen];
        tmid[k] = s[0];
        invw[k] = 1.0 / W[k];
        for (int g = 0; g < 2; g++)
            for (int j = 0; j < 7; j++)
                th[(size_t)(g * 7 + j) * kLanes + k] =
                    double2{s[1 + g * kRangeLen + 2 * j], s[1 + g * kRangeLen + 2 * j + 1]};
    }
    // ---- pressure-dependent reactions of each species ----
    std::vector<int32_t> poff(kLanes + 1, 0);
    std::vector<int2> pent;
    for (int k = 0; k < kLanes; k++) {
        if (k < K)
            for (const auto &e : inc[k])
                if ((rx[e.first].kind & 7) != kRxnElem) pent.push_back(int2{e.first, e.second});
        poff[k + 1] = (int32_t)pent.size();
    }
    // ---- one block ----
    const size_t o_rx = place(blk, rxa), o_rw = place(blk, rw), o_gat = place(blk, gat), o_xs = place(blk, xseg),
                 o_jn = place(blk, jcnt), o_jr = place(blk, jrc), o_jc = place(blk, jcon), o_th = place(blk, th),
                 o_tm = place(blk, tmid), o_iw = place(blk, invw), o_po = place(blk, poff), o_pe = place(blk, pent);
    t.rx = (const double2 *)(base + o_rx);
    t.rw = (const uint32_t *)(base + o_rw);
    t.gat = (const uint4 *)(base + o_gat);
    t.xseg = (const int32_t *)(base + o_xs);
    t.jcnt = (const int2 *)(base + o_jn);
    t.jrc = (const uint32_t *)(base + o_jr);
    t.jcon = (const uint32_t *)(base + o_jc);
    t.th = (const double2 *)(base + o_th);
    t.tmid = (const double *)(base + o_tm);
    t.invw = (const double *)(base + o_iw);
    t.poff = (const int32_t *)(base + o_po);
    t.pent = (const int2 *)(base + o_pe);
    return blk;
}

}  // namespace chem
