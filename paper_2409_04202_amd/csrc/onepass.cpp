// The one-pass form of a plan (onepass_kernel, encoding in onepass.hpp): per
// segment of element positions, the expression that every buffer ends with
// there, as its leaves in computing order; the tiling and the kernel
// instance.  Host only.
#include <algorithm>
#include <map>
#include <vector>

#include "exec_state.hpp"

namespace arp {

namespace {

// The values of one segment: a buffer's row as the plan finds it, or a fold
// of k >= 2 values (a copy names its source's value).
struct Values {
    struct Val {
        int32_t leaf;      // buffer, or -1 (a fold)
        int32_t in, k;     // a fold's inputs: ins[in .. in + k) in source order
    };
    std::vector<Val> vals;
    std::vector<int32_t> ins;
    std::vector<int32_t> cur;  // per buffer: its value, -1: its row, untouched

    explicit Values(int32_t n) : cur(size_t(n), -1) {}
    void clear() {
        vals.clear();
        ins.clear();
        std::fill(cur.begin(), cur.end(), -1);
    }
    int32_t of(int32_t b) {
        int32_t& c = cur[size_t(b)];
        if (c < 0) {
            c = int32_t(vals.size());
            vals.push_back({b, 0, 0});
        }
        return c;
    }
    // The phases are hazard-free: no later step of a phase reads or writes
    // what an earlier one wrote, so updating at once keeps its reads.
    void step(const XStep& x) {
        int32_t out;
        if (x.srcs.size() == 1) {
            out = of(x.srcs[0]);
        } else {
            const int32_t in = int32_t(ins.size());
            for (int32_t b : x.srcs) ins.push_back(of(b));
            out = int32_t(vals.size());
            vals.push_back({-1, in, int32_t(x.srcs.size())});
        }
        for (int32_t d : x.dsts) cur[size_t(d)] = out;
    }
};

// Leaves of value v in computing order, appended to w; false when there are
// more than n of them (a value used twice) or too many sums put aside.  `level`
// counts the folds that v is an operand of: each brings a leaf besides v's, so
// at n of them there are too many leaves, whatever lies below (which may be as
// many folds as the plan has phases).
struct Emit {
    const Values& vs;
    std::vector<uint32_t>& w;
    size_t most;       // words allowed
    bool rounds;       // step results are rounded (bf16)
    int32_t max_depth = 0;

    bool run(int32_t v, int32_t depth, size_t level = 0) {
        if (level >= most) return false;
        max_depth = std::max(max_depth, depth);
        const Values::Val& x = vs.vals[size_t(v)];
        if (x.leaf >= 0) {
            if (w.size() >= most) return false;
            w.push_back(uint32_t(x.leaf));
            return true;
        }
        // a step of two sources adds the folded one first: a chain of them
        // needs no sum put aside
        const bool swap = x.k == 2 && vs.vals[size_t(vs.ins[size_t(x.in)])].leaf >= 0 &&
                          vs.vals[size_t(vs.ins[size_t(x.in) + 1])].leaf < 0;
        for (int32_t i = 0; i < x.k; ++i) {
            const int32_t u = vs.ins[size_t(x.in + (swap ? 1 - i : i))];
            const bool is_fold = vs.vals[size_t(u)].leaf < 0;
            const size_t at = w.size();
            const bool aside = i > 0 && is_fold;
            if (depth + int32_t(aside) > kOneMaxDepth || !run(u, depth + int32_t(aside), level + 1))
                return false;
            if (!is_fold) continue;
            if (aside) {
                w[at] |= kOnePush;
                w.back() += 1u << kOnePopShift;
            } else if (rounds) {
                w.back() |= kOneRound;
            }
        }
        return true;
    }
};

}  // namespace

static bool team_tiles(int32_t n, int64_t tiles16) {
    return n >= kOneTeamMinN && tiles16 <= kOneTeamTiles;
}
static int64_t tiles_of(const Plan& p) {  // of 1 KiB of a buffer
    return (p.N * p.esize + 1023) / 1024;
}
bool onepass_teams(const Plan& p) { return team_tiles(p.n, tiles_of(p)); }
static bool team16(int32_t n, int64_t tiles16) {
    return tiles16 <= (n >= kOneTeamManyN ? kOneTeam16Tiles * 3 / 2 : kOneTeam16Tiles);
}
int32_t team_waves(const Plan& p) {
    return !onepass_teams(p) ? 0 : team16(p.n, tiles_of(p)) ? 16 : 4;
}
// Instance and tile for `tiles16` tiles of 64 16-byte vectors (see
// onepass.hpp for what was measured).  Instances with U > 1 are for launches
// that are resident at once, which their wavefronts' registers limit (kOneWide)
// and, at a fifth less than would fit, the sums that they put aside in LDS,
// depth * U * 64 each.
OneConf one_config(int32_t n, int64_t tiles16, int32_t depth, int32_t dtype, bool chain) {
    const bool bf16 = dtype == AR_BF16;
    if (team_tiles(n, tiles16)) return {team16(n, tiles16) ? ONE_TEAM16 : ONE_TEAM4, 4, 1, 1};
    if (tiles16 <= kOneNarrowTiles) return {ONE_LB4, 4, 1, 4};
    if (n >= kOneWideMinN)
        for (const OneWide& w : kOneWide) {
            if (bf16 != w.bf16 || tiles16 < w.from || tiles16 > w.to || (chain && !w.chain)) continue;
            const int64_t units = (tiles16 + w.u - 1) / w.u;
            const int64_t lds = int64_t(depth) * w.u * 1024 * (bf16 ? 2 : 1);
            if (lds == 0 || units * 5 <= kNumCUs * (kLdsBytesPerCU / lds) * 4)
                return {w.kind, 16, w.u, 1};
        }
    return {n < 8 ? ONE_U1B4 : n < 16 ? ONE_U1B8 : ONE_U1B16, 16, 1, 1};
}

static void build(const Plan& p, const ExecState& ex, OnePlan& one) {
    const int32_t n = p.n;
    const int64_t VEC = 16 / p.esize;
    if (n < 2 || n > kOneMaxN || p.N < VEC || ex.phases.empty()) return;
    std::vector<int64_t> cuts;
    for (const XPhase& xp : ex.phases)
        for (const XStep& x : xp.steps)
            if (x.end > x.begin) {
                cuts.push_back(x.begin);
                cuts.push_back(x.end);
            }
    std::sort(cuts.begin(), cuts.end());
    cuts.erase(std::unique(cuts.begin(), cuts.end()), cuts.end());
    // every position must be covered
    if (cuts.size() < 2 || cuts.front() != 0 || cuts.back() != p.N) return;
    const size_t nseg = cuts.size() - 1;
    if (nseg > size_t(kOneMaxSegs)) return;
    auto seg_of = [&](int64_t x) {
        return size_t(std::lower_bound(cuts.begin(), cuts.end(), x) - cuts.begin());
    };
    // the steps of each segment, in phase order
    std::vector<std::vector<const XStep*>> steps(nseg);
    int64_t covered = 0;
    one.max_k = one.max_dst = 0;
    one.nsteps = 0;
    for (const XPhase& xp : ex.phases)
        for (const XStep& x : xp.steps) {
            if (x.end <= x.begin) continue;
            const size_t a = seg_of(x.begin), b = seg_of(x.end);
            covered += int64_t(b - a) * int64_t(x.srcs.size() + x.dsts.size());
            if (covered > kOneMaxWork) return;
            for (size_t s = a; s < b; ++s) steps[s].push_back(&x);
            one.max_k = std::max(one.max_k, int32_t(x.srcs.size()));
            one.max_dst = std::max(one.max_dst, int32_t(x.dsts.size()));
            ++one.nsteps;
        }
    std::map<std::vector<uint32_t>, int32_t> known;  // leaves -> first word
    Values vs(n);
    std::vector<uint32_t> w;
    one.depth = one.pushes = 0;
    for (size_t s = 0; s < nseg; ++s) {
        vs.clear();
        for (const XStep* x : steps[s]) vs.step(*x);
        const int32_t v = vs.cur[0];
        if (v < 0 || vs.vals[size_t(v)].leaf >= 0) return;
        for (int32_t b = 1; b < n; ++b)
            if (vs.cur[size_t(b)] != v) return;
        w.clear();
        Emit em{vs, w, size_t(n), p.dtype == AR_BF16};
        if (!em.run(v, 0)) return;
        one.depth = std::max(one.depth, em.max_depth);
        // neighbours with the same expression are one segment
        if (!one.segs.empty() && one.segs.back().nleaf == int32_t(w.size()) &&
            std::equal(w.begin(), w.end(), one.prog.begin() + one.segs.back().off)) {
            one.segs.back().hi = cuts[s + 1];
            continue;
        }
        auto it = known.find(w);
        if (it == known.end()) {
            if (one.prog.size() + w.size() > size_t(kOneMaxWords)) return;
            it = known.emplace(w, int32_t(one.prog.size())).first;
            one.prog.insert(one.prog.end(), w.begin(), w.end());
        }
        one.segs.push_back({cuts[s], cuts[s + 1], it->second, int32_t(w.size())});
        int32_t pushes = 0;
        for (uint32_t x : w) pushes += (x & kOnePush) != 0;
        one.pushes = std::max(one.pushes, pushes);
        one.chain = one.chain || (p.dtype == AR_BF16 && em.max_depth == 0 && w.size() > 2 &&
                                  (w[1] & kOneRound) != 0);
    }
    one.conf = one_config(n, tiles_of(p), one.depth, p.dtype, one.chain);
    if (one.conf.u == 1 && one.conf.lb == 16 && n >= kOneManyMinN) {
        const int64_t bytes = int64_t(n) * p.N * p.esize;
        const bool whole = std::all_of(one.segs.begin(), one.segs.end(),
                                       [&](const OneSeg& sg) { return sg.lo % VEC == 0; });
        if (one.cm && tiles_of(p) > kOneManyTiles) one.many = 2;
        else if (whole && n < kOneFewN && bytes >= kOneFewBytes)
            one.many = tiles_of(p) > kOneManyTiles / 2 || bytes < kOneFewBytesTo;
    }
    const int64_t vec = one.conf.lb / p.esize;
    const int64_t te = 64 * vec * one.conf.u;
    std::vector<int64_t> nt;
    int64_t used = 0, most = 0;
    for (const OneSeg& sg : one.segs) {
        // counted from the vector boundary before it (buffers on 16-byte
        // boundaries); from its start there are no more
        nt.push_back((sg.hi - (sg.lo & ~(vec - 1)) + te - 1) / te);
        used += nt.back();
        most = std::max(most, nt.back());
    }
    const int64_t all = most * int64_t(one.segs.size());
    if (std::max(used, all) > kMaxBlocks) return;
    one.tiles_per_seg = most;
    one.nunits = all;
    if (used * 5 < all * 4) {  // uneven segments: a table
        one.nunits = used;
        for (size_t s = 0; s < one.segs.size(); ++s)
            for (int64_t t = 0; t < nt[s]; ++t) one.tiles.push_back(make_int2(int(s), int(t)));
    }
    one.ok = true;
}

void build_onepass(const Plan& p, const ExecState& ex, OnePlan& one) {
    if (one.tried) return;
    one.tried = true;
    // more than three eighths of the last-level cache: stream past it (n = 64
    // over 2^19 fp32, 128 MiB: 46 us, cached 56; over 2^18, 64 MiB: cached 21 us,
    // streamed 23)
    one.cm = int64_t(p.n) * p.N * p.esize >= kOneNtBytes ? 3 : 0;
    one.bytes = 2 * int64_t(p.n) * p.N * p.esize;
    build(p, ex, one);
    if (one.ok) return;
    one = OnePlan();
    one.tried = true;
}

// A wavefront's work and the bytes, ns.
static double one_wave_time(const Plan& p, const OnePlan& one) {
    if (onepass_teams(p))
        return kOneTeamLatNs +
               double(p.n) * (kOneTeamLeafNs + (one.chain ? kOneTeamRoundNs : 0.0)) +
               double(one.pushes) * kOneTeamPushNs;
    return kOneLatNs + double(p.n) * (kOneLeafNs + (one.chain ? kOneRoundNs : 0.0)) +
           double(one.pushes) * kOnePushNs;
}
static double one_mem_time(const Plan& p) {
    const double bytes = double(p.n) * double(p.N) * p.esize;
    return 2.0 * bytes / (bytes >= double(kOneNtBytes) ? kOneBytesPerNs : kOneCachedBytesPerNs);
}
double onepass_time(const Plan& p, const OnePlan& one) {
    const double w = one_wave_time(p, one), m = one_mem_time(p);
    return kLaunchNs + std::max(w, m) + (onepass_teams(p) ? 1.0 : kOneOverlap) * std::min(w, m);
}
bool onepass_streams(const Plan& p, const OnePlan& one) {
    return one_mem_time(p) >= one_wave_time(p, one);
}

bool onepass_beats_slice(const Plan& p, const OnePlan& one, bool resident) {
    const int64_t tiles = tiles_of(p);
    if (p.n == 2 && !one.cm && !resident)
        return tiles >= kOnePairTiles && 2 * p.N * p.esize < kOneFewBytes;
    return !resident || one.conf.u > 1 || one.conf.lb < 16 || !one.cm || one.many ||
           p.n < kOneRowsMinN || tiles <= kOneManyTiles / 2;
}

}  // namespace arp
