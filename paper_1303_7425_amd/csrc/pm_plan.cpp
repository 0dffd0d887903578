// Host planner: see pm_plan.hpp.
#include "pm_plan.hpp"

#include <stdio.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <vector>

#include "../../include/polymul.h"

namespace pm {

static std::mutex g_tune_mu;
static std::map<TuneClass, TuneChoice> g_tune_cache;

bool tune_lookup(const TuneClass &c, TuneChoice &choice) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune_cache.find(c);
    if (it == g_tune_cache.end()) return false;
    choice = it->second;
    return true;
}

void tune_store(const TuneClass &c, const TuneChoice &choice) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache[c] = choice;
}

void tune_reset() {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache.clear();
}

// Text file, one choice per line: ring dense log2pairs tile_cfg combine digits,
// and a 1 behind them where the choice was faster than the automatic path too.
int tune_save(const char *path) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    FILE *f = fopen(path, "w");
    if (!f) return PM_EINVAL;
    fprintf(f, "# polymul tuning: ring dense log2pairs tile_cfg combine digits\n");
    for (auto &kv : g_tune_cache)
        fprintf(f, "%d %d %d %d %d %d%s\n", kv.first.ring, kv.first.dense, kv.first.log2pairs, kv.second.tile_cfg,
                kv.second.combine, kv.second.digits, kv.second.over_auto ? " 1" : "");
    return fclose(f) == 0 ? PM_OK : PM_EINVAL;
}

int tune_load(const char *path) {
    FILE *f = fopen(path, "r");
    if (!f) return PM_EINVAL;
    std::vector<std::pair<TuneClass, TuneChoice>> got;
    char line[256];
    int rc = PM_OK;
    while (fgets(line, sizeof line, f)) {
        if (line[0] == '#' || line[0] == '\n') continue;
        int r, d, l, t, c, g, over = 0;
        if (sscanf(line, "%d %d %d %d %d %d %d", &r, &d, &l, &t, &c, &g, &over) < 6 || r < 0 || r > 4 || d < 0 || d > 1 ||
            l < 0 || l > 127 || t < -1 || t >= N_TILE_CFGS || c < -1 || c > 3 || g < -1 || g > 1) {
            rc = PM_EINVAL;
            break;
        }
        got.push_back({TuneClass{r, d, l}, TuneChoice{t, c, g, over == 1}});
    }
    fclose(f);
    if (rc != PM_OK) return rc;  // nothing is taken from a malformed file
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &e : got) g_tune_cache[e.first] = e.second;
    return PM_OK;
}

// Digit widths of the radix passes over the keys' significant bits: 8 bits
// per pass with the remainder in the last (RADIX_DIGITS_GREEDY), or the same
// number of passes with widths as equal as possible, wider ones first
// (RADIX_DIGITS_BALANCED): fewer digit values give longer runs per digit and
// fuller cache lines in the scatter.
void set_digits(Plan &P, int schedule) {
    int shift = 0;
    for (int p = 0; p < P.passes; p++) {
        int w;
        if (schedule == RADIX_DIGITS_GREEDY) {
            w = std::min(RADIX_BITS, std::max(1, P.max_bits - shift));
        } else {
            const int rest = std::max(P.passes, P.max_bits - shift), left = P.passes - p;
            w = std::min(RADIX_BITS, (rest + left - 1) / left);
        }
        P.dsh[p] = (unsigned char)shift;
        P.dbits[p] = (unsigned char)w;
        shift += w;
    }
}

int log2_floor(uint64_t x) {
    int b = -1;
    while (x) {
        b++;
        x >>= 1;
    }
    return b;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t stats_region_bytes(int nseg, int nvars) {
    return align256(stats_bytes(nseg, nvars)) + align256((size_t)nseg * 2 * sizeof(uint32_t));
}

static int bitlen128(unsigned __int128 x) {
    int b = 0;
    while (x) {
        b++;
        x >>= 1;
    }
    return b;
}

// One way to run a product by prefix groups (SEG_GRP, SEG_GRPD).
struct GpTry {
    bool ok = false;
    GrpSeg g{};
    int64_t ibound = 0, items = 0, nres = 0;
    int64_t bytes = 0;  // of workspace
};

// What the general plan's pass finds out about prefix groups.
struct GpProbe {
    std::vector<int64_t> old_bytes, bytes;  // workspace of every product's arrays: in the general plan, by prefix groups
    bool pays = false;                      // some product's groups pay
};

constexpr double GP_MIN_PAIRS = 4096;  // a product of fewer is not tried: latencies bound every path there, planning too

// The split of a product's keys into prefix and bin, from sizes and ranges
// alone.  way 1: bins that fit direct cells, with a few to a work item for
// the degree box (so that items can be cut to an even size: box cells over 16
// rounds of the device, 512 to GP_CELLS); way 2: bins that only fit the
// presence bitmap (sparse), or up to all direct cells (degree box).  The fewest
// prefix variables that do: fewer groups, larger blocks.
static GpTry gp_try(int nvars, const VarParam *vp, int64_t na, int64_t nb, unsigned __int128 box, bool dense, double cus,
                    int way, bool f64) {
    GpTry o;
    const double pairs = (double)na * (double)nb;
    if (na >= (int64_t)1 << 27 || nb >= (int64_t)1 << 27) return o;  // byte offsets of terms: 32 bits
    if (std::min(na, nb) > 65536) return o;  // pairs of one monomial: see gp_split
    if (!dense && (unsigned __int128)na * nb > 0xFFFFFFFFull) return o;
    const int64_t target =
        (int64_t)std::min<unsigned __int128>(GP_CELLS, std::max<unsigned __int128>(512, (unsigned __int128)((double)box / (cus * 16))));
    if (f64 && way != 1) return o;
    const uint64_t fit = f64 ? (uint64_t)GP_F64_CELLS : dense ? (way == 1 ? (uint64_t)target / 4 : (uint64_t)GP_CELLS)
                               : (way == 1 ? (uint64_t)GP_CELLS : (uint64_t)GP_MAX_S);
    const double most_bins = dense ? 2147483648.0 : std::max(way == 1 ? 16384.0 : 65536.0, pairs / 4);
    GrpSeg &g = o.g;
    for (int d = 1; d <= nvars && !o.ok; d++) {
        const VarParam &v = vp[d - 1];
        if (v.range == 0 || v.range > 0xFFFFFFFFull) return o;
        if (v.stride > fit) continue;
        const unsigned __int128 bins = box / v.stride;
        if ((double)bins > most_bins) return o;
        if (!dense && way == 2 && v.stride <= (uint64_t)GP_CELLS) return o;
        // (a bin of more pairs than there are cells takes several rounds of ranks: one variable more
        // where its bins are still too wide for direct cells; 3000 x 3000 terms of 5^8 exponents 677 us, by work items 611)
        if (!dense && way == 2 && pairs / (double)bins > GP_CELLS && d < nvars && vp[d].stride > (uint64_t)GP_CELLS) continue;
        g.S = (uint32_t)v.stride;
        g.d = (uint32_t)d;
        g.nbins = (uint32_t)bins;
        o.ok = true;
    }
    if (!o.ok) return o;
    const int64_t nt = na + nb;
    o.bytes = (int64_t)(sizeof(GpTerm) + 8) * nt + 4 * ((int64_t)g.nbins + 1) + 18 * 256 +
              GP_PAD * (int64_t)sizeof(GpTerm) + 4 * (nt / GP_PART + 2);
    if (dense) {
        // runs of K bins, cut into work items of about 1/12 of a workgroup's
        // share (512 workgroups), at least 2048 pairs
        g.K = (uint32_t)vp[g.d - 1].range;
        const int64_t runs = g.nbins / g.K, least = gp_run_items(g.K, g.S, 0);
        const double t = std::max(2048.0, pairs / (24.0 * cus));
        while (pairs / (double)(1ull << g.csh) + 1e6 > 4e9) g.csh++;
        g.T = (uint32_t)std::max(1.0, t / (double)(1ull << g.csh));
        g.nsb = (runs + GP_SB - 1) / GP_SB;
        o.ibound = runs * (least + 2) + (int64_t)(pairs / t * 1.1 * (double)(1u << g.csh)) + 64;
        o.items = runs * least + (int64_t)(pairs / t);
        o.bytes += g.nsb * (4 * GP_SB + 20) + o.ibound * ((int64_t)sizeof(GpItem) + 5);
        return o;
    }
    if (f64) {
        // one wave per work item: its bins fit the wave's cells
        const int fc = g.S <= 1024 ? 1024 : g.S <= 2048 ? 2048 : GP_F64_CELLS;
        g.T = (uint32_t)std::min(2048.0, std::max(256.0, pairs / (16.0 * cus)));
        g.span_bins = std::max<uint32_t>(1, (uint32_t)fc / g.S);
        g.heavy = 0xFFFFFFFFu;
        g.nsb = ((int64_t)g.nbins + GP_SB - 1) / GP_SB;
        o.nres = (int64_t)std::min((unsigned __int128)na * nb, box);
        const int64_t cross = ((int64_t)g.nbins + g.span_bins - 1) / g.span_bins + g.nsb;
        o.ibound = std::min<int64_t>((int64_t)(pairs / g.T) + cross + 2 * g.nsb, g.nbins) + 1;
        o.items = std::max<int64_t>((int64_t)(pairs / g.T), cross);
        o.bytes += g.nsb * (4 * GP_SB + 20) + o.ibound * ((int64_t)sizeof(GpItem) + 5) + 12 * o.nres;
        return o;
    }
    // work items of about 4096 pairs, fewer while that leaves compute units idle
    g.T = (uint32_t)std::min(4096.0, std::max(512.0, pairs / (4.0 * cus)));
    g.span_bins = std::max<uint32_t>(1, (1u << GP_SPAN_LOG) / g.S);
    // a bin that alone fills the direct cells to a quarter and more (with
    // S <= GP_CELLS / 2 several fit and stay together up to gp.T pairs)
    g.heavy = g.S <= (uint32_t)GP_CELLS && 2 * g.S > (uint32_t)GP_CELLS ? g.S / 4 : 0xFFFFFFFFu;
    g.nsb = ((int64_t)g.nbins + GP_SB - 1) / GP_SB;
    o.nres = (int64_t)std::min((unsigned __int128)na * nb, box);
    // starts of work items: the first bin of a super-bin, a crossing of a
    // multiple of T (or of a span), a heavy bin and the one after it
    const int64_t span_cross = ((int64_t)g.nbins + g.span_bins - 1) / g.span_bins + g.nsb;
    o.ibound = (int64_t)(pairs / g.T) + span_cross + 2 * g.nsb;
    o.ibound += 2 * (int64_t)(pairs / std::min<uint32_t>(g.heavy, gl_pairs(19) / 4));  // (also gp_list's)
    o.ibound = std::min<int64_t>(o.ibound, g.nbins) + 1;
    o.items = std::max<int64_t>((int64_t)(pairs / g.T), (g.nbins + g.span_bins - 1) / g.span_bins);
    o.bytes += g.nsb * (4 * GP_SB + 20) + o.ibound * ((int64_t)sizeof(GpItem) + 5) + 12 * o.nres;
    return o;
}

// Small blocks: their pairs are listed (k_gp_list).  The sparser the product,
// the wider the key span of a work item.
static void gp_list(GpTry &t, double pairs, unsigned __int128 box, double cus) {
    GrpSeg &g = t.g;
    const double density = pairs / (double)box;
    uint32_t sl = 17;
    while (sl < 19 && density * (double)(1u << sl) < gl_pairs(sl) * 2.0 / 3) sl++;
    g.rows = sl;
    // a work item has its share of T pairs and at most one bin that is not heavy
    g.T = (uint32_t)std::min(gl_pairs(sl) * 0.75, std::max(512.0, pairs / (4.0 * cus)));
    g.heavy = gl_pairs(sl) / 4;
    g.span_bins = std::max<uint32_t>(1, (1u << sl) / g.S);
    t.items = std::max<int64_t>((int64_t)(pairs / g.T), (g.nbins + g.span_bins - 1) / g.span_bins);
}

// Whether the operands' groups make that split pay.  Every work item looks
// every outer group up (at most two lookups per pair, where the staged path
// spends hundreds of instructions); a block below four pairs leaves most of
// its lanes idle.  The bitmap needs some pairs per span to pay for its scan.
static bool gp_pays(const GpTry &t, double gf, double gg, int64_t na, int64_t nb, unsigned __int128 box, bool dense,
                    int way, bool f64) {
    const double pairs = (double)na * (double)nb;
    if (gf < 1 || gg < 1) return false;
    const double cells = std::min<double>(t.g.nbins, gf * gg) * t.g.S;  // of the non-empty bins, at most
    if (f64) {
        // a wave adds one row of one inner group at a time: a step per outer
        // term and inner group, which the radix sort's cost per pair buys
        // from about two columns on; lookups: f's groups for every work item
        // (non-empty bins: a few dozen per group where the groups form a regular set)
        const double items = std::min<double>(t.items, 32 * (gf + gg) + pairs / t.g.T);
        if ((double)nb / gg < 4 || items * gf > pairs) return false;
        // Measured costs, in ps: a non-empty bin's work item about 7 ns, a row's
        // step by how many waves the cells leave on a compute unit, a block;
        // against the sort's 32 per pair and more for a long operand (16 x
        // 300000 terms of 31^5 exponents 1272 us, by the sort 439; 3000 x 3000
        // of 8^6 421, 314; 1000 x 20000 of 61^3 678, 521).
        const double cols = (double)nb / gg, steps = (double)na * gg * std::ceil(cols / 64);
        const double step = t.g.S <= 1024 ? 100 : t.g.S <= 2048 ? 140 : 210;
        const double bins = std::min(std::min<double>(t.items, 16 * (gf + gg) + pairs / t.g.T), gf * gg);
        // the fullest bin's rows come one after another, 32 ns each; the sort
        // sums long runs of like terms one by one
        if (steps / std::max(gf, gg) * 32000 > 90e6 + (pairs > 32 * cells ? 64 : 32) * pairs) return false;
        return bins * 7000 + steps * step + gf * gg * 100 <= 20e6 + 32 * pairs + 400 * (double)(na + nb);
    }
    if ((double)t.items * std::min(gf, gg) > (t.g.rows ? 8 : 2) * pairs) return false;
    if (!t.g.rows || dense) {
        // A bin is one work item, however many pairs it has: where the operands
        // have few groups the fullest one, a block of each, outlasts the rest
        // (1378 x 8605 terms in 3 groups each 8.5 ms, by the staged work items
        // 0.24).  One workgroup takes at least 0.35 ns per pair in direct cells,
        // 0.2 per pair and sweep in ranks: two sweeps and one more per 4096 keys.
        // The staged work items take 15 ps per pair beyond what both have, and
        // three times that where fine bins hold few pairs or more than a work
        // item's.
        const double most = pairs / std::max(gf, gg);
        const double each = t.g.S <= (uint32_t)GP_CELLS ? 350 : 200 * (1 + std::ceil(std::min<double>(most, t.g.S) / GP_CELLS));
        const bool slow = !dense && (8 * cells > pairs || 8 * (double)box > 4096 * cells);
        if (most * each > (slow ? 200e6 + 45 * pairs : 60e6 + 15 * pairs)) return false;
    }
    // beyond 32-bit keys the alternative is the pair-index sort, some 62 ps per
    // pair; a listed work item takes 27 ns and its pairs 34 ps with their
    // placement, a pair of groups 18 ps (300 x 20000 terms of 4^12 exponents
    // 961 us, by the sort 495)
    if (t.g.rows && !dense && box > (unsigned __int128)0xFFFFFFFFull && (double)t.items * 27000 + 18 * gf * gg > 75e6 + 28 * pairs)
        return false;
    const double block = pairs / (gf * gg);
    if (dense) return block * t.g.nbins / t.items >= 4;
    if (pairs / (double)box * t.g.span_bins * t.g.S < (t.g.rows ? 24 : 256)) return false;
    return way == 1 ? block >= 4 : t.g.rows || block >= 1.5;
}

// A product that one workgroup sorts and sums in LDS: TINY_PAIRS is what its
// LDS holds, and up to there it is the fastest path at every ring and density
// (57 x 61 random FP64 terms in 6 variables: 121 us by the radix sort, now 55).
static bool tiny_fits(int64_t na, int64_t nb, unsigned __int128 box) {
    return (unsigned __int128)na * nb <= (unsigned)TINY_PAIRS && box <= (unsigned __int128)0xFFFFFFFFull;
}

// counted: the minima's upper halves hold group counts (smask takes them off).
// probe: the general plan, and what prefix groups would need and whether some
// product's pay; without it such products run by them, and with `tiny` one
// that fits runs by a single workgroup.
static int plan_core(int nvars, int bits, int ring, const std::vector<SegInput> &in, const uint64_t *stats,
                     const uint32_t *flags, const Tuning &tune_in, Plan &P, int cus, uint64_t smask, bool counted,
                     GpProbe *probe, bool tiny = false) {
    const int S = (int)in.size();
    P = Plan();
    P.nseg = S;
    P.nvars = nvars;
    P.bits = bits;
    P.ring = ring;
    const uint64_t fmask = bits == 64 ? ~0ull : ((1ull << bits) - 1);

    // validation verdicts, most fundamental first
    uint32_t all = 0;
    for (int q = 0; q < S; q++) all |= flags[2 * q] | flags[2 * q + 1];
    if (all & ST_BADBITS) return PM_EINVAL;
    if (all & ST_UNSORTED) return PM_EUNSORTED;
    if (all & ST_RANGE) return PM_ERANGE;

    P.segs.resize(S);
    P.vars.resize((size_t)S * nvars);
    P.bound.assign(S, 0);
    std::vector<unsigned __int128> box(S, 0);
    int max_bits = 0;
    bool need_u64 = false;
    for (int q = 0; q < S; q++) {
        DevSeg &d = P.segs[q];
        d = DevSeg();
        d.fk = in[q].fk;
        d.fc = in[q].fc;
        d.gk = in[q].gk;
        d.gc = in[q].gc;
        d.na = in[q].na;
        d.nb = in[q].nb;
        d.var_off = (int64_t)q * nvars;
        if (d.na == 0 || d.nb == 0) {
            d.mode = SEG_EMPTY;
            continue;
        }
        const uint64_t *st = stats + (size_t)q * 4 * nvars;  // f: min[nv] max[nv], g: min[nv] max[nv]
        uint64_t fmin[MAX_VARS], gmin[MAX_VARS];
        const uint64_t *fmax = st + nvars, *gmax = st + 3 * nvars;
        for (int v = 0; v < nvars; v++) {
            fmin[v] = st[v] & smask;
            gmin[v] = st[2 * nvars + v] & smask;
        }
        unsigned __int128 b = 1;
        bool big = false;
        uint64_t lo_key = 0;
        for (int v = 0; v < nvars; v++) {
            if (fmax[v] > fmask - gmax[v]) return PM_EOVERFLOW;
            unsigned __int128 r = (unsigned __int128)(fmax[v] + gmax[v]) - (fmin[v] + gmin[v]) + 1;
            VarParam &vp = P.vars[(size_t)q * nvars + v];
            vp.shift = (uint32_t)((nvars - 1 - v) * bits);
            vp.mask = fmask;
            vp.minf = fmin[v];
            vp.ming = gmin[v];
            vp.range = (uint64_t)r;  // 0 encodes 2^64 (one full-width variable)
            if (r <= 0xFFFFFFFFull) vp.rdiv = make_div32((uint32_t)r);
            lo_key += (fmin[v] + gmin[v]) << vp.shift;
            if (!big) {
                b *= r;
                if (b >> 64) big = true;
            }
        }
        // strides: stride_v = prod_{w > v} range_w
        unsigned __int128 st_acc = 1;
        for (int v = nvars - 1; v >= 0; v--) {
            VarParam &vp = P.vars[(size_t)q * nvars + v];
            vp.stride = (uint64_t)st_acc;
            unsigned __int128 r = vp.range ? vp.range : ((unsigned __int128)1 << 64);
            st_acc *= r;
            if (st_acc >> 65) st_acc = (unsigned __int128)1 << 65;  // only reached when box > 2^64
        }
        d.lo_key = lo_key;
        box[q] = big ? ((unsigned __int128)1 << 64) : b;
        const unsigned __int128 prod = (unsigned __int128)d.na * (unsigned __int128)d.nb;
        const unsigned __int128 bnd = std::min(prod, box[q]);
        P.bound[q] = (int64_t)bnd;
        // path
        // the degree box when it is small against the pairs, and also for a
        // product that no sparse path can take (their staged items address
        // pairs with 32 bits)
        const bool sparse_too_big = prod > (unsigned __int128)0xFFFFFFFFull;
        const bool can_dense = tune_in.allow_dense && ring != RING_F64 && box[q] <= (unsigned __int128)tune_in.dense_max_cells &&
                               ((double)box[q] * tune_in.dense_ratio <= (double)prod || sparse_too_big);
        if (can_dense) {
            d.mode = SEG_DENSE;
        } else {
            d.mode = SEG_RAW;  // decided for the whole launch below
        }
    }

    // automatic settings: the autotuner's choice for the largest product's class
    Tuning tune = tune_in;
    bool over_auto = false;
    {
        int big = -1;
        unsigned __int128 bigp = 0;
        for (int q = 0; q < S; q++) {
            const unsigned __int128 pr = (unsigned __int128)P.segs[q].na * P.segs[q].nb;
            if (P.segs[q].mode != SEG_EMPTY && pr > bigp) {
                bigp = pr;
                big = q;
            }
        }
        if (big >= 0) {
            P.cls = TuneClass{ring, P.segs[big].mode == SEG_DENSE ? 1 : 0, log2_floor((uint64_t)bigp)};
            TuneChoice c;
            if (tune_in.remembered && tune_lookup(P.cls, c)) {
                if (tune.tile_cfg < 0) tune.tile_cfg = c.tile_cfg;
                if (tune.combine < 0 && !P.cls.dense) tune.combine = c.combine;  // (a box's choice times no sparse mode)
                if (tune.digits < 0) tune.digits = c.digits;
                over_auto = c.over_auto;
            }
        }
    }

    // prefix groups, where an explicit setting does not ask for another path
    std::vector<GpTry> gt(S);
    double all_pairs = 0;
    for (int q = 0; q < S; q++) all_pairs += (double)P.segs[q].na * (double)P.segs[q].nb;
    for (int q = 0; q < S; q++) {
        DevSeg &d = P.segs[q];
        const bool dense = d.mode == SEG_DENSE;
        if (d.mode == SEG_EMPTY) continue;
        // an explicit tile shape or sparse mode is what runs; a remembered one
        // leaves these paths alone unless it was timed against them
        if (dense ? tune_in.tile_cfg >= 0 : tune_in.combine != -1) continue;
        if (over_auto && (dense ? 1 : 0) == P.cls.dense && log2_floor((uint64_t)d.na * (uint64_t)d.nb) == P.cls.log2pairs) continue;
        if (tiny && tiny_fits(d.na, d.nb, box[q])) {
            d.mode = SEG_TINY;
            continue;
        }
        if ((double)d.na * (double)d.nb < GP_MIN_PAIRS) continue;
        // compute units that the product's share of the launch keeps busy (work
        // items as for the whole chip each made a burst of 14 products of 0.2 to
        // 4 million pairs spend 780 us in their reductions)
        const double share = std::max(1.0, cus * ((double)d.na * (double)d.nb / all_pairs));
        for (int way = 1; way <= 2 && !gt[q].ok; way++) {
            GpTry t = gp_try(nvars, &P.vars[(size_t)q * nvars], d.na, d.nb, box[q], dense, share, way, ring == RING_F64);
            if (!t.ok) continue;
            if (probe) probe->bytes[q] = std::max(probe->bytes[q], t.bytes);
            if (!counted || (probe && probe->pays)) continue;
            const uint64_t *st = stats + (size_t)q * 4 * nvars;
            const double gf = (double)(st[t.g.d - 1] >> 32), gg = (double)(st[2 * nvars + t.g.d - 1] >> 32);
            const double pairs = (double)d.na * (double)d.nb;
            // prefixes within the operands' ranges, which their groups are some of
            double cf = 1, cg = 1;
            for (uint32_t v = 0; v < t.g.d; v++) {
                cf *= (double)(st[nvars + v] - (st[v] & smask)) + 1;
                cg *= (double)(st[3 * nvars + v] - (st[2 * nvars + v] & smask)) + 1;
            }
            const double fill = gg < gf ? gf / cf : gg / cg;  // share of them that the inner operand has
            // pairs that an outer group has with the bins of a work item, if the inner operand has all of them
            const double bins = dense ? (double)t.g.nbins / (double)t.items
                                      : std::max(1.0, std::min<double>(t.g.span_bins, (double)t.g.nbins * t.g.T / pairs));
            const double met = pairs / (gf * gg) * bins;
            // (blocks of a pair or two take 8 times as long as a term each: 10002 by
            // 10002 of 100000 exponents 4422 us, 376; small blocks far apart twice as
            // long as listed: 3917 x 7693 terms in 1600 clusters 1244 us, 631)
            const bool single = dense && t.g.S == 1 && met * fill < 40;  // one term to a prefix, few prefixes to a work item
            if (gf >= 1 && gg >= 1 && (met < 32 || ((dense || pairs < 16 * gf * gg) && met * fill < 16) || single)) {
                if (dense) t.g.rows = 1;
                else if (ring != RING_F64) gp_list(t, pairs, box[q], share);
            }
            if (single) {
                // The wider bins of way 2 take half of the time where there are
                // enough of them (100 x 100 exponents squared 857 us, 329; a
                // tenth of 300 x 300 426, 170).  Else, terms side by side in full
                // lattices make a wave's lanes meet in the same cells, and the
                // tile kernel takes 0.7 of the time (20000 by 20000 terms in one
                // variable 2803 us, 2362; half of 20 x 2000 exponents squared
                // 1118, 2472).
                const GpTry w = gp_try(nvars, &P.vars[(size_t)q * nvars], d.na, d.nb, box[q], dense, share, 2, false);
                if ((w.ok && w.g.S > 1 && w.g.nbins >= share / 2) || (gf > 0.6 * cf && gg > 0.6 * cg)) continue;
            }
            // so few bins leave compute units idle (39 bins: 1368 us, by tiles 411; 199 bins: 329, 570)
            if (dense && way == 2 && t.g.nbins < share / 2) continue;
            if (!gp_pays(t, gf, gg, d.na, d.nb, box[q], dense, way, ring == RING_F64)) continue;
            if (probe) {
                probe->pays = true;
            } else {
                gt[q] = t;
                gt[q].g.swap = gg < gf ? 1 : 0;
                if (ring == RING_F64) {
                    gt[q].g.swap = 0;  // row-major sums: f's groups are the rows
                    P.gp_fc = std::max(P.gp_fc, t.g.S <= 1024 ? 1024 : t.g.S <= 2048 ? 2048 : GP_F64_CELLS);
                }
                d.mode = dense ? SEG_GRPD : SEG_GRP;
            }
        }
    }
    for (int q = 0; q < S; q++) {
        const int m = P.segs[q].mode;
        if (m == SEG_EMPTY || m == SEG_GRP || m == SEG_GRPD || m == SEG_TINY) continue;
        if (m == SEG_RAW) max_bits = std::max(max_bits, bitlen128(box[q] - 1));
        if (box[q] > (unsigned __int128)0xFFFFFFFFull) need_u64 = true;
    }
    P.ksize = need_u64 ? 8 : 4;
    P.passes = (max_bits + RADIX_BITS - 1) / RADIX_BITS;
    P.max_bits = max_bits;

    // one sort mode per launch: pair indices (products regenerated in the
    // reduction, FP64 summed in row-major order) or LDS-combined coefficients
    // (exact rings only; needs a free hash sentinel, i.e. box < 2^(8*ksize)).
    bool idx_fits = true, sentinel_ok = true;
    for (int q = 0; q < S; q++) {
        if (P.segs[q].mode != SEG_RAW) continue;
        if ((unsigned __int128)P.segs[q].na * P.segs[q].nb > 0xFFFFFFFFull) idx_fits = false;
        if (box[q] >= ((unsigned __int128)1 << 64)) sentinel_ok = false;
    }
    // output-key intervals: 32-bit compressed keys and 32-bit pair indices
    if (P.ksize == 4 && idx_fits && tune.combine == 2) {
        for (int q = 0; q < S; q++) {
            if (P.segs[q].mode != SEG_RAW) continue;
            DevSeg &d = P.segs[q];
            d.mode = SEG_IVAL;
            const double target = std::max(1.0, (double)d.na * (double)d.nb / 32768.0);
            int64_t l = (int64_t)std::ceil(std::sqrt(target)) - 1;
            l = std::max<int64_t>(0, std::min<int64_t>(l, 63));
            l = std::min<int64_t>(l, std::min(d.na, d.nb));
            d.iv_l = l;
        }
    }
    // output-key work items: products with 32-bit compressed keys and pair
    // indices whose single monomials can never hold more than BK_CAP pairs
    // (at most min(na, nb) pairs share a monomial)
    // (automatic for the exact rings; FP64 sorts each work item by row and key
    // in LDS, slower than the pair-index sort, so only on request)
    if (P.ksize == 4 && (tune.combine == 3 || (tune.combine == -1 && ring != RING_F64))) {
        for (int q = 0; q < S; q++) {
            DevSeg &d = P.segs[q];
            if (d.mode != SEG_RAW) continue;
            if ((unsigned __int128)d.na * d.nb > 0xFFFFFFFFull || std::min(d.na, d.nb) > BK_CAP) continue;
            d.mode = SEG_BKT;
        }
        idx_fits = true;
        sentinel_ok = true;
        for (int q = 0; q < S; q++) {
            if (P.segs[q].mode != SEG_RAW) continue;
            if ((unsigned __int128)P.segs[q].na * P.segs[q].nb > 0xFFFFFFFFull) idx_fits = false;
            if (box[q] >= ((unsigned __int128)1 << 64)) sentinel_ok = false;
        }
    }
    bool combine = ring != RING_F64 && sentinel_ok && (tune.combine == 1 || !idx_fits);
    if (!combine && !idx_fits) return PM_ENOMEM;  // FP64 product of more than 2^32 - 1 term pairs
    P.raw = combine ? 0 : 1;
    P.vsize = combine ? 8 : 4;
    for (int q = 0; q < S; q++)
        if (P.segs[q].mode == SEG_RAW && combine) P.segs[q].mode = SEG_COMBINE;
    // the combine path stages at most one item per term pair and addresses a
    // product's staging slots and sort partitions with 32-bit positions
    for (int q = 0; q < S; q++)
        if (P.segs[q].mode == SEG_COMBINE && (unsigned __int128)P.segs[q].na * P.segs[q].nb > 0xFFFFFFFFull)
            return PM_ENOMEM;
    bool any_sparse = false;
    for (int q = 0; q < S; q++) any_sparse |= P.segs[q].mode == SEG_RAW || P.segs[q].mode == SEG_COMBINE;
    if (!any_sparse) P.passes = 0;
    if (P.raw && any_sparse && P.passes == 0) P.passes = 1;  // pass 0 also generates the items
    set_digits(P, tune.digits == RADIX_DIGITS_GREEDY ? RADIX_DIGITS_GREEDY : RADIX_DIGITS_BALANCED);

    // tile shape: explicit, or the largest one that still gives >= 512 tiles
    // over the tiled products (at least two per compute unit); the sparse
    // combine path keeps the smallest table load (32 x 64 into 4096 slots).
    int64_t tiled_pairs = 0;
    bool any_combine = false;
    for (int q = 0; q < S; q++) {
        const DevSeg &d = P.segs[q];
        if (d.mode == SEG_COMBINE || d.mode == SEG_DENSE) tiled_pairs += d.na * d.nb;
        if (d.mode == SEG_COMBINE) any_combine = true;
    }
    if (tune.tile_cfg >= 0 && tune.tile_cfg < N_TILE_CFGS && (!any_combine || tile_cfg_combines(tune.tile_cfg))) {
        P.tile_cfg = tune.tile_cfg;
    } else if (any_combine) {
        P.tile_cfg = 0;
    } else {
        // a degree box with few pairs per cell (under 16) gives tiles with few
        // like terms: a tile of more pairs than table slots would overflow
        // its table into global atomics, so the shape stays at 64 x 64
        int top = N_TILE_CFGS - 1;
        for (int q = 0; q < S; q++) {
            const DevSeg &d = P.segs[q];
            if (d.mode == SEG_DENSE && (unsigned __int128)d.na * d.nb < 16 * box[q]) top = std::min(top, 1);
        }
        P.tile_cfg = 0;
        for (int c = top; c >= 0; c--) {
            if (tiled_pairs / ((int64_t)TILE_CFGS[c].tm * TILE_CFGS[c].tn) >= 512) {
                P.tile_cfg = c;
                break;
            }
        }
    }
    const TileCfg tc = TILE_CFGS[P.tile_cfg];

    // queues and offsets
    P.tile_pre.push_back(0);
    P.dpart_pre.push_back(0);
    P.cpre.push_back(0);
    int64_t nstage = 0, nbox = 0, nck = 0;
    bool split = false;
    for (int q = 0; q < S; q++) {
        DevSeg &d = P.segs[q];
        if (d.mode == SEG_EMPTY) P.nempty++;
        const bool grp = d.mode == SEG_GRP || d.mode == SEG_GRPD;
        const bool own = grp || d.mode == SEG_TINY;  // compresses its operands itself
        d.ck_f = nck;
        nck += own ? 0 : d.na;
        d.ck_g = nck;
        nck += own ? 0 : d.nb;
        P.cpre.push_back(P.cpre.back() + (own ? 0 : d.na));
        P.cpre.push_back(P.cpre.back() + (own ? 0 : d.nb));
        if (d.mode == SEG_TINY) {
            d.nb_div = make_div32((uint32_t)d.nb);
            d.bk_fs = bitlen128(box[q] - 1);
            P.ntiny++;
        }
        if (grp) {
            const GpTry &t = gt[q];
            d.gp = t.g;
            d.gp.bq = (uint32_t)P.ngp++;
            if (P.gp_sb_pre.empty()) P.gp_sb_pre.push_back(0);
            d.gp.tf = P.gp_nterm;
            d.gp.tg = P.gp_nterm + d.na;
            P.gp_nterm += d.na + d.nb;
            d.gp.lut = P.gp_nlut;
            P.gp_nlut += (int64_t)t.g.nbins + 1;
            d.gp.hist = P.gp_nsb * GP_SB;
            d.gp.sb_first = P.gp_nsb;
            P.gp_nsb += t.g.nsb;
            P.gp_ibound += t.ibound;
            P.gp_nres += t.nres;
            P.gp_maxbins = std::max<int64_t>(P.gp_maxbins, t.g.nbins);
            P.gp_maxunits = std::max<int64_t>(P.gp_maxunits, std::min(d.na, d.nb) * ((std::max(d.na, d.nb) + GP_LUT_I - 1) / GP_LUT_I));
            d.nb_div = make_div32(t.g.S);
            P.gp_seg.push_back(q);
            P.gp_sb_pre.push_back(P.gp_nsb);
            split |= std::max(d.na, d.nb) > GP_SPLIT;
            if (d.mode == SEG_GRPD) {
                P.ngp_box++;
                P.gp_dpairs += (double)d.na * (double)d.nb;
            } else {
                P.ngp_sparse++;
                if (t.g.rows) P.ngp_list++;
            }
        }
        if (d.mode == SEG_COMBINE || d.mode == SEG_DENSE) {
            const int64_t tmn = (d.na + tc.tm - 1) / tc.tm, tnn = (d.nb + tc.tn - 1) / tc.tn;
            d.tile_first = P.tile_pre.back();
            d.tiles_n = tnn;
            P.tile_seg.push_back(q);
            P.tile_pre.push_back(P.tile_pre.back() + tmn * tnn);
        }
        if (d.mode == SEG_RAW) d.nb_div = make_div32((uint32_t)d.nb);
        if (d.mode == SEG_IVAL) {
            d.nb_div = make_div32((uint32_t)d.nb);
            d.stage_base = nstage;
            d.stage_bound = d.na * d.nb;
            nstage += (d.stage_bound + 63) & ~(int64_t)63;
            d.iv_samp_off = P.iv_nsamp;
            P.iv_nsamp += (d.iv_l + 1) * (d.iv_l + 1);
            d.iv_spl_off = P.iv_nspl;
            P.iv_nspl += (d.iv_l + 1) * (d.iv_l + 1) + 2;
            if (P.iv_pre.empty()) P.iv_pre.push_back(0);
            P.iv_seg.push_back(q);
            P.iv_pre.push_back(P.iv_pre.back() + (d.iv_l + 1) * (d.iv_l + 1) + 1);
            P.iv_maxrows = std::max<int64_t>(P.iv_maxrows, d.na);
            P.nival++;
        }
        if (d.mode == SEG_COMBINE || d.mode == SEG_RAW) {
            d.stage_base = nstage;
            d.stage_bound = d.na * d.nb;
            nstage += (d.stage_bound + 63) & ~(int64_t)63;  // products start on 64-item boundaries
            P.nparts_bound += (d.stage_bound + PART - 1) / PART;
            P.nsparse++;
        }
        if (d.mode == SEG_BKT) {
            // fine bins of about BK_BIN_PAIRS pairs each (at least one super-bin)
            const uint64_t pairs = (uint64_t)d.na * (uint64_t)d.nb;
            const uint64_t target = std::max<uint64_t>(BK_SB, pairs / BK_BIN_PAIRS);
            const uint64_t cells = (uint64_t)box[q];
            int fs = 0;
            while (((cells + (1ull << fs) - 1) >> fs) > target) fs++;
            const int64_t nbins = (int64_t)((cells + (1ull << fs) - 1) >> fs);
            const int64_t nsb = (nbins + BK_SB - 1) / BK_SB;
            d.bk_fs = fs;
            // exact rings: work items span at most 2^BK_RANK_LOG keys, so each
            // one is summed by rank in LDS without a sort
            d.bk_span_bins = (ring != RING_F64 && fs <= BK_RANK_LOG) ? (1 << (BK_RANK_LOG - fs)) : 0;
            d.bk_bin_off = P.bk_nbins;
            d.bk_sb_first = P.bk_nsb;
            d.bk_nsb = nsb;
            P.bk_nbins += nsb * BK_SB;
            P.bk_nsb += nsb;
            // generation tiles: up to BK_TN_MAX columns (a power of two), BK_TILE slots
            int tnl = 0;
            while ((1ll << tnl) < d.nb && (1 << tnl) < BK_TN_MAX) tnl++;
            d.bk_tnl = tnl;
            const int64_t tm = BK_TILE >> tnl, tn = 1ll << tnl;
            d.bk_tiles_n = (d.nb + tn - 1) / tn;
            d.bk_tile_first = P.bk_ntiles;
            if (P.bk_tile_pre.empty()) P.bk_tile_pre.push_back(0), P.bk_sb_pre.push_back(0);
            P.bk_ntiles += ((d.na + tm - 1) / tm) * d.bk_tiles_n;
            P.bk_tile_pre.push_back(P.bk_ntiles);
            P.bk_sb_pre.push_back(P.bk_nsb);
            P.bk_seg.push_back(q);
            // two consecutive work items of a super-bin hold more than BK_CAP
            // pairs, so a super-bin of p pairs has at most 2 ceil(p / BK_CAP) + 1
            // (or the first spans bk_span_bins bins)
            const int64_t span_items = d.bk_span_bins ? 2 * nsb * ((BK_SB + d.bk_span_bins - 1) / d.bk_span_bins) : 0;
            P.bk_wi_bound += 2 * (int64_t)((pairs + BK_CAP - 1) / BK_CAP) + 3 * nsb + 1 + span_items;
            P.bk_nstage += (int64_t)pairs;
            // a work item over BK_CAP pairs is one fine bin: at most 2^fs result terms
            const uint64_t fat_items = pairs / (BK_CAP + 1);
            P.bk_fat_cap += (int64_t)std::min<uint64_t>(pairs, fat_items << fs);
            d.nb_div = make_div32((uint32_t)d.nb);
            P.nbk++;
        }
        if (probe) {
            const int64_t pairs = d.na * d.nb;
            int64_t &b = probe->old_bytes[q];
            if (d.mode == SEG_BKT) b = 4 * (d.na + d.nb) + 12 * pairs + 6 * d.bk_nsb * BK_SB;
            if (d.mode == SEG_RAW || d.mode == SEG_COMBINE) b = 2 * (int64_t)(P.ksize + P.vsize) * pairs;
        }
        if (d.mode == SEG_DENSE || d.mode == SEG_GRPD) {
            d.stage_base = nbox;
            d.stage_bound = (int64_t)box[q];
            nbox += d.stage_bound;
            if (d.mode == SEG_GRPD) continue;
            d.dpart_first = P.dpart_pre.back();
            P.dseg.push_back(q);
            P.dpart_pre.push_back(P.dpart_pre.back() + (d.stage_bound + PART - 1) / PART);
            P.ndense++;
        }
    }
    if (split) {
        P.gp_pt_pre.push_back(0);
        for (int32_t q : P.gp_seg)
            for (int64_t n : {P.segs[q].na, P.segs[q].nb}) P.gp_pt_pre.push_back(P.gp_pt_pre.back() + (n + GP_PART - 1) / GP_PART);
    }
    P.ntiles = P.tile_pre.back();
    P.ndparts = P.dpart_pre.back();
    P.nstage = nstage;
    if (P.iv_pre.empty()) P.iv_pre.push_back(0);
    P.iv_items = P.iv_pre.back();
    P.iv_grid = (int)std::max<int64_t>(1, std::min<int64_t>(P.iv_items, (int64_t)cus * 2));
    P.nbox = nbox;
    P.nck = nck;
    // digit counts of pair-index sorts regenerate keys from an LDS copy of
    // the product's compressed operand keys, up to 64 KB (two workgroups per
    // CU); larger products read them from global memory
    // Pair-index sorts regenerate each key from the operands' compressed keys
    // while those stay cache resident (gathers that hit in L2) and every
    // product's keys fit the digit count's LDS copy; otherwise (over 1 MB of
    // them in one launch, as in large batches, or a product with more than
    // 64 KB of them) the generating pass writes the keys and later passes
    // carry them.
    P.ck_fit = 1;
    P.ck_lds = 0;
    for (int q = 0; q < S; q++) {
        const int64_t m = P.segs[q].na + P.segs[q].nb;
        if (P.segs[q].mode != SEG_RAW) continue;
        if (m * P.ksize <= (64 << 10)) P.ck_lds = std::max<int64_t>(P.ck_lds, m);
        else P.ck_fit = 0;
    }
    if (!P.ck_fit) P.ck_lds = 0;
    P.ix = P.ck_fit && (int64_t)nck * P.ksize <= (int64_t)1 << 20;

    // workspace layout
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    P.r_stats.off = take(stats_bytes(S, nvars));
    P.r_stats.bytes = stats_bytes(S, nvars);
    P.r_flags.off = take((size_t)S * 2 * 4);
    P.r_flags.bytes = (size_t)S * 2 * 4;
    // descriptors side by side: the block of a few products fits a kernel's arguments
    auto small = [&](size_t bytes) {
        size_t o = off;
        off = (off + bytes + 15) & ~(size_t)15;
        return o;
    };
    const size_t desc0 = off;
    P.o_segs = small(sizeof(DevSeg) * S);
    P.o_vars = small(sizeof(VarParam) * S * nvars);
    P.o_tile_pre = small(8 * P.tile_pre.size());
    P.o_tile_seg = small(4 * std::max<size_t>(1, P.tile_seg.size()));
    P.o_dpart_pre = small(8 * P.dpart_pre.size());
    P.o_dseg = small(4 * std::max<size_t>(1, P.dseg.size()));
    P.o_cpre = small(8 * P.cpre.size());
    P.o_iv_pre = small(8 * P.iv_pre.size());
    P.o_iv_seg = small(4 * std::max<size_t>(1, P.iv_seg.size()));
    P.o_bk_tile_pre = small(8 * std::max<size_t>(1, P.bk_tile_pre.size()));
    P.o_bk_seg = small(4 * std::max<size_t>(1, P.bk_seg.size()));
    P.o_bk_sb_pre = small(8 * std::max<size_t>(1, P.bk_sb_pre.size()));
    if (P.ngp) {
        P.o_gp_seg = small(4 * P.gp_seg.size());
        P.o_gp_sb_pre = small(8 * P.gp_sb_pre.size());
        P.o_gp_pt_pre = small(8 * P.gp_pt_pre.size());
    }
    off = align256(off);
    P.r_desc.off = desc0;
    P.r_desc.bytes = off - desc0;
    const size_t zero0 = off;
    P.o_dyn = take(sizeof(DevSegDyn) * S);
    P.o_counters = take(4 * CNT_COUNT);
    P.o_look_red = take((size_t)8 * std::max<int64_t>(1, P.nparts_bound));
    P.o_look_cmp = take((size_t)8 * std::max<int64_t>(1, P.ndparts));
    P.o_look_tile = take((size_t)8 * std::max<int64_t>(1, P.ntiles));
    // (boxes of prefix-group products are stored whole and need no zeroing)
    const bool zero_box = P.ntiles > 0;
    if (zero_box) P.o_box = take((size_t)8 * std::max<int64_t>(1, nbox));
    if (P.ngp) {
        P.o_gp_hist = take((size_t)4 * GP_SB * std::max<int64_t>(1, P.gp_nsb));
        P.o_gp_look = take((size_t)16 * std::max<int64_t>(1, P.gp_nsb));
        P.o_gp_usum = take((size_t)4 * ((P.gp_ibound >> GP_USUM_LOG) + 1));
    }
    P.o_bk_hist = take((size_t)4 * std::max<int64_t>(1, P.bk_nbins));
    P.o_bk_fill = take((size_t)4 * std::max<int64_t>(1, P.bk_wi_bound));
    P.o_bk_fatfill = take(8);
    // sort blocks fill the radix passes' resident workgroups
    P.kl = P.raw && P.ix && os_keys_in_lds(P.ck_lds, P.ksize, P.vsize);
    const int64_t resident = (int64_t)cus * (P.kl ? 2 : os_resident(P.ksize, P.vsize));
    // A workgroup's pass time goes with the blocks it takes times pblk: when
    // some pblk up to PBLK_MAX makes one block per resident workgroup, take
    // the smallest; otherwise (many rounds, where the ticket queue balances
    // finer blocks better) blocks of at most 16 partitions.
    P.pblk = 0;
    for (int64_t pb = 1; pb <= PBLK_MAX && !P.pblk; pb++) {
        int64_t nb = 0;
        for (int q = 0; q < S; q++) {
            const DevSeg &d = P.segs[q];
            if (d.mode != SEG_RAW && d.mode != SEG_COMBINE) continue;
            nb += ((d.stage_bound + PART - 1) / PART + pb - 1) / pb;
        }
        if (nb <= resident) P.pblk = pb;
    }
    if (!P.pblk) P.pblk = std::max<int64_t>(1, std::min<int64_t>(16, (P.nparts_bound + resident - 1) / resident));
    // range counters of the radix passes, two sets by pass parity (zeroed here,
    // then each counting kernel clears the other set for the next pass)
    P.nrng = (P.nparts_bound / P.pblk + S + 1) / RNG + S + 1;
    P.rscan = 0;
    for (int q = 0; q < S; q++) {
        const DevSeg &d = P.segs[q];
        if (d.mode != SEG_RAW && d.mode != SEG_COMBINE) continue;
        const int64_t np = (d.stage_bound + PART - 1) / PART, nb = (np + P.pblk - 1) / P.pblk;
        if ((nb + RNG - 1) / RNG > RSUM_MAX) P.rscan = 1;
    }
    P.o_rtot = take((size_t)8 * RADIX * 2 * P.nrng);
    P.r_zero.off = zero0;
    P.r_zero.bytes = off - zero0;
    if (!zero_box) P.o_box = take((size_t)8 * std::max<int64_t>(1, nbox));
    if (P.ngp) {
        P.o_gp_pt_cnt = take((size_t)4 * (P.gp_pt_pre.empty() ? 0 : P.gp_pt_pre.back()));
        P.o_gp_term = take(sizeof(GpTerm) * (size_t)(P.gp_nterm + GP_PAD));
        P.o_gp_pfx = take((size_t)4 * P.gp_nterm);
        P.o_gp_start = take((size_t)4 * (P.gp_nterm + 2 * P.ngp));
        P.o_gp_ng = take((size_t)8 * P.ngp);
        P.o_gp_lut = take((size_t)4 * P.gp_nlut);
        P.o_gp_sbit = take((size_t)4 * (P.gp_nsb + 1));
        P.o_gp_item = take(sizeof(GpItem) * (size_t)std::max<int64_t>(1, P.gp_ibound));
        P.o_gp_u = take((size_t)4 * std::max<int64_t>(1, P.gp_ibound));
        P.o_gp_rkey = take((size_t)4 * std::max<int64_t>(1, P.gp_nres));
        P.o_gp_rcoef = take((size_t)8 * std::max<int64_t>(1, P.gp_nres));
    }
    P.o_ppre = take((size_t)8 * (S + 1));
    P.o_chpre = take((size_t)8 * (S + 1));
    P.o_rpre = take((size_t)8 * (S + 1));
    P.o_pbase = take((size_t)8 * RADIX * S);
    P.o_pcnt = take((size_t)8 * std::max<int64_t>(1, P.nparts_bound));
    P.o_ctot = take((size_t)8 * RADIX * (P.nparts_bound / P.pblk + S + 1));
    P.o_iv_samp = take((size_t)P.ksize * std::max<int64_t>(1, P.iv_nsamp));
    P.o_iv_spl = take((size_t)P.ksize * std::max<int64_t>(1, P.iv_nspl));
    P.o_iv_cur = take((size_t)4 * std::max<int64_t>(1, (int64_t)P.iv_grid * P.iv_maxrows));
    P.o_iv_items = take((size_t)16 * std::max<int64_t>(1, P.iv_items));
    P.o_iv_off = take((size_t)8 * std::max<int64_t>(1, P.iv_items));
    P.o_ck = take((size_t)P.ksize * std::max<int64_t>(1, nck));
    P.o_bk_wbin = take((size_t)2 * std::max<int64_t>(1, P.bk_nbins));
    P.o_bk_sbtot = take((size_t)4 * std::max<int64_t>(1, P.bk_nsb));
    P.o_bk_sbwi = take((size_t)4 * std::max<int64_t>(1, P.bk_nsb));
    P.o_bk_sbtb = take((size_t)4 * (P.bk_nsb + 1));
    P.o_bk_sbpre = take((size_t)8 * std::max<int64_t>(1, P.bk_nsb));
    P.o_bk_wi = take(sizeof(BkWi) * std::max<int64_t>(1, P.bk_wi_bound));
    P.o_bk_stage = take((size_t)8 * std::max<int64_t>(1, P.bk_nstage));
    P.o_bk_rkey = take((size_t)4 * std::max<int64_t>(1, P.bk_nstage));
    P.o_bk_tlist = take((size_t)8 * 512 * std::max<int64_t>(1, P.bk_ntiles));  // BK_TL bins per tile
    P.o_bk_tcnt = take((size_t)4 * std::max<int64_t>(1, P.bk_ntiles));
    P.o_bk_u = take((size_t)4 * std::max<int64_t>(1, P.bk_wi_bound));
    P.o_bk_opre = take((size_t)8 * std::max<int64_t>(1, P.bk_wi_bound));
    P.o_bk_fbase = take((size_t)8 * std::max<int64_t>(1, P.bk_wi_bound));
    P.o_bk_fatc = take((size_t)8 * std::max<int64_t>(1, P.bk_fat_cap));
    const int64_t nstageA = P.nival ? 1 : nstage;
    P.o_stAk = take((size_t)P.ksize * std::max<int64_t>(1, nstageA));
    P.o_stAv = take((size_t)P.vsize * std::max<int64_t>(1, nstageA));
    P.o_stBk = take((size_t)P.ksize * std::max<int64_t>(1, nstage));
    P.o_stBv = take((size_t)(P.nival ? 8 : P.vsize) * std::max<int64_t>(1, nstage));
    P.total = off;
    return PM_OK;
}

int plan_build(int nvars, int bits, int ring, const std::vector<SegInput> &in, const uint64_t *stats,
               const uint32_t *flags, const Tuning &tune, Plan &P, int cus, bool counted, int64_t limit) {
    const size_t S = in.size();
    // with wider fields (one variable) a minimum takes the whole word
    counted = counted && bits <= 32;
    const uint64_t smask = counted ? 0xFFFFFFFFull : ~0ull;
    GpProbe probe;
    probe.old_bytes.assign(S, 0);
    probe.bytes.assign(S, 0);
    int rc = plan_core(nvars, bits, ring, in, stats, flags, tune, P, cus, smask, counted, &probe);
    if (rc) return rc;
    int64_t more = 0, any = 0;
    for (size_t q = 0; q < S; q++) {
        any += probe.bytes[q];
        more += std::max<int64_t>(0, probe.bytes[q] - probe.old_bytes[q]);
    }
    P.report = P.total + (any ? align256((size_t)more + 4096) : 0);
    const size_t report = P.report, general = P.total;
    // a product on its own only: a launch of several, some of them such, has
    // faulted the GPU once, for a reason not found
    const bool tiny = tune.tiny && S == 1 && P.segs[0].mode != SEG_EMPTY && tiny_fits(in[0].na, in[0].nb, 1);
    if (limit < (int64_t)general || !(probe.pays || tiny)) return PM_OK;
    Plan G;
    rc = plan_core(nvars, bits, ring, in, stats, flags, tune, G, cus, smask, counted, nullptr, tiny);
    if (rc || !(G.ngp || G.ntiny) || (int64_t)G.total > limit) return PM_OK;
    P = std::move(G);
    P.total = std::max(P.total, general);
    P.report = report;
    return PM_OK;
}

}  // namespace pm
