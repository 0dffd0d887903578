// Prefix groups (SEG_GRP, SEG_GRPD): products whose term pairs are generated
// where they are summed.  Included by pm_kernels.hip.
//
// The mixed-radix compressed key adds digit by digit without carries, so the
// key of a pair (i, j) splits at any variable boundary into a prefix (the
// leading gp.d variables, value P_i + P_j) and a low part (below S, the number
// of cells of the remaining variables).  Sorted operands are runs of terms of
// equal prefix ("groups"), and the pairs of output prefix b are exactly the
// blocks (group of prefix p) x (group of prefix b - p).  One workgroup owns a
// range of consecutive output prefixes ("bins") and forms all of its pairs
// itself, from contiguous pieces of both operands, in LDS cells: no pair is
// staged in memory, counted or scattered one by one.  This is Algorithm 1's
// output interval with FindEdge done once per group instead of once per row.
//   k_gp_heads   groups per part of the operands, where some operand is large
//   k_gp_prep    compressed terms, group lists, zeroing of the per-call state
//   k_gp_lut     first inner term of every prefix; SEG_GRP: pairs per bin, one
//                addition per pair of groups
//   k_gp_coarse  SEG_GRPD: pairs per run of gp.K bins
//   k_gp_cut     bins to work items of about gp.T pairs
//   k_gp_reduce  work items summed in LDS: sparse results to staging
//                (SEG_GRP), degree-box cells stored directly (SEG_GRPD)
//   k_gp_list    the same for products of small blocks, whose pairs are listed
//                in LDS first
//   k_gp_copy    result offsets, keys decompressed, terms to h
#pragma once

namespace pm {

constexpr int GPP_T = 1024;  // threads of k_gp_prep (four terms each per step)

typedef u32 u32x3 __attribute__((ext_vector_type(3)));

struct GpOperand {
    const GpTerm *t;
    const u32 *pfx, *start;
    u32 n, groups;
};

__device__ inline GpOperand gp_operand(const Ctx &C, const DevSeg &s, int bq, int side) {
    GpOperand o;
    const i64 off = uniform64(side ? s.gp.tg : s.gp.tf);
    o.t = C.gp_term + off;
    o.pfx = C.gp_pfx + off;
    o.start = C.gp_start + off + 2 * bq + side;  // one more entry than terms per operand
    o.n = uniform32((u32)(side ? s.nb : s.na));
    o.groups = uniform32(C.gp_ng[2 * bq + side]);
    return o;
}

// Part x of the operands' parts (gp_pt_pre, or one part per operand): the
// operand's index and its terms [b0, b1).
struct GpPart {
    int op;
    i64 b0, b1;
};
__device__ inline GpPart gp_part(const Ctx &C, bool split, int x) {
    GpPart p;
    p.op = split ? seg_search(C.gp_pt_pre, 2 * C.ngp, (i64)x) : x;
    const DevSeg &s = C.segs[C.gp_seg[p.op >> 1]];
    const i64 n = (p.op & 1) ? s.nb : s.na;
    p.b0 = split ? (x - C.gp_pt_pre[p.op]) * GP_PART : 0;
    p.b1 = split ? min(n, p.b0 + GP_PART) : n;
    return p;
}

// Groups that start in every part, where an operand has several.  (One
// workgroup alone takes 1.2 ms for a million terms, most of it latency.)
__global__ __launch_bounds__(GPP_T) void k_gp_heads(Ctx C) {
    __shared__ u32 s_sum[GPP_T / 64];
    const GpPart pt = gp_part(C, true, blockIdx.x);
    const DevSeg &s = C.segs[C.gp_seg[pt.op >> 1]];
    const u64 *key = (pt.op & 1) ? s.gk : s.fk;
    const u32 psh = C.vars[s.var_off + s.gp.d - 1].shift;
    u64 k[GP_PART / GPP_T], prev[GP_PART / GPP_T];
#pragma unroll
    for (int e = 0; e < GP_PART / GPP_T; e++) {
        const i64 i = min(pt.b0 + e * GPP_T + threadIdx.x, pt.b1 - 1);
        k[e] = key[i];
        prev[e] = key[max(i - 1, (i64)0)];
    }
    u32 hd = 0;
#pragma unroll
    for (int e = 0; e < GP_PART / GPP_T; e++) {
        const i64 i = pt.b0 + e * GPP_T + threadIdx.x;
        if (i < pt.b1 && (i == 0 || ((k[e] ^ prev[e]) >> psh) != 0)) hd++;
    }
    u32 tot;
    (void)block_excl_scan<u32, GPP_T>(hd, s_sum, tot);
    if (threadIdx.x == 0) C.gp_pt_cnt[blockIdx.x] = tot;
}

// Workgroups [0, nop): one part of an operand each (split: of several, whose
// group counts k_gp_heads has left).  The others clear [zp, zp + zn).
__global__ __launch_bounds__(GPP_T) void k_gp_prep(Ctx C, int nop, bool split, u64 *zp, i64 zn) {
    if ((int)blockIdx.x >= nop) {
        for (i64 i = (i64)(blockIdx.x - nop) * GPP_T + threadIdx.x; i < zn; i += (i64)(gridDim.x - nop) * GPP_T)
            zp[i] = 0;
        return;
    }
    __shared__ u32 s_hi[MAX_VARS], s_lo[MAX_VARS], s_sh[MAX_VARS];
    __shared__ u64 s_mn[MAX_VARS];
    __shared__ u32 s_scan[GPP_T / 64];
    const GpPart pt = gp_part(C, split, blockIdx.x);
    const int bq = pt.op >> 1, side = pt.op & 1;
    const DevSeg &s = C.segs[C.gp_seg[bq]];
    const int nv = C.nvars, d = (int)s.gp.d;
    const VarParam *vp = C.vars + s.var_off;
    for (int v = threadIdx.x; v < nv; v += GPP_T) {
        s_hi[v] = v < d ? (u32)(vp[v].stride / s.gp.S) : 0;
        s_lo[v] = v < d ? 0 : (u32)vp[v].stride;
        s_sh[v] = vp[v].shift;
        s_mn[v] = side ? vp[v].ming : vp[v].minf;
    }
    __syncthreads();
    const u64 mask = vp[0].mask;
    const u64 *key = side ? s.gk : s.fk, *coef = side ? s.gc : s.fc;
    const i64 n = side ? s.nb : s.na;
    const i64 off = side ? s.gp.tg : s.gp.tf;
    GpTerm *out = C.gp_term + off;
    u32 *pfx = C.gp_pfx + off, *start = C.gp_start + off + 2 * bq + side;
    const u32 S = s.gp.S, psh = s_sh[d - 1];
    // coefficient words: 31 and 30 bits mod p, else 32 and 32
    const u32 csh = C.ring == RING_MODP ? 31 : 32, cmask = C.ring == RING_MODP ? 0x7FFFFFFFu : ~0u;
    u32 ng = 0;
    if (split) {  // groups of the operand's earlier parts
        u32 x = 0;
        for (i64 i = C.gp_pt_pre[pt.op] + threadIdx.x; i < (i64)blockIdx.x; i += GPP_T) x += C.gp_pt_cnt[i];
        (void)block_excl_scan<u32, GPP_T>(x, s_scan, ng);
    }
    // the next step's terms are loaded before this one's are scanned
    u64 nk[4], nc[4], np = 0;
    auto load = [&](i64 i0) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const i64 i = min(i0 + e, n - 1);
            nk[e] = key[i];
            nc[e] = coef[i];
        }
        np = key[max(min(i0, n) - 1, (i64)0)];
    };
    load(pt.b0 + (i64)threadIdx.x * 4);
    for (i64 b = pt.b0; b < pt.b1; b += GPP_T * 4) {
        const i64 i0 = b + (i64)threadIdx.x * 4;
        u64 k[4], c[4], prev = np;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            k[e] = nk[e];
            c[e] = nc[e];
        }
        if (b + GPP_T * 4 < pt.b1) load(i0 + GPP_T * 4);
        u32 p[4], lo[4], hd = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            p[e] = lo[e] = 0;
            for (int v = 0; v < nv; v++) {
                const u32 x = (u32)(((k[e] >> s_sh[v]) & mask) - s_mn[v]);
                p[e] += x * s_hi[v];
                lo[e] += x * s_lo[v];
            }
            const i64 i = i0 + e;
            if (i < n && (i == 0 || ((k[e] ^ prev) >> psh) != 0)) hd |= 1u << e;
            prev = k[e];
        }
        u32 tot;
        u32 at = ng + block_excl_scan<u32, GPP_T>((u32)__popc(hd), s_scan, tot);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const i64 i = i0 + e;
            if (i < n) out[i] = GpTerm{(u32)c[e] & cmask, (u32)(c[e] >> csh), p[e] * S + lo[e], p[e]};
            if ((hd >> e) & 1u) {
                pfx[at] = p[e];
                start[at] = (u32)i;
                at++;
            }
        }
        ng += tot;
    }
    if (threadIdx.x == 0 && pt.b1 == n) {
        start[ng] = (u32)n;
        C.gp_ng[2 * bq + side] = ng;
    }
}
static_assert(GP_PART % (GPP_T * 4) == 0, "steps of a part");

// lut[b]: first inner term of prefix b or more (b up to and including nbins).
// SEG_GRP: pairs of every bin, each pair of groups adding its block's size.
__global__ __launch_bounds__(256) void k_gp_lut(Ctx C) {
    for (int bq = blockIdx.y; bq < C.ngp; bq += gridDim.y) {
        const DevSeg &s = C.segs[C.gp_seg[bq]];
        const int so = (int)uniform32(s.gp.swap);
        const GpOperand I = gp_operand(C, s, bq, 1 - so), O = gp_operand(C, s, bq, so);
        const u32 nbins = uniform32(s.gp.nbins);
        u32 *lut = C.gp_lut + uniform64(s.gp.lut);
        for (u32 b = blockIdx.x * 256 + threadIdx.x; b <= nbins; b += gridDim.x * 256) {
            u32 lo = 0, hi = I.groups;
            while (lo < hi) {
                const u32 mid = (lo + hi) >> 1;
                if (I.pfx[mid] < b) lo = mid + 1;
                else hi = mid;
            }
            lut[b] = I.start[lo];
        }
        if (s.mode != SEG_GRP) continue;
        u32 *hist = C.gp_hist + uniform64(s.gp.hist);
        // a wave takes one outer group and GP_LUT_I inner ones (with all of them,
        // one outer group by 160000 inner ones took 0.8 ms, one wave's latencies)
        const u32 nw = gridDim.x * 4, ni = (I.groups + GP_LUT_I - 1) / GP_LUT_I;
        const u64 nu = (u64)O.groups * ni;
        for (u64 x = (u64)uniform32(blockIdx.x * 4 + (threadIdx.x >> 6)); x < nu; x += nw) {
            const u32 o = (u32)(x / ni), i0 = (u32)(x - (u64)o * ni) * GP_LUT_I, i1 = min(i0 + GP_LUT_I, I.groups);
            const u32 p = O.pfx[o], r = O.start[o + 1] - O.start[o];
            for (u32 i = i0 + (threadIdx.x & 63); i < i1; i += 64)
                atomicAdd(&hist[p + I.pfx[i]], r * (I.start[i + 1] - I.start[i]));
        }
    }
}

// SEG_GRPD: pairs of every run of K bins (the bins of one value of the
// variables before the last prefix variable), enough to cut the work evenly.
// A wave takes 16 outer groups and 64 runs of the inner operand, adds up the
// rows of the groups in one run and meets its runs with them.
__global__ __launch_bounds__(256) void k_gp_coarse(Ctx C) {
    const u32 lane = threadIdx.x & 63, nw = gridDim.x * 4;
    for (int bq = blockIdx.y; bq < C.ngp; bq += gridDim.y) {
        const DevSeg &s = C.segs[C.gp_seg[bq]];
        if (s.mode != SEG_GRPD) continue;
        const GpOperand O = gp_operand(C, s, bq, (int)uniform32(s.gp.swap));
        const u32 K = uniform32(s.gp.K), nc = uniform32(s.gp.nbins) / K;
        const u32 *lut = C.gp_lut + uniform64(s.gp.lut);
        u32 *hist = C.gp_hist + uniform64(s.gp.hist);
        // pairs in units of 2^gp.csh, so that a count stays below 2^32
        const u32 csh = uniform32(s.gp.csh);
        const u32 nq = (nc + 63) / 64;
        for (u32 x = uniform32(blockIdx.x * 4 + (threadIdx.x >> 6)); x < (O.groups + 15) / 16 * nq; x += nw) {
            const u32 o = x / nq * 16 + lane, i = x % nq * 64 + lane;
            const bool in = lane < 16 && o < O.groups;
            u32 c = ~0u, r = 0, n = 0;
            if (in) {
                c = O.pfx[o] / K;
                r = O.start[o + 1] - O.start[o];
            }
            if (i < nc) n = lut[(i + 1) * K] - lut[i * K];
            u64 todo = __ballot(in);
            while (todo) {
                const u32 l = (u32)__ffsll((unsigned long long)todo) - 1;
                const u32 cc = (u32)__builtin_amdgcn_readlane((int)c, (int)l);
                const u64 same = __ballot(c == cc);
                todo &= ~same;
                u64 rows = 0;
                for (u64 m = same; m; m &= m - 1)
                    rows += (u32)__builtin_amdgcn_readlane((int)r, (int)__ffsll((unsigned long long)m) - 1);
                if (n && cc + i < nc) atomicAdd(&hist[cc + i], (u32)((rows * n + (1u << csh) - 1) >> csh));
            }
        }
    }
}

// ---------------------------------------------------------------------------
// k_gp_cut: one workgroup per super-bin of GP_SB bins, four bins per thread.
// A non-empty bin starts a work item when it is the super-bin's first, when
// the pairs before it cross a multiple of gp.T, when it enters another span of
// gp.span_bins bins (what the presence bitmap covers), or when it or the bin
// before it is dense enough to fill direct cells by itself.  Work items keep
// key order: their places and their staging offsets (at most min(pairs, S)
// results per bin) are prefix sums over the super-bins, by a look-back.
// SEG_GRPD: the counted bins are runs of K bins; a run is cut into work items
// of equal width to a bin, as many as its pairs ask for and its cells need
// (gp_run_items).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BC_T) void k_gp_cut(Ctx C) {
    __shared__ u32 s_pre[GP_SB + 1];
    __shared__ u32 s_scan[BC_T / 64];
    __shared__ u32 s_max[BC_T / 64];
    __shared__ u32 s_sb;
    __shared__ u64 s_ibase, s_mbase;
    if (threadIdx.x == 0) s_sb = atomicAdd(&C.counters[CNT_GP_CUT], 1u);
    __syncthreads();
    const i64 sb = (i64)uniform32(s_sb);
    const int bq = seg_search(C.gp_sb_pre, C.ngp, sb);
    const int q = C.gp_seg[bq];
    const DevSeg &s = C.segs[q];
    const u32 lsb = (u32)(sb - C.gp_sb_pre[bq]);
    const u32 t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint4 hv = *(const uint4 *)(C.gp_hist + s.gp.hist + (i64)lsb * GP_SB + 4 * t);
    const u32 h[4] = {hv.x, hv.y, hv.z, hv.w};
    const u32 S = s.gp.S, T = s.gp.T, span = s.gp.span_bins, heavy = s.gp.heavy;
    u32 tot, mtot;
    u32 run = block_excl_scan<u32, BC_T>(h[0] + h[1] + h[2] + h[3], s_scan, tot);
    u32 m[4], ms = 0;
    for (int k = 0; k < 4; k++) {
        s_pre[4 * t + k] = run;
        run += h[k];
        m[k] = s.gp.K ? 0u : min(h[k], S);
        ms += m[k];
    }
    if (t == BC_T - 1) s_pre[GP_SB] = tot;
    const u32 mpre = block_excl_scan<u32, BC_T>(ms, s_scan, mtot);
    if (w == 1) {  // staging offset of the super-bin
        const u64 pre = lookback_wave(C.gp_look + C.gp_nsb, 0, sb, 203u, mtot, &C.counters[CNT_ERR_SPIN]);
        if (lane == 0) s_mbase = pre;
    }
    // last non-empty bin (plus one) before this thread's
    u32 mine = 0;
    for (int k = 0; k < 4; k++)
        if (h[k]) mine = 4 * t + k + 1;
    u32 x = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const u32 y = __shfl_up(x, d, 64);
        if (lane >= (u32)d) x = max(x, y);
    }
    if (lane == 63) s_max[w] = x;
    __syncthreads();
    u32 pv = __shfl_up(x, 1, 64), all = 0;
    if (lane == 0) pv = 0;
    for (u32 i = 0; i < BC_T / 64; i++) {
        if (i < w) pv = max(pv, s_max[i]);
        all = max(all, s_max[i]);
    }
    const u32 pv0 = pv;
    u32 st = 0, np[4], nsum = 0;
    const u32 K = s.gp.K;
    for (int k = 0; k < 4; k++) {
        np[k] = 0;
        const u32 b = 4 * t + k;
        if (K && (u64)(lsb * GP_SB + b) * K < s.gp.nbins)
            np[k] = gp_run_items(K, S, h[k] / T + 1);
        if (K) nsum += np[k];
        if (K || !h[k]) continue;
        bool start = pv == 0;
        if (!start) {
            const u32 a = pv - 1, ha = s_pre[pv] - s_pre[a];
            start = s_pre[b] / T != s_pre[a] / T || b / span != a / span || h[k] >= heavy || ha >= heavy;
        }
        if (start) st |= 1u << k;
        pv = b + 1;
    }
    u32 ni;
    u32 it = block_excl_scan<u32, BC_T>((u32)__popc(st) + nsum, s_scan, ni);
    if (w == 0) {
        const u64 pre = lookback_wave(C.gp_look, 0, sb, 204u, ni, &C.counters[CNT_ERR_SPIN]);
        if (lane == 0) s_ibase = pre;
    }
    __syncthreads();
    u64 end = s_ibase + ni;
    if ((i64)end > C.gp_ibound) {  // never planned: keep every item inside the arrays
        if (t == 0) atomicOr(&C.counters[CNT_ERR_SPIN], 32u);
        end = (u64)C.gp_ibound;
    }
    if (t == 0) {
        C.gp_sbit[sb] = (u32)min(s_ibase, (u64)C.gp_ibound);
        if (sb == C.gp_nsb - 1) C.gp_sbit[C.gp_nsb] = (u32)end;
    }
    if (K) {
        // a thread per work item (a single variable's run has thousands of them,
        // which one thread took 1.3 ms to write): its run is found by a search
        for (int k = 0; k < 4; k++) {
            s_pre[4 * t + k] = it;
            it += np[k];
        }
        __syncthreads();
        for (u32 x = t; x < ni; x += BC_T) {
            u32 lo = 0, hi = GP_SB - 1;  // last run that starts at x or before
            while (lo < hi) {
                const u32 mid = (lo + hi + 1) >> 1;
                if (s_pre[mid] <= x) lo = mid;
                else hi = mid - 1;
            }
            const i64 at = (i64)(s_ibase + x);
            if (at >= C.gp_ibound) break;
            const u32 b0 = (lsb * GP_SB + lo) * K, e = x - s_pre[lo];
            const u32 n = (lo + 1 < (u32)GP_SB ? s_pre[lo + 1] : ni) - s_pre[lo];
            GpItem &I = C.gp_item[at];
            I.bin_lo = b0 + gp_run_bin(K, n, e);
            I.bin_hi = b0 + gp_run_bin(K, n, e + 1);
            I.q = q;
            I.pre = I.end = 0;
            I.off = 0;
        }
        return;
    }
    u64 off = s_mbase + mpre;
    pv = pv0;
    for (int k = 0; k < 4; k++) {
        const u32 b = 4 * t + k;
        if ((st >> k) & 1u) {
            const i64 at = (i64)(s_ibase + it);
            if (it > 0 && at - 1 < C.gp_ibound) {
                C.gp_item[at - 1].bin_hi = lsb * GP_SB + pv;
                C.gp_item[at - 1].end = s_pre[pv];
            }
            if (at < C.gp_ibound) {
                GpItem &I = C.gp_item[at];
                I.bin_lo = lsb * GP_SB + b;
                I.q = q;
                I.off = off;
                I.pre = s_pre[b];
                if (it + 1 == ni) {
                    I.bin_hi = lsb * GP_SB + all;
                    I.end = tot;
                }
            }
            it++;
        }
        if (h[k]) pv = b + 1;
        off += m[k];
    }
}

// ---------------------------------------------------------------------------
// k_gp_reduce.  Cells: direct (cell = key inside the work item, at most
// GP_CELLS), else ranked: a presence bitmap over the work item's key span
// gives every present key its rank, the pairs are formed a second time and
// accumulate in the cell of their rank, GP_CELLS ranks per round.
// ---------------------------------------------------------------------------
constexpr int GR_T = 512;
constexpr int GR_NW = GR_T / 64;
constexpr int GR_CPT = GP_CELLS / GR_T;  // cells per thread
constexpr int GR_WIDE = 448, GR_NARROW = 512;  // pieces listed at a time
constexpr u32 GP_SPAN = 1u << GP_SPAN_LOG;
static_assert(GP_SPAN / 64 == GR_T * 4, "each thread scans four bitmap words");

// Cells of the modular rings hold the sum A of the products modulo 2^64 and the
// sum H of their top 16 bits (GP_HI) apart.  At most 2^16 products meet in a
// cell (the planner's condition), so the full sum lies in
// [2^48 H, 2^48 H + 2^64), which tells how often A wrapped: an accumulation
// needs no look at the old value (no returned atomic, no wrap to repair).
template <int RING>
constexpr bool gp_split() {
    return RING == RING_MODP || RING == RING_MODQ;
}
constexpr int GP_HI = 48;

// a * b in a form that is congruent.  Mod p the coefficients come split at bit
// 31 (k_gp_prep): with T = a0 b1 + a1 b0 < 2^62 the product is
// a0 b0 + 2^31 T + 2^62 a1 b1, and 2^61 = 1, so it is congruent to
// a0 b0 + 2 a1 b1 + (T >> 30) + 2^31 (T mod 2^30) < 2^63: four multiply-adds
// and five more instructions.
template <int RING>
__device__ inline u64 gp_mul(u32 a0, u32 a1, u32 b0, u32 b1) {
    if constexpr (RING == RING_MODP) {
        const u64 T = (u64)a1 * b0 + (u64)a0 * b1;
        const u64 r = (u64)a1 * (b1 << 1) + (u64)a0 * b0;
        const u32 tl = (u32)T;
        return r + (T >> 30) + (((u64)((tl >> 1) & 0x1FFFFFFFu) << 32) | (tl << 31));
    } else {
        return ring_mul<RING>(((u64)a1 << 32) | a0, ((u64)b1 << 32) | b0);
    }
}

// The sum of a cell.
template <int RING>
__device__ inline u64 gp_join(u64 A, u32 H) {
    const u32 k = (H + 0xFFFFu - (u32)(A >> GP_HI)) >> (64 - GP_HI);  // A + 2^64 k
    if constexpr (RING == RING_MODP) {
        const u64 r = (A & P61) + (A >> 61) + 8 * k;  // 2^64 = 8
        return r >= P61 ? r - P61 : r;
    } else {
        return addmodq(A >= Q64 ? A - Q64 : A, Q64_C * k);  // 2^64 = 59
    }
}

// LDS of a work item.  Direct: acc u64[GP_CELLS], then (modular rings)
// hi u32[GP_CELLS].  Ranked, over the same memory: acc u64[GP_CELLS],
// rkey u16[GP_CELLS] (key modulo 2^16), bm u64[GP_SPAN / 64] and
// pre u16[GP_SPAN / 64].  Everything but rkey and pre is zero between uses.
struct GrLds {
    static constexpr int HI = GP_CELLS * 8;
    static constexpr int RKEY = GP_CELLS * 8;
    static constexpr int BM = RKEY + GP_CELLS * 2;
    static constexpr int PRE = BM + (int)GP_SPAN / 8;
    static constexpr int RANKED = PRE + (int)GP_SPAN / 64 * 2;
};
static_assert(GP_SPAN_LOG <= 17, "a ranked key is its lower 16 bits and which half of the span it is in");

enum { GP_DIRECT = 0, GP_MARK = 1, GP_RANK = 2 };

// What one pair does: its cell's accumulation, or its key's mark.
template <int RING, int MODE>
__device__ inline void gp_pair(unsigned char *mem, const u32x3 a, const u32x3 b, u32 key, u32 wbase, bool ok) {
    if constexpr (MODE == GP_MARK) {
        if (ok) atomicOr((u32 *)(mem + GrLds::BM) + (key >> 5), 1u << (key & 31));
    } else {
        const u64 v = gp_mul<RING>(a.x, a.y, b.x, b.y);
        if (ok) {
            u32 c = key;
            if constexpr (MODE == GP_RANK) {
                const u32 w = key >> 6;
                const u64 bits = ((const u64 *)(mem + GrLds::BM))[w];
                c = ((const unsigned short *)(mem + GrLds::PRE))[w] +
                    (u32)__popcll(bits & ((1ull << (key & 63)) - 1)) - wbase;
                if (c < (u32)GP_CELLS) ring_atomic_acc<RING>((u64 *)mem + c, v);
            } else {
                atomicAdd((unsigned long long *)mem + c, (unsigned long long)v);
                if constexpr (gp_split<RING>()) atomicAdd((u32 *)(mem + GrLds::HI) + c, (u32)(v >> GP_HI));
            }
        }
    }
}

// A term at a byte offset from a uniform base: coefficient and key.  (Three
// words: a loaded word that nothing reads would be taken for a free register
// while the load is still under way, and its next use would wait for it.)
__device__ inline u32x3 gp_term(const GpTerm *base, u32 off) {
    return *(const __attribute__((address_space(1))) u32x3 *)((const char *)base + off);
}

// Pieces of a block, GP_U steps of a wave each.  A wide piece is 33 to 64
// columns (inner terms, one per lane) by GP_U rows (outer terms, the same for
// every lane: one scalar load of all of them, so that the vector memory path,
// which takes 12 cycles for a load whatever its lanes ask for, only carries
// the columns).  A narrow piece has 2^lg >= columns lanes across and 2^(6-lg)
// stretches of GP_U rows side by side.
constexpr u32 GP_U = 4;
typedef u32 u32x16a __attribute__((ext_vector_type(16), aligned(16)));

struct GpWide {
    u32x3 b;
    u32x16a a;
    u32 cols, rows;
};

// Loads past the piece's rows and columns stay inside the term array and its
// padding (GP_PAD terms) and are not used.
__device__ inline void gp_load_wide(GpWide &p, const uint4 *list, u32 k, const GpTerm *to, const GpTerm *ti) {
    const uint4 e = list[k];
    const u32 row = uniform32(e.x), col = uniform32(e.y), rc = uniform32(e.z);
    p.rows = rc & 0xFFFFu;
    p.cols = rc >> 16;
    p.b = gp_term((const GpTerm *)((const char *)ti + col), (threadIdx.x & 63) * (u32)sizeof(GpTerm));
    p.a = *(const __attribute__((address_space(4))) u32x16a *)((const char *)to + row);
}

template <int RING, int MODE>
__device__ inline void gp_run_wide(const GpWide &p, unsigned char *mem, u32 base, u32 wbase) {
    const bool in = (threadIdx.x & 63) < p.cols;
    const u32 kb = p.b.z - base;
#pragma unroll
    for (u32 u = 0; u < GP_U; u++) {
        const u32x3 a = {p.a[4 * u], p.a[4 * u + 1], p.a[4 * u + 2]};
        if (u < p.rows) gp_pair<RING, MODE>(mem, a, p.b, a.z + kb, wbase, in);
    }
}

struct GpNarrow {
    u32x3 b, a[GP_U];
    u32 r, R;     // this lane's first row; rows (0 for a lane without a column)
    u32 steps;    // (uniform)
};

__device__ inline void gp_load_narrow(GpNarrow &p, const uint4 *list, u32 k, const GpTerm *to, const GpTerm *ti) {
    const uint4 e = list[k];
    const u32 row = uniform32(e.x), col = uniform32(e.y), rc = uniform32(e.z), lg = uniform32(e.w);
    const u32 lane = threadIdx.x & 63, c = lane & ((1u << lg) - 1), rows = rc & 0xFFFFu;
    p.steps = (rows + (64u >> lg) - 1) >> (6 - lg);
    p.r = (lane >> lg) * p.steps;  // stretches apart: neighbouring rows often have neighbouring keys
    p.R = c < (rc >> 16) ? rows : 0u;
    p.b = gp_term((const GpTerm *)((const char *)ti + col), c * (u32)sizeof(GpTerm));
#pragma unroll
    for (u32 u = 0; u < GP_U; u++)
        p.a[u] = gp_term((const GpTerm *)((const char *)to + row), (p.r + u) * (u32)sizeof(GpTerm));
}

template <int RING, int MODE>
__device__ inline void gp_run_narrow(const GpNarrow &p, unsigned char *mem, u32 base, u32 wbase) {
    const u32 kb = p.b.z - base;
#pragma unroll
    for (u32 u = 0; u < GP_U; u++)
        if (u < p.steps) gp_pair<RING, MODE>(mem, p.a[u], p.b, p.a[u].z + kb, wbase, p.r + u < p.R);
}

// The listed pieces, a wave per piece, each piece's terms loaded while the
// one before is worked on (the last one's once more instead of a branch).
template <int RING, int MODE>
__device__ inline void gp_pieces(unsigned char *mem, const uint4 *wide, u32 nw, const uint4 *narrow, u32 nn,
                                 const GpTerm *to, const GpTerm *ti, u32 base, u32 wbase) {
    const u32 w = uniform32(threadIdx.x >> 6);
    if (w < nw) {
        u32 k = w;
        GpWide p, q;
        gp_load_wide(p, wide, k, to, ti);
        while (true) {
            k += GR_NW;
            gp_load_wide(q, wide, min(k, nw - 1), to, ti);
            gp_run_wide<RING, MODE>(p, mem, base, wbase);
            if (k >= nw) break;
            k += GR_NW;
            gp_load_wide(p, wide, min(k, nw - 1), to, ti);
            gp_run_wide<RING, MODE>(q, mem, base, wbase);
            if (k >= nw) break;
        }
    }
    // (the narrow ones from the other end of the waves)
    u32 k = GR_NW - 1 - w;
    if (k < nn) {
        GpNarrow p, q;
        gp_load_narrow(p, narrow, k, to, ti);
        while (true) {
            k += GR_NW;
            gp_load_narrow(q, narrow, min(k, nn - 1), to, ti);
            gp_run_narrow<RING, MODE>(p, mem, base, wbase);
            if (k >= nn) break;
            k += GR_NW;
            gp_load_narrow(p, narrow, min(k, nn - 1), to, ti);
            gp_run_narrow<RING, MODE>(q, mem, base, wbase);
            if (k >= nn) break;
        }
    }
}

// What a thread keeps of its first outer group from one work item to the next.
struct GpOuter {
    u32 p, i0, rows;  // prefix, first row, rows (0: no such group)
    u32 j0, nc;       // columns in the work item at hand
};

__device__ inline void gp_cols(const u32 *lut, u32 p, u32 B0, u32 B1, u32 &j0, u32 &nc) {
    j0 = nc = 0;
    if (p < B1) {
        j0 = gload(lut + (B0 > p ? B0 - p : 0u));
        nc = gload(lut + (B1 - p)) - j0;
    }
}

// List counters, by parity of the listing: wide and narrow pieces, and what is
// left (1: pieces that did not fit, 2: outer groups).
struct GpCtl {
    u32 nw[2], nn[2], more[2];
};

// Forms every pair of output prefixes [B0, B1): lists the blocks' pieces, a
// thread per outer group, and runs them whenever the list fills up.
// `before` runs between the first listing and its pieces.
template <int RING, int MODE, typename Before>
__device__ inline void gp_sweep(const GpOperand &O, const GpOperand &I, const u32 *lut, u32 B0, u32 B1, u32 base,
                                unsigned char *mem, uint4 *list, GpCtl *ctl, u32 &par, const GpOuter &F, u32 wbase,
                                Before &&before) {
    uint4 *wide = list, *narrow = list + GR_WIDE;
    u32 og = threadIdx.x;
    u32 i0 = 0, rows = 0, j0 = 0, nc = 0;
    u32 nwide = 0, nnarrow = 0;  // pieces still to be listed
    u32 wc = 0, wr = 0, nr = 0;  // next wide piece: column, row; next narrow piece: row
    const u32 lane = threadIdx.x & 63;
    bool first = true;
    while (true) {
        u32 flags, nw, nn;
        while (true) {
            if (!(nwide | nnarrow) && og < O.groups) {
                if (og == threadIdx.x) {
                    i0 = F.i0;
                    j0 = F.j0;
                    nc = F.nc;
                    rows = F.rows;
                } else {
                    gp_cols(lut, gload(O.pfx + og), B0, B1, j0, nc);
                    if (nc) {
                        i0 = gload(O.start + og);
                        rows = gload(O.start + og + 1) - i0;
                    }
                }
                og += GR_T;
                wc = wr = nr = 0;
                if (nc && rows) {
                    const u32 rest = nc & 63;
                    nwide = ((nc + 31) >> 6) * ((rows + GP_U - 1) / GP_U);
                    if (rest && rest <= 32) {
                        const u32 lg = rest > 1 ? 32u - (u32)__clz((int)(rest - 1)) : 0u;
                        nnarrow = (rows + (GP_U << (6 - lg)) - 1) >> (8 - lg);
                    }
                }
            }
            const u32 iw = wave_scan_dpp(nwide), in = wave_scan_dpp(nnarrow);
            const u32 tw = (u32)__builtin_amdgcn_readlane((int)iw, 63), tn = (u32)__builtin_amdgcn_readlane((int)in, 63);
            u32 aw = 0, an = 0;
            if (lane == 0) {
                if (tw) aw = atomicAdd(&ctl->nw[par], tw);
                if (tn) an = atomicAdd(&ctl->nn[par], tn);
            }
            aw = uniform32(aw) + iw - nwide;
            an = uniform32(an) + in - nnarrow;
            for (u32 e = aw; e < (u32)GR_WIDE && nwide; e++, nwide--) {
                wide[e] = make_uint4((i0 + wr) * (u32)sizeof(GpTerm), (j0 + wc) * (u32)sizeof(GpTerm),
                                     min(rows - wr, GP_U) | (min(nc - wc, 64u) << 16), 6u);
                wr += GP_U;
                if (wr >= rows) {
                    wr = 0;
                    wc += 64;
                }
            }
            for (u32 e = an; e < (u32)GR_NARROW && nnarrow; e++, nnarrow--) {
                const u32 cols = nc & 63, lg = cols > 1 ? 32u - (u32)__clz((int)(cols - 1)) : 0u;
                const u32 ch = min(rows - nr, GP_U << (6 - lg));
                narrow[e] = make_uint4((i0 + nr) * (u32)sizeof(GpTerm), (j0 + nc - cols) * (u32)sizeof(GpTerm),
                                       ch | (cols << 16), lg);
                nr += ch;
            }
            const u32 mine = (__ballot((nwide | nnarrow) != 0) ? 1u : 0u) | (__ballot(og < O.groups) ? 2u : 0u);
            if (lane == 0 && mine) atomicOr(&ctl->more[par], mine);
            __syncthreads();
            flags = uniform32(ctl->more[par]);
            nw = uniform32(ctl->nw[par]);
            nn = uniform32(ctl->nn[par]);
            if (flags != 2 || nw >= (u32)GR_WIDE / 2 || nn >= (u32)GR_NARROW / 2) break;
            __syncthreads();  // every thread has read the counters
            if (threadIdx.x == 0) ctl->more[par] = 0;
            __syncthreads();
        }
        par ^= 1u;
        if (threadIdx.x == 0) {  // the next listing's counters: read by everyone before the last pieces
            ctl->nw[par] = 0;
            ctl->nn[par] = 0;
            ctl->more[par] = 0;
        }
        if (first) before();
        first = false;
        gp_pieces<RING, MODE>(mem, wide, min(nw, (u32)GR_WIDE), narrow, min(nn, (u32)GR_NARROW), O.t, I.t, base, wbase);
        __syncthreads();
        if (!flags) break;
    }
}

// The same with a thread per outer term, each walking its own columns: for
// operands whose groups hold a term or two.
template <int RING>
__device__ inline void gp_rows(const GpOperand &O, const GpOperand &I, const u32 *lut, u32 B0, u32 B1, u32 base,
                               unsigned char *mem) {
    for (u32 i = threadIdx.x; i < O.n; i += GR_T) {
        const u32x3 a = gp_term(O.t, i * (u32)sizeof(GpTerm));
        u32 j0, nc;
        gp_cols(lut, gload(&O.t[i].pfx), B0, B1, j0, nc);
        const u32 ka = a.z - base;
        for (u32 c = 0; c < nc; c += 4) {
            u32x3 b[4];
#pragma unroll
            for (u32 u = 0; u < 4; u++) b[u] = gp_term(I.t, (j0 + c + u) * (u32)sizeof(GpTerm));
#pragma unroll
            for (u32 u = 0; u < 4; u++)
                if (c + u < nc) gp_pair<RING, GP_DIRECT>(mem, a, b[u], b[u].z + ka, 0u, true);
        }
    }
    __syncthreads();
}

// The work items of SEG_GRPD products (BOX: every cell is stored; part k of n
// of the list) or of SEG_GRP products.  The first work items of a workgroup
// are its own, the later ones come from a counter (an addition to one address
// by many workgroups takes about 10 ns each).  The next work item's
// descriptor and its columns (first outer group of every thread) are loaded
// while the current one runs.
template <int RING, bool BOX>
__global__ __launch_bounds__(GR_T) __attribute__((amdgpu_waves_per_eu(4))) void k_gp_reduce(Ctx C, i64 part, i64 nparts) {
    constexpr bool SPLIT = gp_split<RING>();
    constexpr int DIRECT = GP_CELLS * (SPLIT ? 12 : 8);
    constexpr int MEM = BOX ? DIRECT : (DIRECT > GrLds::RANKED ? DIRECT : GrLds::RANKED);
    __shared__ __align__(16) unsigned char s_mem[MEM];
    __shared__ uint4 s_list[GR_WIDE + GR_NARROW];
    __shared__ GpCtl s_ctl;
    __shared__ u32 s_w[GR_NW];
    __shared__ u32 s_tn[2];  // by parity: read after the barrier that ends a work item, while the other is written
    u64 *acc = (u64 *)s_mem;
    u32 *counter = &C.counters[BOX ? CNT_GP_BOX : CNT_GP_REDUCE];
    // every array starts at zero and is left so
    for (u32 e = threadIdx.x; e < (u32)MEM / 16; e += GR_T) ((uint4 *)s_mem)[e] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x == 0) s_ctl = GpCtl{{0, 0}, {0, 0}, {0, 0}};
    __syncthreads();
    const i64 nall = (i64)uniform32(C.gp_sbit[C.gp_nsb]);
    const i64 tb = nall * part / nparts, ntk = nall * (part + 1) / nparts, G = gridDim.x;
    const i64 own = max((i64)2, BOX ? 0 : (ntk - tb) / G * 3 / 8);  // work items of its own per workgroup
    i64 t = tb + blockIdx.x, t1 = t + G;
    i64 round = 2;
    u32 par = 0, lpar = 0;
    const u32 lane = threadIdx.x & 63, w = uniform32(threadIdx.x >> 6);
    auto item = [&](i64 t) -> GpItem {
        GpItem it{};
        if (t < ntk) it = C.gp_item[t];
        return it;
    };
    GpItem d0 = item(t), d1 = item(t1);
    int qc = -1;  // product whose fields are held
    u32 S = 1, rowmode = 0;
    GpOperand O, I;
    const u32 *lut = nullptr;
    u64 *box = nullptr;
    GpOuter F{};
    bool have = false;  // F's columns are the coming work item's
    bool mine = false;  // the product is of this kernel's kind
    while (t < ntk) {
        const int q = (int)uniform32((u32)d0.q);
        const u32 B0 = uniform32(d0.bin_lo), B1 = uniform32(d0.bin_hi);
        const u64 off = (u64)uniform64((i64)d0.off);
        if (q != qc) {
            const DevSeg &s = C.segs[q];
            const int bq = (int)uniform32(s.gp.bq), so = (int)uniform32(s.gp.swap);
            S = uniform32(s.gp.S);
            rowmode = BOX ? uniform32(s.gp.rows) : 0u;
            O = gp_operand(C, s, bq, so);
            I = gp_operand(C, s, bq, 1 - so);
            lut = C.gp_lut + uniform64(s.gp.lut);
            if constexpr (BOX) box = C.box + uniform64(s.stage_base);
            mine = BOX ? uniform32(s.gp.K) != 0 : uniform32(s.gp.K) == 0 && uniform32(s.gp.rows) == 0;
            qc = q;
            F.rows = 0;
            if (threadIdx.x < O.groups) {
                F.p = gload(O.pfx + threadIdx.x);
                F.i0 = gload(O.start + threadIdx.x);
                F.rows = gload(O.start + threadIdx.x + 1) - F.i0;
            }
            have = false;
        }
        if (!have && F.rows) gp_cols(lut, F.p, B0, B1, F.j0, F.nc);
        const GpOuter F0 = F;
        u32 tk = 0;
        auto ahead = [&]() {  // the next work item's columns, the ticket of the one after it
            have = t1 < ntk && (int)uniform32((u32)d1.q) == qc && !rowmode;
            if (have && F.rows) gp_cols(lut, F.p, d1.bin_lo, d1.bin_hi, F.j0, F.nc);
            if (round >= own && threadIdx.x == 0) tk = atomicAdd(counter, 1u);
        };
        if (!mine || rowmode) ahead();
        const u32 base = B0 * S;  // keys are compared modulo 2^32: a work item spans fewer
        const u32 span = (B1 - B0) * S;
        u32 done = 0;  // result terms so far
        if (!mine) {
            // another kernel's product
        } else if (BOX || span <= (u32)GP_CELLS) {
            if (BOX && rowmode) gp_rows<RING>(O, I, lut, B0, B1, base, s_mem);
            else gp_sweep<RING, GP_DIRECT>(O, I, lut, B0, B1, base, s_mem, s_list, &s_ctl, lpar, F0, 0u, ahead);
            // a wave's cells are consecutive, a lane takes two at a time
            const u32 cw = (span + GR_NW * 128 - 1) / (GR_NW * 128) * 128;
            const u32 c0 = w * cw + lane * 2;
            u64 val[GR_CPT];
            u32 em = 0;
#pragma unroll
            for (int k = 0; k < GR_CPT / 2; k++) {
                const u32 c = c0 + k * 128;
                val[2 * k] = val[2 * k + 1] = 0;
                if ((u32)k * 128 < cw) {
                    ulonglong2 x = *(ulonglong2 *)&acc[c];
                    *(ulonglong2 *)&acc[c] = make_ulonglong2(0, 0);
                    if constexpr (SPLIT) {
                        uint2 *hi = (uint2 *)(s_mem + GrLds::HI + c * 4);
                        const uint2 y = *hi;
                        *hi = make_uint2(0, 0);
                        x.x = gp_join<RING>(x.x, y.x);
                        x.y = gp_join<RING>(x.y, y.y);
                    }
                    val[2 * k] = x.x;
                    val[2 * k + 1] = x.y;
                    if constexpr (BOX) {
                        // (cells beyond the work item are zero: nothing was added)
                        u64 *o = box + ((i64)B0 * S + c);
                        if (c < span) o[0] = x.x;
                        if (c + 1 < span) o[1] = x.y;
                    }
                    if (!ring_is_zero<RING>(x.x)) em |= 1u << (2 * k);
                    if (!ring_is_zero<RING>(x.y)) em |= 2u << (2 * k);
                }
            }
            {
                u32 rk[GR_CPT / 2], before = 0;
#pragma unroll
                for (int k = 0; k < GR_CPT / 2; k++) {
                    const u64 b0 = __ballot((em >> (2 * k)) & 1u), b1 = __ballot((em >> (2 * k + 1)) & 1u);
                    rk[k] = before + mbcnt(b0) + mbcnt(b1);
                    before += (u32)__popcll(b0) + (u32)__popcll(b1);
                }
                if (lane == 0) s_w[w] = before;
                __syncthreads();
                u32 wpre = 0;
#pragma unroll
                for (u32 i = 0; i < (u32)GR_NW; i++) {
                    const u32 v = s_w[i];
                    if (i < w) wpre += v;
                    done += v;
                }
                // the next work item's columns and the ticket are taken here:
                // later their wait would be one for the stores, too
                asm volatile("" : "+v"(F.j0), "+v"(F.nc), "+v"(tk));
#pragma unroll
                for (int k = 0; k < GR_CPT / 2 && !BOX; k++) {
                    u64 at = off + wpre + rk[k];
                    if ((em >> (2 * k)) & 1u) {
                        C.gp_rkey[at] = c0 + k * 128;
                        C.gp_rcoef[at] = val[2 * k];
                        at++;
                    }
                    if ((em >> (2 * k + 1)) & 1u) {
                        C.gp_rkey[at] = c0 + k * 128 + 1;
                        C.gp_rcoef[at] = val[2 * k + 1];
                    }
                }
            }
        } else if constexpr (!BOX) {
            unsigned short *rkey = (unsigned short *)(s_mem + GrLds::RKEY);
            u64 *bm = (u64 *)(s_mem + GrLds::BM);
            unsigned short *pre = (unsigned short *)(s_mem + GrLds::PRE);
            auto none = [] {};
            gp_sweep<RING, GP_MARK>(O, I, lut, B0, B1, base, s_mem, s_list, &s_ctl, lpar, F0, 0u, ahead);
            // rank of a word's first key (thread t: words 4t .. 4t + 3)
            u64 wd[4];
            u32 sum = 0, distinct;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                wd[e] = bm[threadIdx.x * 4 + e];
                sum += (u32)__popcll(wd[e]);
            }
            const u32 ex = block_excl_scan<u32, GR_T>(sum, s_w, distinct);
            {
                u32 r = ex;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    pre[threadIdx.x * 4 + e] = (unsigned short)r;
                    r += (u32)__popcll(wd[e]);
                }
            }
            __syncthreads();
            const u32 lower = pre[GP_SPAN / 128];  // ranks in the lower half of the span
            const u32 half = (u32)GP_SPAN > 65536u ? 65536u : 0u;
            for (u32 wb = 0; wb < distinct; wb += GP_CELLS) {
                // keys of the round's ranks
                u32 r = ex - wb;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    u64 x = wd[e];
                    while (x) {
                        if (r < (u32)GP_CELLS)
                            rkey[r] = (unsigned short)((threadIdx.x * 4 + e) * 64 + (u32)__ffsll((unsigned long long)x) - 1);
                        r++;
                        x &= x - 1;
                    }
                }
                __syncthreads();
                gp_sweep<RING, GP_RANK>(O, I, lut, B0, B1, base, s_mem, s_list, &s_ctl, lpar, F0, wb, none);
                const u32 ncell = min(distinct - wb, (u32)GP_CELLS);
                const u32 cw = (ncell + GR_T - 1) / GR_T * 64;  // cells of a wave
                constexpr int CPT = GP_CELLS / GR_T;
                u64 val[CPT];
                u32 kk[CPT], rk[CPT], em = 0, before = 0;
#pragma unroll
                for (int k = 0; k < CPT; k++) {
                    const u32 c = w * cw + k * 64 + lane;
                    val[k] = 0;
                    kk[k] = 0;
                    if ((u32)k * 64 < cw && c < ncell) {
                        kk[k] = rkey[c] + (wb + c >= lower ? half : 0u);
                        val[k] = ring_cell_final<RING>(acc[c]);
                        acc[c] = 0;
                        if (!ring_is_zero<RING>(val[k])) em |= 1u << k;
                    }
                    const u64 bal = __ballot((em >> k) & 1u);
                    rk[k] = before + mbcnt(bal);
                    before += (u32)__popcll(bal);
                }
                if (lane == 0) s_w[w] = before;
                __syncthreads();
                u32 wpre = 0, tot = 0;
#pragma unroll
                for (u32 i = 0; i < (u32)GR_NW; i++) {
                    const u32 v = s_w[i];
                    if (i < w) wpre += v;
                    tot += v;
                }
#pragma unroll
                for (int k = 0; k < CPT; k++) {
                    if ((em >> k) & 1u) {
                        const u64 at = off + done + wpre + rk[k];
                        C.gp_rkey[at] = kk[k];
                        C.gp_rcoef[at] = val[k];
                    }
                }
                done += tot;
                __syncthreads();
            }
            // the direct cells overlay the keys, the bitmap and its prefix
            for (u32 e = threadIdx.x; e < (u32)(GrLds::RANKED - GrLds::RKEY) / 16; e += GR_T)
                ((uint4 *)(s_mem + GrLds::RKEY))[e] = make_uint4(0, 0, 0, 0);
        }
        if (mine && threadIdx.x == 0) {
            C.gp_u[t] = done;
            atomicAdd(&C.gp_usum[t >> GP_USUM_LOG], done);
        }
        if (round >= own && threadIdx.x == 0) s_tn[par] = tk;
        __syncthreads();
        d0 = d1;
        t = t1;
        t1 = round < own ? tb + blockIdx.x + round * G : tb + own * G + (i64)uniform32(s_tn[par]);
        d1 = item(t1);
        round++;
        par ^= 1u;
    }
}

// ---------------------------------------------------------------------------
// k_gp_list: work items of products whose blocks hold few pairs (gp.rows).
// Such a block leaves most lanes of a wave idle, so the pairs are listed in
// LDS first (a thread per outer group, cheap steps) and worked off with every
// lane.  A work item of at most GL_PAIRS pairs whose keys span more than the
// direct cells is listed once: its pairs' keys and products stay in registers
// between the marks in the presence bitmap and the accumulation by rank.
// Others accumulate in direct cells, GL_CELLS keys per round.
// One workgroup of 1024 threads per compute unit, all of its LDS: larger work
// items look fewer outer groups up and share the bitmap's scan among more
// pairs, which is what bounds it (a sixth of the time forms products).  With a
// thread per outer term walking its columns, twice and more (the way it was),
// 777 x 12345 random terms in 6 variables took 255 us here, now 151 (2^17 keys
// per work item: 241, 2^19: 164, then the scan without bank conflicts); a batch
// of 24 random products up to 217 million pairs 8.1 ms, now 4.8.
// ---------------------------------------------------------------------------
constexpr int GL_T = 1024;
constexpr int GL_NW = GL_T / 64;
constexpr int GL_E = 10;               // pairs of a thread, at most
constexpr int GL_CELLS = 15360;        // direct cells
constexpr int GL_LIST = 3072;          // pairs listed at a time beside direct cells
constexpr int GL_G = 4;                // outer groups of a thread that stay in registers

// Ranked: the list uint2[P] and later, in its place, the cells; rkey u32[P],
// the bitmap of 2^sl bits, pre u16[2^sl / 64], with P = gl_pairs(sl).
// Direct: the cells, the list uint2[GL_LIST].  Behind them the heads, a byte
// per listed pair, zero between uses.
struct GlLds {
    static constexpr int LIST = GL_CELLS * 8;
    static constexpr int HEAD = LIST + GL_LIST * 8;
    static constexpr int MEM = HEAD + GL_E * GL_T;
};
constexpr int gl_ranked_bytes(u32 sl) { return (int)gl_pairs(sl) * 12 + (1 << (sl - 3)) + (1 << (sl - 5)); }
static_assert(gl_ranked_bytes(17) <= GlLds::HEAD && gl_ranked_bytes(18) <= GlLds::HEAD && gl_ranked_bytes(19) <= GlLds::HEAD,
              "one memory for both");
static_assert(gl_pairs(17) <= GL_E * GL_T && gl_pairs(18) <= GL_E * GL_T && gl_pairs(19) <= GL_E * GL_T, "pairs of a thread");

// The part of a block that a thread has not listed yet: byte offsets of the
// next pair's terms and of the block's columns, pairs left.
struct GlBlock {
    u32 i, j, jlo, jhi, left;
};

// The list holds the first pair of every row (byte offsets of its two terms),
// and again the one at every multiple of 64 that the row covers; heads marks
// these places.  So the 64 pairs of a wave find their rows by a ballot.
__device__ inline void gl_row(uint2 *list, unsigned char *head, u32 pos, u32 i, u32 j, u32 len) {
    list[pos] = make_uint2(i, j);
    head[pos] = 1;
    for (u32 b = (pos | 63) + 1; b < pos + len; b += 64) {
        list[b] = make_uint2(i, j + (b - pos) * (u32)sizeof(GpTerm));
        head[b] = 1;
    }
}

// The terms of listed pair pos (a wave's are 64 consecutive ones from a
// multiple of 64; past the list's end: some term's, within the padding).
__device__ inline uint2 gl_pair(const uint2 *list, unsigned char *head, u32 pos) {
    const u64 m = __ballot(head[pos] != 0);
    head[pos] = 0;
    const u32 d = m ? (u32)__clzll((long long)(m << (63 - (pos & 63)))) : 0u;
    uint2 p = list[pos - d];
    p.y += d * (u32)sizeof(GpTerm);
    return m ? p : make_uint2(0, 0);
}

template <int RING>
__global__ __launch_bounds__(GL_T) void k_gp_list(Ctx C) {
    constexpr u32 TB = (u32)sizeof(GpTerm);
    constexpr u64 WRAP = RING == RING_MODP ? 8 : Q64_C;
    __shared__ __align__(16) unsigned char s_mem[GlLds::MEM];
    __shared__ u32 s_w[GL_NW], s_n[2], s_more[2], s_tn[2];
    u64 *acc = (u64 *)s_mem;
    const u32 tid = threadIdx.x, lane = tid & 63, w = uniform32(tid >> 6);
    unsigned char *head = s_mem + GlLds::HEAD;
    for (u32 e = tid; e < (u32)(GL_E * GL_T) / 16; e += GL_T) ((uint4 *)head)[e] = make_uint4(0, 0, 0, 0);
    if (tid < 2) s_n[tid] = s_more[tid] = 0;
    __syncthreads();
    const i64 ntk = (i64)uniform32(C.gp_sbit[C.gp_nsb]), G = gridDim.x;
    const i64 own = max((i64)2, ntk / G * 3 / 8);  // work items of its own, see k_gp_reduce
    i64 t = blockIdx.x, t1 = t + G, round = 2;
    u32 par = 0, lpar = 0;
    auto item = [&](i64 t) -> GpItem {
        GpItem it{};
        if (t < ntk) it = C.gp_item[t];
        return it;
    };
    GpItem d0 = item(t), d1 = item(t1);
    int qc = -1;
    u32 S = 1, sl = 17;
    GpOperand O, I;
    const u32 *lut = nullptr;
    u32 gp[GL_G] = {};                 // prefixes of a thread's first groups (~0: no such group)
    u32 cj[GL_G] = {}, ce[GL_G] = {};  // their columns in the work item: [cj, ce)
    bool have = false, mine = false;
    while (t < ntk) {
        const int q = (int)uniform32((u32)d0.q);
        const u32 B0 = uniform32(d0.bin_lo), B1 = uniform32(d0.bin_hi), np = uniform32(d0.end - d0.pre);
        const u64 off = (u64)uniform64((i64)d0.off);
        if (q != qc) {
            const DevSeg &s = C.segs[q];
            const int bq = (int)uniform32(s.gp.bq), so = (int)uniform32(s.gp.swap);
            S = uniform32(s.gp.S);
            sl = uniform32(s.gp.rows);
            O = gp_operand(C, s, bq, so);
            I = gp_operand(C, s, bq, 1 - so);
            lut = C.gp_lut + uniform64(s.gp.lut);
            mine = uniform32(s.gp.K) == 0 && sl != 0;
            qc = q;
#pragma unroll
            for (int k = 0; k < GL_G; k++) {
                const u32 og = tid + k * GL_T;
                gp[k] = og < O.groups && mine ? gload(O.pfx + og) : ~0u;
            }
            have = false;
        }
        auto columns = [&](u32 b0, u32 b1) {
#pragma unroll
            for (int k = 0; k < GL_G; k++) {
                const bool in = gp[k] < b1;  // (else lut[0] twice: none; loads without a branch: all of them under way at once)
                cj[k] = gload(lut + (in && b0 > gp[k] ? b0 - gp[k] : 0u));
                ce[k] = gload(lut + (in ? b1 - gp[k] : 0u));
            }
        };
        if (!have) columns(B0, B1);
        u32 tk = 0;
        auto ahead = [&]() {  // the next work item's columns, the ticket of the one after it
            have = t1 < ntk && (int)uniform32((u32)d1.q) == qc;
            if (have) columns(uniform32(d1.bin_lo), uniform32(d1.bin_hi));
            if (round >= own && tid == 0) tk = atomicAdd(&C.counters[CNT_GP_LIST], 1u);
        };
        // (taken before the stores: later their wait would be one for the stores, too)
        auto taken = [&]() {
            asm volatile("" : "+v"(cj[0]), "+v"(cj[1]), "+v"(cj[2]), "+v"(cj[3]), "+v"(ce[0]), "+v"(ce[1]),
                         "+v"(ce[2]), "+v"(ce[3]), "+v"(tk));
        };
        // Lists the work item's pairs, cap at a time, and calls use(count).
        auto pairs = [&](uint2 *list, u32 cap, auto &&use) {
            GlBlock B{0, 0, 0, 0, 0};
            u32 og = tid;
            int k = 0;
            while (true) {
                bool room = true;
                while (room && __ballot(B.left || og < O.groups)) {
                    if (!B.left && og < O.groups) {
                        u32 j0, nc;
                        if (k < GL_G) {
                            j0 = k == 0 ? cj[0] : k == 1 ? cj[1] : k == 2 ? cj[2] : cj[3];
                            nc = (k == 0 ? ce[0] : k == 1 ? ce[1] : k == 2 ? ce[2] : ce[3]) - j0;
                        } else {
                            gp_cols(lut, gload(O.pfx + og), B0, B1, j0, nc);
                        }
                        if (nc) {
                            const u32 i0 = gload(O.start + og), rows = gload(O.start + og + 1) - i0;
                            B.i = i0 * TB;
                            B.j = B.jlo = j0 * TB;
                            B.jhi = (j0 + nc) * TB;
                            B.left = rows * nc;
                        }
                        og += GL_T;
                        k++;
                    }
                    const u32 want = min(B.left, cap);
                    const u32 inc = wave_scan_dpp(want);
                    const u32 tot = (u32)__builtin_amdgcn_readlane((int)inc, 63);
                    u32 at = 0;
                    if (tot && lane == 0) at = atomicAdd(&s_n[lpar], tot);
                    at = uniform32(at);
                    room = at + tot <= cap;
                    at += inc - want;
                    const u32 take = at < cap ? min(want, cap - at) : 0u;
                    // long blocks by the whole wave, a lane per row, the others a lane each
                    const bool lg = take > 128;
                    for (u64 m = __ballot(lg); m; m &= m - 1) {
                        const int l = __ffsll((unsigned long long)m) - 1;
                        const u32 bi = (u32)__builtin_amdgcn_readlane((int)B.i, l);
                        const u32 jl = (u32)__builtin_amdgcn_readlane((int)B.jlo, l);
                        const u32 c0 = ((u32)__builtin_amdgcn_readlane((int)B.j, l) - jl) / TB;  // listed before of this row
                        const u32 nc = ((u32)__builtin_amdgcn_readlane((int)B.jhi, l) - jl) / TB;
                        const u32 ba = (u32)__builtin_amdgcn_readlane((int)at, l);
                        const u32 end = c0 + (u32)__builtin_amdgcn_readlane((int)take, l);
                        const u32 nr = (end + nc - 1) / nc;
                        for (u32 r = lane; r < nr; r += 64) {
                            const u32 s0 = max(r * nc, c0), s1 = min(r * nc + nc, end);
                            gl_row(list, head, ba + s0 - c0, bi + r * TB, jl + (s0 - r * nc) * TB, s1 - s0);
                        }
                        if ((int)lane == l) {
                            const u32 r = end / nc;
                            B.i = bi + r * TB;
                            B.j = jl + (end - r * nc) * TB;
                        }
                    }
                    for (u32 e = 0; e < (lg ? 0u : take);) {
                        const u32 len = min((B.jhi - B.j) / TB, take - e);
                        gl_row(list, head, at + e, B.i, B.j, len);
                        e += len;
                        B.j += len * TB;
                        if (B.j == B.jhi) {
                            B.j = B.jlo;
                            B.i += TB;
                        }
                    }
                    B.left -= take;
                }
                if (__ballot(B.left || og < O.groups) && lane == 0) s_more[lpar] = 1;
                __syncthreads();
                const u32 n = min(uniform32(s_n[lpar]), cap);
                const bool more = uniform32(s_more[lpar]) != 0;
                lpar ^= 1u;
                if (tid == 0) s_n[lpar] = s_more[lpar] = 0;  // read by everyone before the barrier above
                use(n);
                __syncthreads();
                if (!more) break;
            }
        };
        const u32 base = B0 * S, span = (B1 - B0) * S;
        u32 done = 0;
        // Stages the non-zero ones of n cells; last: the work item's last cells.
        auto emit = [&](u32 n, auto &&key, bool last) {
            const u32 cw = (n + GL_T - 1) / GL_T * 64;  // cells of a wave
            const u32 c1 = min(w * cw + cw, n);
            u32 mine_n = 0;
            for (u32 c = w * cw; c < c1; c += 256) {
                u64 y[4];
#pragma unroll
                for (u32 e = 0; e < 4; e++) y[e] = acc[min(c + e * 64, c1 - 1) + lane];
#pragma unroll
                for (u32 e = 0; e < 4; e++)
                    mine_n += c + e * 64 + lane < c1 && !ring_is_zero<RING>(ring_cell_final<RING>(y[e])) ? 1u : 0u;
            }
            const u32 inc = wave_scan_dpp(mine_n);
            if (lane == 63) s_w[w] = inc;
            if (last) ahead();
            __syncthreads();
            const u32 sw = s_w[lane & (GL_NW - 1)];
            const u32 wi = wave_scan_dpp(lane < (u32)GL_NW ? sw : 0u);
            const u32 tot = (u32)__builtin_amdgcn_readlane((int)wi, 63);
            u32 at = w ? (u32)__builtin_amdgcn_readlane((int)wi, (int)w - 1) : 0u;
            taken();
            u32 *rk = C.gp_rkey + off + done;
            u64 *rc = C.gp_rcoef + off + done;
            for (u32 c = w * cw; c < c1; c += 128) {
                u64 y[2];
                u32 k[2];
#pragma unroll
                for (u32 e = 0; e < 2; e++) {
                    const u32 x = min(c + e * 64, c1 - 1) + lane;
                    y[e] = acc[x];
                    k[e] = key(x);
                }
#pragma unroll
                for (u32 e = 0; e < 2; e++) {
                    const u64 val = ring_cell_final<RING>(y[e]);
                    const bool in = c + e * 64 + lane < c1 && !ring_is_zero<RING>(val);
                    const u64 em = __ballot(in);
                    if (in) {
                        rk[at + mbcnt(em)] = k[e];
                        rc[at + mbcnt(em)] = val;
                    }
                    at += (u32)__popcll(em);
                }
            }
            done += tot;
        };
        if (!mine) {
            ahead();  // another kernel's product
        } else if (np <= gl_pairs(sl) && span > (u32)GL_CELLS) {
            const u32 P = gl_pairs(sl);
            u32 *rkey = (u32 *)(s_mem + P * 8);
            u64 *bm = (u64 *)(s_mem + P * 12);
            unsigned short *pre = (unsigned short *)(s_mem + P * 12 + (1u << (sl - 3)));
            for (u32 e = tid; e < 1u << (sl - 7); e += GL_T) ((uint4 *)bm)[e] = make_uint4(0, 0, 0, 0);
            u32 x[GL_E];  // key, then rank; ~0: no pair
            u64 v[GL_E];
            const uint2 *list = (const uint2 *)s_mem;
            pairs((uint2 *)s_mem, P, [&](u32 n) {
#pragma unroll
                for (int e = 0; e < GL_E; e++) x[e] = ~0u;
#pragma unroll
                for (int e0 = 0; e0 < GL_E; e0 += GL_E / 2) {
                    if ((u32)e0 * GL_T >= n) break;
                    u32x3 a[GL_E / 2], b[GL_E / 2];
#pragma unroll
                    for (int e = 0; e < GL_E / 2; e++) {
                        const uint2 p = gl_pair(list, head, tid + (e0 + e) * GL_T);
                        a[e] = gp_term(O.t, p.x);
                        b[e] = gp_term(I.t, p.y);
                    }
#pragma unroll
                    for (int e = 0; e < GL_E / 2; e++) {
                        if (tid + (e0 + e) * GL_T < n) {
                            x[e0 + e] = a[e].z + b[e].z - base;
                            atomicOr((u32 *)bm + (x[e0 + e] >> 5), 1u << (x[e0 + e] & 31));
                        }
                        v[e0 + e] = gp_mul<RING>(a[e].x, a[e].y, b[e].x, b[e].y);
                    }
                }
            });
            // rank of a word's first key (a wave has consecutive words, a lane every 64th of them)
            u32 distinct;
            {
                const u32 nw = 1u << (sl - 16), w0 = w * nw * 64 + lane;
                u32 cnt[8], sum = 0;
#pragma unroll
                for (u32 e = 0; e < 8; e++) {
                    cnt[e] = 0;
                    if (e < nw) cnt[e] = (u32)__popcll(bm[w0 + e * 64]);
                    sum += cnt[e];
                }
                const u32 tot = (u32)__builtin_amdgcn_readlane((int)wave_scan_dpp(sum), 63);
                if (lane == 0) s_w[w] = tot;
                __syncthreads();
                const u32 sw = s_w[lane & (GL_NW - 1)];
                const u32 wi = wave_scan_dpp(lane < (u32)GL_NW ? sw : 0u);
                distinct = (u32)__builtin_amdgcn_readlane((int)wi, 63);
                u32 r = w ? (u32)__builtin_amdgcn_readlane((int)wi, (int)w - 1) : 0u;
#pragma unroll
                for (u32 e = 0; e < 8; e++) {
                    if (e >= nw) break;
                    const u32 inc = wave_scan_dpp(cnt[e]);
                    pre[w0 + e * 64] = (unsigned short)(r + inc - cnt[e]);
                    r += (u32)__builtin_amdgcn_readlane((int)inc, 63);
                }
            }
            for (u32 c = tid; c < distinct; c += GL_T) acc[c] = 0;
            __syncthreads();
            {
#pragma unroll
                for (int e0 = 0; e0 < GL_E; e0 += GL_E / 2) {
                    if ((u32)e0 * GL_T >= np) break;
                    u64 old[GL_E / 2];
#pragma unroll
                    for (int e = 0; e < GL_E / 2; e++) {
                        u32 &y = x[e0 + e];
                        old[e] = 0;
                        if (y == ~0u) continue;
                        const u32 key = y;
                        y = pre[y >> 6] + (u32)__popcll(bm[y >> 6] & ((1ull << (y & 63)) - 1));
                        rkey[y] = key;
                        old[e] = atomicAdd((unsigned long long *)acc + y, (unsigned long long)v[e0 + e]);
                    }
                    if constexpr (gp_split<RING>()) {
#pragma unroll
                        for (int e = 0; e < GL_E / 2; e++)
                            if (x[e0 + e] != ~0u && old[e] + v[e0 + e] < old[e]) ring_atomic_acc<RING>(acc + x[e0 + e], WRAP);
                    }
                }
            }
            __syncthreads();
            emit(distinct, [&](u32 c) { return rkey[c]; }, true);
        } else {
            uint2 *list = (uint2 *)(s_mem + GlLds::LIST);
            const u32 nwin = (span + GL_CELLS - 1) / GL_CELLS, width = (span + nwin - 1) / nwin;
            for (u32 w0 = 0; w0 < span; w0 += width) {
                for (u32 c = tid; c < width; c += GL_T) acc[c] = 0;
                const u32 sub = base + w0;
                pairs(list, GL_LIST, [&](u32 n) {
                    u32x3 a[GL_LIST / GL_T], b[GL_LIST / GL_T];
                    if (!n) return;
#pragma unroll
                    for (int e = 0; e < GL_LIST / GL_T; e++) {
                        const uint2 p = gl_pair(list, head, tid + e * GL_T);
                        a[e] = gp_term(O.t, p.x);
                        b[e] = gp_term(I.t, p.y);
                    }
#pragma unroll
                    for (int e = 0; e < GL_LIST / GL_T; e++) {
                        const u32 x = a[e].z + b[e].z - sub;
                        const u64 v = gp_mul<RING>(a[e].x, a[e].y, b[e].x, b[e].y);
                        if (tid + e * GL_T < n && x < width) ring_atomic_acc<RING>(acc + x, v);
                    }
                });
                emit(width, [&](u32 c) { return w0 + c; }, w0 + width >= span);
                __syncthreads();  // the next round clears the cells
            }
        }
        if (mine && tid == 0) {
            C.gp_u[t] = done;
            atomicAdd(&C.gp_usum[t >> GP_USUM_LOG], done);
        }
        if (round >= own && tid == 0) s_tn[par] = tk;
        __syncthreads();
        d0 = d1;
        t = t1;
        t1 = round < own ? blockIdx.x + round * G : own * G + (i64)uniform32(s_tn[par]);
        d1 = item(t1);
        round++;
        par ^= 1u;
    }
}

// ---------------------------------------------------------------------------
// k_gp_f64: FP64 work items.  Every monomial's products are added left to
// right in row-major order, so one wave takes a whole work item and adds one
// row at a time: the LDS additions of a wave are carried out in the order it
// issues them, none waits for another, and a row meets a monomial at most once.
// Rows ascend (f's groups are the outer ones); of a block with more than 64
// columns the last ones come first, since a monomial's later rows meet it in
// earlier columns.  FC: LDS cells of a wave (a work item's key span).
// ---------------------------------------------------------------------------
// A piece: up to 64 rows, a lane each, read across lanes one after another
// (scalar loads would share their wait counter with the LDS additions), and
// up to 64 columns, a lane each.
struct GpRows {
    u32x3 a, b;
    u32 cols, rows;  // 0 rows: no more pieces
};

template <int FC>
__global__ __launch_bounds__(64) void k_gp_f64(Ctx C) {
    __shared__ __align__(16) double acc[FC];
    const u32 lane = threadIdx.x;
    for (u32 c = lane; c < (u32)FC; c += 64) acc[c] = 0.0;
    const i64 nt = (i64)uniform32(C.gp_sbit[C.gp_nsb]), G = gridDim.x;
    const i64 own = max((i64)1, nt / G / 2);
    i64 t = blockIdx.x, round = 1;
    int qc = -1;
    u32 S = 1;
    GpOperand O, I;
    const u32 *lut = nullptr;
    GpItem it{};
    if (t < nt) it = C.gp_item[t];
    while (t < nt) {
        const int q = (int)uniform32((u32)it.q);
        const u32 B0 = uniform32(it.bin_lo), B1 = uniform32(it.bin_hi);
        const u64 off = (u64)uniform64((i64)it.off);
        if (q != qc) {
            const DevSeg &s = C.segs[q];
            const int bq = (int)uniform32(s.gp.bq);
            S = uniform32(s.gp.S);
            O = gp_operand(C, s, bq, 0);
            I = gp_operand(C, s, bq, 1);
            lut = C.gp_lut + uniform64(s.gp.lut);
            qc = q;
        }
        u32 tk = 0;
        if (round >= own && lane == 0) tk = atomicAdd(&C.counters[CNT_GP_REDUCE], 1u);
        const u32 base = B0 * S, span = (B1 - B0) * S;
        // outer groups, 64 at a time, a lane each: prefix and rows are loaded
        // two steps ahead, the columns one step ahead
        GpOuter c1{}, c2{};
        auto fetch = [&](u32 g) {
            GpOuter o{};
            const u32 at = min(g + lane, O.groups);
            o.p = g + lane < O.groups ? gload(O.pfx + at) : ~0u;
            o.i0 = gload(O.start + at);
            o.rows = gload(O.start + min(at + 1, O.groups));
            return o;
        };
        u32 g = 0;
        c1 = fetch(0);
        gp_cols(lut, c1.p, B0, B1, c1.j0, c1.nc);
        c2 = fetch(64);
        u64 todo = 0;
        bool more = true;
        GpOuter cur{};
        u32 i0 = 0, R = 0, j0 = 0, N = 0, r = 0;
        i32 cc = -1;
        auto next = [&](GpRows &p) {
            p.rows = 0;
            if (r >= R) {
                r = 0;
                cc -= 64;
                if (cc < 0) {
                    while (!todo && more) {
                        cur = c1;
                        todo = __ballot(cur.nc != 0);
                        g += 64;
                        more = g < O.groups;
                        if (more) {
                            c1 = c2;
                            gp_cols(lut, c1.p, B0, B1, c1.j0, c1.nc);
                            c2 = fetch(g + 64);
                        }
                    }
                    if (!todo) {  // no more pieces, now and in every later call
                        R = 0;
                        cc = -1;
                        return;
                    }
                    const int l = (int)__ffsll((unsigned long long)todo) - 1;
                    todo &= todo - 1;
                    i0 = (u32)__builtin_amdgcn_readlane((int)cur.i0, l);
                    R = (u32)__builtin_amdgcn_readlane((int)cur.rows, l) - i0;
                    j0 = (u32)__builtin_amdgcn_readlane((int)cur.j0, l);
                    N = (u32)__builtin_amdgcn_readlane((int)cur.nc, l);
                    cc = (i32)((N - 1) & ~63u);
                }
            }
            p.rows = min(R - r, 64u);
            p.cols = min(N - (u32)cc, 64u);
            p.b = gp_term((const GpTerm *)((const char *)I.t + (j0 + (u32)cc) * (u32)sizeof(GpTerm)),
                          lane * (u32)sizeof(GpTerm));
            p.a = gp_term((const GpTerm *)((const char *)O.t + (i0 + r) * (u32)sizeof(GpTerm)), lane * (u32)sizeof(GpTerm));
            r += 64;
        };
        auto run = [&](const GpRows &p) {
            const bool in = lane < p.cols;
            const double b = __longlong_as_double((long long)(((u64)p.b.y << 32) | p.b.x));
            const u32 kb = p.b.z - base;
            auto row = [&](u32 u) {
                const u64 a = ((u64)(u32)__builtin_amdgcn_readlane((int)p.a.y, (int)u) << 32) |
                              (u32)__builtin_amdgcn_readlane((int)p.a.x, (int)u);
                const double v = __longlong_as_double((long long)a) * b;
                unsafeAtomicAdd(&acc[(u32)__builtin_amdgcn_readlane((int)p.a.z, (int)u) + kb], v);
            };
            if (in) {
                u32 u = 0;
                for (; u + 4 <= p.rows; u += 4) {
                    row(u);
                    row(u + 1);
                    row(u + 2);
                    row(u + 3);
                }
                for (; u < p.rows; u++) row(u);
            }
        };
        GpRows p0, p1, p2;
        next(p0);
        next(p1);
        while (p0.rows) {
            next(p2);
            run(p0);
            if (!p1.rows) break;
            next(p0);
            run(p1);
            if (!p2.rows) break;
            next(p1);
            run(p2);
        }
        // the next work item's descriptor
        const i64 tn = round < own ? (i64)blockIdx.x + round * G : own * G + (i64)uniform32(tk);
        GpItem nx{};
        if (tn < nt) nx = C.gp_item[tn];
        u32 done = 0;
        // four cells of a lane at a time (a sum is never -0: it started at +0)
        for (u32 c0 = 0; c0 < span; c0 += 256) {
            ulonglong2 x[2];
#pragma unroll
            for (int e = 0; e < 2; e++) x[e] = *(ulonglong2 *)&acc[c0 + e * 128 + lane * 2];
            if (!__ballot((x[0].x | x[0].y | x[1].x | x[1].y) != 0)) continue;
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const u32 c = c0 + e * 128 + lane * 2;
                *(ulonglong2 *)&acc[c] = make_ulonglong2(0, 0);
                const u64 b0 = __ballot(x[e].x != 0), b1 = __ballot(x[e].y != 0);
                u64 at = off + done + mbcnt(b0) + mbcnt(b1);
                if (x[e].x) {
                    C.gp_rkey[at] = c;
                    C.gp_rcoef[at] = x[e].x;
                    at++;
                }
                if (x[e].y) {
                    C.gp_rkey[at] = c + 1;
                    C.gp_rcoef[at] = x[e].y;
                }
                done += (u32)__popcll(b0) + (u32)__popcll(b1);
            }
        }
        if (lane == 0) {
            C.gp_u[t] = done;
            atomicAdd(&C.gp_usum[t >> GP_USUM_LOG], done);
        }
        t = tn;
        it = nx;
        round++;
    }
}

// ---------------------------------------------------------------------------
// k_gp_copy: a workgroup takes a run of consecutive work items; its waves share
// the terms of a large one and take the small ones in turn.  The result offset of the first one is the sum of the term counts of
// the product's earlier ones (gp_usum holds them per 2^GP_USUM_LOG items; every
// wave adds them up for itself).
// ---------------------------------------------------------------------------
constexpr int GC_T = 256;
constexpr int GC_B = 4;  // terms per lane per batch

__device__ inline u64 gp_range_sum(const u32 *v, i64 a, i64 b) {
    u64 x = 0;
    for (i64 i = a + (threadIdx.x & 63); i < b; i += 64) x += v[i];
    return x;
}

// The fields of one product that placing its terms takes.
struct GpOut {
    u64 *hk, *hc;
    const u64 *box;
    i64 cap, last;
    u64 lo_key;
    const VarParam *vp;
    Div32 sd;
    int d, nvars;
};

// Term at of h: cell x of the work item that starts at bin b.
__device__ inline void gp_put(const GpOut &o, i64 at, u32 b, u32 x, u64 coef) {
    if (at >= o.cap) return;
    u32 hi = div32(x, o.sd);
    u32 low = x - hi * o.sd.d;
    hi += b;
    u64 key = o.lo_key;
    for (int v = o.nvars - 1; v >= 0; v--) {
        const Div32 dv{uniform32(o.vp[v].rdiv.m), uniform32(o.vp[v].rdiv.s1), uniform32(o.vp[v].rdiv.s2),
                       uniform32(o.vp[v].rdiv.d)};
        const u32 y = v >= o.d ? low : hi;
        const u32 z = div32(y, dv);
        key += (u64)(y - z * dv.d) << uniform32(o.vp[v].shift);
        if (v >= o.d) low = z;
        else hi = z;
    }
    o.hk[at] = key;
    o.hc[at] = coef;
}

__global__ __launch_bounds__(GC_T) void k_gp_copy(Ctx C) {
    const i64 nt = (i64)uniform32(C.gp_sbit[C.gp_nsb]);
    const u32 lane = threadIdx.x & 63, w = uniform32(threadIdx.x >> 6);
    constexpr u32 NW = GC_T / 64;
    const i64 t0 = nt * blockIdx.x / gridDim.x, t1 = nt * (blockIdx.x + 1) / gridDim.x;
    if (t0 >= t1) return;
    int q = (int)uniform32((u32)C.gp_item[t0].q), qc = -1;
    u64 at0;
    {
        const i64 f = (i64)uniform32(C.gp_sbit[C.segs[q].gp.sb_first]);
        const i64 m = (i64)1 << GP_USUM_LOG;
        const i64 f1 = min((f + m - 1) & ~(m - 1), t0), g1 = max(t0 & ~(m - 1), f1);
        u64 x = gp_range_sum(C.gp_u, f, f1) + gp_range_sum(C.gp_u, g1, t0);
        if (g1 > f1) x += gp_range_sum(C.gp_usum, f1 >> GP_USUM_LOG, g1 >> GP_USUM_LOG);
        at0 = (u64)uniform64((i64)wave_sum_u64(x));
    }
    GpOut o{};
    GpItem ci{};
    u32 cu = 0;
    for (i64 t = t0; t < t1; t++) {
        const u32 l = (u32)(t - t0) & 63;
        if (l == 0) {  // descriptors and counts of the next 64 work items, a lane each
            const i64 i = min(t + lane, t1 - 1);
            ci = C.gp_item[i];
            cu = C.gp_u[i];
        }
        const u32 bin_lo = (u32)__builtin_amdgcn_readlane((int)ci.bin_lo, (int)l);
        const u32 bin_hi = (u32)__builtin_amdgcn_readlane((int)ci.bin_hi, (int)l);
        q = __builtin_amdgcn_readlane(ci.q, (int)l);
        const u64 off = ((u64)(u32)__builtin_amdgcn_readlane((int)(ci.off >> 32), (int)l) << 32) |
                        (u32)__builtin_amdgcn_readlane((int)(u32)ci.off, (int)l);
        const u32 u = (u32)__builtin_amdgcn_readlane((int)cu, (int)l);
        if (q != qc) {
            const DevSeg &s = C.segs[q];
            if (qc >= 0) at0 = 0;
            o.hk = (u64 *)uniform64((i64)s.hk);
            o.hc = (u64 *)uniform64((i64)s.hc);
            o.cap = uniform64(s.cap);
            o.lo_key = (u64)uniform64((i64)s.lo_key);
            o.vp = C.vars + uniform64(s.var_off);
            o.sd = Div32{uniform32(s.nb_div.m), uniform32(s.nb_div.s1), uniform32(s.nb_div.s2), uniform32(s.nb_div.d)};
            o.d = (int)uniform32(s.gp.d);
            o.nvars = C.nvars;
            o.box = uniform32(s.gp.K) ? C.box + uniform64(s.stage_base) : nullptr;
            o.last = (i64)uniform32(C.gp_sbit[uniform64(s.gp.sb_first) + uniform64(s.gp.nsb)]) - 1;
            qc = q;
        }
        const bool share = !o.box && u > 64 * GC_B;
        if (!share && (l & (NW - 1)) != w) {
            // another wave's
        } else if (o.box) {
            // the non-zero cells of the degree box
            const u64 *cell = o.box + (i64)bin_lo * o.sd.d;
            const u32 n = (bin_hi - bin_lo) * o.sd.d;
            u64 at = at0;
            for (u32 c0 = 0; c0 < n && u; c0 += 64 * GC_B) {
                u64 v[GC_B];
#pragma unroll
                for (int e = 0; e < GC_B; e++) v[e] = cell[min(c0 + e * 64 + lane, n - 1)];
#pragma unroll
                for (int e = 0; e < GC_B; e++) {
                    const bool in = v[e] && c0 + e * 64 + lane < n;
                    const u64 bal = __ballot(in);
                    if (in) gp_put(o, (i64)(at + mbcnt(bal)), bin_lo, c0 + e * 64 + lane, v[e]);
                    at += (u64)__popcll(bal);
                }
            }
        } else {
            const u32 *rk = C.gp_rkey + off;
            const u64 *rc = C.gp_rcoef + off;
            for (u32 r0 = share ? w * (64 * GC_B) : 0u; r0 < u; r0 += share ? NW * 64 * GC_B : 64 * GC_B) {
                u32 ck[GC_B];
                u64 cv[GC_B];
#pragma unroll
                for (int e = 0; e < GC_B; e++) {
                    const u32 r = min(r0 + e * 64 + lane, u - 1);
                    ck[e] = rk[r];
                    cv[e] = rc[r];
                }
#pragma unroll
                for (int e = 0; e < GC_B; e++) {
                    const u32 r = r0 + e * 64 + lane;
                    if (r < u) gp_put(o, (i64)(at0 + r), bin_lo, ck[e], cv[e]);
                }
            }
        }
        at0 += u;
        if (t == o.last && threadIdx.x == 0) *C.segs[q].n_out = (i64)at0;
    }
}

}  // namespace pm
