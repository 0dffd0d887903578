// A product of a few thousand term pairs on its own (SEG_TINY): one workgroup,
// one launch.  Included by pm_kernels.hip.
//
// The other paths take 4 to 12 launches of 5 to 20 us for such a product, most
// of it latency.  Here one workgroup forms every pair's compressed key, sorts
// keys and pair indices in LDS (stable 6-bit digits, ranks within a wave by
// ballots), multiplies in sorted order and sums each run of equal keys from its
// first pair on, which is row-major order: FP64 sums are those of the pair-index
// sort bit by bit.  Latency bounds it (a chain of barriers per digit): 57 x 61
// random FP64 terms in 6 variables took 12 launches and 121 us, now 31 us here
// and 55 us with the validation before it.
#pragma once

namespace pm {

constexpr int TINY_T = 1024;
constexpr int TINY_NW = TINY_T / 64;
constexpr int TINY_E = TINY_PAIRS / TINY_T;  // pairs of a thread
constexpr int TINY_IDX = 13;                 // bits of a pair index
static_assert(TINY_PAIRS == 1 << TINY_IDX, "pair indices");
constexpr int TINY_D = 6;  // digit bits: five passes over the 30-bit keys of 6 variables (5 bits, six passes: 33 us, 6: 31)

// zp, zn: per-call state to be cleared (no other kernel runs).
template <int RING>
__global__ __launch_bounds__(TINY_T) void k_tiny(Ctx C, u64 *zp, i64 zn) {
    __shared__ u64 s_x[TINY_PAIRS];                                 // key and pair index
    __shared__ __align__(16) unsigned char s_v[TINY_PAIRS * 8 + 16];  // operand keys, then products
    __shared__ u32 s_cnt[TINY_NW << TINY_D], s_w[TINY_NW];
    const u32 tid = threadIdx.x, lane = tid & 63, w = uniform32(tid >> 6);
    for (i64 i = tid; i < zn; i += TINY_T) zp[i] = 0;
    const DevSeg &s = C.segs[0];
    const u32 na = (u32)uniform64(s.na), nb = (u32)uniform64(s.nb), N = na * nb;
    const VarParam *vp = C.vars + uniform64(s.var_off);
    const int nv = C.nvars;
    const Div32 dnb{uniform32(s.nb_div.m), uniform32(s.nb_div.s1), uniform32(s.nb_div.s2), uniform32(s.nb_div.d)};
    u32 *ck = (u32 *)s_v;  // f's keys, then g's: na + nb <= TINY_PAIRS + 1
    for (u32 i = tid; i < na + nb; i += TINY_T) {
        const bool second = i >= na;
        const u64 k = second ? s.gk[i - na] : s.fk[i];
        u32 c = 0;
        for (int v = 0; v < nv; v++)
            c += (u32)(((k >> vp[v].shift) & vp[v].mask) - (second ? vp[v].ming : vp[v].minf)) * (u32)vp[v].stride;
        ck[i] = c;
    }
    __syncthreads();
    // a wave has consecutive pairs, a lane every 64th of them
    const u32 ne = (N + TINY_T - 1) / TINY_T, p0 = w * ne * 64 + lane;
    u64 x[TINY_E];
#pragma unroll
    for (u32 e = 0; e < (u32)TINY_E; e++) {
        x[e] = ~0ull;  // past the end: sorts last
        const u32 p = p0 + e * 64;
        if (e < ne && p < N) {
            const u32 r = div32(p, dnb);
            x[e] = ((u64)(ck[r] + ck[na + p - r * nb]) << TINY_IDX) | p;
        }
    }
    const u32 bits = uniform32((u32)s.bk_fs);  // of a key
    for (u32 sh = TINY_IDX; sh < TINY_IDX + bits; sh += TINY_D) {
        if (tid < (u32)TINY_NW << TINY_D) s_cnt[tid] = 0;
        __syncthreads();
        volatile u32 *cnt = s_cnt + (w << TINY_D);
        u32 rk[TINY_E];
#pragma unroll
        for (u32 e = 0; e < (u32)TINY_E; e++) {
            rk[e] = 0;
            if (e >= ne) continue;
            const u32 d = (u32)(x[e] >> sh) & ((1u << TINY_D) - 1);
            u64 same = ~0ull;
#pragma unroll
            for (int b = 0; b < TINY_D; b++) {
                const u64 m = __ballot((d >> b) & 1u);
                same &= (d >> b) & 1u ? m : ~m;
            }
            const u32 before = cnt[d], at = mbcnt(same);
            rk[e] = before + at;
            // (a wave's LDS accesses are carried out in order: every lane has read)
            if (at == 0) cnt[d] = before + (u32)__popcll(same);
        }
        __syncthreads();
        // first place of every digit and wave, digits first
        const u32 ci = ((tid & (TINY_NW - 1)) << TINY_D) + (tid >> 4);
        const bool in = tid < (u32)TINY_NW << TINY_D;
        const u32 c = in ? s_cnt[ci] : 0u;
        const u32 inc = wave_scan_dpp(c);
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        {
            const u32 wi = wave_scan_dpp(lane < (u32)TINY_NW ? s_w[lane & (TINY_NW - 1)] : 0u);
            const u32 wp = w ? (u32)__builtin_amdgcn_readlane((int)wi, (int)w - 1) : 0u;
            if (in) s_cnt[ci] = wp + inc - c;
        }
        __syncthreads();
#pragma unroll
        for (u32 e = 0; e < (u32)TINY_E; e++)
            if (e < ne) s_x[cnt[(u32)(x[e] >> sh) & ((1u << TINY_D) - 1)] + rk[e]] = x[e];
        __syncthreads();
#pragma unroll
        for (u32 e = 0; e < (u32)TINY_E; e++)
            if (e < ne) x[e] = s_x[p0 + e * 64];
    }
    if (bits == 0) {  // one output monomial: in order already
#pragma unroll
        for (u32 e = 0; e < (u32)TINY_E; e++)
            if (e < ne) s_x[p0 + e * 64] = x[e];
    }
    __syncthreads();  // (also: the operand keys have been read)
    u64 *val = (u64 *)s_v;
#pragma unroll
    for (u32 e = 0; e < (u32)TINY_E; e++) {
        if (e >= ne || p0 + e * 64 >= N) continue;
        const u32 p = (u32)x[e] & (TINY_PAIRS - 1), r = div32(p, dnb);
        val[p0 + e * 64] = ring_mul<RING>(s.fc[r], s.gc[p - r * nb]);
    }
    __syncthreads();
    u64 sum[TINY_E];
    u32 em = 0, rk[TINY_E], before = 0;
#pragma unroll
    for (u32 e = 0; e < (u32)TINY_E; e++) {
        rk[e] = 0;
        sum[e] = 0;
        if (e >= ne) continue;
        const u32 at = p0 + e * 64;
        const u64 key = x[e] >> TINY_IDX;
        if (at < N && (at == 0 || s_x[at - 1] >> TINY_IDX != key)) {
            u64 y = val[at];
            for (u32 k = at + 1; k < N && s_x[k] >> TINY_IDX == key; k++) y = ring_add<RING>(y, val[k]);
            sum[e] = y;
            if (!ring_is_zero<RING>(y)) em |= 1u << e;
        }
        const u64 m = __ballot((em >> e) & 1u);
        rk[e] = before + mbcnt(m);
        before += (u32)__popcll(m);
    }
    if (lane == 0) s_w[w] = before;
    __syncthreads();
    const u32 wi = wave_scan_dpp(lane < (u32)TINY_NW ? s_w[lane & (TINY_NW - 1)] : 0u);
    const u32 wp = w ? (u32)__builtin_amdgcn_readlane((int)wi, (int)w - 1) : 0u;
    if (tid == 0) *s.n_out = (i64)(u32)__builtin_amdgcn_readlane((int)wi, 63);
    const i64 cap = s.cap;
#pragma unroll
    for (u32 e = 0; e < (u32)TINY_E; e++) {
        const i64 at = (i64)(wp + rk[e]);
        if (!((em >> e) & 1u) || at >= cap) continue;
        u64 key = s.lo_key;
        u32 y = (u32)(x[e] >> TINY_IDX);
        for (int v = nv - 1; v >= 0; v--) {
            const Div32 dv{uniform32(vp[v].rdiv.m), uniform32(vp[v].rdiv.s1), uniform32(vp[v].rdiv.s2),
                           uniform32(vp[v].rdiv.d)};
            const u32 z = div32(y, dv);
            key += (u64)(y - z * dv.d) << uniform32(vp[v].shift);
            y = z;
        }
        s.hk[at] = key;
        s.hc[at] = sum[e];
    }
}

}  // namespace pm
