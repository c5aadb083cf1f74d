// The replica step: the fused step of the renewal tau-leap (FlashSpread,
// arXiv 2604.22092, Algorithm 3) for unit-weight sims of several replicas
// with constant shedding and fixed steps.  Same draws, states, ages and counts
// as step_body (fs_step.hpp).
//
// What bounds it: with one lane per (node, replica) unit, each of a node's R
// lanes loads the same columns and extracts one bit of the same bitmap word,
// and every 64-unit chunk pays a whole wavefront of Philox rounds for the few
// lanes that draw: 269 vector instructions per chunk, issue-bound at 3.3 times
// the step's memory floor.  So the two phases use different lane mappings:
//  gather  one lane per node and block of W = 2^LGW replicas: a column is
//          loaded once, and one load of W bits brings W replicas' infectivity.
//          The bits of eight edges are added by carry-save adders on bit
//          planes (one three-input logic operation per sum or carry), and
//          the planes are spread into one byte per unit in LDS;
//  units   one lane per unit, chunk after chunk: state, age, hazard table,
//          and the byte.  Units that draw are packed into an LDS queue, and
//          every 64 of them get one wavefront of Philox and the comparison.
// A wavefront owns a group of W chunks (64 W consecutive units).
//
// Measured (traced step launches, one MI355X, general step / replica step):
// Barabasi-Albert m = 4, N = 3e5, 16 replicas, FP32 56.0 / 29.5 us over 300 steps
// of an epidemic and 52 / 27 with few infectious units (111 vector instructions
// per chunk); m = 5, N = 1e6, 16 replicas 155 / 74 us; Erdos-Renyi mean degree 10,
// N = 3e4, 64 replicas 23.4 / 11.4 us.  At m = 4 wavefronts wait for memory 42% of
// their cycles and to issue 32%, and move 2.6 TB/s: what is left there is the
// latency of the chain columns -> bits -> bytes -> units (5 of 14 us of a
// wavefront's life in the gather, one L1 lookup per edge and compute unit and
// cycle) and the issue of the draws; at N = 1e6, the state and age traffic.
#pragma once

#include "fs_step.hpp"

namespace fsk {

// Rows have at most REPS_MAX_DEG light edges: seven planes hold the count, and
// it fits the unit's byte.
constexpr uint32_t REPS_TPB = STREAM_TPB;
// Chunks whose loads are in flight together, and wavefronts per SIMD, by group
// width.  Groups of 4 and of 8 chunks fit 96 vector registers with few spills or
// none, so five wavefronts share a SIMD: the 5000 groups of regular d = 6, N =
// 2e4, R = 64 run at once (compact, 11.3 us per step with four, 9.3 with five).
// Groups of 16 need the four chunks' loads in flight more (Barabasi-Albert 4, N =
// 3e5, R = 16 in groups of 16: 33.7 us, two chunks and five wavefronts 35.2).  Draws queued: at
// most 63 left over plus every unit of those chunks.
constexpr int reps_ns(int lgw) { return lgw == 3 ? 2 : 4; }
constexpr int reps_waves(int lgw) { return lgw == 4 ? 4 : 5; }
// Queue entry: the unit in its group (10 bits), its state, and whether the
// first word is the age of a unit whose hazard is yet to be evaluated.
constexpr uint32_t REPS_EVAL = 0x80000000u;

template <int LGW>
struct RepsShared {
    static constexpr int W = 1 << LGW;
    static constexpr int NW = REPS_TPB / 64;
    uint32_t cnt[4 * 64];          // transitions per (replica, compartment left)
    uint32_t press[NW][16 * W];    // one byte per unit of the group
    uint2 q[NW][64 + reps_ns(LGW) * 64];        // (rate or age, unit in the group | state << 10 | REPS_EVAL)
    uint32_t id[NW][64];           // the caller's node id of each gather lane
    uint32_t flip[NW][2 * W];      // infectivity bits changed by the draws
    uint32_t pq[NW][PUSHQ];        // pushes of binned rows
    uint32_t pb[NW][64], px[NW][64];
};

__device__ __forceinline__ uint32_t add_sum(uint32_t a, uint32_t b, uint32_t c) { return a ^ b ^ c; }
__device__ __forceinline__ uint32_t add_carry(uint32_t a, uint32_t b, uint32_t c) { return (a & b) | (c & (a | b)); }

// A += the eight one-bit numbers x (bit r of every word belongs to replica r);
// plane p of A holds bit p of the sums.
__device__ __forceinline__ void add8(uint32_t (&A)[7], const uint32_t (&x)[8])
{
    const uint32_t s0 = add_sum(x[0], x[1], x[2]), c0 = add_carry(x[0], x[1], x[2]);
    const uint32_t s1 = add_sum(x[3], x[4], x[5]), c1 = add_carry(x[3], x[4], x[5]);
    const uint32_t s2 = add_sum(x[6], x[7], s0), c2 = add_carry(x[6], x[7], s0);
    const uint32_t t = add_sum(c0, c1, c2), d0 = add_carry(c0, c1, c2);
    // ones: s1, s2 and A[0]; twos: t and the carry; fours: d0 and the carries
    const uint32_t a0 = A[0], e0 = add_carry(s1, s2, a0);
    A[0] = add_sum(s1, s2, a0);
    const uint32_t a1 = A[1], e1 = add_carry(t, e0, a1);
    A[1] = add_sum(t, e0, a1);
    const uint32_t a2 = A[2], e2 = add_carry(d0, e1, a2);
    A[2] = add_sum(d0, e1, a2);
    uint32_t c = e2;
#pragma unroll
    for (int p = 3; p < 7; ++p) {
        const uint32_t v = A[p];
        A[p] = v ^ c;
        c = v & c;
    }
}

// The W infectivity bits of one source for this lane's replica block, or 0
// where take is not set (no memory request).
template <int LGW>
__device__ __forceinline__ uint32_t block_bits(rsrc_t gbits, uint32_t col, int32_t lgR, uint32_t rep0, bool take)
{
    const uint32_t b = (col << lgR) + rep0;
    const int off = take ? (int)(b >> 3) : (int)OOB;
    if (LGW == 4) return __builtin_amdgcn_raw_buffer_load_b16(gbits, off, 0, 0);
    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b8(gbits, off, 0, 0);
    if (LGW == 3) return v;
    return __builtin_amdgcn_ubfe(v, b & 7u, 1u << LGW);
}

// The launch's arguments in constant memory.  Narrow groups read them in every
// part of the step through a pointer the compiler cannot follow (fresh_args), so
// it loads what the part uses there instead of holding all of them from the
// start on, spilled to vector lanes (73 of them, now 18).  With groups of 16 the
// later loads cost more than the spills (Barabasi-Albert 5, N = 1e6, R = 16: 87.8
// us held, 89.4 read anew).
typedef const __attribute__((address_space(4))) StepArgs* ArgsPtr;
template <int LGW>
__device__ __forceinline__ ArgsPtr fresh_args(ArgsPtr p)
{
    if (LGW < 4) asm volatile("" : "+s"(p));
    return p;
}

// The lane's number, formed where it is asked for: neither it nor an address
// formed from it is held through the whole walk.
__device__ __forceinline__ uint32_t fresh_lane()
{
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, in_vgpr(0u)));
}

template <int STORAGE, int LGW>
__device__ __forceinline__ void reps_body(ArgsPtr args, uint32_t step_off, RepsShared<LGW>& S, uint32_t block,
                                          uint32_t nblocks)
{
    const auto& a = *args;
    using state_t = typename Store<STORAGE>::state_t;
    using age_t = typename Store<STORAGE>::age_t;
    constexpr uint32_t W = 1u << LGW;
    constexpr int NW = RepsShared<LGW>::NW;
    constexpr int NS = reps_ns(LGW);
    constexpr int SUBS = (int)W / NS;
    static_assert(W >= NS, "a group holds at least one sub-batch");

    const uint32_t tid = threadIdx.x;
    const uint32_t lane0 = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t lgR = a.lgR;
    const uint32_t R = 1u << lgR;
    const int32_t lgNB = lgR - LGW;     // replica blocks per node (log2)
    const uint32_t rows = 64u >> lgNB;  // nodes per group
    const uint32_t total = (uint32_t)a.n << lgR;
    const uint32_t nchunks = (total + 63) >> 6;
    const uint32_t ngroups = (nchunks + W - 1) >> LGW;
    const rsrc_t tabr = make_rsrc(a.htab, a.htab_len * 16u);
    const float dt = a.dt;
    const uint8_t* press8 = (const uint8_t*)S.press[wave];

    for (uint32_t i = tid; i < 4 * R; i += REPS_TPB) S.cnt[i] = 0;
    if (lane0 < 2 * W) S.flip[wave][lane0] = 0;
    __syncthreads();

    uint32_t qn = 0; // queued draws (wave-uniform)

    uint32_t kk = 0;
    HubCtx H;
    H.on = a.hub_T != nullptr;
    H.n = 0;
    H.q = S.pq[wave];
    H.pb = S.pb[wave];
    H.px = S.px[wave];
    H.t_prev = H.t_cur = H.d_cur = H.d_clr = H.d_next = 0;
    H.base = H.on ? (uint32_t)a.hub_base << lgR : 0xFFFFFFFFu;
    H.tr = make_rsrc(a.hub_T, H.on ? 5u * a.hub_units * 4u : 0u);

    // the densest rows of a degree-sorted order come last: taken first, they
    // do not make the launch's tail
    for (uint32_t g0 = block * NW + wave; g0 < ngroups; g0 += nblocks * NW) {
        const auto& a = *fresh_args<LGW>(args);
        const uint32_t g = __builtin_amdgcn_readfirstlane(ngroups - 1u - g0);
        const uint32_t lane = fresh_lane();
        const uint32_t q = lane >> lgNB;
        const uint32_t rep0 = (lane & ((1u << lgNB) - 1u)) << LGW;
        const uint32_t u0 = g << (6 + LGW);
        const uint32_t nvalid = min(64u * W, total - u0);
        const uint32_t n0 = u0 >> lgR;
        const uint32_t node = n0 + q;
        const bool valid = node < (uint32_t)a.n;
        const rsrc_t str = make_rsrc((state_t*)a.state + u0, nvalid * (uint32_t)sizeof(state_t));
        const rsrc_t agr = make_rsrc((age_t*)a.age + u0, nvalid * (uint32_t)sizeof(age_t));

        // ---- loads that need no other load's result: the first chunks'
        // state and age, the first sixteen columns of the rows
        uint32_t xs[NS], as[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            xs[i] = BufIO<state_t>::ld(str, (uint32_t)i * 64u + lane);
            as[i] = BufIO<age_t>::ld(agr, (uint32_t)i * 64u + lane);
        }
        // (the step index too, by a vector load: every scalar wait before it is
        // needed would wait for a scalar one)
        const auto ctl = __builtin_amdgcn_raw_buffer_load_b64(make_rsrc(a.ctl, 8u), 0, 0, 0);
        uint32_t base, ud;
        uint32_t id = node;
        uint32_t d = 0; // this lane's light edges
        if (a.udeg >= 0) {
            ud = (uint32_t)a.udeg;
            base = g * rows * ud;
        } else {
            const uint2 meta = a.chunk_meta[g];
            base = __builtin_amdgcn_readfirstlane(meta.x);
            ud = __builtin_amdgcn_readfirstlane(meta.y);
            id = valid ? (uint32_t)a.orig_id[node] : 0u;
        }
        const bool mixed = ud == MIXED_CHUNK;
        if (mixed) {
            d = valid ? (uint32_t)a.ldeg[node] : 0u;
            if (d == HEAVY_ROW) d = 0u;
        } else {
            d = valid ? ud : 0u;
        }
        const unsigned long long leads = __ballot((lane & ((1u << lgNB) - 1u)) == 0u);
        // The columns of edges j0 .. j0 + 7 of the rows: where every row has
        // ud light edges, slot j of row q at j * rows + q; else (binned rows
        // hold no light edge) run j lists the j-th edge of the rows with more
        // than j edges, from slot `base` on, which moves past the runs read.
        auto columns = [&](uint32_t j0, uint32_t (&c)[8]) {
            if (!mixed) {
                const rsrc_t cr = make_rsrc(a.col_t + base, ud * rows * 4u);
#pragma unroll
                for (int j = 0; j < 8; ++j) c[j] = ld32(cr, ((j0 + (uint32_t)j) * rows + q) << 2);
                return;
            }
            const unsigned long long below = leads & ((1ull << (q << lgNB)) - 1ull);
            uint32_t idx[8], n8 = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const unsigned long long m = __ballot(d > j0 + (uint32_t)j);
                idx[j] = n8 + (uint32_t)__popcll(m & below);
                n8 += (uint32_t)__popcll(m & leads);
            }
            const rsrc_t cr = make_rsrc(a.col_t + base, n8 * 4u);
#pragma unroll
            for (int j = 0; j < 8; ++j) c[j] = ld32(cr, d > j0 + (uint32_t)j ? idx[j] << 2 : OOB);
            base += n8;
        };
        auto any = [&](uint32_t j0) { return __ballot(d > j0) != 0ull; };
        uint32_t c0[8], c1[8];
        bool m0 = any(0u), m1 = any(8u); // the first and second eight hold edges
        if (m0) columns(0u, c0);
        if (m1) columns(8u, c1);

        // ---- loads that need the first ones: the step index's bitmap, the
        // hazard-table entries of the first chunks
        // (E and I lanes; the others read nothing and get 0)
        float t0[NS], tE[NS], tI[NS];
        auto load_table = [&]() {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const float mf = rintf(age_units(age_from_raw<age_t>(as[i])) * a.htab_inv);
                const bool want = xs[i] - 1u < 2u && mf < (float)a.htab_len;
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(tabr, want ? (int)((uint32_t)mf << 4) : (int)OOB, 0, 0);
                t0[i] = __uint_as_float(t[0]);
                tE[i] = __uint_as_float(t[1]);
                tI[i] = __uint_as_float(t[2]);
            }
        };
        const unsigned long long k = (((unsigned long long)__builtin_amdgcn_readfirstlane(ctl[1]) << 32) |
                                      __builtin_amdgcn_readfirstlane(ctl[0])) + step_off;
        kk = (uint32_t)k;
        const rsrc_t gbits = make_rsrc((k & 1) ? a.iota1 : a.iota0, ((total + 511u) >> 9) << 6);
        if (H.on) {
            const uint32_t HU = a.hub_units;
            const uint32_t k2 = kk & 1u;
            // k mod 3 (2^32 = 1 mod 3)
            const uint32_t k3 = ((uint32_t)(k >> 32) % 3u + kk % 3u) % 3u;
            H.t_prev = in_vgpr((k2 ^ 1u) * HU);
            H.t_cur = in_vgpr(k2 * HU);
            H.d_cur = in_vgpr((2u + k3) * HU);
            H.d_next = in_vgpr((2u + (k3 + 1u) % 3u) * HU);
            H.d_clr = in_vgpr((2u + (k3 + 2u) % 3u) * HU);
        }
        load_table();

        // ---- gather: one lane per (node, replica block), sixteen edges at a
        // time; the next columns are on their way while these bits are
        uint32_t A[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
        uint32_t maxd = 0; // edges counted per row, at most (wave-uniform)
        for (uint32_t j0 = 0; m0; j0 += 16) {
            uint32_t x0[8], x1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x0[j] = block_bits<LGW>(gbits, c0[j], lgR, rep0, d > j0 + (uint32_t)j);
            if (m1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x1[j] = block_bits<LGW>(gbits, c1[j], lgR, rep0, d > j0 + 8u + (uint32_t)j);
            }
            const bool two = m1;
            m0 = any(j0 + 16u);
            m1 = any(j0 + 24u);
            if (m0) columns(j0 + 16u, c0);
            if (m1) columns(j0 + 24u, c1);
            add8(A, x0);
            if (two) add8(A, x1);
            maxd = j0 + (two ? 16u : 8u);
        }
        if (!mixed) maxd = ud;
        // planes to bytes: four bits to the low bits of four bytes by one
        // 24-bit multiplication (replica r of the block is byte r)
        uint32_t by[W / 4] = {};
#pragma unroll
        for (int p = 0; p < 7; ++p) {
            if ((maxd >> p) == 0u) break;
#pragma unroll
            for (uint32_t w = 0; w < W / 4; ++w)
                by[w] += (__umul24(__builtin_amdgcn_ubfe(A[p], 4u * w, 4u), 0x204081u) & 0x01010101u) << p;
        }
#pragma unroll
        for (uint32_t w = 0; w < W / 4; ++w) S.press[wave][lane * (W / 4) + w] = by[w];
        S.id[wave][lane] = id;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        const bool hub_group = H.on && u0 + 64u * W > H.base;
        uint32_t w_lo = 0, w_hi = 0; // lane c: the next infectivity word of chunk c, before the draws

        // the queued draws [qn - m, qn), one per lane (m <= 64)
        auto draw = [&](uint32_t m) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            qn -= m;
            bool fire = false;
            uint32_t l = 0, x = 0;
            if (lane < m) {
                const uint2 e = S.q[wave][qn + lane];
                l = e.y & 1023u;
                x = (e.y >> 10) & 3u;
                // (an age the table does not hold: its hazard is evaluated here)
                float lam = __uint_as_float(e.x);
                if (e.y & REPS_EVAL) lam = unit_hazard(a.hz_dev, a.same_kind, lam, x == (uint32_t)ST_I);
                const uint32_t nid = S.id[wave][l >> LGW];
                uint32_t k0 = __builtin_amdgcn_readfirstlane(a.key0), k1 = __builtin_amdgcn_readfirstlane(a.key1),
                         ks = __builtin_amdgcn_readfirstlane(kk);
                asm volatile("" : "+s"(k0), "+s"(k1), "+s"(ks));
                const uint32_t w = fsd::philox4x32_10(make_uint4(nid, ks, l & (R - 1u), 0u), k0, k1).x >> 8;
                fire = fsd::bernoulli((float)w * 0x1p-24f, lam * dt);
            }
            const unsigned long long fm = __ballot(fire);
            if (fm == 0ull) return;
            // the transitions: state, age 0 (after the chunk's age store:
            // stores of one wavefront to one address keep their order)
            BufIO<state_t>::st(str, fire ? l : OOB_ELEM, x + 1u);
            BufIO<age_t>::st(agr, fire ? l : OOB_ELEM, 0u);
            if (fire) {
                atomicAdd(&S.cnt[(l & (R - 1u)) * 4u + x], 1u);                         // LDS
                if (x != (uint32_t)ST_S) atomicXor(&S.flip[wave][l >> 5], 1u << (l & 31u)); // LDS
            }
            if (H.on) {
                const bool push = fire && x != (uint32_t)ST_S;
                const unsigned long long pm = __ballot(push);
                if (pm != 0ull) {
                    const uint32_t cnt = (uint32_t)__popcll(pm);
                    if (H.n + cnt > PUSHQ) flush_pushes(a, H, lane);
                    if (push)
                        H.q[H.n + (uint32_t)__popcll(pm & ((1ull << lane) - 1ull))] =
                            (u0 + l) | (x == (uint32_t)ST_I ? 0x80000000u : 0u);
                    H.n += cnt;
                }
            }
        };

        // ---- units: one lane per unit, NS chunks at a time
#pragma unroll 1
        for (int sub = 0; sub < SUBS; ++sub) {
            const uint32_t cb = (uint32_t)sub * NS;
            // the next chunks' loads, then the ages' stores: what is waited
            // for below was issued before the stores
            uint32_t xn[NS], an[NS];
            if (sub + 1 < SUBS) {
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    xn[i] = BufIO<state_t>::ld(str, (cb + NS + (uint32_t)i) * 64u + lane);
                    an[i] = BufIO<age_t>::ld(agr, (cb + NS + (uint32_t)i) * 64u + lane);
                }
            }
            uint32_t ht[NS], hd[NS];
            if (hub_group) {
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const uint32_t l = (cb + (uint32_t)i) * 64u + lane;
                    const bool hub = l < nvalid && u0 + l >= H.base;
                    const uint32_t h = hub ? u0 + l - H.base : 0u;
                    ht[i] = ld32(H.tr, hub ? (H.t_prev + h) << 2 : OOB);
                    hd[i] = ld32(H.tr, hub ? (H.d_cur + h) << 2 : OOB);
                    if (LGW < 4) ht[i] += hd[i]; // (one register each)
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NS; ++i)
                BufIO<age_t>::st(agr, (cb + (uint32_t)i) * 64u + lane,
                                 age_to_raw(age_next(age_from_raw<age_t>(as[i]), dt)));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const uint32_t c = cb + (uint32_t)i;
                const uint32_t l = c * 64u + lane;
                const uint32_t x = xs[i];
                const float ag = age_units(age_from_raw<age_t>(as[i]));
                float p = (float)press8[l];
                if (hub_group) {
                    const bool hub = l < nvalid && u0 + l >= H.base;
                    if (__ballot(hub) != 0ull) {
                        const uint32_t h = hub ? u0 + l - H.base : 0u;
                        const uint32_t pp = LGW < 4 ? ht[i] : ht[i] + hd[i];
                        st32(H.tr, hub ? (H.t_cur + h) << 2 : OOB, pp);
                        st32(H.tr, hub ? (H.d_clr + h) << 2 : OOB, 0u);
                        if (hub) p = (float)pp;
                    }
                }
                // rate: beta * pressure for S, the hazard for E and I, 0 for R
                const float lam = x == (uint32_t)ST_S ? a.beta * p : x == (uint32_t)ST_I ? tI[i] : tE[i];
                const bool miss = x - 1u < 2u && t0[i] != ag;
                const unsigned long long mI = __ballot(x == (uint32_t)ST_I);
                w_lo = lane == c ? (uint32_t)mI : w_lo;
                w_hi = lane == c ? (uint32_t)(mI >> 32) : w_hi;
                uint32_t word = __float_as_uint(lam), code = l | (x << 10);
                bool need = lam > 0.0f;
                if (__ballot(miss) != 0ull) { // (ages a state load set, or past the table)
                    if (miss) {
                        word = __float_as_uint(ag);
                        code |= REPS_EVAL;
                        need = true;
                    }
                }
                const unsigned long long m = __ballot(need);
                if (need)
                    S.q[wave][qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                        make_uint2(word, code);
                qn += (uint32_t)__popcll(m);
            }
            if (sub + 1 < SUBS) {
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    xs[i] = xn[i];
                    as[i] = an[i];
                }
                load_table();
            }
            // whole wavefronts of draws, and after the last chunks the rest
            const uint32_t least = sub + 1 < SUBS ? 64u : 1u;
            while (qn >= least) draw(min(qn, 64u));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the next infectivity words of the group's chunks
        if (lane < W) {
            const uint32_t f0 = S.flip[wave][2 * lane], f1 = S.flip[wave][2 * lane + 1];
            // (a zero made here: one held through the walk is spilled to scratch
            // memory, and a kernel with scratch starts later)
            const uint32_t zero = in_vgpr(0u);
            S.flip[wave][2 * lane] = zero;
            S.flip[wave][2 * lane + 1] = zero;
            const uint32_t c = (g << LGW) + lane;
            const auto& f = *fresh_args<LGW>(args);
            if (c < nchunks) ((uint2*)((kk & 1u) ? f.iota0 : f.iota1))[c] = make_uint2(w_lo ^ f0, w_hi ^ f1);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    const auto& b = *fresh_args<LGW>(args);
    if (H.on && H.n > 0) flush_pushes(b, H, fresh_lane());

    // this workgroup's transitions; the reduce kernel turns their sums into
    // counts (the counts before the step, plus and minus the transitions)
    __syncthreads();
    uint32_t* out = b.part + ((size_t)step_off * nblocks + block) * (4 * R);
    for (uint32_t i = wave * 64u + fresh_lane(); i < 4 * R; i += REPS_TPB) out[i] = S.cnt[i];
}

} // namespace fsk
