// The Markovian engine (FlashSpread, arXiv 2604.22092, Section "Markovian
// engine", Algorithm "Markovian Engine: One Tau-Leaping Step") for gfx950.
//
// Rates are piecewise constant: S nodes beta * I_i (I_i: infectious
// in-neighbours, unit weights), E nodes sigma, I nodes gamma, R nodes 0.
// One step is two launches, inside a captured graph:
//   step   (dense, then sparse): one wavefront per workgroup folds the rate
//          partials of the previous launch into Lambda and max lambda (exact
//          integers) and takes tau = min(theta N / Lambda, p_max / max lambda,
//          tau_max) while the workgroup's states and influences are on their
//          way; every node with a positive rate draws and applies its
//          transition; then (Inertial Mode) each node whose infectiousness
//          changed adds +-1 to the pending influence of its out-neighbours
//          (integer atomics: exact and order-independent).  Pending, because
//          other workgroups still read the influences of this step.  Without
//          I -> S (SEIR, SIR) only susceptible targets are updated: no other
//          node reads its influence again;
//   rates  (dense): adds the pending changes to the influences (without I -> S
//          only to nodes still susceptible: one that leaves S in this step was
//          pushed to or not by who came first, and keeps the influence it left
//          with), or (Control Mode: many events in the step) recounts every
//          influence from the incoming CSR, and writes per-workgroup partials
//          (sum of S influences, max S influence, #E, #I) and counts; after a
//          step without transitions it keeps the old ones.
// Both modes give the same integer influences on every node that can still
// read them (every susceptible node; every node under SIS), so results do not
// depend on which ran.  Per-step counts, tau and event totals go to rings on the
// device; a launch sequence ends with the count reduce, which also advances
// the step index.
//
// What bounds it is latency: a step's dense arrays are 9 MB at N = 1e6 (2 us),
// and its chain is two launches, the tau fold, the draws, and list -> target ->
// state -> atomic.  Draws, pushes and rates as three launches with one lane per
// node and one per event took 8.1 + 9.7 + 4.8 us (Erdos-Renyi d = 8, SIR, 600
// steps); four nodes per lane loaded at once, draws packed and eight lanes per
// event take 7.9 + 4.5 us (loaded, stepped and read 15.3 -> 7.9 ms).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "fs_device.hpp"
#include "fs_runtime.hpp"

namespace fsm {

using namespace fsi;

constexpr uint32_t MTPB = 1024;  // most threads per workgroup
constexpr uint32_t NPL = 4;      // consecutive nodes per lane
constexpr uint32_t MAX_REGIONS = 1024;
constexpr uint32_t EV_LEAVE = 0x80000000u;
// fired[] of a workgroup that left its pushes out (many events): the rates
// launch recounts.
constexpr uint32_t SKIPPED = 0x80000000u;

struct MkArgs {
    uint8_t* state;
    int32_t* infl;
    const int32_t* row_ptr; // incoming CSR (internal order)
    const int32_t* col_ind;
    const int32_t* out_ptr; // outgoing CSR (internal order)
    const int32_t* out_ind;
    const int32_t* orig_id; // caller's id of each node: the draws are keyed by it
    int32_t* pending;       // influence changes of the current step, zero between steps
    uint32_t* ev_cnt;       // [G] events of the current step per workgroup
    uint32_t* fired;        // [G] transitions of the current step (events or not) | SKIPPED
    uint4* rpart;           // [G]: (sum of S influences, max S influence, #E, #I)
    uint4* wcnt;            // [G]: counts after the last step
    uint32_t* part;         // count partials [slot][G][4]
    float* tau_hist;        // [H]
    uint32_t* ev_hist;      // [H]
    double* elapsed;        // one value: the simulated time
    const Ctl* ctl;
    uint32_t n, G, span, H;
    uint32_t step_off;
    int32_t model;          // FS_MARKOV_*
    float beta, sigma, gamma;
    double theta, p_max, tau_max;
    uint32_t key0, key1;
    uint32_t inertial_max;  // events per step up to which pushes update the influence
    uint32_t wg_max;        // events of one workgroup up to which it pushes
    int32_t force_control;  // rates launch after a state change: recount everything
};

__device__ __forceinline__ int next_state(int model, int x)
{
    if (x == ST_S) return model == FS_MARKOV_SEIR ? ST_E : ST_I;
    if (x == ST_E) return ST_I;
    if (x == ST_I) return model == FS_MARKOV_SIS ? ST_S : ST_R;
    return x;
}

// Sum (or maximum) of v over the wavefront, wave-uniform: lane-crossing adds
// within rows of 16, then across rows (a shuffle would go through LDS, and the
// folds sit on the launches' critical path).
template <bool MAX>
__device__ __forceinline__ uint32_t wave_fold(uint32_t v)
{
    auto op = [](uint32_t x, uint32_t y) { return MAX ? max(x, y) : x + y; };
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false)); // row_shr:1
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false)); // row_shr:2
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false)); // row_shr:4
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false)); // row_shr:8
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false)); // row_bcast:15
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false)); // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// tau of Algorithm "Markovian Engine" from the per-workgroup partials of the
// rates launch (one wave; every workgroup folds them in the same order).  The
// sums are exact: an influence sum is at most the edge count, below 2^31.
__device__ double markov_tau(const MkArgs& a, uint32_t lane)
{
    uint32_t A = 0, M = 0, nE = 0, nI = 0;
    for (uint32_t g = lane; g < a.G; g += 64) {
        const uint4 v = a.rpart[g];
        A += v.x;
        M = max(M, v.y);
        nE += v.z;
        nI += v.w;
    }
    A = wave_fold<false>(A);
    M = wave_fold<true>(M);
    nE = wave_fold<false>(nE);
    nI = wave_fold<false>(nI);
    const double L = (double)a.beta * (double)A + (double)a.sigma * (double)nE + (double)a.gamma * (double)nI;
    double mx = (double)a.beta * (double)M;
    if (nE > 0) mx = fmax(mx, (double)a.sigma);
    if (nI > 0) mx = fmax(mx, (double)a.gamma);
    double tau = a.tau_max;
    if (L > 0.0) tau = fmin(tau, a.theta * (double)a.n / L);
    if (mx > 0.0) tau = fmin(tau, a.p_max / mx);
    return tau;
}

// The four states of a lane's nodes i .. i + 3 (state is padded past n), the
// ones past `end` as 7, which is no compartment.
__device__ __forceinline__ uint32_t load_states(const uint8_t* state, uint32_t i, uint32_t end)
{
    uint32_t w = 0x07070707u;
    if (i < end) {
        w = *(const uint32_t*)(state + i);
        const uint32_t nv = end - i;
        if (nv < NPL) w |= 0x07070707u << (8u * nv);
    }
    return w;
}

__global__ __launch_bounds__(MTPB) void mk_step_kernel(MkArgs a)
{
    constexpr uint32_t NW = MTPB / 64;
    __shared__ uint32_t s_lam[NW][64 * NPL]; // queued draws of each wave: the rate,
    __shared__ uint32_t s_who[NW][64 * NPL]; // the node in the tile | state << 16,
    __shared__ uint32_t s_key[NW][64 * NPL]; // and the caller's node id
    __shared__ uint32_t s_event[MTPB * NPL]; // node | EV_LEAVE when it stopped being infectious
    __shared__ uint32_t s_ev, s_fired;
    __shared__ double s_tau;
    const uint32_t tpb = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long k = a.ctl->step + a.step_off;
    const uint32_t base = blockIdx.x * a.span;
    const uint32_t end = min(a.n, base + a.span);
    uint32_t events = 0, fired = 0; // of the whole workgroup (thread 0's hold)
    bool pushing = a.inertial_max != 0u;
    float tf = 0.0f;
    for (uint32_t tile = base; tile < end; tile += tpb * NPL) {
        const uint32_t i = tile + tid * NPL;
        const uint32_t w = load_states(a.state, i, end);
        int4 f = make_int4(0, 0, 0, 0);
        if (i < end) f = *(const int4*)(a.infl + i);
        if (tile == base && wave == 0) {
            const double t = markov_tau(a, lane);
            if (lane == 0) {
                s_tau = t;
                if (blockIdx.x == 0) {
                    a.tau_hist[k % a.H] = (float)t;
                    *a.elapsed += t;
                }
            }
        }
        if (tid == 0) {
            s_ev = 0;
            s_fired = 0;
        }
        __syncthreads();
        tf = (float)s_tau;
        // the nodes with a positive rate, packed
        uint32_t qn = 0;
        const int fl[NPL] = {f.x, f.y, f.z, f.w};
        uint32_t key[NPL];
        float lam[NPL];
#pragma unroll
        for (uint32_t j = 0; j < NPL; ++j) {
            const uint32_t x = (w >> (8u * j)) & 7u;
            lam[j] = x == (uint32_t)ST_S ? a.beta * (float)fl[j] : x == (uint32_t)ST_E ? a.sigma : x == (uint32_t)ST_I ? a.gamma : 0.0f;
            key[j] = lam[j] > 0.0f ? (uint32_t)a.orig_id[i + j] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < NPL; ++j) {
            const bool need = lam[j] > 0.0f;
            const unsigned long long m = __ballot(need);
            if (need) {
                const uint32_t at = qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                s_lam[wave][at] = __float_as_uint(lam[j]);
                s_who[wave][at] = (tid * NPL + j) | (((w >> (8u * j)) & 7u) << 16);
                s_key[wave][at] = key[j];
            }
            qn += (uint32_t)__popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint32_t nfire = 0;
        for (uint32_t q0 = 0; q0 < qn; q0 += 64) {
            bool fire = false, ev = false;
            uint32_t node = 0;
            int x = ST_R;
            if (q0 + lane < qn) {
                const uint32_t who = s_who[wave][q0 + lane];
                node = tile + (who & 0xFFFFu);
                x = (int)(who >> 16);
                const uint4 r = fsd::philox4x32_10(make_uint4(s_key[wave][q0 + lane], (uint32_t)k, 0u, 0u), a.key0, a.key1);
                fire = fsd::bernoulli((float)(r.x >> 8) * 0x1p-24f, __uint_as_float(s_lam[wave][q0 + lane]) * tf);
                if (fire) {
                    const int xn = next_state(a.model, x);
                    a.state[node] = (uint8_t)xn;
                    ev = (xn == ST_I) != (x == ST_I);
                }
            }
            nfire += (uint32_t)__popcll(__ballot(fire));
            const unsigned long long m = __ballot(ev);
            if (m) {
                uint32_t pos = 0;
                if (lane == 0) pos = atomicAdd(&s_ev, (uint32_t)__popcll(m)); // LDS
                pos = __builtin_amdgcn_readfirstlane(pos);
                if (ev) s_event[pos + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = node | (x == ST_I ? EV_LEAVE : 0u);
            }
        }
        if (lane == 0 && nfire) atomicAdd(&s_fired, nfire); // LDS
        __syncthreads();
        const uint32_t nev = s_ev;
        events += nev;
        fired += s_fired;
        // (a step of many events is recounted anyway: past its share of them
        // a workgroup leaves the pushes to the recount)
        if (events > a.wg_max) pushing = false;
        if (pushing) {
            // eight lanes per event take eight targets each at a time (their
            // ids, then their states, then the atomics); lists of more than 64
            // targets (hubs) are left to whole waves
            const bool all = a.model == FS_MARKOV_SIS;
            const int32_t* __restrict__ out_ind = a.out_ind;
            const uint8_t* state = a.state;
            auto push = [&](uint32_t t0, uint32_t t1, uint32_t at, uint32_t stride, int d) {
                for (uint32_t t = t0 + at; t < t1; t += 8 * stride) {
                    int32_t tg[8];
                    bool go[8];
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) tg[u] = t + u * stride < t1 ? out_ind[t + u * stride] : -1;
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) go[u] = tg[u] >= 0 && (all || state[tg[u]] == ST_S);
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u)
                        if (go[u]) atomicAdd(&a.pending[tg[u]], d);
                }
            };
            const uint32_t sub = lane & 7u;
            for (uint32_t e0 = wave * 8; e0 < nev; e0 += tpb / 8) {
                const uint32_t e = e0 + (lane >> 3);
                const uint32_t v = e < nev ? s_event[e] : 0u;
                const uint32_t node = v & ~EV_LEAVE;
                const uint32_t t0 = e < nev ? (uint32_t)a.out_ptr[node] : 0u;
                const uint32_t t1 = e < nev ? (uint32_t)a.out_ptr[node + 1] : 0u;
                const bool lng = t1 - t0 > 64u;
                if (!lng) push(t0, t1, sub, 8u, (v & EV_LEAVE) ? -1 : 1);
                for (unsigned long long lm = __ballot(lng && sub == 0u); lm != 0ull; lm &= lm - 1ull) {
                    const int l = __builtin_ctzll(lm);
                    const uint32_t u0 = (uint32_t)__shfl((int)t0, l, 64), u1 = (uint32_t)__shfl((int)t1, l, 64);
                    const uint32_t lv = (uint32_t)__shfl((int)v, l, 64);
                    push(u0, u1, lane, 64u, (lv & EV_LEAVE) ? -1 : 1);
                }
            }
        }
        if (tile + tpb * NPL < end) __syncthreads(); // (the event list is reused)
    }
    if (tid == 0) {
        a.ev_cnt[blockIdx.x] = events;
        a.fired[blockIdx.x] = fired | (pushing ? 0u : SKIPPED);
    }
}

// The influences after a step (its pending changes, or in Control Mode and
// after a state change a recount), and the partials and counts of the new
// states.
__global__ __launch_bounds__(MTPB) void mk_rates_kernel(MkArgs a)
{
    constexpr uint32_t NW = MTPB / 64;
    __shared__ uint4 s_p[NW], s_c[NW];
    __shared__ uint32_t s_t[NW][2];
    const uint32_t tpb = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = tpb >> 6;
    const unsigned long long k = a.ctl->step + a.step_off;
    const uint32_t base = blockIdx.x * a.span;
    const uint32_t end = min(a.n, base + a.span);
    // the first tile's arrays and the step's totals, together
    uint32_t i = base + tid * NPL;
    uint32_t w = load_states(a.state, i, end);
    int4 f = make_int4(0, 0, 0, 0), d = make_int4(0, 0, 0, 0);
    if (i < end) {
        f = *(const int4*)(a.infl + i);
        d = *(const int4*)(a.pending + i);
    }
    uint32_t ev = 0, fi = 0, skip = 0;
    for (uint32_t g = tid; g < a.G; g += tpb) {
        ev += a.ev_cnt[g];
        const uint32_t v = a.fired[g];
        fi += v & ~SKIPPED;
        skip |= v & SKIPPED;
    }
    ev = wave_fold<false>(ev);
    fi = wave_fold<false>(fi);
    if (__ballot(skip != 0u) != 0ull) fi |= SKIPPED;
    if (lane == 0) {
        s_t[wave][0] = ev;
        s_t[wave][1] = fi;
    }
    __syncthreads();
    ev = fi = skip = 0;
    for (uint32_t v = 0; v < nw; ++v) {
        ev += s_t[v][0];
        fi += s_t[v][1] & ~SKIPPED;
        skip |= s_t[v][1] & SKIPPED;
    }
    uint4* part = (uint4*)a.part + (size_t)a.step_off * a.G + blockIdx.x;
    if (!a.force_control) {
        if (blockIdx.x == 0 && tid == 0) a.ev_hist[k % a.H] = ev;
        // a step without transitions changed nothing: the partials still hold
        if (fi == 0) {
            if (tid == 0) *part = a.wcnt[blockIdx.x];
            return;
        }
    }
    const bool all = a.model == FS_MARKOV_SIS;
    // (pushes left out by a workgroup, in a step of few events: the recount
    // stands for them and touches the nodes they would have)
    const bool recount = a.force_control || ev > a.inertial_max;
    const bool control = recount || skip != 0u;
    uint32_t A = 0, M = 0, nE = 0, nI = 0, nS = 0;
    if (control) {
        for (uint32_t v = base + tid; v < end; v += tpb) {
            const int x = (int)a.state[v];
            int c = 0;
            if (recount || all || x == ST_S) {
                for (int32_t e = a.row_ptr[v]; e < a.row_ptr[v + 1]; ++e) c += a.state[a.col_ind[e]] == ST_I;
                a.infl[v] = c;
            }
            a.pending[v] = 0;
            if (x == ST_S) {
                A += (uint32_t)c;
                M = max(M, (uint32_t)c);
            }
            nS += x == ST_S;
            nE += x == ST_E;
            nI += x == ST_I;
        }
    } else {
        for (uint32_t tile = base; tile < end; tile += tpb * NPL) {
            if (tile != base) {
                i = tile + tid * NPL;
                w = load_states(a.state, i, end);
                f = d = make_int4(0, 0, 0, 0);
                if (i < end) {
                    f = *(const int4*)(a.infl + i);
                    d = *(const int4*)(a.pending + i);
                }
            }
            if ((d.x | d.y | d.z | d.w) != 0) {
                auto add = [&](int v, int c, uint32_t j) { return all || ((w >> (8u * j)) & 7u) == (uint32_t)ST_S ? v + c : v; };
                f = make_int4(add(f.x, d.x, 0), add(f.y, d.y, 1), add(f.z, d.z, 2), add(f.w, d.w, 3));
                *(int4*)(a.infl + i) = f;
                *(int4*)(a.pending + i) = make_int4(0, 0, 0, 0);
            }
            const int fl[NPL] = {f.x, f.y, f.z, f.w};
#pragma unroll
            for (uint32_t j = 0; j < NPL; ++j) {
                const uint32_t v = (w >> (8u * j)) & 7u ? 0u : (uint32_t)fl[j]; // S nodes only
                A += v;
                M = max(M, v);
            }
            const uint32_t b0 = w & 0x01010101u, b1 = (w >> 1) & 0x01010101u;
            nS += (uint32_t)__popc(~(b0 | b1) & 0x01010101u);
            nE += (uint32_t)__popc(b0 & ~b1);
            nI += (uint32_t)__popc(b1 & ~b0);
        }
    }
    A = wave_fold<false>(A);
    M = wave_fold<true>(M);
    nE = wave_fold<false>(nE);
    nI = wave_fold<false>(nI);
    nS = wave_fold<false>(nS);
    if (lane == 0) {
        s_p[wave] = make_uint4(A, M, nE, nI);
        s_c[wave].x = nS;
    }
    __syncthreads();
    if (tid == 0) {
        uint4 t = make_uint4(0, 0, 0, 0);
        uint32_t S = 0;
        for (uint32_t v = 0; v < nw; ++v) {
            t.x += s_p[v].x;
            t.y = max(t.y, s_p[v].y);
            t.z += s_p[v].z;
            t.w += s_p[v].w;
            S += s_c[v].x;
        }
        a.rpart[blockIdx.x] = t;
        const uint4 c = make_uint4(S, t.z, t.w, end - base - S - t.z - t.w);
        a.wcnt[blockIdx.x] = c;
        if (!a.force_control) *part = c;
    }
}

__global__ void mk_seed_kernel(uint8_t* state, const int64_t* nodes, int64_t count, int32_t comp)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < count) state[nodes[j]] = (uint8_t)comp;
}

// States (and influences) between the caller's node order and the internal
// one (orig: internal -> caller's id, nullptr for the identity).
__global__ void mk_put_kernel(uint8_t* state, const uint8_t* src, const int32_t* orig, uint32_t n)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) state[i] = src[orig ? (uint32_t)orig[i] : i];
}

__global__ void mk_get_kernel(const uint8_t* state, const int32_t* infl, const int32_t* orig, uint32_t n,
                              uint8_t* dst_state, int32_t* dst_infl)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t c = orig ? (uint32_t)orig[i] : i;
    dst_state[c] = state[i];
    dst_infl[c] = infl[i];
}

__global__ void mk_clear_kernel(double* elapsed, double value)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *elapsed = value;
}

} // namespace fsm

using namespace fsr;
using fsm::MkArgs;

struct fs_markov {
    fs_graph* g = nullptr;
    fs_markov_params p{};
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    uint8_t* d_state = nullptr;
    int32_t* d_infl = nullptr;
    int32_t* d_pending = nullptr;
    uint4* d_wcnt = nullptr;
    uint32_t tpb = 1024; // threads per workgroup
    uint32_t* d_ev_cnt = nullptr;
    uint32_t* d_fired = nullptr;
    uint4* d_rpart = nullptr;
    uint32_t* d_part = nullptr;
    uint32_t* d_hist = nullptr;
    float* d_tau = nullptr;
    uint32_t* d_evh = nullptr;
    double* d_elapsed = nullptr;
    fsi::Ctl* d_ctl = nullptr;
    uint32_t G = 0, span = 0, H = 1024, chunk = 64;
    int64_t step = 0, hist_from = 0;
    MkArgs args{};
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

// The outgoing CSR of a graph's internal order, built on first use and kept
// with the graph (the transpose of its incoming rows).
fs_status ensure_out_csr(fs_graph* g)
{
    std::lock_guard<std::mutex> lk(g->layout_mu);
    if (g->d_out_ptr) return FS_OK;
    const int64_t n = g->n;
    std::vector<int32_t> ptr((size_t)n + 1, 0), ind((size_t)g->nnz);
    for (int64_t e = 0; e < g->nnz; ++e) ptr[(size_t)g->h_col_ind[(size_t)e] + 1] += 1;
    for (int64_t j = 0; j < n; ++j) ptr[(size_t)j + 1] += ptr[(size_t)j];
    std::vector<int32_t> fill(ptr.begin(), ptr.end() - 1);
    for (int64_t i = 0; i < n; ++i)
        for (int32_t e = g->h_row_ptr[(size_t)i]; e < g->h_row_ptr[(size_t)i + 1]; ++e)
            ind[(size_t)fill[(size_t)g->h_col_ind[(size_t)e]]++] = (int32_t)i;
    int32_t *dp = nullptr, *di = nullptr;
    hipError_t e;
    if ((e = dev_alloc((void**)&dp, ptr.size() * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&di, std::max<size_t>(ind.size(), 1) * 4)) != hipSuccess) {
        dev_free(dp);
        return fail(FS_ERR_OUT_OF_MEMORY, std::string("outgoing CSR: ") + hipGetErrorString(e));
    }
    if ((e = hipMemcpy(dp, ptr.data(), ptr.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
        (!ind.empty() && (e = hipMemcpy(di, ind.data(), ind.size() * 4, hipMemcpyHostToDevice)) != hipSuccess)) {
        dev_free(dp);
        dev_free(di);
        return fail(FS_ERR_DEVICE, std::string("outgoing CSR upload: ") + hipGetErrorString(e));
    }
    g->d_out_ptr = dp;
    g->d_out_ind = di;
    return FS_OK;
}

void release_markov(fs_markov* m)
{
    if (!m) return;
    if (m->stream) (void)hipStreamSynchronize(m->stream); // (blocks may return to a caller's allocator)
    if (m->exec) (void)hipGraphExecDestroy(m->exec);
    if (m->graph) (void)hipGraphDestroy(m->graph);
    for (void* p : {(void*)m->d_state, (void*)m->d_infl, (void*)m->d_pending, (void*)m->d_wcnt, (void*)m->d_ev_cnt, (void*)m->d_fired,
                    (void*)m->d_rpart,
                    (void*)m->d_part, (void*)m->d_hist, (void*)m->d_tau, (void*)m->d_evh, (void*)m->d_elapsed,
                    (void*)m->d_ctl})
        dev_free(p);
    if (m->own_stream && m->stream) (void)hipStreamDestroy(m->stream);
    if (m->g) m->g->users.fetch_sub(1);
    delete m;
}

// After a change of states from the host: recount every influence and the
// rate partials the next draw folds.
hipError_t refresh(fs_markov* m)
{
    MkArgs a = m->args;
    a.force_control = 1;
    a.step_off = 0;
    void* argv[] = {&a};
    return hipLaunchKernel((const void*)&fsm::mk_rates_kernel, dim3(m->G), dim3(m->tpb), argv, 0, m->stream);
}

struct MkSeq {
    std::vector<MkArgs> step;
    fsi::Ctl* ctl;
    const uint32_t* part;
    uint32_t G, C, H, r;
    uint32_t* hist;
};

void make_seq(fs_markov* m, uint32_t r, MkSeq& q)
{
    q.step.assign(r, m->args);
    for (uint32_t j = 0; j < r; ++j) q.step[j].step_off = j;
    q.ctl = m->d_ctl;
    q.part = m->d_part;
    q.G = m->G;
    q.C = 4;
    q.H = m->H;
    q.r = r;
    q.hist = m->d_hist;
}

fs_status build_exec(fs_markov* m, uint32_t b)
{
    MkSeq q;
    make_seq(m, b, q);
    FS_HIP(hipGraphCreate(&m->graph, 0));
    hipGraphNode_t prev = nullptr;
    auto add = [&](const void* fn, dim3 grid, dim3 block, void** argv) -> fs_status {
        hipKernelNodeParams kp{};
        kp.func = const_cast<void*>(fn);
        kp.gridDim = grid;
        kp.blockDim = block;
        kp.kernelParams = argv;
        hipGraphNode_t node;
        FS_HIP(hipGraphAddKernelNode(&node, m->graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp));
        prev = node;
        return FS_OK;
    };
    fs_status st;
    for (uint32_t j = 0; j < b; ++j) {
        void* argv[] = {&q.step[j]};
        if ((st = add((const void*)&fsm::mk_step_kernel, dim3(m->G), dim3(m->tpb), argv)) != FS_OK) return st;
        if ((st = add((const void*)&fsm::mk_rates_kernel, dim3(m->G), dim3(m->tpb), argv)) != FS_OK) return st;
    }
    uint32_t* no_base = nullptr;
    void* rargv[] = {&q.ctl, &q.part, &q.G, &q.C, &q.hist, &q.H, &no_base};
    if ((st = add(fsk::reduce_kernel_fn(), dim3(q.r), dim3(fsi::RED_TPB), rargv)) != FS_OK) return st;
    FS_HIP(hipGraphInstantiate(&m->exec, m->graph, nullptr, nullptr, 0));
    return FS_OK;
}

fs_status launch_seq(fs_markov* m, uint32_t r)
{
    MkSeq q;
    make_seq(m, r, q);
    for (uint32_t j = 0; j < r; ++j) {
        void* argv[] = {&q.step[j]};
        FS_HIP(hipLaunchKernel((const void*)&fsm::mk_step_kernel, dim3(m->G), dim3(m->tpb), argv, 0, m->stream));
        FS_HIP(hipLaunchKernel((const void*)&fsm::mk_rates_kernel, dim3(m->G), dim3(m->tpb), argv, 0, m->stream));
    }
    uint32_t* no_base = nullptr;
    void* rargv[] = {&q.ctl, &q.part, &q.G, &q.C, &q.hist, &q.H, &no_base};
    FS_HIP(hipLaunchKernel(fsk::reduce_kernel_fn(), dim3(r), dim3(fsi::RED_TPB), rargv, 0, m->stream));
    return FS_OK;
}

} // namespace

#define FS_GUARD_BEGIN try {
#define FS_GUARD_END                                                                            \
    }                                                                                           \
    catch (const std::bad_alloc&) { return fail(FS_ERR_OUT_OF_MEMORY, "host allocation failed"); } \
    catch (const std::exception& e) { return fail(FS_ERR_DEVICE, e.what()); }                   \
    catch (...) { return fail(FS_ERR_DEVICE, "unknown exception"); }

extern "C" {

fs_status fs_markov_create(fs_graph* g, const fs_markov_params* p, fs_markov** out)
{
    FS_GUARD_BEGIN
    if (!out) return fail(FS_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!g || !p) return fail(FS_ERR_INVALID_ARG, "NULL graph or params");
    if (g->d_weights) return fail(FS_ERR_INVALID_ARG, "the Markovian engine runs unit-weight graphs");
    if (p->model != FS_MARKOV_SEIR && p->model != FS_MARKOV_SIR && p->model != FS_MARKOV_SIS)
        return fail(FS_ERR_INVALID_ARG, "model must be FS_MARKOV_SEIR, FS_MARKOV_SIR or FS_MARKOV_SIS");
    auto finite_ge0 = [](double v) { return v >= 0.0 && std::isfinite(v); };
    if (!finite_ge0(p->beta) || !finite_ge0(p->gamma) || (p->model == FS_MARKOV_SEIR && !finite_ge0(p->sigma)))
        return fail(FS_ERR_INVALID_ARG, "rates must be finite and >= 0");
    if (!(p->theta > 0.0) || !(p->p_max > 0.0) || !(p->tau_max > 0.0) || !std::isfinite(p->theta) ||
        !std::isfinite(p->p_max) || !std::isfinite(p->tau_max))
        return fail(FS_ERR_INVALID_ARG, "theta, p_max and tau_max must be finite and > 0");
    if (p->history_len < 0 || p->history_len == 1) return fail(FS_ERR_INVALID_ARG, "history_len must be 0 or >= 2");
    if (p->steps_per_graph < 0 || p->steps_per_graph > 100000)
        return fail(FS_ERR_INVALID_ARG, "steps_per_graph out of range");
    if (p->inertial_max < -1) return fail(FS_ERR_INVALID_ARG, "inertial_max must be -1, 0 or positive");
    DeviceGuard dg(g->device);
    fs_status st = ensure_out_csr(g);
    if (st != FS_OK) return st;
    fs_markov* m = new fs_markov();
    m->g = g;
    g->users.fetch_add(1);
    m->p = *p;
    m->device = g->device;
    m->H = p->history_len ? (uint32_t)p->history_len : 1024u;
    m->chunk = (uint32_t)std::max(p->steps_per_graph, 64);
    const uint32_t n = (uint32_t)g->n;
    int cus = 0;
    hipError_t e;
    auto bad = [&](hipError_t err, const char* what) {
        release_markov(m);
        return fail(err == hipErrorOutOfMemory ? FS_ERR_OUT_OF_MEMORY : FS_ERR_DEVICE,
                    std::string(what) + ": " + hipGetErrorString(err));
    };
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device)) != hipSuccess)
        return bad(e, "device attribute");
    // one workgroup region per compute unit, in whole wavefronts
    m->G = (uint32_t)std::max<int64_t>(1, std::min<int64_t>({(int64_t)cus, (int64_t)fsm::MAX_REGIONS,
                                                              ((int64_t)n + 63) / 64}));
    m->span = (((n + m->G - 1) / m->G) + 63) / 64 * 64;
    m->G = (n + m->span - 1) / m->span;
    // four nodes per lane, in whole wavefronts (larger regions in tiles)
    m->tpb = std::min(fsm::MTPB, (m->span / fsm::NPL + 63) / 64 * 64);
    const size_t padded = ((size_t)n + 255) / 256 * 256;
    if (p->stream) {
        m->stream = (hipStream_t)p->stream;
    } else {
        if ((e = hipStreamCreateWithFlags(&m->stream, hipStreamNonBlocking)) != hipSuccess) return bad(e, "stream");
        m->own_stream = true;
    }
    const size_t part_words = (size_t)m->chunk * m->G * 4;
    if ((e = dev_alloc((void**)&m->d_state, padded)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_infl, padded * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_pending, padded * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_wcnt, (size_t)m->G * sizeof(uint4))) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_ev_cnt, (size_t)m->G * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_fired, (size_t)m->G * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_rpart, (size_t)m->G * sizeof(uint4))) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_part, part_words * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_hist, (size_t)m->H * 16)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_tau, (size_t)m->H * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_evh, (size_t)m->H * 4)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_elapsed, 8)) != hipSuccess ||
        (e = dev_alloc((void**)&m->d_ctl, sizeof(fsi::Ctl))) != hipSuccess)
        return bad(e, "device allocation");
    if ((e = hipMemsetAsync(m->d_state, 0, padded, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_infl, 0, padded * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_pending, 0, padded * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_ev_cnt, 0, (size_t)m->G * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_fired, 0, (size_t)m->G * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_hist, 0, (size_t)m->H * 16, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_tau, 0, (size_t)m->H * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_evh, 0, (size_t)m->H * 4, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_elapsed, 0, 8, m->stream)) != hipSuccess ||
        (e = hipMemsetAsync(m->d_ctl, 0, sizeof(fsi::Ctl), m->stream)) != hipSuccess)
        return bad(e, "initialisation");
    MkArgs& a = m->args;
    a.state = m->d_state;
    a.infl = m->d_infl;
    a.row_ptr = g->d_row_ptr;
    a.col_ind = g->d_col_ind;
    a.out_ptr = g->d_out_ptr;
    a.out_ind = g->d_out_ind;
    a.orig_id = g->d_orig;
    a.pending = m->d_pending;
    a.wcnt = m->d_wcnt;
    a.ev_cnt = m->d_ev_cnt;
    a.fired = m->d_fired;
    a.rpart = m->d_rpart;
    a.part = m->d_part;
    a.tau_hist = m->d_tau;
    a.ev_hist = m->d_evh;
    a.elapsed = m->d_elapsed;
    a.ctl = m->d_ctl;
    a.n = n;
    a.G = m->G;
    a.span = m->span;
    a.H = m->H;
    a.model = p->model;
    a.beta = (float)p->beta;
    a.sigma = (float)p->sigma;
    a.gamma = (float)p->gamma;
    a.theta = p->theta;
    a.p_max = p->p_max;
    a.tau_max = p->tau_max;
    a.key0 = (uint32_t)p->seed;
    a.key1 = (uint32_t)(p->seed >> 32);
    // automatic threshold: pushes while the step's events touch fewer edges
    // than a recount reads (events * mean degree < nnz / 8)
    const double dmean = std::max(1.0, g->mean_degree);
    a.inertial_max = p->inertial_max == -1 ? 0u
                   : p->inertial_max > 0   ? (uint32_t)std::min<int64_t>(p->inertial_max, 0xFFFFFFFFll)
                                           : (uint32_t)std::max(1.0, (double)g->nnz / 8.0 / dmean);
    // (four times an even share: uneven regions still push)
    a.wg_max = (uint32_t)std::min<uint64_t>(0xFFFFFFFFull, 4ull * a.inertial_max / m->G + 64ull);
    if ((e = refresh(m)) != hipSuccess || (e = hipStreamSynchronize(m->stream)) != hipSuccess)
        return bad(e, "initialisation");
    *out = m;
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_destroy(fs_markov* m)
{
    FS_GUARD_BEGIN
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    DeviceGuard dg(m->device);
    hipError_t e = hipStreamSynchronize(m->stream);
    release_markov(m);
    if (e != hipSuccess) return fail(FS_ERR_DEVICE, std::string("pending work failed: ") + hipGetErrorString(e));
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_seed(fs_markov* m, int64_t count, const int64_t* nodes, int32_t compartment)
{
    FS_GUARD_BEGIN
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    if (compartment < 0 || compartment > 3) return fail(FS_ERR_INVALID_ARG, "compartment must be in [0, 3]");
    if (count < 0) return fail(FS_ERR_INVALID_ARG, "count < 0");
    if (count == 0) return FS_OK;
    if (!nodes) return fail(FS_ERR_INVALID_ARG, "nodes is NULL");
    std::vector<int64_t> internal((size_t)count);
    for (int64_t j = 0; j < count; ++j) {
        if (nodes[j] < 0 || nodes[j] >= m->g->n) return fail(FS_ERR_INVALID_ARG, "seed node out of range");
        internal[(size_t)j] = m->g->h_inv.empty() ? nodes[j] : m->g->h_inv[(size_t)nodes[j]];
    }
    DeviceGuard dg(m->device);
    StreamBuf tmp(m->stream);
    FS_HIP(hipMallocAsync(&tmp.p, (size_t)count * 8, m->stream));
    FS_HIP(hipMemcpyAsync(tmp.p, internal.data(), (size_t)count * 8, hipMemcpyHostToDevice, m->stream));
    hipLaunchKernelGGL(fsm::mk_seed_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, m->stream,
                       m->d_state, (const int64_t*)tmp.p, count, compartment);
    FS_HIP(hipGetLastError());
    FS_HIP(refresh(m));
    FS_HIP(hipStreamSynchronize(m->stream));
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_set_state(fs_markov* m, const int32_t* state, int64_t step_index, double elapsed)
{
    FS_GUARD_BEGIN
    if (!m || !state) return fail(FS_ERR_INVALID_ARG, "NULL argument");
    if (step_index < -1) return fail(FS_ERR_INVALID_ARG, "step_index must be >= -1");
    if (!(elapsed >= 0.0) || !std::isfinite(elapsed)) return fail(FS_ERR_INVALID_ARG, "elapsed must be finite and >= 0");
    const size_t n = (size_t)m->g->n;
    DeviceGuard dg(m->device);
    const int64_t new_step = step_index >= 0 ? step_index : m->step;
    StreamBuf tmp(m->stream);
    FS_HIP(hipMallocAsync(&tmp.p, n, m->stream));
    bool bad_state = false, bad_age = false;
    const fs_status st = copy_in(m->device, m->stream, n, state, (uint8_t*)tmp.p, nullptr, nullptr, 0, false, &bad_state,
                                 &bad_age);
    if (bad_state) return fail(FS_ERR_INVALID_ARG, "state values must lie in [0, 3]");
    if (st != FS_OK) return st;
    hipLaunchKernelGGL(fsm::mk_put_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, m->stream, m->d_state,
                       (const uint8_t*)tmp.p, m->g->h_orig.empty() ? (const int32_t*)nullptr : m->g->d_orig, (uint32_t)n);
    FS_HIP(hipGetLastError());
    hipLaunchKernelGGL(fsm::mk_clear_kernel, dim3(1), dim3(64), 0, m->stream, m->d_elapsed, elapsed);
    FS_HIP(hipGetLastError());
    FS_HIP(fsk::launch_set_ctl(m->d_ctl, (unsigned long long)new_step, m->stream));
    FS_HIP(refresh(m));
    FS_HIP(hipStreamSynchronize(m->stream));
    if (step_index >= 0) {
        m->step = step_index;
        m->hist_from = step_index;
    }
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_step(fs_markov* m, int64_t n_steps)
{
    FS_GUARD_BEGIN
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    if (n_steps < 0) return fail(FS_ERR_INVALID_ARG, "n_steps < 0");
    DeviceGuard dg(m->device);
    const int b = m->p.steps_per_graph;
    int64_t left = n_steps;
    if (b > 0) {
        if (!m->exec) {
            fs_status st = build_exec(m, (uint32_t)b);
            if (st != FS_OK) return st;
        }
        for (; left >= b; left -= b) FS_HIP(hipGraphLaunch(m->exec, m->stream));
    }
    while (left > 0) {
        const uint32_t r = (uint32_t)std::min<int64_t>(left, m->chunk);
        fs_status st = launch_seq(m, r);
        if (st != FS_OK) return st;
        left -= r;
    }
    m->step += n_steps;
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_sync(fs_markov* m)
{
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    DeviceGuard dg(m->device);
    FS_HIP(hipStreamSynchronize(m->stream));
    return FS_OK;
}

fs_status fs_markov_get_state(fs_markov* m, int32_t* state, int32_t* influence, int64_t* step_index, double* elapsed)
{
    FS_GUARD_BEGIN
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    DeviceGuard dg(m->device);
    const size_t n = (size_t)m->g->n;
    double el = 0.0;
    StreamBuf tmp(m->stream);
    FS_HIP(hipMallocAsync(&tmp.p, n * 5, m->stream));
    uint8_t* d_state = (uint8_t*)tmp.p + n * 4;
    hipLaunchKernelGGL(fsm::mk_get_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, m->stream,
                       (const uint8_t*)m->d_state, (const int32_t*)m->d_infl,
                       m->g->h_orig.empty() ? (const int32_t*)nullptr : m->g->d_orig, (uint32_t)n, d_state,
                       (int32_t*)tmp.p);
    FS_HIP(hipGetLastError());
    const fs_status st = copy_out(m->device, m->stream, n, d_state, state, tmp.p, influence, 4);
    if (st != FS_OK) return st;
    FS_HIP(hipMemcpyAsync(&el, m->d_elapsed, 8, hipMemcpyDeviceToHost, m->stream));
    FS_HIP(hipStreamSynchronize(m->stream));
    if (step_index) *step_index = m->step;
    if (elapsed) *elapsed = el;
    return FS_OK;
    FS_GUARD_END
}

fs_status fs_markov_history(fs_markov* m, int64_t first_step, int64_t n, int64_t* counts, double* taus, int64_t* events)
{
    FS_GUARD_BEGIN
    if (!m) return fail(FS_ERR_INVALID_ARG, "engine is NULL");
    if (n < 0) return fail(FS_ERR_INVALID_ARG, "n < 0");
    if (n == 0) return FS_OK;
    if (first_step < m->hist_from || first_step + n > m->step || m->step - first_step > (int64_t)m->H)
        return fail(FS_ERR_INVALID_ARG, "steps outside the recorded window");
    DeviceGuard dg(m->device);
    std::vector<uint32_t> h((size_t)m->H * 4), ev(m->H);
    std::vector<float> t(m->H);
    FS_HIP(hipMemcpyAsync(h.data(), m->d_hist, h.size() * 4, hipMemcpyDeviceToHost, m->stream));
    FS_HIP(hipMemcpyAsync(t.data(), m->d_tau, t.size() * 4, hipMemcpyDeviceToHost, m->stream));
    FS_HIP(hipMemcpyAsync(ev.data(), m->d_evh, ev.size() * 4, hipMemcpyDeviceToHost, m->stream));
    FS_HIP(hipStreamSynchronize(m->stream));
    for (int64_t j = 0; j < n; ++j) {
        const size_t slot = (size_t)((first_step + j) % m->H);
        if (counts)
            for (int q = 0; q < 4; ++q) counts[4 * j + q] = h[slot * 4 + (size_t)q];
        if (taus) taus[j] = t[slot];
        if (events) events[j] = ev[slot];
    }
    return FS_OK;
    FS_GUARD_END
}

} // extern "C"
