// Resident iteration: one launch runs whole CFR iterations of a game that fits the LDS of the chip's
// CUs, about 5 ms of them.
//
// Level by level, a small or middle-sized game's iteration is bound by its launches (two sweeps
// of one launch per level, 3 to 5 us each) and not by what they compute. Here the game is cut into a
// trunk and subtrees of at most a given size: a workgroup takes a bin of whole subtrees and runs both
// sweeps over them in its LDS, with only workgroup barriers between levels, and the workgroups meet
// twice per pass:
//   A. every bin: the reach of its roots (the trunk's edges on their paths), then phase i takes the
//      reach of the bin's level i + 1 (Eq. excepted_reach_probabilities_matrix_recurrence and its
//      own-reach twin, odd wavefronts) and the values of its level n - 1 - i (Eq.
//      expected_payoffs_matrix_recurrence, even wavefronts), which do not depend on one another;
//      then each player node's regret contributions (Eq. instantaneous_counterfactual_regret,
//      multiplied out) and own reach (Eq. player_reach_probability) go to its slot;
//   B. after a barrier, per infoset the sums of its members' slots and the update (Eqs.
//      average_counterfactual_regrets_vector, average_strategy_profile_vector,
//      next_strategy_profile); the first workgroup runs the trunk's sweeps (level by level from
//      the subtrees' values) and its infosets; another barrier.
// A game that fits one workgroup has no trunk and no team (RES_SOLO): strategy, regrets, sums and
// contributions lie in LDS too.
//
// What crosses workgroups goes through agent-scope atomic accesses (performed at the point of
// coherence; no cache is written back or invalidated). A team of at most 32 forms on one XCD:
// there a dependent access takes about 0.17 us and a barrier 0.8 to 1.1 us; across XCDs 0.5 us, and
// with 256 arrivals on one counter 3.7 us, which is why they meet in groups of kResGroup first. A
// team is the workgroups that are running when it forms (they register; the first closes the
// registration after a bounded wait), so every member of a barrier is resident and every wait ends,
// whatever else the GPU runs; workgroups that come late leave at once, and a smaller team takes its
// bins in turn.
//
// Sums are formed in the order of the level-by-level launches, so that the two agree bit for bit: the
// public-block engine's for two players (values by action, chance nodes by lane groups and a
// butterfly, infosets by member; one larger than a chunk of those launches is their exception), the
// node engine's for general sums (sum_order.hpp: with sums of its own order, as first built, general
// sums took 87 us per iteration at 2.1 million nodes of three players; in this order, compiled for four
// players and for eight, 67 us).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "resident.hpp"
#include "sum_order.hpp"

namespace cfr {

namespace {

constexpr uint32_t kResClosed = 0x80000000u;
constexpr int kResMaxThreads = 1024;

__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float pos_(float a) { return fmaxf(a, 0.0f); }
__device__ __forceinline__ double pos_(double a) { return fmax(a, 0.0); }

template <bool SOLO, class F>
__device__ __forceinline__ F get(const F* p) {
    if constexpr (SOLO) return *p;
    else return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool SOLO, class F>
__device__ __forceinline__ void put(F* p, F v) {
    if constexpr (SOLO) *p = v;
    else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 16 bytes (aligned) at once. Between workgroups: written through to the point of coherence, as the
// agent-scope stores are (sc1). The wait state keeps the next write of the data registers behind
// the store's read of them.
template <bool SOLO>
__device__ __forceinline__ void put_vec(float* p, const float (&v)[4]) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 x = {v[0], v[1], v[2], v[3]};
    if constexpr (SOLO) *reinterpret_cast<f4*>(p) = x;
    else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(x) : "memory");
}
template <bool SOLO>
__device__ __forceinline__ void put_vec(double* p, const double (&v)[2]) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    const d2 x = {v[0], v[1]};
    if constexpr (SOLO) *reinterpret_cast<d2*>(p) = x;
    else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(x) : "memory");
}

__device__ __forceinline__ uint32_t agent_load(const ResTeam::Line& p) {
    return __hip_atomic_load(&p.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t agent_add(ResTeam::Line& p, uint32_t v) {
    return __hip_atomic_fetch_add(&p.v, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The XCD that this wavefront runs on (hardware register XCC_ID, bits 0-3).
__device__ __forceinline__ uint32_t xcc_id() {
    return __builtin_amdgcn_s_getreg(20 | (31 << 11)) & 15u;
}

// Joins the team (thread 0): the workgroup's place in it, or -1; `size` is the team's size.
__device__ __forceinline__ int join_team(ResTeam* t, uint32_t want, uint32_t& size) {
    if (want <= kResXcd) {
        const uint32_t me = xcc_id() + 1;
        uint32_t first = 0;
        __hip_atomic_compare_exchange_strong(&t->xcc.v, &first, me, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (first != 0 && first != me) return -1;
    }
    const uint32_t place = agent_add(t->reg, 1);
    if ((place & kResClosed) || place >= want) return -1;
    if (place == 0) {
        // at most 20 us (the 100 MHz clock) for the others to arrive
        const uint64_t t0 = wall_clock64();
        while (agent_load(t->reg) < want && wall_clock64() - t0 < 2000) __builtin_amdgcn_s_sleep(1);
        size = __hip_atomic_fetch_or(&t->reg.v, kResClosed, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        size = size < want ? size : want;
        __hip_atomic_store(&t->size.v, size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        // the first member is running and closes the team within its bounded wait
        while ((size = agent_load(t->size)) == 0) __builtin_amdgcn_s_sleep(1);
    }
    return static_cast<int>(place);
}

// Leaves the launch (thread 0): the last workgroup clears the team for the next launch.
__device__ __forceinline__ void leave_team(ResTeam* t) {
    if (agent_add(t->exited, 1) == gridDim.x - 1) {
        put<false>(&t->xcc.v, 0u);
        put<false>(&t->reg.v, 0u);
        put<false>(&t->size.v, 0u);
        put<false>(&t->bar.v, 0u);
        for (int g = 0; g < kResTeam / kResGroup; ++g) put<false>(&t->group[g].v, 0u);
        put<false>(&t->exited.v, 0u);
    }
}

// NP: 0 for two players and zero sum, else the most players (kMaxPlayers).
template <class F, int MODE, int NP>
__global__ void __launch_bounds__(kResMaxThreads) k_resident(Resident<F> r, UpdateRule rule,
                                                             int32_t passes, int32_t n) {
#pragma clang fp contract(off)
    constexpr bool SOLO = MODE == RES_SOLO;
    constexpr int CM = NP > 0 ? NP : 1, RM = NP > 0 ? NP : 2;  // at most so many columns, planes
    constexpr int kLaneUnroll = NP > 0 ? 1 : 4;  // (several columns' reads ahead spill)
    extern __shared__ __attribute__((aligned(16))) unsigned char s_raw[];
    __shared__ Rec4 s_tab[kResMaxDepth + 3];
    __shared__ F s_red[NP > 0 ? kWideWaves : 1][NP > 0 ? NP : 1];
    __shared__ int s_place;
    __shared__ uint32_t s_size;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nt = blockDim.x, nw = nt >> 6;
    const int D = r.D;
    const int32_t P = NP > 0 ? r.players : 1;       // value columns
    const int32_t planes = NP > 0 ? r.players : 2;  // players' reach planes
    const int32_t mn = r.max_nodes, mr = r.max_ranks;
    int place = 0;
    int32_t team = 1;
    if constexpr (!SOLO) {
        if (tid == 0) {
            uint32_t size = 0;
            s_place = join_team(r.team, r.team_size, size);
            s_size = size;
            if (s_place < 0) leave_team(r.team);
        }
        __syncthreads();
        place = s_place;
        team = static_cast<int32_t>(s_size);
        if (place < 0) return;
    }
    // LDS: the decision nodes' records (team: the first and third word of each), value columns, reach
    // planes, then (team) the probabilities of the edges into the nodes or (solo) the state and
    // the contributions
    constexpr int kRecBytes = SOLO ? 16 : 8;
    Rec4* const rec4 = reinterpret_cast<Rec4*>(s_raw);
    int2* const rec2 = reinterpret_cast<int2*>(s_raw);
    F* const val = reinterpret_cast<F*>(s_raw + static_cast<int64_t>(kRecBytes) * ((mr + 1) & ~1));
    F* const reach = val + static_cast<int64_t>(P) * mn;
    F* const sig = reach + static_cast<int64_t>(planes) * mr;
    F* const prob = SOLO ? sig : r.prob;
    F* const R = SOLO ? prob + r.Qp + r.Q0 : r.R;
    F* const S = SOLO ? R + r.Qp : r.S;
    constexpr int64_t V16 = 16 / sizeof(F);
    const int64_t con_at = P * int64_t{mn} + planes * int64_t{mr} + 3 * int64_t{r.Qp} + r.Q0;
    F* const con = SOLO ? val + (con_at + V16 - 1) / V16 * V16 : r.con;
    auto structure = [&](int32_t x) {  // {first child | own node << 16, parent | actor << 16 | k << 20}
        if constexpr (SOLO) return make_int2(rec4[x].x, rec4[x].z);
        else return rec2[x];
    };
    if constexpr (SOLO) {
        for (int i = tid; i < r.Qp + r.Q0; i += nt) prob[i] = r.prob[i];
        for (int i = tid; i < r.Qp; i += nt) R[i] = r.R[i];
        for (int i = tid; i < r.Qp; i += nt) S[i] = r.S[i];
    }
    const int64_t T0 = *r.T;  // counted at the launch's end
    uint32_t arrivals = 0;
    auto barrier = [&]() {
        if constexpr (SOLO) {
            __syncthreads();
        } else {
            // every store of the workgroup has reached the point of coherence before it arrives
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) {
                // the last of a group's members arrives for the group
                const int g = place / kResGroup;
                const uint32_t members = min(kResGroup, team - g * kResGroup);
                const uint32_t groups = (team + kResGroup - 1) / kResGroup;
                ++arrivals;
                if (agent_add(r.team->group[g], 1) + 1 == arrivals * members)
                    agent_add(r.team->bar, 1);
                while (static_cast<int32_t>(agent_load(r.team->bar) - arrivals * groups) < 0)
                    __builtin_amdgcn_s_sleep(1);
            }
            __syncthreads();
        }
    };

    // ---- one bin's sweeps and contributions
    // the bins are the trunk, of the first workgroup, and the others', taken in turn (a team of one
    // takes all); a workgroup with one bin keeps what does not change in LDS
    const int32_t b_lo = SOLO ? 0 : team > 1 && place == 0 ? r.bins : max(1, place);
    const int32_t b_step = team > 1 ? team - 1 : 1;
    const bool keeps = team > 1 ? place == 0 || b_lo + b_step >= r.bins : SOLO;
    int32_t loaded = -1;
    // operands of the loaded bin's ranks tid, tid + threads: kept over the iterations
    constexpr int KR = 2;
    int32_t slot_r[KR], y_r[KR];
    F rc_r[KR];
    auto sweep = [&](int32_t b, int32_t mask, bool keep) {
        const bool trunk = !SOLO && b == 0;
        const Rec4* tab = r.table + static_cast<int64_t>(b) * (D + 3);
        if (loaded != b) {
            __syncthreads();
            for (int i = tid; i < D + 3; i += nt) s_tab[i] = tab[i];
            __syncthreads();
        }
        const int32_t rbase = s_tab[D + 1].x, n_nodes = s_tab[D + 1].y, n_ranks = s_tab[D + 1].z;
        const int32_t nbase = s_tab[D + 1].w;
        const int l0 = s_tab[D + 2].x, nl = s_tab[D + 2].y;  // levels with decision nodes
        auto rlo = [&](int l) { return l <= D ? s_tab[l].y : n_ranks; };
        const Rec4* rec = r.rec + rbase;
        if (loaded != b) {
            // records, terminal values (a decision node's is computed before it is read), sigma_0
            for (int32_t c = 0; c < P; ++c) {
                const F* pay = r.pay + c * r.NB + nbase;
#pragma unroll 4
                for (int32_t i = tid; i < n_nodes; i += nt) val[c * mn + i] = pay[i];
            }
#pragma unroll
            for (int u = 0; u < KR; ++u) {
                const int32_t x = tid + u * nt;
                slot_r[u] = x < n_ranks ? r.slot[rbase + x] : 0;
                rc_r[u] = x < n_ranks ? r.reach_c[rbase + x] : F(0);
                y_r[u] = x < n_ranks ? rec[x].y : 0;
            }
#pragma unroll 4
            for (int32_t x = tid; x < n_ranks; x += nt) {
                const Rec4 q = rec[x];
                if constexpr (SOLO) rec4[x] = q;
                else rec2[x] = make_int2(q.x, q.z);
            }
            if constexpr (!SOLO) {
                // (a level's chance nodes are its last: 16 lanes each)
                __syncthreads();
                for (int l = l0; l < l0 + nl; ++l) {
                    const int32_t hi = rlo(l + 1), lo = hi - s_tab[l].w;
                    for (int32_t x = lo + (tid >> 4); x < hi; x += nt >> 4) {
                        const int2 q = rec2[x];
                        const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
                        const int32_t e0 = rec[x].y & 0x0FFFFFFF;
                        for (int32_t a = tid & 15; a < k; a += 16) sig[(q.x & 0xFFFF) + a] = prob[e0 + a];
                    }
                }
            }
            loaded = keeps ? b : -1;
            __syncthreads();
        }
        if (trunk) {
            // the subtrees' values
            for (int32_t c = 0; c < P; ++c)
                for (int32_t x = tid; x < r.roots; x += nt)
                    val[c * mn + r.ext[x]] = get<SOLO>(&r.root_val[c * r.roots + x]);
        }
        if constexpr (!SOLO) {
            // the strategy at the bin's player nodes, by the children it leads to
            auto stage = [&](int32_t x, int32_t y) {
                if ((static_cast<uint32_t>(y) >> 28) == 0) return;
                const int2 q = structure(x);
                const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
                const int32_t c0 = q.x & 0xFFFF, e0 = y & 0x0FFFFFFF;
                F s[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) s[a] = get<SOLO>(&prob[e0 + min(a, k - 1)]);
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    if (a < k) sig[c0 + a] = s[a];
                for (int32_t a = 4; a < k; ++a) sig[c0 + a] = get<SOLO>(&prob[e0 + a]);
            };
#pragma unroll
            for (int u = 0; u < KR; ++u)
                if (tid + u * nt < n_ranks) stage(tid + u * nt, y_r[u]);
#pragma unroll 2
            for (int32_t x = tid + KR * nt; x < n_ranks; x += nt) stage(x, rec[x].y);
        }
        // the roots' reach
        const int32_t x0 = s_tab[D + 2].z, x1 = s_tab[D + 2].w;
        if (SOLO || trunk) {
            if (tid < planes) reach[tid * mr] = F(1);
        } else {
            for (int32_t x = x0 + tid; x < x1; x += nt) {
                F p[RM];
#pragma unroll
                for (int k = 0; k < RM; ++k) p[k] = F(1);
#pragma unroll 4
                for (int i = 0; i < r.path_len; ++i) {
                    const int32_t e = r.path[i * r.roots + x];
                    const int32_t actor = static_cast<int32_t>(static_cast<uint32_t>(e) >> 28);
                    const F s = actor > 0 ? get<SOLO>(&prob[e & 0x0FFFFFFF]) : F(1);
#pragma unroll
                    for (int k = 0; k < RM; ++k)
                        if (k == actor - 1) p[k] *= s;
                }
                const int32_t d = r.root_rank[x];
#pragma unroll
                for (int k = 0; k < RM; ++k)
                    if (k < planes) reach[k * mr + d] = p[k];
            }
        }
        __syncthreads();
        // even wavefronts take the values, odd ones the reach (a few wavefronts issue one
        // instruction at a time: short code beats reading ahead here)
        const bool downward = wave & 1;
        const int32_t step = nw / 2 * 64, base = (wave >> 1) * 64, at = base + lane;
        for (int i = 0; i < nl; ++i) {
            const int l = l0 + nl - 1 - i, sums = s_tab[l].z, g = sums & kResLanes;
            // nodes that share lanes from rch: chance nodes (general sums: in small levels)
            const int32_t r1 = rlo(l + 1);
            const int32_t rch = NP > 0 && !(sums & kResGrouped) ? r1 : r1 - s_tab[l].w;
            if (downward) {
                const int ld = l0 + 1 + i;
                const int32_t end = i + 1 < nl ? rlo(ld + 1) : 0;
                for (int32_t x = rlo(ld) + at; x < end; x += step) {
                    const int2 q = structure(x);
                    const int32_t pr = q.y & 0xFFFF, actor = (q.y >> 16) & 15;
                    if (actor == 15) continue;  // a subtree's root
                    F s = F(1);
                    if constexpr (SOLO) s = prob[rec4[x].w];
                    else s = sig[static_cast<uint32_t>(q.x) >> 16];
#pragma unroll
                    for (int k = 0; k < RM; ++k)
                        if (k < planes) {
                            const F p = reach[k * mr + pr];
                            reach[k * mr + x] = k == actor - 1 ? p * s : p;
                        }
                }
            } else {
                for (int32_t x = rlo(l) + at; x < rch; x += step) {
                    const int2 q = structure(x);
                    const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
                    const int32_t c0 = q.x & 0xFFFF;
                    const F* const s = SOLO ? prob + (rec4[x].y & 0x0FFFFFFF) : sig + c0;
                    F* const own = val + (static_cast<uint32_t>(q.x) >> 16);
                    const F* const w = val + c0;
                    if constexpr (NP == 0) {
                        F v = F(0);
#pragma unroll 4
                        for (int32_t a = 0; a < k; ++a) v = fma_(s[a], w[a], v);
                        *own = v;
                    } else {
                        // a column at a time (all at once spill), its first four children, as good as
                        // always all, together
                        F s4[4];
#pragma unroll
                        for (int a = 0; a < 4; ++a) s4[a] = s[min(a, k - 1)];
                        for (int32_t c = 0; c < P; ++c) {
                            const F* const wc = w + c * mn;
                            F ch[4];
#pragma unroll
                            for (int a = 0; a < 4; ++a) ch[a] = wc[min(a, k - 1)];
                            F v = F(0);
                            if (!(sums & kResGrouped)) {
#pragma unroll
                                for (int a = 0; a < 4; ++a)
                                    if (a < k) v = fma_(s4[a], ch[a], v);
#pragma unroll 4
                                for (int32_t a = 4; a < k; ++a) v = fma_(s[a], wc[a], v);
                            } else {
                                // the butterfly over 64 lanes with a child each (at most 16 have one)
#pragma unroll
                                for (int a = 0; a < 4; ++a) ch[a] = a < k ? s4[a] * ch[a] : F(0);
                                F odd = ch[1] + ch[3];
                                v = ch[0] + ch[2];
                                if (k > 4) {
                                    auto at = [&](int32_t i) { return i < k ? s[i] * wc[i] : F(0); };
                                    v = odd = F(0);
#pragma unroll 1
                                    for (int a = 0; a < 4; ++a) {
                                        const F p = (at(a) + at(a + 8)) + (at(a + 4) + at(a + 12));
                                        if (a & 1) odd += p;
                                        else v += p;
                                    }
                                }
                                v += odd;
                            }
                            own[c * mn] = v;
                        }
                    }
                }
                if (r1 > rch) {
                    // a node by a lane group, then a butterfly
                    const int32_t items = (r1 - rch) << g;
                    for (int32_t bs = base; bs < items; bs += step) {
                        bool ok = bs + lane < items;
                        const int32_t x = rch + ((bs + lane) >> g);
                        const int2 q = ok ? structure(x) : make_int2(0, 0);
                        const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
                        if (NP > 0 && (sums & kResWide) && k > 64) ok = false;  // (below)
                        const int32_t c0 = q.x & 0xFFFF;
                        const F* s = sig + c0;
                        if constexpr (SOLO) s = prob + (ok ? rec4[x].y & 0x0FFFFFFF : 0);
                        // (every column's butterfly step together: one waits for the one before)
                        F v[CM];
#pragma unroll
                        for (int c = 0; c < CM; ++c) v[c] = F(0);
#pragma unroll kLaneUnroll
                        for (int32_t a = lane & ((1 << g) - 1); a < (ok ? k : 0); a += 1 << g)
#pragma unroll
                            for (int c = 0; c < CM; ++c)
                                if (c < P) v[c] = fma_(s[a], val[c * mn + c0 + a], v[c]);
                        for (int off = (1 << g) >> 1; off > 0; off >>= 1)
#pragma unroll
                            for (int c = 0; c < CM; ++c)
                                if (c < P) v[c] += __shfl_xor(v[c], off, 64);
                        if (ok && (lane & ((1 << g) - 1)) == 0) {
#pragma unroll
                            for (int c = 0; c < CM; ++c)
                                if (c < P) val[c * mn + (static_cast<uint32_t>(q.x) >> 16)] = v[c];
                        }
                    }
                }
            }
            if (NP > 0 && (sums & kResWide)) {
                // its nodes of more than 64 children by the workgroup: wavefront w of kWideWaves takes
                // children 64 w + lane, then every 64 kWideWaves-th; the wavefronts' sums in order
                for (int32_t x = rch; x < r1; ++x) {
                    const int2 q = structure(x);
                    const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
                    if (k <= 64) continue;
                    const int32_t c0 = q.x & 0xFFFF;
                    const F* const s = SOLO ? prob + (rec4[x].y & 0x0FFFFFFF) : sig + c0;
                    for (int w = wave; w < kWideWaves; w += nw)
                        for (int32_t c = 0; c < P; ++c) {
                            F v = F(0);
                            for (int32_t a = 64 * w + lane; a < k; a += 64 * kWideWaves)
                                v = fma_(s[a], val[c * mn + c0 + a], v);
                            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
                            if (lane == 0) s_red[w][c] = v;
                        }
                    __syncthreads();
                    if (tid < P) {
                        F sum = F(0);
                        for (int w = 0; w < kWideWaves; ++w) sum += s_red[w][tid];
                        val[tid * mn + (static_cast<uint32_t>(q.x) >> 16)] = sum;
                    }
                    __syncthreads();
                }
            }
            __syncthreads();
        }
        // contributions of the pass's players' nodes
        auto contribute = [&](int32_t x, int32_t y, int32_t slot, F rc) {
            const int32_t who = static_cast<int32_t>(static_cast<uint32_t>(y) >> 28);
            if (who == 0 || !((mask >> (who - 1)) & 1)) return;
            const int2 q = structure(x);
            const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(q.y) >> 20);
            const int32_t c0 = q.x & 0xFFFF;
            const int32_t col = NP > 0 ? who - 1 : 0;
            F* const to = con + slot;
            F cf = rc, own = F(0);
            if constexpr (NP > 0) {
#pragma unroll
                for (int c = 0; c < RM; ++c)
                    if (c < planes) {
                        const F p = reach[c * mr + x];
                        if (c == who - 1) own = p;
                        else cf *= p;
                    }
            } else {
                const F p1 = reach[x], p2 = reach[mr + x];
                cf = (who == 2 ? p1 : p2) * cf;
                own = who == 2 ? p2 : p1;
            }
            const F u = val[col * mn + (static_cast<uint32_t>(q.x) >> 16)];
            const F* const w = val + col * mn + c0;
            // 16 bytes at a time: k contributions, the own reach, padding
            constexpr int V = 16 / sizeof(F);
            for (int32_t a = 0; a <= k; a += V) {
                F o[V];
#pragma unroll
                for (int e = 0; e < V; ++e)
                    o[e] = a + e < k ? cf * (w[min(a + e, k - 1)] - u) : own;
                put_vec<SOLO>(to + a, o);
            }
        };
#pragma unroll
        for (int u = 0; u < KR; ++u)
            if (tid + u * nt < n_ranks) contribute(tid + u * nt, y_r[u], slot_r[u], rc_r[u]);
        for (int32_t x = tid + KR * nt; x < n_ranks; x += nt)
            contribute(x, rec[x].y, r.slot[rbase + x], r.reach_c[rbase + x]);
        if (!SOLO && !trunk)
            for (int32_t c = 0; c < P; ++c)
                for (int32_t x = x0 + tid; x < x1; x += nt)
                    put<SOLO>(&r.root_val[c * r.roots + x],
                              val[c * mn + (static_cast<uint32_t>(structure(r.root_rank[x]).x) >> 16)]);
        if (keep) {
            // the launch's last iteration: node values and reach for inspection
            for (int32_t c = 0; c < P; ++c)
                for (int32_t i = tid; i < n_nodes; i += nt) r.val[c * r.NB + nbase + i] = val[c * mn + i];
            for (int32_t c = 0; c < planes; ++c)
                for (int32_t x = tid; x < n_ranks; x += nt)
                    r.reach[static_cast<int64_t>(c) * r.ND + rbase + x] = reach[c * mr + x];
        }
    };

    // ---- the infosets: 1 << (alog + mlog) lanes each, actions in the low bits; the first workgroup
    // of a team takes the trunk's, the others the rest
    const int alog = r.alog, mlog = r.mlog, hlog = alog + mlog;
    const bool split = !SOLO && team > 1;
    const int32_t h_lo = split && place > 0 ? r.trunk_sets : 0;
    const int32_t h_hi = split && place == 0 ? r.trunk_sets : r.Hp;
    const int32_t h_wg = split && place > 0 ? place - 1 : 0, h_wgs = split && place > 0 ? team - 1 : 1;
    // (consecutive groups of a wavefront's infosets go to different workgroups)
    const int32_t hstep = h_wgs * nt >> hlog;
    const int32_t hw = h_lo + (((wave * h_wgs + h_wg) * 64) >> hlog);  // the wavefront's first infoset
    const int32_t h0 = hw + (lane >> hlog);
    const int j = lane & ((1 << alog) - 1), ms = (lane >> alog) & ((1 << mlog) - 1);
    const int gbase = lane & ~((1 << hlog) - 1);
    const Rec4 own_set = h0 < h_hi ? r.sets[h0] : Rec4{0, 0, 0, 0};

    __syncthreads();
    for (int32_t it = 0; it < n; ++it) {
        const F t = static_cast<F>(T0 + it + 1);
        F wt = rule.linear ? t : F(1);
        F d_pos = F(1), d_neg = F(1), d_avg = F(1);
        if (rule.variant == 2) {
            wt = F(1);
            dcfr_discounts(rule, t, d_pos, d_neg, d_avg);
        }
        for (int32_t pass = 0; pass < passes; ++pass) {
            const int32_t mask = passes > 1 ? 1 << pass : rule.players;
            const bool keep = it == n - 1 && pass == passes - 1;
            for (int32_t b = b_lo; b < r.bins; b += b_step) sweep(b, mask, keep);
            barrier();
            if (!SOLO && place == 0) {
                sweep(0, mask, keep);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
            }
            // (every lane of a wavefront runs the same rounds; groups past the end idle)
            for (int32_t hb = hw, first = 1; hb < h_hi; hb += hstep, first = 0) {
                const int32_t h = hb + (lane >> hlog);
                const bool in = h < h_hi;
                const Rec4 s = first ? own_set : in ? r.sets[h] : Rec4{0, 0, 0, 0};
                const int32_t k = s.w & 0xFFFFFF, who = s.w >> 24;
                const bool act = in && ((mask >> (who - 1)) & 1) && j < k;
                F ro = F(0), so = F(0), po = F(0);
                if (act && ms == 0) {
                    ro = R[s.x + j];
                    so = S[s.x + j];
                    po = get<SOLO>(&prob[s.x + j]);
                }
                // members four (times the lanes over members) at a time, their reads together. Two
                // players: added in member order. General sums, whose infosets can hold hundreds of
                // members: in the order of r.waves wavefronts (sum_order.hpp)
                F racc = F(0), own = F(0);
                const int32_t stride = res_stride(k, sizeof(F));
                const int32_t members = act ? s.z : 0;
                if constexpr (NP > 0) {
                    // lane t of a wavefront's 64 has the members t, t + 64 waves, ...: this one stands
                    // for the lanes ms + (q << mlog), whose sums meet as in the wavefront's
                    // butterfly (q in bit-reversed order: the far halves first), then over its own
                    // neighbours. Lanes and wavefronts past every infoset's members add nothing and
                    // are left out; four are read together.
                    auto read = [&](int32_t m, int32_t column) {
                        const F x = get<SOLO>(&con[s.y + max(min(m, members - 1), 0) * stride + column]);
                        return m < members ? x : F(0);
                    };
                    if (!__any(members > min(64, 4 << mlog))) {
                        constexpr int kQ[4] = {0, 2, 1, 3};
                        F xr[4], xo[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            xr[i] = read(ms + (kQ[i] << mlog), j);
                            xo[i] = read(ms + (kQ[i] << mlog), k);
                        }
                        racc = (xr[0] + xr[1]) + (xr[2] + xr[3]);
                        own = (xo[0] + xo[1]) + (xo[2] + xo[3]);
                        for (int off = 1 << hlog >> 1; off >= 1 << alog; off >>= 1) {
                            racc += __shfl_xor(racc, off, 64);
                            own += __shfl_xor(own, off, 64);
                        }
                    } else {
                        int lq = 0, wu = 1;  // log2 of the q's, wavefronts
                        while (lq < 6 - mlog && __any(members > 1 << (lq + mlog))) ++lq;
                        while (wu < r.waves && __any(members > 64 * wu)) ++wu;
                        // contributions and own reaches together, in double precision one after
                        // the other (together they spill)
                        constexpr int U = sizeof(F) == 4 ? 2 : 1;
                        for (int t = 0; t < 2; t += U) {
                            F total[U], half[4][U];
#pragma unroll
                            for (int u = 0; u < U; ++u) total[u] = F(0);
                            for (int b = 0; b < wu << lq; b += 4) {
                                F x[4][U];
                                int32_t m[4];
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const int q =
                                        static_cast<int>(__brev((b + i) & ((1 << lq) - 1)) >> 1 >> (31 - lq));
                                    m[i] = b + i < wu << lq ? 64 * ((b + i) >> lq) + ms + (q << mlog) : members;
#pragma unroll
                                    for (int u = 0; u < U; ++u) x[i][u] = read(m[i], t + u == 0 ? j : k);
                                }
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    for (int32_t mm = m[i] + 64 * r.waves; mm < members; mm += 64 * r.waves)
#pragma unroll
                                        for (int u = 0; u < U; ++u) x[i][u] += read(mm, t + u == 0 ? j : k);
                                int parts = min(4 >> lq, wu - (b >> lq));  // complete but for their lanes
                                if (lq >= 1) {
#pragma unroll
                                    for (int u = 0; u < U; ++u) {
                                        x[0][u] += x[1][u];
                                        x[1][u] = x[2][u] + x[3][u];
                                        if (lq >= 2) x[0][u] += x[1][u];
                                    }
                                }
                                if (lq >= 2) {
                                    parts = 1;
#pragma unroll
                                    for (int i = 0; i < 4; ++i)
                                        if (parts != 0 && i < lq - 2) {  // a complete half joins its other half
                                            const bool second = (b >> (2 + i)) & 1;
#pragma unroll
                                            for (int u = 0; u < U; ++u) {
                                                if (second) x[0][u] = half[i][u] + x[0][u];
                                                else half[i][u] = x[0][u];
                                            }
                                            if (!second) parts = 0;
                                        }
                                }
                                if (parts > 0)
                                    for (int off = 1 << hlog >> 1; off >= 1 << alog; off >>= 1)
#pragma unroll
                                        for (int i = 0; i < 4; ++i)
                                            if (i < parts)
#pragma unroll
                                                for (int u = 0; u < U; ++u)
                                                    x[i][u] += __shfl_xor(x[i][u], off, 64);
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (i < parts)
#pragma unroll
                                        for (int u = 0; u < U; ++u) total[u] += x[i][u];
                            }
                            if (t == 0) racc = total[0];
                            if (t == 1 || U == 2) own = total[U - 1];
                        }
                    }
                } else if (mlog == 0) {
                    for (int32_t m = 0; m < members; m += 4) {
                        F xr[4], xo[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const F* from = con + s.y + min(m + i, members - 1) * stride;
                            xr[i] = get<SOLO>(&from[j]);
                            xo[i] = get<SOLO>(&from[k]);
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (m + i < members) {
                                racc += xr[i];
                                own += xo[i];
                            }
                    }
                } else {
                    for (int32_t m = 0; __any(m < members); m += 4 << mlog) {
                        F xr[4], xo[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            xr[i] = xo[i] = F(0);
                            if (members > 0) {
                                const F* from =
                                    con + s.y + min(m + (i << mlog) + ms, members - 1) * stride;
                                xr[i] = get<SOLO>(&from[j]);
                                xo[i] = get<SOLO>(&from[k]);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            for (int q = 0; q < 1 << mlog; ++q) {
                                const F a = __shfl(xr[i], gbase + j + (q << alog), 64);
                                const F o = __shfl(xo[i], gbase + j + (q << alog), 64);
                                if (m + (i << mlog) + q < members) {
                                    racc += a;
                                    own += o;
                                }
                            }
                    }
                }
                F rn = F(0);
                if (act && ms == 0) {
                    rn = NP == 0 && who == 2 ? ro - racc : ro + racc;
                    if (rule.variant == 1) rn = pos_(rn);
                    else if (rule.variant == 2) rn *= rn > F(0) ? d_pos : d_neg;
                    R[s.x + j] = rn;
                    const F sn = fma_(wt * own, po, so);
                    S[s.x + j] = rule.variant == 2 ? sn * d_avg : sn;
                }
                const F pr = pos_(rn);
                F sum = F(0);
                for (int a0 = 0; a0 < 1 << alog; a0 += 4) {
                    F x[4];
#pragma unroll
                    for (int a = 0; a < 4; ++a) x[a] = __shfl(pr, gbase + ((a0 + a) & ((1 << alog) - 1)), 64);
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        if (a0 + a < k) sum += x[a];
                }
                if (act && ms == 0)
                    put<SOLO>(&prob[s.x + j], sum > F(0) ? pr / sum : F(1) / static_cast<F>(k));
            }
            barrier();
        }
    }
    if constexpr (SOLO) {
        for (int i = tid; i < r.Qp; i += nt) r.prob[i] = prob[i];
        for (int i = tid; i < r.Qp; i += nt) r.R[i] = R[i];
        for (int i = tid; i < r.Qp; i += nt) r.S[i] = S[i];
        if (tid == 0) *r.T = T0 + n;
    } else if (tid == 0) {
        if (place == 0) *r.T = T0 + n;  // (every member read it before the first barrier)
        leave_team(r.team);
    }
}

__global__ void k_resident_reset(ResTeam* team) {
    uint32_t* w = reinterpret_cast<uint32_t*>(team);
    for (int i = threadIdx.x; i < static_cast<int>(sizeof(ResTeam) / 4); i += blockDim.x) w[i] = 0;
}

template <class F>
__global__ void k_resident_pay(int64_t N, int64_t NB, int32_t cols, const int32_t* __restrict__ node,
                               const F* __restrict__ payoff, F* __restrict__ pay) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= NB) return;
    const int32_t v = node[i];
    for (int32_t c = 0; c < cols; ++c) pay[c * NB + i] = payoff[c * N + v];
}

template <class F>
size_t lds_bytes(const Resident<F>& r) {
    const int64_t P = r.players > 0 ? r.players : 1, planes = r.players > 0 ? r.players : 2;
    const int64_t recs = ((r.max_ranks + 1) & ~1) * int64_t{r.mode == RES_SOLO ? 16 : 8};
    int64_t n = P * r.max_nodes + planes * r.max_ranks;
    if (r.mode == RES_SOLO) n += 3 * int64_t{r.Qp} + r.Q0 + r.n_con + 16 / sizeof(F);
    else n += r.max_nodes;
    return static_cast<size_t>(recs + n * static_cast<int64_t>(sizeof(F)));
}

}  // namespace

template <class F>
void resident_shape(Resident<F>& r, const ResPlan& p) {
    r.mode = p.mode;
    r.bins = p.bins;
    r.team_size = std::min(p.bins, kResTeam);
    r.trunk_sets = p.trunk_sets;
    r.roots = p.roots;
    r.path_len = p.path_len;
    r.NB = r.N + p.roots;
    r.max_nodes = p.max_nodes;
    r.max_ranks = p.max_ranks;
    r.n_con = p.contributions;
    r.alog = 0;
    while ((1 << r.alog) < p.max_actions) ++r.alog;
    r.mlog = 0;
    const int32_t each = r.players > 0 ? 4 : 16;  // members of a lane
    while (r.alog + r.mlog < 6 && (each << r.mlog) < p.mean_members) ++r.mlog;
    r.waves = p.waves;
    // a solo game's threads follow its widest work (fewer wavefronts meet sooner)
    int32_t threads = kResMaxThreads;
    if (r.mode == RES_SOLO) {
        const int64_t items = std::max<int64_t>(r.max_ranks, int64_t{r.Hp} << (r.alog + r.mlog));
        threads = 128;
        while (threads < kResMaxThreads && threads < items) threads *= 2;
    }
    r.threads = threads;
}

template <class F>
void launch_resident_pay(const Resident<F>& r, const F* payoff, hipStream_t st) {
    hipLaunchKernelGGL(k_resident_pay<F>, dim3(static_cast<unsigned>((r.NB + 255) / 256)), dim3(256), 0, st,
                       r.N, r.NB, r.players > 0 ? r.players : 1, reinterpret_cast<const int32_t*>(r.val),
                       payoff, r.pay);
}

template <class F>
void launch_resident_reset(const Resident<F>& r, hipStream_t st) {
    hipLaunchKernelGGL(k_resident_reset, dim3(1), dim3(256), 0, st, r.team);
}

template <class F>
void launch_resident(const Resident<F>& r, const UpdateRule& rule, bool alternating, int32_t n,
                     hipStream_t st) {
    const int32_t passes = alternating ? (r.players > 0 ? r.players : 2) : 1;
    const int32_t most = resident_launch_iterations(r, passes);
    const size_t lds = lds_bytes(r);
    // workgroups go to the XCDs in turn: eight per member of a one-XCD team bring them to each
    Resident<F> team = r;
    team.team_size = resident_workgroups(r);
    const int32_t grid = team.team_size <= kResXcd && r.mode == RES_TEAM ? 8 * team.team_size : team.team_size;
    for (int64_t i = 0; i < n; i += most) {
        const int32_t m = static_cast<int32_t>(std::min<int64_t>(most, n - i));
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(r.threads), lds, st, team, rule, passes, m);
        };
        if (r.players > 0) {
            const bool few = r.players <= 4;
            if (r.mode == RES_SOLO) few ? go(k_resident<F, RES_SOLO, 4>) : go(k_resident<F, RES_SOLO, kMaxPlayers>);
            else few ? go(k_resident<F, RES_TEAM, 4>) : go(k_resident<F, RES_TEAM, kMaxPlayers>);
        } else {
            if (r.mode == RES_SOLO) go(k_resident<F, RES_SOLO, 0>);
            else go(k_resident<F, RES_TEAM, 0>);
        }
    }
}

#define CFR_RES_INSTANTIATE(F)                                                                \
    template void resident_shape<F>(Resident<F>&, const ResPlan&);                            \
    template void launch_resident_pay<F>(const Resident<F>&, const F*, hipStream_t);          \
    template void launch_resident_reset<F>(const Resident<F>&, hipStream_t);                  \
    template void launch_resident<F>(const Resident<F>&, const UpdateRule&, bool, int32_t,    \
                                     hipStream_t);
CFR_RES_INSTANTIATE(float)
CFR_RES_INSTANTIATE(double)
#undef CFR_RES_INSTANTIATE

}  // namespace cfr
