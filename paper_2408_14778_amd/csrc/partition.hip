// Device side of the subtree-partitioned, out-of-core iteration.
//
// The host link bounds it: 57 GB/s by copy, 53 GB/s by loads of a kernel, against 5 TB/s of device
// memory. So every node below the resident levels is read once per pass, by the kernel that uses it,
// as 4 bytes and a bit (double precision: 8 bytes and a bit): a decision node's infoset, from which
// its player, fan-out and edges follow, or a terminal's payoff; the children's places are prefix
// sums of the fan-outs. Copying windows of full records (21 and 25 bytes a node) and running their
// levels as launches of their own took 3.08 ms per iteration of a game of 3,309,121 nodes cut at
// level 7 (13 windows, 209 launches).
#include "partition.hpp"

#include <cstring>

namespace cfr {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }

template <class F>
struct WordOf;
template <>
struct WordOf<float> {
    using T = uint32_t;
};
template <>
struct WordOf<double> {
    using T = uint64_t;
};

__device__ __forceinline__ void load_part(const uint32_t* p, uint32_t (&w)[kStreamPart]) {
    const uint4 a = *reinterpret_cast<const uint4*>(p);
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
}
__device__ __forceinline__ void load_part(const uint64_t* p, uint64_t (&w)[kStreamPart]) {
    const ulonglong2 a = reinterpret_cast<const ulonglong2*>(p)[0];
    const ulonglong2 b = reinterpret_cast<const ulonglong2*>(p)[1];
    w[0] = a.x; w[1] = a.y; w[2] = b.x; w[3] = b.y;
}

// What a code stands for: the first edge and the fan-out, and who acts.
struct Sets {
    int32_t Hp, Qp;
    const int32_t *q_offset, *cq_offset;
    const int8_t* infoset_player;
};
__device__ __forceinline__ void decode(const Sets& s, int32_t code, int32_t& edge, int32_t& k, int& who) {
    const bool chance = code >= s.Hp;
    const int32_t* o = chance ? s.cq_offset + (code - s.Hp) : s.q_offset + code;
    const int32_t a = o[0];
    k = o[1] - a;
    edge = chance ? s.Qp + a : a;
    who = chance ? 0 : s.infoset_player[code];
}

// The regret contributions and own reach of a player's node with value u, added to the per-pair
// and per-infoset accumulators (signs and reaches as the node engine's bottom-up pass);
// child_value(a): the value of action a's child.
template <class F, class V>
__device__ __forceinline__ void add_node(int who, int32_t h, int32_t edge, int32_t k, F u, F r1, F r2,
                                         F rc, const V& child_value, F* rtilde, F* pibar) {
    const F cf = (who == 1 ? r2 : r1) * rc;
    const F w = who == 1 ? cf : -cf;
    for (int32_t a = 0; a < k; ++a) unsafeAtomicAdd(&rtilde[edge + a], w * (child_value(a) - u));
    unsafeAtomicAdd(&pibar[h], who == 1 ? r1 : r2);
}

// A level between the cuts, top-down: terminals write their value, the others their children's reach.
template <class F>
__global__ void k_mid_down(int32_t n, int32_t id0, int64_t N, Sets s, const int32_t* __restrict__ code,
                           const int32_t* __restrict__ child, const F* __restrict__ pay,
                           const F* __restrict__ prob, F* __restrict__ value, F* __restrict__ reach) {
    const int32_t i = static_cast<int32_t>(blockIdx.x) * kThreads + static_cast<int32_t>(threadIdx.x);
    if (i >= n) return;
    const int32_t h = code[i], id = id0 + i;
    if (h < 0) {
        value[id] = pay[i];
        return;
    }
    int32_t edge, k;
    int who;
    decode(s, h, edge, k, who);
    const F r1 = reach[id], r2 = reach[N + id], rc = reach[2 * N + id];
    const int32_t c0 = child[i];
    for (int32_t a = 0; a < k; ++a) {
        const F p = prob[edge + a];
        reach[c0 + a] = who == 1 ? r1 * p : r1;
        reach[N + c0 + a] = who == 2 ? r2 * p : r2;
        reach[2 * N + c0 + a] = who == 0 ? rc * p : rc;
    }
}

// The same level bottom-up.
template <class F>
__global__ void k_mid_up(int32_t n, int32_t id0, int64_t N, Sets s, const int32_t* __restrict__ code,
                         const int32_t* __restrict__ child, const F* __restrict__ prob,
                         F* __restrict__ value, const F* __restrict__ reach, F* __restrict__ rtilde,
                         F* __restrict__ pibar) {
    const int32_t i = static_cast<int32_t>(blockIdx.x) * kThreads + static_cast<int32_t>(threadIdx.x);
    if (i >= n) return;
    const int32_t h = code[i], id = id0 + i;
    if (h < 0) return;
    int32_t edge, k;
    int who;
    decode(s, h, edge, k, who);
    const int32_t c0 = child[i];
    F u = F(0);
    for (int32_t a = 0; a < k; ++a) u = fma_(prob[edge + a], value[c0 + a], u);
    value[id] = u;
    if (who > 0)
        add_node(who, h, edge, k, u, reach[id], reach[N + id], reach[2 * N + id],
                 [&](int32_t a) { return value[c0 + a]; }, rtilde, pibar);
}

// A run of subtrees, one workgroup: every record is read once from host memory and staged with the
// edge probabilities in LDS, in which both sweeps then run (a level costs an LDS barrier instead
// of a launch). Only the accumulators and the roots' reach and value are in device memory.
template <class F>
__global__ void __launch_bounds__(kThreads) k_stream_run(const StreamUnit* __restrict__ units,
                                                         const typename WordOf<F>::T* __restrict__ stream,
                                                         int32_t cap, int64_t N, Sets s,
                                                         const F* __restrict__ prob,
                                                         F* __restrict__ value, F* __restrict__ reach,
                                                         F* __restrict__ rtilde, F* __restrict__ pibar) {
    using W = typename WordOf<F>::T;
    constexpr int kPart = kStreamPart, kWaves = kThreads / 64;
    extern __shared__ uint64_t s_mem[];
    __shared__ int32_t s_sum[kWaves];
    // per node: edge probability, value (a decision's code until then: words of one type, so that a
    // code's read stays ahead of the value's write), reaches; first edge; who (2 bits), fan-out
    // (12) and first child (12)
    F* const s_prob = reinterpret_cast<F*>(s_mem);
    W* const s_word = reinterpret_cast<W*>(s_prob + cap);
    F *const s_r1 = reinterpret_cast<F*>(s_word + cap), *const s_r2 = s_r1 + cap, *const s_rc = s_r2 + cap;
    int32_t* const s_edge = reinterpret_cast<int32_t*>(s_rc + cap);
    uint32_t* const s_meta = reinterpret_cast<uint32_t*>(s_edge + cap);
    uint16_t* const s_level = reinterpret_cast<uint16_t*>(s_meta + cap);  // cap + 2 level offsets
    auto value_of = [&](int i) { return __builtin_bit_cast(F, s_word[i]); };
    auto first_child = [&](int i) { return static_cast<int>(s_meta[i] >> 14); };

    const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const StreamUnit u = units[blockIdx.x];
    const int n = u.n, roots = u.roots;
    const uint32_t* bits = reinterpret_cast<const uint32_t*>(stream + u.at);
    const int bit_words = (((n + 31) / 32 * 4 + static_cast<int>(sizeof(W)) - 1) /
                               static_cast<int>(sizeof(W)) + kPart - 1) / kPart * kPart;
    const W* rec = stream + u.at + bit_words;
    for (int i = tid; i < roots; i += kThreads) {
        const int64_t id = u.id0 + i;
        s_r1[i] = reach[id];
        s_r2[i] = reach[N + id];
        s_rc[i] = reach[2 * N + id];
    }
    int carry = roots;  // first child of the next part's first node
    for (int base = 0; base < n; base += kPart * kThreads) {
        const int i0 = base + kPart * tid;
        W w[kPart] = {};
        uint32_t dec = 0;
        if (i0 < n) {
            load_part(rec + i0, w);
            dec = bits[i0 >> 5] >> (i0 & 31);
        }
        int32_t edge[kPart], k[kPart];
        int who[kPart];
        int mine = 0;
#pragma unroll
        for (int j = 0; j < kPart; ++j) {
            edge[j] = k[j] = 0;
            who[j] = 3;
            if (i0 + j < n && ((dec >> j) & 1) != 0)
                decode(s, static_cast<int32_t>(w[j]), edge[j], k[j], who[j]);
            mine += k[j];
        }
        int before = mine;
        for (int off = 1; off < 64; off <<= 1) {
            const int x = __shfl_up(before, off, 64);
            if (lane >= off) before += x;
        }
        if (lane == 63) s_sum[wave] = before;
        before -= mine;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) {
            const int x = s_sum[v];
            if (v < wave) before += x;
            all += x;
        }
        __syncthreads();
        int c = carry + before;
        carry += all;
#pragma unroll
        for (int j = 0; j < kPart; ++j) {
            if (i0 + j < n) {
                s_word[i0 + j] = w[j];
                s_edge[i0 + j] = edge[j];
                s_meta[i0 + j] = static_cast<uint32_t>(who[j]) | static_cast<uint32_t>(k[j]) << 2 |
                                 static_cast<uint32_t>(c) << 14;
            }
#pragma unroll 4
            for (int a = 0; a < k[j]; ++a) s_prob[c + a] = prob[edge[j] + a];
            c += k[j];
        }
    }
    __syncthreads();
    int levels = 0;
    for (int lo = 0, hi = roots; lo < hi; ++levels) {
        if (tid == 0) s_level[levels] = static_cast<uint16_t>(lo);
        const int end = hi < n ? first_child(hi) : n;
        for (int i = lo + tid; i < hi; i += kThreads) {
            const uint32_t m = s_meta[i];
            const int who = m & 3, k = (m >> 2) & 0xfff, c = m >> 14;
            const F r1 = s_r1[i], r2 = s_r2[i], rc = s_rc[i];
            for (int a = c; a < c + k; ++a) {
                const F p = s_prob[a];
                s_r1[a] = who == 1 ? r1 * p : r1;
                s_r2[a] = who == 2 ? r2 * p : r2;
                s_rc[a] = who == 0 ? rc * p : rc;
            }
        }
        lo = hi;
        hi = end;
        __syncthreads();
    }
    int hi = n;
    for (int l = levels - 1; l >= 0; --l) {
        const int lo = s_level[l];
        for (int i = lo + tid; i < hi; i += kThreads) {
            const uint32_t m = s_meta[i];
            const int who = m & 3, k = (m >> 2) & 0xfff, c = m >> 14;
            if (who == 3) continue;
            F v = F(0);
            for (int a = c; a < c + k; ++a) v = fma_(s_prob[a], value_of(a), v);
            const int32_t h = static_cast<int32_t>(s_word[i]);
            s_word[i] = __builtin_bit_cast(W, v);
            if (who > 0)
                add_node(who, h, s_edge[i], k, v, s_r1[i], s_r2[i], s_rc[i],
                         [&](int32_t a) { return value_of(c + a); }, rtilde, pibar);
        }
        hi = lo;
        __syncthreads();
    }
    for (int i = tid; i < roots; i += kThreads) value[u.id0 + i] = value_of(i);
}

template <class F>
size_t run_lds(int32_t cap) {
    return static_cast<size_t>(cap) * (5 * sizeof(F) + 8 + 2) + 8;
}

template <class T>
int pinned(T** p, int64_t bytes) {
    *p = nullptr;
    if (bytes <= 0) return 0;
    return hipHostMalloc(reinterpret_cast<void**>(p), static_cast<size_t>(bytes),
                         hipHostMallocDefault) == hipSuccess
               ? 0
               : -1;
}

}  // namespace

template <class F>
int PartDev<F>::upload() {
    StreamPlan& P = plan;
    const int64_t mid = static_cast<int64_t>(P.mid_code.size());
    const size_t unit_bytes = P.units.size() * sizeof(StreamUnit);
    const size_t stream_bytes = static_cast<size_t>(P.words) * sizeof(F);
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_stream_run<F>),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(run_lds<F>(kStreamMax))) != hipSuccess)
        return -1;
    if (pinned(&h_stream, static_cast<int64_t>(stream_bytes)) ||
        pinned(&h_units, static_cast<int64_t>(unit_bytes)) ||
        pinned(&h_code, mid * int64_t{sizeof(int32_t)}) ||
        pinned(&h_child, mid * int64_t{sizeof(int32_t)}) || pinned(&h_pay, mid * int64_t{sizeof(F)})) {
        release();
        return -1;
    }
    if (stream_bytes > 0)
        std::memcpy(h_stream,
                    sizeof(F) == 8 ? static_cast<const void*>(P.stream64.data()) : P.stream32.data(),
                    stream_bytes);
    if (unit_bytes > 0) std::memcpy(h_units, P.units.data(), unit_bytes);
    if (mid > 0) {
        std::memcpy(h_code, P.mid_code.data(), mid * sizeof(int32_t));
        std::memcpy(h_child, P.mid_child.data(), mid * sizeof(int32_t));
        for (int64_t i = 0; i < mid; ++i) h_pay[i] = static_cast<F>(P.mid_pay[i]);
    }
    // the host vectors are no longer needed: the pinned copies are what each pass reads
    P.stream32 = {};
    P.stream64 = {};
    P.units = {};
    P.mid_code = {};
    P.mid_child = {};
    P.mid_pay = {};
    return 0;
}

template <class F>
void PartDev<F>::release() {
    for (void* p : {h_stream, static_cast<void*>(h_units), static_cast<void*>(h_code),
                    static_cast<void*>(h_child), static_cast<void*>(h_pay)})
        if (p != nullptr) (void)hipHostFree(p);
    h_stream = nullptr;
    h_units = nullptr;
    h_code = h_child = nullptr;
    h_pay = nullptr;
}

template <class F>
void launch_partitioned_pass(const DevT<F>& d, const PartDev<F>& Pd, const UpdateRule& rule,
                             hipStream_t st) {
    const StreamPlan& P = Pd.plan;
    const int32_t* lo = Pd.level_offset.data();
    const int32_t cut = P.cut, nl = P.split - cut + 1;
    const Sets s{static_cast<int32_t>(d.Hp), static_cast<int32_t>(d.Qp), d.q_offset, d.cq_offset,
                 d.infoset_player};
    auto blocks = [](int32_t n) { return dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads)); };
    // resident top-down: levels 1 .. cut
    launch_top_reach(d, lo, cut, rule.count ? d.T : nullptr, st);
    for (int32_t g = 0; g < P.groups; ++g) {
        // (stream order keeps a group's use of the window after the group before it)
        const size_t at = static_cast<size_t>(g) * nl;
        for (int32_t i = 0; i + 1 < nl; ++i)
            if (P.count[at + i] > 0)
                hipLaunchKernelGGL(k_mid_down<F>, blocks(P.count[at + i]), dim3(kThreads), 0, st,
                                   P.count[at + i], P.id[at + i], d.N, s, Pd.h_code + P.rec[at + i],
                                   Pd.h_child + P.rec[at + i], Pd.h_pay + P.rec[at + i], d.prob,
                                   d.value, d.reach);
        const int32_t u0 = P.unit0[g], u1 = P.unit0[g + 1];
        if (u1 > u0)
            hipLaunchKernelGGL(k_stream_run<F>, dim3(static_cast<unsigned>(u1 - u0)), dim3(kThreads),
                               run_lds<F>(P.max_unit), st, Pd.h_units + u0,
                               static_cast<const typename WordOf<F>::T*>(Pd.h_stream), P.max_unit, d.N,
                               s, d.prob, d.value, d.reach, d.rtilde, d.pibar);
        for (int32_t i = nl - 2; i >= 0; --i)
            if (P.count[at + i] > 0)
                hipLaunchKernelGGL(k_mid_up<F>, blocks(P.count[at + i]), dim3(kThreads), 0, st,
                                   P.count[at + i], P.id[at + i], d.N, s, Pd.h_code + P.rec[at + i],
                                   Pd.h_child + P.rec[at + i], d.prob, d.value, d.reach, d.rtilde,
                                   d.pibar);
    }
    launch_top_values(d, lo, cut, st);  // resident bottom-up: levels cut - 1 .. 0
    launch_infoset_pass(d, rule, rule.count != 0, st);
}

template struct PartDev<float>;
template struct PartDev<double>;
template void launch_partitioned_pass<float>(const DevT<float>&, const PartDev<float>&,
                                             const UpdateRule&, hipStream_t);
template void launch_partitioned_pass<double>(const DevT<double>&, const PartDev<double>&,
                                              const UpdateRule&, hipStream_t);

}  // namespace cfr
