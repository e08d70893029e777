// Warm-start network kernels for gfx950: BF16 MFMA GEMMs with FP32 accumulation, the masked
// softmax cross-entropy, Adam, the poker-subgame feature extractor and the warm start of
// cumulative regrets from predicted strategies.
//
// The network (3 layers, ReLU) maps infoset features to a distribution over action slots;
// the warm start turns it into initial cumulative regrets R0(h, a) = w * m(h) * p(h, a),
// where m(h) is the magnitude of h's regrets after one iteration from zero. CFR from zero
// regrets remains the fallback (the caller decides, by exploitability).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "mlp.hpp"

namespace cfr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int64_t gid() {
    return static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
}

inline unsigned blocks_for(int64_t n, int t) { return static_cast<unsigned>((n + t - 1) / t); }

// C = epilogue(A . B) on 32 x 32 tiles, one wavefront per tile, v_mfma_f32_32x32x16_bf16.
// A(i, k) = A[i * a_i + k * a_k] (M x K), B(k, j) = B[k * b_k + j * b_j] (K x N), bf16.
// Operand fragments: lane l holds A rows i = l % 32 and B columns j = l % 32, with the 8
// k-values 8 * (l / 32) .. + 7 of the current 16-wide k step; the 32 x 32 FP32 result has
// element e of lane l at row 8 * (e / 4) + 4 * (l / 32) + e % 4, column l % 32.
// Epilogue: + bias[j] (if bias), then mode 0: store FP32; 1: relu, store BF16; 2: multiply by
// (gate[i, j] > 0) (the ReLU derivative of the layer's output), store BF16.
// Split K (weight gradients, where K is the batch): workgroup z of gridDim.z takes k in
// [z kps, (z + 1) kps) and stores its FP32 partial tile to part[z][M][N]; k_sum_splits adds the
// partials in z order (deterministic) and applies mode 0.
__global__ void __launch_bounds__(64) k_gemm(int M, int N, int K, const __bf16* __restrict__ A,
                                             int64_t a_i, int64_t a_k,
                                             const __bf16* __restrict__ B, int64_t b_k,
                                             int64_t b_j, const float* __restrict__ bias, int mode,
                                             const __bf16* __restrict__ gate, float* __restrict__ Cf,
                                             __bf16* __restrict__ Cb, int64_t ldc, int kps,
                                             float* __restrict__ part) {
    const int lane = threadIdx.x;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    const int r = lane & 31, half = lane >> 5;
    const int ai = m0 + r, bj = n0 + r;
    const int kbeg = blockIdx.z * kps;
    const int kend = min(K, kbeg + kps);
    floatx16 acc = {};
    for (int k0 = kbeg; k0 < kend; k0 += 16) {
        bf16x8 fa, fb;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + 8 * half + j;
            const bool kin = k < kend;
            fa[j] = (kin && ai < M) ? A[ai * a_i + k * a_k] : static_cast<__bf16>(0.0f);
            fb[j] = (kin && bj < N) ? B[k * b_k + bj * b_j] : static_cast<__bf16>(0.0f);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = m0 + 8 * (e >> 2) + 4 * half + (e & 3);
        const int j = n0 + r;
        if (i >= M || j >= N) continue;
        if (gridDim.z > 1) {
            part[(static_cast<int64_t>(blockIdx.z) * M + i) * N + j] = acc[e];
            continue;
        }
        float v = acc[e];
        if (bias != nullptr) v += bias[j];
        const int64_t o = static_cast<int64_t>(i) * ldc + j;
        if (mode == 0) {
            Cf[o] = v;
        } else if (mode == 1) {
            Cb[o] = static_cast<__bf16>(fmaxf(v, 0.0f));
        } else {
            const float g = static_cast<float>(gate[o]);
            Cb[o] = static_cast<__bf16>(g > 0.0f ? v : 0.0f);
        }
    }
}

// The same product on TM x TM output tiles (TM = 128 or 64) staged through LDS, for operands of
// at least 64 rows and columns. Workgroup of 256 threads = 4 wavefronts in 2 x 2, each a
// TM/2 x TM/2 quarter (TM/64 x TM/64 MFMA tiles of 32 x 32); the K loop steps by 32, two
// 16-wide MFMA steps per slice. Both operands sit in LDS k-contiguous (A as [m][k], B transposed
// as [n][k]) with rows padded to 40 elements (80 bytes: eight lanes reading or writing 16 bytes
// each cover the 32 banks once), so every fragment read and every slice write is a 16-byte LDS
// access. The next slice is loaded from memory into registers while the current one is
// multiplied (two LDS buffers, one barrier per slice). An operand is loaded along k when it is
// k-contiguous (AKC / BKC: 16-byte loads of 8-element granules) and otherwise one element per k
// with the wavefront's lanes on consecutive rows (each load instruction reads one contiguous run
// of the row dimension). The loads are branch-free: addresses are clamped into the operand and
// out-of-range values replaced by zero, so that the loads of the next slice stay in flight
// while the current one is multiplied. Epilogue and split K as in k_gemm.
constexpr int kTK = 32, kTPad = 40;

__device__ __forceinline__ uint32_t bf16_bits(__bf16 x) {
    return __builtin_bit_cast(unsigned short, x);
}

// EPT bf16 values of one thread's share of a slice, packed two to a 32-bit word.
template <int EPT>
struct Slice {
    uint4 w[EPT / 8];
};

// One operand's slice (TM rows: m, or n for B; kTK k-values) into registers. x_r, x_k: the
// operand's strides along its rows and along k; r0: the tile's first row; k0: the slice's first
// k; rows and kend bound the operand. KC: k-contiguous (x_k == 1, x_r and kend multiples of 8,
// 16-byte aligned base); otherwise x_r == 1.
template <int TM, bool KC>
__device__ __forceinline__ void load_slice(const __bf16* __restrict__ X, int64_t x_r, int64_t x_k,
                                           int r0, int rows, int k0, int kend, int tid,
                                           Slice<TM / 8>& sl) {
    constexpr int EPT = TM / 8;           // elements per thread
    constexpr int TPR = kTK / EPT;        // threads per row (k-contiguous mapping)
    if constexpr (KC) {
        const int r = r0 + tid / TPR, k = k0 + EPT * (tid % TPR);
        const __bf16* row = X + static_cast<int64_t>(min(r, rows - 1)) * x_r;
#pragma unroll
        for (int g = 0; g < EPT / 8; ++g) {
            const int kg = k + 8 * g;
            const uint4 v = *reinterpret_cast<const uint4*>(row + min(kg, kend - 8));
            const bool ok = r < rows && kg < kend;
            sl.w[g].x = ok ? v.x : 0u;
            sl.w[g].y = ok ? v.y : 0u;
            sl.w[g].z = ok ? v.z : 0u;
            sl.w[g].w = ok ? v.w : 0u;
        }
    } else {
        // one row per thread, EPT consecutive k; consecutive lanes take consecutive rows
        const int r = r0 + tid % TM, k = k0 + EPT * (tid / TM);
        const __bf16* col = X + min(r, rows - 1);
        uint32_t h[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const uint32_t v = bf16_bits(col[static_cast<int64_t>(min(k + e, kend - 1)) * x_k]);
            h[e] = (r < rows && k + e < kend) ? v : 0u;
        }
#pragma unroll
        for (int q = 0; q < EPT / 8; ++q) {
            sl.w[q].x = h[8 * q + 0] | (h[8 * q + 1] << 16);
            sl.w[q].y = h[8 * q + 2] | (h[8 * q + 3] << 16);
            sl.w[q].z = h[8 * q + 4] | (h[8 * q + 5] << 16);
            sl.w[q].w = h[8 * q + 6] | (h[8 * q + 7] << 16);
        }
    }
}

// Writes a slice loaded by load_slice into the LDS tile T[row][k] (row stride kTPad).
template <int TM, bool KC>
__device__ __forceinline__ void store_slice(__bf16 (*T)[kTPad], int tid, const Slice<TM / 8>& sl) {
    constexpr int EPT = TM / 8, TPR = kTK / EPT;
    const int r = KC ? tid / TPR : tid % TM;
    const int k = KC ? EPT * (tid % TPR) : EPT * (tid / TM);
    uint4* d = reinterpret_cast<uint4*>(&T[r][k]);
#pragma unroll
    for (int q = 0; q < EPT / 8; ++q) d[q] = sl.w[q];
}

template <int TM, bool AKC, bool BKC>
__global__ void __launch_bounds__(256) k_gemm_tile(int M, int N, int K, const __bf16* __restrict__ A,
                                                   int64_t a_i, int64_t a_k,
                                                   const __bf16* __restrict__ B, int64_t b_k,
                                                   int64_t b_j, const float* __restrict__ bias,
                                                   int mode, const __bf16* __restrict__ gate,
                                                   float* __restrict__ Cf, __bf16* __restrict__ Cb,
                                                   int64_t ldc, int kps, float* __restrict__ part) {
    constexpr int NT = TM / 64;  // MFMA tiles per wavefront along each dimension
    __shared__ __attribute__((aligned(16))) __bf16 As[2][TM][kTPad];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][TM][kTPad];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
    const int kbeg = blockIdx.z * kps, kend = min(K, kbeg + kps);
    // B is addressed as [n][k]: its row stride is b_j, its k stride b_k
    Slice<TM / 8> sa, sb;
    load_slice<TM, AKC>(A, a_i, a_k, m0, M, kbeg, kend, tid, sa);
    load_slice<TM, BKC>(B, b_j, b_k, n0, N, kbeg, kend, tid, sb);
    store_slice<TM, AKC>(As[0], tid, sa);
    store_slice<TM, BKC>(Bs[0], tid, sb);
    __syncthreads();
    floatx16 acc[NT][NT] = {};
    const int r = lane & 31, half = lane >> 5;
    int buf = 0;
    for (int k0 = kbeg; k0 < kend; k0 += kTK) {
        // the last slice reloads itself (in range, unused): no branch around the loads
        const int kn = k0 + kTK < kend ? k0 + kTK : k0;
        load_slice<TM, AKC>(A, a_i, a_k, m0, M, kn, kend, tid, sa);
        load_slice<TM, BKC>(B, b_j, b_k, n0, N, kn, kend, tid, sb);
#pragma unroll
        for (int ks = 0; ks < kTK / 16; ++ks) {
            bf16x8 fa[NT], fb[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                fa[t] = *reinterpret_cast<const bf16x8*>(
                    &As[buf][wm * (TM / 2) + t * 32 + r][ks * 16 + 8 * half]);
                fb[t] = *reinterpret_cast<const bf16x8*>(
                    &Bs[buf][wn * (TM / 2) + t * 32 + r][ks * 16 + 8 * half]);
            }
#pragma unroll
            for (int tm = 0; tm < NT; ++tm)
#pragma unroll
                for (int tn = 0; tn < NT; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[tm], fb[tn],
                                                                          acc[tm][tn], 0, 0, 0);
        }
        // unconditional (the other buffer was last read before the previous barrier), so that
        // the loads above are issued before the multiplies rather than sunk into a branch
        store_slice<TM, AKC>(As[buf ^ 1], tid, sa);
        store_slice<TM, BKC>(Bs[buf ^ 1], tid, sb);
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int tm = 0; tm < NT; ++tm)
#pragma unroll
        for (int tn = 0; tn < NT; ++tn)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int i = m0 + wm * (TM / 2) + tm * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                const int j = n0 + wn * (TM / 2) + tn * 32 + r;
                if (i >= M || j >= N) continue;
                const float a = acc[tm][tn][e];
                if (gridDim.z > 1) {
                    part[(static_cast<int64_t>(blockIdx.z) * M + i) * N + j] = a;
                    continue;
                }
                float v = a;
                if (bias != nullptr) v += bias[j];
                const int64_t o = static_cast<int64_t>(i) * ldc + j;
                if (mode == 0) {
                    Cf[o] = v;
                } else if (mode == 1) {
                    Cb[o] = static_cast<__bf16>(fmaxf(v, 0.0f));
                } else {
                    const float g = static_cast<float>(gate[o]);
                    Cb[o] = static_cast<__bf16>(g > 0.0f ? v : 0.0f);
                }
            }
}

// Products with at most kNarrow output columns and a k-contiguous A (the action-slot layer):
// half a wavefront per row, lane l taking k = c + 8 l' .. + 7 of every 256-wide chunk c (l' =
// l % 32: one 16-byte load per lane, so the half-wavefront reads one contiguous 512-byte run of
// the row), each lane accumulating all N columns in FP32, then a butterfly over the 32 lanes in
// a fixed order. B is staged once per workgroup in LDS as FP32, ordered [chunk][e][lane][n] so
// that for each e the 32 lanes read consecutive N-float groups (no bank conflicts). Each
// wavefront takes kNarrowRows rows: the loads of all of them are issued before the first
// multiply. Epilogue as k_gemm (no split K). Needs ceil(K / 256) * 256 * N <= kNarrowLds, a row
// stride a multiple of 8 and a 16-byte aligned A.
constexpr int kNarrow = 8;
constexpr int kNarrowRows = 8;
constexpr int kNarrowLds = 8192;

__global__ void __launch_bounds__(256) k_gemm_narrow(int M, int N, int K,
                                                     const __bf16* __restrict__ A, int64_t a_i,
                                                     const __bf16* __restrict__ B, int64_t b_k,
                                                     int64_t b_j, const float* __restrict__ bias,
                                                     int mode, const __bf16* __restrict__ gate,
                                                     float* __restrict__ Cf,
                                                     __bf16* __restrict__ Cb, int64_t ldc) {
    extern __shared__ float Wl[];
    const int Kp = (K + 255) / 256 * 256;
    for (int t = threadIdx.x; t < Kp * N; t += blockDim.x) {
        const int n = t % N, q = t / N;
        const int l = q % 32, e = (q / 32) % 8, c = q / 256;
        const int k = 256 * c + 8 * l + e;
        Wl[t] = k < K ? static_cast<float>(B[static_cast<int64_t>(k) * b_k + n * b_j]) : 0.0f;
    }
    __syncthreads();
    constexpr int P = kNarrowRows / 2;  // row pairs per wavefront
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l = lane & 31, half = lane >> 5;
    const int base = (blockIdx.x * 4 + wave) * kNarrowRows + half;
    float acc[P][kNarrow];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int n = 0; n < kNarrow; ++n) acc[p][n] = 0.0f;
#pragma unroll 1
    for (int c = 0; c < K; c += 256) {
        const int k = c + 8 * l;
        uint4 xw[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int i = min(base + 2 * p, M - 1);
            const uint4 v = *reinterpret_cast<const uint4*>(A + static_cast<int64_t>(i) * a_i +
                                                            min(k, K - 8));
            const bool ok = k < K;  // K is a multiple of 8
            xw[p].x = ok ? v.x : 0u;
            xw[p].y = ok ? v.y : 0u;
            xw[p].z = ok ? v.z : 0u;
            xw[p].w = ok ? v.w : 0u;
        }
        const float* wl = Wl + (c / 256) * 256 * N;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float w[kNarrow];
#pragma unroll
            for (int n = 0; n < kNarrow; ++n) w[n] = n < N ? wl[(e * 32 + l) * N + n] : 0.0f;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const uint32_t wd = e / 2 == 0 ? xw[p].x : e / 2 == 1 ? xw[p].y
                                    : e / 2 == 2 ? xw[p].z : xw[p].w;
                const float x = static_cast<float>(__builtin_bit_cast(
                    __bf16, static_cast<unsigned short>(wd >> (16 * (e % 2)))));
#pragma unroll
                for (int n = 0; n < kNarrow; ++n) acc[p][n] = fmaf(x, w[n], acc[p][n]);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int n = 0; n < kNarrow; ++n)
            for (int off = 16; off > 0; off >>= 1) acc[p][n] += __shfl_xor(acc[p][n], off, 32);
    if (l != 0) return;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = base + 2 * p;
        if (i >= M) break;
#pragma unroll
        for (int n = 0; n < kNarrow; ++n) {
            if (n >= N) break;
            float v = acc[p][n];
            if (bias != nullptr) v += bias[n];
            const int64_t o = static_cast<int64_t>(i) * ldc + n;
            if (mode == 0) {
                Cf[o] = v;
            } else if (mode == 1) {
                Cb[o] = static_cast<__bf16>(fmaxf(v, 0.0f));
            } else {
                const float g = static_cast<float>(gate[o]);
                Cb[o] = static_cast<__bf16>(g > 0.0f ? v : 0.0f);
            }
        }
    }
}

// Column c of `splits` partials part[z][cols], by one wavefront: lane l adds partials l, l + 64, ...
// in order, then a butterfly over the 64 lanes in a fixed order.
__device__ __forceinline__ float sum_split_col(int splits, int cols, const float* __restrict__ part,
                                               int c, int lane) {
    float s = 0.0f;
    for (int z = lane; z < splits; z += 64) s += part[static_cast<int64_t>(z) * cols + c];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
}

__global__ void __launch_bounds__(256) k_sum_cols(int cols, int splits,
                                                  const float* __restrict__ part,
                                                  float* __restrict__ out) {
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (c >= cols) return;
    const float s = sum_split_col(splits, cols, part, c, lane);
    if (lane == 0) out[c] = s;
}

// Column j of rows [y rps, (y + 1) rps) of a BF16 [rows x cols] matrix, with four interleaved
// accumulators combined in a fixed order.
__device__ __forceinline__ float colsum_rows(int rows, int cols, int rps,
                                             const __bf16* __restrict__ G, int y, int j) {
    const int r0 = y * rps, r1 = min(rows, r0 + rps);
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int i = r0;
#pragma unroll 8
    for (; i + 4 <= r1; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] += static_cast<float>(G[static_cast<int64_t>(i + u) * cols + j]);
    }
    for (; i < r1; ++i) s[0] += static_cast<float>(G[static_cast<int64_t>(i) * cols + j]);
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// Column sums (bias gradients), split over rows: workgroup (x, y) takes 64 columns (one per lane,
// coalesced rows) and rows [y rps, (y + 1) rps), into part[y][cols].
__global__ void __launch_bounds__(64) k_colsum_part(int rows, int cols, int rps,
                                                    const __bf16* __restrict__ G,
                                                    float* __restrict__ part) {
    const int j = blockIdx.x * 64 + threadIdx.x;
    if (j >= cols) return;
    part[static_cast<int64_t>(blockIdx.y) * cols + j] = colsum_rows(rows, cols, rps, G, blockIdx.y, j);
}

// Adam's step constants and one parameter's step (FP32 master value, moments updated in place);
// the new value is returned.
struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ float adam_step(const AdamStep& a, float gi, float& w, float& m, float& v) {
    const float mi = a.b1 * m + (1.0f - a.b1) * gi;
    const float vi = a.b2 * v + (1.0f - a.b2) * gi * gi;
    m = mi;
    v = vi;
    const float wi = w - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    w = wi;
    return wi;
}

// Adam on FP32 master parameters; refreshes the BF16 copy used by the GEMMs.
__global__ void k_adam(int64_t n, float* __restrict__ w, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, __bf16* __restrict__ wb,
                       AdamStep a) {
    const int64_t i = gid();
    if (i >= n) return;
    const float wi = adam_step(a, g[i], w[i], m[i], v[i]);
    if (wb != nullptr) wb[i] = static_cast<__bf16>(wi);
}

// Where element (k, j) of a K x H weight matrix lies in its copy packed in MFMA fragment order:
// fragment (t, s) is the 64 lanes' 8 elements, lane l's W[16 s + 8 (l / 32) + 0 .. 7][32 t + l % 32].
__device__ __forceinline__ int64_t fragment_at(int K, int k, int j) {
    const int64_t f = static_cast<int64_t>(j / 32) * (K / 16) + k / 16;
    return (f * 64 + j % 32 + 32 * ((k % 16) / 8)) * 8 + k % 8;
}

// One row of k_softmax_xent from registers (slots past A: mask 0): the gradients into g, the
// row's share of the loss returned.
template <int NA>
__device__ __forceinline__ float softmax_xent_row(int B, const float* z, const float* tv,
                                                  const float* mk, float* g) {
    bool on[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) on[a] = mk[a] > 0.0f;
    float mx = -3.0e38f;
#pragma unroll
    for (int a = 0; a < NA; ++a)
        if (on[a]) mx = fmaxf(mx, z[a]);
    float se = 0.0f, tsum = 0.0f;
#pragma unroll
    for (int a = 0; a < NA; ++a)
        if (on[a]) {
            se += __expf(z[a] - mx);
            tsum += tv[a];
        }
    const float lse = mx + __logf(se);
    float l = 0.0f;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        g[a] = 0.0f;
        if (on[a]) {
            const float p = __expf(z[a] - lse);
            l -= tv[a] * (z[a] - lse);
            g[a] = (p * tsum - tv[a]) / static_cast<float>(B);
        }
    }
    return l / static_cast<float>(B);
}

// The three layers of a run of rows in one kernel, and for a training step the whole row-wise part
// of the backward pass with them. A workgroup of four wavefronts takes 32 RT rows: their input,
// then each hidden layer in turn, lies in one LDS tile; the wavefronts split a layer's columns
// (H = 64: columns and rows), so that the workgroup reads the weights once for all its rows.
// The products are formed transposed, D(j, i) = sum_k W(k, j) x(i, k): the weights are the
// MFMA's A operand, the rows its B operand, so that a lane ends with groups of four
// consecutive columns j of one row i: bias, ReLU and rounding write 8 bytes to LDS at once.
// Weights come from BF16 copies packed in fragment order (one coalesced kilobyte per fragment,
// L2-resident), several k-steps ahead of their use (the fewer rows a wavefront multiplies per
// step, the further ahead: kAhead(row tiles)).
// The last layer is split over the wavefronts by k: wavefront w takes the groups of 8
// consecutive k whose number is w mod 4, its weights read from LDS (one address for all lanes),
// and the partial sums meet in LDS.
// Every element is computed as by the per-layer kernels (k_gemm_tile, k_gemm, k_gemm_narrow), bit
// for bit: the same BF16 operands, FP32 accumulation over k in the same 16-wide MFMA steps, the
// same rounding of the hidden layers, the same tree over the last layer's sums (groups l and
// l ^ 16 first, then ^ 8, ^ 4, ^ 2, ^ 1).
// F: a multiple of 16 up to kFusedMaxF; H 64, 128 or 256; A <= kNarrow.
// Bound by the matrix units, fed from LDS and L2: 65,536 rows of 96 -> 256 -> 256 -> 4 take 15.7 to 16.2 us,
// 740 TFLOP/s, against 42 to 45 us with one wavefront per 32 rows, each reading all the weights.
constexpr int kFusedMaxF = 128;
constexpr int kAhead(int rpw) { return rpw >= 4 ? 4 : rpw == 2 ? 8 : 16; }

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// A layer's weights as a wavefront reads them: its TPC column tiles' fragments (packed at wp, tile
// c's from wp + c n 512, this lane's 8 elements) of n = KS k-steps (KS = 0: n at run time), the
// first PD steps loaded by load(). The multiply then adds, step by step, the products with the
// wavefront's RPW row tiles (rows x + 32 r LD .., this lane's row and k-half).
// Loads and stores complete in order, so load() comes before the stores of the layer before.
template <int TPC, int KS, int PD>
struct LayerWeights {
    const __bf16* wp;
    int n;
    bf16x8 w[PD][TPC];
    __device__ __forceinline__ bf16x8 at(int c, int s) const {
        return *reinterpret_cast<const bf16x8*>(wp + (static_cast<int64_t>(c) * n + s) * 512);
    }
    __device__ __forceinline__ void load(const __bf16* p, int steps) {
        wp = p;
        n = KS > 0 ? KS : steps;
#pragma unroll
        for (int s = 0; s < PD; ++s)
#pragma unroll
            for (int c = 0; c < TPC; ++c) w[s][c] = at(c, KS > 0 ? s : (s < n ? s : n - 1));
        // (the compiler would otherwise move the loads down to their use)
        __builtin_amdgcn_sched_barrier(0);
    }
    template <int RPW, bool FIRST = false>
    __device__ __forceinline__ void step(int s, const __bf16* x, int LD, const bf16x8 (&ws)[TPC],
                                         floatx16 (&acc)[RPW][TPC]) const {
        bf16x8 fx[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r)
            fx[r] = *reinterpret_cast<const bf16x8*>(x + 32 * r * LD + 16 * s);
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int c = 0; c < TPC; ++c)
                acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    ws[c], fx[r], FIRST ? floatx16{} : acc[r][c], 0, 0, 0);
    }
    template <int RPW>
    __device__ __forceinline__ void multiply(const __bf16* x, int LD, floatx16 (&acc)[RPW][TPC]) {
        if constexpr (KS > 0) {
            step<RPW, true>(0, x, LD, w[0], acc);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (s > 0) step<RPW>(s, x, LD, w[s % PD], acc);
                if (s + PD < KS) {
#pragma unroll
                    for (int c = 0; c < TPC; ++c) w[s % PD][c] = at(c, s + PD);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            static_assert(KS > 0 || PD == 1, "a run-time step count is loaded one step ahead");
#pragma unroll
            for (int r = 0; r < RPW; ++r)
#pragma unroll
                for (int c = 0; c < TPC; ++c) acc[r][c] = floatx16{};
#pragma unroll 1
            for (int s = 0; s < n; ++s) {
                bf16x8 cur[TPC];
#pragma unroll
                for (int c = 0; c < TPC; ++c) {
                    cur[c] = w[0][c];
                    w[0][c] = at(c, s + 1 < n ? s + 1 : s);  // (the last step's is unused)
                }
                step<RPW>(s, x, LD, cur, acc);
            }
        }
    }
};

// What a training step needs besides the forward pass's operands (TRAIN).
struct TrainOut {
    const float* target;   // M x A
    const float* mask;     // M x A
    const __bf16* W2B;     // W2 packed for dZ2 . W2^T (k: the layer's outputs)
    __bf16 *A1, *A2;       // M x H: the hidden layers
    __bf16 *dZ3, *dZ2, *dZ1;  // M x A, M x H, M x H
    float* loss;           // one partial per workgroup
};

// Copies the tile's rows m0 .. (those below M) of H columns to dst (M x H).
template <int H, int ROWS>
__device__ __forceinline__ void store_tile(const __bf16* T, int LD, __bf16* __restrict__ dst, int m0,
                                           int M) {
    constexpr int G = H / 8;
#pragma unroll 4
    for (int q = threadIdx.x; q < ROWS * G; q += 256) {
        const int row = q / G, c = 8 * (q % G);
        if (m0 + row < M)
            *reinterpret_cast<uint4*>(dst + static_cast<int64_t>(m0 + row) * H + c) =
                *reinterpret_cast<const uint4*>(T + row * LD + c);
    }
}

// NA: A rounded up to 4 or 8 (four columns' partial sums leave room for two workgroups of 128
// rows on a CU).
template <int H, int RT, int KS1, int NA, bool TRAIN>
__global__ void __launch_bounds__(256, TRAIN ? 1 : 2) k_mlp_rows(int M, int F, int A,
                                                     const __bf16* __restrict__ X,
                                                     const __bf16* __restrict__ W1P,
                                                     const float* __restrict__ b1,
                                                     const __bf16* __restrict__ W2P,
                                                     const float* __restrict__ b2,
                                                     const __bf16* __restrict__ W3T,
                                                     const float* __restrict__ b3,
                                                     float* __restrict__ Z, TrainOut tr) {
    constexpr int ROWS = 32 * RT;
    // row stride of the LDS tile (elements; input and hidden rows both fit): 16-byte aligned rows,
    // eight consecutive rows start on different banks
    constexpr int LD = (H > kFusedMaxF ? H : kFusedMaxF) + 8;
    constexpr int WC = H / 32 < 4 ? H / 32 : 4;  // wavefronts along the columns
    constexpr int WR = 4 / WC;                   // and along the rows
    constexpr int TPC = H / 32 / WC;             // column tiles of a wavefront
    constexpr int RPW = RT / WR;                 // row tiles of a wavefront
    static_assert(RPW >= 1, "too few rows for four wavefronts");
    constexpr int PD = kAhead(RPW) < H / 16 ? kAhead(RPW) : H / 16;
    constexpr int PD1 = KS1 == 0 ? 1 : KS1 < PD ? KS1 : PD;
    __shared__ __attribute__((aligned(16))) __bf16 T[ROWS * LD];
    // the hidden layers' biases, then (they are no longer needed) the last layer's partial sums
    constexpr int kPart = 4 * ROWS * NA > 2 * H ? 4 * ROWS * NA : 2 * H;
    __shared__ __attribute__((aligned(16))) float s_mem[kPart];
    __shared__ __attribute__((aligned(16))) float s_w3[H][NA];  // (columns past A: unused)
    float(*s_part)[ROWS][NA] = reinterpret_cast<float(*)[ROWS][NA]>(s_mem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, half = lane >> 5;
    const int m0 = blockIdx.x * ROWS;
    const int ct0 = (wave % WC) * TPC;         // the wavefront's first column tile
    const int row0 = (wave / WC) * RPW * 32;   // and first row
    LayerWeights<TPC, KS1, PD1> w1;
    LayerWeights<TPC, H / 16, PD> w2;
    w1.load(W1P + (static_cast<int64_t>(ct0) * (F / 16) * 64 + lane) * 8, F / 16);
    // stage the input rows (zero past M): 8-element granules, 16-byte loads
    {
        const int gpr = F / 8;  // granules per row
        for (int q = tid; q < ROWS * gpr; q += 256) {
            const int row = q / gpr, c = 8 * (q % gpr);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (m0 + row < M)
                v = *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(m0 + row) * F + c);
            *reinterpret_cast<uint4*>(&T[row * LD + c]) = v;
        }
        for (int q = tid; q < 2 * H; q += 256) s_mem[q] = q < H ? b1[q] : b2[q - H];
        for (int q = tid; q < H; q += 256)
#pragma unroll
            for (int n = 0; n < NA; ++n)
                s_w3[q][n] = static_cast<float>(W3T[static_cast<int64_t>(min(n, A - 1)) * H + q]);
    }
    float tgt[NA], msk[NA];  // TRAIN: thread tid's row
    if constexpr (TRAIN) {
#pragma unroll
        for (int n = 0; n < NA; ++n) {
            const bool in = tid < ROWS && m0 + tid < M && n < A;
            tgt[n] = in ? tr.target[static_cast<int64_t>(m0 + tid) * A + n] : 0.0f;
            msk[n] = in ? tr.mask[static_cast<int64_t>(m0 + tid) * A + n] : 0.0f;
        }
    }
    __syncthreads();
    const __bf16* xr = &T[(row0 + r) * LD + 8 * half];
    const int64_t wat = (static_cast<int64_t>(ct0) * (H / 16) * 64 + lane) * 8;
    floatx16 acc[RPW][TPC];
    uint32_t gate1[RPW][TPC], gate2[RPW][TPC];  // TRAIN: bit e: element e of the tile is > 0
    // bias, ReLU, rounding to BF16 into the tile (over the layer's input: every wavefront is past
    // its reads of it), and the ReLU's gate
    auto hidden = [&](const float* bias, uint32_t (&gate)[RPW][TPC]) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < TPC; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = (ct0 + c) * 32 + 8 * q + 4 * half;
                const float4 bv = *reinterpret_cast<const float4*>(bias + j);
                const float b[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
                for (int t = 0; t < RPW; ++t) {
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e] = static_cast<__bf16>(fmaxf(acc[t][c][4 * q + e] + b[e], 0.0f));
                    *reinterpret_cast<bf16x4*>(&T[(row0 + 32 * t + r) * LD + j]) = v;
                    if constexpr (TRAIN) {
                        if (q == 0) gate[t][c] = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            gate[t][c] |= (static_cast<float>(v[e]) > 0.0f ? 1u : 0u) << (4 * q + e);
                    }
                }
            }
        __syncthreads();
    };
    w1.template multiply<RPW>(xr, LD, acc);
    w2.load(W2P + wat, H / 16);
    hidden(s_mem, gate1);
    if constexpr (TRAIN) store_tile<H, ROWS>(T, LD, tr.A1, m0, M);
    w2.template multiply<RPW>(xr, LD, acc);
    hidden(s_mem + H, gate2);
    if constexpr (TRAIN) {
        w2.load(tr.W2B + wat, H / 16);  // the backward pass's
        store_tile<H, ROWS>(T, LD, tr.A2, m0, M);
    }
    // layer 3: groups g = wave + 4 j of 8 consecutive k; an FMA chain over a group's k, then the
    // tree over j (j ^ 4, ^ 2, ^ 1: the groups 16, 8 and 4 apart). A lane takes rows lane and
    // lane + 64 together: each group's weights (the same address in every lane) serve both.
    {
        constexpr int NR = ROWS > 64 ? ROWS / 64 : 1;
        constexpr int kOrder[8] = {0, 4, 2, 6, 1, 5, 3, 7};  // the tree's leaves, left to right
        float sum[NR][NA], half_[NR][NA], keep[NR][NA];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int j = kOrder[jj];
            float p[NR][NA];
#pragma unroll
            for (int u = 0; u < NR; ++u)
#pragma unroll
                for (int n = 0; n < NA; ++n) p[u][n] = 0.0f;
            if (32 * j < H) {
                bf16x8 xv[NR];
#pragma unroll
                for (int u = 0; u < NR; ++u)
                    xv[u] = *reinterpret_cast<const bf16x8*>(
                        &T[(ROWS >= 64 ? lane + 64 * u : r) * LD + 8 * (wave + 4 * j)]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float* wk = s_w3[8 * (wave + 4 * j) + e];
#pragma unroll
                    for (int u = 0; u < NR; ++u)
#pragma unroll
                        for (int n = 0; n < NA; ++n)
                            p[u][n] = fmaf(static_cast<float>(xv[u][e]), wk[n], p[u][n]);
                }
            }
#pragma unroll
            for (int u = 0; u < NR; ++u)
#pragma unroll
                for (int n = 0; n < NA; ++n) {
                    if (jj % 2 == 0) half_[u][n] = p[u][n];
                    else half_[u][n] += p[u][n];
                    if (jj == 1 || jj == 5) keep[u][n] = half_[u][n];
                    if (jj == 3) sum[u][n] = keep[u][n] + half_[u][n];
                    if (jj == 7) sum[u][n] = sum[u][n] + (keep[u][n] + half_[u][n]);
                }
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int row = ROWS >= 64 ? lane + 64 * u : r;
            if (ROWS >= 64 || lane < 32)
#pragma unroll
                for (int n = 0; n < NA; ++n) s_part[wave][row][n] = sum[u][n];
        }
    }
    __syncthreads();
    if constexpr (!TRAIN) {
        for (int t = tid; t < ROWS * A; t += 256) {
            const int row = t / A, n = t % A;
            if (m0 + row < M)
                Z[static_cast<int64_t>(m0 + row) * A + n] =
                    ((s_part[0][row][n] + s_part[2][row][n]) +
                     (s_part[1][row][n] + s_part[3][row][n])) + b3[n];
        }
    } else {
        __shared__ __attribute__((aligned(16))) __bf16 s_dz3[ROWS][kNarrow];
        __shared__ float s_loss[4];
        // masked softmax cross-entropy, one thread per row (as k_softmax_xent)
        float l = 0.0f;
        if (tid < ROWS) {
            bf16x8 g8 = {};
            if (m0 + tid < M) {
                const int64_t b = m0 + tid;
                float z[NA], g[NA];
#pragma unroll
                for (int n = 0; n < NA; ++n)
                    z[n] = n < A ? ((s_part[0][tid][n] + s_part[2][tid][n]) +
                                    (s_part[1][tid][n] + s_part[3][tid][n])) + b3[n]
                                 : 0.0f;
                l = softmax_xent_row<NA>(M, z, tgt, msk, g);
#pragma unroll
                for (int n = 0; n < NA; ++n)
                    if (n < A) {
                        g8[n] = static_cast<__bf16>(g[n]);
                        tr.dZ3[b * A + n] = g8[n];
                    }
            }
            *reinterpret_cast<bf16x8*>(&s_dz3[tid][0]) = g8;
        }
        for (int off = 32; off > 0; off >>= 1) l += __shfl_down(l, off, 64);
        if (lane == 0) s_loss[wave] = l;
        __syncthreads();
        if (tid == 0)
            tr.loss[blockIdx.x] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
        // the gated products with a layer's weights, rounded into the tile
        auto gated = [&](const uint32_t (&gate)[RPW][TPC]) {
#pragma unroll
            for (int c = 0; c < TPC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int t = 0; t < RPW; ++t) {
                        bf16x4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e] = static_cast<__bf16>(
                                (gate[t][c] >> (4 * q + e)) & 1 ? acc[t][c][4 * q + e] : 0.0f);
                        *reinterpret_cast<bf16x4*>(
                            &T[(row0 + 32 * t + r) * LD + (ct0 + c) * 32 + 8 * q + 4 * half]) = v;
                    }
            __syncthreads();
        };
        // dZ2 = (dZ3 . W3^T) gated: one 16-wide k-step, zero past A
        {
            bf16x8 fx[RPW];
#pragma unroll
            for (int t = 0; t < RPW; ++t) {
                fx[t] = bf16x8{};
                if (half == 0)
                    fx[t] = *reinterpret_cast<const bf16x8*>(&s_dz3[row0 + 32 * t + r][0]);
            }
#pragma unroll
            for (int c = 0; c < TPC; ++c) {
                bf16x8 fw = {};
#pragma unroll
                for (int n = 0; n < NA; ++n)
                    if (half == 0 && n < A)
                        fw[n] = static_cast<__bf16>(s_w3[(ct0 + c) * 32 + r][n]);  // exact
#pragma unroll
                for (int t = 0; t < RPW; ++t)
                    acc[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw, fx[t], floatx16{}, 0, 0, 0);
            }
        }
        gated(gate2);
        store_tile<H, ROWS>(T, LD, tr.dZ2, m0, M);
        // dZ1 = (dZ2 . W2^T) gated
        w2.template multiply<RPW>(xr, LD, acc);
        __syncthreads();  // every wavefront is past its reads of dZ2
        gated(gate1);
        store_tile<H, ROWS>(T, LD, tr.dZ1, m0, M);
    }
}

// The weight and bias gradients of a training step in one launch, as partials over runs of rows
// (k_train_update adds them): jobs in the order of TrainJobs. A weight job is one 64 x 64 tile of
// L^T R over the rows [z kps, (z + 1) kps): both operands are read along their rows (16 bytes: 8
// columns of one row) and stored to LDS transposed, two rows' values to a 32-bit word, so that
// the fragments read 8 consecutive k as k_gemm_tile's do; the k-steps and the splits are those
// of launch_gemm, so every partial equals its. A bias job sums 4 x rps rows of 64 columns, one
// wavefront per rps rows, as k_colsum_part. Bound by its loads and the transposition through LDS: 14.5 us
// for 4,096 rows (a step was 27 launches and 178 us; its three take 40 us, 52 with the caller's wait).
struct TrainJobs {
    int B, F, H, A;
    const __bf16 *X, *A1, *A2, *dZ1, *dZ2, *dZ3;
    float *pw1, *pw2, *pw3;       // weight partials [split][M][N]
    float *pb1, *pb2, *pb3;       // bias partials [split][N]
    int splits1, kps1;            // of W1
    int splits, kps;              // of W2
    int splits3, kps3;            // of W3
    int csplits, rps;             // of the column sums
    int n1, n2, n3, nb1, nb3;     // workgroups of each kind (b2 as b1)
};

// One 64 x 64 tile of L^T R: L is B x ldl, R is B x ldr, tile columns ml0 of L and nr0 of R (ml, nr
// columns in all), rows kbeg .. kend. W8: R's rows are read 16 bytes at a time, else by element.
template <bool W8>
__device__ __forceinline__ void grad_tile(const __bf16* __restrict__ L, int ldl, int ml, int ml0,
                                          const __bf16* __restrict__ R, int ldr, int nr, int nr0,
                                          int kbeg, int kend, float* __restrict__ out,
                                          __bf16 (*As)[64][kTPad], __bf16 (*Bs)[64][kTPad]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, half = lane >> 5;
    // threads 0-127 load L's slice, 128-255 R's: granule g (8 columns) of rows 2 p and 2 p + 1
    const bool left = tid < 128;
    const int t = tid & 127, g = t / 16, p = t % 16;
    uint4 v[2];
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + 2 * p + u;
            v[u] = make_uint4(0u, 0u, 0u, 0u);
            if (k >= kend) continue;
            if (left) {
                if (ml0 + 8 * g < ml)
                    v[u] = *reinterpret_cast<const uint4*>(L + static_cast<int64_t>(k) * ldl + ml0 +
                                                           8 * g);
            } else if constexpr (W8) {
                v[u] = *reinterpret_cast<const uint4*>(R + static_cast<int64_t>(k) * ldr + nr0 + 8 * g);
            } else if (g == 0) {  // at most 8 columns
                uint32_t h[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    h[j] = j < nr ? bf16_bits(R[static_cast<int64_t>(k) * ldr + j]) : 0u;
                v[u] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                  h[6] | (h[7] << 16));
            }
        }
    };
    auto store = [&](int buf) {
        __bf16(*S)[kTPad] = left ? As[buf] : Bs[buf];
        const uint32_t a[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
        const uint32_t b[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t lo = (a[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
            const uint32_t hi = (b[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
            *reinterpret_cast<uint32_t*>(&S[8 * g + j][2 * p]) = lo | (hi << 16);
        }
    };
    load(kbeg);
    store(0);
    __syncthreads();
    floatx16 acc = {};
    int buf = 0;
    for (int k0 = kbeg; k0 < kend; k0 += kTK) {
        load(k0 + kTK);  // zeros past kend
#pragma unroll
        for (int ks = 0; ks < kTK / 16; ++ks) {
            const bf16x8 fa =
                *reinterpret_cast<const bf16x8*>(&As[buf][wm * 32 + r][ks * 16 + 8 * half]);
            const bf16x8 fb =
                *reinterpret_cast<const bf16x8*>(&Bs[buf][wn * 32 + r][ks * 16 + 8 * half]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc, 0, 0, 0);
        }
        store(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = ml0 + wm * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
        const int j = nr0 + wn * 32 + r;
        if (i < ml && j < nr) out[static_cast<int64_t>(i) * nr + j] = acc[e];
    }
}

__global__ void __launch_bounds__(256) k_train_grads(TrainJobs q) {
    __shared__ __attribute__((aligned(16))) __bf16 As[2][64][kTPad];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][64][kTPad];
    int b = blockIdx.x;
    const int tn = q.H / 64, tm1 = (q.F + 63) / 64;
    if (b < q.n2) {  // dW2 = A1^T dZ2
        const int z = b / (tn * tn), t = b % (tn * tn);
        grad_tile<true>(q.A1, q.H, q.H, 64 * (t / tn), q.dZ2, q.H, q.H, 64 * (t % tn), z * q.kps,
                        min(q.B, (z + 1) * q.kps), q.pw2 + static_cast<int64_t>(z) * q.H * q.H, As, Bs);
        return;
    }
    b -= q.n2;
    if (b < q.n1) {  // dW1 = X^T dZ1
        const int z = b / (tm1 * tn), t = b % (tm1 * tn);
        grad_tile<true>(q.X, q.F, q.F, 64 * (t / tn), q.dZ1, q.H, q.H, 64 * (t % tn), z * q.kps1,
                        min(q.B, (z + 1) * q.kps1), q.pw1 + static_cast<int64_t>(z) * q.F * q.H, As, Bs);
        return;
    }
    b -= q.n1;
    if (b < q.n3) {  // dW3 = A2^T dZ3
        const int z = b / tn, t = b % tn;
        grad_tile<false>(q.A2, q.H, q.H, 64 * t, q.dZ3, q.A, q.A, 0, z * q.kps3,
                         min(q.B, (z + 1) * q.kps3), q.pw3 + static_cast<int64_t>(z) * q.H * q.A, As,
                         Bs);
        return;
    }
    b -= q.n3;
    // column sums: four splits per workgroup
    const __bf16* G = q.dZ1;
    float* part = q.pb1;
    int cols = q.H;
    if (b >= 2 * q.nb1) {
        b -= 2 * q.nb1;
        G = q.dZ3;
        part = q.pb3;
        cols = q.A;
    } else if (b >= q.nb1) {
        b -= q.nb1;
        G = q.dZ2;
        part = q.pb2;
    }
    const int cg = (cols + 63) / 64;
    const int y = 4 * (b / cg) + static_cast<int>(threadIdx.x >> 6);
    const int j = 64 * (b % cg) + static_cast<int>(threadIdx.x & 63);
    if (y >= q.csplits || j >= cols) return;
    part[static_cast<int64_t>(y) * cols + j] = colsum_rows(q.B, cols, q.rps, G, y, j);
}

// Adds a step's partials (as k_sum_splits and k_sum_cols), applies Adam (as k_adam) and writes
// every BF16 copy of the new weights: workgroups [0, nw) one thread per weight, then one
// wavefront per bias; the last workgroup adds the loss partials in order. Bound by the partials' reads:
// 6 us at 96 -> 256 -> 256 -> 4.
__global__ void __launch_bounds__(256) k_train_update(TrainJobs q, int nw, int nl,
                                                      const float* __restrict__ lpart,
                                                      float* __restrict__ loss, float* __restrict__ w,
                                                      float* __restrict__ g, float* __restrict__ m,
                                                      float* __restrict__ v, __bf16* __restrict__ wb,
                                                      __bf16* __restrict__ wbT,
                                                      __bf16* __restrict__ wbP, AdamStep ad) {
    const int F = q.F, H = q.H, A = q.A;
    const int64_t o1 = static_cast<int64_t>(F) * H, o2 = o1 + H, o3 = o2 + static_cast<int64_t>(H) * H,
                  o4 = o3 + H, o5 = o4 + static_cast<int64_t>(H) * A;
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ float s_l[4];
        float l = 0.0f;
        for (int t = threadIdx.x; t < nl; t += 256) l += lpart[t];
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        if ((threadIdx.x & 63) == 0) s_l[threadIdx.x >> 6] = l;
        __syncthreads();
        if (threadIdx.x == 0) *loss = (s_l[0] + s_l[1]) + (s_l[2] + s_l[3]);
        return;
    }
    if (static_cast<int>(blockIdx.x) >= nw) {
        // bias c of [b1 | b2 | b3]
        const int c = (blockIdx.x - nw) * 4 + static_cast<int>(threadIdx.x >> 6);
        if (c >= 2 * H + A) return;
        const int lane = threadIdx.x & 63;
        const float* part = c < H ? q.pb1 : c < 2 * H ? q.pb2 : q.pb3;
        const int cols = c < 2 * H ? H : A, j = c < H ? c : c < 2 * H ? c - H : c - 2 * H;
        const int64_t i = c < H ? o1 + j : c < 2 * H ? o3 + j : o5 + j;
        const float s = sum_split_col(q.csplits, cols, part, j, lane);
        if (lane == 0) {
            g[i] = s;
            wb[i] = static_cast<__bf16>(adam_step(ad, s, w[i], m[i], v[i]));
        }
        return;
    }
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t n1 = static_cast<int64_t>(F) * H, n2 = static_cast<int64_t>(H) * H,
                  n3 = static_cast<int64_t>(H) * A;
    if (e >= n1 + n2 + n3) return;
    const int which = e < n1 ? 1 : e < n1 + n2 ? 2 : 3;
    const int64_t at = which == 1 ? e : which == 2 ? e - n1 : e - n1 - n2;
    const float* part = which == 1 ? q.pw1 : which == 2 ? q.pw2 : q.pw3;
    const int64_t size = which == 1 ? n1 : which == 2 ? n2 : n3;
    const int splits = which == 1 ? q.splits1 : which == 2 ? q.splits : q.splits3;
    float s = 0.0f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) s += part[z * size + at];
    const int64_t i = which == 1 ? at : which == 2 ? o2 + at : o4 + at;
    g[i] = s;
    const __bf16 x = static_cast<__bf16>(adam_step(ad, s, w[i], m[i], v[i]));
    wb[i] = x;
    const int cols = which == 3 ? A : H, k = static_cast<int>(at / cols), j = static_cast<int>(at % cols);
    if (which == 1) {
        wbT[static_cast<int64_t>(j) * F + k] = x;
        wbP[fragment_at(F, k, j)] = x;
    } else if (which == 2) {
        wbT[n1 + static_cast<int64_t>(j) * H + k] = x;
        wbP[n1 + fragment_at(H, k, j)] = x;
        wbP[n1 + n2 + fragment_at(H, j, k)] = x;  // the backward pass reads W2^T
    } else {
        wbT[n1 + n2 + static_cast<int64_t>(j) * H + k] = x;
    }
}

// Packs the K x H weight matrix W (given transposed, WT[j][k]) in MFMA fragment order.
__global__ void k_pack_fragments(int K, int H, const __bf16* __restrict__ WT,
                                 __bf16* __restrict__ dst) {
    const int64_t i = gid();
    if (i >= static_cast<int64_t>(K) * H) return;
    const int k = static_cast<int>(i % K), j = static_cast<int>(i / K);
    dst[fragment_at(K, k, j)] = WT[i];
}

// dst[c][r] = src[r][c] for a rows x cols BF16 matrix (the transposed weight copies).
__global__ void k_transpose_bf16(int rows, int cols, const __bf16* __restrict__ src,
                                 __bf16* __restrict__ dst) {
    const int64_t t = gid();
    if (t >= static_cast<int64_t>(rows) * cols) return;
    const int64_t r = t / cols, c = t % cols;
    dst[c * rows + r] = src[t];
}

// Masked softmax cross-entropy per row: loss += -(1/B) sum_a mask t log p, and
// dZ[b, a] = mask (p tsum - t) / B in BF16.
__global__ void k_softmax_xent(int B, int A, const float* __restrict__ Z,
                               const float* __restrict__ target, const float* __restrict__ mask,
                               __bf16* __restrict__ dZ, float* __restrict__ loss) {
    const int64_t b = gid();
    float l = 0.0f;
    if (b < B) {
        const float* z = Z + b * A;
        const float* t = target + b * A;
        const float* mk = mask + b * A;
        float mx = -3.0e38f;
        for (int a = 0; a < A; ++a)
            if (mk[a] > 0.0f) mx = fmaxf(mx, z[a]);
        float se = 0.0f, tsum = 0.0f;
        for (int a = 0; a < A; ++a)
            if (mk[a] > 0.0f) {
                se += __expf(z[a] - mx);
                tsum += t[a];
            }
        const float lse = mx + __logf(se);
        for (int a = 0; a < A; ++a) {
            float g = 0.0f;
            if (mk[a] > 0.0f) {
                const float p = __expf(z[a] - lse);
                l -= t[a] * (z[a] - lse);
                g = (p * tsum - t[a]) / static_cast<float>(B);
            }
            dZ[b * A + a] = static_cast<__bf16>(g);
        }
        l /= static_cast<float>(B);
    }
    // wave reduction then one atomic per wave
    for (int off = 32; off > 0; off >>= 1) l += __shfl_down(l, off, 64);
    if ((threadIdx.x & 63) == 0 && loss != nullptr) atomicAdd(loss, l);
}

// Sums split partials part[z][M][N] over z in order into C (row stride ldc), one thread per
// element.
__global__ void k_sum_splits(int M, int N, int splits, const float* __restrict__ part,
                             float* __restrict__ C, int64_t ldc) {
    const int64_t t = gid();
    if (t >= static_cast<int64_t>(M) * N) return;
    const int64_t i = t / N, j = t % N;
    float s = 0.0f;
    for (int z = 0; z < splits; ++z) s += part[(static_cast<int64_t>(z) * M + i) * N + j];
    C[i * ldc + j] = s;
}

__global__ void k_to_bf16(int64_t n, const float* __restrict__ src, __bf16* __restrict__ dst) {
    const int64_t i = gid();
    if (i < n) dst[i] = static_cast<__bf16>(src[i]);
}

// Poker-subgame features. Descriptor fields (int16): see mlp.hpp. A workgroup builds kFeatRows
// rows in LDS (zeroed, then the few non-zero entries written, four threads per row) and stores
// them with consecutive threads on consecutive 16-byte granules (VEC: F a multiple of 8, X and
// desc 16-byte aligned; else element by element). Bound by its stores: 200,001 rows of 96 in 15 us (2.5
// TB/s; 262 us with a thread per row writing element by element).
constexpr int kFeatRows = 64;
constexpr int kFeatLd = 88;  // kFeatures rounded up to granules of 8

template <bool VEC>
__global__ void __launch_bounds__(256) k_features(int64_t n, int F, const int16_t* __restrict__ desc,
                                                  const float* __restrict__ beliefs,
                                                  __bf16* __restrict__ X) {
    __shared__ __attribute__((aligned(16))) int16_t s_desc[kFeatRows * kDescFields];
    __shared__ __attribute__((aligned(16))) __bf16 s_x[kFeatRows][kFeatLd];
    const int tid = threadIdx.x;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kFeatRows;
    const int rows = static_cast<int>(min<int64_t>(kFeatRows, n - row0));
    if constexpr (VEC) {
        if (tid < 2 * rows)
            reinterpret_cast<uint4*>(s_desc)[tid] =
                reinterpret_cast<const uint4*>(desc + row0 * kDescFields)[tid];
    } else {
        for (int t = tid; t < rows * kDescFields; t += 256) s_desc[t] = desc[row0 * kDescFields + t];
    }
    for (int t = tid; t < kFeatRows * kFeatLd / 8; t += 256)
        reinterpret_cast<uint4*>(&s_x[0][0])[t] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const int row = tid & (kFeatRows - 1), part = tid / kFeatRows;
    if (row < rows) {
        const int16_t* d = s_desc + row * kDescFields;
        __bf16* f = s_x[row];
        const __bf16 one = static_cast<__bf16>(1.0f);
        const int player = d[kDPlayer], own = d[kDOwn];
        if (part == 0) {
            const int rnd = d[kDRound], raises = d[kDRaises], last = d[kDLast];
            if (own >= 0 && own < 13) f[own] = one;                   // own rank 0..12
            f[13 + (player == 1 ? 0 : 1)] = one;                      // player
            if (rnd >= 0 && rnd < 3) f[15 + rnd] = one;               // absolute round
            for (int i = 0; i < 3; ++i) {                             // board multi-hot
                const int c = d[kDBoard0 + i];
                if (c >= 0 && c < 13) f[18 + c] = one;
            }
            if (raises >= 0 && raises < 4) f[31 + raises] = one;      // raises this round
            if (last >= 0 && last < 5) f[35 + last] = one;            // last action
            for (int i = 0; i < 4; ++i)                               // legal slots
                if ((d[kDMask] >> i) & 1) f[44 + i] = one;
            f[80] = one;                                              // bias input
        } else if (part == 1) {
            const float stack = static_cast<float>(d[kDStack]);
            const float cme = static_cast<float>(d[kDCMe]), cop = static_cast<float>(d[kDCOpp]);
            f[40] = static_cast<__bf16>(cme / stack);                 // commitments and pot
            f[41] = static_cast<__bf16>(cop / stack);
            f[42] = static_cast<__bf16>((cme + cop) / stack);
            f[43] = static_cast<__bf16>((cop - cme) / fmaxf(cme + cop, 1.0f));
            f[48] = static_cast<__bf16>(static_cast<float>(d[kDDepth]) / 16.0f);
            f[49] = static_cast<__bf16>(static_cast<float>(d[kDCap]) / 3.0f);
            f[50] = static_cast<__bf16>(logf(stack) / logf(1000.0f));
            f[51] = static_cast<__bf16>(static_cast<float>(d[kDRanks]) / 13.0f);
        } else {
            // root beliefs: the opponent's range over ranks and my win chance, then my own range
            const int64_t seat = part == 2 ? 2 - player : player - 1;
            const float* b = beliefs + (static_cast<int64_t>(d[kDGame]) * 2 + seat) * 13;
            float bv[13];
#pragma unroll
            for (int i = 0; i < 13; ++i) bv[i] = b[i];
            float below = 0.0f, above = 0.0f;
#pragma unroll
            for (int i = 0; i < 13; ++i) {
                f[(part == 2 ? 52 : 65) + i] = static_cast<__bf16>(bv[i]);
                if (i < own) below += bv[i];
                if (i > own) above += bv[i];
            }
            if (part == 2) {
                f[78] = static_cast<__bf16>(below);
                f[79] = static_cast<__bf16>(above);
            }
        }
    }
    __syncthreads();
    if constexpr (VEC) {
        const int gpr = F / 8;
        for (int q = tid; q < rows * gpr; q += 256) {
            const int rw = q / gpr, c = 8 * (q % gpr);
            const uint4 v = c < kFeatLd ? *reinterpret_cast<const uint4*>(&s_x[rw][c])
                                        : make_uint4(0u, 0u, 0u, 0u);
            *reinterpret_cast<uint4*>(X + (row0 + rw) * F + c) = v;
        }
    } else {
        for (int64_t q = tid; q < static_cast<int64_t>(rows) * F; q += 256) {
            const int rw = static_cast<int>(q / F), c = static_cast<int>(q % F);
            X[(row0 + rw) * F + c] = c < kFeatLd ? s_x[rw][c] : static_cast<__bf16>(0.0f);
        }
    }
}

// Masked softmax of logits over the legal slots, scattered to pair order: action a of infoset
// h is the a-th legal slot; probs[q_off[h] + a].
__global__ void k_probs_to_pairs(int64_t n, int A, const float* __restrict__ Z,
                                 const int16_t* __restrict__ desc, const int64_t* __restrict__ q_off,
                                 float* __restrict__ probs) {
    const int64_t h = gid();
    if (h >= n) return;
    const int mask = desc[h * kDescFields + kDMask];
    const float* z = Z + h * A;
    float mx = -3.0e38f;
    for (int s = 0; s < A; ++s)
        if ((mask >> s) & 1) mx = fmaxf(mx, z[s]);
    float se = 0.0f;
    for (int s = 0; s < A; ++s)
        if ((mask >> s) & 1) se += __expf(z[s] - mx);
    int a = 0;
    for (int s = 0; s < A; ++s)
        if ((mask >> s) & 1) probs[q_off[h] + a++] = __expf(z[s] - mx) / se;
}

// R0(h, a) = w * m(h) * p(h, a) with m(h) = sum_a max(R(h, a), 0) of the current state,
// S = 0, then regret matching. Pairs in the solver's order; p read through q_input.
__global__ void k_warm_start(int64_t Hp, const int32_t* __restrict__ q_offset,
                             const int32_t* __restrict__ q_input, const float* __restrict__ probs,
                             float w, float* __restrict__ R, float* __restrict__ S,
                             float* __restrict__ sigma) {
    const int64_t h = gid();
    if (h >= Hp) return;
    const int32_t o = q_offset[h], k = q_offset[h + 1] - o;
    float m = 0.0f;
    for (int32_t a = 0; a < k; ++a) m += fmaxf(R[o + a], 0.0f);
    float pos = 0.0f;
    for (int32_t a = 0; a < k; ++a) {
        const float r = w * m * probs[q_input[o + a]];
        R[o + a] = r;
        S[o + a] = 0.0f;
        pos += fmaxf(r, 0.0f);
    }
    for (int32_t a = 0; a < k; ++a)
        sigma[o + a] = pos > 0.0f ? fmaxf(R[o + a], 0.0f) / pos : 1.0f / static_cast<float>(k);
}

}  // namespace

namespace {

// Splits of a K-long reduction in steps of `step` and the k-values of each (the last may have
// fewer); one split unless `split` and K is long.
void split_k(int K, int step, bool split, int& splits, int& kps) {
    splits = split && K >= 2 * kSplitK ? std::min(kMaxSplits, K / kSplitK) : 1;
    kps = ((K + splits - 1) / splits + step - 1) / step * step;
    splits = (K + kps - 1) / kps;
}

// Splits of a column sum over `rows` rows and the rows of each.
void split_rows(int rows, int& splits, int& rps) {
    // 32 rows per split, at most kColsumMaxSplits partials
    splits = std::max(1, std::min(kColsumMaxSplits, rows / 32));
    rps = (rows + splits - 1) / splits;
}

}  // namespace

void launch_gemm(int M, int N, int K, const void* A, int64_t a_i, int64_t a_k, const void* B,
                 int64_t b_k, int64_t b_j, const float* bias, int mode, const void* gate, float* Cf,
                 void* Cb, int64_t ldc, hipStream_t st, float* part) {
    const auto* a = static_cast<const __bf16*>(A);
    const auto* b = static_cast<const __bf16*>(B);
    const auto* g = static_cast<const __bf16*>(gate);
    auto* cb = static_cast<__bf16*>(Cb);
    // a few output columns from a k-contiguous A: half a wavefront per row
    const int Kp = (K + 255) / 256 * 256;
    if (N <= kNarrow && a_k == 1 && a_i % 8 == 0 && K % 8 == 0 && Kp * N <= kNarrowLds &&
        (reinterpret_cast<uintptr_t>(a) % 16) == 0 &&
        (part == nullptr || mode != 0 || bias != nullptr || K < 2 * kSplitK)) {
        const int rows_per_wg = 4 * kNarrowRows;
        hipLaunchKernelGGL(k_gemm_narrow, dim3((M + rows_per_wg - 1) / rows_per_wg), dim3(256),
                           static_cast<size_t>(Kp) * N * sizeof(float), st, M, N, K, a, a_i, b, b_k,
                           b_j, bias, mode, g, Cf, cb, ldc);
        return;
    }
    // LDS tiles where both output dimensions fill them and each operand is k-contiguous (rows
    // of 8-element granules, 16-byte aligned) or row-contiguous; the other skinny products stay
    // on one wavefront per 32 x 32 tile
    auto aligned16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) % 16) == 0; };
    const bool akc = a_k == 1 && a_i % 8 == 0 && K % 8 == 0 && aligned16(a);
    const bool bkc = b_k == 1 && b_j % 8 == 0 && K % 8 == 0 && aligned16(b);
    const bool tiled = M >= 64 && N >= 64 && K >= kTK && (akc || a_i == 1) && (bkc || b_j == 1);
    const int step = tiled ? kTK : 16;
    // split K only for FP32 outputs without bias (weight gradients) when K is long
    int splits = 1, kps = 0;
    split_k(K, step, part != nullptr && mode == 0 && bias == nullptr, splits, kps);
    if (tiled) {
        // 128 x 128 tiles when they alone give the chip a few workgroups per CU, else 64 x 64
        const int64_t big = int64_t{(N + 127) / 128} * ((M + 127) / 128) * splits;
        const int tm = big >= 512 ? 128 : 64;
        dim3 grid((N + tm - 1) / tm, (M + tm - 1) / tm, splits);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, M, N, K, a, a_i, a_k, b, b_k, b_j,
                               bias, mode, g, Cf, cb, ldc, kps, part);
        };
        if (tm == 128) {
            if (akc && bkc) go(k_gemm_tile<128, true, true>);
            else if (akc) go(k_gemm_tile<128, true, false>);
            else if (bkc) go(k_gemm_tile<128, false, true>);
            else go(k_gemm_tile<128, false, false>);
        } else {
            if (akc && bkc) go(k_gemm_tile<64, true, true>);
            else if (akc) go(k_gemm_tile<64, true, false>);
            else if (bkc) go(k_gemm_tile<64, false, true>);
            else go(k_gemm_tile<64, false, false>);
        }
    } else {
        dim3 grid((N + 31) / 32, (M + 31) / 32, splits);
        hipLaunchKernelGGL(k_gemm, grid, dim3(64), 0, st, M, N, K, a, a_i, a_k, b, b_k, b_j, bias,
                           mode, g, Cf, cb, ldc, kps, part);
    }
    if (splits > 1)
        hipLaunchKernelGGL(k_sum_splits, dim3(blocks_for(int64_t{M} * N, 256)), dim3(256), 0, st, M,
                           N, splits, part, Cf, ldc);
}

void launch_softmax_xent(int B, int A, const float* Z, const float* target, const float* mask,
                         void* dZ, float* loss, hipStream_t st) {
    hipLaunchKernelGGL(k_softmax_xent, dim3(blocks_for(B, 256)), dim3(256), 0, st, B, A, Z, target,
                       mask, static_cast<__bf16*>(dZ), loss);
}

bool mlp_fused_shape(int F, int H, int A, const void* X) {
    return F % 16 == 0 && F <= kFusedMaxF && A <= kNarrow && (H == 64 || H == 128 || H == 256) &&
           (reinterpret_cast<uintptr_t>(X) % 16) == 0;
}

namespace {

// Rows per workgroup: 128 once that gives every CU one workgroup (and two of them fit a CU: a
// forward pass, A at most 4), else 64, else 32 (H = 64: at least 64), so that fewer rows spread over more CUs.
template <int H, int NA, bool TRAIN, class Go>
void with_rows(int M, int F, Go go) {
    auto rows = [&](auto rt) {
        constexpr int RT = decltype(rt)::value;
        const dim3 grid((M + 32 * RT - 1) / (32 * RT));
        if (F == 96) go(k_mlp_rows<H, RT, 6, NA, TRAIN>, grid);
        else go(k_mlp_rows<H, RT, 0, NA, TRAIN>, grid);
    };
    // Rows per workgroup: more of them share a read of the weights, fewer fill more CUs. The lines lie
    // where there is a workgroup for each of the 256 CUs (96 -> 256 -> 256 -> 4, forward with 32, 64,
    // 128 rows: 16,384 rows all within the 9.4 us that a call costs the host, 24,576 rows 12.5, 9.9,
    // 11.2 us, 32,768 rows 15.1, 11.2, 11.5 us, 65,536 rows 25.7, 18.0, 15.7 us; a training step of
    // 4,096 rows 52 us with 32, 55 us with 64). Training keeps 64 at most: its backward pass's
    // accumulators leave no registers for 128.
    if (NA == 4 && !TRAIN && M >= 128 * 256) rows(std::integral_constant<int, NA == 4 && !TRAIN ? 4 : 2>{});
    else if (H == 64 || M >= 64 * 256) rows(std::integral_constant<int, 2>{});
    else rows(std::integral_constant<int, H == 64 ? 2 : 1>{});
}

template <int NA, bool TRAIN, class Go>
void with_hidden(int M, int F, int H, Go go) {
    if (H == 64) with_rows<64, NA, TRAIN>(M, F, go);
    else if (H == 128) with_rows<128, NA, TRAIN>(M, F, go);
    else with_rows<256, NA, TRAIN>(M, F, go);
}

template <bool TRAIN, class Go>
void with_shape(int M, int F, int H, int A, Go go) {
    if (A <= 4) with_hidden<4, TRAIN>(M, F, H, go);
    else with_hidden<8, TRAIN>(M, F, H, go);
}

}  // namespace

bool launch_mlp_forward(int M, int F, int H, int A, const void* X, const void* W1P, const float* b1,
                        const void* W2P, const float* b2, const void* W3T, const float* b3,
                        float* Z, hipStream_t st) {
    if (!mlp_fused_shape(F, H, A, X)) return false;
    with_shape<false>(M, F, H, A, [&](auto kernel, dim3 grid) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, M, F, A, static_cast<const __bf16*>(X),
                           static_cast<const __bf16*>(W1P), b1, static_cast<const __bf16*>(W2P), b2,
                           static_cast<const __bf16*>(W3T), b3, Z, TrainOut{});
    });
    return true;
}

int64_t mlp_train_part_floats(int F, int H, int A) {
    const int64_t f = F, h = H, a = A;
    return kMaxSplits * (f * h + h * h + h * a) + kColsumMaxSplits * (2 * h + a) + kMaxLossParts;
}

bool launch_mlp_train(int B, int F, int H, int A, const TrainArgs& t, hipStream_t st) {
    // (a step of 64 rows, 96 -> 256 -> 256 -> 4: 37 us with the caller's wait against 108 us layer by
    // layer; of 4,096 rows 52 against 153 us)
    if (!mlp_fused_shape(F, H, A, t.x)) return false;
    float* p = t.part;
    TrainJobs q{};
    q.B = B; q.F = F; q.H = H; q.A = A;
    q.X = static_cast<const __bf16*>(t.x);
    q.A1 = t.A1; q.A2 = t.A2; q.dZ1 = t.dZ1; q.dZ2 = t.dZ2; q.dZ3 = t.dZ3;
    // (the steps that launch_gemm takes for these shapes)
    split_k(B, F >= 64 ? kTK : 16, true, q.splits1, q.kps1);
    split_k(B, kTK, true, q.splits, q.kps);
    split_k(B, 16, true, q.splits3, q.kps3);
    split_rows(B, q.csplits, q.rps);
    auto take = [&](int64_t n) {
        float* r = p;
        p += n;
        return r;
    };
    q.pw1 = take(int64_t{kMaxSplits} * F * H);
    q.pw2 = take(int64_t{kMaxSplits} * H * H);
    q.pw3 = take(int64_t{kMaxSplits} * H * A);
    q.pb1 = take(int64_t{kColsumMaxSplits} * H);
    q.pb2 = take(int64_t{kColsumMaxSplits} * H);
    q.pb3 = take(int64_t{kColsumMaxSplits} * A);
    float* lpart = take(kMaxLossParts);
    const int tn = H / 64, tm1 = (F + 63) / 64, cgs = (q.csplits + 3) / 4;
    q.n2 = tn * tn * q.splits;
    q.n1 = tm1 * tn * q.splits1;
    q.n3 = tn * q.splits3;
    q.nb1 = cgs * tn;
    q.nb3 = cgs;
    int rows_wg = 0;
    bool fits = true;
    with_shape<true>(B, F, H, A, [&](auto kernel, dim3 grid) {
        rows_wg = static_cast<int>(grid.x);
        fits = rows_wg <= kMaxLossParts;
        if (!fits) return;
        const TrainOut out{t.target, t.mask, t.W2B, t.A1, t.A2, t.dZ3, t.dZ2, t.dZ1, lpart};
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, B, F, A, q.X, t.W1P, t.b1, t.W2P, t.b2,
                           t.W3T, t.b3, static_cast<float*>(nullptr), out);
    });
    if (!fits) return false;
    hipLaunchKernelGGL(k_train_grads, dim3(q.n1 + q.n2 + q.n3 + 2 * q.nb1 + q.nb3), dim3(256), 0, st,
                       q);
    const int nw = static_cast<int>(blocks_for(int64_t{F} * H + int64_t{H} * H + int64_t{H} * A, 256));
    hipLaunchKernelGGL(k_train_update, dim3(nw + (2 * H + A + 3) / 4 + 1), dim3(256), 0, st, q, nw,
                       rows_wg, lpart, t.loss, t.w, t.g, t.m, t.v, t.wb, t.wbT, t.wbP,
                       AdamStep{t.lr, t.beta1, t.beta2, t.eps, t.c1, t.c2});
    return true;
}

void launch_pack_fragments(int K, int H, const void* WT, void* dst, hipStream_t st) {
    const int64_t n = int64_t{K} * H;
    if (n > 0 && K % 16 == 0 && H % 32 == 0)
        hipLaunchKernelGGL(k_pack_fragments, dim3(blocks_for(n, 256)), dim3(256), 0, st, K, H,
                           static_cast<const __bf16*>(WT), static_cast<__bf16*>(dst));
}

void launch_transpose_bf16(int rows, int cols, const void* src, void* dst, hipStream_t st) {
    const int64_t n = int64_t{rows} * cols;
    if (n > 0)
        hipLaunchKernelGGL(k_transpose_bf16, dim3(blocks_for(n, 256)), dim3(256), 0, st, rows, cols,
                           static_cast<const __bf16*>(src), static_cast<__bf16*>(dst));
}

void launch_colsum(int rows, int cols, const void* G, float* out, hipStream_t st, float* part) {
    int splits = 1, rps = 0;
    split_rows(rows, splits, rps);
    hipLaunchKernelGGL(k_colsum_part, dim3((cols + 63) / 64, splits), dim3(64), 0, st, rows, cols,
                       rps, static_cast<const __bf16*>(G), part);
    hipLaunchKernelGGL(k_sum_cols, dim3((cols + 3) / 4), dim3(256), 0, st, cols, splits, part, out);
}

void launch_adam(int64_t n, float* w, const float* g, float* m, float* v, void* wb, float lr,
                 float b1, float b2, float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, w, g, m, v,
                       static_cast<__bf16*>(wb), AdamStep{lr, b1, b2, eps, c1, c2});
}

void launch_to_bf16(int64_t n, const float* src, void* dst, hipStream_t st) {
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, src,
                       static_cast<__bf16*>(dst));
}

void launch_features(int64_t n, int F, const int16_t* desc, const float* beliefs, void* X,
                     hipStream_t st) {
    const dim3 grid(blocks_for(n, kFeatRows));
    auto* x = static_cast<__bf16*>(X);
    const bool vec = F % 8 == 0 && (reinterpret_cast<uintptr_t>(X) % 16) == 0 &&
                     (reinterpret_cast<uintptr_t>(desc) % 16) == 0;
    if (vec) hipLaunchKernelGGL(k_features<true>, grid, dim3(256), 0, st, n, F, desc, beliefs, x);
    else hipLaunchKernelGGL(k_features<false>, grid, dim3(256), 0, st, n, F, desc, beliefs, x);
}

void launch_probs_to_pairs(int64_t n, int A, const float* Z, const int16_t* desc,
                           const int64_t* q_off, float* probs, hipStream_t st) {
    hipLaunchKernelGGL(k_probs_to_pairs, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, A, Z, desc,
                       q_off, probs);
}

void launch_warm_start(int64_t Hp, const int32_t* q_offset, const int32_t* q_input,
                       const float* probs, float w, float* R, float* S, float* sigma, hipStream_t st) {
    hipLaunchKernelGGL(k_warm_start, dim3(blocks_for(Hp, 256)), dim3(256), 0, st, Hp, q_offset,
                       q_input, probs, w, R, S, sigma);
}

}  // namespace cfr
