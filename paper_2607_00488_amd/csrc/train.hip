// Training step of the surrogate network on gfx950 (train.h), for hidden layers
// of 256 outputs.  The products, the order of their sums and every rounding are
// those of the layer-by-layer GEMMs with K-split slabs that networks of other
// widths run; what is fused is the passes between them.
//
// Matrix operands come straight from memory (L2) into the registers of
// v_mfma_f32_32x32x16_bf16: a fragment is 32 rows x 16 reduction indices, lane
// (li, lh) holding indices 8 lh .. 8 lh + 7 of row li, and every producer writes
// its matrices in that order (train.h), so that a fragment is one 1 KB run.
#include "train.h"

#include <cmath>
#include <utility>

namespace nr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int H = kFusedHidden;
constexpr int kKp = H + 8;         // padded input width of layers 1 to 3
constexpr int kRows = 32;          // points per work-group of the chained layers
constexpr int kLda = H + 24;       // LDS row (bf16): 16-byte aligned, zeros to 272
constexpr int kThreads = 256;

__device__ inline bf16x8 frag(const bf16* p) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    return *reinterpret_cast<const bf16x8*>(&v);
}
__device__ inline bf16x8 zero8() {
    const uint4 v = make_uint4(0u, 0u, 0u, 0u);
    return *reinterpret_cast<const bf16x8*>(&v);
}
__device__ inline f32x16 zero16() {
    f32x16 v;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = 0.f;
    return v;
}
// row of register r in a 32 x 32 block
__device__ inline int blk_row(int r, int lh) { return (r >> 2) * 8 + lh * 4 + (r & 3); }

__device__ inline float silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.f + __expf(-z));
}
__device__ inline float dsilu(float v, float z) {
    const float sg = 1.f / (1.f + __expf(-z));
    return v * sg * (1.f + z * (1.f - sg));
}

// Fragment `step` of row block `rb` of a matrix in fragment order.
__device__ inline bf16x8 frag_of(const bf16* x, int rb, int step, int steps) {
    return frag(x + ((size_t)rb * steps + step) * 512 + (threadIdx.x & 63) * 8);
}

// Columns [0, n_col) of the points in LDS as rows of a matrix whose reduction
// runs over the points: eight of them per 16-byte store.
__device__ inline void store_t(const bf16 (*As)[kLda], int n_col, bf16* dst, int steps, int m0, int B) {
    for (int c = threadIdx.x; c < n_col * (kRows / 8); c += kThreads) {
        const int col = c % n_col, p = c / n_col * 8;
        if (m0 + p >= B) continue;
        bf16 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = As[p + e][col];
        *reinterpret_cast<uint4*>(dst + frag_at(col, m0 + p, steps)) = *reinterpret_cast<const uint4*>(v);
    }
}

// --------------------------------------------------------------- forward
// Input map and the three hidden layers of 32 points per work-group, the
// activations in LDS: wave w forms outputs 64 w .. 64 w + 63 (points as the row
// operand).  Every layer's weights are in flight before the first layer starts
// (one wave per SIMD holds them all): the chain was bound by their latency, layer
// by layer.
template <int NKS>
__device__ __forceinline__ void load_weights(const bf16* __restrict__ W, bf16x8 w[NKS][2]) {
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int y = 0; y < 2; ++y) w[ks][y] = frag_of(W, wave * 2 + y, ks, NKS);
}

template <int NKS>
__device__ __forceinline__ void fwd_layer(bf16 (*As)[kLda], const bf16x8 w[NKS][2], float* z, int m0,
                                          int B) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    f32x16 acc[2] = {zero16(), zero16()};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&As[li][ks * 16 + lh * 8]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w[ks][0], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w[ks][1], acc[1], 0, 0, 0);
    }
    __syncthreads();  // every wave has read this layer's input
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int p = blk_row(r, lh), o = wave * 64 + y * 32 + li;
            As[p][o] = (bf16)silu(acc[y][r]);
            if (m0 + p < B) z[(size_t)(m0 + p) * H + o] = acc[y][r];
        }
    __syncthreads();
}

__global__ __launch_bounds__(kThreads, 1) void k_train_fwd(TrainFwd a) {
    __shared__ __attribute__((aligned(16))) bf16 As[kRows][kLda];
    const int tid = threadIdx.x, m0 = blockIdx.x * kRows;
    bf16x8 w0[2][2], w1[17][2], w2[17][2];
    load_weights<2>(a.wf[0], w0);
    load_weights<17>(a.wf[1], w1);
    load_weights<17>(a.wf[2], w2);
    __builtin_amdgcn_sched_barrier(0);
    for (int q = tid; q < kRows * (kLda / 8); q += kThreads)
        *reinterpret_cast<uint4*>(&As[q / (kLda / 8)][q % (kLda / 8) * 8]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    if (tid < kRows) {
        const int p = min(m0 + tid, a.B - 1);
        const double* th = a.theta + (a.idx ? a.idx[p] : (long long)p) * kNTheta;
        for (int i = 0; i < kNTheta; ++i)
            As[tid][i] = bf16_of(2.0 * (th[i] - a.lo[i]) / (a.hi[i] - a.lo[i]) - 1.0);
        As[tid][kNTheta] = (bf16)1.f;
        As[tid][H] = (bf16)1.f;  // the bias input of the later layers
    }
    __syncthreads();
    store_t(As, 32, a.b.xt, a.b.steps, m0, a.B);
    fwd_layer<2>(As, w0, a.b.z[0], m0, a.B);
    store_t(As, H, a.b.ht[0], a.b.steps, m0, a.B);
    fwd_layer<17>(As, w1, a.b.z[1], m0, a.B);
    store_t(As, H, a.b.ht[1], a.b.steps, m0, a.B);
    fwd_layer<17>(As, w2, a.b.z[2], m0, a.B);
    store_t(As, H, a.b.ht[2], a.b.steps, m0, a.B);
    // 272 columns: the bias column and the zeros after it are in the tile
    constexpr int KS = (kKp + 15) / 16;
    for (int c = tid; c < kRows * KS * 2; c += kThreads) {
        const int r = c % kRows, k = c / kRows * 8;
        *reinterpret_cast<uint4*>(a.b.h2 + frag_at(m0 + r, k, KS)) =
            *reinterpret_cast<const uint4*>(&As[r][k]);
    }
}

// ---------------------------------------------------- output layer, loss
// 128 points x 128 outputs per work-group, waves 2 x 2; the targets of a wave's
// block are loaded before its products.  d(loss)/dY leaves twice, as rows of
// points and as rows of outputs, each through LDS in whole 256-byte runs.  Bound
// by those streams (targets 4 B, dY 2 x 2 B per output).
constexpr int kTS = 128 + 8;  // LDS row of a staged tile

__global__ __launch_bounds__(kThreads, 2) void k_train_mse(TrainMse a) {
    __shared__ __attribute__((aligned(16))) bf16 T1[128][kTS];  // [point][output]
    __shared__ __attribute__((aligned(16))) bf16 T2[128][kTS];  // [output][point]
    __shared__ double red[4];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;
    const int m0 = blockIdx.y * 128, n0 = blockIdx.x * 128;
    const int n_last = a.N - 1, m_last = a.B - 1 - m0;  // last valid row of the tile
    __shared__ long long rows[128];  // first target of every point
    if (tid < 128) {
        const int p = m0 + min(tid, m_last);
        rows[tid] = (a.idx ? a.idx[p] : (long long)p) * a.N;
    }
    __syncthreads();
    float t[2][2][16];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float* tb = a.t + rows[wm * 64 + x * 32 + blk_row(r, lh)];
#pragma unroll
            for (int y = 0; y < 2; ++y)
                t[x][y][r] = tb[min(n0 + wn * 64 + y * 32 + li, n_last)];
        }
    f32x16 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = zero16();
    constexpr int NKS = (kKp + 15) / 16, D = 3;
    bf16x8 fa[D][2], fb[D][2];
    // row blocks past the last point or output: any of them, never stored
    const int rb_a = m0 / 32 + wm * 2, rb_b = n0 / 32 + wn * 2;
    const int last_a = (a.B - 1) / 32, last_b = n_last / 32;
    auto load = [&](int ks, bf16x8 u[2], bf16x8 v[2]) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            u[x] = frag_of(a.b.h2, min(rb_a + x, last_a), ks, NKS);
            v[x] = frag_of(a.wf, min(rb_b + x, last_b), ks, NKS);
        }
    };
#pragma unroll
    for (int ks = 0; ks < D; ++ks) load(ks, fa[ks], fb[ks]);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        bf16x8 u[2], v[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            u[x] = fa[ks % D][x];  // zeros past the columns in both
            v[x] = fb[ks % D][x];
        }
        if (ks + D < NKS) load(ks + D, fa[ks % D], fb[ks % D]);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
                acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[x], v[y], acc[x][y], 0, 0, 0);
    }
    double lsum = 0.0;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int nl = wn * 64 + y * 32 + li;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16 d[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 4 * q + e, ml = wm * 64 + x * 32 + blk_row(r, lh);
                    const float rr = acc[x][y][r] - t[x][y][r];
                    d[e] = (bf16)(a.scale * 2.f * rr);
                    if (ml <= m_last && n0 + nl <= n_last) lsum += (double)rr * rr;
                    T1[ml][nl] = d[e];
                }
                *reinterpret_cast<uint2*>(&T2[nl][wm * 64 + x * 32 + 8 * q + 4 * lh]) =
                    *reinterpret_cast<const uint2*>(d);
            }
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
    if (lane == 0) red[wave] = lsum;
    __syncthreads();
    if (tid == 0)
        a.tile_loss[blockIdx.y * gridDim.x + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    const int n_steps = frag_steps(a.N);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = tid + i * kThreads, row = c & 127, k = (c >> 7) * 8;
        if (row <= m_last && n0 + k < a.N)
            *reinterpret_cast<uint4*>(a.b.dy + frag_at(m0 + row, n0 + k, n_steps)) =
                *reinterpret_cast<const uint4*>(&T1[row][k]);
        if (n0 + row < a.N && k <= m_last)
            *reinterpret_cast<uint4*>(a.b.dyt + frag_at(n0 + row, m0 + k, a.b.steps)) =
                *reinterpret_cast<const uint4*>(&T2[row][k]);
    }
}

// ------------------------------------------------------- split products
// One tile of C[m][n] = sum_k A[m][k] B[n][k], both in fragment order, the sum
// taken in chunks: round by round every G waves form one chunk of the whole
// tile (BM x BN blocks of 32 x 32 each), then the threads add the round's chunks in order to their elements
// (element tid + i T of the tile, rows of 32 BN).  No partial sums leave the
// work-group, where the K-split GEMM wrote and read back a slab per chunk.
template <int BM, int BN, int NW, int G>
struct SplitTile {
    static constexpr int D = 3;  // stages in flight; deeper ones spill
    static constexpr int T = NW * G * 64, TM = 32 * BM * G, TN = 32 * BN, EPT = TM * TN / T;
    static_assert(TM * TN % T == 0, "whole elements per thread");

    // ahead(): loads for after the sum, issued behind the last products
    template <class Ahead>
    static __device__ __forceinline__ void run(const bf16* __restrict__ A, const bf16* __restrict__ B,
                                               int M, int N, int K, int steps, TrainSplit sp, int m0,
                                               int n0, float (*part)[TM][TN], float v[EPT], Ahead ahead) {
        const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
        // uniform: addresses in scalar registers
        const int w0 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = w0 / G, g = w0 % G;
        const bf16 *ap[BM], *bp[BN];  // row blocks past the last: any, never stored
#pragma unroll
        for (int x = 0; x < BM; ++x)
            ap[x] = A + (size_t)min(m0 / 32 + g * BM + x, (M - 1) / 32) * steps * 512;
#pragma unroll
        for (int y = 0; y < BN; ++y)
            bp[y] = B + (size_t)min(n0 / 32 + y, (N - 1) / 32) * steps * 512;
#pragma unroll
        for (int i = 0; i < EPT; ++i) v[i] = 0.f;
        for (int q0 = 0; q0 < sp.n_split; q0 += NW) {
            const int q = q0 + wave;
            if (q < sp.n_split) {
                const int kb = q * sp.chunk, ke = min(K, kb + sp.chunk);
                f32x16 acc[BM][BN];
#pragma unroll
                for (int x = 0; x < BM; ++x)
#pragma unroll
                    for (int y = 0; y < BN; ++y) acc[x][y] = zero16();
                struct Stage {  // 16 reduction indices
                    bf16x8 a[BM], b[BN];
                };
                auto load = [&](int k, Stage& s) {
#pragma unroll
                    for (int x = 0; x < BM; ++x) s.a[x] = frag(ap[x] + k * 32 + lane * 8);
#pragma unroll
                    for (int y = 0; y < BN; ++y) s.b[y] = frag(bp[y] + k * 32 + lane * 8);
                };
                auto compute = [&](const Stage& s) {
#pragma unroll
                    for (int x = 0; x < BM; ++x)
#pragma unroll
                        for (int y = 0; y < BN; ++y)
                            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                s.a[x], s.b[y], acc[x][y], 0, 0, 0);
                };
                const int nst = (ke - kb) / 16;
                if (nst > 0) {  // D - 1 stages ahead; the loads past the end repeat the last
                    Stage st[D];
                    auto at = [&](int i) { return kb + min(i, nst - 1) * 16; };
#pragma unroll
                    for (int d = 0; d < D - 1; ++d) load(at(d), st[d]);
                    int i = 0;
                    for (; i + D <= nst; i += D)
#pragma unroll
                        for (int d = 0; d < D; ++d) {
                            load(at(i + d + D - 1), st[(d + D - 1) % D]);
                            compute(st[d]);
                        }
#pragma unroll
                    for (int d = 0; d < D - 1; ++d)
                        if (i + d < nst) compute(st[d]);
                }
                // the last indices, a multiple of eight: 16 at a time, zeros past
                // the end
                for (int k = kb + nst * 16; k < ke; k += 16) {
                    const bool ok = k + lh * 8 < ke;
#pragma unroll
                    for (int x = 0; x < BM; ++x) {
                        const bf16x8 f = frag(ap[x] + k * 32 + lane * 8), u = ok ? f : zero8();
#pragma unroll
                        for (int y = 0; y < BN; ++y) {
                            const bf16x8 w = frag(bp[y] + k * 32 + lane * 8);
                            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                u, ok ? w : zero8(), acc[x][y], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int x = 0; x < BM; ++x)
#pragma unroll
                    for (int y = 0; y < BN; ++y)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            part[wave][32 * (g * BM + x) + blk_row(r, lh)][32 * y + li] = acc[x][y][r];
            }
            if (q0 + NW >= sp.n_split) ahead();
            __syncthreads();
            const int nq = min(NW, sp.n_split - q0);
            for (int w = 0; w < nq; ++w) {
                const float* p = &part[w][0][0];
#pragma unroll
                for (int i = 0; i < EPT; ++i) v[i] += p[tid + i * T];
            }
            __syncthreads();
        }
    }
};

// dZ_2 = (dY W_3) SiLU'(Z_2): 32 points x 64 units per work-group, sixteen waves,
// a chunk of 256 outputs each (a batch of 2048 fills the 256 CUs once; 64 x 64
// tiles of eight waves filled half of them, in two rounds: 17.5 -> 11.8 us at
// N = 4096).  Work-groups of the same points run on one XCD (eight apart), whose
// L2 then serves dY to all four of them.
typedef SplitTile<1, 2, 16, 1> DhTile;

__global__ __launch_bounds__(DhTile::T) void k_train_dh(TrainDh a) {
    __shared__ float part[16][DhTile::TM][DhTile::TN];
    float v[DhTile::EPT];
    const int u = blockIdx.x >> 3, n0 = (u & 3) * 64, m0 = ((u >> 2) * 8 + (blockIdx.x & 7)) * DhTile::TM;
    if (m0 >= a.B) return;
    float z[DhTile::EPT];
    DhTile::run(a.b.dy, a.wt, a.B, H, a.N, frag_steps(a.N), a.sp, m0, n0, part, v, [&] {
#pragma unroll
        for (int i = 0; i < DhTile::EPT; ++i) {
            const int e = threadIdx.x + i * DhTile::T;
            z[i] = a.b.z[2][(size_t)min(m0 + e / DhTile::TN, a.B - 1) * H + n0 + e % DhTile::TN];
        }
    });
#pragma unroll
    for (int i = 0; i < DhTile::EPT; ++i) {
        const int e = threadIdx.x + i * DhTile::T, m = m0 + e / DhTile::TN, n = n0 + e % DhTile::TN;
        if (m >= a.B) continue;
        a.b.dz2[frag_at(m, n, H / 16)] = (bf16)dsilu(v[i], z[i]);
    }
}

// dZ_1 and dZ_0 of 32 points per work-group, as the forward chain; the chunks of
// a layer's reduction are summed one after the other in registers.
__device__ __forceinline__ void load_z(const float* z, int m0, int B, f32x16 zv[2]) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            zv[y][r] = z[(size_t)min(m0 + blk_row(r, lh), B - 1) * H + wave * 64 + y * 32 + li];
}

__device__ __forceinline__ void bwd_layer(bf16 (*As)[kLda], const bf16x8 w[H / 16][2], TrainSplit sp,
                                          const f32x16 zv[2]) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    constexpr int NKS = H / 16;
    f32x16 acc[2] = {zero16(), zero16()}, v[2] = {zero16(), zero16()};
    const int cks = sp.chunk / 16;
    int left = cks;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&As[li][ks * 16 + lh * 8]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w[ks][0], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w[ks][1], acc[1], 0, 0, 0);
        if (--left == 0 || ks == NKS - 1) {
            left = cks;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                v[y] += acc[y];
                acc[y] = zero16();
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            As[blk_row(r, lh)][wave * 64 + y * 32 + li] = (bf16)dsilu(v[y][r], zv[y][r]);
    __syncthreads();
}

__global__ __launch_bounds__(kThreads, 1) void k_train_hidden(TrainHidden a) {
    __shared__ __attribute__((aligned(16))) bf16 As[kRows][kLda];
    const int tid = threadIdx.x, m0 = blockIdx.x * kRows;
    bf16x8 w1[H / 16][2], w0[H / 16][2];
    f32x16 z1[2], z0[2];
    load_weights<H / 16>(a.wt[0], w1);
    load_z(a.b.z[1], m0, a.B, z1);
    load_weights<H / 16>(a.wt[1], w0);
    load_z(a.b.z[0], m0, a.B, z0);
    __builtin_amdgcn_sched_barrier(0);
    for (int c = tid; c < kRows * (H / 8); c += kThreads) {
        const int r = c % kRows, k = c / kRows * 8;  // rows past the last point: never stored
        *reinterpret_cast<uint4*>(&As[r][k]) =
            *reinterpret_cast<const uint4*>(a.b.dz2 + frag_at(m0 + r, k, H / 16));
    }
    __syncthreads();
    store_t(As, H, a.b.dzt[2], a.b.steps, m0, a.B);
    bwd_layer(As, w1, a.sp, z1);
    store_t(As, H, a.b.dzt[1], a.b.steps, m0, a.B);
    bwd_layer(As, w0, a.sp, z0);
    store_t(As, H, a.b.dzt[0], a.b.steps, m0, a.B);
}

// Every layer's weight gradient with its Adam step: 64 x 96 tiles of G, two waves
// per chunk; a matrix's tiles of the same outputs run on one XCD.  The parameters
// and moments are asked for behind the last products.  Six waves of whole tiles,
// with the moments loaded after the sum: 30.8 -> 26.8 us at N = 4096, 2048 points.
// The thread that ends up with an element of G updates its parameter, its
// moments and its BF16 copies (those in fragment order through LDS).
// Tiles of 64 x 32, eight pairs of waves, where few tiles of a long reduction leave
// the chip idle (the rule: launch_train_w).
typedef SplitTile<1, 3, 6, 2> WTile;
typedef SplitTile<1, 1, 8, 2> WTileSmall;

template <class Tile, int NW>
__global__ __launch_bounds__(Tile::T) void k_train_w(TrainW a) {
    __shared__ __attribute__((aligned(16))) union {
        float part[NW][Tile::TM][Tile::TN];
        struct {
            bf16 f[Tile::TM][Tile::TN + 8], t[Tile::TN][Tile::TM + 8];
        } w;
    } sh;
    int li = 3;
    while (li > 0 && (int)blockIdx.x < a.l[li].first) --li;
    const TrainLayer& L = a.l[li];
    const int nt = (L.N + Tile::TN - 1) / Tile::TN, t = (int)blockIdx.x - L.first, u = t >> 3;
    const int m0 = (u / nt * 8 + (t & 7)) * Tile::TM, n0 = u % nt * Tile::TN;
    if (m0 >= L.M) return;
    float v[Tile::EPT], ow[Tile::EPT], om[Tile::EPT], ov[Tile::EPT];
    Tile::run(L.A, L.Bm, L.M, L.N, a.B, a.steps, L.sp, m0, n0, sh.part, v, [&] {
#pragma unroll
        for (int i = 0; i < Tile::EPT; ++i) {
            const int e = threadIdx.x + i * Tile::T;
            const size_t o = (size_t)min(m0 + e / Tile::TN, L.M - 1) * L.N +
                             min(n0 + e % Tile::TN, L.N - 1);
            ow[i] = L.w[o];
            om[i] = L.m[o];
            ov[i] = L.v[o];
        }
    });
#pragma unroll
    for (int i = 0; i < Tile::EPT; ++i) {
        const int e = threadIdx.x + i * Tile::T, ml = e / Tile::TN, nl = e % Tile::TN;
        if (m0 + ml >= L.M || n0 + nl >= L.N) continue;
        const size_t o = (size_t)(m0 + ml) * L.N + n0 + nl;
        const float g = v[i];
        // fused as the layer-by-layer step's Adam kernel is
        const float m = fmaf(1.f - a.b1, g, a.b1 * om[i]);
        const float s = fmaf(g, (1.f - a.b2) * g, a.b2 * ov[i]);
        const float w = ow[i] - a.lr * (m / a.bc1) / (sqrtf(s / a.bc2) + a.eps);
        L.g[o] = g;
        L.m[o] = m;
        L.v[o] = s;
        L.w[o] = w;
        L.w16[o] = (bf16)w;
        sh.w.f[ml][nl] = sh.w.t[nl][ml] = (bf16)w;
    }
    __syncthreads();
    const int sm = frag_steps(L.M), sn = frag_steps(L.N);
    // M and N are multiples of eight: whole 16-byte pieces
    for (int c = threadIdx.x; c < Tile::TN * (Tile::TM / 8); c += Tile::T) {
        const int nl = c % Tile::TN, ml = c / Tile::TN * 8;
        if (n0 + nl < L.N && m0 + ml < L.M)
            *reinterpret_cast<uint4*>(L.wt + frag_at(n0 + nl, m0 + ml, sm)) =
                *reinterpret_cast<const uint4*>(&sh.w.t[nl][ml]);
    }
    for (int c = threadIdx.x; c < Tile::TM * (Tile::TN / 8); c += Tile::T) {
        const int ml = c % Tile::TM, nl = c / Tile::TM * 8;
        if (n0 + nl < L.N && m0 + ml < L.M)
            *reinterpret_cast<uint4*>(L.wf + frag_at(m0 + ml, n0 + nl, sn)) =
                *reinterpret_cast<const uint4*>(&sh.w.f[ml][nl]);
    }
}

__global__ void k_train_ones(bf16* ht, int steps) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= steps * 16) return;
    for (int r = 0; r < 8; ++r) ht[frag_at(H + r, p, steps)] = (bf16)(r == 0 ? 1.f : 0.f);
}

// One element of the padded matrix per thread.
__global__ void k_train_pack(TrainPack a) {
    const int pm = (a.M + 31) / 32 * 32, pn = (a.N + 31) / 32 * 32;
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)pm * pn) return;
    const int m = (int)(e / pn), n = (int)(e % pn);
    const bf16 w = m < a.M && n < a.N ? a.w[(size_t)m * a.N + n] : (bf16)0.f;
    const int sm = frag_steps(a.M), sn = frag_steps(a.N);
    if (n < sn * 16) a.wf[frag_at(m, n, sn)] = w;
    if (m < sm * 16) a.wt[frag_at(n, m, sm)] = w;
}

bool split_ok(const TrainSplit& s, int K) {
    return s.chunk > 0 && s.chunk % 32 == 0 && s.n_split > 0 && (long)s.chunk * s.n_split >= K &&
           (long)s.chunk * (s.n_split - 1) < K;
}

}  // namespace

hipError_t launch_train_fwd(const TrainFwd& a, hipStream_t s) {
    if (a.B <= 0 || a.B % 8 || a.b.steps * 16 < (a.B + 31) / 32 * 32) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_train_fwd, dim3((a.B + kRows - 1) / kRows), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_mse(const TrainMse& a, hipStream_t s) {
    if (a.N <= 0 || a.N % 8 || a.B % 8 || a.b.steps * 16 < a.B || a.N >= (1 << 24))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_train_mse, dim3((a.N + 127) / 128, (a.B + 127) / 128), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_dh(const TrainDh& a, hipStream_t s) {
    if (a.N % 8 || !split_ok(a.sp, a.N)) return hipErrorInvalidValue;
    const int n_mt = (a.B + DhTile::TM - 1) / DhTile::TM;
    hipLaunchKernelGGL(k_train_dh, dim3((n_mt + 7) / 8 * 8 * 4), dim3(DhTile::T), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_hidden(const TrainHidden& a, hipStream_t s) {
    if (!split_ok(a.sp, H)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_train_hidden, dim3((a.B + kRows - 1) / kRows), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_w(TrainW a, hipStream_t s) {
    const auto tiles = [&](int tm, int tn) {  // of all layers; their first work-groups
        int n = 0, all = 0;
        for (int l = 0; l < 4; ++l) {
            const int nt = (a.l[l].N + tn - 1) / tn;
            a.l[l].first = n;
            n += (a.l[l].M + 8 * tm - 1) / (8 * tm) * 8 * nt;
            all += (a.l[l].M + tm - 1) / tm * nt;
        }
        return std::pair<int, int>(n, all);
    };
    for (int l = 0; l < 4; ++l)
        if (a.l[l].M % 8 || a.l[l].N % 8 || !split_ok(a.l[l].sp, a.B)) return hipErrorInvalidValue;
    auto n = tiles(WTile::TM, WTile::TN);
    // Four layers of up to 1024 outputs are 76 tiles or fewer: a large batch went
    // through them one work-group a compute unit, and most of the units idle.  Four
    // steps, large tiles -> small: 262144 x 64 13.0 -> 9.5 ms (layer by layer 11.2),
    // 131072 x 256 7.0 -> 5.5 (6.8), 65536 x 1024 4.90 -> 4.81, 2048 x 256 273 -> 229
    // us; 124 tiles, 65536 x 2048: 6.96 and 7.02 ms.
    if (n.second < 100) {
        n = tiles(WTileSmall::TM, WTileSmall::TN);
        hipLaunchKernelGGL((k_train_w<WTileSmall, 8>), dim3(n.first), dim3(WTileSmall::T), 0, s, a);
    } else {
        hipLaunchKernelGGL((k_train_w<WTile, 6>), dim3(n.first), dim3(WTile::T), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_train_ones(bf16* ht, int steps, hipStream_t s) {
    hipLaunchKernelGGL(k_train_ones, dim3((steps * 16 + 255) / 256), dim3(256), 0, s, ht, steps);
    return hipGetLastError();
}

hipError_t launch_train_pack(const TrainPack& a, hipStream_t s) {
    const long n = (long)((a.M + 31) / 32 * 32) * ((a.N + 31) / 32 * 32);
    hipLaunchKernelGGL(k_train_pack, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace nr
