// affine forward/backward (paper, Section 2: the affine layer is the matrix
// product of the inputs with the weights plus a broadcast bias row, and its
// backward returns the input, weight and bias gradients in that order) on the
// gfx950 matrix cores.
//
// One strided GEMM kernel serves all three products:
//   forward  out = X W + b        (A = X,        B = W)
//   dX = g W^T                    (A = g,        B = W viewed transposed)
//   dW = X^T g                    (A = X viewed transposed, B = g)
// where g = dout masked to out_fwd > 0 when a relu mask is given.  Column sums
// of g (db) use a separate fixed-order kernel.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace dmlnn {
namespace {

constexpr int kMaxNK = 8;    // waves per block, each a k range of the block's tile

struct GemmArgs {
    const void *A, *Amask;  // A(i,k) = A[i*sAm + k*sAk]; mask has the same strides
    const void *B, *Bmask;  // B(k,j) = B[k*sBk + j*sBn]
    const void *bias;       // per column j, or null
    void *C;                // C[i*ldc + j]
    void *part;             // [splits][M][N] partial products when splits > 1
    const void *xmask;      // C is zeroed where xmask[i*ldc + j] <= 0 (or null)
    long long sAm, sAk, sBk, sBn, ldc;
    int M, N, K, relu;
};

// The k order of an MFMA fragment.  k is walked in groups of 16 (four MFMA
// k-steps).  Inside a group the k order is permuted so that an operand stored
// with k contiguous (X for the forward product, g and W for dX) is read with
// 16-byte vector loads: lane quarter q holds k = 2q, 2q+1, 8+2q, 9+2q of the
// group in its four steps (fp64; for fp32 k = 4q..4q+3).  Each step still
// covers four distinct k, the four steps cover the group, and both operands
// use the same order, so the products are unchanged.  A 16-row fragment then
// reads 64 contiguous bytes per row per load instead of 32, which halves the
// L1 cache accesses that bound these loads.  Operands with rows contiguous
// keep per-step loads (16 lanes read one 16-element row piece).
template <typename T>
struct GemmFrag {
    // position in the group of k-step u for lane quarter q
    static __device__ __forceinline__ int kpos(int q, int u)
    {
        if (sizeof(T) == 8) return (u & 1) + 2 * q + 8 * (u >> 1);
        return 4 * q + u;
    }
    // the four values of a k-contiguous row at group start p (16-byte aligned)
    static __device__ __forceinline__ void vload(const T *p, int q, T (&v)[4])
    {
        if constexpr (sizeof(T) == 8) {
            const double2 lo = *reinterpret_cast<const double2 *>(p + 2 * q);
            const double2 hi = *reinterpret_cast<const double2 *>(p + 8 + 2 * q);
            v[0] = lo.x;
            v[1] = lo.y;
            v[2] = hi.x;
            v[3] = hi.y;
        } else {
            const float4 x = *reinterpret_cast<const float4 *>(p + 4 * q);
            v[0] = x.x;
            v[1] = x.y;
            v[2] = x.z;
            v[3] = x.w;
        }
    }
};

// A block owns one output tile of WT x WT MFMA tiles (16 x 16 each) and
// `nk` waves; the waves of the tile's `splits` blocks walk contiguous,
// balanced ranges of whole 16-k groups, in (block, wave) order, reading their
// MFMA fragments straight from global memory.  WT = 2 (32 x 32 per wave: two
// A and two B fragments feed four MFMAs per k-step) halves the operand
// fetches per MFMA against WT = 1 for products with long K; WT = 1 keeps more
// blocks for short K or a narrow output.  The waves of a block add their
// partial tiles through LDS in wave order; with splits > 1 each block writes
// its sum to its own slice of the workspace and a second kernel adds the
// slices in split order, so the result is deterministic for a given split
// count.  The products of a LeNet-sized step are too small to fill the GPU by
// tiles alone (the 64 x 512 forward from K = 3136 has 32 tiles of 32 x 32):
// the k split over blocks is what lets most CUs take part.
//
// These products are bound by the latency and the CU's fetch rate of their
// operand loads, not by the matrix cores, so groups are loaded BATCH at a
// time, one batch ahead (two register sets), so one batch's loads are in
// flight while the previous batch's MFMAs issue.  Rows and columns past the
// matrix edge read a clamped (valid) row or column; they only feed outputs
// that are not stored.  A partial last group (K not a multiple of 16) reads
// clamped k and zeroes both operands past K.  A relu mask is loaded beside its
// operand and applied just before the MFMA.  With `xmask`, each output (i, j)
// is multiplied by (xmask[i, j] > 0) before it is stored (the relu backward
// of the layer below, folded into dX).
template <typename T, bool MA, bool MB, bool VA, bool VB, int BATCH, int WT>
__global__ __launch_bounds__(kMaxNK * kWave) void gemm_kernel(GemmArgs g)
{
    using MF = Mfma<T>;
    using FR = GemmFrag<T>;
    constexpr int TE = 16 * WT;  // tile edge
    extern __shared__ __align__(16) unsigned char smem[];
    T *s_red = reinterpret_cast<T *>(smem);  // [wave][TE * TE]

    const int lane = lane_id(), wave = wave_id();
    const int nk = blockDim.x / kWave;
    const int tm = (g.M + TE - 1) / TE;
    const int ntile = gridDim.x, splits = gridDim.y;
    // Blocks are dealt to the 8 XCDs round-robin and each XCD has its own L2:
    // renumber (tile, split), tile fastest with row tiles first, so that each
    // XCD owns a contiguous run and the row tiles of a column strip share one
    // L2 copy of that strip of B (for the LeNet forward a 12.8 MB weight).
    const int t = xcd_logical_block(blockIdx.x + ntile * blockIdx.y, ntile * splits);
    const int tile = t % ntile, split = t / ntile;
    const int i0 = (tile % tm) * TE, j0 = (tile / tm) * TE;
    const int G = (g.K + 15) / 16;
    const long long R = (long long)splits * nk, r = (long long)split * nk + wave;
    const int g_lo = (int)(r * G / R), g_hi = (int)((r + 1) * G / R);
    const int ngrp = g_hi - g_lo;
    const bool ragged = (g.K & 15) != 0 && g_hi == G;  // this range holds the partial group
    const T *A = reinterpret_cast<const T *>(g.A);
    const T *Am = reinterpret_cast<const T *>(g.Amask);
    const T *B = reinterpret_cast<const T *>(g.B);
    const T *Bm = reinterpret_cast<const T *>(g.Bmask);
    const int li = lane & 15, q = lane >> 4;
    long long arow[WT], bcol[WT];
#pragma unroll
    for (int x = 0; x < WT; ++x) {
        arow[x] = (long long)min(i0 + 16 * x + li, g.M - 1) * g.sAm;
        bcol[x] = (long long)min(j0 + 16 * x + li, g.N - 1) * g.sBn;
    }

    struct Grp {
        T a[WT][4], b[WT][4];
        T am[WT][4], bm[WT][4];  // used only with a mask (MA / MB)
    };
    // one group of 16 k from k0; `part`: the partial last group of K
    auto load_grp = [&](int k0, bool part, Grp &f) {
        if (part) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + FR::kpos(q, u), kc = min(k, g.K - 1);
                const bool in = k < g.K;
#pragma unroll
                for (int x = 0; x < WT; ++x) {
                    const long long oa = arow[x] + (long long)kc * g.sAk;
                    const T av = A[oa];
                    f.a[x][u] = in ? av : T(0);
                    if (MA) f.am[x][u] = Am[oa];
                    const long long ob = (long long)kc * g.sBk + bcol[x];
                    const T bv = B[ob];
                    f.b[x][u] = in ? bv : T(0);
                    if (MB) f.bm[x][u] = Bm[ob];
                }
            }
            return;
        }
#pragma unroll
        for (int x = 0; x < WT; ++x) {
            if constexpr (VA) {
                FR::vload(A + arow[x] + k0, q, f.a[x]);
                if constexpr (MA) FR::vload(Am + arow[x] + k0, q, f.am[x]);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const long long oa = arow[x] + (long long)(k0 + FR::kpos(q, u)) * g.sAk;
                    f.a[x][u] = A[oa];
                    if (MA) f.am[x][u] = Am[oa];
                }
            }
            if constexpr (VB) {
                FR::vload(B + bcol[x] + k0, q, f.b[x]);
                if constexpr (MB) FR::vload(Bm + bcol[x] + k0, q, f.bm[x]);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const long long ob = (long long)(k0 + FR::kpos(q, u)) * g.sBk + bcol[x];
                    f.b[x][u] = B[ob];
                    if (MB) f.bm[x][u] = Bm[ob];
                }
            }
        }
    };
    typename MF::acc_t acc[WT][WT];
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int y = 0; y < WT; ++y) acc[x][y] = MF::zero();
    auto mma_grp = [&](const Grp &f) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            T av[WT], bv[WT];
#pragma unroll
            for (int x = 0; x < WT; ++x) {
                av[x] = MA ? (f.am[x][u] > T(0) ? f.a[x][u] : T(0)) : f.a[x][u];
                bv[x] = MB ? (f.bm[x][u] > T(0) ? f.b[x][u] : T(0)) : f.b[x][u];
            }
#pragma unroll
            for (int x = 0; x < WT; ++x)
#pragma unroll
                for (int y = 0; y < WT; ++y) acc[x][y] = MF::mma(av[x], bv[y], acc[x][y]);
        }
    };
    auto load_batch = [&](int b, Grp (&f)[BATCH]) {
#pragma unroll
        for (int c = 0; c < BATCH; ++c) {
            const int gi = b * BATCH + c;
            if (gi < ngrp) load_grp((g_lo + gi) * 16, ragged && gi == ngrp - 1, f[c]);
        }
    };
    auto mma_batch = [&](int b, const Grp (&f)[BATCH]) {
#pragma unroll
        for (int c = 0; c < BATCH; ++c)
            if (b * BATCH + c < ngrp) mma_grp(f[c]);
    };
    const int nbatch = (ngrp + BATCH - 1) / BATCH;
    Grp f0[BATCH], f1[BATCH];
    if (nbatch > 0) load_batch(0, f0);
    int i = 0;
    for (; i + 1 < nbatch; i += 2) {
        load_batch(i + 1, f1);
        mma_batch(i, f0);
        if (i + 2 < nbatch) load_batch(i + 2, f0);
        mma_batch(i + 1, f1);
    }
    if (i < nbatch) mma_batch(i, f0);

    T *C = reinterpret_cast<T *>(g.C);
    T *P = reinterpret_cast<T *>(g.part);
    const T *bias = reinterpret_cast<const T *>(g.bias);
    const T *xm = reinterpret_cast<const T *>(g.xmask);
    auto store = [&](int ii, int j, T v) {
        if (ii >= g.M || j >= g.N) return;
        if (splits == 1) {
            if (bias) v += bias[j];
            v = relu_if(v, g.relu);
            if (xm && !(xm[(long long)ii * g.ldc + j] > T(0))) v = T(0);
            C[(long long)ii * g.ldc + j] = v;
        } else {
            P[((long long)split * g.M + ii) * g.N + j] = v;
        }
    };
    if (nk == 1) {  // one wave: no partial tiles to add
#pragma unroll
        for (int x = 0; x < WT; ++x)
#pragma unroll
            for (int y = 0; y < WT; ++y)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
                    store(i0 + 16 * x + MF::row(lane, rr), j0 + 16 * y + li, acc[x][y][rr]);
        return;
    }
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int y = 0; y < WT; ++y)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                s_red[wave * TE * TE + (16 * x + MF::row(lane, rr)) * TE + 16 * y + li] =
                    acc[x][y][rr];
    __syncthreads();
    for (int e = threadIdx.x; e < TE * TE; e += blockDim.x) {
        T v = s_red[e];
        for (int w = 1; w < nk; ++w) v += s_red[w * TE * TE + e];
        store(i0 + e / TE, j0 + e % TE, v);
    }
}

// C = act(sum over splits of the partial products + bias), splits added in
// order; zero where xmask (if given) is not positive.
template <typename T>
__global__ __launch_bounds__(256) void gemm_split_reduce(const T *part, const T *bias,
                                                         const T *xmask, T *C, int M, int N,
                                                         long long ldc, int splits, int relu)
{
    const long long MN = (long long)M * N;
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= MN) return;
    const int ii = (int)(e / N), j = (int)(e - (long long)ii * N);
    T v = part[e];
    for (int s = 1; s < splits; ++s) v += part[s * MN + e];
    if (bias) v += bias[j];
    v = relu_if(v, relu);
    if (xmask && !(xmask[(long long)ii * ldc + j] > T(0))) v = T(0);
    C[(long long)ii * ldc + j] = v;
}

// db[j] = sum_i g[i, j], g masked by out_fwd > 0 if given.  A block covers 16
// columns with 16 row phases each: thread (j, ph) sums rows ph, ph+16, ... in
// order, and the 16 phase sums are added in phase order (deterministic).
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T *G, const T *mask, T *db, int N,
                                                     int M)
{
    __shared__ T s_part[16][17];
    const int jl = threadIdx.x & 15, ph = threadIdx.x >> 4;
    const int j = blockIdx.x * 16 + jl;
    T s = T(0);
    if (j < M) {
        // eight rows' loads in flight, added in order (a load each waited for took
        // 11 us for 512 x 1000 in fp32; here 5)
        for (int i = ph; i < N; i += 16 * 8) {
            T v[8], m[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const size_t o = (size_t)min(i + 16 * u, N - 1) * M + j;
                v[u] = G[o];
                m[u] = mask ? mask[o] : T(1);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + 16 * u < N) s += m[u] > T(0) ? v[u] : T(0);
        }
    }
    s_part[ph][jl] = s;
    __syncthreads();
    if (ph == 0 && j < M) {
        T t = s_part[0][jl];
        for (int q = 1; q < 16; ++q) t += s_part[q][jl];
        db[j] = t;
    }
}

// An operand takes the vector loads when k is contiguous and every row start
// is 16-byte aligned.
template <typename T>
bool vec_ok(const void *p, long long s_row, long long s_k)
{
    constexpr long long e = 16 / sizeof(T);  // elements per 16 bytes
    return s_k == 1 && s_row % e == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0;
}

template <typename T, bool MA, bool MB, int BATCH, int WT>
auto pick_gemm(bool va, bool vb)
{
    return va ? (vb ? gemm_kernel<T, MA, MB, true, true, BATCH, WT>
                    : gemm_kernel<T, MA, MB, true, false, BATCH, WT>)
              : (vb ? gemm_kernel<T, MA, MB, false, true, BATCH, WT>
                    : gemm_kernel<T, MA, MB, false, false, BATCH, WT>);
}

template <typename T, int WT>
auto pick_masked(const GemmArgs &g, bool va, bool vb)
{
    // fp64 with a mask holds one group per batch (registers); the rest two
    constexpr int BM = sizeof(T) == 8 ? 1 : 2;
    return g.Amask ? pick_gemm<T, true, false, BM, WT>(va, vb)
                   : (g.Bmask ? pick_gemm<T, false, true, BM, WT>(va, vb)
                              : pick_gemm<T, false, false, 2, WT>(va, vb));
}

}  // namespace

// Tile, waves per block and block k splits of an M x N x K product.
//   wt: 32 x 32 tiles (wt = 2) when both output edges are 32 or more and K
//       has four 16-k groups or more; else 16 x 16;
//   nk: up to 8 waves per tile while the tiles alone give fewer than 2048
//       waves (eight per CU), two groups or more each;
//   splits: only when a wave would otherwise walk more than 8 groups and the
//       grid is still short of 2048 waves: about four groups per wave, at most
//       what the workspace holds (splits x M x N elements).
GemmPlan gemm_plan(int M, int N, int K, size_t elem, size_t workspace_bytes)
{
    GemmPlan p;
    const long long G = (K + 15) / 16;
    p.wt = (M >= 32 && N >= 32 && G >= 4) ? 2 : 1;
    const int te = 16 * p.wt;
    const long long tiles = (long long)((M + te - 1) / te) * ((N + te - 1) / te);
    const long long want = 2048;
    long long nk = std::min<long long>(kMaxNK, std::max<long long>(1, G / 2));
    nk = std::max<long long>(1, std::min(nk, (want + tiles - 1) / tiles));
    long long s = 1;
    if (G > 8 * nk && tiles * nk < want) {
        s = std::min((G + 4 * nk - 1) / (4 * nk), (want + tiles * nk - 1) / (tiles * nk));
        const long long fit = (long long)(workspace_bytes / ((size_t)M * N * elem));
        s = std::min(std::min(s, fit), 65535LL);
        if (s < 2) s = 1;
    }
    p.nk = (int)nk;
    p.splits = (int)s;
    p.workspace_bytes = s > 1 ? (size_t)s * M * N * elem : 0;
    return p;
}

namespace {

template <typename T>
hipError_t gemm(GemmArgs g, void *workspace, size_t workspace_bytes, hipStream_t s)
{
    if (g.Amask && g.Bmask) return hipErrorInvalidValue;  // one masked operand at most
    const GemmPlan p = gemm_plan(g.M, g.N, g.K, sizeof(T), workspace ? workspace_bytes : 0);
    g.part = p.splits > 1 ? workspace : nullptr;
    const bool va = vec_ok<T>(g.A, g.sAm, g.sAk) && (!g.Amask || vec_ok<T>(g.Amask, g.sAm, g.sAk));
    const bool vb = vec_ok<T>(g.B, g.sBn, g.sBk) && (!g.Bmask || vec_ok<T>(g.Bmask, g.sBn, g.sBk));
    auto k = p.wt == 2 ? pick_masked<T, 2>(g, va, vb) : pick_masked<T, 1>(g, va, vb);
    const int te = 16 * p.wt;
    const size_t lds = p.nk > 1 ? (size_t)p.nk * te * te * sizeof(T) : 0;
    hipError_t e = allow_dynamic_lds(k, lds);
    if (e != hipSuccess) return e;
    const int tiles = ((g.M + te - 1) / te) * ((g.N + te - 1) / te);
    hipLaunchKernelGGL(k, dim3(tiles, p.splits), dim3(p.nk * kWave), lds, s, g);
    if ((e = hipGetLastError()) != hipSuccess || p.splits == 1) return e;
    const long long MN = (long long)g.M * g.N;
    hipLaunchKernelGGL(gemm_split_reduce<T>, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<const T *>(g.part), reinterpret_cast<const T *>(g.bias),
                       reinterpret_cast<const T *>(g.xmask), reinterpret_cast<T *>(g.C), g.M,
                       g.N, g.ldc, p.splits, g.relu);
    return hipGetLastError();
}

}  // namespace

// The affine products as conv passes of a 1x1 filter over one image of a row:
//   out = X W    forward: image W (D channels of M pixels), filters X (N x D);
//   dX = g W^T   backward_filter: image W, gradient g (N "filters" of M pixels);
//   dW = X^T g   backward_data: gradient g, filters X.
// The gather kernels' LDS tiles carry large products at fewer fetches than the
// fragments of each wave, but have fewer blocks (a long narrow product, 1000 x 4001 x
// 101 in fp32: out 40 us, gathered 72; dW 26 and 32), so every edge is 256 or more,
// and multiply-adds at least
//   - fp32, dX and dW: 2.5e8 (512 x 2048 x 1000: dX 38 -> 32 us, dW 45 -> 38; 256 x
//     1501 x 801: 41 -> 29, 18 -> 17.6; the LeNet layer 64 x 3136 x 512 has 1e8);
//   - fp32 out, fp64 dX: 2e9 (1024 x 4096 x 1024: 162 -> 116 and 251 -> 171; 512 x
//     2048 x 1000: 39 and 41, 57 and 61);
//   - fp64 out and dW: never (at these sizes 207 and 208, 61 and 80; 204 and 269, 59
//     and 71).
ConvDims affine_dims(int N, int D, int M)
{
    return ConvDims{1, D, 1, M, N, 1, 1, 1, 0, 1, M};
}

GatherPlan affine_gather(int dtype, int product, int N, int D, int M)
{
    if (std::min(N, std::min(D, M)) < 256 || (dtype == 0 && product != 1)) return GatherPlan{};
    if ((double)N * D * M < (dtype == 1 && product != 0 ? 2.5e8 : 2e9)) return GatherPlan{};
    const ConvDims d = affine_dims(N, D, M);
    if (product == 1) return gather_wgrad_plan(dtype, d, 1);
    return gather_plan(dtype, product == 2, d, false);
}

size_t affine_workspace_bytes(int dtype, int N, int D, int M)
{
    const size_t el = dtype == 0 ? 8 : 4;
    const size_t big = ~(size_t)0;
    size_t w = gemm_plan(N, M, D, el, big).workspace_bytes;                  // out = X W
    w = std::max(w, gemm_plan(N, D, M, el, big).workspace_bytes);            // dX = g W^T
    w = std::max(w, gemm_plan(D, M, N, el, big).workspace_bytes);            // dW = X^T g
    return w;
}

hipError_t launch_affine_fwd(int dtype, const void *X, const void *W, const void *b, void *out,
                             int N, int D, int M, int relu, void *workspace,
                             size_t workspace_bytes, hipStream_t s)
{
    const GatherPlan p = affine_gather(dtype, 0, N, D, M);
    if (p.MW)
        return launch_gather(dtype, false, p, W, nullptr, X, b, out, affine_dims(N, D, M), relu, s, 1);
    GemmArgs g = {};
    g.A = X;
    g.sAm = D;
    g.sAk = 1;
    g.B = W;
    g.sBk = M;
    g.sBn = 1;
    g.bias = b;
    g.C = out;
    g.ldc = M;
    g.M = N;
    g.N = M;
    g.K = D;
    g.relu = relu;
    return dtype == 0 ? gemm<double>(g, workspace, workspace_bytes, s)
                      : gemm<float>(g, workspace, workspace_bytes, s);
}

hipError_t launch_affine_bwd(int dtype, const void *dout, const void *X, const void *W,
                             const void *out_fwd, void *dX, void *dW, void *db, int N, int D,
                             int M, int relu_input, void *workspace, size_t workspace_bytes,
                             hipStream_t s)
{
    hipError_t e;
    const GatherPlan px = affine_gather(dtype, 1, N, D, M), pw = affine_gather(dtype, 2, N, D, M);
    const ConvDims dims = affine_dims(N, D, M);
    if (dX && px.MW) {
        e = launch_gather_wgrad(dtype, px, W, dout, out_fwd, dX, nullptr, nullptr, nullptr, dims, s,
                                relu_input ? X : nullptr);
        if (e != hipSuccess) return e;
    } else if (dX) {  // dX[n, d] = sum_m g[n, m] W[d, m]  (times X[n, d] > 0 with relu_input)
        GemmArgs g = {};
        g.xmask = relu_input ? X : nullptr;
        g.A = dout;
        g.Amask = out_fwd;
        g.sAm = M;
        g.sAk = 1;
        g.B = W;
        g.sBk = 1;
        g.sBn = M;
        g.C = dX;
        g.ldc = D;
        g.M = N;
        g.N = D;
        g.K = M;
        e = dtype == 0 ? gemm<double>(g, workspace, workspace_bytes, s)
                       : gemm<float>(g, workspace, workspace_bytes, s);
        if (e != hipSuccess) return e;
    }
    if (dW && pw.MW) {
        const GatherPlan p = out_fwd ? gather_plan(dtype, true, dims, true) : pw;
        if ((e = launch_gather(dtype, true, p, dout, out_fwd, X, nullptr, dW, dims, 0, s)) != hipSuccess)
            return e;
    } else if (dW) {  // dW[d, m] = sum_n X[n, d] g[n, m]
        GemmArgs g = {};
        g.A = X;
        g.sAm = 1;
        g.sAk = D;
        g.B = dout;
        g.Bmask = out_fwd;
        g.sBk = M;
        g.sBn = 1;
        g.C = dW;
        g.ldc = M;
        g.M = D;
        g.N = M;
        g.K = N;
        e = dtype == 0 ? gemm<double>(g, workspace, workspace_bytes, s)
                       : gemm<float>(g, workspace, workspace_bytes, s);
        if (e != hipSuccess) return e;
    }
    if (db) {
        dim3 grid((M + 15) / 16);
        if (dtype == 0)
            hipLaunchKernelGGL(colsum_kernel<double>, grid, dim3(256), 0, s, (const double *)dout,
                               (const double *)out_fwd, (double *)db, N, M);
        else
            hipLaunchKernelGGL(colsum_kernel<float>, grid, dim3(256), 0, s, (const float *)dout,
                               (const float *)out_fwd, (float *)db, N, M);
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace dmlnn
