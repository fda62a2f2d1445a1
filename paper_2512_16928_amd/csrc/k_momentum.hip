// K1: momentum accumulate fused with the line-norm reduction.
//
// M <- fl32(M + G) in place (Algorithm 1, accumulate step) and, for every line of
// the selection axis, the l1 norm (Select_alpha, Default rule) and the
// squared l2 norm (for ||M[K]||_F, the Newton-Schulz normalisation).
// The l1 norm is accumulated in double-double from the fp32 values and
// rounded once at the end, which gives the exactly rounded sum unless the
// exact sum lies within ~n*2^-106 (relative) of an fp64 rounding boundary.
//
// Row mode: one wave per row (four rows per 256-thread block); every lane
// streams 4-element vectors (16 B of M, 8 B of bf16 G), eight vectors in
// flight, and the wave reduces in a fixed shuffle order. M and G are
// streamed with non-temporal loads and stores (each is touched once), but for
// the ends of long rows and short rows in some launches (momentum_rows).
// Column mode: M is only read here (the gather pass rewrites whole rows of
// M once the selection is known, so the sum is stored once); each thread
// owns 4 adjacent columns of a block of rows and writes double-double
// partials, and a second pass folds the row blocks in order. The row blocks
// and the fold depend on the matrices' shape and number, so the last bits of
// the squared norms do too. No floating-point atomics anywhere: results are
// run-to-run bitwise reproducible.
#include "dion2_device.h"

namespace dion2 {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ void accumulate(double x, double& hi, double& lo, double& s2) {
    double s, e;
    two_sum(hi, x, s, e);
    hi = s;
    lo += e;
    s2 += x * x;
}

// Fixed-order wave reduction of (hi, lo, s2); result valid in every lane.
__device__ __forceinline__ void wave_reduce(double& hi, double& lo, double& s2) {
    for (int off = 32; off > 0; off >>= 1) {
        double ohi = __shfl_xor(hi, off);
        double olo = __shfl_xor(lo, off);
        double os2 = __shfl_xor(s2, off);
        dd_add(hi, lo, ohi, olo);
        s2 += os2;
    }
}

constexpr int kRowsPerBlock = kThreads / 64;
constexpr int kRowVecs = 8;   // 4-element vectors per lane in flight
constexpr int64_t kRowChunk = 64 * 4 * kRowVecs;   // entries of a row a wave takes at once

// What a row has past its whole chunks is taken one vector at a time through
// the caches, or (BATCHED) with all its loads before its first store, past
// the caches like the chunks and for any length. Through the caches wins
// behind whole chunks, until a launch's rests together, about 1.3 GB, outgrow
// them (us, cached and BATCHED: 8 x 4096 x 11008 681 and 709, 32 x 2000 x 4000
// 453 and 459; 64 x 2000 x 3584 837 and 815), and for rows of one or two vectors
// in a launch that the 256 MB last-level cache about holds (200 x 256 x 256: the
// step 77 and 83; 1000 x 256 x 256 331 and 327). BATCHED wins on rows between,
// where one vector at a time is a chain of up to eight waits (64 x 1000 x 2000
// 234 and 211, 1 x 1000 x 2000 11 and 8.5), and with fp32 G behind whole chunks
// in launches of less than a wave a SIMD (1 x 512 x 4000 12.3 and 10.8; with
// bf16 G 12.4 and 13.1).
template <typename GT, bool BATCHED>
__global__ __launch_bounds__(kThreads) void momentum_rows(MatSet ms, int64_t rows, int64_t cols,
                                                          double* __restrict__ l1,
                                                          double* __restrict__ sq) {
    const int b = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (row >= rows) return;   // whole wave
    float* __restrict__ M = ms.m(b) + row * cols;
    const GT* __restrict__ G = ms.g<GT>(b) + row * cols;
    typedef typename Quad<GT>::V GRaw;
    // four independent accumulators (element v of each vector goes to set v)
    // keep the fp64 dependency chains short; they are folded in a fixed order
    double h4[4] = {0.0, 0.0, 0.0, 0.0}, l4[4] = {0.0, 0.0, 0.0, 0.0}, q4[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t c = 0;
    for (; c + kRowChunk <= cols; c += kRowChunk) {
        float m[kRowVecs][4], g[kRowVecs][4];
#pragma unroll
        for (int u = 0; u < kRowVecs; ++u) {
            unpack4(ldg_nt<float4>(M + c + (u * 64 + lane) * 4), m[u]);
            unpack4(ldg_nt<GRaw>(G + c + (u * 64 + lane) * 4), g[u]);
        }
#pragma unroll
        for (int u = 0; u < kRowVecs; ++u) {
#pragma unroll
            for (int v = 0; v < 4; ++v) m[u][v] = m[u][v] + g[u][v];
            stg_nt(M + c + (u * 64 + lane) * 4, make_float4(m[u][0], m[u][1], m[u][2], m[u][3]));
#pragma unroll
            for (int v = 0; v < 4; ++v) accumulate(fabs((double)m[u][v]), h4[v], l4[v], q4[v]);
        }
    }
    if constexpr (!BATCHED) {   // the row's length is a multiple of 4
        for (int64_t cc = c + lane * 4; cc < cols; cc += 64 * 4) {
            float m[4], g[4];
            load4(M + cc, m);
            load4(G + cc, g);
#pragma unroll
            for (int v = 0; v < 4; ++v) m[v] = m[v] + g[v];
            stg(M + cc, make_float4(m[0], m[1], m[2], m[3]));
#pragma unroll
            for (int v = 0; v < 4; ++v) accumulate(fabs((double)m[v]), h4[v], l4[v], q4[v]);
        }
    } else if (c < cols) {
        // (memory counters retire in issue order); entries past the end count as zero
        float4 mr[kRowVecs];
        GRaw gr[kRowVecs];
#pragma unroll
        for (int u = 0; u < kRowVecs; ++u) {
            if (c + u * 256 >= cols) break;   // uniform
            const int64_t cc = c + (u * 64 + lane) * 4;
            mr[u] = load_quad(M + cc, cols - cc);
            gr[u] = load_quad(G + cc, cols - cc);
        }
#pragma unroll
        for (int u = 0; u < kRowVecs; ++u) {
            if (c + u * 256 >= cols) break;
            const int64_t cc = c + (u * 64 + lane) * 4;
            float m[4], g[4];
            unpack4(mr[u], m);
            unpack4(gr[u], g);
#pragma unroll
            for (int v = 0; v < 4; ++v) m[v] = m[v] + g[v];
            store_quad(M + cc, make_float4(m[0], m[1], m[2], m[3]), cols - cc);
#pragma unroll
            for (int v = 0; v < 4; ++v) accumulate(fabs((double)m[v]), h4[v], l4[v], q4[v]);
        }
    }
    double hi = h4[0], lo = l4[0], s2 = q4[0];
#pragma unroll
    for (int v = 1; v < 4; ++v) {
        dd_add(hi, lo, h4[v], l4[v]);
        s2 += q4[v];
    }
    wave_reduce(hi, lo, s2);
    if (lane == 0) {
        l1[(int64_t)b * rows + row] = hi + lo;
        sq[(int64_t)b * rows + row] = s2;
    }
}

// Column mode, partial sums of a block of rb_rows rows; the row blocks shrink
// with the launch (momentum_col_blocks), since 256 rows a thread left one 8192
// x 2048 matrix 64 blocks and 145 us, where 64 rows a block take 24.
//
// From about three waves a SIMD on (kStreamWaves), rows of whole vectors: a wave
// streams 256 columns down the whole row block, a row at a time; the waves,
// not the loads of one, cover the latency, and the registers must leave room
// for eight a SIMD. Blocks of four adjacent waves where they tile the row, else
// of one. Bound by memory: 16 x 8192 x 2048 242 us, 256 x 2048 x 1408 741; with
// a wave's eight rows in flight, as below, 261 and 771. (5 x 11008 x 4096, 3440
// waves: 231 with the fold, 241 below.)
constexpr int64_t kStreamWaves = 3328;

int64_t stream_waves(int64_t cols, int64_t nrb, int batch) { return (cols + 255) / 256 * nrb * batch; }

template <typename GT>
__global__ __launch_bounds__(kThreads) void momentum_cols_stream(MatSet ms, int64_t rows, int64_t cols, int rb_rows,
                                                                 int nrb, double* __restrict__ part) {
    constexpr int VEC = 4;
    const int b = blockIdx.z;
    const int rb = blockIdx.y;
    const int64_t c0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * VEC;
    if (c0 >= cols) return;
    const int64_t r0 = (int64_t)rb * rb_rows;
    const int64_t r1 = r0 + rb_rows < rows ? r0 + rb_rows : rows;
    const float* __restrict__ M = ms.m(b);
    const GT* __restrict__ G = ms.g<GT>(b);
    double hi[VEC], lo[VEC], s2[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) hi[v] = lo[v] = s2[v] = 0.0;
#pragma unroll 4
    for (int64_t r = r0; r < r1; ++r) {
        const float* p = M + r * cols + c0;
        const GT* q = G + r * cols + c0;
        float m[VEC], g[VEC];
        unpack4(ldg_nt<float4>(p), m);
        unpack4(ldg_nt<typename Quad<GT>::V>(q), g);
#pragma unroll
        for (int v = 0; v < VEC; ++v) m[v] = m[v] + g[v];
#pragma unroll
        for (int v = 0; v < VEC; ++v) accumulate(fabs((double)m[v]), hi[v], lo[v], s2[v]);
    }
    double* out = part + ((int64_t)b * nrb + rb) * 3 * cols;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        out[c0 + v] = hi[v];
        out[cols + c0 + v] = lo[v];
        out[2 * cols + c0 + v] = s2[v];
    }
}

// Smaller launches: a block covers 256 columns, each wave a contiguous quarter
// of the rows, kColUnroll of them loaded at once, and the quarters are folded
// in row order (3072 waves of the other kernel, us with it and here: 64 x 2048 x
// 1408 226 and 190, 12 x 8192 x 2048 216 and 203; 2048 waves, 8 x 8192 x 2048:
// 182 and 131).
constexpr int kColUnroll = 8;

template <typename GT, bool RAGGED>
__global__ __launch_bounds__(kThreads) void momentum_cols_partial(MatSet ms, int64_t rows,
                                                                  int64_t cols, int rb_rows,
                                                                  int nrb,
                                                                  double* __restrict__ part) {
    constexpr int VEC = 4;
    constexpr int kW = kThreads / 64;   // waves that share a column
    __shared__ double fold[kW - 1][3][VEC][64];
    const int b = blockIdx.z;
    const int rb = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = ((int64_t)blockIdx.x * 64 + lane) * VEC;
    const int64_t n = cols - c0;   // columns of this lane that exist
    const bool in = n > 0;
    const int64_t quarter = rb_rows / kW;
    const int64_t r0 = (int64_t)rb * rb_rows + wave * quarter;
    const int64_t r1 = r0 + quarter < rows ? r0 + quarter : rows;
    const float* __restrict__ M = ms.m(b);
    const GT* __restrict__ G = ms.g<GT>(b);
    typedef typename Quad<GT>::V GRaw;
    double hi[VEC], lo[VEC], s2[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) hi[v] = lo[v] = s2[v] = 0.0;
    auto add = [&](const float4& mr, const GRaw& gr) {
        float m[VEC], g[VEC];
        unpack4(mr, m);
        unpack4(gr, g);
#pragma unroll
        for (int v = 0; v < VEC; ++v) accumulate(fabs((double)(m[v] + g[v])), hi[v], lo[v], s2[v]);
    };
    if (in) {   // (the loads of lanes with four columns need no other branch)
        int64_t r = r0;
        for (; r + kColUnroll <= r1; r += kColUnroll) {
            float4 m[kColUnroll];
            GRaw g[kColUnroll];
#pragma unroll
            for (int u = 0; u < kColUnroll; ++u) {
                if constexpr (RAGGED) {
                    m[u] = load_quad(M + (r + u) * cols + c0, n);
                    g[u] = load_quad(G + (r + u) * cols + c0, n);
                } else {
                    m[u] = ldg_nt<float4>(M + (r + u) * cols + c0);
                    g[u] = ldg_nt<GRaw>(G + (r + u) * cols + c0);
                }
            }
#pragma unroll
            for (int u = 0; u < kColUnroll; ++u) add(m[u], g[u]);
        }
        for (; r < r1; ++r) add(load_quad<RAGGED>(M + r * cols + c0, n), load_quad<RAGGED>(G + r * cols + c0, n));
    }
    if (wave > 0) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            fold[wave - 1][0][v][lane] = hi[v];
            fold[wave - 1][1][v][lane] = lo[v];
            fold[wave - 1][2][v][lane] = s2[v];
        }
    }
    __syncthreads();
    if (wave > 0 || !in) return;
    double* out = part + ((int64_t)b * nrb + rb) * 3 * cols;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
#pragma unroll
        for (int w = 0; w < kW - 1; ++w) {
            dd_add(hi[v], lo[v], fold[w][0][v][lane], fold[w][1][v][lane]);
            s2[v] += fold[w][2][v][lane];
        }
        if (!RAGGED || v < n) {
            out[c0 + v] = hi[v];
            out[cols + c0 + v] = lo[v];
            out[2 * cols + c0 + v] = s2[v];
        }
    }
}

// The row blocks folded in order: WAYS groups of threads of a block take a
// contiguous share of the row blocks each, and the shares are folded in
// order. Latency-bound in small launches (one thread a column over 32 row
// blocks took 12 us, sixteen take 4); a launch with blocks enough folds a
// column by one thread, coalesced and without the second stage (256 x 2048 x
// 1408: 17.9 us with sixteen, 11.7 with one; 64 x 2048 x 1408: 8.1 with
// sixteen, 5.2 with four).
template <int WAYS>
__global__ __launch_bounds__(kThreads) void momentum_cols_final(const double* __restrict__ part,
                                                                int nrb, int64_t cols,
                                                                double* __restrict__ l1,
                                                                double* __restrict__ sq) {
    constexpr int kCols = kThreads / WAYS;
    const int b = blockIdx.y;
    const int cl = threadIdx.x % kCols, way = threadIdx.x / kCols;
    const int64_t c = (int64_t)blockIdx.x * kCols + cl;
    const int per = (nrb + WAYS - 1) / WAYS;
    const int q0 = way * per < nrb ? way * per : nrb;
    const int q1 = q0 + per < nrb ? q0 + per : nrb;
    double hi = 0.0, lo = 0.0, s2 = 0.0;
    if (c < cols) {
        const double* p = part + ((int64_t)b * nrb + q0) * 3 * cols + c;
#pragma unroll 4
        for (int rb = q0; rb < q1; ++rb, p += 3 * cols) {
            dd_add(hi, lo, p[0], p[cols]);
            s2 += p[2 * cols];
        }
    }
    if constexpr (WAYS > 1) {
        __shared__ double fold[3][WAYS][kCols];
        fold[0][way][cl] = hi;
        fold[1][way][cl] = lo;
        fold[2][way][cl] = s2;
        __syncthreads();
        if (way > 0) return;
        for (int w = 1; w < WAYS; ++w) {
            dd_add(hi, lo, fold[0][w][cl], fold[1][w][cl]);
            s2 += fold[2][w][cl];
        }
    }
    if (c >= cols) return;
    l1[(int64_t)b * cols + c] = hi + lo;
    sq[(int64_t)b * cols + c] = s2;
}

template <typename GT>
hipError_t launch_typed(const MomentumArgs& a, int axis, hipStream_t s) {
    if (axis == 0) {
        dim3 grid((unsigned)((a.rows + kRowsPerBlock - 1) / kRowsPerBlock), (unsigned)a.batch);
        const int64_t lines = a.rows * a.batch;
        const bool cached = a.cols >= kRowChunk ? lines * (a.cols % kRowChunk) <= int64_t(1) << 27
                                                : a.cols <= 512 && lines * a.cols <= int64_t(1) << 25;
        if (a.cols % 4 == 0 && cached && (sizeof(GT) == 2 || a.cols < kRowChunk || lines >= 1024))
            hipLaunchKernelGGL((momentum_rows<GT, false>), grid, dim3(kThreads), 0, s, a.ms, a.rows, a.cols, a.l1, a.sq);
        else
            hipLaunchKernelGGL((momentum_rows<GT, true>), grid, dim3(kThreads), 0, s, a.ms, a.rows, a.cols, a.l1, a.sq);
    } else {
        auto launch = [&](auto kernel, int threads, int64_t cols) {
            const dim3 grid((unsigned)((a.cols + cols - 1) / cols), (unsigned)a.nrb, (unsigned)a.batch);
            hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, a.ms, a.rows, a.cols, a.rb_rows, a.nrb, a.part);
        };
        if (a.cols % 4) launch(momentum_cols_partial<GT, true>, kThreads, 256);
        else if (stream_waves(a.cols, a.nrb, a.batch) < kStreamWaves)
            launch(momentum_cols_partial<GT, false>, kThreads, 256);
        else if (a.cols % (kThreads * 4) == 0) launch(momentum_cols_stream<GT>, kThreads, kThreads * 4);
        else launch(momentum_cols_stream<GT>, 64, 256);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        auto fold = [&](auto kernel, int ways) {
            const int cols = kThreads / ways;
            const dim3 grid((unsigned)((a.cols + cols - 1) / cols), (unsigned)a.batch);
            hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, a.part, a.nrb, a.cols, a.l1, a.sq);
        };
        const int64_t blocks = (a.cols + kThreads - 1) / kThreads * a.batch;   // of one thread a column
        if (blocks >= 1024) fold(momentum_cols_final<1>, 1);
        else if (blocks >= 256) fold(momentum_cols_final<4>, 4);
        else fold(momentum_cols_final<16>, 16);
    }
    return hipGetLastError();
}

}  // namespace

// Row blocking of the column-mode reduction: blocks of 256 rows keep the
// partials small next to the matrix (24 bytes for 1280 or more); a launch
// of fewer than four blocks a compute unit halves them, down to 32 rows, as
// long as the partials fit in part_bytes.
int64_t momentum_col_blocks(int64_t rows, int64_t cols, int batch, size_t part_bytes, int* rb_rows) {
    const int64_t strips = (cols + 255) / 256 * batch;
    auto blocks = [&](int rb) { return (rows + rb - 1) / rb; };
    int rb = 256;
    while (rb > 32 && strips * blocks(rb) < 1024 &&
           (size_t)batch * (size_t)blocks(rb / 2) * 3 * (size_t)cols * sizeof(double) <= part_bytes)
        rb /= 2;
    *rb_rows = rb;
    return blocks(rb);
}

hipError_t launch_momentum(const MomentumArgs& a, int axis, int g_bf16, hipStream_t s) {
    return g_bf16 ? launch_typed<uint16_t>(a, axis, s) : launch_typed<float>(a, axis, s);
}

}  // namespace dion2
