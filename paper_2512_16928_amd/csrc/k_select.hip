// K2: Select_alpha -- the k lines of largest l1 norm (Default rule), or k
// lines uniformly at random (Random rule) from counter-based Philox keys.
//
// One block per matrix. Norms are non-negative fp64, so their
// bit patterns order like unsigned integers; NaN is mapped to +inf's pattern
// (a corrupted line ranks first and shows in W). An MSD radix select over
// the 64-bit keys, 8 bits per pass with an LDS histogram, finds the k-th
// largest key T and how many of the lines equal to T are still needed; the
// digit of each pass comes from a scan of the histogram by a wave. A
// second sweep in index order keeps every key > T and the lowest-indexed
// keys == T (ties to the lower index) and compacts them into K, which
// therefore comes out ascending. Up to kRegLines lines the keys live in
// registers (select_reg); beyond, they are read again in every pass
// (select_any).
//
// The block also sums the selected lines' squared l2 norms in a fixed order
// and stores 1 / (||M[K]||_F + eps), the Newton-Schulz normalisation, and
// optionally rank[i] = the number of selected lines below i (i <= d_sel),
// which the column-mode gather uses to place line i at rank[i].
#include "dion2_device.h"

namespace dion2 {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr uint64_t kInfBits = 0x7ff0000000000000ull;
constexpr int kRegLines = 8192;   // lines whose keys fit a block's registers

// Random rule: Philox-4x32-10 (Salmon, Moraes, Dror and Shaw, SC 2011), ten
// rounds of two 32 x 32 -> 64-bit products with the halves swapped and the
// round key mixed in, the key bumped by the Weyl constants between rounds.
// The line's key is the first two output words, high first.
__device__ __forceinline__ uint64_t philox_line_key(uint32_t line, uint32_t matrix, uint64_t step,
                                                    uint64_t seed) {
    uint32_t c0 = line, c1 = matrix, c2 = (uint32_t)step, c3 = (uint32_t)(step >> 32);
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
        const uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    return ((uint64_t)c0 << 32) | c1;
}

__device__ __forceinline__ uint64_t key_of(double v) {
    uint64_t u = (uint64_t)__double_as_longlong(v);
    u &= 0x7fffffffffffffffull;           // -0.0 orders as +0.0
    return u > kInfBits ? kInfBits : u;   // NaN ranks as +inf
}

// Keys ordered so that the k largest are taken: l1 norms as they are,
// Philox keys complemented (the k smallest keys win; equal keys stay
// equal, so ties still go to the lower index).
__device__ __forceinline__ uint64_t make_key(const SelectArgs& a, const double* nrm, int b, int i) {
    return a.rule ? ~philox_line_key((uint32_t)i, (uint32_t)(a.matrix0 + b), a.step, a.seed) : key_of(nrm[i]);
}

// Inclusive prefix sum over the wave's lanes, on the VALU's own lane shifts.
__device__ __forceinline__ unsigned wave_incl(unsigned v) {
    auto add = [&](unsigned x) { v += x; };
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15, rows 1 and 3
    add((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31, rows 2 and 3
    return v;
}

// At most kRegLines lines: thread t holds lines R t .. R t + R - 1. The block
// is latency-bound (one per matrix, a few dependent rounds between
// barriers), so the rounds are few: the passes start at the highest bit in
// which any two keys differ, stop as soon as a whole bin is taken, use a
// histogram each (cleared up front) and are scanned by every wave for
// itself; the squared norms are fetched with the keys; one scan of packed
// (above T, equal to T) counts places every line. 2048 lines: 15.7 us with
// eight passes over keys in LDS, 6.6 us now; 256 lines 10.0 and 4.5.
template <int T, int R>
__global__ __launch_bounds__(T) void select_reg(SelectArgs a) {
    constexpr int W = T / 64;
    constexpr int kPasses = 8;
    const int b = blockIdx.x;
    const double* __restrict__ nrm = a.l1 + (int64_t)b * a.d_sel;
    int32_t* __restrict__ out = a.sel + (int64_t)b * a.k;
    int32_t* __restrict__ rank = a.rank ? a.rank + (int64_t)b * (a.d_sel + 1) : nullptr;
    __shared__ unsigned hist[kPasses][256];
    __shared__ uint64_t wdiff[W];
    __shared__ unsigned wtot[W];
    __shared__ double red[W];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = threadIdx.x * R;

    uint64_t key[R];
    double q[R];
    const uint64_t key0 = make_key(a, nrm, b, 0);
    uint64_t diff = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = i0 + r < a.d_sel ? i0 + r : a.d_sel - 1;
        key[r] = make_key(a, nrm, b, i);
        q[r] = a.sq ? a.sq[(int64_t)b * a.d_sel + i] : 0.0;
    }
    for (int i = threadIdx.x; i < kPasses * 256; i += T) (&hist[0][0])[i] = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) diff |= key[r] ^ key0;   // (lines past the end repeat the last)
    for (int off = 32; off > 0; off >>= 1) diff |= __shfl_xor(diff, off);
    if (lane == 0) wdiff[wave] = diff;
    __syncthreads();
    diff = 0;
    for (int w = 0; w < W; ++w) diff |= wdiff[w];

    // `top` bits of the keys are decided: the common ones, then a digit a pass
    int low = diff ? 64 - __builtin_clzll(diff) : 0;   // undecided low bits
    uint64_t prefix = low < 64 ? key0 >> low << low : 0;
    uint64_t mask = low < 64 ? ~0ull << low : 0;
    unsigned need = (unsigned)a.k;   // how many still to take at or below the current prefix
    for (int pass = 0; low > 0; ++pass) {
        const int shift = low > 8 ? low - 8 : 0;
        const unsigned dmask = (1u << (low - shift)) - 1u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool in = i0 + r < a.d_sel && (key[r] & mask) == prefix;
            if (in) atomicAdd(&hist[pass][(unsigned)(key[r] >> shift) & dmask], 1u);
        }
        __syncthreads();
        // lane l owns bins 4l .. 4l+3; the digit is the largest d whose
        // suffix count reaches `need`
        unsigned c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = hist[pass][4 * lane + u];
        const unsigned own = c[0] + c[1] + c[2] + c[3];
        const unsigned incl = wave_incl(own);
        unsigned above = (unsigned)__builtin_amdgcn_readlane((int)incl, 63) - incl;   // in the higher lanes' bins
        unsigned digit = 0, left = 0, count = 0;
        bool here = false;
#pragma unroll
        for (int u = 3; u >= 0; --u) {
            if (above < need && above + c[u] >= need) {
                here = true;
                digit = 4 * lane + u;
                left = need - above;
                count = c[u];
            }
            above += c[u];
        }
        const int src = __builtin_ctzll(__ballot(here));
        digit = (unsigned)__builtin_amdgcn_readlane((int)digit, src);
        need = (unsigned)__builtin_amdgcn_readlane((int)left, src);
        count = (unsigned)__builtin_amdgcn_readlane((int)count, src);
        prefix |= (uint64_t)digit << shift;
        mask |= (uint64_t)dmask << shift;
        low = shift;
        if (count == need) break;   // every key with this prefix goes in
    }
    // keys above the decided bits go in, and the first `need` of those that equal them
    unsigned n_gt = 0, n_eq = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool valid = i0 + r < a.d_sel;
        n_gt += valid && (key[r] & mask) > prefix ? 1u : 0u;
        n_eq += valid && (key[r] & mask) == prefix ? 1u : 0u;
    }
    const unsigned packed = n_gt | (n_eq << 16);   // at most 8192 lines each
    const unsigned incl = wave_incl(packed);
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    unsigned before = incl - packed;
    for (int w = 0; w < W; ++w) before += w < wave ? wtot[w] : 0u;
    unsigned gt = before & 0xffffu, eq = before >> 16;
    double fro = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = i0 + r;
        if (i < a.d_sel) {
            const unsigned pos = gt + (eq < need ? eq : need);   // selected lines before i
            const bool above = (key[r] & mask) > prefix, equal = (key[r] & mask) == prefix;
            if (above || (equal && eq < need)) {
                out[pos] = i;
                fro += q[r];
            }
            if (rank) rank[i] = (int)pos;
            gt += above ? 1u : 0u;
            eq += equal ? 1u : 0u;
        }
    }
    // fixed-order reduction of the selected squared norms
    for (int off = 32; off > 0; off >>= 1) fro += __shfl_xor(fro, off);
    if (lane == 0) red[wave] = fro;
    __syncthreads();
    if (threadIdx.x == 0) {
        double f = 0.0;
        for (int w = 0; w < W; ++w) f += red[w];
        if (a.sq) {   // a zero X with eps = 0: scale 0 (X / (||X||_F + eps) -> 0 as eps -> 0+)
            const double d = sqrt(f) + a.eps;
            a.scale[b] = d > 0.0 ? 1.0 / d : 0.0;
        }
        if (rank) rank[a.d_sel] = a.k;
    }
}

// Exclusive prefix count of `flag` over the block in thread order, and the
// block total. Uses wave ballots and one LDS round.
__device__ __forceinline__ int block_excl_prefix(bool flag, int* wave_tot, int& total) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const uint64_t mask = __ballot(flag);
    const int within = __popcll(mask & ((1ull << lane) - 1ull));
    __syncthreads();   // wave_tot may still be read by the previous call
    if (lane == 0) wave_tot[wave] = __popcll(mask);
    __syncthreads();
    int before = 0;
    total = 0;
    for (int w = 0; w < kWaves; ++w) {
        const int t = wave_tot[w];
        before += (w < wave) ? t : 0;
        total += t;
    }
    return before + within;
}

__global__ __launch_bounds__(kThreads) void select_any(SelectArgs a) {
    const int b = blockIdx.x;
    const double* __restrict__ nrm = a.l1 + (int64_t)b * a.d_sel;
    const double* __restrict__ sq = a.sq ? a.sq + (int64_t)b * a.d_sel : nullptr;
    int32_t* __restrict__ out = a.sel + (int64_t)b * a.k;
    int32_t* __restrict__ rank = a.rank ? a.rank + (int64_t)b * (a.d_sel + 1) : nullptr;

    __shared__ unsigned hist[256];
    __shared__ uint64_t s_prefix;
    __shared__ int s_need;
    __shared__ int wave_tot[kWaves];
    __shared__ double red[kWaves];

    auto key_at = [&](int i) { return make_key(a, nrm, b, i); };
    const int lane = threadIdx.x & 63;

    uint64_t prefix = 0, mask = 0;
    int need = a.k;   // how many still to take at or below the current prefix
    for (int shift = 56; shift >= 0; shift -= 8) {
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
        for (int base = 0; base < a.d_sel; base += kThreads) {
            const int i = base + threadIdx.x;
            const uint64_t key = i < a.d_sel ? key_at(i) : 0;
            const bool in = i < a.d_sel && (key & mask) == prefix;
            const unsigned digit = (unsigned)(key >> shift) & 0xffu;
            // one atomic per wave when every candidate lane has the same digit
            const uint64_t cand = __ballot(in);
            if (cand == 0) continue;
            const int first = __builtin_ctzll(cand);
            const unsigned d0 = __shfl(digit, first);
            if (__ballot(in && digit != d0) == 0) {
                if (lane == first) atomicAdd(&hist[d0], (unsigned)__popcll(cand));
            } else if (in) {
                atomicAdd(&hist[digit], 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            // lane l owns bins 4l .. 4l+3; above[l] = count in bins > 4l+3
            unsigned c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = hist[4 * lane + q];
            const unsigned own = c[0] + c[1] + c[2] + c[3];
            unsigned incl = own;   // inclusive suffix sum over lanes >= l
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const unsigned v = __shfl_down(incl, off);
                if (lane + off < 64) incl += v;
            }
            unsigned above = incl - own;
            // the digit is the largest d whose suffix count reaches `need`
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                if (above < (unsigned)need && above + c[q] >= (unsigned)need) {
                    s_prefix = prefix | ((uint64_t)(4 * lane + q) << shift);
                    s_need = need - (int)above;
                }
                above += c[q];
            }
        }
        __syncthreads();
        prefix = s_prefix;
        need = s_need;
        mask |= 0xffull << shift;
    }
    // prefix == T (the k-th largest key); `need` of the keys equal to T go in.
    const uint64_t T = prefix;
    int taken = 0, ties_seen = 0;
    double fro = 0.0;
    for (int base = 0; base < a.d_sel; base += kThreads) {
        const int i = base + threadIdx.x;
        const bool valid = i < a.d_sel;
        const uint64_t key = valid ? key_at(i) : 0;
        const bool eq = valid && key == T;
        int eq_total;
        const int eq_rank = ties_seen + block_excl_prefix(eq, wave_tot, eq_total);
        const bool pick = valid && (key > T || (eq && eq_rank < need));
        int pick_total;
        const int pos = taken + block_excl_prefix(pick, wave_tot, pick_total);
        if (pick) {
            out[pos] = i;
            if (sq) fro += sq[i];
        }
        if (rank && valid) rank[i] = pos;   // selected lines before i
        taken += pick_total;
        ties_seen += eq_total;
    }
    // fixed-order reduction of the selected squared norms
    for (int off = 32; off > 0; off >>= 1) fro += __shfl_xor(fro, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = fro;
    __syncthreads();
    if (threadIdx.x == 0) {
        double f = 0.0;
        for (int w = 0; w < kWaves; ++w) f += red[w];
        if (sq) {   // a zero X with eps = 0: scale 0 (X / (||X||_F + eps) -> 0 as eps -> 0+)
            const double d = sqrt(f) + a.eps;
            a.scale[b] = d > 0.0 ? 1.0 / d : 0.0;
        }
        if (rank) rank[a.d_sel] = a.k;
    }
}

}  // namespace

hipError_t launch_select(const SelectArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.batch);
#define DION2_SELECT(T, R) hipLaunchKernelGGL((select_reg<T, R>), grid, dim3(T), 0, s, a)
    // four waves up to 1024 lines (cheaper barriers), sixteen beyond
    if (a.d_sel <= 256) DION2_SELECT(256, 1);
    else if (a.d_sel <= 512) DION2_SELECT(256, 2);
    else if (a.d_sel <= 1024) DION2_SELECT(256, 4);
    else if (a.d_sel <= 2048) DION2_SELECT(1024, 2);
    else if (a.d_sel <= 4096) DION2_SELECT(1024, 4);
    else if (a.d_sel <= kRegLines) DION2_SELECT(1024, 8);
    else hipLaunchKernelGGL(select_any, grid, dim3(kThreads), 0, s, a);
#undef DION2_SELECT
    return hipGetLastError();
}

}  // namespace dion2
