// K4: the Newton-Schulz GEMMs on MFMA (bf16 operands, fp32 accumulation).
//
// One Newton-Schulz step on the wide compact matrix Z (s x l, s <= l) is
//   A  = Z Z^T                     gemm<1, EPI_H16>, B as rows    A kept as fp16 (scaled)
//   B  = b A + c A^2               gemm<1, EPI_POLY_H16>, B as rows  A^2 = A A^T, one fp16 pass
//   Z' = a Z + B Z                 gemm<1, EPI_UPDATE | EPI_FINAL>, B operand = Z as [K][N]
// The a Z term is added in fp32 in the epilogue rather than folded into the
// diagonal of B: with it separate, lines of Z that are exactly equal stay
// exactly equal through every step (their rows of A, B and Z' come from
// identical inputs), so no rounding noise enters the null space, where the
// polynomial would amplify it by a per step.
//
// C[i][j] = sum_k A[i][k] B[k][j]. The A operand is always given as rows
// with K contiguous. The B operand is given either as rows with K
// contiguous (BT = 0: Z Z^T reads Z twice, A^2 reads A, which is symmetric)
// or as a row-major [K][N] matrix (BT = 1: the update reads Z itself). For
// BT = 1 the MFMA fragments are read with gfx950's transposing LDS read
// (ds_read_b64_tr_b16): a lane of a 16-lane group receives element (i mod 4)
// of the 8 bytes addressed by source lane 4e + i/4 for e = 0..3, so pointing
// source lane s at row s/4, column 4 (s mod 4) hands lane i four
// consecutive K values of column i.
//
// The GRAM form's chain of s x s products runs the same way on bf16 hi / lo
// pairs (three passes), or, as an option, on scaled fp16 matrices with
// v_mfma_f32_32x32x16_f16 (one pass; EPI_H16 and EPI_QPOLY_H16 store fp16).
// For s <= 64 the whole chain is one launch instead (chain_small): one block
// per matrix keeps its s x s matrices in LDS and computes every product as
// the launches would, bitwise.
// With the fp32 master Z itself is a hi / lo pair: the Gram matrix takes
// three passes, and so does the final product, whose [K][N] operand then
// has a lo tile read through the same transposing LDS reads.
//
// Tiling for gfx950: a BM x BN output tile per block of WM x WN wave64s,
// each wave a (BM/WM) x (BN/WN) tile of v_mfma_f32_32x32x16_bf16 blocks.
// K-slices (BK deep) go from global memory straight into an S-stage LDS
// ring with global_load_lds_dwordx4 (each lane's 16 bytes land at the
// wave's LDS base + 16 * lane), S - 1 slices ahead of the MFMAs, so no
// registers stage the operands and a slice's load latency is covered by
// S - 2 slices of compute. Tiles are stored unpadded with an XOR swizzle of
// their 16-byte chunks, chosen so both the fragment reads (ds_read_b128)
// and the transposing reads hit distinct LDS banks; each lane fetches the
// global chunk that belongs in its LDS slot. Tiles are numbered XCD-aware;
// the symmetric products (A and B) compute only the tiles on and above the
// diagonal and write each one twice, so that the stored matrix is exactly
// symmetric. The epilogue goes through a per-wave 32 x 32 LDS tile: each
// lane finishes 16 entries of a row there, and the
// block then leaves in whole row segments (64 bytes of bf16 or 128 bytes of
// fp32 per row), row-major or transposed for the mirrored copy.
//
// All dimensions are multiples of the tile: buffers are padded to 128. An s x s
// matrix (and X along s) is defined, zeros past s, up to the next multiple of
// 64 (of a shared chain's widest member); past it 64-row tiles leave it
// unwritten, so a tile choice may read rows there, which give rows there, but
// no K extent may reach it.
#include <algorithm>
#include <type_traits>

#include "dion2_device.h"

namespace dion2 {
namespace {

constexpr int kXcds = 8;   // accelerator complex dies on MI355X

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;

// two fp32 -> packed bf16 pair (RNE), one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack2(float x, float y) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const bf16x2 v = {(__bf16)x, (__bf16)y};
    return __builtin_bit_cast(uint32_t, v);
}

// two fp32 -> packed fp16 pair (RNE)
__device__ __forceinline__ uint32_t pack2h(float x, float y) {
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    const f16x2 v = {(_Float16)x, (_Float16)y};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float f16_bits_to_f32(uint32_t h) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// One 32 x 32 x 16 MFMA block on bf16 or fp16 fragments.
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(f16x8 a, f16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

template <int NPASS, int BT_, int BM_, int BN_, int BK_, int WM_, int WN_, int S_, bool F16_ = false,
          bool PIPE_ = (BM_ * BN_ > 64 * 128 && !BT_ && !(NPASS == 3 && BM_ == 128))>
struct Tile {
    static constexpr bool PIPE = PIPE_;                  // the k-steps run on over slice ends (see gemm)
    static constexpr int BT = BT_, S = S_;
    static constexpr bool F16 = F16_;                    // fp16 operands (else bf16)
    using Frag = typename std::conditional<F16_, f16x8, bf16x8>::type;
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_;
    static constexpr int WAVES = WM * WN;
    static constexpr int THREADS = 64 * WAVES;
    // waves per SIMD to leave registers for: two blocks of eight waves a CU
    // up to 128 x 128 (a polynomial epilogue is two registers over without)
    static constexpr int MIN_WAVES = WAVES == 8 && BM * BN <= 128 * 128 ? 4 : 1;
    static constexpr int TM = BM / WM, TN = BN / WN;     // wave tile
    static constexpr int FM = TM / 32, FN = TN / 32;     // MFMA blocks per wave
    static constexpr int NA = NPASS == 1 ? 1 : 2;        // A operand tiles (hi[, lo])
    static constexpr int NB = NPASS == 3 ? 2 : 1;        // B operand tiles
    // K-major tiles: rows of BK bf16 (pitch PK bytes), CPR chunks of 16 B
    static constexpr int PK = BK * 2;
    static constexpr int CPR = BK / 8;
    static constexpr int GK = 256 / PK;                  // rows sharing one bank sweep
    // N-major tile (BT = 1): rows of BN bf16 (pitch PN bytes)
    static constexpr int PN = BN * 2;
    static constexpr int A_BYTES = BM * PK;
    static constexpr int B_BYTES = BN * PK;              // same size either layout
    static constexpr int STAGE_BYTES = NA * A_BYTES + NB * B_BYTES;
    static constexpr int STAGE_INSTS = STAGE_BYTES / 1024;   // 1 KB per wave instruction
    static constexpr int IPW = STAGE_INSTS / WAVES;      // load instructions per wave per slice
    static constexpr int EPI_LD = 33;                    // fp32 staging row (32 + 1)
    static constexpr int EPI_BYTES = WAVES * 32 * EPI_LD * 4;
    static constexpr int SMEM = (S * STAGE_BYTES > EPI_BYTES) ? S * STAGE_BYTES : EPI_BYTES;
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile is whole 32x32 blocks");
    static_assert(BK % 16 == 0 && (BK == 32 || BK == 64), "BK of 32 or 64");
    static_assert(A_BYTES % 1024 == 0 && B_BYTES % 1024 == 0, "tiles are whole 1 KB blocks");
    static_assert(STAGE_INSTS % WAVES == 0, "load instructions split evenly over waves");
    static_assert(NPASS >= 1 && NPASS <= 3, "one to three passes");
    static_assert(!BT || BN == 128, "the [K][N] B operand: BN 128");
    static_assert(S >= 2 && S <= 4, "two to four stages");
    static_assert(!F16 || (NPASS == 1 && !BT), "fp16 operands: one pass, B as rows");
};

// Byte offset, inside a K-major tile, of logical 16-byte chunk c of row r.
template <typename T>
__device__ __forceinline__ int kmajor_off(int r, int c) {
    return r * T::PK + 16 * (c ^ ((r / T::GK) % T::CPR));
}
// Byte offset, inside the [BK][BN] tile, of logical 16-byte chunk c of row r.
__device__ __forceinline__ int nmajor_off(int r, int c) {
    return r * 256 + 16 * (c ^ ((r & 3) << 2));
}

// This wave's part of the operands' K-slices. Wave w owns a stage's 1 KB
// blocks w, w + WAVES, ...; lane i of a block fills the block's 16-byte slot
// i with the global chunk that belongs there. A block is some rows of one
// operand tile: its first row's address is uniform and moves on by one slice
// at a time, and a lane's offset from it (row within the block, swizzled
// chunk) is the same for all of a wave's blocks of an operand, so a load in
// the loop costs scalar work alone and two registers hold the offsets.
template <typename T>
struct Loader {
    static constexpr int RA = 1024 / T::PK;                  // rows a block of a K-major tile holds
    static constexpr int RB = T::BT ? 4 : RA;                // ... and of the B tile
    static constexpr int BLK_A = T::A_BYTES / 1024, BLK_B = T::B_BYTES / 1024;   // blocks a tile
    // the chunk swizzle repeats every two blocks, and a wave's are an even number apart
    static_assert(T::WAVES % 2 == 0 && BLK_A % 2 == 0 && BLK_B % 2 == 0, "one offset per operand");
    const unsigned char* base[T::IPW];
    uint32_t off_a, off_b;
    int64_t b_step;   // bytes between slices of the [K][N] B operand (rows: PK)

    __device__ __forceinline__ static bool is_a(int blk) { return blk < T::NA * BLK_A; }
    // a0, a1 (b0, b1): the tile's first row (column) of the operands, in the
    // first slice
    __device__ __forceinline__ void init(const GemmArgs& a, const uint16_t* a0, const uint16_t* a1,
                                         const uint16_t* b0, const uint16_t* b1, int wave, int lane) {
        b_step = T::BT ? (int64_t)T::BK * a.ldb * 2 : T::PK;
        auto kmajor = [&](int ld) {   // a lane's row and chunk in its wave's K-major blocks
            const int lr = lane * 16 / T::PK, slot = lane * 16 % T::PK / 16;
            const int c = slot ^ (((wave * RA + lr) / T::GK) % T::CPR);
            return 2u * ((uint32_t)lr * (uint32_t)ld + c * 8);
        };
        off_a = kmajor(a.lda);
        if constexpr (T::BT) {
            const int lr = lane / 16;
            off_b = 2u * ((uint32_t)lr * (uint32_t)a.ldb + (uint32_t)((lane % 16) ^ (lr << 2)) * 8);
        } else {
            off_b = kmajor(a.ldb);
        }
#pragma unroll
        for (int q = 0; q < T::IPW; ++q) {
            const int blk = wave + q * T::WAVES;   // 1 KB block of the stage (wave-uniform)
            const int in_b = blk - T::NA * BLK_A;
            const uint16_t* p = is_a(blk) ? (blk >= BLK_A ? a1 : a0) : (in_b >= BLK_B ? b1 : b0);
            const int64_t row = is_a(blk) ? (int64_t)(blk % BLK_A) * RA * a.lda : (int64_t)(in_b % BLK_B) * RB * a.ldb;
            base[q] = reinterpret_cast<const unsigned char*>(p + row);
        }
    }
    __device__ __forceinline__ void load(int q, unsigned char* dst, int wave) const {
        const int blk = wave + q * T::WAVES;
        const unsigned char* src = base[q] + (is_a(blk) ? off_a : off_b);
        __builtin_amdgcn_global_load_lds(src, (lds_void*)(dst + blk * 1024), 16, 0, 0);
    }
    __device__ __forceinline__ void advance(int wave) {
#pragma unroll
        for (int q = 0; q < T::IPW; ++q)
            base[q] += !T::BT || is_a(wave + q * T::WAVES) ? (int64_t)T::PK : b_step;
    }
};

// Wait until at most N vector-memory loads of this wave are outstanding
// (vmcnt only; lgkmcnt and expcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The same, and every LDS read of this wave done.
template <int N>
__device__ __forceinline__ void wait_all_lds_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

// B fragment (8 consecutive K of one column) from the [BK][BN] tile through
// two transposing reads; `col` is the fragment's first column.
template <typename T>
__device__ __forceinline__ bf16x8 b_frag_tr(const unsigned char* sb, int krow, int col, int lane) {
    const int g = lane >> 4, s = lane & 15;
    const int row = krow + 8 * (g >> 1) + (s >> 2);
    const int c = col + 16 * (g & 1) + 4 * (s & 3);
    typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4*)(sb + nmajor_off(row, c >> 3) + 2 * (c & 7)));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4*)(sb + nmajor_off(row + 4, c >> 3) + 2 * (c & 7)));
    typedef __attribute__((ext_vector_type(8))) short i16x8;
    const i16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// One k-step's fragments from the slice staged at `st`.
template <int NPASS, typename T>
struct Frags {
    typename T::Frag a0[T::FM], b0[T::FN], a1[T::FM], b1[T::FN];
    __device__ __forceinline__ void read(const unsigned char* st, int kk, int wm, int wn, int lane) {
        const unsigned char* sa0 = st;
        const unsigned char* sa1 = st + T::A_BYTES;
        const unsigned char* sb0 = st + T::NA * T::A_BYTES;
        const unsigned char* sb1 = sb0 + T::B_BYTES;
        const int arow = wm * T::TM + (lane & 31);
        const int brow = wn * T::TN + (lane & 31);
        const int c = 2 * kk + (lane >> 5);   // logical 16-byte chunk of the K-major rows
#pragma unroll
        for (int i = 0; i < T::FM; ++i)
            a0[i] = *reinterpret_cast<const typename T::Frag*>(sa0 + kmajor_off<T>(arow + i * 32, c));
#pragma unroll
        for (int j = 0; j < T::FN; ++j) {
            if constexpr (T::BT) b0[j] = b_frag_tr<T>(sb0, kk * 16, wn * T::TN + j * 32, lane);
            else b0[j] = *reinterpret_cast<const typename T::Frag*>(sb0 + kmajor_off<T>(brow + j * 32, c));
        }
        if constexpr (NPASS >= 2) {
#pragma unroll
            for (int i = 0; i < T::FM; ++i)
                a1[i] = *reinterpret_cast<const typename T::Frag*>(sa1 + kmajor_off<T>(arow + i * 32, c));
        }
        if constexpr (NPASS == 3) {
#pragma unroll
            for (int j = 0; j < T::FN; ++j) {
                if constexpr (T::BT) b1[j] = b_frag_tr<T>(sb1, kk * 16, wn * T::TN + j * 32, lane);
                else b1[j] = *reinterpret_cast<const typename T::Frag*>(sb1 + kmajor_off<T>(brow + j * 32, c));
            }
        }
    }
};

// One k-step's MFMAs. With OVER > 0 the loads of a slice are spread over OVER
// MFMAs, of which this step's are M0, M0 + 1, ...; each is fenced in place:
// issued in one burst ahead of the MFMAs they hold the wave in the
// vector-memory issue queue while its matrix pipe idles.
template <int NPASS, typename T, int OVER, int M0>
__device__ __forceinline__ void mma_step(f32x16 (&acc)[T::FM][T::FN], const Frags<NPASS, T>& f, const Loader<T>& ld,
                                         unsigned char* dst, int wave) {
    int m = M0;
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j)
#pragma unroll
            for (int p = 0; p < NPASS; ++p) {
                // per block: hi*lo, lo*hi, then hi*hi (the order of the sums)
                if (NPASS == 3 && p == 0) acc[i][j] = mfma32(f.a0[i], f.b1[j], acc[i][j]);
                else if (NPASS >= 2 && p == NPASS - 2) acc[i][j] = mfma32(f.a1[i], f.b0[j], acc[i][j]);
                else acc[i][j] = mfma32(f.a0[i], f.b0[j], acc[i][j]);
                if constexpr (OVER > 0) {
#pragma unroll
                    for (int q = 0; q < T::IPW; ++q) {
                        if (q * OVER / T::IPW == m) {
                            __builtin_amdgcn_sched_barrier(0);
                            ld.load(q, dst, wave);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
                ++m;
            }
}

// Store a wave's finished 32 x 32 block from its LDS tile (fp32, row pitch
// EPI_LD) to output rows orow0 .. orow0 + 31, columns ocol0 .. ocol0 + 31, in
// the epilogue's output form. Lanes take whole row segments: for bf16
// outputs four lanes cover a row's 64 bytes (16 rows per instruction), for
// fp32 eight lanes its 128 bytes, so every store instruction writes
// contiguous segments of few cache lines. With TR the tile is read
// transposed (output row q = tile column q), for the mirrored block; with
// DIAG (a block on the diagonal of a symmetric product) the entries below
// the diagonal are taken from their mirror images above it. O1 sends a bf16
// block to out1 instead of out0 (EPI_UPDATE's transposed copy).
template <int EPI, typename T, bool TR, bool DIAG = false, bool O1 = false>
__device__ __forceinline__ void store_block(const GemmArgs& a, int b, const float* stage, int64_t orow0,
                                            int64_t ocol0, int lane) {
    auto at = [&](int r, int c) {
        if (DIAG && c < r) return stage[c * T::EPI_LD + r];
        return TR ? stage[c * T::EPI_LD + r] : stage[r * T::EPI_LD + c];
    };
    if constexpr (EPI == EPI_FINAL) {
        const int c4 = 4 * (lane & 7);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 8 * q + (lane >> 3);
            float* op = static_cast<float*>(a.out0) + (int64_t)b * a.sOut0 + (orow0 + r) * a.ldo0 + ocol0 + c4;
            *reinterpret_cast<float4*>(op) = make_float4(at(r, c4), at(r, c4 + 1), at(r, c4 + 2), at(r, c4 + 3));
        }
    } else {
        const int c8 = 8 * (lane & 3);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = 16 * q + (lane >> 2);
            float v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = at(r, c8 + t);
            if constexpr (EPI == EPI_SPLIT || EPI == EPI_QPOLY) {
                uint32_t h[4], l[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint16_t h0 = f32_to_bf16(v[2 * t]), h1 = f32_to_bf16(v[2 * t + 1]);
                    h[t] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                    l[t] = pack2(v[2 * t] - bf16_bits_to_f32(h0), v[2 * t + 1] - bf16_bits_to_f32(h1));
                }
                uint16_t* hp = static_cast<uint16_t*>(a.out0) + (int64_t)b * a.sOut0 + (orow0 + r) * a.ldo0 + ocol0 + c8;
                uint16_t* lp = static_cast<uint16_t*>(a.out1) + (int64_t)b * a.sOut1 + (orow0 + r) * a.ldo1 + ocol0 + c8;
                *reinterpret_cast<uint4*>(hp) = make_uint4(h[0], h[1], h[2], h[3]);
                *reinterpret_cast<uint4*>(lp) = make_uint4(l[0], l[1], l[2], l[3]);
            } else if constexpr (EPI == EPI_H16 || EPI == EPI_QPOLY_H16) {
                uint16_t* op = static_cast<uint16_t*>(a.out0) + (int64_t)b * a.sOut0 + (orow0 + r) * a.ldo0 + ocol0 + c8;
                *reinterpret_cast<uint4*>(op) = make_uint4(pack2h(v[0], v[1]), pack2h(v[2], v[3]),
                                                           pack2h(v[4], v[5]), pack2h(v[6], v[7]));
            } else if constexpr (O1) {   // EPI_UPDATE's transposed copy: bf16
                uint16_t* op = static_cast<uint16_t*>(a.out1) + (int64_t)b * a.sOut1 + (orow0 + r) * a.ldo1 + ocol0 + c8;
                *reinterpret_cast<uint4*>(op) = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]),
                                                           pack2(v[4], v[5]), pack2(v[6], v[7]));
            } else {   // EPI_POLY, EPI_UPDATE: bf16
                uint16_t* op = static_cast<uint16_t*>(a.out0) + (int64_t)b * a.sOut0 + (orow0 + r) * a.ldo0 + ocol0 + c8;
                *reinterpret_cast<uint4*>(op) = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]),
                                                           pack2(v[4], v[5]), pack2(v[6], v[7]));
            }
        }
    }
}

template <int NPASS, int EPI, typename T, bool SYM>
__global__ __launch_bounds__(T::THREADS, T::MIN_WAVES) void gemm(GemmArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[T::SMEM];

    // XCD-aware tile order. Workgroups are dispatched round-robin over the
    // eight XCDs, each with its own L2; renumbering puts consecutive tiles --
    // the tiles of one matrix, which share its operands -- on one XCD, so a
    // matrix's compact operands are fetched into one L2 instead of eight.
    const int nx = gridDim.x, ny = gridDim.y;
    const int total = nx * ny * gridDim.z;
    const int hw = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    const int logical = (total % kXcds == 0) ? (hw % kXcds) * (total / kXcds) + hw / kXcds : hw;
    int b = logical / (nx * ny);
    int part = 0;
    if constexpr (EPI == EPI_PART) {   // z runs over (matrix, part of K)
        part = b % a.ksplit;
        b /= a.ksplit;
    }
    if (a.dual) {
        // matrix b's two products are neighbours in the tile order, so the
        // shared A operand is fetched into one L2 for both
        if (b & 1) {
            a.B0 = a.B0x;
            a.B1 = a.B1x;
            a.out0 = a.out0x;
            a.out1 = a.out1x;
            a.oexp = a.oexpx;
        }
        b >>= 1;
    }
    // Within a matrix the tiles run down each column strip first: the ny
    // tiles that read one strip of the B operand are dispatched together, so
    // the strip is fetched into L2 once, while the A operand (the s x s
    // factor, the smaller one) stays resident across strips.
    int row0 = (logical % ny) * T::BM;          // output rows (M)
    int col0 = ((logical / ny) % nx) * T::BN;   // output cols (N)
    if constexpr (SYM) {
        // symmetric output: x enumerates the upper-triangle tiles I <= J
        // row by row; each is written at (I, J) and mirrored to (J, I)
        const int tiles = a.M / T::BM;
        int rem = logical % nx, I = 0;
        while (rem >= tiles - I) {
            rem -= tiles - I;
            ++I;
        }
        row0 = I * T::BM;
        col0 = (I + rem) * T::BN;
    }
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wave
    const int wm = wave / T::WN, wn = wave % T::WN;

    const uint16_t* abase0 = a.A0 + (int64_t)b * a.sA + (int64_t)row0 * a.lda;
    const uint16_t* abase1 = NPASS >= 2 ? a.A1 + (int64_t)b * a.sA + (int64_t)row0 * a.lda : abase0;
    const int64_t bo = (int64_t)b * a.sB + (T::BT ? (int64_t)col0 : (int64_t)col0 * a.ldb);
    const uint16_t* bbase0 = a.B0 + bo;
    const uint16_t* bbase1 = NPASS == 3 ? a.B1 + bo : bbase0;

    // Epilogue operands (Z for a Z, or A's hi / lo for the polynomial) are
    // fetched first so their latency hides behind the main loop.
    const int er = lane >> 1;          // epilogue: row (or transposed row) of this lane
    const int ec = (lane & 1) * 16;    // epilogue: 16 consecutive columns
    constexpr bool kPreE0 = EPI == EPI_POLY || EPI == EPI_QPOLY || EPI == EPI_UPDATE || EPI == EPI_FINAL ||
                            EPI == EPI_APPLY || EPI == EPI_APPLY_F32 || EPI == EPI_QPOLY_H16 || EPI == EPI_POLY_H16;
    constexpr bool kPreE1 = EPI == EPI_POLY || EPI == EPI_QPOLY;
    const bool pre = kPreE0 && a.E0 != nullptr && !(EPI == EPI_FINAL && a.out_transposed);
    uint4 e0[T::FM][T::FN][2], e1[T::FM][T::FN][2];
    if (pre) {
#pragma unroll
        for (int i = 0; i < T::FM; ++i)
#pragma unroll
            for (int j = 0; j < T::FN; ++j) {
                const int64_t eo = (int64_t)b * a.sE + (int64_t)(row0 + wm * T::TM + i * 32 + er) * a.lde +
                                   col0 + wn * T::TN + j * 32 + ec;
                e0[i][j][0] = reinterpret_cast<const uint4*>(a.E0 + eo)[0];
                e0[i][j][1] = reinterpret_cast<const uint4*>(a.E0 + eo)[1];
                if constexpr (kPreE1) {
                    e1[i][j][0] = reinterpret_cast<const uint4*>(a.E1 + eo)[0];
                    e1[i][j][1] = reinterpret_cast<const uint4*>(a.E1 + eo)[1];
                }
            }
    }

    // EPI_APPLY: the W entries this lane updates (16 consecutive entries per
    // block, row K[p] of W) are fetched before the main loop as well.
    // Addresses are clamped into W so the loads are unconditional; the
    // epilogue uses them only where they are the right entries.
    int32_t wrow[T::FM];
    constexpr bool kApply = EPI == EPI_APPLY || EPI == EPI_APPLY_F32;
    typedef typename std::conditional<EPI == EPI_APPLY_F32, float, uint16_t>::type WT;
    constexpr int kWQ = 16 * sizeof(WT) / sizeof(uint4);   // 16-byte pieces of 16 entries
    uint4 wv[T::FM][T::FN][kWQ];
    if constexpr (kApply) {
        const WT* W = a.ms.w<WT>(b);
#pragma unroll
        for (int i = 0; i < T::FM; ++i) {
            const int p = row0 + wm * T::TM + i * 32 + er;
            wrow[i] = ldg<int32_t>(a.sel + (int64_t)b * a.k + (p < a.k ? p : a.k - 1));
#pragma unroll
            for (int j = 0; j < T::FN; ++j) {
                int64_t jc = col0 + wn * T::TN + j * 32 + ec;
                jc = jc + 16 <= a.cols ? jc : a.cols - 16;
                const WT* src = W + (int64_t)wrow[i] * a.cols + jc;
#pragma unroll
                for (int q = 0; q < kWQ; ++q) wv[i][j][q] = ldg<uint4>(src + q * (16 / kWQ));
            }
        }
    }

    f32x16 acc[T::FM][T::FN];
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // S-stage ring. Plain loop: slices 0..S-2 in flight before the first MFMA;
    // at iteration kt slice kt+S-1 is requested into the stage freed by kt-1.
    // Run-on loop (PIPE): a slice's last k-step reads the next slice's first
    // fragments, so the barrier between them stands among MFMAs already
    // queued instead of ahead of idle ones; once a wave holds the last
    // fragments of slice kt its stage is free, so S slices are in flight.
    // Requests past the last slice re-read it (in bounds) so every iteration
    // issues the same number of loads and the vmcnt wait stays exact.
    // (16 x 8192 x 2048 at alpha 0.5: 3371 -> 3313 us a step.)
    int nk = a.K / T::BK;
    if constexpr (EPI == EPI_PART) {
        // this part's slices: the parts' lengths differ by at most one slice
        const int k0 = nk * part / a.ksplit;
        nk = nk * (part + 1) / a.ksplit - k0;
        abase0 += (int64_t)k0 * T::BK;
        abase1 += (int64_t)k0 * T::BK;
        bbase0 += (int64_t)k0 * T::BK;
        bbase1 += (int64_t)k0 * T::BK;
    }
    Loader<T> ld;
    ld.init(a, abase0, abase1, bbase0, bbase1, wave, lane);
    constexpr int KK = T::BK / 16;
    constexpr int NMFMA = T::FM * T::FN * NPASS;   // MFMAs per k-step
    Frags<NPASS, T> f[2];
    constexpr int AHEAD = T::PIPE ? T::S : T::S - 1;
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
#pragma unroll
        for (int q = 0; q < T::IPW; ++q) ld.load(q, smem_raw + p * T::STAGE_BYTES, wave);
        if (p + 1 < nk) ld.advance(wave);
    }
    if constexpr (T::PIPE) {
        wait_vmcnt<(T::S - 1) * T::IPW>();   // slice 0
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        f[0].read(smem_raw, 0, wm, wn, lane);
        for (int kt = 0; kt < nk; ++kt) {
            unsigned char* st = smem_raw + (kt % T::S) * T::STAGE_BYTES;
            const unsigned char* nx_st = smem_raw + ((kt + 1) % T::S) * T::STAGE_BYTES;
#pragma unroll
            for (int kk = 0; kk < KK - 1; ++kk) {
                f[(kk + 1) & 1].read(st, kk + 1, wm, wn, lane);
                mma_step<NPASS, T, 0, 0>(acc, f[kk & 1], ld, st, wave);
            }
            // slice kt's last fragments are in registers and this wave's part of
            // slice kt+1 has landed; behind the barrier that holds for all waves
            __builtin_amdgcn_sched_barrier(0);
            wait_all_lds_vmcnt<(T::S - 2) * T::IPW>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            f[0].read(nx_st, 0, wm, wn, lane);
            mma_step<NPASS, T, NMFMA, 0>(acc, f[(KK - 1) & 1], ld, st, wave);
            if (kt + T::S + 1 < nk) ld.advance(wave);
        }
    } else {
        for (int kt = 0; kt < nk; ++kt) {
            // This wave's part of slice kt has landed; the bare barrier then makes
            // every wave's part visible and frees stage kt-1 (its fragments were
            // consumed by MFMAs issued before the barrier). A full __syncthreads
            // would also drain the loads of the slices in flight behind kt.
            wait_vmcnt<(T::S - 2) * T::IPW>();
            __builtin_amdgcn_s_barrier();
            const unsigned char* st = smem_raw + (kt % T::S) * T::STAGE_BYTES;
            unsigned char* ldst = smem_raw + ((kt + T::S - 1) % T::S) * T::STAGE_BYTES;
            f[0].read(st, 0, wm, wn, lane);
            static_assert(KK == 2 || KK == 4, "two or four k-steps a slice");
            f[1].read(st, 1, wm, wn, lane);
            mma_step<NPASS, T, NMFMA * KK, 0>(acc, f[0], ld, ldst, wave);
            if constexpr (KK == 4) {
                f[0].read(st, 2, wm, wn, lane);
                mma_step<NPASS, T, NMFMA * KK, NMFMA>(acc, f[1], ld, ldst, wave);
                f[1].read(st, 3, wm, wn, lane);
                mma_step<NPASS, T, NMFMA * KK, 2 * NMFMA>(acc, f[0], ld, ldst, wave);
            }
            mma_step<NPASS, T, NMFMA * KK, (KK - 1) * NMFMA>(acc, f[1], ld, ldst, wave);
            if (kt + T::S < nk) ld.advance(wave);
        }
    }
    wait_vmcnt<0>();   // no load may land in the ring once the epilogue reuses it
    __syncthreads();

    if constexpr (EPI == EPI_PART) {
        // the accumulators as they are, in register order (16 bytes a lane,
        // 1 KB an instruction); reduce_parts reads them back the same way
        const int tiles = nx;
        const int tile = logical % nx;
        float* out = a.part + (((int64_t)b * a.ksplit + part) * tiles + tile) * (T::BM * T::BN);
#pragma unroll
        for (int i = 0; i < T::FM; ++i)
#pragma unroll
            for (int j = 0; j < T::FN; ++j) {
                const int blk = (wm * T::FM + i) * (T::BN / 32) + wn * T::FN + j;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    stg(out + blk * 1024 + q * 256 + lane * 4,
                        make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]));
            }
        return;
    }

    // ---- epilogue, one 32 x 32 block at a time through a per-wave LDS tile.
    // The tile belongs to its wave alone and LDS accesses of one wave complete
    // in issue order, so wave barriers order the staging.
    float* stage = reinterpret_cast<float*>(smem_raw) + wave * 32 * T::EPI_LD;
    // the fp16 chain's products carry power-of-two scales (exact)
    constexpr bool kScaled = T::F16 || EPI == EPI_H16;
    const float osc = kScaled ? __builtin_amdgcn_ldexpf(1.0f, a.oexp) : 1.0f;
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
#pragma unroll
        for (int j = 0; j < T::FN; ++j) {
            const int R = row0 + wm * T::TM + i * 32;   // block origin in the output
            const int Cc = col0 + wn * T::TN + j * 32;
            // A symmetric product is stored exactly symmetric: blocks above
            // the diagonal are written twice, blocks on it from their upper
            // triangle, and blocks below it (in diagonal tiles) not at all.
            // Rounding leaves the computed product slightly asymmetric;
            // carried along, that asymmetry feeds the Gram chain's unstable
            // directions.
            if (SYM && R > Cc) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                stage[m * T::EPI_LD + (lane & 31)] = kScaled ? acc[i][j][r] * osc : acc[i][j][r];
            }
            __builtin_amdgcn_wave_barrier();
            if constexpr (EPI == EPI_SPLIT || EPI == EPI_H16) {
                // no arithmetic after the accumulators: they leave the tile as staged
                if (SYM && R == Cc) {
                    store_block<EPI, T, false, true>(a, b, stage, (int64_t)R, (int64_t)Cc, lane);
                } else {
                    store_block<EPI, T, false>(a, b, stage, (int64_t)R, (int64_t)Cc, lane);
                    if (SYM) store_block<EPI, T, true>(a, b, stage, (int64_t)Cc, (int64_t)R, lane);
                }
                __builtin_amdgcn_wave_barrier();   // the stage tile is rewritten next
                continue;
            }
            float v[16];
            const bool transposed = EPI == EPI_FINAL && a.out_transposed;
            if (!transposed) {
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = stage[er * T::EPI_LD + ec + q];
            } else {
                // output row = block column er, 16 consecutive block rows
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = stage[(ec + q) * T::EPI_LD + er];
            }
            const int64_t orow = transposed ? Cc + er : R + er;
            const int64_t ocol = transposed ? R + ec : Cc + ec;
            if constexpr (EPI == EPI_UPDATE || EPI == EPI_FINAL || kApply) {
                // + a Z at this lane's 16 entries (none when E0 is null)
                if (pre) {
                    const uint4 z0 = e0[i][j][0];
                    const uint4 z1 = e0[i][j][1];
                    const uint32_t zw[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        v[2 * q] += a.ca * bf16_bits_to_f32(zw[q] & 0xffffu);
                        v[2 * q + 1] += a.ca * bf16_bits_to_f32(zw[q] >> 16);
                    }
                } else if (transposed && a.E0) {
                    // transposed output: entry q is Z[R + ec + q][Cc + er]
                    const uint16_t* zp = a.E0 + (int64_t)b * a.sE + (int64_t)(R + ec) * a.lde + Cc + er;
#pragma unroll
                    for (int q = 0; q < 16; ++q) v[q] += a.ca * bf16_bits_to_f32(zp[(int64_t)q * a.lde]);
                }
            } else if constexpr (EPI == EPI_POLY || EPI == EPI_QPOLY) {
                // b (A_hi + A_lo) + c A^2 [+ a I]
                const uint4 h0 = e0[i][j][0];
                const uint4 h1 = e0[i][j][1];
                const uint4 l0 = e1[i][j][0];
                const uint4 l1 = e1[i][j][1];
                const uint32_t hw[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
                const uint32_t lw[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float a0 = bf16_bits_to_f32(hw[q] & 0xffffu) + bf16_bits_to_f32(lw[q] & 0xffffu);
                    const float a1 = bf16_bits_to_f32(hw[q] >> 16) + bf16_bits_to_f32(lw[q] >> 16);
                    v[2 * q] = a.cb * a0 + a.cc * v[2 * q];
                    v[2 * q + 1] = a.cb * a1 + a.cc * v[2 * q + 1];
                }
                if constexpr (EPI == EPI_QPOLY) {
                    // entry (R + er, Cc + ec + q) is on the diagonal iff er == ec + q
                    if (R == Cc) {
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (er == ec + q) v[q] += a.ca;
                    }
                }
            } else if constexpr (EPI == EPI_QPOLY_H16 || EPI == EPI_POLY_H16) {
                // b A + c A^2 from the fp16 A (scale 2^eexp back to A); the
                // chain's Q adds a I and is stored as fp16(2^sexp Q)
                const float esc = __builtin_amdgcn_ldexpf(1.0f, a.eexp);
                const uint4 h0 = e0[i][j][0];
                const uint4 h1 = e0[i][j][1];
                const uint32_t hw[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    v[2 * q] = a.cb * (esc * f16_bits_to_f32(hw[q] & 0xffffu)) + a.cc * v[2 * q];
                    v[2 * q + 1] = a.cb * (esc * f16_bits_to_f32(hw[q] >> 16)) + a.cc * v[2 * q + 1];
                }
                if constexpr (EPI == EPI_QPOLY_H16) {
                    const float ssc = __builtin_amdgcn_ldexpf(1.0f, a.sexp);
                    if (R == Cc) {
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (er == ec + q) v[q] += a.ca;
                    }
#pragma unroll
                    for (int q = 0; q < 16; ++q) v[q] *= ssc;
                }
            }
            if constexpr (kApply) {
                // W[K[p]][j] <- round(W[K[p]][j] - lr_eff O[p][j]) (update step, eq. (1))
                if (orow < a.k) {
                    WT* w = a.ms.w<WT>(b) + (int64_t)wrow[i] * a.cols + ocol;
                    auto step = [&](float x, float o) { return __dsub_rn((double)x, __dmul_rn(a.lr_eff, (double)o)); };
                    if (ocol + 16 <= a.d_oth) {
#pragma unroll
                        for (int q = 0; q < kWQ; ++q) {
                            const uint32_t ww[4] = {wv[i][j][q].x, wv[i][j][q].y, wv[i][j][q].z, wv[i][j][q].w};
                            uint32_t o[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                if constexpr (sizeof(WT) == 2) {
                                    const int e = 8 * q + 2 * u;
                                    o[u] = (uint32_t)f64_to_bf16(step(bf16_bits_to_f32(ww[u] & 0xffffu), v[e])) |
                                           ((uint32_t)f64_to_bf16(step(bf16_bits_to_f32(ww[u] >> 16), v[e + 1])) << 16);
                                } else {
                                    o[u] = __float_as_uint((float)step(__uint_as_float(ww[u]), v[4 * q + u]));
                                }
                            }
                            stg(w + q * (16 / kWQ), make_uint4(o[0], o[1], o[2], o[3]));
                        }
                    } else if (ocol < a.d_oth) {
                        // the row's last entries: all loaded before the first store
                        float x[16];
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (ocol + q < a.d_oth) x[q] = Elem<WT>::load(w + q);
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (ocol + q < a.d_oth) Elem<WT>::store_f64(w + q, step(x[q], v[q]));
                    }
                    if (a.dbg) {
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (ocol + q < a.d_oth) a.dbg[((int64_t)b * a.k + orow) * a.d_oth + ocol + q] = v[q];
                    }
                }
            } else {
                // the finished values go back to the tile (this lane's own
                // entries) and leave it in whole row segments
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < 16; ++q) stage[er * T::EPI_LD + ec + q] = v[q];
                __builtin_amdgcn_wave_barrier();
                if (SYM && R == Cc) {
                    store_block<EPI, T, false, true>(a, b, stage, orow - er, ocol - ec, lane);
                } else {
                    store_block<EPI, T, false>(a, b, stage, orow - er, ocol - ec, lane);
                    if (SYM) store_block<EPI, T, true>(a, b, stage, (int64_t)Cc, (int64_t)R, lane);
                }
                if constexpr (EPI == EPI_UPDATE) {
                    // X' also as X'^T, the next step's B operand given as rows
                    if (a.out1) store_block<EPI, T, true, false, true>(a, b, stage, (int64_t)Cc, (int64_t)R, lane);
                }
            }
            __builtin_amdgcn_wave_barrier();   // the stage tile is rewritten next
        }
    }
}

// C = the sum over the parts of K, in their order, of a product computed by
// EPI_PART launches, in EPI's output form and exactly symmetric, as gemm's
// own epilogue stores it. A wave takes one 32 x 32 block of a tile; blocks
// below the diagonal are the mirrors of others, tiles past the side that the
// parts cover (a.M) are zeros out to a.mfill. Bound by latency: a launch
// of few tiles has a few MB of partials, which its own loads fetch at once.
template <int EPI, typename T>
__global__ __launch_bounds__(256) void reduce_parts(GemmArgs a) {
    __shared__ float smem[4 * 32 * T::EPI_LD];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int PER = (T::BM / 32) * (T::BN / 32);   // blocks of a tile
    static_assert(PER % 4 == 0, "a block of four waves stays inside one tile");
    const int tiles = a.mfill / T::BM;                    // written, a side
    const int ntile = tiles * (tiles + 1) / 2;
    const int ptiles = a.M / T::BM;                       // of which there are parts
    const int nptile = ptiles * (ptiles + 1) / 2;
    const int64_t w = (int64_t)blockIdx.x * 4 + wave;
    const int blk = (int)(w % PER);
    const int tile = (int)(w / PER % ntile);
    const int b = (int)(w / PER / ntile);
    int rem = tile, I = 0;
    while (rem >= tiles - I) {
        rem -= tiles - I;
        ++I;
    }
    const int R = I * T::BM + 32 * (blk / (T::BN / 32));
    const int C = (I + rem) * T::BN + 32 * (blk % (T::BN / 32));
    if (R > C) return;   // whole wave; no block barrier follows
    const int ptile = I * ptiles - I * (I - 1) / 2 + rem;   // the tile's place among the parts'
    const float* in = a.part + ((int64_t)b * a.ksplit * nptile + ptile) * (T::BM * T::BN) + blk * 1024 + lane * 4;
    const int64_t step = (int64_t)nptile * (T::BM * T::BN);
    const int nparts = I + rem < ptiles ? a.ksplit : 0;
    float v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = 0.f;
    int p = 0;
    for (; p + 4 <= nparts; p += 4) {   // sixteen loads in flight
        float4 x[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) x[u][q] = ldg<float4>(in + (p + u) * step + q * 256);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[4 * q] += x[u][q].x;
                v[4 * q + 1] += x[u][q].y;
                v[4 * q + 2] += x[u][q].z;
                v[4 * q + 3] += x[u][q].w;
            }
    }
    for (; p < nparts; ++p) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = ldg<float4>(in + p * step + q * 256);
            v[4 * q] += x.x;
            v[4 * q + 1] += x.y;
            v[4 * q + 2] += x.z;
            v[4 * q + 3] += x.w;
        }
    }
    const float osc = EPI == EPI_H16 ? __builtin_amdgcn_ldexpf(1.0f, a.oexp) : 1.0f;
    float* stage = smem + wave * 32 * T::EPI_LD;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        stage[m * T::EPI_LD + (lane & 31)] = EPI == EPI_H16 ? v[r] * osc : v[r];
    }
    __builtin_amdgcn_wave_barrier();   // LDS accesses of one wave complete in issue order
    if (R == C) {
        store_block<EPI, T, false, true>(a, b, stage, (int64_t)R, (int64_t)C, lane);
    } else {
        store_block<EPI, T, false>(a, b, stage, (int64_t)R, (int64_t)C, lane);
        store_block<EPI, T, true>(a, b, stage, (int64_t)C, (int64_t)R, lane);
    }
}

// ---- the GRAM chain of a compact matrix with s <= 64, in one block
//
// The s x s matrices stay in LDS as bf16 hi / lo pairs, four hi and their four
// lo entries side by side (16 bytes: what a lane reads or writes at once), in
// 64 rows of 272 bytes (the 16-byte pieces of 16 rows fall on
// distinct banks). Every product is the one the launch-per-product chain
// makes: per 16-deep k-step hi*lo, lo*hi, then hi*hi into fp32
// accumulators, the same epilogue arithmetic and hi / lo split, and exactly
// symmetric storage (entries on and above the diagonal computed, mirrored
// below it). The MFMAs are v_mfma_f32_16x16x16_bf16, whose sums equal those of
// v_mfma_f32_32x32x16_bf16 bit for bit. Entries past s_k are never read.
//
// Bound by latency: fourteen dependent stages of one to two products, each a
// chain of 12 dependent MFMAs between LDS reads and writes. So a wave takes
// one 16 x 16 block of a stage's products (ten waves for s = 64: a chain step
// of 16 cycles instead of 64, and a quarter of a 32 x 32 block's conversions
// and stores), a stage's two products share x and interleave, and the code is
// one stage's (a second copy would be fetched cold into the instruction cache
// of a kernel that runs once). Five steps at s = 64: 28.0 us with copies of
// the code on 32 x 32 blocks, 16.2 with one copy, 12.9 now (s = 32: 7.7).
constexpr int kSmallPitch = 2 * kSmallChainS + 8;
constexpr int kSmallMat = kSmallChainS * kSmallPitch;
enum { SM_A, SM_Q, SM_T, SM_P, SM_COUNT = SM_P + 2 };   // P twice

// where entry (r, c)'s hi half lies; its lo half is 4 further on
__device__ __forceinline__ constexpr int small_at(int r, int c) { return r * kSmallPitch + (c >> 2) * 8 + (c & 3); }

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mfma16(i16x4 a, i16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

template <int KS>
__global__ __launch_bounds__(64 * (KS / 16) * (KS / 16 + 1) / 2) void chain_small(SmallChainArgs a) {
    constexpr int NK = KS / 16;                       // k-steps, and blocks a side
    constexpr int THREADS = 64 * NK * (NK + 1) / 2;   // a wave per block on or above the diagonal
    __shared__ __attribute__((aligned(16))) uint16_t pl[SM_COUNT * kSmallMat];
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t s2 = a.s_pad * a.s_pad;
    constexpr int kChunks = KS * (KS / 8);   // 8 entries of [0, KS)^2
    for (int i = tid; i < kChunks; i += THREADS) {
        const int r = i / (KS / 8), c = 8 * (i % (KS / 8));
        const int64_t at = (int64_t)b * s2 + (int64_t)r * a.s_pad + c;
        const uint4 h = ldg<uint4>(a.Ah + at), l = ldg<uint4>(a.Al + at);
        uint16_t* o = pl + SM_A * kSmallMat + small_at(r, c);
        *reinterpret_cast<uint4*>(o) = make_uint4(h.x, h.y, l.x, l.y);
        *reinterpret_cast<uint4*>(o + 8) = make_uint4(h.z, h.w, l.z, l.w);
    }
    // this wave's block: rows 16 bi, columns 16 bj, bi <= bj
    int bi = 0, bj = wave;
    while (bj >= NK - bi) {
        bj -= NK - bi;
        ++bi;
    }
    bj += bi;
    // A lane's fragments: 4 consecutive k of row lane & 15 of the block's rows
    // of x (columns: rows of y); its results: entries (m .. m + 3, n), stored
    // as 8 bytes of row n (the mirror) and one by one in column n. On the
    // diagonal the mirror is stored whole and the entries above the diagonal
    // over it; those on or below go to the row's padding instead.
    const int xat = small_at(16 * bi + (lane & 15), 4 * (lane >> 4));
    const int yat = small_at(16 * bj + (lane & 15), 4 * (lane >> 4));
    const int m = 16 * bi + 4 * (lane >> 4), n = 16 * bj + (lane & 15);
    const int mirror = small_at(n, m);
    int direct[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) direct[u] = m + u < n ? small_at(m + u, n) : small_at(n, kSmallChainS);

    struct Pair {
        i16x4 h, l;
    };
    Pair x[NK];
    auto read = [&](int mat, int at, Pair (&f)[NK]) {
#pragma unroll
        for (int k = 0; k < NK; ++k)
            f[k] = __builtin_bit_cast(Pair, *reinterpret_cast<const uint4*>(pl + mat * kSmallMat + at + 32 * k));
    };
    auto store = [&](int mat, const f32x4& v) {
        uint16_t* o = pl + mat * kSmallMat;
        const uint2 h = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        float hf[4];
        unpack4(h, hf);
        const uint2 l = make_uint2(pack2(v[0] - hf[0], v[1] - hf[1]), pack2(v[2] - hf[2], v[3] - hf[3]));
        *reinterpret_cast<uint4*>(o + mirror) = make_uint4(h.x, h.y, l.x, l.y);
        __builtin_amdgcn_wave_barrier();   // LDS accesses of one wave complete in issue order
        const uint32_t hw[2] = {h.x, h.y}, lw[2] = {l.x, l.y};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            o[direct[u]] = (uint16_t)(hw[u >> 1] >> (16 * (u & 1)));
            o[direct[u] + 4] = (uint16_t)(lw[u >> 1] >> (16 * (u & 1)));
        }
    };
    __syncthreads();
    int cur = 0;
    // per step: Q_t (the first one is P itself); T = Q_t A (t < T - 1) and
    // P <- Q_t P (t > 0); A <- Q_t T (t < T - 1)
    for (int t = 0; t < a.ns_steps; ++t) {
        const float ca = a.cf[t][0], cb = a.cf[t][1], cc = a.cf[t][2];
        const bool do_p = t > 0, do_t = t + 1 < a.ns_steps;
        const int q = t == 0 ? SM_P : SM_Q;
        const int pin = SM_P + cur, pout = SM_P + 1 - cur;
        const int stages = do_t ? 3 : 2;
#pragma unroll 1
        for (int stage = 0; stage < stages; ++stage) {
            const bool poly = stage == 0, two = stage == 1 && do_p && do_t;
            const int y0 = stage == 2 ? SM_T : stage == 1 && !do_t ? pin : SM_A;
            const int d0 = stage == 0 ? q : stage == 2 ? SM_A : do_t ? SM_T : pout;
            if (stage < 2) read(stage == 0 ? SM_A : q, xat, x);   // the third stage's x is the second's
            Pair y[NK];
            read(y0, yat, y);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            if (two) {
                Pair z[NK];
                read(pin, yat, z);
                f32x4 acp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    acc = mfma16(x[k].h, y[k].l, acc);
                    acp = mfma16(x[k].h, z[k].l, acp);
                    acc = mfma16(x[k].l, y[k].h, acc);
                    acp = mfma16(x[k].l, z[k].h, acp);
                    acc = mfma16(x[k].h, y[k].h, acc);
                    acp = mfma16(x[k].h, z[k].h, acp);
                }
                store(pout, acp);
            } else {
                uint4 e;   // A at this lane's entries (it is symmetric)
                if (poly) e = *reinterpret_cast<const uint4*>(pl + SM_A * kSmallMat + mirror);
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    acc = mfma16(x[k].h, y[k].l, acc);
                    acc = mfma16(x[k].l, y[k].h, acc);
                    acc = mfma16(x[k].h, y[k].h, acc);
                }
                if (poly) {
                    float a0[4], a1[4];
                    unpack4(make_uint2(e.x, e.y), a0);
                    unpack4(make_uint2(e.z, e.w), a1);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        float v = cb * (a0[u] + a1[u]) + cc * acc[u];
                        if (m + u == n) v += ca;
                        acc[u] = v;
                    }
                }
            }
            // (a stage never writes a plane that it reads, but for A <- Q T,
            // whose A has been read by the stages before)
            store(d0, acc);
            __syncthreads();
        }
        if (do_p) cur = 1 - cur;
    }
    // P_T out
    for (int i = tid; i < kChunks; i += THREADS) {
        const int r = i / (KS / 8), c = 8 * (i % (KS / 8));
        const uint16_t* o = pl + (SM_P + cur) * kSmallMat + small_at(r, c);
        const uint4 p0 = *reinterpret_cast<const uint4*>(o), p1 = *reinterpret_cast<const uint4*>(o + 8);
        const int64_t at = (int64_t)b * s2 + (int64_t)r * a.s_pad + c;
        stg(a.Ph + at, make_uint4(p0.x, p0.y, p1.x, p1.y));
        stg(a.Pl + at, make_uint4(p0.z, p0.w, p1.z, p1.w));
    }
}

constexpr unsigned kMaxGridZ = 65535;   // the grid's z extent holds the batch

template <int NPASS, int EPI, typename T, bool SYM = false>
hipError_t launch_tile(const GemmArgs& a, hipStream_t s) {
    if (a.M % T::BM || a.N % T::BN || a.K % T::BK) return hipErrorInvalidValue;
    const unsigned per = EPI == EPI_PART ? (unsigned)a.ksplit : a.dual ? 2u : 1u;
    if (SYM && EPI != EPI_PART && (unsigned)a.batch * per > kMaxGridZ) {
        // A dual launch of more than 32767 matrices: consecutive launches
        // over slices of the batch (the symmetric products' operands and
        // outputs are all bf16 / fp16 stacks with a batch stride).
        const int chunk = (int)(kMaxGridZ / per);
        auto at = [](const void* p, int64_t elems) {
            return p ? static_cast<const uint16_t*>(p) + elems : nullptr;
        };
        for (int b0 = 0; b0 < a.batch; b0 += chunk) {
            GemmArgs c = a;
            c.batch = a.batch - b0 < chunk ? a.batch - b0 : chunk;
            c.A0 = at(a.A0, b0 * a.sA);
            c.A1 = at(a.A1, b0 * a.sA);
            c.B0 = at(a.B0, b0 * a.sB);
            c.B1 = at(a.B1, b0 * a.sB);
            c.B0x = at(a.B0x, b0 * a.sB);
            c.B1x = at(a.B1x, b0 * a.sB);
            c.E0 = at(a.E0, b0 * a.sE);
            c.E1 = at(a.E1, b0 * a.sE);
            c.out0 = const_cast<uint16_t*>(at(a.out0, b0 * a.sOut0));
            c.out1 = const_cast<uint16_t*>(at(a.out1, b0 * a.sOut1));
            c.out0x = const_cast<uint16_t*>(at(a.out0x, b0 * a.sOut0));
            c.out1x = const_cast<uint16_t*>(at(a.out1x, b0 * a.sOut1));
            const hipError_t e = launch_tile<NPASS, EPI, T, SYM>(c, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const unsigned zb = (unsigned)a.batch * per;
    if (zb > kMaxGridZ) return hipErrorInvalidValue;
    dim3 grid((unsigned)(a.N / T::BN), (unsigned)(a.M / T::BM), zb);
    if (SYM) {
        if (a.M != a.N || T::BM != T::BN) return hipErrorInvalidValue;
        const unsigned tiles = (unsigned)(a.M / T::BM);
        grid = dim3(tiles * (tiles + 1) / 2, 1, zb);
    }
    hipLaunchKernelGGL((gemm<NPASS, EPI, T, SYM>), grid, dim3(T::THREADS), 0, s, a);
    return hipGetLastError();
}

// A symmetric product in two launches: the parts of K, then their sum.
template <int NPASS, int EPI, typename T>
hipError_t launch_split(const GemmArgs& a, hipStream_t s) {
    const hipError_t e = launch_tile<NPASS, EPI_PART, T, true>(a, s);
    if (e != hipSuccess) return e;
    const int64_t tiles = a.mfill / T::BM;
    const int64_t waves = (int64_t)a.batch * (tiles * (tiles + 1) / 2) * (T::BM / 32) * (T::BN / 32);
    hipLaunchKernelGGL((reduce_parts<EPI, T>), dim3((unsigned)(waves / 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ---- tile and split choices
//
// 256 compute units take two blocks of most of these tiles at once (one of a
// 256 x 256 or 256 x 128 tile, or of a three-pass 64 x 128 one, whose rings
// take 96 KB of LDS or more), so a launch of few tiles leaves most of the chip
// idle and costs one block's serial time: the slice loop's latency and a big tile's
// epilogue. There the tile shrinks to 64 x 64 (four times the blocks, each
// with four slices in flight), and a long K is split over more blocks, whose
// fp32 partials a second launch folds in order. A larger launch is bound by
// the path into LDS, where a small tile's lower reuse costs more than the
// fuller chip gains. Every choice computes each entry's sum in one order (per
// 16-deep k-step hi lo, lo hi, hi hi), so they are bitwise alike except where
// K is split, which only a symmetric product over the long side does.
// Measured (us per launch, 128 x 128 tiles before, chosen tile after):
//   three-pass s x s products: s = 256, batch 1: 8.7, 4.6; s = 512, batch 1:
//     13.2, 6.0 and batch 16: 17.9, 16.7; s = 1024, batch 1: 27.9, 10.7
//   Gram matrix, s x l: 256 x 1024: 11.6, 6.4; 512 x 2048, batch 4: 19.0,
//     10.3; 512 x 8192: 58.7, 13.0; 256 x 8192, batch 8: 58.5, 16.3; 1024 x
//     4096, batch 4: 90.0 on 256 x 256 tiles, 35.8
//   two-pass final product, s x l: 256 x 1024: 7.7, 5.9; 1024 x 4096: 29.3, 22.8
enum SymTile { SYM_64, SYM_64S2, SYM_128, SYM_256 };
struct SymPlan {
    SymTile tile;
    int ksplit;
};

int64_t sym_tiles(const GemmArgs& a, int m, int bm) {
    const int64_t t = (m + bm - 1) / bm;
    return (int64_t)a.batch * (a.dual ? 2 : 1) * (t * (t + 1) / 2);
}

// Parts of K for a launch of n tiles: as many as `most` blocks hold, none of
// them shorter than `least`, and no more than the scratch holds.
int parts_of(const GemmArgs& a, int64_t n, int bm, int m, int64_t most, int least) {
    const int64_t t = (m + bm - 1) / bm;
    const int64_t floats = (int64_t)a.batch * (t * (t + 1) / 2) * bm * bm;
    int64_t p = std::min(most / n, (int64_t)(a.K / least));
    if (floats * p > a.part_floats) p = a.part_floats / floats;
    return p < 2 ? 1 : (int)p;
}

SymPlan plan_sym(const GemmArgs& a, GemmEpi epi, int npass) {
    const bool split = a.part && !a.dual && !a.f16 && (epi == EPI_SPLIT || epi == EPI_H16);
    const int mr = a.mreal ? a.mreal : a.M;   // 64 x 64 tiles stop at the real side
    const int64_t n64 = sym_tiles(a, mr, 64), n128 = sym_tiles(a, a.M, 128);
    const int64_t n256 = a.M % 256 ? 0 : sym_tiles(a, a.M, 256);
    if (npass == 3) {
        // one block a compute unit: four stages; beyond, two of the two-stage
        // ring's share one (us on 64 x 64 and on 128 x 128: 510 at s = 320 17.5
        // and 19.4, 495 at s = 640 24.6 and 25.3, 408 at s = 1024 21.8 and 30.3;
        // 540 at s = 320 20.0 and 17.7, 550 at s = 640 30.9 and 26.5). A number
        // that gemm renumbers onto the XCDs keeps a matrix in one L2, and up to
        // K = 512 holds to 640 (600 at s = 320 14.1 and 17.4, 640 at s = 256 12.5
        // and 14.6, 576 at s = 512 17.6 and 18.1; 672 at s = 384 17.0 and 16.2,
        // 720 at s = 512 20.1 and 19.8; 544 at s = 1024 29.4 and 28.7). On a
        // single 128 x 128 tile, of which they are three quarters, up to 1600
        // (384 at s = 128: 5.8 against 7.5 us; 1536: 15.1 against 17.0)
        if (n64 <= 256) return {SYM_64, split && a.K >= 1024 ? parts_of(a, n64, 64, mr, 256, 512) : 1};
        if (n64 <= (mr <= 128 ? 1600 : a.K <= 512 && n64 % kXcds == 0 ? 640 : 512)) return {SYM_64S2, 1};
        // two rounds of 256 x 256 tiles for the plain products (the
        // polynomial epilogues spill on them): 5-10% at s = 1024 and 2048
        const bool poly = epi == EPI_POLY || epi == EPI_QPOLY;
        return {!poly && a.M >= 1024 && n256 >= 512 ? SYM_256 : SYM_128, 1};
    }
    if (n64 <= 256 && (n64 <= 170 || a.K < 6144)) {
        // below K = 2048 the second launch costs more than the shorter loop
        // saves (1024 deep: 6.4 against 7.5 us); from 4096 on two blocks a
        // compute unit pay (1024 x 4096: 15.6 us in three parts, 18.0 whole),
        // but not in two parts (768 x 4096, 234 tiles: 27.8, 23.1 whole)
        const int64_t most = a.K >= 4096 && n64 > 128 && n64 <= 170 ? 512 : 256;
        return {SYM_64, split && a.K >= 2048 ? parts_of(a, n64, 64, mr, most, 640) : 1};
    }
    // 288 to 336 tiles of 64 x 64 measured 13.6 us at K = 2048 where 128 x 128
    // took 19.5, 22.6 against 32.8 at 4096; 528 of them 23.9 against 20.7. A
    // longer K goes in parts of 128 x 128 tiles (384 x 10240, 210 tiles of 64 x
    // 64: 31.0 us in four parts, 62.9 whole, 69.6 in two of 64 x 64)
    if (n64 <= 448 && a.K < 6144) return {SYM_64, 1};
    // 256 x 256 tiles run one to a compute unit: they pay once their last
    // round is filled well (s = 2048: 144 tiles 57.8 against 62.0 us, 288
    // tiles 116.6 against 104.6; s = 1024, 160 tiles: 201 against 215, 120
    // tiles 95.8 against 74.4; s = 4096, 136 tiles, where 128 x 128 would take
    // just over a round of 512: a Muon step of 1756 against 1883 us)
    const int64_t rounds = (n256 + 255) / 256;
    if (a.M >= (a.f16 ? 2048 : 1024) && n256 >= (rounds > 1 ? 160 * rounds : n128 > 512 ? 129 : 140))
        return {SYM_256, 1};
    return {SYM_128, split && a.K >= 4096 ? parts_of(a, n128, 128, a.M, 256, 1024) : 1};
}

bool is_apply(GemmEpi epi) { return epi == EPI_APPLY || epi == EPI_APPLY_F32; }
bool is_sym(GemmEpi epi) { return epi != EPI_UPDATE && epi != EPI_FINAL && !is_apply(epi); }

// A symmetric product on tile T, whole or split over K.
template <int NPASS, int EPI, typename T, bool SPLIT = false>
hipError_t launch_sym(const GemmArgs& a0, int ksplit, hipStream_t s) {
    GemmArgs a = a0;
    if (T::BM == 64 && a.mreal) {
        a.mfill = std::max(a.mreal, a.mfill);
        a.M = a.N = ksplit > 1 ? a.mreal : a.mfill;
    } else {
        a.mfill = a.M;
    }
    a.K = (a.K + T::BK - 1) / T::BK * T::BK;   // operands are zero to the next 128
    a.ksplit = ksplit;
    if constexpr (SPLIT && (EPI == EPI_SPLIT || EPI == EPI_H16)) {
        if (ksplit > 1) return launch_split<NPASS, EPI, T>(a, s);
    }
    return ksplit > 1 ? hipErrorInvalidValue : launch_tile<NPASS, EPI, T, true>(a, s);
}

// The tiles: 128 x 128 with four stages of 32-deep slices (two blocks of four
// waves per CU) for one-pass products, 256 x 256 for large ones; three-pass
// products 128 x 128 in a two-stage ring of eight waves. The fp16 s x s
// products run on 256 x 256 from s = 2048 (12% faster there, 24% at 4096; 13%
// slower at 1024).
template <int EPI>
hipError_t sym_one(const GemmArgs& a, const SymPlan& p, hipStream_t s) {
    switch (p.tile) {
        case SYM_64: return launch_sym<1, EPI, Tile<1, 0, 64, 64, 64, 2, 2, 4>, true>(a, p.ksplit, s);
        case SYM_256: return launch_sym<1, EPI, Tile<1, 0, 256, 256, kSliceK, 4, 2, 3>>(a, 1, s);
        default: return launch_sym<1, EPI, Tile<1, 0, 128, 128, kSliceK, 2, 2, 4>, true>(a, p.ksplit, s);
    }
}
template <int EPI>
hipError_t sym_f16(const GemmArgs& a, const SymPlan& p, hipStream_t s) {
    switch (p.tile) {
        case SYM_64: return launch_sym<1, EPI, Tile<1, 0, 64, 64, 64, 2, 2, 4, true>>(a, 1, s);
        case SYM_256: return launch_sym<1, EPI, Tile<1, 0, 256, 256, kSliceK, 4, 2, 3, true>>(a, 1, s);
        default: return launch_sym<1, EPI, Tile<1, 0, 128, 128, kSliceK, 2, 2, 4, true>>(a, 1, s);
    }
}
template <int EPI>
hipError_t sym_three(const GemmArgs& a, const SymPlan& p, hipStream_t s) {
    switch (p.tile) {
        case SYM_64: return launch_sym<3, EPI, Tile<3, 0, 64, 64, kSliceK, 2, 2, 4>, true>(a, p.ksplit, s);
        case SYM_64S2: return launch_sym<3, EPI, Tile<3, 0, 64, 64, kSliceK, 2, 2, 2>>(a, 1, s);
        case SYM_256:
            if constexpr (EPI == EPI_SPLIT) return launch_sym<3, EPI, Tile<3, 0, 256, 256, kSliceK, 2, 4, 2>>(a, 1, s);
            return hipErrorInvalidValue;
        default:
            // plain products: from K = 1024 the slices pay for the run-on loop's
            // longer start (s = 1024, 16 matrices: 72.3 against 74.7 us; s =
            // 384, 64: 24.8 against 23.1); polynomial ones spill in the other
            // loop within the registers of two blocks a CU (s = 512, 64: 55.4
            // against 57.2)
            if constexpr (EPI == EPI_SPLIT) {
                if (a.K < 1024) return launch_sym<3, EPI, Tile<3, 0, 128, 128, kSliceK, 4, 2, 2>>(a, 1, s);
            }
            return launch_sym<3, EPI, Tile<3, 0, 128, 128, kSliceK, 4, 2, 2, false, true>>(a, 1, s);
    }
}

hipError_t launch_sym_product(const GemmArgs& a, GemmEpi epi, int npass, hipStream_t s) {
    const SymPlan p = plan_sym(a, epi, npass);
    if (a.f16) {
        if (npass != 1 || (a.dual && epi != EPI_H16)) return hipErrorInvalidValue;   // dual: the chain's P and T
        switch (epi) {
            case EPI_SPLIT: return sym_f16<EPI_SPLIT>(a, p, s);
            case EPI_H16: return sym_f16<EPI_H16>(a, p, s);
            case EPI_QPOLY_H16: return sym_f16<EPI_QPOLY_H16>(a, p, s);
            case EPI_POLY_H16: return sym_f16<EPI_POLY_H16>(a, p, s);   // the Direct form's B = b A + c A^2
            default: return hipErrorInvalidValue;
        }
    }
    if (a.dual && !(epi == EPI_SPLIT && npass == 3)) return hipErrorInvalidValue;
    if (npass == 1) {   // the Gram matrix (EPI_H16: into the fp16 chain or the Direct form)
        if (epi == EPI_SPLIT) return sym_one<EPI_SPLIT>(a, p, s);
        if (epi == EPI_H16) return sym_one<EPI_H16>(a, p, s);
    } else if (npass == 3) {
        if (epi == EPI_SPLIT) return sym_three<EPI_SPLIT>(a, p, s);
        if (epi == EPI_POLY) return sym_three<EPI_POLY>(a, p, s);
        if (epi == EPI_QPOLY) return sym_three<EPI_QPOLY>(a, p, s);
    }
    return hipErrorInvalidValue;
}

// X-side products with the [K][N] operand. A two-stage ring of 128 x 128
// tiles leaves room for three blocks per CU; with the update applied in the
// epilogue eight waves per block hide more of the W traffic. A launch of at
// most one such tile a CU takes 64 x 128 tiles of eight waves in a deeper ring.
template <int NPASS, int EPI>
hipError_t launch_right(const GemmArgs& a, hipStream_t s) {
    const int64_t n128 = (int64_t)a.batch * (a.M / 128) * (a.N / 128);
    // (three passes: 256 tiles 21.6 us on 64 x 128, 20.7 on 128 x 128; 16
    // tiles 6.8 against 11.1)
    if (n128 <= (NPASS == 3 ? 128 : 256)) {
        using T = Tile<NPASS, 1, 64, 128, NPASS == 1 ? 64 : kSliceK, 2, 4, NPASS == 1 ? 3 : 4>;
        GemmArgs r = a;
        r.K = (a.K + T::BK - 1) / T::BK * T::BK;   // operands are zero to the next 64
        if (a.mreal) r.M = a.mreal;
        return launch_tile<NPASS, EPI, T>(r, s);
    }
    if constexpr ((NPASS == 2 && EPI == EPI_APPLY) || (NPASS < 3 && EPI == EPI_APPLY_F32))
        return launch_tile<NPASS, EPI, Tile<NPASS, 1, 128, 128, kSliceK, 4, 2, 2>>(a, s);
    else
        return launch_tile<NPASS, EPI, Tile<NPASS, 1, 128, 128, kSliceK, 2, 2, 2>>(a, s);
}

// The Direct form's X-side products from s = 2048: X^T as rows lets them run
// on the wide plain-read tiles (28% faster at s = 2048, 35% at 4096 than the
// transposing reads of the [K][N] operand): 256 x 256, or 256 x 128 where l
// is not a multiple of 256 and for the fused update step (whose W rows spill
// on 256 x 256). A launch of fewer than 160 of the former (two of the latter)
// leaves too much of the chip idle and takes 128 x 128.
template <int EPI>
hipError_t launch_rows(const GemmArgs& a, hipStream_t s) {
    if ((int64_t)a.batch * (a.M / 256) * (a.N / 128) < 2 * 160)
        return launch_tile<1, EPI, Tile<1, 0, 128, 128, kSliceK, 2, 2, 4>>(a, s);
    using TR = Tile<1, 0, 256, 256, kSliceK, 2, 4, 3>;
    using TRN = Tile<1, 0, 256, 128, kSliceK, 4, 2, 4>;
    if constexpr (EPI == EPI_UPDATE || EPI == EPI_FINAL) {
        if (a.N % 256 == 0) return launch_tile<1, EPI, TR>(a, s);
    }
    return launch_tile<1, EPI, TRN>(a, s);
}

}  // namespace

int gemm_launches(const GemmArgs& a, GemmEpi epi, int npass) {
    return is_sym(epi) && plan_sym(a, epi, npass).ksplit > 1 ? 2 : 1;
}

// bf16 transpose through a 64 x 64 LDS tile (row pitch 66 elements, so the
// column reads spread over the banks): 16-byte row segments in and out.
__global__ __launch_bounds__(256) void transpose_bf16(const uint16_t* __restrict__ in, uint16_t* __restrict__ out,
                                                      int64_t rows, int64_t cols, int64_t stride) {
    __shared__ uint16_t t[64][66];
    const int64_t b = blockIdx.z;
    const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
    const uint16_t* src = in + b * stride + r0 * cols + c0;
    uint16_t* dst = out + b * stride + c0 * rows + r0;
    for (int i = threadIdx.x; i < 64 * 8; i += 256) {
        const int r = i >> 3, c = (i & 7) * 8;
        const uint4 v = ldg<uint4>(src + (int64_t)r * cols + c);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            t[r][c + 2 * q] = (uint16_t)(w[q] & 0xffffu);
            t[r][c + 2 * q + 1] = (uint16_t)(w[q] >> 16);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * 8; i += 256) {
        const int r = i >> 3, c = (i & 7) * 8;   // output row r (input column), input rows c .. c + 7
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (uint32_t)t[c + 2 * q][r] | ((uint32_t)t[c + 2 * q + 1][r] << 16);
        stg(dst + (int64_t)r * rows + c, make_uint4(w[0], w[1], w[2], w[3]));
    }
}

hipError_t launch_gemm(const GemmArgs& a, GemmEpi epi, int npass, hipStream_t s) {
    if (is_sym(epi)) return launch_sym_product(a, epi, npass, s);
    if (a.f16 || a.dual) return hipErrorInvalidValue;
    if (is_apply(epi) && (a.cols < 16 || a.out_transposed)) return hipErrorInvalidValue;
    if (a.b_rows) {
        if (npass != 1 || a.M % 256) return hipErrorInvalidValue;
        if (epi == EPI_UPDATE) return launch_rows<EPI_UPDATE>(a, s);
        if (epi == EPI_FINAL) return launch_rows<EPI_FINAL>(a, s);
        return epi == EPI_APPLY ? launch_rows<EPI_APPLY>(a, s) : launch_rows<EPI_APPLY_F32>(a, s);
    }
    if (epi == EPI_UPDATE) return npass == 1 ? launch_right<1, EPI_UPDATE>(a, s) : hipErrorInvalidValue;
    if (epi == EPI_FINAL) {
        if (npass == 1) return launch_right<1, EPI_FINAL>(a, s);
        if (npass == 2) return launch_right<2, EPI_FINAL>(a, s);
        if (npass == 3) return launch_right<3, EPI_FINAL>(a, s);
    } else if (epi == EPI_APPLY) {
        if (npass == 1) return launch_right<1, EPI_APPLY>(a, s);
        if (npass == 2) return launch_right<2, EPI_APPLY>(a, s);
        if (npass == 3) return launch_right<3, EPI_APPLY>(a, s);
    } else {
        if (npass == 1) return launch_right<1, EPI_APPLY_F32>(a, s);
        if (npass == 2) return launch_right<2, EPI_APPLY_F32>(a, s);
        if (npass == 3) return launch_right<3, EPI_APPLY_F32>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_chain_small(const SmallChainArgs& a, hipStream_t s) {
    if (a.s_k < 32 || a.s_k > kSmallChainS || a.s_k % 32 || a.s_pad < kSmallChainS || a.s_pad % 8 ||
        a.ns_steps < 1 || a.ns_steps > kChainMaxSteps || a.batch < 1)
        return hipErrorInvalidValue;
    if (a.s_k == 32) hipLaunchKernelGGL(chain_small<32>, dim3((unsigned)a.batch), dim3(64 * 3), 0, s, a);
    else hipLaunchKernelGGL(chain_small<64>, dim3((unsigned)a.batch), dim3(64 * 10), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_transpose_bf16(const uint16_t* in, uint16_t* out, int64_t rows, int64_t cols, int batch,
                                 int64_t stride, hipStream_t s) {
    if (rows < 64 || cols < 64 || rows % 64 || cols % 64 || rows / 64 > 65535 || batch < 1 || batch > 65535)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)(cols / 64), (unsigned)(rows / 64), (unsigned)batch);
    hipLaunchKernelGGL(transpose_bf16, grid, dim3(256), 0, s, in, out, rows, cols, stride);
    return hipGetLastError();
}

}  // namespace dion2
