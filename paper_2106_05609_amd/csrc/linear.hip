// Dense transform of the GNN operators on the matrix cores (gas_linear,
// gas_mlp2):  Y = act(c_identity * Z + c_weight * (Z W) + bias), and the fused
// two-layer MLP of the GIN operator.
//
// This is the only dense contraction of the step (the W of the paper's GCN,
// GCNII and GIN operator equations), so it is the only place MFMA is used.
// fp32 data uses the bf16 instruction on operands split in three (split.h), the fused fp32 MLP
// v_mfma_f32_32x32x2_f32, bf16 data v_mfma_f32_32x32x16_bf16, all with fp32 accumulation.
//
// Tiling: a workgroup of 4 wavefronts (2 x 2) owns a BM x BN tile of Y, each
// wavefront a sub-tile made of 32x32 MFMA blocks.  K is walked in tiles: the
// next A (rows of Z) and B (rows of W) tiles are fetched from global memory
// into registers while the current ones are consumed from LDS.
//   fused fp32 MLP: A is stored [m][k] so that one 128-bit LDS read gives a lane the four
//         k values of four consecutive MFMAs; lanes 0-31 and 32-63 of an MFMA
//         take different k, and A and B agree on which.
//   bf16: both operands need eight consecutive k per lane.  Z is [m][k]
//         already; W is [k][n], so its tiles are transposed on the way into
//         LDS: a thread loads an 8(k) x 8(n) block as eight 16-byte row pieces,
//         regroups it in registers and writes eight 16-byte [n][k] pieces.
// The accumulator of a 32x32 block keeps, in register r of lane (li, lh),
// row 8*(r/4) + 4*lh + r%4 and column li.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "split.h"
#include <mutex>

namespace gas {
namespace {

struct LinArgs {
    const char* Z;   int64_t ldz;      // elements
    const char* W;
    const char* bias;
    char* Y;         int64_t ldy;
    int64_t M;
    int K, N;
    float c_id, c_w;
    int relu;
    int trans_w;                       // W is given as [N][K] (the product is Z W^T of a [N, K] matrix)
    const char* mask; int64_t ldmask;  // optional [M, N]: outputs where mask <= 0 are set to zero
    const int32_t* push_idx = nullptr; // optional (fp32 tile kernel): row m also goes to push_hist[push_idx[m], :]
    char* push_hist = nullptr; int64_t ld_push = 0;
    const char* add = nullptr; int64_t ldadd = 0;     // optional (fp32): [M, N] added before the mask (may be Y itself)
    char* total = nullptr; int64_t ldtotal = 0;       // optional (fp32): [M, N], total += c_total * output
    float c_total = 0.f;
};

struct MlpArgs {
    const char* Z;   int64_t ldz;
    const char* W1;  const char* b1;
    const char* W2;  const char* b2;
    char* Y;         int64_t ldy;
    int64_t M;
    int K, H, N;     // F_in, F_hid (<= kHidMax), F_out
    int relu_out;
};

constexpr int kHidMax = 256;
constexpr int kMlpRowsF32 = 32, kMlpRowsBF16 = 64;     // rows per workgroup of the fused MLP kernels

template <int TM, int TN>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}

__device__ __forceinline__ float bf16_val(const uint16_t* p, int64_t i) { return __uint_as_float((uint32_t)p[i] << 16); }

// ====================================================================== fp32
constexpr int kBK = 32;                    // k per tile
constexpr int kLdA = kBK + 4;              // padded LDS row of the A tile (floats)

// Fetch / stage one BM x kBK tile of a row-major fp32 matrix with row stride ld.
template <int BM, bool VEC>
struct ATileF32 {
    static constexpr int NV = BM * kBK / 4 / 256;
    f32x4 r[NV];
    __device__ __forceinline__ void fetch(const float* Z, int64_t ld, int64_t M, int K, int64_t m0, int k0, int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            const int64_t m = m0 + idx / (kBK / 4);
            const int k = k0 + 4 * (idx % (kBK / 4));
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (m < M) {
                if constexpr (VEC) {
                    if (k < K) v = *reinterpret_cast<const f32x4*>(Z + m * ld + k);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k + e < K) v[e] = Z[m * ld + k + e];
                }
            }
            r[i] = v;
        }
    }
    __device__ __forceinline__ void stage(float (*As)[kLdA], int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            *reinterpret_cast<f32x4*>(&As[idx / (kBK / 4)][4 * (idx % (kBK / 4))]) = r[i];
        }
    }
};

// Fetch / stage one kBK x BN tile of a row-major fp32 [K][N] matrix.
template <int BN, bool VEC>
struct BTileF32 {
    static constexpr int NV = kBK * BN / 4 / 256;
    f32x4 r[NV];
    __device__ __forceinline__ void fetch(const float* W, int K, int N, int k0, int n0, int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            const int k = k0 + idx / (BN / 4), n = n0 + 4 * (idx % (BN / 4));
            if (k < K) {
                if constexpr (VEC) {
                    if (n < N) v = *reinterpret_cast<const f32x4*>(W + (int64_t)k * N + n);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < N) v[e] = W[(int64_t)k * N + n + e];
                }
            }
            r[i] = v;
        }
    }
    __device__ __forceinline__ void stage(float (*Bs)[BN + 4], int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            *reinterpret_cast<f32x4*>(&Bs[idx / (BN / 4)][4 * (idx % (BN / 4))]) = r[i];
        }
    }
};

// acc += A[arow0.., acol0 .. acol0+kBK) * Bs, A an LDS array with row stride lda floats
template <int TM, int TN, int BN>
__device__ __forceinline__ void mfma_tile_f32(const float* A, int lda, int arow0, int acol0,
                                              const float (*Bs)[BN + 4], int bcol0, int li, int lh,
                                              f32x16 (&acc)[TM][TN]) {
#pragma unroll
    for (int kq = 0; kq < kBK / 8; ++kq) {
        f32x4 fa[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = *reinterpret_cast<const f32x4*>(A + (arow0 + 32 * i + li) * lda + acol0 + kq * 8 + lh * 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float fb[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = Bs[kq * 8 + lh * 4 + q][bcol0 + 32 * j + li];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[j], acc[i][j], 0, 0, 0);
        }
    }
}

// The wavefront's 32 x 32 blocks of the output, at row m0 and column n0.  WHOLE: they lie inside the output and the
// strides are below 2^26, so a row's address is a scalar base and one 32-bit lane offset; else every element is checked.
// (With the checks and 64-bit addresses everywhere this took 4 us per 128 x 128 tile, a sixth of the tile's time.)
template <int TM, int TN, bool WHOLE, bool EXTRA, bool PUSH>
__device__ __forceinline__ void store_rows(const LinArgs& a, int64_t m0, int n0, int li, int lh, const f32x16 (&acc)[TM][TN]) {
    const float* bias = reinterpret_cast<const float*>(a.bias);
    float bv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bv[j] = bias && (WHOLE || n0 + 32 * j + li < a.N) ? bias[n0 + 32 * j + li] : 0.f;
    auto at = [&](const char* X, int64_t ld, int64_t row) {       // element (row + 4 lh, n0 + li)
        if constexpr (WHOLE)
            return reinterpret_cast<float*>(const_cast<char*>(X) + (row * ld + n0) * 4 + (uint32_t)((4 * lh * (int)ld + li) * 4));
        else
            return reinterpret_cast<float*>(const_cast<char*>(X) + ((row + 4 * lh) * ld + n0 + li) * 4);
    };
    // the optional operands of eight rows are loaded together, before any of them is needed
    constexpr int R = EXTRA ? 8 : 1;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r0 = 0; r0 < 16; r0 += R) {
            auto row_of = [&](int r) { return m0 + 32 * i + 8 * (r / 4) + r % 4; };
            auto in = [&](int r, int j) { return WHOLE || (row_of(r) + 4 * lh < a.M && n0 + 32 * j + li < a.N); };
            float zv[R][TN], kv[R][TN], av[R][TN], tv[R][TN];
            auto load = [&](float (&v)[R][TN], const char* X, int64_t ld) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float* x = at(X, ld, row_of(r0 + r));
#pragma unroll
                    for (int j = 0; j < TN; ++j) v[r][j] = in(r0 + r, j) ? x[32 * j] : 0.f;
                }
            };
            if constexpr (EXTRA) {
                if (a.c_id != 0.f) load(zv, a.Z, a.ldz);
                if (a.add) load(av, a.add, a.ldadd);
                if (a.mask) load(kv, a.mask, a.ldmask);
                if (a.total) load(tv, a.total, a.ldtotal);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t row = row_of(r0 + r);
                if (!WHOLE && row + 4 * lh >= a.M) continue;
                float* yrow = at(a.Y, a.ldy, row);
                float* trow = EXTRA && a.total ? at(a.total, a.ldtotal, row) : nullptr;
                float* hrow = nullptr;
                if constexpr (PUSH)
                    hrow = reinterpret_cast<float*>(a.push_hist) + n0 + li +
                           (WHOLE ? (uint64_t)(uint32_t)a.push_idx[row + 4 * lh] * (uint32_t)a.ld_push
                                  : (uint64_t)((int64_t)a.push_idx[row + 4 * lh] * a.ld_push));
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if (!WHOLE && n0 + 32 * j + li >= a.N) continue;
                    float y = a.c_w * acc[i][j][r0 + r] + bv[j];
                    if (EXTRA && a.c_id != 0.f) y += a.c_id * zv[r][j];
                    if (EXTRA && a.add) y += av[r][j];
                    if (a.relu) y = fmaxf(y, 0.f);
                    if (EXTRA && a.mask && !(kv[r][j] > 0.f)) y = 0.f;
                    yrow[32 * j] = y;
                    if (EXTRA && a.total) trow[32 * j] = tv[r][j] + a.c_total * y;
                    if constexpr (PUSH) hrow[32 * j] = y;         // Push in the epilogue
                }
            }
        }
}
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const LinArgs& a, int64_t m0, int n0, int li, int lh, const f32x16 (&acc)[TM][TN]) {
    constexpr int64_t kNear = 1 << 26;
    const bool whole = m0 + 32 * TM <= a.M && n0 + 32 * TN <= a.N && a.ldy < kNear && a.ldz < kNear && a.ldmask < kNear &&
                       a.ld_push < kNear && a.ldadd < kNear && a.ldtotal < kNear;
    const bool extra = a.c_id != 0.f || a.mask || a.add || a.total;
    if (!extra && !a.push_idx) {
        if (whole) store_rows<TM, TN, true, false, false>(a, m0, n0, li, lh, acc);
        else store_rows<TM, TN, false, false, false>(a, m0, n0, li, lh, acc);
    } else if (whole && !extra) store_rows<TM, TN, true, false, true>(a, m0, n0, li, lh, acc);
    else if (whole && !a.push_idx) store_rows<TM, TN, true, true, false>(a, m0, n0, li, lh, acc);
    else if (!a.push_idx) store_rows<TM, TN, false, true, false>(a, m0, n0, li, lh, acc);
    else store_rows<TM, TN, false, true, true>(a, m0, n0, li, lh, acc);
}

// Y tile of BM x BN by 2 x 2 wavefronts, operands split into bf16 parts on their way into LDS (split.h).  The column
// tiles of one row tile follow each other on one XCD (workgroups are dealt to the eight XCDs in turn): the second
// reads the rows of Z from that L2.
template <int BM, int BN, int KS, bool TRANS, int WPS>
__global__ __launch_bounds__(256, WPS) void linear_split_kernel(LinArgs a) {
    using G = SplitGemm<BM, BN, 2, 2, KS, true, TRANS>;
    constexpr int TM = G::TM, TN = G::TN;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const float* Z = reinterpret_cast<const float*>(a.Z);
    const float* W = reinterpret_cast<const float*>(a.W);
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned gn = (a.N + BN - 1) / BN, of_xcd = blockIdx.x / 8;
    const int64_t m0 = ((int64_t)(of_xcd / gn) * 8 + blockIdx.x % 8) * BM;
    if (m0 >= a.M) return;                             // the grid is padded to a multiple of eight row tiles
    const int n0 = (int)(of_xcd % gn) * BN;
    const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
    const int64_t ldw = TRANS ? a.K : a.N;
    G g;
    f32x16 acc[TM][TN];
    if (!g.run(Z, a.ldz, m0, a.M, W, ldw, n0, a.N, 0, a.K, reinterpret_cast<uint16_t*>(smem), wm0, wn0, acc))
        plain_tile<TM, TN, true, TRANS>(Z, a.ldz, m0 + wm0, a.M, W, ldw, n0 + wn0, a.N, 0, a.K, acc);
    store_tile<TM, TN>(a, m0 + wm0, n0 + wn0, li, lh, acc);
}

// The same tile by KG groups of WM x WN wavefronts that take the steps of 32 k in turn: where there is at most one tile for a
// compute unit, one wavefront on a SIMD issues a vector instruction every eight cycles, two or more every four to five, and
// its chains of dependent products and LDS reads leave the unit idle.  The sum over the groups goes through LDS.
template <int BM, int BN, int WM, int WN, bool TRANS, int KG>
__global__ __launch_bounds__(64 * WM * WN * KG) void linear_split_groups_kernel(LinArgs a) {
    using G = SplitGemm<BM, BN, WM, WN, 2, true, TRANS, KG>;
    constexpr int TM = G::TM, TN = G::TN;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const float* Z = reinterpret_cast<const float*>(a.Z);
    const float* W = reinterpret_cast<const float*>(a.W);
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = wave / (WM * WN);
    const unsigned gn = (a.N + BN - 1) / BN, of_xcd = blockIdx.x / 8;
    const int64_t m0 = ((int64_t)(of_xcd / gn) * 8 + blockIdx.x % 8) * BM;
    if (m0 >= a.M) return;                             // the grid is padded to a multiple of eight row tiles
    const int n0 = (int)(of_xcd % gn) * BN;
    const int wm0 = wave / WN % WM * (BM / WM), wn0 = wave % WN * (BN / WN);
    const int64_t ldw = TRANS ? a.K : a.N;
    G g;
    f32x16 acc[TM][TN];
    if (!g.run_groups(Z, a.ldz, m0, a.M, W, ldw, n0, a.N, a.K, reinterpret_cast<uint16_t*>(smem), group, wm0, wn0, acc))
        plain_tile<TM, TN, true, TRANS>(Z, a.ldz, m0 + wm0, a.M, W, ldw, n0 + wn0, a.N, 0, a.K, acc);
    if (group == 0) store_tile<TM, TN>(a, m0 + wm0, n0 + wn0, li, lh, acc);
}

// fp32, weights stationary: a matrix of up to 32 KT x 256 stays, split, in the registers of one persistent workgroup of
// eight wavefronts (32 output columns each), and row tiles stream past it: a row is split once, not once per column tile,
// and a weight once per workgroup, not once per row tile.
//
// Products of 16 x 16 x 32, taken transposed (the weights are the first operand): a lane ends up with eight consecutive
// columns of one row, stored as two 16-byte pieces.  LDS holds the three parts of two row tiles: while one is multiplied the
// next is split and written, by wavefronts 0-3 before their products and by 4-7 after theirs, so that of the two wavefronts
// of a SIMD one splits while the other multiplies; one barrier a tile.  The operands of a step are read from LDS one step
// ahead (sched_barrier keeps them there: left to itself the compiler reads each fragment right before its use, 50,000 x 256 x
// 256 then take 50 us).  With 256 columns the registers do not hold all of it: the third parts of the first LS steps lie in LDS (without:
// spills, 54 us).
//
// Bound by the matrix pipe and the vector unit together, at the clock that the power allows (1.7-1.9 GHz; the instructions alone,
// on random operands, reach 1,400-1,900 TFLOP/s): 50,000 x 256 x 256 46 us, by the 128 x 128 tiles above 59; 600,000 rows 454 (1,040 TFLOP/s
// of bf16 products) and 567, with the push 520 and 601.  The same products in the same order of steps, summed by another shape of the
// instruction: one element in 55 differs from the tiles' in its last bits, neither nearer to 64 bits (both 9.0e-8 off at 256 columns).
//
// A tile that holds a value below 2^-110 is staged again times 2^40 (split.h says why), and so are the weights if one of
// them is; a wavefront whose sums are not finite takes its block again with the fp32 instruction.
template <int KT, bool MASK>
struct WsSplit {
    static constexpr int RB = KT <= 4 ? 2 : 1, ROWS = 16 * RB;                  // rows of a tile
    static constexpr int KP = 4 * KT, PITCH = (KP + 7) / 8 * 64;                // pieces of eight k, bf16 elements of a row in LDS
    static constexpr int PLANE = ROWS * PITCH;
    static constexpr int LS = KT == 8 ? (MASK ? 6 : 4) : (KT == 7 ? 2 : 0);     // steps of 32 k whose third parts lie in LDS
    static constexpr int kLdsBytes = 2 * 3 * PLANE * 2 + LS * 2 * 512 * 16 + 32;
};
template <int KT, bool TRANS, bool MASK>
__global__ __launch_bounds__(512) void linear_ws_split_kernel(LinArgs a, int64_t n_tiles) {
    using L = WsSplit<KT, MASK>;
    constexpr int RB = L::RB, ROWS = L::ROWS, KP = L::KP, PITCH = L::PITCH, PLANE = L::PLANE, LS = L::LS;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t* planes = reinterpret_cast<uint16_t*>(smem);                              // [2][3][ROWS][PITCH]
    bf16x8* wlds = reinterpret_cast<bf16x8*>(smem + 2 * 3 * PLANE * 2);                // [LS][2][512]
    uint32_t* low_tile = reinterpret_cast<uint32_t*>(smem + 2 * 3 * PLANE * 2 + LS * 2 * 512 * 16);     // [4], of tile it & 3
    uint32_t* low_w = low_tile + 4;
    const float* Z = reinterpret_cast<const float*>(a.Z);
    const float* W = reinterpret_cast<const float*>(a.W);
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = 32 * wave;                                         // the wavefront's first column
    const int wcol = c0 + 8 * (li >> 2) + (li & 3);                   // column of the lane's weights in block 0 (+ 4 in block 1)
    if (tid < 5) low_tile[tid] = 0;
    __syncthreads();

    auto split8 = [](const float (&x)[8], bf16x8 (&f)[3]) {
        u32x4 h, m, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t u, v, w;
            split_pair(x[2 * e], x[2 * e + 1], u, v, w);
            h[e] = u; m[e] = v; l[e] = w;
        }
        f[0] = __builtin_bit_cast(bf16x8, h);
        f[1] = __builtin_bit_cast(bf16x8, m);
        f[2] = __builtin_bit_cast(bf16x8, l);
    };
    auto least = [](const float (&x)[8], uint32_t low) {
#pragma unroll
        for (int e = 0; e < 8; ++e) low = min(low, 2 * __float_as_uint(x[e]) - 1);
        return low;
    };

    // ---- the thread's piece of a row tile: eight k of one row
    const int prow = tid / KP, piece = tid % KP;
    const int at = prow * PITCH + 8 * (piece ^ (prow & 7));
    const bool stages = ROWS * KP == 512 || prow < ROWS;
    float raw[8];
    auto fetch = [&](int64_t tile) {
        if (!stages) return;
        int64_t m = tile * ROWS + prow;
        m = m < a.M ? m : a.M - 1;
        // no branch around the loads and no write to their registers until stage(): either would wait for what is in flight
        const float* p = Z + m * a.ldz;
        const f32x4 u = *reinterpret_cast<const f32x4_any*>(p + min(8 * piece, a.K - 4));
        const f32x4 v = *reinterpret_cast<const f32x4_any*>(p + min(8 * piece + 4, a.K - 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) { raw[e] = u[e]; raw[4 + e] = v[e]; }
    };
    // columns beyond the last come out zero (a four that begins before the last column and ends beyond was loaded from K - 4)
    auto trim = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int left = a.K - 8 * piece - 4 * q;                  // columns of this four
            float w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[e] = left > e ? raw[4 * q + e] : 0.f;
                if (a.K & 3) {
#pragma unroll
                    for (int l = 1; l < 4; ++l)
                        if (e < l) w[e] = left == l ? raw[4 * q + e + 4 - l] : w[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[4 * q + e] = w[e];
        }
    };
    auto write = [&](int it) {
        bf16x8 f[3];
        split8(raw, f);
#pragma unroll
        for (int part = 0; part < 3; ++part) *reinterpret_cast<bf16x8*>(planes + ((it & 1) * 3 + part) * PLANE + at) = f[part];
    };
    auto stage = [&](int it) {
        if (!stages) return;
        if (a.K != 32 * KT) trim();
        if (least(raw, 0xFFFFFFFFu) < kLeast) low_tile[it & 3] = 1;
        write(it);
    };

    int64_t tile = blockIdx.x;
    const int64_t step = gridDim.x;
    if (tile < n_tiles) fetch(tile);
    bf16x8 wf[KT][2][2], wl[KT > LS ? KT - LS : 1][2];
    auto weights = [&](auto times_up) {
        constexpr bool UP = decltype(times_up)::value;
        uint32_t low = 0xFFFFFFFFu;
        int col = wcol, q = lq;
        // the second, rare pass forms its addresses anew and takes one fragment after the other: nothing is kept for it
        if constexpr (UP) asm volatile("" : "+v"(col), "+v"(q));
#pragma unroll
        for (int s = 0; s < KT; ++s)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int c = min(col + 4 * b, a.N - 1), k0 = 32 * s + 8 * q;        // eight k of one column
                float x[8];
                if (TRANS && k0 + 8 <= a.K) {
                    const f32x4_any* p = reinterpret_cast<const f32x4_any*>(W + (int64_t)c * a.K + k0);
                    const f32x4 u = p[0], v = p[1];
#pragma unroll
                    for (int e = 0; e < 4; ++e) { x[e] = u[e]; x[4 + e] = v[e]; }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int64_t k = min(k0 + e, a.K - 1);
                        const float v = TRANS ? W[(int64_t)c * a.K + k] : W[k * a.N + c];
                        x[e] = k0 + e < a.K ? v : 0.f;
                    }
                }
                low = least(x, low);
                if constexpr (UP) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] *= kUp;
                }
                bf16x8 f[3];
                split8(x, f);
                wf[s][b][0] = f[0];
                wf[s][b][1] = f[1];
                if (s < LS) wlds[(2 * s + b) * 512 + tid] = f[2];
                else wl[s - LS][b] = f[2];
                if constexpr (UP) __builtin_amdgcn_sched_barrier(0);
            }
        if (low < kLeast) *low_w = 1;
    };
    weights(std::false_type());
    if (tile < n_tiles) stage(0);
    if (tile + step < n_tiles) fetch(tile + step);
    __syncthreads();
    const bool scaled_w = __builtin_amdgcn_readfirstlane(*low_w) != 0;
    if (scaled_w) weights(std::true_type());           // (a lane's pieces in LDS are its own)

    const int ocol = c0 + 8 * lq;                                     // the lane's eight output columns
    const bool cols = c0 + 32 <= a.N;
    float kv[MASK ? RB : 1][8];
    auto mask_rows = [&](int64_t m, int rb) {
        if constexpr (MASK) {
            const float* x = reinterpret_cast<const float*>(a.mask) + (m < a.M ? m : a.M - 1) * a.ldmask + ocol;
            if (cols) {
                const f32x4 u = *reinterpret_cast<const f32x4_any*>(x), w = *reinterpret_cast<const f32x4_any*>(x + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { kv[rb][e] = u[e]; kv[rb][4 + e] = w[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) kv[rb][e] = ocol + e < a.N ? x[e] : 0.f;
            }
        }
    };
    // the lane's eight columns of row m
    auto store = [&](int64_t m, int rb, const f32x4 (&acc)[2]) {
        if (m >= a.M) return;
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = a.c_w * acc[e >> 2][e & 3];
        if (a.bias) {
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] += cols || ocol + e < a.N ? reinterpret_cast<const float*>(a.bias)[ocol + e] : 0.f;
        }
        if (a.relu) {
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = fmaxf(y[e], 0.f);
        }
        if constexpr (MASK) {
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = kv[rb][e] > 0.f ? y[e] : 0.f;
        }
        auto put = [&](float* to) {
            if (cols) {
                *reinterpret_cast<f32x4_any*>(to) = f32x4{y[0], y[1], y[2], y[3]};
                *reinterpret_cast<f32x4_any*>(to + 4) = f32x4{y[4], y[5], y[6], y[7]};
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (ocol + e < a.N) to[e] = y[e];
            }
        };
        put(reinterpret_cast<float*>(a.Y) + m * a.ldy + ocol);
        if (a.push_idx) put(reinterpret_cast<float*>(a.push_hist) + (int64_t)a.push_idx[m] * a.ld_push + ocol);
    };
    // the wavefront's columns of 16 rows by the fp32 instruction: four k, one of them a lane's
    auto plain = [&](int64_t m, f32x4 (&acc)[2]) {
        const float* z = Z + (m < a.M ? m : a.M - 1) * a.ldz;
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int k0 = 0; k0 < a.K; k0 += 4) {
            const int64_t k = min(k0 + lq, a.K - 1);
            const bool in = k0 + lq < a.K;
            const float x = in ? z[k] : 0.f;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int64_t c = min(wcol + 4 * b, a.N - 1);
                const float w = TRANS ? W[c * a.K + k] : W[k * a.N + c];
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? w : 0.f, x, acc[b], 0, 0, 0);
            }
        }
    };

    // the large product between two small ones: its sums do not wait for theirs
    constexpr int PZ[6] = {1, 0, 0, 1, 2, 0}, PW[6] = {0, 0, 1, 1, 0, 2}, kLarge = 1;
    const bool early = wave < 4;
    int it = 0;
#pragma unroll 1
    for (; tile < n_tiles; tile += step, ++it) {
        auto advance = [&]() {
            if (tile + step < n_tiles) stage(it + 1);
            if (tile + 2 * step < n_tiles) fetch(tile + 2 * step);
        };
        const bool scaled = __builtin_amdgcn_readfirstlane(low_tile[it & 3]) != 0;         // set before the last barrier
        if (tid == 0) low_tile[(it + 3) & 3] = 0;                                           // the tile before: read by all
        if (scaled) {                                      // staged again, then what was on its way is fetched again
            fetch(tile);
            if (stages) {
                if (a.K != 32 * KT) trim();
#pragma unroll
                for (int e = 0; e < 8; ++e) raw[e] *= kUp;
                write(it);
            }
            if (tile + step < n_tiles) fetch(tile + step);
            __syncthreads();
        }
        if (early) advance();
        if (c0 < a.N) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) mask_rows(tile * ROWS + 16 * rb + li, rb);
            // piece 4 s + lq of row li (+ 16 rb) lies at piece ^ (row & 7): two addresses and constants
            const uint16_t* zp[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) zp[h] = planes + (it & 1) * 3 * PLANE + li * PITCH + 8 * ((4 * h + lq) ^ (li & 7));
            f32x4 acc[RB][2], small[RB][2];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[rb][b] = small[rb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            // Step i = s RB + rb.  The first two parts of its rows are read from LDS one step ahead of its products, the
            // operands of its last two products (third parts) before its first ones.
            bf16x8 z[2][2], z2, third[2];
            auto ahead = [&](int i) {
                const int s = i / RB, rb = i % RB;
#pragma unroll
                for (int part = 0; part < 2; ++part)
                    z[i & 1][part] = *reinterpret_cast<const bf16x8*>(zp[s & 1] + part * PLANE + 16 * rb * PITCH + 64 * (s >> 1));
            };
            ahead(0);
#pragma unroll
            for (int i = 0; i < KT * RB; ++i) {
                const int s = i / RB, rb = i % RB;
                z2 = *reinterpret_cast<const bf16x8*>(zp[s & 1] + 2 * PLANE + 16 * rb * PITCH + 64 * (s >> 1));
#pragma unroll
                for (int b = 0; b < 2; ++b) third[b] = s < LS ? wlds[(2 * s + b) * 512 + tid] : wl[s < LS ? 0 : s - LS][b];
                if (i + 1 < KT * RB) ahead(i + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        f32x4& c = t == kLarge ? acc[rb][b] : small[rb][b];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(PW[t] == 2 ? third[b] : wf[s][b][PW[t] & 1],
                                                                    PZ[t] == 2 ? z2 : z[i & 1][PZ[t] & 1], c, 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            float bad = 0.f;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    acc[rb][b] += small[rb][b];
                    if (scaled || scaled_w) {
                        if (scaled) acc[rb][b] *= 1.f / kUp;
                        if (scaled_w) acc[rb][b] *= 1.f / kUp;
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) bad = fmaf(acc[rb][b][r], 0.f, bad);      // stays 0 for finite values, else NaN
                }
            if (__any(bad != 0.f)) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) plain(tile * ROWS + 16 * rb + li, acc[rb]);
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) store(tile * ROWS + 16 * rb + li, rb, acc[rb]);
        }
        if (!early) advance();
        __syncthreads();
    }
}

// fp32 fused MLP: 32 rows per workgroup; wavefront w owns hidden / output
// columns [64w, 64w+64).  Phase 1 leaves relu(Z W1 + b1) in LDS (fp32), phase 2
// multiplies it by W2 with the hidden tile as the A operand.
template <bool VEC>
__global__ __launch_bounds__(256) void mlp2_f32_kernel(MlpArgs a) {
    constexpr int BM = kMlpRowsF32, BN = 256, TN = 2;
    constexpr int kLdH = kHidMax + 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];   // above the 64 KB static limit
    float (*Hs)[kLdH] = reinterpret_cast<float (*)[kLdH]>(smem);
    float (*As)[kLdA] = reinterpret_cast<float (*)[kLdA]>(smem + sizeof(float) * BM * kLdH);
    float (*Bs)[BN + 4] = reinterpret_cast<float (*)[BN + 4]>(smem + sizeof(float) * BM * (kLdH + kLdA));
    const float* Z = reinterpret_cast<const float*>(a.Z);
    const float* W1 = reinterpret_cast<const float*>(a.W1);
    const float* W2 = reinterpret_cast<const float*>(a.W2);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int wn0 = wave * 64;
    f32x16 acc[1][TN];
    zero_acc(acc);
    ATileF32<BM, VEC> ta;
    BTileF32<BN, VEC> tb;
    ta.fetch(Z, a.ldz, a.M, a.K, m0, 0, tid);
    tb.fetch(W1, a.K, a.H, 0, 0, tid);
    for (int k0 = 0; k0 < a.K; k0 += kBK) {
        __syncthreads();
        ta.stage(As, tid);
        tb.stage(Bs, tid);
        __syncthreads();
        if (k0 + kBK < a.K) {
            ta.fetch(Z, a.ldz, a.M, a.K, m0, k0 + kBK, tid);
            tb.fetch(W1, a.K, a.H, k0 + kBK, 0, tid);
        }
        mfma_tile_f32<1, TN, BN>(&As[0][0], kLdA, 0, 0, Bs, wn0, li, lh, acc);
    }
    const float* b1 = reinterpret_cast<const float*>(a.b1);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int h = wn0 + 32 * j + li;
        const float bv = (b1 && h < a.H) ? b1[h] : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            Hs[8 * (r / 4) + 4 * lh + (r % 4)][h] = h < a.H ? fmaxf(acc[0][j][r] + bv, 0.f) : 0.f;
    }
    zero_acc(acc);
    tb.fetch(W2, a.H, a.N, 0, n0, tid);
    for (int k0 = 0; k0 < a.H; k0 += kBK) {
        __syncthreads();                 // Hs written / previous Bs consumed
        tb.stage(Bs, tid);
        __syncthreads();
        if (k0 + kBK < a.H) tb.fetch(W2, a.H, a.N, k0 + kBK, n0, tid);
        mfma_tile_f32<1, TN, BN>(&Hs[0][0], kLdH, 0, k0, Bs, wn0, li, lh, acc);
    }
    float* Y = reinterpret_cast<float*>(a.Y);
    const float* b2 = reinterpret_cast<const float*>(a.b2);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn0 + 32 * j + li;
        if (n >= a.N) continue;
        const float bv = b2 ? b2[n] : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t m = m0 + 8 * (r / 4) + 4 * lh + (r % 4);
            if (m >= a.M) continue;
            float y = acc[0][j][r] + bv;
            if (a.relu_out) y = fmaxf(y, 0.f);
            Y[m * a.ldy + n] = y;
        }
    }
}

// ====================================================================== bf16
constexpr int kBKh = 64;            // k per tile
constexpr int kLdh = kBKh + 8;      // padded LDS row, in bf16 elements

__device__ __forceinline__ void transpose8x8_bf16(const u32x4 (&in)[8], u32x4 (&out)[8]) {
    // in[r] holds n = 0..7 of k-row r (two per dword); out[c] holds k = 0..7 of column c
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t lo = in[2 * q][c >> 1], hi = in[2 * q + 1][c >> 1];
            out[c][q] = (c & 1) ? ((lo >> 16) | (hi & 0xFFFF0000u)) : ((lo & 0xFFFFu) | (hi << 16));
        }
}

template <int BM>
struct ATileBF16 {
    static constexpr int NV = BM * kBKh / 8 / 256;
    u32x4 r[NV];
    __device__ __forceinline__ void fetch(const uint16_t* Z, int64_t ld, int64_t M, int K, int64_t m0, int k0, int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            const int64_t m = m0 + (idx >> 3);
            const int k = k0 + 8 * (idx & 7);
            r[i] = u32x4{0u, 0u, 0u, 0u};
            if (m < M && k < K) r[i] = *reinterpret_cast<const u32x4*>(Z + m * ld + k);
        }
    }
    __device__ __forceinline__ void stage(uint16_t (*As)[kLdh], int tid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            *reinterpret_cast<u32x4*>(&As[idx >> 3][8 * (idx & 7)]) = r[i];
        }
    }
};

// One kBKh x BN tile of a bf16 weight matrix into Bs[n][k].  Row-major [K][N]: transposed on the way (8 x 8
// blocks).  trans (the matrix is [N][K] row-major): already in the layout the MFMA wants, plain 16-byte copies.
template <int BN>
struct BTileBF16 {
    u32x4 r[8];
    __device__ __forceinline__ void fetch(const uint16_t* W, int K, int N, int k0, int n0, int tid, bool trans = false) {
        if (!trans) {
            if (tid >= BN) return;              // kBKh/8 * BN/8 = BN blocks of 8 x 8
            const int kb = tid / (BN / 8), n = n0 + 8 * (tid % (BN / 8));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = k0 + 8 * kb + i;
                r[i] = u32x4{0u, 0u, 0u, 0u};
                if (k < K && n < N) r[i] = *reinterpret_cast<const u32x4*>(W + (int64_t)k * N + n);
            }
        } else {
#pragma unroll
            for (int i = 0; i < BN / 32; ++i) {  // BN * 8 pieces of 16 bytes over 256 threads
                const int idx = tid + 256 * i;
                const int n = n0 + (idx >> 3), k = k0 + 8 * (idx & 7);
                r[i] = u32x4{0u, 0u, 0u, 0u};
                if (n < N && k < K) r[i] = *reinterpret_cast<const u32x4*>(W + (int64_t)n * K + k);
            }
        }
    }
    __device__ __forceinline__ void stage(uint16_t (*Bs)[kLdh], int tid, bool trans = false) {
        if (!trans) {
            if (tid >= BN) return;
            const int kb = tid / (BN / 8), nb = tid % (BN / 8);
            u32x4 t[8];
            transpose8x8_bf16(r, t);
#pragma unroll
            for (int c = 0; c < 8; ++c) *reinterpret_cast<u32x4*>(&Bs[8 * nb + c][8 * kb]) = t[c];
        } else {
#pragma unroll
            for (int i = 0; i < BN / 32; ++i) {
                const int idx = tid + 256 * i;
                *reinterpret_cast<u32x4*>(&Bs[idx >> 3][8 * (idx & 7)]) = r[i];
            }
        }
    }
};

template <int TM, int TN>
__device__ __forceinline__ void mfma_tile_bf16(const uint16_t* A, int lda, int arow0, int acol0,
                                               const uint16_t (*Bs)[kLdh], int brow0, int li, int lh,
                                               f32x16 (&acc)[TM][TN]) {
#pragma unroll
    for (int kk = 0; kk < kBKh / 16; ++kk) {
        bf16x8 fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(A + (arow0 + 32 * i + li) * lda + acol0 + kk * 16 + 8 * lh));
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fb[j] = __builtin_bit_cast(bf16x8,
                                       *reinterpret_cast<const u32x4*>(&Bs[brow0 + 32 * j + li][kk * 16 + 8 * lh]));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
}

// y = act(c_w acc + bias + c_id Z), masked, of a wavefront's blocks, two bytes a lane
template <int TM, int TN>
__device__ __forceinline__ void store_tile_bf16(const LinArgs& a, int64_t m0, int n0, int li, int lh, const f32x16 (&acc)[TM][TN]) {
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    uint16_t* Y = reinterpret_cast<uint16_t*>(a.Y);
    const uint16_t* bias = reinterpret_cast<const uint16_t*>(a.bias);
    const uint16_t* mask = reinterpret_cast<const uint16_t*>(a.mask);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + 32 * j + li;
            if (n >= a.N) continue;
            const float bv = bias ? bf16_val(bias, n) : 0.f;
            float id[16], keep[16];          // asked for together
            const int64_t mj = m0 + 32 * i + 4 * lh;
            if (a.c_id != 0.f)
#pragma unroll
                for (int r = 0; r < 16; ++r) id[r] = bf16_val(Z, min(mj + 8 * (r / 4) + r % 4, a.M - 1) * a.ldz + n);
            if (mask)
#pragma unroll
                for (int r = 0; r < 16; ++r) keep[r] = bf16_val(mask, min(mj + 8 * (r / 4) + r % 4, a.M - 1) * a.ldmask + n);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = mj + 8 * (r / 4) + r % 4;
                if (m >= a.M) continue;
                float y = a.c_w * acc[i][j][r] + bv;
                if (a.c_id != 0.f) y += a.c_id * id[r];
                if (a.relu) y = fmaxf(y, 0.f);
                if (mask && !(keep[r] > 0.f)) y = 0.f;
                Y[m * a.ldy + n] = (uint16_t)f32_to_bf16(y);
            }
        }
}

// One ROWS x kBKh tile of a bf16 operand whose rows need no alignment beyond their elements', into LDS as [row][q], q the reduced
// index; KC: element (r, q) lies at X[r ld + q], else at X[q ld + r].  Loads are of single elements, a wavefront's side by side
// from an address that it shares (an address a lane takes 100 registers more).  Turned, a lane keeps eight q of its row and writes
// them as 16 bytes.  Rows beyond the last repeat it (nothing stores their products), q beyond the end come out zero.
template <int ROWS, bool KC, int WAVES = 4>
struct AnyTileBF16 {
    static constexpr int NV = ROWS * kBKh / 2 / (64 * WAVES);
    uint16_t lo[NV], hi[NV];      // packed on the way into LDS: before, each pair would be waited for before the next is asked for
    typedef const __attribute__((address_space(1))) char* Row;
    // the next row's address, if there is one: in scalar registers, and not before the row at hand is asked for
    static __device__ __forceinline__ void step(Row& x, int64_t ld, bool more) {
        x += more ? 2 * ld : 0;
        asm volatile("" : "+s"(x) : : "memory");
    }
    static __device__ __forceinline__ uint16_t at(Row x, uint32_t byte) {
        return *reinterpret_cast<const __attribute__((address_space(1))) uint16_t*>(x + byte);
    }
    __device__ __forceinline__ void fetch(const uint16_t* X, int64_t ld, int64_t r0, int64_t r_end, int64_t q0, int64_t q_end, int tid) {
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        const int last = (int)min(r_end - 1 - r0, (int64_t)ROWS), q_last = (int)min(q_end - 1 - q0, (int64_t)kBKh);
        if constexpr (KC) {
            const uint32_t q = 2u * (uint32_t)min(lane, q_last);
            const int row = wave * (ROWS / WAVES);
            Row x = (Row)(X + (r0 + min(row, last)) * ld + q0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                lo[i] = at(x, q);
                step(x, ld, row + 2 * i < last);
                hi[i] = at(x, q);
                step(x, ld, row + 2 * i + 1 < last);
            }
        } else {
#pragma unroll
            for (int u = 0; u < NV / 4; ++u) {
                const int unit = wave * (NV / 4) + u, q = unit / (ROWS / 64) * 8;
                const uint32_t row = 2u * (uint32_t)min(unit % (ROWS / 64) * 64 + lane, last);
                Row x = (Row)(X + (q0 + min(q, q_last)) * ld + r0);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    lo[4 * u + c] = at(x, row);
                    step(x, ld, q + 2 * c < q_last);
                    hi[4 * u + c] = at(x, row);
                    step(x, ld, q + 2 * c + 1 < q_last);
                }
            }
        }
    }
    // left: q of the step inside
    __device__ __forceinline__ void stage(uint16_t (*to)[kLdh], int64_t left, int tid) {
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        if constexpr (KC) {
            const bool in = lane < left;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                to[wave * (ROWS / WAVES) + 2 * i][lane] = in ? lo[i] : (uint16_t)0;
                to[wave * (ROWS / WAVES) + 2 * i + 1][lane] = in ? hi[i] : (uint16_t)0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < NV / 4; ++u) {
                const int unit = wave * (NV / 4) + u, q = unit / (ROWS / 64) * 8;
                u32x4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = ((uint32_t)lo[4 * u + c] | (uint32_t)hi[4 * u + c] << 16) & (q + 2 * c + 1 < left ? 0xFFFFFFFFu : (q + 2 * c < left ? 0xFFFFu : 0u));
                *reinterpret_cast<u32x4*>(&to[unit % (ROWS / 64) * 64 + lane][q]) = v;
            }
        }
    }
};

// Y tile of BM x BN by operands of any alignment and width (odd feature and class counts).  Bound by its loads, of two bytes a lane:
// 16 of every row and column of a step's 64 k a wavefront, so 64 and 32 matrix instructions at 128 x 128.  A thread an output
// before: 50,000 x 256 x 47 312 us and now 14, its input gradient 609 and 18, 256 x 250 1,059 and 31, 11,287 and 30; 500 x 256 x 47 32 and 7.
template <int BM, int BN, bool TRANS>
__global__ __launch_bounds__(256, 2) void linear_bf16_any_kernel(LinArgs a) {
    constexpr int TM = BM / 64, TN = BN / 64;
    __shared__ __attribute__((aligned(16))) uint16_t As[BM][kLdh];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[BN][kLdh];
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const unsigned tn = (unsigned)((a.N + BN - 1) / BN), of_xcd = blockIdx.x / 8;   // a row tile's column tiles follow each other on one XCD
    const int64_t m0 = ((int64_t)(of_xcd / tn) * 8 + blockIdx.x % 8) * BM;
    const int n0 = (int)(of_xcd % tn) * BN;
    if (m0 >= a.M) return;
    const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
    f32x16 acc[TM][TN];
    zero_acc(acc);
    AnyTileBF16<BM, true> ta;
    AnyTileBF16<BN, TRANS> tb;
    const int64_t ldw = TRANS ? a.K : a.N;
    ta.fetch(Z, a.ldz, m0, a.M, 0, a.K, tid);
    tb.fetch(W, ldw, n0, a.N, 0, a.K, tid);
    for (int k0 = 0; k0 < a.K; k0 += kBKh) {
        __syncthreads();
        ta.stage(As, a.K - k0, tid);
        tb.stage(Bs, a.K - k0, tid);
        __syncthreads();
        if (k0 + kBKh < a.K) {
            ta.fetch(Z, a.ldz, m0, a.M, k0 + kBKh, a.K, tid);
            tb.fetch(W, ldw, n0, a.N, k0 + kBKh, a.K, tid);
        }
        mfma_tile_bf16<TM, TN>(&As[0][0], kLdh, wm0, 0, Bs, wn0, li, lh, acc);
    }
    store_tile_bf16<TM, TN>(a, m0 + wm0, n0 + wn0, li, lh, acc);
}

// Y tile of BM x BN, 16-byte loads.  A step's loads are under way while the one before is multiplied; where the units hold few
// tiles, their latency and the turning of W bound it, so tiles are small (64 x 64 at 500 x 256 x 256 7.2 us, 128 x 256 20.1).
template <int BM, int BN>
__global__ __launch_bounds__(256) void linear_bf16_kernel(LinArgs a) {
    constexpr int TM = BM / 64, TN = BN / 64;
    __shared__ __attribute__((aligned(16))) uint16_t As[BM][kLdh];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[BN][kLdh];
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const unsigned tn = (unsigned)((a.N + BN - 1) / BN), of_xcd = blockIdx.x / 8;   // a row tile's column tiles follow each other on one XCD
    const int64_t m0 = ((int64_t)(of_xcd / tn) * 8 + blockIdx.x % 8) * BM;
    const int n0 = (int)(of_xcd % tn) * BN;
    if (m0 >= a.M) return;
    const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
    f32x16 acc[TM][TN];
    zero_acc(acc);
    ATileBF16<BM> ta;
    BTileBF16<BN> tb;
    const bool tr = a.trans_w != 0;
    ta.fetch(Z, a.ldz, a.M, a.K, m0, 0, tid);
    tb.fetch(W, a.K, a.N, 0, n0, tid, tr);
    for (int k0 = 0; k0 < a.K; k0 += kBKh) {
        __syncthreads();
        ta.stage(As, tid);
        tb.stage(Bs, tid, tr);
        __syncthreads();
        if (k0 + kBKh < a.K) {
            ta.fetch(Z, a.ldz, a.M, a.K, m0, k0 + kBKh, tid);
            tb.fetch(W, a.K, a.N, k0 + kBKh, n0, tid, tr);
        }
        mfma_tile_bf16<TM, TN>(&As[0][0], kLdh, wm0, 0, Bs, wn0, li, lh, acc);
    }
    store_tile_bf16<TM, TN>(a, m0 + wm0, n0 + wn0, li, lh, acc);
}

// bf16 fused MLP: 64 rows per workgroup, wavefronts 2 x 2 over (rows, columns).
// Phase 1: hidden = relu(Z W1 + b1) for all F_hid columns, rounded to bf16 into
// LDS.  Phase 2: Y = act(hidden W2 + b2), the hidden tile being the A operand.
// ANY: operands of any alignment and width (AnyTileBF16), by eight wavefronts, whose loads bound it.  A workgroup a row before:
// 50,000 x 81 -> 184 -> 184 429 us and now 44, 500 rows 16.6 and 14.7 (by four wavefronts 19.8).
template <bool ANY>
__global__ __launch_bounds__(ANY ? 512 : 256) void mlp2_bf16_kernel(MlpArgs a) {
    constexpr int BM = kMlpRowsBF16, BN = 256, TN = ANY ? 2 : 4;
    constexpr int kLdHid = kHidMax + 8;
    extern __shared__ __attribute__((aligned(16))) char smem[];   // above the 64 KB static limit
    uint16_t (*Hs)[kLdHid] = reinterpret_cast<uint16_t (*)[kLdHid]>(smem);
    uint16_t (*As)[kLdh] = reinterpret_cast<uint16_t (*)[kLdh]>(smem + 2 * BM * kLdHid);
    uint16_t (*Bs)[kLdh] = reinterpret_cast<uint16_t (*)[kLdh]>(smem + 2 * BM * (kLdHid + kLdh));
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* W1 = reinterpret_cast<const uint16_t*>(a.W1);
    const uint16_t* W2 = reinterpret_cast<const uint16_t*>(a.W2);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int wm0 = (wave / (8 / TN)) * 32, wn0 = wave % (8 / TN) * (32 * TN);
    f32x16 acc[1][TN];
    zero_acc(acc);
    std::conditional_t<ANY, AnyTileBF16<BM, true, 8>, ATileBF16<BM>> ta;
    std::conditional_t<ANY, AnyTileBF16<BN, false, 8>, BTileBF16<BN>> tb;
    auto rows = [&](int k0) {
        if constexpr (ANY) ta.fetch(Z, a.ldz, m0, a.M, k0, a.K, tid);
        else ta.fetch(Z, a.ldz, a.M, a.K, m0, k0, tid);
    };
    auto weights = [&](const uint16_t* W, int K, int N, int k0, int c0) {
        if constexpr (ANY) tb.fetch(W, N, c0, N, k0, K, tid);
        else tb.fetch(W, K, N, k0, c0, tid);
    };
    auto stage_weights = [&](int left) {
        if constexpr (ANY) tb.stage(Bs, left, tid);
        else tb.stage(Bs, tid);
    };
    rows(0);
    weights(W1, a.K, a.H, 0, 0);
    for (int k0 = 0; k0 < a.K; k0 += kBKh) {
        __syncthreads();
        if constexpr (ANY) ta.stage(As, a.K - k0, tid);
        else ta.stage(As, tid);
        stage_weights(a.K - k0);
        __syncthreads();
        if (k0 + kBKh < a.K) {
            rows(k0 + kBKh);
            weights(W1, a.K, a.H, k0 + kBKh, 0);
        }
        mfma_tile_bf16<1, TN>(&As[0][0], kLdh, wm0, 0, Bs, wn0, li, lh, acc);
    }
    const uint16_t* b1 = reinterpret_cast<const uint16_t*>(a.b1);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int h = wn0 + 32 * j + li;
        const float bv = (b1 && h < a.H) ? bf16_val(b1, h) : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = h < a.H ? fmaxf(acc[0][j][r] + bv, 0.f) : 0.f;
            Hs[wm0 + 8 * (r / 4) + 4 * lh + (r % 4)][h] = (uint16_t)f32_to_bf16(v);
        }
    }
    zero_acc(acc);
    weights(W2, a.H, a.N, 0, n0);
    for (int k0 = 0; k0 < a.H; k0 += kBKh) {
        __syncthreads();                 // Hs written / previous Bs consumed
        stage_weights(a.H - k0);
        __syncthreads();
        if (k0 + kBKh < a.H) weights(W2, a.H, a.N, k0 + kBKh, n0);
        mfma_tile_bf16<1, TN>(&Hs[0][0], kLdHid, wm0, k0, Bs, wn0, li, lh, acc);
    }
    uint16_t* Y = reinterpret_cast<uint16_t*>(a.Y);
    const uint16_t* b2 = reinterpret_cast<const uint16_t*>(a.b2);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn0 + 32 * j + li;
        if (n >= a.N) continue;
        const float bv = b2 ? bf16_val(b2, n) : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t m = m0 + wm0 + 8 * (r / 4) + 4 * lh + (r % 4);
            if (m >= a.M) continue;
            float y = acc[0][j][r] + bv;
            if (a.relu_out) y = fmaxf(y, 0.f);
            Y[m * a.ldy + n] = (uint16_t)f32_to_bf16(y);
        }
    }
}

// ---------------------------------------------------------------------- weights-stationary bf16 kernels
// For feature widths up to 256 the whole weight matrix fits in the registers
// of one workgroup: wavefront w of 8 keeps the MFMA B-fragments of columns
// [32w, 32w+32) for every k (K/16 fragments of 8 bf16 per lane), loaded once.
// The workgroup is persistent (one per compute unit) and streams 64-row tiles
// of Z through LDS, so after start-up the only global traffic is Z in and Y
// out: the weights are never re-staged.  ws_bf16_kernel is the single product;
// ws_mlp_bf16_kernel keeps W1 and W2 on separate wavefronts and chains the two
// products of the GIN MLP through an LDS-resident hidden tile.
struct WsArgs {
    const uint16_t* Z;  int64_t ldz;
    const uint16_t* W1; const uint16_t* b1;
    const uint16_t* W2; const uint16_t* b2;
    uint16_t* Y;        int64_t ldy;
    int64_t M, n_tiles;
    int K, H, N;        // single product: H == N is the output width and W2 is unused
    float c_id, c_w;
    int relu1, relu_out;
    int trans_w1;                          // W1 is given as [H][K] (single product only)
    const uint16_t* mask; int64_t ldmask;  // optional [M, N]: outputs where mask <= 0 are set to zero
    const int32_t* push_idx;               // optional: output row m is also stored to push_hist[push_idx[m], :]
    uint16_t* push_hist; int64_t ld_push;
    uint16_t* H_out; int64_t ldh_out;      // optional (fused MLP): the hidden activation is stored as well
};

constexpr int kWsRows = 64;

template <int KT>
__device__ __forceinline__ void load_w_frags(const uint16_t* W, int K, int ncols, int col, int lh, bf16x8 (&f)[KT],
                                             bool trans = false) {
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (trans) {                     // [ncols][K] row-major, K a multiple of 8: the fragment is contiguous
            const int k = 16 * kk + 8 * lh;
            if (k < K && col < ncols) v = *reinterpret_cast<const u32x4*>(W + (int64_t)col * K + k);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 16 * kk + 8 * lh + e;
                uint32_t x = 0;
                if (k < K && col < ncols) x = W[(int64_t)k * ncols + col];
                v[e >> 1] |= x << (16 * (e & 1));
            }
        }
        f[kk] = __builtin_bit_cast(bf16x8, v);
    }
}

// The products are evaluated transposed, D' = W^T Z^T: the weight fragment is
// the MFMA A operand and the Z fragment the B operand (both hold 8 consecutive
// k of one row/column, so the register contents are what they would be the
// other way round).  Then a lane holds, for ONE row m of the tile, 4 groups of
// 4 consecutive output columns, which go to the [m][n] LDS tiles as 8-byte
// stores after a packed hardware fp32->bf16 conversion.
template <int KT1, bool MASK>
__global__ __launch_bounds__(512) void ws_bf16_kernel(WsArgs a) {
    constexpr int LDA = 16 * KT1 + 8;                 // bf16 elements per LDS row of the Z tile
    constexpr int LDY = 256 + 8;                      // ... of the output staging tile
    constexpr int VPR = 2 * KT1;                      // 16-byte vectors per Z-tile row
    constexpr int NVA = (kWsRows * VPR + 511) / 512;  // vectors per thread per tile
    constexpr int MT = kWsRows / 32;                  // 32-row blocks per tile
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);                       // [2][64][LDA]
    uint16_t* Ys = As + 2 * kWsRows * LDA;                                  // [64][LDY]
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // the same in every lane, and known to be

    bf16x8 w1f[KT1];
    load_w_frags<KT1>(a.W1, a.K, a.H, 32 * wave + li, lh, w1f, a.trans_w1 != 0);
    // output columns of this lane: n(q, e) = 32*wave + 8*q + 4*lh + e, q, e in 0..3
    const int nbase = 32 * wave + 4 * lh;
    // bias as fp32 in LDS (read back four at a time in the epilogue: registers are what this kernel is short of)
    float* bias1 = reinterpret_cast<float*>(Ys + kWsRows * LDY);            // [256]
    if (tid < 256) bias1[tid] = (a.b1 && tid < a.H) ? bf16_val(a.b1, tid) : 0.f;

    // Loads are issued unconditionally from a clamped address and zeroed by a select afterwards: with no
    // branch around them the compiler counts outstanding memory operations exactly, and a later wait for one
    // load does not turn into a wait for everything in flight.
    u32x4 ra[NVA];
    const bool k_whole = a.K == 16 * KT1;
    auto fetch = [&](int64_t tile) {
        const uint16_t* base = a.Z + tile * kWsRows * a.ldz;      // the same for every lane; offsets are 32-bit
        const bool full = k_whole && (tile + 1) * kWsRows <= a.M;
#pragma unroll
        for (int i = 0; i < NVA; ++i) {
            const int idx = tid + 512 * i;
            const int row = idx / VPR, k = 8 * (idx % VPR);
            uint32_t off = (uint32_t)row * (uint32_t)a.ldz + (uint32_t)k;
            if (!full) {
                const bool ok = idx < kWsRows * VPR && tile * kWsRows + row < a.M && k < a.K;
                off = ok ? off : 0u;
            } else if (kWsRows * VPR % 512 != 0 && idx >= kWsRows * VPR) {
                off = 0u;
            }
            ra[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off));
        }
    };
    auto stage = [&](int buf, int64_t tile) {          // tile: the one fetch() was called for
        const bool full = k_whole && (tile + 1) * kWsRows <= a.M;
#pragma unroll
        for (int i = 0; i < NVA; ++i) {
            const int idx = tid + 512 * i;
            const int row = idx / VPR, k = 8 * (idx % VPR);
            u32x4 v = ra[i];
            if (!full) {
                const bool ok = tile * kWsRows + row < a.M && k < a.K;
                v = ok ? v : u32x4{0u, 0u, 0u, 0u};
            }
            if (idx < kWsRows * VPR) *reinterpret_cast<u32x4*>(As + (buf * kWsRows + row) * LDA + k) = v;
        }
    };

    // Order of memory operations per tile: the loads of the tile after next are issued BEFORE this tile's
    // output stores and are consumed one iteration later, so they are in flight during the stores and the next
    // tile's MFMAs, and waiting for them never waits for a store (loads and stores retire in issue order).
    constexpr int NPI = (kWsRows * 32 + 511) / 512;   // output vectors per thread per tile at the widest row
    int64_t tile = blockIdx.x;
    if (tile < a.n_tiles) {
        fetch(tile);
        stage(0, tile);
        if (tile + gridDim.x < a.n_tiles) fetch(tile + gridDim.x);
    }
    int buf = 0;
    for (; tile < a.n_tiles; tile += gridDim.x, buf ^= 1) {
        const int64_t next = tile + gridDim.x;
        __syncthreads();                               // (1) Z tile `buf` staged; previous tile fully consumed
        // output vector (row, v) of a thread: row = tid / 32 + 16 i, v = tid % 32 (the staging tile is 32 vectors
        // wide; narrower outputs leave the lanes beyond their width idle)
        const bool out_full = (tile + 1) * kWsRows <= a.M;
        int32_t prow[NPI] = {};                        // history slots of the rows this thread will store
        if (a.push_idx) {
            const int32_t* pi = a.push_idx + tile * kWsRows;
#pragma unroll
            for (int i = 0; i < NPI; ++i) {
                int row = (tid >> 5) + 16 * i;
                if (!out_full) row = tile * kWsRows + row < a.M ? row : 0;
                prow[i] = pi[row];
            }
        }
        // the mask's rows are requested a product ahead of their use (312,500 rows, 256 x 256: 112 -> 98 us; asked for where
        // they are used they wait for the next tile's rows as well)
        u32x4 km[NPI];
        if constexpr (MASK) {
            const uint16_t* mbase = a.mask + tile * kWsRows * a.ldmask;
#pragma unroll
            for (int i = 0; i < NPI; ++i) {
                const int row = (tid >> 5) + 16 * i, v = tid & 31;
                const bool ok = v < (a.N >> 3) && (out_full || tile * kWsRows + row < a.M);
                km[i] = *reinterpret_cast<const u32x4*>(mbase + (ok ? (uint32_t)row * (uint32_t)a.ldmask + 8u * v : 0u));
            }
        }
        const uint16_t* At = As + buf * kWsRows * LDA;
        f32x16 acc[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
        if (32 * wave < a.H) {
#pragma unroll
            for (int kk = 0; kk < KT1; ++kk)
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const bf16x8 fz = __builtin_bit_cast(
                        bf16x8, *reinterpret_cast<const u32x4*>(At + (32 * t + li) * LDA + 16 * kk + 8 * lh));
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1f[kk], fz, acc[t], 0, 0, 0);
                }
        }
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
                const f32x4 bq = *reinterpret_cast<const f32x4*>(bias1 + nbase + 8 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = a.c_w * acc[t][4 * q + e] + bq[e];
                if (a.c_id != 0.f && nbase + 8 * q < a.N) {      // identity term straight from the staged Z tile (K == N)
                    const u32x2 z = *reinterpret_cast<const u32x2*>(At + (32 * t + li) * LDA + nbase + 8 * q);
                    v[0] += a.c_id * bf16_lo(z[0]); v[1] += a.c_id * bf16_hi(z[0]);
                    v[2] += a.c_id * bf16_lo(z[1]); v[3] += a.c_id * bf16_hi(z[1]);
                }
                if (a.relu1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
                }
                *reinterpret_cast<u32x2*>(Ys + (32 * t + li) * LDY + nbase + 8 * q) =
                    u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
        // take delivery of the history slots and of the mask before new loads are queued behind them: the stores below then
        // need no wait that the loads just issued would have to satisfy first
#pragma unroll
        for (int i = 0; i < NPI; ++i) asm volatile("" : "+v"(prow[i]));
        if constexpr (MASK) {
#pragma unroll
            for (int i = 0; i < NPI; ++i) asm volatile("" : "+v"(km[i]));
        }
        if (next < a.n_tiles) {
            stage(buf ^ 1, next);                      // the other buffer: nobody reads it before the next (1)
            if (next + gridDim.x < a.n_tiles) fetch(next + gridDim.x);
        }
        __syncthreads();                               // (3) output tile staged
        {
            const int vpr = a.N >> 3;                  // 16-byte vectors per output row
            uint16_t* ybase = a.Y + tile * kWsRows * a.ldy;
            const int v = tid & 31;
            if (v < vpr) {
#pragma unroll
                for (int i = 0; i < NPI; ++i) {
                    const int row = (tid >> 5) + 16 * i;
                    if (out_full || tile * kWsRows + row < a.M) {
                        u32x4 o = *reinterpret_cast<const u32x4*>(Ys + row * LDY + 8 * v);
                        if constexpr (MASK) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                if (!(bf16_lo(km[i][q]) > 0.f)) o[q] &= 0xFFFF0000u;
                                if (!(bf16_hi(km[i][q]) > 0.f)) o[q] &= 0x0000FFFFu;
                            }
                        }
                        __builtin_nontemporal_store(
                            o, reinterpret_cast<u32x4*>(ybase + ((uint32_t)row * (uint32_t)a.ldy + 8u * v)));
                        if (a.push_idx)      // Push fused into the epilogue: the row goes to its history slot as well
                            __builtin_nontemporal_store(
                                o, reinterpret_cast<u32x4*>(a.push_hist + (int64_t)prow[i] * a.ld_push + 8 * v));
                    }
                }
            }
        }
    }
}

// Weight fragments for a 64-column block, through LDS: the [K][ncols] matrix is staged 128 rows at a time with
// 16-byte loads, and a lane picks the 8 consecutive k of its column out of the staged chunk (the MFMA operand
// wants the matrix transposed).  ncols is a multiple of 8 and W is 16-byte aligned.  All threads of the
// workgroup call this; only those with `mine` keep fragments.
constexpr int kLdW = 256 + 8;
template <int KT, int KTM>
__device__ __forceinline__ void load_w_block_lds(const uint16_t* W, int K, int ncols, uint16_t* Wl, bool mine, int cb,
                                                 int li, int lh, int tid, bf16x8 (&w)[2][KTM]) {
    constexpr int NCH = (KT + 7) / 8;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        __syncthreads();                               // the previous chunk has been read
        for (int idx = tid; idx < 128 * 32; idx += 512) {
            const int r = idx >> 5, v = idx & 31;
            const int k = 128 * c + r;
            u32x4 x = {0u, 0u, 0u, 0u};
            if (k < K && 8 * v < ncols) x = *reinterpret_cast<const u32x4*>(W + (int64_t)k * ncols + 8 * v);
            *reinterpret_cast<u32x4*>(Wl + r * kLdW + 8 * v) = x;
        }
        __syncthreads();
        if (mine) {
#pragma unroll
            for (int kk = 8 * c; kk < 8 * c + 8 && kk < KT; ++kk)
#pragma unroll
                for (int ch = 0; ch < 2; ++ch) {
                    const int col = 64 * cb + 32 * ch + li;
                    u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t x = Wl[(16 * (kk - 8 * c) + 8 * lh + e) * kLdW + col];
                        v[e >> 1] |= x << (16 * (e & 1));
                    }
                    w[ch][kk] = __builtin_bit_cast(bf16x8, v);
                }
        }
    }
    __syncthreads();
}

// Fused two-layer MLP, weights stationary, wavefronts specialised by layer.
//
// Wavefronts 0-3 hold W1 (64 hidden columns each), wavefronts 4-7 hold W2 (64 output columns each); every SIMD
// gets one of each.  The two products are pipelined over tiles: in phase p the first group turns Z tile p into
// hidden tile p (LDS, two buffers) while the second group turns hidden tile p-1 into output tile p-1, so the
// each staged row is read from LDS by four wavefronts instead of eight.  The loads of Z tile p+1 are issued at the
// start of the phase and travel during the products; between the phase's two barriers all wavefronts move data:
// output tile p-1 from its staging tile to Y (and to the history rows), Z tile p+1 from registers to LDS.
// EXACT: K = 16 KT1 and H = N = 256, i.e. every column of every tile exists: the checks on the input columns and
// the output width are compiled out.
template <int KT1, int KT2, bool EXACT>
__global__ __launch_bounds__(512) void ws_mlp_bf16_kernel(WsArgs a) {
    constexpr int LDA = 16 * KT1 + 8, LDH = 16 * KT2 + 8, LDY = 256 + 8;
    constexpr int VPR = 2 * KT1;
    constexpr int NVA = (kWsRows * VPR + 511) / 512;
    constexpr int NPI = (kWsRows * 32 + 511) / 512;
    constexpr int MT = kWsRows / 32;
    constexpr int KTM = KT1 > KT2 ? KT1 : KT2;
    static_assert(KT2 == 16, "the hidden and output staging tiles are 256 columns wide, one 64-column block per wavefront");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);                       // [64][LDA]
    uint16_t* Hs = As + kWsRows * LDA;                                      // [2][64][LDH]
    uint16_t* Ys = Hs + 2 * kWsRows * LDH;                                  // [64][LDY]
    float* bias1 = reinterpret_cast<float*>(Ys + kWsRows * LDY);            // [256]
    float* bias2 = bias1 + 256;                                             // [256]
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // the same in every lane, and known to be
    const int role = wave >> 2, cb = wave & 3;        // role 0: Z W1, role 1: H W2; 64-column block cb

    bf16x8 w[2][KTM];
    load_w_block_lds<KT1, KTM>(a.W1, a.K, a.H, As, role == 0, cb, li, lh, tid, w);
    load_w_block_lds<KT2, KTM>(a.W2, a.H, a.N, As, role == 1, cb, li, lh, tid, w);
    if (tid < 256) {
        bias1[tid] = (a.b1 && tid < a.H) ? bf16_val(a.b1, tid) : 0.f;
        bias2[tid] = (a.b2 && tid < a.N) ? bf16_val(a.b2, tid) : 0.f;
    }

    u32x4 ra[NVA];
    // Per-thread offsets (row, column, LDS address) are recomputed from the thread index where they are used
    // (the index is made opaque there): kept live across the products they would be spilled.  Addresses are a
    // tile base that is the same for every lane plus a 32-bit offset; a tile that lies wholly inside the matrix
    // (all but the last, when the width is a multiple of the MFMA depth) takes a path without per-lane checks.
    const bool k_whole = EXACT || a.K == 16 * KT1;
    auto fetch = [&](int64_t tile, int tl) {          // unconditional loads; clamped addresses where checks are needed
        const uint16_t* base = a.Z + tile * kWsRows * a.ldz;
        const bool full = k_whole && (tile + 1) * kWsRows <= a.M;
#pragma unroll
        for (int i = 0; i < NVA; ++i) {
            const int idx = tl + 512 * i;
            const int row = idx / VPR, k = 8 * (idx % VPR);
            uint32_t off = (uint32_t)row * (uint32_t)a.ldz + (uint32_t)k;
            if (!full) {
                const bool ok = idx < kWsRows * VPR && tile * kWsRows + row < a.M && k < a.K;
                off = ok ? off : 0u;
            } else if (kWsRows * VPR % 512 != 0 && idx >= kWsRows * VPR) {
                off = 0u;
            }
            ra[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off));
        }
    };
    auto stage = [&](int64_t tile, int tl) {          // tile: the one fetch() was called for
        const bool full = k_whole && (tile + 1) * kWsRows <= a.M;
#pragma unroll
        for (int i = 0; i < NVA; ++i) {
            const int idx = tl + 512 * i;
            const int row = idx / VPR, k = 8 * (idx % VPR);
            u32x4 v = ra[i];
            if (!full) {
                const bool ok = tile * kWsRows + row < a.M && k < a.K;
                v = ok ? v : u32x4{0u, 0u, 0u, 0u};
            }
            if (idx < kWsRows * VPR) *reinterpret_cast<u32x4*>(As + row * LDA + k) = v;
        }
    };
    // D[m][64cb .. 64cb+63] = act(X[m][:] Wcols + bias) for the 64 rows of a tile, X and D in LDS.  Transposed
    // products: a lane ends up with 4 consecutive columns of one row per group of four accumulator registers.
    // Columns beyond the width need no check: their weight fragments and biases were loaded as zeros, so they come
    // out as exact zeros (and are zero operands of the next product).
    auto product = [&](auto kt_tag, const uint16_t* X, int ldx, uint16_t* D, int ldd, const float* bias, bool relu) {
        constexpr int KT = decltype(kt_tag)::value;
#pragma unroll
        for (int t = 0; t < MT; ++t) {                 // 32 rows at a time: two accumulator tiles live, not four
            // the accumulators start from the bias of their columns (element 4q+e of a lane is column n0(q)+e)
            f32x16 acc[2];
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 bq = *reinterpret_cast<const f32x4*>(bias + 64 * cb + 32 * ch + 8 * q + 4 * lh);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[ch][4 * q + e] = bq[e];
                }
            // operand fragments are read from LDS PF steps ahead of the MFMAs that use them
            constexpr int PF = KT < 4 ? KT : 4;
            const uint16_t* xrow = X + (32 * t + li) * ldx + 8 * lh;
            u32x4 fx[PF];
#pragma unroll
            for (int j = 0; j < PF; ++j) fx[j] = *reinterpret_cast<const u32x4*>(xrow + 16 * j);
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) {
                const bf16x8 cur = __builtin_bit_cast(bf16x8, fx[kk % PF]);
                if (kk + PF < KT) fx[kk % PF] = *reinterpret_cast<const u32x4*>(xrow + 16 * (kk + PF));
#pragma unroll
                for (int ch = 0; ch < 2; ++ch)
                    acc[ch] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[ch][kk], cur, acc[ch], 0, 0, 0);
            }
            uint16_t* drow = D + (32 * t + li) * ldd + 64 * cb + 4 * lh;
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[ch][4 * q + e];
                        if (relu) v[e] = fmaxf(v[e], 0.f);
                    }
                    *reinterpret_cast<u32x2*>(drow + 32 * ch + 8 * q) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                }
        }
    };

    const int grid = (int)gridDim.x, t0 = (int)blockIdx.x;
    const int n_my = (int)((a.n_tiles - t0 + grid - 1) / grid);   // tiles of this workgroup (>= 1)
    fetch(t0, tid);
    stage(t0, tid);
    __syncthreads();
    for (int p = 0; p <= n_my; ++p) {
        const int64_t t_out = t0 + (int64_t)(p - 1) * grid;        // tile whose output leaves in this phase
        int32_t prow[NPI] = {};
        int tl = tid;
        asm volatile("" : "+v"(tl));
        // output vector (row, v) of a thread: row = tl / 32 + 16 i, v = tl % 32 (the staging tile is 32 vectors wide;
        // narrower outputs leave the lanes beyond their width idle)
        const bool out_full = p >= 1 && (t_out + 1) * kWsRows <= a.M;
        if (a.push_idx && p >= 1) {
            const int32_t* pi = a.push_idx + t_out * kWsRows;
#pragma unroll
            for (int i = 0; i < NPI; ++i) {
                int row = (tl >> 5) + 16 * i;
                if (!out_full) row = t_out * kWsRows + row < a.M ? row : 0;
                prow[i] = pi[row];
            }
        }
        // loads of the next Z tile: issued here, they travel while the matrix pipes work, and are staged
        // between this phase's two barriers
        if (p + 1 < n_my) fetch(t0 + (int64_t)(p + 1) * grid, tl);
        if (role == 0) {
            if (p < n_my)
                product(std::integral_constant<int, KT1>{}, As, LDA, Hs + (p & 1) * kWsRows * LDH, LDH, bias1, true);
        } else {
            if (p >= 1)
                product(std::integral_constant<int, KT2>{}, Hs + ((p - 1) & 1) * kWsRows * LDH, LDH, Ys, LDY, bias2,
                        a.relu_out != 0);
        }
        __syncthreads();                               // Z tile consumed; hidden tile p and output tile p-1 complete
#pragma unroll
        for (int i = 0; i < NPI; ++i) asm volatile("" : "+v"(prow[i]));   // delivered before new loads queue up
        asm volatile("" : "+v"(tl));
        if (p + 1 < n_my) stage(t0 + (int64_t)(p + 1) * grid, tl);
        if (p >= 1) {
            const int vpr = EXACT ? 32 : a.N >> 3;     // 16-byte vectors per output row
            const int tq = __builtin_amdgcn_readfirstlane((int)t_out);   // the tile index, in a scalar register
            uint16_t* ybase = a.Y + (int64_t)tq * kWsRows * a.ldy;
            const int v = tl & 31;
            if (v < vpr) {
#pragma unroll
                for (int i = 0; i < NPI; ++i) {
                    const int row = (tl >> 5) + 16 * i;
                    if (out_full || (int64_t)tq * kWsRows + row < a.M) {
                        const u32x4 o = *reinterpret_cast<const u32x4*>(Ys + row * LDY + 8 * v);
                        __builtin_nontemporal_store(
                            o, reinterpret_cast<u32x4*>(ybase + ((uint32_t)row * (uint32_t)a.ldy + 8u * v)));
                        if (a.push_idx)
                            __builtin_nontemporal_store(
                                o, reinterpret_cast<u32x4*>(a.push_hist + (int64_t)prow[i] * a.ld_push + 8 * v));
                    }
                }
            }
            if (a.H_out) {
                // a training pass reads the hidden activation again: tile p-1 of it is complete and not written
                // before the next phase, so it leaves from its LDS buffer the same way
                const int hvpr = EXACT ? 32 : a.H >> 3;
                const uint16_t* hs = Hs + ((p - 1) & 1) * kWsRows * LDH;
                uint16_t* hbase = a.H_out + (int64_t)tq * kWsRows * a.ldh_out;
                if (v < hvpr) {
#pragma unroll
                    for (int i = 0; i < NPI; ++i) {
                        const int row = (tl >> 5) + 16 * i;
                        if (out_full || (int64_t)tq * kWsRows + row < a.M)
                            __builtin_nontemporal_store(
                                *reinterpret_cast<const u32x4*>(hs + row * LDH + 8 * v),
                                reinterpret_cast<u32x4*>(hbase + ((uint32_t)row * (uint32_t)a.ldh_out + 8u * v)));
                    }
                }
            }
        }
        __syncthreads();                               // next Z tile staged, output staging tile free again
    }
}

template <int KT1, int KT2>
gas_status launch_ws_mlp(const WsArgs& a, hipStream_t s) {
    constexpr int smem = 2 * (kWsRows * (16 * KT1 + 8) + 2 * kWsRows * (16 * KT2 + 8) + kWsRows * (256 + 8)) + 2 * 256 * 4;
    static const hipError_t attr1 = hipFuncSetAttribute(reinterpret_cast<const void*>(ws_mlp_bf16_kernel<KT1, KT2, true>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    static const hipError_t attr2 = hipFuncSetAttribute(reinterpret_cast<const void*>(ws_mlp_bf16_kernel<KT1, KT2, false>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr1);
    GAS_CHECK_HIP(attr2);
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    const int64_t blocks = a.n_tiles < cus ? a.n_tiles : cus;
    if (a.K == 16 * KT1 && a.H == 256 && a.N == 256)
        hipLaunchKernelGGL((ws_mlp_bf16_kernel<KT1, KT2, true>), dim3((unsigned)blocks), dim3(512), smem, s, a);
    else
        hipLaunchKernelGGL((ws_mlp_bf16_kernel<KT1, KT2, false>), dim3((unsigned)blocks), dim3(512), smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

template <int KT1, bool MASK>
gas_status launch_ws_kernel(const WsArgs& a, hipStream_t s) {
    constexpr int smem = 2 * (2 * kWsRows * (16 * KT1 + 8) + kWsRows * (256 + 8)) + 256 * 4;   // + the bias in fp32
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(ws_bf16_kernel<KT1, MASK>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr);
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    const int64_t blocks = a.n_tiles < cus ? a.n_tiles : cus;
    hipLaunchKernelGGL((ws_bf16_kernel<KT1, MASK>), dim3((unsigned)blocks), dim3(512), smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}
template <int KT1>
gas_status launch_ws(const WsArgs& a, hipStream_t s) { return a.mask ? launch_ws_kernel<KT1, true>(a, s) : launch_ws_kernel<KT1, false>(a, s); }

// ====================================================================== backward kernels
// Weight gradient dW[k, j] = c_w * sum_m Z[m, k] * G[m, j]: the reduction runs over the rows.  The rows are cut
// into slabs; a workgroup forms the 128 x 128 tile (tk, tj) of the partial product of one slab in fp32 and
// writes it to the workspace; dw_reduce_kernel adds the slabs in slab order (fixed order, no atomics).
constexpr int kDwTile = 128;

// Rows per slab: a function of the shape alone (the workspace size and the order of the sum follow from it).
// About four workgroups per compute unit, at most 4096 rows (long slabs amortise the partial tile they write),
// at least 128: a small batch then still spreads over the chip instead of queueing in a handful of workgroups.
static int64_t dw_tiles(int K, int N) { return (int64_t)((K + kDwTile - 1) / kDwTile) * ((N + kDwTile - 1) / kDwTile); }
static int64_t dw_slab_rows(int64_t M, int K, int N) {
    int64_t slab = (M * dw_tiles(K, N) + 1023) / 1024;
    slab = (slab + 63) / 64 * 64;
    return slab < 128 ? 128 : (slab > 4096 ? 4096 : slab);
}

// Slab partials for callers that can bring no workspace (gas_linear_bwd_weight_static): a zero-initialised array in
// the code object, one copy per GPU at that GPU's own address.  In host code the array's name is only a handle for
// the runtime; the address a kernel can use comes from hipGetSymbolAddress, asked once per device with that device
// current, and is what the launches are given.
constexpr int64_t kDwScratchBytes = 64ll << 20;
static __device__ __align__(256) unsigned char dw_scratch[kDwScratchBytes];
constexpr int kMaxDevices = 64;

static gas_status dw_scratch_pointer(void** out) {
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {nullptr};
    int dev = -1;
    GAS_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(GAS_ERR_ARG, "gas_linear_bwd_weight_static: device %d", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(dw_scratch));
        if (e != hipSuccess || !p)
            return fail(GAS_ERR_HIP, "gas_linear_bwd_weight_static: no address for the scratch array on device %d: %s",
                        dev, hipGetErrorString(e));
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return GAS_OK;
}

struct DwArgs {
    const char* Z;  int64_t ldz;
    const char* G;  int64_t ldg;
    int64_t M;
    int K, N;                       // F_in, F_out
    float c_w;
    float* partial;                 // [n_slabs][K][N]
    float* dW;                      // [K][N]
    int n_slabs;
    int slab;                       // rows per slab
};

// fp32: both operands split into bf16 parts (split.h), eight consecutive rows of one feature per LDS piece.  The tiles
// of one slab follow each other on one XCD: they read the same rows.
constexpr int kDwSplitKS = 2;
template <int BK, int BN>
__device__ __forceinline__ void dw_split_block(const DwArgs& a, unsigned block, char* smem) {
    using S = SplitGemm<BK, BN, 2, 2, kDwSplitKS, false, false>;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tn = (a.N + BN - 1) / BN, tiles = (a.K + BK - 1) / BK * tn;
    const unsigned of_xcd = block / 8, tile = of_xcd % tiles;
    const int slab = (int)(of_xcd / tiles * 8 + block % 8);
    if (slab >= a.n_slabs) return;                     // the grid is padded to a multiple of eight slabs
    const int k0 = (int)(tile / tn) * BK, n0 = (int)(tile % tn) * BN;
    const int64_t m_begin = (int64_t)slab * a.slab;
    const int64_t m_end = m_begin + a.slab < a.M ? m_begin + a.slab : a.M;
    const int wk0 = (wave >> 1) * (BK / 2), wn0 = (wave & 1) * (BN / 2);
    const float* Z = reinterpret_cast<const float*>(a.Z);
    const float* G = reinterpret_cast<const float*>(a.G);
    S g;
    f32x16 acc[S::TM][S::TN];
    if (!g.run(Z, a.ldz, k0, a.K, G, a.ldg, n0, a.N, m_begin, m_end, reinterpret_cast<uint16_t*>(smem), wk0, wn0, acc))
        plain_tile<S::TM, S::TN, false, false>(Z, a.ldz, k0 + wk0, a.K, G, a.ldg, n0 + wn0, a.N, m_begin, m_end, acc);
    float* out = a.partial + (int64_t)slab * a.K * a.N;
#pragma unroll
    for (int i = 0; i < S::TM; ++i)
#pragma unroll
        for (int j = 0; j < S::TN; ++j) {
            const int n = n0 + wn0 + 32 * j + li;
            if (n >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wk0 + 32 * i + 8 * (r / 4) + 4 * lh + (r % 4);
                if (k < a.K) out[(int64_t)k * a.N + n] = acc[i][j][r];
            }
        }
}
template <int BK, int BN, int WPS>
__global__ __launch_bounds__(256, WPS) void dw_split_kernel(DwArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    dw_split_block<BK, BN>(a, blockIdx.x, smem);
}

// Several weight gradients in one launch: problem i has the workgroups from first[i] on.  A gradient of few rows fills the chip
// for less time than its two launches take: 16 of 21,248 rows of 64 x 64 take 57 us together and 181 one by one, nine of
// 4,000 x 256 x 256 67 and 174.
constexpr int kDwBatch = 16;
struct DwBatch {
    DwArgs p[kDwBatch];
    unsigned first[kDwBatch];
    int count;
};
__device__ __forceinline__ int dw_problem(const DwBatch& b) {
    int i = 0;
    while (i + 1 < b.count && blockIdx.x >= b.first[i + 1]) ++i;
    return i;
}
template <int BK, int BN, int WPS>
__global__ __launch_bounds__(256, WPS) void dw_batch_split_kernel(DwBatch b) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int i = dw_problem(b);
    const DwArgs a = b.p[i];
    dw_split_block<BK, BN>(a, blockIdx.x - b.first[i], smem);
}

// bf16: both operands of an instruction need consecutive rows of one feature.  The rows lie in LDS as they come from memory and
// are transposed on the way out (ds_read_b64_tr_b16: sixteen lanes read four rows of sixteen features, and a lane receives
// one feature of the four rows), two buffers of 64 rows, the next rows in registers during the products: one barrier a step.
// A workgroup of eight wavefronts owns a BK x BN tile of a slab's partial; with both widths at most 256 that is the whole
// partial, and Z and G are read once.
// Bounded by memory: 312,500 rows, 256 x 256: 384 MB with the slabs' partials in 79 us (4.9 TB/s; transposed on the way into
// LDS, with one buffer, whose 16-byte stores met 16 to a bank, 110); 128 x 256, 304 MB, 69 us (in tiles of 128 x 128 81).
// LDS: 16-byte unit u of row r lies at unit u ^ 4 (r & 3), so the 32 bytes that four lanes read of each of four rows, and the
// neighbouring ones that the next sixteen lanes read, fall on banks of their own.
constexpr int kDwRows = 64;
template <int B> __device__ __forceinline__ int dw_lds_unit(int row, int unit) { return row * (B / 8) + (unit ^ (4 * (row & 3))); }

template <int BK, int BN, int WK, bool PASS>
__global__ __launch_bounds__(512) void dw_bf16_kernel(DwArgs a) {
    constexpr int WN = 8 / WK, TK = BK / WK / 32, TN = BN / WN / 32;           // wavefronts, 32 x 32 blocks of one
    constexpr int NZ = kDwRows * BK / 8 / 512, NG = kDwRows * BN / 8 / 512;    // 16-byte units a thread brings
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t* lds = reinterpret_cast<uint16_t*>(smem);                         // [2][64 * BK, then 64 * BN]
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* G = reinterpret_cast<const uint16_t*>(a.G);
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slab = blockIdx.x, k0 = blockIdx.y * BK, n0 = blockIdx.z * BN;
    const int64_t m_begin = (int64_t)slab * a.slab;
    const int64_t m_end = m_begin + a.slab < a.M ? m_begin + a.slab : a.M;
    const int wk0 = (wave / WN) * (32 * TK), wn0 = (wave % WN) * (32 * TN);
    f32x16 acc[TK][TN];
    zero_acc(acc);
    u32x4 rz[NZ], rg[NG];
    // loads from clamped addresses, zeroed by a select: no branch around them
    auto bring = [&](const uint16_t* src, int64_t ld, int64_t m0, int f0, int flim, int idx, int units) {
        const int64_t m = m0 + idx / units;
        const int f = f0 + 8 * (idx % units);
        const bool ok = m < m_end && f < flim;
        const u32x4* p = reinterpret_cast<const u32x4*>(ok ? src + m * ld + f : src);
        const u32x4 v = PASS ? __builtin_nontemporal_load(p) : *p;
        return ok ? v : u32x4{0u, 0u, 0u, 0u};
    };
    auto fetch = [&](int64_t m0) {
#pragma unroll
        for (int i = 0; i < NZ; ++i) rz[i] = bring(Z, a.ldz, m0, k0, a.K, tid + 512 * i, BK / 8);
#pragma unroll
        for (int i = 0; i < NG; ++i) rg[i] = bring(G, a.ldg, m0, n0, a.N, tid + 512 * i, BN / 8);
    };
    auto stage = [&](int buf) {
        u32x4* zt = reinterpret_cast<u32x4*>(lds + buf * kDwRows * (BK + BN));
        u32x4* gt = zt + kDwRows * BK / 8;
#pragma unroll
        for (int i = 0; i < NZ; ++i) zt[dw_lds_unit<BK>((tid + 512 * i) / (BK / 8), (tid + 512 * i) % (BK / 8))] = rz[i];
#pragma unroll
        for (int i = 0; i < NG; ++i) gt[dw_lds_unit<BN>((tid + 512 * i) / (BN / 8), (tid + 512 * i) % (BN / 8))] = rg[i];
    };
    // a lane's eight consecutive rows 16 kk + 8 lh .. + 7 of feature f0 + li, in two reads of four rows
    const int i16 = lane & 15, feat = 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
    auto fragment = [&](const uint16_t* tile, auto width, int f0, int kk) {
        constexpr int B = decltype(width)::value;
        s16x4 h[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = 16 * kk + 8 * lh + 4 * t + (i16 >> 2), f = f0 + feat;
            const uint16_t* p = tile + 8 * dw_lds_unit<B>(row, f >> 3) + (f & 7);
            h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
        }
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        return __builtin_bit_cast(bf16x8, s16x8{h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]});
    };
    fetch(m_begin);
    stage(0);
    if (m_begin + kDwRows < m_end) fetch(m_begin + kDwRows);
    int buf = 0;
    for (int64_t m0 = m_begin; m0 < m_end; m0 += kDwRows, buf ^= 1) {
        __syncthreads();                           // rows m0 .. staged; the other buffer's rows are done with
        const uint16_t* zt = lds + buf * kDwRows * (BK + BN);
        const uint16_t* gt = zt + kDwRows * BK;
#pragma unroll
        for (int kk = 0; kk < kDwRows / 16; ++kk) {
            bf16x8 fa[TK], fb[TN];
#pragma unroll
            for (int i = 0; i < TK; ++i) fa[i] = fragment(zt, std::integral_constant<int, BK>{}, wk0 + 32 * i, kk);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = fragment(gt, std::integral_constant<int, BN>{}, wn0 + 32 * j, kk);
#pragma unroll
            for (int i = 0; i < TK; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (m0 + kDwRows < m_end) {
            stage(buf ^ 1);
            if (m0 + 2 * kDwRows < m_end) fetch(m0 + 2 * kDwRows);
        }
    }
    float* out = a.partial + (int64_t)slab * a.K * a.N;
#pragma unroll
    for (int i = 0; i < TK; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn0 + 32 * j + li;
            if (n >= a.N) continue;
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const int k = k0 + wk0 + 32 * i + 8 * (rr / 4) + 4 * lh + (rr % 4);
                if (k < a.K) out[(int64_t)k * a.N + n] = acc[i][j][rr];
            }
        }
}

// Operands of any alignment and width: tiles of BK x BN, steps of 64 rows, both turned on their way into LDS (AnyTileBF16).  A
// thread an element of a slab's partial before: 50,000 x 256 x 47 358 us and now 19, 250 columns 1,746 and 39, 500 x 256 x 47 17.8 and 8.4.
template <int BK, int BN>
__global__ __launch_bounds__(256, 2) void dw_bf16_any_kernel(DwArgs a) {
    constexpr int TK = BK / 64, TN = BN / 64;
    __shared__ __attribute__((aligned(16))) uint16_t As[BK][kLdh];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[BN][kLdh];
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* G = reinterpret_cast<const uint16_t*>(a.G);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const unsigned tn = (a.N + BN - 1) / BN, tiles = (a.K + BK - 1) / BK * tn, of_xcd = blockIdx.x / 8, tile = of_xcd % tiles;
    const int slab = (int)(of_xcd / tiles * 8 + blockIdx.x % 8);      // the tiles of a slab follow each other on one XCD
    if (slab >= a.n_slabs) return;
    const int k0 = (int)(tile / tn) * BK, n0 = (int)(tile % tn) * BN;
    const int wk0 = (wave >> 1) * (BK / 2), wn0 = (wave & 1) * (BN / 2);
    const int64_t m_begin = (int64_t)slab * a.slab, m_end = min(a.M, m_begin + a.slab);
    f32x16 acc[TK][TN];
    zero_acc(acc);
    AnyTileBF16<BK, false> ta;
    AnyTileBF16<BN, false> tb;
    ta.fetch(Z, a.ldz, k0, a.K, m_begin, m_end, tid);
    tb.fetch(G, a.ldg, n0, a.N, m_begin, m_end, tid);
    for (int64_t m = m_begin; m < m_end; m += kBKh) {
        __syncthreads();
        ta.stage(As, m_end - m, tid);
        tb.stage(Bs, m_end - m, tid);
        __syncthreads();
        if (m + kBKh < m_end) {
            ta.fetch(Z, a.ldz, k0, a.K, m + kBKh, m_end, tid);
            tb.fetch(G, a.ldg, n0, a.N, m + kBKh, m_end, tid);
        }
        mfma_tile_bf16<TK, TN>(&As[0][0], kLdh, wk0, 0, Bs, wn0, li, lh, acc);
    }
    float* out = a.partial + (int64_t)slab * a.K * a.N;
#pragma unroll
    for (int i = 0; i < TK; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn0 + 32 * j + li;
            if (n >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wk0 + 32 * i + 8 * (r / 4) + 4 * lh + (r % 4);
                if (k < a.K) out[(int64_t)k * a.N + n] = acc[i][j][r];
            }
        }
}
template <int BK, int BN>
gas_status launch_dw_any(const DwArgs& a, hipStream_t s) {
    const int64_t tiles = (int64_t)((a.K + BK - 1) / BK) * ((a.N + BN - 1) / BN), blocks = ((int64_t)a.n_slabs + 7) / 8 * 8 * tiles;
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_linear_bwd_weight: too many workgroups for one launch");
    hipLaunchKernelGGL((dw_bf16_any_kernel<BK, BN>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

// dW = c_w * (sum of the slabs' partial tiles).  A workgroup owns 32 consecutive outputs; eight threads per output
// each add every eighth slab in slab order, four loads in flight, and the eight sums are added in a fixed order.
constexpr int kDwReduceOut = 32, kDwReduceWays = 8;
__device__ __forceinline__ void dw_reduce_block(const DwArgs& a, unsigned block, float (*part)[kDwReduceOut]) {
    const int o = threadIdx.x % kDwReduceOut, way = threadIdx.x / kDwReduceOut;
    const int64_t idx = (int64_t)block * kDwReduceOut + o;
    const int64_t per = (int64_t)a.K * a.N;
    float s = 0.f;
    if (idx < per) {
        const float* p = a.partial + idx;
        int sl = way;
        for (; sl + 3 * kDwReduceWays < a.n_slabs; sl += 4 * kDwReduceWays) {
            const float v0 = p[(int64_t)sl * per], v1 = p[(int64_t)(sl + kDwReduceWays) * per],
                        v2 = p[(int64_t)(sl + 2 * kDwReduceWays) * per], v3 = p[(int64_t)(sl + 3 * kDwReduceWays) * per];
            s = ((s + v0) + v1) + v2 + v3;
        }
        for (; sl < a.n_slabs; sl += kDwReduceWays) s += p[(int64_t)sl * per];
    }
    part[way][o] = s;
    __syncthreads();
    if (way == 0 && idx < per) {
        float t = part[0][o];
#pragma unroll
        for (int w = 1; w < kDwReduceWays; ++w) t += part[w][o];
        a.dW[idx] = a.c_w * t;
    }
}
__global__ __launch_bounds__(256) void dw_reduce_kernel(DwArgs a) {
    __shared__ float part[kDwReduceWays][kDwReduceOut];
    dw_reduce_block(a, blockIdx.x, part);
}
__global__ __launch_bounds__(256) void dw_batch_reduce_kernel(DwBatch b) {
    __shared__ float part[kDwReduceWays][kDwReduceOut];
    const int i = dw_problem(b);
    const DwArgs a = b.p[i];
    dw_reduce_block(a, blockIdx.x - b.first[i], part);
}

// ReLU backward, element-wise: GP = GY where Y > 0, else 0
template <bool BF>
__global__ __launch_bounds__(256) void relu_bwd_kernel(const char* GY, int64_t ldgy, const char* Y, int64_t ldy,
                                                       char* GP, int64_t ldgp, int64_t M, int F, int vec) {
    // vec: 16-byte pieces per row (0 = element-wise)
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    constexpr int EB = BF ? 2 : 4;
    if (vec > 0) {
        if (idx >= M * vec) return;
        const int64_t m = idx / vec;
        const int v = (int)(idx % vec);
        const u32x4 g = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(GY + (m * ldgy) * EB) + v);
        const u32x4 y = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(Y + (m * ldy) * EB) + v);
        u32x4 o = g;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (BF) {
                if (!(bf16_lo(y[q]) > 0.f)) o[q] &= 0xFFFF0000u;
                if (!(bf16_hi(y[q]) > 0.f)) o[q] &= 0x0000FFFFu;
            } else {
                if (!(__uint_as_float(y[q]) > 0.f)) o[q] = 0u;
            }
        }
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(GP + (m * ldgp) * EB) + v);
    } else {
        if (idx >= M * F) return;
        const int64_t m = idx / F;
        const int f = (int)(idx % F);
        if constexpr (BF) {
            const uint16_t* y = reinterpret_cast<const uint16_t*>(Y);
            const uint16_t g = reinterpret_cast<const uint16_t*>(GY)[m * ldgy + f];
            reinterpret_cast<uint16_t*>(GP)[m * ldgp + f] = bf16_val(y, m * ldy + f) > 0.f ? g : (uint16_t)0;
        } else {
            const float g = reinterpret_cast<const float*>(GY)[m * ldgy + f];
            reinterpret_cast<float*>(GP)[m * ldgp + f] = reinterpret_cast<const float*>(Y)[m * ldy + f] > 0.f ? g : 0.f;
        }
    }
}

// ====================================================================== launchers
template <int BM, int BN, int KS, int WPS>
gas_status launch_split(const LinArgs& a, hipStream_t s) {
    constexpr int smem = SplitGemm<BM, BN, 2, 2, KS, true, true>::kLdsBytes;
    static_assert(smem <= 65536, "no attribute needed");
    const int64_t gm = ((a.M + BM - 1) / BM + 7) / 8 * 8, gn = (a.N + BN - 1) / BN;
    if (gm * gn > 0x7FFFFFFF) return fail(GAS_ERR_ARG, "gas_linear: problem too large for one launch");
    const dim3 grid((unsigned)(gm * gn)), block(256);
    if (a.trans_w) hipLaunchKernelGGL((linear_split_kernel<BM, BN, KS, true, WPS>), grid, block, smem, s, a);
    else hipLaunchKernelGGL((linear_split_kernel<BM, BN, KS, false, WPS>), grid, block, smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

template <int BM, int BN, int WM, int WN, int KG, bool TRANS>
gas_status launch_groups(const LinArgs& a, hipStream_t s) {
    constexpr int smem = SplitGemm<BM, BN, WM, WN, 2, true, TRANS, KG>::kGroupsLdsBytes;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(linear_split_groups_kernel<BM, BN, WM, WN, TRANS, KG>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr);
    const int64_t gm = ((a.M + BM - 1) / BM + 7) / 8 * 8, gn = (a.N + BN - 1) / BN;
    hipLaunchKernelGGL((linear_split_groups_kernel<BM, BN, WM, WN, TRANS, KG>), dim3((unsigned)(gm * gn)), dim3(64 * WM * WN * KG), smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

// The tile of the fp32 weight gradient: 64 wide where a width fits (21,000 x 64 x 64 in 64 x 64 tiles 8 us, in 128 x 128 15;
// 98,000 x 256 x 64 in 128 x 64 tiles 44 us, in 128 x 128 61).  Shape 2 * (K <= 64) + (N <= 64).
int dw_shape(int K, int N) { return 2 * (K <= 64) + (N <= 64); }
int64_t dw_split_blocks(int shape, int64_t n_slabs, int K, int N) {
    const int bk = shape & 2 ? 64 : 128, bn = shape & 1 ? 64 : 128;
    return (n_slabs + 7) / 8 * 8 * ((K + bk - 1) / bk) * ((N + bn - 1) / bn);
}
template <int BK, int BN, int WPS>
void launch_dw_tile(int64_t blocks, const DwArgs* one, const DwBatch* batch, hipStream_t s) {
    constexpr int smem = SplitGemm<BK, BN, 2, 2, kDwSplitKS, false, false>::kLdsBytes;
    static_assert(smem <= 65536, "no attribute needed");
    if (one) hipLaunchKernelGGL((dw_split_kernel<BK, BN, WPS>), dim3((unsigned)blocks), dim3(256), smem, s, *one);
    else hipLaunchKernelGGL((dw_batch_split_kernel<BK, BN, WPS>), dim3((unsigned)blocks), dim3(256), smem, s, *batch);
}
gas_status launch_dw_blocks(int shape, int64_t blocks, const DwArgs* one, const DwBatch* batch, hipStream_t s) {
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_linear_bwd_weight: problem too large for one launch");
    if (shape == 0) launch_dw_tile<128, 128, 2>(blocks, one, batch, s);
    else if (shape == 1) launch_dw_tile<128, 64, 3>(blocks, one, batch, s);
    else if (shape == 2) launch_dw_tile<64, 128, 3>(blocks, one, batch, s);
    else launch_dw_tile<64, 64, 4>(blocks, one, batch, s);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}
gas_status launch_dw_split(int shape, int64_t n_slabs, const DwArgs& a, hipStream_t s) {
    return launch_dw_blocks(shape, dw_split_blocks(shape, n_slabs, a.K, a.N), &a, nullptr, s);
}

template <int BK, int BN, int WK, bool PASS>
gas_status launch_dw_bf16_tile(const DwArgs& a, hipStream_t s) {
    constexpr int smem = 2 * kDwRows * (BK + BN) * 2;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(dw_bf16_kernel<BK, BN, WK, PASS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr);
    const dim3 grid((unsigned)a.n_slabs, (unsigned)((a.K + BK - 1) / BK), (unsigned)((a.N + BN - 1) / BN));
    hipLaunchKernelGGL((dw_bf16_kernel<BK, BN, WK, PASS>), grid, dim3(512), smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}
template <bool PASS>
gas_status launch_dw_bf16_whole(const DwArgs& a, hipStream_t s) {
    if (a.K <= 128 && a.N <= 128) return launch_dw_bf16_tile<128, 128, 4, PASS>(a, s);
    if (a.K <= 128) return launch_dw_bf16_tile<128, 256, 2, PASS>(a, s);
    if (a.N <= 128) return launch_dw_bf16_tile<256, 128, 4, PASS>(a, s);
    return launch_dw_bf16_tile<256, 256, 4, PASS>(a, s);
}

// One tile for both widths up to 256; beyond, tiles of 128 x 128 (a 256-wide one would leave compute units without any).
// Loads pass the caches by (non-temporal) where one tile has both widths, so that every row is read once, and the rows are of
// 96 MB or more, which the passes between their writing and this call mostly push out of the 256 MB behind the L2s.  us in
// training passes, all weight gradients of one, by and through the caches: GIN of 312,500 rows of 128 254 and 268, of 150,000 of
// 128 and 256 256 and 268; but of 150,000 of 128 160 and 156, GCN of 50,000 of 128 41.5 and 35.7, of 1,432 -> 256 163 and 135.
gas_status launch_dw_bf16(const DwArgs& a, hipStream_t s) {
    if (a.K > 256 || a.N > 256) return launch_dw_bf16_tile<128, 128, 4, false>(a, s);
    return a.M * 2 * (a.K + a.N) >= (96 << 20) ? launch_dw_bf16_whole<true>(a, s) : launch_dw_bf16_whole<false>(a, s);
}

template <int KT, bool TRANS, bool MASK>
gas_status launch_ws_split(const LinArgs& a, hipStream_t s) {
    constexpr int smem = WsSplit<KT, MASK>::kLdsBytes, rows = WsSplit<KT, MASK>::ROWS;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(linear_ws_split_kernel<KT, TRANS, MASK>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr);
    const int64_t n_tiles = (a.M + rows - 1) / rows;
    const unsigned blocks = (unsigned)(n_tiles < 256 ? n_tiles : 256);                     // one per compute unit
    hipLaunchKernelGGL((linear_ws_split_kernel<KT, TRANS, MASK>), dim3(blocks), dim3(512), smem, s, a, n_tiles);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}
template <bool TRANS, bool MASK>
gas_status run_ws_split(const LinArgs& a, hipStream_t s) {
    switch ((a.K + 31) / 32) {
        case 3: return launch_ws_split<3, TRANS, MASK>(a, s);
        case 4: return launch_ws_split<4, TRANS, MASK>(a, s);
        case 5: return launch_ws_split<5, TRANS, MASK>(a, s);
        case 6: return launch_ws_split<6, TRANS, MASK>(a, s);
        case 7: return launch_ws_split<7, TRANS, MASK>(a, s);
        default: return launch_ws_split<8, TRANS, MASK>(a, s);
    }
}

template <int BM, int BN>
gas_status launch_bf16(const LinArgs& a, hipStream_t s) {
    const int64_t blocks = ((a.M + BM - 1) / BM + 7) / 8 * 8 * ((a.N + BN - 1) / BN);
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_linear: problem too large for one launch");
    hipLaunchKernelGGL((linear_bf16_kernel<BM, BN>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

// Y = Z W, every output a chain of fp32 multiply-adds in the order of k (gas_linear_in_order), for operands of any alignment and width.
// Bound by the multiply-adds of the vector units, with few rows by the chain of a tile's steps.  Tiles of 16 R x 64, R x 4 outputs a
// lane, steps of 32 k through LDS; the last step ends with k, so no term is added that is not there.  us, a thread an output with every
// operand out of the caches and so: 50,000 x 256 x 250 880 and 99, 20,000 x 1,433 x 128 1,033 and 152, 2,340 x 745 x 256 158 and 46 (by
// matrix instructions, in another order, 30, 50 and 16; by those of one k, which give the same bits, 96 to 102, 135 and 46: no more a cycle).
template <int R>
__global__ __launch_bounds__(256) void linear_bf16_in_order_kernel(LinArgs a) {
    constexpr int TM = 16 * R, TN = 64, BK = 32, NA = TM * BK / 256, NB = TN * BK / 256;
    typedef float f32xR __attribute__((ext_vector_type(R)));
    __shared__ __attribute__((aligned(16))) float As[BK][TM + (R == 1 ? 1 : 4)];      // [k][row]
    __shared__ __attribute__((aligned(16))) float Bs[BK][TN + 4];                     // [k][column]
    const uint16_t* Z = reinterpret_cast<const uint16_t*>(a.Z);
    const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const unsigned tn = (unsigned)((a.N + TN - 1) / TN), of_xcd = blockIdx.x / 8;     // a row tile's column tiles follow each other on one XCD
    const int64_t m0 = ((int64_t)(of_xcd / tn) * 8 + blockIdx.x % 8) * TM;
    const int n0 = (int)(of_xcd % tn) * TN;
    if (m0 >= a.M) return;
    uint16_t za[NA], wb[NB];
    auto fetch = [&](int k0) {                                      // rows, columns and k beyond the last repeat it
#pragma unroll
        for (int i = 0; i < NA; ++i) za[i] = Z[min(m0 + tid / BK + 256 / BK * i, a.M - 1) * a.ldz + min(k0 + tid % BK, a.K - 1)];
#pragma unroll
        for (int i = 0; i < NB; ++i) wb[i] = W[(int64_t)min(k0 + tid / TN + 256 / TN * i, a.K - 1) * a.N + min(n0 + tid % TN, a.N - 1)];
    };
    float acc[R][4] = {};
    auto step = [&](int k) {
        const f32xR z = *reinterpret_cast<const f32xR*>(&As[k][R * ty]);
        const f32x4 w = *reinterpret_cast<const f32x4*>(&Bs[k][4 * tx]);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(z[i], w[j], acc[i][j]);
    };
    fetch(0);
    for (int k0 = 0; k0 < a.K; k0 += BK) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NA; ++i) As[tid % BK][tid / BK + 256 / BK * i] = __uint_as_float((uint32_t)za[i] << 16);
#pragma unroll
        for (int i = 0; i < NB; ++i) Bs[tid / TN + 256 / TN * i][tid % TN] = __uint_as_float((uint32_t)wb[i] << 16);
        __syncthreads();
        if (k0 + BK < a.K) {
            fetch(k0 + BK);
#pragma unroll 8
            for (int k = 0; k < BK; ++k) step(k);
        } else {
            for (int k = 0; k < a.K - k0; ++k) step(k);
        }
    }
    uint16_t* Y = reinterpret_cast<uint16_t*>(a.Y);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t m = m0 + R * ty + i;
            const int n = n0 + 4 * tx + j;
            if (m < a.M && n < a.N) Y[m * a.ldy + n] = (uint16_t)f32_to_bf16(acc[i][j]);
        }
}

template <int R>
gas_status launch_in_order(const LinArgs& a, hipStream_t s) {
    const int64_t blocks = ((a.M + 16 * R - 1) / (16 * R) + 7) / 8 * 8 * ((a.N + 63) / 64);
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_linear_in_order: problem too large for one launch");
    hipLaunchKernelGGL(linear_bf16_in_order_kernel<R>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

template <int BM, int BN>
gas_status launch_bf16_any(const LinArgs& a, hipStream_t s) {
    const int64_t blocks = ((a.M + BM - 1) / BM + 7) / 8 * 8 * ((a.N + BN - 1) / BN);
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_linear: problem too large for one launch");
    if (a.trans_w) hipLaunchKernelGGL((linear_bf16_any_kernel<BM, BN, true>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((linear_bf16_any_kernel<BM, BN, false>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

}  // namespace
}  // namespace gas

using namespace gas;

extern "C" {

// Y = act(c_identity * Z + c_weight * (Z op(W)) + bias) with optional output mask; op(W) = W ([F_in, F_out]) or,
// with trans_w, the transpose of a [F_out, F_in] matrix.
struct PushTarget {                 // optional fused Push: output row i also goes to hist[idx[i], :]
    const int32_t* idx = nullptr;
    void* hist = nullptr;
    int64_t n_hist_rows = 0, ld_hist = 0;
};

// rows the kernel did not scatter itself are pushed by the row-copy kernel
static gas_status push_after(const PushTarget& p, const void* Y, int64_t ldy, int64_t n_rows, int32_t F, gas_dtype dt,
                             hipStream_t s) {
    if (!p.idx) return GAS_OK;
    return gas_push(Y, ldy, p.idx, 0, n_rows, F, dt, p.hist, p.n_hist_rows, p.ld_hist, s);
}

static gas_status run_linear(const char* who, const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W,
                             int trans_w, int32_t F_out, const void* bias, gas_dtype dt, float c_identity,
                             float c_weight, int relu, const void* mask, int64_t ldmask, void* Y, int64_t ldy,
                             hipStream_t s, const PushTarget& push = PushTarget(), const void* add = nullptr,
                             int64_t ldadd = 0, float c_total = 0.f, void* total = nullptr, int64_t ldtotal = 0,
                             bool in_order = false) {
    if (push.idx) {
        GAS_REQUIRE(push.hist && push.ld_hist >= F_out && push.n_hist_rows > 0, "%s: bad history table for the fused push", who);
        GAS_REQUIRE(push.hist != Y, "%s: the history table aliases the output", who);
    }
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    GAS_REQUIRE(n_rows >= 0 && F_in > 0 && F_out > 0, "%s: n_rows=%lld widths %d, %d", who, (long long)n_rows, F_in, F_out);
    if (n_rows == 0) return GAS_OK;
    GAS_REQUIRE(Z && W && Y, "%s: null pointer", who);
    GAS_REQUIRE(ldz >= F_in && ldy >= F_out && (!mask || ldmask >= F_out), "%s: row stride smaller than the row", who);
    GAS_REQUIRE(c_identity == 0.f || F_in == F_out, "%s: the identity term needs equal widths", who);
    GAS_REQUIRE(Y != Z, "%s: the output must not alias the input", who);
    LinArgs a;
    a.Z = static_cast<const char*>(Z); a.ldz = ldz;
    a.W = static_cast<const char*>(W);
    a.bias = static_cast<const char*>(bias);
    a.Y = static_cast<char*>(Y); a.ldy = ldy;
    a.M = n_rows; a.K = F_in; a.N = F_out;
    a.c_id = c_identity; a.c_w = c_weight; a.relu = relu;
    a.trans_w = trans_w; a.mask = static_cast<const char*>(mask); a.ldmask = ldmask;
    if (dt == GAS_F32) {
        a.add = static_cast<const char*>(add); a.ldadd = ldadd;
        a.total = static_cast<char*>(total); a.ldtotal = ldtotal; a.c_total = c_total;
        a.push_idx = push.idx; a.push_hist = static_cast<char*>(push.hist); a.ld_push = push.ld_hist;
        // Up to 16 input columns one step of 16 k takes them all.  Up to 64 a tile's loads and stores outweigh its products, and
        // many small workgroups overlap best until their number hides that too (100,000 x 64 x 64: 13.5 us, in 128 x 64 tiles
        // 15.6; 28,000 x 47 x 100: 11, 13 in 128 x 64, 17 in 128 x 128; but 300,000 x 64 x 256: 127, 103 in 128 x 128).  Beyond,
        // a larger tile splits each value for more products, as long as most compute units have a workgroup: 128 x 128
        // where two each are nearly reached (28,000 x 256 x 128, 219 tiles: 23 us, in 128 x 64 18; 50,000 x 256 x 128, 391
        // tiles: 27, in 128 x 64 35), 4,000 x 256 x 256 10 us in 64 x 64 tiles.
        const int64_t tiles = (n_rows + 127) / 128, large = tiles * ((F_out + 127) / 128);
        if (F_in <= 16) return launch_split<64, 64, 1, 4>(a, s);
        // One to two columns of 128 x 128 tiles, in more than one round of the 512 that run at once: the weights stay put instead
        // (33,000 rows 256 -> 256: 32 us, in tiles 48; 50,000 rows 256 -> 136: 40 and 52, 144 -> 256: 36 and 40, 72 -> 256: 27 and 31;
        // below, 26,000 rows 256 -> 256: 27 and 27, 16,000: 20 and 18).  The tiles stay where they do no work for padding, up to
        // 160 whole columns to 256: 96 in less than three rounds (65,000 rows, the transform 27.7 us and with the weights in place
        // 30.3, the input gradient 26.8 and 31.0), 128 and 160 in two full rounds, 897 to 1,024 tiles (65,000 rows of 160: 38.8 and
        // 39.7, 37.1 and 41.3, of 128 33.3 and 32.8, 32.2 and 34.4; at 896 tiles of 160 39.5 and 36.4, 38.1 and 37.7, at 1,026
        // 48.9 and 43.0, 46.6 and 44.5).  With any padding the weights stay (65,000 rows 160 -> 252: 49.1 and 38.7, 47.4 and 41.4).
        if (F_in > 64 && F_in <= 256 && F_out > 128 && F_out <= 256 && large > 512 &&
            c_identity == 0.f && !add && !total && (!mask || trans_w)) {
            const bool unpadded = F_in % 32 == 0 && F_in <= 160 && F_out == 256;
            if (!unpadded || (F_in <= 96 ? large > 1536 : large <= 896 || large > 1024)) {
                if (mask) return run_ws_split<true, true>(a, s);
                return trans_w ? run_ws_split<true, false>(a, s) : run_ws_split<false, false>(a, s);
            }
        }
        if (F_in > 64 || large >= 2048) {
            if (F_out > 64 && large >= 352) return launch_split<128, 128, 2, 2>(a, s);
            if (tiles * ((F_out + 63) / 64) >= 384) return launch_split<128, 64, 2, 3>(a, s);
        }
        // No more than a tile for a compute unit: its steps go to four groups of wavefronts (500 x 1,024 x 1,024: 29.9 -> 24.5 us,
        // 2,500 x 850 x 255 28.0 -> 22.5, 4,000 x 256 x 256 9.8 -> 9.0).  Up to five steps the sum over the groups costs a call
        // that repeats itself more than they save (5,000 x 128 x 64: 5.8 -> 6.1), but right after the aggregation that wrote its
        // input the same call ends 0.8 us earlier, 2,000 x 160 x 128 0.6, 512 x 80 x 64 0.1: that is how passes call it.  A
        // workgroup fills a unit, and the column tiles of a row tile share one of the eight XCDs of 32: at 33 tiles on an
        // XCD one of them waits for a second round (5,120 x 192 x 192, 30 on an XCD: 9.4 and 9.1; 5,400 rows, 33: 11.2 and 16.5).
        // Half as many rows a tile and twice the groups as long as that is one round too: most units are idle then, and each group has
        // half the steps to split (500 x 256 x 256: 9.1 -> 7.5 us, 229 x 2,240 x 224 46.9 -> 31.3, 2,000 x 832 x 128 19.9 -> 14.6;
        // steps of 16 k 38.4, two steps' loads in flight 34; at 64 tiles of 32 x 64 on an XCD, 4,000 x 256 x 256, 12.8 for 9.1).
        auto on_xcd = [&](int rows) { return ((n_rows + rows - 1) / rows + 7) / 8 * ((F_out + 63) / 64); };
        if (F_in > 96 && on_xcd(32) <= 32)
            return trans_w ? launch_groups<32, 64, 1, 2, 8, true>(a, s) : launch_groups<32, 64, 1, 2, 8, false>(a, s);
        if (F_in > 64 && on_xcd(64) <= 32)
            return trans_w ? launch_groups<64, 64, 2, 2, 4, true>(a, s) : launch_groups<64, 64, 2, 2, 4, false>(a, s);
        return launch_split<64, 64, 2, 4>(a, s);
    }
    const bool vec = aligned16(Z) && aligned16(W) && ldz % 8 == 0 && F_in % 8 == 0 && F_out % 8 == 0;
    if (!vec && in_order) {
        // Tiles of 64 rows once they fill the units twice, of 16 while one of 64 a unit would be too many: us by 16, 32 and 64 rows,
        // 2,340 x 745 x 64 39, 48, 70; 2,340 x 745 x 256 46, 52, 71; 5,000 x 745 x 250 66, 62, 72; 20,000 x 1,433 x 128 209, 153, 152.
        const int64_t tiles = (n_rows + 63) / 64 * ((F_out + 63) / 64);
        return tiles <= 256 ? launch_in_order<1>(a, s) : tiles <= 512 ? launch_in_order<2>(a, s) : launch_in_order<4>(a, s);
    }
    if (!vec) {
        // Small tiles until their number fills the units several times (256 -> 250 in 64 x 64 and in larger ones: 5,000 rows
        // 9.5 and 14.1 us, 20,000 17.0 and 17.9, 50,000 34.5 and 30.3; the masked input gradient, whose larger tiles wait longer for
        // the mask, 15.3 and 20.3, 31.5 and 36.0, at 150,000 81 and 76).
        const gas_status st = (n_rows + 63) / 64 * ((F_out + 63) / 64) <= (trans_w ? 4096 : 2048) ? launch_bf16_any<64, 64>(a, s)
                              : F_out <= 64 ? launch_bf16_any<128, 64>(a, s) : launch_bf16_any<128, 128>(a, s);
        if (st != GAS_OK) return st;
        return push_after(push, Y, ldy, n_rows, F_out, dt, s);
    }
    // A workgroup that keeps all weights needs several row tiles to be worth its start, and a tile of 64 x 64 a quarter of that:
    // 500 rows 256 -> 256 in 64 x 64 7.2 us (128 x 256, one wavefront a unit, 20.1), 1,024 inputs 19.8 and 31.5, 16,000 rows 11.2
    // and with the weights in place 16.9, 50,000 33.0 and 27.3; the masked input gradient, which starts sooner because its weights
    // take no turning, 6,000 rows 6.6 and 8.8, 16,000 9.7 and 9.6.  Up to 64 columns six wavefronts of eight would hold no
    // weights: 50,000 rows 256 -> 64 11.2 and 21.6, 300,000 49 and 56.  Wider than the weights-stationary kernel takes: 128 x 128 once small tiles
    // fill the chip (100,000 rows 512 -> 256 98 and 89), but not transposed (90 and 98).
    // With a Push, which that kernel stores itself and a copy of the rows, 3 to 19 us, follows tiles for: up to 128 inputs it starts soon and
    // takes all but the few rows whose tiles are fewest (4,096 rows 128 -> 128 9.9 and 9.6, 9,000 10.4 and 11.3, 16,000 10.6 and 11.7, 128 ->
    // 256 3,000 10.2 both, 9,000 11.1 and 12.5, 16,000 11.8 and 13.7); up to 64 columns tiles only between (128 -> 48 16,000 10.1 and 11.2,
    // 40,000 15.0 and 13.7, 64 -> 64 3,000 7.0 and 9.1, 40,000 11.5 and 12.0).  With more inputs the line stays (256 -> 256 16,000 18.1
    // and 17.1, 24,000 20.9 and 25.4; 256 -> 64 64,000 24.4 and 21.6, 300,000 62 and 77).
    const bool ws = F_in <= 256 && F_out <= 256 && aligned16(Y) && ldy % 8 == 0 &&
        (!mask || (aligned16(mask) && ldmask % 8 == 0)) && ldz < (1 << 24) && ldy < (1 << 24) && ldmask < (1 << 24);
    const bool scatter = ws && push.idx && aligned16(push.hist) && push.ld_hist % 8 == 0;
    const int64_t tiles = (n_rows + 63) / 64 * ((F_out + 63) / 64);
    const bool small = !scatter || F_in > 128 ? (F_out <= 64 && !scatter) || (!ws && trans_w) || tiles <= (trans_w ? 512 : 1024)
                                              : F_in > 64 && (F_out <= 64 ? tiles > 320 && tiles <= 1024 : tiles <= 192);
    if (ws && !small) {
        WsArgs w{};
        w.Z = static_cast<const uint16_t*>(Z); w.ldz = ldz;
        w.W1 = static_cast<const uint16_t*>(W); w.b1 = static_cast<const uint16_t*>(bias);
        w.Y = static_cast<uint16_t*>(Y); w.ldy = ldy;
        w.M = n_rows; w.n_tiles = (n_rows + kWsRows - 1) / kWsRows;
        w.K = F_in; w.H = F_out; w.N = F_out;
        w.c_id = c_identity; w.c_w = c_weight; w.relu1 = relu; w.relu_out = 0;
        w.trans_w1 = trans_w; w.mask = static_cast<const uint16_t*>(mask); w.ldmask = ldmask;
        if (scatter) { w.push_idx = push.idx; w.push_hist = static_cast<uint16_t*>(push.hist); w.ld_push = push.ld_hist; }
        const gas_status st = F_in <= 64 ? launch_ws<4>(w, s) : (F_in <= 128 ? launch_ws<8>(w, s) : launch_ws<16>(w, s));
        return (st != GAS_OK || scatter) ? st : push_after(push, Y, ldy, n_rows, F_out, dt, s);
    }
    const gas_status st = small ? launch_bf16<64, 64>(a, s) : launch_bf16<128, 128>(a, s);
    return st != GAS_OK ? st : push_after(push, Y, ldy, n_rows, F_out, dt, s);
}

gas_status gas_linear_push(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W, int32_t F_out,
                           const void* bias, gas_dtype dt, float c_identity, float c_weight, int relu, void* Y,
                           int64_t ldy, const int32_t* idx, void* hist, int64_t n_hist_rows, int64_t ld_hist,
                           void* stream) {
    GAS_REQUIRE(idx || n_rows == 0, "gas_linear_push: null index array");
    PushTarget p;
    p.idx = idx; p.hist = hist; p.n_hist_rows = n_hist_rows; p.ld_hist = ld_hist;
    return run_linear("gas_linear_push", Z, ldz, n_rows, F_in, W, 0, F_out, bias, dt, c_identity, c_weight, relu,
                      nullptr, 0, Y, ldy, (hipStream_t)stream, p);
}

gas_status gas_linear(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W, int32_t F_out,
                      const void* bias, gas_dtype dt, float c_identity, float c_weight, int relu, void* Y,
                      int64_t ldy, void* stream) {
    return run_linear("gas_linear", Z, ldz, n_rows, F_in, W, 0, F_out, bias, dt, c_identity, c_weight, relu, nullptr,
                      0, Y, ldy, (hipStream_t)stream);
}

gas_status gas_linear_in_order(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W, int32_t F_out, gas_dtype dt,
                               void* Y, int64_t ldy, void* stream) {
    return run_linear("gas_linear_in_order", Z, ldz, n_rows, F_in, W, 0, F_out, nullptr, dt, 0.f, 1.f, 0, nullptr, 0, Y, ldy,
                      (hipStream_t)stream, PushTarget(), nullptr, 0, 0.f, nullptr, 0, true);
}

gas_status gas_linear_bwd_input(const void* GP, int64_t ldgp, int64_t n_rows, int32_t F_out, const void* W,
                                int32_t F_in, gas_dtype dt, float c_identity, float c_weight, const void* mask,
                                int64_t ldmask, void* GZ, int64_t ldgz, void* stream) {
    // GZ = c_identity * GP + c_weight * (GP W^T): a product with the [F_in, F_out] matrix taken transposed
    return run_linear("gas_linear_bwd_input", GP, ldgp, n_rows, F_out, W, 1, F_in, nullptr, dt, c_identity, c_weight,
                      0, mask, ldmask, GZ, ldgz, (hipStream_t)stream);
}

gas_status gas_linear_bwd_input_add(const void* GP, int64_t ldgp, int64_t n_rows, int32_t F_out, const void* W,
                                    int32_t F_in, gas_dtype dt, float c_identity, float c_weight, const void* add,
                                    int64_t ldadd, const void* mask, int64_t ldmask, float c_total, void* total,
                                    int64_t ldtotal, void* GZ, int64_t ldgz, void* stream) {
    const char* who = "gas_linear_bwd_input_add";
    GAS_REQUIRE((!add || ldadd >= F_in) && (!mask || ldmask >= F_in) && (!total || ldtotal >= F_in),
                "%s: row stride smaller than the row", who);
    GAS_REQUIRE(!total || (total != GZ && total != GP && total != add && total != mask), "%s: the total aliases another matrix", who);
    GAS_REQUIRE(!add || add != GZ || ldadd == ldgz, "%s: an output in place of the addend needs its row stride", who);
    hipStream_t s = (hipStream_t)stream;
    if (dt == GAS_F32)
        return run_linear(who, GP, ldgp, n_rows, F_out, W, 1, F_in, nullptr, dt, c_identity, c_weight, 0, mask, ldmask, GZ,
                          ldgz, s, PushTarget(), add, ldadd, c_total, total, ldtotal);
    // bf16: every step rounds to storage, as the calls one after the other do
    GAS_REQUIRE(!add || add != GZ, "%s: bf16 needs an output beside the addend", who);
    gas_status st = run_linear(who, GP, ldgp, n_rows, F_out, W, 1, F_in, nullptr, dt, c_identity, c_weight, 0,
                               add ? nullptr : mask, ldmask, GZ, ldgz, s);
    if (st == GAS_OK && add) st = gas_axpy(add, ldadd, GZ, ldgz, n_rows, F_in, dt, 1.f, GZ, ldgz, stream);
    if (st == GAS_OK && add && mask) st = gas_relu_bwd(GZ, ldgz, mask, ldmask, n_rows, F_in, dt, GZ, ldgz, stream);
    if (st == GAS_OK && total) st = gas_axpy(total, ldtotal, GZ, ldgz, n_rows, F_in, dt, c_total, total, ldtotal, stream);
    return st;
}

int64_t gas_linear_bwd_weight_workspace(int64_t n_rows, int32_t F_in, int32_t F_out) {
    if (n_rows <= 0 || F_in <= 0 || F_out <= 0) return 0;
    const int64_t slab = dw_slab_rows(n_rows, F_in, F_out);
    return ((n_rows + slab - 1) / slab) * (int64_t)F_in * F_out * (int64_t)sizeof(float);
}

// Weight gradient with the slab partials in `workspace` (the caller's, or the library's static array).
static gas_status run_dw(const void* Z, int64_t ldz, const void* GP, int64_t ldgp, int64_t n_rows,
                         int32_t F_in, int32_t F_out, gas_dtype dt, float c_weight, float* dW,
                         void* workspace, int64_t workspace_bytes, bool static_scratch, void* stream) {
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "gas_linear_bwd_weight: unknown dtype %d", (int)dt);
    GAS_REQUIRE(n_rows >= 0 && F_in > 0 && F_out > 0, "gas_linear_bwd_weight: n_rows=%lld widths %d, %d",
                (long long)n_rows, F_in, F_out);
    GAS_REQUIRE(dW, "gas_linear_bwd_weight: null output");
    hipStream_t s = (hipStream_t)stream;
    DwArgs a;
    a.Z = static_cast<const char*>(Z); a.ldz = ldz;
    a.G = static_cast<const char*>(GP); a.ldg = ldgp;
    a.M = n_rows; a.K = F_in; a.N = F_out; a.c_w = c_weight;
    a.partial = static_cast<float*>(workspace); a.dW = dW;
    a.slab = (int)dw_slab_rows(n_rows, F_in, F_out);
    const int64_t n_slabs = (n_rows + a.slab - 1) / a.slab;
    GAS_REQUIRE(n_slabs <= 0x7FFFFFFFLL, "gas_linear_bwd_weight: too many rows");
    a.n_slabs = (int)n_slabs;
    const int64_t per = (int64_t)F_in * F_out;
    const unsigned rblocks = (unsigned)((per + kDwReduceOut - 1) / kDwReduceOut);
    if (n_rows == 0) {                                   // empty sum: dW = 0
        hipLaunchKernelGGL(dw_reduce_kernel, dim3(rblocks), dim3(256), 0, s, a);
        GAS_CHECK_HIP(hipGetLastError());
        return GAS_OK;
    }
    GAS_REQUIRE(Z && GP, "gas_linear_bwd_weight: null pointer");
    GAS_REQUIRE(ldz >= F_in && ldgp >= F_out, "gas_linear_bwd_weight: row stride smaller than the row");
    if (static_scratch) {
        const int64_t need = gas_linear_bwd_weight_workspace(n_rows, F_in, F_out);
        if (need > kDwScratchBytes)
            return fail(GAS_ERR_ARG, "gas_linear_bwd_weight_static: the slab partials of this shape take %lld bytes, "
                        "the library's static scratch array holds %lld; use gas_linear_bwd_weight with a workspace",
                        (long long)need, (long long)kDwScratchBytes);
        const gas_status st = dw_scratch_pointer(&workspace);
        if (st != GAS_OK) return st;
        workspace_bytes = kDwScratchBytes;
        a.partial = static_cast<float*>(workspace);
    }
    GAS_REQUIRE(workspace && workspace_bytes >= gas_linear_bwd_weight_workspace(n_rows, F_in, F_out),
                "gas_linear_bwd_weight: workspace of %lld bytes needed, %lld given",
                (long long)gas_linear_bwd_weight_workspace(n_rows, F_in, F_out), (long long)workspace_bytes);
    const unsigned tk = (unsigned)((F_in + kDwTile - 1) / kDwTile), tn = (unsigned)((F_out + kDwTile - 1) / kDwTile);
    GAS_REQUIRE(tk <= 65535 && tn <= 65535, "gas_linear_bwd_weight: widths too large");
    if (dt == GAS_F32) {
        const gas_status st = launch_dw_split(dw_shape(F_in, F_out), n_slabs, a, s);
        if (st != GAS_OK) return st;
    } else {
        const bool vec = aligned16(Z) && aligned16(GP) && ldz % 8 == 0 && ldgp % 8 == 0 && F_in % 8 == 0 && F_out % 8 == 0;
        if (vec) {
            const gas_status st = launch_dw_bf16(a, s);
            if (st != GAS_OK) return st;
        } else {
            const gas_status st = F_in <= 64 ? (F_out <= 64 ? launch_dw_any<64, 64>(a, s) : launch_dw_any<64, 128>(a, s))
                                             : (F_out <= 64 ? launch_dw_any<128, 64>(a, s) : launch_dw_any<128, 128>(a, s));
            if (st != GAS_OK) return st;
        }
    }
    hipLaunchKernelGGL(dw_reduce_kernel, dim3(rblocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

gas_status gas_linear_bwd_weight(const void* Z, int64_t ldz, const void* GP, int64_t ldgp, int64_t n_rows,
                                 int32_t F_in, int32_t F_out, gas_dtype dt, float c_weight, float* dW,
                                 void* workspace, int64_t workspace_bytes, void* stream) {
    return run_dw(Z, ldz, GP, ldgp, n_rows, F_in, F_out, dt, c_weight, dW, workspace, workspace_bytes, false, stream);
}

int64_t gas_linear_bwd_weights_workspace(int32_t count, const int64_t* n_rows, const int32_t* F_in, const int32_t* F_out,
                                         gas_dtype dt) {
    if (count <= 0 || !n_rows || !F_in || !F_out) return 0;
    int64_t most = 0, launch = 0;
    for (int32_t i = 0; i < count; ++i) {              // bf16: a launch for each; fp32: kDwBatch at a time
        if (dt != GAS_F32 || i % kDwBatch == 0) launch = 0;
        launch += gas_linear_bwd_weight_workspace(n_rows[i], F_in[i], F_out[i]);
        most = std::max(most, launch);
    }
    return most;
}

gas_status gas_linear_bwd_weights(int32_t count, const void* const* Z, const int64_t* ldz, const void* const* GP,
                                  const int64_t* ldgp, const int64_t* n_rows, const int32_t* F_in, const int32_t* F_out,
                                  gas_dtype dt, const float* c_weight, float* const* dW, void* workspace,
                                  int64_t workspace_bytes, void* stream) {
    const char* who = "gas_linear_bwd_weights";
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    GAS_REQUIRE(count >= 0 && (count == 0 || (Z && ldz && GP && ldgp && n_rows && F_in && F_out && c_weight && dW)),
                "%s: count=%d or a null array", who, count);
    for (int32_t i = 0; i < count; ++i) {
        GAS_REQUIRE(n_rows[i] >= 0 && F_in[i] > 0 && F_out[i] > 0, "%s: %d: n_rows=%lld widths %d, %d", who, i, (long long)n_rows[i],
                    F_in[i], F_out[i]);
        GAS_REQUIRE(dW[i] && (n_rows[i] == 0 || (Z[i] && GP[i])), "%s: %d: null pointer", who, i);
        GAS_REQUIRE(n_rows[i] == 0 || (ldz[i] >= F_in[i] && ldgp[i] >= F_out[i]), "%s: %d: row stride smaller than the row", who, i);
    }
    const int64_t need = gas_linear_bwd_weights_workspace(count, n_rows, F_in, F_out, dt);
    GAS_REQUIRE(need == 0 || (workspace && workspace_bytes >= need), "%s: workspace of %lld bytes needed, %lld given", who,
                (long long)need, (long long)workspace_bytes);
    if (dt != GAS_F32) {
        for (int32_t i = 0; i < count; ++i) {
            const gas_status st = gas_linear_bwd_weight(Z[i], ldz[i], GP[i], ldgp[i], n_rows[i], F_in[i], F_out[i], dt, c_weight[i],
                                                        dW[i], workspace, workspace_bytes, stream);
            if (st != GAS_OK) return st;
        }
        return GAS_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    for (int32_t i0 = 0; i0 < count; i0 += kDwBatch) {
        const int32_t n = std::min(count - i0, (int32_t)kDwBatch);
        int64_t at = 0, reduce_blocks = 0, blocks[4] = {0, 0, 0, 0};
        DwBatch tile[4], all;              // by the shape of the tiles, and all of them for the sums over the slabs
        tile[0].count = tile[1].count = tile[2].count = tile[3].count = all.count = 0;
        bool wide = false;                 // where 128 x 128 tiles are launched anyway, half-filled ones cost less than a launch
        for (int32_t i = i0; i < i0 + n; ++i) wide = wide || (n_rows[i] > 0 && F_in[i] > 64 && F_out[i] > 64);
        for (int32_t i = i0; i < i0 + n; ++i) {
            DwArgs a;
            a.Z = static_cast<const char*>(Z[i]); a.ldz = ldz[i];
            a.G = static_cast<const char*>(GP[i]); a.ldg = ldgp[i];
            a.M = n_rows[i]; a.K = F_in[i]; a.N = F_out[i]; a.c_w = c_weight[i];
            a.partial = static_cast<float*>(workspace) + at; a.dW = dW[i];
            a.slab = (int)dw_slab_rows(n_rows[i], F_in[i], F_out[i]);
            const int64_t n_slabs = (n_rows[i] + a.slab - 1) / a.slab, per = (int64_t)F_in[i] * F_out[i];
            GAS_REQUIRE(n_slabs <= 0x7FFFFFFFLL, "%s: too many rows", who);
            a.n_slabs = (int)n_slabs;
            at += n_slabs * per;
            all.p[all.count] = a;
            all.first[all.count++] = (unsigned)reduce_blocks;
            reduce_blocks += (per + kDwReduceOut - 1) / kDwReduceOut;
            if (n_slabs > 0) {
                const int own = dw_shape(F_in[i], F_out[i]), t = wide && own != 3 ? 0 : own;
                tile[t].p[tile[t].count] = a;
                tile[t].first[tile[t].count++] = (unsigned)blocks[t];
                blocks[t] += dw_split_blocks(t, n_slabs, F_in[i], F_out[i]);
            }
            GAS_REQUIRE(reduce_blocks <= 0x7FFFFFFFLL, "%s: too large for one launch", who);
        }
        for (int t = 0; t < 4; ++t) {
            if (blocks[t] == 0) continue;
            const gas_status st = launch_dw_blocks(t, blocks[t], nullptr, &tile[t], s);
            if (st != GAS_OK) return st;
        }
        hipLaunchKernelGGL(dw_batch_reduce_kernel, dim3((unsigned)reduce_blocks), dim3(256), 0, s, all);
        GAS_CHECK_HIP(hipGetLastError());
    }
    return GAS_OK;
}

gas_status gas_linear_bwd_weight_static(const void* Z, int64_t ldz, const void* GP, int64_t ldgp, int64_t n_rows,
                                        int32_t F_in, int32_t F_out, gas_dtype dt, float c_weight, float* dW,
                                        void* stream) {
    return run_dw(Z, ldz, GP, ldgp, n_rows, F_in, F_out, dt, c_weight, dW, nullptr, 0, true, stream);
}

gas_status gas_relu_bwd(const void* GY, int64_t ldgy, const void* Y, int64_t ldy, int64_t n_rows, int32_t F,
                        gas_dtype dt, void* GP, int64_t ldgp, void* stream) {
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "gas_relu_bwd: unknown dtype %d", (int)dt);
    GAS_REQUIRE(n_rows >= 0 && F > 0, "gas_relu_bwd: n_rows=%lld F=%d", (long long)n_rows, F);
    if (n_rows == 0) return GAS_OK;
    GAS_REQUIRE(GY && Y && GP, "gas_relu_bwd: null pointer");
    GAS_REQUIRE(ldgy >= F && ldy >= F && ldgp >= F, "gas_relu_bwd: row stride smaller than F");
    const int eb = elem_bytes(dt);
    const bool vec = aligned16(GY) && aligned16(Y) && aligned16(GP) && (F * eb) % 16 == 0 && (ldgy * eb) % 16 == 0 &&
                     (ldy * eb) % 16 == 0 && (ldgp * eb) % 16 == 0;
    const int v = vec ? F * eb / 16 : 0;
    const int64_t items = vec ? n_rows * v : n_rows * (int64_t)F;
    const int64_t blocks = (items + 255) / 256;
    GAS_REQUIRE(blocks <= 0x7FFFFFFFLL, "gas_relu_bwd: too many elements for one launch");
    const char* gy = static_cast<const char*>(GY);
    const char* y = static_cast<const char*>(Y);
    char* gp = static_cast<char*>(GP);
    if (dt == GAS_BF16)
        hipLaunchKernelGGL(relu_bwd_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, gy, ldgy, y,
                           ldy, gp, ldgp, n_rows, F, v);
    else
        hipLaunchKernelGGL(relu_bwd_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, gy, ldgy,
                           y, ldy, gp, ldgp, n_rows, F, v);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

static gas_status run_mlp2(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W1, int32_t F_hid,
                           const void* b1, const void* W2, int32_t F_out, const void* b2, gas_dtype dt, int relu_out,
                           void* Y, int64_t ldy, void* stream, const PushTarget& push, void* H_out = nullptr,
                           int64_t ldh_out = 0) {
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "gas_mlp2: unknown dtype %d", (int)dt);
    GAS_REQUIRE(!H_out || ldh_out >= F_hid, "gas_mlp2_keep: row stride of the hidden activation smaller than F_hid");
    GAS_REQUIRE(!H_out || (H_out != Y && H_out != Z), "gas_mlp2_keep: the hidden activation aliases Z or Y");
    if (push.idx) {
        GAS_REQUIRE(push.hist && push.ld_hist >= F_out && push.n_hist_rows > 0, "gas_mlp2_push: bad history table");
        GAS_REQUIRE(push.hist != Y, "gas_mlp2_push: the history table aliases the output");
    }
    GAS_REQUIRE(n_rows >= 0 && F_in > 0 && F_hid > 0 && F_out > 0, "gas_mlp2: n_rows=%lld F_in=%d F_hid=%d F_out=%d",
                (long long)n_rows, F_in, F_hid, F_out);
    GAS_REQUIRE(F_hid <= kHidMax, "gas_mlp2: F_hid=%d exceeds %d", F_hid, kHidMax);
    if (n_rows == 0) return GAS_OK;
    GAS_REQUIRE(Z && W1 && W2 && Y, "gas_mlp2: null pointer");
    GAS_REQUIRE(ldz >= F_in && ldy >= F_out, "gas_mlp2: row stride smaller than the row");
    GAS_REQUIRE(Y != Z, "gas_mlp2: Y must not alias Z");
    MlpArgs a;
    a.Z = static_cast<const char*>(Z); a.ldz = ldz;
    a.W1 = static_cast<const char*>(W1); a.b1 = static_cast<const char*>(b1);
    a.W2 = static_cast<const char*>(W2); a.b2 = static_cast<const char*>(b2);
    a.Y = static_cast<char*>(Y); a.ldy = ldy;
    a.M = n_rows; a.K = F_in; a.H = F_hid; a.N = F_out;
    a.relu_out = relu_out;
    hipStream_t s = (hipStream_t)stream;
    const int q = dt == GAS_F32 ? 4 : 8;    // elements per 16 bytes
    const bool vec = aligned16(Z) && aligned16(W1) && aligned16(W2) && ldz % q == 0 && F_in % q == 0 &&
                     F_hid % q == 0 && F_out % q == 0;
    // The fused kernel holds both weight matrices in registers: for a narrow hidden layer most wavefronts hold nothing.  us, two products
    // (without a place for the hidden rows the tiled kernel) and fused:
    // - with that place, hidden 64 wide: 2,000 rows 8.1 and 10.1, 300,000 48 and 72, from 256 inputs 50,000 21.6 and 26.0, 150,000 52.2 and 49.9;
    //   128 wide: 4,096 rows 10.7 and 11.0, 6,000 11.7 and 11.3, 12,000 13.3 and 11.7; 256 wide: 500 rows 14.5 and 14.2, 30,000 39.7 and 20.7;
    // - without it, hidden 64 wide: 4,096 rows 8.7 and 10.1, 24,000 11.4 and 13.6, 60,000 20.7 and 19.2, from 256 inputs 1,000 14.0 and 12.6, 24,000
    //   19.5 and 17.9; 256 wide: 500 rows 20.8 and 14.2.
    // A Push, which the fused kernel stores itself, has a copy of the rows after the others: with the place, hidden 64 wide, 500 rows 12.2 and
    // 10.7, 24,000 15.4 and 15.1, 40,000 17.8 and 18.8, from 256 inputs 500 15.1 and 13.5, 64,000 30.4 and 27.9; 128 wide 4,096 14.7 and 11.7; without it,
    // hidden 64 wide, 500 rows 12.1 and 10.1, 64,000 26.9 and 21.4.
    const bool scatter = push.idx && aligned16(push.hist) && push.ld_hist % 8 == 0;
    const bool fused = F_hid > 128 || (scatter ? !H_out || F_hid > 64 || F_in > 64 || n_rows <= 30000
                                       : H_out ? F_hid > 64 ? n_rows > 5000 : F_in > 128 && n_rows > 100000
                                               : F_hid > 64 || F_in > 128 || n_rows > 30000);
    const bool ws_path = dt == GAS_BF16 && vec && fused && F_in <= 256 && F_out <= 256 && aligned16(Y) && ldy % 8 == 0 &&
                         ldz < (1 << 24) && ldy < (1 << 24) &&             // offsets inside a 64-row tile are 32-bit
                         (!H_out || (aligned16(H_out) && ldh_out % 8 == 0 && ldh_out < (1 << 24)));
    if (H_out && !ws_path) {
        // only the weights-stationary kernel stores the hidden activation on its way: elsewhere two stored linears
        gas_status st = run_linear("gas_mlp2_keep", Z, ldz, n_rows, F_in, W1, 0, F_hid, b1, dt, 0.f, 1.f, 1, nullptr, 0,
                                   H_out, ldh_out, s);
        if (st != GAS_OK) return st;
        return run_linear("gas_mlp2_keep", H_out, ldh_out, n_rows, F_hid, W2, 0, F_out, b2, dt, 0.f, 1.f, relu_out,
                          nullptr, 0, Y, ldy, s, push);
    }
    const int gn = (F_out + 255) / 256;
    if (n_rows > 0x7FFFFFFFLL || gn > 65535) return fail(GAS_ERR_ARG, "gas_mlp2: problem too large for one launch");
    if (dt == GAS_F32) {
        constexpr int smem = 4 * (kMlpRowsF32 * (kHidMax + 4 + kBK + 4) + kBK * (256 + 4));
        static const hipError_t e1 = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp2_f32_kernel<true>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        static const hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp2_f32_kernel<false>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        GAS_CHECK_HIP(e1);
        GAS_CHECK_HIP(e2);
        dim3 grid((unsigned)((n_rows + kMlpRowsF32 - 1) / kMlpRowsF32), (unsigned)gn);
        if (vec) hipLaunchKernelGGL(mlp2_f32_kernel<true>, grid, dim3(256), smem, s, a);
        else hipLaunchKernelGGL(mlp2_f32_kernel<false>, grid, dim3(256), smem, s, a);
    } else if (ws_path) {
        // the kernel scatters the rows itself if the history rows take 16-byte stores; else the row copy follows
        WsArgs w{};
        w.Z = static_cast<const uint16_t*>(Z); w.ldz = ldz;
        w.W1 = static_cast<const uint16_t*>(W1); w.b1 = static_cast<const uint16_t*>(b1);
        w.W2 = static_cast<const uint16_t*>(W2); w.b2 = static_cast<const uint16_t*>(b2);
        w.Y = static_cast<uint16_t*>(Y); w.ldy = ldy;
        w.M = n_rows; w.n_tiles = (n_rows + kWsRows - 1) / kWsRows;
        w.K = F_in; w.H = F_hid; w.N = F_out;
        w.c_id = 0.f; w.c_w = 1.f; w.relu1 = 1; w.relu_out = relu_out;
        if (scatter) { w.push_idx = push.idx; w.push_hist = static_cast<uint16_t*>(push.hist); w.ld_push = push.ld_hist; }
        w.H_out = static_cast<uint16_t*>(H_out); w.ldh_out = ldh_out;
        const gas_status st = F_in <= 128 ? launch_ws_mlp<8, 16>(w, s) : launch_ws_mlp<16, 16>(w, s);
        return (st != GAS_OK || scatter) ? st : push_after(push, Y, ldy, n_rows, F_out, dt, s);
    } else {
        constexpr int smem = 2 * (kMlpRowsBF16 * (kHidMax + 8 + kBKh + 8) + 256 * (kBKh + 8));
        static const hipError_t e1 = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp2_bf16_kernel<false>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        static const hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp2_bf16_kernel<true>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        GAS_CHECK_HIP(e1);
        GAS_CHECK_HIP(e2);
        const dim3 grid((unsigned)((n_rows + kMlpRowsBF16 - 1) / kMlpRowsBF16), (unsigned)gn);
        if (vec) hipLaunchKernelGGL(mlp2_bf16_kernel<false>, grid, dim3(256), smem, s, a);
        else hipLaunchKernelGGL(mlp2_bf16_kernel<true>, grid, dim3(512), smem, s, a);
    }
    GAS_CHECK_HIP(hipGetLastError());
    return push_after(push, Y, ldy, n_rows, F_out, dt, s);
}

gas_status gas_mlp2(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W1, int32_t F_hid,
                    const void* b1, const void* W2, int32_t F_out, const void* b2, gas_dtype dt, int relu_out,
                    void* Y, int64_t ldy, void* stream) {
    return run_mlp2(Z, ldz, n_rows, F_in, W1, F_hid, b1, W2, F_out, b2, dt, relu_out, Y, ldy, stream, PushTarget());
}

gas_status gas_mlp2_push(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W1, int32_t F_hid,
                         const void* b1, const void* W2, int32_t F_out, const void* b2, gas_dtype dt, int relu_out,
                         void* Y, int64_t ldy, const int32_t* idx, void* hist, int64_t n_hist_rows, int64_t ld_hist,
                         void* stream) {
    GAS_REQUIRE(idx || n_rows == 0, "gas_mlp2_push: null index array");
    PushTarget p;
    p.idx = idx; p.hist = hist; p.n_hist_rows = n_hist_rows; p.ld_hist = ld_hist;
    return run_mlp2(Z, ldz, n_rows, F_in, W1, F_hid, b1, W2, F_out, b2, dt, relu_out, Y, ldy, stream, p);
}

gas_status gas_mlp2_keep(const void* Z, int64_t ldz, int64_t n_rows, int32_t F_in, const void* W1, int32_t F_hid,
                         const void* b1, const void* W2, int32_t F_out, const void* b2, gas_dtype dt, int relu_out,
                         void* Y, int64_t ldy, void* H_out, int64_t ldh_out, const int32_t* idx, void* hist,
                         int64_t n_hist_rows, int64_t ld_hist, void* stream) {
    GAS_REQUIRE(H_out || n_rows == 0, "gas_mlp2_keep: null hidden activation");
    GAS_REQUIRE((idx == nullptr) == (hist == nullptr), "gas_mlp2_keep: idx and hist go together");
    PushTarget p;
    p.idx = idx; p.hist = hist; p.n_hist_rows = n_hist_rows; p.ld_hist = ld_hist;
    return run_mlp2(Z, ldz, n_rows, F_in, W1, F_hid, b1, W2, F_out, b2, dt, relu_out, Y, ldy, stream, p, H_out, ldh_out);
}

}  // extern "C"
