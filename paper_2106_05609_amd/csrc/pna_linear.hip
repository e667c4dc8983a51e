// PNA's transform (paper, operator appendix) by the rows' degrees.  Its input is [h | A | s A | A / s]: the row itself, three
// aggregates A and their products with the degree scalers s = log(d + 1) / delta and 1 / s, 2/3 of the columns of a typical
// layer being a scalar times others.  With W = [Wh; Wa; Wb; Wc] cut the same way
//     [h | A | s A | A / s] W = h Wh + A (Wa + s Wb + Wc / s),
// and the matrix in brackets depends on the row's degree d alone.  Rows of one degree share it: they are taken together,
// and a row costs F + 3 F1 columns instead of F + 9 F1 (448 instead of 832 for 256 and 64).  The same for the input gradient,
// whose last 6 F1 columns the aggregation's backward pass only adds up again, and for the weight gradient, where
// dWa, dWb, dWc are the degrees' products A^T G summed with the weights 1, s and 1 / s.
//
// fp32 products of the tiles of split.h, bounded as those are (matrix pipe and vector unit in turn) and by whole rounds of
// workgroups: 50,000 rows, 256 + 64 x 3 -> 256, degrees up to 26: 105 us (nine blocks 158), input gradient 102 (146), weight
// gradient 119 (151), the degrees' matrices 7.  Relative error against 64 bits 2.1e-7 (nine blocks 2.8e-7).
#include "common.h"
#include "split.h"

namespace gas {
namespace {

constexpr int kMaxDegree = 63;                // a degree for every lane
constexpr int kTile = 128;                    // rows of a product's tile
// Rows of a weight gradient's slab, whose partial is of the weights' size: about 128 slabs and one more for a degree, up to the
// 4,096 rows of the plain gradient's.  256 + 64 x 3 -> 256, degrees up to 26, in MB: 50,000 rows 57, 1,000,000 125 (by 512
// rows throughout 908; the nine blocks' plain gradient 209).
constexpr int kSlabStep = 512, kMostSlab = 4096;
inline int slab_rows(int64_t n) {
    const int64_t s = (n + 128 * kSlabStep - 1) / (128 * kSlabStep) * kSlabStep;
    return (int)(s < kSlabStep ? kSlabStep : s > kMostSlab ? kMostSlab : s);
}

// The rows by degree, in a buffer of the caller's: counts, then tiles and slabs (degree, first position, rows), the row
// ids, ascending for each degree, and what the building of the lists needs: of each degree, its rows in every workgroup's share.
struct GroupsHead { int32_t n_tiles, n_slabs, count[kMaxDegree + 1], pad[2]; };
struct Part { int32_t degree, start, rows, pad; };
constexpr int kShare = 1024;                  // rows of a workgroup that counts or lists them
inline int64_t most_tiles(int64_t n, int d) { return n / kTile + d + 1; }
inline int64_t most_slabs(int64_t n, int d) { return n / slab_rows(n) + d + 1; }
inline int64_t shares(int64_t n) { return (n + kShare - 1) / kShare; }
struct Groups {
    GroupsHead* head; Part* tile; Part* slab; int32_t* row; int32_t* share;
    int in_slab;                              // rows of a slab
    Groups(void* p, int64_t n, int d)
        : head(static_cast<GroupsHead*>(p)), tile(reinterpret_cast<Part*>(head + 1)), slab(tile + most_tiles(n, d)),
          row(reinterpret_cast<int32_t*>(slab + most_slabs(n, d))), share(row + n),
          in_slab(slab_rows(n)) {}
};

__device__ __forceinline__ int degree_of(const int32_t* rowptr, int64_t r, int most) {
    return min(max(rowptr[r + 1] - rowptr[r], 0), most);
}

// Sum over the lanes up to this one.
__device__ __forceinline__ int wave_scan(int v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o);
        if ((int)(threadIdx.x & 63) >= o) v += t;
    }
    return v;
}

// The lists in three launches, whose reads and stores are of the size of the row pointer: bounded by the launches and by the turns
// of the third, one for a degree that 64 rows hold.  50,000 rows of up to 26 entries 18 us, 1,000,000 30 us (one launch of a
// workgroup for each degree that walks all rows twice: 48 and 856).
// 1. The workgroup's rows of every degree.
__global__ __launch_bounds__(256) void groups_count_kernel(const int32_t* rowptr, int64_t n, int most, Groups g) {
    __shared__ int count[kMaxDegree + 1];
    const int tid = threadIdx.x;
    if (tid <= kMaxDegree) count[tid] = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * kShare;
    for (int64_t r = r0 + tid; r < min(n, r0 + kShare); r += 256) atomicAdd(&count[degree_of(rowptr, r, most)], 1);
    __syncthreads();
    if (tid <= most) g.share[(int64_t)tid * gridDim.x + blockIdx.x] = count[tid];
}

// 2. One wavefront for a degree: its counts become the rows of the shares before.
__global__ __launch_bounds__(64) void groups_scan_kernel(Groups g, int n_shares) {
    const int lane = threadIdx.x;
    int32_t* c = g.share + (int64_t)blockIdx.x * n_shares;
    int before = 0;
    for (int i0 = 0; i0 < n_shares; i0 += 64) {
        const int own = i0 + lane < n_shares ? c[i0 + lane] : 0;
        const int sum = wave_scan(own);
        if (i0 + lane < n_shares) c[i0 + lane] = before + sum - own;
        before += __shfl(sum, 63);
    }
    if (lane == 0) g.head->count[blockIdx.x] = before;
}

// 3. The workgroup's rows to their places (wavefront w has the w-th quarter of them, 64 at a time); the tiles and slabs of the degrees
// blockIdx.x, blockIdx.x + gridDim.x, ...
__global__ __launch_bounds__(256) void groups_list_kernel(const int32_t* rowptr, int64_t n, int most, Groups g) {
    __shared__ int rows[kMaxDegree + 1], first[kMaxDegree + 1], tile0[kMaxDegree + 1], slab0[kMaxDegree + 1], next[4][kMaxDegree + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    next[wave][lane] = 0;
    if (wave == 0) {                          // lane d: degree d
        const int c = lane <= most ? g.head->count[lane] : 0, t = (c + kTile - 1) / kTile, s = (c + g.in_slab - 1) / g.in_slab;
        const int at = wave_scan(c), tile = wave_scan(t), slab = wave_scan(s);
        rows[lane] = c;
        first[lane] = at - c;
        tile0[lane] = tile - t;
        slab0[lane] = slab - s;
        if (blockIdx.x == 0 && lane == 63) { g.head->n_tiles = tile; g.head->n_slabs = slab; }
    }
    __syncthreads();
    for (int d = blockIdx.x; d <= most; d += gridDim.x) {
        const int c = rows[d], at = first[d];
        for (int i = tid; i * kTile < c; i += 256) g.tile[tile0[d] + i] = Part{d, at + i * kTile, min(kTile, c - i * kTile), 0};
        for (int i = tid; i < (c + g.in_slab - 1) / g.in_slab; i += 256)
            g.slab[slab0[d] + i] = Part{d, at + i * g.in_slab, min(g.in_slab, c - i * g.in_slab), 0};
    }
    constexpr int kSteps = kShare / 256;
    const int64_t r0 = (int64_t)blockIdx.x * kShare + wave * (kShare / 4) + lane;
    int degree[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const int64_t r = r0 + 64 * i;
        degree[i] = r < n ? degree_of(rowptr, r, most) : -1;
        if (r < n) atomicAdd(&next[wave][degree[i]], 1);
    }
    __syncthreads();
    if (tid <= most) {
        int at = first[tid] + g.share[(int64_t)tid * gridDim.x + blockIdx.x];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int c = next[w][tid];
            next[w][tid] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        uint64_t left = __ballot(degree[i] >= 0);
        while (left) {                        // the lanes of one degree at a time, ascending
            const int d = __builtin_amdgcn_readlane(degree[i], __ffsll((unsigned long long)left) - 1);
            const uint64_t same = __ballot(degree[i] == d);
            const int at = next[wave][d];
            if (degree[i] == d) g.row[at + __popcll(same & ((1ull << lane) - 1))] = (int)(r0 + 64 * i);
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) next[wave][d] = at + __popcll(same);
            __builtin_amdgcn_wave_barrier();
            left &= ~same;
        }
    }
}

struct PnaLinArgs {
    Groups g;
    const float* A; int64_t lda;       // forward: [h | A ..]; backward: the gradient
    const float* W;                    // of every degree, one after the other: [F + 3 F1][N]
    int K, N;                          // columns of A that are taken, columns of the output
    float* Y; int64_t ldy;
    int relu;
    const int32_t* push_idx; float* push; int64_t ldp;
};

__device__ __forceinline__ float scaler(int degree, float inv_delta) { return logf((float)degree + 1.f) * inv_delta; }

// blockIdx.y: the degree
__global__ __launch_bounds__(256) void degree_weights_kernel(Groups g, const float* W, int F, int F1, int N, float inv_delta, float* out) {
    const int d = blockIdx.y;
    if (g.head->count[d] == 0) return;
    const int64_t per = (int64_t)(F + 3 * F1) * N, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= per) return;
    float w = W[i];
    if (i >= (int64_t)F * N) {
        const float s = scaler(d, inv_delta);
        w += s * W[i + 3ll * F1 * N] + (d > 0 ? 1.f / s : 0.f) * W[i + 6ll * F1 * N];
    }
    out[d * per + i] = w;
}

// As linear_split_kernel: the column tiles of one row tile follow each other on one XCD.
template <int BN, bool TRANS>
__global__ __launch_bounds__(256, BN == 128 ? 2 : 3) void pna_linear_kernel(PnaLinArgs a) {
    using G = SplitGemm<kTile, BN, 2, 2, 2, true, TRANS, 1, true, false>;
    constexpr int TM = G::TM, TN = G::TN;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned gn = (a.N + BN - 1) / BN, of_xcd = blockIdx.x / 8;
    const int tile = (int)(of_xcd / gn * 8 + blockIdx.x % 8);
    if (tile >= a.g.head->n_tiles) return;
    const Part part = a.g.tile[tile];
    const int n0 = (int)(of_xcd % gn) * BN, wm0 = (wave >> 1) * (kTile / 2), wn0 = (wave & 1) * (BN / 2);
    const float* W = a.W + (int64_t)part.degree * a.K * a.N;
    const int64_t ldw = TRANS ? a.K : a.N, end = part.start + part.rows;
    G g;
    g.ta.idx = a.g.row;
    f32x16 acc[TM][TN];
    if (!g.run(a.A, a.lda, part.start, end, W, ldw, n0, a.N, 0, a.K, reinterpret_cast<uint16_t*>(smem), wm0, wn0, acc))
        plain_tile<TM, TN, true, TRANS, true, false>(a.A, a.lda, part.start + wm0, end, W, ldw, n0 + wn0, a.N, 0, a.K, acc, a.g.row);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int local = wm0 + 32 * i + 8 * (r / 4) + 4 * lh + r % 4;
            if (local >= part.rows) continue;
            const int64_t row = a.g.row[part.start + local];
            float* y = a.Y + row * a.ldy + n0 + wn0 + li;
            float* h = a.push ? a.push + (int64_t)a.push_idx[row] * a.ldp + n0 + wn0 + li : nullptr;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (n0 + wn0 + 32 * j + li >= a.N) continue;
                const float x = a.relu ? fmaxf(acc[i][j][r], 0.f) : acc[i][j][r];
                y[32 * j] = x;
                if (h) h[32 * j] = x;
            }
        }
}

struct PnaDwArgs {
    Groups g;
    const float* Z; int64_t ldz;       // [h | A ..], K columns of it
    const float* G; int64_t ldg;       // [.., N]
    int K, N, F, F1;
    float inv_delta;
    float* partial;                    // [slab][K][N]
    float* dW;                         // [F + 9 F1][N]
};

__global__ __launch_bounds__(256, 2) void pna_dw_kernel(PnaDwArgs a) {
    using S = SplitGemm<kTile, kTile, 2, 2, 2, false, false, 1, true, true>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tn = (a.N + kTile - 1) / kTile, tiles = (a.K + kTile - 1) / kTile * tn, of_xcd = blockIdx.x / 8, tile = of_xcd % tiles;
    const int slab = (int)(of_xcd / tiles * 8 + blockIdx.x % 8);
    if (slab >= a.g.head->n_slabs) return;
    const Part part = a.g.slab[slab];
    const int k0 = (int)(tile / tn) * kTile, n0 = (int)(tile % tn) * kTile, wk0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
    // the slab's row ids in LDS: asked of memory where the rows are, every step waits for them first (139 us, 119 by LDS)
    int32_t* ids = reinterpret_cast<int32_t*>(smem + S::kLdsBytes);
    for (int i = threadIdx.x; i < part.rows; i += 256) ids[i] = a.g.row[part.start + i];
    __syncthreads();
    S g;
    g.ta.idx = g.tb.idx = ids;
    f32x16 acc[S::TM][S::TN];
    if (!g.run(a.Z, a.ldz, k0, a.K, a.G, a.ldg, n0, a.N, 0, part.rows, reinterpret_cast<uint16_t*>(smem), wk0, wn0, acc))
        plain_tile<S::TM, S::TN, false, false, true, true>(a.Z, a.ldz, k0 + wk0, a.K, a.G, a.ldg, n0 + wn0, a.N, 0, part.rows, acc, ids);
    float* out = a.partial + (int64_t)slab * a.K * a.N;
#pragma unroll
    for (int i = 0; i < S::TM; ++i)
#pragma unroll
        for (int j = 0; j < S::TN; ++j) {
            const int n = n0 + wn0 + 32 * j + li;
            if (n >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wk0 + 32 * i + 8 * (r / 4) + 4 * lh + r % 4;
                if (k < a.K) out[(int64_t)k * a.N + n] = acc[i][j][r];
            }
        }
}

// The slabs' partials, in slab order (eight threads an output, every eighth slab each, added in a fixed order): the rows of dWh as
// they are, those of the aggregates with the weights 1, s and 1 / s of the slab's degree.
__global__ __launch_bounds__(256) void pna_dw_reduce_kernel(PnaDwArgs a) {
    __shared__ float part[3][8][32];
    __shared__ float up[kMaxDegree + 1], down[kMaxDegree + 1];
    if (threadIdx.x <= kMaxDegree) {
        const float s = scaler(threadIdx.x, a.inv_delta);
        up[threadIdx.x] = s;
        down[threadIdx.x] = threadIdx.x > 0 ? 1.f / s : 0.f;
    }
    __syncthreads();
    const int o = threadIdx.x % 32, way = threadIdx.x / 32, n_slabs = a.g.head->n_slabs;
    const int64_t per = (int64_t)a.K * a.N, i = (int64_t)blockIdx.x * 32 + o;
    float t[3] = {0.f, 0.f, 0.f};
    if (i < per) {
        for (int s0 = way; s0 < n_slabs; s0 += 32) {
            float x[4];
            int d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = s0 + 8 * u;
                x[u] = s < n_slabs ? a.partial[s * per + i] : 0.f;
                d[u] = s < n_slabs ? a.g.slab[s].degree : 0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t[0] += x[u];
                t[1] = fmaf(up[d[u]], x[u], t[1]);
                t[2] = fmaf(down[d[u]], x[u], t[2]);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) part[b][way][o] = t[b];
    __syncthreads();
    if (way >= 3 || i >= per || (way > 0 && i < (int64_t)a.F * a.N)) return;
    float sum = part[way][0][o];
#pragma unroll
    for (int w = 1; w < 8; ++w) sum += part[way][w][o];
    a.dW[i + 3ll * way * a.F1 * a.N] = sum;
}

template <int BN, bool TRANS>
gas_status launch_linear(const PnaLinArgs& a, int64_t n, int most, hipStream_t s) {
    constexpr int smem = SplitGemm<kTile, BN, 2, 2, 2, true, TRANS, 1, true, false>::kLdsBytes;
    const int64_t blocks = (most_tiles(n, most) + 7) / 8 * 8 * ((a.N + BN - 1) / BN);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(pna_linear_kernel<BN, TRANS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    GAS_CHECK_HIP(attr);
    hipLaunchKernelGGL((pna_linear_kernel<BN, TRANS>), dim3((unsigned)blocks), dim3(256), smem, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}
// 64-column tiles where they leave fewer columns over (50,000 rows of 256 -> 448: seven tiles of 64 102 us, four of 128 110)
template <bool TRANS>
gas_status run_linear(const PnaLinArgs& a, int64_t n, int most, hipStream_t s) {
    return (a.N + 63) / 64 * 64 < (a.N + 127) / 128 * 128 ? launch_linear<64, TRANS>(a, n, most, s) : launch_linear<128, TRANS>(a, n, most, s);
}

gas_status check(const char* who, int64_t n_rows, int32_t max_degree, int32_t F, int32_t F1, int32_t N, float delta) {
    GAS_REQUIRE(n_rows >= 0 && n_rows < (1ll << 30) && max_degree >= 0 && max_degree <= kMaxDegree,
                "%s: n_rows=%lld, degrees up to %d (at most %d)", who, (long long)n_rows, max_degree, kMaxDegree);
    GAS_REQUIRE(F > 0 && F1 > 0 && N > 0 && F <= 65536 && F1 <= 65536 && N <= 65536 && (F + 3ll * F1) * N < (1ll << 29),
                "%s: widths %d, %d, %d", who, F, F1, N);      // 32 weights a workgroup of the last sum: as one_launch
    GAS_REQUIRE(delta > 0.f, "%s: delta must be positive", who);
    return GAS_OK;
}

// Whether workgroups of 256, a multiple of eight parts by `columns`, fit one launch (fewer than 2^32 threads); asked before
// anything is launched.
bool one_launch(int64_t parts, int64_t columns) { return (parts + 7) / 8 * 8 * columns < (1ll << 24); }

gas_status degree_weights(const Groups& g, const void* W, int32_t F, int32_t F1, int32_t N, float delta, int max_degree, void* out,
                          hipStream_t s) {
    const int64_t per = (int64_t)(F + 3 * F1) * N;
    hipLaunchKernelGGL(degree_weights_kernel, dim3((unsigned)((per + 255) / 256), (unsigned)max_degree + 1), dim3(256), 0, s, g,
                       static_cast<const float*>(W), F, F1, N, 1.f / delta, static_cast<float*>(out));
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

}  // namespace
}  // namespace gas

using namespace gas;

extern "C" {

int64_t gas_pna_groups_workspace(int64_t n_rows, int32_t max_degree) {
    if (n_rows < 0 || max_degree < 0 || max_degree > kMaxDegree) return 0;
    return (int64_t)sizeof(GroupsHead) + (int64_t)sizeof(Part) * (most_tiles(n_rows, max_degree) + most_slabs(n_rows, max_degree)) +
           4 * (n_rows + shares(n_rows) * (max_degree + 1));
}

gas_status gas_pna_groups(const int32_t* rowptr, int64_t n_rows, int32_t max_degree, void* groups, void* stream) {
    const gas_status st = check("gas_pna_groups", n_rows, max_degree, 1, 1, 1, 1.f);
    if (st != GAS_OK || n_rows == 0) return st;
    GAS_REQUIRE(rowptr && groups, "gas_pna_groups: null pointer");
    GAS_REQUIRE(aligned16(groups), "gas_pna_groups: the buffer must be 16-byte aligned");
    const Groups g(groups, n_rows, max_degree);
    const unsigned blocks = (unsigned)shares(n_rows);
    hipLaunchKernelGGL(groups_count_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, rowptr, n_rows, (int)max_degree, g);
    hipLaunchKernelGGL(groups_scan_kernel, dim3((unsigned)max_degree + 1), dim3(64), 0, (hipStream_t)stream, g, (int)blocks);
    hipLaunchKernelGGL(groups_list_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, rowptr, n_rows, (int)max_degree, g);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

int64_t gas_pna_linear_workspace(int32_t max_degree, int32_t F, int32_t F1, int32_t F_out) {
    if (max_degree < 0 || F <= 0 || F1 <= 0 || F_out <= 0) return 0;
    return 4ll * (max_degree + 1) * ((int64_t)F + 3 * F1) * F_out;
}

gas_status gas_pna_linear(const void* groups, int64_t n_rows, int32_t max_degree, const void* X, int64_t ldx, int32_t F, int32_t F1,
                          const void* W, int32_t F_out, float delta, int relu, void* Y, int64_t ldy, const int32_t* push_idx,
                          void* push_hist, int64_t ld_push, void* workspace, int64_t workspace_bytes, void* stream) {
    const char* who = "gas_pna_linear";
    gas_status st = check(who, n_rows, max_degree, F, F1, F_out, delta);
    if (st != GAS_OK || n_rows == 0) return st;
    GAS_REQUIRE(groups && X && W && Y && workspace, "%s: null pointer", who);
    GAS_REQUIRE(ldx >= F + 3 * (int64_t)F1 && ldy >= F_out && (!push_hist || ld_push >= F_out), "%s: row stride smaller than the row", who);
    GAS_REQUIRE((push_idx == nullptr) == (push_hist == nullptr), "%s: push_idx and push_hist go together", who);
    GAS_REQUIRE(Y != X, "%s: the output must not alias the input", who);
    GAS_REQUIRE(one_launch(most_tiles(n_rows, max_degree), (F_out + 63) / 64), "%s: too many rows for one launch", who);
    GAS_REQUIRE(workspace_bytes >= gas_pna_linear_workspace(max_degree, F, F1, F_out), "%s: workspace too small", who);
    const Groups g(const_cast<void*>(groups), n_rows, max_degree);
    st = degree_weights(g, W, F, F1, F_out, delta, max_degree, workspace, (hipStream_t)stream);
    if (st != GAS_OK) return st;
    const PnaLinArgs a{g, static_cast<const float*>(X), ldx, static_cast<const float*>(workspace), F + 3 * F1, F_out, static_cast<float*>(Y),
                       ldy, relu, push_idx, static_cast<float*>(push_hist), ld_push};
    return run_linear<false>(a, n_rows, max_degree, (hipStream_t)stream);
}

gas_status gas_pna_linear_bwd_input(const void* groups, int64_t n_rows, int32_t max_degree, const void* G, int64_t ldg, int32_t F,
                                    int32_t F1, const void* W, int32_t F_out, float delta, void* GX, int64_t ldgx, void* workspace,
                                    int64_t workspace_bytes, void* stream) {
    const char* who = "gas_pna_linear_bwd_input";
    gas_status st = check(who, n_rows, max_degree, F, F1, F_out, delta);
    if (st != GAS_OK || n_rows == 0) return st;
    GAS_REQUIRE(groups && G && W && GX && workspace, "%s: null pointer", who);
    GAS_REQUIRE(ldg >= F_out && ldgx >= F + 3 * (int64_t)F1, "%s: row stride smaller than the row", who);
    GAS_REQUIRE(G != GX, "%s: the output must not alias the input", who);
    GAS_REQUIRE(one_launch(most_tiles(n_rows, max_degree), (F + 3 * F1 + 63) / 64), "%s: too many rows for one launch", who);
    GAS_REQUIRE(workspace_bytes >= gas_pna_linear_workspace(max_degree, F, F1, F_out), "%s: workspace too small", who);
    const Groups g(const_cast<void*>(groups), n_rows, max_degree);
    st = degree_weights(g, W, F, F1, F_out, delta, max_degree, workspace, (hipStream_t)stream);
    if (st != GAS_OK) return st;
    const PnaLinArgs a{g, static_cast<const float*>(G), ldg, static_cast<const float*>(workspace), F_out, F + 3 * F1, static_cast<float*>(GX),
                       ldgx, 0, nullptr, nullptr, 0};
    return run_linear<true>(a, n_rows, max_degree, (hipStream_t)stream);
}

int64_t gas_pna_linear_bwd_weight_workspace(int64_t n_rows, int32_t max_degree, int32_t F, int32_t F1, int32_t F_out) {
    if (n_rows < 0 || max_degree < 0 || F <= 0 || F1 <= 0 || F_out <= 0) return 0;
    return 4 * most_slabs(n_rows, max_degree) * ((int64_t)F + 3 * F1) * F_out;
}

gas_status gas_pna_linear_bwd_weight(const void* groups, int64_t n_rows, int32_t max_degree, const void* X, int64_t ldx, const void* G,
                                     int64_t ldg, int32_t F, int32_t F1, int32_t F_out, float delta, float* dW, void* workspace,
                                     int64_t workspace_bytes, void* stream) {
    const char* who = "gas_pna_linear_bwd_weight";
    gas_status st = check(who, n_rows, max_degree, F, F1, F_out, delta);
    if (st != GAS_OK || n_rows == 0) return st;
    GAS_REQUIRE(groups && X && G && dW && workspace, "%s: null pointer", who);
    GAS_REQUIRE(ldx >= F + 3 * (int64_t)F1 && ldg >= F_out, "%s: row stride smaller than the row", who);
    GAS_REQUIRE(workspace_bytes >= gas_pna_linear_bwd_weight_workspace(n_rows, max_degree, F, F1, F_out), "%s: workspace too small", who);
    const Groups g(const_cast<void*>(groups), n_rows, max_degree);
    const PnaDwArgs a{g, static_cast<const float*>(X), ldx, static_cast<const float*>(G), ldg, F + 3 * F1, F_out, F, F1, 1.f / delta,
                      static_cast<float*>(workspace), dW};
    const int64_t tiles = (int64_t)((a.K + kTile - 1) / kTile) * ((a.N + kTile - 1) / kTile);
    GAS_REQUIRE(one_launch(most_slabs(n_rows, max_degree), tiles), "%s: too many rows for one launch", who);
    constexpr int lds = SplitGemm<kTile, kTile, 2, 2, 2, false, false, 1, true, true>::kLdsBytes;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(pna_dw_kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds + 4 * kMostSlab);
    GAS_CHECK_HIP(attr);
    const int64_t blocks = (most_slabs(n_rows, max_degree) + 7) / 8 * 8 * tiles;
    hipLaunchKernelGGL(pna_dw_kernel, dim3((unsigned)blocks), dim3(256), lds + 4 * g.in_slab, (hipStream_t)stream, a);
    hipLaunchKernelGGL(pna_dw_reduce_kernel, dim3((unsigned)(((int64_t)a.K * a.N + 31) / 32)), dim3(256), 0, (hipStream_t)stream, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

}  // extern "C"
