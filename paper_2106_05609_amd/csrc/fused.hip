// One layer of the step in ONE launch for narrow layers (fp32, widths up to 128): the aggregation of Eq. (2) with
// its two sources (fresh in-batch rows, stored halo rows), the dense transform on the aggregated tile while it is
// still in LDS, and the Push of the result.  A deep narrow model (the 64-layer GCNII of the paper's experiments,
// width 64) spends its time on launches, not on bytes: its weight matrix is 16 KB and a whole tile of aggregated
// rows is 8 KB, so the layer needs neither the Z round trip through HBM nor a second launch.
// Wide layers (256) keep their two kernels: there the weights fill the register file of the transform.
#include "common.h"
#include "wave.h"

namespace gas {
namespace {

constexpr int kRows = 32;            // rows of the batch subgraph per tile = two 16-row MFMA blocks
constexpr int kMaxWidth = 128;
typedef f32x4 f32x4_any __attribute__((aligned(4)));      // a 16-byte access at a float's alignment

struct FusedArgs {
    const int32_t* rowptr; const int32_t* src; const float* val;
    int64_t n_rows, n_tiles;
    const float* X; int64_t ldx;
    const float* H; int64_t ldh;
    const float* R; int64_t ldr;
    const float* W; const float* bias;
    float* Y; int64_t ldy;
    float* Zout; int64_t ldzo;       // optional copy of the aggregated rows (a training pass reads them again)
    const int32_t* push_idx; float* PH; int64_t ldp;
    int K, N;                        // widths
    float diag, s_agg, s_res, c_id, c_w;
    int relu;
    // backward pass: aggregated rows are zero where mask <= 0, total += c_total * Y
    const float* mask; int64_t ldm;
    float* total; int64_t ldt;
    float c_total;
};

constexpr int kThreads = 256;        // four wavefronts: eight rows of the tile each

// Workgroups of four wavefronts, looping over tiles of 32 rows.  Per tile:
//   1. aggregation: wavefront w owns rows 8w .. 8w+7; a team of G lanes owns one row at a time, lane j its
//      16-byte pieces j and j + G (P loads per gathered row, each contiguous over the team).  The team reads
//      2 G source indices (and coefficients) with two loads (the next 2 G are requested before the current ones
//      are used); the lane that read an index forms the row's address, the team takes it over by two moves instead of
//      forming it G times.  The rows are gathered eight at a time and folded in index order; the finished row (scaled,
//      plus the diagonal and residual terms, requested before the gathers) goes to the LDS tile Zs.  With width 64 a
//      team is 8 lanes, so a wavefront works on its 8 rows at once and the whole chain (row pointers, indices,
//      rows) is walked once per tile.
//   2. transform: the weights are in registers from the start, wavefront w's 16 output columns (of 64; NB times that
//      for 128) by all k, so the four wavefronts share the products.  16x16x4 fp32 MFMAs, taken transposed: a lane has four
//      consecutive columns of a row, which get c_w * acc + c_id * Z + bias and ReLU and are stored to Y and to the
//      row's history slot as 16 bytes.
// 64 layers of 21,248 rows, width 64, 15 entries a row: 16.4 us each (17.7 with the loads past a row's end not switched off,
// kMaskedGathers; with the addresses formed by every lane, 32x32x2
// products by two of the four wavefronts and the weights in LDS 21.9).  Without the gathers 7.6 us, without the transform
// 13.7: what is left is the gather's chain of two to three batches and the rows that every XCD fetches anew (4.6 TB/s).
// BWD: the same on the adjoint (gas_spmm_t_relu_linear): the pattern is the CSC copy, the activations of the layer below mask
// the aggregated rows, the weights are taken transposed and a running total is kept.  21,248 rows of 64: 14.7 us
// where the aggregation by plan (19) and the input gradient (9) were two launches; the whole pass of 64 layers 3,780 -> 3,426 us.
// <8, 2, 2> spills 6 registers (BWD 11) to keep three wavefronts on a SIMD: 21,248 rows of 50, 64 -> 128, 33.5 us, with two
// and none spilled 41.9 (rows of 5: 15.4 and 15.7).
// Whether a team past its row's end fetches nothing; otherwise it fetches the row's last entry again, which it has just had.  The
// eight teams of a wavefront go by its longest row, two entries in five more than their own.  The mask takes 5 to 8 registers:
// it is on where the compiled kernel keeps its wavefronts on a SIMD and spills nothing for it.  Time without over with the mask, 30
// patterns (500 to 50,000 rows of 5 to 40 entries, even and power law), geometric mean: up to 32 columns to at most 64 1.01
// (BWD 1.02), 33 to 64 1.05 (1.02), 65 to 128 1.08, to more columns from up to 32 1.01, from 65 to 128 1.07 (1.06).  Off:
// 65 to 128 to at most 64 BWD, three wavefronts to two, 21,248 rows of 40 entries 40 -> 48 us; up to 32 to more than 64 BWD, four
// to three, 0.98; 33 to 64 to more than 64, twice the spills, 0.97 to 1.00.  A wavefront with one row of hundreds of entries among
// short ones is the slower with it (500 rows of 8, one of 500, 32 -> 32, 41 -> 45 us); passes over power-law batches of
// 50,000 rows, 32 -> 32, are not (221 -> 205).
template <int G, int P, int NB, bool BWD>
constexpr bool kMaskedGathers = G == 8 ? NB == 1 || (P == 1 && !BWD) : NB == 2 || !BWD;

template <int G, int P, int NB, bool BWD>
__global__ __launch_bounds__(kThreads, G == 8 ? 3 : 2) void spmm_linear_f32_kernel(FusedArgs a) {
    constexpr int KQ = G * P / 4, LDZ = 16 * KQ + 4;                      // steps of 16 k, floats of a row of Zs
    __shared__ __attribute__((aligned(16))) float Zs[kRows * LDZ];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int T = 64 / G, U = 8, RW = kRows / (kThreads / 64);        // teams, gathers in flight per lane (P loads each), rows per wavefront
    const int team = lane / G, j = lane % G;
    // Workgroups go to the eight XCDs in turn and each XCD has its own L2.  Every XCD gets one contiguous eighth
    // of the tiles: consecutive rows of a batch belong to one cluster of the partition and gather mostly from that
    // cluster's rows, which then stay in that XCD's L2 instead of being fetched into all eight.
    const int64_t per_xcd = (a.n_tiles + 7) / 8;
    const int xcd = blockIdx.x & 7;
    const int64_t tile_end = min(a.n_tiles, (xcd + 1) * per_xcd), tile0 = xcd * per_xcd + (blockIdx.x >> 3);
    if (tile0 >= tile_end) return;
    // the first row's pointers are requested before the weights, so the two latencies overlap
    int b_first, e_first;
    {
        const int64_t m = min(tile0 * kRows + wave * RW + team, a.n_rows - 1);
        b_first = a.rowptr[m];
        e_first = a.rowptr[m + 1];
    }
    // weights of k = 16 g + 4 lq .. + 3 and column 16 (wave + 4 b) + li; zero outside the matrix
    f32x4 w[NB][KQ];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < KQ; ++g) {
            const int n = 16 * (wave + 4 * b) + li, k = 16 * g + 4 * lq;
            if constexpr (BWD) {
                w[b][g] = *reinterpret_cast<const f32x4*>(a.W + (int64_t)min(n, a.N - 1) * a.K + min(k, a.K - 4));
            } else {
                const float* p = a.W + (int64_t)min(k, a.K - 4) * a.N + min(n, a.N - 1);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[b][g][e] = p[(int64_t)e * a.N];
            }
        }
    // the padding columns of Zs are cleared once (the aggregation never writes them)
    const int pad = 16 * KQ - a.K;
    for (int idx = tid; idx < kRows * pad; idx += kThreads) Zs[(idx / pad) * LDZ + a.K + idx % pad] = 0.f;

    const bool piece0 = 4 * j < a.K, piece1 = P == 2 && 4 * (j + G) < a.K;
    const int off0 = piece0 ? 16 * j : 0, off1 = piece1 ? 16 * (j + G) : 0;                  // bytes

    for (int64_t tile = tile0; tile < tile_end; tile += gridDim.x >> 3) {
        const int64_t m_tile = tile * kRows;
        // the history rows of output rows li and 16 + li: requested a whole aggregation before the epilogue stores to them
        int slot[2] = {0, 0};
        if (!BWD && a.push_idx) {
#pragma unroll
            for (int h = 0; h < 2; ++h) slot[h] = a.push_idx[min(m_tile + 16 * h + li, a.n_rows - 1)];
        }
        // ---- 1. aggregation
#pragma unroll 1
        for (int r = wave * RW + team; r < (wave + 1) * RW; r += T) {
            const bool row_on = m_tile + r < a.n_rows;
            const int64_t m = row_on ? m_tile + r : a.n_rows - 1;          // a row beyond the last repeats it; nothing stores it
            const bool have = tile == tile0 && r == wave * RW + team;      // requested before the weights
            const int b = have ? b_first : a.rowptr[m], e = have ? e_first : a.rowptr[m + 1];
            f32x4 acc[P], res[P], own[P], act[P];
            auto piece = [&](const float* base, int64_t ld, f32x4 (&v)[P]) {
                const char* row = reinterpret_cast<const char*>(base + m * ld);
                v[0] = *reinterpret_cast<const f32x4*>(row + off0);
                if constexpr (P == 2) v[1] = *reinterpret_cast<const f32x4*>(row + off1);
            };
            if (!BWD && a.R) piece(a.R, a.ldr, res);
            if (!BWD && a.diag != 0.f) piece(a.X, a.ldx, own);
            if constexpr (BWD) piece(a.mask, a.ldm, act);
#pragma unroll
            for (int p = 0; p < P; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
            // entries k + j and k + G + j (the row's last one past its end: a valid address, never folded)
            int s[2];
            float v[2];
            auto fetch = [&](int k) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int at = min(k + G * h + j, e - 1);
                    s[h] = a.src[at];
                    v[h] = a.val ? a.val[at] : 1.f;
                }
            };
            if (b < e) fetch(b);
            for (int k0 = b; k0 < e; k0 += 2 * G) {
                const int cnt = e - k0;
                int lo[2], hi[2], wt[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool fresh = s[h] >= 0;
                    const uint64_t p = (uint64_t)(fresh ? a.X : a.H) + (uint64_t)((int64_t)(fresh ? s[h] : -1 - s[h]) * (fresh ? a.ldx : a.ldh)) * 4;
                    lo[h] = (int)(uint32_t)p;
                    hi[h] = (int)(uint32_t)(p >> 32);
                    wt[h] = __float_as_int(v[h]);
                }
                fetch(min(k0 + 2 * G, e - 1));                            // the next indices, before these are used
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int q = 0; q < G; q += U) {
                        if (G * h + q >= cnt) break;
                        f32x4 x[U][P];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint64_t row = (uint64_t)(uint32_t)team_lane<G>(lo[h], q + u) | ((uint64_t)(uint32_t)team_lane<G>(hi[h], q + u) << 32);
                            if constexpr (kMaskedGathers<G, P, NB, BWD>) {
                                if (G * h + q + u < cnt) {
                                    x[u][0] = load_global<f32x4>(row + off0);
                                    if constexpr (P == 2) x[u][1] = load_global<f32x4>(row + off1);
                                }
                            } else {
                                const char* at = reinterpret_cast<const char*>(row);
                                x[u][0] = *reinterpret_cast<const f32x4*>(at + off0);
                                if constexpr (P == 2) x[u][1] = *reinterpret_cast<const f32x4*>(at + off1);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const float f = __int_as_float(team_lane<G>(wt[h], q + u));
                            if (G * h + q + u < cnt) {
#pragma unroll
                                for (int p = 0; p < P; ++p)
#pragma unroll
                                    for (int c = 0; c < 4; ++c) acc[p][c] = fmaf(f, x[u][p][c], acc[p][c]);
                            }
                        }
                    }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (!(p == 0 ? piece0 : piece1)) continue;
                f32x4 z;
#pragma unroll
                for (int c = 0; c < 4; ++c) z[c] = a.s_agg * acc[p][c];
                if (!BWD && a.diag != 0.f) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) z[c] = fmaf(a.diag, own[p][c], z[c]);
                }
                if (!BWD && a.R) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) z[c] = fmaf(a.s_res, res[p][c], z[c]);
                }
                if constexpr (BWD) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) z[c] = act[p][c] > 0.f ? z[c] : 0.f;
                }
                const int c0 = 4 * (j + G * p);
                *reinterpret_cast<f32x4*>(Zs + r * LDZ + c0) = z;
                if (a.Zout && row_on) *reinterpret_cast<f32x4*>(a.Zout + m * a.ldzo + c0) = z;      // as gas_spmm would have stored it
            }
        }
        // the total's rows are requested before the wait for the tile
        f32x4 sum[BWD ? NB : 1][2];
        if constexpr (BWD) {
            if (a.total) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        sum[b][h] = *reinterpret_cast<const f32x4*>(a.total + min(m_tile + 16 * h + li, a.n_rows - 1) * a.ldt + min(16 * (wave + 4 * b) + 4 * lq, a.N - 4));
            }
        }
        __syncthreads();                 // Zs complete
        // ---- 2. transform of the tile
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int n = 16 * (wave + 4 * b) + 4 * lq;                    // the lane's four columns
            if (16 * (wave + 4 * b) >= a.N) break;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int g = 0; g < KQ; ++g) {
                if (16 * g >= a.K) break;
                f32x4 z[2], f = w[b][g];
#pragma unroll
                for (int h = 0; h < 2; ++h) z[h] = *reinterpret_cast<const f32x4*>(Zs + (16 * h + li) * LDZ + 16 * g + 4 * lq);
                if (16 * g + 16 > a.K && 16 * g + 4 * lq >= a.K) f = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[e], z[h][e], acc[h], 0, 0, 0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t m = m_tile + 16 * h + li;
                if (m >= a.n_rows || n >= a.N) continue;
                f32x4 y;
#pragma unroll
                for (int c = 0; c < 4; ++c) y[c] = a.c_w * acc[h][c];
                if (a.bias) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] += a.bias[n + c];
                }
                if (a.c_id != 0.f) {
                    const f32x4 z = *reinterpret_cast<const f32x4*>(Zs + (16 * h + li) * LDZ + n);
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] = fmaf(a.c_id, z[c], y[c]);
                }
                if (a.relu) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] = fmaxf(y[c], 0.f);
                }
                *reinterpret_cast<f32x4_any*>(a.Y + m * a.ldy + n) = y;
                if constexpr (BWD) {
                    if (a.total) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) sum[b][h][c] += a.c_total * y[c];
                        *reinterpret_cast<f32x4*>(a.total + m * a.ldt + n) = sum[b][h];
                    }
                }
                if (!BWD && a.push_idx) *reinterpret_cast<f32x4_any*>(a.PH + (int64_t)slot[h] * a.ldp + n) = y;      // Push in the epilogue
            }
        }
        __syncthreads();                 // the next tile's aggregation overwrites Zs
    }
}

template <int G, int P, int NB, bool BWD>
gas_status launch_layer(const FusedArgs& a, hipStream_t s) {
    // Workgroups that a CU holds at once, as the compiled kernel's registers and LDS allow: one more would wait for a slot and then
    // walk its tiles alone (100,000 rows of 64, 14 entries each: 42 us, with a grid for four 54 us), one less leaves the others
    // more tiles (60,000 rows of 15, 32 -> 32: 23.2 us by three, 19.5 by the four that fit).
    static const int64_t per_cu = [] {
        int n = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, spmm_linear_f32_kernel<G, P, NB, BWD>, kThreads, 0);
        return e == hipSuccess && n > 0 ? n : 2;
    }();
    const int64_t per_xcd = (a.n_tiles + 7) / 8;                                   // a multiple of eight workgroups
    const unsigned blocks = (unsigned)(8 * (per_xcd < 32 * per_cu ? per_xcd : 32 * per_cu));
    hipLaunchKernelGGL((spmm_linear_f32_kernel<G, P, NB, BWD>), dim3(blocks), dim3(kThreads), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

template <bool BWD>
gas_status run_layer(const FusedArgs& a, hipStream_t s) {
    // lanes per row and 16-byte pieces per lane by the input width, blocks of 16 output columns per wavefront by the output's
    if (a.K <= 32) return a.N <= 64 ? launch_layer<8, 1, 1, BWD>(a, s) : launch_layer<8, 1, 2, BWD>(a, s);
    if (a.K <= 64) return a.N <= 64 ? launch_layer<8, 2, 1, BWD>(a, s) : launch_layer<8, 2, 2, BWD>(a, s);
    return a.N <= 64 ? launch_layer<16, 2, 1, BWD>(a, s) : launch_layer<16, 2, 2, BWD>(a, s);
}

// the arguments of gas_spmm_linear and of gas_spmm_t_relu_linear (and of each of their layers), checked
gas_status check_layer(const char* who, const int32_t* rowptr, const int32_t* src, int64_t n_rows, const void* X, int64_t ldx, const void* hist,
                       int64_t n_hist_rows, int64_t ld_hist, gas_dtype dt, int32_t F_in, const void* R, int64_t ldr, const void* W,
                       int32_t F_out, float c_identity, const void* Y, int64_t ldy, const void* Z_out, int64_t ldz_out,
                       const int32_t* push_idx, const void* push_hist, int64_t n_push_rows, int64_t ld_push) {
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    if (dt != GAS_F32) return fail(GAS_ERR_DTYPE, "%s: fp32 only (use gas_spmm_hist + gas_linear_push)", who);
    GAS_REQUIRE(n_rows >= 0 && n_rows < 0x7FFFFFFFLL, "%s: n_rows=%lld", who, (long long)n_rows);
    GAS_REQUIRE(F_in > 0 && F_out > 0 && F_in <= kMaxWidth && F_out <= kMaxWidth && F_in % 4 == 0 && F_out % 4 == 0,
                "%s: widths %d -> %d: multiples of 4 up to %d only (use gas_spmm_hist + gas_linear_push)", who,
                F_in, F_out, kMaxWidth);
    if (n_rows == 0) return GAS_OK;
    GAS_REQUIRE(rowptr && src && X && W && Y, "%s: null pointer", who);
    GAS_REQUIRE(ldx >= F_in && ldy >= F_out && (!hist || ld_hist >= F_in) && (!R || ldr >= F_in),
                "%s: row stride smaller than the width", who);
    GAS_REQUIRE(n_hist_rows >= 0 && n_push_rows >= 0, "%s: negative table size", who);
    GAS_REQUIRE(c_identity == 0.f || F_in == F_out, "%s: the identity term needs F_in == F_out", who);
    GAS_REQUIRE((push_idx == nullptr) == (push_hist == nullptr), "%s: push_idx and push_hist go together", who);
    GAS_REQUIRE(!push_hist || ld_push >= F_out, "%s: row stride of the push table smaller than F_out", who);
    GAS_REQUIRE(!Z_out || ldz_out >= F_in, "%s: row stride of Z_out smaller than F_in", who);
    const bool al = aligned16(X) && ldx % 4 == 0 && aligned16(W) && (!hist || (aligned16(hist) && ld_hist % 4 == 0)) &&
                    (!R || (aligned16(R) && ldr % 4 == 0)) && (!Z_out || (aligned16(Z_out) && ldz_out % 4 == 0));
    GAS_REQUIRE(al, "%s: rows must be 16-byte aligned (use gas_spmm_hist + gas_linear_push)", who);
    return GAS_OK;
}
gas_status check_layer_bwd(const char* who, const int32_t* colptr, const int32_t* row, int64_t n_cols, const void* G, int64_t ldg,
                           gas_dtype dt, int32_t F, const void* Y, int64_t ldy, const void* GX, int64_t ldgx, const void* W,
                           int32_t F_below, float c_identity, const void* total, int64_t ldtotal, const void* GZ, int64_t ldgz) {
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    if (dt != GAS_F32) return fail(GAS_ERR_DTYPE, "%s: fp32 only (use gas_spmm_t_relu + gas_linear_bwd_input)", who);
    GAS_REQUIRE(n_cols >= 0 && n_cols < 0x7FFFFFFFLL, "%s: n_cols=%lld", who, (long long)n_cols);
    GAS_REQUIRE(F > 0 && F_below > 0 && F <= kMaxWidth && F_below <= kMaxWidth && F % 4 == 0 && F_below % 4 == 0,
                "%s: widths %d, %d: multiples of 4 up to %d only", who, F, F_below, kMaxWidth);
    if (n_cols == 0) return GAS_OK;
    GAS_REQUIRE(colptr && row && G && Y && GX && W && GZ, "%s: null pointer", who);
    GAS_REQUIRE(ldg >= F && ldy >= F && ldgx >= F && ldgz >= F_below && (!total || ldtotal >= F_below),
                "%s: row stride smaller than the width", who);
    GAS_REQUIRE(c_identity == 0.f || F == F_below, "%s: the identity term needs equal widths", who);
    GAS_REQUIRE(G != GX && G != GZ && G != total && GX != GZ && GX != total && Y != GX && Y != GZ && Y != total &&
                    (!total || total != GZ),
                "%s: an output aliases another matrix", who);
    GAS_REQUIRE(aligned16(G) && ldg % 4 == 0 && aligned16(Y) && ldy % 4 == 0 && aligned16(GX) && ldgx % 4 == 0 && aligned16(W) &&
                    (!total || (aligned16(total) && ldtotal % 4 == 0)),
                "%s: rows must be 16-byte aligned (use gas_spmm_t_relu + gas_linear_bwd_input)", who);
    return GAS_OK;
}

}  // namespace
}  // namespace gas

using namespace gas;

extern "C" {

gas_status gas_spmm_linear(const int32_t* rowptr, const int32_t* src, const float* val, int64_t n_rows, const void* X,
                           int64_t ldx, const void* hist, int64_t n_hist_rows, int64_t ld_hist, gas_dtype dt,
                           int32_t F_in, float diag, float s_agg, const void* R, int64_t ldr, float s_res,
                           const void* W, int32_t F_out, const void* bias, float c_identity, float c_weight, int relu,
                           void* Y, int64_t ldy, void* Z_out, int64_t ldz_out, const int32_t* push_idx,
                           void* push_hist, int64_t n_push_rows, int64_t ld_push, void* stream) {
    const gas_status st = check_layer("gas_spmm_linear", rowptr, src, n_rows, X, ldx, hist, n_hist_rows, ld_hist, dt, F_in, R, ldr, W, F_out, c_identity,
                                      Y, ldy, Z_out, ldz_out, push_idx, push_hist, n_push_rows, ld_push);
    if (st != GAS_OK || n_rows == 0) return st;
    FusedArgs a{};
    a.rowptr = rowptr; a.src = src; a.val = val;
    a.n_rows = n_rows; a.n_tiles = (n_rows + kRows - 1) / kRows;
    a.X = reinterpret_cast<const float*>(X); a.ldx = ldx;
    a.H = reinterpret_cast<const float*>(hist); a.ldh = ld_hist;
    a.R = reinterpret_cast<const float*>(R); a.ldr = ldr;
    a.W = reinterpret_cast<const float*>(W); a.bias = reinterpret_cast<const float*>(bias);
    a.Y = reinterpret_cast<float*>(Y); a.ldy = ldy;
    a.Zout = reinterpret_cast<float*>(Z_out); a.ldzo = ldz_out;
    a.push_idx = push_idx; a.PH = reinterpret_cast<float*>(push_hist); a.ldp = ld_push;
    a.K = F_in; a.N = F_out;
    a.diag = diag; a.s_agg = s_agg; a.s_res = s_res; a.c_id = c_identity; a.c_w = c_weight; a.relu = relu;
    return run_layer<false>(a, (hipStream_t)stream);
}

gas_status gas_spmm_t_relu_linear(const int32_t* colptr, const int32_t* row, const float* val, int64_t n_cols,
                                  const void* G, int64_t ldg, gas_dtype dt, int32_t F, float s_agg, const void* Y,
                                  int64_t ldy, void* GX, int64_t ldgx, const void* W, int32_t F_below, float c_identity,
                                  float c_weight, float c_total, void* total, int64_t ldtotal, void* GZ, int64_t ldgz,
                                  void* stream) {
    const gas_status st = check_layer_bwd("gas_spmm_t_relu_linear", colptr, row, n_cols, G, ldg, dt, F, Y, ldy, GX, ldgx, W, F_below,
                                          c_identity, total, ldtotal, GZ, ldgz);
    if (st != GAS_OK || n_cols == 0) return st;
    FusedArgs a{};
    a.rowptr = colptr; a.src = row; a.val = val;
    a.n_rows = n_cols; a.n_tiles = (n_cols + kRows - 1) / kRows;
    a.X = reinterpret_cast<const float*>(G); a.ldx = ldg;
    a.mask = reinterpret_cast<const float*>(Y); a.ldm = ldy;
    a.Zout = reinterpret_cast<float*>(GX); a.ldzo = ldgx;
    a.W = reinterpret_cast<const float*>(W);
    a.Y = reinterpret_cast<float*>(GZ); a.ldy = ldgz;
    a.total = reinterpret_cast<float*>(total); a.ldt = ldtotal; a.c_total = c_total;
    a.K = F; a.N = F_below;
    a.s_agg = s_agg; a.c_id = c_identity; a.c_w = c_weight;
    return run_layer<true>(a, (hipStream_t)stream);
}

gas_status gas_spmm_linear_layers(int32_t count, const int32_t* rowptr, const int32_t* src_first, const int32_t* src,
                                  const float* val, int64_t n_rows, const void* X, int64_t ldx, const void* const* hist,
                                  int64_t n_hist_rows, const int64_t* ld_hist, gas_dtype dt, int32_t F, float s_agg, const void* R,
                                  int64_t ldr, float s_res, const void* const* W, const float* c_identity,
                                  const float* c_weight, int relu_last, void* const* Y, int64_t ldy, void* const* Z_out,
                                  int64_t ldz_out, const int32_t* push_idx, void* const* push_hist, int64_t n_push_rows,
                                  const int64_t* ld_push, void* stream) {
    const char* who = "gas_spmm_linear_layers";
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    GAS_REQUIRE(count >= 0 && n_rows >= 0, "%s: count=%d, n_rows=%lld", who, count, (long long)n_rows);
    if (count == 0 || n_rows == 0) return GAS_OK;
    GAS_REQUIRE(hist && ld_hist && W && c_identity && c_weight && Y && (!push_hist || ld_push), "%s: null pointer", who);
    GAS_REQUIRE((push_idx == nullptr) == (push_hist == nullptr), "%s: push_idx and push_hist go together", who);
    for (int pass = 0; pass < 2; ++pass)                       // every argument is checked before anything is launched
        for (int l = 0; l < count; ++l) {
            const int32_t* ind = l ? src : src_first;
            const void* x = l ? Y[l - 1] : X;
            const int64_t ld = l ? ldy : ldx;
            void* z = Z_out ? Z_out[l] : nullptr;
            void* table = push_hist ? push_hist[l] : nullptr;
            const int32_t* ids = table ? push_idx : nullptr;
            const int64_t ldp = table ? ld_push[l] : 0;
            gas_status st;
            if (pass == 0) {
                st = check_layer(who, rowptr, ind, n_rows, x, ld, hist[l], n_hist_rows, ld_hist[l], dt, F, R, ldr, W[l], F, c_identity[l],
                                 Y[l], ldy, z, ldz_out, ids, table, n_push_rows, ldp);
                if (st == GAS_OK && Y[l] == x) st = fail(GAS_ERR_ARG, "%s: layer %d writes the rows that it reads", who, l);
            } else {
                st = gas_spmm_linear(rowptr, ind, val, n_rows, x, ld, hist[l], n_hist_rows, ld_hist[l], dt, F, 0.f, s_agg, R, ldr, s_res,
                                     W[l], F, nullptr, c_identity[l], c_weight[l], l + 1 < count || relu_last, Y[l], ldy, z, ldz_out, ids,
                                     table, n_push_rows, ldp, stream);
            }
            if (st != GAS_OK) return st;
        }
    return GAS_OK;
}

gas_status gas_spmm_t_relu_linear_layers(int32_t count, const int32_t* colptr, const int32_t* row, const float* val,
                                         int64_t n_cols, const void* G, int64_t ldg, gas_dtype dt, int32_t F, float s_agg,
                                         const void* const* Y, int64_t ldy, void* const* GX, int64_t ldgx, const void* const* W,
                                         const float* c_identity, const float* c_weight, float c_total, void* total,
                                         int64_t ldtotal, void* const* GZ, int64_t ldgz, void* stream) {
    const char* who = "gas_spmm_t_relu_linear_layers";
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    GAS_REQUIRE(count >= 0 && n_cols >= 0, "%s: count=%d, n_cols=%lld", who, count, (long long)n_cols);
    if (count == 0 || n_cols == 0) return GAS_OK;
    GAS_REQUIRE(Y && GX && W && c_identity && c_weight && GZ, "%s: null pointer", who);
    for (int pass = 0; pass < 2; ++pass)
        for (int l = 0; l < count; ++l) {
            const void* g = l ? GZ[l - 1] : G;
            const int64_t ld = l ? ldgz : ldg;
            const gas_status st =
                pass == 0 ? check_layer_bwd(who, colptr, row, n_cols, g, ld, dt, F, Y[l], ldy, GX[l], ldgx, W[l], F, c_identity[l],
                                            total, ldtotal, GZ[l], ldgz)
                          : gas_spmm_t_relu_linear(colptr, row, val, n_cols, g, ld, dt, F, s_agg, Y[l], ldy, GX[l], ldgx, W[l], F,
                                                   c_identity[l], c_weight[l], c_total, total, ldtotal, GZ[l], ldgz, stream);
            if (st != GAS_OK) return st;
        }
    return GAS_OK;
}

}  // extern "C"
