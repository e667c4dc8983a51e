// Neighbourhood aggregation over the batch subgraph (gas_spmm) and its adjoint
// (gas_spmm_t): row-parallel compressed-sparse-row products without atomics.
//
// What is computed is the sum of the paper's Eq. (1)/(2) for the in-batch
// rows, with the edge weights of the GCN / GCNII / GIN operators folded into
// `val`, `diag`, `s_agg` and the residual term.
//
// Mapping to the machine.  A feature row is cut into 16-byte units (a width that
// is no whole number of them: the last unit starts E elements before the row's
// end and shares elements with the one before it, both compute the same sums;
// rows need no alignment beyond their element's); a "team" of G = 2^k lanes (G >= units per row, at most 64) owns one row, so one wavefront
// works on 64/G neighbours at a time and a wavefront-wide load instruction
// always fetches whole contiguous rows.  The wavefront stages 64 column
// indices and weights at a time in registers (one coalesced load) and
// broadcasts them with lane permutes; U independent row loads are in flight
// per lane.  Rows with at most `threshold` entries take one wavefront each.
// Heavier rows (power-law hubs) are cut into chunks of at most `chunk` entries,
// one wavefront per chunk (spmm_chunk_kernel), whose fp32 partial sums go to a
// workspace and are added in a fixed order by spmm_heavy_reduce_kernel; the
// light rows follow in spmm_rows_kernel.  The chunks are cut and ordered by
// windows of the source rows (plan_host.h states the rules; half an L2 unless
// the plan's maker asks for others), so that wavefronts running together gather
// from the same rows.
// Light rows go by slices of a row instead (spmm_slices_kernel) where rows_form() says so.
// The summation order is a
// function of the plan alone, so results are bit-identical from run to run.
#include "common.h"
#include "plan.h"
#include "wave.h"

#include <algorithm>
#include <string.h>
#include <type_traits>
#include <vector>

namespace gas {
namespace {

struct SpmmArgs {
    const int32_t* ptr;
    const int32_t* ind;
    const float* val;
    const char* X;
    int64_t x_stride;     // bytes
    const char* H;        // history table for entries with a negative index (row -1-index), or null
    int64_t h_stride;
    const char* R;
    int64_t r_stride;
    const char* Y;        // optional (MASK kernels): activations of X's type; outputs where Y <= 0 are zero
    int64_t y_stride;
    char* Z;
    int64_t z_stride;
    const int32_t* own;   // the diagonal term's rows: row own[v] of H, or (null) row v of X
    float diag, s_agg, s_res;
    int64_t n_rows, n_diag;
    int units;            // 16-byte units per row of X, the last one may overlap its neighbour
    int F;                // at least one unit's elements
    int threshold;
    const int32_t* chunk;       // plan lists
    int64_t n_chunks;
    const int32_t* heavy;
    int64_t n_heavy;
    float* partial;
    const int32_t* group;       // row groups of the light rows (wave-per-row path)
    int64_t n_groups;
    int xcd_ranges;       // grouped light rows: one contiguous range of groups per XCD, [xcd_start[x], xcd_start[x+1])
    int64_t xcd_start[9];
    int pieces, in_turn;  // rows_form()
};

__device__ __forceinline__ const char* own_row(const SpmmArgs& a, int64_t row) {
    return a.own ? a.H + (int64_t)a.own[row] * a.h_stride : a.X + row * a.x_stride;
}

template <bool XBF>
struct Unit {
    static constexpr int E = XBF ? 8 : 4;   // elements per 16-byte unit
    static __device__ __forceinline__ void fma(float (&acc)[E], float w, const u32x4& v) {
        if constexpr (XBF) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[2 * i] = fmaf(w, bf16_lo(v[i]), acc[2 * i]);
                acc[2 * i + 1] = fmaf(w, bf16_hi(v[i]), acc[2 * i + 1]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fmaf(w, __uint_as_float(v[i]), acc[i]);
        }
    }
};

// 16-byte accesses of rows that are aligned to their elements only (global memory takes them at any byte address)
typedef u32x4 u32x4_at2 __attribute__((aligned(2)));
typedef u32x4 u32x4_at4 __attribute__((aligned(4)));
typedef f32x4 f32x4_at4 __attribute__((aligned(4)));
template <bool BF>
__device__ __forceinline__ u32x4 load_unit(const char* p) {
    if constexpr (BF) return *reinterpret_cast<const u32x4_at2*>(p);
    else return *reinterpret_cast<const u32x4_at4*>(p);
}
// first element of a unit
template <bool XBF>
__device__ __forceinline__ int unit_start(const SpmmArgs& a, int unit) {
    return min(unit * Unit<XBF>::E, a.F - Unit<XBF>::E);
}

template <int G>
__device__ __forceinline__ int bcast_i(int v, int k) {
    if constexpr (G == 64) return __builtin_amdgcn_readlane(v, k);
    else return __shfl(v, k, 64);
}
template <int G>
__device__ __forceinline__ float bcast_f(float v, int k) {
    if constexpr (G == 64) return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
    else return __shfl(v, k, 64);
}

// Sum of val[k] * X[ind[k], :] over k in [begin, end) for this lane's units.
// Afterwards every team of the wavefront holds the full sum.
template <int G, int UPT, int U, bool XBF>
__device__ __forceinline__ void accumulate(const SpmmArgs& a, int begin, int end,
                                           float (&acc)[UPT][Unit<XBF>::E]) {
    constexpr int S = kWave / G;
    constexpr int E = Unit<XBF>::E;
    const int lane = threadIdx.x & 63;
    const int team = lane / G, tl = lane % G;
#pragma unroll
    for (int p = 0; p < UPT; ++p)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[p][e] = 0.f;
    const int nunits = a.units;
    int start[UPT];                            // byte offset of the lane's units in a row
#pragma unroll
    for (int p = 0; p < UPT; ++p) start[p] = unit_start<XBF>(a, tl + p * G) * (XBF ? 2 : 4);
    for (int t = begin; t < end; t += kWave) {
        const int cnt = min(kWave, end - t);
        int my_c = 0;
        float my_w = 0.f;
        if (lane < cnt) {
            my_c = __builtin_nontemporal_load(a.ind + t + lane);     // streamed once: keep it out of the way of X in L2
            my_w = a.val ? __builtin_nontemporal_load(a.val + t + lane) : 1.f;
        }
        for (int j = 0; j < cnt; j += S * U) {
            u32x4 v[U][UPT];
            float w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = j + u * S + team;
                const bool ok = k < cnt;
                const int c = bcast_i<G>(my_c, k & 63);
                const float ww = bcast_f<G>(my_w, k & 63);
                w[u] = ok ? ww : 0.f;
#pragma unroll
                for (int p = 0; p < UPT; ++p) {
                    v[u][p] = u32x4{0u, 0u, 0u, 0u};
                    // index >= 0: row of the mini-batch tensor; index < 0: row -1-index of the history table
                    const bool in_batch = c >= 0;
                    const char* src = (in_batch ? a.X : a.H) +
                                      (int64_t)(in_batch ? c : -1 - c) * (in_batch ? a.x_stride : a.h_stride);
                    if (ok && tl + p * G < nunits) v[u][p] = load_unit<XBF>(src + start[p]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int p = 0; p < UPT; ++p) Unit<XBF>::fma(acc[p], w[u], v[u][p]);
        }
    }
    if constexpr (S > 1) {
#pragma unroll
        for (int off = G; off < kWave; off <<= 1)
#pragma unroll
            for (int p = 0; p < UPT; ++p)
#pragma unroll
                for (int e = 0; e < E; ++e) acc[p][e] += __shfl_xor(acc[p][e], off, 64);
    }
}

// Z[row, unit] = s_agg * acc + diag * X[row, unit] + s_res * R[row, unit], zero where the activation Y is not positive
template <bool XBF, bool ZBF>
__device__ __forceinline__ void epilogue(const SpmmArgs& a, int64_t row, int unit, float (&acc)[Unit<XBF>::E]) {
    constexpr int E = Unit<XBF>::E, EB = XBF ? 2 : 4;
    const int start = unit_start<XBF>(a, unit);
    float z[E];
#pragma unroll
    for (int e = 0; e < E; ++e) z[e] = a.s_agg * acc[e];
    if (a.diag != 0.f && row < a.n_diag) {
        float t[E];
#pragma unroll
        for (int e = 0; e < E; ++e) t[e] = 0.f;
        Unit<XBF>::fma(t, a.diag, load_unit<XBF>(own_row(a, row) + start * EB));
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] += t[e];
    }
    if (a.R) {
        float t[E];
#pragma unroll
        for (int e = 0; e < E; ++e) t[e] = 0.f;
        Unit<XBF>::fma(t, a.s_res, load_unit<XBF>(a.R + row * a.r_stride + start * EB));
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] += t[e];
    }
    if (a.Y) {
        const u32x4 y = load_unit<XBF>(a.Y + row * a.y_stride + start * EB);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float v = XBF ? (e & 1 ? bf16_hi(y[e / 2]) : bf16_lo(y[e / 2])) : __uint_as_float(y[e % 4]);
            z[e] = v > 0.f ? z[e] : 0.f;
        }
    }
    char* zp = a.Z + row * a.z_stride;
    if constexpr (ZBF) {
        static_assert(!ZBF || XBF, "bf16 output needs bf16 input");
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = pack_bf16(z[2 * i], z[2 * i + 1]);
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4_at2*>(zp + start * 2));
    } else {
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
            f32x4 o = {z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]};
            __builtin_nontemporal_store(o, reinterpret_cast<f32x4_at4*>(zp + (start + 4 * q) * 4));
        }
    }
}

// ---- wave-per-row path for rows of exactly 64 vectors of VB bytes (1 KiB or 512 B; chunks of heavy rows 256 B too)
// Short rows are the common case on power-law graphs, and one wavefront per row
// pays three dependent memory latencies (row pointers, indices, feature rows)
// for a handful of gathers.  Here consecutive light rows are bundled at plan
// time into groups of at most 64 entries and 63 rows: the wavefront loads the
// group's row pointers with one load and all its indices and weights with
// another, then streams the gathers of the whole group, 8 in flight per lane,
// flushing a row (epilogue + store) whenever the entry cursor crosses a row
// boundary.  Every lane works on every row (lane l owns bytes [l*VB, (l+1)*VB) of
// the row), all control flow is wavefront-uniform, and the order of summation
// within a row is the stored order.
template <int VB> struct VecOf;
template <> struct VecOf<16> { typedef u32x4 type; };
template <> struct VecOf<8> { typedef u32x2 type; };
typedef uint32_t u32x1 __attribute__((ext_vector_type(1)));
template <> struct VecOf<4> { typedef u32x1 type; };

template <int VB, bool XBF>
struct LaneAcc {
    static constexpr int NW = VB / 4;                 // dwords per lane and row
    static constexpr int E = XBF ? 2 * NW : NW;       // elements per lane and row
    typedef typename VecOf<VB>::type V;
    float v[E];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = 0.f;
    }
    __device__ __forceinline__ void fma(float w, const V& x) {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            if constexpr (XBF) {
                v[2 * i] = fmaf(w, bf16_lo(x[i]), v[2 * i]);
                v[2 * i + 1] = fmaf(w, bf16_hi(x[i]), v[2 * i + 1]);
            } else {
                v[i] = fmaf(w, __uint_as_float(x[i]), v[i]);
            }
        }
    }
};

template <int VB, bool XBF, bool ZBF, bool MASK>
__device__ __forceinline__ void flush_row(const SpmmArgs& a, int64_t row, int lane, LaneAcc<VB, XBF>& acc,
                                          const typename VecOf<VB>::type& own, const typename VecOf<VB>::type& act) {
    // `own` = this lane's piece of X[row, :], `act` of Y[row, :], loaded ahead of time by the caller (only read when
    // diag != 0; MASK)
    typedef typename VecOf<VB>::type V;
    constexpr int E = LaneAcc<VB, XBF>::E, NW = VB / 4;
    float z[E];
#pragma unroll
    for (int e = 0; e < E; ++e) z[e] = a.s_agg * acc.v[e];
    if (a.diag != 0.f && row < a.n_diag) {
        LaneAcc<VB, XBF> t;
        t.clear();
        t.fma(a.diag, own);
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] += t.v[e];
    }
    if (a.R) {
        LaneAcc<VB, XBF> t;
        t.clear();
        t.fma(a.s_res, *reinterpret_cast<const V*>(a.R + row * a.r_stride + (int64_t)lane * VB));
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] += t.v[e];
    }
    if constexpr (MASK) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float v = XBF ? (e & 1 ? bf16_hi(act[e / 2]) : bf16_lo(act[e / 2])) : __uint_as_float(act[e % NW]);
            z[e] = v > 0.f ? z[e] : 0.f;
        }
    }
    char* zp = a.Z + row * a.z_stride;
    if constexpr (ZBF) {
        V o;
#pragma unroll
        for (int i = 0; i < NW; ++i) o[i] = pack_bf16(z[2 * i], z[2 * i + 1]);
        __builtin_nontemporal_store(o, reinterpret_cast<V*>(zp + (int64_t)lane * VB));
    } else if constexpr (XBF) {      // bf16 in, fp32 out: twice the bytes
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            V o;
#pragma unroll
            for (int i = 0; i < NW; ++i) o[i] = __float_as_uint(z[q * NW + i]);
            __builtin_nontemporal_store(o, reinterpret_cast<V*>(zp + (int64_t)lane * 2 * VB + q * VB));
        }
    } else {
        V o;
#pragma unroll
        for (int i = 0; i < NW; ++i) o[i] = __float_as_uint(z[i]);
        __builtin_nontemporal_store(o, reinterpret_cast<V*>(zp + (int64_t)lane * VB));
    }
    acc.clear();
}

template <int VB, bool XBF, bool ZBF, bool MASK>
__device__ __forceinline__ void light_group(const SpmmArgs& a, int64_t g) {
    typedef typename VecOf<VB>::type V;
    constexpr int U = 8;
    const int lane = threadIdx.x & 63;
    const int r0 = a.group[2 * g], nrows = a.group[2 * g + 1] - r0;   // 1 <= nrows <= 63
    const int my_ptr = lane <= nrows ? a.ptr[r0 + lane] : 0;
    const int e0 = __builtin_amdgcn_readlane(my_ptr, 0);
    const int e1 = __builtin_amdgcn_readlane(my_ptr, nrows);
    const int my_own = a.own && lane < nrows ? a.own[r0 + lane] : 0;
    const char* xb = a.X + (int64_t)lane * VB;
    const char* hb = a.H + (int64_t)lane * VB;
    LaneAcc<VB, XBF> acc;
    acc.clear();
    int r = 0;                                                     // row being accumulated (relative to r0)
    int row_end = __builtin_amdgcn_readlane(my_ptr, 1);            // first entry after row r
    // The diagonal term needs X[row, :] at every flush.  Its address depends on the row number alone, so the
    // pieces of the next four rows are kept in flight in a small ring instead of being loaded (and waited for)
    // at the flush itself: rows of 0-1 entries would otherwise pay a full memory latency each.
    constexpr int D = 4;
    V own[D];
    const bool use_diag = a.diag != 0.f;
    auto load_own = [&](int rr) -> V {
        V v{};
        const int64_t row = (int64_t)r0 + rr;
        if (use_diag && rr < nrows && row < a.n_diag)
            v = *reinterpret_cast<const V*>(a.own ? hb + (int64_t)__builtin_amdgcn_readlane(my_own, rr) * a.h_stride : xb + row * a.x_stride);
        return v;
    };
#pragma unroll
    for (int d = 0; d < D; ++d) own[d] = load_own(d);
    // the same for the rows of the mask
    V act[MASK ? D : 1];
    auto load_act = [&](int rr) -> V {
        V v{};
        if (rr < nrows) v = __builtin_nontemporal_load(reinterpret_cast<const V*>(a.Y + ((int64_t)r0 + rr) * a.y_stride + (int64_t)lane * VB));
        return v;
    };
    if constexpr (MASK) {
#pragma unroll
        for (int d = 0; d < D; ++d) act[d] = load_act(d);
    }
    auto flush = [&]() {
        flush_row<VB, XBF, ZBF, MASK>(a, r0 + r, lane, acc, own[0], act[0]);
#pragma unroll
        for (int d = 0; d + 1 < D; ++d) own[d] = own[d + 1];
        own[D - 1] = load_own(r + D);
        if constexpr (MASK) {
#pragma unroll
            for (int d = 0; d + 1 < D; ++d) act[d] = act[d + 1];
            act[D - 1] = load_act(r + D);
        }
        ++r;
    };
    // a single row longer than 64 entries makes its own group: walk it 64 entries at a time
    for (int t = e0; t < e1; t += kWave) {
        const int cnt = min(kWave, e1 - t);
        int my_c = 0;
        float my_w = 0.f;
        if (lane < cnt) {
            my_c = __builtin_nontemporal_load(a.ind + t + lane);
            my_w = a.val ? __builtin_nontemporal_load(a.val + t + lane) : 1.f;
        }
        for (int j = 0; j < cnt; j += U) {
            V v[U];
            float w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = j + u;
                const int c = __builtin_amdgcn_readlane(my_c, k & 63);
                w[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_w), k & 63));
                const bool in_batch = c >= 0;
                const char* src = (in_batch ? xb : hb) +
                                  (int64_t)(in_batch ? c : -1 - c) * (in_batch ? a.x_stride : a.h_stride);
                if (k < cnt) v[u] = *reinterpret_cast<const V*>(src);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = j + u;
                if (k < cnt) {
                    while (t + k >= row_end) {                     // crossed into the next row (or over empty rows)
                        flush();
                        row_end = __builtin_amdgcn_readlane(my_ptr, (r + 1) & 63);
                    }
                    acc.fma(w[u], v[u]);
                }
            }
        }
    }
    while (r < nrows) flush();                                     // last row and trailing empty rows
}

// One chunk of a heavy row on the wave-per-row layout (rows of 64 vectors of VB bytes): every lane owns VB bytes
// of the row, 8 gathers in flight per lane, the fp32 partial sum goes to the chunk's slot of the workspace.
template <int VB, bool XBF, int U>
__device__ __forceinline__ void chunk_wave_per_row(const SpmmArgs& a, int64_t c) {
    typedef typename VecOf<VB>::type V;
    constexpr int E = LaneAcc<VB, XBF>::E;
    const int lane = threadIdx.x & 63;
    const int begin = a.chunk[3 * c + 1], end = a.chunk[3 * c + 2];
    const char* xb = a.X + (int64_t)lane * VB;
    const char* hb = a.H + (int64_t)lane * VB;
    LaneAcc<VB, XBF> acc;
    acc.clear();
    for (int t = begin; t < end; t += kWave) {
        const int cnt = min(kWave, end - t);
        int my_c = 0;
        float my_w = 0.f;
        if (lane < cnt) {
            my_c = __builtin_nontemporal_load(a.ind + t + lane);
            my_w = a.val ? __builtin_nontemporal_load(a.val + t + lane) : 1.f;
        }
        for (int j = 0; j < cnt; j += U) {
            V v[U];
            float w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = j + u;
                const int ci = __builtin_amdgcn_readlane(my_c, k & 63);
                w[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_w), k & 63));
                const bool in_batch = ci >= 0;
                const char* src = (in_batch ? xb : hb) +
                                  (int64_t)(in_batch ? ci : -1 - ci) * (in_batch ? a.x_stride : a.h_stride);
                if (k < cnt) v[u] = *reinterpret_cast<const V*>(src);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (j + u < cnt) acc.fma(w[u], v[u]);
        }
    }
    float* dst = a.partial + (int64_t)a.chunk[3 * c] * a.F + (int64_t)lane * E;
    if constexpr (E == 8) {
        *reinterpret_cast<f32x4*>(dst) = f32x4{acc.v[0], acc.v[1], acc.v[2], acc.v[3]};
        *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc.v[4], acc.v[5], acc.v[6], acc.v[7]};
    } else if constexpr (E == 4) {
        *reinterpret_cast<f32x4*>(dst) = f32x4{acc.v[0], acc.v[1], acc.v[2], acc.v[3]};
    } else if constexpr (E == 2) {
        *reinterpret_cast<u32x2*>(dst) = u32x2{__float_as_uint(acc.v[0]), __float_as_uint(acc.v[1])};
    } else {
        *dst = acc.v[0];
    }
}

// Chunks of heavy rows: one wavefront per chunk, partial sums to the workspace.
// Workgroups take the window-ordered list four chunks at a time.  At most
// four wavefronts per SIMD: fewer chunks in flight keep the gathers of the
// running chunks inside a narrower range of rows (measured: 2-4 % faster than
// 5 or 8, 3 and fewer are slower).
template <int G, int UPT, int U, bool XBF, int VB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void spmm_chunk_kernel(SpmmArgs a) {
    constexpr int E = Unit<XBF>::E;
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= a.n_chunks) return;
    if constexpr (VB > 0) {                 // rows of 64 vectors
        chunk_wave_per_row<VB, XBF, U>(a, c);
        return;
    }
    float acc[UPT][E];
    accumulate<G, UPT, U, XBF>(a, a.chunk[3 * c + 1], a.chunk[3 * c + 2], acc);
    if (lane < G) {
#pragma unroll
        for (int p = 0; p < UPT; ++p) {
            const int unit = lane + p * G;
            if (unit < a.units) {
                float* dst = a.partial + (int64_t)a.chunk[3 * c] * a.F + unit_start<XBF>(a, unit);
#pragma unroll
                for (int q = 0; q < E / 4; ++q)
                    *reinterpret_cast<f32x4_at4*>(dst + 4 * q) =
                        f32x4{acc[p][4 * q], acc[p][4 * q + 1], acc[p][4 * q + 2], acc[p][4 * q + 3]};
            }
        }
    }
}

// ---- rows by slices
// A team of 16 lanes owns one row's slice of up to 16 P pieces of 16 bytes (P pieces a lane); it reads 32 indices with two
// loads, the lane that read an index forms the row's address and the team takes it by data-parallel moves.  Four rows of a
// wavefront walk their chain of dependent loads (row pointers, indices, rows) together, where the kernels of a wavefront a row
// walk one.  A row's entries are folded in the stored order (S: entry k into sum k % S): above 32 units, and for 32 whole
// ones, the sums are the wave-per-row kernel's, bit for bit; below they have as many parts (launch_slices).
// Bounded by that chain and, with inputs that are not in the caches, by the misses.  us, a wavefront a row -> slices, inputs
// that rotate through more than the Infinity Cache holds, 50,000 clustered rows of 11 entries: 47 floats 24 -> 16, 64 28 -> 16,
// 136 50 -> 33, 184 53 -> 39, 248 61 -> 45, 1,433 429 -> 370, 128 bf16 30 -> 15, 136 36 -> 26; 150,000 power-law rows of 69, 64
// floats 421 -> 385; 64,000 clustered rows of 23 entries, 256 floats 184 -> 108.
// Contiguous (in_turn 0): the slices' rows, slice after slice, are cut into eight ranges, one for each XCD, so that a cluster is
// gathered into one L2, of which an XCD then holds a slice of its rows.  In turn: a slice's rows are dealt to the XCDs one after the
// other, for lengths that differ along the batch (a power law's first rows are its longest).
// rows_form() has the line between the forms.  Not kept: slices of 128 bytes, one for each XCD (their rows' lines lie in an
// eighth of an L2's channels: all gathers out of 2,048 rows of 1,024 bytes 2.1 ms whole, 2.7 by 256, 3.7 by 128 bytes), several
// rows a team with the next row's indices requested ahead (its last workgroups end late), rows put in order of length within
// a workgroup, loads past a row's end not switched off, steps without masks where every team has them in full (they cost
// registers: a wavefront less on a SIMD).
constexpr int kSliceRows = 16;      // rows of a workgroup (four wavefronts of four teams)

// H == 2 states its wavefronts because the compiler otherwise keeps all of a row's addresses in registers (fp32 242 instead of 83).
template <int P, bool EVEN, int S, int H, bool XBF, bool ZBF, bool MASK>
__global__ __launch_bounds__(256, H == 1 ? 1 : XBF ? 4 : 5) void spmm_slices_kernel(SpmmArgs a, int slices, int width) {
    constexpr int G = 16, E = Unit<XBF>::E, EB = XBF ? 2 : 4, U = P == 1 ? 8 : 4;
    typedef std::conditional_t<XBF, u32x4_at2, u32x4_at4> Piece;
    const int j = threadIdx.x % G, half = H == 2 ? j / 8 : 0;             // H == 2: a row's entries in turn to the team's halves
    const uint32_t tiles = (uint32_t)((a.n_rows + kSliceRows - 1) / kSliceRows);
    const uint32_t xcd = blockIdx.x & 7, i = blockIdx.x >> 3;             // workgroups go to the eight XCDs in turn
    uint32_t slice, tile;
    if (a.in_turn) {
        slice = blockIdx.x / tiles;
        tile = blockIdx.x - slice * tiles;
    } else {
        const uint32_t jobs = tiles * slices, per = (jobs + 7) / 8, job = xcd * per + i;
        if (i >= per || job >= jobs) return;
        slice = job / tiles;
        tile = job - slice * tiles;
    }
    const int64_t row = (int64_t)tile * kSliceRows + (threadIdx.x / G);
    if (row >= a.n_rows) return;
    const int b = a.ptr[row], e = a.ptr[row + 1];
    if (e - b > a.threshold) return;                                      // heavy row: done by the chunk kernel
    // the lane's units of the slice: j, j + G, ...; a lane past the slice's width loads nothing there if it is the last piece of
    // several, and else the row's last unit or one of the next slice, which it does not store: one condition less for every load
    uint32_t off[P];
    bool mine[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int w = (H == 2 ? j % 8 : j) + G * p, unit = slice * width + w;
        mine[p] = EVEN || (w < width && unit < a.units);
        off[p] = EVEN ? unit * 16 : unit_start<XBF>(a, min(unit, a.units - 1)) * EB;
    }
    static_assert(H == 1 || (P == 1 && !EVEN), "halves are for rows of up to eight units");
    // entries k + j and k + G + j (past the row's end its last one: a valid address, never folded)
    int s[2];
    float v[2];
    auto fetch = [&](int k) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int at = min(k + G * h + j, e - 1);
            s[h] = a.ind[at];
            v[h] = a.val ? a.val[at] : 1.f;
        }
    };
    if (b < e) fetch(b);
    auto piece = [&](const char* base, u32x4 (&t)[P]) {
#pragma unroll
        for (int p = 0; p < P; ++p) t[p] = *reinterpret_cast<const Piece*>(base + off[p]);
    };
    u32x4 own[P], res[P], act[P];
    const bool use_own = a.diag != 0.f && row < a.n_diag;
    if (use_own) piece(own_row(a, row), own);
    if (a.R) piece(a.R + row * a.r_stride, res);
    if constexpr (MASK) piece(a.Y + row * a.y_stride, act);
    float acc[S][P][E];
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int i = 0; i < E; ++i) acc[t][p][i] = 0.f;
    auto entry = [](int v, int u) {
        if constexpr (H == 2) return pair_lane(v, u);
        else return team_lane<G>(v, u);
    };
    for (int k0 = b; k0 < e; k0 += 2 * G) {
        const int cnt = e - k0, left = cnt - half;
        int lo[2], hi[2], wt[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool fresh = s[h] >= 0;
            const uint64_t p = (uint64_t)(fresh ? a.X : a.H) + (uint64_t)((int64_t)(fresh ? s[h] : -1 - s[h]) * (fresh ? a.x_stride : a.h_stride));
            lo[h] = (int)(uint32_t)p;
            hi[h] = (int)(uint32_t)(p >> 32);
            wt[h] = __float_as_int(v[h]);
        }
        fetch(min(k0 + 2 * G, e - 1));                                    // the next indices, before these are used
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < G; q += H * U) {
                if (G * h + q >= cnt) break;
                u32x4 x[U][P];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const u32x2 r = {(uint32_t)entry(lo[h], q + H * u), (uint32_t)entry(hi[h], q + H * u)};
                    if (G * h + q + H * u < left) {
#pragma unroll
                        for (int p = 0; p < P; ++p)
                            if (P == 1 || p + 1 < P || mine[p]) x[u][p] = load_global<Piece>(__builtin_bit_cast(uint64_t, r) + off[p]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float f = __int_as_float(entry(wt[h], q + H * u));
                    if (G * h + q + H * u < left) {
#pragma unroll
                        for (int p = 0; p < P; ++p) Unit<XBF>::fma(acc[u % S][p], f, x[u][p]);
                    }
                }
            }
    }
#pragma unroll
    for (int d = 1; d < S; d *= 2)
#pragma unroll
        for (int t = 0; t + d < S; t += 2 * d)
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int i = 0; i < E; ++i) acc[t][p][i] += acc[t + d][p][i];
    if constexpr (H == 2)
#pragma unroll
        for (int i = 0; i < E; ++i) acc[0][0][i] += other_half(acc[0][0][i]);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (!mine[p] || half) continue;
        float z[E];
#pragma unroll
        for (int i = 0; i < E; ++i) z[i] = a.s_agg * acc[0][p][i];
        if (use_own) Unit<XBF>::fma(z, a.diag, own[p]);
        if (a.R) Unit<XBF>::fma(z, a.s_res, res[p]);
        if constexpr (MASK) {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const float y = XBF ? (i & 1 ? bf16_hi(act[p][i / 2]) : bf16_lo(act[p][i / 2])) : __uint_as_float(act[p][i % 4]);
                z[i] = y > 0.f ? z[i] : 0.f;
            }
        }
        char* zp = a.Z + row * a.z_stride + (int64_t)(off[p] / EB) * (ZBF ? 2 : 4);
        if constexpr (ZBF) {
            u32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = pack_bf16(z[2 * i], z[2 * i + 1]);
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4_at2*>(zp));
        } else {
#pragma unroll
            for (int q = 0; q < E / 4; ++q) {
                f32x4 o = {z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]};
                __builtin_nontemporal_store(o, reinterpret_cast<f32x4_at4*>(zp + 16 * q));
            }
        }
    }
}

// Light rows, finished in one go (epilogue and store).  VB > 0: bundled into
// groups, one wavefront per row (rows of exactly 64 vectors of VB bytes);
// VB == 0: one wavefront per row, teams of G lanes per neighbour.
template <int G, int UPT, int U, bool XBF, bool ZBF, int VB, bool MASK>
__global__ __launch_bounds__(256) void spmm_rows_kernel(SpmmArgs a) {
    if constexpr (VB > 0) {
        // Workgroups go to the eight XCDs in turn and each XCD has its own L2: with xcd_ranges every XCD takes one
        // contiguous range of the groups (equal cost per range), so rows of one cluster of the partition gather
        // into one L2, not eight.  The plan turns this on where the pattern is clustered.
        int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), g_end = a.n_groups;
        if (a.xcd_ranges) {
            const int x = blockIdx.x & 7;
            g = a.xcd_start[x] + (int64_t)(blockIdx.x >> 3) * 4 + (threadIdx.x >> 6);
            g_end = a.xcd_start[x + 1];
        }
        if (g < g_end) light_group<VB, XBF, ZBF, MASK>(a, g);
    } else {
        constexpr int E = Unit<XBF>::E;
        const int lane = threadIdx.x & 63;
        const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
        if (row >= a.n_rows) return;
        const int begin = a.ptr[row], end = a.ptr[row + 1];
        if (end - begin > a.threshold) return;       // heavy row: done by the chunk kernel
        float acc[UPT][E];
        accumulate<G, UPT, U, XBF>(a, begin, end, acc);
        if (lane < G) {
#pragma unroll
            for (int p = 0; p < UPT; ++p)
                if (lane + p * G < a.units) epilogue<XBF, ZBF>(a, row, lane + p * G, acc[p]);
        }
    }
}

// One wavefront per heavy row: add the chunk partials in chunk order.  A hub has hundreds, each a load that the sum would wait
// for: eight are requested together (600,000 rows, 10,600 heavy ones with 634,000 chunks of 256 floats 200 -> 135 us).
template <bool XBF, bool ZBF>
__global__ __launch_bounds__(256) void spmm_heavy_reduce_kernel(SpmmArgs a) {
    const int64_t h = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (h >= a.n_heavy) return;
    constexpr int E = Unit<XBF>::E;
    const int64_t row = a.heavy[h];
    const int first = a.heavy[a.n_heavy + h], last = a.heavy[a.n_heavy + h + 1];
    for (int unit = threadIdx.x & 63; unit < a.units; unit += kWave) {
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.f;
        const float* src = a.partial + (int64_t)first * a.F + unit_start<XBF>(a, unit);
        int c = first;
        for (; c + 8 <= last; c += 8, src += 8 * (int64_t)a.F) {          // eight loads in flight, added in chunk order
            f32x4 v[8][E / 4];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int q = 0; q < E / 4; ++q) v[k][q] = *reinterpret_cast<const f32x4_at4*>(src + k * (int64_t)a.F + 4 * q);
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int q = 0; q < E / 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[4 * q + i] += v[k][q][i];
        }
        for (; c < last; ++c, src += a.F) {
#pragma unroll
            for (int q = 0; q < E / 4; ++q) {
                const f32x4 v = *reinterpret_cast<const f32x4_at4*>(src + 4 * q);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[4 * q + i] += v[i];
            }
        }
        epilogue<XBF, ZBF>(a, row, unit, acc);
    }
}

// Element-wise path for rows shorter than one 16-byte unit: one wavefront per row, one lane per feature.
template <bool XBF, bool ZBF>
__global__ __launch_bounds__(256) void spmm_generic_kernel(SpmmArgs a) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.n_rows) return;
    const int begin = a.ptr[row], end = a.ptr[row + 1];
    auto ld = [](const char* base, int64_t stride, int64_t r, int f) -> float {
        if constexpr (XBF) return __uint_as_float((uint32_t) * reinterpret_cast<const uint16_t*>(base + r * stride + 2 * f) << 16);
        else return *reinterpret_cast<const float*>(base + r * stride + 4 * (int64_t)f);
    };
    for (int f = threadIdx.x & 63; f < a.F; f += kWave) {
        float acc = 0.f;
        for (int k = begin; k < end; ++k) {
            const int c = a.ind[k];
            const float x = c >= 0 ? ld(a.X, a.x_stride, c, f) : ld(a.H, a.h_stride, -1 - c, f);
            acc = fmaf(a.val ? a.val[k] : 1.f, x, acc);
        }
        float z = a.s_agg * acc;
        if (a.diag != 0.f && row < a.n_diag) z += a.diag * ld(own_row(a, row), 0, 0, f);
        if (a.R) z += a.s_res * ld(a.R, a.r_stride, row, f);
        if (a.Y && !(ld(a.Y, a.y_stride, row, f) > 0.f)) z = 0.f;
        if constexpr (ZBF) *reinterpret_cast<uint16_t*>(a.Z + row * a.z_stride + 2 * f) = (uint16_t)f32_to_bf16(z);
        else *reinterpret_cast<float*>(a.Z + row * a.z_stride + 4 * (int64_t)f) = z;
    }
}

template <int G, int UPT, int U, bool XBF, int VB = 0>
gas_status launch_chunks(const SpmmArgs& a, hipStream_t s) {
    const int64_t blocks = (a.n_chunks + 3) / 4;
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_spmm: too many workgroups for one launch");
    hipLaunchKernelGGL((spmm_chunk_kernel<G, UPT, U, XBF, VB>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    return GAS_OK;
}

// `whole`: rows are whole numbers of 16-byte aligned units, as the wave-per-row kernels need
template <bool XBF>
gas_status dispatch_chunks(const SpmmArgs& a, bool whole, hipStream_t s) {
    const int u = a.units;
    if (whole && u == 64) return launch_chunks<64, 1, 8, XBF, 16>(a, s);
    if (whole && u == 32) return launch_chunks<32, 1, 8, XBF, 8>(a, s);
    if (whole && u == 16) return launch_chunks<16, 1, 8, XBF, 4>(a, s);
    if (u <= 8) return launch_chunks<8, 1, 8, XBF>(a, s);
    if (u <= 16) return launch_chunks<16, 1, 8, XBF>(a, s);
    if (u <= 32) return launch_chunks<32, 1, 8, XBF>(a, s);
    if (u <= 64) return launch_chunks<64, 1, 8, XBF>(a, s);
    if (u <= 128) return launch_chunks<64, 2, 4, XBF>(a, s);
    return launch_chunks<64, 4, 2, XBF>(a, s);
}

template <int G, int UPT, int U, bool XBF, bool ZBF, int VB = 0>
gas_status launch_rows(const SpmmArgs& a, hipStream_t s) {
    const int64_t items = VB > 0 ? a.n_groups : a.n_rows;
    int64_t blocks = (items + 3) / 4;
    if (VB > 0 && a.xcd_ranges) {
        int64_t longest = 0;
        for (int x = 0; x < 8; ++x) longest = std::max(longest, a.xcd_start[x + 1] - a.xcd_start[x]);
        blocks = 8 * ((longest + 3) / 4);
    }
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_spmm: too many workgroups for one launch");
    if (blocks > 0) {
        // (the kernels by units look at a.Y themselves)
        if (VB > 0 && a.Y) hipLaunchKernelGGL((spmm_rows_kernel<G, UPT, U, XBF, ZBF, VB, (VB > 0)>), dim3((unsigned)blocks), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((spmm_rows_kernel<G, UPT, U, XBF, ZBF, VB, false>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    }
    return GAS_OK;
}

template <int P, bool XBF, bool ZBF>
gas_status launch_slices(const SpmmArgs& a, bool whole, hipStream_t s) {
    const int slices = (a.units + 16 * P - 1) / (16 * P), width = (a.units + slices - 1) / slices;
    const int64_t jobs = (a.n_rows + kSliceRows - 1) / kSliceRows * slices;
    const int64_t blocks = a.in_turn ? jobs : 8 * ((jobs + 7) / 8);
    if (blocks > 0x7FFFFFFFLL) return fail(GAS_ERR_ARG, "gas_spmm: too many workgroups for one launch");
    const dim3 grid((unsigned)blocks), block(256);
    // As many partial sums a row as a wavefront's teams make of it in the other form: eight up to 8 units, four up to 16, two up to 32, one
    // beyond and for 32 whole units, which a wavefront takes at once there, and so 16 whole ones of bf16 that are rounded to bf16 again (a few
    // values of a batch come out otherwise in four, and moved the gradients of a training step by up to 5e-4).  Root mean square error against 64 bits, 21 entries: in one
    // sum 8.5e-8, in two 6.7e-8; 60: in one 1.4e-7, in two 1.0e-7, in four 8.1e-8, in eight 7.0e-8.  Eight are four in each half of a team,
    // which takes every other entry: no lane is idle at 8 units (us, eight in each lane and so: 200,000 clustered rows of 9 entries, 32 floats
    // 44.5 -> 30.1, 64 bf16 62.6 -> 37.9; 257,000 power-law rows of 19 103.6 -> 86.0, 139.0 -> 103.1; four in each lane 37.1 to 111.5).
    auto launch = [&](auto split) {
        constexpr int H = decltype(split)::value == 8 ? 2 : 1, S = decltype(split)::value / H;
        if (a.Y) hipLaunchKernelGGL((spmm_slices_kernel<P, false, S, H, XBF, ZBF, true>), grid, block, 0, s, a, slices, width);
        else hipLaunchKernelGGL((spmm_slices_kernel<P, false, S, H, XBF, ZBF, false>), grid, block, 0, s, a, slices, width);
    };
    const bool two = a.units < 32 || (a.units == 32 && !whole);
    if constexpr (P == 1) {
        if (a.units <= 8) launch(std::integral_constant<int, 8>());
        else if (XBF && ZBF && a.units == 16 && whole) launch(std::integral_constant<int, 1>());
        else if (a.units <= 16) launch(std::integral_constant<int, 4>());
        else if (two) launch(std::integral_constant<int, 2>());
        else launch(std::integral_constant<int, 1>());
    } else if constexpr (P == 2) {                        // from 17 units on
        // whole slices need no masks: two pieces a lane 40 -> 39 us (adjoint 38 -> 37); one piece a lane has none, and three gain nothing
        if (two) launch(std::integral_constant<int, 2>());
        else if (a.units == slices * 32 && a.units * 16 == a.F * (XBF ? 2 : 4)) {
            if (a.Y) hipLaunchKernelGGL((spmm_slices_kernel<2, true, 1, 1, XBF, ZBF, true>), grid, block, 0, s, a, slices, width);
            else hipLaunchKernelGGL((spmm_slices_kernel<2, true, 1, 1, XBF, ZBF, false>), grid, block, 0, s, a, slices, width);
        } else launch(std::integral_constant<int, 1>());
    } else launch(std::integral_constant<int, 1>());
    return GAS_OK;
}

template <bool XBF, bool ZBF>
gas_status dispatch_units(const SpmmArgs& a, bool whole, hipStream_t s) {
    const int u = a.units;
    if (u > 256) return fail(GAS_ERR_ARG, "feature rows longer than 4096 bytes are not supported (F*size = %d)", u * 16);
    // heavy rows first: chunk partials, then their reduction; the light rows follow on the same stream
    if (a.n_chunks > 0) {
        const gas_status st = dispatch_chunks<XBF>(a, whole, s);
        if (st != GAS_OK) return st;
        hipLaunchKernelGGL((spmm_heavy_reduce_kernel<XBF, ZBF>), dim3((unsigned)((a.n_heavy + 3) / 4)), dim3(256),
                           0, s, a);
    }
    gas_status st;
    if (a.pieces == 1) st = launch_slices<1, XBF, ZBF>(a, whole, s);
    else if (a.pieces == 2) st = launch_slices<2, XBF, ZBF>(a, whole, s);
    else if (a.pieces == 3) st = launch_slices<3, XBF, ZBF>(a, whole, s);
    // rows of exactly 1 KiB or 512 B: grouped wave-per-row path
    else if (whole && a.group && u == 64) st = launch_rows<64, 1, 8, XBF, ZBF, 16>(a, s);
    else if (whole && a.group && u == 32) st = launch_rows<32, 1, 4, XBF, ZBF, 8>(a, s);
    else if (u <= 8) st = launch_rows<8, 1, 2, XBF, ZBF>(a, s);
    else if (u <= 32) st = launch_rows<32, 1, 4, XBF, ZBF>(a, s);
    else if (u <= 64) st = launch_rows<64, 1, 8, XBF, ZBF>(a, s);
    else if (u <= 128) st = launch_rows<64, 2, 4, XBF, ZBF>(a, s);
    else st = launch_rows<64, 4, 2, XBF, ZBF>(a, s);
    if (st != GAS_OK) return st;
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

// How the light rows are taken: by slices of 16 `pieces` units (0: a wavefront a row), contiguous or in turn.  us on rotating
// inputs, a wavefront a row and slices, over clustered patterns of 2,000 to 200,000 rows of 7 to 31 entries and power laws of
// 1,250 to 600,000 rows (mean 2 to 86) with their adjoints:
// - up to 16 units a row fits one slice and always wins (64 floats: 50,000 clustered rows 28 and 16, their adjoint 29 and 15,
//   250,000 power-law rows 326 and 316 forward, 187 and 140 adjoint), but for at most 8 units and few, long rows, where the
//   other form has eight entries in flight beside each other (15,000 rows of 43, 32 floats 23 and 26);
// - 17 to 31 units are one slice of two pieces a lane (136 bf16: 50,000 clustered rows 36 and 26, 600,000 power-law rows 2,337 and
//   2,256); few long rows of a power law keep a wavefront each (50,000 rows of 36, 100 floats 114 and 119);
// - 32 and 64 whole units, 512 and 1,024 bytes, go by 256 bytes (600,000 power-law rows of 84, 256 floats 5.06 and 4.94 ms,
//   adjoint 1.86 and 1.79; 100,000 clustered rows of 10 147 and 101); 64 clustered with two pieces where few entries share a row and
//   the batch is not much more than the L2s hold (50,000 of 11: 43 by one, 39 by two pieces; 75,000 of 7 48 and 43; 64,000 of 23
//   108 and 145); a wavefront a row with more than 28 entries, which fetches a cluster's rows once into its XCD (25,000 of 31:
//   56 and 62), and with fewer than four, grouped (312,500 rows of 0.9, 256 bf16 100 and 132);
// - 33 to 48 units are one slice of three pieces (184 floats: 50,000 clustered rows 53 and 39, adjoint of 250,000 power-law rows 491
//   and 456);
// - 49 to 63 units are two slices that share a cache line: clustered and near the size of the L2s (248 floats: 50,000 rows 61
//   and 45, 100,000 143 and 155; power law 600,000 5.32 and 5.55 ms);
// - wider ones two pieces at a time where they are clustered or few (1,433 floats: 50,000 rows 429 and 370, 5,000 49 and 37; 150,000
//   power-law rows 7.2 and 7.4 ms);
// - few rows are a matter of the chain of loads alone: one piece a lane has eight entries in flight (5,000 rows of 11, 248
//   floats 9.7 and 8.7; 1,250 power-law rows of 19, 184 floats 28 and 17, by three pieces 32).
struct RowsForm { int pieces, in_turn; };
RowsForm rows_form(const gas_plan* plan, int units, bool whole) {
    const int64_t n = plan->n_rows, nnz = plan->nnz, bytes = n * units * 16;
    const bool even = whole && (units == 32 || units == 64);
    if (plan->xcd_ranges) {
        if (units > 64) return {2, 0};
        if (units <= 16 || n <= 8192 || (even && units == 32)) return {1, 0};
        if (units <= 32) return {2, 0};
        if (units <= 48) return {units <= 40 || bytes <= (int64_t)112 << 20 ? 3 : 0, 0};
        if (nnz > 28 * n) return {0, 0};
        if (!even) return {bytes <= (int64_t)80 << 20 ? 2 : 0, 0};
        return {nnz <= 16 * n && bytes <= (int64_t)80 << 20 ? 2 : 1, 0};
    }
    if (units <= 8 && n < 65536) return {0, 0};
    if (n <= 16384) return {units > 64 ? 2 : 1, 0};
    if (units <= 16) return {1, 1};
    if (even) return {nnz < 4 * n ? 0 : 1, 1};
    if (units <= 32) return {n < 65536 && nnz > 24 * n ? 0 : 2, 1};
    return {units <= 48 ? 3 : 0, 1};
}

gas_status run_spmm(const char* who, const gas_plan* plan, const int32_t* ptr, const int32_t* ind, const float* val,
                    float diag, int64_t n_diag, const void* X, int64_t ldx, const void* H, int64_t ldh,
                    gas_dtype dt_x, int32_t F, float s_agg,
                    const void* R, int64_t ldr, float s_res, void* Z, int64_t ldz, gas_dtype dt_z, hipStream_t s,
                    const void* Y = nullptr, int64_t ldy = 0, const int32_t* own = nullptr) {
    if (!valid_dtype(dt_x) || !valid_dtype(dt_z)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype", who);
    if (dt_x == GAS_F32 && dt_z == GAS_BF16)
        return fail(GAS_ERR_DTYPE, "%s: fp32 input with bf16 output is not supported", who);
    GAS_REQUIRE(plan, "%s: null plan", who);
    if (plan->n_rows == 0) return GAS_OK;
    GAS_REQUIRE(ptr && X && Z, "%s: null pointer", who);
    GAS_REQUIRE(plan->nnz == 0 || ind, "%s: null index array", who);
    GAS_REQUIRE(F > 0 && F <= plan->max_F, "%s: F=%d outside (0, plan max_F=%d]", who, F, plan->max_F);
    GAS_REQUIRE(ldx >= F && ldz >= F && (!R || ldr >= F) && (!H || ldh >= F), "%s: row stride smaller than F", who);
    GAS_REQUIRE(!Y || ldy >= F, "%s: row stride of the mask smaller than F", who);
    GAS_REQUIRE(Z != X && Z != R && Z != Y, "%s: output aliases an input", who);
    const int xb = elem_bytes(dt_x), zb = elem_bytes(dt_z);
    // Rows longer than 4096 bytes (a wide input layer) are aggregated panel by panel: the sum is separate for
    // every feature column, so a panel of columns is an aggregation of its own over the same pattern.
    const int64_t panel = 4096 / xb;
    if ((int64_t)F > panel) {
        for (int64_t f0 = 0; f0 < F; f0 += panel) {
            const int32_t fw = (int32_t)std::min<int64_t>(panel, F - f0);
            const gas_status st = run_spmm(who, plan, ptr, ind, val, diag, n_diag, static_cast<const char*>(X) + f0 * xb,
                                           ldx, H ? static_cast<const char*>(H) + f0 * xb : nullptr, ldh, dt_x, fw, s_agg,
                                           R ? static_cast<const char*>(R) + f0 * xb : nullptr, ldr, s_res,
                                           static_cast<char*>(Z) + f0 * zb, ldz, dt_z, s,
                                           Y ? static_cast<const char*>(Y) + f0 * xb : nullptr, ldy, own);
            if (st != GAS_OK) return st;
        }
        return GAS_OK;
    }
    SpmmArgs a;
    a.ptr = ptr; a.ind = ind; a.val = val;
    a.X = static_cast<const char*>(X); a.x_stride = ldx * xb;
    a.H = static_cast<const char*>(H); a.h_stride = ldh * xb;
    a.R = static_cast<const char*>(R); a.r_stride = ldr * xb;
    a.Y = static_cast<const char*>(Y); a.y_stride = ldy * xb;
    a.Z = static_cast<char*>(Z); a.z_stride = ldz * zb;
    a.own = own; a.diag = diag; a.s_agg = s_agg; a.s_res = s_res;
    a.n_rows = plan->n_rows; a.n_diag = n_diag;
    a.units = (F * xb + 15) / 16; a.F = F;
    a.threshold = plan->threshold;
    a.chunk = plan->d_chunk; a.n_chunks = plan->n_chunks;
    a.heavy = plan->d_heavy; a.n_heavy = plan->n_heavy;
    a.partial = plan->d_partial;
    a.group = plan->d_group; a.n_groups = plan->n_groups;
    a.xcd_ranges = plan->xcd_ranges;
    for (int x = 0; x < 9; ++x) a.xcd_start[x] = plan->xcd_start[x];
    const bool whole = (F * xb) % 16 == 0 && aligned16(X) && a.x_stride % 16 == 0 && aligned16(Z) &&
                       a.z_stride % 16 == 0 && (!R || (aligned16(R) && a.r_stride % 16 == 0)) &&
                       (!H || (aligned16(H) && a.h_stride % 16 == 0)) && (!Y || (aligned16(Y) && a.y_stride % 16 == 0));
    const RowsForm form = rows_form(plan, a.units, whole);
    a.pieces = form.pieces; a.in_turn = form.in_turn;
    const bool xbf = dt_x == GAS_BF16, zbf = dt_z == GAS_BF16;
    // From one 16-byte unit on, rows go by units whatever their width and alignment: a row of 1,433 floats 5,000 times,
    // 11 entries each, 49 us (element-wise 254 us).
    if (F * xb >= 16) {
        if (!xbf) return dispatch_units<false, false>(a, whole, s);
        return zbf ? dispatch_units<true, true>(a, whole, s) : dispatch_units<true, false>(a, whole, s);
    }
    const unsigned blocks = (unsigned)((a.n_rows + 3) / 4);
    if (!xbf) hipLaunchKernelGGL((spmm_generic_kernel<false, false>), dim3(blocks), dim3(256), 0, s, a);
    else if (zbf) hipLaunchKernelGGL((spmm_generic_kernel<true, true>), dim3(blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((spmm_generic_kernel<true, false>), dim3(blocks), dim3(256), 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

__global__ __launch_bounds__(256) void fuse_sources_kernel(const int32_t* __restrict__ col, int64_t nnz, int64_t nb,
                                                           const int32_t* __restrict__ n_id,
                                                           int32_t* __restrict__ src) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= nnz) return;
    const int32_t c = col[k];
    src[k] = c < nb ? c : -1 - n_id[c];
}

}  // namespace
}  // namespace gas

using namespace gas;

extern "C" {

gas_status gas_spmm(const gas_plan* plan, const int32_t* rowptr, const int32_t* col, const float* val, float diag,
                    const void* X, int64_t ldx, gas_dtype dt_x, int32_t F, float s_agg, const void* R, int64_t ldr,
                    float s_res, void* Z, int64_t ldz, gas_dtype dt_z, void* stream) {
    return run_spmm("gas_spmm", plan, rowptr, col, val, diag, plan ? plan->n_rows : 0, X, ldx, nullptr, 0, dt_x, F,
                    s_agg, R, ldr, s_res, Z, ldz, dt_z, (hipStream_t)stream);
}

gas_status gas_spmm_t(const gas_plan* plan, const int32_t* colptr, const int32_t* row, const float* val, float diag,
                      float s_agg, int64_t n_diag, const void* G, int64_t ldg, gas_dtype dt_g, int32_t F, void* GX,
                      int64_t ldgx, gas_dtype dt_gx, void* stream) {
    GAS_REQUIRE(n_diag >= 0, "gas_spmm_t: n_diag=%lld", (long long)n_diag);
    return run_spmm("gas_spmm_t", plan, colptr, row, val, diag, n_diag, G, ldg, nullptr, 0, dt_g, F, s_agg, nullptr,
                    0, 0.f, GX, ldgx, dt_gx, (hipStream_t)stream);
}

gas_status gas_spmm_t_relu(const gas_plan* plan, const int32_t* colptr, const int32_t* row, const float* val, float diag,
                           float s_agg, int64_t n_diag, const void* G, int64_t ldg, gas_dtype dt, int32_t F,
                           const void* Y, int64_t ldy, void* GX, int64_t ldgx, void* stream) {
    GAS_REQUIRE(n_diag >= 0, "gas_spmm_t_relu: n_diag=%lld", (long long)n_diag);
    GAS_REQUIRE(Y || !plan || plan->n_rows == 0, "gas_spmm_t_relu: null activations");
    return run_spmm("gas_spmm_t_relu", plan, colptr, row, val, diag, n_diag, G, ldg, nullptr, 0, dt, F, s_agg, nullptr,
                    0, 0.f, GX, ldgx, dt, (hipStream_t)stream, Y, ldy);
}

gas_status gas_spmm_hist(const gas_plan* plan, const int32_t* rowptr, const int32_t* src, const float* val,
                         float diag, const void* X, int64_t ldx, const void* hist, int64_t n_hist_rows,
                         int64_t ld_hist, gas_dtype dt_x, int32_t F, float s_agg, const void* R, int64_t ldr,
                         float s_res, void* Z, int64_t ldz, gas_dtype dt_z, void* stream) {
    GAS_REQUIRE(hist && n_hist_rows > 0, "gas_spmm_hist: null or empty history table");
    GAS_REQUIRE(Z != hist, "gas_spmm_hist: output aliases the history table");
    return run_spmm("gas_spmm_hist", plan, rowptr, src, val, diag, plan ? plan->n_rows : 0, X, ldx, hist, ld_hist,
                    dt_x, F, s_agg, R, ldr, s_res, Z, ldz, dt_z, (hipStream_t)stream);
}

gas_status gas_spmm_table(const gas_plan* plan, const int32_t* rowptr, const int32_t* src, const float* val, float diag,
                          const int32_t* own, const void* table, int64_t n_table_rows, int64_t ld_table, gas_dtype dt_x, int32_t F,
                          float s_agg, void* Z, int64_t ldz, gas_dtype dt_z, void* stream) {
    GAS_REQUIRE(table && n_table_rows > 0, "gas_spmm_table: null or empty table");
    GAS_REQUIRE(diag == 0.f || own, "gas_spmm_table: the diagonal term needs the rows' ids");
    return run_spmm("gas_spmm_table", plan, rowptr, src, val, diag, plan ? plan->n_rows : 0, table, ld_table, table, ld_table, dt_x, F,
                    s_agg, nullptr, 0, 0.f, Z, ldz, dt_z, (hipStream_t)stream, nullptr, 0, own);
}

gas_status gas_fuse_sources(const int32_t* col, int64_t nnz, int64_t nb, const int32_t* n_id, int32_t* src,
                            void* stream) {
    GAS_REQUIRE(nnz >= 0 && nb >= 0, "gas_fuse_sources: nnz=%lld nb=%lld", (long long)nnz, (long long)nb);
    if (nnz == 0) return GAS_OK;
    GAS_REQUIRE(col && n_id && src, "gas_fuse_sources: null pointer");
    const int64_t blocks = (nnz + 255) / 256;
    GAS_REQUIRE(blocks <= 0x7FFFFFFFLL, "gas_fuse_sources: too many entries");
    hipLaunchKernelGGL(fuse_sources_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, col, nnz, nb,
                       n_id, src);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

}  // extern "C"
