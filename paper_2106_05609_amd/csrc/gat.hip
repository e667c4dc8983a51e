// GAT's anisotropic aggregation (paper, operator appendix), one head: attention scores, their softmax over the
// entries of a row and the weighted sum of the gathered rows in ONE pass (running maximum and running sum,
// rescaled block by block), so every neighbour row is gathered once.  The score of an entry needs the whole
// gathered row, which a wavefront holds across its lanes: the dot product with the attention vector is a
// reduction over the lanes.  HBM-bound like the other aggregations.  Several heads side by side in a row are taken
// together by teams of lanes: a row is gathered once, not once per head.
#include "wave.h"

namespace gas {
namespace {

struct GatArgs {
    const int32_t* rowptr; const int32_t* col;
    int64_t n_rows;
    const char* P; int64_t ldp;
    const char* a_dst; const char* a_src;
    char* Z; int64_t ldz;
    int F;                                        // width of a head; head h has columns h F .. of P and Z
    float slope;
    int relu;                                     // ReLU on the output row
    int longest;                                  // no row has more entries
    const int32_t* push_idx;                      // optional: output row v is also stored to push_hist[push_idx[v]]
    char* push_hist; int64_t ld_push;
};

// Rows of at most 64 pieces of 16 bytes, G = 16, 32 or 64 lanes per row (at least the number of pieces).  A
// wavefront's S = 64 / (G H) slots of H teams of G lanes each hold the whole row, a head per team, and take the entries
// in turn (slot t the entries t, t + S, ... of every block of 64), eight at a time per slot: gathers, scores (one
// reduction over the team's lanes for all eight), one rescale of the running sums to the new maximum, then the weighted
// adds.  Every team keeps its own running maximum and sums, and the slots' states are merged pair by pair at the end.  A row of
// more than kLongRow entries is shared by the kLongWaves wavefronts of a workgroup in the same way, block of 64
// entries by block, and their states are merged in wavefront order.  Which lane takes which entry depends on the
// row's length and the width alone, so the result is the same bits on every run.

// running softmax state of one lane: maximum m, sum of weights l, weighted sum acc of its piece
template <int E>
__device__ __forceinline__ void merge_state(float& m, float& l, float (&acc)[E], float mo, float lo, const float (&acco)[E]) {
    const float mm = fmaxf(m, mo);
    // a state that has seen no entry has m = -inf and zero sums
    const float s1 = m > -INFINITY ? expf(m - mm) : 0.f, s2 = mo > -INFINITY ? expf(mo - mm) : 0.f;
    l = l * s1 + lo * s2;
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = acc[i] * s1 + acco[i] * s2;
    m = mm;
}

// The entries of the blocks first, first + stride, ... of row v = [b, e), b < e: afterwards every team of the
// wavefront holds the merged state of all of them.
template <bool BF, int G, int H>
__device__ __forceinline__ void gat_gather(const GatArgs& a, int64_t v, int b, int e, int first, int stride,
                                           float& m, float& l, float (&acc)[Elems<BF>::E]) {
    constexpr int E = Elems<BF>::E, EB = BF ? 2 : 4, U = 8, S = HeadTeams<G, H>::kSlots;
    const HeadTeams<G, H> ht;
    const int lane = threadIdx.x & 63, team = ht.slot;
    const bool on = ht.tl * E < a.F;
    const int64_t own = (int64_t)ht.head * a.F + ht.tl * E;      // the lane's first column
    float ad[E], ar[E], x[E];
    u32x4 t = {0u, 0u, 0u, 0u};
    if (on) t = *reinterpret_cast<const u32x4*>(a.a_dst + own * EB);
    unpack<BF>(t, ad);
    t = u32x4{0u, 0u, 0u, 0u};
    if (on) t = *reinterpret_cast<const u32x4*>(a.a_src + own * EB);
    unpack<BF>(t, ar);
    t = u32x4{0u, 0u, 0u, 0u};
    if (on) t = *reinterpret_cast<const u32x4*>(a.P + (v * a.ldp + own) * EB);
    unpack<BF>(t, x);
    float sv = 0.f;
#pragma unroll
    for (int i = 0; i < E; ++i) sv += ad[i] * x[i];
    sv = team_sum<G>(sv);
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.f;
    for (int k0 = b + 64 * first; k0 < e; k0 += 64 * stride) {
        const int cnt = min(64, e - k0);
        const int mine = lane < cnt ? a.col[k0 + lane] : 0;
        for (int j0 = 0; j0 < cnt; j0 += U * S) {
            u32x4 r[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int kk = j0 + j * S + team;
                int c;
                if constexpr (S == 1) c = __builtin_amdgcn_readlane(mine, kk & 63);
                else c = __shfl(mine, kk & 63);
                r[j] = u32x4{0u, 0u, 0u, 0u};
                if (on && kk < cnt)
                    r[j] = *reinterpret_cast<const u32x4*>(a.P + ((int64_t)c * a.ldp + own) * EB);
            }
            float sc[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                unpack<BF>(r[j], x);
                sc[j] = 0.f;
#pragma unroll
                for (int i = 0; i < E; ++i) sc[j] += ar[i] * x[i];
            }
            // a lane has one of the eight scores, and its weight: formed by every lane they are most of the instructions
            float s = team_sum8_own<G>(sc) + sv;
            s = s > 0.f ? s : a.slope * s;
            s = j0 + ht.tl / (G / 8) * S + team < cnt ? s : -INFINITY;
            const float mb = fmaxf(m, team_max8<G>(s));
            if (mb > -INFINITY) {                         // a team may have had no entry of its own yet
                const float scale = expf(m - mb);         // m = -inf at the start: scale 0 on sums that are 0
                // the eight entries are summed by themselves first: a sum over a long row is then one of few large terms
                const float own_p = expf(s - mb);         // 0 for the padding entries
                float lb = 0.f, part[E];
#pragma unroll
                for (int i = 0; i < E; ++i) part[i] = 0.f;
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const float p = team_value8<G>(own_p, j);
                    lb += p;
                    unpack<BF>(r[j], x);
#pragma unroll
                    for (int i = 0; i < E; ++i) part[i] += p * x[i];
                }
                l = l * scale + lb;
#pragma unroll
                for (int i = 0; i < E; ++i) acc[i] = acc[i] * scale + part[i];
                m = mb;
            }
        }
    }
    // both partners of an exchange compute the same merged state
#pragma unroll
    for (int o = G * H; o < 64; o <<= 1) {
        const float mo = __shfl_xor(m, o), lo = __shfl_xor(l, o);
        float acco[E];
#pragma unroll
        for (int i = 0; i < E; ++i) acco[i] = __shfl_xor(acc[i], o);
        merge_state<E>(m, l, acc, mo, lo, acco);
    }
}

template <bool BF, int G, int H>
__device__ __forceinline__ void gat_finish(const GatArgs& a, int64_t v, float l, float (&acc)[Elems<BF>::E]) {
    constexpr int E = Elems<BF>::E, EB = BF ? 2 : 4;
    const HeadTeams<G, H> ht;
    if (ht.slot > 0 || ht.tl * E >= a.F) return;      // slot 0 stores
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < E; ++i) {
        acc[i] *= inv;
        if (a.relu) acc[i] = fmaxf(acc[i], 0.f);
    }
    const u32x4 y = pack<BF>(acc);
    const int64_t at = (int64_t)ht.head * a.F + ht.tl * E;
    __builtin_nontemporal_store(y, reinterpret_cast<u32x4*>(a.Z + (v * a.ldz + at) * EB));
    if (a.push_idx) __builtin_nontemporal_store(y, reinterpret_cast<u32x4*>(a.push_hist + (a.push_idx[v] * a.ld_push + at) * EB));
}

// one wavefront per row; long rows are left to gat_long_rows_kernel
template <bool BF, int G, int H>
__global__ __launch_bounds__(64) void gat_rows_kernel(GatArgs a) {
    constexpr int E = Elems<BF>::E, EB = BF ? 2 : 4;
    const int64_t v = blockIdx.x;
    const int b = a.rowptr[v], e = a.rowptr[v + 1];
    if (e == b) {
        const HeadTeams<G, H> ht;
        if (ht.slot == 0 && ht.tl * E < a.F) {
            const int64_t at = (int64_t)ht.head * a.F + ht.tl * E;
            *reinterpret_cast<u32x4*>(a.Z + (v * a.ldz + at) * EB) = u32x4{0u, 0u, 0u, 0u};
            if (a.push_idx) *reinterpret_cast<u32x4*>(a.push_hist + (a.push_idx[v] * a.ld_push + at) * EB) = u32x4{0u, 0u, 0u, 0u};
        }
        return;
    }
    if (e - b > kLongRow) return;
    float m, l, acc[E];
    gat_gather<BF, G, H>(a, v, b, e, 0, 1, m, l, acc);
    gat_finish<BF, G, H>(a, v, l, acc);
}

// Workgroup w looks at the rows w, w + gridDim.x, ... (512 of them at a time), and every row of more than kLongRow
// entries among them is gathered by all its wavefronts together.
template <bool BF, int G, int H>
__global__ __launch_bounds__(64 * kLongWaves) void gat_long_rows_kernel(GatArgs a) {
    constexpr int E = Elems<BF>::E, T = 64 * kLongWaves;
    __shared__ int queue[T];
    __shared__ int n_queued;
    __shared__ float red[kLongWaves][E + 2][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int64_t r0 = blockIdx.x; r0 < a.n_rows; r0 += (int64_t)T * gridDim.x) {
        const int nq = queue_long_rows(a.rowptr, a.n_rows, r0, queue, &n_queued);
        for (int q = 0; q < nq; ++q) {
            const int64_t v = queue[q];
            const int b = a.rowptr[v], e = a.rowptr[v + 1];
            float m, l, acc[E];
            gat_gather<BF, G, H>(a, v, b, e, w, kLongWaves, m, l, acc);
            if (w > 0) {
                red[w][E][lane] = m;
                red[w][E + 1][lane] = l;
#pragma unroll
                for (int i = 0; i < E; ++i) red[w][i][lane] = acc[i];
            }
            __syncthreads();
            if (w == 0) {
                for (int o = 1; o < kLongWaves; ++o) {
                    float acco[E];
#pragma unroll
                    for (int i = 0; i < E; ++i) acco[i] = red[o][i][lane];
                    merge_state<E>(m, l, acc, red[o][E][lane], red[o][E + 1][lane], acco);
                }
                gat_finish<BF, G, H>(a, v, l, acc);
            }
            __syncthreads();
        }
    }
}

template <bool BF, int G, int H>
void launch_rows(const GatArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((gat_rows_kernel<BF, G, H>), dim3((unsigned)a.n_rows), dim3(64), 0, s, a);
    if (a.longest <= kLongRow) return;            // 4 us even where it finds none
    const unsigned blocks = long_row_blocks(a.n_rows);
    hipLaunchKernelGGL((gat_long_rows_kernel<BF, G, H>), dim3(blocks), dim3(64 * kLongWaves), 0, s, a);
}

// H heads of at most 64 / H teams of lanes
template <bool BF>
void launch_vec(const GatArgs& a, int H, hipStream_t s) {
    const int G = gat_team<BF>(a.F, H > 1);
    if (G == 64) launch_rows<BF, 64, 1>(a, s);
    else if (G == 32) H == 2 ? launch_rows<BF, 32, 2>(a, s) : launch_rows<BF, 32, 1>(a, s);
    else if (G == 16) H == 4 ? launch_rows<BF, 16, 4>(a, s) : H == 2 ? launch_rows<BF, 16, 2>(a, s) : launch_rows<BF, 16, 1>(a, s);
    else if constexpr (BF) H == 4 ? launch_rows<BF, 8, 4>(a, s) : launch_rows<BF, 8, 2>(a, s);
}

// any alignment, widths up to 64 * NE: lane l owns elements l, l + 64, ...; one entry at a time
template <bool BF, int NE>
__global__ __launch_bounds__(64) void gat_generic_kernel(GatArgs a) {
    const int64_t v = blockIdx.x;
    const int lane = threadIdx.x;
    auto ld = [&](const char* p, int64_t i) -> float {
        if constexpr (BF) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(p)[i] << 16);
        else return reinterpret_cast<const float*>(p)[i];
    };
    const int b = a.rowptr[v], e = a.rowptr[v + 1];
    float ad[NE], ar[NE], acc[NE], x[NE];
    float sv = 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int f = lane + 64 * i;
        ad[i] = f < a.F ? ld(a.a_dst, f) : 0.f;
        ar[i] = f < a.F ? ld(a.a_src, f) : 0.f;
        acc[i] = 0.f;
        if (f < a.F && e > b) sv += ad[i] * ld(a.P, v * a.ldp + f);
    }
    sv = wave_sum(sv);
    float m = -INFINITY, l = 0.f;
    for (int k = b; k < e; ++k) {
        const int64_t c = a.col[k];
        float part = 0.f;
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int f = lane + 64 * i;
            x[i] = f < a.F ? ld(a.P, c * a.ldp + f) : 0.f;
            part += ar[i] * x[i];
        }
        float s = wave_sum(part) + sv;
        s = s > 0.f ? s : a.slope * s;
        const float mb = fmaxf(m, s), scale = expf(m - mb), p = expf(s - mb);
        l = l * scale + p;
#pragma unroll
        for (int i = 0; i < NE; ++i) acc[i] = acc[i] * scale + p * x[i];
        m = mb;
    }
    const float inv = e > b ? 1.f / l : 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int f = lane + 64 * i;
        if (f < a.F) {
            const float y = a.relu ? fmaxf(acc[i] * inv, 0.f) : acc[i] * inv;
            if constexpr (BF) reinterpret_cast<uint16_t*>(a.Z)[v * a.ldz + f] = (uint16_t)f32_to_bf16(y);
            else reinterpret_cast<float*>(a.Z)[v * a.ldz + f] = y;
        }
    }
}

template <bool BF>
gas_status launch_generic(const GatArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.n_rows), block(64);
    if (a.F <= 64) hipLaunchKernelGGL((gat_generic_kernel<BF, 1>), grid, block, 0, s, a);
    else if (a.F <= 256) hipLaunchKernelGGL((gat_generic_kernel<BF, 4>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((gat_generic_kernel<BF, 16>), grid, block, 0, s, a);
    GAS_CHECK_HIP(hipGetLastError());
    return GAS_OK;
}

}  // namespace
}  // namespace gas

using namespace gas;

// The Push is taken with the output row in registers: 50,000 rows of 11 entries, four heads, 256 floats, with a copy of the rows (and
// the launch for long ones) afterwards 119 us, here 98; 3,500 rows of 12, 224 floats, 16.9 and 7.3.
extern "C" gas_status gas_gat_aggregate_push(const int32_t* rowptr, const int32_t* col, int64_t n_rows, int32_t longest, const void* P,
                                             int64_t ldp, gas_dtype dt, int32_t F, int32_t heads, const void* a_dst,
                                             const void* a_src, float negative_slope, int relu, void* Z, int64_t ldz,
                                             const int32_t* push_idx, void* push_hist, int64_t n_hist_rows, int64_t ld_push,
                                             void* stream) {
    const char* who = "gas_gat_aggregate";
    if (!valid_dtype(dt)) return fail(GAS_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dt);
    GAS_REQUIRE(n_rows >= 0 && F > 0 && heads > 0, "%s: n_rows=%lld F=%d heads=%d", who, (long long)n_rows, F, heads);
    GAS_REQUIRE(F <= 1024, "%s: F=%d exceeds 1024", who, F);
    if (n_rows == 0) return GAS_OK;
    GAS_REQUIRE(rowptr && col && P && a_dst && a_src && Z, "%s: null pointer", who);
    GAS_REQUIRE(ldp >= (int64_t)heads * F && ldz >= (int64_t)heads * F, "%s: row stride smaller than the row", who);
    GAS_REQUIRE(Z != P, "%s: the output must not alias the input", who);
    GAS_REQUIRE(n_rows <= 0x7FFFFFFFLL, "%s: too many rows for one launch", who);
    GAS_REQUIRE(!push_idx || (push_hist && push_hist != Z && push_hist != P && ld_push >= (int64_t)heads * F && n_hist_rows > 0),
                "%s: bad history table for the push", who);
    GatArgs a;
    a.rowptr = rowptr; a.col = col; a.n_rows = n_rows;
    a.P = static_cast<const char*>(P); a.ldp = ldp;
    a.a_dst = static_cast<const char*>(a_dst); a.a_src = static_cast<const char*>(a_src);
    a.Z = static_cast<char*>(Z); a.ldz = ldz;
    a.F = F; a.slope = negative_slope; a.relu = relu; a.longest = longest;
    const int e = dt == GAS_BF16 ? 8 : 4, eb = elem_bytes(dt);
    hipStream_t s = (hipStream_t)stream;
    const bool vec = F % e == 0 && F <= 64 * e && ldp % e == 0 && ldz % e == 0 && aligned16(P) && aligned16(Z) &&
                     aligned16(a_dst) && aligned16(a_src);
    const bool scatter = push_idx && vec && ld_push % e == 0 && aligned16(push_hist);      // else a copy of the rows follows
    a.push_idx = scatter ? push_idx : nullptr; a.push_hist = static_cast<char*>(push_hist); a.ld_push = ld_push;
    const int H = !vec ? 1 : (dt == GAS_BF16 ? gat_heads_together<true>(F, heads) : gat_heads_together<false>(F, heads));
    for (int32_t h = 0; h < heads; h += H) {
        gas_status st = GAS_OK;
        if (vec && dt == GAS_BF16) launch_vec<true>(a, H, s);
        else if (vec) launch_vec<false>(a, H, s);
        else st = dt == GAS_BF16 ? launch_generic<true>(a, s) : launch_generic<false>(a, s);
        if (st != GAS_OK) return st;
        GAS_CHECK_HIP(hipGetLastError());
        a.P += (int64_t)H * F * eb; a.Z += (int64_t)H * F * eb;
        a.a_dst += (int64_t)H * F * eb; a.a_src += (int64_t)H * F * eb;
        if (scatter) a.push_hist += (int64_t)H * F * eb;
    }
    return push_idx && !scatter ? gas_push(Z, ldz, push_idx, 0, n_rows, heads * F, dt, push_hist, n_hist_rows, ld_push, stream) : GAS_OK;
}

extern "C" gas_status gas_gat_aggregate_heads(const int32_t* rowptr, const int32_t* col, int64_t n_rows, const void* P,
                                              int64_t ldp, gas_dtype dt, int32_t F, int32_t heads, const void* a_dst,
                                              const void* a_src, float negative_slope, int relu, void* Z, int64_t ldz,
                                              void* stream) {
    return gas_gat_aggregate_push(rowptr, col, n_rows, 0x7FFFFFFF, P, ldp, dt, F, heads, a_dst, a_src, negative_slope, relu, Z, ldz,
                                  nullptr, nullptr, 0, 0, stream);
}

extern "C" gas_status gas_gat_aggregate(const int32_t* rowptr, const int32_t* col, int64_t n_rows, const void* P,
                                        int64_t ldp, gas_dtype dt, int32_t F, const void* a_dst, const void* a_src,
                                        float negative_slope, int relu, void* Z, int64_t ldz, void* stream) {
    return gas_gat_aggregate_heads(rowptr, col, n_rows, P, ldp, dt, F, 1, a_dst, a_src, negative_slope, relu, Z, ldz, stream);
}
