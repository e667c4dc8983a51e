// Helpers shared by the one-wavefront-per-row kernels (PNA and GAT aggregations and their backward passes):
// reductions over the 64 lanes and the 16-byte piece of a feature row that a lane owns.
#pragma once
#include "common.h"

namespace gas {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Sum over the G lanes of a team: the wavefront's aligned groups of G lanes, G a power of two.
template <int G>
__device__ __forceinline__ float team_sum(float v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Eight sums over the lanes of every team of G at once: at each of the first three steps a lane keeps one half of its values,
// adds the partner's copy of that half and hands over the other half, so 4 + 2 + 1 exchanges leave one partial sum per lane,
// and the remaining steps finish it: seven exchanges and more instead of 8 log2 G.  The lane's return value is the total of
// s[tl / (G / 8)], tl its number in the team.
template <int G>
__device__ __forceinline__ float team_sum8_own(const float (&s)[8]) {
    static_assert(G == 8 || G == 16 || G == 32 || G == 64, "teams of 8 to 64 lanes");
    const int lane = threadIdx.x & 63;
    const bool ha = lane & (G / 2), hb = lane & (G / 4), hc = lane & (G / 8);
    float t4[4], t2[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) t4[j] = (ha ? s[j + 4] : s[j]) + __shfl_xor(ha ? s[j] : s[j + 4], G / 2);
#pragma unroll
    for (int j = 0; j < 2; ++j) t2[j] = (hb ? t4[j + 2] : t4[j]) + __shfl_xor(hb ? t4[j] : t4[j + 2], G / 4);
    float t = (hc ? t2[1] : t2[0]) + __shfl_xor(hc ? t2[0] : t2[1], G / 8);
#pragma unroll
    for (int o = G / 16; o > 0; o >>= 1) t += __shfl_xor(t, o);
    return t;
}
// The largest of the eight values that the lanes of a team hold so.
template <int G>
__device__ __forceinline__ float team_max8(float v) {
#pragma unroll
    for (int o = G / 2; o >= G / 8; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// ---- several attention heads in one wavefront
// The row of a node holds H heads side by side.  Team t = lane / G of a wavefront has head t % H of the entry that
// slot t / H works on, so the teams of a slot load one contiguous row, and a head's sums never leave its teams.
template <int G, int H>
struct HeadTeams {
    static_assert(G * H <= 64, "the heads of an entry fit a wavefront");
    static constexpr int kSlots = 64 / (G * H);
    int tl, head, slot;
    __device__ __forceinline__ HeadTeams() {
        const int lane = threadIdx.x & 63;
        tl = lane % G;
        head = lane / G % H;
        slot = lane / (G * H);
    }
    // the same head's lanes of the other slots, added / compared pair by pair
    static __device__ __forceinline__ float over_slots(float v) {
#pragma unroll
        for (int o = G * H; o < 64; o <<= 1) v += __shfl_xor(v, o);
        return v;
    }
    static __device__ __forceinline__ float max_over_slots(float v) {
#pragma unroll
        for (int o = G * H; o < 64; o <<= 1) v = fmaxf(v, __shfl_xor(v, o));
        return v;
    }
};

// A value per head (the same in all lanes of the head) over the W wavefronts of a workgroup in wavefront order; every
// thread calls it; red: W * 4 floats.
template <int W, bool MAX>
__device__ __forceinline__ float across_waves_by_head(float x, int head, bool writer, float (*red)[4]) {
    if constexpr (W == 1) return x;
    if (writer) red[threadIdx.x >> 6][head] = x;
    __syncthreads();
    float r = red[0][head];
#pragma unroll
    for (int o = 1; o < W; ++o) r = MAX ? fmaxf(r, red[o][head]) : r + red[o][head];
    __syncthreads();
    return r;
}

// ---- rows too long for one wavefront
// The one-wavefront-per-row kernels leave a row of more than kLongRow entries to a second launch of kLongBlocks
// workgroups of kLongWaves wavefronts, which take the row's blocks of 64 entries in turn: a hub row of 17,000
// entries is thousands of dependent steps for one wavefront, which the whole launch would wait for.
constexpr int kLongRow = 2048;
constexpr int kLongWaves = 8;
constexpr int kLongBlocks = 2048;                     // 512, 8,192 and 32,768 were measured slower
inline unsigned long_row_blocks(int64_t n_rows) { return (unsigned)(n_rows < kLongBlocks ? n_rows : kLongBlocks); }

// Workgroup w of such a launch looks at the rows w, w + gridDim.x, ..., blockDim.x of them per call (r0 = w, then
// + blockDim.x * gridDim.x): the long ones among them are left in queue[0 .. return value).  Called by every thread
// of the workgroup; the caller passes a barrier between its last use of the queue and the next call.
__device__ __forceinline__ int queue_long_rows(const int32_t* rowptr, int64_t n_rows, int64_t r0, int* queue, int* n_queued,
                                               int longer_than = kLongRow) {
    if (threadIdx.x == 0) *n_queued = 0;
    __syncthreads();
    const int64_t r = r0 + (int64_t)threadIdx.x * gridDim.x;
    if (r < n_rows && rowptr[r + 1] - rowptr[r] > longer_than) queue[atomicAdd(n_queued, 1)] = (int)r;
    __syncthreads();
    return *n_queued;
}

// elements in a 16-byte piece
template <bool BF> struct Elems { static constexpr int E = BF ? 8 : 4; };

template <bool BF>
__device__ __forceinline__ void unpack(const u32x4& r, float (&x)[Elems<BF>::E]) {
    if constexpr (BF) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[2 * i] = bf16_lo(r[i]); x[2 * i + 1] = bf16_hi(r[i]); }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(r[i]);
    }
}
template <bool BF>
__device__ __forceinline__ u32x4 pack(const float (&x)[Elems<BF>::E]) {
    if constexpr (BF) return u32x4{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7])};
    else return u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
}

// ---- how many lanes a head takes (the team), and how many heads a wavefront takes together
// eight: teams of 8 for heads of at most 8 pieces (64 bf16).  The backward pass and several heads together take them; the
// forward pass of one head keeps 16 lanes: with 8 the entries of a short row are spread over eight slots whose eight loads
// stay mostly empty (200,000 rows of 3 entries, 64 bf16: 193 us, with teams of 8 237; 100,000 of 12: 112 and 131; from 30
// entries on teams of 8 are the faster ones, 1,000 rows of 60 13 and 11 us, but a call does not know its rows' lengths).
template <bool BF>
inline int gat_team(int32_t F, bool eight) {
    const int pieces = F / Elems<BF>::E;              // whole pieces, at most 64
    return BF && eight && pieces <= 8 ? 8 : (pieces <= 16 ? 16 : (pieces <= 32 ? 32 : 64));
}
// Powers of two: team numbers split by shifts.  95,000 nodes, 550,000 entries, four heads of 64 floats: 66 us, a
// launch per head 4 x 37 us.
template <bool BF>
inline int gat_heads_together(int32_t F, int32_t heads) {
    int H = 1;
    while (H < 4 && heads % (2 * H) == 0 && gat_team<BF>(F, false) * 2 * H <= 64) H *= 2;
    return H;
}

template <int G> __device__ __forceinline__ int team_lane(int v, int u);
// Value j of the eight that the lanes of a team hold as team_sum8_own leaves them; j a constant wherever this is called.
template <int G>
__device__ __forceinline__ float team_value8(float v, int j) {
    if constexpr (G <= 16) return __int_as_float(team_lane<G>(__float_as_int(v), j * (G / 8)));
    else return __shfl(v, (threadIdx.x & 63 & ~(G - 1)) + j * (G / 8));
}

// Lane u of every team of G lanes to the whole team, by data-parallel moves (row_newbcast: one lane of each 16; for teams
// of eight the two halves of a 16 take their own).  u is a constant wherever this is called.
template <int G>
__device__ __forceinline__ int team_lane(int v, int u) {
#define GAS_CASE(n)                                                                                     \
    case n:                                                                                             \
        if constexpr (G == 16) return __builtin_amdgcn_mov_dpp(v, 0x150 + (n), 0xf, 0xf, true);          \
        else return __builtin_amdgcn_update_dpp(__builtin_amdgcn_mov_dpp(v, 0x150 + (n), 0xf, 0x3, true), v, 0x150 + ((n) + 8) % 16, 0xf, 0xc, false);
    switch (u) {
        GAS_CASE(0) GAS_CASE(1) GAS_CASE(2) GAS_CASE(3) GAS_CASE(4) GAS_CASE(5) GAS_CASE(6) GAS_CASE(7)
        GAS_CASE(8) GAS_CASE(9) GAS_CASE(10) GAS_CASE(11) GAS_CASE(12) GAS_CASE(13) GAS_CASE(14) GAS_CASE(15)
    }
#undef GAS_CASE
    return v;
}

// Lane u of every 16 to the lower eight of them and lane u + 1 to the upper eight.  u is even and a constant wherever this is called.
__device__ __forceinline__ int pair_lane(int v, int u) {
#define GAS_CASE(n) \
    case n: return __builtin_amdgcn_update_dpp(__builtin_amdgcn_mov_dpp(v, 0x150 + (n), 0xf, 0x3, true), v, 0x151 + (n), 0xf, 0xc, false);
    switch (u) {
        GAS_CASE(0) GAS_CASE(2) GAS_CASE(4) GAS_CASE(6) GAS_CASE(8) GAS_CASE(10) GAS_CASE(12) GAS_CASE(14)
    }
#undef GAS_CASE
    return v;
}
// The value of the lane eight further in every 16, around its end (row_ror:8).
__device__ __forceinline__ float other_half(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));
}

}  // namespace gas
