// Products of fp32 operands on the bf16 matrix instructions.
//
// A float is the sum of three bf16 numbers: x = h + m + l with h the nearest bf16 to x, m the nearest to x - h and l
// to x - h - m (8 + 8 + 8 significant bits; both differences are exact).  A product is then taken as
//     a b = ah bh + (ah bm + am bh) + (am bm + ah bl + al bh),
// six v_mfma_f32_32x32x16_bf16 with fp32 accumulation; the three dropped terms are at most 2^-24 of |a b|, an fp32
// rounding of the product (|m| <= 2^-8, |l| <= 2^-17 beside h = 1; 2^-27 of it root mean square for normally
// distributed operands).  Six instructions of 32 cycles do what eight v_mfma_f32_32x32x2_f32 of 64 cycles do: 16 k of
// a 32 x 32 block.  A product that is all there is of its sum (K = 1) is taken by the fp32 instruction, which rounds it
// correctly; from two terms on the fewer roundings of the sum outweigh what is dropped (2.7e-8 against 3.2e-8).
//
// ah bh has an accumulator of its own and the five small terms share another, so the large one is rounded once per 16
// k: the relative error against 64 bits (2-norm, N(0,1) operands) is 9.0e-8 at K = 256 and 1.7e-7 at K = 832, with the
// fp32 instruction 2.9e-7 and 5.2e-7.  With one accumulator for all six it is 2.5e-7 and 4.5e-7, but the instruction's
// rounding has a bias that adds up: a weight gradient over 600,000 rows is 2.1e-6 off (fp32 instruction 8.7e-7, two
// accumulators 3.2e-7).  Sums that only grow, of absolute values, over the same rows: 5.9e-8 (fp32 instruction 7.3e-8).
//
// What bounds it: matrix pipe 52 %, vector instructions of the split 31 % of the cycles by the counters, the clock
// falls to 1.8 GHz under this load; 50,000 x 256 x 256 in 128 x 128 tiles take 59 us (87 us with the fp32 instruction),
// 600,000 rows 567 us (738); products of these sizes keep their weights in registers instead (46 and 454 us,
// linear_ws_split_kernel).  128 x 256 and 256 x 256 tiles split each value for more products but leave one workgroup per
// compute unit: 55-63 us; products and split interleaved by hand in one wavefront, two LDS buffers: 49-56 us (when the
// 128 x 128 tiles took 54).
//
// What the split cannot represent: an infinity, a NaN or a value that rounds to an infinite bf16 makes the accumulator
// non-finite (0 * inf in the terms beside it, if not itself), and a wavefront that finds one takes its block again with
// the fp32 instruction (plain_tile), so such inputs give what fp32 arithmetic gives.  The other end is not seen in the
// result: below 2^-110 the last bits of a value lie under bf16's smallest subnormal, 2^-133 (relative error 2.2e-6 for
// an operand of 2^-116 N(0,1), 5.6e-4 at 2^-124).  So the least non-zero magnitude is kept while staging, and a workgroup
// that met one below 2^-110 takes its tile again with both operands times 2^40: every fp32 number is then represented
// whole, and what leaves the range at the upper end is non-finite, as above.  The search costs one and a half
// instructions a value (4,000 x 256 x 256: 9.7 -> 10.3 us, 50,000 rows 53.7 -> 54.0 us); with such a value in every tile
// 50,000 rows take 92 us (the fp32 instruction 86 us), with one beyond 2^88 as well 211 us.
#pragma once
#include "common.h"

namespace gas {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));      // a 16-byte load at a float's alignment

constexpr float kUp = 0x1p40f;
constexpr uint32_t kLeast = 2 * ((127 - 110) << 23) - 1;      // 2 bits - 1 of 2^-110

// x0, x1 -> their three bf16 parts, packed in pairs
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = pack_bf16(x0, x1);
    const float r0 = x0 - bf16_lo(h), r1 = x1 - bf16_hi(h);
    m = pack_bf16(r0, r1);
    l = pack_bf16(r0 - bf16_lo(m), r1 - bf16_hi(m));
}

// One operand's tile of a workgroup of T threads: ROWS rows (output rows or columns) x 16 KS values of the reduced
// index q.  KC: element (r, q) lies at X[r ld + q] (q contiguous), else at X[q ld + r].  A thread holds pieces of
// eight consecutive q of one row and writes them to LDS as one 16-byte piece per part: [part][row][q], the pieces of a
// row exchanged so that the 16-byte reads of consecutive rows fall on different banks.
// KG groups of T threads each take a tile of their own; a thread's number in its group is `threadIdx.x` itself where there is one
// group (a remainder there changed the order of the kernel's instructions: 6,000 x 498 x 192 in 64 x 64 tiles 22.5 -> 23.3 us).
// IDX: the matrix's rows are those that idx names (KC: row r of the tile is row idx[r] of X; else q is row idx[q]).
template <int ROWS, int KS, bool KC, int T, int KG, bool IDX = false>
struct SplitTile {
    static constexpr int kQ = 16 * KS, kCh = 2 * KS, kPieces = ROWS * kCh;
    static constexpr int kPlane = ROWS * kQ;                              // bf16 elements
    static constexpr int NV = (kPieces + T - 1) / T;
    static_assert(KS == 1 || KS == 2, "two or four pieces a row");
    static_assert(KC || (T % ROWS == 0 && ROWS % 64 == 0), "a thread stays with one row, a wavefront with one piece index");
    const float* p[NV];        // KC: the thread's pieces; else the workgroup's first row, one scalar address for all ...
    uint32_t off;              // ... and the thread's row from there, in bytes: a load is scalar base + 32-bit offset
    float v[NV][8];
    int64_t ld;
    const int32_t* idx = nullptr;

    __device__ __forceinline__ int64_t named(int64_t row) const {
        if constexpr (!IDX) return row;
        else if constexpr (KC) return idx[row];
        else return __builtin_amdgcn_readfirstlane(idx[row]);      // a wavefront has one piece: one q
    }
    static __device__ __forceinline__ unsigned thread() { return KG == 1 ? threadIdx.x : threadIdx.x % T; }
    static __device__ __forceinline__ int row_of(int i) {
        const int idx = thread() + T * i;
        return KC ? idx / kCh : idx % ROWS;
    }
    static __device__ __forceinline__ int piece_of(int i) {
        // q contiguous: neighbouring threads take one row's pieces; else a wavefront has one piece index
        if constexpr (KC) return (thread() + T * i) % kCh;
        else return (__builtin_amdgcn_readfirstlane(thread() >> 6) * 64 + T * i) / ROWS;
    }
    static __device__ __forceinline__ bool holds(int i) { return kPieces % T == 0 || (int)thread() + T * i < kPieces; }
    // where piece `piece` of row `row` lies in a plane
    static __device__ __forceinline__ int at(int row, int piece) {
        return row * kQ + 8 * (KS == 2 ? (piece ^ ((row >> 1) & 3)) : (piece ^ ((row >> 2) & 1)));
    }

    // rows r0 .. r_end - 1; rows beyond take the last one's values, which nothing stores
    __device__ __forceinline__ void init(const float* X, int64_t ld_, int64_t r0, int64_t r_end) {
        ld = ld_;
        const int64_t last = r_end - 1 - r0;
        off = (uint32_t)(row_of(0) < last ? row_of(0) : last) * 4;             // not KC: T is a multiple of ROWS
#pragma unroll
        for (int i = 0; i < NV; ++i)
            p[i] = KC ? X + named(r0 + (row_of(i) < last ? row_of(i) : last)) * ld + 8 * piece_of(i) : X + r0;
    }
    __device__ __forceinline__ void fetch(int64_t q0) {                       // q0 .. q0 + kQ - 1
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (!holds(i)) continue;
            if constexpr (KC) {
                const f32x4 a = *reinterpret_cast<const f32x4_any*>(p[i] + q0);
                const f32x4 b = *reinterpret_cast<const f32x4_any*>(p[i] + q0 + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[i][e] = a[e]; v[i][4 + e] = b[e]; }
            } else if constexpr (IDX) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[i][e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p[i] + named(q0 + 8 * piece_of(i) + e) * ld) + off);
            } else {
                const char* u = reinterpret_cast<const char*>(p[i] + (q0 + 8 * piece_of(i)) * ld);
#pragma unroll
                for (int e = 0; e < 8; ++e, u += ld * 4) v[i][e] = *reinterpret_cast<const float*>(u + off);
            }
        }
    }
    // the same where the step reaches beyond q_end: values from there on repeat the last one until mask() clears them
    // (after the wait for the loads: a select beside each load would wait for each)
    __device__ __forceinline__ void fetch_last(int64_t q0, int64_t q_end) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (!holds(i)) continue;
            const int64_t q = q0 + 8 * piece_of(i);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t k = q + e < q_end ? q + e : q_end - 1;
                v[i][e] = KC ? p[i][k - 8 * piece_of(i)]
                             : *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p[i] + named(k) * ld) + off);
            }
        }
    }
    __device__ __forceinline__ void mask(int left) {             // left: values of the step inside
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] = 8 * piece_of(i) + e < left ? v[i][e] : 0.f;
    }
    // low: the least of 2 bits - 1 over the values staged, as an integer (zeros come out largest)
    template <bool SCALED>
    __device__ __forceinline__ void stage(uint16_t* planes, uint32_t& low) const {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (!holds(i)) continue;
            u32x4 h, m, l;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x0 = v[i][2 * e], x1 = v[i][2 * e + 1];
                if constexpr (SCALED) {
                    x0 *= kUp;
                    x1 *= kUp;
                } else {
                    const uint32_t t0 = 2 * __float_as_uint(x0) - 1, t1 = 2 * __float_as_uint(x1) - 1;
                    low = min(low, min(t0, t1));
                }
                uint32_t a, b, c;
                split_pair(x0, x1, a, b, c);
                h[e] = a; m[e] = b; l[e] = c;
            }
            uint16_t* to = planes + at(row_of(i), piece_of(i));
            *reinterpret_cast<u32x4*>(to) = h;
            *reinterpret_cast<u32x4*>(to + kPlane) = m;
            *reinterpret_cast<u32x4*>(to + 2 * kPlane) = l;
        }
    }
};

// A BM x BN tile of sum_q A(r, q) B(c, q), q_begin <= q < q_end (not empty), by WM x WN wavefronts; `lds` holds kLdsBytes.  acc: the wavefront's TM x TN blocks of 32 x 32, at rows wm0.. and columns wn0..
// of the tile.
template <int BM, int BN, int WM, int WN, int KS, bool AKC, bool BKC, int KG = 1, bool AIDX = false, bool BIDX = false>
struct SplitGemm {
    static constexpr int T = 64 * WM * WN, TM = BM / 32 / WM, TN = BN / 32 / WN;     // threads, 32 x 32 blocks of a wavefront
    using TA = SplitTile<BM, KS, AKC, T, KG, AIDX>;
    using TB = SplitTile<BN, KS, BKC, T, KG, BIDX>;
    static constexpr int kFlag = 3 * (TA::kPlane + TB::kPlane);              // where the flag lies, in bf16 elements
    static constexpr int kLdsBytes = kFlag * 2 + 16;
    TA ta;
    TB tb;

    static __device__ __forceinline__ void products(const uint16_t* lds, int wm0, int wn0, f32x16 (&acc)[TM][TN],
                                                    f32x16 (&small)[TM][TN]) {
        const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
        const uint16_t* B = lds + 3 * TA::kPlane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 fa[3][TM], fb[3][TN];
#pragma unroll
            for (int part = 0; part < 3; ++part) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[part][i] = *reinterpret_cast<const bf16x8*>(lds + part * TA::kPlane + TA::at(wm0 + 32 * i + li, 2 * ks + lh));
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[part][j] = *reinterpret_cast<const bf16x8*>(B + part * TB::kPlane + TB::at(wn0 + 32 * j + li, 2 * ks + lh));
            }
            constexpr int PA[6] = {0, 1, 0, 1, 2, 0}, PB[6] = {0, 0, 1, 1, 0, 2};
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        f32x16& c = t == 0 ? acc[i][j] : small[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[t]][i], fb[PB[t]][j], c, 0, 0, 0);
                    }
        }
    }

    // acc = the products of the operands as they are, or of both times kUp (the products divided by its square at the end)
    template <bool SCALED>
    __device__ __forceinline__ void pass(const float* A, int64_t lda, int64_t a0, int64_t a_end, const float* B, int64_t ldb,
                                         int64_t b0, int64_t b_end, int64_t q_begin, int64_t q_end, uint16_t* lds, int wm0,
                                         int wn0, f32x16 (&acc)[TM][TN]) {
        ta.init(A, lda, a0, a_end);
        tb.init(B, ldb, b0, b_end);
        if (q_begin + TA::kQ <= q_end) {
            ta.fetch(q_begin);
            tb.fetch(q_begin);
        } else {
            ta.fetch_last(q_begin, q_end);
            tb.fetch_last(q_begin, q_end);
        }
        f32x16 small[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = small[i][j][r] = 0.f;
        uint32_t low = 0xFFFFFFFFu;
        auto stage = [&](bool last) {        // last: no whole step follows
            __syncthreads();                 // everyone is done reading the previous step
            ta.template stage<SCALED>(lds, low);
            tb.template stage<SCALED>(lds + 3 * TA::kPlane, low);
            if (!SCALED && last && low < kLeast) *reinterpret_cast<uint32_t*>(lds + kFlag) = 1;
            __syncthreads();
        };
        auto multiply = [&]() {
            __builtin_amdgcn_s_setprio(1);   // the matrix pipe first: the other workgroup splits meanwhile
            products(lds, wm0, wn0, acc, small);
            __builtin_amdgcn_s_setprio(0);
        };
        int64_t q = q_begin;
        for (; q + 2 * TA::kQ <= q_end; q += TA::kQ) {
            stage(false);
            ta.fetch(q + TA::kQ);
            tb.fetch(q + TA::kQ);
            multiply();
        }
        if (q + TA::kQ <= q_end) {           // the last whole step
            stage(true);
            if (q + TA::kQ < q_end) {
                ta.fetch_last(q + TA::kQ, q_end);
                tb.fetch_last(q + TA::kQ, q_end);
            }
            multiply();
            q += TA::kQ;
        }
        if (q < q_end) {                     // a step that is not whole
            ta.mask((int)(q_end - q));
            tb.mask((int)(q_end - q));
            stage(true);
            multiply();
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[i][j][r] += small[i][j][r];
                    if constexpr (SCALED) acc[i][j][r] *= 1.f / (kUp * kUp);
                }
    }

    // The same by KG groups of T threads, each with LDS of its own: group `group` takes every KG-th step, and group 0 ends up with
    // the sum over the groups, added pair by pair (the other groups' acc is of no use afterwards).
    template <bool SCALED>
    __device__ __forceinline__ void pass_groups(const float* A, int64_t lda, int64_t a0, int64_t a_end, const float* B, int64_t ldb,
                                                int64_t b0, int64_t b_end, int64_t q_end, uint16_t* lds, uint32_t* flag, int group,
                                                int wm0, int wn0, f32x16 (&acc)[TM][TN]) {
        uint16_t* mine = lds + group * kFlag;
        ta.init(A, lda, a0, a_end);
        tb.init(B, ldb, b0, b_end);
        auto fetch = [&](int64_t q) {
            if (q + TA::kQ <= q_end) {
                ta.fetch(q);
                tb.fetch(q);
            } else if (q < q_end) {
                ta.fetch_last(q, q_end);
                tb.fetch_last(q, q_end);
            }
        };
        int64_t q = (int64_t)group * TA::kQ;
        fetch(q);
        f32x16 small[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = small[i][j][r] = 0.f;
        uint32_t low = 0xFFFFFFFFu;
        const int64_t rounds = (q_end + KG * TA::kQ - 1) / (KG * TA::kQ);       // the same for every group: they share the barriers
#pragma unroll 1
        for (int64_t r = 0; r < rounds; ++r, q += KG * TA::kQ) {
            const bool on = q < q_end;
            __syncthreads();                     // everyone is done reading the previous step
            if (on) {
                if (q + TA::kQ > q_end) {
                    ta.mask((int)(q_end - q));
                    tb.mask((int)(q_end - q));
                }
                ta.template stage<SCALED>(mine, low);
                tb.template stage<SCALED>(mine + 3 * TA::kPlane, low);
            }
            if (!SCALED && r + 1 == rounds && low < kLeast) *flag = 1;
            __syncthreads();
            if (on) {
                fetch(q + KG * TA::kQ);
                products(mine, wm0, wn0, acc, small);
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] += small[i][j][r];
        // the groups' sums through LDS: [group - 1][block][thread][16], four floats an access
        constexpr int kBlocks = TM * TN;
        static_assert((KG - 1) * kBlocks * T * 16 * 4 <= KG * kFlag * 2, "the sums fit where the operands were");
        float* sums = reinterpret_cast<float*>(lds);
        const int t = threadIdx.x % T;
        __syncthreads();
        if (group > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<f32x4*>(sums + ((((group - 1) * kBlocks + i * TN + j) * 4 + r) * T + t) * 4) =
                            f32x4{acc[i][j][4 * r], acc[i][j][4 * r + 1], acc[i][j][4 * r + 2], acc[i][j][4 * r + 3]};
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        f32x4 part[KG];
                        part[0] = f32x4{acc[i][j][4 * r], acc[i][j][4 * r + 1], acc[i][j][4 * r + 2], acc[i][j][4 * r + 3]};
#pragma unroll
                        for (int g = 1; g < KG; ++g)
                            part[g] = *reinterpret_cast<const f32x4*>(sums + ((((g - 1) * kBlocks + i * TN + j) * 4 + r) * T + t) * 4);
#pragma unroll
                        for (int d = 1; d < KG; d *= 2)           // pair by pair: in a row they lost what shorter sums gain
#pragma unroll
                            for (int g = 0; g + d < KG; g += 2 * d) part[g] += part[g + d];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][j][4 * r + e] = part[0][e];
                    }
            if constexpr (SCALED) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] *= 1.f / (kUp * kUp);
            }
        }
    }

    // run() by KG groups; q from 0.  For group 0 as run(), the others take part and return true with nothing in acc.
    static constexpr int kGroupsLdsBytes = KG * kFlag * 2 + 16;
    __device__ __forceinline__ bool run_groups(const float* A, int64_t lda, int64_t a0, int64_t a_end, const float* B, int64_t ldb,
                                               int64_t b0, int64_t b_end, int64_t q_end, uint16_t* lds, int group, int wm0, int wn0,
                                               f32x16 (&acc)[TM][TN]) {
        uint32_t* flag = reinterpret_cast<uint32_t*>(lds + KG * kFlag);
        if (threadIdx.x == 0) *flag = 0;         // before the first barrier of the pass, which sets it between its last two steps'
        pass_groups<false>(A, lda, a0, a_end, B, ldb, b0, b_end, q_end, lds, flag, group, wm0, wn0, acc);
        if (__builtin_amdgcn_readfirstlane(*flag)) {
            __syncthreads();                     // group 0 is done reading the sums
            pass_groups<true>(A, lda, a0, a_end, B, ldb, b0, b_end, q_end, lds, flag, group, wm0, wn0, acc);
        }
        if (group > 0) return true;
        float bad = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) bad = fmaf(acc[i][j][r], 0.f, bad);
        return !__any(bad != 0.f);
    }

    // acc = the products; whether they stand (not if a value of the wavefront's blocks is not finite): else plain_tile
    __device__ __forceinline__ bool run(const float* A, int64_t lda, int64_t a0, int64_t a_end, const float* B, int64_t ldb,
                                        int64_t b0, int64_t b_end, int64_t q_begin, int64_t q_end, uint16_t* lds, int wm0,
                                        int wn0, f32x16 (&acc)[TM][TN]) {
        if (q_end - q_begin == 1) return false;      // sums of one term: the dropped parts would be all of their error
        uint32_t* flag = reinterpret_cast<uint32_t*>(lds + kFlag);
        if (threadIdx.x == 0) *flag = 0;     // before the first barrier of the pass, which sets it between its last two
        pass<false>(A, lda, a0, a_end, B, ldb, b0, b_end, q_begin, q_end, lds, wm0, wn0, acc);
        if (__builtin_amdgcn_readfirstlane(*flag))
            pass<true>(A, lda, a0, a_end, B, ldb, b0, b_end, q_begin, q_end, lds, wm0, wn0, acc);
        float bad = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) bad = fmaf(acc[i][j][r], 0.f, bad);      // stays 0 for finite values, else NaN
        return !__any(bad != 0.f);
    }
};

// The wavefront's block by the fp32 instruction, straight from memory: rows a_r0.. of A and b_r0.. of B (clamped to
// the last), q0 <= q < q_end.
template <int TM, int TN, bool AKC, bool BKC, bool AIDX = false, bool BIDX = false>
__device__ __forceinline__ void plain_tile(const float* A, int64_t lda, int64_t a_r0, int64_t a_end, const float* B,
                                        int64_t ldb, int64_t b_r0, int64_t b_end, int64_t q0, int64_t q_end,
                                        f32x16 (&acc)[TM][TN], const int32_t* idx = nullptr) {
    auto row_a = [&](int64_t r) { return AIDX ? (int64_t)idx[r] : r; };
    auto row_b = [&](int64_t r) { return BIDX ? (int64_t)idx[r] : r; };
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll 1
    for (int64_t q = q0; q < q_end; q += 2) {                // lanes 0-31 take q, lanes 32-63 q + 1
        const bool in = q + lh < q_end;
        const int64_t qq = in ? q + lh : q;
        float fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int64_t r = a_r0 + 32 * i + li;
            r = r < a_end ? r : a_end - 1;
            fa[i] = AKC ? A[row_a(r) * lda + qq] : A[row_a(qq) * lda + r];
            fa[i] = in ? fa[i] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int64_t r = b_r0 + 32 * j + li;
            r = r < b_end ? r : b_end - 1;
            fb[j] = BKC ? B[row_b(r) * ldb + qq] : B[row_b(qq) * ldb + r];
            fb[j] = in ? fb[j] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
}

}  // namespace
}  // namespace gas
