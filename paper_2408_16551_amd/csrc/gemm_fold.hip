// The dense DFT of Eq. (12) as four quarter-size products on the MFMA units,
// using the symmetry of the Fourier matrix (the operand rows come folded from
// the FIR, fir_fold.h).  With Q = P/4, q = p + 1/2 and j < Q:
//   part 0: C_k = sum_p part0[p] cos(2 pi k q / P), k = 2j
//   part 1: S_k = sum_p part1[p] sin(2 pi k q / P), k = 2j (j > 0), P/2 (j = 0)
//   part 2: C_k, part 3: S_k, k = 2j + 1
//   X_k = exp(i pi k / P) (C_k - i S_k);  complex frames also
//   X_{P-k} = exp(-i pi k / P) (C_k + i S_k), C and S complex.
// P^2/2 (real) or P^2 (complex) flops a frame instead of 2 P^2 or 8 P^2, and an
// operand of P^2/4 entries instead of P^2 or 4 P^2.  Where fold_split says so,
// complex frames arrive in two halves of P/2 (even and odd channels) and take the
// product of size P/2 twice: half the flops again, a quarter of the operand.
//
// As a matrix product: rows r = frame * cf + (re/im), inner index (part, p) of
// length P on both sides, columns j; the accumulator set changes with the
// part, so a tile holds all four results of its (row, j) and its epilogue
// forms whole channels: X_2j, X_2j+1 leave in one 16-byte store, 512
// contiguous bytes per half wave.
#include "internal.h"

#include <type_traits>

namespace tina {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float fvec2 __attribute__((ext_vector_type(2)));
typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));  // channel pairs lie on 8 bytes

// EB: bytes per element; NP: pieces.
template <int FORM> struct FF;
template <> struct FF<FORM_FP32> { static constexpr int EB = 4, NP = 1; };
template <> struct FF<FORM_BF16> { static constexpr int EB = 2, NP = 1; };
template <> struct FF<FORM_BF16X3> { static constexpr int EB = 2, NP = 2; };

// What the rows are: real frames; complex ones, as real and imaginary row; complex
// ones in two halves (one decimation in frequency, fir_fold.h), as four rows.
enum Mode : int { REAL = 0, CPLX = 1, SPLIT = 2 };
template <int MODE> constexpr int kRows = MODE == REAL ? 1 : MODE == CPLX ? 2 : 4;

constexpr int SLAB = 32;      // bytes of a row per MFMA step (8 FP32 or 16 bf16 of K)
constexpr int GROUP_M = 8;    // m-tiles swept per column of j-tiles (4096 complex, BF16: 439 us; 470, 463, 532 at 4, 16, 32)

// FP32 sums every K tile of 32 products by itself and adds the tile sums: C and
// S of a strong channel are as large as the channel, and what their running
// sums lose is left over in the mirrored channel, where C + iS cancels (60 dB
// mix of 4096 channels: worst noise channel 0.175 with one running sum of 1024
// products).
template <int FORM> constexpr bool kTileSums = FORM == FORM_FP32;

template <int TM>
__device__ __forceinline__ void zero(f32x16 (&a)[TM]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) a[i][v] = 0.f;
}
template <int TM>
__device__ __forceinline__ void add_to(f32x16 (&a)[TM], const f32x16 (&b)[TM]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) a[i][v] += b[i][v];
}

// Products of one slab into the accumulators of one part.
template <int FORM, int NP, int TM>
__device__ __forceinline__ void fold_mfma(const uint4 (&af)[TM][NP], const uint4 (&bf)[NP], f32x16 (&acc)[TM]) {
    if constexpr (FORM == FORM_FP32) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int bm = 0; bm < TM; ++bm)
                acc[bm] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, af[bm][0])[e],
                                                               __builtin_bit_cast(f32x4, bf[0])[e], acc[bm], 0, 0, 0);
    } else {
        // hi*hi, then hi*lo and lo*hi for the split form.
#pragma unroll
        for (int term = 0; term < (NP == 2 ? 3 : 1); ++term)
#pragma unroll
            for (int bm = 0; bm < TM; ++bm)
                acc[bm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, af[bm][term == 2 ? 1 : 0]),
                    __builtin_bit_cast(bf16x8, bf[term == 1 ? 1 : 0]), acc[bm], 0, 0, 0);
    }
}

// Writes the channels of one (frame, j): c0 s0 c1 s1 = C, S of k = 2j and of
// 2j + 1 (real frames), w = cos, sin of pi 2j/P and of pi (2j+1)/P.
__device__ __forceinline__ void put16(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<f32x4_a8*>(p) = f32x4_a8{a, b, c, d};
}
// a b + c d, in an order of operations that the compiler cannot choose anew in
// every kernel: all of them give the same bits.
__device__ __forceinline__ float mul2(float a, float b, float c, float d) { return fmaf(a, b, c * d); }
__device__ __forceinline__ void fold_out_real(float* row, int P, int j, const float4& w, float c0, float s0, float c1,
                                              float s1) {
    const float x1r = mul2(w.z, c1, w.w, s1), x1i = mul2(w.w, c1, -w.z, s1);
    if (j == 0) {  // X_0 = C_0 and X_{P/2} = S_{P/2}, both real
        put16(row, c0, 0.0f, x1r, x1i);
        *reinterpret_cast<fvec2*>(row + P) = fvec2{s0, 0.0f};
    } else {
        put16(row + 4 * j, mul2(w.x, c0, w.y, s0), mul2(w.y, c0, -w.x, s0), x1r, x1i);
    }
}
// Complex frames: index 0 = real row, 1 = imaginary row.
// inv != 0: the inverse DFT, the same values times inv = 1/P in the order of
// -k (w already holds the factor, a power of two).
__device__ __forceinline__ void fold_out_cplx(float* row, int P, int j, const float4& w, float inv, const float (&c0)[2],
                                              const float (&s0)[2], const float (&c1)[2], const float (&s1)[2]) {
    const float ur = c1[0] + s1[1], ui = c1[1] - s1[0];  // C - iS
    const float vr = c1[0] - s1[1], vi = c1[1] + s1[0];  // C + iS
    const float x1r = mul2(w.z, ur, -w.w, ui), x1i = mul2(w.w, ur, w.z, ui);
    const float y1r = mul2(w.z, vr, w.w, vi), y1i = mul2(w.z, vi, -w.w, vr);
    if (j == 0) {  // X_0 = C_0, X_{P/2} = S_{P/2}
        const float sc = inv != 0.0f ? inv : 1.0f;
        put16(row, sc * c0[0], sc * c0[1], inv != 0.0f ? y1r : x1r, inv != 0.0f ? y1i : x1i);
        *reinterpret_cast<fvec2*>(row + P) = fvec2{sc * s0[0], sc * s0[1]};
        *reinterpret_cast<fvec2*>(row + 2 * (P - 1)) = inv != 0.0f ? fvec2{x1r, x1i} : fvec2{y1r, y1i};
    } else {
        const float pr = c0[0] + s0[1], pi = c0[1] - s0[0], mr = c0[0] - s0[1], mi = c0[1] + s0[0];
        const float x0r = mul2(w.x, pr, -w.y, pi), x0i = mul2(w.y, pr, w.x, pi);
        const float y0r = mul2(w.x, mr, w.y, mi), y0i = mul2(w.x, mi, -w.y, mr);
        float *up = row + 4 * j, *down = row + 2 * (P - 1 - 2 * j);
        if (inv != 0.0f) {
            put16(up, y0r, y0i, y1r, y1i);
            put16(down, x1r, x1i, x0r, x0i);
        } else {
            put16(up, x0r, x0i, x1r, x1i);
            put16(down, y1r, y1i, y0r, y0i);
        }
    }
}

// The channels of one j of a split frame of P channels (halves t of P/2: channel
// 2k + t is the half's channel k): C, S of the half's channels 2j and 2j + 1 as
// complex numbers, w as above for P/2.  Each store is the two halves' channels,
// 16 bytes, and a lane's four stores are two runs of 32.
struct Quad {
    float c0[2], s0[2], c1[2], s1[2];
};
struct HalfOut {
    float e[2], em[2], o[2], om[2];  // the half's channels 2j, P/2 - 2j, 2j + 1, P/2 - 2j - 1
};
__device__ __forceinline__ HalfOut fold_half(const Quad& q, const float4& w) {
    HalfOut r;
    const float ur = q.c1[0] + q.s1[1], ui = q.c1[1] - q.s1[0], vr = q.c1[0] - q.s1[1], vi = q.c1[1] + q.s1[0];
    r.o[0] = mul2(w.z, ur, -w.w, ui);
    r.o[1] = mul2(w.w, ur, w.z, ui);
    r.om[0] = mul2(w.z, vr, w.w, vi);
    r.om[1] = mul2(w.z, vi, -w.w, vr);
    const float pr = q.c0[0] + q.s0[1], pi = q.c0[1] - q.s0[0], mr = q.c0[0] - q.s0[1], mi = q.c0[1] + q.s0[0];
    r.e[0] = mul2(w.x, pr, -w.y, pi);
    r.e[1] = mul2(w.y, pr, w.x, pi);
    r.em[0] = mul2(w.x, mr, w.y, mi);
    r.em[1] = mul2(w.x, mi, -w.y, mr);
    return r;
}
__device__ __forceinline__ void fold_out_split(float* row, int P, int j, const float4& w, float inv, const Quad& t0,
                                               const Quad& t1) {
    const HalfOut a = fold_half(t0, w), b = fold_half(t1, w);
    if (inv == 0.0f) {
        put16(row + 2 * (4 * j + 2), a.o[0], a.o[1], b.o[0], b.o[1]);
        put16(row + 2 * (P - 4 * j - 2), a.om[0], a.om[1], b.om[0], b.om[1]);
        if (j == 0) {  // k = 0 is C_0; in its mirror's place, S of k = P/4
            put16(row, t0.c0[0], t0.c0[1], t1.c0[0], t1.c0[1]);
            put16(row + P, t0.s0[0], t0.s0[1], t1.s0[0], t1.s0[1]);
        } else {
            put16(row + 8 * j, a.e[0], a.e[1], b.e[0], b.e[1]);
            put16(row + 2 * (P - 4 * j), a.em[0], a.em[1], b.em[0], b.em[1]);
        }
    } else {  // channel n to place P - n, times inv
        put16(row + 2 * (P - 4 * j - 3), b.o[0], b.o[1], a.o[0], a.o[1]);
        put16(row + 2 * (4 * j + 1), b.om[0], b.om[1], a.om[0], a.om[1]);
        if (j == 0) {
            *reinterpret_cast<fvec2*>(row) = fvec2{inv * t0.c0[0], inv * t0.c0[1]};
            *reinterpret_cast<fvec2*>(row + 2 * (P - 1)) = fvec2{inv * t1.c0[0], inv * t1.c0[1]};
            put16(row + 2 * (P / 2 - 1), inv * t1.s0[0], inv * t1.s0[1], inv * t0.s0[0], inv * t0.s0[1]);
        } else {
            put16(row + 2 * (P - 4 * j - 1), b.e[0], b.e[1], a.e[0], a.e[1]);
            put16(row + 2 * (4 * j - 1), b.em[0], b.em[1], a.em[0], a.em[1]);
        }
    }
}

// Entry of the folded operand from the table ct[r] = cos(pi r / P), r < 2P:
// part s, column j, sample p: the angle pi k (2p+1) / P, a sine as the cosine
// P/2 steps earlier.
__device__ __forceinline__ int fold_k(int s, int j, int P) { return s == 1 && j == 0 ? P / 2 : 2 * j + (s >> 1); }
__device__ __forceinline__ int fold_index(int k, int p, bool sine, int P) {
    return (k * (2 * p + 1) + (sine ? 3 * (P / 2) : 0)) & (2 * P - 1);
}

// A block of WGM x WGN waves, each 64 rows x 32 columns of all four parts (128
// accumulators).  FP32: 128 x 64, 256 threads, two blocks a CU (128 x 128 took
// the same time).  16-bit forms: 128 x 128, one block a CU, or 256 x 64 for the
// 64 columns of 256 channels.  Their LDS reads are the bound (three 16-byte
// reads per two products), so long K tiles, few barriers and fewer operand
// bytes from L2 count: 545 / 1212 us for BF16 / BF16x3 at 4096 complex channels
// with the FP32 tile, 439 / 895 us with this one; a second K tile of loads in
// flight made no difference.
// ROWB: bytes of a row per K tile and piece; 128 where two stages fit the LDS.
template <int FORM, int WGM, int WGN>
struct FoldTile {
    static constexpr int NP = FF<FORM>::NP, EB = FF<FORM>::EB;
    static constexpr int BMR = 64 * WGM, BJ = 32 * WGN, NTH = 64 * WGM * WGN;
    static constexpr int ROWB = 2 * NP * (BMR + BJ) * 144 <= 160 * 1024 ? 128 : 64;
    static_assert(2 * NP * (BMR + BJ) * (ROWB + 16) <= 160 * 1024, "two stages fit the LDS");
    static constexpr int RS = ROWB + 16, CPR = ROWB / 16, NSLAB = ROWB / SLAB;
    static constexpr int QCH = BMR * CPR / NTH, BCH = (BJ * CPR + NTH - 1) / NTH;  // chunks per thread and piece
    static constexpr int STAGE = NP * (BMR + BJ) * RS;
    static_assert(BMR * CPR % NTH == 0, "whole chunks per thread");
};

// One tile (rows m0.., columns n0..), called by every thread of the block.
// lds: two stages of K tiles.  TABLE: the B rows are assembled from ct.
template <int FORM, int MODE, int WGM, int WGN, bool TABLE>
__device__ __forceinline__ void fold_tile(const GemmArgs& g, int64_t m0, int64_t n0, uint8_t* lds, const float* ct) {
    constexpr bool IM = MODE != REAL;  // rows in (real, imaginary) pairs
    using G = FoldTile<FORM, WGM, WGN>;
    constexpr int NP = G::NP, RS = G::RS, CPR = G::CPR, NTH = G::NTH, BMR = G::BMR, BJ = G::BJ;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN, lr = lane & 31, lh = lane >> 5;
    const int P = g.K, Q = g.N, lq = 31 - __clz(Q);  // inner length, columns (a power of two)
    const int64_t R = g.F * kRows<MODE>;
    const int64_t pitch = (int64_t)P * G::EB;      // bytes per operand row
    const uint8_t* Ap[2] = {FORM == FORM_FP32 ? (const uint8_t*)g.A : g.Aq, g.Aq1};
    const uint8_t* Bp[2] = {(const uint8_t*)g.B0, (const uint8_t*)g.B1};
    __amdgpu_buffer_rsrc_t ra[NP], rb[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int64_t ar = R - m0 < BMR ? R - m0 : BMR, br = Q - n0 < BJ ? Q - n0 : BJ;
        ra[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(Ap[p] + m0 * pitch), (short)0, (int)(ar * pitch), 0x00020000);
        rb[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(Bp[p] + n0 * pitch), (short)0, (int)(br * pitch), 0x00020000);
    }
    struct Stage {
        uint4 a[NP][G::QCH];
        uint4 b[NP][G::BCH];
    };
    auto load = [&](Stage& r, int st) {
        const int32_t kb = st * G::ROWB;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int i = 0; i < G::QCH; ++i) {
                const int c = tid + i * NTH;
                r.a[p][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          ra[p], (uint32_t)((c / CPR) * pitch + (c % CPR) * 16), kb, 0));
            }
#pragma unroll
            for (int i = 0; i < G::BCH; ++i) {
                const int c = tid + i * NTH;
                if constexpr (TABLE) {
                    const int el = (kb >> 2) + (c % CPR) * 4, s = el >> lq, p0 = el & (Q - 1);
                    const int k = fold_k(s, (int)n0 + c / CPR, P), r0 = fold_index(k, p0, s & 1, P), m = 2 * P - 1;
                    r.b[p][i] = __builtin_bit_cast(uint4, make_float4(ct[r0], ct[(r0 + 2 * k) & m], ct[(r0 + 4 * k) & m],
                                                                      ct[(r0 + 6 * k) & m]));
                } else {
                    r.b[p][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                              rb[p], (uint32_t)((c / CPR) * pitch + (c % CPR) * 16), kb, 0));
                }
            }
        }
    };
    auto store = [&](const Stage& r, int buf) {
        uint8_t* As = lds + buf * G::STAGE;
        uint8_t* Bs = As + NP * BMR * RS;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int i = 0; i < G::QCH; ++i) {
                const int c = tid + i * NTH;
                int row = c / CPR;
                // Complex frames: a wave's 64 rows as 32 real, then 32 imaginary.
                if (IM) row = (row & ~63) | ((row & 1) << 5) | ((row >> 1) & 31);
                *reinterpret_cast<uint4*>(As + p * BMR * RS + row * RS + (c % CPR) * 16) = r.a[p][i];
            }
#pragma unroll
            for (int i = 0; i < G::BCH; ++i) {
                const int c = tid + i * NTH;  // past the tile's rows: loaded as zeros, not stored
                if (BJ * CPR % NTH == 0 || c < BJ * CPR)
                    *reinterpret_cast<uint4*>(Bs + p * BJ * RS + (c / CPR) * RS + (c % CPR) * 16) = r.b[p][i];
            }
        }
    };
    f32x16 acc[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) zero(acc[s]);
    auto compute = [&](int buf, f32x16 (&ac)[2]) {
        const uint8_t* As = lds + buf * G::STAGE;
        const uint8_t* Bs = As + NP * BMR * RS;
#pragma unroll
        for (int sl = 0; sl < G::NSLAB; ++sl) {
            uint4 af[2][NP], bf[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
#pragma unroll
                for (int bm = 0; bm < 2; ++bm)
                    af[bm][p] = *reinterpret_cast<const uint4*>(As + p * BMR * RS + (wm * 64 + bm * 32 + lr) * RS + sl * SLAB + lh * 16);
                bf[p] = *reinterpret_cast<const uint4*>(Bs + p * BJ * RS + (wn * 32 + lr) * RS + sl * SLAB + lh * 16);
            }
            fold_mfma<FORM, NP, 2>(af, bf, ac);
        }
    };

    // Step st multiplies K tile st (part st / nk) from LDS buffer st & 1 while
    // the registers hold tile st + 1; that is then stored to the other buffer
    // and the loads of tile st + 2 are issued.
    const int nk = Q * G::EB / G::ROWB, nst = 4 * nk;
    Stage r;
    load(r, 0);
    __syncthreads();  // the table (and, in a batch, the previous use of LDS) is done
    store(r, 0);
    load(r, 1);
    __syncthreads();
    auto part = [&](int s, f32x16 (&ac)[2]) {
        for (int t = 0; t < nk; ++t) {
            const int st = s * nk + t;
            if constexpr (kTileSums<FORM>) {
                f32x16 ts[2];
                zero(ts);
                compute(st & 1, ts);
                add_to(ac, ts);
            } else {
                compute(st & 1, ac);
            }
            if (st + 1 < nst) store(r, (st + 1) & 1);
            if (st + 2 < nst) load(r, st + 2);
            __syncthreads();
        }
    };
    part(0, acc[0]);
    part(1, acc[1]);
    part(2, acc[2]);
    part(3, acc[3]);

    // Element v of a block: row 8 (v >> 2) + 4 lh + (v & 3), column lr.
    const int j = (int)n0 + wn * 32 + lr;
    if (j >= Q) return;
    const float4 w = reinterpret_cast<const float4*>(g.tw)[j];
    const int64_t fr0 = (m0 + wm * 64) / (IM ? 2 : 1);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int rr = 8 * (v >> 2) + 4 * lh + (v & 3);
        if constexpr (MODE == SPLIT) {
            const int64_t f = (fr0 + rr) / 2;  // rows rr and rr + 1: the frame's halves
            if ((v & 1) == 0 && f < g.F) {
                const Quad t0{{acc[0][0][v], acc[0][1][v]}, {acc[1][0][v], acc[1][1][v]}, {acc[2][0][v], acc[2][1][v]}, {acc[3][0][v], acc[3][1][v]}};
                const Quad t1{{acc[0][0][v + 1], acc[0][1][v + 1]}, {acc[1][0][v + 1], acc[1][1][v + 1]},
                              {acc[2][0][v + 1], acc[2][1][v + 1]}, {acc[3][0][v + 1], acc[3][1][v + 1]}};
                fold_out_split(g.out + f * g.ldo, 2 * P, j, w, g.inv, t0, t1);
            }
        } else if constexpr (IM) {
            const int64_t f = fr0 + rr;
            if (f < g.F) {
                const float c0[2] = {acc[0][0][v], acc[0][1][v]}, s0[2] = {acc[1][0][v], acc[1][1][v]};
                const float c1[2] = {acc[2][0][v], acc[2][1][v]}, s1[2] = {acc[3][0][v], acc[3][1][v]};
                fold_out_cplx(g.out + f * g.ldo, P, j, w, g.inv, c0, s0, c1, s1);
            }
        } else {
#pragma unroll
            for (int bm = 0; bm < 2; ++bm) {
                const int64_t f = fr0 + bm * 32 + rr;
                if (f < g.F)
                    fold_out_real(g.out + f * g.ldo, P, j, w, acc[0][bm][v], acc[1][bm][v], acc[2][bm][v], acc[3][bm][v]);
            }
        }
    }
}

// Few rows: blocks of 32 TM rows x 32 columns (complex frames: TM = 2), one wave
// per part, so that a short call still spreads over the chip (a
// wave of the large tile does four to eight times as much).  Operand rows go
// from memory straight to the MFMA registers, U slabs ahead: what bounds a short
// call is how often it waits for memory.  The four parts meet in LDS.  Same K
// order, same bits as fold_tile.
template <int FORM, int MODE, int TM>
__device__ __forceinline__ void fold_tile_small(const GemmArgs& g, int64_t m0, int64_t n0, float* ex) {
    constexpr bool IM = MODE != REAL;  // rows in (real, imaginary) pairs
    constexpr int NP = FF<FORM>::NP, EB = FF<FORM>::EB, ROWS = 32 * TM;
    constexpr int U = TM == 1 && NP == 1 ? 8 : 4;  // (with two row blocks the registers cost more waves than 8 gain)
    const int lane = threadIdx.x & 63, s = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
    const int P = g.K, Q = g.N;
    const int64_t R = g.F * kRows<MODE>, pitch = (int64_t)P * EB;
    const uint8_t* Ap[2] = {FORM == FORM_FP32 ? (const uint8_t*)g.A : g.Aq, g.Aq1};
    const uint8_t* Bp[2] = {(const uint8_t*)g.B0, (const uint8_t*)g.B1};
    const int part0 = s * Q * EB + lh * 16;
    int64_t ao[TM];
#pragma unroll
    for (int bm = 0; bm < TM; ++bm) {
        const int64_t row = m0 + (IM ? 2 * lr + bm : 32 * bm + lr);
        ao[bm] = (row < R ? row : R - 1) * pitch + part0;  // rows past the end: read, never written
    }
    const int64_t bo = (n0 + lr) * pitch + part0;  // Q is a multiple of 32
    f32x16 acc[TM], ts[TM];
    zero(acc);
    const int ns = Q * EB / SLAB;  // 4 or a multiple of U
    uint4 a[U][TM][NP], b[U][NP];
    auto load = [&](int u, int sl) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int bm = 0; bm < TM; ++bm) a[u][bm][p] = *reinterpret_cast<const uint4*>(Ap[p] + ao[bm] + sl * SLAB);
            b[u][p] = *reinterpret_cast<const uint4*>(Bp[p] + bo + sl * SLAB);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, U <= 4 || u < ns ? u : 0);
    for (int sl = 0; sl < ns; sl += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (U > 4 && sl + u >= ns) break;  // 4 slabs in all
            if constexpr (kTileSums<FORM>) {  // the K tiles of fold_tile: 4 slabs
                if (u % 4 == 0) zero(ts);
                fold_mfma<FORM, NP, TM>(a[u], b[u], ts);
                if (u % 4 == 3) add_to(acc, ts);
            } else {
                fold_mfma<FORM, NP, TM>(a[u], b[u], acc);
            }
            load(u, sl + U + (U > 4 ? u : 0) < ns ? sl + U + u : u & 3);  // past the last: repeats in-range reads
        }
    }
    // ex[part][row][column], 33 floats a row.
#pragma unroll
    for (int bm = 0; bm < TM; ++bm)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            ex[(s * ROWS + bm * 32 + 8 * (v >> 2) + 4 * lh + (v & 3)) * 33 + lr] = acc[bm][v];
    __syncthreads();
    const int jl = threadIdx.x & 31, j = (int)n0 + jl;
    const float4 w = reinterpret_cast<const float4*>(g.tw)[j];
    auto at = [&](int part, int row) { return ex[(part * ROWS + row) * 33 + jl]; };
    for (int i = threadIdx.x >> 5; i < (MODE == SPLIT ? 16 : IM ? 32 : ROWS); i += 8) {
        const int64_t f = m0 / kRows<MODE> + i;
        if (f >= g.F) break;
        float* row = g.out + f * g.ldo;
        if constexpr (MODE == SPLIT) {
            const int a = 2 * i, b = a + 1;
            const Quad t0{{at(0, a), at(0, 32 + a)}, {at(1, a), at(1, 32 + a)}, {at(2, a), at(2, 32 + a)}, {at(3, a), at(3, 32 + a)}};
            const Quad t1{{at(0, b), at(0, 32 + b)}, {at(1, b), at(1, 32 + b)}, {at(2, b), at(2, 32 + b)}, {at(3, b), at(3, 32 + b)}};
            fold_out_split(row, 2 * P, j, w, g.inv, t0, t1);
        } else if constexpr (IM) {
            const float c0[2] = {at(0, i), at(0, 32 + i)}, s0[2] = {at(1, i), at(1, 32 + i)};
            const float c1[2] = {at(2, i), at(2, 32 + i)}, s1[2] = {at(3, i), at(3, 32 + i)};
            fold_out_cplx(row, P, j, w, g.inv, c0, s0, c1, s1);
        } else {
            fold_out_real(row, P, j, w, at(0, i), at(1, i), at(2, i), at(3, i));
        }
    }
}

// Logical tile L of an nm x nn grid: groups of GROUP_M m-tiles sweep all
// j-tiles, so they share each operand block and their own rows in L2.
__device__ __forceinline__ void fold_place(int64_t L, int64_t nm, int64_t nn, int64_t bm, int64_t bj, int64_t& m0,
                                           int64_t& n0) {
    const int64_t full = GROUP_M * nn, grp = L / full, first = grp * GROUP_M;
    const int64_t gsz = min((int64_t)GROUP_M, nm - first), in = L - grp * full;
    m0 = (first + in % gsz) * bm;
    n0 = (in / gsz) * bj;
}

template <int FORM, int MODE, int WGM, int WGN>
__global__ __launch_bounds__((FoldTile<FORM, WGM, WGN>::NTH)) __attribute__((amdgpu_waves_per_eu(2)))
void fold_gemm_kernel(GemmArgs g) {
    using G = FoldTile<FORM, WGM, WGN>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * G::STAGE];
    const int64_t nm = (g.F * kRows<MODE> + G::BMR - 1) / G::BMR, nn = (g.N + G::BJ - 1) / G::BJ;
    int64_t m0, n0;
    fold_place(xcd_logical_block(blockIdx.x, gridDim.x), nm, nn, G::BMR, G::BJ, m0, n0);
    fold_tile<FORM, MODE, WGM, WGN, false>(g, m0, n0, lds, nullptr);
}

template <int FORM, int MODE, int TM>
__global__ __launch_bounds__(256) void fold_gemm_small_kernel(GemmArgs g) {
    constexpr int ROWS = 32 * TM;
    __shared__ float ex[4 * ROWS * 33];
    const int64_t nm = (g.F * kRows<MODE> + ROWS - 1) / ROWS, nn = g.N / 32;
    int64_t m0, n0;
    fold_place(xcd_logical_block(blockIdx.x, gridDim.x), nm, nn, ROWS, 32, m0, n0);
    fold_tile_small<FORM, MODE, TM>(g, m0, n0, ex);
}

// FP32 with the operand assembled from the 2P-entry cosine table (8 P bytes,
// copied to LDS after the K tiles) instead of read: same entries, same bits.
template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void fold_gemm_table_kernel(GemmArgs g) {
    using G = FoldTile<FORM_FP32, 2, 2>;
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn[];
    float* ct = reinterpret_cast<float*>(dyn + 2 * G::STAGE);
    for (int r = threadIdx.x; r < 2 * g.K; r += G::NTH) ct[r] = g.ct[r];
    __syncthreads();
    const int64_t nm = (g.F * kRows<MODE> + G::BMR - 1) / G::BMR, nn = (g.N + G::BJ - 1) / G::BJ;
    int64_t m0, n0;
    fold_place(xcd_logical_block(blockIdx.x, gridDim.x), nm, nn, G::BMR, G::BJ, m0, n0);
    fold_tile<FORM_FP32, MODE, 2, 2, true>(g, m0, n0, dyn, ct);
}

// Batched: block b serves tile b / 8 of XCD b % 8's range of the table's
// folded tiles (fold_batch_tile).
template <int FORM>
__global__ __launch_bounds__(FORM == FORM_FP32 ? 256 : 512) __attribute__((amdgpu_waves_per_eu(2)))
void fold_gemm_batch_kernel(const BatchTable* __restrict__ t) {
    constexpr bool F32 = FORM == FORM_FP32;
    using G = FoldTile<FORM, 2, F32 ? 2 : 4>;
    using G64 = FoldTile<FORM, F32 ? 2 : 4, 2>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * (G::STAGE > G64::STAGE ? G::STAGE : G64::STAGE)];
    const int x = blockIdx.x & 7;
    const int64_t u = t->gfold_bounds[x] + (blockIdx.x >> 3);
    if (u >= t->gfold_bounds[x + 1]) return;
    const int it = batch_find(t->items, t->n_items, u, /*stage=*/5);
    const GemmArgs g = t->items[it].gemm;
    int64_t bm, bj, m0, n0;
    const int64_t rows = g.F * (g.real_pack ? 1 : g.split ? 4 : 2);
    fold_batch_tile(FORM, g.N, bm, bj);
    fold_place(u - t->items[it].gfold_unit0, (rows + bm - 1) / bm, (g.N + bj - 1) / bj, bm, bj, m0, n0);
    if (!F32 && g.N == 64) {
        // 256 channels: whole frames (16-bit forms split from 2048 on).
        if (g.real_pack) fold_tile<FORM, REAL, F32 ? 2 : 4, 2, false>(g, m0, n0, lds, nullptr);
        else fold_tile<FORM, CPLX, F32 ? 2 : 4, 2, false>(g, m0, n0, lds, nullptr);
    } else {
        if (g.real_pack) fold_tile<FORM, REAL, 2, F32 ? 2 : 4, false>(g, m0, n0, lds, nullptr);
        else if (g.split) fold_tile<FORM, SPLIT, 2, F32 ? 2 : 4, false>(g, m0, n0, lds, nullptr);
        else fold_tile<FORM, CPLX, 2, F32 ? 2 : 4, false>(g, m0, n0, lds, nullptr);
    }
}

template <int FORM, int MODE, int WGM, int WGN>
hipError_t launch_fold_wide(const GemmArgs& g, hipStream_t s) {
    using G = FoldTile<FORM, WGM, WGN>;
    const int64_t nm = (g.F * kRows<MODE> + G::BMR - 1) / G::BMR, nn = (g.N + G::BJ - 1) / G::BJ;
    hipLaunchKernelGGL((fold_gemm_kernel<FORM, MODE, WGM, WGN>), dim3((unsigned)(nm * nn)), dim3(G::NTH), 0, s, g);
    return hipGetLastError();
}

// Below 96 tiles of 128 x 128 most CUs would have no large tile (4096 complex
// channels, FP32: 64 of them take 106 us either way, 128 take 166 us against
// 201 us with the small ones; 1024 real channels, BF16x3: 64 take 35 us against
// 31 us, 128 37 us against 58 us).
template <int FORM, int MODE>
hipError_t launch_fold_form(const GemmArgs& g, hipStream_t s) {
    const int64_t R = g.F * kRows<MODE>;
    if (R * g.N < 96 * 128 * 128) {
        // Real frames: 32 rows a block until those are 512 blocks (1024 channels,
        // FP32: 1024 frames 17 us against 21 us with 64 rows, 4096 frames 49 us
        // against 35 us).
        if constexpr (MODE == REAL) {
            const int64_t blocks = (R + 31) / 32 * (g.N / 32);
            if (blocks <= 512) {
                hipLaunchKernelGGL((fold_gemm_small_kernel<FORM, MODE, 1>), dim3((unsigned)blocks), dim3(256), 0, s, g);
                return hipGetLastError();
            }
        }
        const int64_t blocks = (R + 63) / 64 * (g.N / 32);
        hipLaunchKernelGGL((fold_gemm_small_kernel<FORM, MODE, 2>), dim3((unsigned)blocks), dim3(256), 0, s, g);
        return hipGetLastError();
    }
    if constexpr (FORM == FORM_FP32) return launch_fold_wide<FORM, MODE, 2, 2>(g, s);
    else if constexpr (MODE == SPLIT) return launch_fold_wide<FORM, MODE, 2, 4>(g, s);  // from 2048 channels on
    else return g.N == 64 ? launch_fold_wide<FORM, MODE, 4, 2>(g, s) : launch_fold_wide<FORM, MODE, 2, 4>(g, s);
}

template <int MODE>
hipError_t launch_fold_table(const GemmArgs& g, hipStream_t s) {
    using G = FoldTile<FORM_FP32, 2, 2>;
    const int64_t nm = (g.F * kRows<MODE> + G::BMR - 1) / G::BMR, nn = (g.N + G::BJ - 1) / G::BJ;
    static const hipError_t attr = hipFuncSetAttribute((const void*)fold_gemm_table_kernel<MODE>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       2 * G::STAGE + 8 * 8192);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((fold_gemm_table_kernel<MODE>), dim3((unsigned)(nm * nn)), dim3(G::NTH), 2 * G::STAGE + 8 * g.K, s, g);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dft_fold(const GemmArgs& g, hipStream_t s) {
    if (g.F <= 0) return hipSuccess;
    if (g.N * 4 != g.K || g.N < 64 || !g.tw) return hipErrorInvalidValue;
    auto go = [&](auto tag) {
        constexpr int FORM = decltype(tag)::value;
        return g.real_pack ? launch_fold_form<FORM, REAL>(g, s)
               : g.split   ? launch_fold_form<FORM, SPLIT>(g, s)
                           : launch_fold_form<FORM, CPLX>(g, s);
    };
    if (g.ct) {
        if (g.form != FORM_FP32) return hipErrorInvalidValue;
        return g.real_pack ? launch_fold_table<REAL>(g, s) : g.split ? launch_fold_table<SPLIT>(g, s) : launch_fold_table<CPLX>(g, s);
    }
    switch (g.form) {
        case FORM_FP32: return go(std::integral_constant<int, FORM_FP32>{});
        case FORM_BF16: return go(std::integral_constant<int, FORM_BF16>{});
        case FORM_BF16X3: return go(std::integral_constant<int, FORM_BF16X3>{});
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fold_gemm_batch(const BatchTable* t, int form, int grid, hipStream_t s) {
    switch (form) {
        case FORM_FP32: hipLaunchKernelGGL((fold_gemm_batch_kernel<FORM_FP32>), dim3(grid), dim3(256), 0, s, t); break;
        case FORM_BF16: hipLaunchKernelGGL((fold_gemm_batch_kernel<FORM_BF16>), dim3(grid), dim3(512), 0, s, t); break;
        case FORM_BF16X3: hipLaunchKernelGGL((fold_gemm_batch_kernel<FORM_BF16X3>), dim3(grid), dim3(512), 0, s, t); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tina
