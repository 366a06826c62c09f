// Polyphase FIR with folded output: the operand of the folded DFT product
// (gemm_fold.hip).  Instantiated per output mode in fir_fold_*.hip.
//
// The DFT of a frame y[0..P) is taken around the half sample: with
// q = p + 1/2, exp(-2 pi i k p / P) = exp(i pi k / P) exp(-2 pi i k q / P),
// and the cosines and sines of 2 pi k q / P are even and odd under
// q -> P - q and, for even and odd k apart, under q -> P/2 - q.  The four
// samples p, P/2-1-p, P/2+p, P-1-p (p < Q = P/4) therefore enter every channel
// only through four sums, and the P x P product falls apart into four
// products of size Q x Q:
//   a = y[p], b = y[P/2-1-p], c = y[P/2+p], d = y[P-1-p]
//   part 0 (cos, even k): (a+d) + (b+c)     part 1 (sin, even k): (a-d) - (b-c)
//   part 2 (cos, odd k):  (a+d) - (b+c)     part 3 (sin, odd k):  (a-d) + (b-c)
// Only additions, in FP32 before any rounding to the operand type: a part's
// entries have on average the square sum of the samples they replace, so the
// rounding of the operand costs what it did.
//
// A complex frame is two such rows (real, imaginary).  Output: row f * cf + ri,
// P elements, part s at elements [s Q, (s+1) Q).  Where fold_split says so a complex
// frame takes one decimation in frequency first (fold_store_split) and is four rows
// of P/2: its halves' real and imaginary parts.
//
// HBM-bound.  A block holds the four column groups that fold onto each other
// (group g in wave(s) g, GF floats each), walks a run of frames through the
// FIR's register ring (same multiply-adds, same bits as fir_unit), and passes
// up to SB frames at a time through LDS: every wave stores its group, and
// after one barrier (two buffers) every thread reads four floats of each group,
// mirrored where the group runs backwards, and stores the four parts.  The LDS
// traffic (1 write, 1 read per float) is a quarter of its rate at HBM speed.
#pragma once
#include "fir_kernels.h"

namespace tina {
namespace {

// VEC floats per thread, NG column groups (4; 8 for split frames) of GL lanes.
template <int VEC, int NG, int GL>
struct FoldGeom {
    static constexpr int GF = GL * VEC;                   // floats per column group
    static constexpr int NTH = NG * GL;                   // threads per block
    static constexpr int SB = NG == 4 ? 16 / VEC : 512 / GF;  // frames per LDS phase (16 to 32 KB a buffer)
};
template <int VEC, int NG, int GL>
struct FoldSmem {
    float ys[2][FoldGeom<VEC, NG, GL>::SB][NG * FoldGeom<VEC, NG, GL>::GF];
};

__device__ __forceinline__ fvec4 fold_mirror(const fvec4& v, bool cplx) {
    return cplx ? __builtin_shufflevector(v, v, 2, 3, 0, 1) : __builtin_shufflevector(v, v, 3, 2, 1, 0);
}

// Four consecutive elements of a part row, in the operand type.
template <int QM>
__device__ __forceinline__ void fold_put(const FirArgs& a, int64_t el, const float (&v)[4]) {
    if constexpr (QM == QM_NONE) {
        st<true>(reinterpret_cast<fvec4*>(a.y + el), fvec4{v[0], v[1], v[2], v[3]});
    } else {
        static_assert(QM == QM_BF16 || QM == QM_BF16X2 || QM == QM_F8BF16, "operand types of the folded product");
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[i] = bf16_bits(v[i]);
            lo[i] = bf16_bits(v[i] - __builtin_bit_cast(float, hi[i] << 16));
        }
        auto put = [&](uint8_t* base, const uint32_t (&h)[4]) {
            st<true>(reinterpret_cast<uint64_t*>(base + el * 2),
                     (uint64_t)(h[0] | (h[1] << 16)) | ((uint64_t)(h[2] | (h[3] << 16)) << 32));
        };
        put(a.q, hi);
        if constexpr (QM == QM_BF16X2) put(a.q1, lo);
    }
}

// A value as the fold takes it: for FP8 rounded (to nearest even) to the 4
// significant bits of E4M3, on the bit pattern.  The largest floats saturate, as
// E4M3's do.  Infinities and NaNs become NaN by the product with zero (a carry out
// of a NaN's payload alone would leave a zero); a finite value's adds a zero of its
// own sign.
template <int VEC, int QM>
__device__ __forceinline__ typename VecT<VEC>::T fold_value(typename VecT<VEC>::T v) {
    if constexpr (QM == QM_F8BF16) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float x = vget<VEC>(v, i), top = 0x1.ep127f;
            const uint32_t u = __builtin_bit_cast(uint32_t, x);
            const float r = __builtin_bit_cast(float, (u + 0x7ffffu + ((u >> 20) & 1u)) & 0xfff00000u);
            vset<VEC>(v, i, fmaf(x, 0.0f, __builtin_amdgcn_fmed3f(r, -top, top)));
        }
    }
    return v;
}

// Folds and stores `cnt` frames (first frame f0) of LDS buffer ys: column
// block at float offset c0 of each quarter frame.  A thread stores four
// elements of a part at a time: real frames four samples' four parts, complex
// ones two of the parts (even or odd channels) of four samples.
template <int VEC, int GL, int QM>
__device__ __forceinline__ void fold_store(const FirArgs& a,
                                           const float (&ys)[FoldGeom<VEC, 4, GL>::SB][4 * FoldGeom<VEC, 4, GL>::GF],
                                           int64_t f0, int cnt, int c0) {
    using G = FoldGeom<VEC, 4, GL>;
    constexpr int X4 = G::GF / 4;  // float4 positions per group
    const int Q = a.P / 4;
    if (a.cf == 2) {
        for (int it = threadIdx.x; it < cnt * X4; it += G::NTH) {
            const int fr = it / X4, h = (it % X4) / (X4 / 2), x = it % (X4 / 2);  // h: odd channels
            const fvec4* row = reinterpret_cast<const fvec4*>(ys[fr]);
            fvec4 c[2], s[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = 2 * x + i;
                const fvec4 A = row[q], B = fold_mirror(row[X4 + X4 - 1 - q], true);
                const fvec4 C = row[2 * X4 + q], D = fold_mirror(row[3 * X4 + X4 - 1 - q], true);
                const fvec4 e = A + D, e2 = B + C, o = A - D, o2 = B - C;
                c[i] = h ? e - e2 : e + e2;
                s[i] = h ? o + o2 : o - o2;
            }
            const int64_t el = (f0 + fr) * (int64_t)a.W + c0 / 2 + 4 * x + 2 * h * Q;
            fold_put<QM>(a, el, {c[0][0], c[0][2], c[1][0], c[1][2]});
            fold_put<QM>(a, el + Q, {s[0][0], s[0][2], s[1][0], s[1][2]});
            fold_put<QM>(a, el + a.P, {c[0][1], c[0][3], c[1][1], c[1][3]});
            fold_put<QM>(a, el + a.P + Q, {s[0][1], s[0][3], s[1][1], s[1][3]});
        }
    } else {
        for (int it = threadIdx.x; it < cnt * X4; it += G::NTH) {
            const int fr = it / X4, x = it % X4;
            const fvec4* row = reinterpret_cast<const fvec4*>(ys[fr]);
            const fvec4 A = row[x], B = fold_mirror(row[X4 + X4 - 1 - x], false);
            const fvec4 C = row[2 * X4 + x], D = fold_mirror(row[3 * X4 + X4 - 1 - x], false);
            const fvec4 e = A + D, e2 = B + C, o = A - D, o2 = B - C;
            const fvec4 part[4] = {e + e2, o - o2, e - e2, o + o2};
            const int64_t el = (f0 + fr) * (int64_t)a.W + c0 + 4 * x;
#pragma unroll
            for (int s = 0; s < 4; ++s) fold_put<QM>(a, el + s * Q, {part[s][0], part[s][1], part[s][2], part[s][3]});
        }
    }
}

// The same of split complex frames: u = y[p] + y[p + P/2] (even channels) and
// v = (y[p] - y[p + P/2]) exp(-2 pi i p / P) (odd channels), p < P/2, each folded as
// a frame of P/2.  Groups 0-3 hold the places that fold onto each other, groups
// 4-7 the same P/2 samples later.  A thread takes four samples of one half (t)
// and two of its parts (h).
template <int VEC, int GL, int QM>
__device__ __forceinline__ void fold_store_split(const FirArgs& a,
                                                 const float (&ys)[FoldGeom<VEC, 8, GL>::SB][8 * FoldGeom<VEC, 8, GL>::GF],
                                                 int64_t f0, int cnt, int c0) {
    using G = FoldGeom<VEC, 8, GL>;
    constexpr int X4 = G::GF / 4, X8 = G::GF / 8;
    const int H = a.P / 2, Q = a.P / 8, n = cnt * X8;  // half's length, part's length, places
    const fvec2* tw = reinterpret_cast<const fvec2*>(a.split_tw);
    for (int it = threadIdx.x; it < 4 * n; it += G::NTH) {
        const int sub = it / n, pl = it % n, t = sub >> 1, h = sub & 1, fr = pl / X8, x = pl % X8;
        const fvec4* row = reinterpret_cast<const fvec4*>(ys[fr]);
        const int p0 = c0 / 2 + 4 * x;
        // z[g][i]: sample p0 + i of group g (mirrored groups in the order of their folds), as re, im.
        fvec2 z[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = 2 * x + i;
                const bool mir = g & 1;
                const int at = g * X4 + (mir ? X4 - 1 - q : q);
                fvec4 y0 = row[at], y1 = row[at + 4 * X4];
                fvec4 d = t ? y0 - y1 : y0 + y1;
                if (mir) d = fold_mirror(d, true);
                z[g][2 * i] = fvec2{d[0], d[1]};
                z[g][2 * i + 1] = fvec2{d[2], d[3]};
            }
        if (t) {
            // Twiddles of places p, P/4 - 1 - p, P/4 + p, P/2 - 1 - p by those of p and
            // p + 1: w(p), -i w*(p + 1), -i w(p), -w*(p + 1).
            fvec2 w = tw[p0];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const fvec2 w1 = tw[p0 + i + 1];
                auto fwd = [](fvec2 d, fvec2 c) { return fvec2{fmaf(d[0], c[0], d[1] * c[1]), fmaf(d[1], c[0], -(d[0] * c[1]))}; };
                auto bwd = [](fvec2 d, fvec2 c) { return fvec2{fmaf(d[0], c[0], -(d[1] * c[1])), fmaf(d[1], c[0], d[0] * c[1])}; };
                z[0][i] = fwd(z[0][i], w);
                const fvec2 b = bwd(z[1][i], w1), c = fwd(z[2][i], w), d = bwd(z[3][i], w1);
                z[1][i] = fvec2{b[1], -b[0]};
                z[2][i] = fvec2{c[1], -c[0]};
                z[3][i] = fvec2{-d[0], -d[1]};
                w = w1;
            }
        }
        float cr[4], ci[4], sr[4], si[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const fvec2 e = z[0][i] + z[3][i], e2 = z[1][i] + z[2][i], o = z[0][i] - z[3][i], o2 = z[1][i] - z[2][i];
            const fvec2 c = h ? e - e2 : e + e2, s = h ? o + o2 : o - o2;
            cr[i] = c[0];
            ci[i] = c[1];
            sr[i] = s[0];
            si[i] = s[1];
        }
        const int64_t el = (f0 + fr) * (int64_t)a.W + (int64_t)t * a.P + p0 + 2 * h * Q;
        fold_put<QM>(a, el, cr);
        fold_put<QM>(a, el + Q, sr);
        fold_put<QM>(a, el + H, ci);
        fold_put<QM>(a, el + H + Q, si);
    }
}

// Place of a block's thread in the frame: its column group's first float j0, and
// its floats' place in an LDS row.
template <int VEC, int NG, int GL>
struct FoldPlace {
    int c0, j0, slot;
    __device__ __forceinline__ FoldPlace(const FirArgs& a, int cb) {
        using G = FoldGeom<VEC, NG, GL>;
        // Floats that fold four-fold (a frame, or half of one) and a quarter of them.
        const int span = NG == 8 ? a.W / 2 : a.W, quarter = span / 4;
        const int g = threadIdx.x / GL, x = (threadIdx.x % GL) * VEC, gg = g & 3;
        c0 = cb * G::GF;
        j0 = (g >> 2) * span + (gg == 0 ? c0 : gg == 1 ? 2 * quarter - c0 - G::GF : gg == 2 ? 2 * quarter + c0 : span - c0 - G::GF) + x;
        slot = g * G::GF + x;
    }
};

// Column blocks of a frame (a power of two).
template <int VEC, int NG, int GL>
__host__ __device__ __forceinline__ int fold_col_blocks(const FirArgs& a) {
    return a.W / NG / FoldGeom<VEC, NG, GL>::GF;
}

// One unit of up to 16 taps: column block and run of logical block `blk`.  Every
// condition on frames is the same for the whole block, so all its threads meet at
// each barrier.  ph: the LDS buffer of the next phase (a buffer is written again
// two phases later, after every thread has passed the barrier in between, so
// one barrier per phase is enough, across units too).
template <int VEC, int NG, int GL, int MT, int QM>
__device__ __forceinline__ void fir_fold_unit(const FirArgs& a, int TF, int64_t blk, FoldSmem<VEC, NG, GL>& sm, int& ph) {
    using V = typename VecT<VEC>::T;
    using G = FoldGeom<VEC, NG, GL>;
    // Frames walked at a time: whole rings, as many as fill an LDS phase (with one
    // ring a phase, and so a barrier for every M frames, 256 complex channels, BF16,
    // 2^24 samples took 182 us with 1 tap and 133 with 6; now 78 and 80; 104 and 96
    // with the plain product).
    constexpr int BL = fold_block_frames(MT, G::SB);
    const int ncb = fold_col_blocks<VEC, NG, GL>(a);
    const int64_t run = blk / ncb;
    const int64_t f_begin = run * TF;
    if (f_begin >= a.F) return;
    const int64_t f_end = min(a.F, f_begin + TF);
    const FoldPlace<VEC, NG, GL> at(a, (int)(blk & (ncb - 1)));
    const int j0 = at.j0, slot = at.slot;

    V tp[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) tp[m] = load_taps<VEC>(a, MT, m, j0);
    V win[MT];  // ring of input frames, as in fir_unit
    auto flush = [&](int64_t f0, int cnt) {
        __syncthreads();
        if constexpr (NG == 8) fold_store_split<VEC, GL, QM>(a, sm.ys[ph], f0, cnt, at.c0);
        else fold_store<VEC, GL, QM>(a, sm.ys[ph], f0, cnt, at.c0);
        ph ^= 1;
    };
    // Frames [f0, f1) straight from their input frames: blocks that straddle
    // the prefix/chunk boundary, and the tail.  All loads of D frames in flight
    // before the first FMA (195 frames of 1024 channels, 12 taps, half of them such:
    // 10 us; 20 us where the compiler puts waits between the loads).
    constexpr int D = 8 / (MT * VEC) > 1 ? 8 / (MT * VEC) : 1;
    auto direct = [&](int64_t f, int u0, int cnt) {
        V in[D][MT];
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
            for (int m = 0; m < MT; ++m)
                in[d][m] = load_frame<VEC, true>(a, a.g0 + f + (D > 1 ? min(u0 + d, cnt - 1) : u0) - m, j0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            V acc = V(0.0f);
#pragma unroll
            for (int m = 0; m < MT; ++m) acc = __builtin_elementwise_fma(tp[m], in[d][m], acc);
            if (D == 1 || u0 + d < cnt) *reinterpret_cast<V*>(&sm.ys[ph][u0 + d][slot]) = fold_value<VEC, QM>(acc);
        }
    };
    auto slow = [&](int64_t f0, int64_t f1) {
        constexpr int SB = G::SB < BL ? G::SB : BL;
        for (int64_t f = f0; f < f1; f += SB) {
            const int cnt = (int)min((int64_t)SB, f1 - f);
#pragma unroll 1
            for (int u = 0; u < cnt; u += D) direct(f, u, cnt);  // unrolled: up to 250 registers
            flush(f, cnt);
        }
    };
    bool ring_ok = false;
    // n frames from fb on (LEN, whole rings, or at the end fewer: rows past the last
    // read the last one again), through the ring where they lie in the chunk.
    auto walk = [&](auto len, int64_t fb, int n) {
        constexpr int LEN = decltype(len)::value, SB = G::SB < LEN ? G::SB : LEN;
        const int64_t fu = (int64_t)uniform64((uint64_t)fb);
        const int64_t eu = (a.g0 + fu + a.M - 1) * (int64_t)a.W - a.plen;  // block's first float in the chunk
        if (eu < 0) {
            ring_ok = false;
            slow(fb, fb + n);
            return;
        }
        if (!ring_ok) {
#pragma unroll
            for (int d = 1; d < MT; ++d) win[MT - d] = load_frame<VEC, false>(a, a.g0 + fb - d, j0);
        }
        ring_ok = true;
        const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.chunk + eu, (a.nchunk - eu) * 4);
        const uint32_t vin = (uint32_t)j0 * 4u;
        const int32_t w4 = a.W * 4;
#pragma unroll
        for (int sb = 0; sb < LEN; sb += SB) {
            if (sb >= n) break;
            V in[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i)
                if (sb + i < LEN) in[i] = buf_load<VEC, true>(rin, vin, min(sb + i, n - 1) * w4);
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                if (sb + i >= LEN) continue;
                const int u = (sb + i) % MT;
                win[u] = in[i];
                *reinterpret_cast<V*>(&sm.ys[ph][i][slot]) = fold_value<VEC, QM>(fir_point<VEC, MT, true>(tp, win, u, MT));
            }
            flush(fb + sb, min(n - sb, LEN - sb < SB ? LEN - sb : SB));
        }
    };
    int64_t fb = f_begin;
    for (; fb + BL <= f_end; fb += BL) walk(std::integral_constant<int, BL>{}, fb, BL);
    if (fb < f_end) walk(std::integral_constant<int, BL>{}, fb, (int)(f_end - fb));
}

// One unit of more than 16 taps, any number of them: kFoldLong frames at a time,
// their sums in registers, tap after tap, while the input frames they meet move
// through a ring of that length, one older frame a tap (1 + (M - 1) / 32 reads a
// float, all but one of them from L2).  Taps and frames are loaded kFoldAhead taps
// ahead.  In place of rings of 32 and 64 taps in registers, those beyond M behind a
// condition each (512 registers, 584 scalar ones spilled), 1024 real channels, BF16,
// 2^25 samples, the whole call: 24 taps 204 -> 111 us, 64 taps 3510 -> 144 (94 with 16
// taps; 237 and 174 with the plain product).
constexpr int kFoldLong = 32, kFoldAhead = 8;
template <int NG, int GL, int QM>
__device__ __forceinline__ void fir_fold_unit_long(const FirArgs& a, int TF, int64_t blk, FoldSmem<1, NG, GL>& sm, int& ph) {
    using G = FoldGeom<1, NG, GL>;
    constexpr int B = kFoldLong, C = kFoldAhead, SB = G::SB;
    const int ncb = fold_col_blocks<1, NG, GL>(a);
    const int64_t run = blk / ncb;
    const int64_t f_begin = run * TF;
    if (f_begin >= a.F) return;
    const int64_t f_end = min(a.F, f_begin + TF);
    const FoldPlace<1, NG, GL> at(a, (int)(blk & (ncb - 1)));
    const int j0 = at.j0, M = a.M;
    for (int64_t fb = f_begin; fb < f_end; fb += B) {
        const int cnt = (int)min((int64_t)B, f_end - fb);
        float ring[B], acc[B], t[C], x[C], tn[C], xn[C];
        auto ahead = [&](int m) {
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const int k = min(m + i, M - 1);  // past the last: reads in range, not used
                tn[i] = load_taps<1>(a, M, k, j0);
                xn[i] = load_frame<1, false>(a, a.g0 + fb - k, j0);
            }
        };
        ahead(0);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            ring[u] = load_frame<1, false>(a, a.g0 + fb + min(u, cnt - 1), j0);
            acc[u] = -0.0f;  // the first multiply-add gives the product itself
        }
        // Tap m meets frame fb + u - m for output u, in slot (u - m) mod B.
        for (int m0 = 0; m0 < M; m0 += B) {
#pragma unroll
            for (int s = 0; s < B; ++s) {
                if (s % C == 0) {
                    if (m0 + s >= M) break;
#pragma unroll
                    for (int i = 0; i < C; ++i) {
                        t[i] = tn[i];
                        x[i] = xn[i];
                    }
                    ahead(m0 + s + C);
                }
                if (m0 + s < M) {
                    ring[(B - s) % B] = x[s % C];
#pragma unroll
                    for (int u = 0; u < B; ++u) acc[u] = fmaf(t[s % C], ring[(u - s + B) % B], acc[u]);
                }
            }
        }
#pragma unroll
        for (int sb = 0; sb < B; sb += SB) {
            if (sb >= cnt) break;
#pragma unroll
            for (int i = 0; i < SB; ++i) sm.ys[ph][i][at.slot] = fold_value<1, QM>(acc[sb + i]);
            __syncthreads();
            const int n = min(SB, cnt - sb);
            if constexpr (NG == 8) fold_store_split<1, GL, QM>(a, sm.ys[ph], fb + sb, n, at.c0);
            else fold_store<1, GL, QM>(a, sm.ys[ph], fb + sb, n, at.c0);
            ph ^= 1;
        }
    }
}

template <int VEC, int NG, int GL, int MT, int QM>
__global__ __launch_bounds__((FoldGeom<VEC, NG, GL>::NTH)) void fir_fold_kernel(FirArgs a, int TF) {
    __shared__ __attribute__((aligned(16))) FoldSmem<VEC, NG, GL> sm;
    int ph = 0;
    fir_fold_unit<VEC, NG, GL, MT, QM>(a, TF, xcd_logical_block(blockIdx.x, gridDim.x), sm, ph);
}
template <int NG, int GL, int QM>
__global__ __launch_bounds__((FoldGeom<1, NG, GL>::NTH)) void fir_fold_long_kernel(FirArgs a) {
    __shared__ __attribute__((aligned(16))) FoldSmem<1, NG, GL> sm;
    int ph = 0;
    fir_fold_unit_long<NG, GL, QM>(a, kFoldLong, xcd_logical_block(blockIdx.x, gridDim.x), sm, ph);
}

template <int VEC, int NG, int GL, int M0, int MT, int QM>
__device__ __forceinline__ void fir_fold_unit_own_m(const FirArgs& a, int TF, int64_t blk, FoldSmem<VEC, NG, GL>& sm, int& ph) {
    if constexpr (M0 <= MT) {
        if (a.M == M0) fir_fold_unit<VEC, NG, GL, M0, QM>(a, TF, blk, sm, ph);
        else fir_fold_unit_own_m<VEC, NG, GL, M0 + 1, MT, QM>(a, TF, blk, sm, ph);
    }
}

// Persistent batched form, over the table's folded FIR units, each with its item's
// tap count.  LONG: items of more than 16 taps among them (apart, for the registers).
// One float per thread (any alignment); two, a complex sample, in the 16-bit forms
// (whole 128-byte lines of a part row).
template <bool LONG, int QM>
__global__ __launch_bounds__(256) void fir_fold_batch_kernel(const BatchTable* __restrict__ t) {
    constexpr int CV = QM == QM_NONE ? 1 : 2;  // floats per thread of complex items
    __shared__ __attribute__((aligned(16))) union {
        FoldSmem<1, 4, 64> one;
        FoldSmem<CV, 4, 64> cplx;
    } sm;
    static_assert(sizeof(FoldSmem<1, 4, 64>) == sizeof(FoldSmem<CV, 4, 64>), "their buffers coincide");
    int ph = 0;
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3, nbx = gridDim.x >> 3;
    const int64_t end = t->ffold_bounds[x + 1];
    for (int64_t u = t->ffold_bounds[x] + i; u < end; u += nbx) {
        const int it = batch_find(t->items, t->n_items, u, /*stage=*/4);
        const BatchItem& b = t->items[it];
        const FirArgs fa = b.fir;
        const int64_t blk = u - b.ffold_unit0;
        if (LONG && fa.M > 16) fir_fold_unit_long<4, 64, QM>(fa, b.fir_tf, blk, sm.one, ph);
        else if (CV == 2 && fa.cf == 2) fir_fold_unit_own_m<CV, 4, 64, 1, 16, QM>(fa, b.fir_tf, blk, sm.cplx, ph);
        else fir_fold_unit_own_m<1, 4, 64, 1, 16, QM>(fa, b.fir_tf, blk, sm.one, ph);
    }
}
template <bool LONG, int QM>
__global__ __launch_bounds__(512) void fir_fold_split_batch_kernel(const BatchTable* __restrict__ t) {
    __shared__ __attribute__((aligned(16))) FoldSmem<1, 8, 64> sm;
    int ph = 0;
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3, nbx = gridDim.x >> 3;
    const int64_t end = t->fsplit_bounds[x + 1];
    for (int64_t u = t->fsplit_bounds[x] + i; u < end; u += nbx) {
        const int it = batch_find(t->items, t->n_items, u, /*stage=*/6);
        const BatchItem& b = t->items[it];
        const FirArgs fa = b.fir;
        const int64_t blk = u - b.fsplit_unit0;
        if (LONG && fa.M > 16) fir_fold_unit_long<8, 64, QM>(fa, b.fir_tf, blk, sm, ph);
        else fir_fold_unit_own_m<1, 8, 64, 1, 16, QM>(fa, b.fir_tf, blk, sm, ph);
    }
}

template <int VEC, int NG, int GL, int MT, int QM>
hipError_t launch_fold_one(const FirArgs& a, hipStream_t s) {
    using G = FoldGeom<VEC, NG, GL>;
    const int ncb = fold_col_blocks<VEC, NG, GL>(a);
    // Frames per block: two of the unit's blocks (at least 16 frames) so that the
    // halo stays small; fewer, down to one ring, while that leaves CUs without a block.
    constexpr int BL = fold_block_frames(MT, G::SB);
    int TF = 2 * BL < 16 ? ((16 + BL - 1) / BL) * BL : 2 * BL;
    while (TF > MT && TF > 4 && (a.F + TF - 1) / TF * ncb < 512) TF -= TF > BL ? BL : MT;
    const int64_t runs = (a.F + TF - 1) / TF;
    hipLaunchKernelGGL((fir_fold_kernel<VEC, NG, GL, MT, QM>), dim3((unsigned)(runs * ncb)), dim3(G::NTH), 0, s, a, TF);
    return hipGetLastError();
}

template <int NG, int GL, int QM>
hipError_t launch_fold_long(const FirArgs& a, hipStream_t s) {
    const int64_t blocks = (a.F + kFoldLong - 1) / kFoldLong * fold_col_blocks<1, NG, GL>(a);
    hipLaunchKernelGGL((fir_fold_long_kernel<NG, GL, QM>), dim3((unsigned)blocks), dim3(FoldGeom<1, NG, GL>::NTH), 0, s, a);
    return hipGetLastError();
}

template <int VEC, int NG, int GL, int M0, int MTOP, int QM>
hipError_t launch_fold_m(const FirArgs& a, hipStream_t s) {
    if constexpr (M0 <= MTOP) {
        if (a.M == M0) return launch_fold_one<VEC, NG, GL, M0, QM>(a, s);
        return launch_fold_m<VEC, NG, GL, M0 + 1, MTOP, QM>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int QM>
hipError_t launch_fold_qm(const FirArgs& a, hipStream_t s) {
    auto aligned = [&](const void* p) { return ((uintptr_t)p & 15) == 0; };
    const bool al16 = a.plen % 4 == 0 && aligned(a.chunk) && (!a.prefix || aligned(a.prefix));
    if (a.split_tw) {
        // 64 samples a group (a part row's piece fills a 128-byte line in the
        // 16-bit forms) in blocks of 256 threads while their registers hold two
        // blocks a CU: 4096 channels, 2^25 samples, 8 taps, BF16x3: 123 us, 159
        // with one float a thread.  Beyond 8 taps one float (1024 channels, 16
        // taps, FP32: 131 us; 156 with four, 184 with two in 512 threads).
        if (a.M <= 8 && al16) return launch_fold_m<4, 8, 32, 1, 8, QM>(a, s);
        if (a.M <= 16) return launch_fold_m<1, 8, 64, 1, 16, QM>(a, s);
        return launch_fold_long<8, 64, QM>(a, s);
    }
    if (a.M <= 8 && al16 && a.W >= 1024) return launch_fold_m<4, 4, 64, 1, 8, QM>(a, s);
    // 16-bit complex rows: 128 lanes a group, for whole lines as above (1024
    // channels, 16 taps, 2^25 samples, BF16x3, unsplit: 163 us with 64 lanes and
    // half lines, 129 us; FP32 rows the same either way).
    if (QM != QM_NONE && a.cf == 2 && a.M <= 16) return launch_fold_m<1, 4, 128, 1, 16, QM>(a, s);
    if (a.M <= 16) return launch_fold_m<1, 4, 64, 1, 16, QM>(a, s);
    return launch_fold_long<4, 64, QM>(a, s);
}

template <int QM>
hipError_t launch_fold_batch_qm(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s) {
    auto go = [&](auto tag) {
        constexpr bool LONG = decltype(tag)::value;
        if (split) hipLaunchKernelGGL((fir_fold_split_batch_kernel<LONG, QM>), dim3(grid), dim3(512), 0, s, t);
        else hipLaunchKernelGGL((fir_fold_batch_kernel<LONG, QM>), dim3(grid), dim3(256), 0, s, t);
        return hipGetLastError();
    };
    return max_m <= 16 ? go(std::false_type{}) : go(std::true_type{});
}

}  // namespace

// Per-mode entry points (fir_fold_*.hip).
hipError_t launch_fold_f32(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_bf16(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_bf16x2(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_f8bf16(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_batch_f8bf16(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s);
hipError_t launch_fold_batch_f32(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s);
hipError_t launch_fold_batch_bf16(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s);
hipError_t launch_fold_batch_bf16x2(const BatchTable* t, int max_m, bool split, int grid, hipStream_t s);

}  // namespace tina
