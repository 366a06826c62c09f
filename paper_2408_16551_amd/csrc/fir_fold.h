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
// P elements, part s at elements [s Q, (s+1) Q).
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

template <int VEC, int GW>
struct FoldGeom {
    static constexpr int GL = 64 * GW;      // lanes per column group
    static constexpr int GF = GL * VEC;     // floats per column group
    static constexpr int NTH = 4 * GL;      // threads per block
    static constexpr int SB = 16 / VEC;     // frames per LDS phase
};
template <int VEC, int GW>
struct FoldSmem {
    float ys[2][FoldGeom<VEC, GW>::SB][4 * FoldGeom<VEC, GW>::GF];
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
// significant bits of E4M3, on the bit pattern.
template <int VEC, int QM>
__device__ __forceinline__ typename VecT<VEC>::T fold_value(typename VecT<VEC>::T v) {
    if constexpr (QM == QM_F8BF16) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const uint32_t u = __builtin_bit_cast(uint32_t, vget<VEC>(v, i));
            vset<VEC>(v, i, __builtin_bit_cast(float, (u + 0x7ffffu + ((u >> 20) & 1u)) & 0xfff00000u));
        }
    }
    return v;
}

// Folds and stores `cnt` frames (first frame f0) of LDS buffer ys: column
// block at float offset c0 of each quarter frame.  A thread stores four
// elements of a part at a time: real frames four samples' four parts, complex
// ones two of the parts (even or odd channels) of four samples.
template <int VEC, int GW, int QM>
__device__ __forceinline__ void fold_store(const FirArgs& a, const float (&ys)[FoldGeom<VEC, GW>::SB][4 * FoldGeom<VEC, GW>::GF],
                                           int64_t f0, int cnt, int c0) {
    using G = FoldGeom<VEC, GW>;
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

// One unit: column block and run of logical block `blk`.  Every condition on
// frames is the same for the whole block, so all its threads meet at each
// barrier.  ph: the LDS buffer of the next phase (a buffer is written again
// two phases later, after every thread has passed the barrier in between, so
// one barrier per phase is enough, across units too).
template <int VEC, int GW, int MT, bool EXACT, int QM>
__device__ __forceinline__ void fir_fold_unit(const FirArgs& a, int TF, int64_t blk, FoldSmem<VEC, GW>& sm, int& ph) {
    using V = typename VecT<VEC>::T;
    using G = FoldGeom<VEC, GW>;
    constexpr int SB = G::SB < MT ? G::SB : MT;
    const int quarter = a.W / 4, ncb = quarter / G::GF;  // powers of two
    const int cb = (int)(blk & (ncb - 1));
    const int64_t run = blk / ncb;
    const int64_t f_begin = run * TF;
    if (f_begin >= a.F) return;
    const int64_t f_end = min(a.F, f_begin + TF);
    const int M = EXACT ? MT : a.M;
    const int c0 = cb * G::GF;
    const int g = threadIdx.x / G::GL, x = (threadIdx.x % G::GL) * VEC;
    const int j0 = (g == 0 ? c0 : g == 1 ? 2 * quarter - c0 - G::GF : g == 2 ? 2 * quarter + c0 : a.W - c0 - G::GF) + x;
    const int slot = g * G::GF + x;  // this thread's floats in an LDS row

    V tp[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) tp[m] = (EXACT || m < M) ? load_taps<VEC>(a, M, m, j0) : V(0.0f);
    V win[MT];  // ring of input frames, as in fir_unit
    auto direct = [&](int64_t f) {
        V acc = V(0.0f);
#pragma unroll
        for (int m = 0; m < MT; ++m)
            if (EXACT || m < M) acc = __builtin_elementwise_fma(tp[m], load_frame<VEC, true>(a, a.g0 + f - m, j0), acc);
        return acc;
    };
    auto flush = [&](int64_t f0, int cnt) {
        __syncthreads();
        fold_store<VEC, GW, QM>(a, sm.ys[ph], f0, cnt, c0);
        ph ^= 1;
    };
    // Frames [f0, f1) straight from their input frames: blocks that straddle
    // the prefix/chunk boundary, and the tail.
    auto slow = [&](int64_t f0, int64_t f1) {
        for (int64_t f = f0; f < f1; f += SB) {
            const int cnt = (int)min((int64_t)SB, f1 - f);
            for (int u = 0; u < cnt; ++u) *reinterpret_cast<V*>(&sm.ys[ph][u][slot]) = fold_value<VEC, QM>(direct(f + u));
            flush(f, cnt);
        }
    };
    bool ring_ok = false;
    int64_t fb = f_begin;
    for (; fb + MT <= f_end; fb += MT) {
        const int64_t fu = (int64_t)uniform64((uint64_t)fb);
        const int64_t eu = (a.g0 + fu + a.M - 1) * (int64_t)a.W - a.plen;  // block's first float in the chunk
        if (eu < 0) {
            ring_ok = false;
            slow(fb, fb + MT);
            continue;
        }
        if (!ring_ok) {
#pragma unroll
            for (int d = 1; d < MT; ++d)
                win[MT - d] = (EXACT || d < M) ? load_frame<VEC, false>(a, a.g0 + fb - d, j0) : V(0.0f);
        }
        ring_ok = true;
        const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.chunk + eu, (a.nchunk - eu) * 4);
        const uint32_t vin = (uint32_t)j0 * 4u;
        const int32_t w4 = a.W * 4;
#pragma unroll
        for (int sb = 0; sb < MT; sb += SB) {
            V in[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i)
                if (sb + i < MT) in[i] = buf_load<VEC, true>(rin, vin, (sb + i) * w4);
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int u = sb + i;
                if (u >= MT) continue;
                win[u] = in[i];
                *reinterpret_cast<V*>(&sm.ys[ph][i][slot]) = fold_value<VEC, QM>(fir_point<VEC, MT, EXACT>(tp, win, u, M));
            }
            flush(fb + sb, MT - sb < SB ? MT - sb : SB);
        }
    }
    slow(fb, f_end);
}

template <int VEC, int GW, int MT, bool EXACT, int QM>
__global__ __launch_bounds__((FoldGeom<VEC, GW>::NTH)) void fir_fold_kernel(FirArgs a, int TF) {
    __shared__ __attribute__((aligned(16))) FoldSmem<VEC, GW> sm;
    int ph = 0;
    fir_fold_unit<VEC, GW, MT, EXACT, QM>(a, TF, xcd_logical_block(blockIdx.x, gridDim.x), sm, ph);
}

template <int VEC, int M0, int MT, int QM>
__device__ __forceinline__ void fir_fold_unit_own_m(const FirArgs& a, int TF, int64_t blk, FoldSmem<VEC, 1>& sm, int& ph) {
    if constexpr (M0 <= MT) {
        if (a.M == M0) fir_fold_unit<VEC, 1, M0, true, QM>(a, TF, blk, sm, ph);
        else fir_fold_unit_own_m<VEC, M0 + 1, MT, QM>(a, TF, blk, sm, ph);
    }
}

// Persistent batched form, over the table's folded FIR units, with the ring
// unrolled for the item's own tap count up to 16, else 32 or 64 with the taps
// beyond M switched off.  One float per thread (any alignment); two, a complex
// sample, in the 16-bit forms (whole 128-byte lines of a part row).
template <int MAXM, int QM>
__global__ __launch_bounds__(256) void fir_fold_batch_kernel(const BatchTable* __restrict__ t) {
    constexpr int CV = QM == QM_NONE ? 1 : 2;  // floats per thread of complex items
    __shared__ __attribute__((aligned(16))) union {
        FoldSmem<1, 1> one;
        FoldSmem<CV, 1> cplx;
    } sm;
    int ph = 0;
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3, nbx = gridDim.x >> 3;
    const int64_t end = t->ffold_bounds[x + 1];
    for (int64_t u = t->ffold_bounds[x] + i; u < end; u += nbx) {
        const int it = batch_find(t->items, t->n_items, u, /*stage=*/4);
        const BatchItem& b = t->items[it];
        const FirArgs fa = b.fir;
        const int64_t blk = u - b.ffold_unit0;
        if (MAXM <= 16 || fa.M <= 16) {
            if (CV == 2 && fa.cf == 2) fir_fold_unit_own_m<CV, 1, 16, QM>(fa, b.fir_tf, blk, sm.cplx, ph);
            else fir_fold_unit_own_m<1, 1, 16, QM>(fa, b.fir_tf, blk, sm.one, ph);
        } else {
            if constexpr (MAXM == 32) fir_fold_unit<1, 1, 32, false, QM>(fa, b.fir_tf, blk, sm.one, ph);
            if constexpr (MAXM == 64) fir_fold_unit<1, 1, 64, false, QM>(fa, b.fir_tf, blk, sm.one, ph);
        }
    }
}

template <int VEC, int GW, int MT, bool EXACT, int QM>
hipError_t launch_fold_one(const FirArgs& a, hipStream_t s) {
    using G = FoldGeom<VEC, GW>;
    const int ncb = a.W / 4 / G::GF;
    // Frames per block: whole ring blocks, two of them (at least 16 frames) so
    // that the halo stays small; one while that leaves CUs without a block.
    int TF = 2 * MT < 16 ? ((16 + MT - 1) / MT) * MT : 2 * MT;
    while (TF > MT && TF > 4 && (a.F + TF - 1) / TF * ncb < 512) TF -= MT;
    const int64_t runs = (a.F + TF - 1) / TF;
    hipLaunchKernelGGL((fir_fold_kernel<VEC, GW, MT, EXACT, QM>), dim3((unsigned)(runs * ncb)), dim3(G::NTH), 0, s, a, TF);
    return hipGetLastError();
}

template <int VEC, int GW, int M0, int MTOP, int QM>
hipError_t launch_fold_m(const FirArgs& a, hipStream_t s) {
    if constexpr (M0 <= MTOP) {
        if (a.M == M0) return launch_fold_one<VEC, GW, M0, true, QM>(a, s);
        return launch_fold_m<VEC, GW, M0 + 1, MTOP, QM>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int QM>
hipError_t launch_fold_qm(const FirArgs& a, hipStream_t s) {
    auto aligned = [&](const void* p) { return ((uintptr_t)p & 15) == 0; };
    const bool al16 = a.plen % 4 == 0 && aligned(a.chunk) && (!a.prefix || aligned(a.prefix));
    if (a.M <= 8 && al16 && a.W >= 1024) return launch_fold_m<4, 1, 1, 8, QM>(a, s);
    // 16-bit complex rows: 128 lanes a group, so that a part row's piece of 64
    // samples fills a 128-byte line (1024 channels, 16 taps, 2^25 samples, BF16x3:
    // 163 us with 64 lanes and half lines, 129 us; FP32 rows the same either way).
    if (QM != QM_NONE && a.cf == 2 && a.M <= 16) return launch_fold_m<1, 2, 1, 16, QM>(a, s);
    if (a.M <= 16) return launch_fold_m<1, 1, 1, 16, QM>(a, s);
    if (a.M <= 32) return launch_fold_one<1, 1, 32, false, QM>(a, s);
    if (a.M <= 64) return launch_fold_one<1, 1, 64, false, QM>(a, s);
    return hipErrorInvalidValue;
}

template <int QM>
hipError_t launch_fold_batch_qm(const BatchTable* t, int max_m, int grid, hipStream_t s) {
    if (max_m <= 16) hipLaunchKernelGGL((fir_fold_batch_kernel<16, QM>), dim3(grid), dim3(256), 0, s, t);
    else if (max_m <= 32) hipLaunchKernelGGL((fir_fold_batch_kernel<32, QM>), dim3(grid), dim3(256), 0, s, t);
    else hipLaunchKernelGGL((fir_fold_batch_kernel<64, QM>), dim3(grid), dim3(256), 0, s, t);
    return hipGetLastError();
}

}  // namespace

// Per-mode entry points (fir_fold_*.hip).
hipError_t launch_fold_f32(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_bf16(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_bf16x2(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_f8bf16(const FirArgs& a, hipStream_t s);
hipError_t launch_fold_batch_f8bf16(const BatchTable* t, int max_m, int grid, hipStream_t s);
hipError_t launch_fold_batch_f32(const BatchTable* t, int max_m, int grid, hipStream_t s);
hipError_t launch_fold_batch_bf16(const BatchTable* t, int max_m, int grid, hipStream_t s);
hipError_t launch_fold_batch_bf16x2(const BatchTable* t, int max_m, int grid, hipStream_t s);

}  // namespace tina
