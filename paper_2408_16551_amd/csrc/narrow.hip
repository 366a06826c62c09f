// FIR and dense DFT in one kernel for narrow frames (at most 128 floats: up to 128
// real or 64 complex channels; FP32, BF16, BF16x3).  The output must lie apart from
// the input: a block writes its channels while others still read.
//
// A frame of at most 128 floats is a short row of a small product: the tiles
// of the two-kernel path are mostly padding (128 x 256 against 16 columns) and
// its FIR output a round trip of its own.  Here a block stages the input of
// R = 256 L / W consecutive frames and the M - 1 before them in LDS, every
// thread forms L outputs of the FIR (column c of every 256/W-th row, so that a
// wave reads consecutive words), stores them in the operand form, the waves
// take the 32 x 32 tiles of the product (operand fragments straight from L2),
// and the rows leave as one contiguous copy.  Memory-bound: input read once,
// channels written once.  Multiply-adds, roundings and the K order of the
// products are the two-kernel path's: same bits.  2^25 real samples, FP32: 16
// channels, 4 taps 404 -> 83 us; 64 channels, 8 taps 229 -> 114 us (bytes at the
// rate of a copy: 53 us; the FIR's LDS reads, M a float, and at 128 floats the
// product bound the rest).
#include "internal.h"

#include <type_traits>

namespace tina {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any float's address
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int FORM> struct NF;
template <> struct NF<FORM_FP32> { static constexpr int EB = 4, NP = 1; };
template <> struct NF<FORM_BF16> { static constexpr int EB = 2, NP = 1; };
template <> struct NF<FORM_BF16X3> { static constexpr int EB = 2, NP = 2; };

struct NarrowArgs {
    FirArgs x;   // y, q unused
    GemmArgs g;  // A unused
};

// LDS: input rows (later the output rows), then the operand pieces, W + 16 / EB
// elements a row.
template <int FORM>
size_t narrow_lds(int W, int M, int64_t ldo, int R) {
    const int64_t in = (int64_t)(R + M - 1) * W, out = R * ldo;
    return 4 * (size_t)(((in > out ? in : out) + 3) / 4 * 4) + (size_t)NF<FORM>::NP * R * (W * NF<FORM>::EB + 16);
}

template <int FORM, int L>
__global__ __launch_bounds__(256) void narrow_kernel(NarrowArgs na) {
    constexpr int EB = NF<FORM>::EB, NP = NF<FORM>::NP;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FirArgs& a = na.x;
    const GemmArgs& g = na.g;
    const int W = a.W, M = a.M, R = 256 * L / W, RS = W * EB + 16;
    const int tid = threadIdx.x;
    const int64_t f0 = blockIdx.x * (int64_t)R;
    const int nrow = (int)min((int64_t)R, a.F - f0);
    float* xs = reinterpret_cast<float*>(lds);
    const int64_t in = (int64_t)(R + M - 1) * W, outf = R * g.ldo;
    uint8_t* As = lds + 4 * (((in > outf ? in : outf) + 3) / 4 * 4);

    // Input: float e0 + i of prefix ++ chunk, zeros past the last frame.
    const int64_t e0 = (a.g0 + f0) * (int64_t)W;
    const int valid = (nrow + M - 1) * W, total = (R + M - 1) * W;
    const float* src = a.chunk + (e0 - a.plen);
    if (e0 >= a.plen) {
        for (int i = tid; i < total / 4; i += 256)
            reinterpret_cast<f32x4*>(xs)[i] =
                4 * i < valid ? __builtin_nontemporal_load(reinterpret_cast<const f32x4_a4*>(src + 4 * i)) : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
        for (int i = tid; i < total; i += 256) {
            const int64_t e = e0 + i;
            xs[i] = i >= valid ? 0.0f : e >= a.plen ? a.chunk[e - a.plen] : a.prefix ? a.prefix[e] : 0.0f;
        }
    }
    __syncthreads();

    // FIR, tap 0 times the newest frame first (as fir_point).
    const int c = tid & (W - 1), q = tid / W, RB = 256 / W;
    float acc[L];
    {
        const float* xr = xs + (M - 1) * W + tid;  // row q of the tile, column c
        const float* tp = a.taps + (int64_t)(M - 1) * a.P + c / a.cf;
        const float t0 = *tp;
#pragma unroll
        for (int l = 0; l < L; ++l) acc[l] = t0 * xr[256 * l];
        for (int m = 1; m < M; ++m) {
            const float t = tp[-(int64_t)m * a.P];
#pragma unroll
            for (int l = 0; l < L; ++l) acc[l] = fmaf(t, xr[256 * l - m * W], acc[l]);
        }
    }
#pragma unroll
    for (int l = 0; l < L; ++l) {
        uint8_t* at = As + (l * RB + q) * RS + c * EB;
        if constexpr (FORM == FORM_FP32) {
            *reinterpret_cast<float*>(at) = acc[l];
        } else {
            const uint16_t hi = __builtin_bit_cast(uint16_t, (__bf16)acc[l]);
            *reinterpret_cast<uint16_t*>(at) = hi;
            if constexpr (NP == 2)
                *reinterpret_cast<uint16_t*>(at + R * RS) =
                    __builtin_bit_cast(uint16_t, (__bf16)(acc[l] - __builtin_bit_cast(float, (uint32_t)hi << 16)));
        }
    }
    __syncthreads();

    // Product: 32 x 32 tiles, the slabs of 32 bytes of a row in order.
    const int lane = tid & 63, wave = tid >> 6, lr = lane & 31, lh = lane >> 5;
    const int ct = (W + 31) / 32, nt = R / 32 * ct, ns = W * EB / 32;
    const uint8_t* Bp[2] = {(const uint8_t*)g.B0, (const uint8_t*)g.B1};
    for (int ti = wave; ti < nt; ti += 4) {
        const int n = ti % ct * 32 + lr, r0 = ti / ct * 32;
        const bool col = n < g.N;
        const int64_t bo = (int64_t)(col ? n : 0) * W * EB + lh * 16;  // columns past the last: read, not stored
        const uint8_t* ar = As + (r0 + lr) * RS + lh * 16;
        f32x16 d;
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll 4
        for (int s = 0; s < ns; ++s) {
            uint4 av[NP], bv[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                av[p] = *reinterpret_cast<const uint4*>(ar + p * R * RS + s * 32);
                bv[p] = *reinterpret_cast<const uint4*>(Bp[p] + bo + s * 32);
            }
            if constexpr (FORM == FORM_FP32) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    d = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, av[0])[e],
                                                             __builtin_bit_cast(f32x4, bv[0])[e], d, 0, 0, 0);
            } else {
#pragma unroll
                for (int term = 0; term < (NP == 2 ? 3 : 1); ++term)
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[term == 2 ? 1 : 0]),
                                                                __builtin_bit_cast(bf16x8, bv[term == 1 ? 1 : 0]), d, 0, 0, 0);
            }
        }
        if (col) {
            const int oc = g.real_pack && n < 2 ? (n == 0 ? 0 : (int)g.N) : n;
            float* o = xs + oc;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = r0 + 8 * (v >> 2) + 4 * lh + (v & 3);
                o[row * g.ldo] = d[v];
                if (g.real_pack && n < 2) o[row * g.ldo + 1] = 0.0f;  // Im X_0, Im X_{P/2}
            }
        }
    }
    __syncthreads();
    float* out = g.out + f0 * g.ldo;  // 8-byte aligned, whole pairs
    const int pairs = (int)(nrow * g.ldo / 2);
    for (int i = tid; i < pairs; i += 256)
        __builtin_nontemporal_store(reinterpret_cast<const f32x2*>(xs)[i], reinterpret_cast<f32x2*>(out) + i);
}

template <int FORM, int L>
hipError_t launch_narrow_l(const NarrowArgs& na, hipStream_t s) {
    const int R = 256 * L / na.x.W;
    const size_t lds = narrow_lds<FORM>(na.x.W, na.x.M, na.g.ldo, R);
    static const hipError_t attr = hipFuncSetAttribute((const void*)narrow_kernel<FORM, L>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((narrow_kernel<FORM, L>), dim3((unsigned)((na.x.F + R - 1) / R)), dim3(256), lds, s, na);
    return hipGetLastError();
}

template <int FORM>
hipError_t launch_narrow_form(const NarrowArgs& na, hipStream_t s) {
    // The smallest blocks with 32 rows: several on a CU cover each other's
    // phases (64 real channels, 8 taps, 2^25 samples, FP32: 144, 119 and 114 us
    // with 32, 16 and 8 outputs a thread).  Narrower rows: 8 outputs, 4 while 8
    // leave CUs without a block.
    if (na.x.W == 128) return launch_narrow_l<FORM, 16>(na, s);
    if (na.x.W == 64 || na.x.F * na.x.W >= 512 * 2048) return launch_narrow_l<FORM, 8>(na, s);
    return launch_narrow_l<FORM, 4>(na, s);
}

}  // namespace

bool narrow_supported(const FirArgs& x, const GemmArgs& g) {
    // 128 complex channels: the operand fragments of 256 x 256 entries a block of
    // 32 rows reads from L2 take longer than the round trip saved (2^24 samples,
    // 8 taps: FP32 278 against 225 us, BF16x3 219 against 132 us).
    // Frames of 128 floats in the 16-bit forms with 9 to 16 or 32 taps (exact rings in
    // the two kernels' FIR): its LDS reads, M a float, bound a long call here.  2^25
    // floats, one and two kernels: BF16 12 taps 102 and 96 us, 16 taps 122 and 109, 32
    // taps 172 and 111; BF16x3 141 and 133, 159 and 148, 205 and 142; at 2^23 9 to 16
    // taps 26-47 and 31-44, 32 taps from 2^22 on 22-36 and 23-30.  Also 32 taps over
    // 128 floats in FP32 (123 and 119 at 2^24) and over 64 in BF16 (71 and 64).
    const int64_t fl = x.F * x.W;
    const bool wide = x.W == 128, f32 = g.form == FORM_FP32;
    if (fl >= 1 << 24 && ((wide && !f32 && x.M >= 9 && x.M <= 16) ||
                          (x.M == 32 && (wide || (x.W == 64 && g.form == FORM_BF16)))))
        return false;
    if (fl >= 1 << 22 && wide && !f32 && x.M == 32) return false;
    return x.W <= 128 && x.M <= 32 && !g.compensated && g.K == x.W && g.N == x.W &&
           (g.form == FORM_FP32 || g.form == FORM_BF16 || g.form == FORM_BF16X3);
}

hipError_t launch_narrow(const FirArgs& x, const GemmArgs& g, hipStream_t s) {
    if (x.F <= 0) return hipSuccess;
    if (!narrow_supported(x, g) || !g.B0) return hipErrorInvalidValue;
    NarrowArgs na;
    na.x = x;
    na.g = g;
    switch (g.form) {
        case FORM_FP32: return launch_narrow_form<FORM_FP32>(na, s);
        case FORM_BF16: return launch_narrow_form<FORM_BF16>(na, s);
        default: return launch_narrow_form<FORM_BF16X3>(na, s);
    }
}

}  // namespace tina
