// Factored DFT across the branches (the paper allows a "Discrete or Fast"
// Fourier transform after the FIR, Sec. 5.2): the result of Eq. (12) by a
// mixed-radix FFT (decimation in time in Stockham's self-sorting order), two or
// three passes of radix 16 with a last pass of radix 2 to 16, in FP32.
//
// Memory-bound: a frame is read once (P values) and written once; about
// 5 P log2 P flops are a twentieth of the vector units' time at HBM speed.
// N = P points for a complex frame, P/2 for a real one (neighbouring samples
// as real and imaginary part, untangled at the end).  A thread holds 16 points
// in registers, N / 16 threads a frame, 256 threads a block, 256 / (N / 16)
// frames at a time; between passes the points change hands in LDS, one float2
// of padding after every 16 so that both the strided writes and the contiguous
// reads spread over the banks.  Frames of up to 64 threads (N <= 1024) lie in
// one wave and need no block barrier.  A thread's twiddles do not change from
// frame to frame and stay in registers; the grid is persistent.
//
// 2^26 complex samples, 4096 channels: this stage 0.74-0.87 ms as two
// 64-point products on the FP32 matrix units (their flops were the bound, 0.59
// of the peak).
#include <math.h>

#include <type_traits>

#include "internal.h"

namespace tina {
namespace {

// Multiply-adds are written out, so that every kernel rounds alike.
#pragma clang fp contract(off)

struct cf32 {
    float x, y;
};
__device__ __forceinline__ cf32 operator+(cf32 a, cf32 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cf32 operator-(cf32 a, cf32 b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cf32 mul(cf32 a, cf32 w) {
    return {__builtin_fmaf(a.x, w.x, -(a.y * w.y)), __builtin_fmaf(a.x, w.y, a.y * w.x)};
}
__device__ __forceinline__ cf32 mul_mi(cf32 a) { return {a.y, -a.x}; }  // times -i

__device__ __forceinline__ void dft2(cf32& a, cf32& b) {
    const cf32 s = a + b;
    b = a - b;
    a = s;
}
__device__ __forceinline__ void dft4(cf32& a, cf32& b, cf32& c, cf32& d) {
    const cf32 s = a + c, t = a - c, u = b + d, v = mul_mi(b - d);
    a = s + u;
    b = t + v;
    c = s - u;
    d = t - v;
}
// exp(-2 pi i e / 16)
__device__ __forceinline__ cf32 times_w16(cf32 a, int e) {
    constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508977f, r = 0.70710678118654752f;
    switch (e) {
        case 0: return a;
        case 1: return mul(a, {c1, -s1});
        case 2: return {r * (a.x + a.y), r * (a.y - a.x)};
        case 3: return mul(a, {s1, -c1});
        case 4: return mul_mi(a);
        case 6: return {r * (a.y - a.x), -r * (a.x + a.y)};
        default: return mul(a, {-c1, s1});  // 9
    }
}
// R-point DFT of v[0], v[1], ..., v[R-1] in place, natural order.
template <int R>
__device__ __forceinline__ void dft(cf32 (&v)[16], int at) {
    if constexpr (R == 2) {
        dft2(v[at], v[at + 1]);
    } else if constexpr (R == 4) {
        dft4(v[at], v[at + 1], v[at + 2], v[at + 3]);
    } else if constexpr (R == 8) {  // 2 x 4: X[k1 + 2 k2]
        cf32 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = v[at + i];
            b[i] = v[at + 4 + i];
            dft2(a[i], b[i]);
            b[i] = times_w16(b[i], 2 * i);
        }
        dft4(a[0], a[1], a[2], a[3]);
        dft4(b[0], b[1], b[2], b[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[at + 2 * i] = a[i];
            v[at + 2 * i + 1] = b[i];
        }
    } else if constexpr (R == 16) {  // 4 x 4: X[k1 + 4 k2]
        cf32 a[4][4];  // [k1][b]
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            cf32 t[4] = {v[b], v[b + 4], v[b + 8], v[b + 12]};
            dft4(t[0], t[1], t[2], t[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k][b] = times_w16(t[k], b * k);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            dft4(a[k][0], a[k][1], a[k][2], a[k][3]);
#pragma unroll
            for (int b = 0; b < 4; ++b) v[k + 4 * b] = a[k][b];
        }
    }
}

// cos, sin of 2 pi r / P in FP64, rounded to FP32.
__global__ void fft_twiddle_kernel(float* tw, int P) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= P) return;
    double s, c;
    sincospi(2.0 * (double)r / (double)P, &s, &c);
    tw[2 * r] = __double2float_rn(c);
    tw[2 * r + 1] = __double2float_rn(s);
}

template <int N, bool CPLX>
struct FftGeom {
    static constexpr int P = CPLX ? N : 2 * N;
    static constexpr int T = N / 16;          // threads per frame
    static constexpr int FPB = 256 / T;       // frames per block and turn
    static constexpr int R2 = N >= 256 ? 16 : N / 16;    // second pass (Ns = 16)
    static constexpr int R3 = N >= 256 ? N / 256 : 1;    // third pass (Ns = 256); 1: none
    static constexpr int ROW = N + N / 16;    // padded points of a frame in LDS
    static constexpr bool WAVE = T <= 64;     // a frame's threads lie in one wave
};

__device__ __forceinline__ int pad16(int i) { return i + (i >> 4); }

// The threads of a frame meet: all their LDS writes so far are seen.
template <bool WAVE>
__device__ __forceinline__ void frame_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

constexpr int kFftLds = 256 * 17;  // points: FPB * ROW of every N

// Frames f0 + g, f0 + g + step, ... below F of y and out (g < FPB: the thread's
// place in the block), by every thread of the block.
template <int N, bool CPLX>
__device__ __forceinline__ void fft_frames(const float* __restrict__ y, int64_t ldy, float* __restrict__ out, int64_t ldo,
                                           int64_t f0, int64_t F, int64_t step, const float* __restrict__ twf, cf32* lds,
                                           int tid) {
    using G = FftGeom<N, CPLX>;
    constexpr int T = G::T, R2 = G::R2, R3 = G::R3;
    constexpr int B2 = 16 / R2, B3 = R3 > 1 ? 16 / R3 : 1;  // butterflies per thread
    static_assert(G::FPB * G::ROW == kFftLds, "every N fills the same LDS");
    const cf32* tw = reinterpret_cast<const cf32*>(twf);
    const int t = tid % T, g = tid / T;
    cf32* buf = lds + g * G::ROW;
    constexpr int S = G::P / N;  // W_N^x = table entry S x
    auto w = [&](int x) {
        const cf32 e = tw[x & (G::P - 1)];
        return cf32{e.x, -e.y};
    };
    cf32 w2[B2][R2 > 1 ? R2 - 1 : 1], w3[B3][R3 > 1 ? R3 - 1 : 1];
#pragma unroll
    for (int b = 0; b < B2; ++b)
#pragma unroll
        for (int r = 1; r < R2; ++r) w2[b][r - 1] = w(((t + b * T) & 15) * r * (N / (16 * R2)) * S);
    if constexpr (R3 > 1) {
#pragma unroll
        for (int b = 0; b < B3; ++b)
#pragma unroll
            for (int r = 1; r < R3; ++r) w3[b][r - 1] = w((t + b * T) * r * S);
    }
    cf32 wu[CPLX ? 1 : 8];  // untangling
    if constexpr (!CPLX) {
#pragma unroll
        for (int i = 0; i < 8; ++i) wu[i] = w(t + i * T);
    }
    for (int64_t fb = f0; fb < F; fb += step) {  // the same turns for the whole block
        const int64_t f = fb + g;
        const bool on = f < F;
        float* const orow = out + f * ldo;
        cf32 v[16];
        if (on) {
            const cf32* z = reinterpret_cast<const cf32*>(y + f * ldy);
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = z[t + r * T];
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = {0.f, 0.f};
        }
        dft<16>(v, 0);
        frame_sync<G::WAVE>();  // the previous frame's last reads are done
#pragma unroll
        for (int r = 0; r < 16; ++r) buf[pad16(16 * t + r)] = v[r];
        frame_sync<G::WAVE>();
        // Second pass: butterfly j = t + b T of N / R2, points j + r N / R2.
#pragma unroll
        for (int b = 0; b < B2; ++b)
#pragma unroll
            for (int r = 0; r < R2; ++r) {
                const cf32 x = buf[pad16(t + b * T + r * (N / R2))];
                v[b * R2 + r] = r ? mul(x, w2[b][r - 1]) : x;
            }
#pragma unroll
        for (int b = 0; b < B2; ++b) dft<R2>(v, b * R2);
        if constexpr (R3 > 1) {
            frame_sync<G::WAVE>();
#pragma unroll
            for (int r = 0; r < 16; ++r) buf[pad16((t >> 4) * 256 + (t & 15) + 16 * r)] = v[r];
            frame_sync<G::WAVE>();
#pragma unroll
            for (int b = 0; b < B3; ++b)
#pragma unroll
                for (int r = 0; r < R3; ++r) {
                    const cf32 x = buf[pad16(t + b * T + r * 256)];
                    v[b * R3 + r] = r ? mul(x, w3[b][r - 1]) : x;
                }
#pragma unroll
            for (int b = 0; b < B3; ++b) dft<R3>(v, b * R3);
        }
        // v[b R + r] is point j + r N / R, j = t + b T, of the last pass.
        constexpr int RL = R3 > 1 ? R3 : R2, BL = 16 / RL;
        if constexpr (CPLX) {
            if (on) {
                cf32* o = reinterpret_cast<cf32*>(orow);
#pragma unroll
                for (int b = 0; b < BL; ++b)
#pragma unroll
                    for (int r = 0; r < RL; ++r) o[t + b * T + r * (N / RL)] = v[b * RL + r];
            }
        } else {
            // Untangle: Z_k of z = y_even + i y_odd; with E = (Z_k + Z*_{N-k}) / 2,
            // O = -i (Z_k - Z*_{N-k}) / 2: X_k = E + W_P^k O, X_{N-k} = (E - W_P^k O)*.
            frame_sync<G::WAVE>();
#pragma unroll
            for (int b = 0; b < BL; ++b)
#pragma unroll
                for (int r = 0; r < RL; ++r) buf[pad16(t + b * T + r * (N / RL))] = v[b * RL + r];
            frame_sync<G::WAVE>();
            if (on) {
                cf32* o = reinterpret_cast<cf32*>(orow);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int k = t + i * T;
                    const cf32 a = buf[pad16(k)], c = buf[pad16((N - k) & (N - 1))];
                    const cf32 e = {0.5f * (a.x + c.x), 0.5f * (a.y - c.y)}, d = {0.5f * (a.x - c.x), 0.5f * (a.y + c.y)};
                    const cf32 wo = mul(mul_mi(d), wu[i]);
                    if (k == 0) {
                        o[0] = {a.x + a.y, 0.0f};
                        o[N] = {a.x - a.y, 0.0f};
                        const cf32 m = buf[pad16(N / 2)];
                        o[N / 2] = {m.x, -m.y};
                    } else {
                        o[k] = e + wo;
                        const cf32 x = e - wo;
                        o[N - k] = {x.x, -x.y};
                    }
                }
            }
        }
    }
}

template <int N, bool CPLX>
__global__ __launch_bounds__(256) void fft_kernel(FftArgs a) {
    __shared__ __attribute__((aligned(16))) cf32 lds[kFftLds];
    constexpr int64_t FPB = FftGeom<N, CPLX>::FPB;
    fft_frames<N, CPLX>(a.y, a.ldy, a.out, a.ldo, blockIdx.x * FPB, a.F, gridDim.x * FPB, a.tw, lds, threadIdx.x);
}

// The frames of several batch items in one launch, whatever their channel
// counts (one launch per count took 7-16 us each in a server's steps, most of
// it latency): a unit is `turns` times as many frames of one item as a block
// holds.  The arithmetic of a frame is fft_kernel's: a batched item's output is
// bit for bit that of its own call.
__global__ __launch_bounds__(256) void fft_batch_kernel(const FftItem* __restrict__ items, int n, int64_t units) {
    __shared__ __attribute__((aligned(16))) cf32 lds[kFftLds];
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        int lo = 0, hi = n - 1;
        while (lo < hi) {  // the last item whose first unit is <= u
            const int mid = (lo + hi + 1) >> 1;
            if (items[mid].unit0 <= u) lo = mid;
            else hi = mid - 1;
        }
        const FftItem it = items[lo];
        // A thread index the compiler cannot see through, so that it does not move
        // the address arithmetic of all ten cases out of the loop (512 registers).
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        auto go = [&](auto n_tag, auto c_tag) {
            constexpr int N = decltype(n_tag)::value;
            constexpr bool CPLX = decltype(c_tag)::value;
            constexpr int64_t FPB = FftGeom<N, CPLX>::FPB;
            const int64_t f0 = (u - it.unit0) * it.turns * FPB, f1 = min(it.F, f0 + it.turns * FPB);
            fft_frames<N, CPLX>(it.y, it.ldy, it.out, it.ldo, f0, f1, FPB, it.tw, lds, tid);
        };
        __syncthreads();  // the previous unit's reads of LDS are done (its frames may have lain in single waves)
        using std::integral_constant;
        switch (it.cplx ? it.P : -it.P) {
            case 256: go(integral_constant<int, 256>{}, std::true_type{}); break;
            case 512: go(integral_constant<int, 512>{}, std::true_type{}); break;
            case 1024: go(integral_constant<int, 1024>{}, std::true_type{}); break;
            case 2048: go(integral_constant<int, 2048>{}, std::true_type{}); break;
            case 4096: go(integral_constant<int, 4096>{}, std::true_type{}); break;
            case -256: go(integral_constant<int, 128>{}, std::false_type{}); break;
            case -512: go(integral_constant<int, 256>{}, std::false_type{}); break;
            case -1024: go(integral_constant<int, 512>{}, std::false_type{}); break;
            case -2048: go(integral_constant<int, 1024>{}, std::false_type{}); break;
            default: go(integral_constant<int, 2048>{}, std::false_type{}); break;
        }
    }
}

template <int N, bool CPLX>
hipError_t launch_fft_n(const FftArgs& a, hipStream_t s) {
    constexpr int64_t FPB = FftGeom<N, CPLX>::FPB;
    const int64_t turns = (a.F + FPB - 1) / FPB;
    const int64_t grid = turns < 4 * (int64_t)a.cus ? turns : 4 * (int64_t)a.cus;  // four blocks per CU (34 KiB of LDS each)
    hipLaunchKernelGGL((fft_kernel<N, CPLX>), dim3((unsigned)grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

bool fft_supported(int P) { return P >= 256 && P <= 4096 && (P & (P - 1)) == 0; }

hipError_t launch_twiddle_table(float* tw, int P, hipStream_t s) {
    hipLaunchKernelGGL(fft_twiddle_kernel, dim3((P + 255) / 256), dim3(256), 0, s, tw, P);
    return hipGetLastError();
}

int fft_frames_per_block(int P, bool cplx) { return 4096 / (cplx ? P : P / 2); }

hipError_t launch_fft_dft(const FftArgs& a, hipStream_t s) {
    if (a.F <= 0) return hipSuccess;
    switch (a.P) {
        case 256: return a.cplx ? launch_fft_n<256, true>(a, s) : launch_fft_n<128, false>(a, s);
        case 512: return a.cplx ? launch_fft_n<512, true>(a, s) : launch_fft_n<256, false>(a, s);
        case 1024: return a.cplx ? launch_fft_n<1024, true>(a, s) : launch_fft_n<512, false>(a, s);
        case 2048: return a.cplx ? launch_fft_n<2048, true>(a, s) : launch_fft_n<1024, false>(a, s);
        case 4096: return a.cplx ? launch_fft_n<4096, true>(a, s) : launch_fft_n<2048, false>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fft_batch(const FftItem* items, int n, int64_t units, int cus, hipStream_t s) {
    if (units <= 0) return hipSuccess;
    const int64_t grid = units < 4 * (int64_t)cus ? units : 4 * (int64_t)cus;
    hipLaunchKernelGGL(fft_batch_kernel, dim3((unsigned)grid), dim3(256), 0, s, items, n, units);
    return hipGetLastError();
}

}  // namespace tina
