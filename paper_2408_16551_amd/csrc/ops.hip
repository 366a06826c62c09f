// Standalone building blocks: unfold (Sec. 4.4, Eq. (17)) and a direct FIR
// filter with arbitrary taps (Sec. 4.3, Eq. (15)).
//
// Unfold: Y[i][j] = x[i*stride + j].  A pure gather whose output is
// width/stride times the input; each thread writes 4 consecutive outputs
// (one 16-byte store when a row holds whole groups of 4).
//
// FIR: y[i] = sum_k a[k] x[i-k].  Up to 16 taps (complex samples: 9) as it stands, on
// the vector units; beyond as a product with the Toeplitz matrix of the taps on the
// FP32 matrix units: 16 consecutive outputs are the rows of a 16 x 16 MFMA tile, 16
// such runs its columns,
//   Y[m][n] = sum_q T[m][q] x[16 n - H + q],  T[m][q] = a[H + m - q], H >= K - 1,
// q < H + 16 in slabs of 16.  The vector units (no packed FP32) reach half the
// matrix units' rate, of which the product wastes 15 / (K + 15); with 129 taps
// over 2^24 samples the vector form took 126 us (34 TFLOP/s, two LDS reads a
// multiply-add), against 26 us for the bytes at the rate of a copy.
#include <stdlib.h>
#include <string.h>

#include <new>
#include <string>

#include "runtime_types.h"
#include "tina_ops.h"

using namespace tina;

namespace {

__global__ __launch_bounds__(256) void unfold_kernel(const float* __restrict__ x, int64_t width, int64_t stride,
                                                     float* __restrict__ y, int64_t total, bool vec) {
    const int64_t n4 = (total + 3) / 4;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n4; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = 4 * t;
        if (vec) {  // width % 4 == 0 and y 16-byte aligned: the 4 outputs share one row
            const int64_t row = e / width, col = e - row * width;
            const float* src = x + row * stride + col;
            *reinterpret_cast<float4*>(y + e) = make_float4(src[0], src[1], src[2], src[3]);
        } else {
            for (int64_t k = e; k < e + 4 && k < total; ++k) {
                const int64_t row = k / width, col = k - row * width;
                y[k] = x[row * stride + col];
            }
        }
    }
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any float's address

// Few taps: four floats a thread straight from its loads, no LDS and no barrier; of a
// thread's loads all but one hit L1, whose rate bounds it as the taps grow.  Bound by HBM
// in long calls, by one load's latency in short ones.  us here, by the product below and
// as the LDS form with a multiply-add a tap that preceded both:
//                                        8 taps              9 taps           16 taps
//   4 M real, one buffer            5.1   8.3   7.4    5.1   8.3   7.7    5.9   8.3   9.2
//   4 M real, buffers in turn       7.8   9.7  10.9    7.8   9.8  11.1    8.1   9.7  12.7
//   2 M complex, one buffer         5.9   7.8   7.4    5.9   7.8   7.6    7.6   7.8   9.2
//   2 M complex, buffers in turn    8.2   9.7  10.9    8.2   9.9  11.2   10.5   9.7  12.7
//   2^26 real                      88.6  93.0   133   85.7  93.0   134   90.8  93.1   141
//   2^26 complex                    182   182   260    181   182   264    266   182   276
// 18 real taps take 98 over 2^26 (92), 10 complex ones 197 (183): the lines below.
constexpr int direct_taps(int cf) { return cf == 1 ? 16 : 9; }
template <int K, int CF>
__global__ __launch_bounds__(256) void fir_direct_kernel(const float* __restrict__ x, int64_t nf,
                                                         const float* __restrict__ taps, float* __restrict__ y) {
    constexpr int H = (CF * (K - 1) + 3) & ~3, L = H / 4 + 1;
    const int64_t b0 = (int64_t)blockIdx.x * 1024, at0 = b0 + 4 * threadIdx.x;
    float t[K];
#pragma unroll
    for (int k = 0; k < K; ++k) t[k] = taps[k];
    auto run = [&](auto edge) {
        f32x4 w[L], acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const int64_t at = at0 - H + 4 * l;  // a multiple of 4
            if (!edge || (at >= 0 && at + 4 <= nf)) {
                w[l] = *reinterpret_cast<const f32x4_a4*>(x + at);
            } else {
                w[l] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (at >= 0)
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (at + e < nf) w[l][e] = x[at + e];
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(t[k], w[(H + e - CF * k) / 4][(H + e - CF * k) % 4], acc[e]);
        if (!edge || at0 + 4 <= nf) {
            *reinterpret_cast<f32x4_a4*>(y + at0) = acc;
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (at0 + e < nf) y[at0 + e] = acc[e];
        }
    };
    if (b0 >= H && b0 + 1024 <= nf) run(std::false_type{});
    else run(std::true_type{});
}

// Four waves of NT column tiles (256 outputs each; complex: NT / 2 for the real
// and NT / 2 for the imaginary parts).  LDS: the block's input, one plane per
// part (from H samples before the block's first output, H = K - 1 rounded up to
// a multiple of 4 so that a float4 of the input is one of a plane), then the taps reversed,
// rt[15 + q] = a[H-q] with zeros around.  A 16-byte read of a lane
// serves four MFMAs (lane group kk holds q = k0 + 4 kk + step on both sides), a
// wave's 64 reads are 1 KB in a row, and a lane's four accumulators are four
// consecutive outputs.
// The zeros of T would turn an infinite or NaN sample into NaN beyond its
// reach, so a block that stages one takes the sums one by one.
template <int NT, int CF>
__global__ __launch_bounds__(256) void fir_toeplitz_kernel(const float* __restrict__ x, int64_t n,
                                                           const float* __restrict__ taps, int K, int S,
                                                           float* __restrict__ y) {
    constexpr int NC = NT / CF, NBP = 4 * NC * 256;  // column tiles and block outputs per plane
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const int plane = NBP + 16 * S, H = (K + 2) & ~3;
    float* rt = sm + CF * plane;
    const int64_t i0 = (int64_t)blockIdx.x * NBP;
    bool odd = false;
    auto check = [&](float v) { odd |= (__builtin_bit_cast(uint32_t, v) & 0x7f800000u) == 0x7f800000u; };
    const int have = NBP + H;  // samples of a plane that an output reaches
    // A block's samples and taps are all in flight before the first LDS store, four
    // floats a load whatever their alignment, in the first and the last block too:
    // calls of a few blocks a CU are bound by these latencies, one after another.
    // Buffers in turn: 2 M complex samples, 12 taps 11.5 -> 9.7 us (as float4s on 16 bytes
    // alone, the edges float by float, the taps after the samples), 65536 complex 4.8 ->
    // 3.3, 4 M real a float off 16 bytes 18.2 -> 10.2.
    const int64_t lo = (i0 - H) * CF, nf = n * CF;  // lo: a multiple of 4
    constexpr int U = CF * NBP / 4 / 256;
    auto tap = [&](int i) {
        const int k = H - (i - 15);
        return (k >= 0 && k < K) ? taps[k] : 0.0f;
    };
    // (Long filters in large blocks, which the products bound, load them after: 2^24
    // real samples, 129 taps 48.7 us against 50.1, 300 taps 88.1 against 90.5; 64 taps
    // 34.3 against 34.2.)
    const bool early = NT < 4 || K <= 96;
    float tap0 = early ? tap(threadIdx.x) : 0.0f;
    auto put = [&](int i, f32x4 v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) check(v[e]);
        if constexpr (CF == 1) {
            *reinterpret_cast<f32x4*>(sm + 4 * i) = v;
        } else {
            *reinterpret_cast<f32x2*>(sm + 2 * i) = f32x2{v[0], v[2]};
            *reinterpret_cast<f32x2*>(sm + plane + 2 * i) = f32x2{v[1], v[3]};
        }
    };
    auto stage = [&](auto fetch, auto tail) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = fetch(256 * u + threadIdx.x);
        for (int i = 256 * U + threadIdx.x; i < CF * have / 4; i += 256) put(i, tail(i, fetch(i)));
#pragma unroll
        for (int u = 0; u < U; ++u) put(256 * u + threadIdx.x, tail(256 * u + threadIdx.x, v[u]));
    };
    if (lo >= 0 && lo + CF * have <= nf) {
        stage([&](int i) -> f32x4 { return *reinterpret_cast<const f32x4_a4*>(x + lo + 4 * i); },
              [](int, f32x4 v) { return v; });
    } else {
        stage(
            [&](int i) -> f32x4 {
                const int64_t at = lo + 4 * i;
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
                if (at >= 0 && at + 4 <= nf) v = *reinterpret_cast<const f32x4_a4*>(x + at);
                return v;
            },
            [&](int i, f32x4 v) {
                const int64_t at = lo + 4 * i;
                if (at >= 0 && at < nf && at + 4 > nf)  // the input ends within
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (at + e < nf) v[e] = x[at + e];
                return v;
            });
    }
    for (int i = threadIdx.x; i < CF * (plane - have); i += 256) sm[(i % CF) * plane + have + i / CF] = 0.0f;
    if (!early) tap0 = tap(threadIdx.x);
    if ((int)threadIdx.x < 16 * S + 16) rt[threadIdx.x] = tap0;
    for (int i = threadIdx.x + 256; i < 16 * S + 16; i += 256) rt[i] = tap(i);
    if (__syncthreads_or(odd)) {
        for (int i = threadIdx.x; i < CF * NBP; i += 256) {
            const int p = i / CF, c = i % CF;
            if (i0 + p >= n) continue;
            const float* b = sm + c * plane + p + H;
            float acc = 0.0f;
            for (int k = 0; k < K; ++k) acc = fmaf(rt[15 + H - k], b[-k], acc);
            y[(i0 + p) * CF + c] = acc;
        }
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, kk = lane >> 4;
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* tp = rt + 15 + 4 * kk - m;
    const float* xp = sm + wave * NC * 256 + 16 * m + 4 * kk;
    for (int k0 = 0; k0 < 16 * S; k0 += 16) {
        float a[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = tp[k0 + s];
        f32x4 b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
            b[t] = *reinterpret_cast<const f32x4*>(xp + (t / NC) * plane + (t % NC) * 256 + k0);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[t][s], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < NC; ++t) {
        const int64_t i = i0 + wave * NC * 256 + t * 256 + 16 * m + 4 * kk;  // (column m of the tile)
        float v[4 * CF];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < CF; ++c) v[e * CF + c] = acc[c * NC + t][e];
        float* o = y + i * CF;
        if (i + 4 <= n) {
#pragma unroll
            for (int e = 0; e < CF; ++e)
                *reinterpret_cast<f32x4_a4*>(o + 4 * e) = f32x4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < n)
#pragma unroll
                    for (int c = 0; c < CF; ++c) o[e * CF + c] = v[e * CF + c];
        }
    }
}

int fir_slabs(int K) { return (((K + 2) & ~3) + 1 + 15 + 15) / 16; }
template <int NT, int CF>
size_t fir_lds(int K) {
    const size_t s16 = 16 * (size_t)fir_slabs(K);
    return sizeof(float) * (CF * (4 * (NT / CF) * 256 + s16) + s16 + 16);
}

template <int NT, int CF>
hipError_t launch_toeplitz(const float* x, int64_t n, const float* taps, int K, float* y, hipStream_t s) {
    constexpr int NBP = 4 * (NT / CF) * 256;
    hipLaunchKernelGGL((fir_toeplitz_kernel<NT, CF>), dim3((unsigned)((n + NBP - 1) / NBP)), dim3(256), (fir_lds<NT, CF>(K)),
                       s, x, n, taps, K, fir_slabs(K), y);
    return hipGetLastError();
}

template <int CF, int K = 1>
hipError_t launch_direct(const float* x, int64_t n, const float* taps, int k, float* y, hipStream_t s) {
    if constexpr (K <= direct_taps(CF)) {
        if (k != K) return launch_direct<CF, K + 1>(x, n, taps, k, y, s);
        const int64_t nf = n * CF;
        hipLaunchKernelGGL((fir_direct_kernel<K, CF>), dim3((unsigned)((nf + 1023) / 1024)), dim3(256), 0, s, x, nf, taps, y);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

}  // namespace

struct tina_fir_s {
    int device = 0;
    int K = 0, cf = 1;
    float* taps = nullptr;
};

extern "C" {

tina_status tina_unfold(const float* d_x, int64_t n, int64_t width, int64_t stride, float* d_y, int64_t cap,
                        int64_t* rows_out, void* stream) {
    if (n < 0 || width < 1 || stride < 1) return fail(TINA_ERR_INVALID_ARGUMENT, "unfold: need n >= 0, width >= 1, stride >= 1");
    const int64_t rows = n < width ? 0 : (n - width) / stride + 1;
    if (rows > 0 && (!d_x || !d_y)) return fail(TINA_ERR_INVALID_ARGUMENT, "unfold: NULL buffer");
    if (rows > cap) return fail(TINA_ERR_INVALID_ARGUMENT, "unfold: output capacity below " + std::to_string(rows) + " rows");
    if (rows_out) *rows_out = rows;
    if (rows == 0) return TINA_OK;
    const int64_t total = rows * width;
    const bool vec = (width % 4 == 0) && ((uintptr_t)d_y % 16 == 0);
    const int64_t blocks = std::min<int64_t>((total / 4 + 255) / 256 + 1, 1 << 20);
    hipLaunchKernelGGL(unfold_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, d_x, width, stride,
                       d_y, total, vec);
    HIP_TRY(hipGetLastError());
    return TINA_OK;
}

tina_status tina_fir_create(int device, const double* taps, int32_t K, int32_t sample_type, tina_fir_t* out) {
    if (!out || !taps) return fail(TINA_ERR_INVALID_ARGUMENT, "fir_create: NULL argument");
    *out = nullptr;
    if (K < 1 || K > 8192) return fail(TINA_ERR_UNSUPPORTED, "fir_create: taps must be in [1, 8192]");
    if (sample_type != TINA_SAMPLE_R32 && sample_type != TINA_SAMPLE_C64)
        return fail(TINA_ERR_INVALID_ARGUMENT, "fir_create: unknown sample type");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return fail(TINA_ERR_INVALID_ARGUMENT, "fir_create: bad device");
    DeviceScope ds(device);
    tina_fir_s* f = new (std::nothrow) tina_fir_s();
    if (!f) return fail(TINA_ERR_OUT_OF_MEMORY, "fir_create: host allocation");
    f->device = device;
    f->K = K;
    f->cf = sample_type == TINA_SAMPLE_C64 ? 2 : 1;
    float* h = (float*)malloc(sizeof(float) * K);
    if (!h) {
        delete f;
        return fail(TINA_ERR_OUT_OF_MEMORY, "fir_create: host allocation");
    }
    for (int k = 0; k < K; ++k) h[k] = (float)taps[k];
    hipError_t e = hipMalloc(&f->taps, sizeof(float) * K);
    if (e == hipSuccess) e = hipMemcpy(f->taps, h, sizeof(float) * K, hipMemcpyHostToDevice);
    free(h);
    if (e != hipSuccess) {
        if (f->taps) (void)hipFree(f->taps);
        delete f;
        return fail(TINA_ERR_OUT_OF_MEMORY, std::string("fir_create: ") + hipGetErrorString(e));
    }
    const int top = 8192;  // the longest filter's LDS: 68 to 112 KB
    (void)hipFuncSetAttribute((const void*)fir_toeplitz_kernel<4, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fir_lds<4, 1>(top));
    (void)hipFuncSetAttribute((const void*)fir_toeplitz_kernel<1, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fir_lds<1, 1>(top));
    (void)hipFuncSetAttribute((const void*)fir_toeplitz_kernel<4, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fir_lds<4, 2>(top));
    (void)hipFuncSetAttribute((const void*)fir_toeplitz_kernel<2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fir_lds<2, 2>(top));
    *out = f;
    return TINA_OK;
}

tina_status tina_fir_destroy(tina_fir_t f) {
    if (!f) return TINA_OK;
    DeviceScope ds(f->device);
    (void)hipDeviceSynchronize();
    (void)hipFree(f->taps);
    delete f;
    return TINA_OK;
}

tina_status tina_fir_execute(tina_fir_t f, const void* d_x, int64_t n, void* d_y, void* stream) {
    if (!f) return fail(TINA_ERR_INVALID_ARGUMENT, "fir_execute: NULL filter");
    if (n < 0) return fail(TINA_ERR_INVALID_ARGUMENT, "fir_execute: negative sample count");
    if (n == 0) return TINA_OK;
    if (!d_x || !d_y) return fail(TINA_ERR_INVALID_ARGUMENT, "fir_execute: NULL buffer");
    const int64_t nf = n * f->cf;
    const uintptr_t xa = (uintptr_t)d_x, ya = (uintptr_t)d_y;
    if (xa % 4 || ya % 4) return fail(TINA_ERR_INVALID_ARGUMENT, "fir_execute: buffers must be 4-byte aligned");
    if (xa < ya + (uintptr_t)nf * 4 && ya < xa + (uintptr_t)nf * 4)
        return fail(TINA_ERR_INVALID_ARGUMENT, "fir_execute: input and output overlap");
    DeviceScope ds(f->device);
    const float* x = (const float*)d_x;
    float* y = (float*)d_y;
    hipStream_t s = (hipStream_t)stream;
    // Blocks of 4096 floats from eight of them a CU on, below that of 1024 (2048
    // where complex): few large blocks a CU end together late (14 taps, buffers in
    // turn, us with large and small blocks: 2.8 M complex samples 13.7 and 13.1, 4 M
    // 16.9 and 16.2; 8 M real 15.4 and 15.6, 16.8 M 25.5 and 26.5; 40 taps: 4 M complex
    // 18.3 and 17.7, 12 M 41.6 and 42.2, 16.8 M real 29.6 and 32.7).
    const bool big = nf >= 2048 * 4096;
    hipError_t e;
    if (f->K <= direct_taps(f->cf))
        e = f->cf == 1 ? launch_direct<1>(x, n, f->taps, f->K, y, s) : launch_direct<2>(x, n, f->taps, f->K, y, s);
    else if (f->cf == 1) e = big ? launch_toeplitz<4, 1>(x, n, f->taps, f->K, y, s) : launch_toeplitz<1, 1>(x, n, f->taps, f->K, y, s);
    else e = big ? launch_toeplitz<4, 2>(x, n, f->taps, f->K, y, s) : launch_toeplitz<2, 2>(x, n, f->taps, f->K, y, s);
    HIP_TRY(e);
    return TINA_OK;
}

}  // extern "C"
