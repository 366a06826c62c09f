// Internal declarations shared by the library's translation units.
// Not part of the ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tina {

// Arithmetic forms of the DFT stage (same values as tina_precision).
enum Form : int {
    FORM_FP32 = 0, FORM_BF16 = 1, FORM_BF16X3 = 2, FORM_FP16 = 3, FORM_FP16X3 = 4, FORM_FP8 = 5, FORM_MXFP8 = 6
};

// Forms with a per-frame scale (the FIR also writes per-frame partial maxima).
inline bool form_scaled(int f) { return f == FORM_FP16 || f == FORM_FP16X3 || f == FORM_FP8; }
// Block-scaled FP8: the FIR writes E4M3 codes plus one E8M0 scale per 32
// floats of a frame, and the GEMM reads them as they are.
inline bool form_mx(int f) { return f == FORM_MXFP8; }
inline int form_pieces(int f) { return (f == FORM_BF16X3 || f == FORM_FP16X3) ? 2 : 1; }
inline int form_elem_bytes(int f) { return f == FORM_FP32 ? 4 : ((f == FORM_FP8 || f == FORM_MXFP8) ? 1 : 2); }
// Bytes of one block-scaled FP8 matrix of `rows` x `k` entries: codes, then
// one scale byte per 32 entries of each row.
inline int64_t mx_codes_bytes(int64_t rows, int64_t k) { return rows * k; }
inline int64_t mx_bytes(int64_t rows, int64_t k) { return rows * k + rows * (k / 32); }

// Map a hardware block index to a logical tile index so that the blocks the
// dispatcher places on one XCD (it deals blocks round-robin over the 8 XCDs)
// receive consecutive logical tiles, which then share that XCD's L2.
__device__ inline int64_t xcd_logical_block(int64_t b, int64_t nb) {
    const int64_t x = b & 7, i = b >> 3;
    const int64_t q = nb >> 3, rmd = nb & 7;
    return x * q + (x < rmd ? x : rmd) + i;
}

// ---------------------------------------------------------------- generation
// Prototype window h[n], n < P*M, in FP64 (sinc x window), plus its FP32 copy.
hipError_t launch_window(double* h64, float* h32, int P, int M, int window, hipStream_t s);
// FP32 copy of FP64 taps (custom window).
hipError_t launch_taps_to_f32(const double* h64, float* h32, int64_t L, hipStream_t s);
// DFT operand Bt[N][K] (row n = output column, K contiguous) in the pieces of
// `form`: piece0 (and piece1 for split forms), element size form_elem_bytes.
// FORM_MXFP8: piece0 = E4M3 codes [N][K], piece1 = E8M0 scales [N][K/32].
hipError_t launch_dft_operand(void* piece0, void* piece1, int P, int complex_input, int form,
                              hipStream_t s, int inverse = 0);
// Block-reversed FP32 taps of the synthesis FIR.
hipError_t launch_synthesis_taps(const double* h64, float* g32, int P, int M, hipStream_t s);

// ----------------------------------------------------------------------- FIR
struct FirArgs {
    const float* prefix;  // history + residue (floats); nullptr = zeros
    int64_t plen;         // floats in the prefix
    const float* chunk;   // new samples (floats)
    int64_t nchunk;       // floats in the chunk
    const float* taps;    // FP32 prototype h[0..P*M)
    float* y;             // output rows
    int64_t ldy;          // floats per output row
    int64_t g0;           // first output frame (frame numbering of prefix-residue ++ chunk)
    int64_t F;            // frames to produce
    int32_t W;            // floats per frame (P * cf)
    int32_t P, M, cf;     // channels, taps, floats per sample
    float* amax;          // optional per-frame partial |y| maxima [F][nparts]
    int32_t nparts;       // filled in by launch_fir
    // Operand-form output instead of y (qmode != 0): piece 0 at q and piece 1
    // at q1, [F][ldq elements] each; qmode 1 block-scaled FP8 (E4M3 codes plus
    // E8M0 scales [F][W/32] at qs), 2 bf16, 3 bf16 hi + lo.
    uint8_t* q;
    uint8_t* q1;
    int64_t ldq;
    uint8_t* qs;
    int32_t qmode;
    // Per-frame scaled operand output (qmode 4 FP8 E4M3, 5 fp16, 6 fp16 hi +
    // lo): launch_fir first finds every frame's maximum (into amax), then its
    // exponent e_f (fexp[f], the frame's values are scaled by 2^-e_f), then
    // writes the scaled codes.
    int32_t* fexp;
    const float* split_tw;  // folded output in two halves: cos, sin of 2 pi r / P, r < P (else nullptr)
};
// Chooses the vector width and unroll; returns the number of partial maxima
// per frame through a.nparts when a.amax is set.
hipError_t launch_fir(FirArgs& a, hipStream_t s);
// Number of partial maxima per frame launch_fir would produce.
int fir_amax_parts(const FirArgs& a);

// dst[i] = ext[start + i], i < count, where ext = prefix ++ chunk (floats).
hipError_t launch_gather_ext(const float* prefix, int64_t plen, const float* chunk, int64_t nchunk,
                             float* dst, int64_t start, int64_t count, hipStream_t s);

// ---------------------------------------------------------------------- GEMM
struct GemmArgs {
    const float* A;        // FIR output [F][K] FP32, row stride lda
    int64_t lda;
    const void* B0;        // Bt piece 0 [N][K]
    const void* B1;        // Bt piece 1 (split forms)
    float* out;            // output rows (floats), row stride ldo
    int64_t ldo;
    int64_t F;
    int32_t K, N;
    int32_t real_pack;     // real input: column 0 -> X_0, column 1 -> X_{P/2}, rest in place
    int32_t form;
    // A in operand form (every form but FP32, whose A is the FP32 rows
    // above): piece 0 / piece 1 [F][lda elements], and for FORM_MXFP8 the
    // E8M0 scales [F][K/32] (then B0/B1 = Bt codes / scales).
    const uint8_t* Aq;
    const uint8_t* Aq1;
    const uint8_t* Aqs;
    const int32_t* fexp;   // per-frame scaled forms with A in operand form: A row f carries 2^-fexp[f]
    int32_t compensated;   // FP32 only: compensated K accumulation (TwoSum per K tile)
    const float* tw;       // FP32 only, non-null: Bt assembled from this P x (cos, sin) twiddle table (B0 unused)
                           // (folded product: cos, sin of pi k / P, k < P/2, for every form)
    const float* ct;       // folded product, FP32 only, non-null: operand assembled from cos(pi r / P), r < 2P
    int32_t split;         // folded product, complex: frames in two halves (K = P/2, N = P/8)
    float inv;             // folded product, complex: 1/P for the inverse DFT (tw times 1/P), else 0
};
hipError_t launch_dft_gemm(const GemmArgs& a, hipStream_t s);

// ------------------------------------------------------------ folded product
// The dense DFT by its symmetry: four Q x Q products, Q = P / 4 (gemm_fold.hip)
// over operand rows the FIR writes folded (fir_fold.h): frames x cf rows of P
// elements.  GemmArgs: A / Aq, Aq1 those rows, B0, B1 the folded operand
// (launch_fold_operand), K = P, N = Q, real_pack, tw (and ct); lda unused.
//
// From 256 channels, in the forms whose operand element needs no frame or
// block scale.  Fewer channels: the column groups are narrower than a wave,
// and the dense product is no longer what bounds a call.
inline bool fold_form(int form) {
    return form == FORM_FP32 || form == FORM_BF16 || form == FORM_BF16X3 || form == FORM_FP8;
}
// Operand form of the folded product.  Per-frame FP8: sums of four E4M3 values
// (whose powers of two need no common frame scale any more) and the
// coefficients in bf16, a rounding an eighth of E4M3's.
inline int fold_operand_form(int form) { return form == FORM_FP8 ? FORM_BF16 : form; }
inline bool fold_supported(int P, int form) { return P >= 256 && fold_form(form); }
// Complex frames take one decimation in frequency before the fold: half the
// product's work for a FIR that writes its rows with twiddles.  FP32 from 512
// channels (the halves are bank sizes of the folded product), 2^25 samples, 16
// taps: 512 channels 316 -> 270 us, 1024 472 -> 360, 32 taps 654 -> 566.  The
// 16-bit products take less time than the FIR until 2048 channels (BF16x3: 1024
// channels 294 us unsplit, 298 split; 2048 398 -> 334, 4096 585 -> 426; BF16: 2048
// 247 and 249, 4096 329 -> 290; FP8 with 8 taps: 2048 251 -> 233), and the longer
// rings cost their FIR more than that gives.
inline bool fold_split(int P, int cf, int form, int M) {
    return cf == 2 && (form == FORM_FP32 ? P >= 512 : P >= 2048 && M <= 16);
}
// The FIR with folded output (a.y, or a.q / a.q1 with a.qmode; ldy, ldq unused).
hipError_t launch_fir_fold(const FirArgs& a, hipStream_t s);
hipError_t launch_dft_fold(const GemmArgs& a, hipStream_t s);
// Folded operand [Q][4 parts][Q] in the pieces of `form`, in FP64 rounded once.
hipError_t launch_fold_operand(void* piece0, void* piece1, int P, int form, hipStream_t s);
// tw: (cos, sin)(pi k / P) times scale (a power of two), k < P/2; ct (optional):
// cos(pi r / P), r < 2P; ones (optional): 2P times 1.
hipError_t launch_fold_tables(float* tw, float* ct, float* ones, int P, float scale, hipStream_t s);
// Floats per thread of the batched folded FIR (its column blocks are 256 times as wide).
inline int fold_batch_vec(int form, int cf, int M) { return form != FORM_FP32 && cf == 2 && M <= 16 ? 2 : 1; }
// ... and floats per column block of a split item: eight groups of 64 lanes.
constexpr int kFoldSplitCols = 8 * 64;
// Frames that a FIR unit of M <= 16 taps walks at a time: whole rings of M, as many
// as sb frames hold (sb: its loads in flight, or the frames of an LDS phase).
constexpr int fold_block_frames(int M, int sb) { return M < sb ? sb / M * M : M; }
// ... and that the batched FIR and folded FIR walk for an item; their units are whole
// numbers of them, whatever the launch's other items.
constexpr int fir_batch_block(int M) { return M > 16 ? 32 : fold_block_frames(M, 8); }
inline int fold_batch_ring(int form, int cf, bool split, int M) {
    return M > 16 ? 32 : fold_block_frames(M, split ? 8 : 16 / fold_batch_vec(form, cf, M));
}
// Tile rows and columns of the batched folded product for N columns.
__host__ __device__ inline void fold_batch_tile(int form, int64_t N, int64_t& bm, int64_t& bj) {
    bm = form != FORM_FP32 && N == 64 ? 256 : 128;
    bj = form == FORM_FP32 || N == 64 ? 64 : 128;
}
// Forms whose A the FIR can write in operand form.
bool gemm_raw_form(int form);

// FIR and dense product in one kernel for frames of at most 128 floats (x.y, x.q
// and g.A unused); bit for bit the two kernels.
bool narrow_supported(const FirArgs& x, const GemmArgs& g);
hipError_t launch_narrow(const FirArgs& x, const GemmArgs& g, hipStream_t s);

// ------------------------------------------------------------- factored DFT
struct FftArgs {
    const float* y;        // FIR output [F][ldy] (P real or P complex values per frame)
    int64_t ldy;
    int64_t F;
    const float* tw;       // cos, sin of 2 pi r / P
    float* out;            // output rows (complex64), row stride ldo floats
    int64_t ldo;
    int32_t P, cplx, cus;
};
bool fft_supported(int P);
// tw (P x 2): cos, sin of 2 pi r / P in FP64, rounded to FP32.
hipError_t launch_twiddle_table(float* tw, int P, hipStream_t s);
hipError_t launch_fft_dft(const FftArgs& a, hipStream_t s);
// Frames a 256-thread block of the factored DFT holds at a time.
int fft_frames_per_block(int P, bool cplx);
// One batch item's frames in a batched factored-DFT launch (device array,
// sorted by unit0): FIR output rows y, output rows out, twiddles tw, and the
// item's first unit of `turns` blocks' frames.
struct FftItem {
    const float* y;
    float* out;
    const float* tw;
    int64_t ldy, ldo, F, unit0;
    int32_t P, cplx, turns, pad_;
};
hipError_t launch_fft_batch(const FftItem* items, int n, int64_t units, int cus, hipStream_t s);

// --------------------------------------------------------------- batched path
// One item of a batched launch: the FIR and GEMM arguments of one stream
// chunk, its first work unit in each stage, and its state update.
struct BatchItem {
    FirArgs fir;            // fir.y points into the batch workspace
    GemmArgs gemm;          // gemm.A == fir.y
    int64_t fir_unit0;      // first FIR unit (256-thread block) of this item
    int64_t gemm_unit0;     // first GEMM tile of this item
    int64_t st_unit0;       // first state-update unit
    int32_t fir_tf;         // frames per FIR thread (fir_single: frames per frame-stage unit)
    int64_t ffold_unit0, fsplit_unit0, gfold_unit0;  // first unit / tile of the folded FIR (whole, split frames) / product
    int32_t fir_single;     // per-frame scaled form: one pass, whole frame rows per unit (frame stage)
    int64_t frame_unit0;    // first unit of the frame stage
    float* st_dst;          // state buffer to fill (nullptr: no state)
    int64_t st_start, st_count;
};

// Device-resident table read by the persistent kernels.  Each stage's units
// are split into 8 contiguous ranges of about equal cost, one per XCD.
struct BatchTable {
    int32_t n_items;
    int32_t pad_;
    int64_t fir_units, gemm_units, st_units, frame_units, ffold_units, fsplit_units, gfold_units;
    int64_t fir_bounds[9], gemm_bounds[9], st_bounds[9], frame_bounds[9], ffold_bounds[9], fsplit_bounds[9], gfold_bounds[9];
    int32_t gemm_bn;        // GEMM tile columns of this launch (kGemmBN or 2 * kGemmBN, or the wide tile's)
    int32_t gemm_wide;      // the launch uses the wide raw-operand tiles
    BatchItem items[1];     // n_items entries follow
};

// Index of the item that owns unit u of a stage (0 FIR, 1 GEMM, 2 state,
// 3 single-pass per-frame FIR, 4 folded FIR, 5 folded product, 6 folded FIR of split frames):
// the last item whose first unit is <= u.
__device__ inline int batch_find(const BatchItem* items, int n, int64_t u, int stage) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        const int64_t s = stage == 0 ? items[mid].fir_unit0
                          : stage == 1 ? items[mid].gemm_unit0
                          : stage == 2 ? items[mid].st_unit0
                          : stage == 3 ? items[mid].frame_unit0
                          : stage == 4 ? items[mid].ffold_unit0
                          : stage == 6 ? items[mid].fsplit_unit0
                                       : items[mid].gfold_unit0;
        if (s <= u) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// GEMM tile geometry shared with the batch planner.
constexpr int kGemmBM = 128, kGemmBN = 128;

// Per-frame scaled qmodes run three launches: partial maxima, per-frame
// exponents, scaled codes.
// frame_stage: per-frame scaled forms also launch the single-pass frame stage
// (the items flagged fir_single).
hipError_t launch_fir_batch(const BatchTable* t, int max_m, bool all_exact, int qmode, int grid, hipStream_t s,
                            bool frame_stage);
// Per-frame scaled items a batch runs in one pass (whole frame rows of 1024
// threads): the floats per thread, or 0 (three launches).  A unit walks the
// item's fir_tf frames (a whole number of ring blocks of M).
int fir_frame_batch_vec(const FirArgs& a);
// FirArgs::qmode the FIR writes for a DFT form (0: FP32 y): every form but
// FP32 takes its operand straight from the FIR.
inline int form_fir_qmode(int form) {
    switch (form) {
        case FORM_MXFP8: return 1;
        case FORM_BF16: return 2;
        case FORM_BF16X3: return 3;
        case FORM_FP8: return 4;
        case FORM_FP16: return 5;
        case FORM_FP16X3: return 6;
        default: return 0;
    }
}
// ... and the folded FIR: as above, FP8 rounded to E4M3's 4 significant bits before folding, then bf16.
inline int fold_fir_qmode(int form) { return form == FORM_FP8 ? 8 : form_fir_qmode(form); }
// qmode values whose codes carry a per-frame scale.
inline bool qmode_frame_scaled(int qm) { return qm >= 4 && qm <= 6; }

// Per-frame scale 2^e with the frame's largest |y| * 2^-e <= limit (448 for
// FP8 E4M3, 32768 for fp16); 0 for a zero or non-finite maximum.
__device__ inline int frame_exponent(float amax, float limit) {
    if (!(amax > 0.0f) || !isfinite(amax)) return 0;
    int e;
    frexpf(amax / limit, &e);  // amax/limit in [2^(e-1), 2^e)
    while (e > -120 && ldexpf(limit, e - 1) >= amax) --e;
    while (e < 120 && ldexpf(limit, e) < amax) ++e;
    return e;
}
// tile_n: the table's GEMM tile columns (kGemmBN for every form; 2 * kGemmBN
// also for FP32 with A in FP32).
// wide: A in operand form on the single-stream path's wide tiles (every
// item's K a whole number of their K tiles; gemm_batch_wide_tile).
hipError_t launch_gemm_batch(const BatchTable* t, int form, bool raw, int tile_n, int grid, hipStream_t s,
                             bool wide = false);
// The wide raw-operand tile (bm x bn) of `form`, if it serves an operand of K
// columns (K a whole number of its K tiles); false for FP32 and other K.
bool gemm_batch_wide_tile(int form, int K, int& bm, int& bn);
hipError_t launch_gather_batch(const BatchTable* t, int grid, hipStream_t s);
// Items with the folded product: their FIR (max_m: largest tap count among
// them, qmode as launch_fir_batch) and their tiles (one block each).
// split: the split items, else the others.
hipError_t launch_fir_fold_batch(const BatchTable* t, int max_m, int qmode, bool split, int grid, hipStream_t s);
hipError_t launch_fold_gemm_batch(const BatchTable* t, int form, int grid, hipStream_t s);

}  // namespace tina
