// Internal declarations shared by the translation units of libbsfa.so (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bsfa {

// Key/value block rows; the library is built for B_N = 64 only.
constexpr int kBlockN = 64;
// Mask words of a query tile that a workgroup which splits the key blocks can put together (256K tokens).
constexpr int kSplitMaskWords = 128;

// Division of numbers below 2^31 by a number fixed at launch: a multiplication and a shift (of the 64-bit
// product), exact because the multiplier exceeds 2^(31+s) / d by less than 2^s / d (Granlund and Montgomery,
// "Division by invariant integers using multiplication", Theorem 4.2).
struct FastDiv {
    uint32_t mul, shift;
    __host__ __device__ uint32_t of(uint32_t n) const { return (uint32_t)(((uint64_t)n * mul) >> shift); }
};
inline FastDiv fast_div(uint32_t d)               // 1 <= d < 2^31
{
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    return {(uint32_t)(((1ull << (31 + s)) + d - 1) / d), 31 + s};
}

// Work items counted off (decode_work): rows of k items each lie above item x, `sum` items in all if they went down to row
// 0; the row that item x is in.  Whole numbers: a product with a reciprocal of 32 bits is off by a row from about two
// million items on (15 to a row), which no sequence that fits the card's memory has, but nothing else keeps out.
__host__ __device__ inline int counted_row(int sum, int x, int k) { return (int)((uint32_t)(sum - x - 1) / (uint32_t)k); }

struct FwdParams {
    const uint16_t *q, *k, *v;       // bf16 or fp16 bit patterns (f16 says which)
    uint16_t *out;
    uint16_t *vt;                    // workspace for the transposed V tiles ([batch][hkv][mkv] tiles of 64 x head_dim
                                     // elements), or null: V is then gathered with transposing LDS reads
    const float *tau;                // [hq] or [hq][tau_tiles]
    uint8_t *k8;                     // workspace for K as fp8 tiles ([batch][hkv][mkv] tiles of 64 x 128 bytes), or null:
                                     // the score product then runs on the 16-bit elements
    const int32_t *seqlens;          // [batch] tokens per batch element, or null (all have seqlen)
    int64_t qsb, qsn, qsh, ksb, ksn, ksh, vsb, vsn, vsh, osb, osn, osh;
    int batch, hq, hkv, group, seqlen, mq, mkv;
    int causal, tau_per_tile, tau_tiles;
    int f16;                         // element type of q, k, v, out: 0 bf16, 1 fp16
    int single_head;                 // 1: never pair the heads of a GQA group in one workgroup
    int gate_mode;                   // 0: block maximum vs threshold; 1: running-maximum predicate (general stages only)
    float scale;                     // 1/sqrt(d): natural score units, used by the gate
    float scale_log2;                // log2(e)/sqrt(d): softmax evaluated with exp2
    unsigned long long *counts;      // [batch][hq][3] or null
    uint32_t *skip_mask;             // [batch][hq][mq][mask_words] or null
    float *block_max;                // [batch][hq][mq][mkv] or null
    float *lse;                      // [batch][seqlen][hq] or null
    int mask_words;
    FastDiv div_tile, div_gsub, div_hkv;   // work decomposition (decode_work): work items per query tile, head groups per
                                           // KV head, KV heads; set by the launch
    int counted;                     // work items that exist are counted off first (decode_work); set by the launch
    uint32_t turn[3];                // workgroups turn[0] .. turn[1] - 1 of an XCD, and from there to turn[2] - 1, take their
                                     // work items in reverse (decode_work); set by the launch
};

// Shapes whose forward calls rewrite V into the workspace, if they are given one and take their key blocks one after
// the other (rewrites_v; with the fp8 score product every call does).  The lines stand at launch_forward.
constexpr bool v_rewrite_pays(int head_dim, int block_m, int seqlen) { return head_dim == 128 && block_m == 128 && seqlen > 12288; }
bool rewrites_v(const FwdParams &p, int head_dim, int block_m);

// Launches the forward kernel (calib == false) or its score/block-maximum half only
// (calib == true: no V, no softmax, no output; block_max must be non-null).  vt may be set where
// rewrites_v says so or k8 is set.
// Returns hipSuccess or the launch error; hipErrorInvalidValue for an unsupported
// (head_dim, block_m) pair.
hipError_t launch_forward(const FwdParams &p, int head_dim, int block_m, bool calib, hipStream_t stream);

bool shape_supported(int head_dim, int block_m, int block_n);

// ---- order statistics of the block maxima on the GPU (bsfa_select.hip) ------------------------
constexpr int kMaxLevels = 64;        // target skip fractions per calibration call
constexpr int kLevelsPerRound = 8;    // levels that share one sweep over the block-maximum dump
struct SelectLevels {
    float f[kMaxLevels];              // target skip fractions, passed to the kernels by value
};
// Bytes of the histogram / state area launch_select needs for hq query heads (multiple of 16).
size_t select_area_bytes(int hq);
// dump: DEVICE [batch][hq][per_head] block maxima, NaN = not gateable.  out_dev: DEVICE
// [n_levels][hq]: per head (batch elements pooled) the order statistic x_r, r = floor(f * n), of its
// n non-NaN values, -inf if r == 0, +inf if r >= n.  area: DEVICE, select_area_bytes(hq) bytes,
// 16-byte aligned; it is cleared by the launch.  Enqueues on stream; no host synchronisation.
hipError_t launch_select(const float *dump, long per_head, int batch, int hq, const SelectLevels &lv, int n_levels,
                         void *area, float *out_dev, hipStream_t stream);

// ---- per-row top-k of the block maxima on the GPU (bsfa_select.hip) ------------------------------
constexpr int kTopkLevels = 64;       // levels per launch
struct TopkLevels {
    int32_t k[kTopkLevels];           // numbers of retained blocks, passed to the kernel by value
};
// dump: DEVICE [rows][mkv] block maxima, NaN = not gateable.  out_dev: DEVICE [n_lv][n_rows]: for the rows
// row0 .. row0 + n_rows - 1 the k-th largest of the non-NaN values, -inf where there are at most k, +inf
// for k = 0.  Enqueues on stream.
hipError_t launch_topk(const float *dump, int mkv, long row0, long n_rows, const TopkLevels &lv, int n_lv, float *out_dev,
                       hipStream_t stream);

// ---- matrix-instruction rate probe (bsfa_probe.hip) --------------------------------------------
constexpr int kProbeThreads = 512;        // 8 waves per workgroup: two per SIMD, as the forward kernel runs
constexpr int kProbeMfmaPerIter = 16;     // 32x32x16 MFMAs per wave and iteration
// operands: DEVICE, 4096 floats; sink: DEVICE, workgroups * kProbeThreads floats.  Enqueues one kernel.
hipError_t launch_mfma_rate_probe(const float *operands, float *sink, int workgroups, int iters, hipStream_t stream);

}  // namespace bsfa
