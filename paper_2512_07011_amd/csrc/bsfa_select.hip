// Order statistics of block maxima on the GPU: per head (the selection half of bsfa_calibrate) and per
// query tile (that of bsfa_calibrate_topk, at the end of this file).
//
// Input: the block-maximum dump of the score kernel, [batch][hq][per_head] floats with NaN where a
// block is not gateable.  For every query head h (all batch elements pooled) and every level l with
// target skip fraction f_l: n = number of non-NaN values, r = floor(f_l * n), result = the value of
// rank r in ascending order (x_r), -inf if r == 0, +inf if r >= n -- the rule of Section 4.2 reduced
// over query positions (the threshold that leaves exactly r blocks below it).
//
// Exact selection by three radix passes over the values' order-preserving 32-bit keys (11 + 11 + 10
// bits): a histogram pass counts, per head, the values whose leading bits equal the prefix found so
// far; a scan pass picks the bin that holds rank r and extends the prefix.  After the third pass the
// prefix is the key of x_r itself.  Up to kLevelsPerRound levels share one sweep over the dump.
#include "bsfa_internal.h"

#include <math.h>

#include <algorithm>

namespace bsfa {

namespace {

constexpr int kBins = 2048;
constexpr int kHistThreads = 512;

struct SelState {            // per (level slot, head)
    uint32_t prefix;         // leading key bits found so far
    uint32_t done;           // 0 searching, 1 result is -inf, 2 result is +inf
    unsigned long long rank; // rank of the wanted value among the values that share the prefix
};

// Layout of the selection area: hist0 [hq][kBins] (pass 0, shared by all levels),
// hist [kLevelsPerRound][hq][kBins] (passes 1 and 2), state [kLevelsPerRound][hq].
__host__ __device__ inline size_t hist0_words(int hq) { return (size_t)hq * kBins; }
__host__ __device__ inline size_t hist_words(int hq) { return (size_t)kLevelsPerRound * hq * kBins; }

__device__ __forceinline__ uint32_t ordered_key(float v)
{
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ void fill_zero_kernel(uint32_t *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Pass 0: per head, histogram of the leading 11 key bits of every value (private copy in LDS,
// flushed with one atomic per non-empty bin).  grid = (chunks, batch * hq).
__global__ void __launch_bounds__(256) hist0_kernel(const float *dump, long per_head, int hq, uint32_t *hist0)
{
    __shared__ uint32_t h[kBins];
    for (int i = threadIdx.x; i < kBins; i += 256) h[i] = 0u;
    __syncthreads();
    const int head = blockIdx.y % hq;
    const float *src = dump + (size_t)blockIdx.y * per_head;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < per_head; i += (long)gridDim.x * 256) {
        const float v = src[i];
        if (v == v) atomicAdd(&h[ordered_key(v) >> 21], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (h[i]) atomicAdd(&hist0[(size_t)head * kBins + i], h[i]);
}

// Passes 1 and 2: values whose leading bits equal a level's prefix are counted by their next bits.
// PASS 1: prefix = 11 bits, bin = bits 20..10.  PASS 2: prefix = 22 bits, bin = bits 9..0.
// One bin of pass 0 (a quarter of a binade) can hold most of a head's maxima, so pass 1 counts in LDS,
// one histogram per level, and flushes the bins that are not empty (32 heads at 32K tokens, 5 levels: 191 us
// with global atomics; with this and the finer split of the sweeps the whole calibration went from 4.25 to
// 4.00 ms).  In pass 2 a prefix of 22 bits leaves next to nothing to count.
template <int PASS>
__global__ void __launch_bounds__(kHistThreads) histn_kernel(const float *dump, long per_head, int hq, int n_lv,
                                                             const SelState *state, uint32_t *hist)
{
    extern __shared__ uint32_t h[];                   // PASS 1: [n_lv][kBins]
    const int head = blockIdx.y % hq;
    uint32_t pre[kLevelsPerRound];
    bool live[kLevelsPerRound];
    bool any = false;
    for (int l = 0; l < kLevelsPerRound; ++l) {
        live[l] = l < n_lv && state[(size_t)l * hq + head].done == 0u;
        pre[l] = live[l] ? state[(size_t)l * hq + head].prefix : 0u;
        any = any || live[l];
    }
    if (!any) return;                                 // (uniform over the workgroup)
    if constexpr (PASS == 1) {
        for (int i = threadIdx.x; i < n_lv * kBins; i += kHistThreads) h[i] = 0u;
        __syncthreads();
    }
    const float *src = dump + (size_t)blockIdx.y * per_head;
    for (long i = (long)blockIdx.x * kHistThreads + threadIdx.x; i < per_head; i += (long)gridDim.x * kHistThreads) {
        const float v = src[i];
        if (!(v == v)) continue;
        const uint32_t key = ordered_key(v);
        const uint32_t lead = PASS == 1 ? key >> 21 : key >> 10;
        const uint32_t bin = PASS == 1 ? (key >> 10) & 2047u : key & 1023u;
#pragma unroll
        for (int l = 0; l < kLevelsPerRound; ++l)
            if (live[l] && lead == pre[l]) {
                if constexpr (PASS == 1) atomicAdd(&h[l * kBins + bin], 1u);
                else atomicAdd(&hist[((size_t)l * hq + head) * kBins + bin], 1u);
            }
    }
    if constexpr (PASS == 1) {
        __syncthreads();
        for (int i = threadIdx.x; i < n_lv * kBins; i += kHistThreads)
            if (h[i]) atomicAdd(&hist[((size_t)(i / kBins) * hq + head) * kBins + i % kBins], h[i]);
    }
}

// Scan: one workgroup per (level slot, head).  PASS 0 also turns the target fraction into a rank.  The
// histogram the next pass adds to is cleared here, by the workgroup that owns it (PASS 1 has read it by then).
template <int PASS>
__global__ void __launch_bounds__(256) scan_kernel(const uint32_t *hist0, uint32_t *hist, int hq, SelectLevels lv, int l0,
                                                   SelState *state, float *out)
{
    __shared__ unsigned long long part[4];
    const int l = blockIdx.x, head = blockIdx.y, t = threadIdx.x;
    SelState &st = state[(size_t)l * hq + head];
    uint32_t *own = hist + ((size_t)l * hq + head) * kBins;
    const uint32_t *h = PASS == 0 ? hist0 + (size_t)head * kBins : own;
    if (PASS != 0 && st.done != 0u) return;           // (uniform over the workgroup)
    uint32_t c[8];
    unsigned long long s = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) { c[i] = h[t * 8 + i]; s += c[i]; }
    if constexpr (PASS != 2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) own[t * 8 + i] = 0u;
    }
    unsigned long long run = s;                       // sum over this lane and the lanes before it, then over the waves
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long x = __shfl_up(run, d);
        if ((t & 63) >= d) run += x;
    }
    if ((t & 63) == 63) part[t >> 6] = run;
    __syncthreads();
    unsigned long long before = run - s, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        before += w < (t >> 6) ? part[w] : 0ull;
        total += part[w];
    }
    unsigned long long rank;
    if (PASS == 0) {
        const unsigned long long n = total;
        const double f = (double)lv.f[l0 + l];
        const double rr = floor(f * (double)n);
        if (rr <= 0.0 || n == 0ull) {
            if (t == 0) { st.done = 1u; out[(size_t)(l0 + l) * hq + head] = -INFINITY; }
            return;
        }
        if (rr >= (double)n) {
            if (t == 0) { st.done = 2u; out[(size_t)(l0 + l) * hq + head] = INFINITY; }
            return;
        }
        rank = (unsigned long long)rr;
    } else {
        rank = st.rank;
    }
    __syncthreads();                                  // every thread has read st.rank before it is rewritten
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (rank >= before && rank < before + c[i]) {         // exactly one bin of one thread
            const uint32_t bin = (uint32_t)(t * 8 + i);
            const uint32_t prefix = PASS == 0 ? bin : PASS == 1 ? (st.prefix << 11) | bin : (st.prefix << 10) | bin;
            st.prefix = prefix;
            st.rank = rank - before;
            if (PASS == 0) st.done = 0u;
            if (PASS == 2) out[(size_t)(l0 + l) * hq + head] = key_value(prefix);
        }
        before += c[i];
    }
}

// The whole selection of a head in one workgroup, for dumps so short that the launches of the passes above cost
// more than the sweeps: the same three radix passes, one histogram per level in LDS, one wave per level to scan it.
// (Seven levels at a time: 56 KiB of histograms.)  Whole calibrations of 32 heads at five levels, seven launches
// against one: 500 tokens 83 -> 50 us, 2000 96 -> 64 us, 8K 305 -> 269 us, 16K 902 -> 896 us; the line is there.
constexpr int kSmallThreads = 1024, kSmallLevels = 7;
constexpr long kSmallValues = 32768;                  // values per head, batch elements pooled (16K tokens)
__global__ void __launch_bounds__(kSmallThreads) select_small_kernel(const float *dump, long per_head, int batch, int hq, SelectLevels lv,
                                                                     int n_levels, float *out)
{
    __shared__ uint32_t h[kSmallLevels][kBins];
    __shared__ uint32_t prefix[kSmallLevels];         // leading key bits found so far
    __shared__ uint32_t live[kSmallLevels];           // still searching
    const int head = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
    for (int l0 = 0; l0 < n_levels; l0 += kSmallLevels) {
        const int n_lv = min(kSmallLevels, n_levels - l0);
        if (t < kSmallLevels) live[t] = t < n_lv ? 1u : 0u;
        uint32_t rank = 0;                            // this wave's level: rank among the values that share the prefix
        for (int pass = 0; pass < 3; ++pass) {
            const int n_hist = pass == 0 ? 1 : n_lv;
            for (int i = t; i < n_hist * kBins; i += kSmallThreads) (&h[0][0])[i] = 0u;
            __syncthreads();
            for (int b = 0; b < batch; ++b) {
                const float *src = dump + ((size_t)b * hq + head) * per_head;
                for (long i = t; i < per_head; i += kSmallThreads) {
                    const float v = src[i];
                    if (!(v == v)) continue;
                    const uint32_t key = ordered_key(v);
                    if (pass == 0) {                  // (all levels share the first histogram)
                        atomicAdd(&h[0][key >> 21], 1u);
                        continue;
                    }
                    const uint32_t lead = pass == 1 ? key >> 21 : key >> 10, bin = pass == 1 ? (key >> 10) & 2047u : key & 1023u;
#pragma unroll
                    for (int l = 0; l < kSmallLevels; ++l)
                        if (live[l] && lead == prefix[l]) atomicAdd(&h[l][bin], 1u);
                }
            }
            __syncthreads();
            if (wave < n_lv && live[wave]) {          // (uniform over the wave)
                const uint32_t *mine = h[pass == 0 ? 0 : wave];
                uint32_t s = 0;
                for (int i = 0; i < kBins / 64; ++i) s += mine[lane * (kBins / 64) + i];
                uint32_t run = s;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t x = __shfl_up(run, d);
                    if (lane >= d) run += x;
                }
                const uint32_t n = __shfl(run, 63);
                float *const dst = out + (size_t)(l0 + wave) * hq + head;
                bool search = true;
                if (pass == 0) {
                    const double rr = floor((double)lv.f[l0 + wave] * (double)n);
                    search = rr > 0.0 && n != 0u && rr < (double)n;
                    rank = search ? (uint32_t)rr : 0u;
                    if (!search && lane == 0) {
                        live[wave] = 0u;
                        *dst = (rr <= 0.0 || n == 0u) ? -INFINITY : INFINITY;
                    }
                }
                if (search) {
                    uint32_t before = run - s, bin = 0, within = 0;
                    bool here = false;
                    for (int i = 0; i < kBins / 64; ++i) {                // exactly one bin of one lane holds the rank
                        const uint32_t c = mine[lane * (kBins / 64) + i];
                        if (rank >= before && rank < before + c) {
                            here = true;
                            bin = (uint32_t)(lane * (kBins / 64) + i);
                            within = rank - before;
                        }
                        before += c;
                    }
                    const int who = __ffsll((unsigned long long)__ballot(here)) - 1;
                    bin = __shfl(bin, who);
                    rank = __shfl(within, who);
                    if (lane == 0) {
                        const uint32_t found = pass == 0 ? bin : (prefix[wave] << (pass == 1 ? 11 : 10)) | bin;
                        prefix[wave] = found;
                        if (pass == 2) *dst = key_value(found);
                    }
                }
            }
            __syncthreads();                          // prefixes and live levels visible; histograms read
        }
    }
}

// k-th largest value of every row of the dump, for the levels of one chunk: one wave per row.  The row's
// ordered keys (NaN: 0, below every value) stay in registers, E to a lane, and the key is built from its top
// bit down: a bit stays set if at least k keys reach the candidate (32 steps of E compares whose ballots are
// counted on the scalar side; no LDS, no memory).  E = 0: rows too long for that are read again in every step.
template <int E>
__global__ void __launch_bounds__(256) topk_kernel(const float *dump, int mkv, long row0, long n_rows, TopkLevels lv, int n_lv, float *out)
{
    const long r = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n_rows) return;
    const int lane = threadIdx.x & 63;
    const float *src = dump + (size_t)(row0 + r) * mkv;
    auto key_at = [&](int x) {
        const float v = x < mkv ? src[x] : NAN;
        return v == v ? ordered_key(v) : 0u;
    };
    uint32_t key[E > 0 ? E : 1];
    if constexpr (E > 0) {
#pragma unroll
        for (int e = 0; e < E; ++e) key[e] = key_at(e * 64 + lane);
    }
    auto count = [&](uint32_t least) {                // keys >= least (wave-uniform)
        int n = 0;
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) n += __popcll(__builtin_amdgcn_ballot_w64(key[e] >= least));
        } else {
            for (int x = 0; x < mkv; x += 64) n += __popcll(__builtin_amdgcn_ballot_w64(key_at(x + lane) >= least));
        }
        return n;
    };
    const int avail = count(1u);
    for (int l = 0; l < n_lv; ++l) {
        const int k = lv.k[l];
        float t;
        if (avail <= k) t = -INFINITY;                // keeps min(k, A) = A blocks
        else if (k == 0) t = INFINITY;
        else {
            uint32_t found = 0u;
            for (int bit = 31; bit >= 0; --bit) {
                const uint32_t cand = found | (1u << bit);
                if (count(cand) >= k) found = cand;
            }
            t = key_value(found);
        }
        if (lane == 0) out[(size_t)l * n_rows + r] = t;
    }
}

}  // namespace

size_t select_area_bytes(int hq)
{
    return (hist0_words(hq) + hist_words(hq)) * sizeof(uint32_t) + (size_t)kLevelsPerRound * hq * sizeof(SelState);
}

hipError_t launch_select(const float *dump, long per_head, int batch, int hq, const SelectLevels &lv, int n_levels,
                         void *area, float *out_dev, hipStream_t stream)
{
    if (n_levels < 1 || n_levels > kMaxLevels || hq < 1 || hq > 65535 || batch < 1 || (long)batch * hq > 65535) return hipErrorInvalidValue;
    if (batch * per_head <= kSmallValues) {
        hipLaunchKernelGGL(select_small_kernel, dim3((unsigned)hq), dim3(kSmallThreads), 0, stream, dump, per_head, batch, hq, lv, n_levels, out_dev);
        return hipGetLastError();
    }
    uint32_t *hist0 = static_cast<uint32_t *>(area);
    uint32_t *hist = hist0 + hist0_words(hq);
    SelState *state = reinterpret_cast<SelState *>(hist + hist_words(hq));
    // one sweep of a head's maxima is split over up to 64 workgroups of 4K values and more (16K: a quarter of the
    // chip at 32 heads and 32K tokens, and the sweep then waits for memory)
    const int chunks = (int)std::min<long>(64, (per_head + 4095) / 4096);
    const dim3 grid_v((unsigned)std::max(chunks, 1), (unsigned)(batch * hq));
    hipLaunchKernelGGL(fill_zero_kernel, dim3(256), dim3(256), 0, stream, hist0, hist0_words(hq));
    hipLaunchKernelGGL(hist0_kernel, grid_v, dim3(256), 0, stream, dump, per_head, hq, hist0);
    for (int l0 = 0; l0 < n_levels; l0 += kLevelsPerRound) {
        const int n_lv = std::min(kLevelsPerRound, n_levels - l0);
        const dim3 grid_s((unsigned)n_lv, (unsigned)hq);
        const size_t lds = (size_t)n_lv * kBins * sizeof(uint32_t);
        hipLaunchKernelGGL((scan_kernel<0>), grid_s, dim3(256), 0, stream, hist0, hist, hq, lv, l0, state, out_dev);
        hipLaunchKernelGGL((histn_kernel<1>), grid_v, dim3(kHistThreads), lds, stream, dump, per_head, hq, n_lv, state, hist);
        hipLaunchKernelGGL((scan_kernel<1>), grid_s, dim3(256), 0, stream, hist0, hist, hq, lv, l0, state, out_dev);
        hipLaunchKernelGGL((histn_kernel<2>), grid_v, dim3(kHistThreads), 0, stream, dump, per_head, hq, n_lv, state, hist);
        hipLaunchKernelGGL((scan_kernel<2>), grid_s, dim3(256), 0, stream, hist0, hist, hq, lv, l0, state, out_dev);
    }
    return hipGetLastError();
}

hipError_t launch_topk(const float *dump, int mkv, long row0, long n_rows, const TopkLevels &lv, int n_lv, float *out_dev,
                       hipStream_t stream)
{
    if (n_lv < 1 || n_lv > kTopkLevels || mkv < 1 || row0 < 0 || n_rows < 1 || (n_rows + 3) / 4 > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((n_rows + 3) / 4));
    // as many registers as the row needs: 8K, 32K, 128K and 256K tokens; longer rows are not kept
    if (mkv <= 64 * 2) hipLaunchKernelGGL((topk_kernel<2>), grid, dim3(256), 0, stream, dump, mkv, row0, n_rows, lv, n_lv, out_dev);
    else if (mkv <= 64 * 8) hipLaunchKernelGGL((topk_kernel<8>), grid, dim3(256), 0, stream, dump, mkv, row0, n_rows, lv, n_lv, out_dev);
    else if (mkv <= 64 * 32) hipLaunchKernelGGL((topk_kernel<32>), grid, dim3(256), 0, stream, dump, mkv, row0, n_rows, lv, n_lv, out_dev);
    else if (mkv <= 64 * 64) hipLaunchKernelGGL((topk_kernel<64>), grid, dim3(256), 0, stream, dump, mkv, row0, n_rows, lv, n_lv, out_dev);
    else hipLaunchKernelGGL((topk_kernel<0>), grid, dim3(256), 0, stream, dump, mkv, row0, n_rows, lv, n_lv, out_dev);
    return hipGetLastError();
}

}  // namespace bsfa
