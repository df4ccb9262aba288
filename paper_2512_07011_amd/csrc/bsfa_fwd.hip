// Block-Sparse FlashAttention forward kernel for gfx950 (MI355X), wave64, bf16 or fp16 MFMA.
//
// One workgroup = QT adjacent query tiles Q_i (B_M = 32 * NWH rows, NWH waves of 32 rows) of HP query heads
// that share a KV head (GQA); it walks the reachable key blocks j in ascending order (Algorithm 1), each tile of
// each head with decisions of its own.
// With KSP > 1 the blocks are dealt to KSP sets of waves, each with a pipeline of its own, whose
// results are put together at the end (small problems: see launch_forward).
//   S_ij^T = K_j Q_i^T        32x32x16 MFMA, fp32 accumulate                      (Eq. 5)
//   s_max  = max S_ij         compared lane by lane; one flag per wave through LDS (Eq. 6)
//   gate   : s_max / sqrt(d) >= T keeps the block; blocks touching the causal boundary bypass
//            the gate (Section 4.1).  One decision per (head, query tile, key block).
//   kept   : V_j is requested only after the decision (and only if some head of the group keeps
//            the block), exp2-based online softmax, O^T += V_j^T P^T.
// The transposed products keep everything of one query row inside one lane pair (l, l^32):
// the S^T accumulator layout (column = query) is already the B-operand layout of the second
// MFMA up to a permutation of the keys, and the same permutation is applied to V when its
// A operand is gathered from LDS with the transposing read, so P never leaves registers.
//
// Software pipeline, one barrier per key block.  The scores of block j+1 are computed while block
// j is finished, so the gate decision is known one block ahead:
//   stage j:  softmax(S_j) -> P_j          (VALU) interleaved with
//             S_{j+1} = K_{j+1} Q^T        (MFMA); per-lane maximum of S_{j+1}; the wave's keep flag
//             (and its block maximum, where somebody asks for it) -> LDS
//             wait for the copies needed next; barrier
//             O^T += V_j^T P_j^T           (MFMA), and between those MFMAs, a few instructions at a
//             time: decide keep_{j+1}; request V_{j+1} (only if kept) and K_{j+KR+1}; running
//             maximum of block j+1; first score operands of block j+2
// K tiles sit in a ring of KR LDS slots and are requested KR+1 blocks ahead, V tiles in two slots;
// both go HBM -> LDS directly, and the waits are partial (vmcnt) so that only the tile needed
// next has to have landed.  With a workspace V arrives pre-transposed (transpose_v_kernel) and its
// operand is a plain 16-byte LDS read; without one it is gathered with the transposing read.
//
// What bounds it.  Long sequences: the matrix pipe at the clock the card holds under this load (a plain
// library product reaches 1360 TFLOP/s here, this kernel 1060 to 1190 dense, busy in 58 to 65 % of the cycles: a key
// block takes the two waves of a SIMD 3540 cycles at 8K tokens and 3160 at 128K, for 2048 of MFMA) and the issue of each
// wave: of a stage that a wave alone on its SIMD needed 3165 cycles for, two side by side needed 3199 (counted in an
// earlier kernel with the same stages; a vector instruction 4.4 cycles, an exponential 8, a taken branch 30, dependent
// ones 8), so every instruction in a wave's way counts, above all between the last score MFMA and the first PV MFMA of a
// block.  Two workgroups of four waves on a CU
// (HP = 1) run independently and hide that stretch for each other; eight waves that share a K/V stream
// (HP = 2) all stand at the same barrier, but read half as much from L2 (see launch_forward for the line).
// Short sequences: the chain of key blocks of the longest tile, about a microsecond a block (64 blocks 66.9 us).
#include "bsfa_dev.h"
#include <algorithm>

namespace bsfa {

struct ScoreTile {
    f32x16 s[2];          // S^T: [32-key half], raw q.k (no 1/sqrt(d)); column = this lane's query
    float mx0;            // fp8 score product: lane maximum of s[0]
    float mx;             // row max of the lane's query, equal in lanes l and l^32
    uint32_t keep;        // gate decision of this wave's head (uniform over the head's waves; a number, so that it
                          // and every branch on it are scalar)
    uint32_t any_keep;    // some head of the workgroup keeps the block (workgroup-uniform): V is fetched
    float alpha;          // kept blocks: factor that rescales the accumulator, if ...
    uint64_t resc;        // ... the running maximum of some row of the wave has grown (the lanes whose row's has)
};

// Waves per SIMD the registers are allocated for: two, or three at head_dim 64 where the LDS holds as many
// workgroups of four waves (8K tokens, 32 heads of width 64, half skip: 306 us with two, 230 us with three).
constexpr int min_waves(int d, int waves, int lds_bytes)
{
    return d == 64 && waves * (160 * 1024 / (lds_bytes + 1024)) >= 12 && waves <= 4 ? 3 : 2;
}

// Workgroups a CU holds, as far as decode_work asks: tiles that are split are left as they are (turned_places)
constexpr int places_of(int d, int waves, int shares) { return shares > 1 || waves != 4 ? 1 : d == 64 ? 3 : 2; }

constexpr int k_slot_bytes(int d) { return d / 8 * kPitch16; }               // (an fp8 tile fills half of its slot)
constexpr int v_slot_bytes(int d) { return d / 8 * v_pitch(d); }

template <int D, int NWH, int HP, int QT, int KSP, int KR, bool CALIB, bool F16, bool VT, bool QK8>
__global__ void __launch_bounds__(NWH * HP * QT * KSP * 64, min_waves(D, NWH * HP * QT * KSP, KSP * (KR * k_slot_bytes(D) + 2 * v_slot_bytes(D)))) bsfa_fwd_kernel(const FwdParams p)
{
    typedef typename Elem<F16>::T el;                    // element type of Q, K, V, P, O
    typedef typename Elem<F16>::x8 bf16x8;               // (the vector names keep the default type's name)
    typedef typename Elem<F16>::x4 bf16x4;
    typedef typename Elem<F16>::x2 bf16x2;
    static_assert(KSP == 1 || (!CALIB && !VT && !QK8), "shares of the key blocks: V in place");
    static_assert(!VT || D == 128, "V from the workspace: head_dim 128");
    constexpr int TEAMS = HP * QT;                       // (head, query tile) pairs of the workgroup: the NWH waves of one decide together
    constexpr int NW = NWH * TEAMS * KSP;
    constexpr int NT = NWH * TEAMS * 64;                  // threads that share one stream of K and V tiles
    constexpr int BM = NWH * 32;
    constexpr int BN = kBlockN;
    constexpr int KS = D / 16;       // MFMA k-steps over the head dim
    constexpr int DB = D / 32;       // 32-row blocks of O^T
    constexpr int CPR = D / 8;       // 16-byte chunks per tile row
    constexpr int NST = 64 * CPR / NT;                   // copy repetitions per 16-bit tile (V; K unless QK8)
    constexpr int NSTK = QK8 ? NST / 2 : NST;            // ... per K tile (fp8 tiles are half the bytes)
    static_assert(!QK8 || (D == 128 && NST >= 2), "fp8 score operands: head_dim 128, at most 512 threads");
    constexpr int ROW_BYTES = D * 2;
    constexpr int NWS = NT / 64;                         // waves that share one stream
    constexpr int PITCH_V = VT ? kPitch16 : v_pitch(D);
    constexpr int KSLOT = k_slot_bytes(D), VSLOT = v_slot_bytes(D);   // LDS bytes of a K and of a V tile
    constexpr int SHARE = KR * KSLOT + (CALIB ? 0 : 2) * VSLOT;       // ... of a stream of tiles
    constexpr int R = KR + 1;        // K tiles are requested R blocks ahead
    constexpr int VR = CALIB ? 0 : 2;
    static_assert(64 * CPR % NT == 0, "every thread copies the same number of chunks");
    static_assert(NST >= 1 && (R < 4 || NSTK * (R - 3) < 64), "copy repetitions");

    __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[KSP * SHARE];
    __shared__ float lds_red[2][NW];                                  // the waves' block maxima, where somebody asks for them
    __shared__ __attribute__((aligned(8))) uint8_t lds_flag[2][NW];   // the waves' keep flags
    __shared__ uint32_t lds_mask[TEAMS][KSP > 1 ? kSplitMaskWords : 1];  // KSP > 1: the tiles' skip masks, put together

    int b, g, h0, i0, n_tok;
    if (!decode_work<HP, QT, BM * QT, CALIB ? 1 : places_of(D, NWH * HP * QT, KSP)>(p, blockIdx.x, b, g, h0, i0, n_tok)) return;
    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ksel = KSP > 1 ? wave_all / (NWH * TEAMS) : 0;   // which share of the key blocks: those with j % KSP == ksel
    const int wave = KSP > 1 ? wave_all % (NWH * TEAMS) : wave_all, tid = wave * 64 + lane;
    const int tsel = wave / NWH, wrow = wave % NWH;      // which (head, query tile), which 32-row slice of it
    const int team = wave_all / NWH;                     // ... and of which share: the NWH waves that decide about a block together
    // V slots first: their gather offsets then fit the 16-bit immediate of the LDS reads
    const uint32_t lds_v0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)lds_raw) + ksel * SHARE;
    const uint32_t lds_k0 = lds_v0 + VR * VSLOT;
    const uint32_t lds_flag0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint8_t *)lds_flag);
    const int h = h0 + tsel / QT, i = i0 + tsel % QT;    // this wave's head and query tile
    const int l32 = lane & 31, hh = lane >> 5;

    const int64_t row0 = (int64_t)i * BM;                 // first query row of the tile
    // n_tok: tokens of this batch element; a sequence that does not fill its last query tile or key
    // block behaves as if padded by repeating its last token (Section 4.3): queries beyond the end are
    // copies of row n_tok - 1 and not stored, key blocks made of padding only are not visited, and in the
    // last real one the keys beyond the end are zeros (copies of the last token in the workspace's tiles),
    // which the causal mask hides from every real row either way.
    const bool real_tile = QT == 1 || row0 < n_tok;       // (with QT > 1 the last tiles of a workgroup may lie beyond the sequence)
    const bool stat_lane = (wrow == 0 && lane == 0 && real_tile);   // one lane per head and tile writes statistics
    const int64_t stat_row = ((int64_t)b * p.hq + h) * p.mq + i;
    if ((int64_t)i0 * BM >= n_tok) {                      // the tiles lie beyond the sequence: empty statistics
        const int htid = tid - tsel * NWH * 64;
        if (i < p.mq && ksel == 0) {
            if (p.block_max)
                for (int jj = htid; jj < p.mkv; jj += NWH * 64) p.block_max[stat_row * p.mkv + jj] = NAN;
            if (p.skip_mask)
                for (int w = htid; w < p.mask_words; w += NWH * 64) p.skip_mask[stat_row * p.mask_words + w] = 0u;
        }
        return;
    }
    const int mkv_tok = (n_tok + BN - 1) / BN;
    const int partial_blk = (n_tok % BN) ? n_tok / BN : -1;   // the block that padding completes, if any
    const int partial_rows = n_tok % BN;
    // reachable blocks: of this wave's tile, and of the workgroup's tiles together
    auto reachable = [&](int tile) { return p.causal ? min((int)(((int64_t)tile * BM + BM + BN - 1) / BN), mkv_tok) : mkv_tok; };
    const int n_tile = real_tile ? reachable(i) : 0, n_blk = QT == 1 ? n_tile : reachable(i0 + QT - 1);
    // causal: blocks [0, n_gate) are gateable, [n_gate, n_tile) touch the boundary.
    // non-causal: blocks [own_lo, own_hi) overlap the tile's own tokens and bypass the gate.
    const int n_gate = p.causal ? (int)((row0 + 1) / BN) : 0;
    const int own_lo = (int)(row0 / BN), own_hi = (int)((row0 + BM + BN - 1) / BN);
    // gateable for all tiles of the workgroup: blocks below all_lo and, without the mask, from all_hi on
    const int all_lo = QT == 1 ? (p.causal ? n_gate : own_lo) : p.causal ? (int)(((int64_t)i0 * BM + 1) / BN) : (int)((int64_t)i0 * BM / BN);
    const int all_hi = QT == 1 ? own_hi : min((int)(((int64_t)(i0 + QT) * BM + BN - 1) / BN), mkv_tok);
    // Block indices from here on: `j` counts the blocks of this wave's share, glob(j) is the key block it stands
    // for, own(x) is the number of its blocks below key block x.  All the same thing unless KSP > 1.
    auto glob = [&](int jl) { return KSP > 1 ? jl * KSP + ksel : jl; };
    auto own = [&](int x) { return KSP > 1 ? max(0, (x - ksel + KSP - 1) / KSP) : x; };
    const int n_own = own(n_blk), own_max = KSP > 1 ? (n_blk + KSP - 1) / KSP : n_own;
    if constexpr (KSP > 1) {
        for (int w = threadIdx.x; w < TEAMS * kSplitMaskWords; w += NW * 64) (&lds_mask[0][0])[w] = 0u;   // (a barrier follows before its first use)
    }

    const uint16_t *kbase = p.k + (int64_t)b * p.ksb + (int64_t)g * p.ksh;
    // VT: V comes from the workspace, one transposed 64-key tile after the other, unit by unit
    const uint16_t *vbase = VT ? p.vt + ((int64_t)b * p.hkv + g) * p.mkv * (int64_t)(BN * D)
                               : p.v + (int64_t)b * p.vsb + (int64_t)g * p.vsh;
    // threshold of this wave's head; tiles past the calibrated length use its last tile's (Section 4.3)
    const float tau_own = CALIB ? -INFINITY      // the score half takes no decisions
                          : !real_tile ? NAN     // (keeps nothing)
                                : p.tau[p.tau_per_tile ? (int64_t)h * p.tau_tiles + min(i, p.tau_tiles - 1) : h];
    // source of this lane's part of a copy's first repetition, and the bytes from one repetition to the next
    const uint32_t koff = QK8 ? (uint32_t)tid * 16u : unit_src_offset<D>(wave, lane, (int)p.ksn);
    const uint32_t voff = VT ? (uint32_t)tid * 16u : unit_src_offset<D>(wave, lane, (int)p.vsn);
    const uint32_t krep = NWS * (QK8 ? (uint32_t)kUnit : (uint32_t)p.ksn * 2u), vrep = NWS * (VT ? (uint32_t)kUnit : (uint32_t)p.vsn * 2u);
    // QK8: K comes from the workspace as fp8 tiles (64 rows of D bytes, unit by unit)
    const uint8_t *k8base = QK8 ? p.k8 + ((int64_t)b * p.hkv + g) * p.mkv * (int64_t)(BN * D) : nullptr;
    const int64_t kstep = (int64_t)BN * p.ksn, vstep = VT ? (int64_t)(BN * D) : (int64_t)BN * p.vsn;
    // Requests of a tile: bytes of K_t and V_t of this wave's share that exist (0: block t lies behind the share's
    // last), and the copies in pieces, one unit of this wave each.  Every stage requests a K tile, existing or not, so
    // that the counts that the waits rely on are the same everywhere.
    const bool last_partial = n_own > 0 && glob(n_own - 1) == partial_blk;
    const uint32_t k_last = last_partial && !QK8 ? row_bytes<D>(partial_rows, (int)p.ksn) : kWholeTile;
    const uint32_t v_last = last_partial && !VT ? row_bytes<D>(partial_rows, (int)p.vsn) : kWholeTile;      // (workspace tiles are padded already)
    auto k_exist = [&](int t) { return t < n_own - 1 ? kWholeTile : t == n_own - 1 ? k_last : 0u; };
    auto v_exist = [&](int t) { return t < n_own - 1 ? kWholeTile : v_last; };
    const uint32_t k_wave = wave * kPitch16, v_wave = wave * PITCH_V;
    auto k_unit = [&](auto rc, uint32_t &off, const i32x4 &rsrc, uint32_t slot) { unit_copy_async<decltype(rc)::value, NWS * kPitch16>(off, krep, rsrc, slot + k_wave); };
    auto v_unit = [&](auto rc, uint32_t &off, const i32x4 &rsrc, uint32_t slot) { unit_copy_async<decltype(rc)::value, NWS * PITCH_V>(off, vrep, rsrc, slot + v_wave); };
    // whole tiles: K_t, whose first row is at `src`, into the ring slot at LDS byte address dst; V_t into slot t & 1
    auto copy_k_from = [&](const unsigned char *src, int t, uint32_t dst) {
        const i32x4 rsrc = tile_rsrc(src, k_exist(t));
        uint32_t off = koff;
        static_for<NSTK>([&](auto rc) { k_unit(rc, off, rsrc, dst); });
    };
    auto copy_v_from = [&](const unsigned char *src, int t) {
        const i32x4 rsrc = tile_rsrc(src, v_exist(t));
        uint32_t off = voff;
        static_for<NST>([&](auto rc) { v_unit(rc, off, rsrc, lds_v0 + (uint32_t)(t & 1) * VSLOT); });
    };
    const unsigned char *const k_bytes = QK8 ? reinterpret_cast<const unsigned char *>(k8base) : reinterpret_cast<const unsigned char *>(kbase) + ksel * kstep * 2;
    const unsigned char *const v_bytes = reinterpret_cast<const unsigned char *>(vbase) + ksel * vstep * 2;
    // bytes from one tile of this wave's share to the next
    const int64_t kstep_b = KSP * (QK8 ? (int64_t)(BN * D) : kstep * 2), vstep_b = KSP * vstep * 2;
    auto copy_k = [&](int t, uint32_t dst) { copy_k_from(k_bytes + t * kstep_b, t, dst); };
    auto copy_v = [&](int t) { copy_v_from(v_bytes + t * vstep_b, t); };

    // Operand gather addresses: bytes inside a tile slot, a base per lane plus constants (see the tile layout).
    // K (A operand of S^T): lane reads key row 32*kb + l32, chunk 2s + hh:  ka_base + 512 kb + 32 s.
    // QK8: rows of 128 bytes; lane reads row 32*kb + l32, head-dim bytes 64s + 32hh .. +31 as two b128:
    // ka_base + 512 kb + 64 s + {0, 16}.
    constexpr int UK = QK8 ? 8 : D / 8;                  // units of a K tile
    const uint32_t ka_base = (uint32_t)((l32 % UK) * kPitch16 + (l32 / UK) * (QK8 ? 128 : ROW_BYTES) + (QK8 ? 32 : 16) * hh);
    // V (A operand of O^T, transposing read of 4 keys x 16 head-dim columns per 16 lanes): lane
    // reads row 16u + 4hh + (L >> 2) (+8 for the second half), 8 bytes.  Which head-dim column an
    // operand row stands for is free (it only permutes the rows of O^T, undone at the final
    // store): at D = 128 operand rows 0-15 of block x are columns 16x .. 16x+15 and rows 16-31 are
    // columns 64+16x .., which puts the two 16-lane groups of a read into different bank halves;
    // at D = 64 rows 0-31 are columns 32x .. 32x+31:
    // va_base + 256 u + 2 X_COLS x + {0, V_HALF}.
    constexpr int G16_COLS = (D == 128) ? 64 : 16;       // column distance of the two 16-lane groups
    constexpr int X_COLS = (D == 128) ? 16 : 32;         // column step of x
    constexpr int V_HALF = (D == 128) ? 8 * v_pitch(D) : ROW_BYTES;   // eight rows further
    const int L = lane & 15, g16 = (lane >> 4) & 1;
    // VT: the tile holds V^T, D rows of 64 keys (128 bytes), the keys of every 16-key step ordered
    // so that the 8 keys a lane multiplies are contiguous.  Lane reads row 32x + l32, chunk 2u + hh, as one b128,
    // va_base + 256 x + 32 u: at about four times the LDS rate of the transposing reads.  (The lanes of a phase of a read come
    // from both 16-row halves of the block, which lie half the banks apart, and meet conflicts: 16 % of the cycles at 128K dense.
    // Halves a multiple of all the banks apart have none and are no faster: 32K 5812 / 5816 us, dense 7668 / 7653, fp8 4295 / 4318.)
    const uint32_t va_base = VT ? (uint32_t)((l32 % 16) * kPitch16 + (l32 / 16) * 128 + 16 * hh)
                                : (uint32_t)((4 * hh + (L >> 2)) * v_pitch(D) + 2 * G16_COLS * g16 + 8 * (L & 3));

    // All K tiles the ring holds are requested before anything else, and what follows block 0 (V_0, K_{R-1}) is left
    // in flight for the first stage: one trip to memory before the pipeline starts instead of two.  A longer ring leaves out
    // what does not exist, which the only tile of a short sequence would wait for (us with / without the requests: 2000 x 10
    // tokens of 8 heads of width 64, ring of 3, 106.7 / 94.8, 300 x 60 21.9 / 20.2, ring of 4 34.7 / 33.5); with two slots the
    // branch costs more than that (100 x 250 tokens of 3 heads 23.5 / 24.1), and a branch for each tile of four, too (58.0 / 58.5).
#pragma unroll
    for (int t = 0; t < KR; ++t)
        if (KR == 2 || t == 0 || n_own > (t < 2 ? 1 : 2)) copy_k(t, lds_k0 + (uint32_t)t * KSLOT);

    // Q_i^T as the B operand: lane holds query (32*wrow + l32), head-dim slice 16s + 8hh .. +7
    // (QK8: slice 64s + 32hh .. +31, rounded to fp8 here, once)
    constexpr int KSQ = QK8 ? D / 64 : KS;               // score MFMA k-steps
    constexpr int NQK = 2 * KSQ;                         // score MFMAs per block: (k-step, 32-key half)
    typedef std::conditional_t<QK8, i32x8, bf16x8> kop_t; // one score operand
    kop_t qreg[KSQ];
    const int q_row = (int)row0 + wrow * 32 + l32;
    {
        const uint16_t *qrow = p.q + (int64_t)b * p.qsb + (int64_t)min(q_row, n_tok - 1) * p.qsn + (int64_t)h * p.qsh;
        if constexpr (QK8) {
#pragma unroll
            for (int s = 0; s < KSQ; ++s)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bf16x8 v8 = *reinterpret_cast<const bf16x8 *>(qrow + 64 * s + 32 * hh + 8 * c);
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = (float)v8[e];
                    int w0, w1;
                    cvt8_fp8(f, w0, w1);
                    qreg[s][2 * c] = w0;
                    qreg[s][2 * c + 1] = w1;
                }
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) qreg[s] = *reinterpret_cast<const bf16x8 *>(qrow + 8 * hh + 16 * s);
        }
    }
    auto qk_mma = [&](const kop_t &a, const kop_t &b, f32x16 c) {
        if constexpr (QK8) return mfma64_fp8(a, b, c);
        else return mfma16(a, b, c);
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[x][e] = 0.f;
    // Running maximum of the row, log2 units (score * log2(e)/sqrt(d)).  The start value is finite, so that rows
    // without a visible key yet need no special case, and below any finite score (fp32 products times
    // log2(e)/sqrt(d)).
    constexpr float M_NONE = -3.0e38f;
    float m_run = M_NONE;
    float l_run = 0.f;         // this lane's share of the running normaliser

    unsigned n_skipped = 0;    // per-head statistics, uniform over the head's waves
    uint32_t mask_word = 0;

    auto is_gated = [&](int j) { return p.causal ? (j < n_gate) : (j < own_lo || j >= own_hi); };

    // Order of the score MFMAs: the two 32-key halves in turn; with fp8 operands (four long MFMAs) one half after
    // the other, so that the first half's maxima are taken while the second half is multiplied (1.5 % faster
    // there, 1 % slower with 16-bit operands).
    constexpr bool HALVES = QK8;
    auto kst = [](int n) { return HALVES ? n % KSQ : n >> 1; };
    auto khalf = [](int n) { return HALVES ? n / KSQ : n & 1; };
    // K operand n (k-step kst(n), 32-key half khalf(n)) of the tile at LDS byte address kaddr (+ka_base)
    auto k_operand = [&](uint32_t kaddr, int n) {
        if constexpr (QK8) {
            const uint32_t at = kaddr + (uint32_t)(512 * khalf(n) + 64 * kst(n));
            const i32x4 lo = *LDS_PTR(const i32x4, at);
            const i32x4 hi = *LDS_PTR(const i32x4, at + 16u);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return *LDS_PTR(const bf16x8, kaddr + (uint32_t)(512 * khalf(n) + 32 * kst(n)));
        }
    };

    constexpr int PD = 4;            // LDS operand reads are issued PD MFMAs ahead of their use (3 to 6 measure within 1 %)
    // ... of the score operands: the fp8 ones are twice as wide and four in all; with three waves to a SIMD four of them
    // are more than the 168 registers hold, and what is spilled comes back inside the loop behind a wait for every copy
    // in flight (8K tokens, 32 heads of width 64, half skip: 256 us with four, 233 with three, 230 with two).  The score half
    // alone has four waves on a SIMD to hide the reads, and at head_dim 128 the LDS is as busy as the matrix pipe there: fewer
    // reads at a time (a calibration on 6000 tokens of 32 heads over 8, four / two, us: 32-row tiles 159.0 / 155.8, 64-row tiles
    // 144.5 / 141.7, 128-row tiles 140.0 / 137.7; 3000 tokens of 3 heads 36.2 / 35.6; at worst 5000 tokens of 32 heads 102.8 / 104.1).
    constexpr int PDK = QK8 || (CALIB ? D == 128 : min_waves(D, NW, KSP * SHARE) == 3) ? 2 : PD;
    // The first PDK score operands of a block are read one phase early (at the end of the previous
    // stage, behind its last MFMAs), so that the score MFMAs do not start with an LDS round trip.
    kop_t kpre[PDK];
    auto prefetch_k = [&](uint32_t kt) {
        uint32_t at = kt + ka_base;
        asm("" : "+v"(at));                                // (else every operand gets a base of its own, and an addition)
#pragma unroll
        for (int n = 0; n < PDK; ++n) kpre[n] = k_operand(at, n);
    };

    auto half_max = [&](ScoreTile &t, int n) {              // after MFMA n, once s[0] is complete
        if (n != KSQ + 1) return;
        t.mx0 = fmaxf(t.s[0][0], t.s[0][1]);
#pragma unroll
        for (int e = 2; e < 16; ++e) t.mx0 = fmaxf(t.mx0, t.s[0][e]);
    };

    // S^T of block j from the K tile at LDS byte address `kt` (MFMA and LDS reads only); the
    // order reads-ahead / MFMA is pinned so that no MFMA waits for a read issued just before it
    auto qk_mfma = [&](ScoreTile &t, uint32_t kt) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) t.s[kb][e] = 0.f;
        const uint32_t kaddr = kt + ka_base;
        kop_t a[NQK + PDK];
#pragma unroll
        for (int n = 0; n < PDK; ++n) a[n] = kpre[n];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NQK; ++n) {
            if (n + PDK < NQK) a[n + PDK] = k_operand(kaddr, n + PDK);
            t.s[khalf(n)] = qk_mma(a[n], qreg[kst(n)], t.s[khalf(n)]);
            if (HALVES) half_max(t, n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Causal mask on boundary blocks, lane / row maxima, and the wave's keep flag into lds_flag[j & 1]: the
    // decision is about the maximum over the head's waves, and  max(m) * c >= T  <=>  some m * c >= T
    // (c > 0, rounding is monotone), so flags are all the waves have to exchange.  The maxima themselves go to
    // lds_red[j & 1] if somebody asks for them (dump, calibration).
    // FAST: the block is known to be gateable (no causal mask).  There every lane compares its own maximum:
    // that takes the cross-lane reductions out of the stretch between the last score MFMA and the barrier;
    // the row maximum the softmax needs is completed after the barrier, for kept blocks only.
    auto reduce_scores = [&](ScoreTile &t, int j, auto fast_tag) {
        constexpr bool FAST = decltype(fast_tag)::value;
        if constexpr (FAST && !CALIB) {
            float mx = -INFINITY;
            if constexpr (HALVES) {
                mx = t.mx0;
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, t.s[1][e]);
            } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, t.s[kb][e]);
            }
            t.mx = mx;                                        // this lane's half of the row
            const bool wave_ge = __builtin_amdgcn_ballot_w64(mx * p.scale >= tau_own) != 0ull;
            if (lane == 0) lds_flag[j & 1][wave_all] = wave_ge ? 1 : 0;
            return;
        }
        const bool gated = FAST ? true : is_gated(glob(j));
        const bool there = QT == 1 || FAST || glob(j) < n_tile;   // (another tile of the workgroup may reach further)
        if constexpr (!FAST) {
            if (p.causal && !gated && there) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int key = glob(j) * BN + 32 * kb + 8 * (e >> 2) + 4 * hh + (e & 3);
                        if (key > q_row) t.s[kb][e] = -INFINITY;
                    }
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, t.s[kb][e]);
        t.mx = pair_max(mx);
        bool ge = there;                                      // blocks that bypass the gate are kept
        if (gated && there) {
            float stat = t.mx, unit = p.scale;                // natural score units (Eq. 5-6)
            if constexpr (!FAST) {
                // the comparison predicate (Section 3): local row maximum minus the running row maximum
                // after this block, natural units; m_run covers the kept blocks before this one.  A row that has
                // seen no finite score yet is at its running maximum whatever this block holds, -inf included.
                if (p.gate_mode) {
                    stat = m_run > M_NONE ? fminf(t.mx * p.scale - m_run * 0.6931471805599453f, 0.f) : 0.f;
                    unit = 1.f;
                }
            }
            const float wm = wave_max_paired(stat) * unit;
            ge = wm >= tau_own;                               // skip iff s_max < T
            if ((CALIB || p.block_max) && lane == 0) lds_red[j & 1][wave_all] = wm;
        }
        if (!CALIB && lane == 0) lds_flag[j & 1][wave_all] = ge ? 1 : 0;
    };

    // the keep flags of team x of the workgroup for a block of parity par, as published before the last barrier
    constexpr int FB = NWH * TEAMS;                       // flag bytes of a stream's waves
    constexpr int FW = FB == 8 ? 2 : 1;                   // ... in words (one access)
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef std::conditional_t<FB == 8, u32x2, std::conditional_t<FB == 4, uint32_t, std::conditional_t<FB == 2, uint16_t, uint8_t>>> flag_t;
    static_assert(FB == 8 || FB == 4 || FB == 2 || FB == 1, "one access reads the flags of a stream");
    auto read_flags = [&](uint32_t (&flags)[FW], int par) {
        const flag_t f = *LDS_PTR(const flag_t, lds_flag0 + (uint32_t)(par * NW + ksel * FB));
        if constexpr (FW == 2) {
            flags[0] = f[0];
            flags[1] = f[1];
        } else {
            flags[0] = f;
        }
    };
    // Decisions from the read flags.  They are consumed here and not earlier (nothing computed from them may be
    // hoisted in front of the PV MFMAs, where it would wait for the LDS read), and made scalar, so that the
    // branches on them are uniform.
    auto decide = [&](ScoreTile &t, const uint32_t (&flags)[FW]) {
        uint32_t w[FW];
#pragma unroll
        for (int x = 0; x < FW; ++x) {
            uint32_t f = flags[x];
            asm volatile("" : "+v"(f));
            w[x] = (uint32_t)__builtin_amdgcn_readfirstlane((int)f);
        }
        constexpr int PER = FW == 2 ? TEAMS / 2 : TEAMS;                // teams of a word
        const uint32_t own_word = FW == 2 && tsel >= PER ? w[FW - 1] : w[0];
        t.keep = PER == 1 ? own_word : (own_word >> (8 * NWH * (tsel % PER))) & ((1u << (8 * NWH % 32)) - 1u);
        t.any_keep = w[0] | w[FW - 1];
    };

    // The mask word of block j, its last: counted, and written if somebody asks for the mask.  mask_word is a shift register
    // (bit j % 32 of a word comes in at the top, 32 / KSP times a word), so it is never cleared and stays scalar.
    auto flush_mask = [&](int j) {
        const uint32_t word = mask_word >> (32 - KSP * ((j & 31) / KSP + 1));
        n_skipped += (unsigned)__builtin_popcount(word);
        if (p.skip_mask && stat_lane && (QT == 1 || (j & ~31) < n_tile)) {
            if constexpr (KSP > 1) atomicOr(&lds_mask[tsel][j >> 5], word);
            else p.skip_mask[stat_row * p.mask_words + (j >> 5)] = word;
        }
    };
    // statistics of block j: decision of this wave's head, and its maximum if asked for
    auto record = [&](uint32_t keep, int jl, auto fast_tag) {
        constexpr bool FAST = decltype(fast_tag)::value;
        const int j = glob(jl);
        mask_word = (mask_word >> KSP) | (keep == 0u && (QT == 1 || FAST || j < n_tile) ? 1u << (32 - KSP + ksel) : 0u);
        if (CALIB || !FAST) {
            if (p.block_max && stat_lane && (QT == 1 || j < n_tile)) {
                float bmax = NAN;
                if (FAST || is_gated(j)) {
                    bmax = lds_red[jl & 1][team * NWH];
#pragma unroll
                    for (int w = 1; w < NWH; ++w) bmax = fmaxf(bmax, lds_red[jl & 1][team * NWH + w]);
                }
                p.block_max[stat_row * p.mkv + j] = bmax;
            }
        }
        if constexpr (!CALIB) {
            if ((j & 31) > 31 - KSP) flush_mask(j);
        }
    };

    // online-softmax update of the running statistics with block `t`: new row max and the
    // accumulator's rescale factor first, then the exponentials, P (bf16) into pb
    // Running maximum and rescale factor for block `t`; most blocks of a long sequence raise no row's maximum and
    // leave both alone.  (A maximum that follows lazily would save most of the other rescales, 3 % on an 8K
    // prompt, but costs precision: against the row's own maximum the largest probabilities sit just below a power
    // of two, where rounding them to 16 bits is most exact.  Error against 64 bits 0.00199 -> 0.00214.)
    // In two pieces and without a branch; `gate` is 0, or -inf to leave everything as it is.
    auto softmax_max = [&](ScoreTile &t, float gate) {
        const float mb = TEAMS > 1 ? fmaf(t.mx, p.scale_log2, gate) : t.mx * p.scale_log2;
        const bool grown = mb > m_run;
        t.resc = __builtin_amdgcn_ballot_w64(grown);
        const float m_new = grown ? mb : m_run;
        t.alpha = m_run - m_new;
        m_run = m_new;
    };
    auto softmax_alpha = [&](ScoreTile &t) {
        t.alpha = __builtin_amdgcn_exp2f(t.alpha);
        l_run *= t.alpha;
    };
    auto softmax_begin = [&](ScoreTile &t) {
        softmax_max(t, 0.f);
        softmax_alpha(t);
    };
    auto softmax_exp = [&](ScoreTile &t, bf16x8 (&pb)[4]) {
        float psum = 0.f;
#pragma unroll
        for (int idx = 0; idx < 32; idx += 2) {
            const int kb = idx >> 4, e = idx & 15;
            const float p0 = __builtin_amdgcn_exp2f(fmaf(t.s[kb][e], p.scale_log2, -m_run));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(t.s[kb][e + 1], p.scale_log2, -m_run));
            const bf16x2 pp = {(el)p0, (el)p1};
            psum = pair_sum(pp, psum);                                       // sum of the rounded values
            pb[idx >> 3][idx & 7] = pp[0];
            pb[idx >> 3][(idx & 7) + 1] = pp[1];
        }
        l_run += psum;
    };
    // softmax_exp(cur) and qk_mfma(nxt) fused.  The exponentials of block j and the score MFMAs
    // of block j+1 are independent: they are written interleaved (per MFMA a few exponentials,
    // their row-sum adds and bf16 packs) and pinned in that order, so that the matrix pipe and
    // the VALU run together.  K operands are read PD MFMAs ahead.
    auto fused_exp_qk = [&](ScoreTile &cur, ScoreTile &nxt, uint32_t kt, bf16x8 (&pb)[4]) {
        const uint32_t kaddr = kt + ka_base;
        kop_t a[NQK + PDK];
#pragma unroll
        for (int n = 0; n < PDK; ++n) a[n] = kpre[n];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) nxt.s[kb][e] = 0.f;
        constexpr int EPM = 32 / NQK;              // exponentials per MFMA (2 at D = 128, 4 at D = 64; 8 with fp8 operands)
        // The exponentials of one MFMA slot are rounded, packed and summed one slot later, so that
        // no instruction waits for a transcendental issued just before it.
        float ex[EPM];
        auto pack = [&](int n) {                   // the pairs computed in slot n
#pragma unroll
            for (int t = 0; t < EPM; t += 2) {
                const int idx = n * EPM + t;
                const bf16x2 pp = {(el)ex[t], (el)ex[t + 1]};
                pb[idx >> 3][idx & 7] = pp[0];
                pb[idx >> 3][(idx & 7) + 1] = pp[1];
            }
        };
#pragma unroll
        for (int n = 0; n < NQK; ++n) {
            if (n + PDK < NQK) a[n + PDK] = k_operand(kaddr, n + PDK);
            nxt.s[khalf(n)] = qk_mma(a[n], qreg[kst(n)], nxt.s[khalf(n)]);
            float nx[EPM];
#pragma unroll
            for (int t = 0; t < EPM; ++t) {
                const int idx = n * EPM + t;
                nx[t] = __builtin_amdgcn_exp2f(fmaf(cur.s[idx >> 4][idx & 15], p.scale_log2, -m_run));
            }
            if (n > 0) pack(n - 1);
            if (HALVES) half_max(nxt, n);
#pragma unroll
            for (int t = 0; t < EPM; ++t) ex[t] = nx[t];
            __builtin_amdgcn_sched_barrier(0);
        }
        pack(NQK - 1);
    };
    // Row sums of the rounded probabilities (the values the second MFMA multiplies).  The dot instructions run on the
    // matrix pipe: measured beside 32x32x16 MFMAs, each run of them stops the pipe for 12 cycles and 4 per instruction,
    // and a chain on one accumulator takes 8 per instruction.  So all sixteen together, on two accumulators, at a place
    // where the pipe stands still anyway: behind the barrier, while the first V operands travel.  (A block's sum is
    // therefore added up in another order here than in softmax_exp, which differs by 32-bit rounding only.)
    auto row_sum = [&](bf16x8 (&pb)[4]) {
        asm volatile("" : "+v"(pb[0]), "+v"(pb[1]), "+v"(pb[2]), "+v"(pb[3]));
        float ps[2] = {0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < 8; t += 2) {
                const bf16x2 pp = {pb[u][t], pb[u][t + 1]};
                ps[(t >> 1) & 1] = pair_sum(pp, ps[(t >> 1) & 1]);
            }
        l_run += ps[0] + ps[1];
        asm volatile("" : "+v"(l_run));
    };

    // O^T += V^T P^T for the V tile at LDS byte address `vt`; operand n = (k-step u = n / DB,
    // head-dim block x = n % DB), read PD MFMAs ahead
    // `hook(n)` runs after MFMA n has been issued (n a compile-time constant): work that only has to
    // happen soon after the barrier goes there in small pieces, beside the matrix pipe instead of in
    // front of it
    constexpr int NPV = 4 * DB;
    auto v_operand = [&](uint32_t vaddr, int n) {
        const int u = n / DB, x = n % DB;
        if constexpr (VT) return *LDS_PTR(const bf16x8, vaddr + (uint32_t)(256 * x + 32 * u));
        const uint32_t at = vaddr + (uint32_t)(256 * u + 2 * X_COLS * x);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, at));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, at + V_HALF));
        const s16x8 av = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, av);
    };
    typedef bf16x8 vops_t[NPV + PD];
    auto pv_reads = [&](vops_t &a, uint32_t vaddr) {
#pragma unroll
        for (int n = 0; n < PD; ++n) a[n] = v_operand(vaddr, n);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pv_mfma = [&](auto nc, const ScoreTile &t, const bf16x8 (&pb)[4], vops_t &a, uint32_t vaddr, auto rescale) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n + PD < NPV) a[n + PD] = v_operand(vaddr, n + PD);
        if constexpr (decltype(rescale)::value) {             // the running maximum has grown: O^T follows, a block of it at a time
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[n][e] *= t.alpha;
        }
        oacc[n % DB] = mfma16(a[n], pb[n / DB], oacc[n % DB]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the first DB MFMAs, one for each block of O^T
    auto pv_head = [&](const ScoreTile &t, const bf16x8 (&pb)[4], vops_t &a, uint32_t vaddr) {
        if (t.resc != 0) static_for<DB>([&](auto nc) { pv_mfma(nc, t, pb, a, vaddr, std::true_type{}); });
        if (opaque(t.resc) == 0) static_for<DB>([&](auto nc) { pv_mfma(nc, t, pb, a, vaddr, std::false_type{}); });
    };
    auto pv_tail = [&](const ScoreTile &t, const bf16x8 (&pb)[4], vops_t &a, uint32_t vaddr, auto hook) {
        static_range<DB, NPV>([&](auto nc) {
            pv_mfma(nc, t, pb, a, vaddr, std::false_type{});
            hook(nc);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    uint32_t kring = (uint32_t)(1 % KR) * KSLOT;     // ring offset of the K slot the next stage reads
    // sources of the copies a stage requests, advanced by one block per stage: K_{j+R} and V_{j+1}
    const unsigned char *k_ahead = k_bytes + R * kstep_b;
    const unsigned char *v_ahead = v_bytes + vstep_b;
    // One pipeline stage: finish block j (`cur`), look ahead to block j+1 (`nxt`).
    // Block j+1 exists (the tile's last block is finished by last_stage).  FAST: it is gateable, so the
    // look-ahead has no mask and fewer conditionals.
    // PRIO: of a SIMD's two waves the one in its PV half goes first.  Where they come out of the same barrier (heads or
    // tiles that share a workgroup) or wait for each other in the end (shares) the later half is over sooner: us without /
    // with, half skip: 32K tokens 5913 / 5825, 28 heads over 4, 4096 tokens in 64-row tiles 117.5 / 114.8, 2 heads of width 64,
    // 8192 tokens 67.0 / 65.0, fp8 scores 32K 4716 / 4689.  Two independent workgroups on a CU are better left alone (8K tokens
    // 433.5 / 436.1), and so are three waves to a SIMD (28 heads of width 64, 8192 tokens in 32-row tiles 237 / 245).
    constexpr bool PRIO = !CALIB && (KSP > 1 || QK8 || (TEAMS > 1 && D == 128));
    auto stage = [&](ScoreTile &cur, ScoreTile &nxt, int j, auto fast_tag) {
        constexpr bool FAST = decltype(fast_tag)::value;
        bf16x8 pb[4];
        const uint32_t kept = CALIB ? 0u : opaque(cur.keep);
        // slot of K_{j+1}; K_{j+R} is requested into the same slot once block j+1 has left it
        // (R = KR + 1), so one ring position per stage is all the bookkeeping there is
        const uint32_t kt_next = lds_k0 + kring;
        kring = (kring + KSLOT == KR * KSLOT) ? 0u : kring + KSLOT;
        const unsigned char *const k_src = k_ahead, *const v_src = v_ahead;
        k_ahead += kstep_b;
        v_ahead += vstep_b;
        if (kept != 0u) {
            fused_exp_qk(cur, nxt, kt_next, pb);
        } else {
            qk_mfma(nxt, kt_next);
        }
        reduce_scores(nxt, j + 1, fast_tag);
        // copies that must have landed before the barrier: V_j (if requested) and K_{j+2}; every
        // younger request (K_{j+3} .. K_{j+R-1}, issued after V_j) may stay in flight
        if constexpr (R >= 4) {
            if (!CALIB && cur.any_keep != 0u) wait_vmcnt<NSTK>();
            else wait_vmcnt<(R >= 4 ? NSTK * (R - 3) : 0)>();
        } else {
            wait_vmcnt<0>();
        }
        wg_barrier();
        uint32_t flags[FW] = {};
        if constexpr (!CALIB) read_flags(flags, (j + 1) & 1);
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
        // The look-ahead -- decision for block j+1, its statistics, the requests for V_{j+1} and
        // K_{j+R}, the running maximum -- in pieces, so that a kept block can issue them between its
        // PV MFMAs a few instructions at a time.
        auto la_decide = [&]() {
            if constexpr (!CALIB) decide(nxt, flags);
            else nxt.keep = 1u;
        };
        auto la_stats = [&]() {
            record(nxt.keep, j + 1, fast_tag);
        };
        if (kept != 0u) {
            if constexpr (!CALIB) {
                const uint32_t vaddr = lds_v0 + (uint32_t)(j & 1) * VSLOT + va_base;
                vops_t a;
                pv_reads(a, vaddr);
                row_sum(pb);
                __builtin_amdgcn_sched_barrier(0);
                pv_head(cur, pb, a, vaddr);
                la_decide();
                const i32x4 krs = tile_rsrc(k_src, k_exist(j + R));
                // The copies are spread over the MFMAs: a run of them fills the queue in front of the memory pipe, and the
                // wave then waits at the next one (40 to 60 cycles each) instead of issuing MFMAs.
                constexpr int SLOTS = NPV - 2 - DB;           // hooks before the last operand reads
                if (nxt.any_keep != 0u) {
                    const i32x4 vrs = tile_rsrc(v_src, FAST ? kWholeTile : v_exist(j + 1));      // (a gateable block is never the partial one)
                    uint32_t ko = koff, vo = voff;
                    constexpr int PER = (NST + NSTK + SLOTS - 1) / SLOTS;
                    pv_tail(cur, pb, a, vaddr, [&](auto nc) {
                        constexpr int s = decltype(nc)::value - DB;
                        static_range<s * PER, (s + 1) * PER>([&](auto cc) {
                            constexpr int c = decltype(cc)::value;
                            if constexpr (c < NST) v_unit(cc, vo, vrs, lds_v0 + (uint32_t)((j + 1) & 1) * VSLOT);
                            else if constexpr (c < NST + NSTK) k_unit(std::integral_constant<int, c - NST>{}, ko, krs, kt_next);
                        });
                        if constexpr (s == SLOTS / 2 - 1) {
                            if constexpr (FAST) nxt.mx = pair_max(nxt.mx);
                        }
                        if constexpr (s == SLOTS / 2) softmax_max(nxt, TEAMS > 1 && nxt.keep == 0u ? -INFINITY : 0.f);
                        if constexpr (s == SLOTS / 2 + 1) softmax_alpha(nxt);
                        if constexpr (s == SLOTS - 1) la_stats();
                        if constexpr (s == SLOTS) prefetch_k(lds_k0 + kring);   // K_{j+2}: landed and visible since the barrier
                    });
                }
                if (opaque(nxt.any_keep) == 0u) {
                    uint32_t ko = koff;
                    constexpr int PER = (NSTK + SLOTS - 1) / SLOTS;
                    pv_tail(cur, pb, a, vaddr, [&](auto nc) {
                        constexpr int s = decltype(nc)::value - DB;
                        static_range<s * PER, (s + 1) * PER>([&](auto cc) {
                            if constexpr (decltype(cc)::value < NSTK) k_unit(cc, ko, krs, kt_next);
                        });
                        if constexpr (s == SLOTS - 1) la_stats();
                        if constexpr (s == SLOTS) prefetch_k(lds_k0 + kring);
                    });
                }
            }
        }
        if (opaque(kept) == 0u) {
            // the operand reads first, so that they travel while the look-ahead is issued (where V is
            // gathered in place the registers do not allow it: there they come last)
            if constexpr (VT || CALIB) prefetch_k(lds_k0 + kring);
            __builtin_amdgcn_sched_barrier(0);
            la_decide();
            if constexpr (!CALIB) {
                if (nxt.any_keep != 0u) {
                    if constexpr (FAST) nxt.mx = pair_max(nxt.mx);
                    softmax_max(nxt, TEAMS > 1 && nxt.keep == 0u ? -INFINITY : 0.f);
                    softmax_alpha(nxt);
                    copy_v_from(v_src, j + 1);
                }
            }
            copy_k_from(k_src, j + R, kt_next);
            la_stats();
            if constexpr (!(VT || CALIB)) prefetch_k(lds_k0 + kring);
        }
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
    };

    // The tile's last block (it touches the causal boundary, or there is no mask): nothing to look ahead to.
    auto last_stage = [&](ScoreTile &cur, int j) {
        if constexpr (!CALIB) {
            bf16x8 pb[4];
            if (cur.keep != 0u) softmax_exp(cur, pb);
            wait_vmcnt<0>();
            wg_barrier();
            if (cur.keep != 0u) {
                const uint32_t vaddr = lds_v0 + (uint32_t)(j & 1) * VSLOT + va_base;
                vops_t a;
                pv_reads(a, vaddr);
                pv_head(cur, pb, a, vaddr);
                pv_tail(cur, pb, a, vaddr, [](auto) {});
            }
        }
    };

    // ---- prologue: scores and decision of block 0 -----------------------------------------------
    ScoreTile ta, tb;
    wait_vmcnt<0>();
    wg_barrier();
    prefetch_k(lds_k0);
    qk_mfma(ta, lds_k0);
    prefetch_k(lds_k0 + kring);                            // K_1 for the first stage
    reduce_scores(ta, 0, std::false_type{});
    wg_barrier();                                       // flags visible, K_0 consumed
    if constexpr (!CALIB) {
        uint32_t flags[FW];
        read_flags(flags, 0);
        decide(ta, flags);
        if (KSP > 1 && n_own == 0) ta.keep = ta.any_keep = 0u;         // a share without blocks
        if (ta.any_keep != 0u) copy_v(0);
        if (ta.keep != 0u) softmax_begin(ta);
    } else {
        ta.keep = 1u;
    }
    copy_k(R - 1, lds_k0);                                 // the slot block 0 has just left
    if (KSP == 1 || n_own > 0) record(ta.keep, 0, std::false_type{});

    // main loop, two stages per trip.  A pair runs the mask-free stages when both of its
    // look-ahead blocks (j+1, j+2) exist and are gateable: every pair below the causal boundary;
    // without the causal mask every pair before the tile's own token range and, in a second
    // segment, every pair behind it (Section 4.3, last sentence: only the own-range blocks bypass the
    // gate).  The remaining blocks take the general stages, one at a time.
    int j = 0;
    for (int seg = 0; seg < 2; ++seg) {
        const int fast_end = (p.gate_mode || (!CALIB && p.block_max)) ? 0 : seg == 0 ? own(all_lo) : (p.causal ? 0 : n_own);
        for (; j + 2 < fast_end; j += 2) {
            stage(ta, tb, j, std::true_type{});
            stage(tb, ta, j + 1, std::true_type{});
        }
        // up to the first block whose look-ahead block lies behind the own range
        const int gen_end = (seg == 0 && !p.causal) ? min(own(all_hi) - 1, n_own - 1) : n_own - 1;
        for (; j < gen_end; ++j) {
            stage(ta, tb, j, std::false_type{});
            ta = tb;
        }
    }
    if constexpr (KSP > 1) {
        if (n_own > 0) last_stage(ta, j);
        for (int x = n_own; x < own_max; ++x) wg_barrier();          // every wave passes own_max barriers since the prologue
    } else {
        last_stage(ta, j);
    }

    if constexpr (CALIB) wait_vmcnt<0>();                 // (the last requests: nothing is in flight when the LDS is given back)

    // ---- statistics ------------------------------------------------------------------------
    if (!CALIB && n_own > 0 && (glob(n_own - 1) & 31) <= 31 - KSP) flush_mask(glob(n_own - 1));     // the last word, begun
    const int htid = tid - tsel * NWH * 64;               // thread index within the waves of a head and tile
    const bool stat_tile = QT == 1 || i < p.mq;
    if (p.block_max && ksel == 0 && stat_tile)
        for (int jj = n_tile + htid; jj < p.mkv; jj += NWH * 64) p.block_max[stat_row * p.mkv + jj] = NAN;
    if constexpr (KSP == 1) {
        if (p.skip_mask && stat_tile)
            for (int w = ((n_tile + 31) >> 5) + htid; w < p.mask_words; w += NWH * 64) p.skip_mask[stat_row * p.mask_words + w] = 0u;
    }
    if (p.counts && stat_lane) {
        unsigned long long *c = p.counts + ((int64_t)b * p.hq + h) * 3;
        const int gateable = p.causal ? n_gate : (p.mkv - (own_hi - own_lo));
        atomicAdd(c + 0, (unsigned long long)n_skipped);
        if (ksel == 0) {
            atomicAdd(c + 1, (unsigned long long)gateable);
            atomicAdd(c + 2, (unsigned long long)n_tile);
        }
    }

    // ---- the shares of a tile's key blocks put together: (m, l, O~) of every further share through LDS ----
    if constexpr (KSP > 1) {
        constexpr int PER_WAVE = 64 * (16 * DB + 2);      // floats
        static_assert((KSP - 1) * NWH * TEAMS * PER_WAVE * 4 <= (int)sizeof(lds_raw), "the tile slots hold the shares");
        float *const part = reinterpret_cast<float *>(lds_raw);
        wait_vmcnt<0>();                                  // (the last requests of a share without blocks)
        wg_barrier();                                     // nobody reads the slots any more; the mask words are complete
        if (p.skip_mask && ksel == 0 && stat_tile)
            for (int w = htid; w < p.mask_words; w += NWH * 64) p.skip_mask[stat_row * p.mask_words + w] = lds_mask[tsel][w];
        if (ksel > 0) {
            float *const mine = part + ((ksel - 1) * NWH * TEAMS + wave) * PER_WAVE + lane;
#pragma unroll
            for (int x = 0; x < DB; ++x)
#pragma unroll
                for (int e = 0; e < 16; ++e) mine[(16 * x + e) * 64] = oacc[x][e];
            mine[16 * DB * 64] = m_run;
            mine[(16 * DB + 1) * 64] = l_run;
        }
        wg_barrier();
        if (ksel > 0) return;
#pragma unroll 1
        for (int sh = 1; sh < KSP; ++sh) {
            const float *const its = part + ((sh - 1) * NWH * TEAMS + wave) * PER_WAVE + lane;
            const float m_its = its[16 * DB * 64], m_new = fmaxf(m_run, m_its);
            const float a_own = __builtin_amdgcn_exp2f(m_run - m_new), a_its = __builtin_amdgcn_exp2f(m_its - m_new);
            m_run = m_new;
            l_run = l_run * a_own + its[(16 * DB + 1) * 64] * a_its;
#pragma unroll
            for (int x = 0; x < DB; ++x)
#pragma unroll
                for (int e = 0; e < 16; ++e) oacc[x][e] = oacc[x][e] * a_own + its[(16 * x + e) * 64] * a_its;
        }
    }

    // ---- O_i = O~_i / l_i, written as bf16 ----------------------------------------------------
    if constexpr (!CALIB) {
        const float l_tot = l_run + __shfl_xor(l_run, 32);
        const float inv = 1.0f / l_tot;
        if (p.lse && hh == 0 && q_row < n_tok)      // L = m + log(l); m_run is in log2 units
            p.lse[((int64_t)b * p.seqlen + q_row) * p.hq + h] = m_run * 0.6931471805599453f + __logf(l_tot);
        // The wave's 32 rows go through LDS, so that a store instruction writes whole rows instead of 16 bytes of each
        // (32 rows of 16 bytes at a time the epilogue took 2.5 us of a workgroup at 128 x 128, all of it waiting for
        // addresses).  Their place is free: the K ring, which nobody reads after the barrier of the last stage, or the
        // share this wave has just merged.  16-byte chunks are XOR-ed with the row, which spreads them over the banks.
        static_assert(KSP > 1 || NWH * TEAMS * 32 * ROW_BYTES <= KR * KSLOT, "the K ring holds the output rows");
        const uint32_t o_lds = KSP > 1 ? (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)lds_raw) + wave * (64 * (16 * DB + 2) * 4)
                                       : lds_k0 + wave * (32 * ROW_BYTES);
        auto swz_o = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
        const uint32_t o_row = o_lds + l32 * ROW_BYTES + 8 * hh;
        asm volatile("" ::: "memory");              // (a merged share has been read; one wave's LDS accesses complete in order)
#pragma unroll
        for (int x = 0; x < DB; ++x)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                // O^T row 8*e4 + 4hh + e of block x -> head-dim column (see the V operand mapping)
                const int m0 = 8 * e4;
                const int d0 = VT ? 32 * x + m0 : X_COLS * x + (m0 < 16 ? m0 : G16_COLS + m0 - 16);
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (el)(oacc[x][4 * e4 + e] * inv);
                *LDS_PTR(bf16x4, o_row + (((d0 >> 3) ^ swz_o(l32)) << 4)) = o;
            }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        uint16_t *op = p.out + (int64_t)b * p.osb + (int64_t)h * p.osh;
#pragma unroll
        for (int it = 0; it < 32 * CPR / 64; ++it) {
            const int row = it * (64 / CPR) + lane / CPR, c = lane % CPR;
            const i32x4 o = *LDS_PTR(const i32x4, o_lds + row * ROW_BYTES + ((c ^ swz_o(row)) << 4));
            const int token = (int)row0 + wrow * 32 + row;
            if (token < n_tok) *reinterpret_cast<i32x4 *>(op + (int64_t)token * p.osn + 8 * c) = o;   // (padding rows of the last tile are not stored)
        }
    }
}

static __global__ void zero_counts_kernel(unsigned long long *c, int n)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) c[t] = 0ull;
}

// V -> workspace, once per forward call: for every (batch, KV head, 64-key block) the tile V_j^T in
// exactly the byte order the forward kernel wants in LDS (see its operand addresses): D rows of 64
// keys; inside a 16-key step the keys are ordered 0-3, 8-11, 4-7, 12-15 (the 8 keys one lane of the
// second MFMA multiplies are then 16 contiguous bytes); unit r of 1024 bytes holds the rows r, r + 16, ... r + 112.
// Rows at and beyond the sequence end repeat the last token (Section 4.3), so the
// tile of a partial block holds finite values everywhere; blocks that lie entirely beyond the end
// are never read and are not written.  One workgroup per tile, through LDS.
static __global__ void __launch_bounds__(256) transpose_v_kernel(const FwdParams p)
{
    constexpr int BN = kBlockN, D = 128, CPR = D / 8, LD = D + 8;
    __shared__ __attribute__((aligned(16))) uint16_t tile[BN * LD];
    const int j = blockIdx.x, g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    if (p.counts && j == 0 && g == 0 && b == 0)       // (saves the launch that would clear them)
        for (int t = tid; t < p.batch * p.hq * 3; t += 256) p.counts[t] = 0ull;
    int n_tok = p.seqlen;
    if (p.seqlens) n_tok = min(max(p.seqlens[b], 0), p.seqlen);
    if (j * BN >= n_tok) return;
    const uint16_t *src = p.v + (int64_t)b * p.vsb + (int64_t)g * p.vsh;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    for (int sigma = tid; sigma < BN * CPR; sigma += 256) {
        const int row = sigma / CPR, cp = sigma % CPR;
        const int tok = min(j * BN + row, n_tok - 1);
        const u32x4 c = *reinterpret_cast<const u32x4 *>(src + (int64_t)tok * p.vsn + 8 * cp);
        *reinterpret_cast<u32x4 *>(&tile[row * LD + 8 * cp]) = c;
    }
    __syncthreads();
    uint16_t *dst = p.vt + (((int64_t)b * p.hkv + g) * p.mkv + j) * (int64_t)(BN * D);
    for (int sigma = tid; sigma < D * 8; sigma += 256) {
        const int d = (sigma >> 6) + 16 * ((sigma >> 3) & 7);
        const int c = sigma & 7;                     // chunk: 16-key step c >> 1, lane half c & 1
        const int u = c >> 1, hh = c & 1;
        uint16_t w[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) w[t] = tile[(16 * u + 8 * (t >> 2) + 4 * hh + (t & 3)) * LD + d];
        u32x4 o;
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = (uint32_t)w[2 * t] | ((uint32_t)w[2 * t + 1] << 16);
        *reinterpret_cast<u32x4 *>(dst + (int64_t)sigma * 8) = o;
    }
}

// K -> workspace as fp8 (e4m3, round to nearest even), once per call, for the fp8 score product: for
// every (batch, KV head, 64-key block) a tile of 64 rows x 128 bytes in the byte order the forward
// kernel wants in LDS (unit r of 1024 bytes holds the rows r, r + 8, ... r + 56).  Rows at and beyond the
// sequence end repeat the last token (Section 4.3).  head_dim 128 only.
template <bool F16>
__global__ void __launch_bounds__(256) quantize_k_kernel(const FwdParams p)
{
    typedef typename Elem<F16>::x8 x8;
    constexpr int BN = kBlockN, D = 128;
    const int j = blockIdx.x, g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    int n_tok = p.seqlen;
    if (p.seqlens) n_tok = min(max(p.seqlens[b], 0), p.seqlen);
    if (j * BN >= n_tok) return;
    const uint16_t *src = p.k + (int64_t)b * p.ksb + (int64_t)g * p.ksh;
    uint8_t *dst = p.k8 + (((int64_t)b * p.hkv + g) * p.mkv + j) * (int64_t)(BN * D);
    for (int sigma = tid; sigma < BN * 8; sigma += 256) {
        const int row = (sigma >> 6) + 8 * ((sigma >> 3) & 7);
        const int c = sigma & 7;                              // head-dim elements 16c .. 16c + 15
        const int tok = min(j * BN + row, n_tok - 1);
        const uint16_t *e = src + (int64_t)tok * p.ksn + 16 * c;
        i32x4 o;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const x8 v8 = *reinterpret_cast<const x8 *>(e + 8 * half);
            float f[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) f[t] = (float)v8[t];
            int w0, w1;
            cvt8_fp8(f, w0, w1);
            o[2 * half] = w0;
            o[2 * half + 1] = w1;
        }
        *reinterpret_cast<i32x4 *>(dst + (int64_t)sigma * 16) = o;
    }
}

// the call's parameters with the divisors of the work decomposition (decode_work), and its workgroups (0: they do
// not fit a launch)
template <int HP, int QT> static unsigned decompose(FwdParams &p)
{
    const long pairs = (long)p.batch * p.hkv, gsub = p.group / HP, mqg = (p.mq + QT - 1) / QT;
    const long per_tile = (pairs >= 8 ? (pairs + 7) / 8 : pairs) * gsub, wide = pairs >= 8 ? 8 : 1;
    if (pairs <= 0 || per_tile <= 0 || per_tile * wide * mqg > 0x7fffffffL) return 0u;
    p.div_tile = fast_div((uint32_t)per_tile);
    p.div_gsub = fast_div((uint32_t)gsub);
    p.div_hkv = fast_div((uint32_t)p.hkv);
    p.turn[0] = p.turn[1] = p.turn[2] = 0;
    const unsigned n = (unsigned)(per_tile * wide * mqg);
    p.counted = p.seqlens && pairs <= 128 && n > 256;
    return n;
}

// K -> workspace as fp8 tiles and V -> workspace as transposed tiles, as far as the call has room for them
static hipError_t launch_prepasses(const FwdParams &p, hipStream_t stream)
{
    if (!p.vt && !p.k8) return hipSuccess;
    if (p.hkv > 65535 || p.batch > 65535) return hipErrorInvalidValue;    // grid y, z limits
    const dim3 tiles((unsigned)p.mkv, (unsigned)p.hkv, (unsigned)p.batch);
    if (p.vt) hipLaunchKernelGGL(transpose_v_kernel, tiles, dim3(256), 0, stream, p);
    if (p.k8 && p.f16) hipLaunchKernelGGL((quantize_k_kernel<true>), tiles, dim3(256), 0, stream, p);
    if (p.k8 && !p.f16) hipLaunchKernelGGL((quantize_k_kernel<false>), tiles, dim3(256), 0, stream, p);
    return hipGetLastError();
}

// Where a CU holds two or three workgroups and a causal call has no more than fill these places twice, the second and
// the third workgroup of every CU are dealt the other way round, so that the longest tiles share their CU with the
// shortest of the rest and not with the next longest.  In order / turned, us, bf16, half skip (dense): head_dim 64,
// 64-row tiles, 2 x 4096 tokens of 12 heads over 4 (768 workgroups) 58.5 / 57.3 (73.8 / 67.7), 12 000 tokens (1128) 210 / 201,
// 4096 tokens of 28 over 4 (896) 63.4 / 61.6; 32-row tiles, 3500 tokens of 32 over 8 57.0 / 54.5; head_dim 128, 32 over 8,
// 2300 tokens (576) 47.4 / 46.7 (56.8 / 56.0), 4096 tokens (1024) 113.9 / 111.3 (148.2 / 141.4); 28 over 4, 4096 tokens in
// 64-row tiles 105.8 / 103.5; at worst 0.8 % slower (3500 tokens of 32 heads half skip 90.7 / 91.4, dense 117.1 / 112.1).  With more
// than that, what is dealt first is soon forgotten (6000 tokens of 32 heads 226 / 226), and tiles that are split are as short
// as the call allows (2300 tokens of 12 over 4, head_dim 64, 29.3 / 31.8).
static void turned_places(FwdParams &p, unsigned workgroups, int places)
{
    const bool xcd = (int64_t)p.batch * p.hkv >= 8;        // (as decode_work counts them)
    const unsigned n = xcd ? workgroups / 8 : workgroups, cus = xcd ? 32 : 256;
    if (places == 1 || !p.causal || p.seqlens || n <= cus || n > 2 * places * cus) return;
    p.turn[0] = cus;
    p.turn[1] = std::min(n, 2 * cus);
    p.turn[2] = std::min(n, places * cus);
}

// forward pass; `spare` bytes of LDS more than a workgroup needs keep others off its CU
template <int D, int NWH, int HP, int QT, int KSP, int KR>
hipError_t launch_fwd(const FwdParams &params, hipStream_t stream, unsigned spare = 0)
{
    FwdParams p = params;
    const dim3 grid(decompose<HP, QT>(p)), threads(NWH * HP * QT * KSP * 64);
    if (grid.x == 0) return hipErrorInvalidValue;
    turned_places(p, grid.x, std::min(places_of(D, NWH * HP * QT, KSP), spare ? 2 : 3));
    constexpr bool WS = NWH == 4 && KSP == 1 && D == 128;      // V (and fp8 K) from the workspace, if the call has one
    if (p.k8 && (!WS || !p.vt)) return hipErrorInvalidValue;
    if (p.counts && !(WS && p.vt)) {                   // (the pass over V clears them)
        const int n = p.batch * p.hq * 3;
        hipLaunchKernelGGL(zero_counts_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, p.counts, n);
    }
    if constexpr (WS) {
        const hipError_t e = launch_prepasses(p, stream);
        if (e != hipSuccess) return e;
    }
#define BSFA_LAUNCH(F16, VT, QK8) hipLaunchKernelGGL((bsfa_fwd_kernel<D, NWH, HP, QT, KSP, KR, false, F16, VT, QK8>), grid, threads, spare, stream, p)
    if constexpr (WS) {
        if (p.k8) {
            if (p.f16) BSFA_LAUNCH(true, true, true);
            else BSFA_LAUNCH(false, true, true);
            return hipGetLastError();
        }
        if (p.vt) {
            if (p.f16) BSFA_LAUNCH(true, true, false);
            else BSFA_LAUNCH(false, true, false);
            return hipGetLastError();
        }
    }
    if (p.f16) BSFA_LAUNCH(true, false, false);
    else BSFA_LAUNCH(false, false, false);
#undef BSFA_LAUNCH
    return hipGetLastError();
}

// score / block-maximum half (calibration)
template <int D, int NWH, int HP, int QT, int KR>
hipError_t launch_scores(const FwdParams &params, hipStream_t stream)
{
    FwdParams p = params;
    const dim3 grid(decompose<HP, QT>(p)), threads(NWH * HP * QT * 64);
    if (grid.x == 0) return hipErrorInvalidValue;
    constexpr bool FP8 = NWH == 4 && D == 128;
    if (p.k8 && !FP8) return hipErrorInvalidValue;     // fp8 score operands need the 128 x 64 tile and head_dim 128
#define BSFA_LAUNCH(F16, QK8) hipLaunchKernelGGL((bsfa_fwd_kernel<D, NWH, HP, QT, 1, KR, true, F16, false, QK8>), grid, threads, 0, stream, p)
    if constexpr (FP8) {
        if (p.k8) {
            const hipError_t e = launch_prepasses(p, stream);
            if (e != hipSuccess) return e;
            if (p.f16) BSFA_LAUNCH(true, true);
            else BSFA_LAUNCH(false, true);
            return hipGetLastError();
        }
    }
    if (p.f16) BSFA_LAUNCH(true, false);
    else BSFA_LAUNCH(false, false);
#undef BSFA_LAUNCH
    return hipGetLastError();
}

// The instantiations are spread over several translation units, compiled side by side from this one file:
// BSFA_PART says which of them this one holds (0: the dispatch, none of them).
// F(head_dim, waves per head and tile, heads, tiles, shares of the key blocks, K ring), S(head_dim, waves per head and tile, heads, tiles, K ring)
#define BSFA_SHAPES_1(F, S) F(128, 4, 1, 1, 1, 2) F(128, 4, 2, 1, 1, 5)
#define BSFA_SHAPES_2(F, S) F(128, 4, 1, 1, 2, 2) F(64, 4, 1, 1, 1, 3) F(64, 4, 1, 1, 2, 3)
#define BSFA_SHAPES_3(F, S) S(128, 4, 2, 1, 4) S(128, 4, 1, 1, 2) S(64, 4, 1, 1, 3) S(128, 2, 2, 1, 2) S(128, 2, 1, 2, 2) S(64, 2, 2, 1, 4) S(64, 2, 1, 2, 4) S(128, 2, 1, 1, 2) S(64, 2, 1, 1, 2)
#define BSFA_SHAPES_4(F, S) F(128, 2, 2, 1, 1, 2) F(128, 2, 1, 2, 1, 2) F(128, 2, 1, 1, 1, 2)
#define BSFA_SHAPES_5(F, S) F(128, 2, 1, 2, 2, 2) F(128, 2, 1, 1, 2, 2) F(64, 2, 1, 1, 4, 2)
#define BSFA_SHAPES_6(F, S) F(64, 1, 2, 1, 1, 2) F(128, 1, 2, 1, 1, 2) F(64, 2, 2, 1, 1, 4) F(64, 2, 1, 2, 1, 4) F(64, 2, 1, 1, 1, 2) F(64, 2, 1, 1, 2, 2)
#define BSFA_SHAPES_7(F, S) F(128, 1, 4, 1, 1, 2) F(128, 1, 2, 2, 1, 2) F(128, 1, 1, 4, 1, 2)
#define BSFA_SHAPES_8(F, S) F(64, 1, 1, 2, 1, 2) F(64, 1, 1, 1, 1, 2) F(128, 1, 1, 4, 2, 2) F(128, 1, 1, 2, 2, 2) F(64, 1, 1, 2, 4, 2)
#define BSFA_SHAPES_9(F, S) F(64, 1, 4, 1, 1, 4) F(64, 1, 2, 2, 1, 4) F(64, 1, 1, 4, 1, 4) F(64, 1, 1, 2, 2, 2)
#define BSFA_SHAPES_10(F, S) S(128, 1, 4, 1, 2) S(128, 1, 2, 2, 2) S(128, 1, 1, 4, 2) S(64, 1, 4, 1, 4) S(64, 1, 2, 2, 4) S(64, 1, 1, 4, 4)
#define BSFA_EXTERN_F(D, N, H, Q, P, K) extern template hipError_t launch_fwd<D, N, H, Q, P, K>(const FwdParams &, hipStream_t, unsigned);
#define BSFA_EXTERN_S(D, N, H, Q, K) extern template hipError_t launch_scores<D, N, H, Q, K>(const FwdParams &, hipStream_t);
#define BSFA_DEFINE_F(D, N, H, Q, P, K) template hipError_t launch_fwd<D, N, H, Q, P, K>(const FwdParams &, hipStream_t, unsigned);
#define BSFA_DEFINE_S(D, N, H, Q, K) template hipError_t launch_scores<D, N, H, Q, K>(const FwdParams &, hipStream_t);
#if BSFA_PART == 0
BSFA_SHAPES_1(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_2(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_3(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_4(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_5(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_6(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_7(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_8(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_9(BSFA_EXTERN_F, BSFA_EXTERN_S)
BSFA_SHAPES_10(BSFA_EXTERN_F, BSFA_EXTERN_S)

bool shape_supported(int head_dim, int block_m, int block_n)
{
    if (block_n != kBlockN) return false;
    if (head_dim != 64 && head_dim != 128) return false;
    return block_m == 32 || block_m == 64 || block_m == 128;
}

// Which kernel a call gets.  Figures: us, bf16, 32 query heads over 8 KV heads, half skip, unless stated.
//
// `rows` -- query rows over all heads, twice as many without the causal mask -- is what most lines depend on: a
// tile's key blocks are taken one after the other, so a call takes at least the longest tile's chain, and the chip
// holds 512 workgroups of four waves (rows 65 536 in 128-row tiles).
//  - Up to there the key blocks of a tile may be dealt to two sets of waves (KSP = 2, split_of): half the chain
//    for the same work, at the price of a merge, of a K/V stream for each set, and of half the places: a split
//    workgroup of eight waves has a CU to itself.  One set against two, 128-row tiles:
//     * as long as every workgroup has a place (8 heads over 2, 256 tiles): 1000 tokens 25.1 / 22.2, 2048 tokens
//       37.6 / 31.7, 4096 tokens 66.9 / 53.1, 512 tokens dense 17.3 / 16.8.  (Below that the merge costs more than the
//       chain, 300 tokens dense 12.3 / 12.6, 64 tokens 7.0 / 9.1, but a call then takes the host 11 us; and an element
//       gets the bits of a call of its own as long as the batch has no more workgroups than that.)
//     * with up to two workgroups to a place it takes a chain of 20 blocks or more (8 x 1000 tokens of 8 heads, 512 tiles,
//       27.3 / 31.7; 2 x 2048 tokens of 12 over 4, 384, 35.9 / 35.4, dense 42.8 / 39.1; 3000 tokens of 16 over 8, 384,
//       48.4 / 41.5), and of 32 where nearly every place is taken (turned_places: 1700 tokens of 32 heads, 448 tiles,
//       32.8 / 36.6, dense 38.4 / 39.7; 2048 tokens 41.2 / 41.1, dense 48.2 / 47.1), at head_dim 64 of 28 (1900 tokens of 28 over
//       4, 420 tiles, half skip 26.2 / 26.4, dense 31.5 / 29.9; 1700 tokens of 32 heads, 27 blocks, 25.3 / 26.0, 28.5 / 28.4).
//       Elements of different lengths leave places free and are not turned: 20 blocks there too (2 x up to 1900 tokens of 14
//       over 2 33.1 / 28.6, head_dim 64 27.1 / 21.7; 4 x up to 1700 of 8 over 8 33.0 / 27.7), unless every XCD has a single
//       element's KV head, and that of the longest as many tiles as without lengths (4 x up to 1700 of 8 over 2 34.6 / 35.9).
//     * beyond that nothing is gained but for the longest chains (9 x 1536 tokens of 4 heads, whose KV heads lie
//       unevenly on the XCDs, 35.4 / 46.4, 2125 tokens of 32 heads 44.1 / 51.4; 2 heads, 34K tokens 548 / 460), and
//       from rows 65 536 on tiles are not split (2 heads, 49K tokens 918 / 950).
//     * with lengths the lines count the longest element's tokens for every element, as nothing else is known here.  What a
//       split gives there depends on the others: 4 x up to 3000 tokens of 8 heads, 768 tiles, 55.7 / 50.8, 2 x up to 3000 of 16 over
//       8, 768, 62.7 / 70.6, 4 x up to 2000 of 16 over 8, 1024, 40.8 / 50.4.
//  - Tiles of 64 and 32 rows: a workgroup takes several, so that it has the waves of a 128-row tile (narrow: of 64 rows) on
//    one K/V stream.  What that leaves is the question above, with workgroups counted in 128 or in 64 rows (n128, n64; one
//    set of waves on 128 rows / two on 128 / two on 64, at head_dim 64 four on 64 as well).  Figures of 64-row tiles; those of
//    32 rows, on the same workgroups, lie up to 10 % above them on both sides of a line (2 x 1700 tokens of 12 over 4 34.9 / 30.6 /
//    39.7 and 36.5 / 31.8 / 43.5; 3000 tokens of 20 over 4 57.6 / 53.6 / 73.9 and 59.5 / 56.4 / 79.4; width 64, 1100 tokens of 28 over
//    4, one on 128 / two on 64 / four on 64, 19.5 / 14.2 / 19.8 and 20.0 / 15.2 / 20.5):
//     * head_dim 128.  2 heads, 4800 tokens (n64 150) 76 / 56 / 46, 14 400 tokens (450) 211 / 148 / 126, 12 heads over 4, 2384
//       tokens (456) 44 / 35.2 / 34.1; from n64 512 on a CU that holds two workgroups of 64 rows has a wave too few (2709 tokens,
//       516: - / 39.1 / 43.0), and short chains gain less than the second workgroup costs (28 heads over 4, 1026 tokens, 476:
//       22.9 / 21.4 / 23.8; 32 heads, 650 tokens, 352: 17.4 / 16.8 / 18.2): narrow up to 256 workgroups, up to 512 from 24 key
//       blocks on.  Two on 128 as for 128-row tiles (8 over 8, 8000 tokens 129 / 115, 11 200 tokens 217 / 221), but for chains of
//       fewer than 8 blocks (one on 64 / one on 128 / two on 128: 64 x 100 tokens of 3 heads 9.2 / 9.4 / 10.7, of 4 over 2 - / 8.9 /
//       10.8, 8 x 250 of 12 over 4 11.4 / 12.1 / 12.5; 8 blocks, 4 x 450 of 12 over 4 15.0 / 15.2 / 14.5).
//     * head_dim 64 (one on 128 / two on 64 / four on 64; two workgroups of two sets on a CU, one of four).  2 heads, 4800
//       tokens 59 / 35 / 28.5, 16K (512) 188 / 105 / 89; 8 over 8, 2632 tokens (336) - / 23.6 / 21.4, 4096 tokens (512, 64
//       blocks) - / 32.2 / 32.6; 12 over 4, 784 tokens (156, 13 blocks) - / 10.6 / 11.2: four up to 256 workgroups from 16 key
//       blocks on, up to 384 from 40, up to 512 from 96.  Two up to 512, up to 1024 from 18 blocks on (28 over 4, 1161 tokens
//       18.7 / 14.6; 3 x 1000 tokens of 12 over 4, 16 blocks, 18.4 / 18.9), up to 1536 from 100 on (12 over 4, 7445 tokens
//       101 / 98; 32 heads, 2776 tokens 41 / 46).
//       32-row tiles of fewer than four key blocks are not split (as above; they were not before they shared workgroups).
//  - V is rewritten into the workspace only where the pass over it pays for itself, which takes its reuse by many
//    query tiles: head_dim 128, 128-row tiles, beyond 12K tokens.  In place / rewritten, single heads: 8K tokens
//    408 / 411, 12K 899 / 900, 16K 1569 / 1565, 32K 6075 / 6026 (dense 8166 / 8093); 64 heads over 8, whose reuse is
//    twice that: 8K 814 / 810, 12K 1779 / 1760; 16 over 8: 12K 451 / 456, 24K 1724 / 1718; 8 over 8, the least
//    reuse: 12K 238 / 247, 24K 876 / 881, 32K 1542 / 1549 and dense even.  At head_dim 64 it never paid (8K tokens
//    256 / 268, 32K 3690 / 3810 with an earlier kernel) and is not built.  The fp8 score product is built for the
//    rewritten V.
//  - Heads of a GQA group that share a workgroup share one K/V stream in LDS.  128-row tiles have waves enough
//    without that, and two independent workgroups on a CU hide each other's barriers: single heads against pairs,
//    8K tokens 408 / 416 (dense 542 / 534), 20K 2406 / 2483 (3191 / 3182), 24K 3474 / 3553 (4575 / 4583), and more the
//    more is skipped (24K, 90 %: 2444 / 2662).  But they read twice as much from L2 for a launch that the card's power
//    limits: 32K dense 8186 / 8074, half skip 6195 / 6212; 128K 2.5 % slower at half skip.  So pairs beyond 24K
//    tokens; with the fp8 score product, whose K stream is half as wide, beyond 64K (16K tokens 6 % faster single,
//    64K 2 %).  Without the mask, where all tiles are equally long, beyond 3K (3072 tokens 128 / 147, 4096 209 / 207,
//    16K dense 4008 / 3946).
//    A causal call of 865 to 1024 tiles, nearly two for each of the 512 places, is the exception: from 8K tokens on
//    pairs are faster there, unless most is skipped (single / pairs: 8 heads over 2, 16K tokens dense 569 / 521, half
//    434 / 407, 90 % 289 / 305; 16 over 8, 8K tokens 295 / 272, 225 / 212, 156 / 166).
//    Smaller tiles share a stream in any case: heads of a group where they can (two of 64 rows; four, or two and two tiles, of
//    32), else adjacent query tiles, which costs at most 1.3 % more (8K tokens in 64-row tiles 414 / 419, of width 64 239 / 242,
//    in 32-row tiles of width 64 254 / 247).  Before, a tile of an odd group was a workgroup of one or two waves on a stream of
//    its own (tile alone / tiles together: 28 heads over 4, 4096 tokens in 64-row tiles 128 / 110, in 32-row tiles 255 / 119; 12
//    over 4, 9151 tokens in 32-row tiles 570 / 254; width 64, 28 over 4, 8192 tokens 240 / 218, 355 / 222).
//    A 64-row tile of width 128 is left alone where every tile has a place, and where a sequence is a single tile (alone / with
//    the next: 24 x 190 tokens of 6 over 2, 432 tiles, 10.8 / 11.9; 300 x 60 of 3 over 1, 904, 14.0 / 16.5; 64 x 130 of 3 heads, 576,
//    12.6 / 11.7), and with elements of different lengths, which leave places free, up to 640 tiles, from 8 key blocks on 1024,
//    from 12 on 1152 (4 x up to 900 tokens of 16 heads, 960, 21.1 / 23.4; 3 x up to 3000 of 8, 1128, 50.0 / 56.1; 8 x up to 500 of 12
//    over 4, 768, 15.1 / 16.7, of 16, 1024, 16.5 / 17.2; 100 x up to 100 of 3 over 1, 624, 9.5 / 11.3; 64 x up to 127 of 6 over 2, 768, 14.2 /
//    12.4; 16 x up to 300 of 12 over 4, 960, 15.1 / 13.3; 4 x up to 600 of 28 over 4, 1120, 19.6 / 18.8;
//    3 x up to 2000 of 16, 1536, 43.2 / 43.3; 2 x up to 5000, 2528, 164 / 126).
//    A 64-row tile of width 64 of an odd group likewise (four alone or three pairs to a CU), in sequences of four tiles or
//    fewer also where both take more rounds (64 x 130 tokens of 3 heads, 576 tiles, 8.4 / 9.3; 1000 tokens of 40 over 8, 640,
//    16.9 / 18.5, dense 19.5 / 20.4; 300 x 60 of 3 heads 8.0 / 11.3; 200 x 180, 1800, 15.1 / 18.5; 150 x 250, 1824, 16.1 / 18.5;
//    100 x 250, 1248, 14.2 / 13.6; 300 x 90, 3600, 24.6 / 25.3).  With elements of different lengths a tile is left alone up to rows
//    262 144 where heads are even or on their own (4 x up to 2000 tokens of 16 heads 28.9 / 31.0, 3 x up to 7000 of 8 over 8
//    86 / 92; 2 x up to 5000 of 32 heads, rows 320 000, 155 / 143), and where three or more heads of an odd group read the same K and
//    V up to rows 196 608 and 40 key blocks, and in sequences of up to two tiles (100 x up to 100 tokens of 3 heads 7.6 / 9.4, 300 x up to 128
//    12.7 / 14.6; 16 x up to 300 tokens of 28 over 4 15.7 / 18.5; 4 x up to 900 of 12 over 4 16.0 / 18.2; 6 x
//    up to 2500 41.8 / 43.3; 2 x up to 3000 of 28 over 4 72.2 / 70.5, 2 x up to 5000 of 12 over 4 83 / 78).
//    A workgroup of several 32-row tiles has waves without one where a sequence is a single tile: heads alone share there (one
//    tile / several: 2000 x 10 tokens of 4 over 2 41.4 / 47.1, of width 64 21.7 / 30.3; width 64, of 3 heads 24.4 / 40.2, 300 x 30 tokens
//    6.2 / 10.3; four heads or, up to 1024 heads, two: 64 x 20 of 8 over 2 6.3 / 5.4, 300 x 30 10.0 / 10.8).  Tiles of width 64 of an odd
//    group are put together in twos or fours as 64-row tiles are alone or together: (twos / fours: 64 x 130 tokens of 3 heads 7.8 / 9.1,
//    1000 of 40 over 8 17.5 / 19.1, 200 x 180 of 3 over 1 15.8 / 18.7, 100 x 250 14.9 / 13.5), with elements of different lengths up to
//    rows 81 920 or six key blocks (4 x up to 900 tokens of 16 heads 17.1 / 18.3, 3 x up to 3000 of 8 40.1 / 42.8, 16 x up to 300 of 28 over
//    4 16.2 / 18.4; 8 x up to 500 15.2 / 14.3, 2 x up to 5000 of 12 over 4 87 / 80).
//  - 128-row tiles of head_dim 64: the CU holds three workgroups.  For a causal call of 513 to 768 tiles, which all
//    three would hold at once, two to a CU are faster beyond 4K tokens (three / two: 8 heads over 8, 12K tokens
//    165.5 / 155.3; 2 heads, 49K tokens 624 / 590; 28 heads over 4, 3500 tokens 52.8 / 56.4).
//  - The score half alone (calibration) has registers and LDS to spare and shares where it can.  128-row tiles from
//    rows 262 144 on (whole calibrations, single / pairs: 8K tokens 268.9 / 270.3, 16K 913 / 904); 64-row tiles always
//    (500 tokens 46.0 / 46.4, 16K 1106 / 922; head_dim 64 595 / 541); 32-row tiles four (16K single 1571, pairs 1093,
//    four 919; head_dim 64 748, 682, 542; up to 1000 tokens all within 1 us).  64-row tiles of an odd group are alone up to 256
//    tiles, at head_dim 64 and in sequences of up to four 512 (589 tokens of 12 over 4, 120 tiles, alone / in twos 16.5 / 17.3, head_dim 64 14.8 / 15.8; 800 of 28
//    over 4, 364, 19.0 / 18.8, 16.6 / 16.8; 8 x 200 of 12 over 4, 384, 21.1 / 21.5, 20.1 / 20.8).
// Results do not depend on how heads share; the split does change the order of sums, so it must not depend on
// single_head or on the workspace, between which results are equal bit for bit.
static int64_t dispatch_rows(const FwdParams &p) { return (int64_t)p.batch * p.hq * p.seqlen * (p.causal ? 1 : 2); }

// workgroups of one head and `rows` query rows, with the empty ones that deal KV heads to XCDs
static int64_t workgroups_of(const FwdParams &p, int rows)
{
    const int64_t kv = (int64_t)p.batch * p.hkv, heads = (kv >= 8 ? (kv + 7) / 8 * 8 : kv) * p.group;
    return heads * ((p.seqlen + rows - 1) / rows);
}

// How a tile's key blocks are dealt, and for tiles of 64 and 32 rows how many query rows a workgroup takes (tiles of
// 128 rows are a workgroup each).
struct Split {
    int shares;           // sets of waves that the key blocks of a tile are dealt to
    bool narrow;          // 64 query rows to a workgroup instead of 128
};
static Split split_of(const FwdParams &p, int head_dim, int block_m)
{
    // (the comparison predicate depends on the order of the blocks; the mask words of a split tile must fit the LDS)
    if (p.k8 || p.gate_mode || p.mask_words > kSplitMaskWords) return {1, false};
    const int64_t kv = (int64_t)p.batch * p.hkv, n64 = workgroups_of(p, 64), n128 = workgroups_of(p, 128);
    if (block_m < 128 && (block_m == 64 || p.mkv >= 4)) {
        if (head_dim == 128) {
            if (n64 <= 256 || (p.causal && n64 <= 512 && p.mkv >= 24)) return {2, true};
        } else {
            if (n64 <= 256 ? p.mkv >= 16 : p.causal && n64 <= 512 && p.mkv >= (n64 <= 384 ? 40 : 96)) return {4, true};
            if (n64 <= 512 || (p.causal && n64 <= 1536 && p.mkv >= (n64 <= 1024 ? 18 : 100))) return {2, true};
        }
    }
    if (block_m < 128 && (head_dim == 64 || (block_m == 32 && p.mkv < 4))) return {1, false};
    const int taken = p.seqlens && kv != 8 ? 20 : head_dim == 64 ? 28 : 32;      // the line where nearly every place is taken
    const bool split = dispatch_rows(p) <= 65536 && ((n128 <= 256 && (block_m == 128 || p.mkv >= 8)) || (p.causal && p.mkv >= (n128 <= 400 ? 20 : n128 <= 512 ? taken : 64)));
    return {split ? 2 : 1, false};
}

// Whether a 64-row tile that shares its workgroup with no other head is left alone, and not put together with the next one:
// where that takes no more rounds of workgroups (`one`, `pair`: places of the chip for tiles alone and for pairs); with
// elements of different lengths, whose workgroups are fewer than that, up to `lengths` tiles and where there is no next one.
static bool tile_alone(const FwdParams &p, int64_t one, int64_t pair, int64_t lengths)
{
    const int64_t n64 = workgroups_of(p, 64), n128 = workgroups_of(p, 128);
    return p.seqlens ? n64 <= lengths || p.seqlen <= 64 : (n64 + one - 1) / one <= (n128 + pair - 1) / pair;
}

bool rewrites_v(const FwdParams &p, int head_dim, int block_m)
{
    return v_rewrite_pays(head_dim, block_m, p.seqlen) && split_of(p, head_dim, block_m).shares == 1;
}

hipError_t launch_forward(const FwdParams &p, int head_dim, int block_m, bool calib, hipStream_t stream)
{
    if (!shape_supported(head_dim, block_m, kBlockN)) return hipErrorInvalidValue;
    // the copies address a tile with 32-bit byte offsets
    if (p.ksn * 128 > 0x7fff0000LL || p.vsn * 128 > 0x7fff0000LL) return hipErrorInvalidValue;
    const bool two = p.group % 2 == 0 && !p.single_head, four = p.group % 4 == 0 && !p.single_head;
    const int64_t rows = dispatch_rows(p);
    const bool d128 = head_dim == 128;
    if (calib) {
        if (block_m == 128)
            return !d128 ? launch_scores<64, 4, 1, 1, 3>(p, stream)
                 : two && rows > 262144 ? launch_scores<128, 4, 2, 1, 4>(p, stream) : launch_scores<128, 4, 1, 1, 2>(p, stream);
        if (block_m == 64 && !two && workgroups_of(p, 64) <= (d128 && p.mq > 4 ? 256 : 512))
            return d128 ? launch_scores<128, 2, 1, 1, 2>(p, stream) : launch_scores<64, 2, 1, 1, 2>(p, stream);
        if (block_m == 64)
            return d128 ? (two ? launch_scores<128, 2, 2, 1, 2>(p, stream) : launch_scores<128, 2, 1, 2, 2>(p, stream))
                        : (two ? launch_scores<64, 2, 2, 1, 4>(p, stream) : launch_scores<64, 2, 1, 2, 4>(p, stream));
        return d128 ? (four ? launch_scores<128, 1, 4, 1, 2>(p, stream) : two ? launch_scores<128, 1, 2, 2, 2>(p, stream) : launch_scores<128, 1, 1, 4, 2>(p, stream))
                    : (four ? launch_scores<64, 1, 4, 1, 4>(p, stream) : two ? launch_scores<64, 1, 2, 2, 4>(p, stream) : launch_scores<64, 1, 1, 4, 4>(p, stream));
    }
    const Split split = split_of(p, head_dim, block_m);
    if (block_m == 128) {
        if (split.shares == 2) return d128 ? launch_fwd<128, 4, 1, 1, 2, 2>(p, stream) : launch_fwd<64, 4, 1, 1, 2, 3>(p, stream);
        const bool filling = p.causal && !p.seqlens && !p.k8 && p.seqlen >= 8192 && rows > 110592 && rows <= 131072;
        if (d128 && two && (filling || p.seqlen > (p.k8 ? 65536 : p.causal ? 24576 : 3072))) return launch_fwd<128, 4, 2, 1, 1, 5>(p, stream);
        if (d128) return launch_fwd<128, 4, 1, 1, 1, 2>(p, stream);
        const bool two_to_a_cu = p.causal && !p.seqlens && p.seqlen > 4096 && rows > 65536 && rows <= 98304;
        return launch_fwd<64, 4, 1, 1, 1, 3>(p, stream, two_to_a_cu ? 16384 : 0);       // (41 KiB and these: a third does not fit)
    }
    if (block_m == 64) {
        if (d128 && split.narrow) return launch_fwd<128, 2, 1, 1, 2, 2>(p, stream);
        if (d128 && split.shares == 2) return launch_fwd<128, 2, 1, 2, 2, 2>(p, stream);
        if (d128 && two) return launch_fwd<128, 2, 2, 1, 1, 2>(p, stream);
        if (d128) return tile_alone(p, 512, 512, p.mkv >= 12 ? 1152 : p.mkv >= 8 ? 1024 : 640) ? launch_fwd<128, 2, 1, 1, 1, 2>(p, stream) : launch_fwd<128, 2, 1, 2, 1, 2>(p, stream);
        if (split.shares > 1) return split.shares == 4 ? launch_fwd<64, 2, 1, 1, 4, 2>(p, stream) : launch_fwd<64, 2, 1, 1, 2, 2>(p, stream);
        if (two) return p.seqlens && rows <= 262144 ? launch_fwd<64, 2, 1, 1, 1, 2>(p, stream) : launch_fwd<64, 2, 2, 1, 1, 4>(p, stream);
        const bool alone = p.seqlens ? p.mq <= 2 || (p.group == 1 ? rows <= 262144 : rows <= 196608 && p.mkv <= 40)
                                     : tile_alone(p, 1024, 768, 0) && (p.mq <= 4 || workgroups_of(p, 64) <= 1024);
        return alone ? launch_fwd<64, 2, 1, 1, 1, 2>(p, stream) : launch_fwd<64, 2, 1, 2, 1, 4>(p, stream);
    }
    if (d128 && split.narrow) return launch_fwd<128, 1, 1, 2, 2, 2>(p, stream);
    if (d128 && split.shares == 2) return launch_fwd<128, 1, 1, 4, 2, 2>(p, stream);
    const bool one_tile = p.mq == 1;                       // (then a workgroup of several tiles would have waves without one)
    if (d128 && two && !four && one_tile) return launch_fwd<128, 1, 2, 1, 1, 2>(p, stream);
    if (d128) return four ? launch_fwd<128, 1, 4, 1, 1, 2>(p, stream) : two ? launch_fwd<128, 1, 2, 2, 1, 2>(p, stream) : launch_fwd<128, 1, 1, 4, 1, 2>(p, stream);
    if (split.shares > 1) return split.shares == 4 ? launch_fwd<64, 1, 1, 2, 4, 2>(p, stream) : launch_fwd<64, 1, 1, 2, 2, 2>(p, stream);
    if (two && one_tile && (!four || workgroups_of(p, 64) <= 1024)) return launch_fwd<64, 1, 2, 1, 1, 2>(p, stream);
    if (two) return four ? launch_fwd<64, 1, 4, 1, 1, 4>(p, stream) : launch_fwd<64, 1, 2, 2, 1, 4>(p, stream);
    if (one_tile) return launch_fwd<64, 1, 1, 1, 1, 2>(p, stream);
    const bool narrow = p.seqlens ? rows <= 81920 || p.mkv <= 6 : tile_alone(p, 1024, 768, 0) && (p.mkv <= 4 || workgroups_of(p, 64) <= 1024);
    return narrow ? launch_fwd<64, 1, 1, 2, 1, 2>(p, stream) : launch_fwd<64, 1, 1, 4, 1, 4>(p, stream);
}

#elif BSFA_PART == 1
BSFA_SHAPES_1(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 2
BSFA_SHAPES_2(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 3
BSFA_SHAPES_3(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 4
BSFA_SHAPES_4(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 5
BSFA_SHAPES_5(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 6
BSFA_SHAPES_6(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 7
BSFA_SHAPES_7(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 8
BSFA_SHAPES_8(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 9
BSFA_SHAPES_9(BSFA_DEFINE_F, BSFA_DEFINE_S)
#elif BSFA_PART == 10
BSFA_SHAPES_10(BSFA_DEFINE_F, BSFA_DEFINE_S)
#endif

}  // namespace bsfa
