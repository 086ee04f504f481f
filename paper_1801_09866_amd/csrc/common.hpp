// Shared device-side definitions of the RNNLM frame scorer (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rnnlm.h"

namespace rn {

typedef unsigned long long u64;   // the integer type HIP 64-bit atomics take

constexpr u64 kPhi = 0x9E3779B97F4A7C15ull;   // SplitMix64 increment (2^64 / golden ratio)
constexpr int kMaxLH = 2048;                       // largest L*H (codes staged in LDS)
constexpr int kMaxCW = kMaxLH / 2;                 // largest code-word count (EXACT: 2 per word)
constexpr int kPlanMaxHist = 2048;                 // frame planner limits (LDS tables)
constexpr int kPlanMaxQuery = 8192;

// Counter slots in the device counter array (int64 each).
enum Ctr {
    C_HC_SIZE = 0, C_SC_SIZE, C_FRAMES, C_QUERIES, C_SCORE_HITS, C_QUERY_DUPS, C_COMPUTED,
    C_HISTS, C_HIST_HITS, C_HIST_DUPS, C_GRU_ROWS, C_HIST_INS, C_HIST_REJ, C_SCORE_INS,
    C_SCORE_REJ, C_FRAME_M, C_STAGED, C_NEAR_CAP, C_DONE, C_ROW_FLAGS, C_FRAME_FLAGS, C_N
};

// QRec flag bits above the 2-bit base status (COMPUTED or Q_DUP)
constexpr int QF_CAND = 16;    // first of its key with a cached history key: may be admitted
constexpr int QF_PROBE = 32;   // the history key was cached before the frame: probe the LM cache

// Frame arguments as the kernels see them.
struct FrameArgs {
    int n_hist, n_query;
    const float *hist_vec;
    const u64 *hist_ptr;   // optional per-history row addresses (replace hist_vec)
    const int32_t *hist_words, *q_hist, *q_tgt;
    float *scores, *hnew;
    uint8_t *q_status, *h_status;
    int32_t *q_rep, *h_rep;
    u64 *h_hash;
};

// smallest fp32 bit pattern >= 10^-j, j = 0..20 (decimal decade boundaries)
struct DecadeTab {
    uint32_t lo[21];
};

// History-cache index record (open addressing, 16 B): slot -1 = empty.
struct HcIdx {
    u64 hash;
    int slot;   // dense entry (codes + h') of this key
    int word;   // GRU input word of the key
};

// LM-query cache entry (open addressing, 32 B, key stored in place): hs -1 = empty.
struct ScEnt {
    int hs;     // history-cache slot of the query's history key
    int w2, w3; // MaxEnt context words of the key (-1 where the orders do not use them)
    int t;      // target word
    float val;  // stored fp32 score
    int pad[3];
};

// What the scorer needs per query beyond its words, written by the frame
// planner (16 B); the words (f_qwords) come from the keys kernel.
struct QRec {
    u64 hptr;   // address of the history's top-layer h'
    int flags;  // bits 0-1 base status (COMPUTED / Q_DUP), QF_CAND, QF_PROBE; bits 6.. staging slot
    int hs;     // history-cache slot after the frame (-1: not cached)
};

// What the frame planner reads per history, written by the keys kernel as
// one 16-byte record.
struct HistRec {
    u64 hash;   // 64-bit key hash
    int slot;   // history-cache slot found before the frame; if none, negative: ~slot is the
                // row's ScaleCode (0 without split operands)
    int w1;     // GRU input word (clamped into [0, V))
};

// What a GRU launch on split operands has to know of its weights (w_flags) and
// rows (C_ROW_FLAGS, gathered by the keys kernel; C_FRAME_FLAGS, set by the
// planner): some have no packed form; some have parts with scales of their own
// (bit F_SCALE0 << layer).
enum GruFlags : unsigned { F_PLAIN = 1, F_SCALE0 = 2 };

// Cache probes read the linear-probe sequence kProbeWin records at a time,
// one record per lane (tables have at least 64 slots).
constexpr int kProbeShift = 4;
constexpr int kProbeWin = 1 << kProbeShift;

// Independent decode sessions per context (one frame each per launch).
constexpr int kMaxSessions = 8;

// Everything a kernel needs to know about one context (passed by value). The
// per-session state (caches, counters, per-frame scratch) of session s lives
// s * sess_stride bytes after session 0's; session_view() shifts the pointers.
struct Dev {
    // configuration
    int V, E, H, L, LH, wdtype, me_log2, me_order, qmode, qdigits, max_hist, max_query, CW;
    int sessions;
    long long sess_stride;
    long long cap_hist, cap_query;
    unsigned long long seed;
    uint32_t hi_mask, si_mask;
    // weights (borrowed) and packed GRU weights [3H][Kx + H] per layer
    const void *Wp[2];
    const float *b_ih[2];
    const void *Wl;    // the layer a GRU launch computes: Wp[layer], b_ih[layer] (set per launch, so
    const float *bl;   // that no argument load waits for the layer index)
    const void *U_out;
    const float *b_out;
    const float *maxent;
    // Split operands (split: fp32 weights, sign or rounded history keys): every
    // GRU operand value, times a power of two, as the sum of two fp16 numbers. Packed weights (Wp), and per layer
    // one packed row [Kx + H] per history of each session (apk, rows of
    // apk_row bytes, session-major; null: none of this applies). w_exp: per layer and unit, the exponents of
    // its weight rows' scales (bytes: reset, update, candidate; x: input part, y:
    // recurrent part), and in x's last byte 1 for a unit with a non-finite weight. w_flags: per layer, GruFlags of its weights.
    // bf16 models pack rows too for launches that compute on them (split is
    // set per launch): bf16 values, 64 per line; each part of a row ends at a pair of
    // lines (apk_h: where its history part begins).
    const void *emb;
    char *apk[2];
    unsigned apk_row[2], apk_h[2];
    int sess0;   // session whose state the pointers below address
    int split;
    uint2 *w_exp[2];
    const uint2 *wel;   // w_exp of the layer a GRU launch computes
    unsigned *w_flags;
    const void *Wih[2], *Whh[2];   // the caller's weights
    const void *Wf[2];             // packed weights in the order the matrix instructions read them
    // history cache: index + dense entries
    HcIdx *hc_idx;
    u64 *hc_codes;    // [cap_hist][CW]
    float *hc_val;    // [cap_hist][LH]
    // LM-query cache, and the scores admitted this frame (entered into the
    // table by the next frame's keys kernel, so probes always see the cache as
    // it was before the frame)
    ScEnt *sc_tab;
    ScEnt *sc_stage;  // [max_query]
    // statistics and sticky error bits
    long long *ctr;
    unsigned *derr;
    // per-frame history scratch
    u64 *f_codes;     // [max_hist][CW]
    HistRec *f_hrec;  // key hash, cache slot before the frame, input word
    int *f_hstat, *f_hslot;
    u64 *f_hptr;      // device address of each history's h' (all layers)
    int *f_roww;      // GRU input word (w-1) of row r
    u64 *f_rowh;      // address of row r's history vector (all layers)
    u64 *f_rowdst;    // where row r writes its h'
    u64 *f_rowi;      // packed operands: row r's history index | its ScaleCode << 32
    float *f_hval;    // [max_hist][LH] h' of rows the cache did not admit
    // bf16 weights: the GEMM's A operand, rounded to bf16 once per frame
    uint16_t *f_hbf;  // [max_hist][LH] each history row (written by the keys kernel)
    u64 *f_rowhb;     // address of row r's bf16 history row
    uint16_t *f_xbf;  // two layers: [max_hist][H] the first layer's h' of row r (its tiles' epilogue)
    // per-frame query scratch
    int4 *f_qkey;     // (history index, w-2, w-3, target) for exact key checks
    int4 *f_qwords;   // (w-1, w-2, w-3, target) of each query, as the scorer reads them
    QRec *f_qrec;
    int *f_qcand;     // admission candidates (used when the cache is nearly full)
    int4 *f_part;     // per scoring block: (computed, duplicates, hits, admitted), folded later
    // normaliser partials [256][n_tiles] of (max, sum exp)
    float2 *ln_part;
};

template <class T>
__host__ __device__ __forceinline__ T *shift_ptr(T *p, long long o) {
    return reinterpret_cast<T *>(reinterpret_cast<uintptr_t>(p) + o);
}

// The context as seen by session s: its own caches, counters and scratch.
// The host applies it to the first frame of a launch, and kernels to later
// frames relative to that one, so a one-frame launch reads every pointer
// straight from its arguments.
__host__ __device__ __forceinline__ Dev session_view(const Dev &d0, int s) {
    Dev d = d0;
    const long long o = (long long)s * d0.sess_stride;
    d.sess0 += s;
    d.hc_idx = shift_ptr(d.hc_idx, o);
    d.hc_codes = shift_ptr(d.hc_codes, o);
    d.hc_val = shift_ptr(d.hc_val, o);
    d.sc_tab = shift_ptr(d.sc_tab, o);
    d.sc_stage = shift_ptr(d.sc_stage, o);
    d.ctr = shift_ptr(d.ctr, o);
    d.derr = shift_ptr(d.derr, o);
    d.f_codes = shift_ptr(d.f_codes, o);
    d.f_hrec = shift_ptr(d.f_hrec, o);
    d.f_hstat = shift_ptr(d.f_hstat, o);
    d.f_hslot = shift_ptr(d.f_hslot, o);
    d.f_hptr = shift_ptr(d.f_hptr, o);
    d.f_roww = shift_ptr(d.f_roww, o);
    d.f_rowh = shift_ptr(d.f_rowh, o);
    d.f_rowdst = shift_ptr(d.f_rowdst, o);
    d.f_rowi = shift_ptr(d.f_rowi, o);
    d.f_hval = shift_ptr(d.f_hval, o);
    d.f_hbf = shift_ptr(d.f_hbf, o);
    d.f_rowhb = shift_ptr(d.f_rowhb, o);
    d.f_xbf = shift_ptr(d.f_xbf, o);
    d.f_qkey = shift_ptr(d.f_qkey, o);
    d.f_qwords = shift_ptr(d.f_qwords, o);
    d.f_qrec = shift_ptr(d.f_qrec, o);
    d.f_qcand = shift_ptr(d.f_qcand, o);
    d.f_part = shift_ptr(d.f_part, o);
    return d;
}

// The frames of one launch (at most one per session), with each kernel's
// block ranges: entry e's blocks of a role start at off[e] (off[n] = total).
template <int N>
struct FrameBlockT {
    FrameArgs f[N];
    int sess[N];          // session of entry e, relative to entry 0's (the launch's Dev)
    int n;                // entries
    int hoff[N + 1];      // keys kernel: history blocks
    int qoff[N + 1];      // keys kernel: query-key blocks
    int soff[N + 1];      // keys kernel: staged-insert blocks
    int npart[N];         // scoring blocks of the session's last frame still to fold
    int boff[N + 1];      // scoring kernel: entry e's blocks (its query blocks, then its
    int qblk[N];          //   qblk[e] = ... history blocks) start at boff[e]
};
using FrameBlock = FrameBlockT<kMaxSessions>;
// What a kernel takes: a launch of one frame passes that frame's arguments
// only, a kilobyte less per launch to write and to read (32 frames of 16
// histories and 64 queries: 628 to 640 us, with all sessions' arguments 660 to 669).
template <bool MULTI>
using LaunchBlock = FrameBlockT<MULTI ? kMaxSessions : 1>;

template <bool MULTI>
inline LaunchBlock<MULTI> launch_block(const FrameBlock &fb) {
    if constexpr (MULTI) {
        return fb;
    } else {
        FrameBlockT<1> o;
        o.f[0] = fb.f[0];
        o.sess[0] = fb.sess[0];
        o.n = 1;
        for (int k = 0; k < 2; ++k) {
            o.hoff[k] = fb.hoff[k];
            o.qoff[k] = fb.qoff[k];
            o.soff[k] = fb.soff[k];
            o.boff[k] = fb.boff[k];
        }
        o.npart[0] = fb.npart[0];
        o.qblk[0] = fb.qblk[0];
        return o;
    }
}

// scoring blocks of each session's last frame whose counts are still to fold
struct FoldParts {
    int npart[kMaxSessions];
};

// entry whose range [off[e], off[e+1]) holds b (off[0] = 0 <= b < off[n])
__device__ __forceinline__ int entry_of(const int *off, int n, int b) {
    int e = 0;
    while (e + 1 < n && b >= off[e + 1]) ++e;
    return e;
}

__device__ __forceinline__ u64 mix64(u64 z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// round-to-nearest-even fp32 -> bf16 (inputs are finite)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// four fp32 as four bf16 (RNE), lowest element in the lowest half-word
__device__ __forceinline__ uint2 pack_bf16x4(float4 a) {
    uint2 r;
    r.x = (uint32_t)f32_to_bf16(a.x) | ((uint32_t)f32_to_bf16(a.y) << 16);
    r.y = (uint32_t)f32_to_bf16(a.z) | ((uint32_t)f32_to_bf16(a.w) << 16);
    return r;
}

// Split operands. A row (the input or the recurrent part of a GRU row's operands,
// or of one gate and unit's weights) whose largest |value| has the
// biased exponent e is scaled by 2^(140 - e), which puts that value into
// [2^13, 2^14), and each scaled value v becomes hi = fp16(v), lo = fp16(v - hi).
// hi + lo is v within 2^-22 of itself, and within 2^-38 of the row's largest
// value where lo is subnormal. Exponents are held in [14, 254], so that the
// scale and its inverse are normal; 255 (a non-finite value) has no packed form.
__device__ __forceinline__ float split_scale(int e) { return __uint_as_float((unsigned)(267 - e) << 23); }
__device__ __forceinline__ int split_unscale(int e) { return e - 140; }   // exponent of the inverse
__device__ __forceinline__ int split_exp(unsigned max_bits) {
    const int e = (int)(max_bits >> 23);
    return e < 14 ? 14 : e;
}

// Exponents of the two parts, from the bits of their largest |value|s. A part
// takes the other's where that is larger by at most 2^8 (its values then
// are within 2^-30 of its largest), or where it is all zeros: equal exponents
// spare the GRU a change of scale between the parts, and the parts of
// ordinary rows and weights are that close.
struct PartExp {
    int x, h;
};
__device__ __forceinline__ PartExp part_exps(unsigned mx, unsigned mh) {
    const int x = split_exp(mx), h = split_exp(mh), e = max(x, h);
    return {mx == 0 || x + 8 >= e ? e : x, mh == 0 || h + 8 >= e ? e : h};
}

// ScaleCode: the exponents of a history's packed rows in 31 bits. The second
// layer's input (the first layer's h') is scaled by its bound, which is at least 1.
constexpr unsigned kNoScale = 0x7FFFFFFFu;   // no packed form
__device__ __forceinline__ unsigned scale_code(PartExp e0, PartExp e1) {
    return (unsigned)e0.x | ((unsigned)e0.h << 8) | ((unsigned)e1.h << 16) | ((unsigned)(e1.x - 127) << 24);
}
__device__ __forceinline__ PartExp scale_of(unsigned code, int layer) {
    if (layer == 0) return {(int)(code & 0xFF), (int)((code >> 8) & 0xFF)};
    return {(int)((code >> 24) & 0x7F) + 127, (int)((code >> 16) & 0xFF)};
}
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void split8(const float (&v)[8], float scale, uint4 &hi, uint4 &lo) {
    half8_t h, l;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float x = v[k] * scale;
        h[k] = (_Float16)x;
        l[k] = (_Float16)(x - (float)h[k]);
    }
    hi = __builtin_bit_cast(uint4, h);
    lo = __builtin_bit_cast(uint4, l);
}

// Lines of a packed row's part of K values, in pairs: 32 split values or 64 bf16 each.
template <bool SP>
__host__ __device__ __forceinline__ int part_lines(int K) {
    return SP ? K / 32 : (K / 64 + 1) / 2 * 2;
}

// A launch of at most this many histories runs a bf16 GRU on packed rows. The
// host knows the histories only, which bound the rows (the uncached ones). The
// packed tiles are faster while their four-way split of K keeps a few tiles
// per CU busy; the other kernel's 64-unit tiles read each operand less often, and
// wide models have more tiles. GRU us on other and packed tiles, one layer, by
// rows. E = 512, H = 1024: 64: 12.7 and 7.9, 512: 20.1 and 16.0, 768: 25.0 and
// 23.3, 1024: 26.9 and 27.0, 2048: 43.1 and 48.2 (two layers, 1024: 55.4 and
// 57.1; E = 64, 1024: 23.4 and 25.4). E = 512, H = 2048: 256: 26.6 and 20.2, 512:
// 34.9 and 34.1, 768: 46.4 and 47.5, 1024: 53.2 and 61.7. At H = 512 they cross at
// 1400 rows, at H = 256 at 2048.
__host__ __forceinline__ int packed_hists(int H) { return H <= 1024 ? 1024 : (1 << 20) / H; }

// A history handle is bad when null or not 16-byte aligned.
__device__ __forceinline__ bool bad_handle(u64 p) { return p == 0 || (p & 15); }

// The row a history handle names; a bad handle is replaced by a row of the
// workspace, so that no access leaves valid memory.
__device__ __forceinline__ const float *handle_row(const Dev &d, u64 p) {
    return bad_handle(p) ? d.f_hval : reinterpret_cast<const float *>(p);
}

// Address of history i's L*H vector: a row of hist_vec, or its handle (a bad
// one is replaced as above and reported through *bad).
__device__ __forceinline__ const float *hist_row(const Dev &d, const FrameArgs &f, int i, bool &bad) {
    if (!f.hist_ptr) return f.hist_vec + (size_t)i * d.LH;
    const u64 p = f.hist_ptr[i];
    bad = bad_handle(p);
    return handle_row(d, p);
}

// Index of the calling wave in its block, as a scalar. The compiler cannot
// prove threadIdx.x >> 6 uniform across a wave; branches on a value it takes
// for divergent become exec-masked regions, and a matrix instruction inside
// such a region still writes its accumulator when no lane is active. Every
// branch around an MFMA must therefore depend on scalars only.
// Load through a pointer known to address global memory. Pointers read from
// memory or chosen by a select are generic to the compiler, which then emits
// flat loads (they also count against the LDS wait counter); this spells out
// the global address space.
template <typename T>
__device__ __forceinline__ T ldg(const void *p) {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8 || sizeof(T) == 4, "16-, 8- or 4-byte loads");
    if constexpr (sizeof(T) == 4) {
        const unsigned v = *reinterpret_cast<const __attribute__((address_space(1))) unsigned *>(reinterpret_cast<uintptr_t>(p));
        return __builtin_bit_cast(T, v);
    } else {
        typedef unsigned int raw __attribute__((ext_vector_type(sizeof(T) / 4)));
        const raw v = *reinterpret_cast<const __attribute__((address_space(1))) raw *>(reinterpret_cast<uintptr_t>(p));
        return __builtin_bit_cast(T, v);
    }
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ u64 wave_sum_u64(u64 v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// 64-bit hash of a query key (for table placement only); `a` identifies the
// history key (its cache slot, or its 64-bit key hash within a frame)
__device__ __forceinline__ u64 query_hash(u64 a, int b, int c, int d) {
    u64 g = mix64(a + kPhi);
    g = mix64(g ^ (u64)(uint32_t)(b + 2));
    g = mix64(g ^ (u64)(uint32_t)(c + 2));
    return mix64(g ^ (u64)(uint32_t)(d + 1));
}

// Counts of the last frame's scoring blocks (per-block records, written
// without atomics), added into a copy of the counters `c` held in LDS. Run by
// one block; every thread must call it.
__device__ __forceinline__ void fold_partials(const Dev &d, int n, long long *c, int *s_red) {
    int a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    for (int b = threadIdx.x; b < n; b += blockDim.x) {
        const int4 p = d.f_part[b];
        a0 += p.x; a1 += p.y; a2 += p.z; a3 += p.w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a0 += __shfl_xor(a0, o, 64);
        a1 += __shfl_xor(a1, o, 64);
        a2 += __shfl_xor(a2, o, 64);
        a3 += __shfl_xor(a3, o, 64);
    }
    if (threadIdx.x < 4) s_red[threadIdx.x] = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&s_red[0], a0);
        atomicAdd(&s_red[1], a1);
        atomicAdd(&s_red[2], a2);
        atomicAdd(&s_red[3], a3);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        c[C_COMPUTED] += s_red[0];
        c[C_QUERY_DUPS] += s_red[1];
        c[C_SCORE_HITS] += s_red[2];
        c[C_SCORE_INS] += s_red[3];
        c[C_SC_SIZE] += s_red[3];
    }
    __syncthreads();
}

// slot of the order-n MaxEnt n-gram (w-1 .. w-(n-1), target) in a 2^log2 table
// order-n MaxEnt feature: the order seeds a fold of the n-1 context words
// (most recent first), then the target; the prefix (everything before the
// target) is shared by all targets after the same context
__device__ __forceinline__ u64 maxent_prefix(int order, int w1, int w2, int w3) {
    u64 g = mix64((u64)order * kPhi);
    g = mix64(g ^ (u64)(w1 + 1));
    if (order >= 3) g = mix64(g ^ (u64)(w2 + 1));
    if (order >= 4) g = mix64(g ^ (u64)(w3 + 1));
    return g;
}

__device__ __forceinline__ uint32_t maxent_slot(int order, int w1, int w2, int w3, int tgt, int log2) {
    const u64 g = mix64(maxent_prefix(order, w1, w2, w3) ^ (u64)(tgt + 1));
    return (uint32_t)(g & ((1ull << log2) - 1));
}

}  // namespace rn
