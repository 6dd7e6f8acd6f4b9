// Internal definitions shared by the library's translation units: workspace
// layouts, launch descriptors and small device helpers.  Nothing here is part
// of the public ABI (include/growpage.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "growpage.h"

namespace gp {

constexpr int kPage = 16;                 // tokens per page
// waves per decode workgroup: one LDS page (keys and values of one head, 4 to
// 16 KiB) per wave, 64 KiB at most
constexpr int decode_waves(int elem, int D) { return elem * D > 256 ? 4 : 8; }
#ifndef GP_DECODE_WORKGROUPS
#define GP_DECODE_WORKGROUPS 768
#endif
constexpr int kDecodeWorkgroups = GP_DECODE_WORKGROUPS;    // decode workgroups of a call, all KV heads, about
#ifndef GP_DECODE_MIN_RUN
#define GP_DECODE_MIN_RUN 2
#endif
constexpr int kDecodeMinRun = GP_DECODE_MIN_RUN;           // pages a decode wave takes at least
constexpr int kDecodeShortRun = 8;        // runs up to this many pages: one round of workgroups only
constexpr int kDecodeOwnRun = 6;          // pages per wave up to which all requests take a workgroup each (see decode_kernel)
constexpr int kDecodeResident = 512;      // decode workgroups that 256 CUs hold at once
#ifndef GP_WIDE_MERGE
#define GP_WIDE_MERGE 64
#endif
constexpr int kWideMerge = GP_WIDE_MERGE; // (KV head, request) pairs below which the merge takes 1024 threads each
constexpr int kPrefixSlotPages = 64;      // pages of one partial slot of a shared prefix, about
constexpr int kMaxPrefixSlotPages = 128;  // and at most (LDS id table)
constexpr int kMaxDecodePages = 8192;     // table width the decode calls accept
constexpr size_t kScratchBytes = size_t(8) << 20;   // static scratch of gp_decode_attention_noalloc
constexpr int kMaxBoundaryPages = 4096;                    // table width the boundary calls accept
constexpr int kMaxBnd = 2048;             // boundary requests one apply, select, decide or compact call takes
constexpr int kStatBlock = 64;            // candidate tokens per softmax-statistics block (one wave)
constexpr int kProbChunk = 1024;          // tokens per weight/score work item
constexpr int kCompactChunk = 256;        // slots per compaction work item
constexpr int kMaxLayers = 64;            // layers one gp_boundary_apply call can take
constexpr size_t kAlign = 256;

__host__ __device__ inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------- layouts --

// One step of the dual-timescale EMA (Sec. 3.2) for one element: the fp64
// value beta * prev + (1 - beta) * x with products and the sum rounded one at
// a time (no fused multiply-add), then rounded once to float32.  Every kernel
// that updates summaries goes through this, so they agree bit for bit.
__device__ inline float ema_step(float prev, float x, double beta, double one_minus_beta) {
#pragma clang fp contract(off)
    const double a = beta * (double)prev;
    const double b = one_minus_beta * (double)x;
    return (float)(a + b);
}

// Short tables: one workgroup per (KV head, request), so that no request spans
// two and the merge launch falls away.  Its time is that of the pages a wave takes
// one after the other, 4 us and 0.8 per page (bf16, d 64) or 1.0 (d 128); equal runs
// and their merge take 10 us or more at any length.  Up to nine pages per wave it is
// always the shorter (4 requests of 366-1100 tokens, 12/12 heads, d 64: 9.7 us a
// call against 12.5; one of 950, 32/8, d 128: 11.5 and 11.8), up to eight where P.V of
// a 4 KB page runs in 4 x 4 products (16 of up to 1100 tokens, 4/4, d 128: 15.2 with
// nine, 13.6 in equal runs).  With enough (KV head, request) pairs for half the chip
// equal runs cost more: up to 16 pages (16 of 633-1900, 12/12, d 64: 15.7 against
// 19.2), 10 of 4 KB or more (16 of 550-1100, 32/8, d 128: 14.5 and 16.7; at eleven 18.1
// and 18.1).  With about two workgroups per CU up to 16 of any size (64 of up to 1900,
// 32/8, d 128: 60.4 and 64.6).  waves: of a workgroup; quad: see Page in gp_decode.hip.
__host__ __device__ inline bool decode_own(int max_pages, int R, int Hkv, int page_bytes, int waves, bool quad) {
    const int per = cdiv(max_pages, waves);
    const int64_t pairs = (int64_t)R * Hkv;
    return per <= (quad && page_bytes > 2048 ? 8 : 9) || (pairs >= 128 && per <= (page_bytes <= 2048 ? 16 : 10)) || (pairs >= 448 && per <= 16);
}
// ... of four waves instead of eight (pages of 2 KB) where as many workgroups are
// there: more of them fit a CU, fewer waves have no page (8/8 heads, d 64, up to 200
// tokens: 256 requests 15.8 us against 20.3, 128 10.3 against 11.2; 16 requests of up
// to 500 tokens the other way round, 9.8 against 8.1).
__host__ __device__ inline bool decode_own_narrow(int R, int Hkv) { return (int64_t)R * Hkv >= 512; }

struct DecodeWs {
    size_t partial, lens, prefix, total;
    size_t plain;                 // bytes a call without a shared prefix touches
    int W, slots, pslots;
};

// What gp_decode_attention_noalloc compares with its scratch, as growpage.h states it:
// one (max, sum, o) partial per 64 pages of table width and one more, and three words
// per request.
__host__ __device__ inline size_t decode_chunked_bytes(int R, int Hq, int D, int max_pages) {
    const int chunks = cdiv(max_pages, cdiv(max_pages, cdiv(max_pages, 64)));
    return align_up((size_t)R * (chunks + 1) * Hq * (D + 2) * sizeof(float)) + align_up((size_t)R * 3 * sizeof(int32_t));
}

// Work split of decode attention (see decode_kernel): W workgroups per KV head
// take equal runs of the batch's pages; partial slot (workgroup + request).
// W: kDecodeWorkgroups over all KV heads, one and a half times what the CUs hold
// at once; fewer if the widest batch of this shape has fewer runs of
// kDecodeMinRun pages.  A workgroup pays 3-4 us for its way to the first page
// (lengths, page id, page), so short batches (runs of kDecodeShortRun pages or
// less) are split over the resident ones only: 40 short requests and a new
// token 44.0 us, 45.2 / 46.9 / 53 with 768 / 1024 / 2048 workgroups.  Long ones
// take about the same time with 512 to 1024 (Qwen3-8B layer of 64 requests 96.6
// / 96.6 / 97.4 us, 99.2 with 2048; 256 requests 482 / 484 / 486, 490), but a
// second round evens out workgroups that started late because another stream
// held their CU: a step with the boundary calls beside decode takes 153 us with
// 512, 144 with 768.  Runs of two pages at least: one request of 6001 tokens
// 13.6 us against 16.2 with one.
__host__ __device__ inline DecodeWs decode_ws(int R, int Hq, int Hkv, int D, int max_pages, int waves) {
    DecodeWs w;
    const size_t unit = (size_t)Hq * (D + 2) * sizeof(float);          // one slot of every KV head
    w.W = cdiv(kDecodeWorkgroups, Hkv);
    const int64_t most = (int64_t)R * max_pages;
    if (most < (int64_t)w.W * waves * kDecodeMinRun) w.W = (int)((most + waves * kDecodeMinRun - 1) / (waves * kDecodeMinRun));
    // a batch that the static scratch takes fits it (fewer workgroups from 673 KV heads of
    // eight query heads on, where one request's partials are two slots of 4 MiB)
    const size_t lens = align_up((size_t)R * 5 * sizeof(int32_t));
    if (decode_chunked_bytes(R, Hq, D, max_pages) <= kScratchBytes) {
        const int64_t fit = (int64_t)((kScratchBytes - lens - kAlign) / unit) - R;
        if (w.W > fit) w.W = (int)fit;
    }
    if (w.W < 1) w.W = 1;
    w.slots = w.W + R;
    // partial slots of a shared prefix per request
    const int chunks = cdiv(max_pages, cdiv(max_pages, cdiv(max_pages, kPrefixSlotPages)));
    w.pslots = chunks > 1 ? chunks - 1 : 1;
    size_t off = 0;
    w.partial = off;    // float: [Hkv][slots][G][D + 2] (o, max, sum)
    off = align_up(off + unit * w.slots);
    w.lens = off;       // int32, each [R]: tokens attended (-1: held), token appended (0/1), first partial
                        // slot, slots the merge folds (0: none), prefix pass read (0/1)
    off += lens;
    w.plain = off;
    w.prefix = off;     // float: [R][Hkv][pslots][G][D + 2], partials of a shared prefix
    off = align_up(off + unit * R * w.pslots);
    w.total = off;
    return w;
}

struct ScoreWs {
    size_t cand, expz, part, weights, total;
    int cmax, nch;
};

// cmax = (max_pages - 1) * page: the most candidates any request can have.
__host__ __device__ inline ScoreWs score_ws(int Rb, int Hq, int Hkv, int max_pages) {
    ScoreWs w;
    const int G = Hq / Hkv;
    w.cmax = max_pages > 1 ? (max_pages - 1) * kPage : 0;
    w.nch = cdiv(w.cmax > 0 ? w.cmax : 1, kStatBlock);
    size_t off = 0;
    w.cand = off;     // [Rb] int32: candidates of the event (0: not a boundary), written by the logits
    off = align_up(off + (size_t)Rb * sizeof(int32_t));
    w.expz = off;     // [Rb][Hkv][2G][cmax] float: exp(z - block max), z the fp64 logit
    off = align_up(off + (size_t)Rb * Hkv * 2 * G * w.cmax * sizeof(float));
    w.part = off;     // [Rb][Hkv][nch][2G][2] double: block max, block sum of exp
    off = align_up(off + (size_t)Rb * Hkv * w.nch * 2 * G * 2 * sizeof(double));
    w.weights = off;  // [Rb][Hkv][2][cmax] float
    off = align_up(off + (size_t)Rb * Hkv * 2 * w.cmax * sizeof(float));
    w.total = off;
    return w;
}

struct ApplyWs {
    size_t req, hdr, nshc, shflag, old_table, released, evict, border, total;
    int ncc, npc;
};

// Per boundary request scratch (int32 fields).
// RQ_SKIP: written by the selection, 1 if it skipped the request as a
// certain grow (its lists and border rows were not made).
enum { RQ_R = 0, RQ_P, RQ_FLAGS, RQ_NSH, RQ_POP, RQ_DEC, RQ_SKIP, RQ_STRIDE = 8 };
// Call header (int32): free count before pops, after pops, released pages.
enum { HDR_FC0 = 0, HDR_FC1, HDR_NREL, HDR_SIZE = 4 };
constexpr int kPageBlock = 1024;  // pages per work item when walking a page-table row
// Eviction lists per (layer, boundary request, KV head): slots [0, 16) for a
// Compress & Hold, [16, 48) for a shrink.  Rows move down by at most 32 slots.
constexpr int kShrinkEvict = 2 * kPage;
constexpr int kEvictSlots = kPage + kShrinkEvict;
constexpr int kBorderRows = kShrinkEvict;
constexpr int kBordersPerGroup = 4;   // chunk boundaries whose border rows one workgroup saves

__host__ __device__ inline ApplyWs apply_ws(int Rb, int Hkv, int D, int elem, int max_pages,
                                            int n_layers) {
    ApplyWs w;
    w.ncc = cdiv(max_pages * kPage, kCompactChunk);
    w.npc = cdiv(max_pages, kPageBlock);
    size_t off = 0;
    w.req = off;        // [Rb][RQ_STRIDE]
    off = align_up(off + (size_t)Rb * RQ_STRIDE * sizeof(int32_t));
    w.hdr = off;        // [HDR_SIZE]
    off = align_up(off + HDR_SIZE * sizeof(int32_t));
    w.nshc = off;       // [Rb][npc] shared pages per block of the table row
    off = align_up(off + (size_t)Rb * w.npc * sizeof(int32_t));
    w.shflag = off;     // [Rb][max_pages] uint8: page shared when the call starts
    off = align_up(off + (size_t)Rb * max_pages);
    w.old_table = off;  // [Rb][max_pages]
    off = align_up(off + (size_t)Rb * max_pages * sizeof(int32_t));
    w.released = off;   // [Rb * max_pages]
    off = align_up(off + (size_t)Rb * max_pages * sizeof(int32_t));
    w.evict = off;      // [L][Rb][Hkv][kEvictSlots]
    off = align_up(off + (size_t)n_layers * Rb * Hkv * kEvictSlots * sizeof(int32_t));
    w.border = off;     // [L][Rb][Hkv][ncc][2][kBorderRows][D] elements
    off = align_up(off + (size_t)n_layers * Rb * Hkv * w.ncc * 2 * kBorderRows * D * elem);
    w.total = off;
    return w;
}

// ------------------------------------------------------------ launch args --

constexpr int kMaxPrefixGroups = 16;      // prefix groups one shared decode call takes
constexpr int kPrefixWaves = 4;           // waves per workgroup of the shared-prefix pass

struct DecodeArgs {
    const void *k, *v;
    bool aligned;                 // k and v are multiples of 16 (float32: others take a slower path)
    const int32_t *page_table, *num_pages, *seq_lens;
    const void *q;
    void *out;
    // summary update folded into the launch (gp_decode_step); qstate == nullptr: none
    const void *q_pre;
    const int32_t *slot_ids;
    const uint8_t *init;
    float *qstate;
    int M;
    double beta_s, beta_l;
    // the step's new token folded into the launch (gp_decode_step with k_new):
    // written at slot m_r of every request with room and attended to; with
    // advance != 0 the merge pass then advances seq_lens and positions
    void *k_w, *v_w;              // the pools, written at the new token's slot
    const void *k_new, *v_new;    // [R][Hkv][D]; nullptr: no token
    int32_t *seq_lens_w, *positions;
    int advance;
    float *partial, *prefix;      // workspace regions (DecodeWs)
    int32_t *lens;
    // shared-prefix decode (gp_decode_attention_shared): requests
    // [g_first, g_first + g_num) share the first g_pages pages of g_first's
    // table; workgroup blocks [g_blk0[g], g_blk0[g + 1]) of the prefix pass
    int ngroups;
    int g_first[kMaxPrefixGroups], g_num[kMaxPrefixGroups], g_pages[kMaxPrefixGroups];
    int g_blk0[kMaxPrefixGroups + 1], g_slots[kMaxPrefixGroups];
    int R, Hkv, max_pages, pool_pages, W, W1, min_run, slots, pslots;   // W1: workgroups per KV head that fit at once
    float qscale;      // scale * log2(e); float32 caches: rounded down, and the rest of it
    float qscale_lo;   // (> 0, so that an infinite score times it keeps its sign)
};

struct SummaryArgs {
    const void *q;
    const int32_t *slot_ids;
    const uint8_t *init;
    float *qstate;
    int R, HqD, M;
    double beta_s, beta_l;
};

struct AppendArgs {
    void *k[kMaxLayers];
    void *v[kMaxLayers];
    int32_t *page_table, *num_pages, *seq_lens, *positions;
    const void *k_new, *v_new, *q_pre;
    const int32_t *slot_ids;
    const uint8_t *init;
    float *qstate;
    int R, Hq, Hkv, M, max_pages, pool_pages, n_layers;
    double beta_s, beta_l;
};

struct ScoreArgs {
    const void *k;
    const int32_t *page_table, *num_pages, *seq_lens;
    const void *q_pre;
    const float *qstate;
    const int32_t *slot_ids, *positions, *bnd;
    int32_t *k_counts;
    float *scores;
    double *part;
    int32_t *cand;    // [Rb] candidates per event, 0 if the entry is not a boundary (logits -> later kernels)
    float *expz;
    float *weights;
    int Rb, Hq, Hkv, M, max_pages, pool_pages, max_cand, cmax, nch, R;
    double scale, theta, p;
    int metric;       // GP_METRIC_*
    int lg_iters;     // statistics blocks per logits workgroup (set at launch)
};

struct ApplyArgs {
    int32_t *page_table, *num_pages, *seq_lens, *refcount, *free_list, *free_count;
    const int32_t *bnd, *k_counts;
    const float *scores;
    int32_t *decisions;
    float *delta;
    long long *counters;
    int32_t *req, *hdr, *nshc, *old_table, *released, *evict;
    uint8_t *shflag;
    unsigned char *border;
    int R, Rb, Hkv, max_pages, pool_pages, max_cand, n_layers, ncc, npc, k_loc, reserve;
    double tau;
    // policy variant (GP_POLICY_*) and its constants
    int policy, fixed_pages, min_cap;
    float compress_prob;
    double shrink_threshold;
    const float *draws;
    int layout;       // GP_LAYOUT_*
    int hold;         // mark compressing requests held (negative seq_len)
    int skip_grows;   // the selection may skip requests whose decision can only be a grow
};

struct LayerPtrs {
    void *k, *v;
};

// ---------------------------------------------------------------- launchers --

hipError_t launch_summaries(gp_dtype_t dt, const SummaryArgs &a, hipStream_t s);
hipError_t launch_append(gp_dtype_t dt, int D, const AppendArgs &a, hipStream_t s);
hipError_t launch_decode(gp_dtype_t dt, int D, int G, const DecodeArgs &a, int stages, hipStream_t s);
hipError_t launch_score(gp_dtype_t dt, int D, int G, const ScoreArgs &a, int stages, hipStream_t s);
// Stages of the boundary apply (selection, decision, compaction).
constexpr int kStageSelect = 1, kStageDecide = 2, kStageCompact = 4;

hipError_t launch_apply(gp_dtype_t dt, int D, const ApplyArgs &a, const LayerPtrs *layers, int stages,
                        hipStream_t s);
hipError_t launch_release(int32_t *seq_lens, int R, hipStream_t s);
hipError_t launch_stream_read(const void *src, size_t bytes, uint32_t *out, hipStream_t s);

// ---------------------------------------------------------- device helpers --

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// float -> bfloat16, round to nearest even; NaN stays NaN.
__device__ inline uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

}  // namespace gp
