// Paged GQA decode attention (Sec. 3.1, attention-output equation), split over
// the resident pages of the whole batch.
//
// Work split.  Per KV head the batch is one flat list of pages: the pages of
// request 0, then of request 1, and so on (U pages, read off the lengths by
// every workgroup itself).  The waves take equal runs of L consecutive pages of
// it, whatever requests they belong to, so all workgroups have the same amount
// of work; the next page's keys and values are on their way across request
// boundaries too.  (Short requests, few enough, take a workgroup each instead: see
// decode_own and the split below.)  A wave that meets the end of a request writes that request's result (or its partial, if the request began
// before the wave's run) and goes on with the next; at the end the workgroup
// merges the runs its waves left open, and requests that span workgroups are
// folded by merge_kernel from one (o, max, sum) partial per workgroup, at slot
// (workgroup + request) of the KV head (the pair only ever grows along the
// list, so slots are distinct).
// Why: with a (KV head, 64-page chunk, request) grid most of the workgroups of
// a batch with mixed lengths were empty (28 k of 35 k at 256 requests, table
// width 1028), a request's chunks set the workgroups' durations, and one
// request gave 48 workgroups to 256 CUs.
//
// A workgroup serves the whole GQA group of its KV head (G query heads), so
// every K/V byte is read from HBM once per step.  The KV head is the fastest
// grid index: the eight heads of a page are read at about the same time.
//
// Bound: HBM.  Algorithmic bytes per resident token and KV head:
// 2 * d * sizeof(elem) (K and V), plus the page-table entries, q and out.  A
// copy of the kernel's loads without arithmetic (equal runs, 4 KiB head slices
// of randomly placed pages) reads 6.5-6.9 TB/s; a plain streaming read 7.04.
#include "gp_internal.h"

namespace gp {

namespace {

template <typename T>
struct Traits;

template <>
struct Traits<uint16_t> {
    __device__ static inline void store(uint16_t *p, float x) { *p = f32_to_bf16(x); }
    __device__ static inline float load(const uint16_t *p) { return bf16_to_f32(*p); }
};

template <>
struct Traits<float> {
    __device__ static inline void store(float *p, float x) { *p = x; }
    __device__ static inline float load(const float *p) { return *p; }
};

constexpr float kNegInf = -__builtin_huge_valf();

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef short bf16x4s_t __attribute__((ext_vector_type(4)));
// 16 and 8 bytes as a caller's buffers may lie: at any multiple of the element
typedef u32x4_t u32x4_e2_t __attribute__((aligned(2)));
typedef u32x4_t u32x4_e4_t __attribute__((aligned(4)));
typedef f32x4_t f32x4_e4_t __attribute__((aligned(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef f32x2_t f32x2_e4_t __attribute__((aligned(4)));
__device__ inline u32x4_t load16(const uint16_t *p) { return *reinterpret_cast<const u32x4_e2_t *>(p); }
__device__ inline u32x4_t load16(const float *p) { return *reinterpret_cast<const u32x4_e4_t *>(p); }
__device__ inline void store16(uint16_t *p, const u32x4_t &x) { *reinterpret_cast<u32x4_e2_t *>(p) = x; }
__device__ inline void store16(float *p, const u32x4_t &x) { *reinterpret_cast<u32x4_e4_t *>(p) = x; }
__device__ inline f32x2_t load8(const float *p) { return *reinterpret_cast<const f32x2_e4_t *>(p); }
__device__ inline void store8(float *p, float x, float y) { *reinterpret_cast<f32x2_e4_t *>(p) = f32x2_t{x, y}; }

// s_waitcnt immediates: vmcnt(0) (vmcnt in bits 3:0 and 15:14, the others at
// their maximum); and the cache-policy operand of a direct-to-LDS load that
// marks it non-temporal: K and V are read exactly once per step, so the caches
// do not keep them at the expense of data that is reused (page tables,
// partials, the workspaces of boundary kernels beside decode); it also raises
// the read rate itself (6.0 against 6.8 TB/s in the copy without arithmetic).
constexpr int kWaitVm0 = 0x0F70;
// all but the newest n (< 64) vector memory operations
constexpr int wait_vm(int n) { return kWaitVm0 | (n & 15) | (n >> 4) << 14; }
constexpr int kCpolNT = 2;
typedef const __attribute__((address_space(1))) void global_cvoid_t;
typedef __attribute__((address_space(3))) void lds_void_t;

// LDS reads of a stage that direct-to-LDS loads fill, with their own wait.  As
// builtins or plain loads the compiler makes every such read wait for all
// direct-to-LDS loads in flight (s_waitcnt vmcnt(0)), also for those of the
// next page, which cost the decode kernels a second memory latency per page;
// here the caller waits for the loads it needs (wait_vm) first.
__device__ inline uint32_t lds_addr(const void *p) {
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const char *)p;
}
__device__ inline void lds_read16(uint32_t a0, uint32_t a1, u32x4_t &x0, u32x4_t &x1) {
    __asm__ volatile(
        "ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(x0), "=&v"(x1) : "v"(a0), "v"(a1) : "memory");
}
__device__ inline void lds_read16(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x4_t &x0, u32x4_t &x1,
                                  u32x4_t &x2, u32x4_t &x3) {
    __asm__ volatile(
        "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
__device__ inline void lds_read8(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2_t &x0, u32x2_t &x1,
                                 u32x2_t &x2, u32x2_t &x3) {
    __asm__ volatile(
        "ds_read_b64 %0, %4\n\tds_read_b64 %1, %5\n\tds_read_b64 %2, %6\n\tds_read_b64 %3, %7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// four transposed 16-bit reads (ds_read_b64_tr_b16)
__device__ inline void lds_read_tr(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2_t &x0, u32x2_t &x1,
                                   u32x2_t &x2, u32x2_t &x3) {
    __asm__ volatile(
        "ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %5\n\tds_read_b64_tr_b16 %2, %6\n\t"
        "ds_read_b64_tr_b16 %3, %7\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}

// ------------------------------------------------------------ lane helpers --
// wave-uniform value, in a scalar register
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// x of lane i's partners in the other three rows of 16 lanes (lanes i ^ 16,
// i ^ 32, i ^ 48) folded in: v_permlane16_swap and v_permlane32_swap exchange
// rows in the vector ALU, where a shuffle would go through LDS.
__device__ inline float cross_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ inline float cross_sum(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// x of the lane N places before, around the row of 16 lanes
template <int N>
__device__ inline float row_ror(float x) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + N, 0xf, 0xf, false));
}

// element i (wave-uniform) of an array that nothing writes during the kernel,
// by a scalar load: it is counted apart from the pages in flight, so waiting for
// it does not drain them
__device__ inline int scalar_load(const int32_t *p, int64_t i) {
    return ((const __attribute__((address_space(4))) int32_t *)p)[i];
}

// inclusive prefix sum over the wave (DPP row shifts and row broadcasts)
__device__ inline int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// ------------------------------------------------------------ request view --
// What the pass covers of one request: its resident tokens m, whether the
// step's new token goes in (room: a token is given and the last page has a
// free slot, Sec. 3.1 paged cache), the tokens attended, the pages before the
// covered range (base) and the pages covered (n).  A held request keeps its
// place in the flat list (m = -seq_len - 1), so that a request's output does not
// depend on which others are held; its pages are passed over.
struct ReqView {
    int m, m_attn, base, n;
    bool held, room;
};

template <bool STEP, bool PREFIX>
__device__ inline ReqView req_view(const DecodeArgs &a, int r, int m_in, int P_in) {
    ReqView v;
    const int P = min(max(P_in, 0), a.max_pages);
    v.held = m_in < 0;
    v.m = min(v.held ? -m_in - 1 : m_in, P * kPage);
    v.room = STEP && !v.held && v.m < P * kPage;
    v.m_attn = v.m + (v.room ? 1 : 0);
    v.base = 0;
    if constexpr (PREFIX) {
        // The shared pages come from the prefix pass if the request is not
        // held, holds the prefix's pages and tokens and more, and has the
        // leader's page ids on all prefix pages.  The split goes by the first
        // and the last of them (a compaction replaces every shared page); the
        // wave that begins the request compares them all, and takes the prefix
        // pages itself if they differ.
        int pp = 0, first = 0;
        for (int g = 0; g < a.ngroups; ++g)
            if (r >= a.g_first[g] && r < a.g_first[g] + a.g_num[g]) {
                pp = a.g_pages[g];
                first = a.g_first[g];
            }
        const int32_t *row = a.page_table + (size_t)r * a.max_pages, *lead = a.page_table + (size_t)first * a.max_pages;
        const int last = max(pp - 1, 0);
        const bool same = (row[0] == lead[0]) & (row[last] == lead[last]);
        if (same && pp > 0 && m_in > pp * kPage && P_in > pp && P_in <= a.max_pages && m_in <= P_in * kPage) v.base = pp;
    }
    v.n = cdiv(v.m_attn, kPage) - v.base;
    return v;
}
template <bool STEP, bool PREFIX>
__device__ inline ReqView req_view(const DecodeArgs &a, int r) {
    return req_view<STEP, PREFIX>(a, r, a.seq_lens[r], a.num_pages[r]);
}

// The page of K or V that one wave has in flight, by element type: how it is
// laid out in LDS, and the two products on it.
//
// Both products run on the matrix cores, with the scores computed transposed:
// S^T = K.Q^T (16 tokens x 16 columns, the G query heads and 16 - G zero
// ones) leaves tokens 4 kg + e of head n in lane (n, kg) = (lane % 16, lane /
// 16), which is the layout P^T needs as the B operand of O^T += V^T.P^T; every
// lane then owns output dims of one head, so the softmax rescale needs no lane
// exchange, and the cost does not depend on G.
//
// QUAD (few query heads per KV head): P.V on v_mfma_f32_4x4x1f32, sixteen
// outer products of four dims and four heads each, in float32 throughout.  The
// columns of S^T repeat the heads (column n is head n % 4), so that every quad
// of lanes has P of its row's tokens as the B operand in place; lane (n, kg)
// brings dims 4 n .. + 3 of token 4 kg + e, and the four rows of lanes are
// added up at the end of a request (gather).
//
// What a lane holds of a request: the head `head(n)`, its first GROUPS groups
// of four consecutive dims, group j from `group_dim(j, n, kg)`.
template <typename T, int D, bool QUAD>
struct Page;

// O^T of the QUAD products: acc[4 g + c][i] of lane (n, kg) is dim 64 g + 4 (n
// / 4 * 4 + i) + c of head n % 4, summed over the tokens of row kg.  The sums
// over the rows, with the four dims 4 c' .. + 3 of each left in one row:
// v_permlane32_swap and v_permlane16_swap put the halves (rows) of two values
// side by side, so that each addition sums one value in one half and the other
// in the other.
__device__ inline float pair32(float x, float y) {    // rows 0, 1: x, rows 2, 3: y, each of both halves
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float pair16(float x, float y) {    // rows 0, 2: x, rows 1, 3: y, each of both rows of a half
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int D>
struct QuadOut {
    static constexpr int ACC = D / 16, GROUPS = D / 64;
    __device__ static inline int head(int n) { return n & 3; }
    __device__ static inline int group_dim(int j, int n, int kg) { return 64 * j + 4 * (n / 4 * 4 + kg); }
    __device__ static inline void gather(const f32x4_t (&acc)[ACC], f32x4_t (&o)[GROUPS]) {
#pragma unroll
        for (int j = 0; j < GROUPS; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4_t &x = acc[4 * j + c];
                o[j][c] = pair16(pair32(x[0], x[2]), pair32(x[1], x[3]));
            }
    }
};

// bfloat16: S^T on v_mfma_f32_16x16x32_bf16; P split into two bfloat16 terms
// (hi + lo carry its float32 value to about 2^-17) and O^T on
// v_mfma_f32_16x16x16bf16_1k with V^T by transposed LDS reads
// (ds_read_b64_tr_b16).  Keys are XOR-swizzled on the way in: unit u (16
// bytes) of row R sits at R UPR + (u ^ R % UPR), so that the 16 rows of a
// score-layout read fall on distinct banks; values at u ^ 2 (R % (UPR / 2)),
// so that the transposed reads of 4 rows x 2 units do.
template <int D, bool QUAD>
struct PageBf16 {
    static constexpr int UPR = D / 8;                 // 16-byte units per row
    static constexpr int BYTES = kPage * D * 2;       // keys or values of one page and head
    static constexpr int LOADS = BYTES / 1024;        // load instructions (64 lanes x 16 bytes) per page
    static constexpr int WAVES = decode_waves(2, D);  // per workgroup: 64 KiB of pages at most
    static constexpr int RPI = 64 / UPR;              // rows per load instruction
    static constexpr int KK = D / 32;                 // product steps over the head dims

    // byte offset of this lane's unit in load instruction q of keys or values,
    // less 1024 q (the instruction's immediate): row R = q RPI + lane / UPR, unit
    // (lane % UPR) swizzled by R, which splits into a part of the lane and one of
    // q (their bits are disjoint)
    __device__ static inline uint32_t koff(int lane) {
        return (uint32_t)(lane / UPR * UPR + ((lane % UPR) ^ (lane / UPR))) * 16;
    }
    static constexpr uint32_t kflip(int q) { return q * RPI % UPR * 16; }
    // values: as the transposed reads want them (see above); QUAD: rows R and R +
    // 4, which one read takes together, on different halves of the banks
    __device__ static inline uint32_t voff(int lane) {
        const int R = lane / UPR, u = lane % UPR;
        if constexpr (QUAD) return (uint32_t)(D == 64 ? (R ^ (R / 4 & 1)) * UPR + u : R * UPR + u) * 16;
        return (uint32_t)(R * UPR + (u ^ (2 * (R % (UPR / 2))))) * 16;
    }
    static constexpr uint32_t vflip(int q) {
        return QUAD ? (D == 64 ? 0 : (q & 1) * 128) : 2 * (q * RPI % (UPR / 2)) * 16;
    }
    // LDS offset of this lane's key reads, to be xored with 64 kk (operand kk)
    __device__ static inline uint32_t kread(int n, int kg) { return (n * UPR + (kg ^ (n % UPR))) * 16; }
    // Q of the lane's head as the B operand: unit kk of lane (n, kg) is head dims 32 kk + 8 kg .. + 7
    static constexpr int QREGS = KK;
    __device__ static inline int qdim(int j, int n, int kg) { return 32 * j + 8 * kg; }
    __device__ static inline f32x4_t scores(uint32_t ka, const u32x4_t (&q)[QREGS]) {
        u32x4_t kx[KK];
        if constexpr (KK == 4) lds_read16(ka, ka ^ 64, ka ^ 128, ka ^ 192, kx[0], kx[1], kx[2], kx[3]);
        else lds_read16(ka, ka ^ 64, kx[0], kx[1]);
        f32x4_t st = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kx[kk]),
                                                         __builtin_bit_cast(bf16x8_t, q[kk]), st, 0, 0, 0);
        }
        return st;
    }
};

template <int D>
struct Page<uint16_t, D, false> : PageBf16<D, false> {
    using B = PageBf16<D, false>;
    static constexpr int UPR = B::UPR, DT = D / 16, ACC = DT;     // O^T tiles of 16 dims
    // LDS offset of this lane's transposed reads, to be xored with 32 t (tile t)
    __device__ static inline uint32_t vread(int n, int kg) {
        // V^T tile t as the A operand by transposed reads: lane j of group kg
        // names row R = 4 kg + j / 4, dims 16 t + 4 (j % 4); lane n receives
        // tokens 4 kg .. + 3 at dim 16 t + n
        const int R = 4 * kg + n / 4, qd = n % 4;
        return (R * UPR + ((qd / 2) ^ (2 * (R % (UPR / 2))))) * 16 + (qd & 1) * 8;
    }
    // O^T += V^T.P^T; ntok: tokens of the page (slots past the last may hold
    // anything: 0 x inf would reach o, so they read as zero)
    static constexpr int VREGS = DT;
    typedef u32x2_t v_t;
    __device__ static inline void read_values(uint32_t va, int, v_t (&vx)[VREGS]) {
#pragma unroll
        for (int t = 0; t < DT; t += 4)
            lds_read_tr(va ^ 32 * t, va ^ 32 * (t + 1), va ^ 32 * (t + 2), va ^ 32 * (t + 3), vx[t], vx[t + 1], vx[t + 2], vx[t + 3]);
    }
    __device__ static inline void weigh(uint32_t va, v_t (&vx)[VREGS], bool read, const float (&p)[4], int ntok,
                                        f32x4_t (&ot)[DT], int kg) {
        bf16x4s_t phi, plo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const __bf16 hb = (__bf16)p[e];               // round to nearest even
            phi[e] = __builtin_bit_cast(short, hb);
            plo[e] = __builtin_bit_cast(short, (__bf16)(p[e] - (float)hb));   // p - hi is exact in float32
        }
#pragma unroll
        for (int t0 = 0; t0 < DT; t0 += 4) {
            if (!read) {
                u32x2_t *x = vx + t0;
                lds_read_tr(va ^ 32 * t0, va ^ 32 * (t0 + 1), va ^ 32 * (t0 + 2), va ^ 32 * (t0 + 3), x[0], x[1], x[2], x[3]);
            }
#pragma unroll
            for (int t = t0; t < t0 + 4; ++t) {
                bf16x4s_t vt = __builtin_bit_cast(bf16x4s_t, vx[t]);
                if (ntok < kPage) {                       // wave-uniform
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (4 * kg + e >= ntok) vt[e] = 0;
                }
                ot[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, phi, ot[t], 0, 0, 0);
                ot[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, plo, ot[t], 0, 0, 0);
            }
        }
    }
    static constexpr int GROUPS = DT;
    __device__ static inline int head(int n) { return n; }
    __device__ static inline int group_dim(int j, int n, int kg) { return 16 * j + 4 * kg; }
    __device__ static inline void gather(const f32x4_t (&ot)[ACC], f32x4_t (&o)[GROUPS]) {
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) o[j] = ot[j];
    }
};

// The weights stay float32 and the values are widened (exactly), so a product
// is as exact as a float32 multiply-add, and an infinite value weighs as one
// (a second bfloat16 term of P may be negative).  16 (d = 64) or 32 products
// of 8 cycles per page: 9 % of the cycles that a page's transfer gives a SIMD.
template <int D>
struct Page<uint16_t, D, true> : PageBf16<D, true>, QuadOut<D> {
    using B = PageBf16<D, true>;
    static constexpr int UPR = B::UPR, ACC = QuadOut<D>::ACC, NU = D / 64;
    // LDS offset of this lane's reads: dims 4 n .. + 3 of token 4 kg + e of 64-dim
    // group g at + e UPR 16, xored by e's and g's parts
    __device__ static inline uint32_t vread(int n, int kg) {
        if constexpr (D == 64) return (4 * kg * UPR) * 16 + 8 * n;
        return (4 * kg * UPR) * 16 + (8 * n ^ (kg & 1) * 128);
    }
    __device__ static inline uint32_t vtoken(uint32_t va, int e, int kg) {
        return D == 64 ? va + (e ^ (kg & 1)) * UPR * 16 : va + e * UPR * 16;
    }
    static constexpr int VREGS = 4 * NU;
    typedef u32x2_t v_t;
    __device__ static inline void read_group(uint32_t va, int kg, int j, v_t *x) {
        lds_read8(vtoken(va, 0, kg) ^ j * 128, vtoken(va, 1, kg) ^ j * 128, vtoken(va, 2, kg) ^ j * 128,
                  vtoken(va, 3, kg) ^ j * 128, x[0], x[1], x[2], x[3]);
    }
    __device__ static inline void read_values(uint32_t va, int kg, v_t (&vx)[VREGS]) {
#pragma unroll
        for (int j = 0; j < NU; ++j) read_group(va, kg, j, vx + 4 * j);
    }
    __device__ static inline void weigh(uint32_t va, v_t (&vx)[VREGS], bool read, const float (&p)[4], int ntok,
                                        f32x4_t (&acc)[ACC], int kg) {
#pragma unroll
        for (int j = 0; j < NU; ++j) {
            if (!read) read_group(va, kg, j, vx + 4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u32x2_t v = vx[4 * j + e];
                if (ntok < kPage && 4 * kg + e >= ntok) v = u32x2_t{0u, 0u};
                f32x4_t *o = acc + 4 * j;
                o[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_lo(v[0]), p[e], o[0], 0, 0, 0);
                o[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_hi(v[0]), p[e], o[1], 0, 0, 0);
                o[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_lo(v[1]), p[e], o[2], 0, 0, 0);
                o[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_hi(v[1]), p[e], o[3], 0, 0, 0);
            }
        }
    }
};

// float32, eight query heads per KV head: both products on
// v_mfma_f32_16x16x4f32 (float32 products and sums).  The contraction takes the
// head dims of a 16-byte key unit one by one, unit 4 j + kg in lane group kg; P.V
// takes tokens 4 kg + e in step e, so P is in place, and the value units of a row
// as they lie: row n of O^T tile 4 j + c is dim 64 j + 4 n + c.  Keys are
// swizzled (u ^ R % 16); a value read is one 256-byte run per row.  Every product
// sums four terms on its own and the sums are added as a tree: chained, a score
// of d = 128 lost a quarter of a digit more (error against 64 bits 1.4 times as
// large at one page).
template <int D>
struct Page<float, D, false> {
    static constexpr int UPR = D / 4;
    static constexpr int BYTES = kPage * D * 4;
    static constexpr int LOADS = BYTES / 1024;
    static constexpr int WAVES = decode_waves(4, D);
    static constexpr int RPI = 64 / UPR;
    static constexpr int NJ = D / 16;                 // key units per lane
    static constexpr int DT = D / 16, ACC = DT;

    __device__ static inline uint32_t koff(int lane) {
        return (uint32_t)(lane / UPR * UPR + ((lane % UPR) ^ (lane / UPR))) * 16;
    }
    static constexpr uint32_t kflip(int q) { return q * RPI * 16; }
    __device__ static inline uint32_t voff(int lane) { return lane * 16; }
    static constexpr uint32_t vflip(int) { return 0; }
    // key operand j: xor 64 j; values of token 4 kg + e, unit n + 16 j: plus (e UPR + 16 j) 16
    __device__ static inline uint32_t kread(int n, int kg) { return (n * UPR + (kg ^ n)) * 16; }
    __device__ static inline uint32_t vread(int n, int kg) { return (4 * kg * UPR + n) * 16; }
    static constexpr int QREGS = NJ;
    __device__ static inline int qdim(int j, int n, int kg) { return 16 * j + 4 * kg; }
    __device__ static inline f32x4_t mfma4(uint32_t x, uint32_t y) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x), __uint_as_float(y), f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
    }
    __device__ static inline f32x4_t scores(uint32_t ka, const u32x4_t (&q)[QREGS]) {
        f32x4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j0 = 0; j0 < NJ; j0 += 4) {
            u32x4_t kx[4];
            lds_read16(ka ^ 64 * j0, ka ^ 64 * (j0 + 1), ka ^ 64 * (j0 + 2), ka ^ 64 * (j0 + 3), kx[0], kx[1], kx[2], kx[3]);
            f32x4_t st[16];                           // sums of four dims, added as a tree
#pragma unroll
            for (int i = 0; i < 16; ++i) st[i] = mfma4(kx[i / 4][i % 4], q[j0 + i / 4][i % 4]);
#pragma unroll
            for (int n = 8; n > 0; n /= 2)
#pragma unroll
                for (int c = 0; c < n; ++c) st[c] += st[c + n];
            sum = j0 == 0 ? st[0] : sum + st[0];
        }
        return sum;
    }
    static constexpr int VREGS = 1;
    typedef u32x2_t v_t;
    __device__ static inline void read_values(uint32_t, int, v_t (&)[VREGS]) {}
    __device__ static inline void weigh(uint32_t va, v_t (&)[VREGS], bool, const float (&p)[4], int ntok, f32x4_t (&ot)[DT],
                                        int kg) {
        f32x4_t pv[DT];                               // the page's own sum, then added to the run's
#pragma unroll
        for (int e0 = 0; e0 < 4; e0 += 8 / (D / 32)) {    // four reads at a time
            constexpr int NE = 8 / (D / 32), NU = D / 64; // tokens and units per token of one batch
            u32x4_t vx[4];
            auto at = [&](int k) { return va + ((e0 + k / NU) * UPR + 16 * (k % NU)) * 16; };
            lds_read16(at(0), at(1), at(2), at(3), vx[0], vx[1], vx[2], vx[3]);
#pragma unroll
            for (int j = 0; j < NU; ++j) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    f32x4_t x[NE];
#pragma unroll
                    for (int i = 0; i < NE; ++i)
                        x[i] = mfma4(4 * kg + e0 + i < ntok ? vx[i * NU + j][c] : 0u, __float_as_uint(p[e0 + i]));
#pragma unroll
                    for (int n = NE / 2; n > 0; n /= 2)
#pragma unroll
                        for (int i = 0; i < n; ++i) x[i] += x[i + n];
                    pv[4 * j + c] = e0 == 0 ? x[0] : pv[4 * j + c] + x[0];
                }
            }
            static_assert(NE * NU == 4, "four reads per batch");
        }
#pragma unroll
        for (int t = 0; t < DT; ++t) ot[t] += pv[t];
    }
    static constexpr int GROUPS = DT;
    __device__ static inline int head(int n) { return n; }
    __device__ static inline int group_dim(int j, int n, int kg) { return 64 * (j / 4) + 16 * kg + 4 * (j % 4); }
    __device__ static inline void gather(const f32x4_t (&ot)[ACC], f32x4_t (&o)[GROUPS]) {
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) {
            const int t = 4 * (j / 4), e = j % 4;
            o[j] = f32x4_t{ot[t][e], ot[t + 1][e], ot[t + 2][e], ot[t + 3][e]};
        }
    }
};

// float32, up to four query heads: both products on v_mfma_f32_4x4x1f32, which
// a page costs a quarter of the cycles of the sixteen columns above (512 at d =
// 128).  Scores: block (n / 4, kg) of lanes multiplies tokens 4 kg .. + 3 with
// the four heads over the 16-byte key units n / 4 + 4 j, and the four blocks of
// a row are added with row rotations, so that the scores of row kg's tokens end
// in every quad of the row.  Keys are swizzled by u ^ 4 (R % 4): the sixteen
// units that a row of lanes reads at once lie on distinct banks.
template <int D>
struct Page<float, D, true> : QuadOut<D> {
    static constexpr int UPR = D / 4;
    static constexpr int BYTES = kPage * D * 4;
    static constexpr int LOADS = BYTES / 1024;
    static constexpr int RPI = 64 / UPR;
    static constexpr int NJ = D / 16, NU = D / 64;
    static constexpr int ACC = QuadOut<D>::ACC;

    __device__ static inline uint32_t koff(int lane) {
        const int R = lane / UPR;                     // (% 4, of the first instruction's rows)
        return (uint32_t)(R * UPR + ((lane % UPR) ^ 4 * R)) * 16;
    }
    static constexpr uint32_t kflip(int q) { return q * RPI % 4 * 64; }
    __device__ static inline uint32_t voff(int lane) { return lane * 16; }
    static constexpr uint32_t vflip(int) { return 0; }
    // key operand j: xor 64 j; values of token 4 kg + e, unit n + 16 j: plus (e UPR + 16 j) 16
    __device__ static inline uint32_t kread(int n, int kg) {
        return ((4 * kg + n % 4) * UPR + n / 4 + 4 * (n % 4)) * 16;
    }
    __device__ static inline uint32_t vread(int n, int kg) { return (4 * kg * UPR + n) * 16; }
    static constexpr int QREGS = NJ;
    __device__ static inline int qdim(int j, int n, int kg) { return 16 * j + 4 * (n / 4); }
    __device__ static inline f32x4_t scores(uint32_t ka, const u32x4_t (&q)[QREGS]) {
        f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j0 = 0; j0 < NJ; j0 += 4) {
            u32x4_t kx[4];
            lds_read16(ka ^ 64 * j0, ka ^ 64 * (j0 + 1), ka ^ 64 * (j0 + 2), ka ^ 64 * (j0 + 3), kx[0], kx[1], kx[2], kx[3]);
            f32x4_t st[4];                            // by the place in the unit (short sums, added as a tree)
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    st[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(kx[k][e]), __uint_as_float(q[j0 + k][e]),
                                                               k == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : st[e], 0, 0, 0);
            st[0] = (st[0] + st[1]) + (st[2] + st[3]);
            x = j0 == 0 ? st[0] : x + st[0];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] += row_ror<8>(x[e]);
            x[e] += row_ror<4>(x[e]);
        }
        return x;
    }
    static constexpr int VREGS = 1;
    typedef u32x2_t v_t;
    __device__ static inline void read_values(uint32_t, int, v_t (&)[VREGS]) {}
    __device__ static inline void weigh(uint32_t va, v_t (&)[VREGS], bool, const float (&p)[4], int ntok, f32x4_t (&acc)[ACC],
                                        int kg) {
        constexpr int NE = 4 / NU;                    // tokens per four reads
#pragma unroll
        for (int e0 = 0; e0 < 4; e0 += NE) {
            u32x4_t vx[4];
            auto at = [&](int k) { return va + ((e0 + k / NU) * UPR + 16 * (k % NU)) * 16; };
            lds_read16(at(0), at(1), at(2), at(3), vx[0], vx[1], vx[2], vx[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = e0 + k / NU, j = k % NU;
                const bool in = 4 * kg + e < ntok;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[4 * j + c] = __builtin_amdgcn_mfma_f32_4x4x1f32(in ? __uint_as_float(vx[k][c]) : 0.0f, p[e],
                                                                        acc[4 * j + c], 0, 0, 0);
            }
        }
    }
};

template <typename T, int D>
constexpr int waves_of() { return decode_waves(sizeof(T), D); }
template <typename T, int D>
constexpr int page_bytes_of() { return kPage * D * (int)sizeof(T); }
// The query heads per KV head of which P.V runs in QUAD products.  bfloat16, more
// heads: the two-term P of four or eight heads costs the matrix cores less.  float32:
// as far as one product's columns go.
template <typename T>
constexpr bool quad_heads(int G) { return sizeof(T) == 2 ? G <= 2 : G <= 4; }

// Calls whose values go to registers as soon as they are there (8 or 16 of them), so
// that the next page is requested whole before this one's weights are formed: a
// wave's pages follow each other 0.8 us apart instead of 0.95 (d = 64).  Not in the
// equal runs of d = 128, which it would take past the 96 registers that leave other
// kernels' waves room beside two workgroups (107 with one query head, for 1 %).
template <typename T>
constexpr bool early_values(int D, int OWN) { return sizeof(T) == 2 && (D == 64 || OWN > 0); }

// One page slice into LDS: instruction q takes at(q) (less 1024 (q % 4)) to
// stage + 1024 q (the immediate offset moves source and destination).
// Direct-to-LDS loads of 16 bytes want addresses that are multiples of 16; float32
// pools that lie at another multiple of 4 go through registers.
template <int LOADS, bool ANY, typename At>
__device__ inline void load_page(At at, char *stage, bool aligned, int lane) {
    if constexpr (ANY) {
        if (!aligned) {                               // (uniform over the grid)
#pragma unroll
            for (int q = 0; q < LOADS; ++q)
                *reinterpret_cast<u32x4_t *>(stage + q * 1024 + lane * 16) =
                    load16(reinterpret_cast<const float *>(at(q) + q % 4 * 1024));
            return;
        }
    }
#pragma unroll
    for (int q = 0; q < LOADS; q += 4) {
        lds_void_t *const to = (lds_void_t *)(stage + q * 1024);
        __builtin_amdgcn_global_load_lds((global_cvoid_t *)at(q), to, 16, 0, kCpolNT);
        __builtin_amdgcn_global_load_lds((global_cvoid_t *)at(q + 1), to, 16, 1024, kCpolNT);
        if constexpr (LOADS > 2) {
            __builtin_amdgcn_global_load_lds((global_cvoid_t *)at(q + 2), to, 16, 2048, kCpolNT);
            __builtin_amdgcn_global_load_lds((global_cvoid_t *)at(q + 3), to, 16, 3072, kCpolNT);
        }
    }
}

// One output: a sum of weights that is not positive (no tokens, scores of -inf or
// NaN) gives zero, in whichever pass the output is written.
__device__ inline float divided(float o, float l) { return l > 0.0f ? o / l : 0.0f; }
// four consecutive outputs
__device__ inline void store_out(uint16_t *p, const f32x4_t &o, float l) {
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    typedef bf16x4_t bf16x4_e2_t __attribute__((aligned(2)));
    bf16x4_t x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = (__bf16)divided(o[e], l);
    *reinterpret_cast<bf16x4_e2_t *>(p) = x;
}
__device__ inline void store_out(float *p, const f32x4_t &o, float l) {
    *reinterpret_cast<f32x4_e4_t *>(p) = f32x4_t{divided(o[0], l), divided(o[1], l), divided(o[2], l), divided(o[3], l)};
}

// Waves per SIMD that the registers are to leave room for.  Workgroups of one
// request at 2 KB pages: 6 and 5 (80 and 96 registers); held to 64 registers they
// spilled up to 9 of them, 5-20 % of a step with a token, and nothing was gained by
// the room (256 requests of 64-200 tokens, 8/4 heads: 9.0 us a call at 5, 6 or 7).
template <typename T, int D, int OWN>
constexpr int decode_occupancy() {
    if (waves_of<T, D>() < 8) return 2;
    if (OWN == 0) return 4;
    return OWN < waves_of<T, D>() ? 6 : sizeof(T) == 2 ? 5 : 4;
}

// MODE 0: decode attention; 1: gp_decode_step with the step's new token (the
// summary update is in the merge pass); 2: the private tails of
// gp_decode_attention_shared.
//
// Per wave one LDS page of keys and one of values, filled by direct-to-LDS
// loads, each instruction one contiguous 1 KiB of the head's slice; the keys
// are refilled as soon as the scores are formed, the values once P.V has read
// them (or the registers have: early_values), and each wait is for exactly the loads it needs.  Sixteen waves per CU
// (bf16, d = 128) keep the memory busy while some of them compute: the copy of
// the loads reads 6.7-6.8 TB/s whether or not a wave pauses for 1000 cycles
// between a page's arrival and its refill; eight waves with two pages each read
// 6.9 TB/s without the pause and 6.2-6.4 with it.
// OWN > 0: short tables, workgroup r of OWN waves takes request r (see decode_own).
template <typename T, int D, int G, int MODE, int OWN>
__global__ __launch_bounds__((64 * (OWN ? OWN : waves_of<T, D>())))
    __attribute__((amdgpu_waves_per_eu(decode_occupancy<T, D, OWN>()))) void
decode_kernel(DecodeArgs a) {
    static_assert(!OWN || MODE != 2, "a shared-prefix call is always merged");
    constexpr bool STEP = MODE == 1, PREFIX = MODE == 2;
    using Pg = Page<T, D, quad_heads<T>(G)>;
    constexpr int NW = OWN ? OWN : waves_of<T, D>();
    constexpr int NT = 64 * NW;
    constexpr int LOADS = Pg::LOADS, ACC = Pg::ACC;
    constexpr bool EARLY = early_values<T>(D, OWN);
    // per wave its pages (keys, values); when they are read, the wave's o goes
    // where the first keys were
    constexpr int STAGE = 2 * Pg::BYTES;
    static_assert(G * D * 4 <= STAGE, "merge buffer");
    __shared__ __attribute__((aligned(1024))) char s_wave[NW][STAGE];
    __shared__ float s_ml[NW][G][2];                  // (max, sum) of each wave's open part
    __shared__ int s_open[NW][3];                     // its request; flags first page 1, last page 2, tail 4; request written

    const int h = blockIdx.x, wg = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int hn = Pg::head(n);                       // the lane's query head of the group
    const int Hkv = a.Hkv, Hq = Hkv * G, R = a.R;

    // this wave's run [f0, f1) of the flat list; the request at f0, its first page's
    // place in the list, and its length
    int f0, f1, r = -1, a0 = 0, m_in = 0, P_in = 0;
    int parts = 0;                                    // OWN: waves that have a part of the request
    if constexpr (OWN > 0) {
        r = wg;
        m_in = scalar_load(a.seq_lens, r);
        P_in = scalar_load(a.num_pages, r);
        const ReqView v = req_view<STEP, PREFIX>(a, r, m_in, P_in);
        const int run = cdiv(v.n, NW);
        f0 = min(wave * run, v.n);
        f1 = v.held ? f0 : min(f0 + run, v.n);
        parts = v.held || v.n == 0 ? 0 : cdiv(v.n, run);
        if (h == 0 && tid == 0) {                     // for the merge pass (see below): nothing to fold
            a.lens[r] = v.held ? -1 : v.m_attn;
            a.lens[R + r] = v.room ? 1 : 0;
            a.lens[2 * R + r] = a.lens[3 * R + r] = a.lens[4 * R + r] = 0;
        }
        if (v.n == 0 && !v.held) {                    // no tokens
            T *o = reinterpret_cast<T *>(a.out) + ((size_t)r * Hq + (size_t)h * G) * D;
            for (int i = 4 * tid; i < G * D; i += 4 * NT) store_out(o + i, f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0.0f);
        }
    } else {
        // ---- the split: U pages in all, L per wave; the request at the run's start.
        // Thread t takes request base + t; the prefix sums meet in LDS.  (Rolled up:
        // the code before the first page is fetched cold by every CU.)
        __shared__ int s_sum[NW], s_incl[NT], s_len[NT], s_np[NT];
        int any_long = 0;                                 // (sign) a request of the last block has too many pages for a workgroup
        auto scan_block = [&](int base, int acc) {        // inclusive sums of the block's requests; its end
            const int r = min(base + tid, R - 1), sl = a.seq_lens[r], np = a.num_pages[r];
            const int x = base + tid < R ? req_view<STEP, PREFIX>(a, r, sl, np).n : 0;
            const int incl = wave_scan(x), mark = __ballot(x > kDecodeOwnRun * NW) ? 1 << 31 : 0;
            if (base > 0) __syncthreads();                // (the previous block has been read)
            if (lane == 63) s_sum[wave] = incl | mark;
            __syncthreads();
            int before = acc, all = acc;
            any_long = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int t = s_sum[w] & 0x7fffffff;
                any_long |= s_sum[w];
                if (w < wave) before += t;
                all += t;
            }
            s_incl[tid] = before + incl;
            s_len[tid] = sl;
            s_np[tid] = np;
            __syncthreads();
            return all;
        };
        int U = 0;
        for (int base = 0; base < R; base += NT) U = uni(scan_block(base, U));
        const int L = max(max(a.min_run, cdiv(U, a.W * NW)), min(kDecodeShortRun, cdiv(U, a.W1 * NW)));
        // Short requests in a wide table, few enough for a workgroup each, take one each,
        // as OWN: nothing to merge, and the merge launch finds that at once.  Up to
        // kDecodeOwnRun pages per wave; us a call at 512 table columns, equal runs and so:
        // 4 requests of 100-250 tokens, 12/12 heads, d 64, 12.2 and 8.5; 16 of 60-120 at 8/1,
        // d 128, 17.3 and 9.0; 64 of 100-500 at 32/8, d 128, 22.1 and 18.4; with eight pages per
        // wave 16 of 100-1000 at 8/4, d 64, 11.9 and 13.7.
        const bool own = R <= a.W && R <= NT && uni(any_long) >= 0;
        if (wg == a.W - 1) {                              // (the workgroup with the fewest pages)
            // for the merge pass, per request: tokens attended (-1: held), whether a
            // token went in, and the partial slots it folds (first, count; count 0:
            // this pass writes the output); outputs of requests without tokens
            int acc = 0;
            for (int base = 0; base < R; base += 64) {
                const int r = base + lane;
                const ReqView v = req_view<STEP, PREFIX>(a, min(r, R - 1));
                const int np = r < R ? v.n : 0, incl = wave_scan(np), a0 = acc + incl - np;
                acc += __builtin_amdgcn_readlane(incl, 63);
                if (base / 64 % NW != wave || r >= R) continue;
                if (h == 0) {
                    // (the lengths are read a second time here: should another stream be
                    // writing them, the slots named still lie in the workspace)
                    const int ws = own ? r : min(a0 / L / NW, a.W - 1);
                    const int we = own || np == 0 ? ws : min((a0 + np - 1) / L / NW, a.W - 1);
                    a.lens[r] = v.held ? -1 : v.m_attn;
                    a.lens[R + r] = v.room ? 1 : 0;
                    a.lens[2 * R + r] = ws + r;
                    a.lens[3 * R + r] = np > 0 && (we > ws || v.base > 0) ? we - ws + 1 : 0;
                    if (!(PREFIX && v.base > 0)) a.lens[4 * R + r] = 0;   // (else: the wave that begins the request)
                }
                if (np == 0 && !v.held) {
                    T *o = reinterpret_cast<T *>(a.out) + ((size_t)r * Hq + (size_t)h * G) * D;
                    for (int i = 0; i < G * D; i += 4) store_out(o + i, f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0.0f);
                }
            }
        }
        if (own ? wg >= R : wg * NW * L >= U) return;     // (uniform over the workgroup)

        f0 = min((wg * NW + wave) * L, U);
        f1 = min(f0 + L, U);
        if (own) {
            r = wg;
            m_in = uni(s_len[r]);
            P_in = uni(s_np[r]);
            const int n_ = uni(req_view<STEP, PREFIX>(a, r, m_in, P_in).n), run = cdiv(n_, NW);
            a0 = uni(s_incl[r]) - n_;
            f0 = a0 + min(wave * run, n_);
            f1 = a0 + min((wave + 1) * run, n_);
        }
        for (int base = 0, acc = 0; base < R && !own; base += NT) {
            if (R > NT) {                                 // (one block is still in LDS)
                __syncthreads();
                acc = uni(scan_block(base, acc));
            }
            for (int j = 0; j < NT && r < 0 && f0 < f1; j += 64) {
                const unsigned long long past = __ballot(base + j + lane < R && s_incl[j + lane] > f0);
                if (past) {
                    const int l = j + uni(__builtin_ctzll(past));
                    r = base + l;
                    m_in = uni(s_len[l]);
                    P_in = uni(s_np[l]);
                    a0 = uni(s_incl[l]) - uni(req_view<STEP, PREFIX>(a, r, m_in, P_in).n);
                }
            }
        }
    }

    char *const mine = s_wave[wave];
    const size_t page_bytes = (size_t)Hkv * Pg::BYTES;
    const char *const kpool = reinterpret_cast<const char *>(a.k) + (size_t)h * Pg::BYTES;
    const char *const vpool = reinterpret_cast<const char *>(a.v) + (size_t)h * Pg::BYTES;
    // this lane's offsets in a page slice and in its LDS copy.  (Made opaque on
    // each page: hoisted out of the loop, their variants for every instruction
    // would take two dozen registers and push the kernel past the 96 that leave
    // room for other kernels' waves beside two of its workgroups.)
    uint32_t ko = Pg::koff(lane), vo = Pg::voff(lane);
    uint32_t kr = lds_addr(mine) + Pg::kread(n, kg), vr = lds_addr(mine) + Pg::BYTES + Pg::vread(n, kg);
    auto request_keys = [&](int phys) {
        const char *src = kpool + (size_t)phys * page_bytes;
        __asm__ volatile("" : "+v"(ko));
        load_page<LOADS, sizeof(T) == 4>([&](int q) { return src + (size_t)((ko ^ Pg::kflip(q)) + (q - q % 4) * 1024u); }, mine,
                                        a.aligned, lane);
    };
    auto request_values = [&](int phys) {
        const char *src = vpool + (size_t)phys * page_bytes;
        __asm__ volatile("" : "+v"(vo));
        load_page<LOADS, sizeof(T) == 4>([&](int q) { return src + (size_t)((vo ^ Pg::vflip(q)) + (q - q % 4) * 1024u); },
                                        mine + Pg::BYTES, a.aligned, lane);
    };

    // ---- one request's part of the run: pages [p, pend) of its covered pages
    int p = 0, pend = 0, nseg = 0, base = 0, m_attn = 0;
    bool whole = false;                               // the part begins with the request's first page
    const int32_t *row = nullptr;
    int idn = -1;                                     // page id at the cursor, requested ahead
    auto request_id = [&]() { idn = scalar_load(row, min(max(base + p, 0), a.max_pages - 1)); };
    // enters request r (uniform) at its covered page `from`; the step's new token
    // goes into the cache here, before the page that takes it is requested
    auto enter = [&](const ReqView &v, int from) {
        base = uni(v.base);
        nseg = uni(v.n);
        m_attn = uni(v.m_attn);
        p = from;
        pend = min(nseg, f1 - a0);
        whole = from == 0;
        row = a.page_table + (size_t)r * a.max_pages;
        if constexpr (PREFIX) {
            if (base > 0 && whole) {
                const int32_t *lead = nullptr;
                for (int g = 0; g < a.ngroups; ++g)
                    if (r >= a.g_first[g] && r < a.g_first[g] + a.g_num[g])
                        lead = a.page_table + (size_t)a.g_first[g] * a.max_pages;
                bool ok = true;
                for (int j = lane; j < base; j += 64) ok = ok && row[j] == lead[j];
                const bool match = __all(ok);
                if (h == 0 && lane == 0) a.lens[4 * R + r] = match ? 1 : 0;
                if (!match) p = -base;                // this wave takes the prefix pages too
            }
        }
        if constexpr (STEP) {
            const int pn = uni(v.m) / kPage, slot = uni(v.m) % kPage;
            if (uni(v.room) && pn >= p && pn < pend) {
                constexpr int NU = D * (int)sizeof(T) / 16;          // 16-byte units of one row
                const int id = scalar_load(row, pn);
                if (lane < 2 * NU && id >= 0 && id < a.pool_pages) {
                    const bool isv = lane >= NU;
                    const int u = isv ? lane - NU : lane;
                    constexpr int EPU = 16 / (int)sizeof(T);
                    const u32x4_t x = load16(reinterpret_cast<const T *>(isv ? a.v_new : a.k_new) +
                                             ((size_t)r * Hkv + h) * D + u * EPU);
                    store16(reinterpret_cast<T *>(isv ? a.v_w : a.k_w) +
                                (((size_t)id * Hkv + h) * kPage + slot) * D + u * EPU, x);
                }
                // (rare: once per request and head) the row is in memory before its page is requested
                __builtin_amdgcn_s_waitcnt(kWaitVm0);
            }
        }
    };
    // from page `from` of request r on, the next request that has pages for this
    // wave (false: none before the run's end); known: m_in and P_in are r's
    auto seek = [&](int from, bool known) {
        while (r >= 0 && r < R && a0 < f1) {
            if (!known) {
                m_in = scalar_load(a.seq_lens, r);
                P_in = scalar_load(a.num_pages, r);
            }
            known = false;
            const ReqView v = req_view<STEP, PREFIX>(a, r, m_in, P_in);
            const int n_ = uni(v.n);
            if (!v.held && n_ > from) {
                enter(v, from);
                request_id();
                return true;
            }
            a0 += n_;
            from = 0;
            ++r;
        }
        return false;
    };
    u32x4_t q[Pg::QREGS];                             // Q of the current request
    // (uniform bases and 32-bit lane offsets, here and in finish: 64-bit lane
    // addresses kept across the loop would cost registers)
    const uint32_t q_at = (uint32_t)(min(hn, G - 1) * D + Pg::qdim(0, n, kg));
    auto load_q = [&](int rr) {
        const T *src = reinterpret_cast<const T *>(a.q) + ((size_t)rr * Hq + (size_t)h * G) * D;
#pragma unroll
        for (int j = 0; j < Pg::QREGS; ++j) {
            const u32x4_t x = load16(src + (q_at + (uint32_t)(Pg::qdim(j, 0, 0))));
            q[j] = hn < G ? x : u32x4_t{};
        }
    };

    f32x4_t ot[ACC];
    float mrun, lrun;                                 // the lane's head: running max (log2 units), this lane's share of the sum
    auto clear = [&]() {
        mrun = kNegInf;
        lrun = 0.0f;
#pragma unroll
        for (int t = 0; t < ACC; ++t) ot[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto part_of = [&](int rr) { return a.partial + ((size_t)h * a.slots + wg + rr) * G * (D + 2); };
    // the finished part of request rr: its output if the wave has all of it, else its partial
    auto finish = [&](int rr, bool direct) {
        const float l = cross_sum(lrun);
        f32x4_t og[Pg::GROUPS];
        Pg::gather(ot, og);
        uint32_t nn = hn, dd = Pg::group_dim(0, n, kg);
        __asm__ volatile("" : "+v"(nn), "+v"(dd));
        if (hn < G) {
            if (direct) {
                T *o = reinterpret_cast<T *>(a.out) + ((size_t)rr * Hq + (size_t)h * G) * D;
                const uint32_t at = nn * D + dd;
#pragma unroll
                for (int j = 0; j < Pg::GROUPS; ++j)
                    store_out(o + (at + (uint32_t)Pg::group_dim(j, 0, 0)), og[j], l);
            } else {
                float *pt = part_of(rr);
                const uint32_t at = nn * (D + 2) + dd;
#pragma unroll
                for (int j = 0; j < Pg::GROUPS; ++j) {
                    float *o = pt + (at + (uint32_t)Pg::group_dim(j, 0, 0));
                    store8(o, og[j][0], og[j][1]);
                    store8(o + 2, og[j][2], og[j][3]);
                }
                if (n == hn && kg == 0) store8(pt + (nn * (D + 2) + D), mrun, l);
            }
        }
    };

    // what the wave leaves for the workgroup's merge: the request whose part
    // reaches the end of its run without being a whole request, whether it holds
    // the request's first or last page, and the request whose partial it wrote
    // on the way (at most one: the one its run began in)
    int open_r = -1, wrote_r = -1;
    bool open_first = false, open_last = false, open_tail = false;
    // A page on its way: where it is and whose it is.
    struct Ahead {
        int phys, r, p, base, m_attn;
        bool valid, last, first_of, ends;             // last page of the wave's part; part begins / ends the request
    };
    // the page at the cursor (r, p), then the cursor to the next page
    bool more = false;
    auto take = [&]() {
        Ahead x;
        x.valid = more;
        x.phys = -1;
        x.r = r;
        x.p = p;
        x.base = base;
        x.m_attn = m_attn;
        x.last = p + 1 >= pend;
        x.first_of = whole;
        x.ends = pend == nseg;
        if (more) {
            x.phys = idn >= 0 && idn < a.pool_pages ? idn : -1;
            if (!x.last) {
                ++p;
                request_id();
            } else {
                a0 += nseg;
                ++r;
                more = seek(0, false);
            }
        }
        return x;
    };
    if (f0 < f1) more = seek(f0 - a0, true);
    if (more) {
        load_q(r);
        clear();
        // cur is computed, nxt takes its place in LDS (the first round only requests)
        Ahead cur = {-1, 0, 0, 0, 0, false, false, false, false};
        while (true) {
            const Ahead nxt = take();
            const bool has = cur.phys >= 0, has1 = nxt.phys >= 0;
            const int ntok = min(kPage, cur.m_attn - (cur.base + cur.p) * kPage);
            f32x4_t sx = {0.0f, 0.0f, 0.0f, 0.0f};
            typename Pg::v_t vx[Pg::VREGS];
            if (has) {                                // wave-uniform
                // the keys: requested after them are the page's values
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(wait_vm(LOADS));
                __builtin_amdgcn_sched_barrier(0);
                __asm__ volatile("" : "+v"(kr));
                sx = Pg::scores(kr, q);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (EARLY) {
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);
                    __builtin_amdgcn_sched_barrier(0);
                    __asm__ volatile("" : "+v"(vr));
                    Pg::read_values(vr, kg, vx);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (has1) request_keys(nxt.phys);
            if (EARLY && has1) request_values(nxt.phys);
            if (has) {
                // online softmax of the lane's head over tokens 4 kg + e
                float sc[4], ml = kNegInf;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sc[e] = 4 * kg + e < ntok ? sx[e] * a.qscale : kNegInf;
                    ml = fmaxf(ml, sc[e]);
                }
                const float mn = fmaxf(mrun, cross_max(ml));
                const float top = mn == kNegInf ? 0.0f : mn;
                if (__any(mn != mrun)) {              // skip while no head's max has moved
                    const float alpha = exp2f(mrun - top);
                    lrun *= alpha;
#pragma unroll
                    for (int t = 0; t < ACC; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) ot[t][e] *= alpha;
                    mrun = mn;
                }
                // weights; the instruction by itself flushes those below 2^-126
                float lowest = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // float32: the distance to the maximum rounded once, not the score, the
                    // scale and the distance each (a third of the output's error at d = 64)
                    if constexpr (sizeof(T) == 4)
                        sc[e] = 4 * kg + e < ntok ? fmaf(sx[e], a.qscale_lo, fmaf(sx[e], a.qscale, -top)) : kNegInf;
                    else
                        sc[e] -= top;
                    lowest = fminf(lowest, sc[e]);
                }
                if (ntok < kPage) {                   // (not the slots past the last token)
                    lowest = 0.0f;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (4 * kg + e < ntok) lowest = fminf(lowest, sc[e]);
                }
                if (__any(lowest < -126.0f)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc[e] = exp2f(sc[e]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc[e] = __builtin_amdgcn_exp2f(sc[e]);
                }
                lrun += (sc[0] + sc[1]) + (sc[2] + sc[3]);
                if constexpr (!EARLY) {
                    // the values: requested after them are the next page's keys
                    __builtin_amdgcn_sched_barrier(0);
                    if (has1) __builtin_amdgcn_s_waitcnt(wait_vm(LOADS));
                    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
                    __builtin_amdgcn_sched_barrier(0);
                    __asm__ volatile("" : "+v"(vr));
                }
                Pg::weigh(vr, vx, EARLY, sc, ntok, ot, kg);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!EARLY && has1) request_values(nxt.phys);
            if (cur.valid && cur.last) {
                const bool all = cur.first_of && cur.ends;        // the wave has the whole request
                if (!nxt.valid) {
                    open_first = cur.first_of;
                    open_last = cur.ends;
                    open_tail = cur.base > 0;         // (a prefix pass has the pages before)
                    if (all && cur.base == 0) finish(cur.r, true);
                    else open_r = cur.r;
                    break;
                }
                finish(cur.r, all && cur.base == 0);
                if (!cur.first_of) wrote_r = cur.r;
                load_q(nxt.r);
                clear();
            }
            cur = nxt;
        }
    }

    // ---- the workgroup's merge of the open parts
    if (open_r >= 0) {
        const float l = cross_sum(lrun);
        f32x4_t og[Pg::GROUPS];
        Pg::gather(ot, og);
        if (hn < G) {
            float *o = reinterpret_cast<float *>(mine) + hn * D;
#pragma unroll
            for (int j = 0; j < Pg::GROUPS; ++j) *reinterpret_cast<f32x4_t *>(o + Pg::group_dim(j, n, kg)) = og[j];
            if (n == hn && kg == 0) {
                s_ml[wave][hn][0] = mrun;
                s_ml[wave][hn][1] = l;
            }
        }
    }
    // the parts of waves [w0, w1) of request rr (m1, pt: and the partial that the
    // wave after them wrote, folded last, as if it had left its part open).  A
    // workgroup of one request asks for all waves' values before it uses the first:
    // a loop over them pays an LDS latency each (0.5-1 us of a call).  Among short
    // requests, of two or three waves, the loop is the shorter one.
    auto fold = [&](int w0, int w1, int rr, bool more_, bool direct) {
        float *pt = part_of(rr);
        T *out = reinterpret_cast<T *>(a.out) + ((size_t)rr * Hq + (size_t)h * G) * D;
        constexpr int EPT = (G * D + NT - 1) / NT;
        float M[EPT], Ls[EPT], Os[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = min(tid + e * NT, G * D - 1), g = i / D, dd = i % D;
            const float *q = pt + (size_t)g * (D + 2);
            const float m1 = more_ ? q[D] : kNegInf;
            M[e] = m1;
            Ls[e] = Os[e] = 0.0f;
            auto add = [&](float mw, float lw, float ow) {
                const float fw = mw == kNegInf ? 0.0f : exp2f(mw - M[e]);
                Ls[e] += lw * fw;
                Os[e] += ow * fw;
            };
            if (OWN || w1 - w0 == NW) {               // (uniform)
                float mw[NW], lw[NW], ow[NW];
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    mw[w] = s_ml[w][g][0];
                    lw[w] = s_ml[w][g][1];
                    ow[w] = reinterpret_cast<const float *>(s_wave[w])[i];
                }
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    if (w >= w1) mw[w] = kNegInf;
                    M[e] = fmaxf(M[e], mw[w]);
                }
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    if (w < w1) add(mw[w], lw[w], ow[w]);
            } else {
                for (int w = w0; w < w1; ++w) M[e] = fmaxf(M[e], s_ml[w][g][0]);
                for (int w = w0; w < w1; ++w)
                    add(s_ml[w][g][0], s_ml[w][g][1], reinterpret_cast<const float *>(s_wave[w])[i]);
            }
            const float f1_ = m1 == kNegInf ? 0.0f : exp2f(m1 - M[e]);
            if (more_) {
                Ls[e] += q[D + 1] * f1_;
                Os[e] += q[dd] * f1_;
            }
        }
        if (more_ && !direct) __syncthreads();         // every thread has read the partial that is replaced
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = tid + e * NT, g = i / D, dd = i % D;
            if (i >= G * D) continue;
            if (direct) {
                Traits<T>::store(out + i, divided(Os[e], Ls[e]));
            } else {
                pt[(size_t)g * (D + 2) + dd] = Os[e];
                if (dd == 0) store8(pt + (size_t)g * (D + 2) + D, M[e], Ls[e]);
            }
        }
    };
    if constexpr (OWN > 0) {
        __syncthreads();
        if (parts > 1) fold(0, parts, wg, false, true);    // (one part: its wave wrote the output)
    } else {
        if (lane == 0) {
            s_open[wave][0] = open_r;
            s_open[wave][1] = (open_first ? 1 : 0) | (open_last ? 2 : 0) | (open_tail ? 4 : 0);
            s_open[wave][2] = wrote_r;
        }
        __syncthreads();
        const int reqs = s_open[lane % NW][0], ends = s_open[lane % NW][1], wrote = s_open[lane % NW][2];
        for (int w0 = 0; w0 < NW;) {
            const int rr = __builtin_amdgcn_readlane(reqs, w0);
            if (rr < 0) {
                ++w0;
                continue;
            }
            int w1 = w0 + 1;                          // waves [w0, w1) left parts of request rr open
            while (w1 < NW && __builtin_amdgcn_readlane(reqs, w1) == rr) ++w1;
            // the wave after them may have written the rest of rr as this workgroup's partial
            const bool more_ = w1 < NW && __builtin_amdgcn_readlane(wrote, w1) == rr;
            const int begin = __builtin_amdgcn_readlane(ends, w0), end = __builtin_amdgcn_readlane(ends, w1 - 1);
            const bool all = (begin & 1) && (more_ || (end & 2));
            fold(w0, w1, rr, more_, all && !(begin & 4));
            w0 = w1;
        }
    }
}

// ---------------------------------------------------------------------------
// Shared-prefix pass (gp_decode_attention_shared; App. E.2 keeps a common
// prefix in reference-counted blocks that many requests read).  Work item =
// (KV head h, prefix slot c, block of 4 * 16 / G requests of one group).  The
// prefix is split evenly over its slots; a slot's pages are read once per
// workgroup, kPrefixBatch at a time, straight into LDS by direct-to-LDS loads
// (the next batch in flight while this one is computed), and each of the four
// waves serves 16 query rows (16 / G requests x G heads) over all of them.
// Per page a wave computes S^T = K.Q^T on v_mfma_f32_16x16x32_bf16 (the keys
// as the A operand), so that every lane holds four tokens of one query row; an
// online softmax per row; and O^T += V^T.P^T on v_mfma_f32_16x16x16bf16_1k,
// with V^T read by ds_read_b64_tr_b16 and P, already in the B layout, split
// into two bfloat16 terms (hi + lo carry 16 significant bits, so P.V keeps
// float32-level accuracy while the values stay exact bfloat16).  Every lane
// holds output dims of one row, so the rescale needs no lane exchange.  The
// slot's (o, max, sum) per row go to partial slot c of each request; the
// private tails follow in the next slots and the merge folds them together.
// A request reads the pass only if it is not held, holds at least the
// prefix's tokens and its table matches the group leader's on every prefix
// page; otherwise the tail pass covers all of its pages (both passes make the
// same test).
// Bound: HBM on the tails; the prefix pages are read once per block of
// requests instead of once per request.
// The pass stages kPrefixBatch pages (keys and values) per round and keeps
// two rounds in LDS.
constexpr int kPrefixBatch = 4;

// Whether request r may read a prefix pass of pp pages: not held, more pages
// and tokens than the prefix, within its table (the chunk pass makes the same
// test); both passes also require the leader's page ids on every prefix page.
__device__ inline bool prefix_reader(const DecodeArgs &a, int r, int pp) {
    const int m = a.seq_lens[r], P = a.num_pages[r];
    return m > pp * kPage && P > pp && P <= a.max_pages && m <= P * kPage;
}

template <int D, int G>
__global__ __launch_bounds__(64 * kPrefixWaves) void prefix_kernel(DecodeArgs a) {
    constexpr int KK = D / 32;            // S^T MFMA steps per page
    constexpr int NW = kPrefixWaves;
    constexpr int NT = 64 * NW;
    constexpr int RPW = 16 / G;           // requests per wave (16 query rows)
    constexpr int RPB = NW * RPW;         // requests per workgroup
    constexpr int DT = D / 16;            // O^T tiles of 16 dims
    constexpr int UPR = D / 8;            // 16-byte units per row
    constexpr int UPP = kPage * UPR;      // units of one page of one head (keys or values)
    constexpr int NB = kPrefixBatch;      // pages per round
    constexpr int RPI = 64 / UPR;         // rows per load instruction
    constexpr int IPP = 2 * UPP / 64;     // load instructions per page (keys, then values)
    constexpr int IPW = NB * IPP / NW;    // load instructions per wave and round
    static_assert((NB * IPP) % NW == 0 && UPP % 64 == 0, "staging layout");
    __shared__ __attribute__((aligned(16))) uint4 s_stage[2][NB][2][UPP];   // [round % 2][page][keys, values]
    __shared__ int s_ids[kMaxPrefixSlotPages];
    __shared__ int s_match[RPB];

    const int h = blockIdx.x, c = blockIdx.y, blk = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    int gi = 0;
    while (gi + 1 < a.ngroups && blk >= a.g_blk0[gi + 1]) ++gi;
    const int first = a.g_first[gi], nreq = a.g_num[gi], ppages = a.g_pages[gi];
    const int r0 = first + (blk - a.g_blk0[gi]) * RPB;
    // the prefix split evenly over its slots (cs <= kMaxPrefixSlotPages pages each)
    const int cs = cdiv(ppages, a.g_slots[gi]);
    const int p_begin = c * cs, p_end = min(ppages, p_begin + cs);
    const int Hkv = a.Hkv, Hq = Hkv * G;
    const int32_t *lead = a.page_table + (size_t)first * a.max_pages;

    // which requests of the block read the pass (the same test in every
    // workgroup of the block, so they agree without talking)
    for (int j = tid; j < RPB; j += NT) {
        const int r = r0 + j;
        s_match[j] = r < first + nreq && prefix_reader(a, r, ppages) ? 1 : 0;
    }
    for (int k = tid; k < p_end - p_begin; k += NT) {
        const int pid = lead[p_begin + k];
        s_ids[k] = pid >= 0 && pid < a.pool_pages ? pid : -1;
    }
    __syncthreads();
    for (int e = tid; e < RPB * ppages; e += NT) {
        const int j = e / ppages, pg = e % ppages;
        if (s_match[j] && a.page_table[(size_t)(r0 + j) * a.max_pages + pg] != lead[pg]) s_match[j] = 0;
    }
    __syncthreads();
    if (p_begin >= ppages) return;
    int any = 0;
    for (int j = 0; j < RPB; ++j) any |= s_match[j];
    if (!any) return;                                    // uniform

    // this wave's 16 query rows (row n = request wave * RPW + n / G, head
    // n % G) as the B operand of S^T = K Q^T: lane (n, kg) holds dims
    // 32 kk + 8 kg .. + 7
    const int jq = wave * RPW + n / G;
    const bool rowq = s_match[jq] != 0;
    bf16x8_t qb[KK];
    {
        const uint16_t *qp = reinterpret_cast<const uint16_t *>(a.q) +
                             ((size_t)(rowq ? r0 + jq : first) * Hq + (size_t)h * G + n % G) * D;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const bf16x8_t x = __builtin_bit_cast(bf16x8_t, load16(qp + kk * 32 + kg * 8));
            qb[kk] = rowq ? x : bf16x8_t{};
        }
    }

    const uint16_t *kpool = reinterpret_cast<const uint16_t *>(a.k);
    const uint16_t *vpool = reinterpret_cast<const uint16_t *>(a.v);
    const size_t head_off = (size_t)h * kPage * D;
    const size_t page_elems = (size_t)Hkv * kPage * D;
    const int npage = p_end - p_begin;
    // Round rr's pages rr NB .. rr NB + NB - 1 go to stage rr % 2, each load
    // instruction one contiguous run of RPI rows; the waves split the
    // instructions.  Unit u of row R sits at R UPR + (u ^ fk(R)) for keys,
    // fk(R) = R % UPR (a score-layout read of 16 rows hits 16 bank groups),
    // and at R UPR + (u ^ fv(R)) for values, fv(R) = 2 (R % (UPR / 2)) (the
    // transposed reads of 4 rows x 2 units hit distinct bank groups).  An
    // invalid page id reads page 0 (its scores are masked).
    auto issue = [&](int rr) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const int e = wave * IPW + i, j = e / IPP, w2 = e % IPP;
            const int k = rr * NB + j;
            if (k < npage) {                             // wave-uniform
                const bool isv = w2 >= IPP / 2;
                const int q = isv ? w2 - IPP / 2 : w2;
                const int R = q * RPI + lane / UPR, s = lane % UPR;
                const int u = s ^ (isv ? 2 * (R % (UPR / 2)) : R % UPR);
                const uint16_t *src = (isv ? vpool : kpool) + (size_t)max(s_ids[k], 0) * page_elems + head_off +
                                      (size_t)R * D + u * 8;
                __builtin_amdgcn_global_load_lds((global_cvoid_t *)src,
                                                 (lds_void_t *)(&s_stage[rr & 1][j][isv][q * 64]), 16, 0, kCpolNT);
            }
        }
    };

    float mrun = kNegInf, lrun = 0.0f;   // row n: running max (log2 units), this lane's share of the sum
    f32x4_t o[DT];                       // O^T tile t: lane (n, kg) holds dims 16 t + 4 kg + e of row n
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    auto page = [&](const uint4 *ks, const uint4 *vs, bool valid) {
        bf16x8_t kc[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            kc[kk] = __builtin_bit_cast(bf16x8_t, ks[n * UPR + ((4 * kk + kg) ^ (n % UPR))]);
        f32x4_t st = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kc[kk], qb[kk], st, 0, 0, 0);
        // online softmax of row n; this lane has tokens 4 kg + e
        float s[4], ml = kNegInf;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = valid ? st[e] * a.qscale : kNegInf;
            ml = fmaxf(ml, s[e]);
        }
        ml = fmaxf(ml, __shfl_xor(ml, 16, 64));
        ml = fmaxf(ml, __shfl_xor(ml, 32, 64));
        const float mn = fmaxf(mrun, ml);
        // arguments are <= 0: the hardware exp2 needs no range fix-up
        const float alpha = mn == kNegInf ? 1.0f : __builtin_amdgcn_exp2f(mrun - mn);
        float p[4], psum = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = mn == kNegInf ? 0.0f : __builtin_amdgcn_exp2f(s[e] - mn);
            psum += p[e];
        }
        lrun = lrun * alpha + psum;
        mrun = mn;
        if (__any(alpha != 1.0f)) {                      // skip while no row's max has moved
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[t][e] *= alpha;
        }
        // P^T as the B operand (tokens 4 kg + e of row n) in two bf16 terms
        bf16x4s_t phi, plo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const __bf16 hb = (__bf16)p[e];              // round to nearest even
            phi[e] = __builtin_bit_cast(short, hb);
            plo[e] = __builtin_bit_cast(short, (__bf16)(p[e] - (float)hb));   // p - hi is exact in float32
        }
        // V^T tile t as the A operand by transposed reads: lane j of group kg
        // names row R = 4 kg + j / 4, dims 16 t + 4 (j % 4) (unit 2 t + (j % 4)
        // / 2, half (j % 4) % 2); lane n receives the values of tokens
        // 4 kg .. 4 kg + 3 at dim 16 t + n
        const int R = 4 * kg + n / 4, qd = n % 4;
        const char *vrow = reinterpret_cast<const char *>(vs + R * UPR) + (qd & 1) * 8;
        const int fv = 2 * (R % (UPR / 2));
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const bf16x4s_t vt = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) bf16x4s_t *)(vrow + ((2 * t + qd / 2) ^ fv) * 16));
            o[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, phi, o[t], 0, 0, 0);
            o[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, plo, o[t], 0, 0, 0);
        }
    };

    issue(0);
    for (int rr = 0; rr * NB < npage; ++rr) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0);            // this wave's part of round rr has landed
        __syncthreads();                                 // all of it; every wave is done with round rr - 1
        if ((rr + 1) * NB < npage) issue(rr + 1);        // into the stage round rr - 1 used
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int k = rr * NB + j;
            if (k < npage) page(s_stage[rr & 1][j][0], s_stage[rr & 1][j][1], s_ids[k] >= 0);
        }
    }

    // partials of row n: o of dims 16 t + 4 kg + e, (max, sum) by the kg 0 lanes
    lrun += __shfl_xor(lrun, 16, 64);
    lrun += __shfl_xor(lrun, 32, 64);
    if (rowq) {
        float *part = a.prefix + (((size_t)(r0 + jq) * Hkv + h) * a.pslots + c) * G * (D + 2) +
                      (size_t)(n % G) * (D + 2);
#pragma unroll
        for (int t = 0; t < DT; ++t) *reinterpret_cast<f32x4_e4_t *>(part + 16 * t + 4 * kg) = o[t];
        if (kg == 0) {
            part[D] = mrun;
            part[D + 1] = lrun;
        }
    }
}

// ------------------------------------------------------------------- merge --
// Second pass: one workgroup per (KV head, request) folds the (max, sum, o)
// partials of a request that spans workgroups (or reads a prefix pass).
// Running it as its own launch lets the kernel boundary publish the partials;
// a device-scope fence per workgroup would write back and invalidate the L2 of
// every XCD thousands of times per step.  A thread holds pairs of dims and
// folds every NS-th slot, eight slots' loads in flight; with few (KV head,
// request) pairs the workgroups are larger, so that more slots are in flight
// (one request of a long context has dozens).
//
// gp_decode_step: the summaries of query heads [h G, h G + G) are updated here
// (Sec. 4.1) rather than in the chunk pass, where the memory round trip it adds
// lengthened the workgroups that end the grid.  The slot is requested first,
// the query and the old values with the partials' bookkeeping, and the update
// is stored after the output.  A held request, or with a new token one without
// room, keeps its summaries.
template <typename T, int D, int G, int NT>
__global__ __launch_bounds__(NT) void merge_kernel(DecodeArgs a) {
    using Tr = Traits<T>;
    constexpr int GD2 = G * D / 2;                   // pairs of output dims
    constexpr int EP = (GD2 + NT - 1) / NT;          // pairs per thread
    constexpr int NS = GD2 < NT ? NT / GD2 : 1;      // threads per pair
    constexpr int BATCH = EP > 1 ? 4 : 8;            // slots in flight per thread and pair
    static_assert(GD2 % NT == 0 || NT % GD2 == 0, "thread layout");
    __shared__ float4 s_red[NS > 1 ? NT : 1];
    const int h = blockIdx.x, r = blockIdx.y;
    const int tid = threadIdx.x;
    const int R = a.R, Hq = a.Hkv * G;
    constexpr int FE = (G * D + NT - 1) / NT;        // summary elements per thread
    float f_q[FE], f_s[FE], f_l[FE];
    float *fS = nullptr;
    int f_slot = -1;
    bool f_init = false;
    if (a.qstate) {
        f_slot = a.slot_ids[r];
        f_init = a.init[r] != 0;
    }
    const int m = a.lens[r], took = a.lens[R + r], first = a.lens[2 * R + r], cnt = a.lens[3 * R + r];
    const bool pre = a.ngroups > 0 && a.lens[4 * R + r] != 0;
    if (m < 0) return;                               // held
    if (a.qstate && f_slot >= 0 && f_slot < a.M) {
        const T *qp = reinterpret_cast<const T *>(a.q_pre) + ((size_t)r * Hq + (size_t)h * G) * D;
        fS = a.qstate + (size_t)f_slot * 2 * Hq * D + (size_t)h * G * D;
#pragma unroll
        for (int e = 0; e < FE; ++e) {
            const int i = min(tid + NT * e, G * D - 1);
            f_q[e] = Tr::load(qp + i);
            f_s[e] = fS[i];
            f_l[e] = fS[(size_t)Hq * D + i];
        }
    }
    if (a.advance && h == 0 && tid == 0 && took) {   // the request took the step's token
        a.seq_lens_w[r] = m;
        if (a.positions) a.positions[r] += 1;
    }
    if (cnt > 0) {
        int npre = 0;
        if (pre)
            for (int g = 0; g < a.ngroups; ++g)
                if (r >= a.g_first[g] && r < a.g_first[g] + a.g_num[g]) npre = a.g_slots[g];
        const int total = npre + cnt;
        const float *pp = a.prefix + ((size_t)r * a.Hkv + h) * a.pslots * G * (D + 2);
        const float *pt = a.partial + ((size_t)h * a.slots + first) * G * (D + 2);
        const int sg = NS > 1 ? tid / GD2 : 0;
        float M[EP], Ls[EP], Ox[EP], Oy[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) {
            const int i = 2 * (NS > 1 ? tid % GD2 : tid + e * NT);
            const int off = (i / D) * (D + 2);
            M[e] = kNegInf;
            Ls[e] = Ox[e] = Oy[e] = 0.0f;
            for (int k0 = sg; k0 < total; k0 += NS * BATCH) {
                f32x2_t ml[BATCH], o[BATCH];
#pragma unroll
                for (int b = 0; b < BATCH; ++b) {
                    const int k = min(k0 + b * NS, total - 1);
                    const float *q = (k < npre ? pp + (size_t)k * G * (D + 2) : pt + (size_t)(k - npre) * G * (D + 2)) + off;
                    ml[b] = load8(q + D);
                    o[b] = load8(q + i % D);
                }
                float mn = M[e];
#pragma unroll
                for (int b = 0; b < BATCH; ++b)
                    if (k0 + b * NS < total) mn = fmaxf(mn, ml[b][0]);
                const float f0 = M[e] == kNegInf ? 0.0f : exp2f(M[e] - mn);
                Ls[e] *= f0;
                Ox[e] *= f0;
                Oy[e] *= f0;
                M[e] = mn;
#pragma unroll
                for (int b = 0; b < BATCH; ++b) {
                    if (k0 + b * NS < total && ml[b][0] != kNegInf) {
                        const float f = exp2f(ml[b][0] - mn);
                        Ls[e] += ml[b][1] * f;
                        Ox[e] += o[b][0] * f;
                        Oy[e] += o[b][1] * f;
                    }
                }
            }
        }
        if constexpr (NS > 1) {
            s_red[tid] = make_float4(M[0], Ls[0], Ox[0], Oy[0]);
            __syncthreads();
            if (tid < GD2) {
                // (sixteen at a time: all 32 of a small head at once do not fit the registers)
#pragma unroll 16
                for (int k = 0; k < NS; ++k) M[0] = fmaxf(M[0], s_red[tid + k * GD2].x);
                Ls[0] = Ox[0] = Oy[0] = 0.0f;
#pragma unroll 16
                for (int k = 0; k < NS; ++k) {
                    const float4 x = s_red[tid + k * GD2];
                    const float f = x.x == kNegInf ? 0.0f : exp2f(x.x - M[0]);
                    Ls[0] += x.y * f;
                    Ox[0] += x.z * f;
                    Oy[0] += x.w * f;
                }
            }
        }
        T *out = reinterpret_cast<T *>(a.out) + ((size_t)r * Hq + (size_t)h * G) * D;
        if (NS == 1 || tid < GD2) {
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                const int i = 2 * (NS > 1 ? tid : tid + e * NT);
                Tr::store(out + i, divided(Ox[e], Ls[e]));
                Tr::store(out + i + 1, divided(Oy[e], Ls[e]));
            }
        }
    }
    if (fS && (a.k_new == nullptr || took)) {
        const double cs_ = 1.0 - a.beta_s, cl_ = 1.0 - a.beta_l;
#pragma unroll
        for (int e = 0; e < FE; ++e) {
            const int i = tid + NT * e;
            if (i < G * D) {
                fS[i] = f_init ? f_q[e] : ema_step(f_s[e], f_q[e], a.beta_s, cs_);
                fS[(size_t)Hq * D + i] = f_init ? f_q[e] : ema_step(f_l[e], f_q[e], a.beta_l, cl_);
            }
        }
    }
}

template <typename T, int D>
hipError_t launch_g(int G, const DecodeArgs &a, int stages, hipStream_t s) {
    const dim3 grid(a.Hkv, a.W), mgrid(a.Hkv, a.R);
    constexpr bool bf16 = sizeof(T) == 2;
    constexpr int NW = waves_of<T, D>(), NT = 64 * NW;
    constexpr int NN = page_bytes_of<T, D>() <= 2048 ? 4 : NW;        // (see decode_own_narrow)
    // the step variant with a new token and the tails of the shared-prefix
    // decode are their own instantiations, so plain decode attention carries
    // none of their code (a step call's summary update is in the merge pass:
    // without a new token its chunk pass is plain decode attention)
    const int mode = a.ngroups > 0 ? 2 : a.k_new != nullptr ? 1 : 0;
    // the merge pass also advances the lengths when a token went in, updates
    // the summaries of a step call, and folds the prefix partials of a
    // shared-prefix call; with a workgroup per request there is nothing to fold
    const bool own = mode != 2 && decode_own(a.max_pages, a.R, a.Hkv, page_bytes_of<T, D>(), NW, quad_heads<T>(G));
    const bool narrow = own && decode_own_narrow(a.R, a.Hkv);
    const bool chunks = stages & GP_DECODE_CHUNKS, prefix = (stages & GP_DECODE_PREFIX) && mode == 2,
               merge = (stages & GP_DECODE_MERGE) &&
                       (!own || (a.k_new && a.advance) || a.qstate);
    const bool wide = (int64_t)a.Hkv * a.R < kWideMerge;
    // prefix pass grid: (KV head, prefix slot, request block)
    int max_ps = 1;
    for (int g = 0; g < a.ngroups; ++g) max_ps = max(max_ps, a.g_slots[g]);
    const dim3 pgrid(a.Hkv, max_ps, max(a.g_blk0[a.ngroups], 1));
    switch (G) {
#define GP_CASE(GG)                                                                \
    case GG:                                                                       \
        if constexpr (bf16) {                                                      \
            if (prefix) prefix_kernel<D, GG><<<pgrid, 64 * kPrefixWaves, 0, s>>>(a); \
            if (chunks && mode == 2) decode_kernel<T, D, GG, 2, 0><<<grid, NT, 0, s>>>(a); \
        }                                                                          \
        if (chunks && mode == 1 && own) {                                         \
            if (NN < NW && narrow) decode_kernel<T, D, GG, 1, NN><<<mgrid, 64 * NN, 0, s>>>(a); \
            else decode_kernel<T, D, GG, 1, NW><<<mgrid, NT, 0, s>>>(a);            \
        }                                                                          \
        if (chunks && mode == 1 && !own) decode_kernel<T, D, GG, 1, 0><<<grid, NT, 0, s>>>(a); \
        if (chunks && mode == 0 && own) {                                         \
            if (NN < NW && narrow) decode_kernel<T, D, GG, 0, NN><<<mgrid, 64 * NN, 0, s>>>(a); \
            else decode_kernel<T, D, GG, 0, NW><<<mgrid, NT, 0, s>>>(a);            \
        }                                                                          \
        if (chunks && mode == 0 && !own) decode_kernel<T, D, GG, 0, 0><<<grid, NT, 0, s>>>(a); \
        if (merge && wide) merge_kernel<T, D, GG, 1024><<<mgrid, 1024, 0, s>>>(a); \
        if (merge && !wide) merge_kernel<T, D, GG, 256><<<mgrid, 256, 0, s>>>(a);  \
        break;
        GP_CASE(1) GP_CASE(2) GP_CASE(4) GP_CASE(8)
#undef GP_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(gp_dtype_t dt, int D, int G, const DecodeArgs &a, int stages, hipStream_t s) {
    if (dt == GP_BF16)
        return D == 128 ? launch_g<uint16_t, 128>(G, a, stages, s) : launch_g<uint16_t, 64>(G, a, stages, s);
    return D == 128 ? launch_g<float, 128>(G, a, stages, s) : launch_g<float, 64>(G, a, stages, s);
}

}  // namespace gp
