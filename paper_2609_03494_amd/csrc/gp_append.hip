// Step prologue of the decode loop: the current token's K and V go into the
// paged cache of every layer and the dual-timescale summaries take their EMA
// step (Sec. 3.1 paged KV cache, Sec. 3.2 EMA equation, App. E.1 query-state
// pool), for every request that is in the step's batch and has room.
//
// Work item = (request, layer): the workgroups of a request read its resident
// length and none of them changes it; a second, tiny launch advances lengths
// and positions once every write of the first is done.  (One workgroup per
// request that walked the layers one after the other and advanced the length
// itself spent its time on the round trips of each layer: 779 us at 64
// requests x 36 layers of 32/8 heads, d 128, where the traffic is 189 MB;
// 49 us now, 3.8 TB/s of reads and writes.)  A
// call of one layer has nothing to spread: its workgroups advance the lengths
// themselves, in one launch; so do those of a call small enough for one workgroup
// per request (append_flat_kernel).  Held requests (seq_len < 0) and requests whose
// pages are full (at a capacity boundary, waiting for a decision) take no token
// and keep their summaries.  The summary arithmetic is ema_step, the same as
// the summaries kernel's, so the two agree bit for bit.
//
// Bound: HBM with many layers (2 x 4 B x 2 views per query element, read and
// written, are most of it), launch latency with one.
#include "gp_internal.h"

namespace gp {

namespace {

template <typename T>
__device__ inline float load_elem(const T *p, size_t i);
template <>
__device__ inline float load_elem<float>(const float *p, size_t i) { return p[i]; }
template <>
__device__ inline float load_elem<uint16_t>(const uint16_t *p, size_t i) { return bf16_to_f32(p[i]); }

// The page that takes the token of request r (-1: the request takes none), and
// its resident length m.
__device__ inline int append_page(const AppendArgs &a, int r, int &m) {
    const int P = a.num_pages[r];
    m = a.seq_lens[r];
    if (m < 0 || P <= 0 || P > a.max_pages || m >= P * kPage) return -1;
    const int pid = a.page_table[(size_t)r * a.max_pages + m / kPage];
    return pid >= 0 && pid < a.pool_pages ? pid : -1;
}

// four consecutive elements of a query, widened
__device__ inline float4 load4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ inline float4 load4(const uint16_t *p) {
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    return make_float4(bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y));
}
__device__ inline float4 ema4(const float4 &s, const float4 &x, double b, double c) {
    return make_float4(ema_step(s.x, x.x, b, c), ema_step(s.y, x.y, b, c), ema_step(s.z, x.z, b, c),
                       ema_step(s.w, x.w, b, c));
}

// Grid (request, layer).  VEC: every pointer is 16-byte aligned (torch's own
// allocations are; a caller's sub-array need not be), so rows move in 16-byte
// units and a thread takes four summary elements at a time, the loads of
// kUnroll such groups in flight together; otherwise one element at a time.
constexpr int kUnroll = 4;
template <typename T, int D, bool VEC>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a) {
    const int r = blockIdx.x, l = blockIdx.y, tid = threadIdx.x;
    const int slot = a.slot_ids[r];
    const bool has_slot = slot >= 0 && slot < a.M;
    const bool init = a.init != nullptr && a.init[r] != 0;
    int m;
    const int pid = append_page(a, r, m);
    if (pid < 0) return;
    const int HkvD = a.Hkv * D, HqD = a.Hq * D;
    const double cs = 1.0 - a.beta_s, cl = 1.0 - a.beta_l;
    // K, V: token slot m % 16 of page pid, every KV head
    const T *kn = reinterpret_cast<const T *>(a.k_new) + ((size_t)l * a.R + r) * HkvD;
    const T *vn = reinterpret_cast<const T *>(a.v_new) + ((size_t)l * a.R + r) * HkvD;
    T *kp = reinterpret_cast<T *>(a.k[l]);
    T *vp = reinterpret_cast<T *>(a.v[l]);
    // summaries of layer l: [M][2][Hq][D] slice of the [L][M][2][Hq][D] pool
    const T *q = reinterpret_cast<const T *>(a.q_pre) + ((size_t)l * a.R + r) * HqD;
    float *S = a.qstate + ((size_t)l * a.M + (has_slot ? slot : 0)) * 2 * HqD;
    float *Lv = S + HqD;
    if constexpr (VEC) {
        constexpr int EPU = 16 / sizeof(T), UPR = D / EPU;     // elements per unit, units per row
        for (int i = tid; i < 2 * a.Hkv * UPR; i += 256) {
            const bool isv = i >= a.Hkv * UPR;
            const int u = isv ? i - a.Hkv * UPR : i, h = u / UPR, w = u % UPR;
            const uint4 x = reinterpret_cast<const uint4 *>(isv ? vn : kn)[u];
            const size_t dst = (((size_t)pid * a.Hkv + h) * kPage + m % kPage) * D;
            reinterpret_cast<uint4 *>((isv ? vp : kp) + dst)[w] = x;
        }
        if (has_slot) {
            const int n4 = HqD / 4;
            for (int base = tid; base < n4; base += 256 * kUnroll) {
                float4 x[kUnroll], s[kUnroll], w[kUnroll];
#pragma unroll
                for (int k = 0; k < kUnroll; ++k) {
                    const int i = min(base + 256 * k, n4 - 1);
                    x[k] = load4(q + 4 * i);
                    s[k] = load4(S + 4 * i);
                    w[k] = load4(Lv + 4 * i);
                }
#pragma unroll
                for (int k = 0; k < kUnroll; ++k) {
                    const int i = base + 256 * k;
                    if (i < n4) {
                        *reinterpret_cast<float4 *>(S + 4 * i) = init ? x[k] : ema4(s[k], x[k], a.beta_s, cs);
                        *reinterpret_cast<float4 *>(Lv + 4 * i) = init ? x[k] : ema4(w[k], x[k], a.beta_l, cl);
                    }
                }
            }
        }
    } else {
        for (int i = tid; i < HkvD; i += 256) {
            const size_t dst = (((size_t)pid * a.Hkv + i / D) * kPage + m % kPage) * D + i % D;
            kp[dst] = kn[i];
            vp[dst] = vn[i];
        }
        if (has_slot) {
            for (int i = tid; i < HqD; i += 256) {
                const float x = load_elem<T>(q, i);
                S[i] = init ? x : ema_step(S[i], x, a.beta_s, cs);
                Lv[i] = init ? x : ema_step(Lv[i], x, a.beta_l, cl);
            }
        }
    }
    if (gridDim.y > 1) return;                       // advance_kernel follows
    __syncthreads();
    if (tid == 0) {
        a.seq_lens[r] = m + 1;
        a.positions[r] += 1;
    }
}

// Few layers and short rows: one launch of one workgroup per request, all of whose
// 16-byte units (K and V of every layer, groups of four summary elements) are in
// flight at once, so the workgroup advances the length itself.  Up to kFlatUnits
// of them, one round: the second launch costs a host that launches call by call
// 4 us (12 layers of 16/4 heads, d 64, 16 requests: 25.4 us a call against 29.9),
// and the GPU 1 us (2 layers of 4/2 heads, d 64: 5.4 against 6.1 in a graph).
// With more units the CUs that hold no request are missed: 5 layers of 32/8
// heads, d 128, in two rounds 10.7 us in a graph against 7.2.
constexpr int kFlatThreads = 1024, kFlatUnits = kUnroll * kFlatThreads;
template <typename T, int D>
__global__ __launch_bounds__(kFlatThreads) void append_flat_kernel(AppendArgs a) {
    const int r = blockIdx.x, tid = threadIdx.x;
    const int slot = a.slot_ids[r];
    const bool has_slot = slot >= 0 && slot < a.M;
    const bool init = a.init != nullptr && a.init[r] != 0;
    int m;
    const int pid = append_page(a, r, m);
    if (pid < 0) return;
    constexpr int EPU = 16 / sizeof(T), UPR = D / EPU;         // elements per unit, units per row
    const int HkvD = a.Hkv * D, HqD = a.Hq * D;
    const double cs = 1.0 - a.beta_s, cl = 1.0 - a.beta_l;
    const int half = a.Hkv * UPR, KV = 2 * half, U = KV + (has_slot ? HqD / 4 : 0), N = a.n_layers * U;
    if (tid < N) {                                   // (waves without a unit have nothing to load)
        float4 x[kUnroll], s[kUnroll], w[kUnroll];
        T *kv[kUnroll];
        float *S[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int i = min(tid + kFlatThreads * k, N - 1), l = i / U, u = i - l * U;
            kv[k] = nullptr;
            if (u < KV) {
                const bool isv = u >= half;
                const int j = isv ? u - half : u, h = j / UPR;
                x[k] = reinterpret_cast<const float4 *>(reinterpret_cast<const T *>(isv ? a.v_new : a.k_new) +
                                                        ((size_t)l * a.R + r) * HkvD)[j];
                kv[k] = reinterpret_cast<T *>(isv ? a.v[l] : a.k[l]) +
                        (((size_t)pid * a.Hkv + h) * kPage + m % kPage) * D + (j % UPR) * EPU;
            } else {
                const int j = 4 * (u - KV);
                S[k] = a.qstate + ((size_t)l * a.M + slot) * 2 * HqD + j;
                x[k] = load4(reinterpret_cast<const T *>(a.q_pre) + ((size_t)l * a.R + r) * HqD + j);
                s[k] = *reinterpret_cast<const float4 *>(S[k]);
                w[k] = *reinterpret_cast<const float4 *>(S[k] + HqD);
            }
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            if (tid + kFlatThreads * k >= N) break;
            if (kv[k]) {
                *reinterpret_cast<float4 *>(kv[k]) = x[k];
            } else {
                *reinterpret_cast<float4 *>(S[k]) = init ? x[k] : ema4(s[k], x[k], a.beta_s, cs);
                *reinterpret_cast<float4 *>(S[k] + HqD) = init ? x[k] : ema4(w[k], x[k], a.beta_l, cl);
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        a.seq_lens[r] = m + 1;
        a.positions[r] += 1;
    }
}

__global__ __launch_bounds__(64) void advance_kernel(AppendArgs a) {
    const int r = blockIdx.x * 64 + threadIdx.x;
    int m;
    if (r < a.R && append_page(a, r, m) >= 0) {
        a.seq_lens[r] = m + 1;
        a.positions[r] += 1;
    }
}

template <typename T, int D>
void launch_td(const AppendArgs &a, hipStream_t s) {
    uintptr_t bits = reinterpret_cast<uintptr_t>(a.k_new) | reinterpret_cast<uintptr_t>(a.v_new) |
                     reinterpret_cast<uintptr_t>(a.q_pre) | reinterpret_cast<uintptr_t>(a.qstate);
    for (int l = 0; l < a.n_layers; ++l)
        bits |= reinterpret_cast<uintptr_t>(a.k[l]) | reinterpret_cast<uintptr_t>(a.v[l]);
    const dim3 grid(a.R, a.n_layers);
    const int units = 2 * a.Hkv * (D * (int)sizeof(T) / 16) + a.Hq * (D / 4);         // of a request, per layer
    if (bits % 16 == 0 && a.n_layers > 1 && (int64_t)units * a.n_layers <= kFlatUnits) {
        append_flat_kernel<T, D><<<a.R, kFlatThreads, 0, s>>>(a);
        return;
    }
    if (bits % 16 == 0)
        append_kernel<T, D, true><<<grid, 256, 0, s>>>(a);
    else
        append_kernel<T, D, false><<<grid, 256, 0, s>>>(a);
    if (a.n_layers > 1) advance_kernel<<<cdiv(a.R, 64), 64, 0, s>>>(a);
}

}  // namespace

hipError_t launch_append(gp_dtype_t dt, int D, const AppendArgs &a, hipStream_t s) {
    if (a.R == 0) return hipSuccess;
    if (dt == GP_BF16)
        D == 128 ? launch_td<uint16_t, 128>(a, s) : launch_td<uint16_t, 64>(a, s);
    else
        D == 128 ? launch_td<float, 128>(a, s) : launch_td<float, 64>(a, s);
    return hipGetLastError();
}

}  // namespace gp
