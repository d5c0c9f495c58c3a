// Routing baselines with a materialised proxy map (the standard routing the paper compares
// against, Section 2 after Eq. block_proxy): the full proxy map s_hat = s * Qbar Kbar^T is
// written to memory, then every row is traversed again by a top-k or a top-p rule.  These
// kernels exist to measure what on-the-fly routing avoids; the forward pass never uses them.
//
//   proxy_map_kernel   s_hat[bh][i][j], f32, 64 x 64 output tiles on the f32 matrix instructions
//   topk_kernel        k largest proxies of a row: binary search for the k-th largest order-preserving key,
//                      ties to the lower key-block index
//   topp_kernel        shortest decreasing prefix of Softmax(s_hat_i) with mass >= p: binary search for the
//                      smallest kept key, by the mass above it
//
// Top-k and top-p give a row to one wave, with the row's keys in registers (lane l holds the blocks l + 64 i), so
// that a count is a ballot, the mask words are the ballots themselves and nothing waits at a barrier.
#include "sol_attn_internal.h"

#include <cmath>

namespace sol {
namespace {

// Order-preserving map of a float to an unsigned key (larger float -> larger key).
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// s_hat[bh][i][j] = scale * Qbar[bh][i] . Kbar[bh][j], j < NKr.  grid (ceil(NKr/64),
// ceil(NQ/64), BH), 256 threads: a wave owns 32 x 32 outputs, queries on the rows of
// v_mfma_f32_32x32x2_f32 and keys on its lanes, so every accumulator register is stored as two runs of 32
// consecutive j.  The lane halves of the instruction's k dimension hold d = 8u + 4hh + e in step 4u + e: a
// lane's operands of four steps are 16 consecutive bytes.  Bound by latency (one round of loads, d/2 MFMAs,
// the stores); at 12 x 256 x 512 x 128 it takes 12 us, 24 us with 4 x 4 outputs a thread from LDS.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void proxy_map_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar,
                                                        float* __restrict__ shat, int NQ, int NK, int NKr, float scale) {
    constexpr int NU = D / 8;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r32 = lane & 31, hh = lane >> 5;
    const int j = blockIdx.x * 64 + 32 * (wave & 1) + r32, i0 = blockIdx.y * 64 + 32 * (wave >> 1), bh = blockIdx.z;
    const float* qp = qbar + ((size_t)bh * NQ + min(i0 + r32, NQ - 1)) * D + 4 * hh;
    const float* kp = kbar + ((size_t)bh * NK + min(j, NKr - 1)) * D + 4 * hh;
    f32x4 qv[NU], kv[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        qv[u] = *reinterpret_cast<const f32x4*>(qp + 8 * u);
        kv[u] = *reinterpret_cast<const f32x4*>(kp + 8 * u);
    }
    f32x16 acc[2] = {f32x16{}, f32x16{}};   // two chains
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(qv[u][e], kv[u][e], acc[e & 1], 0, 0, 0);
    if (j >= NKr) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + 8 * (r >> 2) + 4 * hh + (r & 3);
        if (i < NQ) shat[((size_t)bh * NQ + i) * NKr + j] = scale * (acc[0][r] + acc[1][r]);
    }
}

// Order-preserving keys of the row's entries j0 + lane + 64 i; 0, below every key, past the row's end.
template <int KPL>
__device__ __forceinline__ void load_keys(const float* __restrict__ row, int NKr, int j0, uint32_t (&key)[KPL]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int j = j0 + lane + 64 * i;
        key[i] = j < NKr ? order_key(row[j]) : 0u;
    }
}

__device__ __forceinline__ void store_words(uint32_t* __restrict__ words, int MW, int i, uint64_t bits) {
    const int lane = threadIdx.x & 63;
    if (lane < 2 && 2 * i + lane < MW) words[2 * i + lane] = (uint32_t)(bits >> (32 * lane));
}

// Lanes below this one whose bit is set.
__device__ __forceinline__ int bits_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---------------------------------------------------------------------------
// Top-k of each row.  WPR waves per row (1, or all four of a workgroup), KPL keys a lane (64 KPL WPR >= NKr), wave w
// holding the entries from 64 KPL w on.  The largest K with at least k keys >= K is built bit by bit; keys above
// K are kept, and of the keys equal to K the lowest indices until k are kept.  The search stops at a K with
// exactly k keys >= K.  3,072 rows of 512: 9 us, against 75 us with a workgroup per row and a radix select in
// LDS whose digit scan ran on one thread.  Rows past TOPK_ROW4 entries take four waves: see launch_topk.
// ---------------------------------------------------------------------------
template <int KPL, int WPR>
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ shat, uint32_t* __restrict__ mask,
                                                   long long rows, int NKr, int MW, int k) {
    static_assert(WPR == 1 || WPR == 4, "a wave or a workgroup per row");
    __shared__ int part[2][4];
    const int wave = threadIdx.x >> 6, j0 = WPR == 1 ? 0 : wave * 64 * KPL;
    const long long r = (long long)blockIdx.x * (4 / WPR) + (WPR == 1 ? wave : 0);
    if (r >= rows) return;
    uint32_t key[KPL];
    load_keys<KPL>(shat + r * NKr, NKr, j0, key);
    // Sum over the row's waves; `before` receives the sum over the waves before this one.  The two sets of partial
    // sums alternate, so one barrier per call is enough.
    int turn = 0;
    auto row_sum = [&](int v, int* before) __attribute__((always_inline)) -> int {
        if constexpr (WPR == 1) {
            if (before) *before = 0;
            return v;
        } else {
            turn ^= 1;
            if ((threadIdx.x & 63) == 0) part[turn][wave] = v;
            __syncthreads();
            int sum = 0, pre = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int x = part[turn][w];
                if (w < wave) pre += x;
                sum += x;
            }
            if (before) *before = __builtin_amdgcn_readfirstlane(pre);
            return __builtin_amdgcn_readfirstlane(sum);   // the same in every wave: uniform control flow
        }
    };
    uint32_t kth = 0u;
    int above = -1;   // keys > kth, once known to be needed
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand = kth | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) cnt += __popcll(__ballot(key[i] >= cand));
        cnt = row_sum(cnt, nullptr);
        if (cnt >= k) kth = cand;
        if (cnt == k) {
            above = 0;   // exactly k keys >= kth: every one equal to it is kept too
            break;
        }
    }
    int take_eq = k;     // how many of the keys equal to kth are kept
    if (above < 0) {
        above = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) above += __popcll(__ballot(key[i] > kth));
        take_eq = k - row_sum(above, nullptr);
    }
    uint32_t* words = mask + r * MW;
    // Should kth be 0, the padding's keys equal it too, but they come last and take_eq entries of the row do before them.
    int seen = 0;
    if constexpr (WPR > 1) {
        int mine = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) mine += __popcll(__ballot(key[i] == kth));
        row_sum(mine, &seen);
    }
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const bool is_eq = key[i] == kth;
        const uint64_t eq = __ballot(is_eq);
        store_words(words, MW, j0 / 64 + i, __ballot(key[i] > kth || (is_eq && seen + bits_below(eq) < take_eq)));
        seen += __popcll(eq);
    }
}

// Sum over the wave, the same value in every lane: quad and row rotations (DPP), then half and quarter swaps, all on
// the VALU.
__device__ __forceinline__ float wave_sum(float x) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));    // lane ^ 1
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));    // lane ^ 2
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, false));   // rotate by 4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false));   // rotate by 8
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// ---------------------------------------------------------------------------
// Top-p of each row.  A wave per row, KPL keys a lane.  In decreasing order (equal proxies by increasing index) an
// entry is kept while the mass before it, of the weights exp(s - s_max), is below p times the total.  The mass
// above a key falls as the key grows, so the kept entries are those with keys >= c, the smallest key whose mass
// above is below the limit: c is built bit by bit from sums over the lanes' weights (a sum over fewer
// terms in the same order is never larger, so the search is consistent), and among the entries equal to c the
// first few are kept.  3,072 rows of 512: 13 us, against 37 us with a bitonic sort and a prefix sum.
// ---------------------------------------------------------------------------
template <int KPL>
__global__ __launch_bounds__(256) void topp_kernel(const float* __restrict__ shat, uint32_t* __restrict__ mask,
                                                   long long rows, int NKr, int MW, float p) {
    const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float* row = shat + r * NKr;
    const int lane = threadIdx.x & 63;
    uint32_t key[KPL];
    load_keys<KPL>(row, NKr, 0, key);
    uint32_t kmax = 0u;
#pragma unroll
    for (int i = 0; i < KPL; ++i) kmax = max(kmax, key[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
    const float smax = __uint_as_float((kmax & 0x80000000u) ? (kmax & 0x7FFFFFFFu) : ~kmax);   // inverse of order_key
    float w[KPL], part = 0.f;
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int j = lane + 64 * i;
        w[i] = j < NKr ? __expf(row[j] - smax) : 0.f;
        part += w[i];
    }
    const float limit = p * wave_sum(part);
    auto mass_above = [&](uint32_t c) __attribute__((always_inline)) -> float {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < KPL; ++i) m += key[i] > c ? w[i] : 0.f;
        return wave_sum(m);
    };
    uint32_t* words = mask + r * MW;
    // A row with a proxy of +inf or not a number, or with -inf throughout, has no softmax: no block is kept.  The test
    // is on the limit's bits (positive and finite otherwise), since comparisons assume numbers here.
    if (__float_as_uint(limit) - 1u >= 0x7F7FFFFFu) {
        for (int w0 = lane; w0 < MW; w0 += 64) words[w0] = 0u;
        return;
    }
    uint32_t low = 0u;   // the mass above `low` reaches the limit (above 0 it is the total, and p <= 1)
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand = low | (1u << bit);
        if (!(mass_above(cand) < limit)) low = cand;
    }
    const uint32_t c = low + 1u;   // the smallest value whose mass above is below the limit
    const float above = mass_above(c);
    int seen = 0;
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const bool is_eq = key[i] == c;
        const uint64_t eq = __ballot(is_eq);
        store_words(words, MW, i,
                    __ballot(key[i] > c || (is_eq && above + (float)(seen + bits_below(eq)) * w[i] < limit)));
        seen += __popcll(eq);
    }
}

// Keys per lane: the smallest power of two (at least 4) that covers the row.  Top-k rows of more than TOPK_ROW4
// entries are dealt to four waves.
constexpr int TOPK_ROW4 = 2048;
template <int KPL>
void launch_topk(const float* shat, uint32_t* mask, long long rows, int NKr, int MW, int k, hipStream_t st) {
    if constexpr (KPL < 32) {
        if (NKr > 64 * KPL) return launch_topk<2 * KPL>(shat, mask, rows, NKr, MW, k, st);
    }
    if (NKr > TOPK_ROW4) {
        if (NKr <= 4096) topk_kernel<16, 4><<<dim3((unsigned)rows), dim3(256), 0, st>>>(shat, mask, rows, NKr, MW, k);
        else topk_kernel<32, 4><<<dim3((unsigned)rows), dim3(256), 0, st>>>(shat, mask, rows, NKr, MW, k);
        return;
    }
    topk_kernel<KPL, 1><<<dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st>>>(shat, mask, rows, NKr, MW, k);
}
template <int KPL>
void launch_topp(const float* shat, uint32_t* mask, long long rows, int NKr, int MW, float p, hipStream_t st) {
    if constexpr (KPL < 64) {
        if (NKr > 64 * KPL) return launch_topp<2 * KPL>(shat, mask, rows, NKr, MW, p, st);
    }
    topp_kernel<KPL><<<dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st>>>(shat, mask, rows, NKr, MW, p);
}

}  // namespace

hipError_t launch_route_materialized(const float* qbar, const float* kbar, float* shat, uint32_t* mask, int BH, int NQ,
                                     int NK, int NKr, int d, int rule, float param, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)d);
    const dim3 g((NKr + 63) / 64, (NQ + 63) / 64, BH);
    if (d == 128) proxy_map_kernel<128><<<g, dim3(256), 0, st>>>(qbar, kbar, shat, NQ, NK, NKr, scale);
    else proxy_map_kernel<64><<<g, dim3(256), 0, st>>>(qbar, kbar, shat, NQ, NK, NKr, scale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int MW = (NKr + 31) / 32;
    const long long rows = (long long)BH * NQ;
    if (rule == 0) launch_topk<4>(shat, mask, rows, NKr, MW, (int)param, st);
    else launch_topp<4>(shat, mask, rows, NKr, MW, param, st);
    return hipGetLastError();
}

}  // namespace sol
