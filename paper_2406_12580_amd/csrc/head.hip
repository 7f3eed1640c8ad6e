// The prediction head's three products (logits = h E^T, dE = dlogits^T h, dh = dlogits E)
// in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums).
//
//   C[i][j] = sum_k A(i, k) B(j, k)
//
// An operand's element (r, k) is at r * ld + k (k contiguous) or at k * ld + r.  Operands
// go from memory straight into MFMA registers, without LDS: a lane holds row lane % 32 of
// its operand, and since both operands may take the contraction in any common order, half
// h of the wave takes k = k0 + 8 h .. + 7 of every 16, which is two 16-byte loads where k
// is contiguous; where r is, 32 lanes read 128 consecutive bytes.
//
// Work decomposition.  A workgroup of 8 waves; WK = 1: each wave has its own 32 x 32 NJ
// tile (logits, whose contraction is D); WK = 8: the waves split the contraction of one
// tile into ranges, whose sums meet in LDS and are added in range order (the gradients,
// whose outputs are few tiles: V / 32 and B / 32 of them with contractions over B and V).
//
// Measured at B = 2048, V = 3416, D = 64 (0.9 GFLOP each, 6 us at the fp32 matrix rate;
// logits 28 MB): logits 25 us, dE 34 us, dh 18 us, bound by the latency of operands that
// come straight from L2 and by the tiles there are (107 workgroups for dE); the
// library's fp32 products took 32, 105 (27 workgroups, each over all 2048 rows) and
// 37 us.  At B = 200, V = 12000: 13, 12 and 15 us against 11, 8 and 650 us (dh with the
// whole contraction over V in a few workgroups).
#include "device_common.hpp"
#include "gemm.hpp"
#include "launch.hpp"

namespace recblr {
namespace head {

constexpr int NW = 8, NT = NW * kWave, KS = 16;  // waves, threads, k of a register buffer

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

struct Params {
    const float* a;
    const float* b;
    float* c;
    int64_t lda, ldb, ldc, I, J, K;
    int64_t jt;       // workgroups along J
    int64_t it;       // along I
    int64_t S;        // along K (WK > 1): each stores its own C, `part` floats apart
    int64_t part;
};

// Eight contraction steps of one lane's row: k .. k + 7.
template <bool KC>
__device__ __forceinline__ void load8(const float* p, int64_t ld, int64_t r, int64_t k,
                                      float (&v)[8]) {
    if constexpr (KC) {
        const float* const q = p + r * ld + k;
        const f4u x = *(const f4u*)q, y = *(const f4u*)(q + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = x[e];
            v[4 + e] = y[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[(k + e) * ld + r];
    }
}
// ... zero from kend on.
template <bool KC>
__device__ __forceinline__ void load8_tail(const float* p, int64_t ld, int64_t r, int64_t k,
                                           int64_t kend, float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
        v[e] = k + e < kend ? p[KC ? r * ld + k + e : (k + e) * ld + r] : 0.0f;
}

template <bool KA, bool KB, int WK, int NJ>
__global__ __launch_bounds__(NT) void head_kernel(Params P) {
    __shared__ float part[WK > 1 ? NW * NJ * 16 * kWave : 1];
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), half = lane >> 5;
    const int64_t bz = WK > 1 ? blockIdx.x / (P.jt * P.it) : 0;
    const int64_t bt = blockIdx.x - bz * (P.jt * P.it);
    const int64_t bi = bt / P.jt, bj = bt - bi * P.jt;
    const int64_t i0 = bi * 32;
    const int64_t j0 = (bj * (WK > 1 ? 1 : NW) + (WK > 1 ? 0 : w)) * (32 * NJ);
    if (j0 >= P.J) return;  // WK = 1 only: the whole wave, and no barrier follows
    // rows past the end read the last one: their results are not stored
    const int64_t ra = i0 + (lane & 31) < P.I ? i0 + (lane & 31) : P.I - 1;
    int64_t rb[NJ];
#pragma unroll
    for (int n = 0; n < NJ; ++n) {
        const int64_t j = j0 + 32 * n + (lane & 31);
        rb[n] = j < P.J ? j : P.J - 1;
    }
    const int64_t nr = WK > 1 ? WK * P.S : 1;
    const int64_t per = ((P.K + nr - 1) / nr + KS - 1) / KS * KS;
    const int64_t kb = WK > 1 ? (bz * WK + w) * per : 0;
    const int64_t ke = kb + per < P.K ? kb + per : P.K;
    f16v acc[NJ];
#pragma unroll
    for (int n = 0; n < NJ; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.0f;
    float a[2][8], b[2][NJ][8];
    auto load = [&](int s, int64_t k) {
        load8<KA>(P.a, P.lda, ra, k + 8 * half, a[s]);
#pragma unroll
        for (int n = 0; n < NJ; ++n) load8<KB>(P.b, P.ldb, rb[n], k + 8 * half, b[s][n]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int s) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int n = 0; n < NJ; ++n)
                acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s][e], b[s][n][e], acc[n], 0, 0, 0);
    };
    // whole groups, the next one's loads in flight (past the last one: that one again)
    const int64_t full = kb < ke ? (ke - kb) / KS : 0;
    auto at = [&](int64_t g) { return kb + (g < full ? g : full - 1) * KS; };
    if (full > 0) load(0, kb);
    for (int64_t g = 0; g < full; g += 2) {
        load(1, at(g + 1));
        mul(0);
        load(0, at(g + 2));
        if (g + 1 < full) mul(1);
    }
    if (kb + full * KS < ke) {
        const int64_t k = kb + full * KS + 8 * half;
        load8_tail<KA>(P.a, P.lda, ra, k, ke, a[0]);
#pragma unroll
        for (int n = 0; n < NJ; ++n) load8_tail<KB>(P.b, P.ldb, rb[n], k, ke, b[0][n]);
        mul(0);
    }
    // accumulator v of lane: row 8 (v / 4) + 4 half + v % 4, column lane % 32
    if constexpr (WK == 1) {
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
            const int64_t j = j0 + 32 * n + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t i = i0 + 8 * (v / 4) + 4 * half + (v & 3);
                if (i < P.I && j < P.J) P.c[i * P.ldc + j] = acc[n][v];
            }
        }
    } else {
#pragma unroll
        for (int n = 0; n < NJ; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                part[((w * NJ + n) * 16 + v) * kWave + lane] = acc[n][v];
        __syncthreads();
        // wave w sums accumulators 2 w and 2 w + 1 of every block
#pragma unroll
        for (int n = 0; n < NJ; ++n)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int v = 2 * w + u;
                float s = part[(n * 16 + v) * kWave + lane];
#pragma unroll
                for (int q = 1; q < NW; ++q) s += part[((q * NJ + n) * 16 + v) * kWave + lane];
                const int64_t i = i0 + 8 * (v / 4) + 4 * half + (v & 3);
                const int64_t j = j0 + 32 * n + (lane & 31);
                if (i < P.I && j < P.J) P.c[bz * P.part + i * P.ldc + j] = s;
            }
    }
}

int64_t ceil_div(int64_t n, int64_t d) { return (n + d - 1) / d; }

template <bool KA, bool KB, int WK, int NJ>
hipError_t launch(Params P, hipStream_t stream) {
    P.jt = ceil_div(P.J, 32 * NJ * (WK > 1 ? 1 : NW));
    P.it = ceil_div(P.I, 32);
    const int64_t n = P.jt * P.it * P.S;
    if (n >= (int64_t)1 << 31) return hipErrorInvalidValue;
    hipLaunchKernelGGL((head_kernel<KA, KB, WK, NJ>), dim3((unsigned)n), dim3(NT), 0, stream, P);
    return hipGetLastError();
}

}  // namespace head

hipError_t launch_head_logits(const float* h, const float* E, float* logits, int64_t B, int64_t V,
                              int64_t D, hipStream_t stream) {
    return head::launch<true, true, 1, 2>(
        head::Params{h, E, logits, D, D, V, B, V, D, 0, 0, 1, 0}, stream);
}
hipError_t launch_head_dE(const float* dlogits, const float* h, float* dE, int64_t B, int64_t V,
                          int64_t D, hipStream_t stream) {
    return head::launch<false, false, head::NW, 2>(
        head::Params{dlogits, h, dE, V, D, D, V, D, B, 0, 0, 1, 0}, stream);
}
hipError_t launch_head_dh(const float* dlogits, const float* E, float* dh, int64_t B, int64_t V,
                          int64_t D, float* ws, hipStream_t stream) {
    // Few tiles: the contraction over V split over workgroups as well, at least 64 items a
    // wave, and their parts summed by a second launch (B = 200, V = 12000, D = 64: 79 us
    // with 14 workgroups).
    const int64_t tiles = head::ceil_div(B, 32) * (D / 32);
    int64_t S = 256 / tiles;
    if (S > V / (64 * head::NW)) S = V / (64 * head::NW);
    if (S < 2) S = 1;
    const hipError_t e = head::launch<true, false, head::NW, 1>(
        head::Params{dlogits, E, S > 1 ? ws : dh, V, D, D, B, D, V, 0, 0, S, B * D}, stream);
    if (e != hipSuccess || S == 1) return e;
    return launch_colsum(ws, S, B * D, dh, nullptr, stream);  // S <= 256: no workspace
}

}  // namespace recblr
