// The linear sub-layers of the model for rows of D = 64: the position-wise
// feed-forward one, and (below) the projections around the gated layer.
//
// Feed-forward, Q = SiLU(X W1^T + b1) W2^T
// + b2 with D = 64 inputs and F = 256 hidden units (fp32), forward and backward in
// one kernel each: of the hidden tensors (F wide, four times the rows' size) only
// A = X W1^T + b1 is stored, by the forward for the backward; SiLU(A) and its
// gradient exist in registers only.
//
// Work decomposition.  A workgroup of 8 waves walks tiles of 32 rows; wave w owns
// hidden units 32 w .. 32 w + 31 for the whole launch, with its parts of the weights
// in registers.  Rows are staged in LDS once a tile as bf16 planes.  A product's
// accumulator holds 4-element runs of one index in each lane, which is an operand
// of the next product once that one's contraction is taken in the same (permuted)
// order, so A -> SiLU -> product stays inside the wave:
//   forward   A^T[f][row] = W1 X^T, then Q^T[d][row] += W2 SiLU(A)^T over the wave's f;
//   backward  dP[row][f] = dQ W2, dA = dP SiLU'(A), then dW1^T[d][f] += X^T dA and
//             dW2[d][f] += dQ^T SiLU(A) over the rows (accumulators in registers for
//             the whole range of rows); dX^T[d][row] = W1^T dA^T contracts f, for which
//             dA is transposed through the wave's own LDS.
// The 8 waves' parts of Q or dX meet in LDS, summed in a fixed order.
//
// Arithmetic.  Products whose results go on through the model keep fp32 accuracy:
// operands split into three bf16 planes (24 bits), the six products of weight 2^-18
// and more of the full one, accumulated in fp32.  Weight gradients take the 3-term
// split.  (An infinite operand gives NaN, its lower planes being inf - inf; what follows
// each of these products is a LayerNorm, which makes NaN of an infinity too.)
//
// Measured at M = 409600: forward 205 us (A written, 0.63 GB: 122 us at copy speed;
// matrix cores busy 80 us), backward 255 us (0.84 GB with dX read and written: 162 us;
// matrix cores 123 us, vector instructions about as long, two waves a SIMD in step
// with each other).  Layer by layer, with the hidden tensors written and read between
// four linear kernels and two weight-gradient kernels: 326 and 630 us.
#include "device_common.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"
#include "wave_tile.hpp"
#include "gemm.hpp"

namespace recblr {
namespace ffn {

using namespace wtile;

constexpr int D = 64, F = 256, TR = 32, NW = 8, NT = NW * kWave;
constexpr int kPlane = TR * D * 2;                 // bytes of a plane of a row tile
constexpr int kExch = NW * 8 * kWave * 16;         // parts of Q or dX, fp32
constexpr int kTrans = 32 * 32 * 2;                // a plane of a wave's dA block
constexpr int64_t kPart = kFfnGrads;               // [dW1 | db1 | dW2 | db2]
static_assert(kPart == 2 * F * D + F + D);

// Chunk j (16 bytes of 128) of row r of a plane at j ^ swz(r): 16 rows of one chunk,
// and 4 rows of 4 chunks, land on distinct banks.
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 1) << 2 | ((r >> 2) & 3); }

// Planes 0 (high) to 2 of both: the products above 2^-27 of the full one.
__device__ __forceinline__ f16v mma6(const b8 (&a)[3], const b8 (&b)[3], f16v c) {
    c = mfma(a[1], b[1], c);
    c = mfma(a[0], b[2], c);
    c = mfma(a[2], b[0], c);
    c = mfma(a[0], b[1], c);
    c = mfma(a[1], b[0], c);
    return mfma(a[0], b[0], c);
}
__device__ __forceinline__ f16v mma3(const b8 (&a)[2], b8 b0, b8 b1, f16v c) {
    c = mfma(a[0], b1, c);
    c = mfma(a[1], b0, c);
    return mfma(a[0], b0, c);
}

// a and b as bf16 pairs: out[0] + out[1] + out[2] to 2^-26 of the value.
struct Tri {
    uint32_t p[3];
};
__device__ __forceinline__ Tri split3(float a, float b) {
    Tri t;
    t.p[0] = bf16_pair(a, b);
    a -= __uint_as_float(t.p[0] << 16);
    b -= __uint_as_float(t.p[0] & 0xffff0000u);
    t.p[1] = bf16_pair(a, b);
    t.p[2] = bf16_pair(a - __uint_as_float(t.p[1] << 16),
                               b - __uint_as_float(t.p[1] & 0xffff0000u));
    return t;
}
// Eight values as three operand planes.
__device__ __forceinline__ void planes3(const float (&v)[8], b8 (&out)[3]) {
    uint32_t u[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const Tri t = split3(v[2 * i], v[2 * i + 1]);
#pragma unroll
        for (int p = 0; p < 3; ++p) u[p][i] = t.p[p];
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
        out[p] = __builtin_bit_cast(b8, u4v{u[p][0], u[p][1], u[p][2], u[p][3]});
}

// One thread's quad of a row tile (row tid / 16, inputs 4 (tid % 16) ..).
__device__ __forceinline__ u4v fetch_quad(const float* p, int64_t m, int64_t end, int tid) {
    const int64_t n = end - m < TR ? end - m : TR;
    return __builtin_amdgcn_raw_buffer_load_b128(
        rsrc(p + m * D, n > 0 ? (uint32_t)(n * D * 4) : 0u), tid * 16, 0, 0);
}
// ... into NP planes at dst (rows past the end were read as zero).
template <int NP>
__device__ __forceinline__ void stage_quad(char* dst, u4v q, int tid) {
    const int r = tid >> 4, c = tid & 15;
    char* const at = dst + r * (D * 2) + (((c >> 1) ^ swz(r)) << 4) + (c & 1) * 8;
    const Tri a = split3(__uint_as_float(q[0]), __uint_as_float(q[1]));
    const Tri b = split3(__uint_as_float(q[2]), __uint_as_float(q[3]));
#pragma unroll
    for (int p = 0; p < NP; ++p) *(u2v*)(at + p * kPlane) = u2v{a.p[p], b.p[p]};
}
// The three planes of a row fragment: row lane % 32, inputs 16 ks + 8 (lane / 32) ..
__device__ __forceinline__ void row_frag(const char* src, int ks, int ln, b8 (&f)[3]) {
    const int r = ln & 31;
    const int base = r * (D * 2) + (((ln >> 5) ^ swz(r)) << 4);
#pragma unroll
    for (int p = 0; p < 3; ++p) f[p] = *(const b8*)(src + (base ^ (ks << 5)) + p * kPlane);
}

// The two planes of a transposed fragment: input 32 db + lane % 32, k = rows of the half
// tile s in the order of an accumulator's (16 s + 4 h .. + 3, 16 s + 8 + 4 h .. + 3).
__device__ __forceinline__ void col_frag(const char* src, int db, int s, int ln, b8 (&f)[2]) {
    const int r0 = 4 * (ln >> 5) + ((ln >> 2) & 3), c0 = 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
    const int tb = r0 * (D * 2) + (((c0 >> 3) ^ swz(r0)) << 4) + (c0 & 7) * 2;
    const int o = tb ^ (db << 6);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int k = s * (16 * D * 2) + p * kPlane;
        f[p] = tr_pair(src + o + k, src + (o ^ 32) + k + 8 * D * 2);
    }
}
// A wave's [32 units][32 rows] block through its own LDS: written by half tiles (lane:
// unit, rows as col_frag's), read as an operand (lane: row, k = units 16 s + 8 h ..).
__device__ __forceinline__ void put_block(char* tp, int s, int ln, const b8 (&v)[3]) {
    const int u = ln & 31;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const u4v d4 = __builtin_bit_cast(u4v, v[p]);
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *(u2v*)(tp + p * kTrans + u * 64 + (((4 * s + 2 * k + (ln >> 5)) ^ (u >> 2)) << 3)) =
                u2v{d4[2 * k], d4[2 * k + 1]};
    }
}
__device__ __forceinline__ void get_block(const char* tp, int s, int ln, b8 (&f)[3]) {
    const int ub = (8 * (ln >> 5) + ((ln >> 2) & 3)) * 64 +
                   (((4 * ((ln >> 4) & 1) + (ln & 3)) ^ (2 * (ln >> 5))) << 3);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const char* const base = tp + p * kTrans + s * 1024;
        f[p] = tr_pair(base + (ub ^ (s << 5)), base + (ub ^ (s << 5) ^ 8) + 256);
    }
}
// Eight values as two operand planes.
__device__ __forceinline__ void planes2(const float (&v)[8], b8 (&out)[2]) {
    uint32_t u[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const fastmm::u2v p = fastmm::split2(v[2 * i], v[2 * i + 1]);
        u[0][i] = p.x;
        u[1][i] = p.y;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
        out[p] = __builtin_bit_cast(b8, u4v{u[p][0], u[p][1], u[p][2], u[p][3]});
}
// A wave's part of [64][32 rows] (two accumulators) into the exchange, and piece
// `piece` of 8 (rows lane % 32, columns 8 piece + 4 h ..) summed over the 8 waves.
__device__ __forceinline__ void put_part(char* ex, int w, int ln, const f16v (&o)[2]) {
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f4*)(ex + ((w * 8 + db * 4 + q) * kWave + ln) * 16) =
                f4{o[db][4 * q], o[db][4 * q + 1], o[db][4 * q + 2], o[db][4 * q + 3]};
}
__device__ __forceinline__ f4 sum_parts(const char* ex, int piece, int ln, f4 sum) {
#pragma unroll
    for (int k = 0; k < NW; ++k) sum += *(const f4*)(ex + ((k * 8 + piece) * kWave + ln) * 16);
    return sum;
}
// Byte offset of that piece in a row tile.
__device__ __forceinline__ uint32_t dx_off(int ln, int piece) {
    return (uint32_t)((ln & 31) * D + 8 * piece + 4 * (ln >> 5)) * 4;
}
__device__ __forceinline__ u4v bits4(f4 v) { return __builtin_bit_cast(u4v, v); }

struct FwdParams {
    const float* x;
    const float* w1;
    const float* b1;
    const float* w2;
    const float* b2;
    float* a;
    float* q;
    int64_t M;
};

__global__ __launch_bounds__(NT, 2) void ffn_fwd_kernel(FwdParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const xp = smem;                    // [2][3 planes]
    char* const exch = smem + 2 * 3 * kPlane; // [2]
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), h = lane >> 5;
    const int64_t tiles = (P.M + TR - 1) / TR;
    int64_t t = blockIdx.x;
    if (t >= tiles) return;

    b8 w1[4][3], w2[2][2][3];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {  // unit 32 w + lane % 32, inputs 16 ks + 8 h ..
        const float* const p = P.w1 + (32 * w + (lane & 31)) * D + 16 * ks + 8 * h;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[e];
        planes3(v, w1[ks]);
    }
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int s = 0; s < 2; ++s) {  // output 32 db + lane % 32, units in A's order
            const float* const p = P.w2 + (32 * db + (lane & 31)) * F + 32 * w + 16 * s + 4 * h;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = p[e + (e & 4)];
            planes3(v, w2[db][s]);
        }
    float b1[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) b1[v] = P.b1[32 * w + 8 * (v / 4) + 4 * h + (v & 3)];
    const f4 b2 = *(const f4*)(P.b2 + 8 * w + 4 * h);  // this wave's piece of Q

    stage_quad<3>(xp, fetch_quad(P.x, t * TR, P.M, threadIdx.x), threadIdx.x);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    lds_barrier();
    for (int par = 0; t < tiles; t += gridDim.x, par ^= 1) {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const int64_t m = t * TR;
        const u4v next = fetch_quad(P.x, m + gridDim.x * TR, P.M, tid);
        const char* const src = xp + par * 3 * kPlane;
        f16v a;
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = b1[v];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            b8 f[3];
            row_frag(src, ks, ln, f);
            a = mma6(w1[ks], f, a);
        }
        const int64_t n = P.M - m < TR ? P.M - m : TR;
        const __amdgpu_buffer_rsrc_t ars = rsrc(P.a + m * F, (uint32_t)(n * F * 4));
        const uint32_t ao = (uint32_t)((ln & 31) * F + 32 * w + 4 * (ln >> 5)) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(
                u4v{__float_as_uint(a[4 * q]), __float_as_uint(a[4 * q + 1]),
                    __float_as_uint(a[4 * q + 2]), __float_as_uint(a[4 * q + 3])},
                ars, ao + 32 * q, 0, 0);
        f16v y[2];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) y[db][v] = 0.0f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = a[8 * s + e] * sigmoid(a[8 * s + e]);
            b8 p[3];
            planes3(v, p);
#pragma unroll
            for (int db = 0; db < 2; ++db) y[db] = mma6(w2[db][s], p, y[db]);
        }
        char* const ex = exch + par * kExch;
        put_part(ex, w, ln, y);
        stage_quad<3>(xp + (par ^ 1) * 3 * kPlane, next, tid);
        lds_barrier();
        const f4 sum = sum_parts(ex, w, ln, b2);
        const __amdgpu_buffer_rsrc_t qrs = rsrc(P.q + m * D, (uint32_t)(n * D * 4));
        __builtin_amdgcn_raw_buffer_store_b128(
            bits4(sum), qrs, dx_off(ln, w), 0, 0);
    }
}

struct BwdParams {
    const float* x;
    const float* dq;
    const float* a;
    const float* w1;
    const float* w2;
    float* dx;         // dx += ...
    float* part;       // [ranges][kPart]
    int64_t M, ranges, rows;
};

__global__ __launch_bounds__(NT, 2) void ffn_bwd_kernel(BwdParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const qp = smem;                          // dQ [2][3 planes]
    char* const xp = qp + 2 * 3 * kPlane;           // X [2][2 planes]
    char* const trans = xp + 2 * 2 * kPlane;        // dA [8 waves][3 planes][32 f][32 rows]
    char* const exch = trans + NW * 3 * kTrans;
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), h = lane >> 5;
    const int64_t row0 = blockIdx.x * P.rows;
    const int64_t row1 = row0 + P.rows < P.M ? row0 + P.rows : P.M;
    if (row0 >= row1) return;

    b8 w2[4][3], w1t[2][2][3];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {  // unit 32 w + lane % 32, outputs 16 ks + 8 h ..
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = P.w2[(16 * ks + 8 * h + e) * F + 32 * w + (lane & 31)];
        planes3(v, w2[ks]);
    }
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int s = 0; s < 2; ++s) {  // input 32 db + lane % 32, units 16 s + 8 h ..
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = P.w1[(32 * w + 16 * s + 8 * h + e) * D + 32 * db + (lane & 31)];
            planes3(v, w1t[db][s]);
        }
    f16v dw1[2], dw2[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) dw1[db][v] = dw2[db][v] = 0.0f;
    float db1 = 0.0f;
    f4 db2 = f4{0.0f, 0.0f, 0.0f, 0.0f};

    float a[16];  // of rows 8 (v / 4) + 4 h + v % 4, unit 32 w + lane % 32
    auto load_a = [&](int64_t m, int ln) {
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const __amdgpu_buffer_rsrc_t rs = rsrc(P.a + m * F, n > 0 ? (uint32_t)(n * F * 4) : 0u);
        const uint32_t o = (uint32_t)(4 * (ln >> 5) * F + 32 * w + (ln & 31)) * 4;
#pragma unroll
        for (int v = 0; v < 16; ++v)
            a[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rs, o, (8 * (v / 4) + (v & 3)) * F * 4, 0));
    };
    auto stage = [&](int par, u4v xq, u4v dqq, int tid) {
        stage_quad<3>(qp + par * 3 * kPlane, dqq, tid);
        stage_quad<2>(xp + par * 2 * kPlane, xq, tid);
#pragma unroll
        for (int k = 0; k < 4; ++k) db2[k] += __uint_as_float(dqq[k]);
    };
    {
        const u4v dqq = fetch_quad(P.dq, row0, row1, threadIdx.x);
        const u4v xq = fetch_quad(P.x, row0, row1, threadIdx.x);
        stage(0, xq, dqq, threadIdx.x);
    }
    load_a(row0, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing pending enters the loop
    lds_barrier();
    int par = 0;
    char* const tp = trans + w * 3 * kTrans;
    for (int64_t m = row0; m < row1; m += TR, par ^= 1) {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const char* const dqs = qp + par * 3 * kPlane;
        const char* const xs = xp + par * 2 * kPlane;
        // ---- dP[row][f]
        f16v dp;
#pragma unroll
        for (int v = 0; v < 16; ++v) dp[v] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            b8 f[3];
            row_frag(dqs, ks, ln, f);
            dp = mma6(f, w2[ks], dp);
        }
        // ---- SiLU and its gradient, then the weight gradients, 16 rows at a time.
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float act[8], da[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float av = a[8 * s + e], sg = sigmoid(av);
                act[e] = av * sg;
                da[e] = dp[8 * s + e] * (sg * fmaf(av, 1.0f - sg, 1.0f));
                db1 += da[e];
            }
            b8 ap[2], dap[3];
            planes3(da, dap);
            planes2(act, ap);
            put_block(tp, s, ln, dap);
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                b8 xf[2], qf[2];
                col_frag(dqs, db, s, ln, qf);
                col_frag(xs, db, s, ln, xf);
                dw2[db] = mma3(qf, ap[0], ap[1], dw2[db]);
                dw1[db] = mma3(xf, dap[0], dap[1], dw1[db]);
            }
        }
        load_a(m + TR, ln);
        const u4v dqn = fetch_quad(P.dq, m + TR, row1, tid);
        const u4v xn = fetch_quad(P.x, m + TR, row1, tid);
        const __amdgpu_buffer_rsrc_t drs = rsrc(P.dx + m * D, (uint32_t)(n * D * 4));
        const u4v dd = __builtin_amdgcn_raw_buffer_load_b128(drs, dx_off(ln, w), 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        wave_fence();  // get_block reads what other lanes put
        // ---- this wave's part of dX^T
        f16v o[2];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.0f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            b8 f[3];
            get_block(tp, s, fresh(lane), f);
#pragma unroll
            for (int db = 0; db < 2; ++db) o[db] = mma6(w1t[db][s], f, o[db]);
        }
        lds_barrier();  // the last tile's parts have been read
        put_part(exch, w, fresh(lane), o);
        stage(par ^ 1, xn, dqn, tid);
        lds_barrier();
        const int ls = fresh(lane);
        const f4 sum = sum_parts(exch, w, ls, __builtin_bit_cast(f4, dd));
        __builtin_amdgcn_raw_buffer_store_b128(bits4(sum), drs, dx_off(ls, w), 0, 0);
    }

    // ---- partial sums of this range
    float* const part = P.part + blockIdx.x * kPart;
    const int f = 32 * w + (lane & 31);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int d = 32 * db + 8 * q + 4 * h;
            *(f4*)(part + f * D + d) = f4{dw1[db][4 * q], dw1[db][4 * q + 1], dw1[db][4 * q + 2],
                                          dw1[db][4 * q + 3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) part[F * D + F + (d + e) * F + f] = dw2[db][4 * q + e];
        }
    db1 += __shfl_xor(db1, 32);
    if (h == 0) part[F * D + f] = db1;
    lds_barrier();  // the last parts have been read
    *(f4*)(exch + threadIdx.x * 16) = db2;
    lds_barrier();
    if (threadIdx.x < D) {
        float s = 0.0f;
        for (int r = 0; r < TR; ++r)
            s += *(const float*)(exch + (r * 16 + threadIdx.x / 4) * 16 + threadIdx.x % 4 * 4);
        part[2 * F * D + F + threadIdx.x] = s;
    }
}

// ---- the projections around the gated layer: Hx = X Wx^T + bx, Hz = X Wz^T + bz and
// O = y Wo^T + bo, with X and O 64 wide and Hx, Hz, y 128 wide (E).
// Each of their large tensors moves once: with linear kernels and weight-gradient
// kernels of their own the input side's backward read dHx and dHz twice and updated dx
// twice.  At M = 409600, before -> now (floor at copy speed): input side forward 180 ->
// 120 us (101), backward 328 -> 172 us (142); output side backward 171 -> 108 us (101).
constexpr int E = 128;
constexpr int64_t kInPart = kProjInGrads;    // [dWx | dbx | dWz | dbz]
constexpr int64_t kOutPart = kProjOutGrads;  // [dWo | dbo]
static_assert(kInPart == 2 * (E * D + E) && kOutPart == E * D + D);

struct InFwdParams {
    const float* x;
    const float* wx;
    const float* bx;
    const float* wz;
    const float* bz;
    float* hx;
    float* hz;
    int64_t M;
};

// Hx and Hz from one reading of X: ffn_fwd_kernel's first product, its waves' units
// those of Wx, then those of Wz.
__global__ __launch_bounds__(NT, 4) void proj_in_fwd_kernel(InFwdParams P) {
    __shared__ __attribute__((aligned(16))) char xp[2 * 3 * kPlane];
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), h = lane >> 5;
    const int64_t tiles = (P.M + TR - 1) / TR;
    int64_t t = blockIdx.x;
    if (t >= tiles) return;
    const int u0 = 32 * (w & 3);
    const float* const wt = w < 4 ? P.wx : P.wz;
    const float* const bt = w < 4 ? P.bx : P.bz;
    float* const out = w < 4 ? P.hx : P.hz;
    b8 w1[4][3];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const float* const p = wt + (u0 + (lane & 31)) * D + 16 * ks + 8 * h;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[e];
        planes3(v, w1[ks]);
    }
    float b1[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) b1[v] = bt[u0 + 8 * (v / 4) + 4 * h + (v & 3)];
    stage_quad<3>(xp, fetch_quad(P.x, t * TR, P.M, threadIdx.x), threadIdx.x);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    lds_barrier();
    for (int par = 0; t < tiles; t += gridDim.x, par ^= 1) {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const int64_t m = t * TR;
        const u4v next = fetch_quad(P.x, m + gridDim.x * TR, P.M, tid);
        f16v a;
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = b1[v];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            b8 f[3];
            row_frag(xp + par * 3 * kPlane, ks, ln, f);
            a = mma6(w1[ks], f, a);
        }
        const int64_t n = P.M - m < TR ? P.M - m : TR;
        const __amdgpu_buffer_rsrc_t rs = rsrc(out + m * E, (uint32_t)(n * E * 4));
        const uint32_t o = (uint32_t)((ln & 31) * E + u0 + 4 * (ln >> 5)) * 4;
        stage_quad<3>(xp + (par ^ 1) * 3 * kPlane, next, tid);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(
                bits4(f4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]}), rs, o + 32 * q, 0,
                0);
        lds_barrier();
    }
}

struct InBwdParams {
    const float* x;
    const float* dhx;
    const float* dhz;
    const float* wx;
    const float* wz;
    float* dx;    // dx += ...
    float* part;  // [ranges][kInPart]
    int64_t M, ranges, rows;
};

// Both data and both weight gradients of the input projections: ffn_bwd_kernel with
// its dA read (dHx for waves 0 to 3, dHz for 4 to 7) in place of formed.
__global__ __launch_bounds__(NT, 2) void proj_in_bwd_kernel(InBwdParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const xp = smem;                    // X [2][2 planes]
    char* const trans = xp + 2 * 2 * kPlane;  // [8 waves][3 planes][32 units][32 rows]
    char* const exch = trans + NW * 3 * kTrans;
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), h = lane >> 5;
    const int64_t row0 = blockIdx.x * P.rows;
    const int64_t row1 = row0 + P.rows < P.M ? row0 + P.rows : P.M;
    if (row0 >= row1) return;
    const int u0 = 32 * (w & 3);
    const float* const wt = w < 4 ? P.wx : P.wz;
    const float* const da_in = w < 4 ? P.dhx : P.dhz;

    b8 w1t[2][2][3];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int s = 0; s < 2; ++s) {  // input 32 db + lane % 32, units 16 s + 8 h ..
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = wt[(u0 + 16 * s + 8 * h + e) * D + 32 * db + (lane & 31)];
            planes3(v, w1t[db][s]);
        }
    f16v dw[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) dw[db][v] = 0.0f;
    float dbs = 0.0f;
    float a[16];  // of rows 8 (v / 4) + 4 h + v % 4, unit u0 + lane % 32
    auto load_a = [&](int64_t m, int ln) {
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const __amdgpu_buffer_rsrc_t rs = rsrc(da_in + m * E, n > 0 ? (uint32_t)(n * E * 4) : 0u);
        const uint32_t o = (uint32_t)(4 * (ln >> 5) * E + u0 + (ln & 31)) * 4;
#pragma unroll
        for (int v = 0; v < 16; ++v)
            a[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rs, o, (8 * (v / 4) + (v & 3)) * E * 4, 0));
    };
    stage_quad<2>(xp, fetch_quad(P.x, row0, row1, threadIdx.x), threadIdx.x);
    load_a(row0, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing pending enters the loop
    lds_barrier();
    int par = 0;
    char* const tp = trans + w * 3 * kTrans;
    for (int64_t m = row0; m < row1; m += TR, par ^= 1) {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const char* const xs = xp + par * 2 * kPlane;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float da[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                da[e] = a[8 * s + e];
                dbs += da[e];
            }
            b8 dap[3];
            planes3(da, dap);
            put_block(tp, s, ln, dap);
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                b8 xf[2];
                col_frag(xs, db, s, ln, xf);
                dw[db] = mma3(xf, dap[0], dap[1], dw[db]);
            }
        }
        load_a(m + TR, ln);
        const u4v xn = fetch_quad(P.x, m + TR, row1, tid);
        const __amdgpu_buffer_rsrc_t drs = rsrc(P.dx + m * D, (uint32_t)(n * D * 4));
        const u4v dd = __builtin_amdgcn_raw_buffer_load_b128(drs, dx_off(ln, w), 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        wave_fence();  // get_block reads what other lanes put
        f16v o[2];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.0f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            b8 f[3];
            get_block(tp, s, ln, f);
#pragma unroll
            for (int db = 0; db < 2; ++db) o[db] = mma6(w1t[db][s], f, o[db]);
        }
        lds_barrier();  // the last tile's parts have been read
        put_part(exch, w, ln, o);
        stage_quad<2>(xp + (par ^ 1) * 2 * kPlane, xn, tid);
        lds_barrier();
        const f4 sum = sum_parts(exch, w, ln, __builtin_bit_cast(f4, dd));
        __builtin_amdgcn_raw_buffer_store_b128(bits4(sum), drs, dx_off(ln, w), 0, 0);
    }
    float* const part = P.part + blockIdx.x * kInPart + (w >> 2) * (E * D + E);
    const int u = u0 + (lane & 31);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f4*)(part + u * D + 32 * db + 8 * q + 4 * h) =
                f4{dw[db][4 * q], dw[db][4 * q + 1], dw[db][4 * q + 2], dw[db][4 * q + 3]};
    dbs += __shfl_xor(dbs, 32);
    if (h == 0) part[E * D + u] = dbs;
}

struct OutBwdParams {
    const float* y;
    const float* dout;
    const float* w;
    float* dy;
    float* part;  // [ranges][kOutPart]
    int64_t M, ranges, rows;
};

constexpr int NTO = 256;  // 4 waves of 32 of the 128 inputs

// Data and weight gradients of the output projection: ffn_bwd_kernel's dP = dQ W2, here
// stored, and its dW2.
__global__ __launch_bounds__(NTO, 2) void proj_out_bwd_kernel(OutBwdParams P) {
    __shared__ __attribute__((aligned(16))) char qp[2 * 3 * kPlane];
    const int lane = threadIdx.x & (kWave - 1), w = wave_id(), h = lane >> 5;
    const int64_t row0 = blockIdx.x * P.rows;
    const int64_t row1 = row0 + P.rows < P.M ? row0 + P.rows : P.M;
    if (row0 >= row1) return;
    b8 wf[4][3];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {  // input 32 w + lane % 32, outputs 16 ks + 8 h ..
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = P.w[(16 * ks + 8 * h + e) * E + 32 * w + (lane & 31)];
        planes3(v, wf[ks]);
    }
    f16v dw[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) dw[db][v] = 0.0f;
    f4 dbo = f4{0.0f, 0.0f, 0.0f, 0.0f};
    float a[16];  // y of rows 8 (v / 4) + 4 h + v % 4, input 32 w + lane % 32
    auto load_a = [&](int64_t m, int ln) {
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const __amdgpu_buffer_rsrc_t rs = rsrc(P.y + m * E, n > 0 ? (uint32_t)(n * E * 4) : 0u);
        const uint32_t o = (uint32_t)(4 * (ln >> 5) * E + 32 * w + (ln & 31)) * 4;
#pragma unroll
        for (int v = 0; v < 16; ++v)
            a[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rs, o, (8 * (v / 4) + (v & 3)) * E * 4, 0));
    };
    auto stage = [&](int par, u4v q0, u4v q1, int tid) {
        stage_quad<3>(qp + par * 3 * kPlane, q0, tid);
        stage_quad<3>(qp + par * 3 * kPlane, q1, tid + NTO);
#pragma unroll
        for (int k = 0; k < 4; ++k) dbo[k] += __uint_as_float(q0[k]) + __uint_as_float(q1[k]);
    };
    {
        const u4v q0 = fetch_quad(P.dout, row0, row1, threadIdx.x);
        const u4v q1 = fetch_quad(P.dout, row0, row1, threadIdx.x + NTO);
        stage(0, q0, q1, threadIdx.x);
    }
    load_a(row0, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing pending enters the loop
    lds_barrier();
    int par = 0;
    for (int64_t m = row0; m < row1; m += TR, par ^= 1) {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const char* const qs = qp + par * 3 * kPlane;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = a[8 * s + e];
            b8 ap[2];
            planes2(v, ap);
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                b8 qf[2];
                col_frag(qs, db, s, ln, qf);
                dw[db] = mma3(qf, ap[0], ap[1], dw[db]);
            }
        }
        load_a(m + TR, ln);
        const u4v q0 = fetch_quad(P.dout, m + TR, row1, tid);
        const u4v q1 = fetch_quad(P.dout, m + TR, row1, tid + NTO);
        __builtin_amdgcn_sched_barrier(0);
        f16v dp;
#pragma unroll
        for (int v = 0; v < 16; ++v) dp[v] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            b8 f[3];
            row_frag(qs, ks, ln, f);
            dp = mma6(f, wf[ks], dp);
        }
        const __amdgpu_buffer_rsrc_t rs = rsrc(P.dy + m * E, (uint32_t)(n * E * 4));
        const uint32_t o = (uint32_t)(4 * (ln >> 5) * E + 32 * w + (ln & 31)) * 4;
        stage(par ^ 1, q0, q1, tid);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dp[v]), rs, o,
                                                  (8 * (v / 4) + (v & 3)) * E * 4, 0);
        lds_barrier();
    }
    float* const part = P.part + blockIdx.x * kOutPart;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            part[(32 * db + 8 * (v / 4) + 4 * h + (v & 3)) * E + 32 * w + (lane & 31)] = dw[db][v];
    *(f4*)(qp + threadIdx.x * 16) = dbo;  // free after the last barrier
    lds_barrier();
    if (threadIdx.x < D) {
        float s = 0.0f;
        for (int r = 0; r < NTO / 16; ++r)
            s += *(const float*)(qp + (r * 16 + threadIdx.x / 4) * 16 + threadIdx.x % 4 * 4);
        part[E * D + threadIdx.x] = s;
    }
}

constexpr int kInBwdSmem = 2 * 2 * kPlane + NW * 3 * kTrans + kExch;
constexpr int kFwdSmem = 2 * 3 * kPlane + 2 * kExch;
constexpr int kBwdSmem = 2 * 5 * kPlane + NW * 3 * kTrans + kExch;

// `most` workgroups (one or two per compute unit), a tile or more each: every range
// leaves a partial of its weight gradients to sum, but few rows in few ranges leave the
// chip idle (model step of 2000 rows, two layers: 437 us with at least 256 rows a range,
// 376 with 64, 371 with 32; 20000 rows, one layer: 411, 375 and 370 us).
constexpr int64_t kMinRows = TR;
void split(int64_t M, int64_t most, int64_t* ranges, int64_t* rows) {
    int64_t n = (M + kMinRows - 1) / kMinRows;
    n = n < most ? n : most;
    *rows = ((M + n - 1) / n + TR - 1) / TR * TR;
    *ranges = (M + *rows - 1) / *rows;
}

}  // namespace ffn

bool sublayers_fused_applies(int64_t M, int64_t D, std::initializer_list<const void*> ptrs) {
    uintptr_t a = 0;
    for (const void* p : ptrs) a |= (uintptr_t)p;
    return M > 0 && D == ffn::D && a % 16 == 0;
}

size_t sublayers_fused_workspace(int64_t M) {
    if (M <= 0) return 0;
    int64_t one, two, rows;
    ffn::split(M, 256, &one, &rows);
    ffn::split(M, 512, &two, &rows);
    const int64_t a = one * ffn::kPart, b = two * ffn::kOutPart;
    return (size_t)(a > b ? a : b) * sizeof(float);
}

size_t sublayers_fused_colsum(int64_t M) {
    if (M <= 0) return 0;
    int64_t one, two, rows;
    ffn::split(M, 256, &one, &rows);
    ffn::split(M, 512, &two, &rows);
    size_t w = colsum_workspace(one, ffn::kPart);
    if (colsum_workspace(one, ffn::kInPart) > w) w = colsum_workspace(one, ffn::kInPart);
    if (colsum_workspace(two, ffn::kOutPart) > w) w = colsum_workspace(two, ffn::kOutPart);
    return w;
}

hipError_t launch_ffn_forward(const float* x, const float* w1, const float* b1, const float* w2,
                              const float* b2, float* a, float* q, int64_t M, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    hipError_t e = allow_dynamic_lds((const void*)ffn::ffn_fwd_kernel, ffn::kFwdSmem, lds_set);
    if (e != hipSuccess) return e;
    const int64_t tiles = (M + ffn::TR - 1) / ffn::TR;
    const dim3 grid((unsigned)(tiles < 256 ? tiles : 256));
    hipLaunchKernelGGL(ffn::ffn_fwd_kernel, grid, dim3(ffn::NT), ffn::kFwdSmem, stream,
                       ffn::FwdParams{x, w1, b1, w2, b2, a, q, M});
    return hipGetLastError();
}

hipError_t launch_ffn_backward(const float* x, const float* dq, const float* a, const float* w1,
                               const float* w2, float* dx, float* grads, int64_t M, float* part,
                               void* colsum_ws, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    hipError_t e = allow_dynamic_lds((const void*)ffn::ffn_bwd_kernel, ffn::kBwdSmem, lds_set);
    if (e != hipSuccess) return e;
    int64_t ranges, rows;
    ffn::split(M, 256, &ranges, &rows);
    hipLaunchKernelGGL(ffn::ffn_bwd_kernel, dim3((unsigned)ranges), dim3(ffn::NT), ffn::kBwdSmem,
                       stream, ffn::BwdParams{x, dq, a, w1, w2, dx, part, M, ranges, rows});
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_colsum(part, ranges, ffn::kPart, grads, colsum_ws, stream);
}

hipError_t launch_proj_in_forward(const float* x, const float* wx, const float* bx,
                                  const float* wz, const float* bz, float* hx, float* hz,
                                  int64_t M, hipStream_t stream) {
    const int64_t tiles = (M + ffn::TR - 1) / ffn::TR;
    const dim3 grid((unsigned)(tiles < 512 ? tiles : 512));
    hipLaunchKernelGGL(ffn::proj_in_fwd_kernel, grid, dim3(ffn::NT), 0, stream,
                       ffn::InFwdParams{x, wx, bx, wz, bz, hx, hz, M});
    return hipGetLastError();
}

hipError_t launch_proj_in_backward(const float* x, const float* dhx, const float* dhz,
                                   const float* wx, const float* wz, float* dx, float* grads,
                                   int64_t M, float* part, void* colsum_ws, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    hipError_t e =
        allow_dynamic_lds((const void*)ffn::proj_in_bwd_kernel, ffn::kInBwdSmem, lds_set);
    if (e != hipSuccess) return e;
    int64_t ranges, rows;
    ffn::split(M, 256, &ranges, &rows);
    hipLaunchKernelGGL(ffn::proj_in_bwd_kernel, dim3((unsigned)ranges), dim3(ffn::NT),
                       ffn::kInBwdSmem, stream,
                       ffn::InBwdParams{x, dhx, dhz, wx, wz, dx, part, M, ranges, rows});
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_colsum(part, ranges, ffn::kInPart, grads, colsum_ws, stream);
}

hipError_t launch_proj_out_backward(const float* y, const float* dout, const float* w, float* dy,
                                    float* grads, int64_t M, float* part, void* colsum_ws,
                                    hipStream_t stream) {
    int64_t ranges, rows;
    ffn::split(M, 512, &ranges, &rows);
    hipLaunchKernelGGL(ffn::proj_out_bwd_kernel, dim3((unsigned)ranges), dim3(ffn::NTO), 0, stream,
                       ffn::OutBwdParams{y, dout, w, dy, part, M, ranges, rows});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_colsum(part, ranges, ffn::kOutPart, grads, colsum_ws, stream);
}

}  // namespace recblr
