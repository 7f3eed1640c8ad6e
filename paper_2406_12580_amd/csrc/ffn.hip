// The position-wise feed-forward sub-layer of the model, Q = SiLU(X W1^T + b1) W2^T
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
// split.
//
// Measured at M = 409600: forward 205 us (A written, 0.63 GB: 122 us at copy speed;
// matrix cores busy 80 us), backward 255 us (0.84 GB with dX read and written: 162 us;
// matrix cores 123 us, vector instructions about as long, two waves a SIMD in step
// with each other).  Layer by layer, with the hidden tensors written and read between
// four linear kernels and two weight-gradient kernels: 326 and 630 us.
#include "device_common.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"
#include "gemm.hpp"

namespace recblr {
namespace ffn {

constexpr int D = 64, F = 256, TR = 32, NW = 8, NT = NW * kWave;
constexpr int kPlane = TR * D * 2;                 // bytes of a plane of a row tile
constexpr int kExch = NW * 8 * kWave * 16;         // parts of Q or dX, fp32
constexpr int kTrans = 32 * 32 * 2;                // a plane of a wave's dA block
constexpr int64_t kPart = kFfnGrads;               // [dW1 | db1 | dW2 | db2]
static_assert(kPart == 2 * F * D + F + D);

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s4 lds_s4;

// Chunk j (16 bytes of 128) of row r of a plane at j ^ swz(r): 16 rows of one chunk,
// and 4 rows of 4 chunks, land on distinct banks.
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 1) << 2 | ((r >> 2) & 3); }

__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vector memory stays in flight
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                             0x00020000);
}
__device__ __forceinline__ int fresh(int lane) {
    asm volatile("" : "+v"(lane));  // addresses are formed again in each tile, not kept
    return lane;
}
__device__ __forceinline__ b8 tr_pair(const char* p0, const char* p1) {
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p0);
    const s4 c = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p1);
    return __builtin_bit_cast(b8, __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ f16v mfma(b8 a, b8 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
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
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f4*)(ex + ((w * 8 + db * 4 + q) * kWave + ln) * 16) =
                    f4{y[db][4 * q], y[db][4 * q + 1], y[db][4 * q + 2], y[db][4 * q + 3]};
        stage_quad<3>(xp + (par ^ 1) * 3 * kPlane, next, tid);
        lds_barrier();
        f4 sum = b2;
#pragma unroll
        for (int o = 0; o < NW; ++o) sum += *(const f4*)(ex + ((o * 8 + w) * kWave + ln) * 16);
        const __amdgpu_buffer_rsrc_t qrs = rsrc(P.q + m * D, (uint32_t)(n * D * 4));
        __builtin_amdgcn_raw_buffer_store_b128(
            u4v{__float_as_uint(sum[0]), __float_as_uint(sum[1]), __float_as_uint(sum[2]),
                __float_as_uint(sum[3])},
            qrs, (uint32_t)((ln & 31) * D + 8 * w + 4 * (ln >> 5)) * 4, 0, 0);
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
        // X^T and dQ^T fragments: input 32 db + lane % 32, rows in A's order
        const int r0 = 4 * (ln >> 5) + ((ln >> 2) & 3), c0 = 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
        const int tb = r0 * (D * 2) + (((c0 >> 3) ^ swz(r0)) << 4) + (c0 & 7) * 2;
        const int fl = ln & 31;
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
            {
                uint32_t u[2][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const fastmm::u2v p = fastmm::split2(act[2 * i], act[2 * i + 1]);
                    u[0][i] = p.x;
                    u[1][i] = p.y;
                }
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    ap[p] = __builtin_bit_cast(b8, u4v{u[p][0], u[p][1], u[p][2], u[p][3]});
            }
            // dA into the wave's [f][row] planes: rows 16 s + 4 h .., 16 s + 8 + 4 h ..
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const u4v d4 = __builtin_bit_cast(u4v, dap[p]);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    *(u2v*)(tp + p * kTrans + fl * 64 +
                            (((4 * s + 2 * k + (ln >> 5)) ^ (fl >> 2)) << 3)) =
                        u2v{d4[2 * k], d4[2 * k + 1]};
            }
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                b8 xf[2], qf[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int o = tb ^ (db << 6);
                    const int k = s * (16 * D * 2) + p * kPlane;
                    qf[p] = tr_pair(dqs + o + k, dqs + (o ^ 32) + k + 8 * D * 2);
                    xf[p] = tr_pair(xs + o + k, xs + (o ^ 32) + k + 8 * D * 2);
                }
                dw2[db] = mma3(qf, ap[0], ap[1], dw2[db]);
                dw1[db] = mma3(xf, dap[0], dap[1], dw1[db]);
            }
        }
        load_a(m + TR, ln);
        const u4v dqn = fetch_quad(P.dq, m + TR, row1, tid);
        const u4v xn = fetch_quad(P.x, m + TR, row1, tid);
        const __amdgpu_buffer_rsrc_t drs = rsrc(P.dx + m * D, (uint32_t)(n * D * 4));
        const uint32_t dxo = (uint32_t)((ln & 31) * D + 8 * w + 4 * (ln >> 5)) * 4;
        const u4v dd = __builtin_amdgcn_raw_buffer_load_b128(drs, dxo, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // ---- this wave's part of dX^T
        f16v o[2];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.0f;
        const int ub = (8 * (ln >> 5) + ((ln >> 2) & 3)) * 64 +
                       (((4 * ((ln >> 4) & 1) + (ln & 3)) ^ (2 * (ln >> 5))) << 3);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            b8 f[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const char* const base = tp + p * kTrans + s * 1024;
                f[p] = tr_pair(base + (ub ^ (s << 5)), base + (ub ^ (s << 5) ^ 8) + 256);
            }
#pragma unroll
            for (int db = 0; db < 2; ++db) o[db] = mma6(w1t[db][s], f, o[db]);
        }
        lds_barrier();  // the last tile's parts have been read
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f4*)(exch + ((w * 8 + db * 4 + q) * kWave + ln) * 16) =
                    f4{o[db][4 * q], o[db][4 * q + 1], o[db][4 * q + 2], o[db][4 * q + 3]};
        stage(par ^ 1, xn, dqn, tid);
        lds_barrier();
        f4 sum = *(const f4*)(exch + (w * kWave + ln) * 16);
#pragma unroll
        for (int k = 1; k < NW; ++k) sum += *(const f4*)(exch + ((k * 8 + w) * kWave + ln) * 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) sum[k] += __uint_as_float(dd[k]);
        __builtin_amdgcn_raw_buffer_store_b128(
            u4v{__float_as_uint(sum[0]), __float_as_uint(sum[1]), __float_as_uint(sum[2]),
                __float_as_uint(sum[3])},
            drs, dxo, 0, 0);
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

constexpr int kFwdSmem = 2 * 3 * kPlane + 2 * kExch;
constexpr int kBwdSmem = 2 * 5 * kPlane + NW * 3 * kTrans + kExch;

template <typename K>
hipError_t allow_lds(K kern, int bytes) {
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// One workgroup per compute unit; at least 256 rows a range (each leaves a partial).
void split(int64_t M, int64_t* ranges, int64_t* rows) {
    int64_t n = (M + 255) / 256;
    n = n < 256 ? n : 256;
    *rows = ((M + n - 1) / n + TR - 1) / TR * TR;
    *ranges = (M + *rows - 1) / *rows;
}

}  // namespace ffn

bool ffn_fused_applies(int64_t M, int64_t D, int64_t F, std::initializer_list<const void*> ptrs) {
    uintptr_t a = 0;
    for (const void* p : ptrs) a |= (uintptr_t)p;
    return M > 0 && D == ffn::D && F == ffn::F && a % 16 == 0;
}

int64_t ffn_backward_ranges(int64_t M) {
    if (M <= 0) return 0;
    int64_t n, rows;
    ffn::split(M, &n, &rows);
    return n;
}

hipError_t launch_ffn_forward(const float* x, const float* w1, const float* b1, const float* w2,
                              const float* b2, float* a, float* q, int64_t M, hipStream_t stream) {
    static const hipError_t attr = ffn::allow_lds(ffn::ffn_fwd_kernel, ffn::kFwdSmem);
    if (attr != hipSuccess) return attr;
    const int64_t tiles = (M + ffn::TR - 1) / ffn::TR;
    const dim3 grid((unsigned)(tiles < 256 ? tiles : 256));
    hipLaunchKernelGGL(ffn::ffn_fwd_kernel, grid, dim3(ffn::NT), ffn::kFwdSmem, stream,
                       ffn::FwdParams{x, w1, b1, w2, b2, a, q, M});
    return hipGetLastError();
}

hipError_t launch_ffn_backward(const float* x, const float* dq, const float* a, const float* w1,
                               const float* w2, float* dx, float* grads, int64_t M, float* part,
                               void* colsum_ws, hipStream_t stream) {
    static const hipError_t attr = ffn::allow_lds(ffn::ffn_bwd_kernel, ffn::kBwdSmem);
    if (attr != hipSuccess) return attr;
    int64_t ranges, rows;
    ffn::split(M, &ranges, &rows);
    hipLaunchKernelGGL(ffn::ffn_bwd_kernel, dim3((unsigned)ranges), dim3(ffn::NT), ffn::kBwdSmem,
                       stream, ffn::BwdParams{x, dq, a, w1, w2, dx, part, M, ranges, rows});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_colsum(part, ranges, ffn::kPart, grads, colsum_ws, stream);
}

}  // namespace recblr
