// Layer backward in one kernel for D = 128: the gate pre-activations of section
// 3.2 (z = W x + b) formed again, the adjoint scan of eq:linrnn, the gate
// gradients, and both projection gradients (dx += dz W and dW = dz^T x), so that
// neither z nor dz reaches HBM.  It reads x, h and dLoss/dh and writes dx.
// For the gated layer of Algorithm alg:gated_recurrent (GATE, fp32) it is the
// whole backward of the core: it reads hx, hz, h and dy, forms x' =
// SiLU(conv(hx)) and dh = dy SiLU(hz), and writes dhz and, through the conv's
// transpose, dhx; neither x' nor dx' reaches HBM either.
//
// Work decomposition.  A workgroup of 8 waves (one per compute unit) walks
// whole batch rows from their last step to their first, in tiles of 64 steps x
// all 128 channels, with the adjoint's carry in a register, and goes on to row
// blockIdx + gridDim.  Per tile:
//   A  wave w owns channels 16 w .. 16 w + 15: z of both gates for its channels
//      (32 columns of v_mfma_f32_32x32x16_bf16, K = 128, x planes in LDS, W
//      fragments streamed from L2), then per lane one channel at 8 consecutive
//      steps per 32-step block: alpha, the run's aggregate, the carry through the
//      four lanes of a channel, and the gate gradients.  dz_r and dz_i go to LDS
//      as bf16 hi and lo planes [gate][channel][step]; dx's direct term replaces
//      x in its LDS tile.
//   B  dW += dz^T x (256 x 128, accumulators in registers for the whole launch;
//      K = the tile's 64 steps), then dx = direct + dz W (64 x 128, K = 256)
//      straight to memory.  The operand whose contraction index is not
//      contiguous in LDS is read through the transposing LDS loads.
//   C  the next tile's x, loaded into registers during B, goes to LDS.
// With GATE a lane holds one channel's steps in C too (x planes are [channel][step]
// then, and the operand that needs the transposing reads is the other one): it
// forms x' from hx and the three steps before, and between B and C it takes its
// channel's whole dx' from the LDS tile back through the conv, walking the tiles
// from the end as the adjoint does, so that dc of the three later steps is at hand.
// Products of two fp32 operands are the 3-term bf16 split of fastmm (hi*hi +
// hi*lo + lo*hi); bf16 operands are one exact plane.  The sums over steps and rows (db, dLambda,
// the conv's gradients) are fp32 within a tile and double across tiles; they and dW
// leave as one fp32 partial per workgroup, summed in double in a fixed order by
// reduce_kernel.  Nothing depends on the order in which workgroups run.
//
// What it replaces and costs (256 x 2048 x 128 fp32): the fused scan, which
// wrote dz (8 B an element), dx += dz W and dW = dz^T x, which read it again:
// 750 us; this kernel 405-410 us, 16 B an element.  Bound by the vector ALU and
// the matrix cores one after the other: of 822 K cycles per SIMD (SQ counters)
// the ALU issues in 375 K (70 instructions an element, 6 of them
// transcendental) and the matrix cores run in 295 K (3 products of 3 terms);
// HBM latency adds 20 us (timed with every tile read from the same rows).
// What it took: W fragments are asked for before anything slow (vector memory
// completes in order, and a fragment queued behind dx's stores or the next
// tile's loads waits for them: 436 -> 405 us), one gate's W per wave instead of
// one 32-step block (W is then read once per tile), and LDS addresses formed
// again in each tile (kept across the loop they spill: 630 us).  Tiles of 32
// steps with two tiles in flight, so that one wave of a SIMD is in A while the
// other is in B, measured 630 us: twice the W traffic, and every stage then
// waits for loads queued by the one before it.  The gated backward at
// 2048 x 200 x 128: 540 us, against 470 us for the same kernel on x' from memory
// plus 230 us of conv passes around it (and 780 us + 230 us with separate
// kernels); its loads are spread over B, the conv and z because all at once in
// flight they spill (595 us).
#include "device_common.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"
#include "wave_tile.hpp"

namespace recblr {
namespace fbw {

using namespace wtile;

constexpr int D = 128;            // channels
constexpr int TS = 64;            // steps per tile
constexpr int NW = 8;             // waves per workgroup
constexpr int NT = NW * kWave;

struct Params {
    const void* x;        // [B][L][D] TX: x, or hx (GATE)
    const void* h;        // [B][L][D] TH
    const void* g;        // [B][L][D] TH: dLoss/dh, or dy (GATE)
    const void* gz;       // GATE: hz
    void* gdz;            // GATE: dhz
    void* dx;             // [B][L][D] TX: dx, or dhx (GATE)
    const float* h0;      // [B][D] or null
    const float* dhT;     // [B][D] or null
    float* dh0;           // [B][D] or null
    const void* pz;       // packed W for z and for dx (pack_kernel)
    const void* px;
    const void* br;       // [D] TW or null
    const void* bi;
    const float* lam;
    float* part_w;        // [gridDim.x][2 D][D]
    float* part_c;        // [gridDim.x][kCols][D]: db_r, db_i, sum of dLoss/dq r and
                          // (GATE) the conv's bias and tap gradients
    int64_t L, B;
    const float* cw;      // GATE: conv taps [D][K]
    const float* cb;      // GATE: conv bias [D] or null
    int K;
};

// 16-byte chunk permutations of the LDS tiles.  A bf16 row of x (256 bytes)
// stores chunk j at j ^ swz16(r): the 16 rows of one pass of a fragment read
// ({0..7, 16..23} or {8..15, 24..31}) land on distinct chunks, and so do the four
// rows x 64 bytes of a transposing read.  A row of the fp32 tile (512 bytes)
// stores chunk j at j ^ swz32(r): the rows 8 apart of a scan access, and the
// rows 4 apart of an accumulator access, differ.  A dz row (128 bytes: one
// channel's 64 steps) stores chunk j at j ^ swzdz(r).
__device__ __forceinline__ int swz16(int r) {
    return ((r & 3) << 2) | ((r >> 2) & 1) | ((r >> 3) & 2);
}
__device__ __forceinline__ int swz32(int r) { return (((r >> 3) & 3) << 2) ^ ((r << 1) & 8); }
__device__ __forceinline__ int swzdz(int r) { return ((r & 2) << 1) | ((r >> 2) & 3); }

// Four values summed over the four 16-lane rows of the wave: row r gets value r's sum.
__device__ __forceinline__ float row_sums(float a, float b, float c, float d) {
    swap16(a, b);  // a: rows 0 and 2 of a, of b; b: rows 1 and 3 of a, of b
    swap16(c, d);
    a += b;
    c += d;
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(c), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One element through a buffer resource (reads past it give 0).
template <typename T>
__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    if constexpr (sizeof(T) == 4)
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    else
        return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0) << 16);
}
template <typename T>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, 2);
    else
        __builtin_amdgcn_raw_buffer_store_b16(from_f32<bf16>(v).bits, r, off, 0, 0);
}

template <typename TX, typename TW, bool GATE>
struct Geo {
    static constexpr bool kXf32 = sizeof(TX) == 4;
    static constexpr int PX = kXf32 ? 2 : 1;             // x planes
    static constexpr int PW = sizeof(TW) == 4 ? 2 : 1;   // W planes
    static constexpr int kXPlane = TS * D * 2;
    static constexpr int kRaw = TS * D * 4;  // fp32 tile: x (fp32 I/O), then dx's direct term
    static constexpr int kDzPlane = 2 * D * TS * 2;
    static constexpr int kSmem = PX * kXPlane + (GATE ? 2 : 1) * kRaw + 2 * kDzPlane;
    static constexpr int kCols = GATE ? 3 + 1 + kConvTaps : 3;  // columns of part_c
    static constexpr int kXLoads = TS * D * (int)sizeof(TX) / (NT * 16);  // 16-byte loads a thread
};

template <typename TX, typename TH, typename TW, bool GATE>
__global__ __launch_bounds__(NT, 2) void fused_bwd_kernel(Params P) {
    using G = Geo<TX, TW, GATE>;
    constexpr int PX = G::PX, PW = G::PW;
    constexpr int EX = (int)sizeof(TX), EH = (int)sizeof(TH);
    static_assert(!GATE || (EX == 4 && EH == 4 && PW == 2), "the gated layer's backward is fp32");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const xpl = smem;                       // x planes [PX][TS][D], GATE [PX][D][TS]
    char* const raw = smem + PX * G::kXPlane;     // fp32 [TS][D]: x, then dx's direct term
    char* const dzp = raw + G::kRaw;              // dz planes [2][2 D][TS]
    char* const hxt = dzp + 2 * G::kDzPlane;      // GATE: fp32 [TS][D], hx

    const int lane = threadIdx.x & (kWave - 1);
    const int w = wave_id();
    int64_t b = blockIdx.x;
    if (b >= P.B) return;

    const uint32_t xbytes = (uint32_t)(P.L * D * EX), hbytes = (uint32_t)(P.L * D * EH);
    const int ntiles = (int)((P.L + TS - 1) / TS);

    f16v dw[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) dw[a][c][v] = 0.0f;
    float nbr, nbi, carry = 0.0f;
    ChannelConst cc;
    // Totals over the workgroup's tiles of the lane's channel, lane row rho: db_r, db_i,
    // dLoss/dq r or (GATE) the conv bias's gradient, and (GATE) the gradient of tap rho.
    double total = 0.0, total_w = 0.0;
    // GATE: the lane's channel's taps and bias, the last tile's part of the bias's gradient,
    // dc of the three steps after the tile, hx of the three before it
    float wt[GATE ? 4 : 1], cbv = 0.0f, dcb = 0.0f, later[GATE ? 3 : 1], before[GATE ? 3 : 1];
    {
        const int ch = 16 * w + (lane & 15);
        nbr = P.br ? -load((const TW*)P.br + ch) * kLog2e : 0.0f;
        nbi = P.bi ? -load((const TW*)P.bi + ch) * kLog2e : 0.0f;
        cc = channel_const(P.lam[ch]);
        if constexpr (GATE) {
            cbv = P.cb ? P.cb[ch] : 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) wt[j] = j < P.K ? P.cw[ch * P.K + j] : 0.0f;
        }
    }

    // ---- weight fragments from L2 (fragment order: one 16-byte load a lane)
    const uint32_t wbytes = (uint32_t)(2 * D * D * 2 * PW);
    const __amdgpu_buffer_rsrc_t zrs = rsrc(P.pz, wbytes), prs = rsrc(P.px, wbytes);
    const int nb = w & 3, gate = w >> 2;  // dx part of this wave: 32 inputs, one gate
    const int wm = w & 3, wn = w >> 2;  // dW block: 64 outputs x 64 inputs
    b8 wf[4][PW];  // ring of k-steps, for z and then for dx
    auto load_w = [&](__amdgpu_buffer_rsrc_t r, int first, int ks, int ln) {
#pragma unroll
        for (int p = 0; p < PW; ++p)
            wf[ks & 3][p] = __builtin_bit_cast(
                b8, __builtin_amdgcn_raw_buffer_load_b128(
                        r, ln * 16, ((first + ks) * PW + p) * kWave * 16, 0));
    };

    // ---- loads of one tile into registers
    u4v xr[GATE ? 1 : G::kXLoads];
    float hx[GATE ? 2 : 1][GATE ? 8 : 1], hxb[GATE ? 3 : 1];
    float gv[2][8], hp[2][8], zv[GATE ? 2 : 1][GATE ? 8 : 1], ht[GATE ? 2 : 1];
    float h0v, dhTv;  // h_{-1} and dhT where the tile starts or ends its row, else 0
    auto fetch = [&](int64_t b, int s) {
        const int ln = fresh(lane);
        const int rho = ln >> 4, ch = 16 * w + (ln & 15);
        const __amdgpu_buffer_rsrc_t xrs = rsrc((const char*)P.x + b * P.L * D * EX, xbytes);
        const __amdgpu_buffer_rsrc_t hrs = rsrc((const char*)P.h + b * P.L * D * EH, hbytes);
        const __amdgpu_buffer_rsrc_t grs = rsrc((const char*)P.g + b * P.L * D * EH, hbytes);
        const uint32_t t0 = (uint32_t)s * TS;
        // (no load is conditional, so that the wait counts stay exact: one that does
        // not apply reads past its resource)
        dhTv = bload<float>(rsrc(P.dhT + b * D, P.dhT && s == ntiles - 1 ? D * 4 : 0), ch * 4);
        h0v = bload<float>(rsrc(P.h0 + b * D, P.h0 && s == 0 ? D * 4 : 0),
                           rho == 0 ? ch * 4 : D * 4);
        // a thread takes 8 channels (two 16-byte chunks in fp32, one in bf16) of
        // rows 4 w + lane / 16 and 32 + that
#pragma unroll
        for (int q = 0; q < (GATE ? 0 : 2); ++q) {
            const uint32_t off = ((t0 + 32 * q + 4 * w + ln / 16) * D + 8 * (ln % 16)) * EX;
#pragma unroll
            for (int k = 0; k < G::kXLoads / 2; ++k)
                xr[q * (G::kXLoads / 2) + k] =
                    __builtin_amdgcn_raw_buffer_load_b128(xrs, off + 16 * k, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const uint32_t off = ((t0 + 32 * m + 8 * rho) * D + ch) * EH;
#pragma unroll
            for (int i = 0; i < (GATE ? 0 : 8); ++i) gv[m][i] = bload<TH>(grs, off + i * D * EH);
            // h_{t-1}: before step 0 the offset wraps past the resource (0)
            hp[m][0] = bload<TH>(hrs, off - D * EH);
#pragma unroll
            for (int i = 1; i < 8; ++i) hp[m][i] = bload<TH>(hrs, off + (i - 1) * D * EH);
        }
        if constexpr (GATE) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
                ht[m] = bload<TH>(hrs, ((t0 + 32 * m + 8 * rho + 7) * D + ch) * EH);
        }
    };
    // GATE: dy and hz, asked for in the middle of z's products (with the other loads they
    // spill) and used after r and alpha.
    auto fetch_g = [&](int64_t b, int s, int ln) {
        if constexpr (GATE) {
            const int rho = ln >> 4, ch = 16 * w + (ln & 15);
            const __amdgpu_buffer_rsrc_t grs = rsrc((const char*)P.g + b * P.L * D * EH, hbytes);
            const __amdgpu_buffer_rsrc_t zrs = rsrc((const char*)P.gz + b * P.L * D * EH, hbytes);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const uint32_t off = (((uint32_t)s * TS + 32 * m + 8 * rho) * D + ch) * EH;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    gv[m][i] = bload<TH>(grs, off + i * D * EH);
                    zv[m][i] = bload<TH>(zrs, off + i * D * EH);
                }
            }
        }
    };
    // GATE: hx of the lane's channel at its 16 steps, and before the tile.  Asked for
    // after dx's products, whose registers these loads take (in flight with the others
    // they spill), and in flight through the conv's backward.
    auto fetch_hx = [&](int64_t b, int s) {
        if constexpr (GATE) {
            const int ln = fresh(lane);
            const int rho = ln >> 4, ch = 16 * w + (ln & 15);
            const __amdgpu_buffer_rsrc_t xrs = rsrc((const char*)P.x + b * P.L * D * EX, xbytes);
            const uint32_t t0 = (uint32_t)s * TS;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const uint32_t off = ((t0 + 32 * m + 8 * rho) * D + ch) * EX;
#pragma unroll
                for (int i = 0; i < 8; ++i) hx[m][i] = bload<TX>(xrs, off + i * D * EX);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)  // before step 0 the offset wraps past the resource (0)
                hxb[k] = bload<TX>(xrs, ((t0 - 3 + k) * D + ch) * EX);
        }
    };
    // ---- the loaded x of a tile to LDS: bf16 planes and (fp32) the tile itself.
    // GATE: x' = SiLU(conv(hx)) of the lane's channel; the columns of hx and x' that a
    // wave writes are those that it alone reads.
    auto stage = [&]() {
        const int ln = fresh(lane);
        if constexpr (GATE) {
            const int rho = ln >> 4, ch = 16 * w + (ln & 15);
            char* const hb = hxt + (8 * rho) * (D * 4) + ch * 4;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int i = 0; i < 8; ++i) *(float*)(hb + (32 * m + i) * (D * 4)) = hx[m][i];
            wave_fence();  // the window's first steps are other lanes'
#pragma unroll
            for (int k = 0; k < 3; ++k) before[k] = hxb[k];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                float win[11];  // steps 32 m + 8 rho - 3 ..
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int row = 32 * m + 8 * rho - 3 + k;  // before the tile: read row 0
                    float v = *(const float*)(hxt + (row < 0 ? 0 : row) * (D * 4) + ch * 4);
                    asm volatile("" : "+v"(v));  // read by every lane, without a branch
                    win[k] = m == 0 && rho == 0 ? before[k] : v;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) win[3 + i] = hx[m][i];
                float xo[8];
                char* const rbase = raw + (8 * rho) * (D * 4) + (((ch >> 2) ^ (4 * rho)) << 4) +
                                    (ch & 3) * 4;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float c = cbv;
#pragma unroll
                    for (int j = 0; j < 4; ++j) c = fmaf(wt[j], win[3 + i - j], c);
                    xo[i] = c * sigmoid(c);
                    *(float*)((i < 4 ? rbase : raw + ((rbase - raw) ^ 128)) +
                              (32 * m + i) * (D * 4)) = xo[i];
                }
                u4v hi, lo;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const fastmm::u2v p = fastmm::split2(xo[2 * q], xo[2 * q + 1]);
                    hi[q] = p.x;
                    lo[q] = p.y;
                }
                char* const dst = xpl + ch * (TS * 2) + ((rho ^ swzdz(ch) ^ (4 * m)) << 4);
                *(u4v*)dst = hi;
                *(u4v*)(dst + G::kXPlane) = lo;
            }
            return;
        }
        const int r = 4 * w + ln / 16, jb = ln % 16;
        char* const pos = xpl + r * (D * 2) + ((jb ^ swz16(r)) << 4);
        char* const pr = raw + r * (D * 4) + (((2 * jb) ^ swz32(r)) << 4);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if constexpr (G::kXf32) {
                const u4v v0 = xr[2 * q], v1 = xr[2 * q + 1];
                *(u4v*)(pr + q * (32 * D * 4)) = v0;
                *(u4v*)(pr + q * (32 * D * 4) + 16) = v1;
                const auto f = [](uint32_t u) { return __uint_as_float(u); };
                const fastmm::u2v p0 = fastmm::split2(f(v0[0]), f(v0[1])),
                                  p1 = fastmm::split2(f(v0[2]), f(v0[3])),
                                  p2 = fastmm::split2(f(v1[0]), f(v1[1])),
                                  p3 = fastmm::split2(f(v1[2]), f(v1[3]));
                *(u4v*)(pos + q * (32 * D * 2)) = u4v{p0.x, p1.x, p2.x, p3.x};
                *(u4v*)(pos + q * (32 * D * 2) + G::kXPlane) = u4v{p0.y, p1.y, p2.y, p3.y};
            } else {
                *(u4v*)(pos + q * (32 * D * 2)) = xr[q];
            }
        }
    };

    // ---- stage A.  NB: 32-step blocks that hold steps; FULL: no step past L.
    auto stage_a = [&](int64_t b, int s, auto nb_tag, auto full_tag) {
        constexpr int NB = decltype(nb_tag)::value;
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t t0 = (int64_t)s * TS;
        const int lim = P.L - t0 < TS ? (int)(P.L - t0) : TS;  // valid rows
        const int ln = fresh(lane);
        const int rho = ln >> 4, ch = 16 * w + (ln & 15);
        const bool odd = rho & 1, upper = rho >= 2;
        if (s == ntiles - 1) carry = dhTv;
        // z
        f16v acc[NB];
        {
            // x rows (operand rows permuted by sigma) x channels 16 kk + 8 (lane / 32) ..
            // + 7; GATE: channel rows, 4 steps of sigma's order a lane
            const int r = sigma(ln & 31);
            const int kr = 8 * (ln >> 5) + ((ln >> 2) & 3);
            const int base = GATE ? kr * (TS * 2) +
                                        (((2 * (ln & 1) + ((ln >> 4) & 1)) ^ swzdz(kr)) << 4) +
                                        4 * (ln & 2)
                                  : r * (D * 2) + (((ln >> 5) ^ swz16(r)) << 4);
            f16v zero;
#pragma unroll
            for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
                for (int m = 0; m < NB; ++m) {
                    b8 a[PX];
#pragma unroll
                    for (int p = 0; p < PX; ++p) {
                        if constexpr (GATE)
                            a[p] = tr_pair(xpl + (base ^ (m << 6)) + kk * (16 * TS * 2) +
                                               p * G::kXPlane,
                                           xpl + (base ^ (m << 6) ^ 16) + kk * (16 * TS * 2) +
                                               4 * TS * 2 + p * G::kXPlane);
                        else
                            a[p] = *(const b8*)(xpl + (base ^ (kk << 5)) + m * (32 * D * 2) +
                                                p * G::kXPlane);
                    }
                    acc[m] = mma<PX, PW>(a, wf[kk & 3], kk == 0 ? zero : acc[m]);
                }
                if (kk < 4) load_w(zrs, 8 * w, kk + 4, ln);
                if (kk == 3) fetch_g(b, s, ln);
                __builtin_amdgcn_sched_barrier(GATE ? 0 : 0x38F);  // the loads stay where they are
            }
        }
        // every lane gets z_r and z_i of channel ch at steps 32 m + 8 rho + i; r and alpha
        float al[NB][8];
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float zr = acc[m][i], zi = acc[m][i + 8];
                swap16(zr, zi);
                const float r = fast_rcp(1.0f + fast_exp2(fmaf(zr, -kLog2e, nbr)));
                acc[m][i] = r;
                acc[m][i + 8] = zi;
                al[m][i] = fast_exp2(r * cc.neg_s_l2);
            }
        // output gate: dh = dy SiLU(hz), dhz = dy h SiLU'(hz)
        if constexpr (GATE) {
            const __amdgpu_buffer_rsrc_t ors = rsrc((char*)P.gdz + b * P.L * D * EH, hbytes);
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const uint32_t off = (uint32_t)((t0 + 32 * m + 8 * rho) * D + ch) * EH;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float z = zv[m][i], y = gv[m][i];
                    const float sg = sigmoid(z);
                    const float hv = i == 7 ? ht[m] : hp[m][i < 7 ? i + 1 : 0];
                    gv[m][i] = y * (z * sg);
                    bstore<TH>(ors, off + i * D * EH, y * hv * (sg * fmaf(z, 1.0f - sg, 1.0f)));
                }
            }
        }
        // the lane's run (later steps first)
        Seg run[NB];
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            Seg sg{1.0f, 0.0f};
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                const float a = al[m][i];
                Seg e{a, a * gv[m][i]};
                if constexpr (!FULL) {
                    const bool ok = 32 * m + 8 * rho + i < lim;
                    e.A = ok ? e.A : 1.0f;
                    e.H = ok ? e.H : 0.0f;
                }
                sg = compose(e, sg);
            }
            run[m] = sg;
        }
        // the four runs of a block: what comes before this lane's, and the total
        Seg excl[NB], tot[NB];
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            const Seg p{row_partner(run[m].A, odd), row_partner(run[m].H, odd)};
            const Seg pair = odd ? compose(p, run[m]) : compose(run[m], p);
            const Seg e1 = odd ? Seg{1.0f, 0.0f} : p;
            const Seg o{half_partner(pair.A, upper), half_partner(pair.H, upper)};
            tot[m] = upper ? compose(o, pair) : compose(pair, o);
            excl[m] = upper ? e1 : compose(e1, o);
        }
        hp[0][0] += h0v;  // one of the two is 0
        // gate gradients, from the last step back
        float sr = 0.0f, si = 0.0f, sl = 0.0f;
#pragma unroll
        for (int m = NB - 1; m >= 0; --m) {
            float eps = fmaf(excl[m].A, carry, excl[m].H);
            carry = fmaf(tot[m].A, carry, tot[m].H);
            float dzr[8], dzi[8];
            char* const rbase = raw + (8 * rho) * (D * 4) + (((ch >> 2) ^ (4 * rho)) << 4) +
                                (ch & 3) * 4;
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                const int row = 32 * m + 8 * rho + i;
                // swz32 of the row: 4 rho, and 8 for i >= 4
                float* const rp = (float*)((i < 4 ? rbase : raw + ((rbase - raw) ^ 128)) +
                                           (32 * m + i) * (D * 4));
                float xv;
                if constexpr (G::kXf32)
                    xv = *rp;
                else
                    xv = __uint_as_float((uint32_t)(*(const uint16_t*)(
                                             xpl + row * (D * 2) +
                                             (((ch >> 3) ^ swz16(8 * rho + i)) << 4) +
                                             (ch & 7) * 2)) << 16);
                const float r = acc[m][i], a = al[m][i];
                const float ig = fast_rcp(1.0f + fast_exp2(fmaf(acc[m][i + 8], -kLog2e, nbi)));
                const float delta = gv[m][i] + eps;
                const float mm = one_minus_exp_neg(r * cc.two_s, a);
                const float rs = mm > 0.0f ? fast_rsq(mm) : 0.0f;  // 1 / sqrt(1 - alpha^2)
                const float v = delta * ig * rs;
                const float dxv = v * mm;      // delta beta
                const float gs = dxv * xv;     // dLoss/dbeta i sqrt(1 - alpha^2)
                const float gq = a * fmaf(-delta, hp[m][i], a * (v * xv));  // dLoss/dq
                float lq = gq * r;
                *rp = dxv;
                dzr[i] = cc.s * fmaf(-lq, r, lq);
                dzi[i] = fmaf(-gs, ig, gs);
                if constexpr (FULL) {
                    eps = a * delta;
                } else {
                    const bool ok = row < lim;
                    dzr[i] = ok ? dzr[i] : 0.0f;
                    dzi[i] = ok ? dzi[i] : 0.0f;
                    lq = ok ? lq : 0.0f;
                    eps = ok ? a * delta : eps;
                }
                sr += dzr[i];
                si += dzi[i];
                sl += lq;
            }
            // dz planes: 8 steps of one channel are one 16-byte chunk
#pragma unroll
            for (int gate = 0; gate < 2; ++gate) {
                u4v hi, lo;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const fastmm::u2v p = gate == 0 ? fastmm::split2(dzr[2 * q], dzr[2 * q + 1])
                                                    : fastmm::split2(dzi[2 * q], dzi[2 * q + 1]);
                    hi[q] = p.x;
                    lo[q] = p.y;
                }
                char* const dst = dzp + (gate * D + ch) * (TS * 2) +
                                  ((rho ^ swzdz(ch) ^ (4 * m)) << 4);
                *(u4v*)dst = hi;
                *(u4v*)(dst + G::kDzPlane) = lo;
            }
        }
        total += (double)row_sums(sr, si, sl, dcb);
        if (s == 0 && rho == 0 && P.dh0) P.dh0[b * D + ch] = carry;
    };

    // ---- GATE: dx' of the lane's channel (whole, in the fp32 tile) back through the conv:
    // dc = dx' SiLU'(c), dhx_t = sum_j w_j dc_{t+j}, and the tap and bias gradients
    auto conv_back = [&](int64_t b, int s, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        if constexpr (GATE) {
            const int64_t t0 = (int64_t)s * TS;
            const int lim = P.L - t0 < TS ? (int)(P.L - t0) : TS;
            const int ln = fresh(lane);
            const int rho = ln >> 4, ch = 16 * w + (ln & 15);
            const __amdgpu_buffer_rsrc_t drs = rsrc((char*)P.dx + b * P.L * D * EX, xbytes);
            char* const rbase = raw + (8 * rho) * (D * 4) + (((ch >> 2) ^ (4 * rho)) << 4) +
                                (ch & 3) * 4;
            const int from = ((ln + 16) & 63) * 4;  // the lane of the next 8 steps
            if (s == ntiles - 1) later[0] = later[1] = later[2] = 0.0f;
            float nx[3];
            float sb = 0.0f, sw[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int m = 1; m >= 0; --m) {
                __builtin_amdgcn_sched_barrier(0);
                float win[11], dc[11];
#pragma unroll
                for (int k = 0; k < 11; ++k) {
                    const int row = 32 * m + 8 * rho - 3 + k;
                    float v = *(const float*)(hxt + (row < 0 ? 0 : row) * (D * 4) + ch * 4);
                    asm volatile("" : "+v"(v));  // read by every lane, without a branch
                    win[k] = k < 3 && m == 0 && rho == 0 ? before[k < 3 ? k : 0] : v;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float dxv = *(const float*)((i < 4 ? rbase : raw + ((rbase - raw) ^ 128)) +
                                                      (32 * m + i) * (D * 4));
                    float c = cbv;
#pragma unroll
                    for (int j = 0; j < 4; ++j) c = fmaf(wt[j], win[3 + i - j], c);
                    const float sg = sigmoid(c);
                    dc[i] = dxv * (sg * fmaf(c, 1.0f - sg, 1.0f));
                    if constexpr (!FULL) dc[i] = 32 * m + 8 * rho + i < lim ? dc[i] : 0.0f;
                    sb += dc[i];
#pragma unroll
                    for (int j = 0; j < 4; ++j) sw[j] = fmaf(dc[i], win[3 + i - j], sw[j]);
                }
                // dc of the three steps after the lane's: the next lane's, across the block
                // the later block's or tile's first lane's
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float n = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(
                        from, (int)__float_as_uint(dc[k])));
                    dc[8 + k] = rho == 3 ? (m == 1 ? later[k] : nx[k]) : n;
                    if (m == 1) nx[k] = n;
                    else later[k] = n;
                }
                if (m == 0) {  // ahead of the last stores (behind them: 2048 x 200 530 -> 547 us)
                    dcb = sb;  // joins `total` with the next tile's sums
                    total_w += (double)row_sums(sw[0], sw[1], sw[2], sw[3]);
                }
                const uint32_t off = (uint32_t)((t0 + 32 * m + 8 * rho) * D + ch) * EX;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    bstore<TX>(drs, off + i * D * EX,
                               fmaf(wt[0], dc[i], fmaf(wt[1], dc[i + 1],
                                                       fmaf(wt[2], dc[i + 2], wt[3] * dc[i + 3]))));
            }
            wave_fence();  // stage() overwrites the steps that other lanes read here
        }
    };

    int s = ntiles - 1;
    fetch(b, s);
    fetch_hx(b, s);
    stage();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) load_w(zrs, 8 * w, ks, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing pending enters the loop
    lds_barrier();

    for (;;) {
        const int64_t t0 = (int64_t)s * TS;
        const int lim = P.L - t0 < TS ? (int)(P.L - t0) : TS;  // valid rows
        int64_t nrow = b;
        int ns = s - 1;
        if (ns < 0) {
            nrow = b + gridDim.x;
            ns = ntiles - 1;
        }
        const bool has_next = nrow < P.B;
        if (lim == TS)
            stage_a(b, s, std::integral_constant<int, 2>{}, std::true_type{});
        else if (lim > 32)
            stage_a(b, s, std::integral_constant<int, 2>{}, std::false_type{});
        else
            stage_a(b, s, std::integral_constant<int, 1>{}, std::false_type{});
        // ---- dx's first weight fragments, then the next tile's loads, which stay in
        // flight through stage B (vector memory completes in order: fragments
        // asked for after them would wait for them)
        {
            const int ln = fresh(lane);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) load_w(prs, 16 * nb + 8 * gate, ks, ln);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!GATE && has_next) fetch(nrow, ns);
        lds_barrier();
        // ---- dW += dz^T x: rows (outputs) 64 wm + 32 u + lane % 32 at steps 16 ks +
        // 8 (lane / 32) .. + 7, against inputs 64 wn + 32 v + lane % 32 at the same steps
        {
            const int ln = fresh(lane);
            const int row = 64 * wm + (ln & 31);
            const int abase = row * (TS * 2) + (((ln >> 5) ^ swzdz(row)) << 4);
            const int kr = 8 * (ln >> 5) + ((ln >> 2) & 3);
            const int col = 64 * wn + 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
            const int bbase = kr * (D * 2) + (((col >> 3) ^ swz16(kr)) << 4) + (col & 7) * 2;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks == 2 && lim <= 32) break;
                b8 a[2][2], c[2][PX];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        a[u][p] = *(const b8*)(dzp + (abase ^ (ks << 5)) + u * (32 * TS * 2) +
                                               p * G::kDzPlane);
                // steps + 16 ks: swz16 bit 1; inputs + 32 v: chunk bit 2; steps + 4: swz16 bit 0
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int p = 0; p < PX; ++p) {
                        if constexpr (GATE) {
                            const int in = 64 * wn + (ln & 31);
                            const int o = in * (TS * 2) + (((ln >> 5) ^ swzdz(in)) << 4);
                            c[v][p] = *(const b8*)(xpl + (o ^ (ks << 5)) + v * (32 * TS * 2) +
                                                   p * G::kXPlane);
                            continue;
                        }
                        const int o = bbase ^ (v << 6) ^ ((ks & 1) << 5);
                        c[v][p] = tr_pair(xpl + o + ks * (16 * D * 2) + p * G::kXPlane,
                                          xpl + (o ^ 16) + ks * (16 * D * 2) + 4 * D * 2 +
                                              p * G::kXPlane);
                    }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 2; ++v) dw[u][v] = mma<2, PX>(a[u], c[v], dw[u][v]);
            }
        }
        // ---- dx = direct + dz W: wave w forms 32 inputs over the 128 channels of one
        // gate (its weights are read once), steps 32 m + lane % 32, channels (k)
        // 16 ks + 8 (lane / 32) .. + 7; the gates' parts meet in the fp32 tile
        // (both blocks of 32 steps always: rows past L are dropped by the stores' range
        // check, and a branch here would blur the wait counts)
        {
            const int ln = fresh(lane);
            const int kr = 8 * (ln >> 5) + ((ln >> 2) & 3);
            const int st = 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
            const int base = (gate * D + kr) * (TS * 2) + (((st >> 3) ^ swzdz(kr)) << 4) +
                             (st & 7) * 2;
            // o[0]: the block that the other gate's wave stores, o[1]: this wave's own
            f16v o[2], zero;
#pragma unroll
            for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int ob = base ^ ((m == gate ? 1 : 0) << 6);  // steps + 32: chunk bit 2
                    b8 a[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        a[p] = tr_pair(dzp + ob + ks * (16 * TS * 2) + p * G::kDzPlane,
                                       dzp + (ob ^ 16) + ks * (16 * TS * 2) + 4 * TS * 2 +
                                           p * G::kDzPlane);
                    o[m] = mma<2, PW>(a, wf[ks & 3], ks == 0 ? zero : o[m]);
                }
                // the freed slots take the next tile's first z fragments (asked for after
                // dx's stores, they would wait for those)
                if (ks < 4)
                    load_w(prs, 16 * nb + 8 * gate, ks + 4, ln);
                else
                    load_w(zrs, 8 * w, ks - 4, ln);
                __builtin_amdgcn_sched_barrier(0x38F);
            }
            const __amdgpu_buffer_rsrc_t drs = rsrc((char*)P.dx + b * P.L * D * EX, xbytes);
            const int col = 32 * nb + (ln & 31), r0 = 4 * (ln >> 5);
            // swz32 of row 32 m + r0 + 8 (v / 4) + v % 4: 4 (v / 4), and 8 for the upper half
            const int dbase = r0 * (D * 4) + (((col >> 2) ^ swz32(r0)) << 4) + (col & 3) * 4;
            const auto rp = [&](int m, int v) {
                return (float*)(raw + (dbase ^ ((v / 4) << 6)) +
                                (32 * m + 8 * (v / 4) + (v & 3)) * (D * 4));
            };
#pragma unroll
            for (int v = 0; v < 16; ++v) *rp(1 - gate, v) += o[0][v];
            lds_barrier();
            if constexpr (GATE) {
#pragma unroll
                for (int v = 0; v < 16; ++v) *rp(gate, v) += o[1][v];
            } else {
                const uint32_t off = (uint32_t)((t0 + 32 * gate + r0) * D + col) * EX;
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    bstore<TX>(drs, off + (8 * (v / 4) + (v & 3)) * D * EX,
                               *rp(gate, v) + o[1][v]);
            }
        }
        lds_barrier();  // every wave is done with the tile's planes
        if constexpr (GATE) {
            if (has_next) {
                fetch_hx(nrow, ns);
                fetch(nrow, ns);
            }
            if (lim == TS)
                conv_back(b, s, std::true_type{});
            else
                conv_back(b, s, std::false_type{});
        }
        if (!has_next) break;
        stage();
        lds_barrier();
        b = nrow;
        s = ns;
    }

    // ---- this workgroup's partial sums
    const int rho = lane >> 4, ch = 16 * w + (lane & 15);
    float* const pw = P.part_w + (int64_t)blockIdx.x * 2 * D * D;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 64 * wm + 32 * u + 8 * (v / 4) + 4 * (lane >> 5) + (v & 3);
                const int col = 64 * wn + 32 * c + (lane & 31);
                pw[row * D + col] = dw[u][c][v];
            }
    float* const pc = P.part_c + (int64_t)blockIdx.x * G::kCols * D;
    if constexpr (GATE) {
        total += (double)row_sums(0.0f, 0.0f, 0.0f, dcb);
        pc[(4 + rho) * D + ch] = (float)total_w;
    }
    if (GATE || rho < 3) pc[rho * D + ch] = (float)total;
}

// The weights in fragment order, as bf16 hi and lo planes (bf16 weights: one).
// pz: [wave 8][k-step 8][plane][lane][8]: column lane % 32 of wave w is z_r of
// channel 16 w + lane % 16 (lane % 32 < 16) or its z_i, k = 16 step + 8 (lane / 32) + e.
// px: [block 4][k-step 16][plane][lane][8]: input 32 block + lane % 32, k (output:
// W_r's rows, then W_i's) = 16 step + 8 (lane / 32) + e.
template <typename TW>
__global__ __launch_bounds__(256) void pack_kernel(const TW* __restrict__ wr,
                                                   const TW* __restrict__ wi, uint16_t* pz,
                                                   uint16_t* px) {
    constexpr int PW = sizeof(TW) == 4 ? 2 : 1;
    const int e = blockIdx.x * 256 + threadIdx.x;  // one of 2 * 2 D D elements
    const bool z = e < 2 * D * D;
    const int k = (z ? e : e - 2 * D * D);
    const int el = k & 7, lane = (k >> 3) & 63, rest = k >> 9;
    float v;
    if (z) {
        const int step = rest & 7, w = rest >> 3, col = lane & 31;
        const TW* src = col < 16 ? wr : wi;
        v = load(src + (16 * w + (col & 15)) * D + 16 * step + 8 * (lane >> 5) + el);
    } else {
        const int step = rest & 15, blk = rest >> 4;
        const int o = 16 * step + 8 * (lane >> 5) + el, in = 32 * blk + (lane & 31);
        v = load((o < D ? wr : wi) + (o & (D - 1)) * D + in);
    }
    uint16_t* dst = (z ? pz : px) + ((int64_t)rest * PW * 64 + lane) * 8 + el;
    const bf16 hi = from_f32<bf16>(v);
    dst[0] = hi.bits;
    if constexpr (PW == 2) dst[64 * 8] = from_f32<bf16>(v - to_f32(hi)).bits;
}

// dW, db and dLambda from the workgroups' partials, in double and in a fixed
// order: 16 groups of rows, each in ascending order, then the groups.
__global__ __launch_bounds__(256) void reduce_kernel(const float* __restrict__ part_w,
                                                     const float* __restrict__ part_c, int rows,
                                                     const float* __restrict__ lam, float* dwr,
                                                     float* dwi, float* dbr, float* dbi,
                                                     float* dlambda, int cols, float* dcw,
                                                     float* dcb, int K) {
    constexpr int kCols = 16, kGroups = 16;  // 16 x 4 columns a block, 16 row groups
    __shared__ double red[kGroups][kCols * 4];
    const int c = threadIdx.x % kCols, g = threadIdx.x / kCols;
    constexpr int kWBlocks = 2 * D * D / (kCols * 4);
    const bool isw = blockIdx.x < kWBlocks;
    const int64_t col = ((int64_t)(isw ? blockIdx.x : blockIdx.x - kWBlocks) * kCols + c) * 4;
    const float* src = (isw ? part_w : part_c) + col;
    const int64_t stride = isw ? 2 * D * D : cols * D;
    const int per = (rows + kGroups - 1) / kGroups;
    const int r0 = g * per, r1 = r0 + per < rows ? r0 + per : rows;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int r = r0; r < r1; ++r) {
        const f4 v = *(const f4*)(src + r * stride);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += (double)v[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) red[g][c * 4 + k] = acc[k];
    __syncthreads();
    if (threadIdx.x >= kCols * 4) return;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kGroups; ++q) s += red[q][threadIdx.x];
    const int64_t o = (int64_t)(isw ? blockIdx.x : blockIdx.x - kWBlocks) * kCols * 4 + threadIdx.x;
    if (isw) {
        if (o < D * D) dwr[o] = (float)s;
        else dwi[o - D * D] = (float)s;
    } else if (o < D) {
        dbr[o] = (float)s;
    } else if (o < 2 * D) {
        dbi[o - D] = (float)s;
    } else if (o < 3 * D) {
        const double lv = (double)lam[o - 2 * D];
        dlambda[o - 2 * D] = (float)(s / (1.0 + exp(-lv)));
    } else if (o < 4 * D) {
        if (dcb) dcb[o - 3 * D] = (float)s;
    } else {
        const int64_t j = (o - 4 * D) / D, d = (o - 4 * D) % D;
        if (j < K) dcw[d * K + j] = (float)s;
    }
}

constexpr int kMaxGroups = 256;  // workgroups: one per compute unit
constexpr int kMaxCols = Geo<float, float, true>::kCols;

constexpr size_t pack_bytes(int planes) { return (size_t)2 * D * D * 2 * planes; }

template <typename TX, typename TH, typename TW, bool GATE>
hipError_t launch(const Params& P, int grid, hipStream_t stream) {
    auto kern = fused_bwd_kernel<TX, TH, TW, GATE>;
    constexpr int smem = Geo<TX, TW, GATE>::kSmem;
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t e = allow_dynamic_lds((const void*)kern, smem, lds_set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NT), smem, stream, P);
    return hipGetLastError();
}

}  // namespace fbw

bool fused2_backward_applies(int64_t B, int64_t L, int64_t D, IoType io, const void* x,
                             const void* h, const void* dx, bool gated) {
    if (D != fbw::D || B <= 0 || L <= 0 || (gated && io != IoType::kF32)) return false;
    if (((uintptr_t)x | (uintptr_t)h | (uintptr_t)dx) % 16 != 0) return false;
    if ((L + fbw::TS) * D * (int64_t)io_bytes(io) >= ((int64_t)1 << 31)) return false;
    // A workgroup walks whole rows, 256 of them in a round, and a step of a round takes
    // 0.16 us (fp32; gated 0.22, bf16 0.12) with few rows and 0.22 (0.30, 0.16) with all
    // 256; the separate kernels take 1.32 ns (1.99, 0.98) a row and step and 5 to 20 us
    // more for their launches.  So a part-filled last round pays from about 142 rows on, a
    // full round before it makes up for 110 rows of that, and the launches for
    // kSaved row-steps (steps in whole tiles).  Backward, separate kernels -> this one, us
    // (fp32 layer / bf16 layer / gated):
    //   rows x steps   taken                                 not taken
    //   32 x 64        32 -> 27, 30 -> 28, 69 -> 29
    //   32 x 200       -, -, 78 -> 65                        38 -> 50, 36 -> 41
    //   128 x 1024     203 -> 187, 153 -> 144, 308 -> 265
    //   128 x 8192     -                    1427 -> 1480, 1049 -> 1114, 2084 -> 2105
    //   256 x 2048     691 -> 459, 514 -> 338, 1044 -> 612
    //   257 x 2048     -                       718 -> 780, 530 -> 594, 1053 -> 1065
    //   300 x 2048     844 -> 795, 624 -> 598, 1237 -> 1088
    const int64_t rows = B % fbw::kMaxGroups, rounds = B / fbw::kMaxGroups;
    const int64_t steps = (L + fbw::TS - 1) / fbw::TS * fbw::TS;
    const int64_t kSaved = gated ? 34000 : io == IoType::kF32 ? 14400 : 16200;
    return rows == 0 || (142 - rows - 110 * rounds) * steps <= kSaved;
}

size_t fused2_backward_workspace(int64_t B, int64_t L, int64_t D) {
    if (D != fbw::D || B <= 0 || L <= 0) return 0;
    const size_t grid = (size_t)(B < fbw::kMaxGroups ? B : fbw::kMaxGroups);
    return 2 * fbw::pack_bytes(2) + grid * (2 * D * D + fbw::kMaxCols * D) * sizeof(float);
}

hipError_t launch_fused2_backward(const Fused2BwdArgs& a, hipStream_t stream) {
    using namespace fbw;
    const int grid = (int)(a.B < kMaxGroups ? a.B : kMaxGroups);
    char* const pz = (char*)a.ws;
    char* const px = pz + pack_bytes(2);
    float* const part_w = (float*)(px + pack_bytes(2));
    float* const part_c = part_w + (size_t)grid * 2 * D * D;
    const bool f32 = a.io == IoType::kF32;
    const dim3 pgrid(4 * D * D / 256);
    if (f32)
        hipLaunchKernelGGL(pack_kernel<float>, pgrid, dim3(256), 0, stream, (const float*)a.wr,
                           (const float*)a.wi, (uint16_t*)pz, (uint16_t*)px);
    else
        hipLaunchKernelGGL(pack_kernel<bf16>, pgrid, dim3(256), 0, stream, (const bf16*)a.wr,
                           (const bf16*)a.wi, (uint16_t*)pz, (uint16_t*)px);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const Params P{a.x,  a.h,  a.gy ? a.gy : a.dh, a.gz, a.gdz, a.dx,   a.h0,   a.dhT, a.dh0,
                   pz,   px,   a.br,               a.bi, a.lambda, part_w, part_c, a.L,  a.B,
                   a.cw, a.cb, a.K};
    if (a.gy)
        e = launch<float, float, float, true>(P, grid, stream);
    else if (f32)
        e = launch<float, float, float, false>(P, grid, stream);
    else
        e = launch<bf16, bf16, bf16, false>(P, grid, stream);
    if (e != hipSuccess) return e;
    const int cols = a.gy ? kMaxCols : 3;
    hipLaunchKernelGGL(reduce_kernel, dim3(2 * D * D / 64 + cols * D / 64), dim3(256), 0, stream,
                       part_w, part_c, grid, a.lambda, a.dwr, a.dwi, a.dbr, a.dbi, a.dlambda, cols,
                       a.dcw, a.dcb, a.K);
    return hipGetLastError();
}

}  // namespace recblr
