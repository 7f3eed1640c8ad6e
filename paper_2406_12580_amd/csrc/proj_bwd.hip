// Both gradient products of the gate projections (section 3.2) in one pass over
// dz, for D in {64, 128, 192, 256}:
//   dx += [dz_r | dz_i] [W_r; W_i]   and   [dW_r; dW_i] = [dz_r | dz_i]^T x,
// db = column sums of dz.  dz (fp32, 8 bytes an element: the largest stream of
// the layer backward) is read once instead of once per product.
//
// Work decomposition.  The M rows are split into contiguous ranges and the D
// inputs into column blocks of 32 CB (D = 256: two of 128, whose dW, 512 x 128
// fp32, takes half of the register file; the two workgroups of a range sit on one
// XCD and read the same dz through its L2).  A workgroup of 8 waves walks its
// range in tiles of 32 rows:
//   * dz rows become bf16 hi and lo planes [row][2 D] in LDS (two buffers: the next
//     tile's are staged while this one is multiplied), x its planes [row][32 CB];
//   * dW += dz^T x over the 32 rows, accumulators in registers for the whole
//     range; both operands run across LDS rows and are read through the
//     transposing LDS loads;
//   * dx: wave w forms 32 columns over one gate's K = D (W fragments streamed from
//     L2 in fragment order), the two gates' parts meet in LDS, and the sum with
//     dx's direct term goes back to memory.
// fp32 operands take the 3-term bf16 split (hi*hi + hi*lo + lo*hi), bf16 ones are
// one exact plane.  dW and db leave as one fp32 partial per range, summed in
// double in a fixed order.
//
// What bounds it at D = 256, M = 262144, bf16 (0.80 GB: 155 us at copy speed): 317
// us, of which the matrix cores are busy for 140 us and the splitting of dz, done by
// both column blocks, for about as long; the two products in kernels of their own
// (gemm.hip) take 220 + 181 us.  Two barriers a tile and dz staged before the first
// of them let one wave's splitting run beside another's products: with one tile
// buffer and three barriers 370 us.
#include "device_common.hpp"
#include "gemm.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"
#include "wave_tile.hpp"

namespace recblr {
namespace pbw {

using namespace wtile;

constexpr int TR = 32;             // rows per tile
constexpr int NW = 8, NT = NW * kWave;

struct Params {
    const float* dzr;
    const float* dzi;
    const void* x;     // TX
    void* dx;          // TD, direct term on entry
    const void* pw;    // W in fragment order (launch_prepare_scan)
    float* part_w;     // [ranges][2 D][D]
    float* part_b;     // [ranges][2 D]
    int64_t M, ranges, rows;  // rows: per range (a multiple of TR)
};

template <int D>
struct Geo {
    // 32-column blocks of a workgroup
    static constexpr int CB = D == 256 ? 4 : D == 192 ? 3 : D / 32;
    static constexpr int NCB = D / (32 * CB);                        // column blocks
    static constexpr int OB = 2 * D / 32;                            // 32-row blocks of dW
    static constexpr int PO = (OB + NW - 1) / NW;                    // of a wave
    static constexpr int WO = OB / PO;                               // waves along dW's rows
    static constexpr int WC = NW / WO < CB ? (NW / WO < 1 ? 1 : NW / WO) : CB;  // along its columns
    static constexpr int PC = CB / WC;                               // 32-column blocks of a wave
    static constexpr int kDzPlane = TR * 2 * D * 2;
    static constexpr int kXPlane = TR * 256;                         // rows of 128 inputs at most
    static constexpr int kX = 32 * CB * TR * 4;                      // the exchange: half of dx
    static constexpr int kExch = kX / 2 * 2;
    static constexpr int QPR = D / 4;                                // quads of a row of one dz
    static constexpr int kQuads = TR * QPR / NT;                     // of a thread
    static constexpr int kPer = D == 192 ? 3 : 1;                    // distinct columns of a thread
    static_assert(kQuads * NT == TR * QPR && WO * PO == OB && WC * PC == CB, "whole blocks");
    static constexpr size_t smem(int px) { return 2 * 2 * kDzPlane + px * kXPlane + kExch; }
};

// Chunk j of row r of a plane at j ^ swz(r): the 16 rows of one pass of a row
// fragment read land on distinct chunks, the four rows x 64 bytes of a
// transposing read in distinct 64-byte groups.
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

template <typename TX, typename TW, typename TD, int D>
__global__ __launch_bounds__(NT, 2) void dxdw_kernel(Params P) {
    using G = Geo<D>;
    constexpr int PX = sizeof(TX) == 4 ? 2 : 1, PW = sizeof(TW) == 4 ? 2 : 1;
    constexpr int EX = (int)sizeof(TX), ED = (int)sizeof(TD);
    constexpr int kRing = PW == 2 ? 2 : 4;  // W k-steps in flight
    constexpr int kXq = 32 * G::CB * TR * EX / 16;  // 16-byte chunks of an x tile
    constexpr int kXl = (kXq + NT - 1) / NT;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const dz0 = smem;                                   // [2][hi, lo][TR][2 D]
    char* const xpl = smem + 4 * G::kDzPlane;                 // [PX][TR][128]
    float* const exch = (float*)(xpl + PX * G::kXPlane);      // [CB][2][8][64 lanes]
    const int lane = threadIdx.x & (kWave - 1), w = wave_id();
    // Workgroups 8 apart (one XCD) take the column blocks of one range.
    const int64_t rg = blockIdx.x / (8 * G::NCB) * 8 + blockIdx.x % 8;
    const int cb = (int)(blockIdx.x / 8 % G::NCB);
    const int64_t row0 = rg * P.rows;
    const int64_t row1 = row0 + P.rows < P.M ? row0 + P.rows : P.M;
    if (rg >= P.ranges || row0 >= row1) return;

    // dW blocks of this wave: rows 32 PO wo .., columns 32 PC wc ..
    const int wo = w % G::WO, wc = w / G::WO;
    const bool dw_on = wc < G::WC;
    // dx block: 32 columns, one gate
    const int nb = w % G::CB, gate = w / G::CB;
    const bool dx_on = gate < 2;

    f16v dw[G::PO][G::PC];
#pragma unroll
    for (int a = 0; a < G::PO; ++a)
#pragma unroll
        for (int c = 0; c < G::PC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) dw[a][c][v] = 0.0f;
    float dbs[2][G::kPer][4];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int p = 0; p < G::kPer; ++p)
#pragma unroll
            for (int k = 0; k < 4; ++k) dbs[g][p][k] = 0.0f;

    const __amdgpu_buffer_rsrc_t prs = rsrc(P.pw, (uint32_t)(2 * D * D * 2 * PW));
    const int wbase = ((cb * G::CB + nb) * (2 * D / 16) + gate * (D / 16)) * PW * kWave * 16;
    b8 wf[kRing][PW];
    auto load_w = [&](int ks, int ln) {
#pragma unroll
        for (int p = 0; p < PW; ++p)
            wf[ks % kRing][p] = __builtin_bit_cast(
                b8, __builtin_amdgcn_raw_buffer_load_b128(prs, ln * 16,
                                                          wbase + (ks * PW + p) * kWave * 16, 0));
    };

    u4v zq[2][G::kQuads];
    u4v xq[kXl];
    auto fetch = [&](int64_t m) {  // rows past the range read as zero
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
        const __amdgpu_buffer_rsrc_t rr = rsrc(P.dzr + m * D, n > 0 ? (uint32_t)(n * D * 4) : 0u);
        const __amdgpu_buffer_rsrc_t ri = rsrc(P.dzi + m * D, n > 0 ? (uint32_t)(n * D * 4) : 0u);
        const __amdgpu_buffer_rsrc_t rx =
            rsrc((const char*)P.x + m * D * EX, n > 0 ? (uint32_t)(n * D * EX) : 0u);
#pragma unroll
        for (int q = 0; q < G::kQuads; ++q) {
            zq[0][q] = __builtin_amdgcn_raw_buffer_load_b128(rr, (q * NT + tid) * 16, 0, 0);
            zq[1][q] = __builtin_amdgcn_raw_buffer_load_b128(ri, (q * NT + tid) * 16, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < kXl; ++q) {
            const int o = q * NT + tid;
            constexpr int cpr = 32 * G::CB * EX / 16;
            const int r = o / cpr, c = o % cpr;
            xq[q] = __builtin_amdgcn_raw_buffer_load_b128(
                rx, o < kXq ? (uint32_t)((r * D + cb * 32 * G::CB) * EX + c * 16) : 0x7FFFFFFFu, 0,
                0);
        }
    };
    auto stage_dz = [&](char* dzp) {
        const int ln = fresh(lane) & 63;
        const int tid = w * kWave + ln;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float s[G::kPer][4];
#pragma unroll
            for (int p = 0; p < G::kPer; ++p)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[p][k] = 0.0f;
#pragma unroll
            for (int q = 0; q < G::kQuads; ++q) {
                // where rows are whole fractions of a wave, the wave's part of the row is scalar
                const int o = q * NT + tid;
                const int r = kWave % G::QPR == 0 ? (q * NT + w * kWave) / G::QPR + ln / G::QPR
                                                  : o / G::QPR;
                const int c = (kWave % G::QPR == 0 ? ln : o) % G::QPR + g * G::QPR;
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = __uint_as_float(zq[g][q][k]);
                const fastmm::u2v p0 = fastmm::split2(v[0], v[1]), p1 = fastmm::split2(v[2], v[3]);
                char* const dst = dzp + r * (2 * D * 2) + (((c >> 1) ^ swz(r)) << 4) + (c & 1) * 8;
                *(u2v*)dst = u2v{p0.x, p1.x};
                *(u2v*)(dst + G::kDzPlane) = u2v{p0.y, p1.y};
#pragma unroll
                for (int k = 0; k < 4; ++k) s[q % G::kPer][k] += v[k];
            }
#pragma unroll
            for (int p = 0; p < G::kPer; ++p)
#pragma unroll
                for (int k = 0; k < 4; ++k) dbs[g][p][k] += s[p][k];
        }
    };
    auto stage_x = [&]() {
        const int ln = fresh(lane);
        const int tid = w * kWave + ln;
#pragma unroll
        for (int q = 0; q < kXl; ++q) {
            const int o = q * NT + tid;
            if (kXq % NT != 0 && o >= kXq) break;
            constexpr int cpr = 32 * G::CB * EX / 16;
            const int r = o / cpr, c = o % cpr;
            if constexpr (PX == 2) {
                const auto f = [](uint32_t u) { return __uint_as_float(u); };
                const fastmm::u2v p0 = fastmm::split2(f(xq[q][0]), f(xq[q][1])),
                                  p1 = fastmm::split2(f(xq[q][2]), f(xq[q][3]));
                char* const dst = xpl + r * 256 + (((c >> 1) ^ swz(r)) << 4) + (c & 1) * 8;
                *(u2v*)dst = u2v{p0.x, p1.x};
                *(u2v*)(dst + G::kXPlane) = u2v{p0.y, p1.y};
            } else {
                *(u4v*)(xpl + r * 256 + ((c ^ swz(r)) << 4)) = xq[q];
            }
        }
    };

    fetch(row0);
    stage_dz(dz0);
    stage_x();
    if (dx_on) {
#pragma unroll
        for (int ks = 0; ks < kRing; ++ks) load_w(ks, lane);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing pending enters the loop
    lds_barrier();
    int par = 0;
    // dx of this wave's half block: the direct term on its way in, the result on its way out
    float dd[8];
    auto dx_off = [&](int ln) {
        return dx_on ? (uint32_t)(((16 * gate + 4 * (ln >> 5)) * D + cb * 32 * G::CB + 32 * nb +
                                   (ln & 31)) * ED)
                     : 0x7FFFFF00u;  // past the resource
    };
    auto dx_rsrc = [&](int64_t m) {
        const int64_t n = row1 - m < TR ? row1 - m : TR;
        return rsrc((char*)P.dx + m * D * ED, (uint32_t)(n * D * ED));
    };
    auto load_dx = [&](int64_t m) {
        const __amdgpu_buffer_rsrc_t drs = dx_rsrc(m);
        const uint32_t off = dx_off(fresh(lane));
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const uint32_t o = off + (8 * (v / 4) + (v & 3)) * D * ED;
            if constexpr (ED == 4)
                dd[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(drs, o, 0, 0));
            else
                dd[v] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(drs, o, 0, 0)
                                        << 16);
        }
    };
    auto store_dx = [&](int64_t m) {
        const __amdgpu_buffer_rsrc_t drs = dx_rsrc(m);
        const uint32_t off = dx_off(fresh(lane));
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const uint32_t o = off + (8 * (v / 4) + (v & 3)) * D * ED;
            if constexpr (ED == 4)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dd[v]), drs, o, 0, 0);
            else
                __builtin_amdgcn_raw_buffer_store_b16(from_f32<bf16>(dd[v]).bits, drs, o, 0, 0);
        }
    };

    // Vector memory completes in order, so everything slow (the last tile's stores,
    // this one's direct term, the next one's loads) is issued after dx's weight
    // fragments and is in flight through dW's products.
    for (int64_t m = row0; m < row1; m += TR, par ^= 1) {
        char* const dzp = dz0 + par * 2 * G::kDzPlane;
        // ---- dx: this gate's part
        f16v o, zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
        if (dx_on) {
            const int ln = fresh(lane);
            const int r = ln & 31;
            const int base = r * (2 * D * 2) + (((ln >> 5) ^ swz(r)) << 4);
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) {
                b8 a[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    // even first chunk of the k-step: XOR below 16 chunks, then steps of 256
                    const int k = gate * (D / 8) + 2 * ks;
                    a[p] = *(const b8*)(dzp + (base ^ ((k & 15) << 4)) + (k >> 4) * 256 +
                                        p * G::kDzPlane);
                }
                o = mma<2, PW>(a, wf[ks % kRing], ks == 0 ? zero : o);
                load_w((ks + kRing) % (D / 16), ln);  // past the end: the next tile's first
                __builtin_amdgcn_sched_barrier(0x38F);
            }
            // the half of the rows that the other gate's wave stores
            float* const e = exch + ((nb * 2 + 1 - gate) * 8) * kWave + ln;
#pragma unroll
            for (int v = 0; v < 8; ++v) e[v * kWave] = gate ? o[v] : o[8 + v];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (m > row0) store_dx(m - TR);
        load_dx(m);
        fetch(m + TR);
        __builtin_amdgcn_sched_barrier(0);
        // ---- dW += dz^T x
        if (dw_on) {
            const int ln = fresh(lane);
            const int kr = 8 * (ln >> 5) + ((ln >> 2) & 3);
            const int oc = 32 * G::PO * wo + 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
            const int ic = 32 * G::PC * wc + 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
            const int ab = kr * (2 * D * 2) + (((oc >> 3) ^ swz(kr)) << 4) + (oc & 7) * 2;
            const int xb = kr * 256 + (((ic >> 3) ^ swz(kr)) << 4) + (ic & 7) * 2;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {  // rows + 16: swz unchanged; + 4: its bit 0
                b8 a[G::PO][2], c[G::PC][PX];
#pragma unroll
                for (int u = 0; u < G::PO; ++u)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int o = ab ^ ((u & 3) << 6);
                        const int k = ks * (16 * 2 * D * 2) + p * G::kDzPlane + (u >> 2) * 256;
                        a[u][p] = tr_pair(dzp + o + k, dzp + (o ^ 16) + k + 4 * 2 * D * 2);
                    }
#pragma unroll
                for (int v = 0; v < G::PC; ++v)
#pragma unroll
                    for (int p = 0; p < PX; ++p) {
                        const int o = xb ^ (v << 6);
                        const int k = ks * (16 * 256) + p * G::kXPlane;
                        c[v][p] = tr_pair(xpl + o + k, xpl + (o ^ 16) + k + 4 * 256);
                    }
#pragma unroll
                for (int u = 0; u < G::PO; ++u)
#pragma unroll
                    for (int v = 0; v < G::PC; ++v) dw[u][v] = mma<2, PX>(a[u], c[v], dw[u][v]);
            }
        }
        stage_dz(dz0 + (par ^ 1) * 2 * G::kDzPlane);
        lds_barrier();
        if (dx_on) {
            const float* const e = exch + ((nb * 2 + gate) * 8) * kWave + fresh(lane);
#pragma unroll
            for (int v = 0; v < 8; ++v) {  // direct term + (gate r's part + gate i's part)
                const float own = gate ? o[8 + v] : o[v], other = e[v * kWave];
                dd[v] += own + other;
            }
        }
        stage_x();
        lds_barrier();
    }
    store_dx(row0 + (row1 - row0 - 1) / TR * TR);

    // ---- partial sums of this range
    if (dw_on) {
        float* const pw = P.part_w + rg * 2 * D * D + cb * 32 * G::CB;
#pragma unroll
        for (int u = 0; u < G::PO; ++u)
#pragma unroll
            for (int c = 0; c < G::PC; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 32 * (G::PO * wo + u) + 8 * (v / 4) + 4 * (lane >> 5) + (v & 3);
                    pw[row * D + 32 * (G::PC * wc + c) + (lane & 31)] = dw[u][c][v];
                }
    }
    if (cb == 0) {  // db: the threads that hold a column, in order
        float* const red = (float*)smem;  // [NT][2][kPer][4]: free after the last barrier
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int p = 0; p < G::kPer; ++p)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    red[((threadIdx.x * 2 + g) * G::kPer + p) * 4 + k] = dbs[g][p][k];
        lds_barrier();
        for (int c = threadIdx.x; c < 2 * D; c += NT) {
            const int g = c / D, quad = c % D / 4;
            float s = 0.0f;
            for (int p = 0; p < G::kPer; ++p)  // thread t's p-th quad: (p NT + t) % QPR
                for (int t = (quad + G::kPer * NT * G::QPR - p * NT) % G::QPR; t < NT; t += G::QPR)
                    s += red[((t * 2 + g) * G::kPer + p) * 4 + c % 4];
            P.part_b[rg * 2 * D + c] = s;
        }
    }
}

struct Split {
    int64_t ranges, rows;
};
// One workgroup per compute unit (two at D = 64, whose dW is small), and at least two
// tiles a range: each range leaves a partial dW to sum, but few ranges leave the chip
// idle.  Layer forward + backward, bf16, with at least 256, 64 and 32 rows a range: 4000
// rows of D = 256 78, 64 and 67 us; 8000 of D = 128 66, 55 and 56; 20000 of D = 64 53,
// 47 and 47.
constexpr int64_t kMinRows = 2 * TR;
Split split(int64_t M, int64_t D) {
    const int64_t ncb = D == 256 || D == 192 ? 2 : 1;
    const int64_t most = (D == 64 ? 512 : 256) / ncb;
    int64_t n = (M + kMinRows - 1) / kMinRows;
    n = n < most ? n : most;
    const int64_t rows = ((M + n - 1) / n + TR - 1) / TR * TR;
    return Split{(M + rows - 1) / rows, rows};
}

template <typename TX, typename TW, typename TD, int D>
hipError_t launch_d(const Params& P, hipStream_t stream) {
    auto kern = dxdw_kernel<TX, TW, TD, D>;
    constexpr int smem = (int)Geo<D>::smem(sizeof(TX) == 4 ? 2 : 1);
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t e = allow_dynamic_lds((const void*)kern, smem, lds_set);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)((P.ranges + 7) / 8 * 8 * Geo<D>::NCB);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), smem, stream, P);
    return hipGetLastError();
}

template <typename TX, typename TW, typename TD>
hipError_t launch(int64_t D, const Params& P, hipStream_t stream) {
    switch (D) {
        case 64: return launch_d<TX, TW, TD, 64>(P, stream);
        case 128: return launch_d<TX, TW, TD, 128>(P, stream);
        case 192: return launch_d<TX, TW, TD, 192>(P, stream);
        default: break;
    }
    if constexpr (sizeof(TX) == 2) {
        if (D == 256) return launch_d<TX, TW, TD, 256>(P, stream);
    }
    return hipErrorInvalidValue;
}

// Where one pass is the faster one (the whole layer or gated step, us, two kernels
// -> this one):
//   bf16 x, every D: layer, M = 600 to 131072: D = 64 61 -> 57 and 90 -> 81, D = 128
//     (M = 8192) 72 -> 66, D = 192 (M = 65536) 207 -> 199, D = 256 (M = 131072) 472 -> 437;
//   fp32 x, D = 64: layer 62 -> 55 (M = 600) and 108 -> 88 (65536), gated 125 -> 112 and
//     194 -> 173; D = 128 likewise;
//   fp32 x, D = 192: layer 79 -> 82 at M = 600, 96 -> 96 at 8192, 173 -> 161 at 28749,
//     gated 441 -> 419 at 65536: from 16384 rows on;
//   fp32 x, D = 256: never (725 -> 765 at M = 131072): both planes of x and three
//     products a block do not fit beside 256 accumulators.
bool takes(int64_t M, int64_t D, IoType x_io) {
    if (M <= 0) return false;
    if (D == 64 || D == 128) return true;
    if (D == 192) return x_io == IoType::kBf16 || M >= 16384;
    return D == 256 && x_io == IoType::kBf16;
}

}  // namespace pbw

bool project_backward_both_applies(int64_t M, int64_t D, IoType x_io, const void* dzr,
                                   const void* dzi, const void* x, const void* dx,
                                   const void* ws) {
    const uintptr_t a =
        (uintptr_t)dzr | (uintptr_t)dzi | (uintptr_t)x | (uintptr_t)dx | (uintptr_t)ws;
    return pbw::takes(M, D, x_io) && a % 16 == 0;  // 16-byte loads and stores
}

size_t project_backward_both_workspace(int64_t M, int64_t D) {
    if (!pbw::takes(M, D, IoType::kF32) && !pbw::takes(M, D, IoType::kBf16)) return 0;
    return (size_t)pbw::split(M, D).ranges * (size_t)(2 * D * D + 2 * D) * sizeof(float);
}

hipError_t launch_project_backward_both(const float* dzr, const float* dzi, const void* x,
                                        const void* pack, void* dx, float* dwr, float* dbr,
                                        float* dwi, float* dbi, int64_t M, int64_t D, IoType x_io,
                                        IoType w_io, void* ws, const DlambdaRows& dl,
                                        hipStream_t stream) {
    const pbw::Split sp = pbw::split(M, D);
    float* const part_w = (float*)ws;
    float* const part_b = part_w + sp.ranges * 2 * D * D;
    const pbw::Params P{dzr, dzi, x, dx, pack, part_w, part_b, M, sp.ranges, sp.rows};
    hipError_t e;
    if (x_io == IoType::kBf16)
        e = pbw::launch<bf16, bf16, bf16>(D, P, stream);
    else if (w_io == IoType::kBf16)
        e = pbw::launch<float, bf16, float>(D, P, stream);
    else
        e = pbw::launch<float, float, float>(D, P, stream);
    if (e != hipSuccess) return e;
    return launch_dw_reduce(part_w, part_b, sp.ranges, D, dwr, dbr, dwi, dbi, dl, stream);
}

}  // namespace recblr
