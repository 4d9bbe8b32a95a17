// Matrix-core kernels of the learned surrogate: 3x3x3 "valid" convolutions over
// channels-last BF16 grids with FP32 accumulation (v_mfma_f32_32x32x16_bf16), their
// two gradients, the loss and the Adam update. A method addition: the paper has no
// surrogate; the network and its training are defined in the public header.
//
// Every layer is an implicit GEMM. Forward: rows = output nodes, columns = the 32
// (padded) output channels, reduction over 27 taps x input channels, weights in
// registers; on wide grids the input marches through LDS by planes (k_conv_fwd_zm), on
// narrower ones rows of output nodes share three staged planes (k_conv_rows).
// Input gradient: rows = input nodes, columns = input channels, reduction over taps x
// output channels (the transposed weights), by k_conv_rows too. Weight gradient: one
// 32 x 32 tile (input x output channels) per tap, reduction over nodes staged in LDS
// and read transposed; partial sums meet in FP32 atomics (k_conv_wgrad).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace lbfd {
namespace sg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16;

constexpr int NL = 4;                                  // layers
constexpr int CO = 32;                                 // padded output channels of every layer
constexpr int CIN_REAL[NL] = {6, 32, 32, 32};
constexpr int CIN_PAD[NL] = {16, 32, 32, 32};
constexpr int COUT_REAL[NL] = {32, 32, 32, 7};
constexpr int NOUT = 7;                                // network outputs: 3 + 3 flux coefficients, the exchange
constexpr int IN_CH = 16;                              // channels of an input grid (6 used)

__host__ __device__ constexpr long long layer_params(int l) { return 27LL * CIN_REAL[l] * COUT_REAL[l] + COUT_REAL[l]; }
__host__ __device__ constexpr long long n_params()
{
    return layer_params(0) + layer_params(1) + layer_params(2) + layer_params(3);
}

// Round to nearest even; NaN stays NaN.
__device__ __forceinline__ u16 f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}
__device__ __forceinline__ float bf2f(u16 h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 frag(const u16 *p) { return __builtin_bit_cast(bf16x8, *(const u32x4 *)p); }
__device__ __forceinline__ bf16x8 frag_zero() { return __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u}); }

// Row of the 32 x 32 result held by register r of a lane in lane group kg (the
// column is the lane index mod 32).
__device__ __forceinline__ int acc_row(int r, int kg) { return 8 * (r >> 2) + 4 * kg + (r & 3); }

// BF16 weights in fragment order: the 16 bytes of lane l for tap t and the c-th sixteen of the
// NC = CIN / 16 reduction channels are at ((t NC + c) 64 + l) 8, so a wavefront reads a
// fragment as 1 KB in a row (in rows of a channel each lane's 16 bytes sat 64 bytes from its
// neighbour's, four times the cache accesses).
__host__ __device__ constexpr long long frag_at(int t, int nc, int k, int col)
{
    return (((long long)t * nc + k / 16) * 64 + (k % 16) / 8 * 32 + col) * 8 + k % 8;
}

// Lane l gets v of lane l xor 32.
__device__ __forceinline__ float other_half(float v, bool low)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(low ? r[1] : r[0]);
}
template <int CTRL> __device__ __forceinline__ uint32_t quad_mov(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}

// Four rows of one channel in every lane -> four channels of one row: the lanes of a quad hold
// channels c .. c + 3 (c = lane column, a multiple of 4 at the first of them) of rows 0 .. 3;
// lane q of the quad ends with row q, channels c .. c + 3, rounded to BF16 (nearest even).
__device__ __forceinline__ uint2 quad_rows(float v0, float v1, float v2, float v3, int lane)
{
    const uint32_t p01 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)v0, (__bf16)v1});
    const uint32_t p23 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)v2, (__bf16)v3});
    // odd lanes take the odd row of the pair
    const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
    const uint32_t a = __builtin_amdgcn_perm(quad_mov<0xB1>(p01), p01, sel);
    const uint32_t b = __builtin_amdgcn_perm(quad_mov<0xB1>(p23), p23, sel);
    const bool hi = (lane & 2) != 0;
    const uint32_t got = quad_mov<0x4E>(hi ? a : b);
    return hi ? uint2{got, b} : uint2{a, got};
}

// Forward layer on wide grids: out[m][o] = act(b[o] + sum_{tap,i} in[m + tap][i] w[tap][i][o]).
// in: channels-last BF16, wb: BF16 in fragment order, out: BF16 [M][32], or with OUTF32 FP32
// [M][NOUT] (the first NOUT channels, no activation).
//
// A workgroup owns columns of ZX x ZY output nodes (x, y) over zc consecutive output planes;
// wavefront w computes output rows y0 + 2 w and y0 + 2 w + 1, which share every weight
// fragment. Input planes (ZY + 2 rows of 32 nodes) rotate through four LDS slots; each is
// fetched into registers two planes ahead of the one being computed. The three x-taps share
// one input fragment: for tap q the partial sums P_q[j] = sum in[x0 + j] w_q are kept per
// input node j of the row, and out[x0 + i] = P_0[i] + P_1[i + 1] + P_2[i + 2] (i < ZX = 30).
//
// Bound: the matrix cores, and the instructions issued between their own. So the weights of QR of
// the three x-taps stay in registers, as many as the vector registers hold without copies from
// the accumulation registers (which cost four instructions a product), and the others are read
// from LDS, once for two rows. A wavefront per SIMD is all the registers allow with 32 input
// channels, so nothing else hides what comes after the products: the shifted sum, bias,
// rounding and stores of a plane are issued between the matrix instructions of the next one
// (two sets of accumulators), and the shift by one and two rows is a register renaming but
// for every fourth row (a swap of the wavefront's halves), where it went through an LDS scratch.
// Columns are dealt to the XCDs in contiguous runs, whose neighbours share rows in one L2.
// 264^3 input nodes: 6 -> 32 channels 924 -> 572 us, 32 -> 32 1436 -> 1242 us (780 TFLOP/s; the
// matrix cores are busy half the cycles and the clock falls to 1.7 GHz under this
// load), 32 -> 7 686 -> 609 us.
constexpr int ZX = 30, ZY = 8;
// Workgroups that share a compute unit, and x-taps whose weights stay in registers.
template <int CIN> __host__ __device__ constexpr int zm_per_cu() { return CIN == 16 ? 2 : 1; }
template <int CIN, bool RELU, bool OUTF32>
__global__ __launch_bounds__(256, (zm_per_cu<CIN>())) void k_conv_fwd_zm(
    const u16 *__restrict__ in, const u16 *__restrict__ wb, const float *__restrict__ bias, void *__restrict__ out,
    int Di, int Hi, int Wi, int nbx, int nby, int nbz, int zc, long long ncol)
{
    constexpr int CP = CIN + 8;                   // node stride in LDS (elements)
    constexpr int PR = ZY + 2;                    // input rows of a plane
    constexpr int PLANE = PR * 32 * CP;           // elements of a plane slot
    constexpr int NC = CIN / 16;                  // reduction fragments per tap
    constexpr int PCS = CIN / 8;                  // 16-byte pieces per node
    constexpr int PIECES = PR * 32 * PCS;         // 16-byte pieces per plane
    constexpr int PPT = (PIECES + 255) / 256;     // pieces per thread
    __shared__ __attribute__((aligned(16))) u16 ring[4 * PLANE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int mr = lane & 31, kg = lane >> 5;
    const int Do = Di - 2, Ho = Hi - 2, Wo = Wi - 2;
    // The last layer (NOUT = 7 outputs) takes 16 x 16 x 32 matrix instructions: 16
    // output columns instead of 32, half the matrix work; every other layer 32 x 32 x 16.
    constexpr bool N16 = OUTF32;
    constexpr bool TWO = zm_per_cu<CIN>() == 1;   // two sets of accumulators
    constexpr int NCB = N16 ? CIN / 32 : NC;      // weight fragments per tap
    constexpr int QR = N16 ? 3 : 1, QL = 3 - QR;  // x-taps with weights in registers, in LDS
    const int l16 = lane & 15, k16 = lane >> 4;
    __shared__ __attribute__((aligned(16))) u16 wl[QL > 0 ? 9 * NCB * QL * 64 * 8 : 8];
    bf16x8 Bw[9][QR][NCB];
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
            const u16 *p = wb + (N16 ? frag_at(t, NC, c * 32 + k16 * 8, l16) : frag_at(t, NC, c * 16 + kg * 8, mr));
            const int ap = t / 3, q = t % 3;
            if (q < QR) Bw[ap][q][c] = frag(p);
            else if (wave == ap % 4) *(bf16x8 *)&wl[(((ap * NCB + c) * QL + q - QR) * 64 + lane) * 8] = frag(p);
        }
    const float bv = bias[N16 ? l16 : mr];
    const long long pstride = (long long)Hi * Wi * CIN;   // elements between input planes
    const long long oplane = (long long)Ho * Wo;
    // accumulators of a plane: per row P_q of 32 rows x 32 columns, or 2 x (16 x 16)
    struct Acc {
        f32x16 w[2][N16 ? 1 : 3];
        f32x4 n[2][N16 ? 3 : 1][2];
    };
    Acc s0, s1;
    // this XCD's run of columns
    const long long run = (ncol + 7) / 8, c0 = (long long)(blockIdx.x & 7u) * run;
    const long long cend = c0 + run < ncol ? c0 + run : ncol;
    for (long long col = c0 + (blockIdx.x >> 3); col < cend; col += gridDim.x >> 3) {
        long long r = col;
        const int bxi = (int)(r % nbx);
        r /= nbx;
        const int byi = (int)(r % nby);
        r /= nby;
        const int bzi = (int)(r % nbz);
        const long long b = r / nbz;
        const int x0 = bxi * ZX, y0 = byi * ZY, z0 = bzi * zc;
        const int nzo = min(zc, Do - z0);
        // this thread's pieces of a plane: offset from the column's first input node in
        // plane z0 (-1 outside the grid: zeros, which only reach outputs that are not
        // stored) and place in a slot
        const u16 *cbase = in + (((b * Di + z0) * Hi + y0) * (long long)Wi + x0) * CIN;
        int off[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            const int piece = i % PCS, node = i / PCS;
            const bool ok = i < PIECES && x0 + (node & 31) < Wi && y0 + (node >> 5) < Hi;
            off[k] = ok ? ((node >> 5) * Wi + (node & 31)) * CIN + piece * 8 : -1;
        }
        const auto fetch = [&](int pz, u32x4 *v) __attribute__((always_inline)) {
            const bool inz = z0 + pz < Di;
            const u16 *pb = cbase + pz * pstride;
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                v[k] = off[k] >= 0 && inz ? *(const u32x4 *)(pb + off[k]) : u32x4{0u, 0u, 0u, 0u};
        };
        const auto put = [&](int slot, const u32x4 *v) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                const int i = (int)threadIdx.x + 256 * k;
                if (i < PIECES) *(u32x4 *)&ring[slot * PLANE + (i / PCS) * CP + (i % PCS) * 8] = v[k];
            }
        };
        // planes 0-2 in slots 0-2; plane 3 in flight in registers (it is stored at the
        // end of plane 0, plane 4 fetched meanwhile)
        u32x4 nx0[PPT], nx1[PPT];
        fetch(0, nx0);
        fetch(1, nx1);
        put(0, nx0);
        fetch(2, nx0);
        put(1, nx1);
        put(2, nx0);
        if (nzo > 1) fetch(3, nx0);
        __syncthreads();
        const int y = y0 + 2 * wave;
        const int full = min(ZX, Wo - x0);   // output nodes of a row tile
        const int lim[2] = {y < Ho ? full : 0, y + 1 < Ho ? full : 0};
        // output node x0 + i of row y + w at plane z0 + iz is node orow + w Wo + iz oplane + i
        const long long orow = ((b * Do + z0) * Ho + y) * (long long)Wo + x0;
        // part h of the last step of row w of plane iz: shifted sum, bias, activation, store
        const auto finish = [&](int h, int w, const Acc &p, int iz, bool on) __attribute__((always_inline)) {
            const long long o0 = orow + (w ? Wo : 0) + iz * oplane;
            const int n = on ? lim[w] : 0;
            if constexpr (N16) {
                // rows 16 h + 4 k16 + r: the next row is the next register, or the first one of
                // the next sixteen lanes
                const auto next = [&](const f32x4 *q, int e) __attribute__((always_inline)) {
                    const float v = k16 == 0 && h == 0 ? q[1][e] : q[h][e];
                    return __int_as_float(__builtin_amdgcn_ds_bpermute(((lane + 16) & 63) * 4, __float_as_int(v)));
                };
                const f32x4 *P0 = p.n[w][0], *P1 = p.n[w][1], *P2 = p.n[w][2];
                const float x1 = next(P1, 0), x20 = next(P2, 0), x21 = next(P2, 1);
                const float v[4] = {P0[h][0] + P1[h][1] + P2[h][2] + bv, P0[h][1] + P1[h][2] + P2[h][3] + bv,
                                    P0[h][2] + P1[h][3] + x20 + bv, P0[h][3] + x1 + x21 + bv};
                const int i = 16 * h + 4 * k16;
                float *o = (float *)out + (o0 + i) * NOUT + l16;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (l16 < NOUT && i + e < n) o[e * NOUT] = v[e];
            } else {
                // rows 8 h + 4 kg + r: the next row is the next register, or the first one of the
                // other half (of the next eight rows, for the upper half)
                const bool low = kg == 0;
                const auto next = [&](const f32x16 &q, int e) __attribute__((always_inline)) {
                    const float up = h < 3 ? q[4 * h + 4 + e] : 0.0f;
                    return other_half(low ? up : q[4 * h + e], low);
                };
                const f32x16 &P0 = p.w[w][0], &P1 = p.w[w][1], &P2 = p.w[w][2];
                const float x1 = next(P1, 0), x20 = next(P2, 0), x21 = next(P2, 1);
                float v[4] = {P0[4 * h] + P1[4 * h + 1] + P2[4 * h + 2] + bv,
                              P0[4 * h + 1] + P1[4 * h + 2] + P2[4 * h + 3] + bv,
                              P0[4 * h + 2] + P1[4 * h + 3] + x20 + bv, P0[4 * h + 3] + x1 + x21 + bv};
                if (RELU)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
                const uint2 pk = quad_rows(v[0], v[1], v[2], v[3], lane);
                // the row as a buffer of its own length: stores past its end (and all of them with
                // `on` false) are dropped, without a branch among the matrix instructions
                const auto rs = __builtin_amdgcn_make_buffer_rsrc((u16 *)out + o0 * CO, 0, n * CO * 2, 0x00020000);
                const int at = ((8 * h + 4 * kg + (lane & 3)) * CO + (mr & ~3)) * 2;
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{pk.x, pk.y}, rs, at, 0, 0);
            }
        };
        constexpr int PARTS = N16 ? 2 : 4;   // parts of a row's last step
        // one output plane; cur holds plane iz + 3, nxt receives plane iz + 4 (the two
        // register sets swap roles every plane, so the loop below takes planes in pairs)
        const auto plane = [&](int iz, u32x4 *cur, u32x4 *nxt, Acc &now, const Acc &prev) __attribute__((always_inline)) {
            if (iz + 2 < nzo) fetch(iz + 4, nxt);
            constexpr int NG = 9 * NCB;   // input fragments of a plane and row
            // fragment g = ((a 3 + p) NCB + c) of row w (N16: of its half)
            const auto afrag = [&](int g, int w, int half) __attribute__((always_inline)) {
                const int a = g / (3 * NCB), p = (g / NCB) % 3, c = g % NCB;
                const u16 *row = ring + ((iz + a) & 3) * PLANE + (2 * wave + w + p) * 32 * CP;
                return frag(N16 ? row + (16 * half + l16) * CP + c * 32 + k16 * 8 : row + mr * CP + c * 16 + kg * 8);
            };
#pragma unroll
            for (int w = 0; w < 2; ++w)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if constexpr (N16) now.n[w][q][0] = now.n[w][q][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    else
#pragma unroll
                        for (int e = 0; e < 16; ++e) now.w[w][q][e] = 0.0f;
                }
            // fragments are read one step ahead of their matrix instructions
            bf16x8 A[2][2][2], B[2][3];
            const auto read = [&](int g) __attribute__((always_inline)) {
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    A[g & 1][w][0] = afrag(g, w, 0);
                    if (N16) A[g & 1][w][1] = afrag(g, w, 1);
                }
#pragma unroll
                for (int q = QR; q < 3; ++q) B[g & 1][q] = frag(&wl[((g * QL + q - QR) * 64 + lane) * 8]);
            };
            read(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g + 1 < NG) read(g + 1);
                const int ap = g / NCB, c = g % NCB;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const bf16x8 Bq = q < QR ? Bw[ap][q < QR ? q : 0][c] : B[g & 1][q];
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        if constexpr (N16) {
                            now.n[w][q][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[g & 1][w][0], Bq, now.n[w][q][0], 0, 0, 0);
                            now.n[w][q][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[g & 1][w][1], Bq, now.n[w][q][1], 0, 0, 0);
                        } else {
                            now.w[w][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[g & 1][w][0], Bq, now.w[w][q], 0, 0, 0);
                        }
                    }
                }
                // a part of the plane before, every other step
                if (TWO && g % 2 == 1 && g / 2 < 2 * PARTS) finish(g / 2 % PARTS, g / 2 / PARTS, prev, iz - 1, iz > 0);
                if (N16) __builtin_amdgcn_sched_barrier(0);
            }
            if (TWO && !N16) {
                // a few of those instructions after every matrix instruction, not all at once
#pragma unroll
                for (int i = 0; i < 6 * NG; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // matrix
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // vector
                }
            }
            if (iz + 1 < nzo) put((iz + 3) & 3, cur);
            if (!TWO)
#pragma unroll
                for (int h = 0; h < 2 * PARTS; ++h) finish(h % PARTS, h / PARTS, now, iz, true);
            __syncthreads();
        };
        for (int iz = 0; iz < nzo; iz += 2) {
            plane(iz, nx0, nx1, s0, TWO ? s1 : s0);
            if (iz + 1 < nzo) plane(iz + 1, nx1, nx0, TWO ? s1 : s0, s0);
        }
        if (TWO)
#pragma unroll
            for (int h = 0; h < 2 * PARTS; ++h) {
                if (nzo & 1) finish(h % PARTS, h / PARTS, s0, nzo - 1, true);
                else finish(h % PARTS, h / PARTS, s1, nzo - 1, true);
            }
        // (every wavefront is past its last read of the slots: plane() ends with a barrier)
    }
}

// Output planes of a column of k_conv_fwd_zm, for `columns` columns over the whole depth Do and a
// grid of at most `most` workgroups: the fewest rounds, each as long as its planes and
// the time of some three more that a column takes to start (2 and 5 measure the same). More
// than ZC gain nothing. Grids of few columns in the plane are cut along z until all
// workgroups have one: four layers over 72^3 input nodes 323 -> 108 us, 12 x 12 x 68 86 -> 31,
// 208 x 9 x 208 314 -> 85, 100^3 326 -> 221, 264^3 3320 -> 3220 (always 32 planes before).
constexpr int ZC = 32, COL_START = 3;
inline int planes_per_column(long long columns, int Do, long long most)
{
    int best = 1;
    long long least = 0;
    for (int zc = 1; zc <= ZC && zc <= Do; ++zc) {
        const long long n = columns * ((Do + zc - 1) / zc), wgs = std::min((n + 7) / 8 * 8, most);
        const long long cost = ((n + 7) / 8 + wgs / 8 - 1) / (wgs / 8) * (zc + COL_START);
        if (zc == 1 || cost <= least) {
            least = cost;
            best = zc;
        }
    }
    return best;
}

// The same sums over rows of a narrower grid, output nodes in their order in memory.
//
// FWD:   out[m][o] = max(0, b[o] + sum_{tap,i} in[m + tap][i] w[tap][i][o])   BF16 [M][32]
// LAST:  out[m][o] = b[o] + the same sum, FP32 [M][NOUT]
// DGRAD: out[v][i] = [mask[v][i] > 0] sum_{tap,o} in[v - tap][o] w[tap][o][i], BF16 [M][32]:
//        the input gradient, with the ReLU of the layer below applied (mask: that layer's
//        output); in: the output gradient, zero outside its grid.
// in: channels-last BF16 [B][Ds][Hs][Ws][CIN], wb in fragment order; output grid Do, Ho, Wo (Ds - 2
// .. for the forward layers, Ds + 2 .. for DGRAD).
//
// A unit of work is ry rows of one output plane, or rz whole planes. Its input (rz + 2 planes of
// ry + 2 rows of Wo + 2 nodes) is staged in LDS while the unit before is computed (two buffers, registers in
// between); consecutive output nodes, whatever rows they lie in, form the 32-row tiles of the
// matrix instructions, so narrow rows waste nothing. The weights stay in registers, a wavefront
// per SIMD; each wavefront takes tiles in pairs that share a weight fragment. Units are
// dealt to the XCDs in contiguous runs (neighbouring planes share an L2).
//
// Bound: LDS reads and the matrix cores alike (an input fragment a matrix instruction). The
// kernels before it read those fragments from global memory, 64 bytes from lane to lane:
// 8 tiles of 40^3, 32 -> 32 channels 92 -> 42 us, 32 -> 7 51 -> 35, 6 -> 32 55 -> 32, input
// gradient 119 -> 49 (66 with its mask read where it is applied); a 24^3 grid 30 -> 9 us a layer.
enum { FWD = 0, LAST = 1, DGRAD = 2 };
constexpr int ROWS_NODES = 1000;   // staged nodes of a unit at most (two buffers fill the LDS)
// PLANES: rz may be more than one (its divisions cost units of rows 2 to 4 %).
template <int CIN, int KIND, bool PLANES>
__global__ __launch_bounds__(256, 1) void k_conv_rows(const u16 *__restrict__ in, const u16 *__restrict__ wb,
                                                     const float *__restrict__ bias, const u16 *__restrict__ mask,
                                                     void *__restrict__ out, int Ds, int Hs, int Ws, int Do, int Ho,
                                                     int Wo, int ry, int nyb, int planes, int nzb, int units)
{
    const int rz = PLANES ? planes : 1;
    constexpr int CP = CIN + 8, NC = CIN / 16, PCS = CIN / 8;
    constexpr int PPT = (ROWS_NODES * PCS + 255) / 256;
    constexpr int OFF = KIND == DGRAD ? 2 : 0;
    __shared__ __attribute__((aligned(16))) u16 buf[2][ROWS_NODES * CP];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int mr = lane & 31, kg = lane >> 5;
    const int SW = Wo + 2, SR = ry + 2, nodes = (rz + 2) * SR * SW;
    bf16x8 Bw[27][NC];
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
        for (int c = 0; c < NC; ++c) Bw[t][c] = frag(wb + frag_at(t, NC, c * 16 + kg * 8, mr));
    const float bv = KIND == DGRAD ? 0.0f : bias[mr];
    // place of this thread's staged pieces: plane, row, x (relative to the unit)
    int place[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int node = ((int)threadIdx.x + 256 * k) / PCS;
        const int t = node / SW, s = t / SR;
        place[k] = node < nodes ? s << 20 | (t - s * SR) << 10 | (node - t * SW) : -1;
    }
    const int part = (int)threadIdx.x % PCS * 8;   // 256 is a multiple of PCS
    struct Unit { int b, z, y0; };
    const auto unit_of = [&](int u) {
        Unit w;
        const int t = u / nyb;
        w.y0 = (u - t * nyb) * ry;
        w.b = t / (PLANES ? nzb : Do);
        w.z = (t - w.b * (PLANES ? nzb : Do)) * rz;
        return w;
    };
    u32x4 v[PPT];
    const auto fetch = [&](int u) __attribute__((always_inline)) {
        const Unit w = unit_of(u);
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int z = w.z - OFF + (place[k] >> 20), y = w.y0 - OFF + ((place[k] >> 10) & 1023), x = (place[k] & 1023) - OFF;
            const bool ok = place[k] >= 0 && (uint32_t)z < (uint32_t)Ds && (uint32_t)y < (uint32_t)Hs && (uint32_t)x < (uint32_t)Ws;
            v[k] = ok ? *(const u32x4 *)(in + (((long long)(w.b * Ds + z) * Hs + y) * Ws + x) * CIN + part) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    const auto put = [&](u16 *d) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (place[k] >= 0) *(u32x4 *)&d[((int)threadIdx.x + 256 * k) / PCS * CP + part] = v[k];
    };
    // NT tiles from tile t on of the unit in s; n: its output nodes, m0: the first one
    const auto tiles = [&](auto NTC, const u16 *s, int t, int n, long long m0) __attribute__((always_inline)) {
        constexpr int NT = decltype(NTC)::value;
        const u16 *base[NT];
        f32x16 acc[NT];
        // the mask's words are fetched before the products that they are applied to: with one
        // wavefront per SIMD nothing else hides their latency
        [[maybe_unused]] uint2 mk[NT][4];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int j = min(32 * (t + i) + mr, n - 1), yy = j / Wo;
            const int row = PLANES ? yy + 2 * (yy / Ho) : yy;   // two rows between the planes of a unit
            base[i] = s + (row * SW + (j - yy * Wo)) * CP + kg * 8;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
            if constexpr (KIND == DGRAD)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    mk[i][h] = *(const uint2 *)&mask[(m0 + min(32 * (t + i) + 8 * h + 4 * kg + (lane & 3), n - 1)) * CO + (mr & ~3)];
        }
#pragma unroll
        for (int ap = 0; ap < 9; ++ap) {
            const int a = KIND == DGRAD ? 2 - ap / 3 : ap / 3, p = KIND == DGRAD ? 2 - ap % 3 : ap % 3;
            const int row = (a * SR + p) * SW * CP;
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    bf16x8 A[NT];
#pragma unroll
                    for (int i = 0; i < NT; ++i) A[i] = frag(base[i] + row + (KIND == DGRAD ? 2 - q : q) * CP + c * 16);
#pragma unroll
                    for (int i = 0; i < NT; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i], Bw[ap * 3 + q][c], acc[i], 0, 0, 0);
                }
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int j0 = 32 * (t + i);
            if constexpr (KIND == LAST) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int j = j0 + acc_row(e, kg);
                    if (mr < NOUT && j < n) ((float *)out)[(m0 + j) * NOUT + mr] = acc[i][e] + bv;
                }
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        o[e] = acc[i][4 * h + e];
                        if (KIND == FWD) o[e] = fmaxf(o[e] + bv, 0.0f);
                    }
                    uint2 pk = quad_rows(o[0], o[1], o[2], o[3], lane);
                    const int j = j0 + 8 * h + 4 * kg + (lane & 3);
                    if (j >= n) continue;
                    const long long at = (m0 + j) * CO + (mr & ~3);
                    if constexpr (KIND == DGRAD) {
                        // x > 0 for a ReLU output: its bits are not zero and its sign is clear
                        const uint2 x = mk[i][h];
                        const auto keep = [](uint32_t g, uint32_t w) {
                            const uint32_t lo = w & 0xffffu, hi = w >> 16;
                            return g & ((lo - 1u < 0x7fffu ? 0xffffu : 0u) | (hi - 1u < 0x7fffu ? 0xffff0000u : 0u));
                        };
                        pk = uint2{keep(pk.x, x.x), keep(pk.y, x.y)};
                    }
                    *(uint2 *)&((u16 *)out)[at] = pk;
                }
            }
        }
    };
    const int run = (units + 7) / 8, u0 = (int)(blockIdx.x & 7u) * run, uend = min(u0 + run, units);
    const int step = (int)gridDim.x >> 3;
    int u = u0 + (int)(blockIdx.x >> 3), cur = 0;
    if (u >= uend) return;
    fetch(u);
    put(buf[0]);
    __syncthreads();
    for (; u < uend; u += step, cur ^= 1) {
        const bool more = u + step < uend;
        if (more) fetch(u + step);
        const Unit w = unit_of(u);
        const int n = (PLANES ? min(rz, Do - w.z) : 1) * min(ry, Ho - w.y0) * Wo, nt = (n + 31) / 32, per = (nt + 3) / 4;
        const long long m0 = ((long long)(w.b * Do + w.z) * Ho + w.y0) * Wo;
        const int tend = min(nt, (wave + 1) * per);
        int t = wave * per;
        for (; t + 1 < tend; t += 2) tiles(std::integral_constant<int, 2>{}, buf[cur], t, n, m0);
        if (t < tend) tiles(std::integral_constant<int, 1>{}, buf[cur], t, n, m0);
        if (more) put(buf[cur ^ 1]);
        __syncthreads();
    }
}

// Unit of k_conv_rows for an output grid: the fewest rounds over `cus` workgroups, each as long
// as the wavefront with the most tiles (54 matrix instructions of 32 cycles a tile with 32 input
// channels, and some 1500 cycles a unit for its start, end and barrier). Several planes where one
// has few tiles: 512 grids of 12^3 input nodes, four layers, 188 us with one plane a unit.
struct RowsUnit {
    int ry, rz;
};
inline RowsUnit rows_unit(int B, int Do, int Ho, int Wo, int cus)
{
    RowsUnit best{1, 1};
    double least = -1.0;
    const auto consider = [&](int ry, int rz) {
        const long long units = (long long)B * ((Do + rz - 1) / rz) * ((Ho + ry - 1) / ry);
        const int tiles = (rz * ry * Wo + 31) / 32;
        const double cost = (double)((units + cus - 1) / cus) * (54.0 * 32.0 * ((tiles + 3) / 4) + 1500.0);
        if (least >= 0.0 && cost >= least) return;
        least = cost;
        best = RowsUnit{ry, rz};
    };
    for (int ry = 1; ry <= Ho && 3 * (ry + 2) * (Wo + 2) <= ROWS_NODES; ++ry) consider(ry, 1);
    for (int rz = 2; rz <= Do && (rz + 2) * (Ho + 2) * (Wo + 2) <= ROWS_NODES; ++rz) consider(Ho, rz);
    return best;
}

// Weight gradient of a layer: dw[tap][i][o] += sum_v x[v + tap][i] dy[v][o] over the output nodes
// v, and the bias gradient db[o] += sum_v dy[v][o]. x: BF16 layer input [B][Di][Hi][Wi][CIN]; dy: BF16
// [B][Do][Ho][Wo][32]; dw: FP32 [27][CIN][32].
//
// Per tap a 32 x 32 product (input x output channels) whose reduction runs over the nodes. A
// unit is ry rows of an output plane: its dy and the three planes of x around it are staged in
// LDS once for all 27 taps (two buffers; the next unit is in flight in registers meanwhile),
// channels fastest as in memory, and the fragments, which need a channel's values at
// consecutive nodes, come from LDS reads that transpose (a lane names any node, so a tap is
// an address offset and rows of any length follow each other without gaps). Wavefront w
// keeps the sums of seven taps (w mod 4; the 28th is a row of ones: the bias gradient) over
// every other sixteen nodes (w / 4); a persistent workgroup adds them to dw with atomics once.
//
// Bound: the latency of staging a unit (some 3 us against 1 us of products) and, at the end, the
// atomics (some 14 of 53 us on 8 tiles of 40^3; 22 of 60 with all workgroups adding in the same
// order). The kernel before it read x and dy once per tap and transposed them by 2-byte LDS
// stores: 112 -> 53 us with 32 input channels, 112 -> 48 with 16.
constexpr int WG_T = 512;
constexpr int WG_TAPS = 7;       // taps of a wavefront
constexpr int WG_NODES = 1000;   // staged nodes (x and dy) of a unit at most
typedef short i16x4 __attribute__((ext_vector_type(4)));
// Eight nodes of this lane's channel: elements 0-3 from address a, 4-7 from b. Sixteen lanes
// read four nodes of sixteen channels, lane l the channels 4 (l mod 4) .. of node l / 4, and
// lane l receives channel l of the four nodes.
__device__ __forceinline__ bf16x8 frag_tr(const u16 *a, const u16 *b)
{
    typedef __attribute__((address_space(3))) i16x4 L;
    struct { i16x4 lo, hi; } r = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)a), __builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)b)};
    return __builtin_bit_cast(bf16x8, r);
}
template <int CIN>
__global__ __launch_bounds__(WG_T, 2) void k_conv_wgrad(const u16 *__restrict__ x, const u16 *__restrict__ dy,
                                                       float *__restrict__ dw, float *__restrict__ db, int Di, int Hi,
                                                       int Wi, int ry, int nyb, int units)
{
    constexpr int XP = CIN + 8, DP = CO + 8;   // node strides in LDS (elements)
    constexpr int PPT = (WG_NODES * (CO / 8) + WG_T - 1) / WG_T;
    // one buffer: x nodes, then dy nodes; the sums of wavefronts 4-7 at the end
    constexpr int BUF = WG_NODES * DP;
    constexpr int SUMS = 4 * WG_TAPS * 16 * 64;
    __shared__ __attribute__((aligned(16))) u16 buf[2 * BUF];
    static_assert(SUMS * 4 <= 4 * BUF, "the sums reuse the buffers");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int set = wave & 3, half = wave >> 2;
    const int mr = lane & 31, kg = lane >> 5, l16 = lane & 15;
    const int Do = Di - 2, Ho = Hi - 2, Wo = Wi - 2, SR = ry + 2;
    const int xn = 3 * SR * Wi, dn = (ry * Wo + 15) / 16 * 16;   // staged nodes of x, of dy (padded)
    const int xpieces = xn * (CIN / 8), pieces = xpieces + dn * (CO / 8);
    const uint32_t inv = ((1u << 20) + (uint32_t)Wo - 1u) / (uint32_t)Wo;   // k / Wo = k inv >> 20 for k < WG_NODES
    int tofs[WG_TAPS];   // this wavefront's taps: offset of their x node
#pragma unroll
    for (int j = 0; j < WG_TAPS; ++j) {
        const int t = min(set * WG_TAPS + j, 26);
        tofs[j] = ((t / 9 * SR + t / 3 % 3) * Wi + t % 3) * XP;
    }
    const bool ones = set == 3;
    const bf16x8 one = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
    f32x16 acc[WG_TAPS];
#pragma unroll
    for (int j = 0; j < WG_TAPS; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
    // this thread's staged pieces of 16 bytes: plane, row and x of an x node, or node of dy
    int place[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int i = (int)threadIdx.x + WG_T * k;
        if (i < xpieces) {
            const int node = i / (CIN / 8), t = node / Wi, s = t / SR;
            place[k] = s << 20 | (t - s * SR) << 10 | (node - t * Wi);
        } else {
            place[k] = i < pieces ? 1 << 30 | (i - xpieces) / (CO / 8) : -1;
        }
    }
    u32x4 v[PPT];
    struct Unit { int b, z, y0; };
    const auto unit_of = [&](int u) {
        Unit w;
        const int t = u / nyb;
        w.y0 = (u - t * nyb) * ry;
        w.b = t / Do;
        w.z = t - w.b * Do;
        return w;
    };
    const auto fetch = [&](int u) __attribute__((always_inline)) {
        const Unit w = unit_of(u);
        const int n = min(ry, Ho - w.y0) * Wo;
        const u16 *xb = x + ((long long)(w.b * Di + w.z) * Hi + w.y0) * Wi * CIN;
        const u16 *db_ = dy + ((long long)(w.b * Do + w.z) * Ho + w.y0) * Wo * CO;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = (int)threadIdx.x + WG_T * k;
            v[k] = u32x4{0u, 0u, 0u, 0u};
            if (place[k] < 0) continue;
            if (place[k] >> 30) {
                if ((place[k] & 0xfffff) < n) v[k] = *(const u32x4 *)(db_ + (long long)(i - xpieces) * 8);
            } else {
                const int s = place[k] >> 20, rr = (place[k] >> 10) & 1023, xx = place[k] & 1023;
                if (w.y0 + rr < Hi) v[k] = *(const u32x4 *)(xb + (((long long)s * Hi + rr) * Wi + xx) * CIN + i % (CIN / 8) * 8);
            }
        }
    };
    const auto put = [&](u16 *d) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = (int)threadIdx.x + WG_T * k;
            if (place[k] < 0) continue;
            u16 *p = place[k] >> 30 ? d + xn * XP + (i - xpieces) / (CO / 8) * DP + (i - xpieces) % (CO / 8) * 8
                                    : d + i / (CIN / 8) * XP + i % (CIN / 8) * 8;
            *(u32x4 *)p = v[k];
        }
    };
    const int run = (units + 7) / 8, u0 = (int)(blockIdx.x & 7u) * run, uend = min(u0 + run, units);
    const int step = (int)gridDim.x >> 3;
    int u = u0 + (int)(blockIdx.x >> 3), cur = 0;
    if (u >= uend) return;
    fetch(u);
    put(buf);
    __syncthreads();
    // channels this lane reads (x: 16 channels repeat), and its node within four
    const int dch = (mr >> 4) * 16 + (l16 & 3) * 4, xch = CIN == 16 ? (l16 & 3) * 4 : dch, sub = kg * 8 + (l16 >> 2);
    for (; u < uend; u += step, cur ^= 1) {
        const bool more = u + step < uend;
        if (more) fetch(u + step);
        const Unit w = unit_of(u);
        const int n = min(ry, Ho - w.y0) * Wo;
        const u16 *xs = buf + cur * BUF, *ds = xs + xn * XP;
        for (int k0 = 16 * half; k0 < n; k0 += 32) {
            const u16 *xa[2], *da[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = k0 + sub + 4 * h;
                da[h] = ds + k * DP + dch;
                const int c = min(k, n - 1);   // past the end dy is zero
                const int yy = (int)((uint32_t)c * inv >> 20);
                xa[h] = xs + (yy * Wi + (c - yy * Wo)) * XP + xch;
            }
            const bf16x8 B = frag_tr(da[0], da[1]);
            bf16x8 A[WG_TAPS];
#pragma unroll
            for (int j = 0; j < WG_TAPS; ++j) A[j] = frag_tr(xa[0] + tofs[j], xa[1] + tofs[j]);
            if (ones) A[WG_TAPS - 1] = one;
#pragma unroll
            for (int j = 0; j < WG_TAPS; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[j], B, acc[j], 0, 0, 0);
        }
        if (more) put(buf + (cur ^ 1) * BUF);
        __syncthreads();
    }
    float *sums = (float *)buf;
    if (half)
#pragma unroll
        for (int j = 0; j < WG_TAPS; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sums[((set * WG_TAPS + j) * 16 + e) * 64 + lane] = acc[j][e];
    __syncthreads();
    if (!half)
#pragma unroll
        for (int j = 0; j < WG_TAPS; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sums[((set * WG_TAPS + j) * 16 + e) * 64 + lane] += acc[j][e];
    __syncthreads();
    // every workgroup starts at another place: in step they would all add to the same lines
    constexpr int G = 4 * WG_TAPS * 16;
    const int rot = (int)(blockIdx.x * (unsigned)G / gridDim.x);
    for (int q = wave; q < G; q += WG_T / 64) {
        const int g = q + rot < G ? q + rot : q + rot - G, t = g >> 4, i = acc_row(g & 15, kg);
        const float s = sums[g * 64 + lane];
        if (s == 0.0f) continue;
        if (t == 27) {
            if (i == 0) atomicAdd(&db[mr], s);
        } else if (i < CIN) {
            atomicAdd(&dw[((long long)t * CIN + i) * CO + mr], s);
        }
    }
}

// Rows of a unit of k_conv_wgrad: the fewest rounds, each as long as its sixteens of nodes (seven
// matrix instructions of 32 cycles for every other one) and some 2000 cycles besides.
inline int rows_per_wgrad_unit(int B, int Do, int Ho, int Wo, int cus)
{
    int best = 1;
    double least = 0.0;
    for (int ry = 1; ry <= Ho && 3 * (ry + 2) * (Wo + 2) + (ry * Wo + 15) / 16 * 16 <= WG_NODES; ++ry) {
        const long long units = (long long)B * Do * ((Ho + ry - 1) / ry);
        const double cost = (double)((units + cus - 1) / cus) * (7.0 * 32.0 * 2.0 * ((ry * Wo + 31) / 32) + 2000.0);
        if (ry == 1 || cost < least) {
            least = cost;
            best = ry;
        }
    }
    return best;
}

// Conservative form of the output (the network's 7 channels per node n of a T^3
// tile: flux coefficients f_psi,a, f_phi,a, a = x, y, z, and the exchange s):
//   A_psi[n] = W[n] s[n] - sum_a (Wf_a[n] f_psi,a[n] - Wf_a[n - e_a] f_psi,a[n - e_a])
//   A_phi[n] = -ratio W[n] s[n] - sum_a (Xf_a[n] f_phi,a[n] - Xf_a[n - e_a] f_phi,a[n - e_a])
// with face weights Wf_a[n] = (W[n] + W[n + e_a])/2 (the same for X), on the
// interior nodes [1, T - 2]^3. t holds per node (W dpsi / dpsi_s, X dphi / dphi_s, W, X).
__device__ __forceinline__ void cons_changes(const float *o, const float *t, int T, long long base, int i, int j,
                                             int l, float ratio, float &Ap, float &Af)
{
    const long long n = base + ((long long)l * T + j) * T + i;
    const long long st[3] = {1, T, (long long)T * T};
    const float Wn = t[4 * n + 2], Xn = t[4 * n + 3];
    Ap = Wn * o[NOUT * n + 6];
    Af = -ratio * Wn * o[NOUT * n + 6];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const long long u = n + st[a], d = n - st[a];
        Ap -= 0.5f * (Wn + t[4 * u + 2]) * o[NOUT * n + a];
        Ap += 0.5f * (t[4 * d + 2] + Wn) * o[NOUT * d + a];
        Af -= 0.5f * (Xn + t[4 * u + 3]) * o[NOUT * n + 3 + a];
        Af += 0.5f * (t[4 * d + 3] + Xn) * o[NOUT * d + 3 + a];
    }
}

// Loss of B tiles of T^3 output nodes: squared error of the conservative form
// against the targets, summed into *acc (FP64), and the output gradient dy (BF16
// [M][32], channels NOUT.. zero) of scale/2 times that sum: per node the adjoint
// of the form above, from the residuals g = scale (A - target) of the node and of
// its upper neighbours.
__global__ __launch_bounds__(256) void k_cons_loss(const float *__restrict__ o, const float *__restrict__ t, int T,
                                                  long long M, float ratio, float scale, double *__restrict__ acc,
                                                  u16 *__restrict__ dy)
{
    __shared__ double sh[256];
    double s = 0.0;
    const long long TT = (long long)T * T * T;
    for (long long m = (long long)blockIdx.x * 256 + threadIdx.x; m < M; m += (long long)gridDim.x * 256) {
        const long long b = m / TT, r = m - b * TT, base = b * TT;
        const int i = (int)(r % T), j = (int)((r / T) % T), l = (int)(r / ((long long)T * T));
        const auto inner = [&](int ii, int jj, int ll) {
            return ii >= 1 && jj >= 1 && ll >= 1 && ii <= T - 2 && jj <= T - 2 && ll <= T - 2;
        };
        // residuals at the node (gp0, gf0) and at its upper neighbours along x, y, z
        float gp[4] = {0, 0, 0, 0}, gf[4] = {0, 0, 0, 0};
        const int ci[4] = {i, i + 1, i, i}, cj[4] = {j, j, j + 1, j}, cl[4] = {l, l, l, l + 1};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (!inner(ci[c], cj[c], cl[c])) continue;
            float Ap, Af;
            cons_changes(o, t, T, base, ci[c], cj[c], cl[c], ratio, Ap, Af);
            const long long nc = base + ((long long)cl[c] * T + cj[c]) * T + ci[c];
            const float rp = Ap - t[4 * nc], rf = Af - t[4 * nc + 1];
            if (c == 0) s += (double)rp * rp + (double)rf * rf;
            gp[c] = scale * rp;
            gf[c] = scale * rf;
        }
        const long long n = base + r;
        const float Wn = t[4 * n + 2], Xn = t[4 * n + 3];
        float d[8];
        const long long st[3] = {1, T, (long long)T * T};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            // face between n and n + e_a: out of n (g at n), into n + e_a (g there)
            const bool up_in = (a == 0 ? i : a == 1 ? j : l) + 1 <= T - 1;
            const float Wf = up_in ? 0.5f * (Wn + t[4 * (n + st[a]) + 2]) : 0.0f;
            const float Xf = up_in ? 0.5f * (Xn + t[4 * (n + st[a]) + 3]) : 0.0f;
            d[a] = Wf * (gp[1 + a] - gp[0]);
            d[3 + a] = Xf * (gf[1 + a] - gf[0]);
        }
        d[6] = Wn * (gp[0] - ratio * gf[0]);
        d[7] = 0.0f;
        u32x4 head = {(uint32_t)f2bf(d[0]) | ((uint32_t)f2bf(d[1]) << 16),
                      (uint32_t)f2bf(d[2]) | ((uint32_t)f2bf(d[3]) << 16),
                      (uint32_t)f2bf(d[4]) | ((uint32_t)f2bf(d[5]) << 16), (uint32_t)f2bf(d[6])};
        u32x4 zero = {0u, 0u, 0u, 0u};
        u32x4 *dd = (u32x4 *)&dy[m * CO];
        dd[0] = head;
        dd[1] = zero;
        dd[2] = zero;
        dd[3] = zero;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(acc, sh[0]);
}

// Device views of the parameters. Master weights in parameter order; gradients and
// the BF16 copies in the padded layouts of the kernels above.
struct Net {
    float *master, *m, *v;      // FP32 [n_params]
    float *gw[NL];              // FP32 [27][CIN_PAD][32] weight gradients
    float *gb[NL];              // FP32 [32] bias gradients
    u16 *wb[NL];                // BF16 forward weights in fragment order (reduction over input channels)
    u16 *wt[NL];                // BF16 transposed weights in fragment order (reduction over output channels)
    float *bias[NL];            // FP32 [32]
};

// Where parameter index k lives: layer, and either (tap, i, o) of a weight or o of a bias.
__device__ __forceinline__ void param_site(long long k, int &l, int &tap, int &i, int &o, bool &is_bias)
{
    l = 0;
    while (l < NL - 1 && k >= layer_params(l)) k -= layer_params(l++);
    const long long nw = 27LL * CIN_REAL[l] * COUT_REAL[l];
    is_bias = k >= nw;
    if (is_bias) {
        o = (int)(k - nw);
        tap = i = 0;
    } else {
        o = (int)(k % COUT_REAL[l]);
        const long long r = k / COUT_REAL[l];
        i = (int)(r % CIN_REAL[l]);
        tap = (int)(r / CIN_REAL[l]);
    }
}

// Adam step (adam != 0, t = step count after this step) or a plain copy of the master
// weights (adam == 0), then the BF16 copies and FP32 biases the kernels read.
__global__ __launch_bounds__(256) void k_adam_pack(Net net, int adam, float lr, float b1, float b2, float eps,
                                                  float c1, float c2)
{
    const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
    if (k >= n_params()) return;
    int l, tap, i, o;
    bool is_bias;
    param_site(k, l, tap, i, o, is_bias);
    float w = net.master[k];
    if (adam) {
        const float g = is_bias ? net.gb[l][o] : net.gw[l][((long long)tap * CIN_PAD[l] + i) * CO + o];
        const float m = b1 * net.m[k] + (1.0f - b1) * g;
        const float v = b2 * net.v[k] + (1.0f - b2) * g * g;
        net.m[k] = m;
        net.v[k] = v;
        w -= lr * (m / c1) / (sqrtf(v / c2) + eps);
        net.master[k] = w;
    }
    if (is_bias) {
        net.bias[l][o] = w;
    } else {
        const u16 h = f2bf(w);
        net.wb[l][frag_at(tap, CIN_PAD[l] / 16, i, o)] = h;
        if (l > 0) net.wt[l][frag_at(tap, CO / 16, o, i)] = h;   // the first layer's input has no gradient
    }
}

__global__ __launch_bounds__(256) void k_zero(u32x4 *p, long long n)
{
    const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
    if (k < n) p[k] = u32x4{0u, 0u, 0u, 0u};
}

// Gradients in parameter order (for export).
__global__ __launch_bounds__(256) void k_grad_flat(Net net, float *out)
{
    const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
    if (k >= n_params()) return;
    int l, tap, i, o;
    bool is_bias;
    param_site(k, l, tap, i, o, is_bias);
    out[k] = is_bias ? net.gb[l][o] : net.gw[l][((long long)tap * CIN_PAD[l] + i) * CO + o];
}

}  // namespace sg
}  // namespace lbfd
