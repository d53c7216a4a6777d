// Learned preconditioner: bfloat16 matrix-core convolutions (forward and
// adjoint), weight gradients with fixed-order reductions, weight preparation
// and the Adam update.
#include "lp_common.hpp"

#include <algorithm>
#include <type_traits>

namespace rpcg {

__device__ __forceinline__ void tap_offset(int t, int &dz, int &dy, int &dx)
{
    dz = t / 9 - 1;
    dy = (t / 3) % 3 - 1;
    dx = t % 3 - 1;
}

// Implicit-GEMM convolution on gfx950's 16x16x32 bfloat16 MFMA, computing
// D[co][cell] = sum_k W[co][k] In[k][cell] for 16 output channels (rows M,
// padded) by 16 cells along x (columns N). Lane l supplies A[m = l%16][k =
// 8(l/16) + j] and B[k][n = l%16] for j < 8 and receives D[4(l/16) + j][l%16]
// for j < 4: four output channels of one cell, stored as one 8-byte unit.
//
// The weights are the A operands and stay in registers for the whole kernel.
// K runs over the taps of one input plane: for each dz, the nine (dy, dx)
// taps go in chunks of 32 = two taps of 16 input channels (five chunks, the
// last half empty) or eight taps of 4 (two chunks). A wavefront owns one
// y-line of 16 cells and a run of CONV_ZR z-planes and streams the input
// planes along z: the B operands of input plane p (read straight from memory,
// zeros outside the grid) feed the three output planes p + 1, p, p - 1
// (dz = -1, 0, +1) with that dz's weights, so each input fragment is loaded
// once per line and used three times; output plane p - 1 is complete after
// plane p and is written. No LDS, no barriers; a plane's loads are issued
// at its start and their latency is covered by the other wavefronts of the
// SIMD (about 110 registers a lane leave room for three or four; loading the
// next plane ahead would double the operand registers and halve that).
constexpr int CONV_BX = 16;    // cells along x of a line
constexpr int CONV_LINES = 4;                      // wavefronts (y-lines) per workgroup
constexpr int CONV_ZR = 16;                        // output planes per wavefront

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef short v8s __attribute__((ext_vector_type(8)));

template <int CIN>
__host__ __device__ constexpr int conv_chunks() { return CIN == 16 ? 5 : 2; }

// Tap (dy, dx) of entry e < 9 of the nine taps of a plane (row-major in dy, dx).
__device__ __forceinline__ int tap9_dy(int e) { return e / 3 - 1; }
__device__ __forceinline__ int tap9_dx(int e) { return e % 3 - 1; }

// Taps of chunk q held by operand lanes of group kb: CIN = 16, tap e =
// 2q + kb/2, channels 8(kb%2) .. + 7; CIN = 4, taps e = 8q + 2kb and
// 8q + 2kb + 1, channels 0 .. 3 of each. e >= 9 is an empty half.
template <int CIN>
__device__ __forceinline__ int chunk_tap(int q, int kb, int h)
{
    return CIN == 16 ? 2 * q + (kb >> 1) : 8 * q + 2 * kb + h;
}

// A operands: W[t][co][ci] of the chunk's taps in the dz plane dzi (0, 1, 2
// for dz = -1, 0, +1), zeros for empty halves.
template <int CIN>
__device__ __forceinline__ v8s load_wchunk(const bf16_t *__restrict__ wt, int dzi, int q, int co, int kb)
{
    v8s a = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (CIN == 16) {
        const int e = chunk_tap<16>(q, kb, 0);
        if (e < 9) a = *(const v8s *)(wt + ((9 * dzi + e) * 16 + co) * 16 + 8 * (kb & 1));
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = chunk_tap<4>(q, kb, h);
            if (e < 9) {
                const v4s w = *(const v4s *)(wt + ((9 * dzi + e) * 16 + co) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) a[4 * h + j] = w[j];
            }
        }
    }
    return a;
}

// B operands of input plane z for the line (x0 + n, y): the chunk's taps at
// (x0 + n + dx, y + dy, z), zeros outside the grid or for empty halves.
template <int CIN>
__device__ __forceinline__ void load_bplane(v8s (&bq)[conv_chunks<CIN>()], const bf16_t *__restrict__ inb, int N,
                                            int x0, int y, int z, int n, int kb)
{
    const bool zin = z >= 0 && z < N;
#pragma unroll
    for (int q = 0; q < conv_chunks<CIN>(); ++q) {
        v8s b = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < (CIN == 16 ? 1 : 2); ++h) {
            const int e = chunk_tap<CIN>(q, kb, h);
            const int X = x0 + n + tap9_dx(e), Y = y + tap9_dy(e);
            if (e < 9 && zin && X >= 0 && X < N && Y >= 0 && Y < N) {
                const long long cell = ((long long)z * N + Y) * N + X;
                if constexpr (CIN == 16) {
                    b = *(const v8s *)(inb + cell * 16 + 8 * (kb & 1));
                } else {
                    const v4s v = *(const v4s *)(inb + cell * 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) b[4 * h + j] = v[j];
                }
            }
        }
        bq[q] = b;
    }
}

template <int CIN, int COUT, int EPI>
__global__ void __launch_bounds__(64 * CONV_LINES) k_lp_conv(int nb, int N, const bf16_t *__restrict__ in,
                                                             const bf16_t *__restrict__ wt,
                                                             const float *__restrict__ bias,
                                                             const bf16_t *__restrict__ mask, float *__restrict__ pre,
                                                             bf16_t *__restrict__ act)
{
    constexpr int NCH = conv_chunks<CIN>();
    const int lane = threadIdx.x & 63, kb = lane >> 4, n = lane & 15;
    const int wave = threadIdx.x >> 6;
    // tiles (system, z-run, x-tile, y-group), y-group fastest; each XCD takes a
    // contiguous range of them when the count allows (neighbours share its L2)
    const int tiles_x = (N + CONV_BX - 1) / CONV_BX, tiles_y = (N + CONV_LINES - 1) / CONV_LINES;
    const int runs = (N + CONV_ZR - 1) / CONV_ZR;
    const long long ntiles = (long long)nb * runs * tiles_x * tiles_y;
    long long tile = blockIdx.x;
    if (ntiles % 8 == 0) tile = (tile % 8) * (ntiles / 8) + tile / 8;
    const int ty = (int)(tile % tiles_y);
    long long r = tile / tiles_y;
    const int tx = (int)(r % tiles_x);
    r /= tiles_x;
    const int zr = (int)(r % runs);
    const long long b = r / runs;
    const int x0 = tx * CONV_BX, y = ty * CONV_LINES + wave, z0 = zr * CONV_ZR;
    const int z1 = min(z0 + CONV_ZR, N);
    if (y >= N) return; // wavefront-uniform; no barriers in this kernel
    const long long N3 = (long long)N * N * N;
    const bf16_t *__restrict__ inb = in + b * N3 * CIN;
    v8bf w[3][NCH];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int q = 0; q < NCH; ++q) w[d][q] = __builtin_bit_cast(v8bf, load_wchunk<CIN>(wt, d, q, n, kb));
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI != EPI_MASK && 4 * kb < COUT)
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[j] = bias[4 * kb + j];
    const int x = x0 + n;
    v4f a_prev = {0.f, 0.f, 0.f, 0.f}, a_cur = a_prev, a_next = a_prev; // outputs p - 1, p, p + 1
    for (int p = z0 - 1; p <= z1; ++p) {
        v8s bq[NCH];
        load_bplane<CIN>(bq, inb, N, x0, y, p, n, kb);
#pragma unroll
        for (int q = 0; q < NCH; ++q) {
            const v8bf bb = __builtin_bit_cast(v8bf, bq[q]);
            a_next = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0][q], bb, a_next, 0, 0, 0); // dz = -1: output p + 1
            a_cur = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1][q], bb, a_cur, 0, 0, 0);   // dz = 0: output p
            a_prev = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2][q], bb, a_prev, 0, 0, 0); // dz = +1: output p - 1
        }
        const int z = p - 1; // complete
        if (z >= z0 && x < N && 4 * kb < COUT) {
            const long long cell = b * N3 + ((long long)z * N + y) * N + x;
            if (EPI == EPI_RELU) {
                v4s o;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = a_prev[j] + bv[j];
                    o[j] = (short)f32_to_bf16(v > 0.f ? v : 0.f);
                }
                *(v4s *)(act + cell * COUT + 4 * kb) = o;
                if (pre)
                    *(v4f *)(pre + cell * COUT + 4 * kb) =
                        (v4f){a_prev[0] + bv[0], a_prev[1] + bv[1], a_prev[2] + bv[2], a_prev[3] + bv[3]};
            } else if (EPI == EPI_LINEAR) {
                *(v4f *)(pre + cell * COUT + 4 * kb) =
                    (v4f){a_prev[0] + bv[0], a_prev[1] + bv[1], a_prev[2] + bv[2], a_prev[3] + bv[3]};
            } else {
                // the relu of the forward layer was active where its stored
                // (bfloat16) activation is nonzero
                const v4s mk = *(const v4s *)(mask + cell * COUT + 4 * kb);
                v4s o;
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = (short)f32_to_bf16(mk[j] != 0 ? a_prev[j] : 0.f);
                *(v4s *)(act + cell * COUT + 4 * kb) = o;
            }
        }
        a_prev = a_cur;
        a_cur = a_next;
        a_next = (v4f){0.f, 0.f, 0.f, 0.f};
    }
}

// Weight gradient dW[t][co][ci] = sum over cells of dout[cell][co] in[cell + off(t)][ci]
// and bias gradient db[co] = sum of dout[cell][co], on 16x16x32 MFMA with
// M = co, N = ci and K = 32 cells along x: lane l supplies dout at cells
// 8(l/16) + j of channel l%16 (A) and the input at the same cells shifted by
// the tap, channel l%16 (B). A workgroup is three wavefronts, one per dz,
// each holding the nine tap tiles of its plane, and walks its items (system,
// z-run, y-line, 32-cell x-segment) one z-plane at a time. Per plane it
// stages the dout row of the plane and the three input rows y - 1 .. y + 1 of the
// next plane into LDS (zeros outside the grid), so every input row is loaded
// once and read by the three wavefronts (dz = -1, 0, +1 read the planes z - 1,
// z, z + 1); the loads of the next DW_PF planes are in flight in registers under
// the current plane's products. Four input planes and two dout rows are held, so
// a plane needs one barrier: what is staged beside the products is read after it.
//
// The operands run along cells, the activations along channels: the rows are
// turned while they are staged. A thread takes a pair of cells of eight (or
// all four) channels and writes one 32-bit word of two cells per channel; the
// operand of dx = -1 is then one 16-byte read, that of dx = +1 the same words one
// on, and dx = 0 between them the words shifted by a cell. Gathering each operand
// value with a 16-bit read of its own (38 a lane and plane instead of 7) and
// packing them bounded this kernel: 2.1 M cells, 16 -> 4, 16 -> 16 and 4 -> 16
// channels 86, 86 and 99 -> 47, 48 and 46 us (one plane in flight: 76, 74 and 63 us), now bound by
// the chain of a step (LDS writes, barrier, LDS reads, products) on four
// workgroups a CU. Rows past a layer's four channels repeat them; nothing
// reads their sums.
constexpr int DW_SEG = 32; // cells along x per item (the K of one product)
constexpr int DW_ZR = 64;  // z-planes per item
constexpr int DW_XP = DW_SEG / 2 + 1; // staged pairs of input cells per row (x0 - 1 .. x0 + 32)
// words of a channel's row: 16-byte units, and 16 channels of a unit in 64 different banks
constexpr int DW_CS = 20;
constexpr int DW_PF = 4;  // planes in flight
constexpr unsigned DW_OUT = 0xFFFFFFF0u; // past every buffer

// A staged unit: two cells of eight channels (or of all four), one word of two
// cells per channel when written.
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
template <int C>
struct DwUnit {
    typedef typename std::conditional<C == 16, v4u, v2u>::type word_t;
    word_t a, b;
    // the two cells at byte offsets o0, o1 (past the buffer: zeros)
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, unsigned o0, unsigned o1)
    {
        if constexpr (C == 16) {
            a = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o0, 0, 0));
            b = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o1, 0, 0));
        } else {
            a = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o0, 0, 0));
            b = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o1, 0, 0));
        }
    }
    __device__ __forceinline__ void store(unsigned *dst) // dst: word of the first channel's row
    {
        asm volatile("" : "+v"(a), "+v"(b)); // not taken up, and so waited for, before this place
#pragma unroll
        for (int w = 0; w < (C == 16 ? 4 : 2); ++w) {
            dst[(2 * w) * DW_CS] = __builtin_amdgcn_perm(b[w], a[w], 0x05040100);
            dst[(2 * w + 1) * DW_CS] = __builtin_amdgcn_perm(b[w], a[w], 0x07060302);
        }
    }
};

template <int CIN, int COUT>
struct DwShared {
    unsigned ring[4][3][CIN][DW_CS]; // input [plane][dy][channel][cell pair]
    unsigned drow[2][COUT][DW_CS];   // dout [plane][channel][cell pair]
    unsigned nowhere[64 + 7 * DW_CS]; // what threads without a unit write
};

// The items of one wavefront: DZ = 0, 1, 2 for dz = -1, 0, +1. The first two
// stage the input, the third dout, the middle one sums the bias gradient. Each role
// has a loop of its own: with branches in it, a wait would have to assume
// the loads of the other side too and so wait for the newest.
template <int CIN, int COUT, int DZ>
__device__ __forceinline__ void dw_items(int nb, int N, long long slot, long long slots, const bf16_t *__restrict__ in,
                                         const bf16_t *__restrict__ dout, v4f (&acc)[9], float &bsum,
                                         DwShared<CIN, COUT> &sh)
{
    constexpr bool ISD = DZ == 2;
    constexpr int C = ISD ? COUT : CIN;
    constexpr int UPC = C == 16 ? 2 : 1;                                    // channel groups per cell
    constexpr int ROW = ISD ? DW_SEG / 2 : DW_XP, UNITS = (ISD ? 1 : 3) * ROW * UPC; // staged units per plane
    static_assert(UNITS <= (ISD ? 64 : 128), "a unit per thread");
    const int lane = threadIdx.x & 63, kb = lane >> 4, c16 = lane & 15;
    const int segs = (N + DW_SEG - 1) / DW_SEG, runs = (N + DW_ZR - 1) / DW_ZR;
    const long long items = (long long)nb * runs * N * segs;
    const long long NN = (long long)N * N, N3 = NN * N;
    // this thread's unit: cell pair up of row ur, channels 8 uq ..
    const int un = ISD ? lane : (int)threadIdx.x;
    const bool mine = un < UNITS;
    const int uq = mine ? un % UPC : 0, up = mine ? un / UPC % ROW : 0, ur = mine ? un / (UPC * ROW) : 0;
    for (long long it = slot; it < items; it += slots) { // workgroup-uniform
        const int seg = (int)(it % segs);
        long long r = it / segs;
        const int y = (int)(r % N);
        r /= N;
        const int zr = (int)(r % runs);
        const long long b = r / runs;
        const int x0 = seg * DW_SEG;
        const int z0 = zr * DW_ZR, z1 = min(z0 + DW_ZR, N);
        // byte offsets of the unit's cells in plane zb, the first that the item reads
        const int zb = max(z0 - 1, 0), ze = min(z1 + 1, N);
        const int X = ISD ? x0 + 2 * up : x0 - 1 + 2 * up, Y = ISD ? y : y + ur - 1;
        const bool row_in = mine && Y >= 0 && Y < N;
        const bool in0 = row_in && X >= 0 && X < N, in1 = row_in && X + 1 < N; // X >= -1
        const unsigned plane = (unsigned)(NN * C * 2);
        const unsigned cell = (unsigned)(((long long)Y * N + X) * C * 2 + 16 * uq);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((ISD ? dout : in) + (b * N3 + zb * NN) * C), 0, (int)((ze - zb) * plane), 0x00027000);
        // the input is staged one plane ahead of dout: step z stages input z + 1 and dout z
        auto load = [&](DwUnit<C> &u, int z) { // plane z, zeros outside the grid
            const bool zin = z >= zb && z < ze;
            const unsigned o = (unsigned)(z - zb) * plane + cell;
            u.load(rs, in0 && zin ? o : DW_OUT, in1 && zin ? o + 2u * C : DW_OUT);
        };
        auto store = [&](DwUnit<C> &u, int z) {
            unsigned *dst = ISD ? &sh.drow[z & 1][8 * uq][up] : &sh.ring[z & 3][ur][8 * uq][up];
            u.store(mine ? dst : &sh.nowhere[lane]);
        };
        constexpr int LEAD = ISD ? 0 : 1;
        DwUnit<C> pre[DW_PF];
        __syncthreads(); // the previous item's readers are done
        if constexpr (!ISD) {
            DwUnit<C> u0, u1;
            load(u0, z0 - 1);
            load(u1, z0);
            store(u0, z0 - 1);
            store(u1, z0);
        }
#pragma unroll
        for (int u = 0; u < DW_PF; ++u) load(pre[u], z0 + LEAD + u);
        auto step = [&](DwUnit<C> &u, int z) {
            store(u, z + LEAD);
            load(u, z + LEAD + DW_PF);
            __syncthreads(); // a wavefront that is ahead stages other planes than the others read
            // A: dout at cells 8 kb + j of channel c16; B: of the three rows of plane z + dz the
            // staged cells 8 kb .. 8 kb + 9 = x - 1 .. x + 8 of channel c16
            v4u a = *(const v4u *)&sh.drow[z & 1][c16 & (COUT - 1)][4 * kb], w[3];
            unsigned last[3];
#pragma unroll
            for (int dyi = 0; dyi < 3; ++dyi) {
                const unsigned *row = sh.ring[(z + DZ + 3) & 3][dyi][c16 & (CIN - 1)] + 4 * kb;
                w[dyi] = *(const v4u *)row;
                last[dyi] = row[4];
            }
            // all reads in flight at once, and none again for another register tuple
            asm volatile("" : "+v"(a), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(last[0]), "+v"(last[1]), "+v"(last[2]));
            if constexpr (DZ == 1) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bsum += bf16_to_f32((bf16_t)a[j]);
                    bsum += bf16_to_f32((bf16_t)(a[j] >> 16));
                }
            }
            const v8bf av = __builtin_bit_cast(v8bf, a);
#pragma unroll
            for (int dyi = 0; dyi < 3; ++dyi) {
                const v4u &q = w[dyi];
                const v4u mid = {__builtin_amdgcn_alignbit(q[1], q[0], 16), __builtin_amdgcn_alignbit(q[2], q[1], 16),
                                 __builtin_amdgcn_alignbit(q[3], q[2], 16), __builtin_amdgcn_alignbit(last[dyi], q[3], 16)};
                const v4u bq[3] = {q, mid, {q[1], q[2], q[3], last[dyi]}};
#pragma unroll
                for (int dxi = 0; dxi < 3; ++dxi)
                    acc[3 * dyi + dxi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(v8bf, bq[dxi]),
                                                                                acc[3 * dyi + dxi], 0, 0, 0);
            }
        };
        int z = z0;
        for (; z + DW_PF <= z1; z += DW_PF)
#pragma unroll
            for (int u = 0; u < DW_PF; ++u) step(pre[u], z + u);
#pragma unroll
        for (int u = 0; u < DW_PF - 1; ++u)
            if (z + u < z1) step(pre[u], z + u);
    }
}

template <int CIN, int COUT>
__global__ void __launch_bounds__(192) k_lp_conv_dw(int nb, int N, const bf16_t *__restrict__ in,
                                                    const bf16_t *__restrict__ dout, float *__restrict__ pw,
                                                    float *__restrict__ pb)
{
    __shared__ __attribute__((aligned(16))) DwShared<CIN, COUT> sh;
    const int dzi = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // each XCD takes a contiguous range of the slots (neighbouring rows share its L2)
    const unsigned slot = gridDim.x % 8 == 0 ? blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
    v4f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = (v4f){0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    if (dzi == 0) dw_items<CIN, COUT, 0>(nb, N, slot, gridDim.x, in, dout, acc, bsum, sh);
    else if (dzi == 1) dw_items<CIN, COUT, 1>(nb, N, slot, gridDim.x, in, dout, acc, bsum, sh);
    else dw_items<CIN, COUT, 2>(nb, N, slot, gridDim.x, in, dout, acc, bsum, sh);
    const int lane = threadIdx.x & 63, kb = lane >> 4, c16 = lane & 15;
    // lane l holds dW[9 dzi + t][co = 4(l/16) + j][ci = l%16]
    float *__restrict__ dst = pw + ((long long)slot * LP_TAPS + 9 * dzi) * 256;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(t * 16 + 4 * kb + j) * 16 + c16] = acc[t][j];
    if (dzi == 1) {
        // lane (co, kb) holds the bias partial of cells 8 kb .. 8 kb + 7: sum over kb in order
        const float p1 = __shfl(bsum, c16 + 16, 64), p2 = __shfl(bsum, c16 + 32, 64), p3 = __shfl(bsum, c16 + 48, 64);
        const float tot = ((bsum + p1) + p2) + p3;
        if (kb == 0) pb[slot * 16 + c16] = tot;
    }
}

// Gradient of one layer from the slots in a fixed order: thread group g of
// an element sums the slots g, g + 16, ... in increasing order, then the 16
// group sums are added in group order. Weights in the [tap][out][in] layout
// of the parameters (the slots hold [tap][16][16]), then the bias.
__global__ void __launch_bounds__(256) k_lp_reduce(int nslots, int cout, int cin, const float *__restrict__ pw,
                                                   const float *__restrict__ pb, float *__restrict__ gw,
                                                   float *__restrict__ gb)
{
    __shared__ float part[16][17];
    const int nw = LP_TAPS * cout * cin;
    const int e = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + e;
    float s = 0.f;
    if (i < nw) {
        const int t = i / (cout * cin), o = (i / cin) % cout, c = i % cin;
        const int src = (t * 16 + o) * 16 + c;
#pragma unroll 8
        for (int k = g; k < nslots; k += 16) s += pw[(long long)k * LP_TAPS * 256 + src];
    } else if (i < nw + cout) {
#pragma unroll 8
        for (int k = g; k < nslots; k += 16) s += pb[k * 16 + (i - nw)];
    }
    part[g][e] = s;
    __syncthreads();
    if (g == 0 && i < nw + cout) {
        float tot = 0.f;
        for (int q = 0; q < 16; ++q) tot += part[q][e];
        if (i < nw) gw[i] = tot;
        else gb[i - nw] = tot;
    }
}

__global__ void k_lp_prep(const float *__restrict__ p, bf16_t *w1, bf16_t *w2, bf16_t *w3, bf16_t *w2t, bf16_t *w3t)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < LP_TAPS * 16 * 16) {
        const int t = e / 256, o = (e / 16) % 16, i = e % 16;
        // layer 2 forward [t][o][i] and adjoint [26 - t][i][o]
        const bf16_t v2 = f32_to_bf16(p[LP_OFF_W2 + (t * LP_HID + o) * LP_HID + i]);
        w2[e] = v2;
        w2t[((LP_TAPS - 1 - t) * 16 + i) * 16 + o] = v2;
        // layer 3 forward [t][o][i], o < 4 (rows 4..15 zero)
        w3[e] = o < LP_COUT ? f32_to_bf16(p[LP_OFF_W3 + (t * LP_COUT + o) * LP_HID + i]) : (bf16_t)0;
    }
    if (e < LP_TAPS * 16 * 4) {
        const int t = e / 64, o = (e / 4) % 16, i = e % 4;
        // layer 1 forward [t][o][i] (4 inputs)
        w1[e] = f32_to_bf16(p[LP_OFF_W1 + (t * LP_HID + o) * LP_CIN + i]);
        // layer 3 adjoint: inputs are its 4 outputs, outputs its 16 inputs: [26 - t][ci = o][co = i]
        w3t[((LP_TAPS - 1 - t) * 16 + o) * 4 + i] = f32_to_bf16(p[LP_OFF_W3 + (t * LP_COUT + i) * LP_HID + o]);
    }
}

// Adam with bias correction (Kingma and Ba, 2015).
__global__ void k_lp_adam(int n, float *__restrict__ p, const float *__restrict__ gr, float *__restrict__ m,
                          float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = gr[i];
    const float mi = b1 * m[i] + (1.f - b1) * g;
    const float vi = b2 * v[i] + (1.f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (__builtin_sqrtf(vi / c2) + eps);
}

hipError_t launch_lp_conv(int cin, int cout, int epi, int nb, int N, const bf16_t *in, const bf16_t *wt,
                          const float *bias, const bf16_t *mask, float *pre, bf16_t *act, hipStream_t s)
{
    const long long tiles = (long long)nb * ((N + CONV_ZR - 1) / CONV_ZR) * ((N + CONV_BX - 1) / CONV_BX) *
                            ((N + CONV_LINES - 1) / CONV_LINES);
    if (tiles <= 0) return hipSuccess;
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int grid = (int)tiles;
    const int block = 64 * CONV_LINES;
    if (cin == 4 && cout == 16 && epi == EPI_RELU)
        k_lp_conv<4, 16, EPI_RELU><<<grid, block, 0, s>>>(nb, N, in, wt, bias, mask, pre, act);
    else if (cin == 16 && cout == 16 && epi == EPI_RELU)
        k_lp_conv<16, 16, EPI_RELU><<<grid, block, 0, s>>>(nb, N, in, wt, bias, mask, pre, act);
    else if (cin == 16 && cout == 4 && epi == EPI_LINEAR)
        k_lp_conv<16, 4, EPI_LINEAR><<<grid, block, 0, s>>>(nb, N, in, wt, bias, mask, pre, act);
    else if (cin == 4 && cout == 16 && epi == EPI_MASK)
        k_lp_conv<4, 16, EPI_MASK><<<grid, block, 0, s>>>(nb, N, in, wt, bias, mask, pre, act);
    else if (cin == 16 && cout == 16 && epi == EPI_MASK)
        k_lp_conv<16, 16, EPI_MASK><<<grid, block, 0, s>>>(nb, N, in, wt, bias, mask, pre, act);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_lp_conv_dw(int cin, int cout, int nb, int N, const bf16_t *in, const bf16_t *dout, float *pw,
                             float *pb, int grid, hipStream_t s)
{
    const int block = 192; // one wavefront per dz
    if (cin == 16 && cout == 4)
        k_lp_conv_dw<16, 4><<<grid, block, 0, s>>>(nb, N, in, dout, pw, pb);
    else if (cin == 16 && cout == 16)
        k_lp_conv_dw<16, 16><<<grid, block, 0, s>>>(nb, N, in, dout, pw, pb);
    else if (cin == 4 && cout == 16)
        k_lp_conv_dw<4, 16><<<grid, block, 0, s>>>(nb, N, in, dout, pw, pb);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_lp_reduce(int nslots, int cout, int cin, const float *pw, const float *pb, float *gw, float *gb,
                            hipStream_t s)
{
    const int len = LP_TAPS * cout * cin + cout;
    k_lp_reduce<<<(len + 15) / 16, 256, 0, s>>>(nslots, cout, cin, pw, pb, gw, gb);
    return hipGetLastError();
}

hipError_t launch_lp_prep(const float *params, bf16_t *w1, bf16_t *w2, bf16_t *w3, bf16_t *w2t, bf16_t *w3t,
                          hipStream_t s)
{
    k_lp_prep<<<(LP_TAPS * 256 + 255) / 256, 256, 0, s>>>(params, w1, w2, w3, w2t, w3t);
    return hipGetLastError();
}

hipError_t launch_lp_adam(int n, float *params, const float *grad, float *m, float *v, float lr, float b1, float b2,
                          float eps, int step, hipStream_t s)
{
    const float c1 = 1.f - __builtin_powf(b1, (float)step), c2 = 1.f - __builtin_powf(b2, (float)step);
    k_lp_adam<<<(n + 255) / 256, 256, 0, s>>>(n, params, grad, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

} // namespace rpcg
