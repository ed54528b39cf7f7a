// substrate.hip -- the HyperNEAT substrate layer (the step after the CPPN
// grid queries; the paper supports HyperNEAT, Section 4.3, and the method
// it cites paints a substrate's connection weights with a CPPN).
//
// For every genome g: W[g] is the CPPN's output on all S x S pairs of the
// side x side grid (row p1 = source point, column p2 = target point, the
// order neat_forward_grid writes them in), the expression threshold prunes
// weak weights (|w| < theta -> 0) and the substrate layer maps the shared
// input planes X [B][S] to Y[g] = tanh(X W'[g]) [B][S].
//
// Y[g] = X W'[g] is a dense contraction (M = B, N = K = S), so it runs on
// the matrix cores: v_mfma_f32_32x32x2_f32, fp32 in and fp32 accumulation
// (the precision of the rest of the path).  A workgroup of four waves owns
// a 128 x 64 tile of one genome's Y (64 x 64 in smaller launches); K
// advances in chunks of 32 staged in LDS (the threshold is applied as W
// enters LDS); each wave owns a 64 x 32 quarter, two 32 x 32 MFMA blocks.
// Operand layout of the 32x32x2 MFMA: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32] and receives D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] in
// its r-th accumulator register.
//
// Both tiles lie in LDS with k contiguous (W transposed as it is stored), and
// lane half l / 32 takes k = 4 (l / 32) .. + 3 of every 8 for both operands,
// one of them per MFMA: any pairing of k serves, and a fragment of four MFMAs
// is one 16-byte read.
//
// What bounds it: the matrix cores.  P = 500, S = B = 256 (16.8 GFLOP): 153 us
// (110 TFLOP/s; the layer alone, without the grid queries that make W); the MFMAs alone, without loads or stores, take 120 us in this
// launch.  16x16x4 blocks with 4-byte LDS reads took 165 us (LDS busy two
// thirds of the time; 16-byte reads halve that), 32x32x2 blocks 158 us, two of
// them per wave 153 us, four 168 us; the next chunk's loads issued ahead of
// the MFMAs 162 us (their registers cost waves); plain instead of
// non-temporal stores no difference.
#include <hip/hip_runtime.h>

#include "act.h"
#include "launch.h"

namespace neat {
namespace {

constexpr int ST_N = 64, ST_KC = 32;
// LDS row stride: 16-byte aligned, and the rows of eight lanes that a 16-byte
// access serves together start four banks apart
constexpr int ST_LD = ST_KC + 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// MT: 32-row blocks of a wave (a workgroup's tile has 64 MT rows)
template <int MT>
__global__ __launch_bounds__(256) void substrate_kernel(SubLaunch L) {
    constexpr int ST_M = 64 * MT;
    __shared__ __align__(16) float xs[ST_M * ST_LD];  // X tile [m][k]
    __shared__ __align__(16) float ws[ST_N * ST_LD];  // W' tile [n][k]
    const int S = L.S, B = L.B;
    const int tiles_m = (B + ST_M - 1) / ST_M, tiles_n = S / ST_N;
    // workgroups are dealt to the 8 XCDs round robin; a genome's go to one, so
    // that its weights are fetched into one L2
    const unsigned bx = blockIdx.x & 7u, per = gridDim.x >> 3, rem = gridDim.x & 7u;
    const long long blk = (long long)(bx * per + min(bx, rem) + (blockIdx.x >> 3));
    const int tn = (int)(blk % tiles_n);
    const long long rest = blk / tiles_n;
    const int tm = (int)(rest % tiles_m);
    const long long g = rest / tiles_m;
    const int m0 = tm * ST_M, n0 = tn * ST_N;
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = 32 * MT * (wave >> 1), wn = 32 * (wave & 1);
    const float *Wg = L.W + (size_t)g * S * S;
    const float theta = L.theta;

    f32x16 acc[MT] = {};

    // staging assignment: X row t / 4, columns 8 (t % 4) ..; W column t % 64,
    // rows 4 (t / 64) .. and 16 further
    const int xr = t >> 2, xc = 8 * (t & 3);
    const int wk = 4 * wave;
    const int li = lane & 31, lk = lane >> 5;
    for (int k0 = 0; k0 < S; k0 += ST_KC) {
        f32x4 x[MT][2] = {};
#pragma unroll
        for (int i = 0; i < MT; ++i)
            if (m0 + 64 * i + xr < B) {
                const f32x4 *src = (const f32x4 *)(L.X + (size_t)(m0 + 64 * i + xr) * S + k0 + xc);
                x[i][0] = src[0];
                x[i][1] = src[1];
            }
        f32x4 w[2];
        const float *wsrc = Wg + (size_t)(k0 + wk) * S + n0 + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) w[h][q] = wsrc[(size_t)(16 * h + q) * S];
        __syncthreads();  // the previous chunk's reads are done
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            *(f32x4 *)(xs + (64 * i + xr) * ST_LD + xc) = x[i][0];
            *(f32x4 *)(xs + (64 * i + xr) * ST_LD + xc + 4) = x[i][1];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // expression threshold: |w| < theta -> 0 (NaN is kept)
#pragma unroll
            for (int q = 0; q < 4; ++q) w[h][q] = fabsf(w[h][q]) < theta ? 0.0f : w[h][q];
            *(f32x4 *)(ws + lane * ST_LD + wk + 16 * h) = w[h];
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < ST_KC; kk += 8) {
            f32x4 a[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
                a[i] = *(const f32x4 *)(xs + (wm + 32 * i + li) * ST_LD + kk + 4 * lk);
            const f32x4 b = *(const f32x4 *)(ws + (wn + li) * ST_LD + kk + 4 * lk);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][q], b[q], acc[i], 0, 0, 0);
        }
    }
    float *Yg = L.Y + (size_t)g * B * S;
    const int n = n0 + wn + li;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * lk + (r & 3);
            if (m < B) __builtin_nontemporal_store(act_tanh(acc[i][r]), Yg + (size_t)m * S + n);
        }
}

}  // namespace

hipError_t substrate_launch(const SubLaunch &L, hipStream_t stream) {
    // Two blocks of rows per wave halve the staging of W per product, but hold
    // twice the registers, and an odd number of 64 rows leaves one empty (one
    // part in 32 more work is what they are worth).  So they are taken for
    // launches of at least 800,000 chunk rows (tiles times S).  The layer alone in
    // us, one block / two (runs differ by 3 percent): P = 500, side 16, B = 256
    // (1,024,000 chunk rows) 178 / 164; P = 31, side 32, B = 256 (1,016,000) 163 /
    // 155; P = 500, side 16, B = 512: 302 / 294; P = 400, side 16, B = 256 (819,000)
    // 125 / 123; P = 300 (614,000) 96 / 96; P = 200 (410,000) 67.6 / 69.7; P = 60,
    // side 24, B = 128 (311,000) 61 / 67.  Past that it is even or costs little
    // where a genome's W is large (P = 100, side 24, B = 256: 161 / 165; P = 60, side
    // 32: 284 / 291).  An odd number of 64 rows: P = 500, side 16, B = 192: 123 / 149.
    const long long rows = ((long long)L.B + 63) / 64;  // of 64
    const bool filled = rows % 2 == 0 || rows > 32;
    const int mt = filled && L.P * ((rows + 1) / 2) * (L.S / ST_N) * L.S >= 800000 ? 2 : 1;
    const long long blocks = (long long)L.P * ((L.B + 64 * mt - 1) / (64 * mt)) * (L.S / ST_N);
    if (blocks == 0) return hipSuccess;
    if (mt == 2)
        hipLaunchKernelGGL(substrate_kernel<2>, dim3((unsigned)blocks), dim3(256), 0, stream, L);
    else
        hipLaunchKernelGGL(substrate_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, stream, L);
    return hipGetLastError();
}

}  // namespace neat
