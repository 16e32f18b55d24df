// gfx950 kernels of the learned sparse-approximate-inverse preconditioner
// (an extension of the paper, which preconditions with scalar Jacobi,
// Section 6).  A per-row network 64 -> 64 -> 64 -> 32 (ReLU, bf16 weights,
// fp32 biases and accumulation on the MFMA units) maps features of row i of A
// to corrections of the Jacobi row: P_{i,c} = fl32((delta_{p,13} + O_{i,p}) /
// a_ii) on A's pattern, p the 27-point slot of (i, c).  Training minimises
// (1/|B|) sum_k ||A P v_k - v_k||^2 over Arnoldi vectors v_k with the
// project's own backward pass and Adam.
//
// MFMA: __builtin_amdgcn_mfma_f32_16x16x16bf16_1k, one wave per 16-row tile.
// Each layer is computed transposed, H^T = W^T X^T, so that the result's
// register layout (lane l holds rows 4(l/16)+r of column l%16) is exactly the
// B-operand layout of the next product: layers chain without data movement.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "../../include/cbgmres.h"
#include "cbg_device.hpp"
#include "cbg_launch.hpp"

namespace cbg {
namespace spai {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NF = 64, NH = 64, NO = 32, NSLOT = 27, CENTER = 13;
constexpr int NBR = 32;     // first neighbour-diagonal feature
// parameter vector: W1 (64x64) b1 (64) W2 (64x64) b2 (64) W3 (64x32) b3 (32)
constexpr int OW1 = 0, OB1 = OW1 + NF * NH, OW2 = OB1 + NH, OB2 = OW2 + NH * NH,
              OW3 = OB2 + NH, OB3 = OW3 + NH * NO, NPARAM = OB3 + NO;
// bf16 weights: W1, W2, W3 back to back
constexpr int QW1 = 0, QW2 = NF * NH, QW3 = QW2 + NH * NH, NWBF = QW3 + NH * NO;
static_assert(NPARAM == CBG_SPAI_NPARAM, "parameter count");
static_assert(NWBF == CBG_SPAI_NWEIGHT, "weight count");

__device__ __forceinline__ uint16_t bf16_of(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);        // round to nearest even (finite inputs)
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float f_of(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// fp64 -> bf16 in one rounding
__device__ __forceinline__ uint16_t bf16_of_d(double v)
{
    return (uint16_t)(rne_code<7, -126, 127>(v) | (sign_of(v) << 15));
}

__device__ __forceinline__ f32x4 mfma(s16x4 a, s16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// 27-point slot of entry (row, col) on an nx*ny*nz grid, or -1.
// Grid position of row i (x fastest); n < 2^31, so 32-bit arithmetic.
struct RowPos {
    int x, y;
};
__device__ __forceinline__ RowPos row_pos(int64_t i, int nx, int ny)
{
    const uint32_t u = (uint32_t)i, q = u / (uint32_t)nx;
    return {(int)(u - q * (uint32_t)nx), (int)(q % (uint32_t)ny)};
}

// Slot (0..26, 13 = the diagonal) of column c in row i on an nx x ny x nz
// grid, or -1 if c is not one of i's 27 stencil neighbours.  A neighbour is
// at offset d = c - i = dz nx ny + dy nx + dx with dx, dy, dz in {-1, 0, 1}
// and its x, y inside the grid (then its z is too, as 0 <= c < n); since
// grid points and indices correspond one to one, a triple that passes these
// tests is the column's true offset.  For nx, ny >= 3 the ranges of d for
// dz = -1, 0, 1 (and then of d - dz nx ny for dy) are disjoint, so the
// triple follows from comparisons; smaller grids try the nine (dz, dy).
__device__ __forceinline__ int slot_at(RowPos r, int64_t i, int64_t c, int nx, int ny)
{
    const int64_t d = c - i, S = (int64_t)nx * ny;
    auto check = [&](int64_t dz, int64_t dy) -> int {
        const int64_t dx = d - dz * S - dy * nx;
        if (dx < -1 || dx > 1)
            return -1;
        const int64_t x = r.x + dx, y = r.y + dy;
        if (x < 0 || x >= nx || y < 0 || y >= ny)
            return -1;
        return (int)((dz + 1) * 9 + (dy + 1) * 3 + (dx + 1));
    };
    if (nx >= 3 && ny >= 3) {
        const int64_t zb = S - nx - 1;            // |d| >= zb only for dz = +-1
        const int64_t dz = d >= zb ? 1 : (d <= -zb ? -1 : 0);
        const int64_t rem = d - dz * S;
        const int64_t dy = rem >= nx - 1 ? 1 : (rem <= -(nx - 1) ? -1 : 0);
        return check(dz, dy);
    }
    for (int dz = -1; dz <= 1; ++dz)
        for (int dy = -1; dy <= 1; ++dy) {
            const int s = check(dz, dy);
            if (s >= 0)
                return s;
        }
    return -1;
}

// Row kernels: a half-wave (32 lanes) per row, HWR rows per 256-thread
// block, lane l on the row's entries l, l + 32, ...: a row's indices and
// values are read as one contiguous run, its outputs written the same way.
// Loops that contain a barrier run the same number of times in every
// half-wave of the block (the block's largest chunk count).
constexpr int HWR = 8;

// Largest number of 32-entry chunks over the block's rows (block-uniform
// call).
__device__ __forceinline__ int block_chunks(int chunks)
{
    __shared__ int m[HWR];
    const int g = threadIdx.x >> 5;
    if ((threadIdx.x & 31) == 0)
        m[g] = chunks;
    __syncthreads();
    int r = 0;
#pragma unroll
    for (int k = 0; k < HWR; ++k)
        r = max(r, m[k]);
    __syncthreads();
    return r;
}

// The diagonal of A (0 where a row stores none).
__global__ __launch_bounds__(256) void k_diag(int n, const int32_t *__restrict__ rp,
                                              const int32_t *__restrict__ ci,
                                              const double *__restrict__ val,
                                              double *__restrict__ diag)
{
    const int g = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (int64_t base = (int64_t)blockIdx.x * HWR; base < n; base += (int64_t)gridDim.x * HWR) {
        const int64_t i = base + g;
        const bool live = i < n;
        const int beg = live ? rp[i] : 0, end = live ? rp[i + 1] : 0;
        const int ch = (end - beg + 31) / 32;
        const int chunks = max(ch, __shfl_xor(ch, 32));          // uniform over the wave
        const double d = hw_row_diag(i, beg, end, chunks, ci, val);
        if (live && lane == 0)
            diag[i] = d;
    }
}

// Orders a wave's LDS accesses across its lanes (its half-waves keep their
// rows in LDS regions of their own, so no block barrier is needed).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int SL_B = 9;                 // entries per batch of the sliced-ELL row walks

// The diagonal from A's sliced-ELL copy with one-byte diagonal indices: a
// lane per row walks the row's CSR-length prefix of the index bytes and
// reads the value of the last entry at offset 0 only (the last in CSR order,
// as k_diag; 0 where a row stores none).
__global__ __launch_bounds__(256) void k_diag_sell(int n, const int32_t *__restrict__ rp,
                                                   const int64_t *__restrict__ sp,
                                                   const uint8_t *__restrict__ sd,
                                                   const double *__restrict__ sv,
                                                   const int32_t *__restrict__ sdiag, int ndiag,
                                                   double *__restrict__ diag)
{
    __shared__ int32_t ldg[CBG_SELL_MAX_DIAG];
    for (int t = threadIdx.x; t < ndiag; t += blockDim.x)
        ldg[t] = sdiag[t];
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t sl = i / 64, beg = sp[sl];
        const int width = (int)((sp[sl + 1] - beg) / 64);
        const int len = rp[i + 1] - rp[i];
        int64_t hit = -1;
        for (int k0 = 0; k0 < len; k0 += SL_B) {
            uint32_t dx[SL_B];
#pragma unroll
            for (int u = 0; u < SL_B; ++u)
                dx[u] = sd[beg + (int64_t)min(k0 + u, width - 1) * 64 + (i & 63)];
#pragma unroll
            for (int u = 0; u < SL_B; ++u)
                if (k0 + u < len && ldg[dx[u]] == 0)
                    hit = beg + (int64_t)(k0 + u) * 64 + (i & 63);
        }
        diag[i] = hit >= 0 ? sv[hit] : 0.0;
    }
}

// Features of each row: f_p = fl32(a_{i,c(p)} / a_ii) and f_{32+p} =
// fl32(a_{c(p),c(p)} / a_ii) on present slots, f_27 = fl32((a_ii -
// sum_{c != i} |a_ic|) / a_ii) with the sum in CSR order, the rest 0; all
// rounded to bf16.  The entries' terms go through the half-wave's own LDS
// region; one lane adds them in CSR order.  (Columns are unique within a
// row, so each slot is written at most once.)
__global__ __launch_bounds__(256) void k_features(int n, const int32_t *__restrict__ rp,
                                                  const int32_t *__restrict__ ci,
                                                  const double *__restrict__ val, int nx, int ny,
                                                  const double *__restrict__ diag,
                                                  uint16_t *__restrict__ feat,
                                                  unsigned *__restrict__ bad)
{
    __shared__ double loff[HWR][32];
    __shared__ uint32_t lfw[HWR][NF / 2];
    const int g = threadIdx.x >> 5, lane = threadIdx.x & 31;
    uint16_t *lf = (uint16_t *)lfw[g];
    for (int64_t i = (int64_t)blockIdx.x * HWR + g; i < n; i += (int64_t)gridDim.x * HWR) {
        const int beg = rp[i], end = rp[i + 1];
        const double d = diag[i];
        const RowPos rpos = row_pos(i, nx, ny);
        lfw[g][lane] = 0u;
        wave_sync();
        double off = 0.0;
        for (int p0 = beg; p0 < end; p0 += 32) {
            const int p = p0 + lane;
            const bool in = p < end;
            const int64_t c = in ? ci[p] : -1;
            const double a = in ? val[p] : 0.0;
            loff[g][lane] = (in && c != i) ? fabs(a) : 0.0;
            const int s = in ? slot_at(rpos, i, c, nx, ny) : -1;
            if (s >= 0) {
                lf[s] = bf16_of((float)(a / d));
                lf[NBR + s] = bf16_of((float)(diag[c] / d));
            }
            wave_sync();
            if (lane == 0) {
                const int m = min(32, end - p0);
                for (int k = 0; k < m; ++k)
                    off += loff[g][k];
            }
            wave_sync();
        }
        if (lane == 0) {
            const double margin = (d - off) / d;
            if (!(d != 0.0) || !isfinite(margin))
                *bad = 1u;
            lf[27] = bf16_of((float)margin);
        }
        wave_sync();
        ((uint32_t *)(feat + i * NF))[lane] = lfw[g][lane];
        wave_sync();
    }
}

// The features of a 64-row slice of A's sliced-ELL copy with one-byte
// diagonal indices (the same values and bits): one wave, lane = row, the
// row's 64 features assembled in an LDS row of its own (odd word stride: the
// 64 rows sit in distinct banks).  The copy keeps each row's entries in CSR
// order, so the lane adds the off-diagonal sum in that order; entries past
// the row's CSR length are padding and skipped.  A batch's values and indices
// are loaded together (indices clamped into the slice), then the neighbours'
// diagonals.  Returns the slots the row stores, one bit each.
constexpr int FS_LD = NF / 2 + 1;       // LDS row stride in 32-bit words

struct SellDix {
    int n, ndiag, nx, ny;
    int64_t nslice;
    const int32_t *rp;
    const int64_t *sp;
    const uint8_t *sd;
    const double *sv;
    const int32_t *sdiag;
};

// What a diagonal says of its entries without their row: the offset col - row
// and, on grids with nx, ny >= 3, where it fixes the triple (see slot_at), the
// slot with dx + 1 and dy + 1 in bits 8 and 10 (-1: no stencil offset).
struct DiagSlot {
    int32_t off, code;
};
__device__ __forceinline__ void stage_diags(DiagSlot *t, const SellDix &A)
{
    for (int k = threadIdx.x; k < A.ndiag; k += blockDim.x) {
        const int32_t d = A.sdiag[k];
        int code = -1;
        if (A.nx >= 3 && A.ny >= 3) {
            const int64_t S = (int64_t)A.nx * A.ny, zb = S - A.nx - 1;
            const int64_t dz = d >= zb ? 1 : (d <= -zb ? -1 : 0), rem = d - dz * S;
            const int64_t dy = rem >= A.nx - 1 ? 1 : (rem <= -(A.nx - 1) ? -1 : 0);
            const int64_t dx = rem - dy * A.nx;
            if (dx >= -1 && dx <= 1)
                code = (int)((dz + 1) * 9 + (dy + 1) * 3 + (dx + 1)) | (int)(dx + 1) << 8 |
                       (int)(dy + 1) << 10;
        }
        t[k] = {d, code};
    }
}

// bf16(fl32(a / d)) with r = fl64(1 / d): a r is within two ulps of a / d, so
// its fl32 is within one of the quotient's, and both round to the same bf16
// unless the fl32's low half is within one of the midpoint 0x8000; then (and
// with !fast: d so small or large that 1 / d loses bits) the division decides.
__device__ __forceinline__ uint16_t bf16_ratio(double a, double d, double r, bool fast)
{
    float f = (float)(a * r);
    const uint32_t low = __float_as_uint(f) & 0xFFFFu;
    if (!fast || low - 0x7FFFu <= 2u)
        f = (float)(a / d);
    return bf16_of(f);
}

__device__ __forceinline__ uint32_t slice_features(const SellDix &A, int64_t sl,
                                                   const DiagSlot *ldg,
                                                   const double *__restrict__ diag, uint32_t *my,
                                                   unsigned *__restrict__ bad)
{
    const int lane = threadIdx.x & 63;
    uint16_t *myh = (uint16_t *)my;
    const int64_t i = sl * 64 + lane;
    const bool live = i < A.n;
    const int64_t ic = live ? i : (int64_t)A.n - 1;
    for (int q = 0; q < NF / 2; ++q)
        my[q] = 0u;
    const int64_t beg = A.sp[sl];
    const int width = (int)((A.sp[sl + 1] - beg) / 64);
    const int len = live ? A.rp[i + 1] - A.rp[i] : 0;
    const double d = diag[ic];
    const RowPos rpos = row_pos(ic, A.nx, A.ny);
    const double r = 1.0 / d;
    const bool fast = fabs(d) >= 0x1p-500 && fabs(d) <= 0x1p500;
    const bool table = A.nx >= 3 && A.ny >= 3;
    const int xin = 2 | (rpos.x > 0 ? 1 : 0) | (rpos.x < A.nx - 1 ? 4 : 0);
    const int yin = 2 | (rpos.y > 0 ? 1 : 0) | (rpos.y < A.ny - 1 ? 4 : 0);
    double off = 0.0;
    uint32_t slots = 0u;
    for (int k0 = 0; k0 < width; k0 += SL_B) {
        double a[SL_B];
        int32_t c[SL_B], code[SL_B];
#pragma unroll
        for (int u = 0; u < SL_B; ++u) {
            const int64_t e = beg + (int64_t)min(k0 + u, width - 1) * 64 + lane;
            a[u] = A.sv[e];
            const DiagSlot ds = ldg[A.sd[e]];
            c[u] = (int32_t)ic + ds.off;
            code[u] = ds.code;
        }
        double dc[SL_B];
#pragma unroll
        for (int u = 0; u < SL_B; ++u)
            dc[u] = diag[min(max(c[u], 0), A.n - 1)];
#pragma unroll
        for (int u = 0; u < SL_B; ++u) {
            if (k0 + u >= len)
                continue;
            if (c[u] != (int32_t)ic)
                off += fabs(a[u]);
            int s = -1;
            if (!table)
                s = slot_at(rpos, ic, c[u], A.nx, A.ny);
            else if (code[u] >= 0 && ((xin >> ((code[u] >> 8) & 3)) & (yin >> (code[u] >> 10)) & 1))
                s = code[u] & 31;
            if (s >= 0) {
                slots |= 1u << s;
                myh[s] = bf16_ratio(a[u], d, r, fast);
                myh[NBR + s] = bf16_ratio(dc[u], d, r, fast);
            }
        }
    }
    if (live) {
        const double margin = (d - off) / d;
        if (!(d != 0.0) || !isfinite(margin))
            *bad = 1u;
        myh[27] = bf16_of((float)margin);
    }
    return slots;
}

// The slice's features out to memory, two rows per store, and (slots not
// null) the slots each row stores.
__global__ __launch_bounds__(256) void k_features_sell(SellDix A, const double *__restrict__ diag,
                                                       uint16_t *__restrict__ feat,
                                                       uint32_t *__restrict__ slots,
                                                       unsigned *__restrict__ bad)
{
    __shared__ DiagSlot ldg[CBG_SELL_MAX_DIAG];
    __shared__ uint32_t lf[4][64 * FS_LD];
    stage_diags(ldg, A);
    __syncthreads();
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int64_t sl = (int64_t)blockIdx.x * 4 + wv; sl < A.nslice; sl += (int64_t)gridDim.x * 4) {
        const uint32_t has = slice_features(A, sl, ldg, diag, lf[wv] + lane * FS_LD, bad);
        if (slots && sl * 64 + lane < A.n)
            slots[sl * 64 + lane] = has;
        wave_sync();
        for (int q = 0; q < 32; ++q) {
            const int r = 2 * q + (lane >> 5);
            const int64_t row = sl * 64 + r;
            if (row < A.n)
                ((uint32_t *)(feat + row * NF))[lane & 31] = lf[wv][r * FS_LD + (lane & 31)];
        }
        wave_sync();
    }
}

// Weights staged in LDS transposed (out-major) so that an A operand
// (4 consecutive k of one output row) is one 8-byte read.
struct WeightsLds {
    uint16_t w1t[NH * NF];   // [out 64][in 64]
    uint16_t w2t[NH * NH];   // [out 64][in 64]
    uint16_t w3t[NO * NH];   // [out 32][in 64]
    float b1[NH], b2[NH], b3[NO];
};

__device__ void stage_weights(WeightsLds &L, const uint16_t *__restrict__ wq,
                              const float *__restrict__ prm)
{
    // four weights (out .. out + 3 of one input) per load
    auto put = [&](uint16_t *t, const uint16_t *w, int ins, int outs) {
        for (int e = 4 * (int)threadIdx.x; e < ins * outs; e += 4 * (int)blockDim.x) {
            const int in = e / outs, out = e % outs;
            const uint2 v = *(const uint2 *)(w + e);
            t[(out + 0) * ins + in] = (uint16_t)v.x;
            t[(out + 1) * ins + in] = (uint16_t)(v.x >> 16);
            t[(out + 2) * ins + in] = (uint16_t)v.y;
            t[(out + 3) * ins + in] = (uint16_t)(v.y >> 16);
        }
    };
    put(L.w1t, wq + QW1, NF, NH);
    put(L.w2t, wq + QW2, NH, NH);
    put(L.w3t, wq + QW3, NH, NO);
    for (int e = threadIdx.x; e < NH; e += blockDim.x) {
        L.b1[e] = prm[OB1 + e];
        L.b2[e] = prm[OB2 + e];
    }
    for (int e = threadIdx.x; e < NO; e += blockDim.x)
        L.b3[e] = prm[OB3 + e];
    __syncthreads();
}

__device__ __forceinline__ s16x4 lds4(const uint16_t *p)
{
    const uint2 v = *(const uint2 *)p;
    s16x4 r;
    r[0] = (short)(v.x & 0xFFFF);
    r[1] = (short)(v.x >> 16);
    r[2] = (short)(v.y & 0xFFFF);
    r[3] = (short)(v.y >> 16);
    return r;
}

// Four bf16 values, round to nearest even, by the hardware's paired conversion
// (the same bits as bf16_of for every float that is not NaN, in 2 instructions
// for about 16; the layers are bound by their VALU work beside the products).
__device__ __forceinline__ s16x4 bf16x4_of(f32x4 v)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(s16x4, __builtin_convertvector(v, bf16x4));
}

__device__ __forceinline__ s16x4 relu_bf16(f32x4 c)
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
        c[q] = fmaxf(c[q], 0.0f);
    return bf16x4_of(c);
}

// The three layers on a 16-row tile: fb holds the tile's features in the B
// layout (lane's row lane % 16, four features per step); h1, h2 and the
// outputs o come in the result layout (lane l: outputs 4 (l / 16) + q of each
// 16, row l % 16).
__device__ __forceinline__ void layers(const WeightsLds &L, const s16x4 (&fb)[NF / 16],
                                       s16x4 (&h1)[4], s16x4 (&h2)[4], f32x4 (&o)[2])
{
    const int lane = threadIdx.x & 63, col = lane & 15, kq = (lane >> 4) * 4;
    // layer 1: H1^T (64 x 16) = W1^T (64 x 64) F^T (64 x 16)
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        f32x4 c;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            c[q] = L.b1[ot * 16 + kq + q];
#pragma unroll
        for (int ks = 0; ks < NF / 16; ++ks)
            c = mfma(lds4(&L.w1t[(ot * 16 + col) * NF + ks * 16 + kq]), fb[ks], c);
        h1[ot] = relu_bf16(c);
    }
    // layer 2: H2^T (64 x 16) = W2^T (64 x 64) H1^T
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        f32x4 c;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            c[q] = L.b2[ot * 16 + kq + q];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            c = mfma(lds4(&L.w2t[(ot * 16 + col) * NH + ks * 16 + kq]), h1[ks], c);
        h2[ot] = relu_bf16(c);
    }
    // layer 3: O^T (32 x 16) = W3^T (32 x 64) H2^T
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) {
        f32x4 c;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            c[q] = L.b3[ot * 16 + kq + q];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            c = mfma(lds4(&L.w3t[(ot * 16 + col) * NH + ks * 16 + kq]), h2[ks], c);
        o[ot] = c;
    }
}

// Forward pass of 16-row tiles: O (n x 32 fp32); optionally the bf16 hidden
// activations H1, H2 (n x 64) for the backward pass.
__global__ __launch_bounds__(256) void k_forward(int n, const uint16_t *__restrict__ feat,
                                                 const uint16_t *__restrict__ wq,
                                                 const float *__restrict__ prm,
                                                 float *__restrict__ O, uint16_t *__restrict__ H1,
                                                 uint16_t *__restrict__ H2)
{
    __shared__ WeightsLds L;
    stage_weights(L, wq, prm);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int col = lane & 15, kq = (lane >> 4) * 4;      // lane's column; first of its 4 k
    const int64_t ntile = ((int64_t)n + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * nw + wave; tile < ntile;
         tile += (int64_t)gridDim.x * nw) {
        const int64_t row = tile * 16 + col;              // this lane's row in the B layout
        const bool live = row < n;
        s16x4 fb[NF / 16], h1[4], h2[4];
        f32x4 o[2];
#pragma unroll
        for (int ks = 0; ks < NF / 16; ++ks)
            fb[ks] = live ? lds4(feat + row * NF + ks * 16 + kq) : s16x4{0, 0, 0, 0};
        layers(L, fb, h1, h2, o);
        if (!live)
            continue;
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
            *(f32x4 *)(O + row * NO + ot * 16 + kq) = o[ot];
        if (H1) {
#pragma unroll
            for (int ot = 0; ot < 4; ++ot) {
                *(uint2 *)(H1 + row * NH + ot * 16 + kq) = __builtin_bit_cast(uint2, h1[ot]);
                *(uint2 *)(H2 + row * NH + ot * 16 + kq) = __builtin_bit_cast(uint2, h2[ot]);
            }
        }
    }
}

// P on A's pattern from the network output (a half-wave per row).
__global__ __launch_bounds__(256) void k_assemble(int n, const int32_t *__restrict__ rp,
                                                  const int32_t *__restrict__ ci,
                                                  const double *__restrict__ val, int nx, int ny,
                                                  const float *__restrict__ O,
                                                  float *__restrict__ pval)
{
    const int g = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (int64_t base = (int64_t)blockIdx.x * HWR; base < n; base += (int64_t)gridDim.x * HWR) {
        const int64_t i = base + g;
        const bool live = i < n;
        const int beg = live ? rp[i] : 0, end = live ? rp[i + 1] : 0;
        const int ch = (end - beg + 31) / 32;
        const int chunks = max(ch, __shfl_xor(ch, 32));
        const double d = hw_row_diag(i, beg, end, chunks, ci, val);
        const RowPos rpos = row_pos(live ? i : 0, nx, ny);
        for (int q = 0; q < chunks; ++q) {
            const int p = beg + q * 32 + lane;
            if (p < end) {
                const int s = slot_at(rpos, i, ci[p], nx, ny);
                double v = 0.0;
                if (s >= 0)
                    v = ((s == CENTER ? 1.0 : 0.0) + (double)O[i * NO + s]) / d;
                pval[p] = (float)v;
            }
        }
    }
}

// float16 code of an fp32 value: one rounding to nearest even (the hardware
// conversion: magnitudes from 65520 up become infinity); NaN the quiet NaN.
__device__ __forceinline__ uint16_t f16_code(float f)
{
    return f != f ? (uint16_t)0x7E00u : __builtin_bit_cast(uint16_t, (_Float16)f);
}

// The stored form's codes: on the slots present in A's row the float16 code
// of O[i][slot], 0 on the others and on rows in [n, ld); slot-major with row
// stride ld.  A block takes PK_ROWS consecutive rows: each half-wave walks
// PK_ROWS / 8 of them (one entry per lane) and puts the row's codes in LDS,
// slot-major; the block then writes each slot's run of PK_ROWS codes with
// one 4-byte store per two rows.
constexpr int PK_ROWS = 128;
constexpr int PK_LD = PK_ROWS + 2;      // LDS row stride: a half-wave's 27 slots in 27 banks

__global__ __launch_bounds__(256) void k_stencil_pack(int n, int64_t ld,
                                                      const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ ci, int nx,
                                                      int ny, const float *__restrict__ O,
                                                      uint16_t *__restrict__ codes)
{
    __shared__ uint32_t lcw[NSLOT * PK_LD / 2];
    uint16_t *lc = (uint16_t *)lcw;
    const int g = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (int64_t base = (int64_t)blockIdx.x * PK_ROWS; base < ld;
         base += (int64_t)gridDim.x * PK_ROWS) {
        for (int e = threadIdx.x; e < NSLOT * PK_LD / 2; e += blockDim.x)
            lcw[e] = 0u;
        __syncthreads();
        for (int r = g; r < PK_ROWS && base + r < n; r += HWR) {
            const int64_t i = base + r;
            const int beg = rp[i], end = rp[i + 1];
            const RowPos rpos = row_pos(i, nx, ny);
            for (int p = beg + lane; p < end; p += 32) {
                const int sl = slot_at(rpos, i, ci[p], nx, ny);
                if (sl >= 0)
                    lc[sl * PK_LD + r] = f16_code(O[i * NO + sl]);
            }
        }
        __syncthreads();
        // ld is even and base a multiple of PK_ROWS: every pair starts 4-byte aligned
        for (int e = threadIdx.x; e < NSLOT * (PK_ROWS / 2); e += blockDim.x) {
            const int sl = e / (PK_ROWS / 2), r = 2 * (e - sl * (PK_ROWS / 2));
            const int64_t i = base + r;
            if (i < ld)
                *(uint32_t *)(codes + (int64_t)sl * ld + i) = lcw[(sl * PK_LD + r) / 2];
        }
        __syncthreads();
    }
}

// The stored form's codes (the same) from the features and the slots each row
// stores: a wave takes 64 rows, runs the layers on their four tiles, puts the
// float16 codes into LDS, slot-major, and writes each slot's run of 64.  The
// outputs (128 bytes a row) stay in registers, and A is not walked again: at
// 128^3 the forward pass and the packing from A took 186 + 210 us as kernels
// of their own, this one 200 us.  Forming the features here too, from LDS, was slower (461 us
// for all three against 242 + 128 + 215): the weights leave two waves per
// SIMD, too few for the chain of loads behind a feature.
__global__ __launch_bounds__(256) void k_forward_codes(int n, int64_t ld,
                                                       const uint16_t *__restrict__ feat,
                                                       const uint32_t *__restrict__ slots,
                                                       const uint16_t *__restrict__ wq,
                                                       const float *__restrict__ prm,
                                                       uint16_t *__restrict__ codes)
{
    __shared__ WeightsLds L;
    __shared__ uint32_t lcw[4][NSLOT * 32];
    stage_weights(L, wq, prm);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int col = lane & 15, kq = (lane >> 4) * 4;
    uint16_t *lc = (uint16_t *)lcw[wv];
    const int64_t runs = ld / 64, step = (int64_t)gridDim.x * 4;     // ld is a multiple of 256
    for (int64_t run = (int64_t)blockIdx.x * 4 + wv; run < runs; run += step) {
        // the four tiles' features and slots in flight together (rows >= n
        // store no slot)
        s16x4 fb[4][NF / 16];
        uint32_t has[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t row = run * 64 + t * 16 + col, rc = min(row, (int64_t)n - 1);
#pragma unroll
            for (int ks = 0; ks < NF / 16; ++ks)
                fb[t][ks] = lds4(feat + rc * NF + ks * 16 + kq);
            has[t] = row < n ? slots[rc] : 0u;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            s16x4 h1[4], h2[4];
            f32x4 o[2];
            layers(L, fb[t], h1, h2, o);
#pragma unroll
            for (int ot = 0; ot < 2; ++ot)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int p = ot * 16 + kq + q;
                    if (p < NSLOT)
                        lc[p * 64 + t * 16 + col] =
                            (has[t] >> p) & 1u ? f16_code(o[ot][q]) : (uint16_t)0;
                }
        }
        wave_sync();
        for (int e = lane; e < NSLOT * 32; e += 64)
            *(uint32_t *)(codes + (int64_t)(e >> 5) * ld + run * 64 + 2 * (e & 31)) = lcw[wv][e];
        wave_sync();
    }
}

// dL/dO (bf16, n x 32) from dL/dP: dO_{i,p} = dP_{i,c(p)} / a_ii (a
// half-wave per row; the row's 32 slots assembled in LDS).
__global__ __launch_bounds__(256) void k_grad_o(int n, const int32_t *__restrict__ rp,
                                                const int32_t *__restrict__ ci,
                                                const double *__restrict__ val, int nx, int ny,
                                                const double *__restrict__ dP,
                                                uint16_t *__restrict__ dO)
{
    __shared__ uint16_t lg[HWR][NO];
    const int g = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (int64_t base = (int64_t)blockIdx.x * HWR; base < n; base += (int64_t)gridDim.x * HWR) {
        const int64_t i = base + g;
        const bool live = i < n;
        const int beg = live ? rp[i] : 0, end = live ? rp[i + 1] : 0;
        const int chunks = block_chunks((end - beg + 31) / 32);
        const double d = hw_row_diag(i, beg, end, chunks, ci, val);
        const RowPos rpos = row_pos(live ? i : 0, nx, ny);
        lg[g][lane] = 0;
        __syncthreads();
        for (int q = 0; q < chunks; ++q) {
            const int p = beg + q * 32 + lane;
            if (p < end) {
                const int s = slot_at(rpos, i, ci[p], nx, ny);
                if (s >= 0)
                    lg[g][s] = bf16_of_d(dP[p] / d);
            }
        }
        __syncthreads();
        if (live)
            dO[i * NO + lane] = lg[g][lane];
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Batched sparse products over K <= 32 vectors stored row-major (n x K).  A
// quad (4 lanes) takes a row and each of its lanes 8 of the K values, so one
// gather instruction fetches 16 rows' worth of an entry and a row's indices
// and values are loaded once, an entry per lane, and passed around the quad
// by DPP.  Bound by those gathers from L2 (64 bytes an entry of fp16 vectors,
// 256 of fp64): at 64^3 and K = 32 the products took 245, 295, 304 and (the
// gradient's dots) 421 us with a lane per value, one entry of two rows per
// instruction; 67, 120 and, the last two in one kernel, 128 us now.  With
// the network's output instead of P's values the first product also forms
// P, and with dO the last one forms dL/dO, which saves P, dL/dP and two more
// passes over A (117 us).
//
// Lane q's values: k = 8 q + e of the fp16 rows (one 16-byte load) and k =
// 8 (e / 2) + 2 q + e % 2 of the fp64 rows (four 16-byte loads, 64 bytes of a
// row per instruction); any other K uses k = q + 4 e, value by value, with the
// index clamped below K so that the loads need no branch (with one, K = 31 took
// 48 us a call on 64 rows, 33 now, 36 with a lane per value).
// ---------------------------------------------------------------------------
constexpr int QROWS = 64;               // rows per block: one per quad

// Blocks are dealt to the 8 XCDs in turn; this numbering gives each XCD a
// contiguous run of row blocks, whose neighbour rows its own L2 then holds (a
// stencil row's gathers reach the planes before and after it).
__device__ __forceinline__ int xcd_block()
{
    const int nb = gridDim.x, x = blockIdx.x & 7;
    return x * (nb >> 3) + min(x, nb & 7) + (int)(blockIdx.x >> 3);
}

template <int CTRL>
__device__ __forceinline__ int quad(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ double quad(double x)
{
    return __hiloint2double(quad<CTRL>(__double2hiint(x)), quad<CTRL>(__double2loint(x)));
}
template <int CTRL>
__device__ __forceinline__ float quad(float x)
{
    return __int_as_float(quad<CTRL>(__float_as_int(x)));
}
constexpr int QUAD_XOR1 = 0xB1, QUAD_XOR2 = 0x4E;
// the value of the quad's lane t (t known after unrolling)
template <typename T>
__device__ __forceinline__ T quad_lane(T x, int t)
{
    return t == 0 ? quad<0x00>(x) : t == 1 ? quad<0x55>(x) : t == 2 ? quad<0xAA>(x) : quad<0xFF>(x);
}

__device__ __forceinline__ double f16_value(uint32_t c)
{
    return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)c);
}

// 8 values of row r of the fp16 vectors
template <bool K32>
__device__ __forceinline__ void quad_v(const uint16_t *__restrict__ Vh, int64_t r, int K, int q,
                                       double *d)
{
    if constexpr (K32) {
        const u32x4 v = *(const u32x4 *)(Vh + r * 32 + q * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            d[2 * e] = f16_value(v[e] & 0xFFFFu);
            d[2 * e + 1] = f16_value(v[e] >> 16);
        }
    } else {
        uint32_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = Vh[r * K + min(q + 4 * e, K - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            d[e] = f16_value(q + 4 * e < K ? v[e] : 0u);
    }
}
// 8 values of row r of the fp64 vectors, and their store
template <bool K32>
__device__ __forceinline__ void quad_x(const double *__restrict__ X, int64_t r, int K, int q,
                                       double *d)
{
    if constexpr (K32) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const f64x2 v = *(const f64x2 *)(X + r * 32 + 4 * e + 2 * q);
            d[e] = v.x;
            d[e + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            d[e] = X[r * K + min(q + 4 * e, K - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            d[e] = q + 4 * e < K ? d[e] : 0.0;
    }
}

// From lane q's k = 8 (e / 2) + 2 q + e % 2 to its k = 8 q + e (the same move
// leads back): a 4 x 4 transpose of pairs within the quad.
__device__ __forceinline__ void quad_transpose(double *d, int q)
{
#pragma unroll
    for (int b = 1; b <= 2; b <<= 1)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i & b)
                continue;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double &lo = d[2 * i + e], &hi = d[2 * (i | b) + e];
                const double send = (q & b) ? lo : hi;
                const double got = b == 1 ? quad<QUAD_XOR1>(send) : quad<QUAD_XOR2>(send);
                if (q & b)
                    lo = got;
                else
                    hi = got;
            }
        }
}

// A row's entries in batches of four, one per lane of the quad: f(p0, whole)
// with whole true_type for a full batch.  In the last, partial one only the
// entries that are there count: a lane past the row's end takes part in the
// moves between lanes with row i's index, and 0 times an infinity there would
// be a NaN.  (The grid's rows of 27 have six full batches, which need no test.)
template <typename Fn>
__device__ __forceinline__ void quad_batches(int beg, int end, Fn f)
{
    int p0 = beg;
    for (; p0 + 4 <= end; p0 += 4)
        f(p0, std::true_type{});
    if (p0 < end)
        f(p0, std::false_type{});
}

// Y = P V.  FROM_O: P_ic = fl32((delta + O[slot]) / a_ii) from the network's
// output and the diagonal (the values k_assemble writes), else P's values.
template <bool K32, bool FROM_O>
__global__ __launch_bounds__(256) void k_quad_pv(int n, int K, const int32_t *__restrict__ rp,
                                                 const int32_t *__restrict__ ci,
                                                 const float *__restrict__ pval,
                                                 const float *__restrict__ O,
                                                 const double *__restrict__ diag, int nx, int ny,
                                                 const uint16_t *__restrict__ Vh,
                                                 double *__restrict__ Y)
{
    const int q = threadIdx.x & 3;
    for (int64_t i = (int64_t)xcd_block() * QROWS + (threadIdx.x >> 2); i < n;
         i += (int64_t)gridDim.x * QROWS) {
        const int beg = rp[i], end = rp[i + 1];
        const RowPos rpos = row_pos(i, nx, ny);
        const double dg = FROM_O ? diag[i] : 1.0;
        double acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            acc[e] = 0.0;
        quad_batches(beg, end, [&](int p0, auto whole) __attribute__((always_inline)) {
            const int p = p0 + q;
            const bool in = whole || p < end;
            const int c = in ? ci[p] : (int)i;
            float a = 0.0f;
            if constexpr (FROM_O) {
                const int sl = in ? slot_at(rpos, i, c, nx, ny) : -1;
                if (sl >= 0)
                    a = (float)(((sl == CENTER ? 1.0 : 0.0) + (double)O[i * NO + sl]) / dg);
            } else {
                a = in ? pval[p] : 0.0f;
            }
            double v[4][8];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                quad_v<K32>(Vh, quad_lane(c, t), K, q, v[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double at = (double)quad_lane(a, t);
                if (whole || p0 + t < end)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[e] = fma(at, v[t][e], acc[e]);
            }
        });
        if constexpr (K32) {
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                f64x2 o = {acc[e], acc[e + 1]};
                *(f64x2 *)(Y + i * 32 + q * 8 + e) = o;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (q + 4 * e < K)
                    Y[i * K + q + 4 * e] = acc[e];
        }
    }
}

// The row sum of val_p X[ci_p] over row i's entries (a quad's 8 values each)
template <bool K32>
__device__ __forceinline__ void quad_row(const int32_t *__restrict__ ci,
                                         const double *__restrict__ val,
                                         const double *__restrict__ X, int64_t i, int beg, int end,
                                         int K, int q, double *acc)
{
#pragma unroll
    for (int e = 0; e < 8; ++e)
        acc[e] = 0.0;
    quad_batches(beg, end, [&](int p0, auto whole) __attribute__((always_inline)) {
        const int p = p0 + q;
        const bool in = whole || p < end;
        const int c = in ? ci[p] : (int)i;
        const double a = in ? val[p] : 0.0;
        double x[4][8];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            quad_x<K32>(X, quad_lane(c, t), K, q, x[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double at = quad_lane(a, t);
            if (whole || p0 + t < end)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc[e] = fma(at, x[t][e], acc[e]);
        }
    });
}

// R = A Y - V, and block partials of ||R||_F^2.
template <bool K32>
__global__ __launch_bounds__(256) void k_quad_residual(int n, int K,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ ci,
                                                       const double *__restrict__ val,
                                                       const double *__restrict__ Y,
                                                       const uint16_t *__restrict__ Vh,
                                                       double *__restrict__ R,
                                                       double *__restrict__ part)
{
    const int q = threadIdx.x & 3;
    double ssq = 0.0;
    for (int64_t i = (int64_t)xcd_block() * QROWS + (threadIdx.x >> 2); i < n;
         i += (int64_t)gridDim.x * QROWS) {
        double acc[8], v[8];
        quad_row<K32>(ci, val, Y, i, rp[i], rp[i + 1], K, q, acc);
        quad_v<K32>(Vh, i, K, q, v);
        if constexpr (K32)
            quad_transpose(v, q);                   // to the fp64 rows' order
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const f64x2 r = {acc[e] - v[e], acc[e + 1] - v[e + 1]};
            ssq = fma(r.x, r.x, ssq);
            ssq = fma(r.y, r.y, ssq);
            if constexpr (K32) {
                *(f64x2 *)(R + i * 32 + 4 * e + 2 * q) = r;
            } else {
                if (q + 4 * e < K)
                    R[i * K + q + 4 * e] = r.x;
                if (q + 4 * e + 4 < K)
                    R[i * K + q + 4 * e + 4] = r.y;
            }
        }
    }
    double m = 0.0;
    block_sum_max(ssq, m);
    if (threadIdx.x == 0)
        part[blockIdx.x] = ssq;
}

// G = scale A^T R on a row, then dP_e = sum_k G[i][k] v_k[c] for its entries:
// dP (TO_O false), or dL/dO (n x 32 bf16) with dO_{i,slot} = bf16(dP_e / a_ii).
template <bool K32, bool TO_O>
__global__ __launch_bounds__(256) void k_quad_grad(int n, int K, const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ ci,
                                                   const double *__restrict__ tval,
                                                   const double *__restrict__ R, double scale,
                                                   const uint16_t *__restrict__ Vh,
                                                   double *__restrict__ dP,
                                                   const double *__restrict__ diag, int nx, int ny,
                                                   uint16_t *__restrict__ dO)
{
    __shared__ u32x4 lrow[TO_O ? QROWS : 1][NO / 8];      // a row's 32 bf16 values
    const int q = threadIdx.x & 3, g = threadIdx.x >> 2;
    for (int64_t i = (int64_t)xcd_block() * QROWS + g; i < n; i += (int64_t)gridDim.x * QROWS) {
        const int beg = rp[i], end = rp[i + 1];
        const RowPos rpos = row_pos(i, nx, ny);
        const double dg = TO_O ? diag[i] : 1.0;
        double gr[8];
        quad_row<K32>(ci, tval, R, i, beg, end, K, q, gr);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            gr[e] *= scale;
        if constexpr (K32)
            quad_transpose(gr, q);                  // to the fp16 rows' order
        if constexpr (TO_O) {
            lrow[g][q] = u32x4{0u, 0u, 0u, 0u};
            wave_sync();
        }
        for (int p0 = beg; p0 < end; p0 += 4) {
            const int p = p0 + q;
            const bool in = p < end;
            const int c = in ? ci[p] : (int)i;
            double mine = 0.0;
            double v[4][8];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                quad_v<K32>(Vh, quad_lane(c, t), K, q, v[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                double s = 0.0;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    s = fma(gr[e], v[t][e], s);
                s += quad<QUAD_XOR1>(s);
                s += quad<QUAD_XOR2>(s);
                if (t == q)
                    mine = s;
            }
            if constexpr (TO_O) {
                const int sl = in ? slot_at(rpos, i, c, nx, ny) : -1;
                if (sl >= 0)
                    ((uint16_t *)lrow[g])[sl] = bf16_of_d(mine / dg);
            } else if (in) {
                dP[p] = mine;
            }
        }
        if constexpr (TO_O) {
            wave_sync();
            *(u32x4 *)(dO + i * NO + q * 8) = lrow[g][q];
            wave_sync();
        }
    }
}

// *loss (+)= scale * sum of the block partials, folded in block order.
__global__ void k_loss_fold(const double *__restrict__ part, int nb, double scale, int accumulate,
                            double *__restrict__ loss)
{
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        s += part[b];
    double m = 0.0;
    block_sum_max(s, m);
    if (threadIdx.x == 0)
        *loss = (accumulate ? *loss : 0.0) + s * scale;
}

// ---------------------------------------------------------------------------
// Backward pass.  Per 16-row tile, one wave: dH2^T = W3 dO^T and dH2 = dO W3^T
// (the same values in two register layouts), dH1 = dH2 W2^T, masked by the
// ReLU and rounded to bf16, then the weight gradients dW3 = H2^T dO, dW2 =
// H1^T dH2 and dW1 = F^T dH1 over the tile's rows, accumulated per wave
// across tiles; bias gradients are column sums.  Each block writes its NPARAM
// partial gradients; k_grad_fold sums blocks in order.
//
// A product over rows needs its operands by column, four rows per lane.  The
// result layout of dH2 and dH1 computed untransposed is that layout (lane l
// holds rows 4 (l / 16) + r of column l mod 16), and for F, H1, H2 and dO a
// lane loads 4 (or 2) consecutive columns of its four rows and packs them by
// column, which makes column tile a the columns 4 j + a (2 j + a): a row is
// one contiguous 128-byte read, and nothing goes through LDS but the weights.
// Latency-bound with one wave per SIMD (160 accumulators a lane), so the next
// tile's loads run under the current tile's 72 products: 386 us at 262,144
// rows with the tile staged in LDS value by value, 56 us now (the fold of the
// blocks' partials took 124 us with 512 of them in turn per parameter).
// ---------------------------------------------------------------------------

// operand 16 x 16 tiles of the weights, one 8-byte value per lane
struct BackLds {
    uint2 w3n[4][2][64];     // [h tile][o step]: W3[16 t + c][16 s + 4 g ..]
    uint2 w3p[4][2][64];     // [h mod 4][o step]: W3[4 c + a][16 s + 4 g ..]
    uint2 w2p[4][4][64];     // [in mod 4][h step]: W2[4 c + a][16 s + 4 g ..]
};

__device__ __forceinline__ s16x4 as_s16x4(uint2 v) { return __builtin_bit_cast(s16x4, v); }
// the low (high) halves of two words
__device__ __forceinline__ uint32_t lo16(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t hi16(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}
// four rows of columns 4 c .. 4 c + 3, by column
__device__ __forceinline__ void by_column(const uint2 (&x)[4], s16x4 (&op)[4])
{
    op[0] = as_s16x4(uint2{lo16(x[0].x, x[1].x), lo16(x[2].x, x[3].x)});
    op[1] = as_s16x4(uint2{hi16(x[0].x, x[1].x), hi16(x[2].x, x[3].x)});
    op[2] = as_s16x4(uint2{lo16(x[0].y, x[1].y), lo16(x[2].y, x[3].y)});
    op[3] = as_s16x4(uint2{hi16(x[0].y, x[1].y), hi16(x[2].y, x[3].y)});
}
// bf16 of the gradient where the activation is positive, else 0
__device__ __forceinline__ s16x4 masked_bf16(f32x4 c, s16x4 act)
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
        c[q] = f_of((uint16_t)act[q]) > 0.0f ? c[q] : 0.0f;
    return bf16x4_of(c);
}
// a column's running sum over the tile's 16 rows in turn, four of them on each
// of its lanes c, c + 16, c + 32, c + 48 (all get the sum)
__device__ __forceinline__ float add_column(float sum, s16x4 v, int c)
{
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float s = sum;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            s += f_of((uint16_t)v[q]);
        sum = __shfl(s, c + 16 * h);
    }
    return sum;
}

// one tile's inputs as a lane loads them
struct TileIn {
    uint2 f[4], h1[4], h2[4];     // rows 4 g + t, columns 4 c ..
    uint32_t dO[4];               // rows 4 g + t, columns 2 c, 2 c + 1
    uint2 dOr[2], h2r[4];         // row c, columns 16 s + 4 g ..
};

__global__ __launch_bounds__(256) void k_backward(int n, const uint16_t *__restrict__ feat,
                                                  const uint16_t *__restrict__ H1,
                                                  const uint16_t *__restrict__ H2,
                                                  const uint16_t *__restrict__ dO,
                                                  const uint16_t *__restrict__ wq,
                                                  float *__restrict__ part)
{
    __shared__ __align__(16) union {
        BackLds w;
        float red[4][NF * NH];
    } L;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int c = lane & 15, g = lane >> 4;
    const uint16_t *w3 = wq + QW3, *w2 = wq + QW2;
    for (int e = wave; e < 8; e += nw) {
        const int t = e >> 1, s = e & 1;
        L.w.w3n[t][s][lane] = *(const uint2 *)(w3 + (16 * t + c) * NO + 16 * s + 4 * g);
        L.w.w3p[t][s][lane] = *(const uint2 *)(w3 + (4 * c + t) * NO + 16 * s + 4 * g);
    }
    for (int e = wave; e < 16; e += nw) {
        const int t = e >> 2, s = e & 3;
        L.w.w2p[t][s][lane] = *(const uint2 *)(w2 + (4 * c + t) * NH + 16 * s + 4 * g);
    }
    __syncthreads();
    f32x4 gw3[4][2], gw2[4][4], gw1[4][4];      // [row tile of W][column tile of W]
    float gb1[4], gb2[4], gb3[2];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            gw2[a][b] = f32x4{0, 0, 0, 0};
            gw1[a][b] = f32x4{0, 0, 0, 0};
            gw3[a][b & 1] = f32x4{0, 0, 0, 0};
        }
        gb1[a] = gb2[a] = gb3[a & 1] = 0.0f;
    }
    const int64_t ntile = ((int64_t)n + 15) / 16, step = (int64_t)gridDim.x * nw;
    // rows >= n read row n - 1 and a zero dO; clear() makes the rest of them 0
    // when the tile's turn comes (an infinite activation of row n - 1 times
    // that dO would be a NaN)
    auto load = [&](int64_t tile, TileIn &x) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t r = tile * 16 + 4 * g + t, rc = min(r, (int64_t)n - 1);
            x.f[t] = *(const uint2 *)(feat + rc * NF + 4 * c);
            x.h1[t] = *(const uint2 *)(H1 + rc * NH + 4 * c);
            x.h2[t] = *(const uint2 *)(H2 + rc * NH + 4 * c);
            x.dO[t] = r < n ? *(const uint32_t *)(dO + rc * NO + 2 * c) : 0u;
        }
        const int64_t r = tile * 16 + c, rc = min(r, (int64_t)n - 1);
#pragma unroll
        for (int s = 0; s < 2; ++s)
            x.dOr[s] = r < n ? *(const uint2 *)(dO + rc * NO + 16 * s + 4 * g) : uint2{0u, 0u};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            x.h2r[t] = *(const uint2 *)(H2 + rc * NH + 16 * t + 4 * g);
    };
    auto clear = [&](int64_t tile, TileIn &x) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (tile * 16 + 4 * g + t >= n)
                x.f[t] = x.h1[t] = x.h2[t] = uint2{0u, 0u};
            if (tile * 16 + c >= n)
                x.h2r[t] = uint2{0u, 0u};
        }
    };
    int64_t tile = (int64_t)blockIdx.x * nw + wave;
    TileIn cur;
    if (tile < ntile)
        load(tile, cur);
    for (; tile < ntile; tile += step) {
        TileIn nxt;
        load(min(tile + step, ntile - 1), nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (tile * 16 + 16 > n)
            clear(tile, cur);
        const s16x4 ob[2] = {as_s16x4(cur.dOr[0]), as_s16x4(cur.dOr[1])};
        s16x4 fc[4], h1c[4], h2c[4], oc[2];
        by_column(cur.f, fc);
        by_column(cur.h1, h1c);
        by_column(cur.h2, h2c);
        oc[0] = as_s16x4(uint2{lo16(cur.dO[0], cur.dO[1]), lo16(cur.dO[2], cur.dO[3])});
        oc[1] = as_s16x4(uint2{hi16(cur.dO[0], cur.dO[1]), hi16(cur.dO[2], cur.dO[3])});
        s16x4 d2t[4], d2[4], d1[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 x = {0, 0, 0, 0}, y = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                x = mfma(as_s16x4(L.w.w3n[t][s][lane]), ob[s], x);
                y = mfma(ob[s], as_s16x4(L.w.w3p[t][s][lane]), y);
            }
            d2t[t] = masked_bf16(x, as_s16x4(cur.h2r[t]));
            d2[t] = masked_bf16(y, h2c[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 x = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4; ++s)
                x = mfma(d2t[s], as_s16x4(L.w.w2p[t][s][lane]), x);
            d1[t] = masked_bf16(x, h1c[t]);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
                gw3[a][b] = mfma(h2c[a], oc[b], gw3[a][b]);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                gw2[a][b] = mfma(h1c[a], d2[b], gw2[a][b]);
                gw1[a][b] = mfma(fc[a], d1[b], gw1[a][b]);
            }
            gb2[a] = add_column(gb2[a], d2[a], c);
            gb1[a] = add_column(gb1[a], d1[a], c);
        }
        gb3[0] = add_column(gb3[0], oc[0], c);
        gb3[1] = add_column(gb3[1], oc[1], c);
        cur = nxt;
    }
    // The block's sums: every wave puts its own into LDS, then each parameter
    // adds the waves in order; W1, W2, and W3 with the biases in turn, since
    // LDS holds 4096 values a wave.  (Waves adding to one array in turn left
    // the others idle: 29.8 us at 64 rows, 9.9 us now.)
    static_assert(OW1 % 4 == 0 && OB1 % 4 == 0 && OW2 % 4 == 0 && OB2 % 4 == 0 && OW3 % 4 == 0 &&
                      OB3 % 4 == 0 && NPARAM % 4 == 0,
                  "four parameters per load and store");
    float *mine = L.red[wave], *out = part + (size_t)blockIdx.x * NPARAM;
    auto fold = [&](int at, int count, int base) {      // parameters base .. from mine[at ..]
        for (int e = 4 * (int)threadIdx.x; e < count; e += 4 * (int)blockDim.x) {
            f32x4 s = *(const f32x4 *)&L.red[0][at + e];
            for (int w = 1; w < nw; ++w)
                s += *(const f32x4 *)&L.red[w][at + e];
            *(f32x4 *)(out + base + e) = s;
        }
    };
    auto put = [&](const f32x4 (&gw)[4][4]) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *(f32x4 *)&mine[(4 * (4 * g + r) + a) * NH + 4 * c] =
                    f32x4{gw[a][0][r], gw[a][1][r], gw[a][2][r], gw[a][3][r]};
    };
    __syncthreads();                            // the weights are done with
    put(gw1);
    __syncthreads();
    fold(0, NF * NH, OW1);
    __syncthreads();
    put(gw2);
    __syncthreads();
    fold(0, NH * NH, OW2);
    __syncthreads();
    constexpr int LB1 = NH * NO, LB2 = LB1 + NH, LB3 = LB2 + NH;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *(float2 *)&mine[(4 * (4 * g + r) + a) * NO + 2 * c] =
                float2{gw3[a][0][r], gw3[a][1][r]};
    if (g == 0) {
        *(f32x4 *)&mine[LB1 + 4 * c] = f32x4{gb1[0], gb1[1], gb1[2], gb1[3]};
        *(f32x4 *)&mine[LB2 + 4 * c] = f32x4{gb2[0], gb2[1], gb2[2], gb2[3]};
        *(float2 *)&mine[LB3 + 2 * c] = float2{gb3[0], gb3[1]};
    }
    __syncthreads();
    fold(0, NH * NO, OW3);
    fold(LB1, NH, OB1);
    fold(LB2, NH, OB2);
    fold(LB3, NO, OB3);
}

// grad[e] (+)= sum over blocks of part[b][e] in fp64: 32 parameters per block,
// eight runs of consecutive blocks each, the runs' sums added in order.
constexpr int FOLD_E = 32, FOLD_RUNS = 8;
__global__ __launch_bounds__(256) void k_grad_fold(const float *__restrict__ part, int nb,
                                                   int accumulate, double *__restrict__ grad)
{
    __shared__ double ls[FOLD_RUNS][FOLD_E];
    const int le = threadIdx.x & (FOLD_E - 1), run = threadIdx.x / FOLD_E;
    const int e = blockIdx.x * FOLD_E + le;
    const int len = (nb + FOLD_RUNS - 1) / FOLD_RUNS, lo = run * len, hi = min(lo + len, nb);
    double s = 0.0;
    if (e < NPARAM) {
#pragma unroll 8
        for (int b = lo; b < hi; ++b)
            s += (double)part[(size_t)b * NPARAM + e];
    }
    ls[run][le] = s;
    __syncthreads();
    if (run == 0 && e < NPARAM) {
#pragma unroll
        for (int r = 1; r < FOLD_RUNS; ++r)
            s += ls[r][le];
        grad[e] = (accumulate ? grad[e] : 0.0) + s;
    }
}

// Adam (Kingma and Ba, 2015) on the fp32 master parameters: moments and
// parameters are formed in FP64 (no contraction) and stored rounded to fp32;
// c1 = 1 - beta1^t and c2 = 1 - beta2^t come from the host.  The bf16
// weights are refreshed as the round-to-nearest-even of the new masters.
__global__ void k_adam(float *__restrict__ prm, float *__restrict__ m1, float *__restrict__ m2,
                       uint16_t *__restrict__ wq, const double *__restrict__ grad, double lr,
                       double b1, double b2, double eps, double c1, double c2)
{
#pragma clang fp contract(off)
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < NPARAM; e += gridDim.x * blockDim.x) {
        const double g = grad[e];
        const float m = (float)(b1 * (double)m1[e] + (1.0 - b1) * g);
        const float v = (float)(b2 * (double)m2[e] + (1.0 - b2) * g * g);
        m1[e] = m;
        m2[e] = v;
        const double mh = (double)m / c1;
        const double vh = (double)v / c2;
        const float p = (float)((double)prm[e] - lr * mh / (sqrt(vh) + eps));
        prm[e] = p;
        int q = -1;
        if (e >= OW1 && e < OB1)
            q = QW1 + (e - OW1);
        else if (e >= OW2 && e < OB2)
            q = QW2 + (e - OW2);
        else if (e >= OW3 && e < OB3)
            q = QW3 + (e - OW3);
        if (q >= 0)
            wq[q] = bf16_of(p);
    }
}

// bf16 weights from the fp32 masters (round to nearest even).
__global__ void k_round_weights(const float *__restrict__ prm, uint16_t *__restrict__ wq)
{
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < NWBF; e += gridDim.x * blockDim.x) {
        const int p = e < QW2 ? OW1 + e : e < QW3 ? OW2 + (e - QW2) : OW3 + (e - QW3);
        wq[e] = bf16_of(prm[p]);
    }
}

// Values of A^T on A's pattern (structurally symmetric A): t_val[p] of
// entry (i, c) is a_ci, found by binary search in row c; a missing mirror
// entry sets *bad.
__global__ __launch_bounds__(256) void k_transpose_values(int n, const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ ci,
                                                          const double *__restrict__ val,
                                                          double *__restrict__ tval,
                                                          unsigned *__restrict__ bad)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        for (int p = rp[i]; p < rp[i + 1]; ++p) {
            const int c = ci[p];
            int lo = rp[c], hi = rp[c + 1] - 1;
            double v = 0.0;
            bool found = false;
            while (lo <= hi) {
                const int mid = (lo + hi) >> 1;
                const int cm = ci[mid];
                if (cm == i) {
                    v = val[mid];
                    found = true;
                    break;
                }
                if (cm < i)
                    lo = mid + 1;
                else
                    hi = mid - 1;
            }
            if (!found)
                *bad = 1u;
            tval[p] = v;
        }
    }
}

// out (n x K, row-major fp16) from K FP64 vectors V[(first + k*stride)*ld ..];
// one rounding to nearest even; magnitudes from 65520 up become infinity.
__global__ __launch_bounds__(256) void k_pack(const double *__restrict__ V, int64_t ld, int n,
                                              int K, int first, int stride,
                                              uint16_t *__restrict__ out)
{
    const int64_t total = (int64_t)n * K;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / K;
        const int k = (int)(e % K);
        const double v = V[(int64_t)(first + (int64_t)k * stride) * ld + i];
        uint32_t c = fabs(v) >= 65520.0 ? 0x7C00u : rne_code<10, -14, 15>(v);
        out[e] = (uint16_t)(c | (sign_of(v) << 15));
    }
}

}  // namespace spai
}  // namespace cbg

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace cbg;
using namespace cbg::spai;

namespace {

constexpr size_t SALIGN = 256;
constexpr int MAXB_ROW = 4096;     // grid cap of the row-parallel kernels
constexpr int MAXB_BACK = 512;     // grid cap of the backward pass (partials)

size_t salign(size_t x) { return (x + SALIGN - 1) / SALIGN * SALIGN; }

struct SpaiWs {
    unsigned *bad;
    double *diag;
    double *dinv;          // 1 / a_ii on cbg_basis_ld(n) rows (stencil apply)
    double *lpart;
    float *gpart;
    uint16_t *feat, *h1, *h2, *dO;
    float *O, *pval;
    double *X0, *X1, *dP;
};

SpaiWs carve_spai(void *ws, int64_t n, int64_t nnz, int64_t K, size_t *total)
{
    uint8_t *base = (uint8_t *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        void *p = base ? base + off : nullptr;
        off = salign(off + bytes);
        return p;
    };
    SpaiWs s;
    s.bad = (unsigned *)take(sizeof(unsigned));
    s.diag = (double *)take(8 * (size_t)n);
    s.dinv = (double *)take(8 * (size_t)((n + 255) / 256 * 256));
    s.lpart = (double *)take(sizeof(double) * MAXB_ROW);
    s.gpart = (float *)take(sizeof(float) * (size_t)MAXB_BACK * NPARAM);
    s.feat = (uint16_t *)take(2 * (size_t)n * NF);
    s.h1 = (uint16_t *)take(2 * (size_t)n * NH);
    s.h2 = (uint16_t *)take(2 * (size_t)n * NH);
    s.dO = (uint16_t *)take(2 * (size_t)n * NO);
    s.O = (float *)take(4 * (size_t)n * NO);
    s.pval = (float *)take(4 * (size_t)nnz);
    s.X0 = (double *)take(8 * (size_t)n * K);
    s.X1 = (double *)take(8 * (size_t)n * K);
    s.dP = (double *)take(8 * (size_t)nnz);
    if (total)
        *total = off;
    return s;
}

bool a16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

bool csr_ok(const cbg_csr *A)
{
    return A && A->n >= 0 && A->nnz >= 0 && A->nnz <= INT32_MAX &&
           (A->n == 0 || (A->row_ptr && (A->nnz == 0 || (A->col_idx && A->val))));
}

// A carries a whole sliced-ELL copy with one-byte diagonal indices
bool sell_dix_of(const cbg_csr *A)
{
    return A->sell_ptr && A->sell_val && A->sell_dix && A->sell_diag && A->sell_ndiag >= 1 &&
           A->sell_ndiag <= CBG_SELL_MAX_DIAG && A->sell_entries >= A->nnz &&
           A->sell_entries % 64 == 0;
}

bool grid_ok(const cbg_csr *A, const int32_t *grid)
{
    return grid && grid[0] > 0 && grid[1] > 0 && grid[2] > 0 &&
           (int64_t)grid[0] * grid[1] * grid[2] == A->n;
}

int row_grid(int64_t rows) { return (int)std::min<int64_t>(std::max<int64_t>((rows + 255) / 256, 1), MAXB_ROW); }
int group_grid(int64_t rows) { return (int)std::min<int64_t>(std::max<int64_t>((rows + 7) / 8, 1), MAXB_ROW); }
int tile_grid(int64_t n, int cap) { return (int)std::min<int64_t>(std::max<int64_t>((n + 63) / 64, 1), cap); }

int slice_grid(int64_t n)
{
    return (int)std::min<int64_t>(std::max<int64_t>(((n + 63) / 64 + 3) / 4, 1), 65536);
}

// The diagonal, from the sliced-ELL copy when A carries one
void enqueue_diag(const cbg_csr *A, double *diag, hipStream_t s)
{
    if (sell_dix_of(A)) {
        const int g = (int)std::min<int64_t>(std::max<int64_t>(((int64_t)A->n + 255) / 256, 1),
                                             65536);
        hipLaunchKernelGGL(k_diag_sell, dim3(g), dim3(256), 0, s, A->n, A->row_ptr,
                           A->sell_ptr, A->sell_dix, A->sell_val, A->sell_diag, A->sell_ndiag,
                           diag);
    } else {
        hipLaunchKernelGGL(k_diag, dim3(group_grid(A->n)), dim3(256), 0, s, A->n, A->row_ptr,
                           A->col_idx, A->val, diag);
    }
}

SellDix sell_dix(const cbg_csr *A, const int32_t grid[3])
{
    return {A->n,        A->sell_ndiag, grid[0],     grid[1],     ((int64_t)A->n + 63) / 64,
            A->row_ptr,  A->sell_ptr,   A->sell_dix, A->sell_val, A->sell_diag};
}

// The features, from the sliced-ELL copy when A carries one
void enqueue_features(const cbg_csr *A, const int32_t grid[3], const double *diag, uint16_t *feat,
                      unsigned *bad, hipStream_t s, uint32_t *slots = nullptr)
{
    if (sell_dix_of(A)) {
        hipLaunchKernelGGL(k_features_sell, dim3(slice_grid(A->n)), dim3(256), 0, s,
                           sell_dix(A, grid), diag, feat, slots, bad);
    } else {
        hipLaunchKernelGGL(k_features, dim3(group_grid(A->n)), dim3(256), 0, s, A->n,
                           A->row_ptr, A->col_idx, A->val, grid[0], grid[1], diag, feat, bad);
    }
}

size_t ws_need(int64_t n, int64_t nnz, int64_t K)
{
    size_t t = 0;
    carve_spai(nullptr, n, nnz, K, &t);
    return t;
}

#define SP_TRY(x)                           \
    do {                                    \
        const hipError_t e_ = (x);          \
        if (e_ != hipSuccess) {             \
            cbg::note_hip_error(e_, __LINE__); \
            (void)hipGetLastError();        \
            return CBG_E_HIP;               \
        }                                   \
    } while (0)

int ws_check(void *ws, size_t ws_bytes, int64_t n, int64_t nnz, int64_t K)
{
    if (!ws || ((uintptr_t)ws & (SALIGN - 1)) || ws_bytes < ws_need(n, nnz, K))
        return CBG_E_WORKSPACE;
    return CBG_OK;
}

// Reads and clears the device flag (synchronous).
int read_flag(unsigned *bad, hipStream_t s, unsigned *out)
{
    SP_TRY(hipMemcpyAsync(out, bad, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    SP_TRY(hipStreamSynchronize(s));
    return CBG_OK;
}

void enqueue_forward(int64_t n, const uint16_t *feat, const uint16_t *w, const float *prm, float *O,
                     uint16_t *h1, uint16_t *h2, hipStream_t s)
{
    // two blocks per CU: what its registers allow; more only stage the
    // weights again (262,144 rows in 2048 blocks: 99 us, 512: 54 us)
    hipLaunchKernelGGL(k_forward, dim3(tile_grid(n, 512)), dim3(256), 0, s, (int)n, feat, w, prm,
                       O, h1, h2);
}

// Loss and gradient of one matrix: with O (the network's output; grid and the
// diagonal in W.diag set) P comes from it and the gradient goes to dO, else P
// is pval and the gradient dP.
template <bool K32>
void enqueue_loss(const cbg_csr *A, const double *tval, const float *pval, const float *O,
                  const int32_t grid[3], int K, const uint16_t *V, double scale, double *loss,
                  int accumulate, double *dP, uint16_t *dO, const SpaiWs &W, hipStream_t s)
{
    const int gb = (int)std::min<int64_t>(std::max<int64_t>(((int64_t)A->n + QROWS - 1) / QROWS, 1),
                                          MAXB_ROW);
    const int nx = O ? grid[0] : 1, ny = O ? grid[1] : 1;
    const double *diag = W.diag;
    if (O)
        hipLaunchKernelGGL((k_quad_pv<K32, true>), dim3(gb), dim3(256), 0, s, A->n, K, A->row_ptr,
                           A->col_idx, pval, O, diag, nx, ny, V, W.X0);
    else
        hipLaunchKernelGGL((k_quad_pv<K32, false>), dim3(gb), dim3(256), 0, s, A->n, K,
                           A->row_ptr, A->col_idx, pval, O, diag, nx, ny, V, W.X0);
    hipLaunchKernelGGL((k_quad_residual<K32>), dim3(gb), dim3(256), 0, s, A->n, K, A->row_ptr,
                       A->col_idx, A->val, (const double *)W.X0, V, W.X1, W.lpart);
    hipLaunchKernelGGL(k_loss_fold, dim3(1), dim3(256), 0, s, (const double *)W.lpart, gb, scale,
                       accumulate, loss);
    if (O)
        hipLaunchKernelGGL((k_quad_grad<K32, true>), dim3(gb), dim3(256), 0, s, A->n, K,
                           A->row_ptr, A->col_idx, tval, (const double *)W.X1, 2.0 * scale, V, dP,
                           diag, nx, ny, dO);
    else
        hipLaunchKernelGGL((k_quad_grad<K32, false>), dim3(gb), dim3(256), 0, s, A->n, K,
                           A->row_ptr, A->col_idx, tval, (const double *)W.X1, 2.0 * scale, V, dP,
                           diag, nx, ny, dO);
}

int enqueue_grad(const cbg_csr *A, const double *tval, const float *pval, const float *O,
                 const int32_t grid[3], int K, const uint16_t *V, double scale, double *loss,
                 int accumulate, double *dP, uint16_t *dO, const SpaiWs &W, hipStream_t s)
{
    // the 16-byte loads of the K = 32 form: V comes from the caller
    if (K == 32 && a16(V))
        enqueue_loss<true>(A, tval, pval, O, grid, K, V, scale, loss, accumulate, dP, dO, W, s);
    else
        enqueue_loss<false>(A, tval, pval, O, grid, K, V, scale, loss, accumulate, dP, dO, W, s);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int enqueue_backward(int64_t n, const uint16_t *feat, const uint16_t *h1, const uint16_t *h2,
                     const uint16_t *dO, const uint16_t *w, double *grad, int accumulate,
                     const SpaiWs &W, hipStream_t s)
{
    const int nb = tile_grid(n, MAXB_BACK);
    hipLaunchKernelGGL(k_backward, dim3(nb), dim3(256), 0, s, (int)n, feat, h1, h2, dO, w,
                       W.gpart);
    hipLaunchKernelGGL(k_grad_fold, dim3((NPARAM + FOLD_E - 1) / FOLD_E), dim3(256), 0, s,
                       (const float *)W.gpart, nb, accumulate, grad);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

}  // namespace

extern "C" {

size_t cbg_spai_workspace_bytes(int32_t n, int64_t nnz, int32_t K)
{
    if (n < 0 || nnz < 0 || K < 0 || K > CBG_SPAI_MAX_K)
        return 0;
    return ws_need(n, nnz, K);
}

int cbg_spai_features(const cbg_csr *A, const int32_t grid[3], uint16_t *feat, void *ws,
                      size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && !a16(feat)) || !feat)
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, 0);
    if (e)
        return e;
    if (A->n == 0)
        return CBG_OK;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, 0, nullptr);
    SP_TRY(hipMemsetAsync(W.bad, 0, sizeof(unsigned), s));
    enqueue_diag(A, W.diag, s);
    enqueue_features(A, grid, (const double *)W.diag, feat, W.bad, s);
    SP_TRY(hipGetLastError());
    unsigned bad = 0;
    if ((e = read_flag(W.bad, s, &bad)))
        return e;
    return bad ? CBG_E_NONFINITE : CBG_OK;
}

int cbg_mlp_forward(int32_t n, const uint16_t *feat, const uint16_t *weights, const float *params,
                    float *out, uint16_t *h1, uint16_t *h2, void *stream)
{
    if (n < 0 || (n > 0 && (!feat || !weights || !params || !out)) || !a16(feat) || !a16(out) ||
        !a16(h1) || !a16(h2) || ((h1 == nullptr) != (h2 == nullptr)) || !a16(weights) ||
        !a16(params))
        return CBG_E_ARG;
    if (n == 0)
        return CBG_OK;
    enqueue_forward(n, feat, weights, params, out, h1, h2, (hipStream_t)stream);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int cbg_spai_assemble(const cbg_csr *A, const int32_t grid[3], const float *out, float *p_val,
                      void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && (!out || !p_val)))
        return CBG_E_ARG;
    if (A->n == 0)
        return CBG_OK;
    hipLaunchKernelGGL(k_assemble, dim3(group_grid(A->n)), dim3(256), 0, (hipStream_t)stream, A->n,
                       A->row_ptr, A->col_idx, A->val, grid[0], grid[1], out, p_val);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int cbg_learned_build(const cbg_csr *A, const int32_t grid[3], const uint16_t *weights,
                      const float *params, float *p_val, void *ws, size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && (!weights || !params || !p_val)) ||
        !a16(weights) || !a16(params))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, 0);
    if (e)
        return e;
    if (A->n == 0)
        return CBG_OK;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, 0, nullptr);
    SP_TRY(hipMemsetAsync(W.bad, 0, sizeof(unsigned), s));
    enqueue_diag(A, W.diag, s);
    enqueue_features(A, grid, (const double *)W.diag, W.feat, W.bad, s);
    enqueue_forward(A->n, W.feat, weights, params, W.O, nullptr, nullptr, s);
    hipLaunchKernelGGL(k_assemble, dim3(group_grid(A->n)), dim3(256), 0, s, A->n, A->row_ptr,
                       A->col_idx, A->val, grid[0], grid[1], (const float *)W.O, p_val);
    SP_TRY(hipGetLastError());
    unsigned bad = 0;
    if ((e = read_flag(W.bad, s, &bad)))
        return e;
    return bad ? CBG_E_NONFINITE : CBG_OK;
}

int cbg_learned_build_stencil(const cbg_csr *A, const int32_t grid[3], const uint16_t *weights,
                              const float *params, uint16_t *p_stencil, void *ws,
                              size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && (!weights || !params || !p_stencil)) ||
        !a16(weights) || !a16(params) || !a16(p_stencil))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, 0);
    if (e)
        return e;
    if (A->n == 0)
        return CBG_OK;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, 0, nullptr);
    const int64_t ld = cbg_basis_ld(A->n);
    SP_TRY(hipMemsetAsync(W.bad, 0, sizeof(unsigned), s));
    enqueue_diag(A, W.diag, s);
    if (sell_dix_of(A)) {
        uint32_t *slots = (uint32_t *)W.O;          // a word a row where 32 outputs would be
        enqueue_features(A, grid, (const double *)W.diag, W.feat, W.bad, s, slots);
        const int gb = (int)std::min<int64_t>(ld / 256, 512);       // two blocks per CU
        hipLaunchKernelGGL(k_forward_codes, dim3(gb), dim3(256), 0, s, A->n, ld, W.feat, slots,
                           weights, params, p_stencil);
    } else {
        enqueue_features(A, grid, (const double *)W.diag, W.feat, W.bad, s);
        enqueue_forward(A->n, W.feat, weights, params, W.O, nullptr, nullptr, s);
        const int gp = (int)std::min<int64_t>((ld + PK_ROWS - 1) / PK_ROWS, MAXB_ROW);
        hipLaunchKernelGGL(k_stencil_pack, dim3(std::max(gp, 1)), dim3(256), 0, s, A->n, ld,
                           A->row_ptr, A->col_idx, grid[0], grid[1], (const float *)W.O,
                           p_stencil);
    }
    SP_TRY(hipGetLastError());
    unsigned bad = 0;
    if ((e = read_flag(W.bad, s, &bad)))
        return e;
    return bad ? CBG_E_NONFINITE : CBG_OK;
}

int cbg_stencil_apply(const cbg_csr *A, const int32_t grid[3], const uint16_t *p_stencil,
                      const double *v, double *z, void *ws, size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && (!p_stencil || !v || !z)) ||
        !a16(p_stencil))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, 0);
    if (e)
        return e;
    if (A->n == 0)
        return CBG_OK;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, 0, nullptr);
    const int64_t ld = cbg_basis_ld(A->n);
    SP_TRY(hipMemsetAsync(W.bad, 0, sizeof(unsigned), s));
    SpmvArgs am{};
    am.n = A->n;
    am.rp = A->row_ptr;
    am.ci = A->col_idx;
    am.val = A->val;
    if (sell_dix_of(A)) {
        am.sp = A->sell_ptr;
        am.sv = A->sell_val;
        am.sd = A->sell_dix;
        am.sdiag = A->sell_diag;
        am.ndiag = A->sell_ndiag;
    }
    launch_jacobi_setup(am, ld, W.dinv, W.bad, s);
    launch_stencil(F_FP64, 1, v, A->n, ld, grid, p_stencil, W.dinv, z, nullptr, nullptr, nullptr,
                   s);
    SP_TRY(hipGetLastError());
    unsigned bad = 0;
    if ((e = read_flag(W.bad, s, &bad)))
        return e;
    return bad ? CBG_E_ARG : CBG_OK;
}

int cbg_csr_transpose_values(const cbg_csr *A, double *t_val, void *ws, size_t ws_bytes,
                             void *stream)
{
    if (!csr_ok(A) || (A->nnz > 0 && !t_val))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, 0);
    if (e)
        return e;
    if (A->n == 0)
        return CBG_OK;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, 0, nullptr);
    SP_TRY(hipMemsetAsync(W.bad, 0, sizeof(unsigned), s));
    hipLaunchKernelGGL(k_transpose_values, dim3(row_grid(A->n)), dim3(256), 0, s, A->n,
                       A->row_ptr, A->col_idx, A->val, t_val, W.bad);
    SP_TRY(hipGetLastError());
    unsigned bad = 0;
    if ((e = read_flag(W.bad, s, &bad)))
        return e;
    return bad ? CBG_E_UNSUPPORTED : CBG_OK;
}

int cbg_spai_pack(const double *V, int64_t ld, int32_t n, int32_t K, int32_t first,
                  int32_t stride, uint16_t *out, void *stream)
{
    if (n < 0 || K < 0 || K > CBG_SPAI_MAX_K || first < 0 || stride < 1 || ld < n ||
        (n > 0 && K > 0 && (!V || !out)))
        return CBG_E_ARG;
    if (n == 0 || K == 0)
        return CBG_OK;
    const int64_t total = (int64_t)n * K;
    hipLaunchKernelGGL(k_pack, dim3(row_grid(total)), dim3(256), 0, (hipStream_t)stream, V, ld, n,
                       K, first, stride, out);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int cbg_spai_grad_p(const cbg_csr *A, const double *t_val, const float *p_val, int32_t K,
                    const uint16_t *V, double scale, double *loss, int32_t accumulate,
                    double *dP, void *ws, size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || K < 1 || K > CBG_SPAI_MAX_K || !loss ||
        (A->n > 0 && (!t_val || !p_val || !V || !dP)) || !isfinite(scale))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, K);
    if (e)
        return e;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, K, nullptr);
    return enqueue_grad(A, t_val, p_val, nullptr, nullptr, K, V, scale, loss, accumulate, dP,
                        nullptr, W, s);
}

int cbg_spai_grad_o(const cbg_csr *A, const int32_t grid[3], const double *dP, uint16_t *dO,
                    void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || (A->n > 0 && (!dP || !dO)) || !a16(dO))
        return CBG_E_ARG;
    if (A->n == 0)
        return CBG_OK;
    hipLaunchKernelGGL(k_grad_o, dim3(group_grid(A->n)), dim3(256), 0, (hipStream_t)stream, A->n,
                       A->row_ptr, A->col_idx, A->val, grid[0], grid[1], dP, dO);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int cbg_mlp_backward(int32_t n, const uint16_t *feat, const uint16_t *h1, const uint16_t *h2,
                     const uint16_t *dO, const uint16_t *weights, double *grad,
                     int32_t accumulate, void *ws, size_t ws_bytes, void *stream)
{
    if (n < 0 || !grad || !weights || (n > 0 && (!feat || !h1 || !h2 || !dO)))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, n, 0, 0);
    if (e)
        return e;
    SpaiWs W = carve_spai(ws, n, 0, 0, nullptr);
    hipStream_t s = (hipStream_t)stream;
    // the kernel's 8-byte loads: an input that is not so aligned is read from a
    // copy in the workspace
    auto aligned = [&](const uint16_t *&p, void *copy, size_t count) {
        if (((uintptr_t)p & 7u) == 0)
            return hipSuccess;
        const hipError_t r = hipMemcpyAsync(copy, p, 2 * count, hipMemcpyDeviceToDevice, s);
        p = (const uint16_t *)copy;
        return r;
    };
    static_assert(sizeof(double) * MAXB_ROW >= 2 * NWBF, "the weights' copy fits the loss partials");
    SP_TRY(aligned(feat, W.feat, (size_t)n * NF));
    SP_TRY(aligned(h1, W.h1, (size_t)n * NH));
    SP_TRY(aligned(h2, W.h2, (size_t)n * NH));
    SP_TRY(aligned(dO, W.dO, (size_t)n * NO));
    SP_TRY(aligned(weights, W.lpart, NWBF));
    return enqueue_backward(n, feat, h1, h2, dO, weights, grad, accumulate, W, s);
}

int cbg_spai_loss_grad(const cbg_csr *A, const double *t_val, const int32_t grid[3],
                       const uint16_t *feat, const uint16_t *weights, const float *params,
                       int32_t K, const uint16_t *V, double scale, double *loss, double *grad,
                       int32_t accumulate, void *ws, size_t ws_bytes, void *stream)
{
    if (!csr_ok(A) || !grid_ok(A, grid) || K < 1 || K > CBG_SPAI_MAX_K || !loss || !grad ||
        !weights || !params || (A->n > 0 && (!t_val || !feat || !V)) || !a16(feat) ||
        !a16(weights) || !a16(params) || !isfinite(scale))
        return CBG_E_ARG;
    int e = ws_check(ws, ws_bytes, A->n, A->nnz, K);
    if (e)
        return e;
    hipStream_t s = (hipStream_t)stream;
    SpaiWs W = carve_spai(ws, A->n, A->nnz, K, nullptr);
    if (A->n == 0) {
        hipLaunchKernelGGL(k_loss_fold, dim3(1), dim3(256), 0, s, (const double *)W.lpart, 0, 0.0,
                           accumulate, loss);
        hipLaunchKernelGGL(k_grad_fold, dim3((NPARAM + FOLD_E - 1) / FOLD_E), dim3(256), 0, s,
                           (const float *)W.gpart, 0, accumulate, grad);
        SP_TRY(hipGetLastError());
        return CBG_OK;
    }
    enqueue_forward(A->n, feat, weights, params, W.O, W.h1, W.h2, s);
    enqueue_diag(A, W.diag, s);
    if ((e = enqueue_grad(A, t_val, nullptr, W.O, grid, K, V, scale, loss, accumulate, nullptr,
                          W.dO, W, s)))
        return e;
    return enqueue_backward(A->n, feat, W.h1, W.h2, W.dO, weights, grad, accumulate, W, s);
}

int cbg_spai_round_weights(const float *params, uint16_t *weights, void *stream)
{
    if (!params || !weights)
        return CBG_E_ARG;
    hipLaunchKernelGGL(k_round_weights, dim3((NWBF + 255) / 256), dim3(256), 0,
                       (hipStream_t)stream, params, weights);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

int cbg_adam_step(float *params, float *m1, float *m2, uint16_t *weights, const double *grad,
                  int64_t t, double lr, double beta1, double beta2, double eps, void *stream)
{
    if (!params || !m1 || !m2 || !weights || !grad || t < 1 || !(lr > 0) || !(beta1 >= 0) ||
        !(beta1 < 1) || !(beta2 >= 0) || !(beta2 < 1) || !(eps > 0))
        return CBG_E_ARG;
    const double c1 = 1.0 - pow(beta1, (double)t), c2 = 1.0 - pow(beta2, (double)t);
    hipLaunchKernelGGL(k_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       params, m1, m2, weights, grad, lr, beta1, beta2, eps, c1, c2);
    SP_TRY(hipGetLastError());
    return CBG_OK;
}

}  // extern "C"
