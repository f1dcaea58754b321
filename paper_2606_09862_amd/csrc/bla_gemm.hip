// Row-major bf16 product Y [m, n] = X [m, k] W [k, n] with float32 accumulation: the projections of
// a layer (the sizes: gemm_takes).
//
// A workgroup of four waves forms a BT x BT tile of Y, each wave a quarter (WT x WT); the reduction
// runs in blocks of 64 staged through LDS, the next block loaded into registers meanwhile.  The
// products are formed transposed (rows: columns of W, columns: tokens), so that a lane holds four
// consecutive elements of a token's row; W is read transposed from its row-major tile
// (ds_read_b64_tr_b16).  Row strides of 36 and of 8 x odd dwords keep both reads free of bank
// conflicts.
//
// With k = D of a few hundred the product moves about as many bytes as it has operations for, and
// what costs is its start: the tiles of one row block run on one XCD, so that X comes from HBM
// once, and three workgroups share a compute unit.  32768 tokens of width 256 to 768 columns take
// 29 us (430 TFLOP/s; the library's kernel 31); keeping a workgroup on its column tile for several
// row blocks, with the next block's first pieces loaded under the last products, took 32.
#include <stdint.h>

#include "bla_device.h"
#include "bla_plan.h"

namespace bla {

template <int BT> struct Gemm {
    static constexpr int BK = 64, WT = BT / 2, NT = WT / 16;  // tiles per wave and direction
    static constexpr int LX = BK + 8, LW = BT + 16;
    static constexpr int PX = BT * BK / 8 / 256, PW = BK * BT / 8 / 256;  // 16-byte pieces per thread
    static_assert(BT == 128 || BT == 64, "row strides");
};

template <int BT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BT == 128 ? 3 : 4))) void gemm_kernel(const bf16* X, const bf16* W, bf16* Y, long long m, int n, int k)
{
    using G = Gemm<BT>;
    using F = bf16x8;
    constexpr int BK = G::BK, WT = G::WT, NT = G::NT, LX = G::LX, LW = G::LW;
    __shared__ __attribute__((aligned(16))) bf16 sX[BT * LX];
    __shared__ __attribute__((aligned(16))) bf16 sW[BK * LW];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wv & 1, wm = wv >> 1;
    // Workgroups are dealt to the eight XCDs by index: the column tiles of one row block share one.
    const int ntn = (n + BT - 1) / BT, xq = blockIdx.x / 8;
    const long long m0 = ((long long)(xq / ntn) * 8 + blockIdx.x % 8) * BT;
    const int n0 = (xq % ntn) * BT;
    if (m0 >= m) return;  // grid padding (whole workgroup, before any barrier)

    // Pieces of the next block: rows past m and columns past n re-read the last ones (their products
    // are not stored); reduction indices past k are zero.
    F px[G::PX], pw[G::PW];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < G::PX; ++i) {
            const int u = tid + 256 * i, row = u / (BK / 8), col = 8 * (u % (BK / 8));
            const long long mr = m0 + row < m ? m0 + row : m - 1;
            px[i] = k0 + col < k ? *reinterpret_cast<const F*>(X + (size_t)mr * k + k0 + col) : zero_frag<bf16>();
        }
#pragma unroll
        for (int i = 0; i < G::PW; ++i) {
            const int u = tid + 256 * i, row = u / (BT / 8), col = 8 * (u % (BT / 8));
            const int nc = n0 + col < n ? n0 + col : n - 8;
            pw[i] = k0 + row < k ? *reinterpret_cast<const F*>(W + (size_t)(k0 + row) * n + nc) : zero_frag<bf16>();
        }
    };
    floatx4 acc[NT][NT];  // [column tile][token tile]
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = zero4();
    load(0);
    for (int k0 = 0; k0 < k; k0 += BK) {
        __syncthreads();  // the previous block is read
#pragma unroll
        for (int i = 0; i < G::PX; ++i) {
            const int u = tid + 256 * i;
            *reinterpret_cast<F*>(sX + (u / (BK / 8)) * LX + 8 * (u % (BK / 8))) = px[i];
        }
#pragma unroll
        for (int i = 0; i < G::PW; ++i) {
            const int u = tid + 256 * i;
            *reinterpret_cast<F*>(sW + (u / (BT / 8)) * LW + 8 * (u % (BT / 8))) = pw[i];
        }
        __syncthreads();
        if (k0 + BK < k) load(k0 + BK);
#pragma unroll
        for (int kb = 0; kb < BK / 32; ++kb) {
            F xf[NT], wf[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) xf[j] = ld_frag_2x8(sX + (wm * WT + 16 * j + r) * LX, kb, g);
#pragma unroll
            for (int i = 0; i < NT; ++i) wf[i] = ld_frag_tr(sW, LW, wn * WT + 16 * i, kb, g, r);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mma(wf[i], xf[j], acc[i][j]);
        }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const long long row = m0 + wm * WT + 16 * j + r;
        if (row < m) {
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int col = n0 + wn * WT + 16 * i + 4 * g;
                if (col < n) st4<bf16>(Y + (size_t)row * n + col, acc[i][j]);
            }
        }
    }
}

// The sizes that this kernel takes from the vendor library.  A workgroup walks its reduction alone, so a long
// one leaves the chip idle where the library splits it (a layer of 16 tokens of width 1536: library 38 us /
// this kernel 55, 200 of 2048 59 / 88); and for large products of widths that are multiples of 256, or past
// 512, the library has kernels that are faster once the device, not its 18 us of host time, is what a
// product takes (one product: 32768 tokens of width 512 to 1536 columns 62 / 71, 8192 22 / 22; 65536 of
// width 256 to 768 columns 42 / 47, 32768 29 / 27; 8528 of 640 to 640 17 / 22, but a whole layer of 4000
// of 640 59 / 51, of 1000 of 1024 43 / 42).  Widths between those it has none for: 65536 of 384 to 1152 118 / 86,
// 131072 of 448 to 448 108 / 83.  Both products of a layer go the same way (n does not matter).
bool gemm_takes(long long m, long long n, long long k)
{
    if (m <= 0 || n <= 0 || k <= 0 || n % 8 || k % 8 || n > INT32_MAX || k > INT32_MAX) return false;
    if (k < 512 && k % 256) return true;
    return (double)m * (double)k * (double)k <= (k <= 768 ? 2.2e9 : k <= 1024 ? 1.1e9 : 0.0);
}

hipError_t launch_gemm(const bf16* X, const bf16* W, bf16* Y, long long m, int n, int k, hipStream_t s)
{
    if (!gemm_takes(m, n, k)) return hipErrorInvalidValue;
    auto grid = [&](int bt) { return ((m + bt - 1) / bt + 7) / 8 * 8 * ((n + bt - 1) / bt); };
    const long long big = grid(128), small = grid(64);
    if (big > INT32_MAX) return hipErrorInvalidValue;
    // 128 x 128 tiles once they give every compute unit one, else 64 x 64 (32768 tokens of width 256:
    // a layer takes 76 us with the large tiles, 82 with the small ones)
    if (big >= 256)
        hipLaunchKernelGGL(gemm_kernel<128>, dim3((unsigned)big), dim3(256), 0, s, X, W, Y, m, n, k);
    else
        hipLaunchKernelGGL(gemm_kernel<64>, dim3((unsigned)small), dim3(256), 0, s, X, W, Y, m, n, k);
    return hipGetLastError();
}

}  // namespace bla
