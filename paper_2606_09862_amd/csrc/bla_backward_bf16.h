// Backward pass of the chunked BLA operator, bf16 operands: the same gradients and the same
// reverse walk as bla_backward.h (whose header states the per-chunk algebra), reorganised so
// that every table read inside the chunk loop comes from LDS.
//
//  * Token tiles (K, V, Q, dO) are staged once, row-major; the orientation with the reduction
//    over tokens is read with the transposing LDS load (ld_frag_tr).
//  * The head's phase table is held in LDS as conj(rho^i) = [cos | -sin] (row i).  It serves the
//    twiddles, the transposed operands of G conj(E), the state rebuilt by subtraction,
//        Z'_in = conj(rho^c) o Z'_out - sum_i conj(rho^i) [k_i | v_i],
//    the H tiles and the adjoint terms of dk and dv without a sign change, when the readout
//    weights are kept as [Re W'' | -Im W''] (which is also conj(W'') as the adjoint update uses
//    it).  The slot matrix scale (A | B) is held once; its transpose (the reduction over slots)
//    is read with ld_frag_tr.
//  * The adjoint is split by head-dim tiles (wave w owns d-tile w, for all modes), so the
//    adjoint terms of dk and dv, Re(rho^j o conj(rho^c) Gam'), are contractions of the wave's
//    own registers against the phase table: no adjoint is published through LDS.
//  * The forward summaries use Z' <- rho^c o (Z' + sum_i conj(rho^i) [k_i | v_i]).
#pragma once

#include "bla_backward.h"
#include "bla_forward_pair.h"

namespace bla {

template <int D, int MP, int SP> struct Bwd16 {
    static constexpr int C = kChunk, NT = C / 16, NTHR = 512, NWS = 4;  // eight waves: two sides of four
    static constexpr int NMT = MP / 16, NDT = D / 16, NST = SP / 16;
    static constexpr int KBD = D / 32, KBM = 2 * MP / 32, KBC = C / 32, KBS = SP / 32;
    // slot rows held in LDS (bla_device.h, slot folding)
    static constexpr bool FOLD = slots_folded(SP);
    static constexpr int HP = slot_rows(SP), NHT = HP / 16, KBH = HP / 32, ABROWS = FOLD ? HP + 1 : SP;
    // waves of a side that share a mode tile (they split its token tiles) and a head-dim tile
    // (they split its keys)
    static constexpr int NRM = NWS / NMT, NRD = NWS / NDT;
    static constexpr int LDQ = D + 12;                // token tiles [C][LDQ] (read both ways)
    static constexpr int LDK = C + 4;                 // Gram tiles [C][LDK]
    static constexpr int LE = 2 * MP + 12;            // phase table [C][LE]; slot matrix [ABROWS][LE]
    // Tiles written row-major by the wave that produces them (8-byte stores) and read
    // transposed (ds_read_b64_tr_b16).  Where the LDS allows it without costing a workgroup
    // per compute unit (PS), they are piece-swizzled (pswz_col) at row strides of 8 x odd
    // (mod 64) dwords, so that neither the stores nor the transposed reads meet bank conflicts;
    // otherwise a stride of 2 (mod 32) dwords keeps the stores conflict-free.
    static constexpr size_t s_elems() { return ((size_t)ABROWS * LE + 7) / 8 * 8; }
    static constexpr size_t lds_bytes(int tp)
    {
        const int ldh = C + tp, ldw = 2 * MP + tp, ldz = D + tp;
        return ((size_t)4 * C * LDQ + (size_t)2 * C * (ldh > LDK ? ldh : LDK) + (size_t)2 * C * ldw +
                (size_t)2 * MP * ldz + (size_t)C * LE + s_elems()) * 2 +
               (size_t)SP * 4 + (size_t)2 * 2 * MP * 4;
    }
    static constexpr bool PS =
        lds_bytes(16) <= kBwdMaxLds && (2 * lds_bytes(16) <= kBwdMaxLds || 2 * lds_bytes(4) > kBwdMaxLds);
    static constexpr int TP = PS ? 16 : 4;
    static constexpr int LDH = C + TP;                // H tiles [query][key]
    static constexpr int LDW = 2 * MP + TP;           // U, Y, then the readout weights: [token][Re m | Im m]
    static constexpr int LDZ = D + TP;                // Z'_k [Re m | Im m][d]
    __device__ static int tcol(int row, int col) { return PS ? pswz_col(row, col) : col; }
    __device__ static bf16x8 ld_t(const bf16* M, int ld, int x0, int kb, int g, int r)
    {
        return PS ? ld_frag_tr_ps(M, ld, x0, kb, g, r) : ld_frag_tr(M, ld, x0, kb, g, r);
    }
    // row fragment (accumulator reduction order) of row `row` of such a tile
    __device__ static bf16x8 ld_row(const bf16* M, int ld, int row, int kb, int g)
    {
        const bf16* q = M + (size_t)row * ld + 32 * kb;
        return join(ld4_lds(q + tcol(row, 4 * g)), ld4_lds(q + 16 + tcol(row, 4 * g)));
    }
    static constexpr size_t A_ELEMS = (size_t)4 * C * LDQ;
    static constexpr size_t G_ELEMS = (size_t)2 * C * (LDH > LDK ? LDH : LDK);
    static constexpr size_t B_ELEMS = (size_t)2 * C * LDW;
    static constexpr size_t Z_ELEMS = (size_t)2 * MP * LDZ;
    static constexpr size_t E_ELEMS = (size_t)C * LE;
    static constexpr size_t S_ELEMS = s_elems();
    static constexpr size_t LDS_BYTES =
        (A_ELEMS + G_ELEMS + B_ELEMS + Z_ELEMS + E_ELEMS + S_ELEMS) * 2 + (size_t)SP * 4 + (size_t)2 * 2 * MP * 4;
    static_assert(LDS_BYTES <= kBwdMaxLds, "backward tiles fit in LDS");
    static_assert((size_t)2 * C * LDH <= G_ELEMS, "H tiles fit in the Gram region");
    // the slot weights handed from one side to the other: four accumulator tiles per query tile in
    // the Gram region, four more in the query tile's own U rows
    static_assert((size_t)NT * (NST < 4 ? NST : 4) * 64 * 16 <= G_ELEMS * 2, "slot weights fit in the Gram region");
    static_assert(NST <= 4 || (size_t)(NST - 4) * 64 * 16 <= (size_t)16 * LDW * 2, "... and in the U rows");
    // staging: 16-byte pieces of the four token tensors
    static constexpr int PIECES = 4 * C * D / 8, PPT = PIECES / NTHR;
    static_assert(PIECES % NTHR == 0 && NMT <= NWS && NDT <= NWS, "tiles split evenly over the waves");
};

__device__ __forceinline__ bf16x8 neg_frag(bf16x8 f)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 u = __builtin_bit_cast(u32x4, f);
    u ^= 0x80008000u;
    return __builtin_bit_cast(bf16x8, u);
}

// Row-major staging of NTEN tensors into [C][ld] tiles (rows past c are zero).
template <int D, int NTEN>
__device__ __forceinline__ void bstage_store_rows(const BStage<bf16, D, NTEN>& st, bf16* const* dst, int ld, int c,
                                                  int tid)
{
    using S = BStage<bf16, D, NTEN>;
    using H = bf16x4;
    const H z = zero_half<bf16>();
#pragma unroll
    for (int i = 0; i < S::PT; ++i) {
        const int u = tid + i * kThreads;
        if ((NTEN * S::UPT) % kThreads == 0 || u < NTEN * S::UPT) {
            const int ten = u / S::UPT, uu = u % S::UPT, dq = uu % (D / 8), tq = uu / (D / 8);
            bf16* rd = dst[ten] + 8 * dq;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool ok = 4 * tq + t < c;
                st_lds<H>(rd + (size_t)(4 * tq + t) * ld, ok ? st.x[i][t][0] : z);
                st_lds<H>(rd + (size_t)(4 * tq + t) * ld + 4, ok ? st.x[i][t][1] : z);
            }
        }
    }
}

// The head's phase table as conj(rho^i) = [cos | -sin] rows into LDS ([C][ld]), from the
// workspace table [C][2MP] of rho^i.
template <int MP, int NTHR = kThreads>
__device__ __forceinline__ void copy_conj_phase(bf16* dst, int ld, const bf16* src, int tid)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int PIECES = kChunk * 2 * MP / 4;
    for (int u = tid; u < PIECES; u += NTHR) {
        const int row = u / (2 * MP / 4), col = (u % (2 * MP / 4)) * 4;
        u32x2 x = *reinterpret_cast<const u32x2*>(src + (size_t)row * 2 * MP + col);
        if (col >= MP) x ^= 0x80008000u;
        *reinterpret_cast<u32x2*>(dst + (size_t)row * ld + col) = x;
    }
}

// cos | sin of m w c (float32, 2MP) for the chunk's length: the LDS row of rho^C, or the
// workspace's phase table for a ragged chunk.
__device__ __forceinline__ const float* rho_row(const float* sRho, int c, int MP)
{
    return c == kChunk ? sRho : sRho + 2 * MP;
}

// sRho[0 .. 2MP): rho^C; sRho[2MP .. 4MP): rho^c of the sequence's last chunk (c = L - (nch-1) C,
// the only chunk that can be shorter).  Both rows live in LDS, so the selected row is read
// with LDS loads (a row chosen between LDS and global memory would be read with flat loads,
// which hold every LDS wait until they return).
template <int NTHR = kThreads>
__device__ __forceinline__ void load_rho_rows(float* sRho, const float* E32h, const BwdArgs& a, int MP, int tid)
{
    const int c_last = a.L - (a.nch - 1) * kChunk;
    for (int i = tid; i < 2 * MP; i += NTHR) {
        sRho[i] = E32h[(size_t)kChunk * 2 * MP + i];
        sRho[2 * MP + i] = E32h[(size_t)c_last * 2 * MP + i];
    }
}

// ---------------------------------------------------------------------------------
// Forward summaries (bf16): per (b, h, summary block) the pre-rotated state after the block's
// tokens from zero, stored as [k|v][re|im][MP][D] (as bwd_fsum_kernel).
//
// Little arithmetic per byte, so what counts is how many loads are in flight: one workgroup takes
// the keys or the values of a block (two per block), stages four chunks ahead in registers and
// one in LDS, and holds its phase fragments in registers.  The waves that share a mode tile split
// its head-dim tiles.  (256 blocks of 8 chunks, d = 64, M = 32: 15.0 -> 10.6 us; 512 of 16 chunks at
// M = 64: 37.5 -> 33.6.)
template <int D, int MP> struct FSum16 {
    static constexpr int C = kChunk, KBC = C / 32, NMT = MP / 16, NDT = D / 16, NW = kThreads / 64;
    static constexpr int NRM = NW / NMT, ODT = (NDT + NRM - 1) / NRM;  // waves per mode tile, head-dim tiles of each
    // K, V and the phase table are read only transposed: row strides of 8 x odd (mod 64) dwords
    // keep those reads free of bank conflicts
    static constexpr int LDQ = D + 16, LE = 2 * MP + 16;
    static constexpr int NPF = 4, PPT = C * D / 8 / kThreads;
    static_assert(NMT <= NW && C * D / 8 % kThreads == 0 && NPF % 2 == 0, "tiles and pieces split evenly");
};

template <int D, int MP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void bwd16_fsum_kernel(BwdArgs a)
{
    using G = FSum16<D, MP>;
    using F = bf16x8;
    constexpr int C = G::C, NDT = G::NDT, ODT = G::ODT, LDQ = G::LDQ, LE = G::LE, NPF = G::NPF;
    constexpr int E_ELEMS = C * LE, X_ELEMS = C * LDQ;
    __shared__ __attribute__((aligned(16))) bf16 lds[2 * X_ELEMS > E_ELEMS ? 2 * X_ELEMS : E_ELEMS];
    __shared__ __attribute__((aligned(16))) float sRhoC[2 * 2 * MP];
    const int tid = threadIdx.x, g = (tid & 63) >> 4, r = tid & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), mt = w % G::NMT, d0 = w / G::NMT * ODT;
    const int side = blockIdx.x & 1, ub = blockIdx.x >> 1;
    const int blk = ub % a.nbk, bh = ub / a.nbk, h = bh % a.H;
    const int ch0 = blk * a.cpb, nch = min(a.cpb, a.nch - ch0);
    const bf16* src = (const bf16*)(side ? a.v : a.k) + (size_t)bh * a.L * D;
    const float* E32h = a.E32 + (size_t)h * (C + 1) * 2 * MP;

    // stages are unconditional (chunks past the block re-read its last): the wait before each
    // store covers exactly that stage's loads
    F st[NPF][G::PPT];
    auto load = [&](F (&x)[G::PPT], int n) {
        const int tok0 = (ch0 + max(min(n, nch - 1), 0)) * C, c = min(C, a.L - tok0);
#pragma unroll
        for (int i = 0; i < G::PPT; ++i) {
            const int u = tid + kThreads * i, row = min(u / (D / 8), c - 1);
            x[i] = ld_global<F>(src + (size_t)tok0 * D + (unsigned)(row * D + 8 * (u % (D / 8))));
        }
    };
    auto store = [&](const F (&x)[G::PPT], int n, bf16* buf) {
        const int c = n < nch ? min(C, a.L - (ch0 + n) * C) : 0;
#pragma unroll
        for (int i = 0; i < G::PPT; ++i) {
            const int u = tid + kThreads * i, row = u / (D / 8);
            st_lds<F>(buf + row * LDQ + 8 * (u % (D / 8)), row < c ? x[i] : zero_frag<bf16>());
        }
    };
#pragma unroll
    for (int i = 0; i < NPF; ++i) load(st[i], i);
    copy_conj_phase<MP>(lds, LE, (const bf16*)a.Etab + (size_t)h * C * 2 * MP, tid);
    load_rho_rows(sRhoC, E32h, a, MP, tid);
    __syncthreads();
    F ef[G::KBC][2];
#pragma unroll
    for (int kb = 0; kb < G::KBC; ++kb)
#pragma unroll
        for (int p = 0; p < 2; ++p) ef[kb][p] = ld_frag_tr(lds, LE, p * MP + 16 * mt, kb, g, r);
    __syncthreads();  // the phase table is in registers: its place takes the chunks
    store(st[0], 0, lds);
    load(st[0], NPF);
    __syncthreads();

    floatx4 Z[2][ODT];  // [d][m] tiles
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < ODT; ++i) Z[p][i] = zero4();
    for (int n0 = 0; n0 < nch; n0 += NPF) {
#pragma unroll
        for (int s = 0; s < NPF; ++s) {
            const int n = n0 + s, s1 = (s + 1) % NPF;
            store(st[s1], n + 1, lds + (s1 & 1) * X_ELEMS);
            load(st[s1], n + 1 + NPF);
            const bf16* X = lds + (s & 1) * X_ELEMS;
            if (n < nch) {
                // Z' <- rho^c o (Z' + sum_i conj(rho^i) x_i)
#pragma unroll
                for (int kb = 0; kb < G::KBC; ++kb)
#pragma unroll
                    for (int i = 0; i < ODT; ++i) {
                        const F xf = ld_frag_tr(X, LDQ, 16 * min(d0 + i, NDT - 1), kb, g, r);
#pragma unroll
                        for (int p = 0; p < 2; ++p) Z[p][i] = mma(xf, ef[kb][p], Z[p][i]);
                    }
                const float* rc = rho_row(sRhoC, min(C, a.L - (ch0 + n) * C), MP);
                const float cc = rc[16 * mt + r], ss = rc[MP + 16 * mt + r];
#pragma unroll
                for (int i = 0; i < ODT; ++i) {
                    const floatx4 re = Z[0][i], im = Z[1][i];
                    Z[0][i] = cc * re - ss * im;
                    Z[1][i] = ss * re + cc * im;
                }
            }
            __syncthreads();  // the next chunk visible; this one's buffer free
        }
    }
    float* S = a.fsum + ((size_t)bh * a.nbk + blk) * 4 * MP * D + (size_t)2 * side * MP * D;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < ODT; ++i)
            if (d0 + i < NDT) st4f(S + ((size_t)p * MP + 16 * mt + r) * D + 16 * (d0 + i) + 4 * g, Z[p][i]);
}

// ---------------------------------------------------------------------------------
// Scans over the block summaries, in place, for sequences cut into many blocks (kBwdScanBlocks):
// summary j becomes the pre-rotated state after block j (from the call's input state), or (ADJ) the
// pre-rotated adjoint before block j (from the gradients of the final state, blocks of segment 0
// excluded).  The walks then read one of them instead of combining them all, each unit its own.
// One thread per mode and four head dims; the loads are issued eight summaries at a time.
template <int D, int MP, bool ADJ>
__global__ __launch_bounds__(kThreads) void bwd16_scan_kernel(BwdArgs a)
{
    constexpr int PER = 2 * MP * D / 4, AHEAD = 8;
    const long long gid = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (gid >= (long long)a.B * a.H * PER) return;
    const int bh = (int)(gid / PER), h = bh % a.H, e = (int)(gid % PER);
    const int side = e / (PER / 2), m = e % (PER / 2) / (D / 4), d = 4 * (e % (D / 4));
    const float* E1 = a.E32 + ((size_t)h * (kChunk + 1) + 1) * 2 * MP;
    const float* in = ADJ ? (side ? a.gv_out : a.gk_out) : (side ? a.sv_in : a.sk_in);
    floatx4 zr = zero4(), zi = zero4();
    if (in && m < a.M) {
        const floatx4 xr = ld4f(in + (((size_t)bh * 2 + 0) * a.M + m) * D + d);
        const floatx4 xi = ld4f(in + (((size_t)bh * 2 + 1) * a.M + m) * D + d);
        const float c1 = E1[m], s1 = E1[MP + m];
        zr = c1 * xr - s1 * xi;
        zi = s1 * xr + c1 * xi;
    }
    // every block but the sequence's last is cpb full chunks long; the adjoint rotates backwards
    float cf, sf, cl, sl;
    bwd_phase(m, (long long)a.cpb * kChunk, a.rperiod[h], cf, sf);
    bwd_phase(m, (long long)a.L - (long long)(a.nbk - 1) * a.cpb * kChunk, a.rperiod[h], cl, sl);
    const int first = ADJ ? a.nbk / a.nseg : 0, cnt = a.nbk - first;
    float* S = (ADJ ? a.asum : a.fsum) + (size_t)bh * a.nbk * 4 * MP * D + (size_t)2 * side * MP * D + (size_t)m * D + d;
    for (int j0 = 0; j0 < cnt; j0 += AHEAD) {
        floatx4 sr[AHEAD], si[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int i = min(j0 + u, cnt - 1), j = ADJ ? a.nbk - 1 - i : i;
            sr[u] = ld4f(S + (size_t)j * 4 * MP * D);
            si[u] = ld4f(S + (size_t)j * 4 * MP * D + (size_t)MP * D);
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (j0 + u >= cnt) continue;
            const int j = ADJ ? a.nbk - 1 - (j0 + u) : j0 + u;
            const float c = j == a.nbk - 1 ? cl : cf, s0 = j == a.nbk - 1 ? sl : sf, s = ADJ ? -s0 : s0;
            const floatx4 nr = c * zr - s * zi + sr[u];
            zi = s * zr + c * zi + si[u];
            zr = nr;
            st4f(S + (size_t)j * 4 * MP * D, zr);
            st4f(S + (size_t)j * 4 * MP * D + (size_t)MP * D, zi);
        }
    }
}

// Summary blocks per sequence from which the scans run.  Measured on whole calls (us, combined in
// the walks / scanned), d = M = 64: one sequence of 2000 tokens 177 / 61, 16 of 2000 with 127 slots
// 265 / 114, 32 of 4096 250 / 191.  At four blocks (the LM layer) the scans would move more bytes
// than the walks read.
constexpr int kBwdScanBlocks = 8;

// ---------------------------------------------------------------------------------
// The reverse walk over one (b, h, segment), bf16.  SUM: adjoint summary only.
//
// Eight waves, two per SIMD, in two sides of four.  Side 0 carries what belongs to the keys and
// queries (Z'_k, its Gram tiles, U, the scores, H_v, Gam'_k, dk), side 1 what belongs to the
// values (Z'_v, Gd, Y, dP, H_q, Gam'_v, dv): the phases below are the same for both, so a wave
// holds half of the state and adjoint registers that one wave per SIMD held, and every SIMD has a
// second chain to issue from while one waits.  Only the softmax crosses over: side 0 hands its
// weights to side 1 in float32.  dq is shared out over all eight at the end.  (One wave per SIMD
// took 401 us for the walk and 153 us for the adjoint summaries at 128 sequences of 4096
// tokens, d = M = S = 64; now 328 and 120.)
template <int D, int MP, int SP, bool SUM>
__global__ __launch_bounds__((Bwd16<D, MP, SP>::NTHR)) void bwd16_kernel(BwdArgs a)
{
    using P = Bwd16<D, MP, SP>;
    using F = bf16x8;
    constexpr int C = P::C, NT = P::NT, NMT = P::NMT, NDT = P::NDT, NTHR = P::NTHR;
    constexpr int KBD = P::KBD, KBM = P::KBM, KBC = P::KBC, NST = P::NST, NHT = P::NHT;
    constexpr int LDQ = P::LDQ, LDK = P::LDK, LDW = P::LDW, LE = P::LE;
    __shared__ __attribute__((aligned(16))) char lds_raw[P::LDS_BYTES];
    bf16* Ks = reinterpret_cast<bf16*>(lds_raw);            // region A: token tiles, row-major
    bf16* Vs = Ks + (size_t)C * LDQ;
    bf16* Qs = Vs + (size_t)C * LDQ;
    bf16* dOs = Qs + (size_t)C * LDQ;
    bf16* GT = Ks + P::A_ELEMS;                              // region G: Gram tiles, slot weights, H tiles
    bf16* GdT = GT + (size_t)C * LDK;
    bf16* HqT = GT;                                          // [query][key], LDH
    bf16* HvT = GT + (size_t)C * P::LDH;
    bf16* UT = GT + P::G_ELEMS;                              // region B: U, Y, then the weights
    bf16* YT = UT + (size_t)C * LDW;
    bf16* WqT = UT;                                          // [token][Re m | Im m], LDW
    bf16* WvT = YT;
    bf16* ZkT = UT + P::B_ELEMS;                             // [Re m | Im m][d] of Z'_k, LDZ
    bf16* sE = ZkT + P::Z_ELEMS;                             // conj(rho^i) rows
    bf16* sAB = sE + P::E_ELEMS;                             // scale (A | B) rows
    int* sTheta = reinterpret_cast<int*>(sAB + P::S_ELEMS);
    float* sRhoC = reinterpret_cast<float*>(sTheta + SP);

    const int tid = threadIdx.x, g = (tid & 63) >> 4, r = tid & 15;
    const int tid_ = tid, g_ = g, r_ = r;  // the chunk loop re-derives its own copies
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int side = wv / P::NWS, w = wv % P::NWS;  // side, and wave within it
    const int mt = w % NMT, rm = w / NMT;           // mode tile, and which of the waves that share it
    const int dt = w % NDT, rd = w / NDT;           // head-dim tile, likewise
    // Token tiles of the waves that share a mode or head-dim tile (causal work grows with the
    // index: 0, 3 | 1, 2 for two, one each for four).
    auto mine = [](int t, int part, int parts) {
        return parts == 1 || (parts == 2 ? ((t == 1 || t == 2) == (part == 1)) : t == part);
    };
    // SUM: one summary block of a segment but the first; otherwise one segment.  last_blk:
    // the last summary block the walk covers.
    const int bps = a.nbk / a.nseg;
    const int nsu = SUM ? a.nbk - bps : a.nseg;
    const int seg = blockIdx.x % nsu + (SUM ? bps : 0), bh = blockIdx.x / nsu, h = bh % a.H;
    const int cpu = SUM ? a.cpb : a.cps;  // chunks per walked unit (block or segment)
    const int ch0 = seg * cpu, nch = min(cpu, a.nch - ch0);
    const int last_blk = SUM ? seg : (seg + 1) * bps - 1;
    const bf16* qb = (const bf16*)a.q + (size_t)bh * a.L * D;
    const bf16* kb_ = (const bf16*)a.k + (size_t)bh * a.L * D;
    const bf16* vb = (const bf16*)a.v + (size_t)bh * a.L * D;
    const bf16* gb = (const bf16*)a.dO + (size_t)bh * a.L * D;
    const float* E32h = a.E32 + (size_t)h * (C + 1) * 2 * MP;
    const double rT = a.rperiod[h];
    const float* rho1 = E32h + 2 * MP;
    const float iscale = 1.f / a.scale;

    // Staging of one chunk: 16-byte pieces of K, V, Q, dO (rows past c re-read row c - 1 and are
    // stored as zeros), loaded a chunk ahead.
    F st[P::PPT];
    auto stage_load = [&](int tok0, int c, int tid) {
#pragma unroll
        for (int i = 0; i < P::PPT; ++i) {
            // a wave's pieces lie in one tensor: uniform base, 32-bit lane offset
            const int u0 = 64 * wv + NTHR * i, ten = u0 / (C * D / 8), u = u0 % (C * D / 8) + (tid & 63);
            const bf16* base = (ten == 0 ? kb_ : ten == 1 ? vb : ten == 2 ? qb : gb) + (size_t)tok0 * D;
            const int row = min(u / (D / 8), c - 1);
            st[i] = ld_global<F>(base + (unsigned)(row * D + 8 * (u % (D / 8))));
        }
    };
    auto stage_store = [&](int c, int tid) {
#pragma unroll
        for (int i = 0; i < P::PPT; ++i) {
            const int u0 = 64 * wv + NTHR * i, ten = u0 / (C * D / 8), u = u0 % (C * D / 8) + (tid & 63);
            const int row = u / (D / 8);
            const F x = row < c ? st[i] : zero_frag<bf16>();
            bf16* d = Ks + (size_t)ten * C * LDQ + (size_t)row * LDQ + 8 * (u % (D / 8));
            st_lds<bf16x4>(d, __builtin_shufflevector(x, x, 0, 1, 2, 3));
            st_lds<bf16x4>(d + 4, __builtin_shufflevector(x, x, 4, 5, 6, 7));
        }
    };
    // first (last in time) chunk's loads go out before the tables are copied
    if (nch > 0) {
        const int tok0 = (ch0 + nch - 1) * C;
        stage_load(tok0, min(C, a.L - tok0), tid);
    }
    copy_conj_phase<MP, NTHR>(sE, LE, (const bf16*)a.Etab + (size_t)h * C * 2 * MP, tid);
    copy_table<bf16, P::ABROWS, 2 * MP, LE, NTHR>(sAB, (const bf16*)a.ABs, tid);
    for (int i = tid; i < SP; i += NTHR) sTheta[i] = slot_threshold<P::FOLD>(a.theta + (size_t)h * SP, i, a.S, SP);
    load_rho_rows<NTHR>(sRhoC, E32h, a, MP, tid);
    const bool last_row = P::FOLD && a.S == SP;  // slot S/2 in row 0 of the mirror set

    // ---- forward state after the segment (pre-rotated, [d][m] tiles): side 0 Z'_k, side 1 Z'_v
    floatx4 Z[2][NDT];
    {
        const int m = 16 * mt + r;
        const bool scanned = a.nbk >= kBwdScanBlocks;  // summary last_blk is the state
        const float* sin_ = scanned ? nullptr : side ? a.sv_in : a.sk_in;
        const float c1 = rho1[m], s1 = rho1[MP + m];
#pragma unroll
        for (int d4 = 0; d4 < NDT; ++d4) {
            floatx4 xr = zero4(), xi = zero4();
            if (sin_ && m < a.M) {
                xr = ld4f(sin_ + (((size_t)bh * 2 + 0) * a.M + m) * D + 16 * d4 + 4 * g);
                xi = ld4f(sin_ + (((size_t)bh * 2 + 1) * a.M + m) * D + 16 * d4 + 4 * g);
            }
            Z[0][d4] = c1 * xr - s1 * xi;
            Z[1][d4] = s1 * xr + c1 * xi;
        }
        for (int sg = scanned ? last_blk : 0; sg <= last_blk; ++sg) {
            const long long len = (long long)min(a.cpb * C, a.L - sg * a.cpb * C);
            const float* S = a.fsum + ((size_t)bh * a.nbk + sg) * 4 * MP * D + (size_t)2 * side * MP * D;
            float cc, ss;
            bwd_phase(m, len, rT, cc, ss);
#pragma unroll
            for (int d4 = 0; d4 < NDT; ++d4) {
                const floatx4 re = Z[0][d4], im = Z[1][d4];
                const floatx4 sr = ld4f(S + (size_t)m * D + 16 * d4 + 4 * g);
                const floatx4 si = ld4f(S + ((size_t)MP + m) * D + 16 * d4 + 4 * g);
                Z[0][d4] = cc * re - ss * im + sr;
                Z[1][d4] = ss * re + cc * im + si;
            }
        }
    }

    // ---- adjoint after the segment (pre-rotated, [m][d] tiles of head-dim tile dt, every mode
    // tile; side 0 Gam'_k, side 1 Gam'_v): Horner over the adjoint summaries of the later segments
    // from rho dLoss/d(final states)
    floatx4 Gm[2][NMT];
    // scanned: summary last_blk + 1 is the adjoint, for every segment but the last
    const bool gscan = a.nbk >= kBwdScanBlocks && last_blk + 1 < a.nbk;
    const float* gout = gscan ? nullptr : side ? a.gv_out : a.gk_out;
#pragma unroll
    for (int m4 = 0; m4 < NMT; ++m4) {
        Gm[0][m4] = Gm[1][m4] = zero4();
        if (!SUM && gout) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 16 * m4 + 4 * g + e;
                if (m < a.M) {
                    const float c1 = rho1[m], s1 = rho1[MP + m];
                    const float xr = gout[(((size_t)bh * 2 + 0) * a.M + m) * D + 16 * dt + r];
                    const float xi = gout[(((size_t)bh * 2 + 1) * a.M + m) * D + 16 * dt + r];
                    Gm[0][m4][e] = c1 * xr - s1 * xi;
                    Gm[1][m4][e] = s1 * xr + c1 * xi;
                }
            }
        }
    }
    if constexpr (!SUM) {
        for (int sg = gscan ? last_blk + 1 : a.nbk - 1; sg > last_blk; --sg) {
            const long long len = (long long)min(a.cpb * C, a.L - sg * a.cpb * C);
            const float* S = a.asum + ((size_t)bh * a.nbk + sg) * 4 * MP * D + (size_t)2 * side * MP * D;
#pragma unroll
            for (int m4 = 0; m4 < NMT; ++m4) {
                floatx4 cc, ss, sr, si;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = 16 * m4 + 4 * g + e;
                    float ce, se;
                    bwd_phase(m, len, rT, ce, se);
                    cc[e] = ce;
                    ss[e] = se;
                    sr[e] = S[(size_t)m * D + 16 * dt + r];
                    si[e] = S[((size_t)MP + m) * D + 16 * dt + r];
                }
                const floatx4 re = Gm[0][m4], im = Gm[1][m4];
                Gm[0][m4] = cc * re + ss * im + sr;
                Gm[1][m4] = cc * im - ss * re + si;
            }
        }
    }
    __syncthreads();  // tables in LDS

    const bf16* Xs = side ? Vs : Ks;      // the side's keys or values ...
    const bf16* Rs = side ? dOs : Qs;     // ... and what they meet: queries or output gradients
    bf16* Gs = side ? GdT : GT;
    bf16* Us = side ? YT : UT;
    for (int n = nch - 1; n >= 0; --n) {
        // lane indices re-derived per chunk (opaque_lane): addresses stay inside the loop
        const int r = opaque_lane(r_), g = opaque_lane(g_), tid = opaque_lane(tid_);
        const int tok0 = (ch0 + n) * C;
        const int c = min(C, a.L - tok0);
        const float* rc = rho_row(sRhoC, c, MP);  // rho^c
        __syncthreads();  // previous chunk done with the token tiles and the weights
        stage_store(c, tid);
        if (n > 0) stage_load(tok0 - C, C, tid);
        __syncthreads();  // token tiles visible

        // ---- phase 1: Z'_in = conj(rho^c) o Z'_out - sum_i conj(rho^i) x_i on the wave's mode
        // tile; Z'_k published for dq; Gram tiles of key tile w
        {
            const float cc = rc[16 * mt + r], ss = rc[MP + 16 * mt + r];
#pragma unroll
            for (int d4 = 0; d4 < NDT; ++d4) {
                const floatx4 re = Z[0][d4], im = Z[1][d4];
                Z[0][d4] = cc * re + ss * im;
                Z[1][d4] = cc * im - ss * re;
            }
        }
#pragma unroll
        for (int kb = 0; kb < KBC; ++kb) {
            F ef[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) ef[p] = neg_frag(ld_frag_tr(sE, LE, p * MP + 16 * mt, kb, g, r));
#pragma unroll
            for (int d4 = 0; d4 < NDT; ++d4) {
                const F xf = ld_frag_tr(Xs, LDQ, 16 * d4, kb, g, r);
#pragma unroll
                for (int p = 0; p < 2; ++p) Z[p][d4] = mma(xf, ef[p], Z[p][d4]);
            }
        }
        if constexpr (!SUM) {
            if (side == 0 && rm == 0) {
#pragma unroll
                for (int d4 = 0; d4 < NDT; ++d4)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int row = p * MP + 16 * mt + r;
                        st_lds<bf16x4>(ZkT + (size_t)row * P::LDZ + P::tcol(row, 16 * d4 + 4 * g), cvt4(Z[p][d4], bf16()));
                    }
            }
        }
        {
            F xf[KBD];
#pragma unroll
            for (int kb = 0; kb < KBD; ++kb) xf[kb] = ld_frag<bf16>(Xs + (size_t)(16 * w + r) * LDQ, 32 * kb, g);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                if (ct < w) continue;
                const int j = 16 * ct + r;
                floatx4 ga = zero4();
#pragma unroll
                for (int kb = 0; kb < KBD; ++kb) ga = mma(xf[kb], ld_frag<bf16>(Rs + (size_t)j * LDQ, 32 * kb, g), ga);
                if (ct == w) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (4 * g + e > r) ga[e] = 0.f;
                }
                st_lds<bf16x4>(Gs + (size_t)j * LDK + 16 * w + 4 * g, cvt4(ga, bf16()));
            }
        }
        __syncthreads();  // Gram tiles visible

        // ---- phase 2 (mode tile mt): U = E o (Q Z'_k^T + G conj(E)), side 1 Y = E o (dO Z'_v^T + Gd conj(E))
        {
            F zf[2][KBD], ef[KBC][2];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int kb = 0; kb < KBD; ++kb) zf[p][kb] = frag_from_acc<bf16>(Z[p][2 * kb], Z[p][2 * kb + 1]);
#pragma unroll
            for (int kb = 0; kb < KBC; ++kb)
#pragma unroll
                for (int p = 0; p < 2; ++p) ef[kb][p] = ld_frag_tr(sE, LE, p * MP + 16 * mt, kb, g, r);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                if (!mine(ct, rm, P::NRM)) continue;
                const int j = 16 * ct + r;
                F xf[KBD];
#pragma unroll
                for (int kb = 0; kb < KBD; ++kb) xf[kb] = ld_frag<bf16>(Rs + (size_t)j * LDQ, 32 * kb, g);
                floatx4 u[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    u[p] = zero4();
#pragma unroll
                    for (int kb = 0; kb < KBD; ++kb) u[p] = mma(zf[p][kb], xf[kb], u[p]);
                }
#pragma unroll
                for (int kb = 0; kb < KBC; ++kb) {
                    if (2 * kb <= ct) {
                        const bf16* grow = Gs + (size_t)j * LDK;
                        const F gf = 2 * kb + 1 <= ct ? ld_frag<bf16>(grow, 32 * kb, g) : ld_frag_lo<bf16>(grow, 32 * kb, g);
#pragma unroll
                        for (int p = 0; p < 2; ++p) u[p] = mma(ef[kb][p], gf, u[p]);
                    }
                }
                // E o X with the stored row [c | -s] of token j
                const floatx4 cs = to_f4(ld4_lds<bf16>(sE + (size_t)j * LE + 16 * mt + 4 * g));
                const floatx4 ns = to_f4(ld4_lds<bf16>(sE + (size_t)j * LE + MP + 16 * mt + 4 * g));
                st_lds<bf16x4>(Us + (size_t)j * LDW + P::tcol(j, 16 * mt + 4 * g), cvt4(cs * u[0] + ns * u[1], bf16()));
                st_lds<bf16x4>(Us + (size_t)j * LDW + P::tcol(j, MP + 16 * mt + 4 * g), cvt4(cs * u[1] - ns * u[0], bf16()));
            }
        }
        __syncthreads();  // U and Y visible; the Gram tiles no longer read

        // ---- phase 3 (query tile w): side 0 the scores and their softmax, side 1 dP; then side 0
        // the readout weights W'' and H_v, side 1 dz, Wq'' and H_q
        {
            const int j = 16 * w + r;
            F uf[KBM];
#pragma unroll
            for (int kb = 0; kb < KBM; ++kb) uf[kb] = P::ld_row(Us, LDW, j, kb, g);
            // products with the slot rows: scores (side 0) or scale dP (side 1); folded, the mirror
            // slots follow the slots
            floatx4 sc[NST];
            if constexpr (P::FOLD) {
                constexpr int KH = KBM / 2;
                floatx4 sp[NHT], sq[NHT];
#pragma unroll
                for (int s4 = 0; s4 < NHT; ++s4) {
                    const bf16* row = sAB + (size_t)(16 * s4 + r) * LE;
                    sp[s4] = sq[s4] = zero4();
#pragma unroll
                    for (int kb = 0; kb < KH; ++kb) {
                        sp[s4] = mma(ld_frag<bf16>(row, 32 * kb, g), uf[kb], sp[s4]);
                        sq[s4] = mma(ld_frag<bf16>(row + MP, 32 * kb, g), uf[KH + kb], sq[s4]);
                    }
                }
                if (last_row) {
#pragma unroll
                    for (int kb = 0; kb < KH; ++kb) {
                        const F f = ld_frag<bf16>(sAB + (size_t)P::HP * LE, 32 * kb, g);
                        sq[0] = mma(r == 0 ? f : zero_frag<bf16>(), uf[kb], sq[0]);
                    }
                }
                fold_scores<NHT>(sp, sq, g);
#pragma unroll
                for (int s4 = 0; s4 < NHT; ++s4) {
                    sc[s4] = sp[s4];
                    sc[NHT + s4] = sq[s4];
                }
            } else {
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) {
                    sc[s4] = zero4();
#pragma unroll
                    for (int kb = 0; kb < KBM; ++kb)
                        sc[s4] = mma(ld_frag<bf16>(sAB + (size_t)(16 * s4 + r) * LE, 32 * kb, g), uf[kb], sc[s4]);
                }
            }
            // where the slot weights of tile s4 pass from side 0 to side 1 (float32, lane order): the
            // Gram region, then this query tile's own U rows
            auto xch = [&](int s4) {
                float* base = s4 < 4 ? reinterpret_cast<float*>(GT) + (size_t)(w * (NST < 4 ? NST : 4) + s4) * 256
                                     : reinterpret_cast<float*>(UT + (size_t)16 * w * LDW) + (size_t)(s4 - 4) * 256;
                return base + 4 * (tid & 63);
            };
            if (side == 0) {
                const long long pos = a.t0 + tok0 + j;
                float mx = -INFINITY;
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) {
                    const intx4 th = *reinterpret_cast<const intx4*>(sTheta + 16 * s4 + 4 * g);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (pos < (long long)th[e]) sc[s4][e] = -INFINITY;
                        mx = fmaxf(mx, sc[s4][e]);
                    }
                }
                mx = rows_max(mx);
                float sum = 0.f;
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float ex = __expf(sc[s4][e] - mx);
                        sc[s4][e] = ex;
                        sum += ex;
                    }
                sum = rows_sum(sum);
                const float inv = __builtin_amdgcn_rcpf(sum);  // sum >= 1: the maximum slot contributes exp(0)
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) {
                    sc[s4] = sc[s4] * inv;
                    st_lds<floatx4>(xch(s4), sc[s4]);
                }
            }
            __syncthreads();  // slot weights visible; U and Y no longer read
            // side 0: P / scale (the slot matrix holds scale (A | B)); side 1: dz = P (dP - sum P dP)
            if (side == 0) {
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) sc[s4] = sc[s4] * iscale;
            } else {
                floatx4 pw[NST];
                float pd = 0.f;
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) {
                    pw[s4] = *(const __attribute__((address_space(3))) floatx4*)xch(s4);
                    sc[s4] = sc[s4] * iscale;
#pragma unroll
                    for (int e = 0; e < 4; ++e) pd += pw[s4][e] * sc[s4][e];
                }
                pd = rows_sum(pd);
#pragma unroll
                for (int s4 = 0; s4 < NST; ++s4) sc[s4] = pw[s4] * (sc[s4] - pd);
            }
            // [Re | -Im] of W'' = (P A - i P B) o rho^j, side 1 of Wq'' = scale (dz A - i dz B) o rho^j
            floatx4 wa[2 * NMT];
#pragma unroll
            for (int t = 0; t < 2 * NMT; ++t) wa[t] = zero4();
            if constexpr (P::FOLD) {
                floatx4 ep[NHT], eq[NHT];
#pragma unroll
                for (int s4 = 0; s4 < NHT; ++s4) {
                    ep[s4] = sc[s4];
                    eq[s4] = sc[NHT + s4];
                }
                fold_weights<NHT>(ep, eq, g);
                F pf[P::KBH], qf[P::KBH];
#pragma unroll
                for (int kb = 0; kb < P::KBH; ++kb) {
                    pf[kb] = frag_from_acc<bf16>(ep[2 * kb], ep[2 * kb + 1]);
                    qf[kb] = frag_from_acc<bf16>(eq[2 * kb], eq[2 * kb + 1]);
                }
#pragma unroll
                for (int t = 0; t < 2 * NMT; ++t)
#pragma unroll
                    for (int kb = 0; kb < P::KBH; ++kb)
                        wa[t] = mma(ld_frag_tr(sAB, LE, 16 * t, kb, g, r), t < NMT ? pf[kb] : qf[kb], wa[t]);
                if (last_row) {
#pragma unroll
                    for (int t = 0; t < NMT; ++t) {
                        F f = zero_frag<bf16>();
                        const bf16 x = sAB[(size_t)P::HP * LE + 16 * t + r];
                        f[0] = g == 0 ? x : (bf16)0.f;
                        wa[t] = mma(f, qf[0], wa[t]);
                    }
                }
            } else {
                F pf[P::KBS];
#pragma unroll
                for (int kb = 0; kb < P::KBS; ++kb) pf[kb] = frag_from_acc<bf16>(sc[2 * kb], sc[2 * kb + 1]);
#pragma unroll
                for (int t = 0; t < 2 * NMT; ++t)
#pragma unroll
                    for (int kb = 0; kb < P::KBS; ++kb) wa[t] = mma(ld_frag_tr(sAB, LE, 16 * t, kb, g, r), pf[kb], wa[t]);
            }
            bf16* Ws = side ? WqT : WvT;
#pragma unroll
            for (int m4 = 0; m4 < NMT; ++m4) {
                const floatx4 cs = to_f4(ld4_lds<bf16>(sE + (size_t)j * LE + 16 * m4 + 4 * g));
                const floatx4 ns = to_f4(ld4_lds<bf16>(sE + (size_t)j * LE + MP + 16 * m4 + 4 * g));
                const floatx4 am = wa[m4], bm = wa[NMT + m4];
                wa[m4] = am * cs - bm * ns;
                wa[NMT + m4] = am * ns + bm * cs;
                st_lds<bf16x4>(Ws + (size_t)j * LDW + P::tcol(j, 16 * m4 + 4 * g), cvt4(wa[m4], bf16()));
                st_lds<bf16x4>(Ws + (size_t)j * LDW + P::tcol(j, MP + 16 * m4 + 4 * g), cvt4(wa[NMT + m4], bf16()));
            }
            if constexpr (!SUM) {
                F wf[KBM];
#pragma unroll
                for (int kb = 0; kb < KBM; ++kb) wf[kb] = frag_from_acc<bf16>(wa[2 * kb], wa[2 * kb + 1]);
                __syncthreads();  // the slot weights in the Gram region are read: it takes the H tiles
                bf16* Hs = side ? HqT : HvT;
#pragma unroll
                for (int kt = 0; kt < NT; ++kt) {
                    floatx4 hh = zero4();
                    if (kt <= w) {
#pragma unroll
                        for (int kb = 0; kb < KBM; ++kb)
                            hh = mma(ld_frag<bf16>(sE + (size_t)(16 * kt + r) * LE, 32 * kb, g), wf[kb], hh);
                        if (kt == w) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (4 * g + e > r) hh[e] = 0.f;
                        }
                    }
                    st_lds<bf16x4>(Hs + (size_t)j * P::LDH + P::tcol(j, 16 * kt + 4 * g), cvt4(hh, bf16()));
                }
            }
        }
        __syncthreads();  // H tiles and weights visible

        // ---- phase 4 (head-dim tile dt): Gam'' = conj(rho^c) o Gam'; dk (side 1: dv) of every key;
        // Gam' <- Gam'' + conj(Wq'')^T Q (side 1: conj(W'')^T dO); then a share of dq
        const bf16* Ws = side ? WvT : WqT;
#pragma unroll
        for (int m4 = 0; m4 < NMT; ++m4) {
            const floatx4 cc = ld4f(rc + 16 * m4 + 4 * g), ss = ld4f(rc + MP + 16 * m4 + 4 * g);
            const floatx4 re = Gm[0][m4], im = Gm[1][m4];
            Gm[0][m4] = cc * re + ss * im;
            Gm[1][m4] = cc * im - ss * re;
        }
        F xtf[KBC];
#pragma unroll
        for (int kb = 0; kb < KBC; ++kb) xtf[kb] = ld_frag_tr(Rs, LDQ, 16 * dt, kb, g, r);
        if constexpr (!SUM) {
            const bf16* Hs = side ? HvT : HqT;
            bf16* out = (bf16*)(side ? a.dv : a.dk) + ((size_t)bh * a.L + tok0) * D;
            // A operand [Re Gam'' | Im Gam''] (rows d, reduction over the 2MP rows)
            F gf[KBM];
#pragma unroll
            for (int kb = 0; kb < KBM; ++kb) {
                // the block's two 16-row tiles in the order [Re tiles | Im tiles]
                const int t0 = 2 * kb, t1 = 2 * kb + 1;
                gf[kb] = frag_from_acc<bf16>(Gm[t0 / NMT][t0 % NMT], Gm[t1 / NMT][t1 % NMT]);
            }
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) {
                if (!mine(kt, rd, P::NRD)) continue;
                const int j = 16 * kt + r;
                floatx4 xa = zero4();
#pragma unroll
                for (int kb = 0; kb < KBC; ++kb)
                    if (2 * kb + 1 >= kt) xa = mma(xtf[kb], P::ld_t(Hs, P::LDH, 16 * kt, kb, g, r), xa);
#pragma unroll
                for (int kb = 0; kb < KBM; ++kb) xa = mma(gf[kb], ld_frag<bf16>(sE + (size_t)j * LE, 32 * kb, g), xa);
                if (j < c) st4<bf16>(out + (unsigned)(j * D + 16 * dt + 4 * g), xa);
            }
        }
#pragma unroll
        for (int kb = 0; kb < KBC; ++kb)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int m4 = 0; m4 < NMT; ++m4)
                    Gm[p][m4] = mma(P::ld_t(Ws, LDW, p * MP + 16 * m4, kb, g, r), xtf[kb], Gm[p][m4]);
        if constexpr (!SUM) {
            // dq of head-dim tile dt: Re(Wq'' Z'_k) + H_q K, the query tiles split over the sides
            // (and over the waves that share the tile)
            F zf[KBM], ktf[KBC];
#pragma unroll
            for (int kb = 0; kb < KBM; ++kb) zf[kb] = P::ld_t(ZkT, P::LDZ, 16 * dt, kb, g, r);
#pragma unroll
            for (int kb = 0; kb < KBC; ++kb) ktf[kb] = ld_frag_tr(Ks, LDQ, 16 * dt, kb, g, r);
            bf16* dqb = (bf16*)a.dq + ((size_t)bh * a.L + tok0) * D;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                if (!mine(tt, P::NRD == 1 ? side : 2 * side + rd, 2 * P::NRD)) continue;
                const int j = 16 * tt + r;
                floatx4 oa = zero4();
#pragma unroll
                for (int kb = 0; kb < KBM; ++kb) oa = mma(zf[kb], P::ld_row(WqT, LDW, j, kb, g), oa);
#pragma unroll
                for (int kb = 0; kb < KBC; ++kb)
                    if (2 * kb <= tt) oa = mma(ktf[kb], P::ld_row(HqT, P::LDH, j, kb, g), oa);
                if (j < c) st4<bf16>(dqb + (unsigned)(j * D + 16 * dt + 4 * g), oa);
            }
        }
    }

    // ---- the adjoint at the segment's start
    if (rd != 0) return;
    if constexpr (SUM) {
        float* S = a.asum + ((size_t)bh * a.nbk + seg) * 4 * MP * D + (size_t)2 * side * MP * D;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int m4 = 0; m4 < NMT; ++m4)
#pragma unroll
                for (int e = 0; e < 4; ++e) S[((size_t)p * MP + 16 * m4 + 4 * g + e) * D + 16 * dt + r] = Gm[p][m4][e];
    } else {
        float* gin = side ? a.gv_in : a.gk_in;
        if (seg != 0 || !gin) return;
#pragma unroll
        for (int m4 = 0; m4 < NMT; ++m4)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 16 * m4 + 4 * g + e;
                if (m >= a.M) continue;
                const float c1 = rho1[m], s1 = rho1[MP + m], re = Gm[0][m4][e], im = Gm[1][m4][e];
                gin[(((size_t)bh * 2 + 0) * a.M + m) * D + 16 * dt + r] = c1 * re + s1 * im;
                gin[(((size_t)bh * 2 + 1) * a.M + m) * D + 16 * dt + r] = c1 * im - s1 * re;
            }
    }
}

template <int D, int MP, int SP>
hipError_t launch_backward16_shape(const BwdArgs& a, hipStream_t s, void* const* ev)
{
    auto mark = [&](int i) -> hipError_t {
        return (ev && ev[i]) ? hipEventRecord((hipEvent_t)ev[i], s) : hipSuccess;
    };
    const unsigned units = (unsigned)(a.B * a.H);
    hipLaunchKernelGGL((bwd16_fsum_kernel<D, MP>), dim3(2 * units * a.nbk), dim3(kThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    const dim3 sgrid((unsigned)(((size_t)units * 2 * MP * D / 4 + kThreads - 1) / kThreads));
    const bool scan = a.nbk >= kBwdScanBlocks;
    if (e == hipSuccess && scan) {
        hipLaunchKernelGGL((bwd16_scan_kernel<D, MP, false>), sgrid, dim3(kThreads), 0, s, a);
        e = hipGetLastError();
    }
    if (e != hipSuccess || (e = mark(0)) != hipSuccess) return e;
    if (a.nseg > 1) {
        const unsigned sum_blocks = (unsigned)(a.nbk - a.nbk / a.nseg);  // blocks of segments 1..nseg-1
        hipLaunchKernelGGL((bwd16_kernel<D, MP, SP, true>), dim3(units * sum_blocks), dim3(Bwd16<D, MP, SP>::NTHR), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (scan) {
            hipLaunchKernelGGL((bwd16_scan_kernel<D, MP, true>), sgrid, dim3(kThreads), 0, s, a);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    if ((e = mark(1)) != hipSuccess) return e;
    hipLaunchKernelGGL((bwd16_kernel<D, MP, SP, false>), dim3(units * a.nseg), dim3(Bwd16<D, MP, SP>::NTHR), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return mark(2);
}

}  // namespace bla
