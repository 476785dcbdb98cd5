// Weight gradients of the heads (chain rule through Section 2.2 with I held
// fixed), each a sum over every selected row r = (b, i) in a fixed order:
//   dW^Q_h = sum_r X[b, I_r]^T dQ_r   (likewise W^K, W^V)    [d x dh]
//   dW^r_h = sum_r dz_r X[b, I_r]                             [d]
//   dW^O_h = sum_r (r_r A_r)^T dY[b, I_r]                     [dh x d]
//            (the forward saved the rows r_r A_r already scaled)
// Dense heads: the same with I = identity and r = 1 (no W^r).
//
// bf16 storage: the gathered-row engine of gemm2.h, see WgradQkvPolicy2 below.
// On the tiled MFMA engine of gemm.h (fp32, and bf16 past that one's reach) the
// contraction index K is the row r, which is
// contiguous in neither operand: both are staged with the engine's 8x8
// register transpose.  wgrad_qkv: M = d, N = 3 dh (+ a 16-column block whose
// first column is dz, so dW^r falls out of the same MFMAs), one workgroup per
// (head, 64 rows of d).  wgrad_o: M = dh, N = d.  The K loop runs over the rows
// in order, so the sums are bitwise reproducible.  When there are too few
// (head, tile) pairs to fill the chip the rows are split into S contiguous
// ranges: each workgroup writes an fp32 partial tile and a second kernel adds
// the S partials in range order (still reproducible).
#include <algorithm>

#include "dxrow.h"
#include "gemm.h"
#include "gemm2.h"
#include "group.h"
#include "kernels.h"

namespace mosa {

namespace {

// SMALL (fp32): one of dW^Q, dW^K, dW^V (or the router column) per workgroup.
template <typename ST, int DH, bool ROUTER, bool GATHER, bool SMALL = false>
struct WgradQkvPolicy {
    static constexpr int NALL = 3 * DH + (ROUTER ? 16 : 0);  // columns of a partial row
    static constexpr int MT = 64, NT = SMALL ? DH : NALL, KC = sizeof(ST) == 2 ? 64 : 32, WM = SMALL ? 2 : 4, WN = 4 / WM;
    static constexpr int NTILES = (NALL + NT - 1) / NT;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = false, B_KCONTIG = false, SPLITK = true;
    struct Args {
        const ST* X;
        const int32_t* I;
        const ST* dQKV;  // [B, H, n, 3*DH]
        const ST* dz16;  // [B, H, n, 16] (the engine of gemm.h)
        ST* dWq;
        ST* dWk;
        ST* dWv;         // [H, d, DH]
        ST* dWr;         // [H, d]
        float* part;     // [S, H, d, NT] fp32 partial sums (S > 1)
        int T, d, H, n, R, mtiles, S, cps;
        FastDiv nd;
        const float* dz; // [B, H, n] (the gathered-row engine)
    };
    struct ARef {};
    struct BRef {};
    // Row r = (b, i) of head h.  The token index t is kept as loaded (the
    // address arithmetic happens in a_kaddr), so the gather load is waited
    // for only when the row infos are stored to LDS, after the chunk's MFMAs.
    struct RowInfo {
        int b;   // batch element, or -1 past the last row
        int t;   // token I_r (gathered) or i (dense)
        int ri;  // selected-row index (b*H + h)*n + i
    };
    __device__ static const ST* a_fallback(const Args& a) { return a.X; }
    __device__ static const ST* b_fallback(const Args& a) { return a.dQKV; }
    __device__ static void tile_split(const Args& a, int logical, int& h, int& m0, int& n0, int& split) {
        const int per = a.H * a.mtiles * NTILES;
        split = logical / per;
        const int rem = logical % per, mn = rem % (a.mtiles * NTILES);
        h = rem / (a.mtiles * NTILES);
        m0 = (mn / NTILES) * MT;
        n0 = (mn % NTILES) * NT;
    }
    __device__ static void k_range(const Args& a, int split, int K, int& kbeg, int& kend) {
        kbeg = split * a.cps * KC;
        kend = min(K, kbeg + a.cps * KC);
    }
    __device__ static int k_size(const Args& a, int) { return a.R; }
    __device__ static ARef a_row(const Args&, int, int) { return {}; }
    __device__ static const ST* a_elem(const Args&, int, const ARef&, int) { return nullptr; }
    __device__ static BRef b_row(const Args&, int, int) { return {}; }
    __device__ static const ST* b_elem(const Args&, int, const BRef&, int) { return nullptr; }
    __device__ static RowInfo row_info(const Args& a, int h, int r) {
        int b, i;
        fast_divmod(a.nd, r < 0 ? 0 : r, b, i);
        const int ri = (b * a.H + h) * a.n + i;
        return {r < 0 ? -1 : b, GATHER ? a.I[ri] : i, ri};
    }
    // A[c][r] = X[b, I_r, c]: row r of the gathered input, c contiguous
    __device__ static const ST* a_kaddr(const Args& a, int, const RowInfo& r, int m8) {
        return a.X + ((size_t)max(r.b, 0) * a.T + r.t) * a.d + min(m8, a.d - 8);
    }
    __device__ static bool a_kok(const Args& a, int, const RowInfo& r, int m8) { return r.b >= 0 && m8 < a.d; }
    // B[r][n] = dQ | dK | dV | (dz, 0...) of row r
    __device__ static const ST* b_kaddr(const Args& a, int, const RowInfo& r, int n8) {
        return n8 < 3 * DH ? a.dQKV + (size_t)r.ri * (3 * DH) + n8
                           : a.dz16 + (size_t)r.ri * 16 + min(n8 - 3 * DH, 8);
    }
    __device__ static bool b_kok(const Args&, int, const RowInfo& r, int n8) { return r.b >= 0 && n8 < NALL; }
    __device__ static void epilogue(const Args& a, int h, int m0, int n0, const float* Cs, int ldc, int tid,
                                    unsigned char*) {
        constexpr int VPR = NT / 8;
        for (int v = tid; v < MT * VPR; v += 256) {
            const int ml = v / VPR, nl = (v % VPR) * 8, nn = n0 + nl;
            const int c = m0 + ml;
            if (c >= a.d || nn >= 3 * DH) continue;
            float x[8];
            cs_load8(Cs, ldc, ml, nl, x);
            ST* W = nn < DH ? a.dWq : (nn < 2 * DH ? a.dWk : a.dWv);
            vec8_store<ST>(W + ((size_t)h * a.d + c) * DH + (nn % DH), vec8_from_f32<ST>(x));
        }
        if (ROUTER && n0 + NT > 3 * DH && tid < MT && m0 + tid < a.d)
            st1<ST>(a.dWr + (size_t)h * a.d + m0 + tid, Cs[tid * ldc + 3 * DH - n0]);
    }
    __device__ static void epilogue_split(const Args& a, int h, int split, int m0, int n0, const float* Cs, int ldc,
                                          int tid) {
        if (a.S == 1) {
            epilogue(a, h, m0, n0, Cs, ldc, tid, nullptr);
            return;
        }
        constexpr int VPR = NT / 4;  // float4 per row
        for (int v = tid; v < MT * VPR; v += 256) {
            const int ml = v / VPR, nl = (v % VPR) * 4, nn = n0 + nl;
            const int c = m0 + ml;
            if (c >= a.d || nn >= NALL) continue;
            const float4 x = *reinterpret_cast<const float4*>(Cs + ml * ldc + nl);
            *reinterpret_cast<float4*>(a.part + (((size_t)split * a.H + h) * a.d + c) * NALL + nn) = x;
        }
    }
};

// Sum of the S partial tiles in split order, then the final stores.
template <typename ST, int DH, bool ROUTER>
__global__ __launch_bounds__(256) void wgrad_qkv_reduce_kernel(const float* __restrict__ part, int S, int H, int d,
                                                               ST* dWq, ST* dWk, ST* dWv, ST* dWr) {
    constexpr int NT = 3 * DH + (ROUTER ? 16 : 0);
    constexpr int G = 3 * DH / 8 + (ROUTER ? 1 : 0);  // 8-column groups written
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= H * d * G) return;
    const int gq = idx % G, hc = idx / G;  // hc = h * d + c
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < S; ++sp) {
        const float* p = part + ((size_t)sp * H * d + hc) * NT + gq * 8;
        const float4 u = reinterpret_cast<const float4*>(p)[0], w = reinterpret_cast<const float4*>(p)[1];
        x[0] += u.x; x[1] += u.y; x[2] += u.z; x[3] += u.w;
        x[4] += w.x; x[5] += w.y; x[6] += w.z; x[7] += w.w;
    }
    const int nn = gq * 8;
    if (nn < 3 * DH) {
        ST* W = nn < DH ? dWq : (nn < 2 * DH ? dWk : dWv);
        vec8_store<ST>(W + (size_t)hc * DH + (nn % DH), vec8_from_f32<ST>(x));
    } else {
        st1<ST>(dWr + hc, x[0]);
    }
}

template <typename ST, int DH, bool GATHER, bool SMALL = false>
struct WgradOPolicy {
    static constexpr int MT = DH, NT = SMALL ? 64 : 128, KC = sizeof(ST) == 2 ? 64 : 32, WM = 2, WN = 2;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = false, B_KCONTIG = false, SPLITK = true;
    struct Args {
        const ST* dY;
        const int32_t* I;
        const ST* A;      // [B, H, n, DH], rows scaled by r
        ST* dWo;          // [H, DH, d]
        float* part;      // [S, H, DH, d] fp32 partial sums (S > 1)
        int T, d, H, n, R, ntiles, S, cps;
        FastDiv nd;
    };
    struct ARef {};
    struct BRef {};
    struct RowInfo {
        int b;   // batch element, or -1 past the last row
        int t;   // token I_r (gathered) or i (dense), as loaded
        int ri;  // selected-row index
    };
    __device__ static const ST* a_fallback(const Args& a) { return a.A; }
    __device__ static const ST* b_fallback(const Args& a) { return a.dY; }
    __device__ static void tile_split(const Args& a, int logical, int& h, int& m0, int& n0, int& split) {
        const int per = a.H * a.ntiles;
        split = logical / per;
        const int rem = logical % per;
        h = rem / a.ntiles;
        m0 = 0;
        n0 = (rem % a.ntiles) * NT;
    }
    __device__ static void k_range(const Args& a, int split, int K, int& kbeg, int& kend) {
        kbeg = split * a.cps * KC;
        kend = min(K, kbeg + a.cps * KC);
    }
    __device__ static int k_size(const Args& a, int) { return a.R; }
    __device__ static ARef a_row(const Args&, int, int) { return {}; }
    __device__ static const ST* a_elem(const Args&, int, const ARef&, int) { return nullptr; }
    __device__ static BRef b_row(const Args&, int, int) { return {}; }
    __device__ static const ST* b_elem(const Args&, int, const BRef&, int) { return nullptr; }
    __device__ static RowInfo row_info(const Args& a, int h, int r) {
        int b, i;
        fast_divmod(a.nd, r < 0 ? 0 : r, b, i);
        const int ri = (b * a.H + h) * a.n + i;
        return {r < 0 ? -1 : b, GATHER ? a.I[ri] : i, ri};
    }
    // A[e][r] = (r_r A_r)[e]
    __device__ static const ST* a_kaddr(const Args& a, int, const RowInfo& r, int m8) {
        return a.A + (size_t)r.ri * DH + m8;
    }
    __device__ static bool a_kok(const Args&, int, const RowInfo& r, int) { return r.b >= 0; }
    // B[r][c] = dY[b, I_r, c]
    __device__ static const ST* b_kaddr(const Args& a, int, const RowInfo& r, int n8) {
        return a.dY + ((size_t)max(r.b, 0) * a.T + r.t) * a.d + min(n8, a.d - 8);
    }
    __device__ static bool b_kok(const Args& a, int, const RowInfo& r, int n8) { return r.b >= 0 && n8 < a.d; }
    __device__ static void epilogue(const Args& a, int h, int, int n0, const float* Cs, int ldc, int tid, unsigned char*) {
        constexpr int VPR = NT / 8;
        for (int v = tid; v < MT * VPR; v += 256) {
            const int e = v / VPR, c = (v % VPR) * 8;
            if (n0 + c >= a.d) continue;
            float x[8];
            cs_load8(Cs, ldc, e, c, x);
            vec8_store<ST>(a.dWo + ((size_t)h * DH + e) * a.d + n0 + c, vec8_from_f32<ST>(x));
        }
    }
    __device__ static void epilogue_split(const Args& a, int h, int split, int m0, int n0, const float* Cs, int ldc,
                                          int tid) {
        if (a.S == 1) {
            epilogue(a, h, m0, n0, Cs, ldc, tid, nullptr);
            return;
        }
        constexpr int VPR = NT / 4;
        for (int v = tid; v < MT * VPR; v += 256) {
            const int e = v / VPR, c = (v % VPR) * 4;
            if (n0 + c >= a.d) continue;
            const float4 x = *reinterpret_cast<const float4*>(Cs + e * ldc + c);
            *reinterpret_cast<float4*>(a.part + (((size_t)split * a.H + h) * DH + e) * a.d + n0 + c) = x;
        }
    }
};

template <typename ST>
__global__ __launch_bounds__(256) void wgrad_o_reduce_kernel(const float* __restrict__ part, int S, size_t n8,
                                                             ST* dWo) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n8) return;
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < S; ++sp) {
        const float* p = part + ((size_t)sp * n8 + idx) * 8;
        const float4 u = reinterpret_cast<const float4*>(p)[0], w = reinterpret_cast<const float4*>(p)[1];
        x[0] += u.x; x[1] += u.y; x[2] += u.z; x[3] += u.w;
        x[4] += w.x; x[5] += w.y; x[6] += w.z; x[7] += w.w;
    }
    vec8_store<ST>(dWo + idx * 8, vec8_from_f32<ST>(x));
}

// bf16 storage, MoSA heads: the multi-stage engine (gemm2.h) with the rows
// gathered through an LDS table, k = r in order over the whole range (no
// split: one workgroup owns its output tile, so the sums are reproducible
// without partials).  Row r = (b, i): the table holds the offsets, in 16-byte
// units, of token row b T + I_r (of X or dY) and of the selected row (b H + h) n
// + i (of dQ | dK | dV or of the scaled attention rows).  The MFMA's A operand is
// the one whose output index is contiguous in memory, interleaved so the
// accumulators go straight to 16-byte stores.
template <class Args>
__device__ __forceinline__ uint2 wgrad_k_row(const Args& a, int h, int k, int sel16) {
    int b, i;
    fast_divmod(a.nd, k, b, i);
    const int ri = (b * a.H + h) * a.n + i;
    return make_uint2((uint32_t)(b * a.T + a.I[ri]) * (uint32_t)(a.d / 8), (uint32_t)ri * (uint32_t)sel16);
}

// Several tiles of d per workgroup, in one pipeline (Args: S workgroups per
// head, cps tiles each), where a tile has few chunks and that still leaves two
// workgroups per CU: with 256 rows per head (8 chunks) a workgroup per tile
// spent as long on its row table (a gather of I) and its first loads as on
// the rest (128 heads, 256 rows, d 1024: 200.9 -> 193.8 us per training step).
inline int wgrad_tiles_per_wg(int H, int tiles, int rows) {
    return std::max(1, std::min({tiles, H * tiles / 512, 1024 / rows}));
}

// dW^{Q,K,V}_h and dW^r_h: M = the 3 dh columns [dQ | dK | dV], N = NT rows of d
// per tile, dW^r as a row product beside the MFMAs (ROW, dz in fp32).  The
// loop is bound by instruction issue and LDS as much as by its MFMAs: offsets
// in the row table instead of row numbers (a multiplication and a select per
// load less) and no 64-column block for the one column dz took the grouped
// launch of 128 heads, 256 rows, d 1024 from 78.8 to 69.6 us, and the dense
// heads' (4 heads, 8192 rows) from 31.5 to 25.0.  128 rows per tile halve the
// LDS reads and the bytes moved into LDS per product: 69.6 -> 67.8 us, with 512
// rows and 64 heads 63.4 -> 59.8.
template <int DH, int NT_>
struct WgradQkvPolicy2 {
    using ST = uint16_t;
    static constexpr int MT = 3 * DH, NT = NT_, KC = DH == 64 ? 32 : 64, WM = DH == 64 ? 2 : 1, WN = 4 / WM, STAGES = 3;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = false, B_KCONTIG = false, KGATHER = true, A_INTERLEAVE = true, EPI_REGS = true;
    static constexpr int A_TAB = 1, B_TAB = 0, MIN_WAVES = 2;
    static constexpr bool MULTI = true, MULTI_A = false, ROW = true;
    static constexpr int STORES = 3 * (NT / WN / 16);  // 3 pairs of row blocks, each column block
    using Args = typename WgradQkvPolicy<ST, DH, true, true>::Args;
    __device__ static void tile(const Args& a, int logical, int& h, int& m0, int& n0) {
        h = logical / a.S;
        m0 = 0;
        n0 = (logical % a.S) * a.cps * NT;
    }
    __device__ static int tiles(const Args& a, int logical) { return min(a.cps, a.mtiles - (logical % a.S) * a.cps); }
    __device__ static int k_size(const Args& a, int) { return a.R; }
    __device__ static uint2 k_row(const Args& a, int h, int k) { return wgrad_k_row(a, h, k, 3 * DH / 8); }
    __device__ static float k_f(const Args& a, int h, int k, int K) {
        int b, i;
        fast_divmod(a.nd, min(k, K - 1), b, i);
        const float v = a.dz[(size_t)(b * a.H + h) * a.n + i];
        return k < K ? v : 0.f;
    }
    __device__ static const ST* a_mlane(const Args& a, int, int m8) { return a.dQKV + m8; }
    __device__ static const ST* b_mlane(const Args& a, int, int n8) { return a.X + n8; }
    // columns m .. m + 7 of row c = n
    __device__ static void store8(const Args& a, int h, int m, int n, const float (&x)[8]) {
        ST* W = m < DH ? a.dWq : (m < 2 * DH ? a.dWk : a.dWv);
        vec8_store<ST>(W + ((size_t)h * a.d + n) * DH + (m % DH), vec8_from_f32<ST>(x));
    }
    __device__ static void store_row(const Args& a, int h, int n, float v) { st1<ST>(a.dWr + (size_t)h * a.d + n, v); }
};

// dW^O_h: M = MT columns c of d per tile (dY rows), N = dh (the scaled
// attention rows).
template <int DH, int MT_>
struct WgradOPolicy2 {
    using ST = uint16_t;
    static constexpr int MT = MT_, NT = DH, KC = 64, WM = 2, WN = 2, STAGES = MT > 64 ? 3 : 4;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = false, B_KCONTIG = false, KGATHER = true, A_INTERLEAVE = true, EPI_REGS = true;
    static constexpr int A_TAB = 0, B_TAB = 1;
    static constexpr bool MULTI = true, MULTI_A = true;
    static constexpr int STORES = (MT / 64) * (DH / 32);  // pairs of row blocks, column blocks
    using Args = typename WgradOPolicy<ST, DH, true>::Args;
    __device__ static void tile(const Args& a, int logical, int& h, int& m0, int& n0) {
        h = logical / a.S;
        m0 = (logical % a.S) * a.cps * MT;
        n0 = 0;
    }
    __device__ static int tiles(const Args& a, int logical) { return min(a.cps, a.ntiles - (logical % a.S) * a.cps); }
    __device__ static int k_size(const Args& a, int) { return a.R; }
    __device__ static uint2 k_row(const Args& a, int h, int k) { return wgrad_k_row(a, h, k, DH / 8); }
    __device__ static const ST* a_mlane(const Args& a, int, int m8) { return a.dY + m8; }
    __device__ static const ST* b_mlane(const Args& a, int, int n8) { return a.A + n8; }
    // columns c = m .. m + 7 of row e = n
    __device__ static void store8(const Args& a, int h, int m, int n, const float (&x)[8]) {
        vec8_store<ST>(a.dWo + ((size_t)h * DH + n) * a.d + m, vec8_from_f32<ST>(x));
    }
};

// Dense heads (bf16) on the same engine: R = B T rows split into S ranges of
// up to 4096 rows (the row table), one fp32 partial tile per range, summed in
// range order by the reduce kernels.  "batch" = h S + s.  Row r of range s:
// row r' = s KS + r of X or dY and row (b Hd + h) T + t of the head.
template <class Args>
__device__ __forceinline__ uint2 wgrad_dense_k_row(const Args& a, int batch, int k, int sel16) {
    const int r = min((batch % a.S) * a.cps + k, a.R - 1);
    int b, t;
    fast_divmod(a.nd, r, b, t);
    return make_uint2((uint32_t)r * (uint32_t)(a.d / 8),
                      (uint32_t)((b * a.H + batch / a.S) * a.T + t) * (uint32_t)sel16);
}

template <int DH>
struct WgradQkvDensePolicy2 : WgradQkvPolicy2<DH, 64> {
    using ST = uint16_t;
    using Base = WgradQkvPolicy2<DH, 64>;
    static constexpr bool MULTI = false, ROW = false;
    using Args = typename Base::Args;  // I unused, cps = rows per range
    __device__ static void tile(const Args& a, int logical, int& batch, int& m0, int& n0) {
        // the heads of one (row range, column tile) side by side (its X block)
        const int h = logical % a.H, rest = logical / a.H;
        batch = h * a.S + rest / a.mtiles;  // h S + s
        m0 = 0;
        n0 = (rest % a.mtiles) * Base::NT;
    }
    __device__ static int k_size(const Args& a, int batch) { return min(a.cps, a.R - (batch % a.S) * a.cps); }
    __device__ static uint2 k_row(const Args& a, int batch, int k) { return wgrad_dense_k_row(a, batch, k, 3 * DH / 8); }
    // fp32 partial: part[s][h][c][3 DH], columns m .. m + 7 of row c = n
    __device__ static void store8(const Args& a, int batch, int m, int n, const float (&x)[8]) {
        const int h = batch / a.S, s = batch % a.S;
        float* p = a.part + (((size_t)s * a.H + h) * a.d + n) * (3 * DH) + m;
        reinterpret_cast<float4*>(p)[0] = make_float4(x[0], x[1], x[2], x[3]);
        reinterpret_cast<float4*>(p)[1] = make_float4(x[4], x[5], x[6], x[7]);
    }
};

template <int DH>
struct WgradODensePolicy2 : WgradOPolicy2<DH, 64> {
    using ST = uint16_t;
    using Base = WgradOPolicy2<DH, 64>;
    static constexpr bool MULTI = false;
    using Args = typename Base::Args;  // I unused, cps = rows per range
    __device__ static void tile(const Args& a, int logical, int& batch, int& m0, int& n0) {
        // the heads of one (row range, column tile) side by side (its dY block)
        const int h = logical % a.H, rest = logical / a.H;
        batch = h * a.S + rest / a.ntiles;  // h S + s
        m0 = (rest % a.ntiles) * Base::MT;
        n0 = 0;
    }
    __device__ static int k_size(const Args& a, int batch) { return min(a.cps, a.R - (batch % a.S) * a.cps); }
    __device__ static uint2 k_row(const Args& a, int batch, int k) { return wgrad_dense_k_row(a, batch, k, DH / 8); }
    // fp32 partial: part[s][h][e][c], columns c = m .. m + 7 of row e = n
    __device__ static void store8(const Args& a, int batch, int m, int n, const float (&x)[8]) {
        const int h = batch / a.S, s = batch % a.S;
        float* p = a.part + (((size_t)s * a.H + h) * DH + n) * a.d + m;
        reinterpret_cast<float4*>(p)[0] = make_float4(x[0], x[1], x[2], x[3]);
        reinterpret_cast<float4*>(p)[1] = make_float4(x[4], x[5], x[6], x[7]);
    }
};

// Row ranges of the dense-head split: about one workgroup per CU (256 for
// `tiles` output tiles per range), each range at most 4096 rows.  Fewer
// ranges mean fewer fp32 partials to write and sum; with 4 dense heads,
// d = 1024 and B T = 8192 rows, 4 ranges beat 2 and 8 (the hybrid layer's
// step: 0.428, 0.406 and 0.410 ms cold), 16 were slower still.
inline int dense_ranges(int R, int tiles, int kc, int& rows) {
    int S = std::max(1, (256 + tiles - 1) / tiles);
    S = std::max(S, (R + 4095) / 4096);
    rows = (R + S - 1) / S;
    rows = (rows + kc - 1) / kc * kc;
    if (rows > 4096) return 0;
    return (R + rows - 1) / rows;
}

// Rows of the k-row table for a gathered range of R rows (0: not usable: the
// table is too long, or a tensor of `tokens` rows of d or `sel` rows of 3 dh
// elements passes the 64 GB that the table's 32-bit offsets of 16-byte units
// reach).
template <class P2>
int wgrad2_table_rows(int R, int d, long long tokens, long long sel, int dh) {
    const int rows = (R + P2::KC - 1) / P2::KC * P2::KC;
    if (R <= 0 || rows > 4096 || d % 64 != 0) return 0;
    if (tokens * d >= 1ll << 35 || sel * 3 * dh >= 1ll << 35) return 0;
    return rows;
}

// Split of the row range: enough workgroups to fill the chip (about 512),
// at least 4 chunks per split.
int choose_splits(int base_tiles, int nchunks, int& cps) {
    int sp = (512 + base_tiles - 1) / base_tiles;
    sp = std::min(sp, std::max(1, nchunks / 4));
    sp = std::max(1, std::min(sp, 64));
    cps = (nchunks + sp - 1) / sp;
    return nchunks > 0 ? (nchunks + cps - 1) / cps : 1;
}

// Splits of a launch of `tiles` output tiles over `rows` rows; small: whether
// the smaller tiles are taken (fp32, when the larger ones with their splits
// leave CUs idle).
struct WgradPlan {
    int S, cps;
    bool small;
};
template <class P, class PS>
WgradPlan wgrad_plan(int tiles, int small_tiles, int rows, bool allow_small) {
    WgradPlan w{1, 0, false};
    const int nchunks = (rows + P::KC - 1) / P::KC;
    w.S = choose_splits(tiles, nchunks, w.cps);
    if (allow_small && w.S * tiles < kFullChip) {
        w.small = true;
        static_assert(P::KC == PS::KC, "same chunks");
        w.S = choose_splits(small_tiles, nchunks, w.cps);
    }
    return w;
}
template <typename ST, int DH, bool ROUTER, bool GATHER>
WgradPlan plan_qkv(int d, int H, int R) {
    using P = WgradQkvPolicy<ST, DH, ROUTER, GATHER>;
    using PS = WgradQkvPolicy<ST, DH, ROUTER, GATHER, true>;
    const int mt = (d + P::MT - 1) / P::MT;
    return wgrad_plan<P, PS>(H * mt, H * mt * PS::NTILES, R, sizeof(ST) == 4);
}
template <typename ST, int DH, bool GATHER>
WgradPlan plan_o(int d, int H, int R) {
    using P = WgradOPolicy<ST, DH, GATHER>;
    using PS = WgradOPolicy<ST, DH, GATHER, true>;
    return wgrad_plan<P, PS>(H * ((d + P::NT - 1) / P::NT), H * ((d + PS::NT - 1) / PS::NT), R, sizeof(ST) == 4);
}

// Stage names of the weight-gradient kernels (MoSA heads / dense heads).
inline const char* wname(bool dense, int which, bool reduce) {
    static const char* const names[2][2][2] = {
        {{"wgrad_qkv", "wgrad_qkv_reduce"}, {"wgrad_o", "wgrad_o_reduce"}},
        {{"wgrad_qkv_dense", "wgrad_qkv_dense_reduce"}, {"wgrad_o_dense", "wgrad_o_dense_reduce"}}};
    return names[dense][which][reduce];
}

template <typename ST, int DH, bool ROUTER, bool GATHER>
int run_qkv_t(const ST* X, const int32_t* I, const ST* dQKV, const ST* dz16, const float* dz, int B, int T, int d, int H, int n,
              ST* dWq, ST* dWk, ST* dWv, ST* dWr, float* part, const Marker& mk, hipStream_t stream) {
    using P = WgradQkvPolicy<ST, DH, ROUTER, GATHER>;
    const bool dense = !GATHER;
    const int mtiles = (d + P::MT - 1) / P::MT, R = B * n;
    if constexpr (sizeof(ST) == 2 && ROUTER && GATHER) {
        using P2 = WgradQkvPolicy2<DH, 64>;
        if (const int rows = wgrad2_table_rows<P2>(R, d, (long long)B * T, (long long)R * H, DH)) {
            const int tl = d / 64, per = wgrad_tiles_per_wg(H, tl, R), wgs = (tl + per - 1) / per;
            typename P::Args a{X, I, dQKV, dz16, dWq, dWk, dWv, dWr, part, T, d, H, n, R, tl, wgs, per, make_fastdiv(n), dz};
            return launch_gemm2<P2>(a, H * wgs, stream, rows) | mk(wname(dense, 0, false));
        }
    }
    if constexpr (sizeof(ST) == 2 && !ROUTER && !GATHER) {
        using P2 = WgradQkvDensePolicy2<DH>;
        int rows;
        const int S = dense_ranges(R, H * (d / 64), P2::KC, rows);
        if (S > 0 && d % 64 == 0 && (long long)R * d < 1ll << 35 && (long long)R * H * 3 * DH < 1ll << 35) {
            typename P2::Args a{X, I, dQKV, dz16, dWq, dWk, dWv, dWr, part, T, d, H, n, R, d / 64, S, rows,
                                make_fastdiv(n)};
            int e = launch_gemm2<P2>(a, S * H * (d / 64), stream, rows);
            e |= mk(wname(dense, 0, false));
            if (e == 0) {
                const int total = H * d * (3 * DH / 8);
                hipLaunchKernelGGL((wgrad_qkv_reduce_kernel<ST, DH, false>), dim3((total + 255) / 256), dim3(256), 0,
                                   stream, part, S, H, d, dWq, dWk, dWv, dWr);
                e = hipGetLastError() == hipSuccess ? 0 : -1;
                e |= mk(wname(dense, 0, true));
            }
            return e;
        }
    }
    const WgradPlan w = plan_qkv<ST, DH, ROUTER, GATHER>(d, H, R);
    const int S = w.S;
    auto go = [&](auto p) {
        using PT = decltype(p);
        typename PT::Args a{X, I, dQKV, dz16, dWq, dWk, dWv, dWr, part, T, d, H, n, R, mtiles, S, w.cps, make_fastdiv(n)};
        return launch_gemm<ST, PT>(a, S * H * mtiles * PT::NTILES, stream);
    };
    int e;
    if constexpr (sizeof(ST) == 4) e = w.small ? go(WgradQkvPolicy<ST, DH, ROUTER, GATHER, true>{}) : go(P{});
    else e = go(P{});
    e |= mk(wname(dense, 0, false));
    if (S > 1 && e == 0) {
        const int total = H * d * (3 * DH / 8 + (ROUTER ? 1 : 0));
        hipLaunchKernelGGL((wgrad_qkv_reduce_kernel<ST, DH, ROUTER>), dim3((total + 255) / 256), dim3(256), 0, stream,
                           part, S, H, d, dWq, dWk, dWv, dWr);
        e = hipGetLastError() == hipSuccess ? 0 : -1;
        e |= mk(wname(dense, 0, true));
    }
    return e;
}

template <typename ST, int DH>
int run_qkv(const ST* X, const int32_t* I, const ST* dQKV, const ST* dz16, const float* dz, int B, int T, int d, int H, int n, ST* dWq,
            ST* dWk, ST* dWv, ST* dWr, float* part, const Marker& mk, hipStream_t stream) {
    if (I)  // MoSA heads: gathered rows and the router column
        return run_qkv_t<ST, DH, true, true>(X, I, dQKV, dz16, dz, B, T, d, H, n, dWq, dWk, dWv, dWr, part, mk, stream);
    return run_qkv_t<ST, DH, false, false>(X, I, dQKV, dz16, dz, B, T, d, H, n, dWq, dWk, dWv, dWr, part, mk, stream);
}

template <typename ST, int DH, bool GATHER>
int run_o_t(const ST* dY, const int32_t* I, const ST* A, int B, int T, int d, int H, int n, ST* dWo, float* part,
            const Marker& mk, hipStream_t stream) {
    using P = WgradOPolicy<ST, DH, GATHER>;
    const bool dense = !GATHER;
    const int R = B * n;
    if constexpr (sizeof(ST) == 2 && GATHER) {
        using P2 = WgradOPolicy2<DH, 64>;
        if (const int rows = wgrad2_table_rows<P2>(R, d, (long long)B * T, (long long)R * H, DH)) {
            const int tl = d / 64, per = wgrad_tiles_per_wg(H, tl, R), wgs = (tl + per - 1) / per;
            typename P::Args a{dY, I, A, dWo, part, T, d, H, n, R, tl, wgs, per, make_fastdiv(n)};
            return launch_gemm2<P2>(a, H * wgs, stream, rows) | mk(wname(dense, 1, false));
        }
    }
    if constexpr (sizeof(ST) == 2 && !GATHER) {
        using P2 = WgradODensePolicy2<DH>;
        int rows;
        const int S = dense_ranges(R, H * (d / 64), P2::KC, rows);
        if (S > 0 && d % 64 == 0 && (long long)R * d < 1ll << 35 && (long long)R * H * 3 * DH < 1ll << 35) {
            typename P2::Args a{dY, I, A, dWo, part, T, d, H, n, R, d / 64, S, rows, make_fastdiv(n)};
            int e = launch_gemm2<P2>(a, S * H * (d / 64), stream, rows);
            e |= mk(wname(dense, 1, false));
            if (e == 0) {
                const size_t n8 = (size_t)H * DH * d / 8;
                hipLaunchKernelGGL((wgrad_o_reduce_kernel<ST>), dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0,
                                   stream, part, S, n8, dWo);
                e = hipGetLastError() == hipSuccess ? 0 : -1;
                e |= mk(wname(dense, 1, true));
            }
            return e;
        }
    }
    const WgradPlan w = plan_o<ST, DH, GATHER>(d, H, R);
    const int S = w.S;
    auto go = [&](auto p) {
        using PT = decltype(p);
        const int nt = (d + PT::NT - 1) / PT::NT;
        typename PT::Args a{dY, I, A, dWo, part, T, d, H, n, R, nt, S, w.cps, make_fastdiv(n)};
        return launch_gemm<ST, PT>(a, S * H * nt, stream);
    };
    int e;
    if constexpr (sizeof(ST) == 4) e = w.small ? go(WgradOPolicy<ST, DH, GATHER, true>{}) : go(P{});
    else e = go(P{});
    e |= mk(wname(dense, 1, false));
    if (S > 1 && e == 0) {
        const size_t n8 = (size_t)H * DH * d / 8;
        hipLaunchKernelGGL((wgrad_o_reduce_kernel<ST>), dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, stream, part,
                           S, n8, dWo);
        e = hipGetLastError() == hipSuccess ? 0 : -1;
        e |= mk(wname(dense, 1, true));
    }
    return e;
}

template <typename ST, int DH>
int run_o(const ST* dY, const int32_t* I, const ST* A, int B, int T, int d, int H, int n, ST* dWo, float* part,
          const Marker& mk, hipStream_t stream) {
    if (I) return run_o_t<ST, DH, true>(dY, I, A, B, T, d, H, n, dWo, part, mk, stream);
    return run_o_t<ST, DH, false>(dY, I, A, B, T, d, H, n, dWo, part, mk, stream);
}

// dW^{Q,K,V,r} and dW^O of the MoSA heads in one launch of the gathered-row
// engine (the two kinds of workgroups share the CUs); 1: not applicable.
template <int DH>
int run_both(const uint16_t* X, const uint16_t* dY, const int32_t* I, const uint16_t* A, const uint16_t* dQKV,
             const uint16_t* dz16, const float* dz, int B, int T, int d, int H, int n, uint16_t* dWq, uint16_t* dWk, uint16_t* dWv,
             uint16_t* dWr, uint16_t* dWo, hipStream_t stream) {
    using ST = uint16_t;
    using PQ = WgradQkvPolicy2<DH, 64>;
    using PO = WgradOPolicy2<DH, 64>;
    const int R = B * n;
    const long long tokens = (long long)B * T, sel = (long long)R * H;
    const int rq = wgrad2_table_rows<PQ>(R, d, tokens, sel, DH), ro = wgrad2_table_rows<PO>(R, d, tokens, sel, DH);
    if (!rq || !ro) return 1;
    const int tl = d / 64, per = wgrad_tiles_per_wg(H, tl, R), wgs = (tl + per - 1) / per;
    typename PQ::Args aq{X, I, dQKV, dz16, dWq, dWk, dWv, dWr, nullptr, T, d, H, n, R, tl, wgs, per, make_fastdiv(n), dz};
    typename PO::Args ao{dY, I, A, dWo, nullptr, T, d, H, n, R, tl, wgs, per, make_fastdiv(n)};
    const int e = launch_gemm2_dual<PQ, PO>(aq, H * wgs, rq, ao, H * wgs, ro, stream);
    return e == -1 ? 1 : e;  // a shape the grouped launch cannot take falls back to two launches
}

// The three products after the attention backward in one launch: dW^{Q,K,V,r},
// dW^O and the per-head dX rows; 1: not applicable.  PQ, PO: the tiles of the
// two weight gradients.
template <class PQ, class PO, int DH>
int run_bwd_proj_t(const uint16_t* X, const uint16_t* dY, const int32_t* I, const uint16_t* A, const uint16_t* dQKV,
                   const uint16_t* dz16, const float* dz, const uint16_t* Wq, const uint16_t* Wk, const uint16_t* Wv,
                   const uint16_t* Wr, int B, int T, int d, int H, int n, uint16_t* dWq, uint16_t* dWk, uint16_t* dWv,
                   uint16_t* dWr, uint16_t* dWo, uint16_t* dXs, hipStream_t stream) {
    using PX = DxProjRowPolicy<DH>;
    const int R = B * n;
    const long long tokens = (long long)B * T, sel = (long long)R * H;
    const int rq = wgrad2_table_rows<PQ>(R, d, tokens, sel, DH), ro = wgrad2_table_rows<PO>(R, d, tokens, sel, DH);
    typename PX::Args ax;
    int nx;
    if (!rq || !ro || !dx_row_args<DH>(dQKV, dz, Wq, Wk, Wv, Wr, B, d, H, n, dXs, ax, nx)) return 1;
    const int tq = d / PQ::NT, pq = wgrad_tiles_per_wg(H, tq, rq), wq = (tq + pq - 1) / pq;
    const int to = d / PO::MT, po = wgrad_tiles_per_wg(H, to, ro), wo = (to + po - 1) / po;
    typename PQ::Args aq{X, I, dQKV, dz16, dWq, dWk, dWv, dWr, nullptr, T, d, H, n, R, tq, wq, pq, make_fastdiv(n), dz};
    typename PO::Args ao{dY, I, A, dWo, nullptr, T, d, H, n, R, to, wo, po, make_fastdiv(n)};
    return launch_group3<Gemm2Job<PQ>, Gemm2Job<PO>, RowGemmJob<PX>>(
        aq, H * wq, Gemm2Job<PQ>::lds(rq), ao, H * wo, Gemm2Job<PO>::lds(ro), ax, nx,
        RowGemmJob<PX>::lds(0), stream);
}

// Whether a CU's 160 KB of LDS hold two workgroups of the grouped launch.
template <class PQ, class PO>
bool two_per_cu(int rows) {
    return 2 * std::max(Gemm2Job<PQ>::lds(rows), Gemm2Job<PO>::lds(rows)) <= 160 * 1024;
}

template <int DH>
int run_bwd_proj(const uint16_t* X, const uint16_t* dY, const int32_t* I, const uint16_t* A, const uint16_t* dQKV,
                 const uint16_t* dz16, const float* dz, const uint16_t* Wq, const uint16_t* Wk, const uint16_t* Wv,
                 const uint16_t* Wr, int B, int T, int d, int H, int n, uint16_t* dWq, uint16_t* dWk, uint16_t* dWv,
                 uint16_t* dWr, uint16_t* dWo, uint16_t* dXs, hipStream_t stream) {
    auto go = [&](auto f) {
        return f(X, dY, I, A, dQKV, dz16, dz, Wq, Wk, Wv, Wr, B, T, d, H, n, dWq, dWk, dWv, dWr, dWo, dXs, stream);
    };
    using PQN = WgradQkvPolicy2<DH, 64>;
    using PON = WgradOPolicy2<DH, 64>;
    if constexpr (DH == 64) {
        using PQW = WgradQkvPolicy2<DH, 128>;
        using POW = WgradOPolicy2<DH, 128>;
        // 128-column tiles where they still give every CU one, unless their
        // rings and row tables (with R rows) let a CU hold one workgroup where
        // those of 64 columns let it hold two: up to 1024 rows two of either,
        // up to 2048 two of 64 columns only, beyond one of either.  Training
        // step with 64 columns against 128, T = 256, k = 64 (us): 27 heads of
        // d 1280, R = 512 124 against 117, 1024 198 / 189, 1536 260 / 273,
        // 2048 331 / 346, 3072 532 / 491; 128 heads of d 1024, 1024 563 / 533,
        // 1536 859 / 890, 2048 1144 / 1182, 3072 1911 / 1713.
        const int rows = (B * n + 63) / 64 * 64;
        if (d % 128 == 0 && H * (d / 128) >= kFullChip &&
            (two_per_cu<PQW, POW>(rows) || !two_per_cu<PQN, PON>(rows)))
            return go(run_bwd_proj_t<PQW, POW, DH>);
    }
    return go(run_bwd_proj_t<PQN, PON, DH>);
}

// Bytes of fp32 partial sums the two launches of one head group need.
template <typename ST, int DH>
size_t partial_bytes(int B, int T, int d, int H, int n, bool router) {
    const int R = B * n;
    if constexpr (sizeof(ST) == 2) {  // MoSA heads on the gathered-row engine: no partials
        // (a tensor past the table's reach takes the fallback, whose partials are kept room for)
        if (router && wgrad2_table_rows<WgradQkvPolicy2<DH, 64>>(R, d, (long long)B * T, (long long)R * H, DH) &&
            wgrad2_table_rows<WgradOPolicy2<DH, 64>>(R, d, (long long)B * T, (long long)R * H, DH))
            return 0;
    }
    // (the plans do not depend on GATHER)
    const int sq = router ? plan_qkv<ST, DH, true, true>(d, H, R).S : plan_qkv<ST, DH, false, false>(d, H, R).S;
    const int so = plan_o<ST, DH, true>(d, H, R).S;
    const size_t nq = 3 * DH + (router ? 16 : 0);
    size_t bq = sq > 1 ? (size_t)sq * H * d * nq * 4 : 0;
    size_t bo = so > 1 ? (size_t)so * H * DH * d * 4 : 0;
    if constexpr (sizeof(ST) == 2) {
        if (!router && d % 64 == 0) {  // dense heads on the multi-stage engine: one partial per row range
            int rows;
            const int sd = dense_ranges(R, H * (d / 64), WgradQkvDensePolicy2<DH>::KC, rows);
            const int so2 = dense_ranges(R, H * (d / 64), WgradODensePolicy2<DH>::KC, rows);
            bq = std::max(bq, (size_t)sd * H * d * 3 * DH * 4);
            bo = std::max(bo, (size_t)so2 * H * DH * d * 4);
        }
    }
    return bq > bo ? bq : bo;
}

}  // namespace

int launch_wgrad(int dtype, const void* X, const void* dY, const int32_t* I, const void* A, const void* dQKV,
                 const void* dz16, const float* dz, int B, int T, int d, int H, int dh, int n, void* dWq, void* dWk,
                 void* dWv, void* dWr, void* dWo, float* part, int which, const Marker& mk, hipStream_t stream) {
    if (H == 0) return 0;
    if (which == 2) {
        // both: one launch on the gathered-row engine where it applies
        if (dtype == kBF16 && I) {
            using ST = uint16_t;
            auto both = dh == 64 ? run_both<64> : run_both<32>;
            const int e = both((const ST*)X, (const ST*)dY, I, (const ST*)A, (const ST*)dQKV, (const ST*)dz16, dz, B, T, d,
                               H, n, (ST*)dWq, (ST*)dWk, (ST*)dWv, (ST*)dWr, (ST*)dWo, stream);
            if (e != 1) return e | mk("wgrad");
        }
        const int e0 = launch_wgrad(dtype, X, dY, I, A, dQKV, dz16, dz, B, T, d, H, dh, n, dWq, dWk, dWv, dWr, dWo, part,
                                    0, mk, stream);
        return e0 | launch_wgrad(dtype, X, dY, I, A, dQKV, dz16, dz, B, T, d, H, dh, n, dWq, dWk, dWv, dWr, dWo, part, 1,
                                 mk, stream);
    }
    if (dtype == kBF16) {
        using ST = uint16_t;
        if (which == 0) {
            auto f = dh == 64 ? run_qkv<ST, 64> : run_qkv<ST, 32>;
            return f((const ST*)X, I, (const ST*)dQKV, (const ST*)dz16, dz, B, T, d, H, n, (ST*)dWq, (ST*)dWk, (ST*)dWv,
                     (ST*)dWr, part, mk, stream);
        }
        auto f = dh == 64 ? run_o<ST, 64> : run_o<ST, 32>;
        return f((const ST*)dY, I, (const ST*)A, B, T, d, H, n, (ST*)dWo, part, mk, stream);
    }
    using ST = float;
    if (which == 0) {
        auto f = dh == 64 ? run_qkv<ST, 64> : run_qkv<ST, 32>;
        return f((const ST*)X, I, (const ST*)dQKV, (const ST*)dz16, dz, B, T, d, H, n, (ST*)dWq, (ST*)dWk, (ST*)dWv,
                 (ST*)dWr, part, mk, stream);
    }
    auto f = dh == 64 ? run_o<ST, 64> : run_o<ST, 32>;
    return f((const ST*)dY, I, (const ST*)A, B, T, d, H, n, (ST*)dWo, part, mk, stream);
}

int launch_bwd_proj(int dtype, const void* X, const void* dY, const int32_t* I, const void* A, const void* dQKV,
                    const void* dz16, const float* dz, const void* Wq, const void* Wk, const void* Wv, const void* Wr,
                    int B, int T, int d, int H, int dh, int n, void* dWq, void* dWk, void* dWv, void* dWr, void* dWo,
                    void* dXs, hipStream_t stream) {
    if (dtype != kBF16 || H == 0 || !I) return 1;
    // few selected rows per head: the per-head streaming kernel
    const int e = launch_bwd_head(dtype, X, dY, I, A, dQKV, dz16, dz, Wq, Wk, Wv, Wr, B, T, d, H, dh, n, dWq, dWk, dWv,
                                  dWr, dWo, dXs, stream);
    if (e != 1) return e;
    using ST = uint16_t;
    auto f = dh == 64 ? run_bwd_proj<64> : run_bwd_proj<32>;
    return f((const ST*)X, (const ST*)dY, I, (const ST*)A, (const ST*)dQKV, (const ST*)dz16, dz, (const ST*)Wq,
             (const ST*)Wk, (const ST*)Wv, (const ST*)Wr, B, T, d, H, n, (ST*)dWq, (ST*)dWk, (ST*)dWv, (ST*)dWr,
             (ST*)dWo, (ST*)dXs, stream);
}

// The gathered-row engine takes dz in fp32; the per-head kernel of few rows and
// the engine of gemm.h take the 16-wide rows.
bool wgrad_reads_dz16(int dtype, int B, int T, int d, int H, int dh, int n) {
    const long long R = (long long)B * n;
    if (dtype != kBF16 || (dh == 64 && R <= kBwdHeadMaxRows)) return true;
    return !(dh == 64 ? wgrad2_table_rows<WgradQkvPolicy2<64, 64>>((int)R, d, (long long)B * T, R * H, 64)
                      : wgrad2_table_rows<WgradQkvPolicy2<32, 64>>((int)R, d, (long long)B * T, R * H, 32));
}

size_t wgrad_partial_bytes(int dtype, int B, int T, int d, int H, int dh, int n, int router) {
    if (H == 0 || n == 0) return 0;
    if (dtype == kBF16)
        return dh == 64 ? partial_bytes<uint16_t, 64>(B, T, d, H, n, router)
                        : partial_bytes<uint16_t, 32>(B, T, d, H, n, router);
    return dh == 64 ? partial_bytes<float, 64>(B, T, d, H, n, router) : partial_bytes<float, 32>(B, T, d, H, n, router);
}

}  // namespace mosa
