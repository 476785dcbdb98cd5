// Gather + grouped Q/K/V projection (paper Section 2.2: X^s = X[I];
// Q = X^s W^Q, K = X^s W^K, V = X^s W^V, computed only for the k selected
// tokens of every head; a dense head is the case I = 0..T-1).
//
// One GEMM per head: B*n gathered rows (b, i) -> token I[b,h,i], 3*dh columns
// (Q | K | V side by side), contraction over d.  fp32: the engine of gemm.h
// (QkvPolicy), the rows gathered once per thread before the K loop, the
// weights W^{Q,K,V}_h [d, dh] transposed 8x8 in registers on their way into
// LDS.  bf16: the engine of gemm2.h (QkvPolicy2), with the attention in the same
// launch where a tile holds whole groups (QkvAttnPolicy).  The output is one packed row [Q | K | V] per selected
// token, so the attention kernels read each token's q, k, v from one row.
// Workgroups of one head are numbered consecutively on one XCD so the head's
// weights are fetched from HBM once into that XCD's L2.
#include "attn_lds.h"
#include "gemm.h"
#include "gemm2.h"
#include "kernels.h"
#include "rope.h"

namespace mosa {

namespace {

// fp32 storage.  SMALL: 32 rows and one of Q, K, V per workgroup.
template <typename ST, int DH, bool SMALL>
struct QkvPolicy {
    static constexpr int MT = SMALL ? 32 : 64, NT = SMALL ? DH : 3 * DH, KC = 32, WM = 2, WN = 2;
    static constexpr int NTILES = 3 * DH / NT;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = true, B_KCONTIG = false;
    struct Args {
        const ST* X;
        const int32_t* I;  // nullptr: identity (dense heads)
        const ST* W0;
        const ST* W1;
        const ST* W2;
        ST* out;  // [B, H, n, 3*DH]
        int T, d, H, n, M, mtiles;
        const float2* rope;  // rotary table [T, DH/4] or nullptr
    };
    struct ARef {
        const ST* p;
    };
    struct BRef {};
    struct RowInfo {
        int k;
    };
    __device__ static const ST* a_fallback(const Args& a) { return a.X; }
    __device__ static const ST* b_fallback(const Args& a) { return a.W0; }

    __device__ static void tile(const Args& a, int logical, int& batch, int& m0, int& n0) {
        const int per = a.mtiles * NTILES, rem = logical % per;
        batch = logical / per;
        m0 = (rem / NTILES) * MT;
        n0 = (rem % NTILES) * NT;
    }
    __device__ static int k_size(const Args& a, int) { return a.d; }
    __device__ static ARef a_row(const Args& a, int h, int m) {
        if (m < 0 || m >= a.M) return {nullptr};
        const int b = m / a.n, i = m % a.n;
        const int t = a.I ? a.I[((size_t)b * a.H + h) * a.n + i] : i;
        return {a.X + ((size_t)b * a.T + t) * a.d};
    }
    __device__ static const ST* a_elem(const Args&, int, const ARef& r, int k) { return r.p ? r.p + k : nullptr; }
    __device__ static BRef b_row(const Args&, int, int) { return {}; }
    __device__ static const ST* b_elem(const Args&, int, const BRef&, int) { return nullptr; }
    __device__ static RowInfo row_info(const Args&, int, int k) { return {k}; }
    __device__ static const ST* a_kaddr(const Args& a, int, const RowInfo&, int) { return a_fallback(a); }
    __device__ static bool a_kok(const Args&, int, const RowInfo&, int) { return false; }
    // B[k][n] = W^{n / DH}_h[k][n % DH]: row k of the [d, DH] weight, n contiguous
    __device__ static const ST* b_kaddr(const Args& a, int h, const RowInfo& r, int n8) {
        const ST* W = n8 < DH ? a.W0 : (n8 < 2 * DH ? a.W1 : a.W2);
        return W + ((size_t)h * a.d + max(r.k, 0)) * DH + (n8 % DH);
    }
    __device__ static bool b_kok(const Args&, int, const RowInfo& r, int) { return r.k >= 0; }
    __device__ static void epilogue(const Args& a, int h, int m0, int n0, const float* Cs, int ldc, int tid,
                                    unsigned char*) {
        constexpr int VPR = NT / 8;  // vectors per row
        for (int v = tid; v < MT * VPR; v += 256) {
            const int ml = v / VPR, c = (v % VPR) * 8;
            const int m = m0 + ml;
            if (m >= a.M) continue;
            const int b = m / a.n, i = m % a.n;
            float x[8];
            cs_load8(Cs, ldc, ml, c, x);
            rope_cols(a, h, b, i, n0 + c, x);
            vec8_store<ST>(a.out + (((size_t)b * a.H + h) * a.n + i) * (3 * DH) + n0 + c, vec8_from_f32<ST>(x));
        }
    }
    // columns c .. c + 7 of row (b, h, i): the rotary encoding of q and k
    __device__ static void rope_cols(const Args& a, int h, int b, int i, int c, float (&x)[8]) {
        if (!a.rope) return;
        const int cq = c < DH ? c : c - DH;  // column within q or k
        if (c >= 2 * DH || cq >= DH / 2) return;
        const int pos = a.I ? a.I[((size_t)b * a.H + h) * a.n + i] : i;
        rope8<DH>(x, cq, a.rope, pos, 1.f);
    }
};

// bf16 storage: the multi-stage engine with direct-to-LDS loads (gemm2.h), as
// the transposed product: A = the three weights as one m-contiguous [d][3 DH]
// operand (M = the packed column), B = RT gathered token rows (k-contiguous,
// clamped to the last row past M).  A lane then holds 8 consecutive packed
// columns of a row, which it rotates, rounds and stores as 16 bytes from its
// registers; no fp32 C tile passes through LDS (that tile's write, its
// read-back and the index divisions of the copy took 6 of the 20.6 us of the
// fused launch below at B = 8, T = 1024, d = 512, 32 heads, k = 128, and its
// 100 KB kept a second workgroup off the CU).
template <int DH, int RT = 128>
struct QkvPolicy2 {
    using ST = uint16_t;
    static constexpr int MT = 3 * DH, NT = RT, KC = DH == 64 ? 32 : 64, WM = DH == 64 ? 2 : 1, WN = 4 / WM, STAGES = 4;
    static constexpr size_t EPI_LDS = 0;
    static constexpr bool A_KCONTIG = false, B_KCONTIG = true, A_INTERLEAVE = true, EPI_REGS = true, EPI_ACC = true;
    struct Args {
        const ST* X;
        const int32_t* I;  // nullptr: identity (dense heads)
        const ST* W0;
        const ST* W1;
        const ST* W2;
        ST* out;  // [B, H, n, 3*DH]
        int T, d, H, n, M;
        const float2* rope;  // rotary table [T, DH/4] or nullptr
        FastDiv nd;          // by n
    };
    struct BRef {
        const ST* p;
    };
    static int row_tiles(int M) { return (M + NT - 1) / NT; }
    __device__ static void tile(const Args& a, int logical, int& batch, int& m0, int& n0) {
        const int rt = (a.M + NT - 1) / NT;
        if (a.I) {  // a head's row tiles side by side: they share its weights
            batch = logical / rt;
            n0 = (logical % rt) * NT;
        } else {  // dense heads: the heads of a row tile side by side (its X rows)
            batch = logical % a.H;
            n0 = (logical / a.H) * NT;
        }
        m0 = 0;
    }
    __device__ static int k_size(const Args& a, int) { return a.d; }
    // A[m][k] = W^{m / DH}_h[k][m % DH]
    __device__ static size_t a_kstride(const Args&, int) { return DH; }
    __device__ static const ST* a_maddr(const Args& a, int h, int k, int m8) {
        const ST* W = m8 < DH ? a.W0 : (m8 < 2 * DH ? a.W1 : a.W2);
        return W + ((size_t)h * a.d + k) * DH + (m8 % DH);
    }
    __device__ static BRef b_row(const Args& a, int h, int m) {
        int b, i;
        fast_divmod(a.nd, min(m, a.M - 1), b, i);
        const int t = a.I ? a.I[((size_t)b * a.H + h) * a.n + i] : i;
        return {a.X + ((size_t)b * a.T + t) * a.d};
    }
    __device__ static const ST* b_elem(const Args&, int, const BRef& r, int k) { return r.p + k; }
    // Every 8-column vector of the tile: rotated (q and k), rounded, stored in
    // its packed row, and handed to use(ml, c, y) (row ml of the tile, packed
    // column c; rows past M hold the clamped last row's values).
    template <class S, class F>
    __device__ static void each_vec8(const Args& a, int h, int n0, const f32x4 (&acc)[S::FM][S::FN], int wm, int wn,
                                     int tid, F use) {
        const int lane = tid & 63, g = lane >> 4, c16 = lane & 15;
        constexpr int HALF = DH / 2;  // rotated columns of q and of k
        ST* dst[S::FN];
        float4 tab[S::FN][2];
#pragma unroll
        for (int j = 0; j < S::FN; ++j) {
            const int m = n0 + wn * S::WTN + 16 * j + c16;
            int b, i;
            fast_divmod(a.nd, min(m, a.M - 1), b, i);
            const size_t ri = ((size_t)b * a.H + h) * a.n + i;
            dst[j] = m < a.M ? a.out + ri * (3 * DH) : nullptr;
            if (a.rope) {  // the pairs of columns 8 g % HALF .. + 7, the same for q and k
                const int pos = a.I ? a.I[ri] : i;
                const float4* t = reinterpret_cast<const float4*>(a.rope + (size_t)pos * (DH / 4) + (8 * g % HALF) / 2);
                tab[j][0] = t[0];
                tab[j][1] = t[1];
            }
        }
#pragma unroll
        for (int p = 0; p < S::FM / 2; ++p) {
            const int c = wm * S::WTM + 32 * p + 8 * g;  // packed column
            const bool rot = a.rope && c < 2 * DH && c % DH < HALF;
#pragma unroll
            for (int j = 0; j < S::FN; ++j) {
                float x[8];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[r] = acc[2 * p][j][r];
                    x[4 + r] = acc[2 * p + 1][j][r];
                }
                if (rot) rope8_tab(x, tab[j][0], tab[j][1], 1.f);
                const uint4 y = vec8_from_f32<ST>(x).v;
                if (dst[j]) *reinterpret_cast<uint4*>(dst[j] + c) = y;
                use(wn * S::WTN + 16 * j + c16, c, y);
            }
        }
    }
    template <class S>
    __device__ static void epi_acc(const Args& a, int h, int, int n0, const f32x4 (&acc)[S::FM][S::FN], int wm, int wn,
                                   int tid, unsigned char*) {
        each_vec8<S>(a, h, n0, acc, wm, wn, tid, [](int, int, const uint4&) {});
    }
};

// QKV projection and attention in one kernel, for groups of n | 128 rows
// (n = 16, 32, 64 or 128): every tile holds whole (b, h) groups, so while the
// epilogue writes the packed Q | K | V rows (kept for the backward pass), the
// same workgroup copies Q, K and V in bf16 into LDS and then runs the attention
// of its groups (attn_lds.h, bit-identical to the separate attention kernel).
// The bf16 tiles (50 KB at 128 rows of 64) fit in the stage buffers, so the
// 80 KB of a workgroup leave room for two per CU, and, with more tiles than
// CUs, the epilogue of one overlaps the loop of the other.
template <int DH, int RT = 128>
struct QkvAttnPolicy : QkvPolicy2<DH, RT> {
    using ST = uint16_t;
    using Base = QkvPolicy2<DH, RT>;
    static constexpr int U = DH / 8, VROWS = RT + 16;
    // bf16 Q and K tiles, then the V tile with 16 zero rows after it (the last
    // group's odd key block reads 16 rows past its end, at weight zero)
    static constexpr size_t EPI_LDS = (size_t)(2 * RT + VROWS) * DH * 2;
    static_assert(RT == 128 || RT == 64, "one or two query blocks per wave");
    static constexpr int QBW = RT / 64;  // query blocks of 16 rows per wave
    struct Args : Base::Args {
        const float* r;  // [B, H, n] router weights of the selected rows
        ST* A;           // [B, H, n, DH]
        float* lse;      // [B, H, n]
        int causal;
        float scale;
    };
    template <class S>
    __device__ static void epi_acc(const Args& a, int h, int, int n0, const f32x4 (&acc)[S::FM][S::FN], int wm, int wn,
                                   int tid, unsigned char* smem) {
        unsigned char* Qs = smem;
        unsigned char* Ks = Qs + (size_t)RT * DH * 2;
        unsigned char* Vs = Ks + (size_t)RT * DH * 2;
        Base::template each_vec8<S>(a, h, n0, acc, wm, wn, tid, [&](int ml, int c, const uint4& y) {
            const int part = c / DH, u = (c % DH) / 8;
            unsigned char* t = part == 0 ? Qs : part == 1 ? Ks : Vs;
            *reinterpret_cast<uint4*>(t + (ml * U + (u ^ (part == 2 ? vt_swz<U>(ml) : kswz(ml, U)))) * 16) = y;
        });
        for (int v = tid; v < (VROWS - RT) * U; v += 256)
            *reinterpret_cast<uint4*>(Vs + (size_t)(RT * U + v) * 16) = make_uint4(0, 0, 0, 0);
        __syncthreads();
        // the score registers sized by n: with 16 rows a 128-key form spends
        // most of its exponentials on masked keys
        if (a.n <= 32) attend<32>(a, h, n0, tid, Qs, Ks, Vs);
        else if (a.n == 64) attend<64>(a, h, n0, tid, Qs, Ks, Vs);
        else if constexpr (RT == 128) attend<128>(a, h, n0, tid, Qs, Ks, Vs);
    }
    // RT / 16 query blocks over 4 waves: 128 rows, blocks w and 7 - w, so that
    // every wave's causal key blocks add up to the same count; 64 rows, block w
    template <int NMAX>
    __device__ static void attend(const Args& a, int h, int n0, int tid, const unsigned char* Qs,
                                  const unsigned char* Ks, const unsigned char* Vs) {
        const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, c16 = lane & 15;
        const int n = a.n, lgb = 31 - __builtin_clz(n / 16);  // query blocks per group: 2^lgb
        for (int j2 = 0; j2 < QBW; ++j2) {
            const int j = j2 ? 7 - wave : wave, gi = j >> lgb, qb = j & ((1 << lgb) - 1), mg = n0 + gi * n;
            if (mg >= a.M) continue;
            const size_t bh = (size_t)(mg >> (lgb + 4)) * a.H + h;
            const int row = gi * n + 16 * qb + c16;
            Frag8<ST> qf[DH / 32];
#pragma unroll
            for (int st = 0; st < DH / 32; ++st)
                qf[st].v = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const uint4*>(Qs + (row * U + ((4 * st + g) ^ kswz(row, U))) * 16));
            attn_lds_block<DH, NMAX>(Ks, Vs, gi * n, qf, n, a.causal, a.scale, qb, a.r ? a.r + bh * n : nullptr,
                                     a.A + bh * n * DH, a.lse + bh * n);
        }
    }
};

// Rows per tile of the gathered heads: 64 where 128-row tiles would be half
// empty or too few to give every CU one (24 tiles of 12 heads, 256 rows each:
// 28.2 us with 128 rows, 21.3 with 64; 17 half-empty ones 10.1 and 7.3), else
// 128, which reads the weights half as often (256 tiles: 30.5 us with 128
// rows, 33.9 with 64; 872: 105 and 110).
inline bool narrow_rows(int M, int H) { return M <= 64 || (long long)H * ((M + 127) / 128) < 256; }

template <typename ST, int DH>
int run(const ST* X, const int32_t* I, const ST* Wq, const ST* Wk, const ST* Wv, int B, int T, int d, int H, int n,
        ST* out, const float2* rope, int narrow, hipStream_t stream) {
    if constexpr (sizeof(ST) == 2) {  // d is a multiple of 64, so of every KC
        auto go = [&](auto rt) {
            using P = QkvPolicy2<DH, decltype(rt)::value>;
            const typename P::Args a{X, I, Wq, Wk, Wv, out, T, d, H, n, B * n, rope, make_fastdiv(n)};
            return launch_gemm2<P>(a, P::row_tiles(B * n) * H, stream);
        };
        return narrow || (I && narrow_rows(B * n, H)) ? go(std::integral_constant<int, 64>{}) : go(std::integral_constant<int, 128>{});
    } else {
        auto go = [&](auto small) {
            using P = QkvPolicy<ST, DH, decltype(small)::value>;
            typename P::Args a{X, I, Wq, Wk, Wv, out, T, d, H, n, B * n, (B * n + P::MT - 1) / P::MT, rope};
            return launch_gemm<ST, P>(a, a.mtiles * H * P::NTILES, stream);
        };
        return (B * n + 63) / 64 * H < kFullChip ? go(std::true_type{}) : go(std::false_type{});
    }
}

}  // namespace

int launch_qkv_attn(int dtype, const void* X, const int32_t* I, const void* Wq, const void* Wk, const void* Wv,
                    int B, int T, int d, int H, int dh, int n, void* QKV, const float2* rope, const float* r,
                    int causal, void* A, float* lse, hipStream_t stream) {
    if (dtype != kBF16 || n < 16 || n % 16 || 128 % n || (dh != 64 && dh != 32)) return 1;
    const float scale = 1.0f / sqrtf((float)dh);
    auto go = [&](auto tag, auto mt) {
        constexpr int DH = decltype(tag)::value;
        using P = QkvAttnPolicy<DH, decltype(mt)::value>;
        typename P::Args a{};
        static_cast<typename P::Base::Args&>(a) = {
            (const uint16_t*)X, I, (const uint16_t*)Wq, (const uint16_t*)Wk, (const uint16_t*)Wv, (uint16_t*)QKV,
            T, d, H, n, B * n, rope, make_fastdiv(n)};
        a.r = r;
        a.A = (uint16_t*)A;
        a.lse = lse;
        a.causal = causal;
        a.scale = scale;
        return launch_gemm2<P>(a, P::row_tiles(B * n) * H, stream);
    };
    // 64-row tiles where the 128-row ones would be half empty or leave CUs idle
    if (n < 128 && narrow_rows(B * n, H))
        return dh == 64 ? go(std::integral_constant<int, 64>{}, std::integral_constant<int, 64>{})
                        : go(std::integral_constant<int, 32>{}, std::integral_constant<int, 64>{});
    return dh == 64 ? go(std::integral_constant<int, 64>{}, std::integral_constant<int, 128>{})
                    : go(std::integral_constant<int, 32>{}, std::integral_constant<int, 128>{});
}

int launch_qkv(int dtype, const void* X, const int32_t* I, const void* Wq, const void* Wk, const void* Wv, int B,
               int T, int d, int H, int dh, int n, void* QKV, const float2* rope, int narrow, hipStream_t stream) {
    if (dtype == kBF16) {
        auto f = dh == 64 ? run<uint16_t, 64> : run<uint16_t, 32>;
        return f((const uint16_t*)X, I, (const uint16_t*)Wq, (const uint16_t*)Wk, (const uint16_t*)Wv, B, T, d, H, n,
                 (uint16_t*)QKV, rope, narrow, stream);
    }
    auto f = dh == 64 ? run<float, 64> : run<float, 32>;
    return f((const float*)X, I, (const float*)Wq, (const float*)Wk, (const float*)Wv, B, T, d, H, n, (float*)QKV,
             rope, 0, stream);
}

}  // namespace mosa
