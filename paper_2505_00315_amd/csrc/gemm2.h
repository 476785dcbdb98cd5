// Multi-stage MFMA GEMM engine for bf16 storage with direct global->LDS loads.
//
//   C[M x N] = sum_k A[M x K] B[K x N]   (fp32 accumulation), one problem per
//   "batch" index, tiles of MT x NT, four waves, K in chunks of KC.
//
// Operands are copied from global memory straight into LDS with 16-byte
// global_load_lds instructions (no register staging): one instruction of a
// wave fills 1 KB of LDS, lane l writing bytes 16 l .. 16 l + 15, and each
// lane chooses the global 16 bytes that belong at its slot.  STAGES chunk
// buffers are in flight; one barrier per chunk.
//
// A k-contiguous operand (rows along M or N, 8 consecutive k per 16 bytes) is
// stored row-major [rows][KC] with the 16-byte units of a row XOR-permuted
// (f(r) below) so that the ds_read_b128 of an MFMA fragment (16 rows, same
// k) hits distinct banks.  An m-contiguous operand (rows along K, e.g. a
// weight W[k][n]) is stored [KC][R] as in memory, units permuted by h(k), and
// its MFMA fragments are read with ds_read_b64_tr_b16, which transposes 4 x 4
// blocks of 16-bit elements across the lanes of a 16-lane group: source lane
// s supplies the address of row kbase + s/4, columns m0 + 4 (s % 4) .. +3, and
// lane i receives rows kbase .. kbase + 3 of column m0 + i.  Two such reads give
// the 8 consecutive k of an MFMA operand, in the same k order as the
// k-contiguous reads.
//
// Policy P (all addresses must be valid for any k in [0, K) and any row; rows
// past the problem are clamped by the policy and their results discarded):
//   MT, NT, KC, WM, WN, STAGES, EPI_LDS; A_KCONTIG, B_KCONTIG;
//   tile(args, logical, batch, m0, n0), k_size(args, batch) (a multiple of KC);
//   k-contiguous: a_row(args, batch, m) -> ARef, a_elem(args, batch, ARef, k)
//                 (likewise b_row / b_elem);
//   m-contiguous: a_maddr(args, batch, k, m8) / b_maddr(args, batch, k, n8) and
//                 a_kstride(args, batch) / b_kstride(args, batch), the element
//                 distance between consecutive k (addresses move linearly in k);
//   epilogue(args, batch, m0, n0, Cs, ldc, tid, extra) as in gemm.h.
//
// Optional (all off by default):
//   KGATHER: the rows along k are gathered (both operands m-contiguous).  The
//     workgroup first fills an LDS table with k_row(args, batch, k) -> uint2 for
//     every k of its range (clamped to the last one in the padded part), and a
//     lane's address for row k is a_mlane(args, batch, m8) + 16 tab[k].x bytes
//     (.y with A_TAB 1; likewise b_mlane / B_TAB): one 64-bit shift and add per
//     load, as the loop has little room for address arithmetic beside the
//     MFMAs.  K need not be a multiple of KC: the rows past K of the last chunk
//     are cleared in LDS.
//   MULTI (with KGATHER and EPI_REGS): a workgroup runs tiles(args, logical)
//     output tiles one after the other, adjacent along M (MULTI_A, the A
//     operand's columns move by MT per tile) or along N (the B operand's by
//     NT), as one pipeline over all their chunks: the row table and the
//     pipeline's fill are paid once, and the next tile's loads are in flight
//     while a tile is stored.  STORES: the number of memory instructions that
//     every wave issues at least while storing a tile (they count in the waits
//     that follow; vector memory operations complete in issue order).
//   ROW (with MULTI): a product of one fp32 weight per k with every column of
//     the B tile beside the MFMAs, out[n] = sum_k f[k] B[k][n], by VALU from
//     the B fragments in registers (the WM waves of a column block share its
//     columns).  Another LDS table holds f = k_f(args, batch, k, K) (0 past K);
//     store_row(args, batch, n, sum) writes a column's sum.
//   A_INTERLEAVE: an m-contiguous A operand whose 16-row MFMA blocks are taken
//     in pairs with interleaved columns (block 2p row i is M index
//     32 p + 8 (i / 4) + i % 4, block 2p + 1 row i is 32 p + 8 (i / 4) + 4 + i % 4),
//     so that a lane's accumulators of a block pair are 8 consecutive M.
//   MIN_WAVES: waves per SIMD the register allocation must allow.
//   CHUNK_ADD (k-contiguous A and B): each MFMA from zero, then one add.
//   EPI_REGS (needs A_INTERLEAVE): no C tile; the engine calls
//     store8(args, batch, m, n, x[8]) for M indices m .. m + 7 at column n, or,
//     where the policy has it, epi_acc<Gemm2Shape<P>>(args, batch, m0, n0, acc,
//     wm, wn, tid, smem) with the wave's accumulators: acc[2 p][j][r] and
//     acc[2 p + 1][j][r] are M indices wm WTM + 32 p + 8 g + r and + 4 + r at
//     column wn WTN + 16 j + lane % 16 of the tile (g = lane / 16).  The
//     stage buffers are free by then (EPI_LDS bytes from smem on).
//   a_tile_hook(args, m0, n0, a_tile, tid, state) / a_hook_done(args, m0, n0,
//     tid, state): called by every thread for each k chunk with that chunk's A
//     tile in LDS (k-contiguous layout above), before the MFMAs of the chunk's
//     last 32-k step, and once after the last chunk; `state` is one double per
//     thread, zero before the first.
#pragma once

#include "gemm.h"

namespace mosa {

typedef __attribute__((address_space(3))) unsigned char lds_u8;

// One wave's 1 KB of LDS from 64 lanes x 16 bytes of global memory
// (global_load_lds_dwordx4: the LDS base goes in M0, lane l writes base +
// 16 l).  Issued as inline assembly so that the compiler does not treat the
// asynchronous LDS write as aliasing every later LDS read and wait for all
// loads in flight; the engine waits for these loads itself (wait_vmcnt).
// `base` is the wave-uniform LDS byte address of the 1 KB block.
__device__ __forceinline__ void lds_load16(const void* g, uint32_t base) {
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(size_t)(const lds_u8*)p; }

// Four 16-bit elements of a transposed 4 x 4 block (see above), issued as
// inline assembly for kernels that place the wait themselves, after work that
// does not need the result.  It is not ready until lds_wait() below; nothing may
// read it earlier.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_tr16(const unsigned char* p) {
    const uint32_t off = (uint32_t)(size_t)(lds_u8*)p;
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(r) : "v"(off) : "memory");
    return r;
}
// The same at p + OFF bytes (the instruction's immediate offset).
template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr16_at(const unsigned char* p) {
    static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
    const uint32_t off = (uint32_t)(size_t)(lds_u8*)p;
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(off), "i"(OFF) : "memory");
    return r;
}
// The same through the builtin: the compiler schedules it and waits for it like
// any LDS read.  For tiles whose direct-to-LDS loads are issued by lds_load16
// (invisible to the compiler), so that no wait on those is added.
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ u32x2 lds_tr16(const unsigned char* p) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds_u8*)p));
}
// Wait for every outstanding LDS read of this wave.
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// Make x depend on the preceding lds_wait() (an empty volatile statement that
// claims to modify x keeps its consumers after the wait).
__device__ __forceinline__ void lds_ready(u32x4& x) { asm volatile("" : "+v"(x)); }

// Unit permutations (both are involutions within a row).
__device__ __forceinline__ int kswz(int r, int lpr) {
    return lpr == 8 ? ((r & 7) ^ ((r >> 3) & 1)) : ((r & 3) ^ ((r >> 2) & 3));
}
template <int U>  // units per m-contiguous row
__device__ __forceinline__ int mswz(int k, int u) {
    if constexpr (U % 16 == 0) return u ^ (2 * ((k & 3) | (((k >> 3) & 1) << 2)));
    else if constexpr (U % 8 == 0) return u ^ (2 * (((k >> 1) & 1) | (((k >> 3) & 1) << 1)));
    else return u;
}

template <class P, class = void> struct G2Gather : std::false_type {};
template <class P> struct G2Gather<P, std::void_t<decltype(P::KGATHER)>> : std::bool_constant<P::KGATHER> {};
template <class P, class = void> struct G2Multi : std::false_type {};
template <class P> struct G2Multi<P, std::void_t<decltype(P::MULTI)>> : std::bool_constant<P::MULTI> {};
template <class P, class = void> struct G2Row : std::false_type {};
template <class P> struct G2Row<P, std::void_t<decltype(P::ROW)>> : std::bool_constant<P::ROW> {};
template <class P, class = void> struct G2MultiA : std::false_type {};
template <class P> struct G2MultiA<P, std::void_t<decltype(P::MULTI_A)>> : std::bool_constant<P::MULTI_A> {};
template <class P, class = void> struct G2Interleave : std::false_type {};
template <class P>
struct G2Interleave<P, std::void_t<decltype(P::A_INTERLEAVE)>> : std::bool_constant<P::A_INTERLEAVE> {};
template <class P, class = void> struct G2MinWaves : std::integral_constant<int, 1> {};
template <class P>
struct G2MinWaves<P, std::void_t<decltype(P::MIN_WAVES)>> : std::integral_constant<int, P::MIN_WAVES> {};
// CHUNK_ADD: every MFMA (32 k) starts from a zero accumulator and is added to
// the running sum with one fp32 add per element (a summation whose error
// bound does not depend on the MFMA's internal accumulation).
template <class P, class = void> struct G2ChunkAdd : std::false_type {};
template <class P> struct G2ChunkAdd<P, std::void_t<decltype(P::CHUNK_ADD)>> : std::bool_constant<P::CHUNK_ADD> {};
template <class P, class = void> struct G2AHook : std::false_type {};
template <class P> struct G2AHook<P, std::void_t<decltype(&P::a_tile_hook)>> : std::true_type {};
template <class P, class = void> struct G2EpiRegs : std::false_type {};
template <class P> struct G2EpiRegs<P, std::void_t<decltype(P::EPI_REGS)>> : std::bool_constant<P::EPI_REGS> {};

template <class P, class = void> struct G2EpiAcc : std::false_type {};
template <class P> struct G2EpiAcc<P, std::void_t<decltype(P::EPI_ACC)>> : std::bool_constant<P::EPI_ACC> {};

// a_koff(args, batch, c) / b_koff(args, batch, c): element offset of k chunk c
// from chunk 0 (k-contiguous operands whose k axis is made of segments, e.g.
// heads, that are not adjacent in memory; the policy keeps KC within one
// segment).  Default: c * KC (times the k-stride of an m-contiguous operand).
template <class P, class = void> struct G2AKoff : std::false_type {};
template <class P>
struct G2AKoff<P, std::void_t<decltype(P::a_koff(std::declval<const typename P::Args&>(), 0, 0))>> : std::true_type {};
template <class P, class = void> struct G2BKoff : std::false_type {};
template <class P>
struct G2BKoff<P, std::void_t<decltype(P::b_koff(std::declval<const typename P::Args&>(), 0, 0))>> : std::true_type {};

template <class P>
struct Gemm2Shape {
    static constexpr int MT = P::MT, NT = P::NT, KC = P::KC, WM = P::WM, WN = P::WN, STAGES = P::STAGES;
    static constexpr int WTM = MT / WM, WTN = NT / WN, FM = WTM / 16, FN = WTN / 16;
    static constexpr int LPR = KC / 8;  // units per k-contiguous row
    static constexpr int A_UNITS = P::A_KCONTIG ? MT * LPR : KC * (MT / 8);
    static constexpr int B_UNITS = P::B_KCONTIG ? NT * LPR : KC * (NT / 8);
    static constexpr int IA = A_UNITS / 256, IB = B_UNITS / 256;  // instructions per wave per chunk
    static constexpr int A_BYTES = A_UNITS * 16, B_BYTES = B_UNITS * 16;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static_assert(WM * WN == 4 && WTM % 16 == 0 && WTN % 16 == 0 && KC % 32 == 0, "tile shape");
    static_assert(A_UNITS % 256 == 0 && B_UNITS % 256 == 0, "whole instructions per wave");
    static_assert(STAGES >= 2 && (STAGES - 1) * (IA + IB) <= 63, "vmcnt range");
    static constexpr bool KG = G2Gather<P>::value, IL = G2Interleave<P>::value, ER = G2EpiRegs<P>::value;
    static constexpr bool CA = G2ChunkAdd<P>::value;
    static constexpr bool MU = G2Multi<P>::value, ROW = G2Row<P>::value;
    static_assert(!ROW || (MU && WM <= 2 && FN % WM == 0), "row weights");
    static_assert(!MU || (KG && ER), "several tiles need gathered k and the register epilogue");
    static_assert(!KG || (!P::A_KCONTIG && !P::B_KCONTIG), "gathered k needs m-contiguous operands");
    static_assert(!IL || (!P::A_KCONTIG && FM % 2 == 0), "interleaved A needs m-contiguous pairs of blocks");
    static_assert(!ER || IL, "register epilogue needs interleaved A");
    static constexpr size_t ctile_bytes = ER ? 0 : (size_t)MT * (NT + 4) * sizeof(float);
    // LDS bytes; the k-row table of a gathered range (8 bytes per row, with row weights 12, of the
    // padded range) follows the stage buffers.
    static constexpr size_t lds_bytes(int ktab_rows = 0) {
        const size_t ops = (size_t)STAGES * STAGE_BYTES + (KG ? (size_t)ktab_rows * (ROW ? 12 : 8) : 0);
        const size_t epi = ctile_bytes + P::EPI_LDS;
        return ops > epi ? ops : epi;
    }
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N <= 63, "vmcnt");
    // gfx9 s_waitcnt: vmcnt [3:0] and [15:14], expcnt [6:4] = 7, lgkmcnt [11:8] = 15
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Scheduling order of a step with NM MFMAs and NR LDS reads: the reads spread
// evenly over the MFMAs.
template <int NM, int NR, int I = 0>
__device__ __forceinline__ void sched_mix() {
    if constexpr (I < NM) {
        constexpr int R = (NR * (I + 1)) / NM - (NR * I) / NM;
        if constexpr (R > 0) __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        sched_mix<NM, NR, I + 1>();
    }
}

// One workgroup's tile of logical index `logical`.
template <class P>
__device__ __forceinline__ void gemm2_body(const typename P::Args& args, int logical, unsigned char* smem) {
    using ST = uint16_t;
    using S = Gemm2Shape<P>;
    constexpr int MT = S::MT, NT = S::NT, KC = S::KC, LPR = S::LPR, STG = S::STAGES;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, c16 = lane & 15;
    int batch, m0, n0;
    P::tile(args, logical, batch, m0, n0);
    const int K = P::k_size(args, batch);
    const int nchunks = S::KG ? (K + KC - 1) / KC : K / KC;
    // gathered: row offsets of the two operands, and the row weights
    uint32_t* ktab = reinterpret_cast<uint32_t*>(smem + STG * S::STAGE_BYTES);
    float* kf = reinterpret_cast<float*>(ktab + 2 * nchunks * KC);
    if constexpr (S::KG) {
        for (int i = tid; i < nchunks * KC; i += 256) {
            const uint2 e = P::k_row(args, batch, min(i, K - 1));
            ktab[i] = e.x;
            ktab[nchunks * KC + i] = e.y;
            if constexpr (S::ROW) kf[i] = P::k_f(args, batch, i, K);
        }
        __syncthreads();
    }

    // Where this lane's 16 bytes of each load instruction come from for chunk
    // 0, and how far they move per chunk (KC elements along k).  Computed once
    // so that the loop does plain pointer arithmetic.
    const ST* asrc[S::IA > 0 ? S::IA : 1];
    const ST* bsrc[S::IB > 0 ? S::IB : 1];
    int akr[S::IA > 0 ? S::IA : 1], bkr[S::IB > 0 ? S::IB : 1];  // gathered: table index within the first chunk
#pragma unroll
    for (int j = 0; j < S::IA; ++j) {
        const int p = 64 * (wave + 4 * j) + lane;  // unit of the tile
        if constexpr (P::A_KCONTIG) {
            const int r = p / LPR, pos = p % LPR;
            asrc[j] = P::a_elem(args, batch, P::a_row(args, batch, m0 + r), 8 * (pos ^ kswz(r, LPR)));
        } else {
            constexpr int U = MT / 8;
            const int kr = p / U, pos = p % U;
            if constexpr (S::KG) {
                asrc[j] = P::a_mlane(args, batch, m0 + 8 * mswz<U>(kr, pos));
                akr[j] = kr + (P::A_TAB ? nchunks * KC : 0);
            } else {
                asrc[j] = P::a_maddr(args, batch, kr, m0 + 8 * mswz<U>(kr, pos));
            }
        }
    }
#pragma unroll
    for (int j = 0; j < S::IB; ++j) {
        const int p = 64 * (wave + 4 * j) + lane;
        if constexpr (P::B_KCONTIG) {
            const int r = p / LPR, pos = p % LPR;
            bsrc[j] = P::b_elem(args, batch, P::b_row(args, batch, n0 + r), 8 * (pos ^ kswz(r, LPR)));
        } else {
            constexpr int U = NT / 8;
            const int kr = p / U, pos = p % U;
            if constexpr (S::KG) {
                bsrc[j] = P::b_mlane(args, batch, n0 + 8 * mswz<U>(kr, pos));
                bkr[j] = kr + (P::B_TAB ? nchunks * KC : 0);
            } else {
                bsrc[j] = P::b_maddr(args, batch, kr, n0 + 8 * mswz<U>(kr, pos));
            }
        }
    }
    size_t astep = KC, bstep = KC;
    if constexpr (!P::A_KCONTIG && !S::KG) astep *= P::a_kstride(args, batch);
    if constexpr (!P::B_KCONTIG && !S::KG) bstep *= P::b_kstride(args, batch);

    // LDS address of this wave's first 1 KB block of a stage (scalar).
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_addr(smem) + 1024 * wave);

    // Gathered k: this lane's table entries for the next chunk to issue, read
    // one iteration ahead so that the LDS latency stays off the issue path.
    uint32_t arv[S::IA > 0 ? S::IA : 1], brv[S::IB > 0 ? S::IB : 1];
    auto load_rows = [&](int c) {
        if constexpr (S::KG) {
            const int cc = min(c, nchunks - 1) * KC;
#pragma unroll
            for (int j = 0; j < S::IA; ++j) arv[j] = ktab[cc + akr[j]];
#pragma unroll
            for (int j = 0; j < S::IB; ++j) brv[j] = ktab[cc + bkr[j]];
        }
    };
    // 16 bytes of a gathered row
    auto gathered = [](const ST* base, uint32_t off16) {
        return reinterpret_cast<const unsigned char*>(base) + ((size_t)off16 << 4);
    };
    // Several tiles: chunks of all of them (`total`); the chunk within its tile
    // and the operand column offset of the next chunk to be issued.
    int total = nchunks, ichunk = 0, ishift = 0;
    if constexpr (S::MU) total = nchunks * P::tiles(args, logical);

    // Issue the loads of chunk c into its stage buffer (chunks past the end
    // load valid, clamped addresses into a buffer nobody reads).  Gathered k:
    // the table entries of chunk c must be in arv / brv (load_rows(c)).
    auto issue_buf = [&](int c, int bidx) {
        const uint32_t buf = lds_wave + bidx * S::STAGE_BYTES;
        const size_t kc = (size_t)min(c, nchunks - 1);
        ptrdiff_t aoff = 0, boff = 0;
        if constexpr (!S::KG) {
            if constexpr (G2AKoff<P>::value) aoff = P::a_koff(args, batch, (int)kc);
            else aoff = (ptrdiff_t)(kc * astep);
            if constexpr (G2BKoff<P>::value) boff = P::b_koff(args, batch, (int)kc);
            else boff = (ptrdiff_t)(kc * bstep);
        }
#pragma unroll
        for (int j = 0; j < S::IA; ++j) {
            if constexpr (S::MU && G2MultiA<P>::value) lds_load16(gathered(asrc[j] + ishift, arv[j]), buf + 4096 * j);
            else if constexpr (S::KG) lds_load16(gathered(asrc[j], arv[j]), buf + 4096 * j);
            else lds_load16(asrc[j] + aoff, buf + 4096 * j);
        }
#pragma unroll
        for (int j = 0; j < S::IB; ++j) {
            if constexpr (S::MU && !G2MultiA<P>::value)
                lds_load16(gathered(bsrc[j] + ishift, brv[j]), buf + S::A_BYTES + 4096 * j);
            else if constexpr (S::KG) lds_load16(gathered(bsrc[j], brv[j]), buf + S::A_BYTES + 4096 * j);
            else lds_load16(bsrc[j] + boff, buf + S::A_BYTES + 4096 * j);
        }
    };

    const int wm = wave / S::WN, wn = wave % S::WN;
    double hook_state = 0.0;
    f32x4 acc[S::FM][S::FN];
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j) acc[i][j] = zero4();

    // Fragment of 8 consecutive k at ks + 8g for operand row `row` (the
    // MFMA's M or N index) from a stage buffer.
    auto frag_k = [&](const unsigned char* t, int row, int ks) {
        const int s = (ks >> 3) + g;
        Frag8<ST> f;
        f.v = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(t + (row * LPR + (s ^ kswz(row, LPR))) * 16));
        return f;
    };
    // m-contiguous fragment: two transposed reads (colstep 8 and odd: the
    // interleaved pairs of A_INTERLEAVE)
    auto frag_m = [&](const unsigned char* t, int mbase, int ks, auto u_tag, int colstep = 4, int odd = 0) {
        constexpr int U = decltype(u_tag)::value;
        const int mcol = mbase + colstep * (c16 & 3) + 4 * odd;
        const int u = mcol >> 3, half = (mcol >> 2) & 1;
        const int k0r = ks + 8 * g + (c16 >> 2);
        const u32x2 lo = lds_tr16(t + (k0r * U + mswz<U>(k0r, u)) * 16 + 8 * half);
        const int k1r = k0r + 4;
        const u32x2 hi = lds_tr16(t + (k1r * U + mswz<U>(k1r, u)) * 16 + 8 * half);
        Frag8<ST> f;
        f.v = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
        return f;
    };
    // Operand fragments of one 32-k step.
    struct Frags {
        Frag8<ST> a[S::FM], b[S::FN];
    };
    auto load_frags = [&](Frags& f, int bidx, int ks) {
        const unsigned char* ta = smem + bidx * S::STAGE_BYTES;
        const unsigned char* tb = ta + S::A_BYTES;
#pragma unroll
        for (int j = 0; j < S::FN; ++j) {
            if constexpr (P::B_KCONTIG) f.b[j] = frag_k(tb, wn * S::WTN + j * 16 + c16, ks);
            else f.b[j] = frag_m(tb, wn * S::WTN + j * 16, ks, std::integral_constant<int, NT / 8>{});
        }
#pragma unroll
        for (int i = 0; i < S::FM; ++i) {
            if constexpr (P::A_KCONTIG) f.a[i] = frag_k(ta, wm * S::WTM + i * 16 + c16, ks);
            else if constexpr (S::IL)
                f.a[i] = frag_m(ta, wm * S::WTM + 32 * (i >> 1), ks, std::integral_constant<int, MT / 8>{}, 8, i & 1);
            else f.a[i] = frag_m(ta, wm * S::WTM + i * 16, ks, std::integral_constant<int, MT / 8>{});
        }
    };
    // several tiles: chunk of the tile being multiplied, chunks since a tile was stored
    int cchunk = 0, since = STG;
    constexpr int RB = S::ROW ? S::FN / S::WM : 1;  // row product: column blocks RB wm .. of this wave
    float rsum[RB] = {};
    auto mfma_step = [&](const Frags& f, int ks) {
        if constexpr (S::ROW) {
            const float4* z = reinterpret_cast<const float4*>(kf + cchunk * KC + ks + 8 * g);
            const float4 z0 = z[0], z1 = z[1];
            const float zv[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                float x[8];
                frag8_to_f32<ST>(S::WM == 2 && wm ? f.b[(S::WM - 1) * RB + j] : f.b[j], x);
#pragma unroll
                for (int e = 0; e < 8; ++e) rsum[j] = fmaf(zv[e], x[e], rsum[j]);
            }
        }
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
#pragma unroll
            for (int j = 0; j < S::FN; ++j) {
                if constexpr (S::CA) {
                    f32x4 part = zero4();
                    mma8(part, f.a[i], f.b[j]);
                    acc[i][j] += part;
                } else {
                    mma8(acc[i][j], f.a[i], f.b[j]);
                }
            }
    };

    // Pipeline.  STAGES - 1 chunks are in flight from global memory to LDS, and
    // the fragments of the next 32-k step are read from LDS into a second
    // register set while the MFMAs of the current step run, so that neither
    // the LDS reads nor their latency add to the MFMA time (with one wave per
    // SIMD nothing else would hide them).  Measured against reads and MFMAs in
    // turn: the grouped backward of 128 heads, 256 rows each, d = 1024 85.4 ->
    // 80.9 us, of 27 heads, 2048 rows each, d = 1280 148 -> 139 us.  At the last step of chunk c: wait
    // for chunk c + 1, one barrier (every wave has then read all of chunk c),
    // the loads of chunk c + STAGES into c's buffer, the reads of chunk c + 1's
    // first step, the MFMAs.  Every wave issues exactly IA + IB loads per chunk,
    // so the wait counts are constants; chunks past the end are not loaded, and
    // the last STAGES - 2 waits are for everything.  An empty K range (no dense
    // heads) issues nothing.
    // The loop is unrolled so that every stage buffer has a constant LDS offset
    // and every register set a constant name.  The last step reads the
    // fragments of a chunk that does not exist (stale, never used), so that the
    // only way out is after MFMAs that always run, through mfma_drain(): the
    // compiler misses the MFMA result hazard on loop-exit edges, where it moves
    // the accumulators to other registers.
    constexpr int KS = KC / 32, L = S::IA + S::IB;
    constexpr int UNROLL = STG * KS % 2 == 0 ? STG : 2 * STG;
    // The table rows of the chunk after the one just issued (c): the next
    // chunk, or with several tiles the first one of the next tile.
    auto next_rows = [&](int c) {
        if constexpr (S::MU) {
            if (++ichunk == nchunks) {
                ichunk = 0;
                ishift += G2MultiA<P>::value ? MT : NT;
            }
            load_rows(ichunk);
        } else {
            load_rows(c + 1);
        }
    };
    // Register epilogue of one tile (lane: M indices 32 p + 8 g .. + 7 of the
    // wave's rows, column c16 of block j).
    auto store_tile = [&](int mt0, int nt0) {
        if constexpr (S::ER && !G2EpiAcc<P>::value) {
#pragma unroll
            for (int p = 0; p < S::FM / 2; ++p)
#pragma unroll
                for (int j = 0; j < S::FN; ++j) {
                    float x[8];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        x[r] = acc[2 * p][j][r];
                        x[4 + r] = acc[2 * p + 1][j][r];
                    }
                    P::store8(args, batch, mt0 + wm * S::WTM + 32 * p + 8 * g, nt0 + wn * S::WTN + 16 * j + c16, x);
                }
        }
    };
    // Gathered, K not a multiple of KC: chunk `cit` of a tile (0 .. nchunks - 1) has
    // landed in stage buffer bidx; clears the rows past K of the last one.
    auto clear_tail = [&](int cit, int bidx) {
        if constexpr (S::KG) {
            const int v = K - cit * KC;  // rows of the chunk that exist
            if (v >= KC) return;
            unsigned char* ta = smem + bidx * S::STAGE_BYTES;
            for (int i = v * (MT / 8) + tid; i < KC * (MT / 8); i += 256)
                *reinterpret_cast<uint4*>(ta + 16 * i) = make_uint4(0, 0, 0, 0);
            for (int i = v * (NT / 8) + tid; i < KC * (NT / 8); i += 256)
                *reinterpret_cast<uint4*>(ta + S::A_BYTES + 16 * i) = make_uint4(0, 0, 0, 0);
            __syncthreads();
        }
    };
    if (total > 0) {
        Frags fr[2];
        load_rows(0);
#pragma unroll
        for (int s = 0; s < STG; ++s) {
            if (s < total) {
                issue_buf(s, s);
                next_rows(s);
            }
        }
        if (total >= STG) wait_vmcnt<(STG - 1) * L>();
        else wait_vmcnt<0>();
        __syncthreads();
        clear_tail(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_frags(fr[0], 0, 0);
        for (int c0 = 0;; c0 += UNROLL) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int c = c0 + u;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int cur = (u * KS + ks) & 1;
                    if (ks + 1 < KS) {
                        load_frags(fr[cur ^ 1], u % STG, 32 * (ks + 1));
                    } else {
                        if constexpr (G2AHook<P>::value)
                            P::a_tile_hook(args, m0, n0, smem + (u % STG) * S::STAGE_BYTES, tid, hook_state);
                        if constexpr (S::MU) {
                            // a tile stored within the last STAGES - 1 chunks: its
                            // stores are younger than the loads of chunk c + 1
                            if (c + STG > total) wait_vmcnt<0>();
                            else if (++since < STG) wait_vmcnt<(STG - 2) * L + P::STORES>();
                            else wait_vmcnt<(STG - 2) * L>();
                        } else {
                            if (c + STG <= total) wait_vmcnt<(STG - 2) * L>();
                            else wait_vmcnt<0>();
                        }
                        __syncthreads();
                        if (c + STG < total) {
                            issue_buf(c + STG, u % STG);
                            next_rows(c + STG);
                        }
                        if constexpr (S::KG) {
                            const int nx = S::MU ? cchunk + 1 : c + 1;  // chunk c + 1 within its tile
                            clear_tail(nx == nchunks ? 0 : nx, (u + 1) % STG);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        load_frags(fr[cur ^ 1], (u + 1) % STG, 0);
                    }
                    mfma_step(fr[cur], 32 * ks);
                    sched_mix<S::FM * S::FN, (P::A_KCONTIG ? 1 : 2) * S::FM + (P::B_KCONTIG ? 1 : 2) * S::FN>();
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (S::MU) {
                    if (++cchunk == nchunks) {
                        cchunk = since = 0;
                        mfma_drain();
                        store_tile(m0, n0);
                        if constexpr (S::ROW) {
#pragma unroll
                            for (int j = 0; j < RB; ++j) {
                                const float v = rows4_sum(rsum[j]);  // the four k groups
                                if (g == 0) P::store_row(args, batch, n0 + wn * S::WTN + 16 * (RB * wm + j) + c16, v);
                                rsum[j] = 0.f;
                            }
                        }
                        if constexpr (G2MultiA<P>::value) m0 += MT;
                        else n0 += NT;
#pragma unroll
                        for (int i = 0; i < S::FM; ++i)
#pragma unroll
                            for (int j = 0; j < S::FN; ++j) acc[i][j] = zero4();
                    }
                }
                if (c + 1 == total) {
                    mfma_drain();
                    goto pipeline_done;
                }
            }
        }
    }
pipeline_done:
    if constexpr (G2AHook<P>::value) P::a_hook_done(args, m0, n0, tid, hook_state);
    wait_vmcnt<0>();  // the trailing loads write into the buffers the C tile reuses
    if constexpr (G2EpiAcc<P>::value) {
        static_assert(S::ER, "accumulator epilogue needs EPI_REGS");
        __syncthreads();
        P::template epi_acc<S>(args, batch, m0, n0, acc, wm, wn, tid, smem);
    } else if constexpr (S::ER) {
        if constexpr (!S::MU) store_tile(m0, n0);
    } else {
        __syncthreads();

        // C tile to LDS: Cs[m][n], row stride NT + 4 floats
        float* Cs = reinterpret_cast<float*>(smem);
        constexpr int LDC = NT + 4;
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
#pragma unroll
            for (int j = 0; j < S::FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    Cs[(wm * S::WTM + i * 16 + 4 * g + r) * LDC + wn * S::WTN + j * 16 + c16] = acc[i][j][r];
        __syncthreads();
        P::epilogue(args, batch, m0, n0, Cs, LDC, tid, smem + S::ctile_bytes);
    }
}

template <class P>
__global__ __launch_bounds__(256, G2MinWaves<P>::value) void gemm2_kernel(const typename P::Args args) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    gemm2_body<P>(args, xcd_logical_id(blockIdx.x, gridDim.x), smem);
}

// Two independent GEMMs in one launch (n1 workgroups of P1, the rest P2),
// mixed on every XCD so that both kinds share its CUs: the blocks an XCD
// receives (every eighth) are its share of P1 first, in index order, then
// its share of P2.
__device__ __forceinline__ void xcd_dual_id(int b, int nb, int n1, int& which, int& idx) {
    const int x = b % 8, j = b / 8;
    const int q = nb / 8, r = nb % 8, q1 = n1 / 8, r1 = n1 % 8;
    const int cnt1 = q1 + (x < r1 ? 1 : 0);
    const int s1 = x * q1 + (x < r1 ? x : r1);                // P1 blocks on lower XCDs
    const int sall = x * q + (x < r ? x : r);                // all blocks on lower XCDs
    if (j < cnt1) {
        which = 0;
        idx = s1 + j;
    } else {
        which = 1;
        idx = (sall - s1) + (j - cnt1);
    }
}

template <class P1, class P2>
__global__ __launch_bounds__(256, (G2MinWaves<P1>::value > G2MinWaves<P2>::value ? G2MinWaves<P1>::value
                                                                                  : G2MinWaves<P2>::value))
void gemm2_dual_kernel(const typename P1::Args a1, const typename P2::Args a2, int n1) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int which, idx;
    xcd_dual_id(blockIdx.x, gridDim.x, n1, which, idx);
    if (which == 0) gemm2_body<P1>(a1, idx, smem);
    else gemm2_body<P2>(a2, idx, smem);
}

// ktab_rows: rows of the k-row table (gathered k: the padded k range).
template <class P>
int launch_gemm2(const typename P::Args& args, int nblocks, hipStream_t stream, int ktab_rows = 0) {
    if (nblocks <= 0) return 0;
    const size_t lds = Gemm2Shape<P>::lds_bytes(ktab_rows);
    if (lds > 160 * 1024) return -1;
    auto kern = gemm2_kernel<P>;
    if (allow_lds((const void*)kern, lds)) return -1;
    hipLaunchKernelGGL(kern, dim3(nblocks), dim3(256), lds, stream, args);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Both GEMMs in one launch (see gemm2_dual_kernel); requires every XCD's
// share of the blocks to hold its share of P1.
template <class P1, class P2>
int launch_gemm2_dual(const typename P1::Args& a1, int n1, int rows1, const typename P2::Args& a2, int n2, int rows2,
                      hipStream_t stream) {
    if (n1 <= 0) return launch_gemm2<P2>(a2, n2, stream, rows2);
    if (n2 <= 0) return launch_gemm2<P1>(a1, n1, stream, rows1);
    const size_t l1 = Gemm2Shape<P1>::lds_bytes(rows1), l2 = Gemm2Shape<P2>::lds_bytes(rows2);
    const size_t lds = l1 > l2 ? l1 : l2;
    if (lds > 160 * 1024) return -1;
    const int nb = n1 + n2;
    for (int x = 0; x < 8; ++x)  // xcd_dual_id's assumption
        if (nb / 8 + (x < nb % 8 ? 1 : 0) < n1 / 8 + (x < n1 % 8 ? 1 : 0)) return -1;
    auto kern = gemm2_dual_kernel<P1, P2>;
    if (allow_lds((const void*)kern, lds)) return -1;
    hipLaunchKernelGGL(kern, dim3(nb), dim3(256), lds, stream, a1, a2, n1);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace mosa
