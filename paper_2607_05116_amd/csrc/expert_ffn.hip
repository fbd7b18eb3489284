// Grouped SwiGLU expert FFN over one rank's experts (Eq. 1, Expert_i(x); the
// experts are SwiGLU FFNs: y = W2 (silu(W1 x) * (W3 x))).
//
// Two grouped GEMMs per call over the ragged experts (row offsets are read on
// the device):
//   gate/up   H[m][j] = silu(X W1^T)[m][j] * (X W3^T)[m][j]   (K = d)
//   down      Y[m][o] = (H W2^T)[m][o]                         (K = inter)
//
// bf16 path (gfx950 MFMA v_mfma_f32_16x16x32_bf16, fp32 accumulation):
//   * Block tile 256 x 256, eight waves (two per SIMD) of 64 x 128 each.
//   * Operands are both K-contiguous (token rows of X / H; weight rows of W).
//     gfx950 direct-to-LDS loads (global_load_lds_dwordx4) fill a double
//     buffer of K = 64 stages: every operand row of a stage is one whole
//     128-byte line, which the direct-to-LDS path moves at about twice the
//     rate of half lines.  A stage is loaded in parts, each issued as soon as
//     the space it takes has been read by every wave (two barriers per stage),
//     so a load has about a stage and a quarter to land.
//   * Half of the waves issue all the direct loads and the other half all the
//     output stores, so no wave's in-order memory counter mixes the two (a
//     wait for a stage never waits for a tile's worth of stores to drain).
//   * Each wave reads its LDS fragments a quarter of a stage ahead of its MFMAs
//     (16 x 16 x 32 MFMAs: half the accumulator reads and writes per flop of
//     the 32 x 32 x 16 form, measured 3-4 % faster on whole calls).
//   * Calls of many rows' capacity run both GEMMs in one persistent kernel with
//     a tile queue per XCD (ffn_fused_bf16_kernel); others run one persistent
//     kernel per GEMM (ffn_gemm_bf16_kernel).  In either, a call whose experts
//     turn out to hold few rows each runs on narrow tiles (narrow_gemm).  Every
//     output element takes the same arithmetic in all of them, so they give
//     identical bits.
//   * Optionally (a combine plan) the down GEMM's epilogue writes the rows of
//     tokens with a single kept expert on the rank, scaled by their gate
//     weight, into the receive-side buffer instead of Y (Sec. II-C local
//     aggregation of a one-term sum).
// fp32 path: fp32 matrix instructions straight from global memory (small shapes).
#include "cap_device.hpp"

#include <type_traits>

namespace cap {
namespace {

constexpr int kMaxExpertsLocal = kMaxE;

// Compile-time loop: f(std::integral_constant<int, 0>) ... f(<N - 1>).
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// ------------------------------------------------------------------ tile scheduler
// Row bounds of every expert.
__device__ __forceinline__ void expert_rows(const int32_t* row_offsets, int E_loc, int max_rows, int* row_begin,
                                            int* row_end) {
    const int base = row_offsets[0];
    for (int l = threadIdx.x; l < E_loc; l += blockDim.x) {
        int b = row_offsets[l] - base, e = row_offsets[l + 1] - base;
        b = max(0, min(b, max_rows));
        e = max(b, min(e, max_rows));
        row_begin[l] = b;
        row_end[l] = e;
    }
}

// Fills mt_prefix[0..E_loc] (m-tiles before each expert) from this thread's own
// expert_rows; ends in a barrier.
template <int BM>
__device__ void build_schedule(int E_loc, int* mt_prefix, const int* row_begin, const int* row_end) {
    for (int l = threadIdx.x; l < E_loc; l += blockDim.x) mt_prefix[l + 1] = (row_end[l] - row_begin[l] + BM - 1) / BM;
    if (threadIdx.x == 0) mt_prefix[0] = 0;
    __syncthreads();
    for (int off = 1; off < E_loc; off <<= 1) {
        int v = 0;
        const int i = threadIdx.x + 1;
        if (i <= E_loc && i > off) v = mt_prefix[i - off];
        __syncthreads();
        if (i <= E_loc) mt_prefix[i] += v;
        __syncthreads();
    }
}

__device__ __forceinline__ int find_expert(const int* mt_prefix, int E_loc, int m_tile) {
    int lo = 0, hi = E_loc - 1;           // largest l with mt_prefix[l] <= m_tile
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (mt_prefix[mid] <= m_tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Workgroups that take part in `total` tiles (a whole round of XCDs more than
// the tiles at most: the rest of the grid has nothing to do), and this one's
// place among them, or -1.  Block b runs on XCD b % 8, so each XCD gets a
// contiguous run of places, and few tiles spread over all XCDs.
__device__ __forceinline__ int worker_count(int total) { return min(static_cast<int>(gridDim.x), (total + 7) & ~7); }
__device__ __forceinline__ int worker_id(int G) {
    const int b = blockIdx.x;
    if (b >= G) return -1;
    return (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
}

// silu(g) = g * sigmoid(g); hardware exp2 and reciprocal (about 1 ulp each),
// far inside the bf16 rounding that H then takes.
__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Scalar base of a direct load: uniform by construction; readfirstlane keeps it
// in scalar registers (widening through uint32_t so the low word is never
// sign-extended).
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b)));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32)));
    return reinterpret_cast<const void*>((hi << 32) | lo);
}

// Wave-wide copies global -> LDS (gfx950 global_load_lds_dwordx4): lane i
// reads 16 bytes at base + voff_i and they land at LDS byte M0 + 16 * i; base
// is a scalar register pair, voff a 32-bit per-lane byte offset, and the
// instruction's immediate offset stays 0 (it would shift the LDS address too).
// They are inline assembly so that the compiler's wait-count pass does not
// treat every later LDS read as aliasing them (it would drain all in-flight
// stages); the kernel waits on them explicitly.  Because the compiler does not
// see the instruction, it also does not insert the wait states the hardware
// needs before it: a VALU write of an SGPR (v_readfirstlane of the base, or a
// reload of a spilled scalar) needs 5 wait states before a vector-memory
// instruction reads it, and an SALU write of M0 needs 1 before an LDS DMA.  The
// statement copies the base with s_mov_b64, which waits for the VALU write by
// itself, is no hazard for the load, and separates it from the M0 write: 3
// issue slots, where an s_nop 4 took 7.
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t off, uint32_t lds_addr) {
    uint64_t b;
    asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(b)
                 : "v"(off), "s"(uniform_ptr(base)), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr))
                 : "memory");
}

// ------------------------------------------------------------------ bf16 MFMA GEMM
// LDS holds kStages stages; a stage is the A tile [BM][64] and the B tile
// [BN][64] (bf16, 128-byte rows).  A stage row is one whole 128-byte line of
// the K-contiguous operand: the direct-to-LDS path moves full lines at about
// twice the rate of half lines, which is what sets the stage depth to K = 64.
// 16-byte chunk c of row r sits at physical chunk c ^ lds_swz(r); fragment
// reads (16 consecutive rows, one chunk) then hit distinct banks for both 128-
// and 256-byte bank windows.
constexpr int kStageK = 64;                 // K per stage
constexpr int kStages = 2;                  // stage kt lives in buffer kt % 2
constexpr int kRowB = kStageK * 2;          // bytes per LDS row
constexpr int kChunks = kRowB / 16;         // 16-byte chunks per row

__device__ __forceinline__ int lds_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Workgroup barrier without the memory fence that __syncthreads() carries (the
// fence would drain every in-flight prefetch).  LDS visibility is ensured by
// explicit waits: vmcnt for the direct-to-LDS loads, and lgkmcnt(0) before a
// barrier that publishes ds_write data (staged outputs, broadcast values); the
// empty asm statements keep memory accesses from being moved across the
// barrier.
__device__ __forceinline__ void block_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(3))) void lds_void;


// ------------------------------------------------------------------ shared tile pieces
// Block tile 256 x 256, eight waves in a 4 x 2 grid, each wave 64 x 128.
constexpr int kBM = 256, kBN = 256, kWavesM = 4, kWavesN = 2;
constexpr int kNW = kWavesM * kWavesN;
constexpr int kNL = kNW / 2;                          // loader waves; the rest are storers
constexpr int kWM = kBM / kWavesM, kWN = kBN / kWavesN;
constexpr int kMI = kWM / 16, kNJ = kWN / 16;         // 16 x 16 MFMA blocks per wave
constexpr int kRowsPerLoad = 1024 / kRowB;            // rows one wave-wide 16-byte load covers
constexpr int kALd = kBM / kRowsPerLoad / kNL;        // direct loads per loader wave per stage
constexpr int kBLd = kBN / kRowsPerLoad / kNL;
constexpr int kStageBytes = (kBM + kBN) * kRowB;
static_assert(kNL % 4 == 0, "one loader and one storer wave per SIMD");
static_assert(kBM % (kRowsPerLoad * kNL) == 0 && kBN % (kRowsPerLoad * kNL) == 0, "load split");
static_assert(kALd + kBLd <= 60, "loads per stage must fit the vmcnt field");
static_assert(kWN % 64 == 0, "gate/up pairs need 64-column wave tiles");
static_assert(kNL == 4 && kBLd == 8 && kRowsPerLoad == 8, "a loader takes 16 rows of each B quarter");
static_assert(kMI == 4 && kNJ == 8, "quarters of two B blocks, A blocks in pairs");
static_assert(kALd * kRowsPerLoad == kWM, "loader wave w loads the A rows that waves of row w read");
static_assert(kStageK == 64, "a stage is two MFMA K steps of 32");
static_assert(kStages == 2, "staging lives in stage buffer 1");

// Per-lane constants of the direct loads and the fragment reads.
struct LaneMap {
    int ld_row;          // direct loads: lane l writes row l / 8 of its 1 KiB block ...
    uint32_t col_b[2];   // ... at physical chunk l % 8, fetching logical chunk (l % 8) ^ swz(row):
                         // the swizzle of row (8 * blk + l / 8) is swz(l / 8) ^ (blk & 1)
    int fr_row, fr_swz, fr_kc;     // fragment reads: row r = ... + lane % 16, K chunk kc(lane / 16)
};
__device__ __forceinline__ LaneMap lane_map(int lane) {
    LaneMap m;
    m.ld_row = lane >> 3;
    const int pc = lane & (kChunks - 1);
    m.col_b[0] = static_cast<uint32_t>((pc ^ lds_swz(m.ld_row)) * 16);
    m.col_b[1] = static_cast<uint32_t>((pc ^ lds_swz(kRowsPerLoad + m.ld_row)) * 16);
    m.fr_row = lane & 15;
    m.fr_swz = lds_swz(m.fr_row);
    // K chunk of lane group g = lane / 16 within a K step: 0, 2, 1, 3, so
    // that lanes l and l + 32 (read in one LDS pass) take chunks of opposite
    // parity and, under the row swizzle, distinct banks
    m.fr_kc = ((lane >> 3) & 2) | (lane >> 5);
    return m;
}

// The same value, opaque to the compiler: what is derived from it is formed
// where it is used, per tile, and not kept in registers across the K loop.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Fragments and MFMAs.  One MFMA K step is K = 32 (two per stage).  Lane
// (r, g) = (lane % 16, lane / 16) reads row r of each 16-row block at 16-byte
// chunk 4 ks + kc(g) of K step ks, kc = (0, 2, 1, 3) (8 consecutive K; A and
// B take the same K positions, so the contraction pairs them correctly
// whatever order the hardware sums them in).  The MFMA takes the weight fragment as its first
// operand, so a lane's 4 accumulators of block (i, j) hold output columns
// 16 j + 4 q + 0..3 of tile row 16 i + r.
__device__ __forceinline__ const bf16x8& frag_at(const uint8_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// Loads of one tile for one loader wave.  A: rows wave * 64 .. + 63, 8 loads a
// stage (lane l of load i: byte offset a_off[i] from the operand base: a tile
// row, clamped to the expert's last, or a gathered row of x), none of them by
// a loader whose own wave computes nothing (a_on: wave row w / 2 has rows; the
// rows 64 w .. it loads come after those).  B: of quarter q
// (rows wn * 128 + 32 q .. + 31 of both wave columns wn) the 16 rows wn =
// wave / 2, 16 (wave % 2) ..: 2 loads a quarter.  The pointers run along K:
// a and b0 / b1 (quarters 0, 1) one stage ahead of c0 / c1 (quarters 2, 3).
struct Loads {
    const char *a, *b0, *b1, *c0, *c1;
    uint32_t a_off[kALd];
    uint32_t b_off[2];
    bool a_on;
};

template <int I>
__device__ __forceinline__ void load_a(const Loads& s, uint32_t a_lds, int buf) {
    lds_dma16(s.a, s.a_off[I], a_lds + buf * kStageBytes + I * 1024);
}
// load I = 0..3 of quarters 0, 1 (half 0) or 2, 3 (half 1)
template <int HALF, int I>
__device__ __forceinline__ void load_b(const Loads& s, uint32_t b_lds, int buf) {
    const char* p = HALF ? (I / 2 ? s.c1 : s.c0) : (I / 2 ? s.b1 : s.b0);
    lds_dma16(p, s.b_off[I % 2],
              b_lds + buf * kStageBytes + (HALF * 64 + (I / 2) * 32 + (I % 2) * kRowsPerLoad) * kRowB);
}
__device__ __forceinline__ void step_half0(Loads& s) { s.a += kRowB; s.b0 += kRowB; s.b1 += kRowB; }
__device__ __forceinline__ void step_half1(Loads& s) { s.c0 += kRowB; s.c1 += kRowB; }
__device__ __forceinline__ void load_half0(Loads& s, bool a_on, uint32_t a_lds, uint32_t b_lds, int buf) {
    if (a_on) static_for<kALd>([&](auto I) { load_a<I.value>(s, a_lds, buf); });
    static_for<4>([&](auto I) { load_b<0, I.value>(s, b_lds, buf); });
    step_half0(s);
}
__device__ __forceinline__ void load_half1(Loads& s, uint32_t b_lds, int buf) {
    static_for<4>([&](auto I) { load_b<1, I.value>(s, b_lds, buf); });
    step_half1(s);
}

// The K loop of one tile: KT stages of K = 64 (KT is even: d % 256 == 0 and
// inter % 128 == 0), stage kt in buffer kt % 2.  A stage is computed in four
// quarters (Q = 0..3: all A blocks with B blocks 2 Q, 2 Q + 1), and each
// quarter's B fragments are read during the quarter before it (two register
// sets in turn).  The A fragments of the next stage replace this one's in
// place: blocks 0, 1 after their last MFMA in quarter 3, blocks 2, 3 at the
// start of the next quarter 0.  So a part of a stage stays in LDS only while
// one or two quarters read it, and its space takes the loads of the stage two
// ahead from then on:
//   barrier a (after quarter 0):  A and B quarters 0, 1 of stage kt are read;
//                                 B quarters 2, 3 of stage kt are complete.
//   barrier c (after quarter 2):  B quarters 2, 3 of stage kt are read; A and
//                                 B quarters 0, 1 of stage kt + 1 are complete.
// A quarter is four groups of four MFMAs; a group starts with its fragment
// reads and ends, in a loader wave, with its direct loads, spread so that the
// address path takes them while the MFMAs run: A of stage kt + 2 in quarters
// 1, 2, its B quarters 0, 1 in quarter 3, its B quarters 2, 3 in quarter 0 of
// stage kt + 1.
//   hook(step)       bookkeeping of the caller, none of it in the middle of the
//                    loop: after barrier a of the first (kFirst) and second
//                    stage (kSecond; both only if KT > 2), of the last but one
//                    (kLast2), before (kPreLast) and after (kLast) that of the
//                    last.
// On entry stage 0 has been issued whole; on return every wave is past its
// last LDS read of the tile (barrier c of the last stage), and buffer 0 was
// free from barrier a of the last stage (the hook may issue the next tile's
// stage 0).
// What bounds it: the board's power (under the counters the MFMA pipes are 73 %
// busy at 1.7 GHz on the 33,234 rows of d = 7168, inter = 2048, where loading
// each stage whole behind one barrier kept them 62 % busy at 1.8 GHz), then the
// LDS, whose fragment reads and direct writes need 256 KB a stage, the time of
// its MFMAs at 128 bytes a clock; on tiles of few stages (a down tile of inter =
// 768 has twelve) also the next tile's stage 1, which cannot be issued before
// the epilogue has given its buffer back.  That call 2328 -> 2131 us, 44,420
// rows of d = 2048, inter = 768 393 -> 358 us, 3,001 rows of d = 2048, inter =
// 1408 98 -> 89 us.  Issuing twelve of a stage's sixteen loads in quarters 1 and
// 2 was no faster, nor a raised wave priority around the MFMAs or for the
// loaders (0 to 2 % slower).
// A wave whose 64 rows all lie past the tile's valid rows (active = false)
// computes nothing: its accumulators stay zero and are never stored.  A loader
// among them loads no A either, and its waits count without those loads: tiles
// of 64 rows or fewer then bring 16 KB of A a stage instead of 32.  (A third
// form of the loop for the loaders of which only the rows they load lie past
// the end was 1 to 4 % slower on 300 rows an expert of d = 7168.)
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// acc += b a^T in place, as inline assembly: with most of the registers taken,
// the register allocator otherwise moves accumulators about (24 spilled
// registers and copies at every tile's end; 2172 -> 2131 us on the 33,234 rows
// of d = 7168, inter = 2048, 372 -> 358 us on 44,420 rows of d = 2048, inter =
// 768).  The compiler inserts no wait states around it: acc_pin and the s_nop
// before and after the K loop separate the MFMAs from the code that writes and
// reads the accumulators; fragment operands come from LDS reads, whose wait it
// does insert.
__device__ __forceinline__ void mfma_acc(f32x4& acc, const bf16x8& b, const bf16x8& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(b), "v"(a));
}
__device__ __forceinline__ void acc_pin(f32x4 (&acc)[kMI][kNJ]) {
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int j = 0; j < kNJ; ++j) asm volatile("" : "+v"(acc[i][j]));
}
enum KStep { kMiddle, kFirst, kSecond, kLast2, kPreLast, kLast };

template <bool LOADER, bool ACTIVE, typename Hook>
__device__ __forceinline__ void k_loop(int KT, const uint8_t* lds, int wm, int wn, int lane, f32x4 (&acc)[kMI][kNJ], Loads& ld, uint32_t a_lds, uint32_t b_lds,
                                       Hook&& hook) {
    constexpr bool LOAD_A = LOADER && ACTIVE;
    constexpr int kA = LOAD_A ? kALd : 0;              // this wave's A loads of a stage
    bf16x8 a[kMI][2], b0[2][2], b1[2][2];
    const LaneMap lm = lane_map(opaque(lane));
    const int pc0 = (lm.fr_kc ^ lm.fr_swz) << 4, pc1 = pc0 ^ 64;
    const uint8_t* const la = lds + (wm * kWM + lm.fr_row) * kRowB;
    const uint8_t* const lb = lds + (kBM + wn * kWN + lm.fr_row) * kRowB;
    // fragment n = 0..3 of A blocks i0, i0 + 1 / of quarter q: K step n / 2
    auto read_a = [&](int buf, int i0, auto Nn) {
        constexpr int n = decltype(Nn)::value;
        a[i0 + n % 2][n / 2] = frag_at(la + buf * kStageBytes + (i0 + n % 2) * 16 * kRowB + (n / 2 ? pc1 : pc0));
    };
    auto read_b = [&](bf16x8 (&b)[2][2], int buf, int q, auto Nn) {
        constexpr int n = decltype(Nn)::value;
        b[n % 2][n / 2] = frag_at(lb + buf * kStageBytes + (2 * q + n % 2) * 16 * kRowB + (n / 2 ? pc1 : pc0));
    };
    // MFMA group g = 0..3 of quarter Q.  Quarters 1, 2: K step g / 2, A blocks
    // 2 (g % 2) ..; quarters 0, 3: A blocks 2 (g / 2) .., K step g % 2 (the A
    // fragments change hands half way).
    auto mfma4 = [&](bf16x8 (&b)[2][2], auto Qn, auto Gn) {
        constexpr int q = decltype(Qn)::value, g = decltype(Gn)::value;
        constexpr bool by_k = q == 1 || q == 2;
        constexpr int ks = by_k ? g / 2 : g % 2, i0 = 2 * (by_k ? g % 2 : g / 2);
#pragma unroll
        for (int i = i0; i < i0 + 2; ++i)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
                mfma_acc(acc[i][2 * q + jj], b[jj][ks], a[i][ks]);
    };
    auto N0 = std::integral_constant<int, 0>{};
    auto N1 = std::integral_constant<int, 1>{};
    auto N2 = std::integral_constant<int, 2>{};
    auto N3 = std::integral_constant<int, 3>{};
    acc_pin(acc);
    asm volatile("s_nop 7");
    if (LOADER) wait_vm<0>();
    block_barrier();                                   // stage 0 visible; buffer 1 free
    if (LOADER) load_half0(ld, LOAD_A, a_lds, b_lds, 1);
    if constexpr (ACTIVE)
        static_for<4>([&](auto N) {
            read_b(b0, 0, 0, N);
            read_a(0, 0, N);
        });
    auto stage = [&](auto BUF, auto STEP) {
        constexpr int buf = decltype(BUF)::value;
        constexpr KStep step = decltype(STEP)::value;
        constexpr bool next1 = step != kLast, next2 = next1 && step != kLast2;   // stages kt + 1, kt + 2 exist
        static_for<4>([&](auto G) {                                            // quarter 0
            if constexpr (ACTIVE) {
                if constexpr (G.value < 2) {
                    read_a(buf, 2, std::integral_constant<int, 2 * G.value>{});
                    read_a(buf, 2, std::integral_constant<int, 2 * G.value + 1>{});
                } else {
                    read_b(b1, buf, 1, std::integral_constant<int, 2 * G.value - 4>{});
                    read_b(b1, buf, 1, std::integral_constant<int, 2 * G.value - 3>{});
                }
                mfma4(b0, N0, G);
            }
            if constexpr (LOADER && next1) load_b<1, G.value>(ld, b_lds, buf ^ 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (LOADER && next1) step_half1(ld);
        if constexpr (step == kLast) hook(std::integral_constant<KStep, kPreLast>{});
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // A, quarters 0 and 1 read
        if constexpr (LOADER) {                                  // quarters 2, 3 of stage kt landed
            wait_vm<next1 ? kA + 8 : 0>();
        }
        block_barrier();                                         // barrier a
        if constexpr (step != kMiddle) hook(STEP);
        static_for<4>([&](auto G) {                                            // quarter 1
            if constexpr (ACTIVE) {
                read_b(b0, buf, 2, G);
                mfma4(b1, N1, G);
            }
            if constexpr (LOAD_A && next2) load_a<G.value>(ld, a_lds, buf);
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<4>([&](auto G) {                                            // quarter 2
            if constexpr (ACTIVE) {
                read_b(b1, buf, 3, G);
                mfma4(b0, N2, G);
            }
            if constexpr (LOAD_A && next2) load_a<4 + G.value>(ld, a_lds, buf);
            __builtin_amdgcn_sched_barrier(0);
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // quarters 2, 3 read
        if constexpr (LOADER && next1) {                         // A, quarters 0, 1 of stage kt + 1 landed
            wait_vm<next2 ? kA + 4 : 4>();
        }
        block_barrier();                                         // barrier c
        static_for<4>([&](auto G) {                                            // quarter 3
            if constexpr (ACTIVE) {
                if constexpr (next1) {
                    if constexpr (G.value < 2) {
                        read_b(b0, buf ^ 1, 0, std::integral_constant<int, 2 * G.value>{});
                        read_b(b0, buf ^ 1, 0, std::integral_constant<int, 2 * G.value + 1>{});
                    } else if constexpr (G.value == 2) {
                        static_for<4>([&](auto N) { read_a(buf ^ 1, 0, N); });
                    }
                }
                mfma4(b1, N3, G);
            }
            if constexpr (LOADER && next2) load_b<0, G.value>(ld, b_lds, buf);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (LOADER && next2) step_half0(ld);
    };
    int kt = 0;
    if constexpr (!LOADER) {
        if (KT > 2) {
            stage(N0, std::integral_constant<KStep, kFirst>{});
            stage(N1, std::integral_constant<KStep, kSecond>{});
            kt = 2;
        }
    }
    for (; kt + 2 < KT; kt += 2) {
        stage(N0, std::integral_constant<KStep, kMiddle>{});
        stage(N1, std::integral_constant<KStep, kMiddle>{});
    }
    stage(N0, std::integral_constant<KStep, kLast2>{});
    stage(N1, std::integral_constant<KStep, kLast>{});
    asm volatile("s_nop 15\n\ts_nop 15");             // the last MFMAs' results are written
    acc_pin(acc);
}

// The four roles of a wave in a tile (wave-uniform): each has a loop of its
// own, all with the same barriers.
template <typename LoadHook, typename StoreHook>
__device__ __forceinline__ void run_k_loop(int KT, const uint8_t* lds, int wm, int wn, int lane,
                                           bool loader, bool active, f32x4 (&acc)[kMI][kNJ], Loads& ld,
                                           uint32_t a_lds, uint32_t b_lds, LoadHook&& load_hook,
                                           StoreHook&& store_hook) {
    if (loader) {
        if (active) k_loop<true, true>(KT, lds, wm, wn, lane, acc, ld, a_lds, b_lds, load_hook);
        else k_loop<true, false>(KT, lds, wm, wn, lane, acc, ld, a_lds, b_lds, load_hook);
    } else {
        if (active) k_loop<false, true>(KT, lds, wm, wn, lane, acc, ld, a_lds, b_lds, store_hook);
        else k_loop<false, false>(KT, lds, wm, wn, lane, acc, ld, a_lds, b_lds, store_hook);
    }
}

// Destination combine folded into the down GEMM's epilogue (Sec. II-C local
// aggregation, Eq. 1): row i of the call whose token has no other kept expert
// on the rank goes to row dst[i] of the receive-side buffer, scaled by its
// gate weight, instead of to Y.  The storer waves load the plan of a down
// tile's rows during its K loop into an LDS table (dst, w per row of the tile).
struct CombinePlan {
    const int32_t* dst;      // [max_rows] receive row, or -1: write Y (nullptr: no combine)
    const float* w;          // [max_rows] gate weight w'
    uint16_t* parts;         // [parts_rows][d] receive-side rows
    int parts_rows;
};

// Two bf16 of a Y row scaled by w the way the destination reduce does it for a
// single term: fp32 fmaf(w, y, 0), then bf16 rounded to nearest even (the
// hardware conversion gives the reduce's bits for finite values); and a 16-byte
// chunk of them.
__device__ __forceinline__ uint32_t scale_pair(uint32_t v, float w) {
    return pack_bf16x2_rne(__builtin_fmaf(w, __uint_as_float(v << 16), 0.0f),
                           __builtin_fmaf(w, __uint_as_float(v & 0xFFFF0000u), 0.0f));
}
__device__ __forceinline__ u32x4 scale_chunk(const u32x4& v, float w) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = scale_pair(v[i], w);
    return o;
}

// Epilogue of a tile of rows [row0, row0 + rows) and block column nt.
// Lane (r, q) = (lane % 16, lane / 16) holds columns 4 q + 0..3 of row r of
// each 16 x 16 block.  For a pair of adjacent blocks (32 output columns) the
// 16-lane rows of the wave swap (permlane16_swap: odd rows of the first
// operand with even rows of the second) so that each lane holds 8 consecutive
// columns: lane (r, q) gets columns 8 (q / 2) + 0..7 of block q % 2 of the
// pair, one 16-byte piece.  Gate/up: the B tile interleaves 32-row blocks of
// W1 and W3, so blocks 4p + {0, 1} and 4p + {2, 3} are the gate and up sums of
// the same 32 outputs; SiLU-and-multiply happens in registers and H is
// rounded to bf16 once.  Loader waves write their pieces to the staging area
// (stage buffer 1), storer waves to the output; after a barrier the storers
// also write the staged rows.  Storers never wait for their stores here.
// Down GEMM with a combine plan (plan_dst != nullptr): a row whose plan entry
// names a receive row in [0, parts_rows) is scaled (by the wave that holds
// its accumulators, before staging) and written there, every other row to
// the output.
template <bool GUP>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[kMI][kNJ], uint16_t* __restrict__ out, int N_out,
                                           int row0, int rows, int nt, int wave, int lane, uint8_t* staging,
                                           const int* plan_dst = nullptr, const float* plan_w = nullptr,
                                           uint16_t* __restrict__ parts = nullptr, int parts_rows = 0) {
    constexpr int OUT_C = GUP ? kWN / 2 : kWN;        // output columns of a wave tile
    constexpr int OUT_RB = OUT_C * 2;                 // bytes per staged output row
    constexpr int OUT_CH = OUT_RB / 16;               // 16-byte chunks per staged row
    constexpr int OUT_RPW = 256 / OUT_RB;             // staged rows per 256-byte bank window
    constexpr int STG_B = kWM * OUT_RB;               // staging bytes per loader wave
    constexpr int NP = OUT_C / 32;                    // 32-column block pairs of a wave's output
    static_assert(kNL * STG_B <= kStageBytes, "staging fits in stage buffer 1");
    static_assert(OUT_RB == 128 || OUT_RB == 256, "staged row layout");
    // staged output rows: 16-byte chunk c of row r at physical chunk
    // c ^ ((r / OUT_RPW) % OUT_CH), conflict-free for column writes (8
    // consecutive rows, one chunk) and row reads
    auto stg_swz = [](int r) { return (r / OUT_RPW) & (OUT_CH - 1); };
    const bool loader = wave < kNL;
    const int wm = wave / kWavesN, wn = wave % kWavesN;
    const int ep_lane = opaque(lane);
    const int ep_row = ep_lane & 15, ep_q = ep_lane >> 4;
    const int ep_c = 2 * (ep_q & 1) + (ep_q >> 1);     // this lane's chunk within a pair's four
    uint8_t* my_stg = staging + (loader ? wave : 0) * STG_B;
    const int out_c0 = (GUP ? nt * (kBN / 2) : nt * kBN) + wn * OUT_C;
#pragma unroll
    for (int i = 0; i < kMI; ++i) {
        if (!loader && wm * kWM + i * 16 >= rows) continue;            // wave-uniform
        const int r = i * 16 + ep_row;                                 // row within the wave tile
        const bool row_ok = wm * kWM + r < rows;
        uint16_t* crow = out + static_cast<size_t>(row0 + wm * kWM + r) * N_out + out_c0;
        int dst = -1;
        float dw = 0.0f;
        if (!GUP && plan_dst && row_ok) {
            dst = plan_dst[wm * kWM + r];
            dw = plan_w[wm * kWM + r];
            if (static_cast<unsigned>(dst) >= static_cast<unsigned>(parts_rows)) dst = -1;
            else if (!loader) crow = parts + static_cast<size_t>(dst) * N_out + out_c0;
        }
#pragma unroll
        for (int pr = 0; pr < NP; ++pr) {
            float v0[4], v1[4];                        // the pair's two output blocks
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (GUP) {
                    v0[e] = silu(acc[i][4 * pr + 0][e]) * acc[i][4 * pr + 2][e];
                    v1[e] = silu(acc[i][4 * pr + 1][e]) * acc[i][4 * pr + 3][e];
                } else {
                    v0[e] = acc[i][2 * pr + 0][e];
                    v1[e] = acc[i][2 * pr + 1][e];
                }
            }
            const uint32_t x0 = pack_bf16x2_rne(v0[0], v0[1]);
            const uint32_t x1 = pack_bf16x2_rne(v0[2], v0[3]);
            const uint32_t y0 = pack_bf16x2_rne(v1[0], v1[1]);
            const uint32_t y1 = pack_bf16x2_rne(v1[2], v1[3]);
            const auto ra = __builtin_amdgcn_permlane16_swap(x0, y0, false, false);
            const auto rb = __builtin_amdgcn_permlane16_swap(x1, y1, false, false);
            u32x4 o;
            o[0] = ra[0]; o[1] = rb[0]; o[2] = ra[1]; o[3] = rb[1];
            const int c = 4 * pr + ep_c;                               // 8-column chunk in the wave tile
            if (dst >= 0) o = scale_chunk(o, dw);
            if (loader) {
                *reinterpret_cast<u32x4*>(my_stg + r * OUT_RB + 16 * (c ^ stg_swz(r))) = o;
            } else if (row_ok) {
                *reinterpret_cast<u32x4*>(crow + 8 * c) = o;
            }
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    block_barrier();                                                   // staging written
    if (!loader) {
        // storer wave w writes the staged tile of loader wave w - kNL
        const int lw = wave - kNL;
        const int lwm = lw / kWavesN, lwn = lw % kWavesN;
        const uint8_t* stg = staging + lw * STG_B;
        const int l_c0 = (GUP ? nt * (kBN / 2) : nt * kBN) + lwn * OUT_C;
        constexpr int ROWS_PER_READ = 1024 / OUT_RB;
#pragma unroll
        for (int r0 = 0; r0 < kWM; r0 += ROWS_PER_READ) {
            if (lwm * kWM + r0 >= rows) break;                          // wave-uniform
            const int r = r0 + ep_lane / OUT_CH;
            const int c = ep_lane % OUT_CH;
            const u32x4 vv = *reinterpret_cast<const u32x4*>(stg + r * OUT_RB + 16 * (c ^ stg_swz(r)));
            if (lwm * kWM + r < rows) {
                uint16_t* orow = out + static_cast<size_t>(row0 + lwm * kWM + r) * N_out;
                if (!GUP && plan_dst) {   // the loader wave scaled the row when it staged it
                    const int dst = plan_dst[lwm * kWM + r];
                    if (static_cast<unsigned>(dst) < static_cast<unsigned>(parts_rows))
                        orow = parts + static_cast<size_t>(dst) * N_out;
                }
                *reinterpret_cast<u32x4*>(orow + l_c0 + 8 * c) = vv;
            }
        }
    }
}

// Loads of tile (expert l, rows [row0, row0 + rows), block column nt) for
// loader wave lw, at stage 0.  Gate/up: A = x (K = d; rows of x through
// row_src if gathered, clamped into [0, x_rows)), B quarters of wave column wn
// are rows nt * 128 + 64 wn + {0, 32} .. + 31 of W1 (quarters 0, 2) and W3
// (quarters 1, 3); down: A = H (K = inter), B quarters are rows
// nt * 256 + 128 wn + 32 q .. + 31 of W2.  Rows past the tile's last valid one
// repeat it.  Lane byte offsets stay below 2^32 (x_rows * pitch does; a tile
// spans 256 rows of at most 2^20 bytes).
__device__ __forceinline__ void tile_loads(Loads& s, bool gu, bool gathered, const uint16_t* A, const uint16_t* B0,
                                           const uint16_t* B1, int l, int row0, int rows, int nt, int lw, int K,
                                           int N_out, int lane, const int32_t* __restrict__ row_src,
                                           int x_rows) {
    const LaneMap lm = lane_map(opaque(lane));
    const uint32_t pitch = static_cast<uint32_t>(K) * 2u;
    s.a = gathered ? reinterpret_cast<const char*>(A) : reinterpret_cast<const char*>(A + static_cast<size_t>(row0) * K);
    s.a_on = lw / kWavesN * kWM < rows;
    const int wn = lw >> 1, h = lw & 1;
    if (gu) {
        const size_t row = static_cast<size_t>(l) * N_out + nt * (kBN / 2) + wn * (kWN / 2) + h * 16;
        s.b0 = reinterpret_cast<const char*>(B0 + row * K);
        s.b1 = reinterpret_cast<const char*>(B1 + row * K);
        s.c0 = s.b0 + static_cast<size_t>(32) * pitch;
        s.c1 = s.b1 + static_cast<size_t>(32) * pitch;
    } else {
        const size_t row = static_cast<size_t>(l) * N_out + nt * kBN + wn * kWN + h * 16;
        s.b0 = reinterpret_cast<const char*>(B0 + row * K);
        s.b1 = s.b0 + static_cast<size_t>(32) * pitch;
        s.c0 = s.b0 + static_cast<size_t>(64) * pitch;
        s.c1 = s.b0 + static_cast<size_t>(96) * pitch;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) s.b_off[i] = (i * kRowsPerLoad + lm.ld_row) * pitch + lm.col_b[i];
#pragma unroll
    for (int i = 0; i < kALd; ++i) {
        int r = min(lw * kALd * kRowsPerLoad + i * kRowsPerLoad + lm.ld_row, rows - 1);
        if (gathered) r = min(max(row_src[row0 + r], 0), x_rows - 1);
        s.a_off[i] = static_cast<uint32_t>(r) * pitch + lm.col_b[(lw * kALd + i) & 1];
    }
}

// ------------------------------------------------------------------ narrow tiles (few rows per expert)
// A call whose experts hold few rows each (decode, small chunks) reads every
// weight once for little arithmetic: what bounds it is the weights' way from
// HBM.  256 x 256 tiles then leave most of the chip idle (an expert has 16
// gate/up tiles at inter = 2048) and keep too little in flight.  On narrow
// tiles, 257 rows over 8 experts of d = 7168, inter = 2048 take 146 us where wide
// tiles take 194 (705 MB of weights: 4.8 TB/s; a large copy moves 5.2 TB/s), 61
// rows over 16 experts of d = 2048, inter = 768 39 us instead of 59.
// Narrow tiles are BM = 64 or 128 rows x 128 weight rows (64 H columns of
// gate/up, or 128 output columns), run by the same eight waves with a ring of
// K = 64 stages (five of 24 KB, or four of 32 KB), all but one of them in
// flight, that runs on across the tiles of a workgroup.  Every wave loads an
// eighth of a stage and computes BM / 2 rows x 32 weight rows.  Stage rows,
// swizzle, fragments and K order are those of the wide tiles, so every output
// element has the same bits.
constexpr int kNbN = 128;                             // weight rows of a narrow tile
static_assert(2 * kNW * kRowsPerLoad == kNbN, "load split");

// Which tiles a call runs on, from its experts' rows (the same everywhere:
// every kernel of the call decides alike): 256 (wide), or the rows of its
// narrow tiles.  Each form's time is modelled as the stages of its busiest
// workgroup times the clocks of a stage with the whole chip at work: the
// narrow forms' are the time their 16 KB of weights take from HBM (2.0 GHz,
// 13 bytes a clock and CU), the wide form's that of its MFMAs.  Measured, us
// (64 / 128 / 256 rows): 257 rows over 8 experts, the most 66, d = 7168, inter =
// 2048: 174 / 146 / 194 (a ninth m-tile costs a second round); 61 rows over 16
// experts, d = 2048, inter = 768: 39 / 41 / 59; 8 experts of 256 rows, d = 2048,
// inter = 1408: 77 / 70 / 75; of 400: 119 / 98 / 73.  Over six layer shapes and
// 16 to 512 rows an expert the rule is within 4 % of the best form but for one
// or four experts of 200 to 512 rows (up to 13 %).  One expert of 800 or more
// rows (shared experts) would run up to a third faster on narrow tiles alone,
// but on the whole chip: beside the routed experts, where a step runs it, it
// costs more than the 64 to 88 workgroups of the wide form, so kNarrowMaxRows
// keeps it there.
constexpr int kNarrowMaxRows = 512;
constexpr int kWideClk = 2400, kNarrow64Clk = 1200, kNarrow128Clk = 1300;

// The schedule of a call's m-tiles, built by wave 0 in registers: row bounds of
// every expert, m-tiles before it (mt_prefix[0..E_loc]) for the chosen tile
// rows, which are returned.  cus > 0: narrow tiles are allowed.  decide: the
// caller needs no schedule of wide tiles.  Every workgroup runs this before its
// first load, so the steps across lanes stop at E_loc, and a call with an
// expert of too many rows skips the model (1,100 rows of d = 256, inter = 128
// 20.4 -> 18.7 us, both launches).
__device__ __forceinline__ int build_call(const int32_t* row_offsets, int E_loc, int max_rows, int d, int inter, int cus,
                                          bool decide, int* mt_prefix, int* row_begin, int* row_end) {
    __shared__ int tile_rows;
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        const int base = row_offsets[0];
        constexpr int kPer = kMaxExpertsLocal / kWave;           // experts per lane: l = c * 64 + lane
        int n[kPer];
        int t64 = 0, t128 = 0, t256 = 0, most = 0;
#pragma unroll
        for (int c = 0; c < kPer; ++c) {
            n[c] = 0;
            const int l = c * kWave + lane;
            if (c * kWave < E_loc) {                             // wave-uniform
                int b = row_offsets[min(l, E_loc)] - base, e = row_offsets[min(l + 1, E_loc)] - base;
                b = max(0, min(b, max_rows));
                e = max(b, min(e, max_rows));
                if (l < E_loc) {
                    row_begin[l] = b;
                    row_end[l] = e;
                    n[c] = e - b;
                }
            }
            t64 += (n[c] + 63) / 64;
            t128 += (n[c] + 127) / 128;
            t256 += (n[c] + 255) / 256;
            most = max(most, n[c]);
        }
        int shift = 8;                                           // tile rows: 2^shift
        if (cus > 0 && !__any(most > kNarrowMaxRows)) {
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {                // sums in lane 0 (lanes past E_loc hold none)
                if (o >= E_loc) break;
                t64 += __shfl_xor(t64, o);
                t128 += __shfl_xor(t128, o);
                t256 += __shfl_xor(t256, o);
            }
            // a workgroup's stages: its share of both GEMMs' tiles, rounded up
            // (in floats: an integer division costs as much as the rest)
            const float per_cu = __builtin_amdgcn_rcpf(static_cast<float>(cus));
            auto stages = [&](int m_tiles, int n_gu, int n_dn) {
                const float m = static_cast<float>(m_tiles) * per_cu;
                return ceilf(m * static_cast<float>(n_gu) - 1e-3f) * static_cast<float>(d / kStageK) +
                       ceilf(m * static_cast<float>(n_dn) - 1e-3f) * static_cast<float>(inter / kStageK);
            };
            const float wide = stages(t256, inter / (kBN / 2), d / kBN) * kWideClk;
            const float n64 = stages(t64, inter / (kNbN / 2), d / kNbN) * kNarrow64Clk;
            const float n128 = stages(t128, inter / (kNbN / 2), d / kNbN) * kNarrow128Clk;
            if (min(n64, n128) < wide) shift = n64 <= n128 ? 6 : 7;
            shift = __builtin_amdgcn_readfirstlane(shift);
        }
        static_assert(kBM == 256, "tile rows by shift");
        const int rows = 1 << shift;
        const bool scan = !(decide && rows == kBM);
        int before = 0;                                          // m-tiles of the experts before this chunk
#pragma unroll
        for (int c = 0; c < kPer; ++c) {
            if (c * kWave >= E_loc || !scan) break;
            int v = (n[c] + rows - 1) >> shift;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                if (o >= E_loc) break;
                const int u = __shfl_up(v, o);
                if (lane >= o) v += u;
            }
            v += before;
            if (c * kWave + lane < E_loc) mt_prefix[c * kWave + lane + 1] = v;
            before = __shfl(v, kWave - 1);
        }
        if (lane == 0) {
            mt_prefix[0] = 0;
            tile_rows = rows;
        }
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(tile_rows);
}

// One GEMM of a call on narrow tiles.  mt_prefix, row_begin, row_end: the
// schedule of BM-row m-tiles.  Tile order: expert, n-tile, m-tile (the m-tiles
// that share weight rows are neighbours, on one XCD).
template <int BM, bool GATEUP, bool GATHER>
__device__ __forceinline__ void narrow_gemm(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
                                            const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
                                            const int* mt_prefix, const int* row_begin, const int* row_end, int E_loc,
                                            int K, int N_out, const int32_t* __restrict__ row_src, int x_rows,
                                            const CombinePlan& cp, const uint8_t* lds) {
    constexpr int MB = BM / 32;                           // 16-row blocks of a wave: block i is rows (2 i + wm) * 16 ..
    constexpr int A_LD = BM / (kNW * kRowsPerLoad), LOADS = A_LD + 2;   // loads per wave and stage
    constexpr int STAGE_B = (BM + kNbN) * kRowB;
    constexpr int RING = kStages * kStageBytes / STAGE_B;
    static_assert(BM == 64 || BM == 128, "built forms");
    const int n_tiles = GATEUP ? N_out / (kNbN / 2) : N_out / kNbN;
    const int total = mt_prefix[E_loc] * n_tiles;
    const int G = worker_count(total);
    int tile = worker_id(G);
    if (tile < 0 || tile >= total) return;
    const int KT = K / kStageK;
    const uint32_t pitch = static_cast<uint32_t>(K) * 2u;
    const int lane = threadIdx.x % kWave;
    const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave));
    const int wm = wave >> 2, wn = wave & 3;
    const LaneMap lm = lane_map(lane);
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));

    struct Tile { int l, row0, rows, nt; };
    auto decode = [&](int t) __attribute__((always_inline)) {
        const int l = __builtin_amdgcn_readfirstlane(find_expert(mt_prefix, E_loc, t / n_tiles));
        const int m0 = __builtin_amdgcn_readfirstlane(mt_prefix[l]);
        const int cnt = __builtin_amdgcn_readfirstlane(mt_prefix[l + 1]) - m0;
        const int u = t - m0 * n_tiles;
        Tile T;
        T.l = l;
        T.nt = u / cnt;
        T.row0 = __builtin_amdgcn_readfirstlane(row_begin[l]) + (u - T.nt * cnt) * BM;
        T.rows = min(BM, __builtin_amdgcn_readfirstlane(row_end[l]) - T.row0);
        return T;
    };

    // The load cursor: the next stage to issue, up to four ahead of the one
    // computed.  A: rows 64 i + 8 wave .. + 7 of the tile (past its valid rows:
    // the last again).  B: tile rows 32 w .. + 15 are W1 rows (or W2 rows) and
    // 32 w + 16 .. + 31 W3 rows (W2 rows) of the output columns 16 w .. (32 w
    // ..) of wave column w; wave 2 w + h loads the 16 rows of half h.
    const char *pa, *pb;
    uint32_t a_off[A_LD];
    const uint32_t b_off0 = lm.ld_row * pitch + lm.col_b[0], b_off1 = (kRowsPerLoad + lm.ld_row) * pitch + lm.col_b[1];
    int it_tile = tile, it_kt = 0, it_buf = 0;
    auto cursor_tile = [&]() __attribute__((always_inline)) {
        const Tile T = decode(it_tile);
        pa = reinterpret_cast<const char*>(GATHER ? A : A + static_cast<size_t>(T.row0) * K);
#pragma unroll
        for (int j = 0; j < A_LD; ++j) {
            const int r0 = j * kNW * kRowsPerLoad + kRowsPerLoad * wave;
            uint32_t r = 0;
            if (GATHER) {
                // the eight rows through scalar loads: a vector load's wait
                // would drain the direct loads in flight
#pragma unroll
                for (int i = 0; i < kRowsPerLoad; ++i) {
                    const int v = row_src[T.row0 + min(r0 + i, T.rows - 1)];
                    r = lm.ld_row == i ? static_cast<uint32_t>(min(max(v, 0), x_rows - 1)) : r;
                }
            } else {
                r = min(r0 + lm.ld_row, T.rows - 1);
            }
            a_off[j] = r * pitch + ((wave & 1) ? lm.col_b[1] : lm.col_b[0]);
        }
        const int h = wave & 1;
        if (GATEUP)
            pb = reinterpret_cast<const char*>((h ? B1 : B0) + (static_cast<size_t>(T.l) * N_out + T.nt * (kNbN / 2) +
                                                                (wave >> 1) * 16) * K);
        else
            pb = reinterpret_cast<const char*>(B0 + (static_cast<size_t>(T.l) * N_out + T.nt * kNbN + wave * 16) * K);
    };
    auto issue = [&]() __attribute__((always_inline)) {
        const uint32_t st = lds_base + it_buf * STAGE_B;
        lds_dma16(pa, a_off[0], st + wave * 1024);
        if constexpr (A_LD > 1) lds_dma16(pa, a_off[A_LD - 1], st + 64 * kRowB + wave * 1024);
        lds_dma16(pb, b_off0, st + BM * kRowB + wave * 2048);
        lds_dma16(pb, b_off1, st + BM * kRowB + wave * 2048 + 1024);
        it_buf = it_buf + 1 == RING ? 0 : it_buf + 1;
        if (++it_kt < KT) {
            pa += kRowB;
            pb += kRowB;
        } else if (it_tile + G < total) {
            it_tile += G;
            it_kt = 0;
            cursor_tile();
        } else {
            it_kt = KT - 1;            // past the end: the last stage again, so that the counts of loads in flight hold
        }
    };

    cursor_tile();
#pragma unroll 1
    for (int i = 0; i < RING - 1; ++i) issue();
    int buf = 0;
    const int pc0 = (lm.fr_kc ^ lm.fr_swz) << 4, pc1 = pc0 ^ 64;
    for (; tile < total; tile += G) {
        const Tile T = decode(tile);
        const int blocks = min(MB, (T.rows - wm * 16 + 31) / 32);     // blocks with valid rows (wave-uniform)
        f32x4 acc[MB][2];
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;
        for (int kt = 0; kt < KT; ++kt) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // this wave has read the stage before
            wait_vm<(RING - 2) * LOADS>();                           // its part of this stage has landed
            block_barrier();
            issue();                                                 // into the buffer of the stage before
            const uint8_t* st = lds + buf * STAGE_B;
            const uint8_t* la = st + (wm * 16 + lm.fr_row) * kRowB;
            const uint8_t* lb = st + (BM + wn * 32 + lm.fr_row) * kRowB;
            bf16x8 b[2][2], a[MB][2];
            if (blocks > 0) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    b[0][ks] = frag_at(lb + (ks ? pc1 : pc0));
                    b[1][ks] = frag_at(lb + 16 * kRowB + (ks ? pc1 : pc0));
                }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                if (i >= blocks) break;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) a[i][ks] = frag_at(la + i * 32 * kRowB + (ks ? pc1 : pc0));
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                if (i >= blocks) break;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], a[i][ks], acc[i][j], 0, 0, 0);
            }
            buf = buf + 1 == RING ? 0 : buf + 1;
        }
        // lane (r, q) holds columns 4 q .. + 3 of row r of each 16 x 16 block
        const int q = lane >> 4;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int r = (2 * i + wm) * 16 + lm.fr_row;
            if (r >= T.rows) continue;
            const size_t grow = static_cast<size_t>(T.row0 + r);
            if constexpr (GATEUP) {
                float h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = silu(acc[i][0][e]) * acc[i][1][e];
                u32x2 o;
                o[0] = pack_bf16x2_rne(h[0], h[1]);
                o[1] = pack_bf16x2_rne(h[2], h[3]);
                *reinterpret_cast<u32x2*>(C + grow * N_out + T.nt * (kNbN / 2) + wn * 16 + 4 * q) = o;
            } else {
                uint16_t* crow = C + grow * N_out;
                int dst = -1;
                float dw = 0.0f;
                if (cp.dst) {
                    dst = cp.dst[grow];
                    dw = cp.w[grow];
                    if (static_cast<unsigned>(dst) >= static_cast<unsigned>(cp.parts_rows)) dst = -1;
                    else crow = cp.parts + static_cast<size_t>(dst) * N_out;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    u32x2 o;
                    o[0] = pack_bf16x2_rne(acc[i][j][0], acc[i][j][1]);
                    o[1] = pack_bf16x2_rne(acc[i][j][2], acc[i][j][3]);
                    if (dst >= 0) {
                        o[0] = scale_pair(o[0], dw);
                        o[1] = scale_pair(o[1], dw);
                    }
                    *reinterpret_cast<u32x2*>(crow + T.nt * kNbN + wn * 32 + j * 16 + 4 * q) = o;
                }
            }
        }
    }
    wait_vm<0>();
}

// ------------------------------------------------------------------ two-kernel bf16 path
// One persistent kernel per GEMM (used for calls of few m-tiles).  Roles:
// loads and stores share one in-order completion counter per wave, so a wave
// that stores its outputs and then waits for a stage would also wait for
// every store to drain (a whole tile of outputs per CU, all CUs at once).  The
// loader waves therefore issue every direct-to-LDS stage load and never store
// to global memory (they stage their outputs in LDS); the storer waves issue
// no loads, write their own and the staged outputs, and never wait for
// stores.  The staging area is stage buffer 1, free from the end of a tile's K
// loop until the next tile fills its stage 1 (one barrier later).
// Tiles are ordered expert, m-tile, n-tile (n fastest: neighbours share the A
// rows); block b runs on XCD b % 8, so the block -> worker map gives each XCD
// a contiguous run of tiles and their operands share that XCD's L2.
// GATHER: row i of A is A[row_src[i]] (A has x_rows rows).
template <bool GATEUP, bool GATHER>
__global__ __launch_bounds__(kNW * kWave, 1) void ffn_gemm_bf16_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
    uint16_t* __restrict__ C, const int32_t* __restrict__ row_offsets, int E_loc, int max_rows, int K,
    int N_out, const int32_t* __restrict__ row_src, int x_rows, CombinePlan cp, int cus, int* __restrict__ sync,
    int n_sync) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kStages * kStageBytes];
    __shared__ int plan_dst[kBM];
    __shared__ float plan_w[kBM];
    __shared__ int mt_prefix[kMaxExpertsLocal + 1];
    __shared__ int row_begin[kMaxExpertsLocal];
    __shared__ int row_end[kMaxExpertsLocal];

    if (sync && blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_sync; i += blockDim.x) sync[i] = 0;
    const int bm = build_call(row_offsets, E_loc, max_rows, GATEUP ? K : N_out, GATEUP ? N_out : K, cus, sync != nullptr,
                              mt_prefix, row_begin, row_end);
    if (bm == 64) {
        narrow_gemm<64, GATEUP, GATHER>(A, B0, B1, C, mt_prefix, row_begin, row_end, E_loc, K, N_out, row_src, x_rows,
                                        cp, lds);
        return;
    }
    if (bm == 128) {
        narrow_gemm<128, GATEUP, GATHER>(A, B0, B1, C, mt_prefix, row_begin, row_end, E_loc, K, N_out, row_src, x_rows,
                                         cp, lds);
        return;
    }
    if (sync) return;
    const int n_tiles = GATEUP ? N_out / (kBN / 2) : N_out / kBN;
    const int total = mt_prefix[E_loc] * n_tiles;
    const int KT = K / kStageK;
    const int lane = threadIdx.x % kWave;
    const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave));
    const bool loader = wave < kNL;
    const int wm = wave / kWavesN, wn = wave % kWavesN;
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
    const uint32_t a_lds = lds_base + wave * kALd * 1024;             // loader waves' parts of a stage
    const uint32_t b_lds = lds_base + (kBM + (wave >> 1) * kWN + (wave & 1) * 16) * kRowB;
    // combine plan of a down tile: each storer lane loads one row's entry in
    // the last stage but one (after the stage where the fused kernel's storers
    // wait for their previous stores to drain) and writes it to the LDS table
    // in the last; the epilogue reads the table after the K loop's final
    // barrier
    const bool comb = !GATEUP && cp.dst != nullptr;
    int pl_d = -1;
    float pl_w = 0.0f;
    auto load_plan = [&](auto step, int r0, int nrows) {
        const int q = (wave - kNL) * kWave + opaque(lane);
        if constexpr (decltype(step)::value == kLast2) {
            pl_d = -1;
            pl_w = 0.0f;
            if (q < nrows) {
                pl_d = cp.dst[r0 + q];
                pl_w = cp.w[r0 + q];
            }
        } else if constexpr (decltype(step)::value == kPreLast) {
            plan_dst[q] = pl_d;
            plan_w[q] = pl_w;
        }
    };

    int row0 = 0, rows = 0, nt = 0;
    Loads ld;
    auto start_tile = [&](int tile) {
        const int m_tile = tile / n_tiles;
        nt = tile % n_tiles;
        // wave-uniform: keep them in scalar registers
        const int l = __builtin_amdgcn_readfirstlane(find_expert(mt_prefix, E_loc, m_tile));
        row0 = __builtin_amdgcn_readfirstlane(row_begin[l] + (m_tile - mt_prefix[l]) * kBM);
        rows = __builtin_amdgcn_readfirstlane(min(kBM, row_end[l] - row0));
        if (!loader) return;
        tile_loads(ld, GATEUP, GATHER, A, B0, B1, l, row0, rows, nt, wave, K, N_out, lane, row_src, x_rows);
        load_half0(ld, ld.a_on, a_lds, b_lds, 0);
        load_half1(ld, b_lds, 0);
    };

    const int G = worker_count(total);
    int tile = worker_id(G);
    if (tile < 0) return;
    if (tile < total) start_tile(tile);
    while (tile < total) {
        f32x4 acc[kMI][kNJ];
#pragma unroll
        for (int i = 0; i < kMI; ++i)
#pragma unroll
            for (int j = 0; j < kNJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

        const int cur_row0 = row0, cur_rows = rows, cur_nt = nt;
        const int next = tile + G;
        // in the last stage buffer 0 is free: the next tile's stage 0 lands
        // during the rest of that stage and the epilogue
        auto load_hook = [&](auto step) {
            if constexpr (decltype(step)::value == kLast) {
                if (next < total) start_tile(next);
            }
        };
        auto store_hook = [&](auto step) {
            if (comb) load_plan(step, cur_row0, cur_rows);
            load_hook(step);
        };
        run_k_loop(KT, lds, wm, wn, lane, loader, wm * kWM < rows, acc, ld, a_lds, b_lds, load_hook, store_hook);
        // buffer 1 is the staging area until the next tile fills its stage 1
        store_tile<GATEUP>(acc, C, N_out, cur_row0, cur_rows, cur_nt, wave, lane, lds + kStageBytes,
                           comb ? plan_dst : nullptr, plan_w, cp.parts, cp.parts_rows);
        tile = next;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// ------------------------------------------------------------------ fused bf16 FFN
// Both GEMMs in one persistent kernel (calls of many m-tiles).  The m-tiles
// (256 expert-sorted rows) are split into one contiguous range per XCD; a
// workgroup reads its XCD from the XCC_ID hardware register.  Each XCD has a
// queue: the gate/up tiles of its m-tiles, then their down tiles, claimed one
// at a time through an atomic counter.  A down tile reads the H rows of its
// m-tile, which gate/up tiles of the same XCD wrote: those stores are in that
// XCD's L2, which its loads read.  Each storer wave adds 1 to its m-tile's
// ready counter once its store counter has drained after a gate/up tile; a
// down tile starts when that counter reaches (gate/up n-tiles) x (storer
// waves).  The gate/up tail thereby overlaps the first down tiles, and each
// XCD reads the weights of only the experts its rows belong to.
//
// The next queue entry is claimed during a tile's first stage, published at
// its second and, for a down tile, its readiness polled two stages before the
// end; a ready tile's first stage is issued before the epilogue, as in the
// two-kernel path.  Counts of this tile's stores are delivered during the next
// tile's second stage, or before any wait.
//
// No wait can deadlock: a workgroup waits (before a down tile) only once every
// gate/up tile of its XCD's queue has been claimed; a gate/up tile is claimed
// only by a running workgroup and never waits, and a workgroup delivers its own
// pending counts before it waits.  Each wait is also bounded (spin_limit
// polls): past it the kernel adds 1 to *wait_err (the caller's counter, or a
// word of the workspace when the caller passes none) and goes on, so a wait
// that gave up is visible to the caller.  A queue no workgroup touched (an XCD
// that ran none of them) is run by the last workgroup to finish, so every tile
// is computed whatever the dispatch.  target_bias is 0; a caller testing the
// give-up path passes 1, which makes every wait's target unreachable, so each
// down tile waits once and gives up after spin_limit polls.
//
// sync (ints, zero at launch): the queue counter of XCD x at
// x * kSyncQueueStride, the workspace error word, the finished-workgroup
// count, then one ready counter per m-tile.
constexpr int kSyncQueueStride = 32;                 // one 128-byte line per queue counter
constexpr int kMaxXcc = 8;
constexpr int kSyncErr = kMaxXcc * kSyncQueueStride;
constexpr int kSyncDone = kSyncErr + 1;
constexpr int kSyncReady = kSyncErr + kSyncQueueStride;
constexpr int kGroupM = 4;                 // m-tiles per group of the queue order
constexpr int kSpinLimit = 1 << 20;        // default polls before a wait gives up

__device__ __forceinline__ int xcc_register() {
    int x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    return x;
}

__device__ __forceinline__ int atomic_add_agent(int* p, int v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool GATHER>
__global__ __launch_bounds__(kNW * kWave, 1) void ffn_fused_bf16_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W3,
    const uint16_t* __restrict__ W2, uint16_t* __restrict__ H, uint16_t* __restrict__ Y,
    const int32_t* __restrict__ row_offsets, int E_loc, int max_rows, int d, int inter,
    const int32_t* __restrict__ row_src, int x_rows, int n_xcc, int* __restrict__ sync,
    int* __restrict__ wait_err, int spin_limit, int target_bias, CombinePlan cp, int cus) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kStages * kStageBytes];
    __shared__ int plan_dst[kBM];
    __shared__ float plan_w[kBM];
    __shared__ int mt_prefix[kMaxExpertsLocal + 1];
    __shared__ int row_begin[kMaxExpertsLocal];
    __shared__ int row_end[kMaxExpertsLocal];
    // LDS broadcasts, one slot per value: each is written by one wave before a
    // barrier and read after it, and not written again before another barrier
    __shared__ int bcast[4];                // next entry; may it start early; finished count; untouched queue

    const int bm = build_call(row_offsets, E_loc, max_rows, d, inter, cus, false, mt_prefix, row_begin, row_end);
    if (bm == 64) {
        narrow_gemm<64, false, false>(H, W2, nullptr, Y, mt_prefix, row_begin, row_end, E_loc, inter, d, nullptr, 0, cp,
                                      lds);
        return;
    }
    if (bm == 128) {
        narrow_gemm<128, false, false>(H, W2, nullptr, Y, mt_prefix, row_begin, row_end, E_loc, inter, d, nullptr, 0,
                                       cp, lds);
        return;
    }
    const int MT = mt_prefix[E_loc];
    const int n_gu = inter / (kBN / 2), n_dn = d / kBN;
    const int target = n_gu * (kNW - kNL) + target_bias;
    int* const ready = sync + kSyncReady;
    const int lane = threadIdx.x % kWave;
    const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave));
    const bool loader = wave < kNL;
    const int wm = wave / kWavesN, wn = wave % kWavesN;
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
    const uint32_t a_lds = lds_base + wave * kALd * 1024;             // loader waves' parts of a stage
    const uint32_t b_lds = lds_base + (kBM + (wave >> 1) * kWN + (wave & 1) * 16) * kRowB;
    // combine plan of a down tile (as in the two-kernel path)
    const bool comb = cp.dst != nullptr;
    int pl_d = -1;
    float pl_w = 0.0f;
    auto load_plan = [&](auto step, int r0, int nrows) {
        const int q = (wave - kNL) * kWave + opaque(lane);
        if constexpr (decltype(step)::value == kLast2) {
            pl_d = -1;
            pl_w = 0.0f;
            if (q < nrows) {
                pl_d = cp.dst[r0 + q];
                pl_w = cp.w[r0 + q];
            }
        } else if constexpr (decltype(step)::value == kPreLast) {
            plan_dst[q] = pl_d;
            plan_w[q] = pl_w;
        }
    };

    // queue of XCD slot x: m-tiles [mb, mb + MX); gate/up entries [0, GU), down [GU, Q)
    int x = xcc_register() % n_xcc;
    int mb = 0, MX = 0, GU = 0, Q = 0;
    int* queue = sync;
    auto set_queue = [&](int xs) {
        mb = (xs * MT) / n_xcc;
        MX = ((xs + 1) * MT) / n_xcc - mb;
        GU = MX * n_gu;
        Q = GU + MX * n_dn;
        queue = sync + xs * kSyncQueueStride;
    };
    // Entry u of a GEMM with nn n-tiles -> (m-tile offset, n-tile): the m-tiles
    // go in groups of kGroupM; within a group the n-tile is the outer index.
    // The workgroups of an XCD then run a block of about kGroupM m-tiles x
    // (CUs / kGroupM) n-tiles at a time, so each operand stream (an m-tile's
    // rows, an n-tile's weight rows) is shared by several running tiles and
    // the expert's weights are streamed into the XCD once per group of
    // m-tiles instead of once per one or two m-tiles.
    auto entry_tile = [&](int u, int nn, int& m_off, int& nt) {
        const int g = u / (kGroupM * nn);
        const int v = u - g * (kGroupM * nn);
        const int gm = min(kGroupM, MX - g * kGroupM);
        m_off = g * kGroupM + v % gm;
        nt = v / gm;
    };

    struct Tile { int gu, m, nt, row0, rows, KT; };
    Tile T{};
    Loads ld;
    auto decode = [&](int t) {
        Tile D;
        D.gu = t < GU ? 1 : 0;
        const int u = D.gu ? t : t - GU;
        int m_off, nt;
        entry_tile(u, D.gu ? n_gu : n_dn, m_off, nt);
        D.m = __builtin_amdgcn_readfirstlane(mb + m_off);
        D.nt = __builtin_amdgcn_readfirstlane(nt);
        D.KT = (D.gu ? d : inter) / kStageK;
        const int l = __builtin_amdgcn_readfirstlane(find_expert(mt_prefix, E_loc, D.m));
        D.row0 = __builtin_amdgcn_readfirstlane(row_begin[l] + (D.m - mt_prefix[l]) * kBM);
        D.rows = __builtin_amdgcn_readfirstlane(min(kBM, row_end[l] - D.row0));
        if (loader) {
            if (D.gu) tile_loads(ld, true, GATHER, X, W1, W3, l, D.row0, D.rows, D.nt, wave, d, inter, lane, row_src, x_rows);
            else tile_loads(ld, false, false, H, W2, nullptr, l, D.row0, D.rows, D.nt, wave, inter, d, lane, nullptr, 0);
        }
        return D;
    };
    auto issue0 = [&]() {
        if (!loader) return;
        load_half0(ld, ld.a_on, a_lds, b_lds, 0);
        load_half1(ld, b_lds, 0);
    };
    // wave 0 waits until m-tile m's H rows are complete, then the workgroup goes on
    auto wait_ready = [&](int m) {
        if (wave == 0 && lane == 0) {
            int polls = 0;
            while (atomic_add_agent(ready + m, 0) < target) {
                if (++polls > spin_limit) {
                    atomic_add_agent(wait_err, 1);
                    break;
                }
                __builtin_amdgcn_s_sleep(4);
            }
        }
        block_barrier();
    };
    // a storer wave counts its drained gate/up stores on the m-tile's counter
    int pending = -1;
    auto deliver = [&]() {
        if (!loader && pending >= 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) atomic_add_agent(ready + pending, 1);
            pending = -1;
        }
    };
    auto claim_blocking = [&]() {
        if (wave == kNL && lane == 0) bcast[0] = atomic_add_agent(queue, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        block_barrier();
        return __builtin_amdgcn_readfirstlane(bcast[0]);
    };

    bool checked_others = false;
    set_queue(x);
    for (;;) {
        int t = claim_blocking();
        if (t < Q) {
            T = decode(t);
            if (!T.gu) wait_ready(T.m);
            issue0();
        }
        while (t < Q) {
            f32x4 acc[kMI][kNJ];
#pragma unroll
            for (int i = 0; i < kMI; ++i)
#pragma unroll
                for (int j = 0; j < kNJ; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

            const Tile C = T;
            const int KT = C.KT;
            const bool ahead = KT >= 4;            // claim, publish and poll inside the K loop
            int claim = 0, poll = 0, nx = Q, early = 0;
            // last stage: buffer 0 is free, and a ready next tile's stage 0
            // lands during the rest of the stage and the epilogue
            auto start_next = [&]() {
                nx = __builtin_amdgcn_readfirstlane(bcast[0]);
                early = __builtin_amdgcn_readfirstlane(bcast[1]);
                if (nx < Q) {
                    T = decode(nx);
                    if (early) issue0();
                }
            };
            const bool active = wm * kWM < C.rows;
            auto load_hook = [&](auto step) {
                if constexpr (decltype(step)::value == kLast) {
                    if (ahead) start_next();
                }
            };
            auto store_hook = [&](auto step) {
                constexpr KStep at = decltype(step)::value;
                if (comb && !C.gu) load_plan(step, C.row0, C.rows);
                if constexpr (at == kSecond) deliver();
                if (ahead && wave == kNL && lane == 0) {
                    if constexpr (at == kFirst) claim = atomic_add_agent(queue, 1);
                    if constexpr (at == kLast2) {
                        if (claim >= GU && claim < Q) {
                            int m_off, nt;
                            entry_tile(claim - GU, n_dn, m_off, nt);
                            poll = atomic_add_agent(ready + mb + m_off, 0);
                        }
                    }
                    if constexpr (at == kPreLast) {
                        bcast[0] = claim;
                        bcast[1] = (claim < GU || claim >= Q || poll >= target) ? 1 : 0;
                    }
                }
                load_hook(step);
            };
            run_k_loop(KT, lds, wm, wn, lane, loader, active, acc, ld, a_lds, b_lds, load_hook, store_hook);
            if (!ahead) {
                deliver();
                if (wave == kNL && lane == 0) bcast[0] = atomic_add_agent(queue, 1);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                block_barrier();
                nx = __builtin_amdgcn_readfirstlane(bcast[0]);
                if (nx < Q) {
                    T = decode(nx);
                    if (nx < GU) {
                        early = 1;
                        issue0();
                    }
                }
            }
            if (C.gu) store_tile<true>(acc, H, inter, C.row0, C.rows, C.nt, wave, lane, lds + kStageBytes);
            else store_tile<false>(acc, Y, d, C.row0, C.rows, C.nt, wave, lane, lds + kStageBytes,
                                   comb ? plan_dst : nullptr, plan_w, cp.parts, cp.parts_rows);
            if (C.gu) pending = C.m;
            if (nx < Q && !early) {
                deliver();                         // the next tile may need this tile's rows
                wait_ready(T.m);
                issue0();
            }
            t = nx;
        }
        deliver();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // The last workgroup to finish runs any queue that none touched.
        if (!checked_others) {
            checked_others = true;
            if (wave == 0 && lane == 0) bcast[2] = atomic_add_agent(sync + kSyncDone, 1);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            block_barrier();
            if (__builtin_amdgcn_readfirstlane(bcast[2]) != static_cast<int>(gridDim.x) - 1) break;
        }
        if (wave == 0 && lane == 0) {
            int found = -1;
            for (int xs = 0; xs < n_xcc && found < 0; ++xs)
                if (atomic_add_agent(sync + xs * kSyncQueueStride, 0) == 0) found = xs;
            bcast[3] = found;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        block_barrier();
        x = __builtin_amdgcn_readfirstlane(bcast[3]);
        if (x < 0) break;
        set_queue(x);
    }
}

// ------------------------------------------------------------------ fp32 GEMM (small shapes)
// One wave computes RB x 16 rows by CB x 16 output columns on fp32 matrix
// instructions (v_mfma_f32_16x16x4_f32: fp32 products and sums), straight from
// global memory: lane (r, g) = (lane % 16, lane / 16) loads 16 bytes of row r
// at K = 16 j + 4 g for both operands, and element e of them feeds the e-th of
// four MFMAs (the same K on both sides).  The loads of a batch of U such steps
// are all issued before its first MFMA.  What bounds the small calls is the
// latency of that chain of loads, so a batch covers K = 128 and the tiles are
// the smallest there are (RB = CB = 1: 169 rows over 4 experts of d = 128,
// inter = 256 take 7 + 8 us; through 64 x 64 LDS tiles with a barrier pair every
// 16 K they took 26 + 42).  Calls with enough rows to fill the chip with larger
// tiles read each operand less often (RB = 4, CB = 2: 1,692 rows over 2 experts
// of d = 328, inter = 717 127 us, 273 through the LDS tiles).
// A4: K is a multiple of 4, so every row is 16-byte aligned.
constexpr int kF32Waves = 4;                 // a wave a tile, in groups of four that share weight rows
// Small tiles, in halves per CU, from which a GEMM takes the large ones, if
// those hold three of the eight small tiles they have room for: up to four
// large tiles per CU take the time of one, small ones a time that grows with
// their number, and less of it for a short K (the loads of one batch cover K =
// 128).  Measured, us (all small / gate/up large): 800 rows over 2 experts of d =
// inter = 1024 (12.5 small tiles per CU) 164 / 145; 1,280 rows over 32 experts
// of d = inter = 512 (12, three of four rows) 68 / 80; 1,400 rows over 2 experts
// of d = 328, inter = 717 (15.5) 93 / 101; 4,000 rows over 2 experts of d = 128,
// inter = 256 (15.6) 29 / 32.
__host__ __device__ constexpr int f32_large_from(int K) { return K <= 128 ? 40 : K < 512 ? 32 : 25; }
// Groups of a workgroup.  Where the rows settle the form on the device, a
// workgroup has as many waves as its CU holds of that kernel and the launch one
// per CU: few tiles then spread over all CUs (of two workgroups the dispatcher
// may put both on one).
constexpr int f32_groups(bool gateup, bool large) { return !large ? 1 : gateup ? 2 : 3; }

template <bool GATEUP, int RB, int CB, bool A4>
__device__ __forceinline__ void f32_tiles(const float* __restrict__ A, const float* __restrict__ B0,
                                          const float* __restrict__ B1, float* __restrict__ C, const int* mt_prefix,
                                          const int* row_begin, const int* row_end, int E_loc, int K, int N_out,
                                          const int32_t* __restrict__ row_src, int x_rows, int first, int step) {
    constexpr int U = RB == 1 ? 8 : 2;       // K steps of 16 per batch of loads
    const int MT = mt_prefix[E_loc];
    const int n_tiles = (N_out + CB * 16 - 1) / (CB * 16);
    const int lane = threadIdx.x % kWave;
    const int r16 = lane & 15, g = lane >> 4;
    // m-tile fastest: the waves of a group share their weight rows
    for (int tile = first; tile < MT * n_tiles; tile += step) {
        const int nt = tile / MT, m_tile = tile - nt * MT;
        const int l = __builtin_amdgcn_readfirstlane(find_expert(mt_prefix, E_loc, m_tile));
        const int row0 = __builtin_amdgcn_readfirstlane(row_begin[l] + (m_tile - mt_prefix[l]) * (RB * 16));
        const int rows = __builtin_amdgcn_readfirstlane(row_end[l]) - row0;
        const int col0 = nt * (CB * 16);
        const float* pa[RB];
        const float* pb[GATEUP ? 2 * CB : CB];        // gate blocks, then up blocks
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            int r = row0 + min(16 * i + r16, rows - 1);          // past the expert's end: its last row again
            if (row_src) r = min(max(row_src[r], 0), x_rows - 1);
            pa[i] = A + static_cast<size_t>(r) * K + 4 * g;
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const size_t n = static_cast<size_t>(l) * N_out + min(col0 + 16 * j + r16, N_out - 1);
            pb[j] = B0 + n * K + 4 * g;
            if constexpr (GATEUP) pb[CB + j] = B1 + n * K + 4 * g;
        }
        constexpr int NB = GATEUP ? 2 * CB : CB;
        // two sums per output, of the even and the odd K steps: half the chain
        // of dependent MFMAs, and less rounding than one running sum
        f32x4 acc[RB][NB], odd[RB][NB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] = odd[i][j][e] = 0.0f;
        // four values of a row at K = k .. k + 3, zero past K
        auto load4 = [&](const float* p, int k) __attribute__((always_inline)) {
            f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (A4) {
                if (k + 4 * g < K) v = *reinterpret_cast<const f32x4*>(p + k);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + 4 * g + e < K) v[e] = p[k + e];
            }
            return v;
        };
        for (int k0 = 0; k0 < K; k0 += 16 * U) {
            f32x4 a[U][RB], b[U][NB];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int i = 0; i < RB; ++i) a[u][i] = load4(pa[i], k0 + 16 * u);
#pragma unroll
                for (int j = 0; j < NB; ++j) b[u][j] = load4(pb[j], k0 + 16 * u);
            }
#pragma unroll
            for (int ue = 0; ue < 4 * U; ++ue) {
                const int u = ue / 8 * 2 + ue % 2, e = ue % 8 / 2;           // even and odd steps in turn
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        f32x4& s = u % 2 ? odd[i][j] : acc[i][j];
                        s = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][j][e], a[u][i][e], s, 0, 0, 0);
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += odd[i][j][e];
        // lane (r, g) holds columns 4 g .. + 3 of row r of each 16 x 16 block
        const bool c4 = (N_out & 3) == 0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (16 * i + r16 >= rows) continue;
            float* crow = C + static_cast<size_t>(row0 + 16 * i + r16) * N_out;
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                const int c = col0 + 16 * j + 4 * g;
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (GATEUP) v[e] = silu(acc[i][j][e]) * acc[i][CB + j][e];
                    else v[e] = acc[i][j][e];
                }
                if (c4) {
                    if (c < N_out) *reinterpret_cast<f32x4*>(crow + c) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < N_out) crow[c + e] = v[e];
                }
            }
        }
    }
}

// LARGE: the row capacity allows large tiles, and the experts' rows, which may
// be far fewer, settle it here, for each GEMM by itself (32 rows over 8 experts
// of d = 2048, inter = 1408 with a capacity of 2,048 rows: 261 us when the
// capacity chose large tiles for both, 67 so).
template <bool GATEUP, bool LARGE, bool A4>
__global__ __launch_bounds__((f32_groups(GATEUP, LARGE) * kF32Waves * kWave)) void ffn_gemm_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ B0, const float* __restrict__ B1,
    float* __restrict__ C, const int32_t* __restrict__ row_offsets, int E_loc, int max_rows, int K, int N_out,
    const int32_t* __restrict__ row_src, int x_rows, int cus) {
    __shared__ int mt_prefix[kMaxExpertsLocal + 1];
    __shared__ int row_begin[kMaxExpertsLocal];
    __shared__ int row_end[kMaxExpertsLocal];
    const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave));
    const int first = (wave / kF32Waves * gridDim.x + blockIdx.x) * kF32Waves + wave % kF32Waves;
    const int step = gridDim.x * f32_groups(GATEUP, LARGE) * kF32Waves;
    expert_rows(row_offsets, E_loc, max_rows, row_begin, row_end);
    build_schedule<16>(E_loc, mt_prefix, row_begin, row_end);
    if constexpr (LARGE) {
        const long long small = static_cast<long long>(mt_prefix[E_loc]) * ((N_out + 15) / 16);
        if (2 * small >= static_cast<long long>(f32_large_from(K)) * cus) {
            __syncthreads();
            build_schedule<64>(E_loc, mt_prefix, row_begin, row_end);
            const long long large = static_cast<long long>(mt_prefix[E_loc]) * ((N_out + 31) / 32);
            if (small >= 3 * large) {
                // gate/up: one wave per SIMD (two read more than the L1 keeps: 2,000
                // rows of d = 2048, inter = 1408 505 us, 568 with two)
                if (!GATEUP || wave < kF32Waves)
                    f32_tiles<GATEUP, 4, 2, A4>(A, B0, B1, C, mt_prefix, row_begin, row_end, E_loc, K, N_out, row_src,
                                                x_rows, first, GATEUP ? static_cast<int>(gridDim.x) * kF32Waves : step);
                return;
            }
            __syncthreads();
            build_schedule<16>(E_loc, mt_prefix, row_begin, row_end);
        }
    }
    f32_tiles<GATEUP, 1, 1, A4>(A, B0, B1, C, mt_prefix, row_begin, row_end, E_loc, K, N_out, row_src, x_rows,
                                first, step);
}

template <bool GATEUP>
void launch_ffn_f32(const float* a, const float* b0, const float* b1, float* c, const int32_t* row_offsets, int E_loc,
                    int max_rows, int K, int N_out, const int32_t* row_src, int x_rows, hipStream_t st) {
    const long long cus = device_cu_count();
    const long long small = (max_rows / 16 + E_loc) * static_cast<long long>((N_out + 15) / 16);   // most there can be
    const long long need = (small + kF32Waves - 1) / kF32Waves;
    auto by_form = [&](auto A4) {
        auto go = [&](auto Large, long long most) {
            constexpr bool large = decltype(Large)::value;
            ffn_gemm_f32_kernel<GATEUP, large, decltype(A4)::value>
                <<<static_cast<int>(need < most ? need : most), f32_groups(GATEUP, large) * kF32Waves * kWave, 0, st>>>(
                    a, b0, b1, c, row_offsets, E_loc, max_rows, K, N_out, row_src, x_rows, static_cast<int>(cus));
        };
        if (2 * small >= f32_large_from(K) * cus) go(std::true_type{}, cus);
        else go(std::false_type{}, 8 * cus);
    };
    // the gate/up GEMM's K is d, a multiple of four
    if constexpr (GATEUP) by_form(std::true_type{});
    else if ((K & 3) == 0) by_form(std::true_type{});
    else by_form(std::false_type{});
}

int persistent_grid(long long tiles_upper) {
    const long long cus = device_cu_count();
    long long g = tiles_upper < cus ? tiles_upper : cus;
    if (g >= 8) g -= g % 8;          // whole XCD rounds
    return static_cast<int>(g < 1 ? 1 : g);
}

// Row capacity from which a bf16 call runs the fused kernel: 32 m-tiles, so
// that every XCD gets several; below it the two-kernel path spreads the few
// m-tiles' n-tiles over all CUs.
constexpr int kFusedMinRows = 32 * kBM;

int fused_sync_ints(int max_rows) { return kSyncReady + (max_rows + kBM - 1) / kBM + kMaxExpertsLocal + 1; }

size_t ffn_h_bytes(int max_rows, int inter, cap_dtype dt) {
    const size_t h = static_cast<size_t>(max_rows) * inter * (dt == CAP_DTYPE_BF16 ? 2 : 4);
    return (h + 255) & ~static_cast<size_t>(255);
}

}  // namespace

// Workspace: H [max_rows][inter], then (bf16) the fused kernel's counters.
size_t ffn_workspace_bytes(int max_rows, int inter, cap_dtype dt) {
    return ffn_h_bytes(max_rows, inter, dt) + (dt == CAP_DTYPE_BF16 ? sizeof(int) * fused_sync_ints(max_rows) : 0);
}

// bf16: d and inter up to 2^19, so that a tile's 256 rows of K = d or inter
// (2^28 bytes) stay far inside the direct loads' 32-bit lane offsets.
cap_status ffn_supported(cap_dtype dt, int d, int inter) {
    if (dt == CAP_DTYPE_BF16)
        return (d % kBN == 0 && inter % (kBN / 2) == 0 && d <= (1 << 19) && inter <= (1 << 19)) ? CAP_OK
                                                                                              : CAP_ERR_UNSUPPORTED;
    return (d % 4 == 0) ? CAP_OK : CAP_ERR_UNSUPPORTED;
}

// row_src == nullptr: xs holds the expert-sorted rows; otherwise row i is
// xs[row_src[i]] and xs has x_rows rows.  row_dst != nullptr (bf16 only): the
// destination combine of single-expert tokens goes into the down GEMM's
// epilogue (row_dst, row_w, parts, parts_rows: CombinePlan).
cap_status expert_ffn_launch(cap_dtype dt, int E_loc, int d, int inter, int max_rows, const void* xs, int x_rows,
                             const int32_t* row_src, const int32_t* row_offsets, const void* w1, const void* w3,
                             const void* w2, void* y, void* ws, const cap_ffn_options* opt, hipStream_t st,
                             const int32_t* row_dst, const float* row_w, void* parts, int parts_rows) {
    const CombinePlan cp{row_dst, row_w, static_cast<uint16_t*>(parts), parts_rows};
    const CombinePlan none{nullptr, nullptr, nullptr, 0};
    if (dt == CAP_DTYPE_BF16) {
        const auto* a = static_cast<const uint16_t*>(xs);
        const auto* b1 = static_cast<const uint16_t*>(w1);
        const auto* b3 = static_cast<const uint16_t*>(w3);
        const auto* b2 = static_cast<const uint16_t*>(w2);
        auto* h = static_cast<uint16_t*>(ws);
        auto* out = static_cast<uint16_t*>(y);
        // The fused kernel maps XCC_ID % n_xcc to a queue: with 8 XCCs the ids
        // are 0..7 (one per XCD); with one XCC all CUs share one L2.  Other
        // partitions take the two-kernel path, which needs no such mapping.
        const int n_xcc = device_xcc_count();
        // narrow tiles are for calls without the options that drive the fused
        // kernel's grid and waits (0: not allowed)
        const int cus = opt && (opt->max_workgroups > 0 || opt->force_wait_timeout) ? 0 : device_cu_count();
        auto gate_up = [&](int g, int* sync, int n_sync) {
            if (row_src)
                ffn_gemm_bf16_kernel<true, true><<<g, kNW * kWave, 0, st>>>(
                    a, b1, b3, h, row_offsets, E_loc, max_rows, d, inter, row_src, x_rows, none, cus, sync, n_sync);
            else
                ffn_gemm_bf16_kernel<true, false><<<g, kNW * kWave, 0, st>>>(
                    a, b1, b3, h, row_offsets, E_loc, max_rows, d, inter, nullptr, 0, none, cus, sync, n_sync);
        };
        if (max_rows >= kFusedMinRows && (n_xcc == kMaxXcc || n_xcc == 1)) {
            int* sync = reinterpret_cast<int*>(static_cast<char*>(ws) + ffn_h_bytes(max_rows, inter, dt));
            int g = persistent_grid(1ll << 30);
            // first launch: clears the counters (a kernel rather than a memset,
            // so that captured graphs hold no memset node) and, if the call
            // runs on narrow tiles, does its gate/up GEMM
            gate_up(g, sync, fused_sync_ints(max_rows));
            CAP_LAUNCH_CHECK();
            // a caller's cap on the grid (with fewer workgroups than XCDs
            // the last one runs the untouched queues)
            if (opt && opt->max_workgroups > 0 && opt->max_workgroups < g) g = opt->max_workgroups;
            int* err = (opt && opt->wait_errors) ? opt->wait_errors : sync + kSyncErr;
            const int spin = (opt && opt->spin_limit > 0) ? opt->spin_limit : kSpinLimit;
            const int bias = (opt && opt->force_wait_timeout) ? 1 : 0;
            if (row_src)
                ffn_fused_bf16_kernel<true><<<g, kNW * kWave, 0, st>>>(a, b1, b3, b2, h, out, row_offsets, E_loc,
                                                                       max_rows, d, inter, row_src, x_rows, n_xcc, sync,
                                                                       err, spin, bias, cp, cus);
            else
                ffn_fused_bf16_kernel<false><<<g, kNW * kWave, 0, st>>>(a, b1, b3, b2, h, out, row_offsets, E_loc,
                                                                        max_rows, d, inter, nullptr, 0, n_xcc, sync,
                                                                        err, spin, bias, cp, cus);
            CAP_LAUNCH_CHECK();
            return CAP_OK;
        }
        const long long mt_upper = (static_cast<long long>(max_rows) + 63) / 64 + E_loc;
        gate_up(persistent_grid(mt_upper * (inter / (kNbN / 2))), nullptr, 0);
        CAP_LAUNCH_CHECK();
        const int g2 = persistent_grid(mt_upper * (d / kNbN));
        ffn_gemm_bf16_kernel<false, false><<<g2, kNW * kWave, 0, st>>>(h, b2, nullptr, out, row_offsets, E_loc,
                                                                       max_rows, inter, d, nullptr, 0, cp, cus,
                                                                       nullptr, 0);
        CAP_LAUNCH_CHECK();
    } else {
        launch_ffn_f32<true>(static_cast<const float*>(xs), static_cast<const float*>(w1), static_cast<const float*>(w3),
                             static_cast<float*>(ws), row_offsets, E_loc, max_rows, d, inter, row_src, x_rows, st);
        CAP_LAUNCH_CHECK();
        launch_ffn_f32<false>(static_cast<const float*>(ws), static_cast<const float*>(w2), nullptr,
                              static_cast<float*>(y), row_offsets, E_loc, max_rows, inter, d, nullptr, 0, st);
        CAP_LAUNCH_CHECK();
    }
    return CAP_OK;
}

}  // namespace cap
