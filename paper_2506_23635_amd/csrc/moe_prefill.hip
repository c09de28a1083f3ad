// moe_prefill.hip -- the expert FFN for many tokens (prefill): a grouped GEMM
// on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16).
//
// A workgroup computes a BM x BN = 256 x 256 tile of C = W X^T for one
// expert: W (the A operand) is 256 output features of the expert's packed
// weights, X (the B operand) is 256 of the expert's token rows (K
// contiguous).  Four waves split the features (4 x 64); each wave owns a
// 64-feature x 256-token block (2 x 8 MFMA blocks of 32 x 32, all 256
// accumulator registers), so each weight slab is re-read by only
// ceil(tokens / 256) workgroups.  One workgroup per CU (128 KiB of LDS),
// one wave per SIMD: latency is hidden by software pipelining alone.
//
//  - A never touches LDS: the packed layout already holds every 32 x 16
//    fragment as 1 KiB in lane order, each fragment is used by exactly one
//    wave, and the wave loads it straight into registers through a ring of
//    three 64-wide K stages.
//  - B (the gathered token rows, shared by all four waves) goes from HBM to
//    LDS by buffer loads with the LDS-direct option, four stages deep; each
//    load reads whole 128-byte lines and the chunks of each row are
//    XOR-swizzled in LDS so that the fragment reads are conflict-free.  The
//    fragments are read into a small register window a few MFMAs ahead,
//    also across stage boundaries.
//  - An expert's partial last token tile skips the MFMAs of token-block
//    pairs past its last row (the padding waste is under 64 rows).
//  - Workgroups are numbered so that consecutive tiles (same weight slab,
//    consecutive token tiles) land on the same XCD and share its L2
//    (find_tile).
//
// gemm<kGateUp>: A = GU slab (gate and up row tiles interleaved), X = the
//   expert's rows of x gathered through row_token; epilogue
//   H = bf16(silu(G) * U) (paper Table tab:vars (e): w1 gate, v1 up).
// gemm<kDown>:   A = DN slab, X = the expert's rows of H; epilogue O fp32.
//
// Token tiles come from the routing's row offsets; the grid is sized for the
// worst case and surplus workgroups, all at its end, exit at once.  Few rows
// per expert take smaller tiles (gemm_mid_kernel below).
#include <algorithm>
#include <type_traits>

#include "moe_common.h"

namespace moe {

constexpr int BM = 256;         // features per workgroup tile
constexpr int BN = 256;         // token rows per workgroup tile
constexpr int BK = 64;          // K per stage (four 16-K MFMA steps)
constexpr int kThreads = 256;   // 4 waves, one per 64-feature slab
constexpr int FB = 2;           // 32-feature MFMA blocks per wave
constexpr int kWaveRt = 2 * FB; // 16-row weight tiles per wave
constexpr int TB = BN / 32;     // 32-token MFMA blocks per tile
constexpr int KS = BK / 16;     // 16-K MFMA steps per stage
constexpr int kRingA = 3;       // register ring of A stages
constexpr int kRingB = 4;       // LDS ring of B stages
constexpr int A_FRAGS = FB * KS;                  // 8 A fragments per wave per stage
constexpr int B_FRAGS = TB * KS;                  // 32 B fragments per stage
constexpr int B_LOADS = B_FRAGS * 64 / kThreads;  // 8 per thread
constexpr int B_STAGE_BYTES = B_FRAGS * kTileBytes;  // 32 KiB
constexpr int kXcds = 8;
constexpr int kBufferFlags = 0x00020000;   // buffer descriptor word 3 (raw dword data, gfx9 family)
constexpr int kNonTemporal = 2;              // buffer cache policy
constexpr int kWaitAll = (0x7 << 4) | (0xF << 8);   // vmcnt 0
static_assert(kRingA == 3, "the K loop is unrolled by three stages");
static_assert(kRingB == 4, "stage s reads B(s), publishes B(s+1), loads B(s+2)");

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

__device__ inline f32x16_t mfma32x32x16(const u32x4_t a, const u32x4_t b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// What a tile's sums become: kGateUp H, kDown O; the plain products of the
// attention block are kDown with their own ends (kQkv, kOut).
enum { kGateUp = 0, kDown = 1, kQkv = 2, kOut = 3 };

// chunk swizzle of B row R in LDS (a function of R mod 16 only, so 32-row
// token blocks share it): rows 0..7 take eight distinct slots, and rows
// 8..15 the complementary (row parity, slot) pairs, so any 8 consecutive
// rows or 16 consecutive rows at one chunk hit distinct banks
__device__ __forceinline__ int b_swizzle(int R) { return (R & 7) ^ ((R >> 3) & 1); }

struct TileCtx {
    __amdgpu_buffer_rsrc_t a_rsrc;  // buffer over the expert's packed slab (GU or DN)
    uint32_t a_off[FB];        // this lane's A byte offset per feature block (stage 0, step 0)
    __amdgpu_buffer_rsrc_t b_rsrc;  // buffer over x (gate/up) or over the tile's rows of H
    uint32_t b_off[B_LOADS];   // byte offsets in b_rsrc of this lane's 16-byte chunk, per load
    uint32_t rd_off[KS];       // LDS byte offsets of this lane's B fragment piece, per K step
    int n_stages;
    int w, lane;
};

// The K loop of one tile on v_mfma_f32_32x32x16_bf16.  A 32 x 16 operand
// fragment is 1 KiB in lane order (lane l: row l%32, K 8(l/32)..+7).
//
// A stage is 32 units (16-K step j, 32-token block t), j-major; a unit is
// one B fragment read from LDS and the two MFMAs (both feature blocks) that
// use it.  B fragments are read kLook units ahead through a small register
// window, also across stage boundaries: the barrier that publishes the next
// stage's B sits kLook units before the end of the current stage.
//
// The global loads are spread over the units (a burst of them would stall
// the wave's in-order issue behind the address unit): stage s issues load q
// of B(s+2) at unit 4q + 1 (into the LDS buffer that stage s-2 used, free
// since stage s-1's barrier), and refills A fragment (fb, j) with A(s+3) two
// units after the last MFMA that reads it.
// kFull: every token block holds rows (branch-free loop); otherwise only the
// first n_pairs pairs of token blocks run their MFMAs.
constexpr int kUnits = KS * TB;   // 32 units per stage
constexpr int kLook = 3;          // B fragments in flight ahead of their MFMAs
constexpr int kWin = kLook + 1;   // B register window
constexpr int kBarrierUnit = kUnits - kLook;
static_assert(kUnits % kWin == 0, "the window index must repeat per stage");
static_assert(kUnits == 4 * B_LOADS, "one B load every four units");

// the unit at which stage s issues B load q of B(s+2)
constexpr int b_load_unit(int q) { return 4 * q + 1; }
// the unit at which stage s refills A fragment (fb, j) with A(s+3): the
// units of K step j are 8j .. 8j+7; the last K step's fragments go after
// the stage (unit kUnits)
constexpr int a_load_unit(int fb, int j) { return j + 1 < KS ? 8 * (j + 1) + 2 * fb : kUnits; }
// vector-memory ops issued after the last load of B(s+1) (stage s-1, unit
// b_load_unit(B_LOADS-1)) up to stage s's barrier; vector-memory ops
// complete in order, so waiting until at most this many are outstanding
// means this wave's part of B(s+1) is in LDS.  The stages after the main
// loop (kTail) issue no A refills: their registers are never read again, and
// the compiler would drop them as dead loads anyway.  The stage before a tail
// stage may be one too, so there only the stage's own B loads before the
// barrier are certain to follow B(s+1).
constexpr int vm_after_last_b(bool kTail)
{
    int n = 0;
    for (int q = 0; q < B_LOADS; ++q)
        if (b_load_unit(q) < kBarrierUnit) ++n;
    if (kTail) return n;
    for (int fb = 0; fb < FB; ++fb)
        for (int j = 0; j < KS; ++j) {
            const int u = a_load_unit(fb, j);
            if (u > b_load_unit(B_LOADS - 1)) ++n;   // rest of stage s-1
            if (u < kBarrierUnit) ++n;               // stage s before the barrier
        }
    return n;
}
static_assert(b_load_unit(B_LOADS - 1) >= kBarrierUnit, "every B(s+1) load precedes the count");
static_assert(vm_after_last_b(false) < 64, "vmcnt holds 6 bits");
// s_waitcnt immediate (gfx9 layout: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] |
// vmcnt[15:14])
constexpr int wait_vm(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }
constexpr int kWaitBStage = wait_vm(vm_after_last_b(false));
constexpr int kWaitBTail = wait_vm(vm_after_last_b(true));

template <bool kFull>
__device__ __forceinline__ void tile_loop(const TileCtx& c, int n_pairs, uint8_t* lds,
                                          f32x16_t (&acc)[FB][TB])
{
    const int n_stages = c.n_stages;
    const int w = c.w;
    u32x4_t ra[kRingA][A_FRAGS];
    u32x4_t bw[kWin];
    // A fragment (fb, j) of stage s: K step j lives in K tile 2s + j/2,
    // second half of the tile for odd j (512 bytes on)
    auto load_a1 = [&](int s, int fb, int j, u32x4_t& dst) {
        dst = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                              c.a_rsrc, c.a_off[fb] + (j / 2) * kTileBytes + (j % 2) * (kTileBytes / 2),
                                              (uint32_t)s * (2 * kTileBytes), 0));
    };
    // B goes global -> LDS directly through buffer loads: a stage of B is
    // 256 rows x 128 bytes (64 K), row-major in LDS with the eight 16-byte
    // chunks of each row XOR-swizzled (see process_tile).  Load q of wave w
    // fills rows 64w + 8q .. +7, so every load reads whole 128-byte lines.
    // Buffer (not global) loads: the compiler counts them in vmcnt only, so
    // the LDS reads of the B window keep exact lgkmcnt waits.
    auto load_b1 = [&](int s, int buf, int q) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            c.b_rsrc,
            (__attribute__((address_space(3))) void*)(&lds[buf * B_STAGE_BYTES +
                                                           (w * B_LOADS + q) * kTileBytes]),
            16, c.b_off[q], (uint32_t)s * (BK * 2), 0, 0);
    };
    // the B fragment of unit u: token block t (rows 32t..), K step j
    auto read_unit = [&](const uint8_t* bbuf, int u) {
        const int j = u / TB, t = u % TB;
        bw[u % kWin] = *reinterpret_cast<const u32x4_t*>(&bbuf[c.rd_off[j] + t * 32 * (BK * 2)]);
    };
    // explicit partial wait + bare barrier: a __syncthreads() release fence
    // would wait for every outstanding LDS DMA (vmcnt 0); the empty asm
    // statements keep the compiler from moving memory operations across it
    auto wait_and_barrier = [&](auto tail) {
        __builtin_amdgcn_s_waitcnt(decltype(tail)::value ? kWaitBTail : kWaitBStage);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // stage s (A in A, B in LDS buffer s % 4).  B loads past the last stage
    // re-read the last stage into buffers no stage reads; A refills are
    // issued in the main loop only (tail is std::true_type after it).
    auto stage = [&](int s, u32x4_t (&A)[A_FRAGS], auto tail) {
        constexpr bool kTail = decltype(tail)::value;
        const uint8_t* bcur = lds + (s % kRingB) * B_STAGE_BYTES;
        const uint8_t* bnext = lds + ((s + 1) % kRingB) * B_STAGE_BYTES;
        const int sb = min(s + 2, n_stages - 1), bbuf = (s + 2) % kRingB;
        const int sa = min(s + kRingA, n_stages - 1);
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            if (u == kBarrierUnit) wait_and_barrier(tail);
            if (u % 4 == 1) load_b1(sb, bbuf, u / 4);
#pragma unroll
            for (int fb = 0; fb < FB; ++fb)
#pragma unroll
                for (int j = 0; j < KS; ++j)
                    if (!kTail && a_load_unit(fb, j) == u) load_a1(sa, fb, j, A[fb * KS + j]);
            if (u + kLook < kUnits)
                read_unit(bcur, u + kLook);
            else
                read_unit(bnext, u + kLook - kUnits);
            __builtin_amdgcn_sched_barrier(0);
            const int j = u / TB, t = u % TB;
            if (kFull || t / 2 < n_pairs) {
#pragma unroll
                for (int fb = 0; fb < FB; ++fb)
                    acc[fb][t] = mfma32x32x16(A[fb * KS + j], bw[u % kWin], acc[fb][t]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int j = 0; j < KS; ++j)
                if (!kTail && a_load_unit(fb, j) == kUnits) load_a1(sa, fb, j, A[fb * KS + j]);
    };

    // prologue: B(0), B(1) and A(0..2); wait for them, then read the first
    // kLook units of stage 0
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < B_LOADS; ++q) load_b1(min(i, n_stages - 1), i, q);
#pragma unroll
    for (int i = 0; i < kRingA; ++i)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int j = 0; j < KS; ++j) load_a1(min(i, n_stages - 1), fb, j, ra[i][fb * KS + j]);
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < kLook; ++u) read_unit(lds, u);
    // three stages per iteration, so that the A ring is indexed statically
    int s = 0;
    for (; s + kRingA <= n_stages; s += kRingA) {
        stage(s + 0, ra[0], std::false_type{});
        stage(s + 1, ra[1], std::false_type{});
        stage(s + 2, ra[2], std::false_type{});
    }
    if (s < n_stages) {
        stage(s, ra[0], std::true_type{});
        if (s + 1 < n_stages) stage(s + 1, ra[1], std::true_type{});
    }
    // the last stages re-issued dummy B loads into LDS: drain them before the
    // workgroup can finish and its LDS be handed to another workgroup
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
}

// A tile of at most 128 token rows (kTB 32-token blocks; an expert's only
// or last tile).  With half of the accumulators free the wave keeps kRingH
// stages of A in flight instead of three: a tile with few rows is bound by
// the latency of its weight stream, not by its MFMAs (three stages: a 64-row
// tile took 121 us of a full one's 155; whole layer at 500 tokens, d 6144, f
// 10752: 1332 -> 1263 us, 400: 1241 -> 1174; no change from 700 tokens on).  B fragments are read one K step
// ahead, across stages too: before the last K step the wave waits for its
// own reads of the stage's buffer and for its part of B(s+1), then a barrier
// publishes both.  At its start stage s issues B(s+3) into the buffer that
// stage s-1 read; A(s + kRingH) refills each fragment after its last use, in
// every stage (past the end it re-reads the last stage), so that the counts
// hold throughout: after B(s+1), issued at the start of stage s-2, came that
// stage's A refills, the B loads and A refills of stage s-1, and the B loads
// and the first three K steps' refills of stage s.
constexpr int kRingH = 6;
constexpr int kHalfTB = TB / 2;

template <int kTB, bool kOnce>
__device__ __forceinline__ void half_loop(const TileCtx& c, uint8_t* lds, f32x16_t (&acc)[FB][kHalfTB])
{
    constexpr int kStage = kTB * 32 * BK * 2;
    constexpr int kWait = wait_vm(2 * kTB + 3 * A_FRAGS - FB);
    static_assert(2 * kTB + 3 * A_FRAGS - FB < 64, "vmcnt holds 6 bits");
    const int n_stages = c.n_stages, w = c.w;
    u32x4_t ra[kRingH][A_FRAGS];
    auto load_a1 = [&](int s, int fb, int j, u32x4_t& dst) {
        dst = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                              c.a_rsrc, c.a_off[fb] + (j / 2) * kTileBytes + (j % 2) * (kTileBytes / 2),
                                              (uint32_t)s * (2 * kTileBytes), kOnce ? kNonTemporal : 0));
    };
    // load q of wave w: rows 32 q + 8 w .. + 7, whole 128-byte lines
    auto load_b = [&](int s, int buf) {
#pragma unroll
        for (int q = 0; q < kTB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                c.b_rsrc, (__attribute__((address_space(3))) void*)(&lds[buf + (q * 4 + w) * kTileBytes]),
                16, c.b_off[q], (uint32_t)s * (BK * 2), 0, 0);
    };
    u32x4_t bw[2][kTB];                        // B fragments of two K steps in turn
    auto read_b = [&](int buf, int j, u32x4_t (&dst)[kTB]) {
#pragma unroll
        for (int t = 0; t < kTB; ++t)
            dst[t] = *reinterpret_cast<const u32x4_t*>(&lds[buf + c.rd_off[j] + t * 32 * (BK * 2)]);
    };
    int cur = 0, prev = (kRingB - 1) * kStage;   // byte offsets of this and the last stage's buffer
    auto stage = [&](int s, u32x4_t (&A)[A_FRAGS]) {
        const int next = cur + kStage == kRingB * kStage ? 0 : cur + kStage;
        const int sa = min(s + kRingH, n_stages - 1);
        load_b(min(s + kRingB - 1, n_stages - 1), prev);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            if (j + 1 == KS) {
                __builtin_amdgcn_s_waitcnt(kWait & ~(0xF << 8));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                read_b(next, 0, bw[0]);
            } else {
                read_b(cur, j + 1, bw[(j + 1) & 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < kTB; ++t)
#pragma unroll
                for (int fb = 0; fb < FB; ++fb)
                    acc[fb][t] = mfma32x32x16(A[fb * KS + j], bw[j & 1][t], acc[fb][t]);
#pragma unroll
            for (int fb = 0; fb < FB; ++fb) load_a1(sa, fb, j, A[fb * KS + j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev = cur;
        cur = next;
    };
#pragma unroll
    for (int i = 0; i < kRingH; ++i)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int j = 0; j < KS; ++j) load_a1(min(i, n_stages - 1), fb, j, ra[i][fb * KS + j]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i + 1 < kRingB; ++i) load_b(min(i, n_stages - 1), i * kStage);
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_b(0, 0, bw[0]);
    for (int s = 0; s < n_stages; s += kRingH) {
        stage(s, ra[0]);
        if (s + 1 < n_stages) stage(s + 1, ra[1]);
        if (s + 2 < n_stages) stage(s + 2, ra[2]);
        if (s + 3 < n_stages) stage(s + 3, ra[3]);
        if (s + 4 < n_stages) stage(s + 4, ra[4]);
        if (s + 5 < n_stages) stage(s + 5, ra[5]);
    }
    // drain the dummy loads before the epilogue takes the LDS
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
}

// barrier for LDS traffic only: this wave's LDS operations are done, its
// global stores may still be on their way
__device__ __forceinline__ void lds_barrier()
{
    constexpr int kWaitLgkm = 0xC07F;   // lgkmcnt 0; vmcnt and expcnt at their maxima
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The end of a tile: kBlocks 32-feature blocks per wave (four waves, wave w
// from row tile rt0 + 2 kBlocks w on) of up to kTBs 32-token blocks, token
// rows row_start .. row_end - 1.  In a block the lane holds token lane % 32
// and features 8g + 4 (lane / 32) + r in register 4g + r (g, r = 0..3).
//
// The sums go through LDS (free after the K loop), so that the workgroup
// writes whole token rows: straight from the registers a store covers 16 or
// 32 bytes of each of 32 rows, and with one workgroup per CU nothing hides
// it (q|k|v of 2048 tokens, rotated here: 197 us from the registers).
//  kGateUp  the block is 16 gate rows (g = 0, 1) and the 16 up rows of the
//           same features (g = 2, 3): H = bf16(silu(G) U), all rows at once
//  kDown    O (fp32), at the K range's offset; here and below 32 token rows
//           at a time, through two buffers in turn
//  kQkv     a row tile of a query or key head holds 8 rotation pairs, the
//           first members in rows 0..7 and the second in rows 8..15 (the
//           packing of rope_row): the fp32 values in natural order, rotated
//           with the token's cos and sin, bf16 q to the workspace, k and v to
//           the cache.  (A kernel of its own read and wrote the product once
//           more: 45 us at 2048 tokens.)  Value rows keep their order, so
//           their "pairs" are 8 features apart and stay unrotated.
//  kOut     o (fp32) and y = bf16(x + o) (x and y may be the same array)
template <int kMode, int kBlocks, int kTBs>
__device__ __forceinline__ void store_tile(const GemmArgs& a, const f32x16_t (&acc)[kBlocks][kTBs],
                                           uint8_t* lds, int rt0, int row_start, int row_end, int w,
                                           int lane, int split)
{
    constexpr int kFeat = 4 * kBlocks * 32;   // features of the workgroup
    const int half = lane >> 5, c = lane & 31, tid = w * 64 + lane;
    const int rows = row_end - row_start;
    if constexpr (kMode == kGateUp) {
        constexpr int kRow = kFeat + 16;      // bytes of a token's H features in LDS, padded
        constexpr int kPieces = kFeat / 16;   // 16-byte pieces of them
#pragma unroll
        for (int t = 0; t < kTBs; ++t) {
            if (t * 32 >= rows) break;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) {
                const f32x16_t v = acc[b][t];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const uint32_t h01 = cvt_pk_bf16(silu_mul(v[4 * g + 0], v[4 * g + 8]),
                                                     silu_mul(v[4 * g + 1], v[4 * g + 9]));
                    const uint32_t h23 = cvt_pk_bf16(silu_mul(v[4 * g + 2], v[4 * g + 10]),
                                                     silu_mul(v[4 * g + 3], v[4 * g + 11]));
                    *reinterpret_cast<uint2*>(
                        &lds[(t * 32 + c) * kRow + ((w * kBlocks + b) * 16 + 8 * g + 4 * half) * 2]) =
                        make_uint2(h01, h23);
                }
            }
        }
        lds_barrier();
#pragma unroll 4
        for (int e = tid; e < rows * kPieces; e += kThreads) {
            const int r = e / kPieces, p = e % kPieces;
            *reinterpret_cast<u32x4_t*>(a.H + (int64_t)(row_start + r) * a.f + rt0 * 8 + p * 8) =
                *reinterpret_cast<const u32x4_t*>(&lds[r * kRow + p * 16]);
        }
    } else {
        constexpr int kRow = kFeat * 4 + 16;  // bytes of a token's sums in LDS, padded
        // pieces of a token's row: 8 packed features (4 + 4 of a row tile) or
        // 4; kIters of the 32 rows' pieces per thread
        constexpr int kPieces = kFeat / (kMode == kQkv ? 8 : 4);
        constexpr int kIters = 32 * kPieces / kThreads;
        const int p = tid % kPieces, r0 = tid / kPieces;   // piece, first row
        constexpr int kStep = kThreads / kPieces;          // rows between a thread's pieces
        const int n0 = (rt0 + p / 2) * kTileRows, head = kMode == kQkv ? n0 / a.hd : 0;
        const int hd = a.hd, e0 = kMode == kQkv ? n0 % hd : 0;
        const bool turn = kMode == kQkv && head < a.heads + a.kv_heads;
        const int f0 = (turn ? e0 / 2 : e0) + p % 2 * 4, gap = turn ? hd / 2 : 8;
        // what the pieces need from memory, loaded a pass ahead: the tokens'
        // cos and sin, or x (rows past the end: the last row's)
        float4 cs[2][kMode == kQkv ? kIters : 1][2];
        uint2 xr[2][kMode == kOut ? kIters : 1];
        auto fetch = [&](int t) {
#pragma unroll
            for (int i = 0; i < kIters; ++i) {
                const int64_t row = min(row_start + t * 32 + r0 + i * kStep, row_end - 1);
                if constexpr (kMode == kQkv) {
                    const float* src = a.cos_sin + (row * (hd / 2) + (turn ? f0 : 0)) * 2;
                    cs[t % 2][i][0] = *reinterpret_cast<const float4*>(src);
                    cs[t % 2][i][1] = *reinterpret_cast<const float4*>(src + 4);
                }
                if constexpr (kMode == kOut)
                    xr[t % 2][i] = *reinterpret_cast<const uint2*>(a.res + row * a.d + rt0 * kTileRows + p * 4);
            }
        };
        fetch(0);
#pragma unroll
        for (int t = 0; t < kTBs; ++t) {
            if (t * 32 >= rows) break;
            uint8_t* buf = lds + t % 2 * (32 * kRow);
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4*>(&buf[c * kRow + ((w * kBlocks + b) * 32 + 8 * g + 4 * half) * 4]) =
                        make_float4(acc[b][t][4 * g], acc[b][t][4 * g + 1], acc[b][t][4 * g + 2],
                                    acc[b][t][4 * g + 3]);
            lds_barrier();
            if (t + 1 < kTBs) fetch(t + 1);
#pragma unroll
            for (int i = 0; i < kIters; ++i) {
                const int r = r0 + i * kStep, row = row_start + t * 32 + r;
                if (row >= row_end) continue;
                if constexpr (kMode == kQkv) {
                    const uint8_t* src = &buf[r * kRow + (p / 2 * 16 + p % 2 * 4) * 4];
                    const float4 x0 = *reinterpret_cast<const float4*>(src);
                    const float4 x1 = *reinterpret_cast<const float4*>(src + 32);
                    const float4 c01 = cs[t % 2][i][0], c23 = cs[t % 2][i][1];
                    float4 y0 = x0, y1 = x1;
                    if (turn) {
                        y0 = make_float4(x0.x * c01.x - x1.x * c01.y, x0.y * c01.z - x1.y * c01.w,
                                         x0.z * c23.x - x1.z * c23.y, x0.w * c23.z - x1.w * c23.w);
                        y1 = make_float4(x1.x * c01.x + x0.x * c01.y, x1.y * c01.z + x0.y * c01.w,
                                         x1.z * c23.x + x0.z * c23.y, x1.w * c23.z + x0.w * c23.w);
                    }
                    float* nat = a.O + (int64_t)row * a.d + head * hd + f0;
                    *reinterpret_cast<float4*>(nat) = x0;
                    *reinterpret_cast<float4*>(nat + gap) = x1;
                    uint16_t* dst =
                        head < a.heads ? a.q + ((int64_t)row * a.heads + head) * hd
                        : turn ? a.kc + ((int64_t)(head - a.heads) * a.max_seq + a.pos0 + row) * hd
                               : a.vc + ((int64_t)(head - a.heads - a.kv_heads) * a.max_seq + a.pos0 + row) * hd;
                    *reinterpret_cast<uint2*>(dst + f0) =
                        make_uint2(cvt_pk_bf16(y0.x, y0.y), cvt_pk_bf16(y0.z, y0.w));
                    *reinterpret_cast<uint2*>(dst + f0 + gap) =
                        make_uint2(cvt_pk_bf16(y1.x, y1.y), cvt_pk_bf16(y1.z, y1.w));
                } else {
                    const int64_t at = (int64_t)row * a.d + rt0 * kTileRows + p * 4;
                    const float4 v = *reinterpret_cast<const float4*>(&buf[r * kRow + p * 16]);
                    *reinterpret_cast<float4*>(a.O + (uint64_t)split * a.split_stride + at) = v;
                    if constexpr (kMode == kOut) {
                        const uint2 x = xr[t % 2][i];
                        *reinterpret_cast<uint2*>(a.y16 + at) =
                            make_uint2(cvt_pk_bf16(__uint_as_float(x.x << 16) + v.x,
                                                   __uint_as_float(x.x & 0xFFFF0000u) + v.y),
                                       cvt_pk_bf16(__uint_as_float(x.y << 16) + v.z,
                                                   __uint_as_float(x.y & 0xFFFF0000u) + v.w));
                    }
                }
            }
        }
    }
}

// One BM x BN tile (feature tile ft, token tile tt) of the grouped GEMM.
template <int kMode>
__device__ __forceinline__ void process_tile(const GemmArgs& a, int e, int row_start, int row_end, bool once, int ft, uint8_t* lds)
{
    const int ntb = (row_end - row_start + 31) / 32;   // 32-token blocks with rows
    const bool half = ntb <= kHalfTB;                  // half_loop's tile

    const int K = kMode == kGateUp ? a.d : a.f;
    const uint64_t KT = (uint64_t)K / kTileK;
    const uint8_t* wbase = a.experts + (uint64_t)(e - a.e_begin) * a.expert_bytes +
                           (kMode == kGateUp ? 0 : a.gu_bytes);

    TileCtx c;
    c.n_stages = K / BK;
    c.lane = threadIdx.x & 63;
    c.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, in an SGPR
    const int lane = c.lane, w = c.w;
    // M is a multiple of BM (the library requires d % 256 == 0 and
    // f % 128 == 0), so every wave's 64-feature slab lies inside the matrix
    const uint64_t rt0 = (uint64_t)ft * (BM / 16) + w * kWaveRt;
    // A: lane l of a 32 x 16 fragment reads row l%32 of the block (row tile
    // rt0 + 2 fb + (l%32)/16, granule row l%16) at K group l/32 of the step.
    // Buffer loads over the expert's slab (the library caps a slab below
    // 2^31 bytes, so offsets fit 32 bits; the size bounds every load).
    const uint64_t slab_bytes = kMode == kGateUp ? a.gu_bytes : a.expert_bytes - a.gu_bytes;
    c.a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wbase), 0, (int)slab_bytes,
                                                 kBufferFlags);
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
        c.a_off[fb] = (uint32_t)tile_offset(rt0 + 2 * fb + ((lane & 31) >> 4), 0, KT) +
                      (uint32_t)(((lane >> 5) * 16) + (lane & 15)) * 16;
    // B: a stage holds, for each of the 256 token rows R of the tile, the
    // 128 bytes of K [64 s, 64 s + 64) as eight 16-byte chunks; chunk c sits
    // in slot c ^ swz(R) so that the MFMA reads (8 consecutive rows at one
    // chunk) fall in distinct LDS banks.  Load q of wave w: lane l reads row
    // R = 64w + 8q + l/8 (a tile of at most
    // 128 rows: R = 32q + 8w + l/8), slot l%8, i.e. chunk (l%8) ^ swz(R).  Gate/up
    // gathers rows of x (the library caps T*d*2 below 2^31, so byte offsets
    // fit 32 bits); down reads the tile's own rows of H through a buffer
    // based at the tile's first row.  The buffer size bounds every load
    // (out-of-range reads return zero).
    if (kMode == kGateUp)
        c.b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.x), 0,
                                                     a.T * a.d * 2, kBufferFlags);
    else
        c.b_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.H + (int64_t)row_start * a.f, 0,
                                                     (row_end - row_start) * a.f * 2, kBufferFlags);
#pragma unroll
    for (int q = 0; q < B_LOADS; ++q) {
        const int R = half ? q % 4 * 32 + w * 8 + (lane >> 3) : w * 64 + q * 8 + (lane >> 3);
        const int row = row_start + R;
        const int rr = row < row_end ? row : row_start;   // rows past the end: any valid row
        const uint32_t chunk = (uint32_t)((lane & 7) ^ b_swizzle(R)) * 16;
        if (kMode == kGateUp)
            c.b_off[q] = (uint32_t)a.row_token[rr] * (uint32_t)a.d * 2 + chunk;
        else
            c.b_off[q] = (uint32_t)(rr - row_start) * (uint32_t)a.f * 2 + chunk;
    }
    // MFMA B operand of K step j, token block t: lane l takes row
    // R = 32t + l%32, chunk 2j + l/32 (swz(R) does not depend on t)
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        const int R = lane & 31;
        c.rd_off[j] = (uint32_t)R * (BK * 2) + (uint32_t)(((2 * j + (lane >> 5)) ^ b_swizzle(R)) * 16);
    }

    if (half) {
        f32x16_t acc[FB][kHalfTB];
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int tb = 0; tb < kHalfTB; ++tb) acc[fb][tb] = f32x16_t{};
        if (ntb <= 2)
            once ? half_loop<2, true>(c, lds, acc) : half_loop<2, false>(c, lds, acc);
        else
            once ? half_loop<4, true>(c, lds, acc) : half_loop<4, false>(c, lds, acc);
        store_tile<kMode, FB, kHalfTB>(a, acc, lds, ft * (BM / 16), row_start, row_end, w, lane, 0);
        return;
    }
    f32x16_t acc[FB][TB];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[fb][tb] = f32x16_t{};

    // full tiles take the branch-free loop; an expert's partial last tile
    // skips the MFMAs of token-block pairs past its last row
    if (ntb == TB)
        tile_loop<true>(c, TB / 2, lds, acc);
    else
        tile_loop<false>(c, (ntb + 1) / 2, lds, acc);

    store_tile<kMode, FB, TB>(a, acc, lds, ft * (BM / 16), row_start, row_end, w, lane, 0);
}

// Measurement only (a.stamps, set by moe_profile_gemm_timeline): workgroup
// blockIdx.x's record of one tile, [0], [1] the constant 100 MHz counter and
// [2], [3] the shader-clock counter around the tile.
__device__ __forceinline__ void write_stamp(const GemmArgs& a, uint64_t r0, uint64_t c0, int ft,
                                            int tt, int rows, int e)
{
    __syncthreads();
    if (threadIdx.x != 0) return;
    const uint64_t r1 = __builtin_amdgcn_s_memrealtime();
    const uint64_t c1 = __builtin_amdgcn_s_memtime();
    uint32_t hw, xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    uint64_t* out = a.stamps + (uint64_t)blockIdx.x * 8;
    out[0] = r0;
    out[1] = r1;
    out[2] = c0;
    out[3] = c1;
    out[4] = (uint64_t)hw | ((uint64_t)xcc << 32);
    out[5] = (uint64_t)ft | ((uint64_t)tt << 16) | ((uint64_t)rows << 32) | ((uint64_t)e << 48);
}

// Numbering: hardware hands block b to XCD b % 8.  Position b / 8 of an
// XCD's sequence takes, expert by expert, one token tile on every eighth
// feature tile, the expert's token tiles fastest: all XCDs stream one
// expert's weights at a time, each keeps that expert's token rows in its
// L2, and the token tiles of an expert read a weight slab through one L2
// one right after the other.  The tiles are counted from the experts' row
// offsets (lane i: local expert i), so that every block up to the last
// tile is live: with blocks for the largest possible count per expert,
// an XCD, which deals its blocks to its shader engines and CUs in turn,
// left up to half of them without a live one (237 workgroups running at a
// time of the 512 that fit).
//
// The feature tiles left over from the groups of eight are dealt in runs of
// consecutive token tiles, whose lengths go on from expert to expert so that
// the XCDs' shares of all tiles differ by one at most.  (Where feature tile ft
// always went to XCD ft % 8, the XCDs past the remainder had nothing of it: 4
// experts of d 2304, f 1152, 9 and 9 tiles of 256 features, 8000 tokens, gate/up
// and down 215 + 143 us, so 174 + 120; on DBRX's gate/up, 84 tiles, a share of 4
// experts with skewed loads, 1300 tokens, whole layer 587 -> 550 us.)
//
// Narrow matrices (below 2048 features) are one list of the experts' tiles, an
// eighth of it for each XCD, so that most experts' weights and token rows are
// read through one L2 (dealt as above every XCD reads every expert's: 32 experts
// of d 512, f 4096, 4000 tokens, down 149 us against 103; 16 of d 1024, f 4096,
// 1900 tokens, 112 against 98).  At 2048 features and more the XCDs stay with one
// expert at a time (8 experts of d 2048, f 8192, 4000 tokens, down 304 us
// against 354 from a list).  Whole layer, 8 experts, top-2, d 256, f 512, 32768
// tokens: 505 us with tile ft on XCD ft % 8, now 335.
constexpr int kNarrow = 2048;      // features

struct TilePos {
    int el;            // local expert, or -1 past the last tile
    int first, rows;   // its rows
    int n_sub, sub;    // its token tiles, and this one
    int before;        // token tiles of the experts before it
    int ft;            // feature tile
};

__device__ __forceinline__ TilePos find_tile(const GemmArgs& a, int block, int n_ftiles, int tile_rows)
{
    // groups of eight, and the rest
    const int n_fg = n_ftiles * tile_rows < kNarrow ? 0 : n_ftiles / kXcds, n_left = n_ftiles - n_fg * kXcds;
    const int pos = block / kXcds, xcd = block % kXcds;
    const int lane = threadIdx.x & 63;
    int first = 0, rows = 0;
    if (a.offsets == nullptr) {              // a plain product: T rows
        rows = lane == 0 ? a.T : 0;
    } else if (lane < a.n_local) {
        first = a.offsets[a.e_begin + lane];
        rows = a.offsets[a.e_begin + lane + 1] - first;
    }
    const int n_sub = (rows + tile_rows - 1) / tile_rows;
    int upto = n_sub;                        // token tiles of the experts up to this lane's
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(upto, off, kWave);
        if (lane >= off) upto += v;
    }
    // this XCD's tiles of the first n token tiles where there are whole
    // groups: those of the groups, and of the n n_left others every eighth
    auto taken = [&](int n) { return n * n_fg + (n * n_left + kXcds - 1 - xcd) / kXcds; };
    // without: its eighth of the list of all tiles
    const int all = __builtin_amdgcn_readlane(upto, kWave - 1) * n_left;
    const int at = all * xcd / kXcds + pos;
    TilePos t{};
    t.el = -1;
    if (n_fg == 0 && at >= all * (xcd + 1) / kXcds) return t;
    t.el = __ffsll((unsigned long long)__ballot(n_fg ? pos < taken(upto) : at < upto * n_left)) - 1;
    if (t.el < 0) return t;
    t.first = __builtin_amdgcn_readlane(first, t.el);
    t.rows = __builtin_amdgcn_readlane(rows, t.el);
    t.n_sub = __builtin_amdgcn_readlane(n_sub, t.el);
    t.before = __builtin_amdgcn_readlane(upto, t.el) - t.n_sub;
    int in_left = at - t.before * n_left;
    if (n_fg) {
        const int in_e = pos - taken(t.before);
        if (in_e < t.n_sub * n_fg) {
            t.sub = in_e % t.n_sub;
            t.ft = in_e / t.n_sub * kXcds + xcd;
            return t;
        }
        // the left-over tiles as eight runs, the first for the XCD on which
        // the expert before it ended
        const int q = (xcd + kXcds * n_left - t.before % kXcds * n_left) % kXcds;
        const int run = t.n_sub * n_left / kXcds, longer = t.n_sub * n_left % kXcds;
        in_left = q * run + min(q, longer) + in_e - t.n_sub * n_fg;
    }
    t.sub = in_left % t.n_sub;
    t.ft = n_fg * kXcds + in_left / t.n_sub;
    return t;
}

template <int kMode>
__global__ __launch_bounds__(kThreads) void gemm_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[kRingB * B_STAGE_BYTES];
    const int M = kMode == kGateUp ? 2 * a.f : a.d;   // a multiple of BM
    const int n_ftiles = M / BM;
    const TilePos tp = find_tile(a, blockIdx.x, n_ftiles, BN);
    if (tp.el < 0) return;
    const int ft = tp.ft, tt = tp.before + tp.sub, e = a.e_begin + tp.el;
    const int row_start = tp.first + tp.sub * BN, row_end = min(row_start + BN, tp.first + tp.rows);
    const bool stamp = a.stamps != nullptr && (int)blockIdx.x < a.max_stamps;
    uint64_t r0 = 0, c0 = 0;
    if (stamp) {
        r0 = __builtin_amdgcn_s_memrealtime();
        c0 = __builtin_amdgcn_s_memtime();
    }
    process_tile<kMode>(a, e, row_start, row_end, tp.n_sub == 1, ft, lds);
    if (stamp) write_stamp(a, r0, c0, ft, tt, row_end - row_start, e);
}

// ---------------------------------------------------------------------------
// Few rows per expert (or few tokens in a plain projection): the same GEMM on
// 128-feature x 128-row tiles.
//
// Here the kernel is bound by the weight stream, and 256 x 256 tiles are too
// few and too long: their last wave leaves CUs idle, and one wave per SIMD
// with three stages of weights in flight does not reach the read rate.  Four
// waves take 32 features each (one MFMA block) of up to four 32-token blocks
// in at most 256 registers and 64 KiB of LDS, so two workgroups share a CU; A
// runs four 64-K stages ahead in registers, B three ahead in LDS.  Token
// blocks that a tile does not have are neither loaded nor multiplied (the
// loop is instantiated for 1 to 4 blocks).  Weights that one tile alone reads
// are loaded nontemporal: the plain policy streams at 6.2 TB/s, the
// nontemporal one at 6.9 (the same addresses, 4 GiB); where several tiles
// share a weight slab it is loaded plain, so that it stays in the L2 for the
// next one.
constexpr int MBM = 128;           // features per workgroup tile
constexpr int MBN = 128;           // token rows per workgroup tile
constexpr int kMidTB = MBN / 32;   // 32-token blocks at most
constexpr int kMidRing = 4;        // A stages in registers
constexpr int kMidRingB = 4;       // B stages in LDS

struct MidCtx {
    __amdgpu_buffer_rsrc_t a_rsrc, b_rsrc;
    uint32_t a_off;            // this lane's A byte offset at the first stage
    uint32_t b_off[kMidTB];    // byte offsets in b_rsrc of this lane's 16-byte chunk, per load
    uint32_t rd_off[KS];       // LDS byte offsets of this lane's B fragment piece, per K step
    int n_stages, w;
    uint32_t s0;               // first stage of the workgroup's K range
};

// Stage s multiplies A(s) (registers) with B(s) (LDS buffer s % 4).  B
// fragments are read one K step ahead, across stages too: before the last K
// step the wave waits for its own reads of this stage's buffer and for its
// part of B(s+1), then a barrier publishes both.  At its start stage s issues
// B(s+3) into the buffer that stage s-1 read; A(s+4) refills each fragment
// after its last use.  Vector-memory operations complete in order: after
// B(s+1), issued at the start of stage s-2, came the four A refills of that
// stage, the B loads and A refills of stage s-1, and the B loads and the
// first three A refills of stage s.  Past the last full round of four stages
// there are no A refills (the compiler would drop them as dead), so only the
// B loads are counted.  B loads past the last stage re-read it into a buffer
// that no later stage reads.
template <int kTB, bool kOnce>
__device__ __forceinline__ void mid_loop(const MidCtx& c, uint8_t* lds, f32x16_t (&acc)[kMidTB])
{
    constexpr int kStage = kTB * 32 * BK * 2;
    constexpr int kWaitMid = wait_vm(2 * kTB + 3 * KS - 1), kWaitMidTail = wait_vm(2 * kTB);
    const int n_stages = c.n_stages, w = c.w;
    u32x4_t ra[kMidRing][KS];
    auto load_a1 = [&](int s, int j, u32x4_t& dst) {
        dst = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                              c.a_rsrc, c.a_off + (j / 2) * kTileBytes + (j % 2) * (kTileBytes / 2),
                                              (c.s0 + (uint32_t)s) * (2 * kTileBytes), kOnce ? kNonTemporal : 0));
    };
    // load q of wave w: rows 32 q + 8 w .. + 7, whole 128-byte lines
    auto load_b = [&](int s, int buf) {
#pragma unroll
        for (int q = 0; q < kTB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                c.b_rsrc,
                (__attribute__((address_space(3))) void*)(&lds[buf + (q * 4 + w) * kTileBytes]),
                16, c.b_off[q], (c.s0 + (uint32_t)s) * (BK * 2), 0, 0);
    };
    u32x4_t bw[2][kTB];                        // B fragments of two K steps in turn
    auto read_b = [&](int buf, int j, u32x4_t (&dst)[kTB]) {
#pragma unroll
        for (int t = 0; t < kTB; ++t)
            dst[t] = *reinterpret_cast<const u32x4_t*>(&lds[buf + c.rd_off[j] + t * 32 * (BK * 2)]);
    };
    int cur = 0, prev = (kMidRingB - 1) * kStage;   // byte offsets of this and the last stage's buffer
    auto stage = [&](int s, u32x4_t (&A)[KS], auto tail) {
        constexpr bool kTail = decltype(tail)::value;
        const int next = cur + kStage == kMidRingB * kStage ? 0 : cur + kStage;
        const int sa = min(s + kMidRing, n_stages - 1);
        load_b(min(s + kMidRingB - 1, n_stages - 1), prev);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            if (j + 1 == KS) {
                // this wave's reads of the stage's buffer and its part of B(s+1)
                __builtin_amdgcn_s_waitcnt((kTail ? kWaitMidTail : kWaitMid) & ~(0xF << 8));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                read_b(next, 0, bw[0]);
            } else {
                read_b(cur, j + 1, bw[(j + 1) & 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < kTB; ++t) acc[t] = mfma32x32x16(A[j], bw[j & 1][t], acc[t]);
            if (!kTail) load_a1(sa, j, A[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev = cur;
        cur = next;
    };
    // A first: its addresses do not wait for the row gather
#pragma unroll
    for (int i = 0; i < kMidRing; ++i)
#pragma unroll
        for (int j = 0; j < KS; ++j) load_a1(min(i, n_stages - 1), j, ra[i][j]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i + 1 < kMidRingB; ++i) load_b(min(i, n_stages - 1), i * kStage);
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_b(0, 0, bw[0]);
    int s = 0;
    for (; s + kMidRing <= n_stages; s += kMidRing) {
        stage(s + 0, ra[0], std::false_type{});
        stage(s + 1, ra[1], std::false_type{});
        stage(s + 2, ra[2], std::false_type{});
        stage(s + 3, ra[3], std::false_type{});
    }
    if (s < n_stages) stage(s, ra[0], std::true_type{});
    if (s + 1 < n_stages) stage(s + 1, ra[1], std::true_type{});
    if (s + 2 < n_stages) stage(s + 2, ra[2], std::true_type{});
    // drain the dummy B loads before the workgroup's LDS can be handed on
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __builtin_amdgcn_s_barrier();
}

template <bool kOnce>
__device__ __forceinline__ void mid_loop_any(int tb, const MidCtx& c, uint8_t* lds, f32x16_t (&acc)[kMidTB])
{
    if (tb == 1)
        mid_loop<1, kOnce>(c, lds, acc);
    else if (tb == 2)
        mid_loop<2, kOnce>(c, lds, acc);
    else if (tb == 3)
        mid_loop<3, kOnce>(c, lds, acc);
    else
        mid_loop<4, kOnce>(c, lds, acc);
}

template <int kMode>
__global__ __launch_bounds__(kThreads, 2) void gemm_mid_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[kMidRingB * MBN * BK * 2];
    const int n_ftiles = (kMode == kGateUp ? 2 * a.f : a.d) / MBM;
    const TilePos tp = find_tile(a, blockIdx.x, n_ftiles * a.k_split, MBN);
    if (tp.el < 0) return;
    const int split = tp.ft / n_ftiles, ft = tp.ft % n_ftiles;
    const int e = a.e_begin + tp.el;
    // an expert's 32-token blocks spread evenly over its token tiles
    const int per_sub = ((tp.rows + 31) / 32 + tp.n_sub - 1) / tp.n_sub * 32;
    const int row_start = tp.first + tp.sub * per_sub;
    const int row_end = min(row_start + per_sub, tp.first + tp.rows);
    if (row_start >= row_end) return;
    const int tb = (row_end - row_start + 31) / 32;   // 32-token blocks with rows

    const int K = kMode == kGateUp ? a.d : a.f;
    const uint64_t KT = (uint64_t)K / kTileK;
    const uint8_t* wbase = a.experts + (uint64_t)(e - a.e_begin) * a.expert_bytes +
                           (kMode == kGateUp ? 0 : a.gu_bytes);
    const int lane = threadIdx.x & 63;
    MidCtx c;
    c.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = c.w, n_all = K / BK;
    c.s0 = (uint32_t)(n_all * split / a.k_split);
    c.n_stages = n_all * (split + 1) / a.k_split - (int)c.s0;
    const uint64_t rt = (uint64_t)ft * (MBM / 16) + w * 2;   // the wave's two 16-row weight tiles
    const uint64_t slab_bytes = kMode == kGateUp ? a.gu_bytes : a.expert_bytes - a.gu_bytes;
    c.a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wbase), 0, (int)slab_bytes,
                                                 kBufferFlags);
    c.a_off = (uint32_t)tile_offset(rt + ((lane & 31) >> 4), 0, KT) +
              (uint32_t)(((lane >> 5) * 16) + (lane & 15)) * 16;
    if (kMode == kGateUp)
        c.b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.x), 0,
                                                     a.T * a.d * 2, kBufferFlags);
    else
        c.b_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.H + (int64_t)row_start * a.f, 0,
                                                     (row_end - row_start) * a.f * 2, kBufferFlags);
#pragma unroll
    for (int q = 0; q < kMidTB; ++q) {
        const int R = q * 32 + w * 8 + (lane >> 3);
        const int row = row_start + R;
        const int rr = row < row_end ? row : row_start;   // rows past the end: any valid row
        const uint32_t chunk = (uint32_t)((lane & 7) ^ b_swizzle(R)) * 16;
        if (kMode == kGateUp)
            c.b_off[q] = (uint32_t)a.row_token[rr] * (uint32_t)a.d * 2 + chunk;
        else
            c.b_off[q] = (uint32_t)(rr - row_start) * (uint32_t)a.f * 2 + chunk;
    }
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        const int R = lane & 31;
        c.rd_off[j] = (uint32_t)R * (BK * 2) + (uint32_t)(((2 * j + (lane >> 5)) ^ b_swizzle(R)) * 16);
    }
    f32x16_t acc[1][kMidTB];
#pragma unroll
    for (int t = 0; t < kMidTB; ++t) acc[0][t] = f32x16_t{};
    if (tp.n_sub == 1)
        mid_loop_any<true>(tb, c, lds, acc[0]);
    else
        mid_loop_any<false>(tb, c, lds, acc[0]);

    store_tile<kMode, 1, kMidTB>(a, acc, lds, ft * (MBM / 16), row_start, row_end, w, lane, split);
}

}  // namespace moe

extern "C" {

int moe_prefill_tile_rows() { return moe::BN; }

// Whether a grouped GEMM of M features per expert takes the 128 x 128 tiles:
// T tokens, k of E experts each, n_local experts here (a plain product: k =
// E = n_local = 1).
//  - Up to about 64 rows per expert the weight stream bounds it (d 6144, f
//    10752, all 16 experts, whole layer, 256 x 256 tiles -> 128 x 128, and
//    with skewed loads: 17 tokens 1023 -> 970 us; 128 tokens (32 rows) 1123 ->
//    1049, skewed 1125 -> 1071; 200 (50 rows) 1147 -> 1088, skewed 1153 ->
//    1133; 260 (65 rows) 1170 -> 1139, skewed 1185 -> 1209; 350 (88 rows) 1213
//    -> 1206, skewed 1239 -> 1313).
//  - With at most 128 tiles of 256 x 256 half of the CUs or more would have
//    none (d 6144: 600 tokens through the 8192-wide projection, 96 tiles,
//    and the 6144-wide one, 72 tiles, the attention block 253 -> 199 us; 1024
//    tokens, 128 and 96 tiles, 299 -> 286; 1400 tokens, 192 and 144 tiles,
//    324 -> 386).
int moe_gemm_mid_tiles(int T, int k, int E, int n_local, int M)
{
    const int64_t pairs = (int64_t)T * k;
    if (pairs <= (int64_t)64 * E) return 1;
    const int64_t rows = (pairs + E - 1) / E;
    return (int64_t)(M / moe::BM) * n_local * ((rows + moe::BN - 1) / moe::BN) <= 128;
}

// Ranges of the reduction of a plain product on 128 x 128 tiles: two where
// the tiles leave half of the CUs idle (d 6144, the attention block: 64
// tokens, 64 and 48 tiles, 144 -> 117 us; 200 tokens, 128 and 96 tiles, 147 ->
// 113; 300 tokens, 192 and 144 tiles, 188 -> 195).
int moe_gemm_plain_split(int T, int M)
{
    if (!moe_gemm_mid_tiles(T, 1, 1, 1, M)) return 1;
    return (int64_t)(M / moe::MBM) * ((T + moe::MBN - 1) / moe::MBN) <= 128 ? 2 : 1;
}

}  // extern "C"

// The grid for n_ft feature tiles (times ranges of K): the token tiles of
// tile_rows rows that a call can have are the full ones and one partial tile
// per expert, and each XCD takes an eighth of all tiles.
static dim3 gemm_grid(const moe::GemmArgs* a, int n_ft, int tile_rows)
{
    const int n = std::min(a->max_rows, a->max_rows / tile_rows + a->n_local) * n_ft;
    return dim3((n + moe::kXcds - 1) / moe::kXcds * moe::kXcds);
}

template <int kMode>
static hipError_t launch_gemm(const moe::GemmArgs* a, hipStream_t s)
{
    const int M = kMode == moe::kGateUp ? 2 * a->f : a->d;
    hipLaunchKernelGGL((moe::gemm_kernel<kMode>), gemm_grid(a, M / moe::BM, moe::BN), dim3(moe::kThreads),
                       0, s, *a);
    return hipGetLastError();
}

template <int kMode>
static hipError_t launch_gemm_mid(const moe::GemmArgs* a, hipStream_t s)
{
    const int M = kMode == moe::kGateUp ? 2 * a->f : a->d;
    hipLaunchKernelGGL((moe::gemm_mid_kernel<kMode>), gemm_grid(a, M / moe::MBM * a->k_split, moe::MBN),
                       dim3(moe::kThreads), 0, s, *a);
    return hipGetLastError();
}

template <int kMode>
static hipError_t launch_any(const moe::GemmArgs* a, hipStream_t s)
{
    return a->mid ? launch_gemm_mid<kMode>(a, s) : launch_gemm<kMode>(a, s);
}

extern "C" hipError_t moe_launch_gemm_gateup(const moe::GemmArgs* a, hipStream_t s)
{
    return launch_any<moe::kGateUp>(a, s);
}

extern "C" hipError_t moe_launch_gemm_down(const moe::GemmArgs* a, hipStream_t s)
{
    return launch_any<moe::kDown>(a, s);
}

extern "C" hipError_t moe_launch_gemm_qkv(const moe::GemmArgs* a, hipStream_t s)
{
    return launch_any<moe::kQkv>(a, s);
}

extern "C" hipError_t moe_launch_gemm_out(const moe::GemmArgs* a, hipStream_t s)
{
    return launch_any<moe::kOut>(a, s);
}
