// Prefill path: bf16 MFMA kernels for gfx950 (v_mfma_f32_16x16x32_bf16, wave64).
//
// Kernel 1  gate_up_mfma:  H[t,j] = bf16( alpha_b(j) * SiLU(<x_t,Wg_j>) * <x_t,Wu_j> )
//           one tile of tokens x neurons per workgroup with TWO fp32 accumulator sets (gate and
//           up), so the gated product of Sec. 3.1's inner bracket is formed in registers and
//           only H (bf16) leaves the CU.
// Kernel 2  down_mfma:     out[t,m] = sum_{j in active runs} H[t,j] * Wd[m,j]
//           one tile of tokens x output features per workgroup; the K loop walks every active
//           run back to back, so the sum over branches of Sec. 3.1 is one fp32 accumulation with
//           no per-branch round trip.  Small outputs are split along K into partial sums that a
//           second kernel adds up in a fixed order.
//
// Both kernels share one main loop: BMT A rows (tokens) against two blocks of 32 NB B rows, waves in
// a WM x 2 arrangement, each wave owning (BMT / WM) x (16 NB + 16 NB) outputs as 16x16 MFMA tiles.
// Tile shapes in use: 256 x (128 + 128) and 256 x (64 + 64) with 8 waves and the whole LDS of a CU,
// 128 x (64 + 64) with 4 waves and either half the LDS (two workgroups per CU) or a deeper ring,
// 64 x (64 + 64) with 4 waves and a ring of whole K tiles (five requested ahead).  The
// 16x16x32 shape is used rather than 32x32x16 because the chip is power limited on this work: with
// random operands a pure stream of 16x16x32 MFMAs sustains 2.0 PFLOP/s, one of 32x32x16 1.7.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace mlpmoe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int BM = 256;          // tokens per tile of the large-tile kernels (and of the routed path's tables)
constexpr int BM_SMALL = 128;    // tokens per tile of the small-tile kernels
constexpr int BNH_MAX = 128;     // rows of each of the two B blocks: 32 * NB, NB = 4 (128) or 2 (64)
// A K tile is 128 bytes (one cache line) of every row: 64 bf16 values or 32 floats; a 16-byte chunk is the unit of
// the loads and the alignment unit of K ranges and neuron tiles.
template <typename E>
struct Elem {
    static constexpr int BK = 128 / sizeof(E), CHUNK = 16 / sizeof(E);
};
constexpr int BK = Elem<uint16_t>::BK;
// The LDS is a ring that keeps the K tile in use and the D tiles requested ahead of it.  Two layouts:
//   alternating (the 256-token tiles): 2 D + 1 parts of equal size, A0 B0 A1 B1 A2 | B2 A3 ...; with D = 2 the
//       ring fills the LDS of a CU (five parts of 32 KiB), half a K tile less than whole stages would need;
//   staged: D + 1 stages, a stage being the A rows followed by the B rows of one K tile.  Nothing is padded, so
//       tiles with fewer A rows than B rows keep more K tiles in flight in the same LDS.
__host__ __device__ constexpr int n_parts(int depth) { return 2 * depth + 1; }
// A part of the alternating ring holds the A rows (BMT tokens), or the B rows (2 blocks of 32 NB), of one K tile.
// 256-token tiles: 32 KiB parts, the ring is the whole LDS of a CU (one workgroup of 8 waves per CU).
// 128-token tiles with NB = 2: 16 KiB parts, 80 KiB per workgroup of 4 waves, two workgroups per CU.
__host__ __device__ constexpr int part_bytes(int bmt, int nb) { return (bmt > 64 * nb ? bmt : 64 * nb) * 128; }
__host__ __device__ constexpr int stage_bytes(int bmt, int nb) { return (bmt + 64 * nb) * 128; }
__host__ __device__ constexpr int lds_bytes(int bmt, int nb, int depth = 2, bool staged = false)
{
    return staged ? (depth + 1) * stage_bytes(bmt, nb) : n_parts(depth) * part_bytes(bmt, nb);
}
constexpr int MFMA_WM = 4;                           // waves along M of the 256-token tiles: 8 waves of 64 x (64+64) outputs
constexpr int SMALL_WM = 2;                          // ... of the 128-token tiles: 4 waves of 64 x (32+32)
constexpr int BM_SLIM = 64;                          // tokens per tile of the slim kernels: 4 waves of 32 x (32+32)
constexpr int SLIM_WM = 2;

// How down_mfma writes its result.  DST_THROUGH: partial sums of at most THROUGH_BYTES, stored past the L2 (sc1), so that the end
// of the kernel has no dirty lines to write back before the sum may start.  us a call, plain / through: 896 x 4864, T = 64 20.9 / 20.3,
// T = 500 34.5 / 33.1, T = 333 in 12 branches, 9 kept 26.4 / 25.7; 2048 x 5504, T = 100 34.7 / 34.1, T = 250 45.5 / 44.0; 3072 x 8192, T = 100 52.7 / 51.6.
// Not for more bytes (4096 x 14336, T = 512, 67 MB: 163.5 / 168.3 with H stored so as well).  Layers whose W_down is larger than
// THROUGH_WEIGHTS and streams from HBM gain less or lose: 4096 x 8192, T = 64 58.3 / 57.8, 5120 x 13824 97.9 / 96.7, 3584 x 18944 104.8 / 103.6, but
// 4096 x 11008 70.9 / 71.8, 4096 x 14336 86.0 / 87.0 and T = 100 92.7 / 93.3.
enum { DST_F32 = 0, DST_BF16 = 1, DST_THROUGH = 2 };
constexpr size_t THROUGH_BYTES = 16u << 20, THROUGH_WEIGHTS = 64u << 20;      // partial sums, W_down
constexpr int STORE_SC1 = 16;           // cache policy of a buffer store: sc1

// 16 zero bytes: K chunks that fall past the end of a range are fetched from here.
__device__ const uint32_t g_zero_chunk[4] = {0, 0, 0, 0};

typedef const __attribute__((address_space(1))) void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

// One wave-wide 16-byte-per-lane load straight into LDS: lane l's data lands at dst + 16*l.
__device__ __forceinline__ void dma16(const void *src, void *lds_dst)
{
    __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)lds_dst, 16, 0, 0);
}

// A fragment piece: one 16-byte chunk per lane.  Lane group lane >> 4 holds a chunk of its own, so a bf16 piece is
// the 32 K values of one 16x16x32 MFMA; a float piece is four 16x16x4 steps, step e taking element e of every chunk.
template <typename E>
struct FragOf {
    typedef bf16x8 type;
};
template <>
struct FragOf<float> {
    typedef f32x4 type;
};
template <typename E>
using Frag = typename FragOf<E>::type;
template <typename E>
constexpr int MFMAS_PER_CHUNK = sizeof(E) == 4 ? 4 : 1;
__device__ __forceinline__ f32x4 mfma_step(bf16x8 r, bf16x8 c, f32x4 acc, int)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(r, c, acc, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_step(f32x4 r, f32x4 c, f32x4 acc, int e)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(r[e], c[e], acc, 0, 0, 0);
}

// Workgroup barrier that waits until at most N of this wave's direct-to-LDS loads (they return
// in issue order) and none of its LDS reads are outstanding.  Written by hand because the
// compiler's own barrier waits for every load, which would drain the multi-stage pipeline.
template <int N>
__device__ __forceinline__ void pipeline_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Position in the flattened list of K tiles (ranges laid end to end).
struct KCursor {
    int run, k;
};

// K ranges of the gate/up projection: the whole model dimension.
struct KSingle {
    int len;
    __device__ __forceinline__ int n_runs() const { return 1; }
    __device__ __forceinline__ int start(int) const { return 0; }
    __device__ __forceinline__ int end(int) const { return len; }
};
// K ranges of the down projection: the active runs of neurons.
struct KRuns {
    const BranchTable &bt;
    __device__ __forceinline__ int n_runs() const { return bt.n_runs; }
    __device__ __forceinline__ int start(int r) const { return bt.run_start[r]; }
    __device__ __forceinline__ int end(int r) const { return bt.run_end[r]; }
};

// K ranges chosen per workgroup at run time (per-token routing: the branches some token of this
// token tile is routed to).  Lane r of every wave holds the bounds of range r; reading them is a
// lane read, not a memory access.
struct KRunsLanes {
    int n, v_start, v_end;
    __device__ __forceinline__ int n_runs() const { return n; }
    __device__ __forceinline__ int start(int r) const { return __builtin_amdgcn_readlane(v_start, r); }
    __device__ __forceinline__ int end(int r) const { return __builtin_amdgcn_readlane(v_end, r); }
};

// Merged ranges of the branches that are active AND flagged in `needed` (B bytes, uniform).
__device__ __forceinline__ KRunsLanes routed_runs(const BranchTable &bt, const uint8_t *needed)
{
    KRunsLanes kr{0, 0, 0};
    const int lane = threadIdx.x & 63;
    int prev_end = -1;
    for (int b = 0; b < bt.B; ++b) {
        if (!((bt.active >> b) & 1ULL) || !needed[b]) continue;
        const int s = bt.off[b], e = bt.off[b + 1];
        if (e == s) continue;
        if (kr.n > 0 && prev_end == s) {
            kr.v_end = lane == kr.n - 1 ? e : kr.v_end;
        } else {
            kr.v_start = lane == kr.n ? s : kr.v_start;
            kr.v_end = lane == kr.n ? e : kr.v_end;
            ++kr.n;
        }
        prev_end = e;
    }
    return kr;
}

template <int BKE, typename KR>
__device__ __forceinline__ KCursor k_seek(const KR &kr, int tile)
{
    KCursor c{0, 0};
    for (int r = 0; r < kr.n_runs(); ++r) {
        const int n = (kr.end(r) - kr.start(r) + BKE - 1) / BKE;
        if (tile < n) {
            c.run = r;
            c.k = kr.start(r) + tile * BKE;
            return c;
        }
        tile -= n;
    }
    c.run = kr.n_runs() - 1;
    c.k = kr.start(c.run);
    return c;
}

// LDS layout.  The LDS is a ring of 2 D + 1 parts (five parts of 32 KiB for the 256-token tiles).  A part
// holds rows of 128 bytes (8 chunks of 8 bf16): either the A rows (tokens) of one K tile, or its B rows (the
// rows of the first B block, then those of the second).  Parts are filled in the order A0 B0 A1 B1 A2 B2 ...,
// part number s going to ring slot s % (2 D + 1), so while K tile i is being used the parts of tiles i+1 ..
// i+D-1 and the A part of tile i+D are landing.  Chunk c of row r is stored at chunk slot c ^ swz(r),
// swz(r) = (r & 7) ^ ((r >> 3) & 1), so that the 16-byte reads of 32 consecutive rows at one
// logical chunk (and of 16 consecutive rows at 4 consecutive chunks) fall on distinct banks.  A direct-to-LDS wave load writes 1 KiB = 8 whole rows,
// and each row is one full 128-byte line of global memory (half lines cost the same L2 -> CU
// transfer as whole ones); the swizzle is applied on the global side: the lane that fills slot p
// of row r fetches logical chunk p ^ swz(r).
//
// Main loop, WM x 2 waves.  A_tile / B0_tile / B1_tile point at the first row of the tile (wave uniform);
// a_valid / b0_valid / b1_valid are the rows that exist from there on (>= 1).  Rows past that
// are clamped to the last valid row: their results are never stored and MFMA rows / columns do
// not mix.  K chunks past the end of a range are read from a zero chunk, in A and in B.
// Schedule of K tile i (two K steps of 32; fragments are double buffered one step ahead):
//   step 0: MFMAs; read step 1's fragments; issue the A part of tile i+D
//   barrier: parts of tile i+1 have landed (only the loads issued after them may be in flight) and
//            every wave has read its last fragments of tile i, whose two ring slots are free again
//   step 1: MFMAs; read step 0's fragments of tile i+1; issue the B part of tile i+D
// The direct loads are spread over the steps (one per wave every other MFMA slot) because a
// CU's vector memory path takes about as long to move a tile as the MFMAs take to consume it:
// issued in bursts, the loads back up in the issue queue and the MFMAs behind them wait.
// NB = 16-row MFMA pieces per B block per wave: 4 (B blocks of 128 rows, a 256 x 256 tile) or 2 (B
// blocks of 64 rows, a 256 x 128 tile, for shapes that would otherwise leave most CUs without a
// tile in the last round).  A B part of 64 + 64 rows fills half of its ring slot.
// Float storage (E = float) differs only in what a 16-byte chunk holds: 4 K elements, fed to four
// v_mfma_f32_16x16x4_f32 one after the other instead of one 16x16x32.
// stops(kt): called with acc0, acc1 the sums over the K tiles before kt, at kt_end and where it said before; gives the next place.
struct NoStops {
    static constexpr bool kSome = false;
    __device__ __forceinline__ int operator()(int) const { return 0; }
};
template <typename F>
struct Stops {
    static constexpr bool kSome = true;
    const F &f;
    int first;
    __device__ __forceinline__ int operator()(int kt) const { return f(kt); }
};
template <int BMT, int WM, int NB, int D, bool kStaged, bool kRowsAreB, typename E, typename KR, typename St = NoStops>
__device__ __forceinline__ void mainloop(const E *__restrict__ A_tile, int lda, int a_valid,
                                         const E *__restrict__ B0_tile,
                                         const E *__restrict__ B1_tile, int ldb, int b0_valid,
                                         int b1_valid, const KR &kr, int kt_begin, int kt_end, char *lds,
                                         f32x4 (&acc0)[BMT / 16 / WM][NB], f32x4 (&acc1)[BMT / 16 / WM][NB],
                                         const St &stops = St{})
{
    constexpr int BKE = Elem<E>::BK, CHUNK = Elem<E>::CHUNK;
    constexpr unsigned ES = sizeof(E);
    constexpr int MI = BMT / 16 / WM;             // 16-row MFMA tiles per wave along M
    constexpr int NWAVES = WM * 2;
    constexpr int BNH = 32 * NB;                  // rows of each B block
    constexpr int PL = BMT / 8 / NWAVES;          // 1 KiB wave-loads per wave per A part
    constexpr int PLB = 8 * NB / NWAVES;          // ... per B part
    constexpr int SLOT = MI * NB >= 2 ? 4 : 2;    // MFMAs (of one chunk element) per slot
    constexpr int N_SLOTS = MI * NB * 2 / SLOT;   // slots per K step
    constexpr int N_PIECES = 2 * NB + MI;         // fragment pieces per K step
    constexpr int RPS = (N_PIECES + N_SLOTS - 1) / N_SLOTS < 2 ? 2 : (N_PIECES + N_SLOTS - 1) / N_SLOTS;   // fragment reads per slot
    // Ring geometry in bytes: where the A part of the first K tile and its B part sit, how far the next tile's
    // parts are from this tile's, and where the ring wraps.
    // direct loads of a part, spread over the slots of a K step: every *_EVERY-th slot issues *_PER of them
    constexpr int A_EVERY = PL <= N_SLOTS ? N_SLOTS / PL : 1, A_PER = PL <= N_SLOTS ? 1 : PL / N_SLOTS;
    constexpr int B_EVERY = PLB <= N_SLOTS ? N_SLOTS / PLB : 1, B_PER = PLB <= N_SLOTS ? 1 : PLB / N_SLOTS;
    constexpr int B_FIRST = kStaged ? BMT * 128 : part_bytes(BMT, NB);
    constexpr int RING_STEP = kStaged ? stage_bytes(BMT, NB) : 2 * part_bytes(BMT, NB);
    constexpr int RING_BYTES = lds_bytes(BMT, NB, D, kStaged);
    static_assert(D >= 2, "one tile in use, at least one more on its way");
    static_assert((N_SLOTS % PL == 0 || PL % N_SLOTS == 0) && (N_SLOTS % PLB == 0 || PLB % N_SLOTS == 0),
                  "loads spread evenly over the slots");
    const int nk = kt_end - kt_begin;
    if (nk <= 0) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // ---- global side: per-lane byte offsets of this wave's loads, relative to the tile pointers
    const int lr = lane >> 3;                     // row inside the 8-row slab of one wave-load
    const int cl0 = (lane & 7) ^ lr;              // logical chunk fetched in even slabs; odd slabs: cl0 ^ 1
    const int a_cl0 = cl0 ^ (wave * PL & 1), b_cl0 = cl0 ^ (wave * PLB & 1);      // ... in this wave's first slab
    const bool second = wave >= NWAVES / 2;       // this wave fills the rows of the second B block
    const int b_valid = second ? b1_valid : b0_valid;
    unsigned a_off[PL], b_off[PLB];
#pragma unroll
    for (int n = 0; n < PL; ++n) {
        const int slab = wave * PL + n;
        const int cl = a_cl0 ^ (n & 1);
        int ra = slab * 8 + lr;
        ra = ra < a_valid ? ra : a_valid - 1;
        a_off[n] = (unsigned)ra * (unsigned)lda * ES + (unsigned)cl * 16u;
    }
#pragma unroll
    for (int n = 0; n < PLB; ++n) {
        const int slab = wave * PLB + n;          // 0 .. 8 NB - 1; the second half are B1's rows
        const int cl = b_cl0 ^ (n & 1);
        int rb = (slab % (4 * NB)) * 8 + lr;
        rb = rb < b_valid ? rb : b_valid - 1;
        b_off[n] = (unsigned)rb * (unsigned)ldb * ES + (unsigned)cl * 16u;
    }
    const char *a_base = reinterpret_cast<const char *>(A_tile);
    const char *b_base = reinterpret_cast<const char *>(second ? B1_tile : B0_tile);
    char *wa_dst = lds + wave * (PL * 1024);      // this wave's slabs inside an A part
    char *wb_dst = lds + wave * (PLB * 1024);     // ... inside a B part
    const char *zero = reinterpret_cast<const char *>(g_zero_chunk);

    // Position of the next part to be issued, per matrix.  `left` counts the tiles not yet
    // issued.  A lane whose chunk lies past the end of the K range, or any lane once no tile is
    // left, reads the zero chunk instead.  Branch free, so that the loads sit in the same basic
    // block as the MFMAs and every part is always the same number of loads.
    struct Issue {
        int run, k, kend, left, off;              // off: byte offset in the ring of the part to be filled next
    };
    auto advance = [&](Issue &q) {                // stays on the last range once the list is exhausted
        q.k += BKE;
        if (q.k >= q.kend && q.run + 1 < kr.n_runs()) {
            ++q.run;
            q.k = kr.start(q.run);
            q.kend = kr.end(q.run);
        }
        --q.left;
        q.off += RING_STEP;
        if (q.off >= RING_BYTES) q.off -= RING_BYTES;
    };
    // what the loads of one part have in common
    struct Part {
        const char *src;                          // tile pointer moved to the part's K offset
        char *dst;                                // this wave's first slab in the part's ring slot
        bool ok[2];                               // chunk inside the K range, for this wave's even / odd loads
    };
    auto part_of = [&](const Issue &q, const char *base, char *w_dst, int first_cl) {
        Part pt;
        const int kend = q.left > 0 ? q.kend : -(1 << 30);
        pt.src = base + (size_t)q.k * ES;
        pt.dst = w_dst + q.off;
        pt.ok[0] = q.k + first_cl * CHUNK < kend;
        pt.ok[1] = q.k + (first_cl ^ 1) * CHUNK < kend;
        return pt;
    };
    auto dma_part = [&](int n, const Part &pt, const unsigned *off) {
        dma16(pt.ok[n & 1] ? pt.src + off[n] : zero, pt.dst + n * 1024);
    };

    // ---- LDS side: per-lane read offsets (bytes) for the 2 K steps of a tile.  A 16x16x32
    // fragment is 16 rows x 32 K: lane l holds row l & 15 and K group l >> 4 (8 elements).  Which
    // 16-byte chunk of the step's 64 bytes a K group reads is free as long as A and B agree (the
    // dot product does not care about the order of K).  The LDS serves lanes l and l + 32 in the
    // same cycle, so K groups g and g + 2 are given ADJACENT chunks (0, 2, 1, 3 -> chunks 0, 1, 2,
    // 3): with the row swizzle the 16 lanes of a cycle then fall on distinct banks.
    const int lrow = lane & 15;
    const int swz = (lane & 7) ^ ((lane >> 3) & 1);      // fragment rows start at multiples of 16
    const int kg = lane >> 4;
    const int kchunk = ((kg & 1) << 1) | (kg >> 1);
    int a_rd[2], b_rd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int slot = (ks * 4 + kchunk) ^ swz;
        a_rd[ks] = (wm * (MI * 16) + lrow) * 128 + slot * 16;
        b_rd[ks] = (wn * (16 * NB) + lrow) * 128 + slot * 16;
    }
    // Fragment pieces of one K step: v[0 .. 2 NB) = the B pieces b0[0..NB), b1[0..NB) (16 rows of the
    // first / second B block each), then the A pieces.  MFMA m uses A piece m / (2 NB) and B piece
    // m % (2 NB).
    struct Frags {
        Frag<E> v[N_PIECES];
    };
    auto read_piece = [&](Frags &f, int g, int a_at, int ks) {
        // the B part of a tile follows its A part (alternating ring: in the next part, which may be the first)
        const int b_at = kStaged ? a_at + B_FIRST : (a_at + B_FIRST < RING_BYTES ? a_at + B_FIRST : 0);
        if (g < 2 * NB)
            f.v[g] = *reinterpret_cast<const Frag<E> *>(lds + b_at + b_rd[ks] + (g / NB) * (BNH * 128) +
                                                       (g % NB) * (16 * 128));
        else
            f.v[g] = *reinterpret_cast<const Frag<E> *>(lds + a_at + a_rd[ks] + (g - 2 * NB) * (16 * 128));
    };
    // kRowsAreB: the B rows (weights) are the MFMA's row operand and the A rows (tokens) its column
    // operand.  In the 16x16 result lane l then holds column l & 15 = one token and rows
    // 4 * (l >> 4) + 0..3 = four consecutive B rows, which the epilogues store as one 8- or 16-byte
    // piece of the token's output row.  Otherwise tokens are the rows.
    // Floats: the second K step of every tile has sums of its own.  Chains of half the length leave less of an error: 896 x 4864, T = 256
    // against float64 9.2e-7 -> 6.4e-7, T = 500 1.1e-6 -> 6.8e-7, in the same time.
    constexpr bool kTwoSums = sizeof(E) == 4;
    f32x4 second0[kTwoSums ? MI : 1][NB], second1[kTwoSums ? MI : 1][NB];
    auto clear_second = [&]() {
#pragma unroll
        for (int i = 0; i < (kTwoSums ? MI : 1); ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) second0[i][j] = second1[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto mfma_n = [&](const Frags &f, int m, int e, bool second_step) {
        const int i = m / (2 * NB), b = m % (2 * NB);
        const Frag<E> r = kRowsAreB ? f.v[b] : f.v[2 * NB + i], c = kRowsAreB ? f.v[2 * NB + i] : f.v[b];
        f32x4 &acc = kTwoSums && second_step ? (b < NB ? second0[kTwoSums ? i : 0][b % NB] : second1[kTwoSums ? i : 0][b % NB])
                                             : (b < NB ? acc0[i][b % NB] : acc1[i][b % NB]);
        acc = mfma_step(r, c, acc, e);
    };
    // One K step, written in the instruction order wanted: slots of {4 MFMAs, then LDS reads of
    // the next step's fragments, then (in evenly spaced slots) one direct load}; nothing may be
    // moved across a slot boundary.  The compiler waits for ALL outstanding LDS reads before the
    // first MFMA of a step (direct-to-LDS loads in flight make it give up exact counting), so the
    // reads are packed into the early slots and the last slots leave them time to land.
    // DMA: 1 loads of the A part pt, 2 loads of the B part pt.
    auto k_step = [&](const Frags &cur_f, Frags &nxt_f, int rd_at, int rd_ks, int dma, const Part &pt) {
#pragma unroll
        for (int g = 0; g < N_SLOTS; ++g) {
            // The two waves of a SIMD take the matrix pipe in turns of four MFMAs.  A wave asks
            // for its turn at priority 1 (first MFMA), holds it at priority 3 (the other wave,
            // asking at 1, cannot cut in, which the older wave otherwise always does) and drops
            // to 0 for its loads and address arithmetic, which then run under the other's turn.
            __builtin_amdgcn_s_setprio(1);
            mfma_n(cur_f, SLOT * g, 0, rd_ks == 0);
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int q = 1; q < SLOT; ++q) mfma_n(cur_f, SLOT * g + q, 0, rd_ks == 0);
#pragma unroll
            for (int e = 1; e < MFMAS_PER_CHUNK<E>; ++e)
#pragma unroll
                for (int q = 0; q < SLOT; ++q) mfma_n(cur_f, SLOT * g + q, e, rd_ks == 0);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < RPS; ++r)
                if (RPS * g + r < N_PIECES) read_piece(nxt_f, RPS * g + r, rd_at, rd_ks);
            if (dma == 1 && g % A_EVERY == 0) {
#pragma unroll
                for (int l = 0; l < A_PER; ++l) dma_part((g / A_EVERY) * A_PER + l, pt, a_off);
            }
            if (dma == 2 && g % B_EVERY == 0) {
#pragma unroll
                for (int l = 0; l < B_PER; ++l) dma_part((g / B_EVERY) * B_PER + l, pt, b_off);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // prologue: the parts of tiles 0 .. D-1 in flight, tile 0 landed
    Issue qa, qb;
    {
        const KCursor c = k_seek<BKE>(kr, kt_begin);
        qa.run = c.run;
        qa.k = c.k;
        qa.kend = kr.end(c.run);
        qa.left = nk;
        qa.off = 0;
        qb = qa;
        qb.off = B_FIRST;
    }
#pragma unroll
    for (int p = 0; p < D; ++p) {
        const Part pa = part_of(qa, a_base, wa_dst, a_cl0), pb = part_of(qb, b_base, wb_dst, b_cl0);
#pragma unroll
        for (int n = 0; n < PL; ++n) dma_part(n, pa, a_off);
#pragma unroll
        for (int n = 0; n < PLB; ++n) dma_part(n, pb, b_off);
        advance(qa);
        advance(qb);
    }
    pipeline_barrier<(D - 1) * (PL + PLB)>();
    Frags f0, f1;
#pragma unroll
    for (int g = 0; g < N_PIECES; ++g) read_piece(f0, g, 0, 0);

    int rd = 0;                                   // byte offset in the ring of the A part of the tile in use
    clear_second();
    int it = 0, until = nk;
    if constexpr (St::kSome) until = stops.first - kt_begin;
    do {
        for (; it < until; ++it) {
            const Part pa = part_of(qa, a_base, wa_dst, a_cl0);
            k_step(f0, f1, rd, 1, 1, pa);             // + A part of tile it+D
            advance(qa);
            // tile it+1 has landed (the newer tiles and the A part just issued may be in flight); tile it's slots are free
            pipeline_barrier<(D - 2) * (PL + PLB) + PL>();
            rd = rd + RING_STEP < RING_BYTES ? rd + RING_STEP : rd + RING_STEP - RING_BYTES;
            const Part pb = part_of(qb, b_base, wb_dst, b_cl0);
            k_step(f1, f0, rd, 0, 2, pb);             // + B part of tile it+D
            advance(qb);
        }
        if constexpr (kTwoSums) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    acc0[i][j] += second0[i][j];
                    acc1[i][j] += second1[i][j];
                }
            clear_second();
        }
        if constexpr (St::kSome) until = stops(kt_begin + it) - kt_begin;
    } while (it < nk);
    pipeline_barrier<0>();                        // LDS may be reused by the caller
}

// Tables whose run boundaries are not multiples of a 16-byte chunk (kEdges).  The neuron tiles of the gate+up
// projection walk the runs rounded OUTWARDS to whole chunks (H is stored for active neurons only); the K ranges of
// the down projection are the runs rounded INWARDS, and the chunks that lie across a boundary, at most two per run,
// are added by edge_steps below: they go from global memory straight into MFMA operand registers, inactive K
// elements masked to 0 in BOTH operands (nothing of a pruned branch reaches the sum, non-finite values included).
// What bounds it: one global load latency per four chunks at the end of a tile.  896 x 4864 in 12 branches of 406 / 405
// neurons, first 9 kept, T = 333: 29 us against 703 us for the general FMA kernels.
constexpr int kMaxEdges = 2 * kMaxRuns;
struct EdgeList {
    int n;
    int col[kMaxEdges];                           // first K element of the chunk
    uint8_t mask[kMaxEdges];                      // bit i: element i of the chunk is active
};
struct NoEdges {};
// Edges of run [s, e): its first chunk (side 0) and its last (side 1), as far as they are partial.  A run inside one
// chunk has its elements in side 0, or in side 1 if it starts at the chunk.  mask 0: no such edge.
template <int CHUNK>
__host__ __device__ inline void run_edge(int s, int e, int side, int &col, unsigned &mask)
{
    const int cs = s / CHUNK * CHUNK, ce = e / CHUNK * CHUNK;
    const unsigned all = (1u << CHUNK) - 1;
    col = side == 0 ? cs : ce;
    if (side == 0) mask = s == cs ? 0u : (all << (s - cs)) & (e - cs < CHUNK ? (1u << (e - cs)) - 1 : all);
    else mask = (e == ce || (ce == cs && s != cs)) ? 0u : (1u << (e - ce)) - 1;
}
// The runs of `raw` rounded inwards, empty ones dropped (lane r holds range r).
template <int CHUNK>
__device__ __forceinline__ KRunsLanes inner_runs(const KRunsLanes &raw)
{
    KRunsLanes in{0, 0, 0};
    const int lane = threadIdx.x & 63;
    for (int r = 0; r < raw.n; ++r) {
        const int s = (raw.start(r) + CHUNK - 1) / CHUNK * CHUNK, e = raw.end(r) / CHUNK * CHUNK;
        if (e <= s) continue;
        in.v_start = lane == in.n ? s : in.v_start;
        in.v_end = lane == in.n ? e : in.v_end;
        ++in.n;
    }
    return in;
}
// chunk & mask, element by element
template <typename E>
__device__ __forceinline__ Frag<E> masked_chunk(const E *p, unsigned mask)
{
    u32x4 v = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t m = sizeof(E) == 4 ? ((mask >> w) & 1u ? 0xffffffffu : 0u)
                                          : ((mask >> (2 * w)) & 1u ? 0x0000ffffu : 0u) | ((mask >> (2 * w + 1)) & 1u ? 0xffff0000u : 0u);
        v[w] &= m;
    }
    return __builtin_bit_cast(Frag<E>, v);
}
// Adds `n` edge chunks to the accumulators of a down tile: four chunks (one per lane group) per step.
// at(i, col, mask) gives chunk i and may be asked with another i in every lane; all lanes of a wave ask together.
template <int MI, int NB, typename E, typename At>
__device__ __forceinline__ void edge_steps(int n, const At &at, const E *__restrict__ A_tile, int lda, int a_valid,
                                           const E *__restrict__ B0_tile, const E *__restrict__ B1_tile, int ldb,
                                           int b0_valid, int b1_valid, f32x4 (&acc0)[MI][NB], f32x4 (&acc1)[MI][NB])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1, lrow = lane & 15;
    for (int i0 = 0; i0 < n; i0 += 4) {
        int col = 0;
        unsigned mask = 0;
        const int i = i0 + (lane >> 4);
        at(i < n ? i : n - 1, col, mask);
        if (i >= n) mask = 0;
        if (mask == 0) col = 0;                   // nothing to add: any chunk that exists
        Frag<E> a[MI];
#pragma unroll
        for (int m = 0; m < MI; ++m) {
            const int r = wm * (MI * 16) + m * 16 + lrow;
            a[m] = masked_chunk(A_tile + (size_t)(r < a_valid ? r : a_valid - 1) * lda + col, mask);
        }
#pragma unroll
        for (int b = 0; b < 2 * NB; ++b) {
            const int r = wn * (16 * NB) + (b % NB) * 16 + lrow, valid = b < NB ? b0_valid : b1_valid;
            const Frag<E> w = masked_chunk((b < NB ? B0_tile : B1_tile) + (size_t)(r < valid ? r : valid - 1) * ldb + col, mask);
#pragma unroll
            for (int e = 0; e < MFMAS_PER_CHUNK<E>; ++e)
#pragma unroll
                for (int m = 0; m < MI; ++m) {
                    f32x4 &acc = b < NB ? acc0[m][b] : acc1[m][b - NB];
                    acc = mfma_step(w, a[m], acc, e);
                }
        }
    }
}

__device__ __forceinline__ float silu_mul(float g, float u)
{
    // SiLU(g) * u with hardware exp2 / rcp (about 1 ulp each)
    const float e = __builtin_amdgcn_exp2f(g * -1.4426950408889634f);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

__device__ __forceinline__ uint16_t to_bf16(float v)
{
    const __bf16 b = (__bf16)v;          // v_cvt_pk_bf16_f32: round to nearest even
    return __builtin_bit_cast(uint16_t, b);
}

// alpha_b * SiLU(g) * u.  kExact: with expf and a division, as the general kernels form it, for the calls that these
// kernels took over from them (float storage, bf16 tables with odd boundaries).  The reciprocal of silu_mul is 0 below
// the smallest normal float, which loses SiLU(g) for g < -87.3 however large u is.
template <bool kExact>
__device__ __forceinline__ float gated(float alpha, float g, float u)
{
    if (!kExact) return alpha * silu_mul(g, u);
    const float s = g / (1.0f + expf(-g));
    return alpha * (s * u);
}
__device__ __forceinline__ void store1(uint16_t *p, float v) { *p = to_bf16(v); }
__device__ __forceinline__ void store1(float *p, float v) { *p = v; }
__device__ __forceinline__ void store4(uint16_t *p, f32x4 v)
{
    u32x2 pk;
    pk.x = (uint32_t)to_bf16(v[0]) | ((uint32_t)to_bf16(v[1]) << 16);
    pk.y = (uint32_t)to_bf16(v[2]) | ((uint32_t)to_bf16(v[3]) << 16);
    *reinterpret_cast<u32x2 *>(p) = pk;
}
__device__ __forceinline__ void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }

// Workgroup id -> output tile.  The hardware deals consecutive workgroup ids round-robin to the
// 8 XCDs, each with its own L2.  Every XCD therefore takes one contiguous eighth of a "grouped"
// tile order (groups of 8 M tiles, M fastest inside a group), so that the 32 workgroups resident
// on an XCD form an 8 x 4 block of tiles and share their A and B tiles through that L2.
// The grid holds 8 * ceil(tiles / 8) ids; ids past the end get no tile.
constexpr int XCDS = 8;
constexpr int kCUs = 256;
constexpr int GROUP_M = 8;
__host__ __device__ inline int ids_per_xcd(long long tiles) { return (int)((tiles + XCDS - 1) / XCDS); }
// position in the grouped tile order -> tile
__device__ __forceinline__ void tile_from_logical(int logical, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int group_sz = GROUP_M * tiles_n;
    const int g = logical / group_sz, rem = logical % group_sz;
    const int m0 = g * GROUP_M;
    const int gsz = tiles_m - m0 < GROUP_M ? tiles_m - m0 : GROUP_M;
    tm = m0 + rem % gsz;
    tn = rem / gsz;
}
__device__ __forceinline__ bool tile_of(int id, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int total = tiles_m * tiles_n;
    const int logical = (id % XCDS) * ids_per_xcd(total) + id / XCDS;
    if (logical >= total) return false;
    const int group_sz = GROUP_M * tiles_n;
    const int g = logical / group_sz, rem = logical % group_sz;
    const int m0 = g * GROUP_M;
    const int gsz = tiles_m - m0 < GROUP_M ? tiles_m - m0 : GROUP_M;
    tm = m0 + rem % gsz;
    tn = rem / gsz;
    return true;
}

// Scratch of the routed kernels, filled by route_tile_list from route[T, B]:
//   tile_need[tm * B + b]  bit h set if some token of half h (128 tokens) of token tile tm (256 tokens) is routed to branch b;
//   counts[g], list[g * stride + i]: the live gate+up tiles of token-tile group g (GROUP_M token tiles), as numbers tn * gsz +
//   (tm - g * GROUP_M), gsz = token tiles in the group.  The lower 16 bits of the words have them by N tile, then by token tile; the
//   upper 16 bits have first those that both halves of their tokens need (list[g * stride + stride - 1] of them), then those that one half
//   needs, plus ROUTE_SECOND if it is the second half, each again by N tile, then by token tile.  Layers with larger numbers (d_inter beyond
//   about 500000) have the first order alone, as whole words.  A tile is live if some token of its token tile is routed to an active
//   branch that owns one of its neurons.
constexpr uint32_t ROUTE_SECOND = 1u << 15;
struct RouteTiles {
    const uint8_t *tile_need;
    const uint32_t *counts;
    const uint32_t *list;
    int stride;
    bool words;           // list entries are whole words
    int most;             // items that the grid has workgroups for
};

// N tile tn (counted over the runs of active branches, tiles of bnh neurons) -> its first neuron and
// the end of its run; false past the last tile.
__device__ __forceinline__ bool neuron_tile(const BranchTable &bt, int tn, int bnh, int &n0, int &n_end)
{
    for (int r = 0; r < bt.n_runs; ++r) {
        const int n = (bt.run_end[r] - bt.run_start[r] + bnh - 1) / bnh;
        if (tn < n) {
            n0 = bt.run_start[r] + tn * bnh;
            n_end = bt.run_end[r];
            return true;
        }
        tn -= n;
    }
    return false;
}

// One tile of the gate+up projection: tokens tm * BMT .., neurons n0 .. min(n0 + 32 NB, n_end) of a run that
// ends at n_end.  lds: lds_bytes(BMT, NB, D) bytes.
template <int BMT, int WM, int NB, int D, bool kStaged, bool kRouted, bool kEdges = false, typename E>
__device__ __forceinline__ void gate_up_tile(const E *__restrict__ X, const E *__restrict__ Wg,
                                             const E *__restrict__ Wu, E *__restrict__ H, int T,
                                             int d_model, int ldh, const uint8_t *__restrict__ route,
                                             const BranchTable &bt, char *lds, int tm, int n0, int n_end)
{
    constexpr int BNH = 32 * NB;
    const int t0 = tm * BMT;

    constexpr int MI = BMT / 16 / WM;
    f32x4 accg[MI][NB], accu[MI][NB];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            accg[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            accu[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

    const BranchLanes br(bt);
    const int nk = (d_model + Elem<E>::BK - 1) / Elem<E>::BK;
    mainloop<BMT, WM, NB, D, kStaged, true>(X + (size_t)t0 * d_model, d_model, T - t0, Wg + (size_t)n0 * d_model,
                       Wu + (size_t)n0 * d_model, d_model, n_end - n0, n_end - n0, KSingle{d_model}, 0, nk,
                       lds, accg, accu);

    // alpha of the tile's neurons -> LDS (the main loop is done with it), from the table in the lanes: a search through
    // the kernel arguments at this point was a chain of loads with nothing to hide it (896 x 4864, 9 of 12 branches, T = 333:
    // the call 34.0 -> 30.4 us; in float, T = 256: 86.4 -> 84.6 us; 4096 x 14336, T = 100, with the batched sum of partial
    // results: 93.2 -> 89.8 us)
    float *al = reinterpret_cast<float *>(lds);
    int *bl = reinterpret_cast<int *>(lds + BNH_MAX * sizeof(float));      // branch of each neuron (routing)
    int *on = reinterpret_cast<int *>(lds + 2 * BNH_MAX * sizeof(float));  // neuron in an active branch (kEdges)
    const int n = n0 + threadIdx.x, n_last = (n0 + BNH < n_end ? n0 + BNH : n_end) - 1;
    int b = br.branch(n0);
    // n_last < d_inter: this ends at the entry that holds d_inter; threads past n_last are not used
    for (int i = b, next; (next = br.next(i)) <= n_last; ++i) b += next <= n ? 1 : 0;
    const float alpha = __shfl(br.v_alpha, b);
    if (threadIdx.x < BNH) {
        al[threadIdx.x] = n < n_end ? alpha : 0.f;
        if (kRouted) bl[threadIdx.x] = b;
        if (kEdges) on[threadIdx.x] = n < n_end && ((bt.active >> b) & 1ULL) ? 1 : 0;
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int tcol = lane & 15, q4 = lane >> 4;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int t = t0 + wm * (MI * 16) + i * 16 + tcol;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int nl = wn * (16 * NB) + j * 16 + 4 * q4;   // first of 4 neurons, tile relative
            // run ends are multiples of a chunk (rounded outwards with kEdges): the four are all inside or all outside
            if (t < T && n0 + nl < n_end) {
                const f32x4 a4 = *reinterpret_cast<const f32x4 *>(al + nl);
                f32x4 h;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[q] = gated<kEdges || sizeof(E) == 4>(a4[q], accg[i][j][q], accu[i][j][q]);
                    if (kRouted) h[q] = route[(size_t)t * bt.B + bl[nl + q]] ? h[q] : 0.f;
                }
                E *dst = H + (size_t)t * ldh + n0 + nl;
                if (kEdges && !(on[nl] & on[nl + 1] & on[nl + 2] & on[nl + 3])) {
                    // the columns of inactive branches are never written
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (on[nl + q]) store1(dst + q, h[q]);
                } else {
                    store4(dst, h);
                }
            }
        }
    }
}

// grid.x = 8 * ids_per_xcd(tilesM * sum over runs of N tiles).
template <int BMT, int WM, int NB, int D, bool kStaged, bool kEdges, typename E>
__global__ void __launch_bounds__(WM * 128)
gate_up_mfma(const E *__restrict__ X, const E *__restrict__ Wg,
             const E *__restrict__ Wu, E *__restrict__ H, int T, int d_model, int d_inter,
             int ldh, int tiles_m, int tiles_n, BranchTable bt)
{
    __shared__ __attribute__((aligned(1024))) char lds[lds_bytes(BMT, NB, D, kStaged)];
    constexpr int BNH = 32 * NB;                  // neurons per tile
    int tm, tn;
    if (!tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    int n0, n_end;
    if (!neuron_tile(bt, tn, BNH, n0, n_end)) return;
    gate_up_tile<BMT, WM, NB, D, kStaged, false, kEdges>(X, Wg, Wu, H, T, d_model, ldh, nullptr, bt, lds, tm, n0, n_end);
}

// The gate+up projection with WIDE tiles for the full rounds of 256 workgroups and smaller tiles for what
// is left, when that is at most half a round: the left-over wide tiles, cut into REST pieces, then fill one
// (shorter) round instead of leaving more than half of the CUs idle for a wide one.  REST = 2: halves of
// 64 neurons (NARROW's tile); REST = 4, when at most a quarter of a round is left: quarters of 128 tokens x
// 64 neurons, run by the same eight waves as 32 x (32 + 32) outputs each.
// Workgroup ids below 8 * wide_per_xcd take wide tiles: id i is tile (i % 8) * P + i / 8 of the grouped
// order, P = ids_per_xcd(wide tiles), i.e. every XCD works through the first wide_per_xcd tiles of its
// contiguous eighth.  The ids above take the rest of each eighth, REST consecutive ids per wide tile (the
// neuron half alternates fastest).  grid.x = 8 * (wide_per_xcd + REST * (P - wide_per_xcd)).
constexpr int QUARTER_D = 3;                          // ring depth of the quarter tiles (7 parts of 16 KiB)
template <int WM, int REST>
__global__ void __launch_bounds__(WM * 128)
gate_up_mfma_mixed(const uint16_t *__restrict__ X, const uint16_t *__restrict__ Wg,
                   const uint16_t *__restrict__ Wu, uint16_t *__restrict__ H, int T, int d_model, int ldh,
                   int tiles_m, int tiles_n, int wide_per_xcd, BranchTable bt)
{
    static_assert(REST == 2 || REST == 4, "halves or quarters of a wide tile");
    static_assert(lds_bytes(BM / 2, 2, QUARTER_D) <= lds_bytes(BM, 4), "the quarter tiles' ring fits the wide tiles' LDS");
    __shared__ __attribute__((aligned(1024))) char lds[lds_bytes(BM, 4)];
    const int total = tiles_m * tiles_n;
    const int P = ids_per_xcd(total);
    const int xcd = blockIdx.x % XCDS;
    const int xcd_end = (xcd + 1) * P < total ? (xcd + 1) * P : total;
    int k = blockIdx.x / XCDS;
    int tm, tn, n0, n_end;
    if (k < wide_per_xcd) {
        const int logical = xcd * P + k;
        if (logical >= xcd_end) return;
        tile_from_logical(logical, tiles_m, tiles_n, tm, tn);
        if (!neuron_tile(bt, tn, 128, n0, n_end)) return;
        gate_up_tile<BM, WM, 4, 2, false, false>(X, Wg, Wu, H, T, d_model, ldh, nullptr, bt, lds, tm, n0, n_end);
    } else {
        k -= wide_per_xcd;
        const int logical = xcd * P + wide_per_xcd + k / REST;
        if (logical >= xcd_end) return;
        tile_from_logical(logical, tiles_m, tiles_n, tm, tn);
        if (!neuron_tile(bt, tn, 128, n0, n_end)) return;
        n0 += (k % 2) * 64;
        if (n0 >= n_end) return;                                   // the run ends in the first half
        if (REST == 2) {
            gate_up_tile<BM, WM, 2, 2, false, false>(X, Wg, Wu, H, T, d_model, ldh, nullptr, bt, lds, tm, n0, n_end);
        } else {
            const int tq = 2 * tm + (k % 4) / 2;                   // token tile of 128
            if (tq * (BM / 2) >= T) return;                        // the last token tile ends in its first half
            gate_up_tile<BM / 2, WM, 2, QUARTER_D, false, false>(X, Wg, Wu, H, T, d_model, ldh, nullptr, bt, lds, tq,
                                                                 n0, n_end);
        }
    }
}

// The gate+up projection with per-token routing.  route[t * B + b] != 0 says token t takes branch b.  Only the live
// tiles are computed: workgroup ids are dealt over the compacted tile list as tile_of() deals them over the full grid
// (one contiguous stretch of the list per XCD), the ids left over exit.  The down projection skips the same (token
// tile, branch) pairs, and H is multiplied by the token's route bit, so that it is exactly 0 where a token does not
// take a branch.
// A live tile that only one half of its 256 tokens needs (sequences of a few hundred tokens end inside nearly every tile: 140
// of about 340 at 4096 x 14336, 16 branches, T = 1900, 7 sequences of 4 branches each) is computed like the others, or for that half
// alone: two quarters of 128 tokens x (64 + 64), which come after the whole tiles, and zeros stored for the other half.  How many
// tiles are live is known on the device only, so every workgroup decides, from when each way would end on 256 CUs:
//   like the others, a last round of at most 64 tiles as quarters, of at most 128 as halves of 256 x (64 + 64);
//   one-half tiles as quarters that start as CUs come free, the other tiles whole;
//   the same with the tiles of the last round that is not full cut into quarters too.
// In units of a whole tile's time a half takes 0.55 and a quarter 0.45, fitted to 392 calls (896 x 4864, 2048 x 8192, 3072 x 18000, 4096 x
// 14336; T = 60 .. 4000; 1 to 16 of 16 branches in 1 to 12 sequences), each timed all three ways.  The first way has to be 4 % longer by
// the estimate: the others ask for the weights of an N tile twice, far apart.  us a call, first / second way, tiles that both halves and
// one half need: 4096 x 14336, T = 60, 0 + 98 tiles 111 / 89; T = 550, 224 + 112 283 / 260; T = 1900, 196 + 147 266 / 246; 2048 x 8192, T = 1900,
// 252 + 104 171 / 156; as long by the estimate: 4096 x 14336, T = 3000, 420 + 77 428 / 454, 3072 x 18000, T = 550, 76 + 170 185 / 206; estimated
// shorter and not so: 3072 x 18000, T = 1398, 393 + 306 467 / 499.
// A workgroup past the last item has a CU to itself for as long as it takes to find out: with room for two per tile, 4176 ids for 240
// live tiles of 3072 x 18000 at T = 3000, the kernel took 90 us, with these ids 85.
// grid.x = 8 * (ids_per_xcd(all tiles) + kCUs / XCDS): `most` is what it holds whatever the split, ways with more items are not taken.
struct RoutedSplit {
    bool merge;           // one-half tiles are computed like the others
    int cut;              // tiles that are cut
    int pieces;           // into so many: 4 quarters or 2 halves
};
constexpr int ROUTED_WHOLE = 100, ROUTED_HALF = 55, ROUTED_QUARTER = 45;
// When `quarters` end that start as CUs come free: `busy` of them after a whole tile (2.2 quarters), the others at once.
__device__ __forceinline__ int routed_quarters_end(int busy, int quarters)
{
    const int idle = kCUs - busy;
    // after a quarters on the idle CUs (the busy ones have done a - 3), or after b on the busy ones (the idle ones b + 2)
    const int a = quarters <= 3 * idle ? (quarters + idle - 1) / idle : (quarters + 3 * busy + kCUs - 1) / kCUs;
    const int left = quarters - 2 * idle, b = left > 0 ? (left + kCUs - 1) / kCUs : 0;
    const int after_idle = a * ROUTED_QUARTER, after_busy = ROUTED_WHOLE + b * ROUTED_QUARTER;
    if (busy == 0) return after_idle;
    const int end = after_idle < after_busy ? after_idle : after_busy;
    return end > ROUTED_WHOLE ? end : ROUTED_WHOLE;
}
__device__ __forceinline__ RoutedSplit routed_split(int both, int singles, const RouteTiles &rt)
{
    const int live = both + singles, live_rest = live % kCUs, rest = both % kCUs;
    const int parts = live_rest == 0 || live_rest > kCUs / 2 ? 1 : (live_rest <= kCUs / 4 ? 4 : 2);
    RoutedSplit best{true, parts == 1 ? 0 : live_rest, parts == 1 ? 4 : parts};
    if (singles == 0 || rt.words) return best;
    int end = live / kCUs * ROUTED_WHOLE +
              (live_rest == 0 ? 0 : (parts == 1 ? ROUTED_WHOLE : (parts == 2 ? ROUTED_HALF : ROUTED_QUARTER)));
    end = both == 0 ? kOffEnd : end * 24 / 25;
    const int rounds = both / kCUs * ROUTED_WHOLE;
    const int cut_end = rounds + routed_quarters_end(0, 2 * singles + 4 * rest), whole_end = rounds + routed_quarters_end(rest, 2 * singles);
    if (cut_end <= end && both + 3 * rest + 2 * singles <= rt.most) {
        best = RoutedSplit{false, rest, 4};
        end = cut_end;
    }
    if (whole_end <= end && both + 2 * singles <= rt.most) best = RoutedSplit{false, 0, 4};
    return best;
}
template <int WM, bool kEdges>
__global__ void __launch_bounds__(WM * 128)
gate_up_mfma_routed(const uint16_t *__restrict__ X, const uint16_t *__restrict__ Wg,
                    const uint16_t *__restrict__ Wu, uint16_t *__restrict__ H, int T, int d_model, int ldh,
                    int tiles_m, const uint8_t *__restrict__ route, RouteTiles rt, BranchTable bt)
{
    constexpr int HALF = BM / 2;
    __shared__ __attribute__((aligned(1024))) char lds[lds_bytes(BM, 4)];
    const int groups = (tiles_m + GROUP_M - 1) / GROUP_M;
    int live = 0, both = 0;                            // live tiles, and those that both halves need
    for (int g = 0; g < groups; ++g) {
        live += (int)rt.counts[g];
        both += (int)rt.list[(size_t)g * rt.stride + rt.stride - 1];
    }
    const RoutedSplit split = routed_split(both, live - both, rt);
    if (split.merge) both = live;
    const int singles = live - both;
    const int wholes = both - split.cut, pieces = 2 * singles + split.pieces * split.cut;
    const int xcd = blockIdx.x % XCDS;
    int k = blockIdx.x / XCDS;
    const int whole_per_xcd = ids_per_xcd(wholes), piece_per_xcd = ids_per_xcd(pieces);
    int whole = -1, single = -1, piece = -1;           // the item: which whole tile or which one-half tile, which piece of it
    if (k < whole_per_xcd) {
        whole = xcd * whole_per_xcd + k;
        if (whole >= wholes) return;
    } else {
        k -= whole_per_xcd;
        const int i = xcd * piece_per_xcd + k;
        if (k >= piece_per_xcd || i >= pieces) return;
        if (i < 2 * singles) {
            single = i / 2;
            piece = i % 2;
        } else {
            whole = wholes + (i - 2 * singles) / split.pieces;
            piece = (i - 2 * singles) % split.pieces;
        }
    }
    int g = 0, at = whole >= 0 ? whole : single;       // entry `at` of the group's whole tiles or one-half tiles
    int first = 0;
    for (;; ++g) {
        const int c = (int)rt.counts[g], w = (int)rt.list[(size_t)g * rt.stride + rt.stride - 1];
        const int n = whole < 0 ? c - w : (split.merge ? c : w);
        first = whole >= 0 ? 0 : w;
        if (at < n || g == groups - 1) break;
        at -= n;
    }
    const uint32_t word = rt.list[(size_t)g * rt.stride + first + at], entry = split.merge ? word % (2 * ROUTE_SECOND) : word >> 16;
    const int e = (int)(rt.words ? word : entry % (split.merge ? 2 * ROUTE_SECOND : ROUTE_SECOND));
    const int m0 = g * GROUP_M;
    const int gsz = tiles_m - m0 < GROUP_M ? tiles_m - m0 : GROUP_M;
    const int tm = m0 + e % gsz, tn = e / gsz;
    int n0, n_end;
    if (!neuron_tile(bt, tn, 128, n0, n_end)) return;
    if (piece < 0) {
        gate_up_tile<BM, WM, 4, 2, false, true, kEdges>(X, Wg, Wu, H, T, d_model, ldh, route, bt, lds, tm, n0, n_end);
        return;
    }
    n0 += (piece % 2) * 64;
    if (n0 >= n_end) return;                                       // the run ends in the first half of the neurons
    if (n_end - n0 > 64) n_end = n0 + 64;
    if (split.pieces == 2) {                                       // then one-half tiles are like the others
        gate_up_tile<BM, WM, 2, 2, false, true, kEdges>(X, Wg, Wu, H, T, d_model, ldh, route, bt, lds, tm, n0, n_end);
        return;
    }
    const int half = 1 + (single >= 0 ? (int)(entry / ROUTE_SECOND) : piece / 2);
    if ((2 * tm + half - 1) * HALF >= T) return;                   // the last token tile ends in its first half
    gate_up_tile<HALF, WM, 2, QUARTER_D, false, true, kEdges>(X, Wg, Wu, H, T, d_model, ldh, route, bt, lds, 2 * tm + half - 1,
                                                              n0, n_end);
    if (single < 0) return;
    // zeros for the other half, neurons n0 .. n_end - 1 (kEdges: those of active branches, noted by gate_up_tile)
    const int *on = reinterpret_cast<const int *>(lds + 2 * BNH_MAX * sizeof(float));
    const int t_first = (2 * tm + 2 - half) * HALF, t_last = t_first + HALF < T ? t_first + HALF : T;
    for (int i = threadIdx.x; i < HALF * 8; i += WM * 128) {
        const int t = t_first + i / 8, nl = i % 8 * 8;
        if (t >= t_last || n0 + nl >= n_end) continue;
        uint16_t *dst = H + (size_t)t * ldh + n0 + nl;
        if constexpr (kEdges) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (on[nl + q]) dst[q] = 0;
        } else {
            *reinterpret_cast<u32x4 *>(dst) = u32x4{0, 0, 0, 0};
        }
    }
}

// grid.x = 8 * ids_per_xcd(splits * tilesM * tilesN); dst = out (splits == 1) or partial[split][T][d_model].
// dst_mode: DST_F32 plain float stores, DST_THROUGH the same past the L2; DST_BF16 (only with splits == 1) dst holds bf16 values, each sum
// rounded once (RNE).
// kRouted: the K loop of token tile tm walks only the branches some token of the tile is routed
// to (tile_need); H is 0 for the tokens of the tile that do not take a branch.
// kEdges: bt holds the runs rounded inwards (kRouted: the table's own runs; the ranges of a tile are rounded here)
// and `edges` (static tables) the partial chunks, which the last K split adds.
// kSpans (no room for the partial results of all splits): workgroup z of a tile goes through splits z * span .. and adds their sums
// up as reduce_partials does, `group` by group, so that the result has the same bits; grid.x = 8 * ids_per_xcd(spans * tilesM * tilesN),
// dst = out for one span, else partial[span][T][d_model].
template <int BMT, int WM, int NB, int D, bool kStaged, bool kRouted, bool kEdges, bool kSpans, typename E>
__global__ void __launch_bounds__(WM * 128)
down_mfma(const E *__restrict__ H, const E *__restrict__ Wd, float *__restrict__ dst, int T,
          int d_model, int d_inter, int ldh, int tiles_m, int tiles_n, int splits, int kt_total, int dst_mode, int span, int group,
          const uint8_t *__restrict__ tile_need, BranchTable bt, std::conditional_t<kEdges && !kRouted, EdgeList, NoEdges> edges)
{
    constexpr int BKE = Elem<E>::BK, CHUNK = Elem<E>::CHUNK;
    static_assert(!kRouted || BMT == BM, "the routed path's tables are per 256 tokens");
    __shared__ __attribute__((aligned(1024))) char lds[lds_bytes(BMT, NB, D, kStaged)];
    // Work items are (split, tile in the grouped order), split slowest, and every XCD takes one contiguous
    // eighth of that list: with K split, an XCD then works on few splits, whose slices of H and W_down are
    // what its L2 has to hold (the 0.5B-shaped layer at T = 2048: 4.7 MB per XCD instead of 12.5 MB).
    const int tiles = tiles_m * tiles_n;
    const long long items = (long long)tiles * (kSpans ? (splits + span - 1) / span : splits);
    const int per_xcd = ids_per_xcd(items);
    const long long item = (long long)(blockIdx.x % XCDS) * per_xcd + blockIdx.x / XCDS;
    if (item >= items) return;
    const int z = (int)(item / tiles);
    int tm, tn;
    tile_from_logical((int)(item % tiles), tiles_m, tiles_n, tm, tn);
    constexpr int BNH = 32 * NB;                  // output features per B block; a tile has two
    const int t0 = tm * BMT, n0 = tn * (2 * BNH);
    KRunsLanes dyn{0, 0, 0}, raw{0, 0, 0};
    if (kRouted) {
        raw = dyn = routed_runs(bt, tile_need + (size_t)tm * bt.B);
        if (kEdges) dyn = inner_runs<CHUNK>(raw);
        kt_total = 0;
        for (int r = 0; r < dyn.n; ++r) kt_total += (dyn.end(r) - dyn.start(r) + BKE - 1) / BKE;
    }
    constexpr int MI = BMT / 16 / WM;
    f32x4 acc0[MI][NB], acc1[MI][NB];
    // the second block of output features may start past d_model: point it at the last row
    const int n1 = n0 + BNH < d_model ? n0 + BNH : d_model - 1;
    const auto first_tile = [&](int part) { return (int)((long long)kt_total * part / splits); };
    const auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                acc0[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                acc1[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    // acc0, acc1 = the sums over K splits first .. last - 1, or since a stop last cleared them
    const auto sum_splits = [&](int first, int last, const auto &stops) {
        clear();
        if (kRouted)
            mainloop<BMT, WM, NB, D, kStaged, true>(H + (size_t)t0 * ldh, ldh, T - t0, Wd + (size_t)n0 * d_inter,
                                        Wd + (size_t)n1 * d_inter, d_inter, d_model - n0, d_model - n1, dyn,
                                        first_tile(first), first_tile(last), lds, acc0, acc1, stops);
        else
            mainloop<BMT, WM, NB, D, kStaged, true>(H + (size_t)t0 * ldh, ldh, T - t0, Wd + (size_t)n0 * d_inter,
                                        Wd + (size_t)n1 * d_inter, d_inter, d_model - n0, d_model - n1, KRuns{bt},
                                        first_tile(first), first_tile(last), lds, acc0, acc1, stops);
        if constexpr (kEdges) {
            const auto edge_at = [&](int i, int &col, unsigned &mask) {
                if constexpr (kRouted) {
                    run_edge<CHUNK>(__shfl(raw.v_start, i >> 1), __shfl(raw.v_end, i >> 1), i & 1, col, mask);
                } else {
                    col = edges.col[i];
                    mask = edges.mask[i];
                }
            };
            int n_edges;
            if constexpr (kRouted) n_edges = 2 * raw.n;
            else n_edges = edges.n;
            if (last == splits)
                edge_steps<MI, NB>(n_edges, edge_at, H + (size_t)t0 * ldh, ldh, T - t0, Wd + (size_t)n0 * d_inter,
                                   Wd + (size_t)n1 * d_inter, d_inter, d_model - n0, d_model - n1, acc0, acc1);
        }
    };
    if constexpr (kSpans) {
        f32x4 sum0[MI][NB], sum1[MI][NB], all0[MI][NB], all1[MI][NB];     // of the group, of the groups before it
        const int first = z * span, last = first + span < splits ? first + span : splits;
        int part = first;
        const auto add_split = [&]() {
            const int nth = part / group - first / group;                  // group of the split, from the first one on
            const bool starts = part == first || part % group == 0;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if (starts && nth > 0) {
                        all0[i][j] = nth == 1 ? sum0[i][j] : all0[i][j] + sum0[i][j];
                        all1[i][j] = nth == 1 ? sum1[i][j] : all1[i][j] + sum1[i][j];
                    }
                    sum0[i][j] = starts ? acc0[i][j] : sum0[i][j] + acc0[i][j];
                    sum1[i][j] = starts ? acc1[i][j] : sum1[i][j] + acc1[i][j];
                }
        };
        const auto next_split = [&](int kt) {
            if (part + 1 == last) return kt;              // the last one: its edges are still to come
            add_split();
            clear();
            ++part;
            return first_tile(part + 1);
        };
        sum_splits(first, last, Stops<decltype(next_split)>{next_split, first_tile(first + 1)});
        add_split();
        const bool one_group = (last - 1) / group == first / group;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                acc0[i][j] = one_group ? sum0[i][j] : all0[i][j] + sum0[i][j];
                acc1[i][j] = one_group ? sum1[i][j] : all1[i][j] + sum1[i][j];
            }
    } else {
        sum_splits(z, z + 1, NoStops{});
    }

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int tcol = lane & 15, q4 = lane >> 4;
    if (dst_mode == DST_THROUGH) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(dst, 0, (unsigned)THROUGH_BYTES, 0x00027000);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int t = t0 + wm * (MI * 16) + i * 16 + tcol;
#pragma unroll
            for (int j = 0; j < 2 * NB; ++j) {
                const int m = n0 + j / NB * BNH + wn * (16 * NB) + j % NB * 16 + 4 * q4;
                if (t < T && m < d_model)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, j < NB ? acc0[i][j % NB] : acc1[i][j % NB]), rsrc,
                                                           (unsigned)(((z * T + t) * d_model + m) * 4), 0, STORE_SC1);
            }
        }
        return;
    }
    float *o = dst + (size_t)z * T * d_model;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int t = t0 + wm * (MI * 16) + i * 16 + tcol;
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int m = n0 + half * BNH + wn * (16 * NB) + j * 16 + 4 * q4;
                // d_model is a multiple of a chunk (4 or 8): the four features are all inside or all outside
                if (t < T && m < d_model) {
                    const f32x4 v = half ? acc1[i][j] : acc0[i][j];
                    if (dst_mode == DST_BF16)
                        store4(reinterpret_cast<uint16_t *>(dst) + (size_t)t * d_model + m, v);
                    else
                        store4(o + (size_t)t * d_model + m, v);
                }
            }
    }
}

constexpr int ROUTE_MAX_TILES_N = 32768;           // N tiles of the gate+up projection the tile list handles

// Fills the routed kernels' scratch (see RouteTiles) for one group of GROUP_M token tiles per
// workgroup.  BNH = neurons per gate+up tile; tiles_n = N tiles over the runs of active branches.
template <int BNH>
__global__ void __launch_bounds__(1024)
route_tile_list(const uint8_t *__restrict__ route, uint8_t *__restrict__ tile_need, uint32_t *__restrict__ counts,
                uint32_t *__restrict__ list, int stride, bool words, int T, int tiles_m, int tiles_n, BranchTable bt)
{
    constexpr int HALVES = 2 * GROUP_M, HALF = BM / 2;
    __shared__ uint8_t need[HALVES][MLPMOE_MAX_BRANCHES];
    __shared__ uint16_t need_bits[MLPMOE_MAX_BRANCHES];    // bit h: half h of the group needs the branch
    __shared__ uint16_t live[ROUTE_MAX_TILES_N];
    __shared__ int s_off[MLPMOE_MAX_BRANCHES + 1], s_run_start[MLPMOE_MAX_BRANCHES], s_run_end[MLPMOE_MAX_BRANCHES];
    __shared__ int wave_both[16], wave_one[16];
    const int B = bt.B;
    const int g = blockIdx.x, m0 = g * GROUP_M;
    const int gsz = tiles_m - m0 < GROUP_M ? tiles_m - m0 : GROUP_M;
    for (int i = threadIdx.x; i < HALVES * MLPMOE_MAX_BRANCHES; i += 1024) (&need[0][0])[i] = 0;
    if (threadIdx.x < 64) {
        // branch table -> LDS, one entry per lane
        const int l = threadIdx.x, r = l < kMaxRuns ? l : kMaxRuns - 1;
        s_off[l] = bt.off[l];
        s_run_start[l] = bt.run_start[r];
        s_run_end[l] = bt.run_end[r];
        if (l == 0) s_off[MLPMOE_MAX_BRANCHES] = bt.off[MLPMOE_MAX_BRANCHES];
    }
    __syncthreads();
    // the group's rows of route are one contiguous stretch of bytes.  Flags already set are not
    // stored again: the LDS serialises the lanes of a store to one address, reads are broadcast
    const size_t base = (size_t)m0 * BM * B;
    const long long t_end = (long long)(m0 + gsz) * BM < T ? (long long)(m0 + gsz) * BM : T;
    const int n_bytes = (int)((t_end - (long long)m0 * BM) * B);
    const uint8_t *rg = route + base;
    // 16 bytes at a time where the pointer allows it, several loads in flight per thread; one
    // division per 16 bytes, the (token, branch) of the following bytes by stepping
    const int n_vec = (reinterpret_cast<uintptr_t>(rg) & 15u) == 0 ? n_bytes / 16 : 0;
    for (int c0 = threadIdx.x; c0 < n_vec; c0 += 4 * 1024) {
        u32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * 1024;
            v[u] = c < n_vec ? *reinterpret_cast<const u32x4 *>(rg + (size_t)c * 16) : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if ((v[u][0] | v[u][1] | v[u][2] | v[u][3]) == 0) continue;
            const int i = (c0 + u * 1024) * 16;
            int t = i / B, b = i - t * B;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                if (((v[u][k / 4] >> (8 * (k % 4))) & 0xffu) && !need[t / HALF][b]) need[t / HALF][b] = 1;
                if (++b == B) {
                    b = 0;
                    ++t;
                }
            }
        }
    }
    for (int i0 = n_vec * 16 + threadIdx.x; i0 < n_bytes; i0 += 8 * 1024) {
        uint8_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * 1024;
            v[u] = i < n_bytes ? rg[i] : (uint8_t)0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v[u]) {
                const int i = i0 + u * 1024;
                if (!need[(i / B) / HALF][i % B]) need[(i / B) / HALF][i % B] = 1;
            }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < gsz * B; i += 1024)
        tile_need[(size_t)m0 * B + i] = need[2 * (i / B)][i % B] | need[2 * (i / B) + 1][i % B] << 1;
    if (threadIdx.x < MLPMOE_MAX_BRANCHES) {
        unsigned bits = 0;
#pragma unroll
        for (int h = 0; h < HALVES; ++h) bits |= need[h][threadIdx.x] ? 1u << h : 0u;
        need_bits[threadIdx.x] = (uint16_t)bits;
    }
    __syncthreads();

    // live[tn]: bits 2 j, 2 j + 1 say that a half of tile (m0 + j, tn) is live; one thread per N tile.  The branch table was
    // copied to LDS above, so that the walks over runs and branches are chains of LDS reads.
    for (int tn = threadIdx.x; tn < tiles_n; tn += 1024) {
        int n0 = 0, n1 = 0, left = tn;
        bool found = false;
        for (int r = 0; r < bt.n_runs; ++r) {
            const int n = (s_run_end[r] - s_run_start[r] + BNH - 1) / BNH;
            if (!found && left < n) {
                n0 = s_run_start[r] + left * BNH;
                n1 = n0 + BNH < s_run_end[r] ? n0 + BNH : s_run_end[r];
                found = true;
            }
            left -= n;
        }
        unsigned bits = 0;
        for (int b = 0; b < B; ++b) {
            const int lo = s_off[b], hi = s_off[b + 1];
            if (!((bt.active >> b) & 1ULL) || hi <= lo || hi <= n0 || lo >= n1) continue;   // owns no neuron of the tile
            bits |= need_bits[b];
        }
        live[tn] = (uint16_t)bits;
    }
    __syncthreads();

    // compaction into both orders of the list: every thread takes a contiguous stretch of N tiles, an exclusive prefix over the
    // threads gives its first positions
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = (tiles_n + 1023) / 1024;
    const int tn0 = threadIdx.x * per;
    const int tn1 = tn0 + per < tiles_n ? tn0 + per : tiles_n;
    const auto both_of = [](unsigned l) { return l & (l >> 1) & 0x5555u; };      // bit 2 j: both halves of tile j
    const auto one_of = [](unsigned l) { return (l ^ (l >> 1)) & 0x5555u; };     // bit 2 j: one of them
    int n_both = 0, n_one = 0;
    for (int tn = tn0; tn < tn1; ++tn) {
        n_both += __popc(both_of(live[tn]));
        n_one += __popc(one_of(live[tn]));
    }
    int incl_both = n_both, incl_one = n_one;
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(incl_both, d), w = __shfl_up(incl_one, d);
        incl_both += lane >= d ? v : 0;
        incl_one += lane >= d ? w : 0;
    }
    if (lane == 63) {
        wave_both[wave] = incl_both;
        wave_one[wave] = incl_one;
    }
    __syncthreads();
    int pos_both = incl_both - n_both, pos_one = incl_one - n_one, all_both = 0, all_one = 0;
    for (int w = 0; w < 16; ++w) {
        pos_both += w < wave ? wave_both[w] : 0;
        pos_one += w < wave ? wave_one[w] : 0;
        all_both += wave_both[w];
        all_one += wave_one[w];
    }
    uint32_t *out = list + (size_t)g * stride;
    uint16_t *out16 = reinterpret_cast<uint16_t *>(out);
    if (threadIdx.x == 0) {
        counts[g] = (uint32_t)(all_both + all_one);
        out[stride - 1] = (uint32_t)all_both;
    }
    for (int tn = tn0; tn < tn1; ++tn)
        for (int j = 0; j < gsz; ++j) {
            const unsigned h = (live[tn] >> (2 * j)) & 3u;
            const uint32_t tile = (uint32_t)(tn * gsz + j);
            const int pos = pos_both + pos_one;
            if (!h) continue;
            if (words) {
                out[pos] = tile;
            } else {
                out16[2 * pos] = (uint16_t)tile;
                out16[2 * (h == 3 ? pos_both : all_both + pos_one) + 1] = (uint16_t)(tile + (h == 2 ? ROUTE_SECOND : 0u));
            }
            if (h == 3) ++pos_both;
            else ++pos_one;
        }
}

// out[i] = sum_z partial[z][i], summed in z order, kGroups: each `group` of them, then the groups: deterministic.  out_bf16: out
// holds bf16 values.
// n4 = pieces of four values (T * d_model is a multiple of 4 on this path; partial is 256-byte, out 16-byte
// aligned).  A thread adds PIECES pieces per trip and has the loads of BATCH partial sums of each in flight.
// Large results are bound by memory: two pieces far apart, one partial sum after the other (512 x 4096, 8 partial sums:
// 13.8 us with event brackets, 16.7 us with one piece and a batch of 8).  Small ones are bound by latency: one piece per
// thread in small workgroups, which spreads them over the chip, and a batch of 8 (128 x 896, 18 partial sums: 9.2 ->
// 6.2 us, 100 x 4096, 8: 6.7 -> 6.3 us).  The line is where one thread per piece fills the chip.
constexpr size_t REDUCE_SMALL_N4 = 256 * 1024;
template <int THREADS, int PIECES, int BATCH, bool kGroups>
__global__ void __launch_bounds__(THREADS)
reduce_partials(const float *__restrict__ partial, float *__restrict__ out, size_t n4, int splits, int group, int out_bf16)
{
    const f32x4 *p4 = reinterpret_cast<const f32x4 *>(partial);
    const size_t stride = (size_t)gridDim.x * THREADS;
    for (size_t i = blockIdx.x * (size_t)THREADS + threadIdx.x; i < n4; i += PIECES * stride) {
        f32x4 s[PIECES], all[PIECES];                     // of the group, of the groups before it
#pragma unroll
        for (int k = 0; k < PIECES; ++k) s[k] = i + k * stride < n4 ? p4[i + k * stride] : f32x4{0.f, 0.f, 0.f, 0.f};
        for (int z = 1; z < splits; z += BATCH) {
            f32x4 v[BATCH][PIECES];
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
                if (z + u < splits) {
#pragma unroll
                    for (int k = 0; k < PIECES; ++k)
                        v[u][k] = i + k * stride < n4 ? p4[(size_t)(z + u) * n4 + i + k * stride] : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
                if (z + u < splits) {
                    if (kGroups && (z + u) % group == 0) {
#pragma unroll
                        for (int k = 0; k < PIECES; ++k) {
                            all[k] = z + u == group ? s[k] : all[k] + s[k];
                            s[k] = v[u][k];
                        }
                        continue;
                    }
#pragma unroll
                    for (int k = 0; k < PIECES; ++k) s[k] += v[u][k];
                }
        }
        if (kGroups) {
#pragma unroll
            for (int k = 0; k < PIECES; ++k) s[k] = all[k] + s[k];
        }
#pragma unroll
        for (int k = 0; k < PIECES; ++k) {
            const size_t j = i + k * stride;
            if (j >= n4) continue;
            if (out_bf16)
                store4(reinterpret_cast<uint16_t *>(out) + j * 4, s[k]);
            else
                store4(out + j * 4, s[k]);
        }
    }
}

int k_tiles(const BranchTable &bt, int bk = BK)
{
    int n = 0;
    for (int r = 0; r < bt.n_runs; ++r) n += ceil_div(bt.run_end[r] - bt.run_start[r], bk);
    return n;
}

// The run lists of a table whose boundaries are not multiples of `chunk`: rounded outwards without overlap (gate+up),
// rounded inwards without empty ones (down), and the partial chunks.  outer / inner keep everything else of bt.
struct UnevenRuns {
    BranchTable outer, inner;
    EdgeList edges;
};
template <int CHUNK>
void uneven_runs(const BranchTable &bt, UnevenRuns &u)
{
    u.outer = u.inner = bt;
    u.outer.n_runs = u.inner.n_runs = u.edges.n = 0;
    for (int r = 0; r < bt.n_runs; ++r) {
        const int s = bt.run_start[r], e = bt.run_end[r];
        const int os = s / CHUNK * CHUNK;
        const int oe = (e + CHUNK - 1) / CHUNK * CHUNK;
        BranchTable &o = u.outer;
        if (o.n_runs > 0 && os <= o.run_end[o.n_runs - 1]) {
            o.run_end[o.n_runs - 1] = oe;             // shares a chunk with the run before it, or touches it
        } else {
            o.run_start[o.n_runs] = os;
            o.run_end[o.n_runs++] = oe;
        }
        const int is = (s + CHUNK - 1) / CHUNK * CHUNK, ie = e / CHUNK * CHUNK;
        if (ie > is) {
            u.inner.run_start[u.inner.n_runs] = is;
            u.inner.run_end[u.inner.n_runs++] = ie;
        }
        for (int side = 0; side < 2; ++side) {
            int col;
            unsigned mask;
            run_edge<CHUNK>(s, e, side, col, mask);
            if (!mask) continue;
            u.edges.col[u.edges.n] = col;
            u.edges.mask[u.edges.n++] = (uint8_t)mask;
        }
    }
}

// Tile shapes.  WIDE: 256 tokens x (128 + 128) rows of B, the shape with the most reuse per byte moved
// into the LDS.  NARROW: 256 x (64 + 64).  SMALL: 128 x (64 + 64) with 4 waves and 80 KiB of LDS, two
// workgroups per CU: four times the tiles of WIDE, the fixed cost of one workgroup (first loads,
// epilogue, hand-over) hidden under the main loop of the other, at 1.6 times WIDE's traffic into the
// LDS per flop.  For layers and batches that give WIDE too few or too short tiles.
// MIXED (gate+up only): WIDE for the full rounds of 256 workgroups, NARROW for a last round that WIDE tiles
// would fill less than half; quarters of a wide tile (128 tokens x (64 + 64)) where they fit one round.
// DEEP: SMALL's tile with four K tiles requested ahead instead of two (a ring of 9 parts, 144 KiB, one
// workgroup per CU): for batches of a few dozen to a hundred tokens, where a launch has about one tile per
// CU and is bound by how many bytes of weights it keeps in flight, not by the matrix cores.
// SLIM: 64 tokens x (64 + 64) with 4 waves and a staged ring of five K tiles requested ahead (144 KiB, one
// workgroup per CU): the A rows of a K tile take a third of a stage, so more bytes of the B operand are in
// flight per CU than with any other shape; for outputs with few token rows per output feature (a down
// projection with a short d_model can then do without a K split) and for gate+up projections whose 64-token tiles fit one
// round of workgroups.
enum TileShape { TILE_WIDE = 0, TILE_NARROW = 1, TILE_SMALL = 2, TILE_MIXED = 3, TILE_DEEP = 4, TILE_SLIM = 5 };
constexpr int N_TILE_SHAPES = 6;
constexpr int DEEP_D = 4, SLIM_D = 5;
// compile-time side of a tile shape: tokens, waves along M, 16-row MFMA pieces per B block and wave, K tiles
// requested ahead, ring layout
template <int BMT_, int WM_, int NB_, int D_, bool kStaged_>
struct ShapeT {
    static constexpr int BMT = BMT_, WM = WM_, NB = NB_, D = D_;
    static constexpr bool kStaged = kStaged_;
};
using ShapeWide = ShapeT<BM, MFMA_WM, 4, 2, false>;
using ShapeNarrow = ShapeT<BM, MFMA_WM, 2, 2, false>;
using ShapeSmall = ShapeT<BM_SMALL, SMALL_WM, 2, 2, false>;
using ShapeDeep = ShapeT<BM_SMALL, SMALL_WM, 2, DEEP_D, false>;
using ShapeSlim = ShapeT<BM_SLIM, SLIM_WM, 2, SLIM_D, true>;
// Float storage: 64 tokens x (32 + 32), 4 waves of 32 x (16 + 16) outputs, 40 KiB, four workgroups per CU.  Bound: the
// float MFMA rate (v_mfma_f32_16x16x4_f32, 256 flop per clock and CU, a sixteenth of bf16's), which this small a tile
// already reaches: it asks the L2 for 16 bytes per clock and CU while the matrix pipe is busy, of about 40 available,
// and small tiles fill the chip at the sizes float storage is used for (4864 neurons and 256 tokens are 608 tiles; the
// 128 x (64 + 64) tile would make 152).  The layer at T = 256: 80 us against 1007 us on the general FMA kernels, error
// against float64 0.64e-6 against 1.5e-6 (rel.).
// Gate+up also with 32 tokens: half the work per tile where 64 leave the last round of workgroups emptier, and with four
// K tiles requested ahead where there are at most two workgroups per CU to hide each other's latency (see pick_f32_tokens).
using ShapeF32 = ShapeT<64, 2, 1, 2, false>;
using ShapeF32Half = ShapeT<32, 2, 1, 2, false>;
using ShapeF32HalfDeep = ShapeT<32, 2, 1, 4, false>;
struct TileDims {
    int bm, bn;       // tokens, B rows per block (a tile has two blocks)
    int per_cu;       // workgroups resident per CU
};
constexpr TileDims kTileDims[N_TILE_SHAPES] = {{BM, 128, 1}, {BM, 64, 1}, {BM_SMALL, 64, 2}, {BM, 128, 1}, {BM_SMALL, 64, 1},
                                               {BM_SLIM, 64, 1}};

long long gate_up_tiles(const BranchTable &bt, int T, TileShape sh)
{
    long long n = 0;
    for (int r = 0; r < bt.n_runs; ++r) n += ceil_div(bt.run_end[r] - bt.run_start[r], kTileDims[sh].bn);
    return n * ceil_div(T, kTileDims[sh].bm);
}

// Estimated duration in microseconds of a launch of the down projection, `tiles` tiles with nk K tiles each that stream
// `bytes` of weights and activations, fitted to measurements on the two benchmark layers (T = 64 .. 4096):
// a K tile of a WIDE tile takes about 1.48 us at the clocks the chip sustains on this work, a NARROW one
// 0.62 of that, a SMALL one 0.4 (two share a CU, each at a quarter of a WIDE tile's flops but bound by the
// traffic into the LDS; an odd one at the end runs alone at about 0.3); the fixed cost of a workgroup
// (first loads, epilogue, hand-over) is about 7.4 / 5.2 us and 1.5 us for SMALL, whose neighbour on the CU
// computes meanwhile; DEEP (SMALL's tile alone on its CU) 0.75 and 4.4 us; SLIM 0.6 and 3.5 us.  A launch that
// has few tiles per CU cannot stream faster than about 3.5 TB/s, 5 TB/s with DEEP's and SLIM's longer queues of
// requests, 3 TB/s with SMALL's (4096 x 14336, T = 200 as 512 SMALL tiles 54.0, as 256 NARROW ones 49.6 us with event brackets;
// T = 256 57.2 and 51.9; 3072 x 8192, T = 160 34.4 and 32.0).
constexpr double kDeepStreamBytesPerUs = 5.0e6;
double launch_cost_us(long long tiles, int nk, TileShape sh, double bytes)
{
    static const double per_k[N_TILE_SHAPES] = {1.48, 0.92, 0.59, 1.48, 0.75, 0.6}, fixed[N_TILE_SHAPES] = {7.4, 5.2, 1.5, 7.4, 4.4, 3.5};
    const long long per_cu = (tiles + kCUs - 1) / kCUs;       // tiles the busiest CU runs, one after the other
    double c;
    if (sh == TILE_SMALL)
        c = (double)(per_cu / 2) * 2 * (nk * per_k[sh] + fixed[sh]) + (double)(per_cu % 2) * (nk * 0.44 + 4.4);
    else
        c = (double)per_cu * (nk * per_k[sh] + fixed[sh]);
    // DEEP keeps twice the bytes in flight
    const double rate = sh == TILE_DEEP || sh == TILE_SLIM ? kDeepStreamBytesPerUs : (sh == TILE_SMALL ? 3.0e6 : 3.5e6);
    return std::max(c, bytes / rate + fixed[sh]);
}

// Wide tiles that MIXED runs as wide, per XCD (32 per full round of 256), or -1 if MIXED does not apply:
// it needs at least one full round and a remainder of at most half a round.
int mixed_wide_per_xcd(long long wide_tiles)
{
    const long long rounds = wide_tiles / kCUs, rest = wide_tiles % kCUs;
    if (rounds < 1 || rest == 0 || rest > kCUs / 2 || wide_tiles > 0x3fffffffLL) return -1;
    return (int)(rounds * (kCUs / XCDS));
}

// Pieces MIXED cuts each left-over wide tile into: quarters when they fit one round, else halves.
int mixed_rest_parts(long long wide_tiles) { return wide_tiles % kCUs <= kCUs / 4 ? 4 : 2; }

// Estimate for a launch of the gate+up projection, whose K loops are as short as d_model: fitted to the kernel alone with
// every shape on twelve layers, 384 x 1024 .. 4096 x 14336, at 18 batches T = 17 .. 4096, and checked on whole calls (half a
// per cent from the fastest shape in the mean).  A round of workgroups takes `round` + nk K tiles of per_k, SMALL 1.45 + 1.05 per K tile
// where two share a CU and 0.73 for an odd one; few tiles stream the weights at the given rate.
// Against launch_cost_us, which is fitted to long K loops: 896 x 4864, T = 64 SMALL 13.9 -> SLIM 11.2 us (with event brackets),
// T = 256 (6 x 38 tiles) SMALL 16.5 -> DEEP 14.8; 2048 x 5504, T = 32 SMALL 31.5 -> SLIM 19.5, T = 200 32.3 -> DEEP 24.8; 3072 x
// 8192, T = 64 46.2 -> SLIM 33.9, T = 200 46.4 -> DEEP 37.9; 4096 x 11008, T = 96 60.7 -> DEEP 44.3.
double gate_up_cost_us(long long tiles, int nk, TileShape sh, double bytes)
{
    static const double per_k[N_TILE_SHAPES] = {1.21, 0.87, 1.05, 1.21, 0.6, 0.394}, round[N_TILE_SHAPES] = {4.5, 2.1, 1.45, 4.5, 3.9, 2.7};
    static const double bytes_per_us[N_TILE_SHAPES] = {3.2e6, 3.9e6, 4.05e6, 3.2e6, 6.1e6, 6.3e6};
    const long long per_cu = (tiles + kCUs - 1) / kCUs;
    const double c = sh == TILE_SMALL ? (double)(per_cu / 2) * (nk * per_k[sh] + round[sh]) + (double)(per_cu % 2) * (nk * 0.73 + round[sh])
                                      : (double)per_cu * (nk * per_k[sh] + round[sh]);
    return std::max(c, bytes / bytes_per_us[sh] + round[sh]);
}

TileShape pick_gate_up_tile(const BranchTable &bt, int T, int d_model)
{
    const int nk = ceil_div(d_model, BK);
    const double bytes = 4.0 * bt.d_eff * d_model;            // W_gate and W_up rows of the active neurons, once
    const long long wide = gate_up_tiles(bt, T, TILE_WIDE);
    TileShape best = TILE_WIDE;
    double best_cost = gate_up_cost_us(wide, nk, TILE_WIDE, bytes);
    for (TileShape sh : {TILE_NARROW, TILE_SMALL, TILE_DEEP, TILE_SLIM}) {
        const double c = gate_up_cost_us(gate_up_tiles(bt, T, sh), nk, sh, bytes);
        if (c < best_cost) {
            best = sh;
            best_cost = c;
        }
    }
    if (mixed_wide_per_xcd(wide) >= 0) {
        // the full rounds as wide tiles, then one round of narrow ones, or of quarters (measured 2 us shorter
        // at 14 K tiles)
        const double c = gate_up_cost_us(wide / kCUs * kCUs, nk, TILE_WIDE, 0.0) + gate_up_cost_us(kCUs, nk, TILE_NARROW, 0.0) -
                         (mixed_rest_parts(wide) == 4 ? 2.0 : 0.0);
        if (c < best_cost) best = TILE_MIXED;
    }
    return best;
}

// Split-K factor of the down projection: fills the chip when the output has few tiles.
int down_splits(int T, int d_model, int k_elems, TileShape sh)
{
    const TileDims &d = kTileDims[sh];
    const long long tiles = (long long)ceil_div(T, d.bm) * ceil_div(d_model, 2 * d.bn);
    const int kt = ceil_div(k_elems > 0 ? k_elems : 1, BK);
    long long s = (long long)kCUs * d.per_cu / tiles;
    if (s > kt / 4) s = kt / 4;
    if (s > 32) s = 32;
    return s < 1 ? 1 : (int)s;
}

// Estimate for a launch of the down projection.  K loops of at most 16 tiles (what a K split of a narrow layer leaves) have
// their operands in the caches: a K tile takes SLIM 0.44 and DEEP 0.6 us there, the first loads and the stores of a SLIM
// workgroup 2.5 us and of a pair of SMALL ones 2.2 us each (896 x 4864 at T = 128 .. 600).  Checked on 260 drawn layers of
// 384 .. 4096 features at T = 17 .. 4096, side by side with the estimate for long loops alone: the call 1.13 times faster
// in the mean with the batched sum, none slower by more than the runs of one side differ.
// SLIM without a K split stays below its long-loop estimate up to 32 tiles, 0.45 and 4.0 us, or a layer of
// 384 to 640 features is split at T >= 1700 where it need not be (448 x 1408, T = 3565: 36.1 us, unsplit 35.0).
constexpr int SHORT_K_TILES = 16;
double down_cost_us(long long tiles, int splits, int nk, TileShape sh, double bytes)
{
    tiles *= splits;
    double c = launch_cost_us(tiles, nk, sh, bytes);
    const double rounds = (double)((tiles + kCUs - 1) / kCUs);
    if (sh == TILE_SLIM && splits == 1 && nk > SHORT_K_TILES && nk <= 2 * SHORT_K_TILES)
        return std::max(rounds * (nk * 0.45 + 4.0), bytes / kDeepStreamBytesPerUs + 4.0);
    if (nk > SHORT_K_TILES) return c;
    if (sh == TILE_SLIM) c = std::max(rounds * (nk * 0.44 + 2.5), bytes / kDeepStreamBytesPerUs + 2.5);
    if (sh == TILE_DEEP) c = std::max(rounds * (nk * 0.6 + 4.4), bytes / kDeepStreamBytesPerUs + 4.4);
    if (sh == TILE_SMALL && rounds >= 2) c += 0.7 * 2 * (int)(rounds / 2);
    return c;
}

// The sum of sp partial results of n floats: about 5 us for small ones, and 3.3 us plus its traffic at 6.5 TB/s.
double reduce_cost_us(int sp, double n) { return sp > 1 ? std::max(5.0, 3.3 + (sp + 1.0) * n * 4.0 / 6.5e6) : 0.0; }

// How the down projection of one call is launched: tile shape and K split (the partial results of a split
// go through the workspace and a second kernel adds them up in a fixed order; adding two halves into
// the result with float atomics instead was measured 2.4 times slower on the 0.5B-shaped layer).
struct DownPlan {
    TileShape shape;
    int splits;
};

DownPlan plan_down(const FwdArgs &a, const BranchTable &bt, bool routed)
{
    const int kt = std::max(1, k_tiles(bt));
    DownPlan best{TILE_WIDE, 1};
    double best_cost = 1e30;
    for (TileShape sh : {TILE_WIDE, TILE_NARROW, TILE_SMALL, TILE_DEEP, TILE_SLIM}) {
        if (a.tile_shape >= 0 && a.tile_shape != (int)TILE_MIXED && a.tile_shape != (int)sh) continue;
        if (routed && kTileDims[sh].bm != BM) continue;
        const TileDims &d = kTileDims[sh];
        const long long tiles = (long long)ceil_div(a.T, d.bm) * ceil_div(a.d_model, 2 * d.bn);
        const int fill = std::min(down_splits(a.T, a.d_model, bt.d_eff, sh), kt);
        // Split as far as it fills the chip or, with SMALL and a short K, as far as gives every CU one workgroup: half the
        // partial sums, and no pair that shares a CU.  896 x 4864 in one run: T = 333 31.3 -> 28.6, T = 600 37.4 -> 34.4,
        // T = 128 (SLIM instead of SMALL) 26.4 -> 25.4 us.
        for (int sp : {fill, fill / 2}) {
            if (sp < 1 || (sp != fill && (sh != TILE_SMALL || ceil_div(kt, sp) > SHORT_K_TILES))) continue;
            if (sp > 1 && (size_t)sp * a.T * a.d_model * sizeof(float) > a.partial_bytes) sp = 1;
            const double c = down_cost_us(tiles, sp, ceil_div(kt, sp), sh, 2.0 * bt.d_eff * (a.d_model + a.T)) +
                             reduce_cost_us(sp, (double)a.T * a.d_model);
            if (c < best_cost) {
                best = DownPlan{sh, sp};
                best_cost = c;
            }
        }
    }
    return best;
}

}  // namespace

int mfma_down_splits(int T, int d_model, int k_elems) { return down_splits(T, d_model, k_elems, TILE_WIDE); }

// Layout of the routed kernels' scratch block (256-byte aligned): tile_need, counts, list.
// The list holds, per group of GROUP_M token tiles, up to GROUP_M * (N tiles) entries; the N tiles
// over runs of active branches number at most d_inter / 128 + one per run.
namespace {
int route_list_stride(int d_inter) { return GROUP_M * (d_inter / BNH_MAX + MLPMOE_MAX_BRANCHES + 1); }
size_t route_need_bytes(int T) { return align_up((size_t)ceil_div(T, BM) * MLPMOE_MAX_BRANCHES, 256); }
size_t route_counts_bytes(int T) { return align_up((size_t)ceil_div(ceil_div(T, BM), GROUP_M) * sizeof(uint32_t), 256); }
}  // namespace

size_t route_scratch_bytes(int T, int d_inter)
{
    if (T < 1) T = 1;
    if (d_inter < 0) d_inter = 0;
    const size_t groups = (size_t)ceil_div(ceil_div(T, BM), GROUP_M);
    return route_need_bytes(T) + route_counts_bytes(T) +
           align_up(groups * route_list_stride(d_inter) * sizeof(uint32_t), 256);
}

// Every table of this width has few enough N tiles for the tile list.
bool mfma_routed_holds(int d_inter) { return d_inter / BNH_MAX + kMaxRuns <= ROUTE_MAX_TILES_N; }

size_t mfma_partial_bytes(int T, int d_model, int d_inter)
{
    // the largest any tile shape asks for
    int s = 1;
    for (TileShape sh : {TILE_WIDE, TILE_NARROW, TILE_SMALL, TILE_DEEP, TILE_SLIM}) s = std::max(s, down_splits(T, d_model, d_inter, sh));
    return s > 1 ? align_up((size_t)s * T * d_model * sizeof(float), 256) : 0;
}

template <typename S, bool kEdges = false, typename E = uint16_t>
static hipError_t launch_gate_up(const FwdArgs &a, const BranchTable &bt)
{
    constexpr int BMT = S::BMT, WM = S::WM, NB = S::NB;
    const int tiles_m = ceil_div(a.T, BMT);
    long long tiles_n = 0;
    for (int r = 0; r < bt.n_runs; ++r) tiles_n += ceil_div(bt.run_end[r] - bt.run_start[r], 32 * NB);
    const long long grid = (long long)XCDS * ids_per_xcd(tiles_m * tiles_n);
    if (grid > 0x7fffffffLL) return note_hip_error("gate_up_mfma grid", hipErrorInvalidValue);
    ProfileScope ps(MLPMOE_KERNEL_GATE_UP_MFMA, a.stream);
    gate_up_mfma<BMT, WM, NB, S::D, S::kStaged, kEdges><<<(unsigned)grid, WM * 128, 0, a.stream>>>(
        static_cast<const E *>(a.x), static_cast<const E *>(a.Wg), static_cast<const E *>(a.Wu), static_cast<E *>(a.H), a.T,
        a.d_model, a.d_inter, a.ldh, tiles_m, (int)tiles_n, bt);
    return launch_status("gate_up_mfma launch");
}

// One launch builds the list of live tiles (and tile_need, which the down projection reads as well), one walks it.
template <bool kEdges>
static hipError_t launch_gate_up_routed(const FwdArgs &a, const BranchTable &bt)
{
    const int tiles_m = ceil_div(a.T, BM);
    long long tiles_n = 0;
    for (int r = 0; r < bt.n_runs; ++r) tiles_n += ceil_div(bt.run_end[r] - bt.run_start[r], BNH_MAX);
    const long long grid = (long long)XCDS * (ids_per_xcd(tiles_m * tiles_n) + kCUs / XCDS);
    if (grid > 0x7fffffffLL) return note_hip_error("gate_up_mfma_routed grid", hipErrorInvalidValue);
    uint8_t *need = a.route_scratch;
    uint32_t *counts = reinterpret_cast<uint32_t *>(a.route_scratch + route_need_bytes(a.T));
    uint32_t *list = reinterpret_cast<uint32_t *>(a.route_scratch + route_need_bytes(a.T) + route_counts_bytes(a.T));
    const int stride = route_list_stride(a.d_inter);
    if ((long long)GROUP_M * tiles_n > stride - 1 || tiles_n > ROUTE_MAX_TILES_N)
        return note_hip_error("route tile list size", hipErrorInvalidValue);
    const bool words = GROUP_M * tiles_n > (long long)ROUTE_SECOND;
    {
        ProfileScope ps(MLPMOE_KERNEL_ROUTE_TILES, a.stream);
        route_tile_list<BNH_MAX><<<ceil_div(tiles_m, GROUP_M), 1024, 0, a.stream>>>(
            a.route, need, counts, list, stride, words, a.T, tiles_m, (int)tiles_n, bt);
    }
    if (launch_status("route_tile_list launch") != hipSuccess) return hipErrorLaunchFailure;
    ProfileScope ps(MLPMOE_KERNEL_GATE_UP_MFMA, a.stream);
    gate_up_mfma_routed<MFMA_WM, kEdges><<<(unsigned)grid, MFMA_WM * 128, 0, a.stream>>>(
        static_cast<const uint16_t *>(a.x), static_cast<const uint16_t *>(a.Wg), static_cast<const uint16_t *>(a.Wu),
        static_cast<uint16_t *>(a.H), a.T, a.d_model, a.ldh, tiles_m, a.route,
        RouteTiles{need, counts, list, stride, words, (int)grid - 2 * XCDS}, bt);
    return launch_status("gate_up_mfma_routed launch");
}

static hipError_t launch_gate_up_mixed(const FwdArgs &a, const BranchTable &bt)
{
    const int tiles_m = ceil_div(a.T, BM);
    long long tiles_n = 0;
    for (int r = 0; r < bt.n_runs; ++r) tiles_n += ceil_div(bt.run_end[r] - bt.run_start[r], BNH_MAX);
    const int wide_per_xcd = mixed_wide_per_xcd(tiles_m * tiles_n);
    if (wide_per_xcd < 0) return note_hip_error("gate_up_mfma_mixed: tile count", hipErrorInvalidValue);
    const int rest_per_xcd = ids_per_xcd(tiles_m * tiles_n) - wide_per_xcd;
    const int parts = mixed_rest_parts(tiles_m * tiles_n);
    const long long grid = (long long)XCDS * (wide_per_xcd + (long long)parts * rest_per_xcd);
    ProfileScope ps(MLPMOE_KERNEL_GATE_UP_MFMA, a.stream);
    const auto kernel = parts == 4 ? gate_up_mfma_mixed<MFMA_WM, 4> : gate_up_mfma_mixed<MFMA_WM, 2>;
    kernel<<<(unsigned)grid, MFMA_WM * 128, 0, a.stream>>>(
        static_cast<const uint16_t *>(a.x), static_cast<const uint16_t *>(a.Wg),
        static_cast<const uint16_t *>(a.Wu), static_cast<uint16_t *>(a.H), a.T, a.d_model, a.ldh, tiles_m,
        (int)tiles_n, wide_per_xcd, bt);
    return launch_status("gate_up_mfma_mixed launch");
}

// bt: the K ranges (kEdges without routing: the inner runs, with their edges).  kSpans: `span` splits in one workgroup.
template <typename S, bool kRouted = false, bool kEdges = false, bool kSpans = false, typename E = uint16_t>
static hipError_t launch_down(const FwdArgs &a, const BranchTable &bt, int splits,
                              const std::conditional_t<kEdges && !kRouted, EdgeList, NoEdges> &edges, int span = 1, int group = 1)
{
    constexpr int BMT = S::BMT, WM = S::WM, NB = S::NB;
    const int tiles_m = ceil_div(a.T, BMT);
    const int tiles_n = ceil_div(a.d_model, 64 * NB);
    const int kt_total = k_tiles(bt, Elem<E>::BK);
    const int sums = kSpans ? ceil_div(splits, span) : splits;      // partial results
    const long long grid = (long long)XCDS * ids_per_xcd((long long)tiles_m * tiles_n * sums);
    if (grid > 0x7fffffffLL) return note_hip_error("down_mfma grid", hipErrorInvalidValue);
    ProfileScope ps(MLPMOE_KERNEL_DOWN_MFMA, a.stream);
    down_mfma<BMT, WM, NB, S::D, S::kStaged, kRouted, kEdges, kSpans><<<(unsigned)grid, WM * 128, 0, a.stream>>>(
        static_cast<const E *>(a.H), static_cast<const E *>(a.Wd),
        sums > 1 ? a.partial : a.out, a.T, a.d_model, a.d_inter, a.ldh, tiles_m, tiles_n, splits, kt_total,
        (a.out_bf16 && sums == 1) ? DST_BF16
                                  : (sums > 1 && (size_t)sums * a.T * a.d_model * sizeof(float) <= THROUGH_BYTES &&
                                             (size_t)a.d_model * a.d_inter * sizeof(E) <= THROUGH_WEIGHTS
                                         ? DST_THROUGH
                                         : DST_F32),
        span, group, a.route_scratch, bt, edges);
    return launch_status("down_mfma launch");
}

// Adds up the partial results of a K split, kGroups: `group` by `group`.
template <bool kGroups = false>
static hipError_t reduce_splits(const FwdArgs &a, int splits, int group = 0)
{
    if (splits < 2) return hipSuccess;
    ProfileScope ps(MLPMOE_KERNEL_SPLITK_REDUCE, a.stream);
    const size_t n4 = (size_t)a.T * a.d_model / 4;
    if (n4 < REDUCE_SMALL_N4) {
        reduce_partials<128, 1, 8, kGroups>
            <<<(unsigned)((n4 + 127) / 128), 128, 0, a.stream>>>(a.partial, a.out, n4, splits, group, a.out_bf16 ? 1 : 0);
    } else {
        const size_t blocks = std::min<size_t>((n4 + 511) / 512, 4096);
        reduce_partials<256, 2, 1, kGroups><<<(unsigned)blocks, 256, 0, a.stream>>>(a.partial, a.out, n4, splits, group, a.out_bf16 ? 1 : 0);
    }
    return launch_status("reduce_partials launch");
}

// The down projection as planned, then the sum of the partial results if K was split through the workspace.
template <bool kRouted, bool kEdges, typename Ed>
static hipError_t down_and_reduce(const FwdArgs &a, const BranchTable &bt, const DownPlan &pl, const Ed &edges)
{
    hipError_t e = hipErrorInvalidValue;
    if (pl.shape == TILE_WIDE) e = launch_down<ShapeWide, kRouted, kEdges>(a, bt, pl.splits, edges);
    else if (pl.shape == TILE_NARROW) e = launch_down<ShapeNarrow, kRouted, kEdges>(a, bt, pl.splits, edges);
    if constexpr (!kRouted) {
        if (pl.shape == TILE_SMALL) e = launch_down<ShapeSmall, false, kEdges>(a, bt, pl.splits, edges);
        else if (pl.shape == TILE_DEEP) e = launch_down<ShapeDeep, false, kEdges>(a, bt, pl.splits, edges);
        else if (pl.shape == TILE_SLIM) e = launch_down<ShapeSlim, false, kEdges>(a, bt, pl.splits, edges);
    }
    if (e != hipSuccess) return hipErrorLaunchFailure;
    return reduce_splits(a, pl.splits);
}

// Per-token routing on the MFMA kernels (wide tiles: how many tiles are live is known only on the
// device).  a.route_scratch is route_scratch_bytes(T, d_inter) bytes, 256-byte aligned.
// uneven: a branch boundary is not a multiple of 8; d_model and d_inter are.
hipError_t launch_mfma_routed_bf16(const FwdArgs &a, const BranchTable &bt, bool uneven)
{
    hipError_t e;
    if (uneven) {
        UnevenRuns u;
        uneven_runs<Elem<uint16_t>::CHUNK>(bt, u);
        e = launch_gate_up_routed<true>(a, u.outer);
    } else {
        e = launch_gate_up_routed<false>(a, bt);
    }
    if (e != hipSuccess) return hipErrorLaunchFailure;
    // 256-token tiles (the routing tables are per 256 tokens); narrow when K is split: half the partial sums
    int splits = down_splits(a.T, a.d_model, bt.d_eff, TILE_WIDE);
    const TileShape sh = splits > 1 ? TILE_NARROW : TILE_WIDE;
    splits = std::min(down_splits(a.T, a.d_model, bt.d_eff, sh), std::max(1, k_tiles(bt)));
    if (splits > 1 && (size_t)splits * a.T * a.d_model * sizeof(float) > a.partial_bytes) splits = 1;
    return uneven ? down_and_reduce<true, true>(a, bt, DownPlan{sh, splits}, NoEdges{})
                  : down_and_reduce<true, false>(a, bt, DownPlan{sh, splits}, NoEdges{});
}

// Float storage.  K split of the down projection in two steps: as many groups as are best where every workgroup has its CU to
// itself, a K tile of 32 floats taking it 0.43 us of matrix pipe and the first loads and the stores about 2 us; then as many splits
// per group as are best where the waits of one workgroup are hidden by others on its CU, a K tile taking 0.6 us alone and 0.42 us each
// of several, and 3 us.  The separate sum takes about 4 us plus its traffic.  A block without room for the partial sums of all splits is
// enough for those of the groups; a workgroup then goes through the splits of its group, or of all groups, without draining its
// ring in between.  us a call with room for all, for the groups, for none: 896 x 4864, T = 256, 8 splits in 4 groups 80.3 / 81.5 / 159.5,
// T = 500 135 / 140 / 190, T = 100 49.7 / 49.5 / 141; 4096 x 14336, T = 256, 2 in 1 784 / - / 889; splitting no further than the groups: 83.8 / - /
// 161, 144 / - / 192, 53.6 / - / 152 and 885 / - / 885.  Depends on T through whole token tiles only.
struct F32Split {
    int groups, per_group;
    int splits() const { return groups * per_group; }
};
static F32Split f32_split(int T, int d_model, int kt)
{
    const long long tiles_m = ceil_div(T, ShapeF32::BMT), tiles = tiles_m * ceil_div(d_model, 64 * ShapeF32::NB);
    const int most = std::max(1, kt / 4) < 16 ? std::max(1, kt / 4) : 16;
    const auto sum_us = [&](int s) { return s > 1 ? 4.0 + (s + 1.0) * (double)(tiles_m * ShapeF32::BMT) * d_model * 4.0 / 5e6 : 0.0; };
    F32Split best{1, 1};
    double best_us = 1e30;
    for (int s = 1; s <= most; ++s) {
        const double us = (double)((tiles * s + kCUs - 1) / kCUs) * (ceil_div(kt, s) * 0.43 + 2.0) + sum_us(s);
        if (us < best_us) {
            best.groups = s;
            best_us = us;
        }
    }
    best_us = 1e30;
    for (int g = 1; g * best.groups <= most; ++g) {
        const int s = g * best.groups;
        const double per_cu = (double)((tiles * s + kCUs - 1) / kCUs), us = ceil_div(kt, s) * std::max(0.6, 0.42 * per_cu) + 3.0 + sum_us(s);
        if (us < best_us) {
            best.per_group = g;
            best_us = us;
        }
    }
    return best;
}

// Token rows per gate+up tile.  Rounds of 64-token tiles against half rounds of 32-token ones, of which a CU holds four at a
// time (the deep form two): a fifth runs alone and hides nothing.  Where both are one round of the chip, the deep form has two
// workgroups per CU with four K tiles asked for each, which pays from about 24 K tiles on.  us of gate+up, 64 / 32 / 32 deep:
//   one round either way: 896 x 4864, T = 64 30.6 / 28.4 / 25.6, 1024 x 4096, T = 100 33.9 / 31.9 / 29.2, 1280 x 3328, T = 100 40.8 / 38.2 / 34.6, 2048 x
//   5504, T = 64 62.7 / 57.5 / 50.3;  512 x 2560, T = 100 16.4 / 16.9 / 17.0, 640 x 1600, T = 200 19.4 / 19.8 / 20.0;
//   more: 896 x 4864, T = 128 39.4 / 34.7 / 38.6, T = 256 53.6 / 58.7 / 57.9, T = 400 84.2 / 76.9 / 85.9; 1280 x 3328, T = 200 52.5 / 46.0 / 51.2;
//   512 x 2560, T = 330 25.6 / 27.3 / 30.4.
constexpr int F32_DEEP_MIN_D = 768;
static int pick_f32_tokens(long long tiles_n, int T, int d_model)
{
    const long long whole = tiles_n * ceil_div(T, ShapeF32::BMT), half = tiles_n * ceil_div(T, ShapeF32Half::BMT);
    const long long cost64 = 2 * ((whole + kCUs - 1) / kCUs), cost32 = (half + kCUs - 1) / kCUs + (half > 4 * kCUs ? 1 : 0);
    return cost32 < cost64 || (cost32 == cost64 && half <= 2 * kCUs && d_model >= F32_DEEP_MIN_D) ? 32 : 64;
}

size_t mfma_partial_bytes_f32(int T, int d_model, int d_inter)
{
    const int s = f32_split(T, d_model, ceil_div(d_inter, Elem<float>::BK)).splits();
    return s > 1 ? align_up((size_t)s * T * d_model * sizeof(float), 256) : 0;
}

template <bool kEdges, typename Ed>
static hipError_t launch_mfma_f32_runs(const FwdArgs &a, const BranchTable &outer, const BranchTable &inner, const Ed &edges)
{
    long long tiles_n = 0;
    for (int r = 0; r < outer.n_runs; ++r) tiles_n += ceil_div(outer.run_end[r] - outer.run_start[r], 32 * ShapeF32::NB);
    const bool half = pick_f32_tokens(tiles_n, a.T, a.d_model) == 32;
    // us of gate+up with two and with four K tiles ahead, 896 x 4864: T = 20 (152 tiles) 27.2 / 18.0, T = 96 (456) 29.6 / 26.2, T = 128 (608) 34.7 / 38.6
    const bool deep = tiles_n * ceil_div(a.T, ShapeF32Half::BMT) <= 2 * kCUs;
    const hipError_t e = !half ? launch_gate_up<ShapeF32, kEdges, float>(a, outer)
                               : (deep ? launch_gate_up<ShapeF32HalfDeep, kEdges, float>(a, outer)
                                       : launch_gate_up<ShapeF32Half, kEdges, float>(a, outer));
    if (e != hipSuccess) return hipErrorLaunchFailure;
    // The order of the sums depends on the sizes and the table alone: at most the splits that the workspace is sized for
    // (short runs have more K tiles than the width they add up to), and a workspace without room for all partial sums
    // changes who adds them up, not the result.
    F32Split sp = f32_split(a.T, a.d_model, k_tiles(inner, Elem<float>::BK));
    const F32Split layer = f32_split(a.T, a.d_model, ceil_div(a.d_inter, Elem<float>::BK));
    sp.groups = std::min(sp.groups, layer.groups);
    sp.per_group = std::min(sp.per_group, layer.splits() / sp.groups);
    const int splits = sp.splits(), group = sp.per_group, groups = sp.groups;
    const size_t room = a.partial_bytes / ((size_t)a.T * a.d_model * sizeof(float));
    if (splits == 1 || (size_t)splits <= room) {
        if (launch_down<ShapeF32, false, kEdges, false, float>(a, inner, splits, edges) != hipSuccess) return hipErrorLaunchFailure;
        return groups > 1 && group > 1 ? reduce_splits<true>(a, splits, group) : reduce_splits(a, splits);
    }
    const int span = (size_t)groups <= room ? group : splits;
    if (launch_down<ShapeF32, false, kEdges, true, float>(a, inner, splits, edges, span, group) != hipSuccess) return hipErrorLaunchFailure;
    return reduce_splits(a, ceil_div(splits, span));
}

// d_model and d_inter are multiples of 4.
hipError_t launch_mfma_f32(const FwdArgs &a, const BranchTable &bt)
{
    UnevenRuns u;
    uneven_runs<Elem<float>::CHUNK>(bt, u);
    bool even = true;
    for (int r = 0; r < bt.n_runs; ++r)
        even = even && bt.run_start[r] % Elem<float>::CHUNK == 0 && bt.run_end[r] % Elem<float>::CHUNK == 0;
    return even ? launch_mfma_f32_runs<false>(a, bt, bt, NoEdges{}) : launch_mfma_f32_runs<true>(a, u.outer, u.inner, u.edges);
}

template <bool kEdges>
static hipError_t launch_gate_up_shape(const FwdArgs &a, const BranchTable &bt, TileShape sh)
{
    switch (sh) {
    case TILE_WIDE: return launch_gate_up<ShapeWide, kEdges>(a, bt);
    case TILE_NARROW: return launch_gate_up<ShapeNarrow, kEdges>(a, bt);
    case TILE_SMALL: return launch_gate_up<ShapeSmall, kEdges>(a, bt);
    case TILE_DEEP: return launch_gate_up<ShapeDeep, kEdges>(a, bt);
    case TILE_SLIM: return launch_gate_up<ShapeSlim, kEdges>(a, bt);
    default: return hipErrorInvalidValue;
    }
}

// uneven: a run boundary is not a multiple of 8 (first-K pruning or branches switched off where B does not divide
// the width); d_model and d_inter are.
hipError_t launch_mfma_bf16(const FwdArgs &a, const BranchTable &bt, bool uneven)
{
    if (uneven) {
        UnevenRuns u;
        uneven_runs<Elem<uint16_t>::CHUNK>(bt, u);
        TileShape gu = pick_gate_up_tile(u.outer, a.T, a.d_model);
        if (gu == TILE_MIXED) gu = TILE_WIDE;
        if (launch_gate_up_shape<true>(a, u.outer, gu) != hipSuccess) return hipErrorLaunchFailure;
        return down_and_reduce<false, true>(a, u.inner, plan_down(a, u.inner, false), u.edges);
    }
    TileShape gu = a.tile_shape >= 0 ? (TileShape)a.tile_shape : pick_gate_up_tile(bt, a.T, a.d_model);
    if (gu == TILE_MIXED && mixed_wide_per_xcd(gate_up_tiles(bt, a.T, TILE_WIDE)) < 0) gu = TILE_WIDE;   // forced where it does not apply
    const hipError_t e = gu == TILE_MIXED ? launch_gate_up_mixed(a, bt) : launch_gate_up_shape<false>(a, bt, gu);
    if (e != hipSuccess) return hipErrorLaunchFailure;
    return down_and_reduce<false, false>(a, bt, plan_down(a, bt, false), NoEdges{});
}

}  // namespace mlpmoe
