// Decode path (T <= 16): bandwidth-bound weight streaming for gfx950.
//
// Every weight element is read exactly once, straight from HBM into MFMA operand registers
// (no LDS staging: there is no reuse to exploit), with the <=16 tokens riding on the N side of
// v_mfma_f32_16x16x32_bf16.  A workgroup owns one tile of 16 weight rows; its waves take
// interleaved 64-element blocks of K, so the workgroup as a whole reads long contiguous
// pieces of every row, and the waves' partial 16x16 results are summed through LDS in a
// fixed order (deterministic).
//
//   decode_gate_up:  a tile is 8 neurons: MFMA rows 0-7 are their W_gate rows, rows 8-15 their
//                    W_up rows, K = d_model; epilogue h = bf16(alpha_b * SiLU(g) * u)
//                                                                        (Sec. 3.1 inner bracket)
//   decode_down:     a tile is 16 output features of W_down, K = active runs of neurons,
//                    epilogue out[t,m] = sum                            (Sec. 3.1 outer sum)
//
// Eight-neuron tiles keep the tile count a multiple of the CU count for the usual widths
// (14336 / 8 = 7 * 256) and never straddle a run boundary (boundaries are multiples of 8).
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace mlpmoe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int KB = 64;   // K elements per wave step: two MFMA steps of 32
// Which 8 of a block's 64 K elements a lane feeds to the two MFMA steps: group q = lane >> 4 takes elements
// q * KQ .. + 7 for the first step and q * KQ + KH .. + 7 for the second.  Any assignment works as long as x
// is loaded the same way (the dot product does not care about the order of K).
constexpr int KQ = 16, KH = 8;

// 16 zero bytes: lanes with nothing to load (token >= T, K chunk past the end of a range) read here.
__device__ const uint32_t g_zero16[4] = {0, 0, 0, 0};

// 16-byte load through the global (not flat) path: every pointer handed in is device memory.
__device__ __forceinline__ u32x4 ld16(const void *p)
{
    typedef const __attribute__((address_space(1))) u32x4 *gptr;
    return *(gptr)p;
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float silu_mul(float g, float u)
{
    const float e = __builtin_amdgcn_exp2f(g * -1.4426950408889634f);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

__device__ __forceinline__ uint16_t to_bf16(float v)
{
    const __bf16 b = (__bf16)v;
    return __builtin_bit_cast(uint16_t, b);
}

// 16-byte loads of at most 2^31 bytes from `base`: lanes without anything to load (!ok) read zeros from past the end.
struct Window {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ Window(const void *base, unsigned bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000)) {}
    __device__ __forceinline__ u32x4 ld16(bool ok, unsigned offset) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? offset : 0xffffffffu, 0, 0);
    }
};

// Uses two registers that were just loaded, so that their loads are waited for here, once, and not at every lane read
// in a loop that has weights in flight.
template <typename A, typename B>
__device__ __forceinline__ void arrived(A &a, B &b)
{
    asm volatile("" : "+v"(a), "+v"(b));
}

// Lane layout of v_mfma_f32_16x16x32_bf16: operand lane l holds row/col (l & 15) and the 8
// K values of group q = l >> 4.  A lane here loads 16 contiguous K values k0+16q .. k0+16q+15
// and feeds the low 8 to one MFMA and the high 8 to the next (KQ, KH); x is loaded with the same
// mapping, so the permutation of K inside a block cancels out.  (Giving each MFMA step 64
// contiguous bytes of a row instead was measured and makes no difference.)
//
// Memory-level parallelism: every wave keeps the loads of U of its K blocks in flight (a ring of
// U register sets: block i is consumed, then the load of block i+U is issued into its place).
// All loads are branch free: a lane with nothing to load points at a zero chunk instead.
// Per-token routing (T <= 16): the set of branches some token of the batch takes, as a 64-bit
// word, folded with the active mask.  Every wave works it out for itself from route[T, B]: lane b
// looks down column b.
__device__ __forceinline__ unsigned long long live_branches(const BranchTable &bt, const uint8_t *route, int T)
{
    const int b = threadIdx.x & 63;
    bool any = false;
    if (b < bt.B)
        for (int t = 0; t < T; ++t) any = any || route[(size_t)t * bt.B + b] != 0;
    return __ballot(any) & bt.active;
}

// The stretches of the intermediate dimension a launch works on.  Without routing they are the
// table's runs of active branches; with routing, one stretch per branch, empty unless the branch is
// live (all branch offsets are then multiples of 8).
// Lane r of every wave holds the bounds of stretch r, so that the cursors read lanes and not memory: one round of
// loads as the kernel starts, in place of a chain of dependent ones before the first weights are asked for.
template <bool kRouted>
struct Stretches {
    int n, v_beg, v_end;
    __device__ __forceinline__ Stretches(const BranchTable &bt, const uint8_t *route, int T)
    {
        const int lane = threadIdx.x & 63;
        if (kRouted) {
            n = bt.B;
            v_beg = bt.off[lane];
            const int next = bt.off[lane + 1];
            v_end = ((live_branches(bt, route, T) >> lane) & 1ULL) ? next : v_beg;
        } else {
            n = bt.n_runs;
            const int r = lane < kMaxRuns ? lane : kMaxRuns - 1;
            v_beg = bt.run_start[r];
            v_end = bt.run_end[r];
        }
    }
    __device__ __forceinline__ int count() const { return n; }
    __device__ __forceinline__ int beg(int r) const { return __builtin_amdgcn_readlane(v_beg, r); }
    __device__ __forceinline__ int end(int r) const { return __builtin_amdgcn_readlane(v_end, r); }
};

// Walks the groups of 8 rows ("tiles") of the stretches in steps: (stretch, tile inside it).
template <bool kRouted>
struct TileCursor {
    int r, t;
    __device__ __forceinline__ TileCursor(const Stretches<kRouted> &st, int tile) : r(0), t(tile) { settle(st); }
    __device__ __forceinline__ void settle(const Stretches<kRouted> &st)
    {
        while (r < st.count()) {
            const int n = (st.end(r) - st.beg(r) + 7) / 8;   // whole tiles but for tables with odd boundaries
            if (t < n) break;
            t -= n;
            ++r;
        }
    }
    __device__ __forceinline__ void advance(const Stretches<kRouted> &st, int step)
    {
        t += step;
        settle(st);
    }
    __device__ __forceinline__ int end(const Stretches<kRouted> &st) const { return st.end(r); }
    // first row of the tile under the cursor, -1 past the last tile
    __device__ __forceinline__ int row0(const Stretches<kRouted> &st) const { return r < st.count() ? st.beg(r) + t * 8 : -1; }
};

template <int NW, int U, bool kGateUp, bool kRouted = false>
__global__ void __launch_bounds__(NW * 64)
decode_kernel(const uint16_t *__restrict__ Xin, int ldx, int T,
              const uint16_t *__restrict__ W0, const uint16_t *__restrict__ W1, int ldw,
              int d_model, uint16_t *__restrict__ Hout, int ldh, float *__restrict__ out, int out_bf16,
              const uint8_t *__restrict__ route, BranchTable bt)
{
    static_assert(NW >= 4, "the final reduction uses 256 threads");
    __shared__ float red[NW][256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    BranchLanes br(bt);
    Stretches<kRouted> st(bt, route, T);
    arrived(br.v_next, br.v_alpha);
    arrived(st.v_beg, st.v_end);

    // tile -> this lane's weight row
    int row0 = 0;
    const uint16_t *wrow;
    if (kGateUp) {
        row0 = TileCursor<kRouted>(st, blockIdx.x).row0(st);
        if (row0 < 0) return;                            // with routing the grid covers all active rows
        wrow = (r16 < 8 ? W0 : W1) + (size_t)(row0 + (r16 & 7)) * ldw;
    } else {
        row0 = blockIdx.x * 16;
        int m = row0 + r16;
        m = m < d_model ? m : d_model - 1;               // clamped rows are computed but never stored
        wrow = W0 + (size_t)m * ldw;
    }
    wrow += q * KQ;
    const bool tok = r16 < T;
    const uint16_t *xp = Xin + (size_t)(tok ? r16 : 0) * ldx + q * KQ;
    const uint16_t *zero = reinterpret_cast<const uint16_t *>(g_zero16);

    // cursor over this wave's blocks: (range, block inside the range); ranges laid end to end
    const int n_ranges = kGateUp ? 1 : st.count();
    auto rbeg = [&](int r) { return kGateUp ? 0 : st.beg(r); };
    auto rend = [&](int r) { return kGateUp ? d_model : st.end(r); };
    int cr = 0, cb = wave;                               // load cursor
    auto settle = [&]() {                                // move past ranges the block index overshoots
        while (cr < n_ranges) {
            const int nb = (rend(cr) - rbeg(cr) + KB - 1) / KB;
            if (cb < nb) break;
            cb -= nb;
            ++cr;
        }
    };
    settle();
    int total = 0;                                       // blocks of this wave in all ranges
    {
        int sk = wave;
        for (int r = 0; r < n_ranges; ++r) {
            const int nb = (rend(r) - rbeg(r) + KB - 1) / KB;
            const int mine = nb > sk ? (nb - sk + NW - 1) / NW : 0;
            total += mine;
            sk = sk + mine * NW - nb;
        }
    }

    u32x4 wa[U][2], xa[U][2];
    auto load_block = [&](int u) {                       // loads the block under the cursor, then advances
        const bool live = cr < n_ranges;
        const int k = live ? rbeg(cr) + cb * KB : 0;
        const int kend = live ? rend(cr) : -1;
        const int kl = k + q * KQ;
        const bool ok0 = kl < kend, ok1 = kl + KH < kend;
        wa[u][0] = ld16(ok0 ? wrow + k : zero);
        wa[u][1] = ld16(ok1 ? wrow + k + KH : zero);
        xa[u][0] = ld16((ok0 && tok) ? xp + k : zero);
        xa[u][1] = ld16((ok1 && tok) ? xp + k + KH : zero);
        cb += NW;
        settle();
    };

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) load_block(u);
    for (int j = 0; j < total; j += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][0]), as_bf16x8(xa[u][0]), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][1]), as_bf16x8(xa[u][1]), acc, 0, 0, 0);
            load_block(u);                               // past the last block this loads zeros
        }
    }

    // cross-wave sum in wave order
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][v * 64 + lane] = acc[v];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    // accumulator layout: register v of lane l is D[row 4*(l>>4)+v][col l&15]
    const int v = wave;
    const int row = 4 * q + v;
    const int t = r16;
    int b = 0;
    float alpha = 0.f;
    if (kGateUp) {
        const int b0 = br.branch(row0 + v), b1 = br.branch(row0 + 4 + v);
        const float alpha0 = br.alpha(b0), alpha1 = br.alpha(b1);
        b = q ? b1 : b0;                                 // rows 0-7: q is 0 or 1
        alpha = q ? alpha1 : alpha0;
    }
    if (t >= T) return;
    if (kGateUp) {
        if (row >= 8) return;                            // rows 8-15 hold the up projection of rows 0-7
        float g = 0.f, up = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            g += red[w][threadIdx.x];
            up += red[w][threadIdx.x + 32];              // row + 8: two lane groups further
        }
        const int n = row0 + row;
        float v = alpha * silu_mul(g, up);
        if (kRouted) v = route[(size_t)t * bt.B + b] ? v : 0.f;
        Hout[(size_t)t * ldh + n] = to_bf16(v);
    } else {
        float s0 = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s0 += red[w][threadIdx.x];
        const int m = row0 + row;
        if (m < d_model) {
            if (out_bf16)
                reinterpret_cast<uint16_t *>(out)[(size_t)t * d_model + m] = to_bf16(s0);
            else
                out[(size_t)t * d_model + m] = s0;
        }
    }
}

// Down projection of wide layers and of a long K, with RT row tiles (16 RT output features) per workgroup and the K blocks dealt to TWO
// workgroups (blockIdx.y).  Every workgroup of the one-tile
// kernel reads all of H, which at 16 tokens is as many bytes as its weight rows, all from the same
// L2; here a block of H is used for two weight fragments and each workgroup reads half of H, a quarter
// of that traffic per weight byte, with all CUs still busy.  The two partial sums of an output are
// added into `out` with float atomics: out must hold zeros when the kernel starts (the gate+up
// kernel that runs before it clears it), and 0 + a + b is the same number in either order, so the
// result does not depend on which workgroup comes first.  RT = 1 with 16 waves: fewer output features and a
// long K (down_long_k).  Few output features or few tokens otherwise: decode_down_rows.
// Slots of the ring past a wave's last block, and absent tokens, read past the end of a buffer: zeros that nobody fetches
// (with the gate+up kernel's last tile likewise: 4096 x 14336, T = 16 70.2 -> 68.8 us a step, T = 4 65.0 -> 64.4).
template <int NW, int U, int RT, bool kRouted = false>
__global__ void __launch_bounds__(NW * 64)
decode_down_split(const uint16_t *__restrict__ Hin, int ldx, int T, const uint16_t *__restrict__ Wd, int ldw,
                  int d_model, float *__restrict__ out, const uint8_t *__restrict__ route, BranchTable bt)
{
    static_assert(NW >= 4, "the final reduction uses 256 threads");
    constexpr int KS = 2;
    __shared__ float red[NW][RT][256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    Stretches<kRouted> st(bt, route, T);
    arrived(st.v_beg, st.v_end);
    const int row0 = blockIdx.x * (16 * RT);
    const Window w(Wd + (size_t)row0 * ldw, 16u * RT * (unsigned)ldw * 2u), h(Hin, (unsigned)T * (unsigned)ldx * 2u);
    unsigned w_lane[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        int m = rt * 16 + r16;
        m = row0 + m < d_model ? m : d_model - 1 - row0; // clamped rows are computed but never stored
        w_lane[rt] = ((unsigned)m * (unsigned)ldw + q * KQ) * 2u;
    }
    const bool tok = r16 < T;
    const unsigned h_lane = ((unsigned)r16 * (unsigned)ldx + q * KQ) * 2u;

    // cursor over this wave's blocks.  The K blocks of all ranges, laid end to end, are cut into KS
    // contiguous parts, one per workgroup (a workgroup then reads long contiguous pieces of its rows);
    // inside its part the waves take the blocks in turn.
    const int n_ranges = st.count();
    int nb_all = 0;
    for (int r = 0; r < n_ranges; ++r) nb_all += (st.end(r) - st.beg(r) + KB - 1) / KB;
    const int part = (nb_all + KS - 1) / KS;
    const int first = wave + (int)blockIdx.y * part, stride = NW;
    const int my_end = (int)(blockIdx.y + 1) * part < nb_all ? (int)(blockIdx.y + 1) * part : nb_all;
    int cr = 0, cb = first;
    auto settle = [&]() {                                // move past ranges the block index overshoots
        while (cr < n_ranges) {
            const int nb = (st.end(cr) - st.beg(cr) + KB - 1) / KB;
            if (cb < nb) break;
            cb -= nb;
            ++cr;
        }
    };
    settle();
    const int total = my_end > first ? (my_end - first + stride - 1) / stride : 0;   // blocks of this wave
    int issued = 0;

    u32x4 wa[U][RT][2], xa[U][2];
    auto load_block = [&](int u) {                       // loads the block under the cursor, then advances
        const bool live = cr < n_ranges && issued < total;     // past its part a wave asks for nothing
        ++issued;
        const int k = live ? st.beg(cr) + cb * KB : 0;
        const int kend = live ? st.end(cr) : -1;
        const int kl = k + q * KQ;
        const bool ok0 = kl < kend, ok1 = kl + KH < kend;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            wa[u][rt][0] = w.ld16(ok0, w_lane[rt] + k * 2);
            wa[u][rt][1] = w.ld16(ok1, w_lane[rt] + (k + KH) * 2);
        }
        xa[u][0] = h.ld16(ok0 && tok, h_lane + k * 2);
        xa[u][1] = h.ld16(ok1 && tok, h_lane + (k + KH) * 2);
        cb += stride;
        settle();
    };

    f32x4 acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) load_block(u);
    for (int j = 0; j < total; j += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][rt][0]), as_bf16x8(xa[u][0]), acc[rt], 0, 0, 0);
                acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][rt][1]), as_bf16x8(xa[u][1]), acc[rt], 0, 0, 0);
            }
            load_block(u);                               // past the last block this loads zeros
        }
    }

    // cross-wave sum in wave order, then this workgroup's half of K goes into out
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][rt][v * 64 + lane] = acc[rt][v];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const int v = threadIdx.x >> 6;
    const int row = 4 * q + v;                           // register v of lane l is D[row 4*(l>>4)+v][col l&15]
    const int t = r16;
    if (t >= T) return;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        float s0 = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s0 += red[w][rt][threadIdx.x];
        const int m = row0 + rt * 16 + row;
        if (m < d_model) atomicAdd(&out[(size_t)t * d_model + m], s0);
    }
}

// Sets n floats to 0 for the down kernel that follows, which adds into them; p may be null.  Called once the first weights are
// requested: loads wait for the stores before them.
__device__ __forceinline__ void clear_floats(float *__restrict__ p, int n, int threads, int grid)
{
    if (p)
        for (int i = blockIdx.x * threads + threadIdx.x; i < n; i += grid * threads) p[i] = 0.f;
}

// Persistent gate+up kernel for layers whose x fits in LDS (T * (d_model*2 + 16) bytes).
// grid is gridDim.x, handed over beside the other arguments: the hidden argument is a cold line of its own that the
// first weight request would wait for.
// One workgroup per CU copies x into LDS once and then walks its tiles (tile t belongs to
// workgroup t % grid, so every CU gets the same number).  The NW waves of the workgroup share each
// tile with interleaved 64-element K blocks, which makes the workgroup read NW*128 contiguous
// bytes of every weight row per step; every wave keeps a ring of U blocks in flight, and the ring
// keeps rolling across tile boundaries, so the loads of the next tile are already under way
// while the partial sums of the current one are reduced through LDS (one barrier per tile, the
// reduction buffer is double buffered).  Each wave's block count per tile is padded to a
// multiple of U with blocks that read a zero chunk, which keeps ring slots compile-time constants.
// x rows are padded by 16 bytes so that the 16 token rows of a fragment fall on distinct banks.
template <int NW, int U, bool kRouted = false>
__global__ void __launch_bounds__(NW * 64)
decode_gate_up_persist(const uint16_t *__restrict__ X, int T, const uint16_t *__restrict__ Wg,
                       const uint16_t *__restrict__ Wu, int d_model, uint16_t *__restrict__ Hout, int ldh,
                       const uint8_t *__restrict__ route, float *__restrict__ clear, int clear_n, int grid, BranchTable bt)
{
    static_assert(NW >= 4, "the reduction uses 256 threads");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *red = reinterpret_cast<float *>(smem);                 // [2][NW][256]
    char *xs = smem + 2 * NW * 256 * sizeof(float);
    const int row_bytes = d_model * 2 + 16;
    const int zero_off = T * row_bytes;                  // 16 zero bytes after the last row
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const bool tok = r16 < T;
    const int x_lane = (tok ? r16 : 0) * row_bytes + q * (KQ * 2);
    const uint16_t *zero = reinterpret_cast<const uint16_t *>(g_zero16);
    const int nblk = (d_model + KB - 1) / KB;
    const int nb_pad = ((nblk + NW - 1) / NW + U - 1) / U * U;    // blocks per wave per tile, padded
    const size_t lane_row_off = (size_t)(r16 & 7) * d_model + q * KQ;
    const uint16_t *wsel = r16 < 8 ? Wg : Wu;

    // with routing the workgroups share out the tiles of the live branches only
    BranchLanes br(bt);
    Stretches<kRouted> st(bt, route, T);
    arrived(br.v_next, br.v_alpha);
    arrived(st.v_beg, st.v_end);

    // load cursor: U blocks ahead of the block being consumed
    TileCursor<kRouted> l_cur(st, blockIdx.x);
    int l_j = 0;
    int l_row0 = l_cur.row0(st);
    const uint16_t *l_wrow = wsel + (size_t)(l_row0 < 0 ? 0 : l_row0) * d_model + lane_row_off;
    u32x4 wa[U][2];
    auto load_next = [&](int u) {
        const int b = wave + NW * l_j;                   // K block inside the tile
        const int kl = b * KB + q * KQ;
        const bool more = l_row0 >= 0;
        wa[u][0] = ld16((more && kl < d_model) ? l_wrow + b * KB : zero);
        wa[u][1] = ld16((more && kl + KH < d_model) ? l_wrow + b * KB + KH : zero);
        if (++l_j == nb_pad) {
            l_j = 0;
            l_cur.advance(st, grid);
            l_row0 = l_cur.row0(st);
            if (l_row0 >= 0) l_wrow = wsel + (size_t)l_row0 * d_model + lane_row_off;
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_next(u);            // the weight stream starts before x is staged

    // x -> LDS, while the first weight blocks are on their way
    {
        const int chunks = T * (d_model / 8);            // 16-byte chunks of x
        for (int i0 = 0; i0 < chunks; i0 += NW * 64 * 8) {
            u32x4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {                // 8 loads in flight per thread
                const int i = i0 + j * (NW * 64) + threadIdx.x;
                v[j] = ld16(i < chunks ? X + (size_t)i * 8 : reinterpret_cast<const uint16_t *>(g_zero16));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = i0 + j * (NW * 64) + threadIdx.x;
                if (i < chunks) {
                    const int t = i / (d_model / 8), c = i % (d_model / 8);
                    *reinterpret_cast<u32x4 *>(xs + t * row_bytes + c * 16) = v[j];
                }
            }
        }
    }
    if (threadIdx.x == 0) *reinterpret_cast<u32x4 *>(xs + zero_off) = u32x4{0, 0, 0, 0};
    __syncthreads();

    clear_floats(clear, clear_n, NW * 64, grid);

    int it = 0;
    TileCursor<kRouted> cur(st, blockIdx.x);
    for (int row0 = cur.row0(st); row0 >= 0; cur.advance(st, grid), row0 = cur.row0(st), ++it) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int j0 = 0; j0 < nb_pad; j0 += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = wave + NW * (j0 + u);
                const int kl = b * KB + q * KQ;
                const int xo0 = (tok && kl < d_model) ? x_lane + b * (KB * 2) : zero_off;
                const int xo1 = (tok && kl + KH < d_model) ? x_lane + b * (KB * 2) + KH * 2 : zero_off;
                const bf16x8 x0 = *reinterpret_cast<const bf16x8 *>(xs + xo0);
                const bf16x8 x1 = *reinterpret_cast<const bf16x8 *>(xs + xo1);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][0]), x0, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][1]), x1, acc, 0, 0, 0);
                load_next(u);                            // refill the slot just consumed
                __builtin_amdgcn_sched_barrier(0);       // keep the ring rolling: no batching of loads
            }
        }
        // cross-wave sum in wave order; rows 0-7 hold g, rows 8-15 hold u of the same neurons
        float *rb = red + (it & 1) * (NW * 256);
#pragma unroll
        for (int v = 0; v < 4; ++v) rb[wave * 256 + v * 64 + lane] = acc[v];
        __syncthreads();
        if (threadIdx.x < 256) {
            const int v = wave;
            const int row = 4 * q + v;                   // register v of lane l is D[row 4*(l>>4)+v][col l&15]
            const int b0 = br.branch(row0 + v), b1 = br.branch(row0 + 4 + v);
            const int b = q ? b1 : b0;                   // rows 0-7: q is 0 or 1
            const float alpha0 = br.alpha(b0), alpha1 = br.alpha(b1);
            const float alpha = q ? alpha1 : alpha0;
            if (row < 8 && tok) {
                float g = 0.f, up = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    g += rb[w * 256 + threadIdx.x];
                    up += rb[w * 256 + threadIdx.x + 32];
                }
                const int n = row0 + row;
                float v = alpha * silu_mul(g, up);
                if (kRouted) v = route[(size_t)r16 * bt.B + b] ? v : 0.f;
                Hout[(size_t)r16 * ldh + n] = to_bf16(v);
            }
        }
    }
}

// waves and ring depth of the instantiations in use: gate+up fallback, down, persistent gate+up
constexpr int DEC_NW1 = 4, DEC_U1 = 8, DEC_NW2 = 8, DEC_U2 = 8, DEC_SNW = 8, DEC_SU = 8;
// The persistent gate+up kernel with the x fragments held in registers instead of LDS: wave w works on
// K blocks w, w + NW, ... of EVERY tile, so the x fragments it needs are the same for every tile and
// are loaded once, XB blocks of 2 x 16 bytes per lane (d_model <= 64 * NW * XB).  Everything else
// (tile order, ring of U weight blocks rolling across tiles, reduction, epilogue, clear) is
// decode_gate_up_persist's.  XB < U (narrow layers): a revolution of the ring spans U / XB tiles, so the
// weight blocks of that many tiles are in flight per wave and no slot is spent on blocks past d_model.
template <int NW, int U, int XB, bool kRouted = false>
__global__ void __launch_bounds__(NW * 64)
decode_gate_up_xreg(const uint16_t *__restrict__ X, int T, const uint16_t *__restrict__ Wg,
                    const uint16_t *__restrict__ Wu, int d_model, uint16_t *__restrict__ Hout, int ldh,
                    const uint8_t *__restrict__ route, float *__restrict__ clear, int clear_n, int grid, BranchTable bt)
{
    static_assert(NW >= 4 && (XB % U == 0 || U % XB == 0), "the reduction uses 256 threads; ring slots are compile-time");
    constexpr int TPR = XB >= U ? 1 : U / XB;     // tiles per revolution of the ring
    __shared__ float red[2][NW][256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const bool tok = r16 < T;
    const uint16_t *zero = reinterpret_cast<const uint16_t *>(g_zero16);
    const size_t lane_row_off = (size_t)(r16 & 7) * d_model + q * KQ;
    const uint16_t *wsel = r16 < 8 ? Wg : Wu;
    BranchLanes br(bt);
    Stretches<kRouted> st(bt, route, T);
    arrived(br.v_next, br.v_alpha);
    arrived(st.v_beg, st.v_end);

    TileCursor<kRouted> l_cur(st, blockIdx.x);
    int l_j = 0;
    int l_row0 = l_cur.row0(st);
    const uint16_t *l_wrow = wsel + (size_t)(l_row0 < 0 ? 0 : l_row0) * d_model + lane_row_off;
    u32x4 wa[U][2];
    auto load_next = [&](int u) {
        const int b = wave + NW * l_j;
        const int kl = b * KB + q * KQ;
        const bool more = l_row0 >= 0;
        wa[u][0] = ld16((more && kl < d_model) ? l_wrow + b * KB : zero);
        wa[u][1] = ld16((more && kl + KH < d_model) ? l_wrow + b * KB + KH : zero);
        if (++l_j == XB) {
            l_j = 0;
            l_cur.advance(st, grid);
            l_row0 = l_cur.row0(st);
            if (l_row0 >= 0) l_wrow = wsel + (size_t)l_row0 * d_model + lane_row_off;
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_next(u);

    // this wave's x fragments, once
    u32x4 xr[XB][2];
    {
        const uint16_t *xp = X + (size_t)(tok ? r16 : 0) * d_model + q * KQ;
#pragma unroll
        for (int j = 0; j < XB; ++j) {
            const int b = wave + NW * j;
            const int kl = b * KB + q * KQ;
            xr[j][0] = ld16((tok && kl < d_model) ? xp + b * KB : zero);
            xr[j][1] = ld16((tok && kl + KH < d_model) ? xp + b * KB + KH : zero);
        }
    }

    clear_floats(clear, clear_n, NW * 64, grid);

    int it = 0;
    TileCursor<kRouted> cur(st, blockIdx.x);
    int row0 = cur.row0(st);
    // one revolution of the ring; more: with the loads of the tiles behind it
    const auto revolve = [&](auto more) {
#pragma unroll
        for (int tt = 0; tt < TPR; ++tt) {           // tile tt of this revolution uses ring slots tt * XB ...
            if (row0 < 0) break;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j0 = 0; j0 < XB; j0 += U) {
#pragma unroll
                for (int ju = 0; ju < (XB < U ? XB : U); ++ju) {
                    const int u = XB < U ? tt * XB + ju : ju;
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][0]), as_bf16x8(xr[j0 + ju][0]), acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wa[u][1]), as_bf16x8(xr[j0 + ju][1]), acc, 0, 0, 0);
                    if (decltype(more)::value) load_next(u);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            float *rb = &red[it & 1][0][0];
#pragma unroll
            for (int v = 0; v < 4; ++v) rb[wave * 256 + v * 64 + lane] = acc[v];
            __syncthreads();
            if (threadIdx.x < 256) {
                const int v = wave;
                const int row = 4 * q + v;                   // register v of lane l is D[row 4*(l>>4)+v][col l&15]
                const int b0 = br.branch(row0 + v), b1 = br.branch(row0 + 4 + v);
                const int b = q ? b1 : b0;                   // rows 0-7: q is 0 or 1
                const float alpha0 = br.alpha(b0), alpha1 = br.alpha(b1);
                const float alpha = q ? alpha1 : alpha0;
                if (row < 8 && tok) {
                    float g = 0.f, up = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        g += rb[w * 256 + threadIdx.x];
                        up += rb[w * 256 + threadIdx.x + 32];
                    }
                    const int n = row0 + row;
                    float v = alpha * silu_mul(g, up);
                    if (kRouted) v = route[(size_t)r16 * bt.B + b] ? v : 0.f;
                    Hout[(size_t)r16 * ldh + n] = to_bf16(v);
                }
            }
            ++it;
            cur.advance(st, grid);
            row0 = cur.row0(st);
        }
    };
    if constexpr (XB == U) {
        // a revolution is a tile: the last one asks for nothing (the zeros it asked for otherwise were 128 KB on a CU's memory
        // path, in front of its last stores)
        while (row0 >= 0 && l_row0 >= 0) revolve(std::true_type{});
        if (row0 >= 0) revolve(std::false_type{});
    } else {
        while (row0 >= 0) revolve(std::true_type{});
    }
}

// ---- narrow layers and small batches ---------------------------------------------------------------
// What bounds them is what a CU's memory path carries and how soon it starts, not HBM: about 40 bytes per clock and CU,
// for lines that come from the L2 and for lanes that read the zero chunk alike.  A ring kernel on 896 x 4864 moves
// 288 KB per CU for 68 KB of W_gate and W_up, the rest being slots past the last tile, K blocks past d_model and token
// columns past T; its down kernel has 112 workgroups with as many loads of H as of W_down.  The kernels below ask for
// weights once, all of them as the kernel starts, and for nothing else: lanes without a token read past the end of a
// buffer, which costs no traffic, and there is a workgroup for every small tile, so that all CUs are busy.
//
// A tile has 8 (or 4) rows, not 16.  Operand lane l of v_mfma_f32_16x16x32_bf16 holds row l & 15 and K group l >> 4, and
// here rows 8 .. 15 are rows 0 .. 7 again at the next 32 K elements: one load takes whole 128-byte lines of 8 rows.  With at
// most 8 tokens the columns 8 .. 15 are the tokens again, at those same K elements, so that one MFMA does both halves: the
// two diagonal blocks of the result are the two partial sums, what is off the diagonal is never used.  With more tokens
// each half has an MFMA and an operand of its own (NG = K groups per MFMA, CT = token columns).

// What E, the storage type, and kEdges, a table whose run boundaries are not multiples of a 16-byte chunk, change: a chunk is
// 8 bf16 values, one MFMA, or 4 floats, four v_mfma_f32_16x16x4_f32; SiLU is formed with expf and a division, as by the
// general kernels.  With kEdges the last tile of a run has fewer rows, and the K blocks of the down projection start at the chunk that a run
// starts in: the elements of a chunk that are not the run's are masked in BOTH operands, so that nothing of a pruned branch
// and no value of H that was never written reaches the sum, non-finite ones included.
template <typename E>
struct RowElem {
    static constexpr int CH = 16 / sizeof(E), KBLK = 8 * CH;    // elements of a chunk, of a 128-byte line
};
template <typename E>
__device__ __forceinline__ f32x4 mfma_chunk(u32x4 w, u32x4 x, f32x4 acc)
{
    if constexpr (sizeof(E) == 2) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w), as_bf16x8(x), acc, 0, 0, 0);
    } else {
        const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc, 0, 0, 0);
        return acc;
    }
}
// the elements lo .. hi - 1 of a chunk
template <typename E>
__device__ __forceinline__ u32x4 keep_elements(u32x4 v, int lo, int hi)
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (sizeof(E) == 4) {
            v[w] = w >= lo && w < hi ? v[w] : 0u;
        } else {
            v[w] &= (2 * w >= lo && 2 * w < hi ? 0x0000ffffu : 0u) | (2 * w + 1 >= lo && 2 * w + 1 < hi ? 0xffff0000u : 0u);
        }
    }
    return v;
}
__device__ __forceinline__ void store_h(uint16_t *p, float v) { *p = to_bf16(v); }
__device__ __forceinline__ void store_h(float *p, float v) { *p = v; }

constexpr int RED_V = 64 + 4, RED_W = 4 * RED_V + 8;     // partial sums in LDS: strides of a register and of a wave (floats)

// Gate+up projection, one workgroup per tile of 8 neurons; wave w takes the K blocks w, w + NW, ..., at most XB of them.
// 896 x 4864 with the ring kernel replaced by this one alone: T = 1 15.9 -> 14.6 us a step, T = 8 16.8 -> 15.8 us,
// T = 16 17.9 -> 17.5 us.  Every workgroup loads all of x, which is why wide layers and batches keep the ring kernel (see
// gate_up_once).  Two tiles per workgroup (half of the x loads): 15.6, 16.7 and 18.3 us; one workgroup per CU with x in
// registers and 4-neuron tiles: 0.5 to 1 us slower than this as well.
template <int NW, int XB, int NG, bool kRouted, bool kEdges, typename E>
__global__ void __launch_bounds__(NW * 64)
decode_gate_up_once(const E *__restrict__ X, int T, const E *__restrict__ Wg,
                    const E *__restrict__ Wu, int d_model, E *__restrict__ Hout, int ldh,
                    const uint8_t *__restrict__ route, float *__restrict__ clear, int clear_n, int grid, BranchTable bt)
{
    constexpr int NM = 2 / NG, CT = 16 / NG, CH = RowElem<E>::CH, KBLK = RowElem<E>::KBLK;
    constexpr unsigned ES = sizeof(E);
    constexpr int PARTS = NW * 64 / (8 * CT) < NW ? NW * 64 / (8 * CT) : NW;     // lanes that add up one output
    __shared__ float red[2][NW * RED_W];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    Stretches<kRouted> st(bt, route, T);
    const BranchLanes br(bt);
    arrived(st.v_beg, st.v_end);
    const TileCursor<kRouted> cur(st, blockIdx.x);
    const int row0 = cur.row0(st);
    if (row0 < 0) {                                      // with routing the grid covers all active rows
        clear_floats(clear, clear_n, NW * 64, grid);
        return;
    }
    constexpr bool kPart = kEdges || sizeof(E) == 4;     // runs of floats are whole chunks of 4: half a tile may be left
    const int rows = kPart && cur.end(st) - row0 < 8 ? cur.end(st) - row0 : 8;
    const E *zero = reinterpret_cast<const E *>(g_zero16);
    const int chunk = (q + 4 * (r16 >> 3)) * CH;         // this lane's K elements of a block
    const int w_row = kPart && (r16 & 7) >= rows ? rows - 1 : r16 & 7;
    const size_t w_off = (size_t)(row0 + w_row) * d_model + chunk;
    const Window x(X, (unsigned)T * (unsigned)d_model * ES);
    const bool tok = r16 % CT < T;
    const int x_k = NG == 2 ? chunk : q * CH;
    const unsigned x_lane = ((unsigned)(r16 % CT) * (unsigned)d_model + x_k) * ES;
    u32x4 wg[XB], wu[XB], xa[XB][NM];
#pragma unroll
    for (int j = 0; j < XB; ++j) {
        const int k = (wave + NW * j) * KBLK;
        wg[j] = ld16(k + chunk < d_model ? Wg + w_off + k : zero);
        wu[j] = ld16(k + chunk < d_model ? Wu + w_off + k : zero);
#pragma unroll
        for (int i = 0; i < NM; ++i)
            xa[j][i] = x.ld16(tok && k + 4 * CH * i + x_k < d_model, x_lane + (k + 4 * CH * i) * ES);
    }
    clear_floats(clear, clear_n, NW * 64, grid);
    f32x4 ag[NM], au[NM];
#pragma unroll
    for (int i = 0; i < NM; ++i) ag[i] = au[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < XB; ++j)
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            ag[i] = mfma_chunk<E>(wg[j], xa[j][i], ag[i]);
            au[i] = mfma_chunk<E>(wu[j], xa[j][i], au[i]);
        }
    // register v of lane l is D[row 4 q + v][col r16]: neuron (4 q + v) % 8, K half q / 2; its columns are those of that half
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        red[0][wave * RED_W + v * RED_V + lane] = NM == 2 && q >= 2 ? ag[NM - 1][v] : ag[0][v];
        red[1][wave * RED_W + v * RED_V + lane] = NM == 2 && q >= 2 ? au[NM - 1][v] : au[0][v];
    }
    __syncthreads();
    // PARTS lanes per output, the neurons of a token side by side: fixed order of the sum
    const int p = lane % PARTS, o = threadIdx.x / PARTS, t = o / 8, row = o % 8;
    float g = 0.f, up = 0.f;
#pragma unroll
    for (int i = 0; i < NW / PARTS; ++i)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int at = (p * (NW / PARTS) + i) * RED_W + row % 4 * RED_V + (row / 4 + 2 * half) * 16 +
                           (NG == 2 ? 8 * half : 0) + t % CT;
            g += red[0][at];
            up += red[1][at];
        }
#pragma unroll
    for (int d = 1; d < PARTS; d <<= 1) {
        g += __shfl_xor(g, d);
        up += __shfl_xor(up, d);
    }
    int bn = br.branch(row0);                            // the tile may span branches: only a run's ends are multiples of 8
    for (int i = bn, next; (next = br.next(i)) <= row0 + rows - 1; ++i) bn += next <= row0 + row ? 1 : 0;
    const float alpha = __shfl(br.v_alpha, bn);
    if (p != 0 || t >= T || t >= CT || row >= rows) return;
    float h = kEdges || sizeof(E) == 4 ? alpha * (g / (1.0f + expf(-g)) * up) : alpha * silu_mul(g, up);
    if (kRouted) h = route[(size_t)t * bt.B + bn] ? h : 0.f;
    store_h(Hout + (size_t)t * ldh + row0 + row, h);
}

// Down projection, one workgroup per R output features and 1 / KS of the K blocks (blockIdx.y); its waves take the blocks
// of SB elements in turn.  KS = 2: the two sums of an output are added into `out` by float atomics, which the gate+up
// kernel before has cleared: 0 + a + b is the same number in either order.  KS = 1: plain stores, float or bf16.
// Fewer rows per workgroup keep more CUs busy and cost more loads of H per weight byte (CT / R of them): see down_shape.
template <int NW, int U, int R, int NG, int KS, bool kRouted, bool kEdges, typename E>
__global__ void __launch_bounds__(NW * 64)
decode_down_rows(const E *__restrict__ Hin, int ldx, int T, const E *__restrict__ Wd, int ldw,
                 int d_model, float *__restrict__ out, int out_bf16, const uint8_t *__restrict__ route, BranchTable bt)
{
    constexpr int CH = RowElem<E>::CH;
    constexpr unsigned ES = sizeof(E);
    constexpr int KG = 16 / R, NM = KG / NG, CT = 16 / NG, SB = 4 * CH * KG;
    constexpr int PARTS = NW * 64 / (R * CT) < NW ? NW * 64 / (R * CT) : NW;
    static_assert(KG % NG == 0 && PARTS >= 1, "K groups per MFMA; a thread for every output");
    __shared__ float red[NW * RED_W];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    Stretches<kRouted> st(bt, route, T);
    arrived(st.v_beg, st.v_end);
    const int row0 = blockIdx.x * R;
    const int rows = d_model - row0 < R ? d_model - row0 : R;
    const Window w(Wd + (size_t)row0 * ldw, (unsigned)rows * (unsigned)ldw * ES);
    const Window h(Hin, (unsigned)T * (unsigned)ldx * ES);
    const int chunk = (q + 4 * (r16 / R)) * CH;          // this lane's K elements of a block
    const bool row_ok = r16 % R < rows, tok = r16 % CT < T;
    const unsigned w_lane = (unsigned)(r16 % R) * (unsigned)ldw * ES;
    const unsigned h_lane = (unsigned)(r16 % CT) * (unsigned)ldx * ES;
    // where the blocks of a stretch start: with kEdges at the chunk that it starts in
    auto first_k = [&](int r) { return kEdges ? st.beg(r) / CH * CH : st.beg(r); };
    auto blocks = [&](int r) { return st.end(r) > st.beg(r) ? (st.end(r) - first_k(r) + SB - 1) / SB : 0; };

    // cursor over this wave's blocks: the blocks of all stretches laid end to end, cut into KS contiguous parts
    int nb_all = 0;
    for (int r = 0; r < st.count(); ++r) nb_all += blocks(r);
    const int part = (nb_all + KS - 1) / KS;
    const int first = (int)blockIdx.y * part + wave;
    const int last = (int)(blockIdx.y + 1) * part < nb_all ? (int)(blockIdx.y + 1) * part : nb_all;
    const int total = last > first ? (last - first + NW - 1) / NW : 0;
    int cr = 0, cb = first, issued = 0;
    auto settle = [&]() {                                // move past stretches the block index overshoots
        while (cr < st.count()) {
            const int nb = blocks(cr);
            if (cb < nb) break;
            cb -= nb;
            ++cr;
        }
    };
    settle();
    u32x4 wa[U], xa[U][NM];
    int k_of[U], beg_of[U], end_of[U];                   // kEdges: first K of the block in the slot, its stretch
    auto load = [&](int u) {                             // the block under the cursor, zeros past this wave's last
        const bool live = cr < st.count() && issued < total;
        ++issued;
        const int k = live ? first_k(cr) + cb * SB : 0;
        const int kend = live ? st.end(cr) : -1;
        wa[u] = w.ld16(row_ok && k + chunk < kend, w_lane + (k + chunk) * ES);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int kx = k + (q + 4 * (i * NG + r16 / CT)) * CH;
            xa[u][i] = h.ld16(tok && kx < kend, h_lane + kx * ES);
        }
        if (kEdges) {
            k_of[u] = k;
            beg_of[u] = live ? st.beg(cr) : 0;
            end_of[u] = kend;
        }
        cb += NW;
        settle();
    };
    f32x4 acc[NM];
#pragma unroll
    for (int i = 0; i < NM; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) load(u);
    for (int j = 0; j < total; j += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kEdges && (k_of[u] < beg_of[u] || k_of[u] + SB > end_of[u])) {
                wa[u] = keep_elements<E>(wa[u], beg_of[u] - k_of[u] - chunk, end_of[u] - k_of[u] - chunk);
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    const int kx = k_of[u] + (q + 4 * (i * NG + r16 / CT)) * CH;
                    xa[u][i] = keep_elements<E>(xa[u][i], beg_of[u] - kx, end_of[u] - kx);
                }
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) acc[i] = mfma_chunk<E>(wa[u], xa[u][i], acc[i]);
            if (j + U < total) load(u);
        }
    }
    // register v of lane l is D[row 4 q + v][col r16]: K group (4 q) / R, whose columns are r16 / CT == group % NG
    const int group = 4 * q / R;
    f32x4 mine = acc[0];
#pragma unroll
    for (int i = 1; i < NM; ++i) mine = group / NG == i ? acc[i] : mine;
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave * RED_W + v * RED_V + lane] = mine[v];
    __syncthreads();
    // PARTS lanes per output, the features of a token side by side (coalesced stores and atomics): fixed order of the sum
    const int p = lane % PARTS, o = threadIdx.x / PARTS, t = o / R, row = o % R;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NW / PARTS; ++i)
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const int d = g * R + row;
            sum += red[(p * (NW / PARTS) + i) * RED_W + d % 4 * RED_V + d / 4 * 16 + g % NG * CT + t % CT];
        }
#pragma unroll
    for (int d = 1; d < PARTS; d <<= 1) sum += __shfl_xor(sum, d);
    if (p != 0 || t >= T || t >= CT || row >= rows) return;
    const size_t at = (size_t)t * d_model + row0 + row;
    if (KS == 2) atomicAdd(&out[at], sum);
    else if (out_bf16) reinterpret_cast<uint16_t *>(out)[at] = to_bf16(sum);
    else out[at] = sum;
}

// The one-tile workgroups start sooner than the ring kernel and load x (2 T d_model bytes) once per 8 neurons (32 d_model bytes
// of weights): the rule bounds what they load of x in all, and with more than 8 tokens, where a K block takes twice the
// loads and registers, d_model as well.  us a call, ring / one tile:
//   T <= 8:  896 x 4800 T = 8 (8.6 MB of x) 12.1 / 11.2, 1280 x 6912 T = 8 (18 MB) 21.2 / 20.2, 1536 x 8256 T = 8 (25 MB) 24.3 / 24.2, 896 x
//     16384 T = 8 (29 MB) 26.0 / 25.4;  past the line 896 x 24576 T = 8 (44 MB) 33.6 / 34.4, 1280 x 16384 T = 8 (42 MB) 37.5 / 38.5, 1280 x
//     32768 T = 8 (84 MB) 66.6 / 68.5.  896 x 65536 T = 1 (15 MB) 69.3 / 68.0, T = 4 (59 MB) 74.2 / 73.1; 1536 x 32768 T = 4 (50 MB) 65.6 / 65.6.
//   T > 8:  640 x 3456 T = 16 (9 MB) 10.8 / 10.3, 896 x 4800 T = 16 (17 MB) 13.5 / 13.3, 1024 x 5504 T = 16 (23 MB) 15.5 / 15.4, 768 x 8192 T =
//     16 (25 MB) 17.8 / 17.7;  past the line 896 x 8192 T = 16 (29 MB) 18.6 / 18.7, 896 x 16384 T = 10 (37 MB) 27.3 / 28.6, T = 16 29.9 / 32.4;
//     1152 x 6208 T = 10 18.9 / 19.9, 1280 x 6912 T = 10 20.4 / 21.3, 1408 x 7552 T = 10 21.6 / 22.8.
constexpr int ONCE_MAX_D = 1536, ONCE_MAX_D_16 = 1024, ONCE_NW = 4;
constexpr long long ONCE_X_BYTES_4 = 64 << 20, ONCE_X_BYTES_8 = 32 << 20, ONCE_X_BYTES_16 = 24 << 20;
constexpr int ONCE_ROUTED_X = 14336;                     // elements of x
constexpr int ROWS_MAX_D = 2048;                         // float storage and odd boundaries: what 8 waves hold of x
bool gate_up_once(int T, int d_model, long long tiles)
{
    const long long x_bytes = 2LL * T * d_model * tiles;
    if (T > 8) return d_model <= ONCE_MAX_D_16 && x_bytes <= ONCE_X_BYTES_16;
    return d_model <= ONCE_MAX_D && x_bytes <= (T > 4 ? ONCE_X_BYTES_8 : ONCE_X_BYTES_4);
}

// Rows per workgroup of decode_down_rows, 0: the kernels for wide layers.  us a step with 4 / 8 / 16 rows and with the
// wide kernels, the gate+up ring kernel before it.
//   float (two workgroups per row tile with 8 and 16 rows, one with 4):
//     896 T = 1 12.9 / 12.9 / 14.3 / 15.9, T = 16 16.8 / 14.8 / 16.7 / 17.9;  1280 T = 8 18.3 / 16.1 / 16.3 / 18.0, T = 16 22.8 /
//     18.6 / 17.9 / 19.2;  2048 T = 1 22.8 / 23.0 / 25.5 / 25.3, T = 8 28.9 / 25.2 / 26.3 / 26.2, T = 16 37.1 / 29.7 / 28.1 / 28.0;
//     2560 T = 1 29.5 / 29.6 / 33.6 / 36.2, T = 16 50.9 / 40.2 / 40.3 / 42.3.  8 rows where 4 are as good: the order of the sum
//     stays that of 64-element blocks.
//     Wide layers, K = 3.5 d_model, 8 rows / wide kernel, T = 1, 2 and 4:  3072 41.2 / 42.6, 41.6 / 42.8, 42.8 / 43.2;  3584 54.2 / 53.9, 55.0 /
//     54.4, 57.2 / 54.6;  4096 64.5 / 64.8, 65.3 / 65.2, 68.1 / 65.6;  5120 103.5 / 115.1, 104.4 / 116.2, 108.6 / 118.6;  6144 138.7 / 147.5,
//     140.1 / 148.8, 147.2 / 151.3;  8192 234.1 / 239.6, 237.0 / 241.3, 247.6 / 242.7;  16384 x 16384 292.0 / 308.8, 294.2 / 310.0.
//   bf16 result (one workgroup per row tile):
//     896 T = 1 12.8 / 14.2 / 16.7 / 18.9, T = 16 16.8 / 17.8 / 21.7 / 22.2;  1280 T = 8 18.3 / 16.5 / 19.8 / 20.7;  2048 T = 16 37.1 /
//     29.8 / 34.5 / 33.8;  2560 T = 16 50.9 / 45.6 / 39.8 / 38.9.
//     4 / 8 rows, K = 4.5 d_model, T = 1, 2 and 4:  1152 13.2 / 13.5, 13.8 / 13.9, 15.2 / 14.7;  1536 17.9 / 17.6, 18.6 / 18.0, 20.4 / 19.1 (K =
//     8256, T = 2 20.7 / 21.2);  1792 21.6 / 22.2, 22.2 / 22.4, 23.9 / 23.2;  2048 25.5 / 26.4, 26.1 / 26.6, 27.9 / 27.2.
//     4 rows / wide kernel, K = 3.5 d_model, T = 1, 2 and 4:  2560 32.3 / 37.0, 33.4 / 37.5, 36.3 / 38.3;  3584 53.8 / 55.4, 55.7 / 56.1, 60.7 /
//     57.1;  4096 63.8 / 67.4, 65.7 / 68.3, 72.1 / 69.3;  6144 137.8 / 153.8, 141.3 / 155.9;  8192 232.7 / 237.2, 238.2 / 239.2, 262.5 / 243.8.
constexpr int WIDE_TILES = 192;                          // row tiles of 16 from which the wide kernels fill the chip
int down_shape(int T, int d_model, bool out_bf16)
{
    const bool few = T <= 2;
    if (out_bf16) return d_model <= 1024 || few ? 4 : (d_model < 2560 ? 8 : 0);
    if (ceil_div(d_model, 16) >= WIDE_TILES) return few ? 8 : 0;
    return T <= 8 || d_model <= 1024 ? 8 : 16;
}

// Layers of 1032 to 3064 features leave decode_down_rows with unequal numbers of workgroups per CU, or with idle CUs; while K is
// short nobody waits for them, a long K is bound by the bytes in flight of the busiest CU, and 16 waves of decode_down_split on a row
// tile have more.  K = neurons of active branches.  us a call, rows / 16 waves, K = 8192, 16384 and 32768:
//   1280 T = 1 17.7 / 18.8, 30.9 / 30.2, 53.7 / 52.8;  T = 8 21.5 / 21.4, 38.5 / 35.7, 68.8 / 63.1;  T = 16 23.5 / 23.8, 39.9 / 38.8, 74.2 / 70.1
//   2048 T = 1 23.5 / 25.4, 41.3 / 40.7, 74.9 / 75.6;  T = 8 25.6 / 26.3, 45.1 / 43.0, 82.0 / 78.9;  T = 16 28.4 / 28.0, 49.0 / 47.1, 88.7 / 85.3
//   2560 T = 1 29.1 / 34.9, 53.7 / 58.3;  T = 8 33.0 / 37.5, 59.5 / 63.4;  T = 16 39.8 / 41.2, 72.2 / 70.3, 138.4 / 131.1
//   1024 T = 1 24.4 / 26.7 (16384), T = 8 47.9 / 54.2 (32768), T = 16 53.7 / 60.9.
bool down_long_k(int T, int d_model, int k)
{
    if (d_model <= 1024 || ceil_div(d_model, 16) >= WIDE_TILES) return false;
    return T > 8 ? k > (d_model <= 2048 ? 8128 : 12288) : d_model <= 2048 && k > 12288;
}

constexpr size_t kStreamLdsMax = 160 * 1024;

}  // namespace

// kFew: sizes that are only taken with at most 8 tokens.
template <int NW, int XB, bool kRouted, bool kEdges, typename E, bool kFew = false>
static void launch_gate_up_once_xb(const FwdArgs &a, const BranchTable &bt, int tiles, float *clear, int clear_n)
{
    auto kernel = decode_gate_up_once<NW, XB, 2, kRouted, kEdges, E>;
    if constexpr (!kFew) kernel = a.T <= 8 ? kernel : decode_gate_up_once<NW, XB, 1, kRouted, kEdges, E>;
    kernel<<<tiles, NW * 64, 0, a.stream>>>(
        static_cast<const E *>(a.x), a.T, static_cast<const E *>(a.Wg), static_cast<const E *>(a.Wu),
        a.d_model, static_cast<E *>(a.H), a.ldh, a.route, clear, clear_n, tiles, bt);
}
// Whole tables in bf16: d_model is at most ONCE_MAX_D, with more than 8 tokens ONCE_MAX_D_16 (not routed).  Odd boundaries and float storage: at most
// ROWS_MAX_D, floats with more than 8 tokens 910 (decode_rows_takes).
template <bool kRouted, bool kEdges = false, typename E = uint16_t>
static void launch_gate_up_once(const FwdArgs &a, const BranchTable &bt, int tiles, float *clear, int clear_n)
{
    constexpr int KBLK = RowElem<E>::KBLK;
    constexpr bool kWhole = !kEdges && !kRouted && sizeof(E) == 2;
    static_assert(ONCE_MAX_D <= 6 * ONCE_NW * KBLK || !kWhole, "K blocks per wave");
    static_assert(ONCE_MAX_D_16 <= 4 * ONCE_NW * KBLK || !kWhole, "more than 8 tokens: at most 4 K blocks per wave");
    static_assert(ROWS_MAX_D <= (sizeof(E) == 2 ? 8 * ONCE_NW : 8 * 8) * KBLK && 910 <= 8 * ONCE_NW * KBLK, "K blocks per wave");
    const int xb = ceil_div(ceil_div(a.d_model, KBLK), ONCE_NW);
    if (xb <= 2) launch_gate_up_once_xb<ONCE_NW, 2, kRouted, kEdges, E>(a, bt, tiles, clear, clear_n);
    else if (xb <= 4) launch_gate_up_once_xb<ONCE_NW, 4, kRouted, kEdges, E>(a, bt, tiles, clear, clear_n);
    else if (xb <= 6) launch_gate_up_once_xb<ONCE_NW, 6, kRouted, kEdges, E, kWhole>(a, bt, tiles, clear, clear_n);
    if constexpr (kEdges || sizeof(E) == 4) {
        if (xb > 6 && xb <= 8) launch_gate_up_once_xb<ONCE_NW, 8, kRouted, kEdges, E>(a, bt, tiles, clear, clear_n);
    }
    if constexpr (sizeof(E) == 4) {
        if (xb > 8 && xb <= 12) launch_gate_up_once_xb<8, 6, kRouted, kEdges, E, true>(a, bt, tiles, clear, clear_n);
        else if (xb > 12) launch_gate_up_once_xb<8, 8, kRouted, kEdges, E, true>(a, bt, tiles, clear, clear_n);
    }
}

// 8 waves with 5 K blocks each requested as the kernel starts (8 blocks of half the size with 16 rows).
template <int R, int NG, int KS, bool kRouted, bool kEdges = false, typename E = uint16_t>
static void launch_down_rows(const FwdArgs &a, const BranchTable &bt)
{
    decode_down_rows<8, R == 16 ? 8 : 5, R, NG, KS, kRouted, kEdges, E><<<dim3(ceil_div(a.d_model, R), KS), 8 * 64, 0, a.stream>>>(
        static_cast<const E *>(a.H), a.ldh, a.T, static_cast<const E *>(a.Wd), a.d_inter, a.d_model, a.out,
        a.out_bf16 ? 1 : 0, a.route, bt);
}

// The sums that two workgroups add into need `out` at zero.  The gate+up kernel clears it beside its own work, except where
// that would take x or weights from its other workgroups: a launch of its own then (896 x 4864, T = 8 in place: one launch more).
static float *cleared_by_gate_up(const FwdArgs &a, bool added_into) { return added_into && !a.in_place ? a.out : nullptr; }
static hipError_t clear_in_place(const FwdArgs &a, bool added_into)
{
    return added_into && a.in_place ? launch_fill_zero(a.out, (size_t)a.T * a.d_model, a.stream) : hipSuccess;
}

// T <= 16, float storage or a bf16 table with odd boundaries (kEdges), sizes that decode_rows_takes accepts.
template <bool kEdges, typename E>
static hipError_t launch_decode_rows_impl(const FwdArgs &a, const BranchTable &bt)
{
    long long tiles = 0;
    for (int r = 0; r < bt.n_runs; ++r) tiles += (bt.run_end[r] - bt.run_start[r] + 7) / 8;
    {
        ProfileScope ps(MLPMOE_KERNEL_DECODE_GATE_UP, a.stream);
        launch_gate_up_once<false, kEdges, E>(a, bt, (int)tiles, cleared_by_gate_up(a, !a.out_bf16), a.T * a.d_model);
    }
    if (launch_status("decode gate+up (rows) launch") != hipSuccess || clear_in_place(a, !a.out_bf16) != hipSuccess)
        return hipErrorLaunchFailure;
    ProfileScope ps(MLPMOE_KERNEL_DECODE_DOWN, a.stream);
    const int rows = down_shape(a.T, a.d_model, a.out_bf16);
    if (!a.out_bf16 && rows == 8)                        // floats: always, 16 rows need more than 8 tokens of more than 1024 features
        a.T <= 8 ? launch_down_rows<8, 2, 2, false, kEdges, E>(a, bt) : launch_down_rows<8, 1, 2, false, kEdges, E>(a, bt);
    if constexpr (sizeof(E) == 2) {
        if (!a.out_bf16 && rows == 16) launch_down_rows<16, 1, 2, false, kEdges, E>(a, bt);
    }
    if constexpr (sizeof(E) == 2) {
        if (a.out_bf16 && rows == 8)
            a.T <= 8 ? launch_down_rows<8, 2, 1, false, kEdges, E>(a, bt) : launch_down_rows<8, 1, 1, false, kEdges, E>(a, bt);
        else if (a.out_bf16)
            a.T <= 4 ? launch_down_rows<4, 4, 1, false, kEdges, E>(a, bt)
                     : (a.T <= 8 ? launch_down_rows<4, 2, 1, false, kEdges, E>(a, bt) : launch_down_rows<4, 1, 1, false, kEdges, E>(a, bt));
    }
    return launch_status("decode down (rows) launch");
}

template <bool kRouted>
static hipError_t launch_decode_impl(const FwdArgs &a, const BranchTable &bt)
{
    long long tiles1 = 0;
    for (int r = 0; r < bt.n_runs; ++r) tiles1 += (bt.run_end[r] - bt.run_start[r]) / 8;
    const int tiles2 = ceil_div(a.d_model, 16);
    if (tiles1 > 0x7fffffffLL) return hipErrorInvalidValue;
    const uint16_t *X = static_cast<const uint16_t *>(a.x);
    uint16_t *H = static_cast<uint16_t *>(a.H);
    const size_t xs_bytes = (size_t)a.T * (a.d_model * 2 + 16) + 16 + 2 * DEC_SNW * 256 * sizeof(float);
    // blocks of K per wave and tile in the persistent kernels, padded to whole ring revolutions
    const int nb_pad = ceil_div(ceil_div(ceil_div(a.d_model, KB), DEC_SNW), DEC_SU) * DEC_SU;
    const bool x_in_regs = nb_pad <= 16;                    // d_model <= 8192: x fragments stay in registers
    const bool persistent = x_in_regs || xs_bytes <= kStreamLdsMax;
    // A float result comes from the down kernel that splits K over two workgroups and adds the halves
    // into `out` with atomics; `out` is cleared by the persistent gate+up kernel, so the pair is only used
    // together.
    const bool split_down = persistent && !a.out_bf16;
    float *clear = cleared_by_gate_up(a, split_down);
    const int clear_n = a.T * a.d_model;
    const uint16_t *Wg = static_cast<const uint16_t *>(a.Wg), *Wu = static_cast<const uint16_t *>(a.Wu);
    // How many tiles of a routed call are live is known on the device only.  Few are, as a rule, and the one-tile workgroups end sooner:
    // 1152 x 6208, T = 12, 1 / 4 / 8 of 16 branches 12.7 / 13.7 / 16.4 us, with the ring kernel 14.2 / 15.2 / 17.7.
    if (kRouted ? a.d_model <= ONCE_MAX_D && a.T * a.d_model <= ONCE_ROUTED_X : gate_up_once(a.T, a.d_model, tiles1)) {
        ProfileScope ps(MLPMOE_KERNEL_DECODE_GATE_UP, a.stream);
        launch_gate_up_once<kRouted>(a, bt, (int)tiles1, clear, clear_n);
        if (launch_status("decode gate+up (one tile per workgroup) launch") != hipSuccess) return hipErrorLaunchFailure;
    } else if (persistent) {
        // per device, set up on the first call there: CU count and the LDS limit of the kernel that stages x
        static std::mutex mu;
        static int cus_of[64] = {0};              // one table per instantiation (attribute is per kernel)
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return note_hip_error("hipGetDevice", e);
        if (dev < 0 || dev >= 64) return note_hip_error("device index", hipErrorInvalidDevice);
        int n_cus;
        {
            std::lock_guard<std::mutex> lock(mu);
            if (cus_of[dev] == 0) {
                hipDeviceProp_t prop;
                e = hipGetDeviceProperties(&prop, dev);
                if (e != hipSuccess) return note_hip_error("hipGetDeviceProperties", e);
                e = hipFuncSetAttribute(
                    reinterpret_cast<const void *>(&decode_gate_up_persist<DEC_SNW, DEC_SU, kRouted>),
                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStreamLdsMax);
                if (e != hipSuccess) return note_hip_error("hipFuncSetAttribute(decode_gate_up_persist)", e);
                cus_of[dev] = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
            }
            n_cus = cus_of[dev];
        }
        const int grid = tiles1 < n_cus ? (int)tiles1 : n_cus;
        ProfileScope ps(MLPMOE_KERNEL_DECODE_GATE_UP, a.stream);
        const int nb_wave = ceil_div(ceil_div(a.d_model, KB), DEC_SNW);      // K blocks per wave and tile
        if (nb_wave <= 2)
            decode_gate_up_xreg<DEC_SNW, DEC_SU, 2, kRouted><<<grid, DEC_SNW * 64, 0, a.stream>>>(
                X, a.T, Wg, Wu, a.d_model, H, a.ldh, a.route, clear, clear_n, grid, bt);
        else if (nb_wave <= 4)
            decode_gate_up_xreg<DEC_SNW, DEC_SU, 4, kRouted><<<grid, DEC_SNW * 64, 0, a.stream>>>(
                X, a.T, Wg, Wu, a.d_model, H, a.ldh, a.route, clear, clear_n, grid, bt);
        else if (nb_pad <= 8)
            decode_gate_up_xreg<DEC_SNW, DEC_SU, 8, kRouted><<<grid, DEC_SNW * 64, 0, a.stream>>>(
                X, a.T, Wg, Wu, a.d_model, H, a.ldh, a.route, clear, clear_n, grid, bt);
        else if (nb_pad <= 16)
            decode_gate_up_xreg<DEC_SNW, DEC_SU, 16, kRouted><<<grid, DEC_SNW * 64, 0, a.stream>>>(
                X, a.T, Wg, Wu, a.d_model, H, a.ldh, a.route, clear, clear_n, grid, bt);
        else
            decode_gate_up_persist<DEC_SNW, DEC_SU, kRouted><<<grid, DEC_SNW * 64, xs_bytes, a.stream>>>(
                X, a.T, Wg, Wu, a.d_model, H, a.ldh, a.route, clear, clear_n, grid, bt);
        if (launch_status("decode gate+up (persistent) launch") != hipSuccess) return hipErrorLaunchFailure;
    } else {
        ProfileScope ps(MLPMOE_KERNEL_DECODE_GATE_UP, a.stream);
        decode_kernel<DEC_NW1, DEC_U1, true, kRouted><<<(unsigned)tiles1, DEC_NW1 * 64, 0, a.stream>>>(
            X, a.d_model, a.T, Wg, Wu, a.d_model, a.d_model, H, a.ldh, nullptr, 0, a.route, bt);
        if (launch_status("decode gate_up launch") != hipSuccess) return hipErrorLaunchFailure;
    }
    if (clear_in_place(a, split_down) != hipSuccess) return hipErrorLaunchFailure;
    ProfileScope ps(MLPMOE_KERNEL_DECODE_DOWN, a.stream);
    // Routed calls: how many neurons some token takes is known on the device only, and walking a stretch per branch costs the many
    // workgroups of a few rows more.  They keep the kernels that are right for a short K: 4096 x 14336, T = 2, 1 / 2 / 4 of 16 branches with
    // 8 rows 17.7 / 18.8 / 23.9 us, with the wide kernel 15.1 / 17.0 / 23.2; 1536 x 16384, T = 16, 1 / 4 branches with 16 waves 18.2 / 22.8, with
    // rows 16.4 / 20.7.
    const bool wide_routed = kRouted && tiles2 >= WIDE_TILES && a.T * (long long)a.d_model > 4096;
    const int rows = !persistent || wide_routed ? 0 : down_shape(a.T, a.d_model, a.out_bf16);
    if (!kRouted && split_down && down_long_k(a.T, a.d_model, bt.d_eff))
        decode_down_split<16, 4, 1><<<dim3(tiles2, 2), 16 * 64, 0, a.stream>>>(
            H, a.ldh, a.T, static_cast<const uint16_t *>(a.Wd), a.d_inter, a.d_model, a.out, a.route, bt);
    else if (split_down && rows == 16)
        launch_down_rows<16, 1, 2, kRouted>(a, bt);
    else if (split_down && rows == 8)
        a.T <= 8 ? launch_down_rows<8, 2, 2, kRouted>(a, bt) : launch_down_rows<8, 1, 2, kRouted>(a, bt);
    else if (split_down)
        decode_down_split<4, 8, 2, kRouted><<<dim3(ceil_div(a.d_model, 32), 2), 4 * 64, 0, a.stream>>>(
            H, a.ldh, a.T, static_cast<const uint16_t *>(a.Wd), a.d_inter, a.d_model, a.out, a.route, bt);
    else if (!kRouted && rows == 8)
        a.T <= 8 ? launch_down_rows<8, 2, 1, false>(a, bt) : launch_down_rows<8, 1, 1, false>(a, bt);
    else if (!kRouted && rows == 4)
        a.T <= 4 ? launch_down_rows<4, 4, 1, false>(a, bt)
                 : (a.T <= 8 ? launch_down_rows<4, 2, 1, false>(a, bt) : launch_down_rows<4, 1, 1, false>(a, bt));
    else if (tiles2 >= WIDE_TILES)
        decode_kernel<DEC_NW2, DEC_U2, false, kRouted><<<tiles2, DEC_NW2 * 64, 0, a.stream>>>(
            H, a.ldh, a.T, static_cast<const uint16_t *>(a.Wd), nullptr, a.d_inter, a.d_model, nullptr,
            a.ldh, a.out, a.out_bf16 ? 1 : 0, a.route, bt);
    else if constexpr (!kRouted)                         // a bf16 result of 2560 to 3064 features
        decode_kernel<16, 4, false><<<tiles2, 1024, 0, a.stream>>>(
            H, a.ldh, a.T, static_cast<const uint16_t *>(a.Wd), nullptr, a.d_inter, a.d_model, nullptr,
            a.ldh, a.out, a.out_bf16 ? 1 : 0, a.route, bt);
    return launch_status("decode_down launch");
}

hipError_t launch_decode_bf16(const FwdArgs &a, const BranchTable &bt) { return launch_decode_impl<false>(a, bt); }

// Per-token routing, T <= 16: the kernels read a.route themselves and need no scratch.
hipError_t launch_decode_routed_bf16(const FwdArgs &a, const BranchTable &bt) { return launch_decode_impl<true>(a, bt); }

// Float storage, and bf16 tables with odd boundaries, at T <= 16: which sizes the row kernels take (else the prefill
// kernels).  The line is where loading x and H once per workgroup, and with more than 8 tokens twice the MFMAs, costs as much as
// the prefill kernels' idle token rows.  us a call, prefill / row kernels:
//   odd boundaries, 12 branches, 9 kept, bf16 result: 1280 x 5000, T = 1 22.1 / 11.1, T = 16 23.0 / 16.6; 1600 x 6000, T = 1 26.2 /
//     14.9, T = 16 27.4 / 22.2; with more active neurons the prefill kernels fill the chip: 1280 features, 9222 neurons T = 12 29.5 / 28.9,
//     T = 16 29.8 / 31.6, 12294 T = 8 28.9 / 27.5, T = 9 29.0 / 30.1, T = 16 29.5 / 36.2, 24582 T = 8 52.0 / 51.0, T = 16 52.8 / 70.3, 49158 T = 4 89.9 /
//     86.9, T = 8 91.0 / 97.5; 1600 features, 9222 T = 9 30.6 / 30.0, T = 12 30.8 / 32.5;
//   floats: 512 x 2048, T = 1 19.4 / 7.8, T = 16 19.9 / 10.3; 896 x 4864, T = 1 31.1 / 19.4, T = 8 30.9 / 22.0, T = 12 31.0 / 31.9; 2048 x
//     8000, T = 1 62.7 / 44.8, T = 8 62.9 / 52.0, T = 12 63.8 / 73.7.
bool decode_rows_takes(int T, int d_model, int d_eff, bool out_bf16, bool is_bf16)
{
    if (T > 16 || d_model > ROWS_MAX_D || down_shape(T, d_model, out_bf16) == 0) return false;
    if (!is_bf16) return T <= 8 || T * d_model <= 8192;
    return T * d_model <= 25600 && (T <= 4 || d_eff <= (T > 8 ? 8192 : 32768));
}

hipError_t launch_decode_rows_bf16(const FwdArgs &a, const BranchTable &bt) { return launch_decode_rows_impl<true, uint16_t>(a, bt); }

// d_model and d_inter are multiples of 4.
hipError_t launch_decode_rows_f32(const FwdArgs &a, const BranchTable &bt)
{
    bool even = true;
    for (int r = 0; r < bt.n_runs; ++r) even = even && bt.run_start[r] % 4 == 0 && bt.run_end[r] % 4 == 0;
    return even ? launch_decode_rows_impl<false, float>(a, bt) : launch_decode_rows_impl<true, float>(a, bt);
}

}  // namespace mlpmoe
