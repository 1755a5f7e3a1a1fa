// MFMA kernels of the two-kernel variant for 65..256 tokens per launch (gfx950).
//
// With more than 64 tokens the block stops being a matrix-vector stream: per weight tile
// there are 8..16 token tiles of MFMA work, too many accumulators for one wavefront and too
// much operand traffic if every wavefront fetched its own copy of the weights.  These
// kernels are the "row-major" end of the Method section's tiling choice carried through: a
// workgroup's eight wavefronts share weight and activation tiles through LDS.  Wavefront
// (tg, kh) owns token group tg of four (1..4 tiles of 16 tokens) and half kh of every step's k
// range: the eight read each weight tile four times per step in all, where eight wavefronts that
// each own tokens over the whole k range read it eight times.  Those operand reads were the
// bound (66 of 70 us of the gate/up kernel at 256 tokens of the 4096 x 14336 layer, the
// loads alone taking less): LDS moves 134 KB per 64 k where it moved 190 KB.  Measured: 61 us there, whole
// call 129 -> 116 us; 8192 x 28672 at 150 tokens (three tiles per group, where 150 tokens had taken the form for
// 256) gate/up 280 -> 205, down 171 -> 122, whole call 443 -> 328 us.
//
// Data movement is the asynchronous global->LDS tile load of the other MFMA kernels,
// organised as a workgroup pipeline:
//   * a step is 64 k (or two such pieces in the gate/up kernel): tiles of 16 rows x 128 bytes (one cache line per row), 2 KB.  In
//     LDS the eight 16-byte pieces of row i sit XOR-swizzled by i / 2, so that the operand reads of 16 rows cover all banks once.
//   * wavefronts 0..3 request the weights, 4..7 the activations.  Loads complete in issue order
//     per wavefront, so a wavefront that requested both would have to wait for its newest
//     activations (one or two steps ahead, out of L2) and with them for every older weight load (several
//     steps ahead, out of HBM): the weights in flight would shrink to what the activations' look-ahead allows.
//   * one LDS-only barrier per step: before it every requesting wavefront waits, by count, for its own
//     loads of the step; after it the step's tiles are whole and the buffers of the step before are free to refill.
//
// Gate/up kernel: workgroup s owns a d_ff slice of at most 8 row tiles (8 rows of W_gate and
// the same 8 of W_up per tile; up to 16 in its wide form).  Down kernel: workgroup (js, cb) owns one 128-column block over
// d_ff split js; W_down is regrouped per lane with v_perm_b32 as in the other down kernels.
// In both the two halves of the k range meet in LDS at the end, each wavefront finishing half of the
// outputs.  The down kernel's sums over the splits are plain stores of partial blocks and a small third launch.
#include <atomic>
#include <algorithm>
#include <type_traits>

#include "dfk_big_plan.h"
#include "dfk_mfma_common.h"

// (the token groups' rows of stamps follow each other)
#define DFK_STAMP_BIG(k) DFK_STAMP_OF(blockIdx.y * (unsigned)per_group + blockIdx.x, k)

namespace dfk {
namespace {

constexpr int kBigWaves = 8;          // 4 token groups x 2 halves of the k range
constexpr int kBigTokensPerLaunch = 256;
constexpr int kBigStepK = 64;         // k (d_ff rows in the down kernel) of one pipeline step
constexpr int kBigTile = 2048;        // 16 rows x 128 bytes

constexpr size_t kL2BytesPerXcd = (size_t)4 << 20;

// Buffers (pipeline steps) of the activations, which come out of L2: two steps ahead is enough (with one: 72 -> 83 us for
// the gate/up kernel at 256 tokens of the 4096 x 14336 layer, 49 -> 66 at 128).  The weights, out of HBM, get what LDS is left,
// up to 8.  Compile-time constants of a kernel, so that the wait of a step is one instruction with a constant count.
constexpr int kBigXBufs = 3;
constexpr int big_w_bufs(int x_step, int w_step) {
    return (kLdsLimit - kBigXBufs * x_step) / w_step < 8 ? (kLdsLimit - kBigXBufs * x_step) / w_step : 8;
}
// 64-k pieces per step of the gate/up kernel.  A step costs about 0.4 us before any multiplication; with few row tiles per slice
// and few token tiles per group that is most of it, so two pieces share one, where LDS still holds three buffers of it (whole
// call: 2432 x 3968 at 65 tokens 36.6 -> 32.8 us, 2560 x 3712 at 107 39.6 -> 37.0, 2304 x 8192 at 104 45.9 -> 43.1).  With one
// token tile per group it gained 10 % at five row tiles (2304 x 9216) and lost 5 % at four (8192 x 7168), so not beyond three.
constexpr int big_gateup_pieces(int TT, int NTC) { return (TT == 1 && NTC <= 3) || (TT == 2 && NTC <= 5) ? 2 : 1; }

// s_waitcnt vmcnt(n) for a run-time n (uniform); more than 63 waits for 63.
__device__ __forceinline__ void wait_vm_exact(int n) {
#define DFK_VM_CASE(k) case k: DFK_WAIT_VM(k); break;
#define DFK_VM_CASE8(k) DFK_VM_CASE(k) DFK_VM_CASE(k + 1) DFK_VM_CASE(k + 2) DFK_VM_CASE(k + 3) \
                        DFK_VM_CASE(k + 4) DFK_VM_CASE(k + 5) DFK_VM_CASE(k + 6) DFK_VM_CASE(k + 7)
    switch (n) {
        DFK_VM_CASE8(0) DFK_VM_CASE8(8) DFK_VM_CASE8(16) DFK_VM_CASE8(24)
        DFK_VM_CASE8(32) DFK_VM_CASE8(40) DFK_VM_CASE8(48)
        DFK_VM_CASE(56) DFK_VM_CASE(57) DFK_VM_CASE(58) DFK_VM_CASE(59) DFK_VM_CASE(60) DFK_VM_CASE(61) DFK_VM_CASE(62)
        default: DFK_WAIT_VM(63); break;
    }
#undef DFK_VM_CASE8
#undef DFK_VM_CASE
    asm volatile("" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vm_const() {
    DFK_WAIT_VM(N < 63 ? N : 63);
    asm volatile("" ::: "memory");
}

// A lane's offset from a scalar base, kept as the 32 bits it is: hoisted out of the loop as a 64-bit value it takes twice the
// registers and a 64-bit add per load instead of the load's own scalar base.
__device__ __forceinline__ unsigned keep32(unsigned o) {
    asm("" : "+v"(o));
    return o;
}

// This lane's byte offset of its MFMA operand within a tile: row q, the 16-byte piece of k group g of half kh.
__device__ __forceinline__ int big_operand_off(int q, int g, int kh) { return q * 128 + (((4 * kh + g) ^ (q >> 1)) & 7) * 16; }

// Step at which a workgroup of the gate/up kernel starts its walk through the k range.  All of them read the same X: in lock-step
// they would ask the same few L2 channels for the same lines at the same moment, so starts differ, as a rule over the whole
// range.  But what is live of X is what lies between the first and the last of an XCD's workgroups (b, b + 8, ...), and that has
// to stay in its 4 MB L2 beside the weights passing through.  Where X is larger than 3 MB the starts are spread over a window of
// 64 steps (2 MB at 256 tokens and 64 k a step) instead: otherwise X came from beyond the L2 again for every workgroup.  The same
// where rows are a multiple of 16 KB apart: there a step's rows lie in the same memory channels, and XCDs that walk in step
// spread the weights better.  Whole call, us, whole range / window / all at step 0: 16384 x 8192 at 256 tokens 455 / 269 / 274,
// 16384 x 16384 at 128 364 / 319 / 352, 12288 x 12288 at 200 285 / 261 / 267, 12288 x 20480 at 200 482 / 444, 8192 x 28672 at 256
// 387 / 376, 8192 x 14336 at 100 148 / 142 / 150, 8192 x 28672 at 80 267 / 264.  On the other side of the line: 9856 x 28032 at
// 111 (2.2 MB) 326 / 332, 5504 x 25216 at 105 193 / 196, 5760 x 29568 at 227 (2.6 MB) 305 / 305, 4096 x 14336 at 128 85.5 / 86.2
// / 90.1.
__device__ __forceinline__ int big_k_start(const MlpArgs& a, int nsteps) {
    const unsigned b = blockIdx.x;
    const size_t row = (size_t)a.d_model * 2;
    const bool window = nsteps > 64 && (a.m_count * row > ((size_t)3 << 20) || row % 16384 == 0);
    return window ? (int)((b >> 3) * 7u & 63u) : (int)(b * 7u % (unsigned)nsteps);
}

// Which (d_ff split, column block) a workgroup of the down kernel takes.  Workgroups are handed to
// the 8 XCDs in turn (workgroup b runs on XCD b % 8) and each XCD has its own L2; all column blocks
// of a split read the same A_2 rows, so a split's workgroups are placed on one XCD (or, with fewer
// than 8 splits, on 8 / splits of them) and those rows are fetched into that L2 once.  Any other
// split count keeps the plain order, and so does a launch whose whole A_2 fits one L2 (the host
// decides: there the plain order measured 2 us faster, at 128 tokens of the 8B shape; beyond,
// the placement gains 1 to 4 us of 60 at 256 tokens of that shape and 13 of 200 on the 70B
// shape).  A bijection from
// [0, S * C) onto S x C in every case.
__device__ __forceinline__ void down_tile_of(int b, int S, int C, bool by_xcd, int& js, int& cb) {
    const int x = b & 7, r = b >> 3;
    if (!by_xcd) {
        js = b / C;
        cb = b - js * C;
    } else if ((S & 7) == 0) {
        js = x + 8 * (r / C);
        cb = r % C;
    } else if ((S == 1 || S == 2 || S == 4) && ((C * S) & 7) == 0) {
        js = x % S;
        cb = (x / S) * (C * S / 8) + r;
    } else {
        js = b / C;
        cb = b - js * C;
    }
}

// Step at which a workgroup of the down kernels starts its split: in step with the split's other column blocks, or (own) in a start of
// its own, against the lock-step on the L2 channels.  In step, what is live of the A_2 rows stays small and XCDs spread W_down over the
// memory channels, which is what counts where A_2 is larger than an L2 and a split's workgroups are on several XCDs, and with wide
// rows of W_down.  Own where a whole split sits on one XCD (down_tile_of, a multiple of 8 splits), or where all of A_2 fits one L2 and
// rows of W_down are below 8 KB or W_down is given as [d_model, d_ff].  Down kernel with its sum, us, own / in step: 16384 x 16384 at 128
// tokens 142 / 117, 9856 x 28032 at 111 148 / 110, 5760 x 29568 at 227 146 / 126; 4096 x 14336 at 256 (on one XCD) 51.9 / 53.0.
// Whole call, own over in step, A_2 below 4 MB, at 80, 128 and 200 tokens: 1792 x 9344 0.988, 0.993, 0.986, 2560 x 6912 0.997, 0.986,
// 1.006, 3072 x 7936 0.987, 0.987, 0.995, 2816 x 9600 0.994, 0.994, 1.011; 4096 x 8192 1.003, 1.002, 1.010, 12288 x 4096 1.012, 1.010,
// 1.003; W_down as [d_model, d_ff]: 2304 x 9216 0.982, 0.986, 0.996, 12288 x 4096 0.977, 0.985, 0.985, 16384 x 4096 0.944, 0.957, 0.988.
template <bool DOWN_T>
__device__ __forceinline__ int big_down_start(const MlpArgs& a, bool by_xcd, int cb, int nsteps) {
    const bool own = by_xcd ? (a.k2_splits & 7) == 0 : DOWN_T || a.d_model < 4096;
    return own ? (int)(cb * 5u % (unsigned)nsteps) : 0;
}

// ---------------------------------------------------------------- gate/up kernel
// NTC: the largest row-tile count of a d_ff slice of the launch (a compile-time constant so that
// a step is straight-line code); every slice has NTC or NTC - 1 row tiles (the missing one's sums are never stored).
//
// DOWN_T: the same pipeline computes the down projection from W_down given as [d_model, d_ff]: Y^T = W_down^T A_2^T has the shape
// of stage one with d_ff as the k range and A_2 in X's place.  Workgroup (js, cb) owns 128 rows of W_down^T (NTC = 8 tiles of 16
// rows of the one matrix) over d_ff split js in whole 64-row steps; the end stores the partial block of the split.
//
// WIDE: slices of up to 16 row tiles (NTC even; NTC to NTC - 2 of them), for layers whose slices of 8 take two or more rounds of
// workgroups on the CUs.  What bounds those is the loads of the two streams: each round reads all of X out of L2 again, 24 KB beside 14 KB of
// weights per step of a workgroup at 150 tokens of the 8192 x 28672 layer.  Sums of that many tiles times both halves of the k range do not fit the
// registers, so wavefront (tg, kh) owns row tiles half kh over the whole k range instead: the same bytes of LDS reads per row tile, and no
// exchange at the end.  It goes through a step's k range in two rounds and reads operands one round ahead (a whole step ahead did not fit
// the registers at three token tiles and 14 row tiles).
template <int TT, typename E, int NTC, bool DOWN_T = false, bool WIDE = false>
__device__ __forceinline__ void gateup_big_body(const MlpArgs& a, unsigned char* lds, const bool by_xcd = false) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane & 15, g = lane >> 4;
    const int tg = wave & 3, kh = wave >> 2;
    int j0, j1, js = 0, cb = 0, k0 = 0;            // rows of the weights; d_ff split, column block and first k (DOWN_T)
    constexpr int KS = DOWN_T || WIDE ? 1 : big_gateup_pieces(TT, NTC);
    constexpr int NR = WIDE ? NTC / 2 : NTC;       // row tiles of a wavefront
    static_assert(!WIDE || (NTC % 2 == 0 && !DOWN_T), "halves of the row tiles");
    int nsteps;
    if (DOWN_T) {
        down_tile_of((int)blockIdx.x, a.k2_splits, a.k2_col_blocks, by_xcd, js, cb);
        const int steps = a.d_ff / kBigStepK;
        int k1;
        share_of((unsigned)steps, (unsigned)a.k2_splits, (unsigned)js, k0, k1);
        nsteps = k1 - k0;
        k0 *= kBigStepK;
        j0 = cb * 128; j1 = j0 + 128;
    } else {
        slice_rows(a.d_ff, a.splits, blockIdx.x, j0, j1);
        nsteps = a.d_model / (kBigStepK * KS);
    }
    const int nt = DOWN_T ? NTC : (j1 - j0) / 8;   // NTC or NTC - 1, with WIDE also NTC - 2 (slices differ by at most one 8-row group)
    const size_t row_bytes = (size_t)(DOWN_T ? a.d_ff : a.d_model) * 2;
    const int tile0 = tg * TT;                     // first token tile of this wavefront's group
    const int t0 = (int)blockIdx.y * a.group_tokens, count = min(a.group_tokens, a.m_count - t0);   // this workgroup's tokens
    const int per_group = DOWN_T ? a.k2_splits * a.k2_col_blocks : a.splits;

    const int rot = DOWN_T ? big_down_start<true>(a, by_xcd, cb, nsteps) : big_k_start(a, nsteps);
    const int prow = lane >> 3, piece = lane & 7;  // a load covers 8 rows: lane l takes row l / 8, and the piece that belongs to its place
    const int lo = big_operand_off(q, g, WIDE ? 0 : kh);
    const int rt0 = WIDE ? kh * NR : 0;            // first row tile of this wavefront

    f32x4 acc[NR][TT];
#pragma unroll
    for (int rt = 0; rt < NR; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (DOWN_T && js >= a.k2_splits) return;       // as in the down kernel below
    DFK_STAMP_BIG(DOWN_T ? 3 : 0);
    constexpr int x_piece = 4 * TT * kBigTile, w_piece = NTC * kBigTile, x_step = KS * x_piece, w_step = KS * w_piece;
    constexpr int nbx = kBigXBufs, nbw = big_w_bufs(x_step, w_step), w_off = nbx * x_step;
    // The steps of a wavefront that requests N weight loads per 64-k piece or (N = -1) activations: of the slice's 2 nt weight
    // loads (half n & 1 of row tile n / 2: the gate rows or the up rows) n = wave, wave + 4, ...; or the two loads of each token
    // tile of its group.
    auto steps = [&](auto n_) {
        constexpr int N = decltype(n_)::value;
        constexpr bool W = N >= 0;
        constexpr int PER = W ? N : 2 * TT, SLOTS = KS * PER;
        constexpr int nb = W ? nbw : nbx;
        const char* const src = (W && DOWN_T ? (const char*)a.Wd + (size_t)(j0 + wave * 8) * row_bytes
                                 : W         ? (const char*)(wave & 1 ? a.Wu : a.Wg) + (size_t)(j0 + (wave >> 1) * 8) * row_bytes
                                             : (const char*)(DOWN_T ? a.a2 : a.X) + (size_t)(a.m_base + t0) * row_bytes) + (size_t)k0 * 2;
        // Byte offset of load i: row 16 i (gate and up rows; 32 i of the one matrix) or 8 i (tokens, the last one for those that
        // do not exist) further on than load 0's; the piece's place changes by half a row (64 bytes) from a tile's rows 0..7 to
        // its rows 8..15.
        const unsigned rb = (unsigned)row_bytes;
        const unsigned off = (unsigned)(W ? prow : tile0 * 16 + prow) * rb, off_last = (unsigned)(count - 1) * rb;
        const unsigned place = (unsigned)(((piece ^ (prow >> 1)) & 7) * 16) ^ (W && (wave & 1) ? 64u : 0u);
        unsigned char* const dst0 = W ? lds + w_off + (wave >> 1) * kBigTile + (wave & 1) * 1024 : lds + tile0 * kBigTile;
        constexpr int buf_bytes = W ? w_step : x_step;
        auto source = [&](int step) { return src + (size_t)(step + rot < nsteps ? step + rot : step + rot - nsteps) * (KS * kBigStepK * 2); };
        auto load = [&](const char* p, unsigned char* dst, int slot) {
            const int u = PER ? slot / PER : 0, i = slot - u * PER;   // (constants)
            const unsigned o = W ? off + (DOWN_T ? 32u : 16u) * i * rb + place : min(off + 8u * i * rb, off_last) + (place ^ (i & 1 ? 64u : 0u));
            __builtin_amdgcn_global_load_lds(p + u * (kBigStepK * 2) + keep32(o), DFK_LDS_PTR(dst + u * (W ? w_piece : x_piece) + i * (W ? 2 * kBigTile : 1024)), 16, 0,
                                             W ? kAuxNonTemporal : 0);
        };
        for (int s = 0; s < nb && s < nsteps; ++s)
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) load(source(s), dst0 + s * buf_bytes, i);

        u32x4 xk[2][KS][TT], wv[2][KS][NR];        // operands of this step (WIDE: round) and of the next
        int xbuf = 0, wbuf = 0, freebuf = 0;
        wait_vm_exact(SLOTS * (min(nb, nsteps) - 1));
        lds_barrier();
#pragma unroll
        for (int u = 0; u < KS; ++u) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) xk[0][u][tt] = *(const u32x4*)(lds + u * x_piece + (tile0 + tt) * kBigTile + lo);
#pragma unroll
            for (int rt = 0; rt < NR; ++rt) wv[0][u][rt] = *(const u32x4*)(lds + w_off + u * w_piece + (rt0 + rt) * kBigTile + lo);
        }
        // The loads of step s + 1 have landed (later ones may be in flight), and every wavefront has read step s:
        // its buffers are free for the loads of step s + nb.
        auto wait_next = [&](int s, auto whole_) {
            if (decltype(whole_)::value || s + nb <= nsteps) wait_vm_const<SLOTS * (nb - 2)>();
            else if (s + 1 < nsteps) wait_vm_exact(SLOTS * (nsteps - s - 2));
            lds_barrier();
            if (++xbuf == nbx) xbuf = 0;
            if (++wbuf == nbw) wbuf = 0;
        };
        if constexpr (WIDE) {
            // MFMAs of round u of a step beside the operand reads of the round behind it, and loads [l0, l1) of step s + nb.
            auto round = [&](auto u_, int s, int l0, int l1, auto whole_) {
                constexpr int cur = decltype(u_)::value, nxt = cur ^ 1;
                const unsigned char* xs = lds + xbuf * x_step + tile0 * kBigTile + (lo ^ (64 * nxt));
                const unsigned char* ws = lds + w_off + wbuf * w_step + rt0 * kBigTile + (lo ^ (64 * nxt));
                const char* p = source(s + nb < nsteps ? s + nb : 0);
                unsigned char* dst = dst0 + freebuf * buf_bytes;
                const bool more = decltype(whole_)::value || s + nb < nsteps;
#pragma unroll
                for (int rt = 0; rt < NR; ++rt) {
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mfma16<E>(wv[cur][0][rt], xk[cur][0][tt], acc[rt][tt]);
                    wv[nxt][0][rt] = *(const u32x4*)(ws + rt * kBigTile);
#pragma unroll
                    for (int tt = rt * TT / NR; tt < (rt + 1) * TT / NR; ++tt) xk[nxt][0][tt] = *(const u32x4*)(xs + tt * kBigTile);
                    if (more) {
#pragma unroll
                        for (int i = l0 + rt * (l1 - l0) / NR; i < l0 + (rt + 1) * (l1 - l0) / NR; ++i) load(p, dst, i);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            constexpr auto first = std::integral_constant<int, 0>{};
            constexpr auto second = std::integral_constant<int, 1>{};
            round(first, nsteps, 0, 0, std::false_type{});
            int s = 0;
            for (; s + nb < nsteps; ++s) {
                wait_next(s, std::true_type{});
                round(second, s, 0, SLOTS / 2, std::true_type{});
                round(first, s, SLOTS / 2, SLOTS, std::true_type{});
                if (++freebuf == nb) freebuf = 0;
            }
            for (; s < nsteps; ++s) {
                wait_next(s, std::false_type{});
                round(second, nsteps, 0, 0, std::false_type{});    // (behind the last step it reads operands that nothing multiplies)
                if (s + 1 < nsteps) round(first, nsteps, 0, 0, std::false_type{});
                if (++freebuf == nb) freebuf = 0;
            }
        } else {
        auto step = [&](int s, auto cur_, auto whole_) {
            constexpr int cur = decltype(cur_)::value, nxt = cur ^ 1;
            wait_next(s, whole_);
            const unsigned char* xs = lds + xbuf * x_step + tile0 * kBigTile + lo;
            const unsigned char* ws = lds + w_off + wbuf * w_step + lo;
            const char* p = source(s + nb < nsteps ? s + nb : 0);
            unsigned char* dst = dst0 + freebuf * buf_bytes;
            const bool more = decltype(whole_)::value || s + nb < nsteps;
            // Loads, operand reads of step s + 1 and MFMAs of step s in turn: in three blocks one after the other, each of the
            // three units idles while the eight wavefronts queue for another (75 us at 256 tokens of the 4096 x 14336 layer).
#pragma unroll
            for (int x = 0; x < KS * NTC; ++x) {
                const int u = x / NTC, rt = x - u * NTC;
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mfma16<E>(wv[cur][u][rt], xk[cur][u][tt], acc[rt][tt]);
                wv[nxt][u][rt] = *(const u32x4*)(ws + u * w_piece + rt * kBigTile);
#pragma unroll
                for (int tt = rt * TT / NTC; tt < (rt + 1) * TT / NTC; ++tt) xk[nxt][u][tt] = *(const u32x4*)(xs + u * x_piece + tt * kBigTile);
                if (more) {
#pragma unroll
                    for (int i = x * SLOTS / (KS * NTC); i < (x + 1) * SLOTS / (KS * NTC); ++i) load(p, dst, i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (++freebuf == nb) freebuf = 0;
        };
        int s = 0;
        // Steps that request another have a loop of their own: with a branch around each row tile's loads the call took, us, 141.9 where
        // it takes 134.2 (4096 x 20480 at 230 tokens), 208.6 / 200.4 (8192 x 18432 at 180), 111.1 / 109.7 (4096 x 14336 at 256).
        for (; s + 1 + nb < nsteps; s += 2) {
            step(s, std::integral_constant<int, 0>{}, std::true_type{});
            step(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
        }
        for (; s + 1 < nsteps; s += 2) {
            step(s, std::integral_constant<int, 0>{}, std::false_type{});
            step(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
        }
        if (s < nsteps) step(s, std::integral_constant<int, 0>{}, std::false_type{});
        }
    };
    constexpr int NMAX = (2 * NTC + 3) / 4;        // a weight wavefront has NMAX loads per step or one less
    if (kh == 1) steps(std::integral_constant<int, -1>{});
    else if ((2 * nt - wave + 3) >> 2 == NMAX) steps(std::integral_constant<int, NMAX>{});
    else steps(std::integral_constant<int, NMAX - 1>{});
    DFK_STAMP_BIG(DOWN_T ? 4 : 2);

    float scale[TT];                               // of the lane's tokens (requested here, used behind the barriers)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
        scale[tt] = !DOWN_T && a.row_scale ? a.row_scale[a.m_base + t0 + min((tile0 + tt) * 16 + q, count - 1)] : 1.f;

    // D tile of (row tile, token tile): lane (q, g) holds token q, tile rows 4g .. 4g+3; rows 0..7
    // are the gate rows, 8..15 the up rows of the same 8 d_ff rows: lanes 32 apart pair up.
    auto store = [&](const f32x4 sum, int rt, int tt) {
        const f32x4 v = sum * scale[tt];
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __shfl_xor(v[i], 32);
        const int m = (tile0 + tt) * 16 + q;
        if (g < 2 && m < count) {
            uint2 pk;
            pk.x = E::pack2(silu_mul_fast(v[0], o[0]), silu_mul_fast(v[1], o[1]));
            pk.y = E::pack2(silu_mul_fast(v[2], o[2]), silu_mul_fast(v[3], o[3]));
            *(uint2*)((uint16_t*)a.a2 + (size_t)(a.m_base + t0 + m) * a.d_ff + j0 + rt * 8 + 4 * g) = pk;
        }
    };
    if constexpr (WIDE) {
#pragma unroll
        for (int rt = 0; rt < NR; ++rt)
            if (rt0 + rt < nt) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) store(acc[rt][tt], rt0 + rt, tt);
            }
        DFK_STAMP_BIG(1);
        return;
    } else {
    // The halves of the k range meet: wavefront (tg, 0) finishes row tiles [0, H), (tg, 1) the others.
    constexpr int H = (NTC + 1) / 2;
    lds_barrier();                                 // nothing in flight and nothing read any more: the buffers are free
    f32x4* mine = (f32x4*)lds + (size_t)wave * (H * TT * 64) + lane;
    const f32x4* theirs = (const f32x4*)lds + (size_t)(wave ^ 4) * (H * TT * 64) + lane;
#pragma unroll
    for (int rt = 0; rt < NTC; ++rt)
        if ((rt < H) == (kh == 1)) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) mine[((rt < H ? rt : rt - H) * TT + tt) * 64] = acc[rt][tt];
        }
    __syncthreads();
    if (DOWN_T) {              // four adjacent columns of the split's partial block, summed by the launch that follows
#pragma unroll
        for (int rt = 0; rt < NTC; ++rt) {
            if ((rt < H) == (kh == 0)) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const f32x4 v = acc[rt][tt] + theirs[((rt < H ? rt : rt - H) * TT + tt) * 64];
                    const int m = (tile0 + tt) * 16 + q;
                    if (m < count) *(f32x4*)(a.P + ((size_t)js * a.m_count + t0 + m) * a.d_model + j0 + rt * 16 + 4 * g) = v;
                }
            }
        }
        DFK_STAMP_BIG(6);
        return;
    }
#pragma unroll
    for (int rt = 0; rt < NTC; ++rt) {
        if ((rt < H) == (kh == 0) && rt < nt) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) store(acc[rt][tt] + theirs[((rt < H ? rt : rt - H) * TT + tt) * 64], rt, tt);
        }
    }
    DFK_STAMP_BIG(1);
    }
}

template <int TT, typename E, int NTC>
__global__ __launch_bounds__(kBigWaves * 64) void k_gateup_big(MlpArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    gateup_big_body<TT, E, NTC>(a, lds);
}
template <int TT, typename E, int NTC>
__global__ __launch_bounds__(kBigWaves * 64) void k_gateup_wide(MlpArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    gateup_big_body<TT, E, NTC, false, true>(a, lds);
}

// ---------------------------------------------------------------- down kernel
template <int TT, typename E>
__device__ __forceinline__ void down_big_body(const MlpArgs& a, const bool by_xcd, unsigned char* lds) {
    __shared__ int flag;
    constexpr int NTHREADS = kBigWaves * 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane & 15, g = lane >> 4;
    const int tg = wave & 3, kh = wave >> 2;
    int js, cb;   // d_ff split and 128-column block of this workgroup (one column block each: checked on the host)
    down_tile_of((int)blockIdx.x, a.k2_splits, a.k2_col_blocks, by_xcd, js, cb);
    int j0, j1;
    slice_rows(a.d_ff, a.k2_splits, js, j0, j1);
    const int rows = j1 - j0;
    const int nsteps = (rows + kBigStepK - 1) / kBigStepK;
    const size_t row_bytes = (size_t)a.d_model * 2;
    const int tile0 = tg * TT;
    const int t0 = (int)blockIdx.y * a.group_tokens, count = min(a.group_tokens, a.m_count - t0);   // this workgroup's tokens
    const int per_group = a.k2_splits * a.k2_col_blocks;

    const int rot = big_down_start<false>(a, by_xcd, cb, nsteps);
    const int prow = lane >> 3, piece = lane & 7;
    const int lo = big_operand_off(q, g, kh);

    f32x4 acc2[8][TT];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc2[c][tt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A workgroup that only fills up a row of the grid (big_down_launch; the order is plain there, so its split would be past the last).
    // Asked here and not on entry, where every workgroup waited for two arguments before it requested the others.  Whole call, us, on entry /
    // here: 896 x 1280 at 234 tokens 18.5 / 18.3; W_down as [d_model, d_ff], 512 x 1152 at 228 18.0 / 17.9, 896 x 1664 at 96 16.45 / 16.26.
    if (js >= a.k2_splits) return;
    DFK_STAMP_BIG(3);
    constexpr int x_step = 4 * TT * kBigTile, w_step = 4 * kTileBytes;
    constexpr int nbx = kBigXBufs, nbw = big_w_bufs(x_step, w_step), w_off = nbx * x_step;
    // Loads per step: wavefronts 0..3 take row u = wave of the four 4 KB tiles (32-row block b, half h) of W_down: rows
    // 32 b + 4 h + 8 g + u of the step, 256 bytes each; 4..7 the two loads of each token tile of their group
    // (A_2: 64 rows = one cache line per token).  Rows past the split are any valid address (zeroed at use).
    auto steps = [&](auto is_w, auto ragged_) {
        constexpr bool W = decltype(is_w)::value, RAGGED = decltype(ragged_)::value;
        constexpr int SLOTS = W ? 4 : 2 * TT;
        constexpr int nb = W ? nbw : nbx;
        const char* const src = W ? (const char*)a.Wd + (size_t)cb * 256 : (const char*)a.a2 + ((size_t)(a.m_base + t0) * a.d_ff + j0) * 2;
        // A_2: byte offsets of the first token's row and of the last that exists (256 tokens x 2 d_ff bytes: below 4 GiB)
        const unsigned a2_row = (unsigned)a.d_ff * 2u;
        const unsigned off = (unsigned)(tile0 * 16 + prow) * a2_row, off_last = (unsigned)(count - 1) * a2_row;
        unsigned char* const dst0 = W ? lds + w_off + wave * 1024 : lds + tile0 * kBigTile;
        constexpr int buf_bytes = W ? w_step : x_step;
        auto first_row = [&](int step) { return (step + rot < nsteps ? step + rot : step + rot - nsteps) * kBigStepK; };
        // A step's address is scalar but for offsets that do not change, unless the split's last step is partial.
        unsigned lane_off[SLOTS];
#pragma unroll
        for (int i = 0; i < SLOTS; ++i)
            lane_off[i] = W ? (unsigned)(((i >> 1) * 32 + (i & 1) * 4 + 8 * g + wave) * row_bytes) + 16u * q
                            : min(off + (unsigned)(8 * i) * a2_row, off_last) + (unsigned)(((piece ^ (((i & 1) * 8 + prow) >> 1)) & 7) * 16);
        auto load = [&](int r0, unsigned char* dst, int i) {
            if (W) {
                const char* p = RAGGED ? src + (size_t)min(j0 + r0 + (i >> 1) * 32 + (i & 1) * 4 + 8 * g + wave, a.d_ff - 1) * row_bytes + 16 * q
                                       : src + (size_t)(j0 + r0) * row_bytes + keep32(lane_off[i]);
                __builtin_amdgcn_global_load_lds(p, DFK_LDS_PTR(dst + i * kTileBytes), 16, 0, kAuxNonTemporal);
            } else {
                const char* p = RAGGED ? src + min(off + (unsigned)(8 * i) * a2_row, off_last) + (size_t)min(r0 + 8 * ((piece ^ (((i & 1) * 8 + prow) >> 1)) & 7), rows - 8) * 2
                                       : src + (size_t)r0 * 2 + keep32(lane_off[i]);
                __builtin_amdgcn_global_load_lds(p, DFK_LDS_PTR(dst + i * 1024), 16, 0, 0);
            }
        };
        for (int s = 0; s < nb && s < nsteps; ++s)
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) load(first_row(s), dst0 + s * buf_bytes, i);

        u32x4 av[2][TT], w[2][8];    // A_2[token q of tile tt][rows 8g .. 8g+7 of block kh]; the same rows of W_down, 8 columns
        const unsigned char* const xs0 = lds + tile0 * kBigTile + lo;
        const unsigned char* const ws0 = lds + w_off + kh * 2 * kTileBytes + lane * 16;
        int xbuf = 0, wbuf = 0, freebuf = 0;
        wait_vm_exact(SLOTS * (min(nb, nsteps) - 1));
        lds_barrier();
#pragma unroll
        for (int r = 0; r < 8; ++r) w[0][r] = *(const u32x4*)(ws0 + (r >> 2) * kTileBytes + (r & 3) * 1024);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) av[0][tt] = *(const u32x4*)(xs0 + tt * kBigTile);
        auto step = [&](int s, auto cur_, auto whole_) {
            constexpr int cur = decltype(cur_)::value, nxt = cur ^ 1;
            if (decltype(whole_)::value || s + nb <= nsteps) wait_vm_const<SLOTS * (nb - 2)>();
            else if (s + 1 < nsteps) wait_vm_exact(SLOTS * (nsteps - s - 2));
            lds_barrier();
            if (++xbuf == nbx) xbuf = 0;
            if (++wbuf == nbw) wbuf = 0;
            const unsigned char* xs = xs0 + xbuf * x_step;
            const unsigned char* ws = ws0 + wbuf * w_step;
            const bool more = decltype(whole_)::value || s + nb < nsteps;
            const int r0 = first_row(more ? s + nb : 0);
            unsigned char* dst = dst0 + freebuf * buf_bytes;
            const int here = first_row(s);
            if (RAGGED && here + kBigStepK > rows && here + kh * 32 + 8 * g >= rows) {   // this lane's eight rows are past the split: they contribute nothing
#pragma unroll
                for (int r = 0; r < 8; ++r) w[cur][r] = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) av[cur][tt] = u32x4{0, 0, 0, 0};
            }
            u32x4 bb[2];                           // operands of a column tile and the next
            auto regroup = [&](int c) {
#pragma unroll
                for (int p = 0; p < 4; ++p) bb[c & 1][p] = __builtin_amdgcn_perm(w[cur][2 * p + 1][c >> 1], w[cur][2 * p][c >> 1], c & 1 ? 0x07060302u : 0x05040100u);
            };
            regroup(0);
            // operand reads of step s + 1, loads and MFMAs of step s in turn, as in the gate/up kernel
#pragma unroll
            for (int c = 0; c < 8; ++c) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc2[c][tt] = mfma16<E>(av[cur][tt], bb[c & 1], acc2[c][tt]);
                if (c < 7) regroup(c + 1);          // beside the MFMAs
                w[nxt][c] = *(const u32x4*)(ws + (c >> 2) * kTileBytes + (c & 3) * 1024);
#pragma unroll
                for (int tt = c * TT / 8; tt < (c + 1) * TT / 8; ++tt) av[nxt][tt] = *(const u32x4*)(xs + tt * kBigTile);
                if (more) {
#pragma unroll
                    for (int i = c * SLOTS / 8; i < (c + 1) * SLOTS / 8; ++i) load(r0, dst, i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (++freebuf == nb) freebuf = 0;
        };
        int s = 0;
        // As in the gate/up kernel (with the regrouping beside the MFMAs, not before them: 8192 x 28672 at 150 tokens, whole call, 306.6 us
        // before, 298.9 with this loop there and here, 294.9 with both); the clamped addresses leave no registers for a second loop.
        for (; !RAGGED && s + 1 + nb < nsteps; s += 2) {
            step(s, std::integral_constant<int, 0>{}, std::true_type{});
            step(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
        }
        for (; s + 1 < nsteps; s += 2) {
            step(s, std::integral_constant<int, 0>{}, std::false_type{});
            step(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
        }
        if (s < nsteps) step(s, std::integral_constant<int, 0>{}, std::false_type{});
    };
    if (rows % kBigStepK == 0) {       // whole steps only: no clamped addresses, nothing to zero
        if (kh == 0) steps(std::true_type{}, std::false_type{});
        else steps(std::false_type{}, std::false_type{});
    } else {
        if (kh == 0) steps(std::true_type{}, std::true_type{});
        else steps(std::false_type{}, std::true_type{});
    }
    DFK_STAMP_BIG(4);

    // D tile (column tile c, token tile tt): lane (q, g) holds tokens 4g .. 4g+3 of the tile, column
    // 8q + c of the block: the lane's 8 column tiles are 8 consecutive columns.  The halves of the k range meet:
    // wavefront (tg, 0) finishes tokens 4g and 4g+1, (tg, 1) tokens 4g+2 and 4g+3.
    lds_barrier();
    f32x4* mine = (f32x4*)lds + (size_t)wave * (TT * 4 * 64) + lane;
    const f32x4* theirs = (const f32x4*)lds + (size_t)(wave ^ 4) * (TT * 4 * 64) + lane;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int x = 0; x < 4; ++x) {              // token i = x / 2 of the partner's two, columns 4 (x & 1) ..
            const int c = 4 * (x & 1);
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = kh == 0 ? acc2[c + e][tt][2 + (x >> 1)] : acc2[c + e][tt][x >> 1];
            mine[(tt * 4 + x) * 64] = v;
        }
    __syncthreads();
    const bool atomic_mode = a.reduce_mode == DFK_REDUCE_ATOMIC;
    const int nb0 = cb * 128;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f32x4 v0 = theirs[(tt * 4 + 2 * i) * 64], v1 = theirs[(tt * 4 + 2 * i + 1) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v0[e] += kh == 0 ? acc2[e][tt][i] : acc2[e][tt][2 + i];
                v1[e] += kh == 0 ? acc2[4 + e][tt][i] : acc2[4 + e][tt][2 + i];
            }
            const int m = (tile0 + tt) * 16 + 4 * g + 2 * kh + i;
            if (m < count) {
                if (atomic_mode) {
                    float* dst = a.yacc + (size_t)m * a.d_model + nb0 + 8 * q;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { acc_add(dst + e, v0[e]); acc_add(dst + 4 + e, v1[e]); }
                } else {       // partial block of the split: plain stores, summed by the launch that follows
                    float* dst = a.P + ((size_t)js * a.m_count + t0 + m) * a.d_model + nb0 + 8 * q;
                    *(f32x4*)dst = v0;
                    *(f32x4*)(dst + 4) = v1;
                }
            }
        }
    }
    if (atomic_mode) {
        drain_own_memory_ops();
        __syncthreads();
        if (tid == 0) flag = arrive_last(a.tickets + cb, (unsigned)a.k2_splits) ? 1 : 0;
        __syncthreads();
        if (!flag) return;
        drain_accumulator<E, NTHREADS>(a, nb0, 128);
    }
}

template <int TT, typename E>
__global__ __launch_bounds__(kBigWaves * 64) void k_down_big(MlpArgs a, int by_xcd) {   // by_xcd: place the workgroups of a d_ff split on one XCD (see down_tile_of)
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    down_big_body<TT, E>(a, by_xcd != 0, lds);
}

// Down projection from W_down given as [d_model, d_ff], 65 tokens and more (and fewer, see wdt_split_pays): the pipeline of the
// gate/up kernel over (d_ff splits) x (blocks of 128 rows of W_down^T).  Its sibling for a few tokens, whose workgroups own rows
// whole so that nothing is summed across them, takes 64 tokens per launch and streams all three weights again for each 64: that,
// not its own pace, bounded it.  Whole call, 4096 x 14336, us: 80 tokens 149 -> 77, 128 173 -> 85, 256 345 -> 108 (the other
// layout, whose weights are regrouped in registers, 115).
template <int TT, typename E>
__global__ __launch_bounds__(kBigWaves * 64) void k_down_t_big(MlpArgs a, int by_xcd) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    gateup_big_body<TT, E, 8, true>(a, lds, by_xcd != 0);
}

// Sum of the splits' partial blocks (counter reduction of the down kernels, this file's and the 64-token pair's): a launch of
// its own spreads it over the whole chip, where the last workgroup of a column block would read them all alone (tens of MB with
// hundreds of tokens; a chain of round trips with a few).  Fixed order (split 0, 1, ...): bitwise reproducible.  One thread per four
// consecutive outputs; all loads of up to BATCH splits are requested before the first is added.  With few outputs it is nothing but
// one round trip, so each CU gets one wavefront and 16 splits one batch: block of 896 x 4864 at 1 and 16 tokens 15.9 -> 15.3, 16.9 -> 16.1
// us against 256 threads a workgroup and batches of 8.
template <typename E, int BATCH, int WAYS>
__global__ __launch_bounds__(256) void k_sum_partials(MlpArgs a) {
    const unsigned w4 = (unsigned)a.d_model >> 2;
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (unsigned)a.m_count * w4) return;
    const size_t blk = (size_t)a.m_count * a.d_model;
    const float* src = a.P + (size_t)4 * idx;
    float4 s[WAYS];
#pragma unroll
    for (int w = 0; w < WAYS; ++w) s[w] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
    for (int js0 = 0; js0 < a.k2_splits; js0 += BATCH) {
        float4 t[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            t[k] = js0 + k < a.k2_splits ? *(const float4*)(src + (size_t)(js0 + k) * blk) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < BATCH; ++k) { s[k % WAYS].x += t[k].x; s[k % WAYS].y += t[k].y; s[k % WAYS].z += t[k].z; s[k % WAYS].w += t[k].w; }
    }
    float4 v = s[0];
#pragma unroll
    for (int w = 1; w < WAYS; ++w) { v.x += s[w].x; v.y += s[w].y; v.z += s[w].z; v.w += s[w].w; }
    store4_plus<E>(a.Y, a.resid, (size_t)a.m_base * a.d_model + (size_t)4 * idx, v);
}

// Every instantiation the launcher uses, spelled out (the host pass otherwise emitted the launch
// stub of only one element type per token-tile count).
#define DFK_INST_GATEUP(NTC)                                                  \
    template __global__ void k_gateup_big<1, BF16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<1, FP16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<2, BF16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<2, FP16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<3, BF16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<3, FP16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<4, BF16, NTC>(MlpArgs);    \
    template __global__ void k_gateup_big<4, FP16, NTC>(MlpArgs);
DFK_INST_GATEUP(1) DFK_INST_GATEUP(2) DFK_INST_GATEUP(3) DFK_INST_GATEUP(4)
DFK_INST_GATEUP(5) DFK_INST_GATEUP(6) DFK_INST_GATEUP(7) DFK_INST_GATEUP(8)
#undef DFK_INST_GATEUP
#define DFK_INST_WIDE(TT, NTC)                                       \
    template __global__ void k_gateup_wide<TT, BF16, NTC>(MlpArgs); \
    template __global__ void k_gateup_wide<TT, FP16, NTC>(MlpArgs);
DFK_INST_WIDE(2, 10) DFK_INST_WIDE(2, 12) DFK_INST_WIDE(2, 14) DFK_INST_WIDE(2, 16)
DFK_INST_WIDE(3, 10) DFK_INST_WIDE(3, 12) DFK_INST_WIDE(3, 14) DFK_INST_WIDE(4, 10)
#undef DFK_INST_WIDE
#define DFK_INST_SUM(BATCH, WAYS)                                          \
    template __global__ void k_sum_partials<BF16, BATCH, WAYS>(MlpArgs);  \
    template __global__ void k_sum_partials<FP16, BATCH, WAYS>(MlpArgs);
DFK_INST_SUM(8, 1) DFK_INST_SUM(16, 1) DFK_INST_SUM(16, 2) DFK_INST_SUM(16, 4) DFK_INST_SUM(16, 8) DFK_INST_SUM(16, 16)
#undef DFK_INST_SUM
#define DFK_INST_DOWN(TT)                                              \
    template __global__ void k_down_big<TT, BF16>(MlpArgs, int);   \
    template __global__ void k_down_big<TT, FP16>(MlpArgs, int);
DFK_INST_DOWN(1) DFK_INST_DOWN(2) DFK_INST_DOWN(3) DFK_INST_DOWN(4)
#undef DFK_INST_DOWN
#define DFK_INST_DOWN_T(TT)                                            \
    template __global__ void k_down_t_big<TT, BF16>(MlpArgs, int); \
    template __global__ void k_down_t_big<TT, FP16>(MlpArgs, int);
DFK_INST_DOWN_T(1) DFK_INST_DOWN_T(2) DFK_INST_DOWN_T(3) DFK_INST_DOWN_T(4)
#undef DFK_INST_DOWN_T

// ---------------------------------------------------------------- host side
unsigned big_groups(const MlpArgs& a) { return (unsigned)((a.m_count + a.group_tokens - 1) / a.group_tokens); }

// LDS of the kernels: activation and weight buffers, or what the two halves of the k range exchange at the end.
size_t big_lds(int x_step, int w_step, size_t end) {
    return std::max((size_t)kBigXBufs * x_step + (size_t)big_w_bufs(x_step, w_step) * w_step, end);
}
size_t big_lds_gateup_nt(int TT, int nt_max) {
    const int ks = big_gateup_pieces(TT, nt_max);
    return big_lds(ks * 4 * TT * kBigTile, ks * nt_max * kBigTile, (size_t)kBigWaves * ((nt_max + 1) / 2) * TT * 1024);
}
size_t big_lds_gateup(const dfk_config_t& c, int TT, int d_ff) { return big_lds_gateup_nt(TT, max_slice_rows(d_ff, c.splits) / 8); }
size_t big_lds_down_t(int TT) { return big_lds(4 * TT * kBigTile, 8 * kBigTile, (size_t)kBigWaves * 4 * TT * 1024); }
size_t big_lds_down(int TT) { return big_lds(4 * TT * kBigTile, 4 * kTileBytes, (size_t)kBigWaves * TT * 4 * 1024); }
constexpr bool big_buffers_fit() {
    for (int tt = 1; tt <= 4; ++tt) {
        if (big_w_bufs(4 * tt * kBigTile, 4 * kTileBytes) < 3) return false;
        for (int n = 1; n <= kBigMaxRowTiles; ++n) {
            const int ks = big_gateup_pieces(tt, n);
            if (big_w_bufs(ks * 4 * tt * kBigTile, ks * n * kBigTile) < 3) return false;
        }
        if (big_wide_tiles(tt) && big_w_bufs(4 * tt * kBigTile, big_wide_tiles(tt) * kBigTile) < 3) return false;
    }
    return true;
}
static_assert(big_buffers_fit(), "weights at least two steps ahead");

template <int TT, typename E, int NTC>
hipError_t launch_big_gateup(const MlpArgs& a, hipStream_t st) {
    static LdsAllowance allowed;   // of this instantiation, per device
    const size_t lds = big_lds_gateup_nt(TT, NTC);
    if (hipError_t e = allow_lds(allowed, (const void*)k_gateup_big<TT, E, NTC>, lds); e != hipSuccess) return e;
    hipLaunchKernelGGL((k_gateup_big<TT, E, NTC>), dim3(a.splits, big_groups(a)), dim3(kBigWaves * 64), lds, st, a);
    return hipGetLastError();
}
template <int TT, typename E, int NTC>
hipError_t launch_big_wide(const MlpArgs& a, hipStream_t st) {
    if constexpr (NTC > big_wide_tiles(TT)) {
        return hipErrorInvalidValue;
    } else {
        static LdsAllowance allowed;   // of this instantiation, per device
        const size_t lds = big_lds(4 * TT * kBigTile, NTC * kBigTile, 0);
        if (hipError_t e = allow_lds(allowed, (const void*)k_gateup_wide<TT, E, NTC>, lds); e != hipSuccess) return e;
        hipLaunchKernelGGL((k_gateup_wide<TT, E, NTC>), dim3(a.splits), dim3(kBigWaves * 64), lds, st, a);
        return hipGetLastError();
    }
}
template <int TT, typename E>
hipError_t launch_big_gateup_n(const MlpArgs& a, hipStream_t st) {
    switch (max_slice_rows(a.d_ff, a.splits) / 8) {
        case 1: return launch_big_gateup<TT, E, 1>(a, st);
        case 2: return launch_big_gateup<TT, E, 2>(a, st);
        case 3: return launch_big_gateup<TT, E, 3>(a, st);
        case 4: return launch_big_gateup<TT, E, 4>(a, st);
        case 5: return launch_big_gateup<TT, E, 5>(a, st);
        case 6: return launch_big_gateup<TT, E, 6>(a, st);
        case 7: return launch_big_gateup<TT, E, 7>(a, st);
        case 8: return launch_big_gateup<TT, E, 8>(a, st);
        case 9: case 10: return launch_big_wide<TT, E, 10>(a, st);
        case 11: case 12: return launch_big_wide<TT, E, 12>(a, st);
        case 13: case 14: return launch_big_wide<TT, E, 14>(a, st);
        case 15: case 16: return launch_big_wide<TT, E, 16>(a, st);
        default: return hipErrorInvalidValue;
    }
}

template <int TT, typename E>
hipError_t launch_big_down(const MlpArgs& a, int row, hipStream_t st) {
    static LdsAllowance allowed;   // of this instantiation, per device
    const size_t lds = big_lds_down(TT);
    const int by_xcd = (size_t)a.m_count * a.d_ff * 2 > kL2BytesPerXcd;
    if (hipError_t e = allow_lds(allowed, (const void*)k_down_big<TT, E>, lds); e != hipSuccess) return e;
    hipLaunchKernelGGL((k_down_big<TT, E>), dim3(row, big_groups(a)), dim3(kBigWaves * 64), lds, st, a, by_xcd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.reduce_mode == DFK_REDUCE_ATOMIC) return e;
    return launch_sum_partials(a, 1, st);
}

template <int TT, typename E>
hipError_t launch_down_t_te(const MlpArgs& a, int row, hipStream_t st) {
    static LdsAllowance allowed;
    const size_t lds = big_lds_down_t(TT);
    const int by_xcd = (size_t)a.m_count * a.d_ff * 2 > kL2BytesPerXcd;
    if (hipError_t e = allow_lds(allowed, (const void*)k_down_t_big<TT, E>, lds); e != hipSuccess) return e;
    hipLaunchKernelGGL((k_down_t_big<TT, E>), dim3(row, big_groups(a)), dim3(kBigWaves * 64), lds, st, a, by_xcd);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    return launch_sum_partials(a, 1, st);
}
template <typename E>
hipError_t launch_sum_e(const MlpArgs& a, int ways, hipStream_t st) {
    const unsigned n4 = (unsigned)a.m_count * (unsigned)(a.d_model / 4);
    const unsigned threads = n4 < 65536 ? 64 : 256;
    const dim3 grid((n4 + threads - 1) / threads), block(threads);
    switch (ways) {
        case 16: hipLaunchKernelGGL((k_sum_partials<E, 16, 16>), grid, block, 0, st, a); break;
        case 8: hipLaunchKernelGGL((k_sum_partials<E, 16, 8>), grid, block, 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_sum_partials<E, 16, 4>), grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_sum_partials<E, 16, 2>), grid, block, 0, st, a); break;
        default:
            if (a.k2_splits <= 8) hipLaunchKernelGGL((k_sum_partials<E, 8, 1>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((k_sum_partials<E, 16, 1>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_sum_partials(const MlpArgs& a, int ways, hipStream_t st) {
    return a.dtype == DFK_FP16 ? launch_sum_e<FP16>(a, ways, st) : launch_sum_e<BF16>(a, ways, st);
}

int mfma_big_tokens_per_launch() { return kBigTokensPerLaunch; }

size_t mfma_big_workgroups(const dfk_config_t& c, int M, int d_ff) {
    const BigLaunch up = big_gateup_launch(M, d_ff, c.splits), down = big_down_launch(M, d_ff, c.k2_splits, c.k2_col_blocks, wdt_split(c), c.reduce == DFK_REDUCE_TICKET);
    return std::max((size_t)up.splits * up.groups, (size_t)down.splits * c.k2_col_blocks * down.groups);
}

// The gate/up kernel alone with one token tile per group: up to 64 tokens per launch.  Paired with
// the down kernel of the 64-token pair for 33..64 tokens (config field kmajor = 3): with three or four token
// tiles the shared weight tiles (read from L2 once per workgroup instead of once per wavefront) pay, while the
// down kernel of this family does not yet.
hipError_t launch_big_gateup_64(const MlpArgs& a, hipStream_t st) {
    if (a.norm_w || a.m_count > 64) return hipErrorInvalidValue;
    MlpArgs b = a;
    b.group_tokens = a.m_count;
    return a.dtype == DFK_FP16 ? launch_big_gateup_n<1, FP16>(b, st) : launch_big_gateup_n<1, BF16>(b, st);
}
bool big_gateup_64_fits(const dfk_config_t& c, int d_model, int d_ff) {
    if (d_model < 128 || d_model % kKC || d_model > kMaxDModel) return false;
    if (c.depth < 3 || c.depth > 4) return false;
    if (max_slice_rows(d_ff, c.splits) / 8 > kBigMaxRowTiles) return false;
    return big_lds_gateup(c, 1, d_ff) <= (size_t)kLdsLimit;
}

bool mfma_big_config_valid(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (c.path != DFK_PATH_MFMA || (dtype != DFK_BF16 && dtype != DFK_FP16) || c.variant != DFK_VARIANT_TWO_KERNEL) return false;
    if (c.kmajor != 2 || c.k2_rows_by_wave != 0 || c.a2_dtype != (int)dtype) return false;
    if (c.reduce != DFK_REDUCE_TICKET && c.reduce != DFK_REDUCE_ATOMIC) return false;
    if ((c.waves != 4 && c.waves != 8) || c.depth < 3 || c.depth > 4) return false;   // depth = buffers of shared tiles
    if (M < 1 || d_model < 128 || d_ff < 8 || d_ff % 8 || d_model % kKC || d_model > kMaxDModel) return false;
    const int ng = d_ff / 8;
    if (c.splits < 1 || c.splits > ng || c.splits > 65535) return false;
    if (max_slice_rows(d_ff, c.splits) / 8 > kBigMaxRowTiles) return false;
    if (c.k2_splits < 1 || c.k2_splits > ng) return false;
    if (c.k2_col_blocks != d_model / 128) return false;                        // one 128-column block per workgroup
    if ((long long)c.k2_splits * c.k2_col_blocks > 65535 || c.k2_col_blocks > kTicketLevel2) return false;
    const int tokens = std::min(M, kBigTokensPerLaunch);
    if (c.reduce == DFK_REDUCE_ATOMIC && (size_t)tokens * d_model * 4 > kYaccBytes) return false;   // fp32 accumulator of one launch
    // (this pair's counter mode keeps one partial block per split and no group sums)
    if (c.reduce == DFK_REDUCE_TICKET && (size_t)c.k2_splits * tokens * d_model * 4 > partial_bytes(M, d_model)) return false;
    return big_lds_gateup(c, big_token_tiles(tokens), d_ff) <= (size_t)kLdsLimit && big_lds_down(big_token_tiles(tokens)) <= (size_t)kLdsLimit;
}

// What the pair launches: the gate/up kernel, the down kernel, the down kernel for W_down as [d_model, d_ff].
enum class BigKernel { GateUp, Down, DownT };
template <int TT, typename E>
static hipError_t launch_big_te(const MlpArgs& a, BigKernel k, int row, hipStream_t st) {
    return k == BigKernel::GateUp ? launch_big_gateup_n<TT, E>(a, st) : k == BigKernel::Down ? launch_big_down<TT, E>(a, row, st) : launch_down_t_te<TT, E>(a, row, st);
}
template <int TT>
static hipError_t launch_big_t(const MlpArgs& a, BigKernel k, int row, hipStream_t st) {
    return a.dtype == DFK_FP16 ? launch_big_te<TT, FP16>(a, k, row, st) : launch_big_te<TT, BF16>(a, k, row, st);
}
static hipError_t launch_big(const MlpArgs& args, BigKernel k, hipStream_t st) {
    MlpArgs a = args;
    const BigLaunch l = k == BigKernel::GateUp ? big_gateup_launch(a.m_count, a.d_ff, a.splits)
                                               : big_down_launch(a.m_count, a.d_ff, a.k2_splits, a.k2_col_blocks, k == BigKernel::DownT, a.reduce_mode == DFK_REDUCE_TICKET);
    (k == BigKernel::GateUp ? a.splits : a.k2_splits) = l.splits;
    a.group_tokens = l.tokens;
    switch (big_token_tiles(a.group_tokens)) {
        case 1: return launch_big_t<1>(a, k, l.row, st);
        case 2: return launch_big_t<2>(a, k, l.row, st);
        case 3: return launch_big_t<3>(a, k, l.row, st);
        case 4: return launch_big_t<4>(a, k, l.row, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_mfma_big(const MlpArgs& a, hipStream_t st) {
    if (a.norm_w) return hipErrorInvalidValue;   // the normalisation is folded into the 64-token pair only
    if (g_stage_mask & 1) {
        if (hipError_t e = launch_big(a, BigKernel::GateUp, st); e != hipSuccess) return e;
    }
    return g_stage_mask & 2 ? launch_big(a, BigKernel::Down, st) : hipSuccess;
}

// W_down as [d_model, d_ff] with the down projection split over d_ff (kmajor = 5, k2_col_blocks = d_model / 128 > 1): up to 64
// tokens the 64-token pair's gate/up kernel, which folds a normalisation, beyond them this file's; then the down kernel above.
bool mfma_wdt_split_valid(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (c.path != DFK_PATH_MFMA || (dtype != DFK_BF16 && dtype != DFK_FP16) || c.variant != DFK_VARIANT_TWO_KERNEL) return false;
    if (c.kmajor != 5 || c.k2_rows_by_wave != 0 || c.a2_dtype != (int)dtype || c.reduce != DFK_REDUCE_TICKET) return false;
    if (M < 1 || d_model < 256 || d_model % 128 || d_model > kMaxDModel || d_ff < 128 || d_ff % 128) return false;
    if (c.k2_col_blocks != d_model / 128 || c.k2_splits < 1 || c.k2_splits > d_ff / kBigStepK) return false;
    if ((long long)c.k2_splits * c.k2_col_blocks > 65535) return false;
    const int tokens = std::min(M, kBigTokensPerLaunch);
    if ((size_t)c.k2_splits * tokens * d_model * 4 > partial_bytes(M, d_model)) return false;
    dfk_config_t g = c;            // its gate/up kernel, as that kernel's own pair asks for it
    g.k2_splits = 1;
    if (M <= mfma_km_tokens_per_launch()) {
        g.kmajor = 1;
        return mfma_km_config_valid(g, M, d_model, d_ff, dtype);
    }
    if ((c.waves != 4 && c.waves != 8) || c.depth < 2 || c.depth > 16) return false;
    g.kmajor = 2; g.waves = 8; g.depth = 3;
    return mfma_big_config_valid(g, M, d_model, d_ff, dtype);
}

hipError_t launch_wdt_split(const MlpArgs& a, const dfk_config_t& c, hipStream_t st) {
    if (g_stage_mask & 1) {
        hipError_t e;
        if (a.M <= mfma_km_tokens_per_launch()) {
            dfk_config_t g = c;
            g.kmajor = 1;
            const int saved = g_stage_mask;
            g_stage_mask = 1;                          // the gate/up kernel only
            e = launch_mfma_km(a, g, st);
            g_stage_mask = saved;
        } else {
            e = a.norm_w ? hipErrorInvalidValue : launch_big(a, BigKernel::GateUp, st);
        }
        if (e != hipSuccess) return e;
    }
    return g_stage_mask & 2 ? launch_big(a, BigKernel::DownT, st) : hipSuccess;
}

}  // namespace dfk
