// Device code of the row-slab forward (the kernel and its launch are in lq_slab.hip): a workgroup takes a slab of at
// most 64 rows of one segment (32 in grouped calls and above rank 64, whose accumulators fill the registers);
//   phase 1: h = x A_a^T over all of d_in (the 8 waves take alternate 64-wide k blocks and add their results in LDS)
//   phase 2: y += s h B_a (the 8 waves take alternate 64-column blocks)
// All global accesses are row-wise 16-byte accesses (an instruction covers 8 rows x 128 contiguous bytes); data
// reaches the MFMA operand layout through slabs of LDS that belong to one wave, so the streaming loops contain no
// workgroup barrier.  Loads are issued ahead into the registers the previous block has just left, unconditionally
// and from clamped addresses, in the order they are consumed, so that the number in flight is static.
#pragma once

#include "lq_internal.h"

namespace lq {
namespace {

constexpr int kSlabRows = 64;          // rows of a unit: up to four 16-row MFMA tiles
constexpr int kKB = 64;                // k elements per block (phase 1), columns per block (phase 2)
constexpr int kPitch = kKB + 8;        // elements per slab row (16-byte aligned, bank spread)
constexpr int kChunk = 32 * kPitch;    // elements of a 32-row slab
constexpr int kSlabBig = 0x7fffffff;
constexpr int kMaxParts = 8;           // column parts a chunk of rows is cut into
constexpr size_t kWaveBytes = 16384;   // LDS of one wave: its slabs, later its share of the reduction buffer

// 16 bytes of an adapter matrix at element offset `off` (< 2^31, see slab_reaches): a wave-uniform base and a 32-bit byte offset per
// lane, the form that needs no 64-bit address arithmetic in vector registers
__device__ __forceinline__ u32x4 load_at(gconst_u16 base, unsigned int off)
{
    typedef const __attribute__((address_space(1))) char* gconst_char;
    return *reinterpret_cast<gconst_u32x4>(reinterpret_cast<gconst_char>(base) + (size_t)(off * 2u));
}

// projections a pass can hold in registers: its accumulators are NP x MTM x NT MFMA tiles (MTM: 16-row tiles
// of the kernel's tallest unit, two in groups)
template <int NT> constexpr int pass_projections() { return NT == 1 ? kMaxProj : NT == 2 ? 3 : 1; }

// =================================================================================================
// phase 1: acc[q][mt][nt] = this wave's share of x[rows] . A_q[ranks]^T for the NP projections of the pass
// (D[row][rank]: lane (c, kg) receives rows 4 kg .. + 3 of tile mt, rank c of tile nt)
// =================================================================================================
// MT: row tiles of this unit, MTM: of the kernel's tallest unit
template <int NT, int NP, int MT, int MTM, bool ZERO_X, class PP>
__device__ __forceinline__ void slab_shrink(const PP& p, const Unit&, const SegInfo (&s)[NP], const int* lds_row,
                                            u16* slab, f32x4 (&acc)[NP][MTM][NT])
{
    constexpr int NJ = 2 * MT;            // load instructions per block of x (8 rows each)
    constexpr int NA = 2 * NT;            // load instructions per block of one A (8 rank rows each)
    constexpr int NCH = (NT + 1) / 2;     // 32-rank chunks of A
    const int lane = lane_id(), w = uniform((int)threadIdx.x / kWave), c = lane & 15, kg = lane >> 4;
    const int r8 = lane >> 3, piece = lane & 7;
    u16* xs = slab;             // [32][kPitch]
    u16* as = slab + kChunk;    // [2][32][kPitch]
    const int rank = s[0].rank;

    const int nblk = (p.d_in + kKB - 1) / kKB;
    const int n_mine = w < nblk ? (nblk - w + kWaves - 1) / kWaves : 0;  // blocks w, w + 8, ...
    if (n_mine == 0) return;  // wave uniform
    // Slabs that run side by side would otherwise all sweep the same k range in step, which (with a power-of-two row
    // pitch) keeps hitting the same few channels; so the sweep starts at a block that depends on the XCD the
    // workgroup runs on (workgroups are dealt to the 8 XCDs in turn).  The slabs of one XCD keep the same order: they
    // share its L2, and slabs of one segment then find the adapter's A there instead of fetching it again.
    const int rot = (int)((((unsigned)blockIdx.x & 7u) * (unsigned)nblk) >> 3);
    auto k_of = [&](int j) {  // first k of this wave's j-th block (past the end: the last one again)
        int b = w + kWaves * min(j, n_mine - 1) + rot;
        if (b >= nblk) b -= nblk;
        return b * kKB;
    };

    const int safe_row = max(lds_row[0], 0);
    const u16* xrow[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const int r = lds_row[r8 + 8 * i];
        xrow[i] = p.x + (long long)(r >= 0 ? r : safe_row) * p.ldx + piece * 8;
    }
    unsigned int aoff[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) aoff[i] = (unsigned int)(min(r8 + 8 * i, rank - 1) * p.d_in);

    // a lane's 8 columns lie wholly inside or wholly beyond d_in; beyond, it re-reads column 0 and A counts as zero.  With
    // ZERO_X (launches above rank 32 and those of units taller than 32 rows) so does x, or an infinity in column 0 would make the
    // row's h a NaN: the zeros are the 16 bytes that pad every row of the slab.  (It costs no time there: 9000 rows of rank 16 to
    // 64, five shapes, all within 0.3 us; a rank-16 decode batch would pay up to 4 %.)
    if (ZERO_X && lane < 32) {
        constexpr u32x4 zero = {0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(xs + lane * kPitch + kKB) = zero;
    }
    static_assert(kPitch >= kKB + 8, "a row's padding holds 16 bytes");
    auto col_of = [&](int k0) { return k0 + piece * 8 < p.d_in ? k0 : -piece * 8; };
    constexpr int XS = NP >= 3 || MT >= 3 ? 1 : 2;  // register sets of x = blocks it is requested ahead (one where registers are short, or a block is 6 to 8 KB already)
    u32x4 xv[XS][NJ];
    // rows 32 half .. 32 half + 31 of a block of x: the x slab holds 32 rows, taller units go through it in two steps
    constexpr int HALVES = (MT + 1) / 2;
    auto x_load_half = [&](int j, int half, u32x4 (&v)[NJ]) {
        const int kc = col_of(k_of(j));
#pragma unroll
        for (int i = 4 * half; i < 4 * half + 4; ++i)
            if (i < NJ) v[i] = *reinterpret_cast<const u32x4*>(xrow[i] + kc);
    };
    auto x_load = [&](int j, u32x4 (&v)[NJ]) {
#pragma unroll
        for (int half = 0; half < HALVES; ++half) x_load_half(j, half, v);
    };
    // The A stream: a block's A is NC chunks (projection q, 32 ranks ch), four load instructions each; chunk n of
    // block j is number j NC + n of the stream, lives in register set (j NC + n) % 2 and goes through LDS buffer
    // (j NC + n) % 2.  A set is refilled with the chunk two further on as soon as it has been written to LDS.
    constexpr int NC = NP * NCH;
    constexpr int NL = NA < 4 ? NA : 4;  // load instructions per chunk
    u32x4 av[2][NL];
    auto a_load = [&](int j, auto chunk, u32x4 (&v)[NL]) {
        constexpr int N = decltype(chunk)::value;  // chunk N of block j (N may run past NC: the blocks further on)
        constexpr int q = (N % NC) / NCH, ch = (N % NC) % NCH;
        const unsigned int kc = (unsigned int)(col_of(k_of(j + N / NC)) + piece * 8);  // >= 0
#pragma unroll
        for (int i2 = 0; i2 < NL; ++i2) v[i2] = load_at(s[q].A, aoff[ch * 4 + i2] + kc);
    };
    // (loads return in order, so they are issued in the order they are consumed, and the scheduler is kept from
    // reordering them: a wait for the oldest then leaves all younger ones in flight)
    x_load(0, xv[0]);
    __builtin_amdgcn_sched_barrier(0);
    a_load(0, std::integral_constant<int, 0>{}, av[0]);
    __builtin_amdgcn_sched_barrier(0);
    a_load(0, std::integral_constant<int, 1>{}, av[1]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (XS == 2) x_load(1, xv[1]);
    __builtin_amdgcn_sched_barrier(0);

    auto block = [&](int j, auto slot) {
        constexpr int J = decltype(slot)::value;
        // x of block j: registers -> slab -> fragments; the registers take block j + XS
        int at[2];  // columns beyond d_in are read from the slab's padding
#pragma unroll
        for (int h = 0; h < 2; ++h) at[h] = !ZERO_X || k_of(j) + 32 * h + kg * 8 < p.d_in ? 32 * h + kg * 8 : kKB;
        u32x4 xf[MT][2];
#pragma unroll
        for (int half = 0; half < HALVES; ++half) {
            if (half > 0) wave_sync();  // the first half's fragments have been read
#pragma unroll
            for (int i = 4 * half; i < 4 * half + 4; ++i)
                if (i < NJ) *reinterpret_cast<u32x4*>(xs + (r8 + 8 * (i & 3)) * kPitch + piece * 8) = xv[J % XS][i];
            x_load_half(j + XS, half, xv[J % XS]);
            __builtin_amdgcn_sched_barrier(0);
            wave_sync();
#pragma unroll
            for (int mt = 2 * half; mt < 2 * half + 2; ++mt)
                if (mt < MT)
#pragma unroll
                    for (int h = 0; h < 2; ++h) xf[mt][h] = *reinterpret_cast<const u32x4*>(xs + ((mt & 1) * 16 + c) * kPitch + at[h]);
        }
        const bool in_cur = k_of(j) + piece * 8 < p.d_in;
        auto chunk = [&](auto index) {
            constexpr int N = decltype(index)::value;
            constexpr int q = N / NCH, ch = N % NCH, S = (J * NC + N) & 1;
            u16* buf = as + S * kChunk;
#pragma unroll
            for (int i2 = 0; i2 < NL; ++i2) {
                constexpr u32x4 zero = {0u, 0u, 0u, 0u};
                const bool live = in_cur && r8 + 8 * (ch * 4 + i2) < rank;
                *reinterpret_cast<u32x4*>(buf + (r8 + 8 * i2) * kPitch + piece * 8) = live ? av[S][i2] : zero;
            }
            a_load(j, std::integral_constant<int, N + 2>{}, av[S]);
            __builtin_amdgcn_sched_barrier(0);
            wave_sync();
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                constexpr int dummy = 0;
                const int nt = ch * 2 + t < NT ? ch * 2 + t : dummy;  // (keeps the dead branch's index inside the array)
                if (ch * 2 + t < NT) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const u32x4 af = *reinterpret_cast<const u32x4*>(buf + (t * 16 + c) * kPitch + 32 * h + kg * 8);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[q][mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xf[mt][h]), as_bf16x8(af),
                                                                                     acc[q][mt][nt], 0, 0, 0);
                    }
                }
            }
        };
        // (a buffer is rewritten two chunks later, behind the wave_sync of the chunk in between; with a single
        // chunk per block, behind the one at the end of the block)
        chunk(std::integral_constant<int, 0>{});
        if constexpr (NC > 1) chunk(std::integral_constant<int, 1>{});
        if constexpr (NC > 2) chunk(std::integral_constant<int, 2>{});
        if constexpr (NC > 3) chunk(std::integral_constant<int, 3>{});
        static_assert(NC <= 4, "the chunks of a block are listed by name");
        wave_sync();  // the x slab is rewritten by the next block
    };
    // (pairs of blocks with a single exit: the accumulators stay where they are across the loop.  An odd last block runs alone:
    // padding it to a pair, with zeros for A, made the h of a row with an infinity there a NaN, and cost 1 to 2 %)
    int j = 0;
    for (; j + 1 < n_mine; j += 2) {
        block(j, std::integral_constant<int, 0>{});
        block(j + 1, std::integral_constant<int, 1>{});
    }
    if (j < n_mine) block(j, std::integral_constant<int, 0>{});
}

// =================================================================================================
// phase 2 for one projection: y[rows][columns of the part] += (scaled h, as bf16 high + low fragments) . B
// D[column][row] with the columns of two MFMA tiles interleaved, so that a lane ends up with 4 consecutive
// columns of a row; every 16-row tile of products makes a round trip through the wave's 4 KB slab to reach the
// row-wise layout y is accessed in.
// =================================================================================================
template <int NT, int MT, bool STREAM, class PP>  // STREAM: y is large, see load_once
__device__ __forceinline__ void slab_expand(const PP&, const Unit& u, const SegInfo& s, const Proj& pj,
                                            const int* lds_row, const u32x4* hf, u16* bs, float* ds, int blk_begin,
                                            int blk_end)
{
    constexpr int NJ = 2 * MT;
    constexpr int NB = 2 * NT;
    constexpr int KSTEPS = (NT + 1) / 2;
    const int lane = lane_id(), w = uniform((int)threadIdx.x / kWave), c = lane & 15, g = lane >> 4;
    const int r8 = lane >> 3, piece = lane & 7;
    const int nblk = blk_end - blk_begin;
    const int n_mine = w < nblk ? (nblk - w + kWaves - 1) / kWaves : 0;
    if (n_mine == 0) return;  // wave uniform
    const int rot = (int)((((unsigned)blockIdx.x & 7u) * (unsigned)nblk) >> 3);  // as in phase 1: one order per XCD
    auto n_of = [&](int j) {  // first column of this wave's j-th block (past the end: the last one again)
        int b = w + kWaves * min(j, n_mine - 1) + rot;
        if (b >= nblk) b -= nblk;
        return (blk_begin + b) * kKB;
    };
    const int safe_row = max(lds_row[0], 0);
    int row[NJ];
    u16* yrow[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        row[i] = lds_row[r8 + 8 * i];
        yrow[i] = pj.y + (long long)(row[i] >= 0 ? row[i] : safe_row) * pj.ldy;
    }
    unsigned int boff[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) boff[i] = (unsigned int)(min(r8 + 8 * i, s.rank - 1) * pj.d_out);

    // The B stream: a block's B is KSTEPS chunks of 32 rank rows, four load instructions each; chunk ks of block j is
    // number j KSTEPS + ks of the stream and lives in register set (j KSTEPS + ks) % 2; a set is refilled with the
    // chunk two further on as soon as it has been written to LDS.
    constexpr int NL = NB < 4 ? NB : 4;  // load instructions per chunk
    u32x4 yv[2][NJ], bv[2][NL];
    auto y_load = [&](int j, u32x4 (&v)[NJ]) {
        const int n_ld = min(n_of(j) + 8 * piece, pj.d_out - 8);
#pragma unroll
        for (int i = 0; i < NJ; ++i) v[i] = load_once<STREAM>(yrow[i] + n_ld);
    };
    auto b_load = [&](int j, auto chunk, u32x4 (&v)[NL]) {
        constexpr int N = decltype(chunk)::value;
        const unsigned int n_ld = (unsigned int)min(n_of(j + N / KSTEPS) + 8 * piece, pj.d_out - 8);
#pragma unroll
        for (int i2 = 0; i2 < NL; ++i2) v[i2] = load_at(s.B, boff[(N % KSTEPS) * 4 + i2] + n_ld);
    };
    // (issued in the order they are consumed, see phase 1; with KSTEPS > 1 both chunks belong to block 0)
    b_load(0, std::integral_constant<int, 0>{}, bv[0]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (KSTEPS == 1) {
        y_load(0, yv[0]);
        __builtin_amdgcn_sched_barrier(0);
        b_load(0, std::integral_constant<int, 1>{}, bv[1]);
    } else {
        b_load(0, std::integral_constant<int, 1>{}, bv[1]);
        __builtin_amdgcn_sched_barrier(0);
        y_load(0, yv[0]);
    }
    __builtin_amdgcn_sched_barrier(0);
    y_load(1, yv[1]);
    __builtin_amdgcn_sched_barrier(0);

    // (live: false for the block that pads an odd count to the pair the loop below runs; it stores nothing)
    auto block = [&](int j, auto slot, bool live_block) {
        constexpr int J = decltype(slot)::value;
        const int n_c = n_of(j) + 8 * piece;
        // B of block j, 32 ranks at a time: registers -> slab -> transposed fragments
        u32x4 bfrag[2][2][KSTEPS];
        auto chunk = [&](auto index) {
            constexpr int ks = decltype(index)::value, S = (J * KSTEPS + ks) & 1;
#pragma unroll
            for (int i2 = 0; i2 < 4; ++i2) {
                constexpr u32x4 zero = {0u, 0u, 0u, 0u};
                u32x4 v = zero;  // rank rows beyond the adapter's (and beyond the tiles of this launch) are zero
                if (i2 < NL && r8 + 8 * (ks * 4 + i2) < s.rank) v = bv[S][i2 < NL ? i2 : 0];
                *reinterpret_cast<u32x4*>(bs + (r8 + 8 * i2) * kPitch + piece * 8) = v;
            }
            b_load(j, std::integral_constant<int, ks + 2>{}, bv[S]);
            __builtin_amdgcn_sched_barrier(0);
            wave_sync();
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    // lane c: column 32 q + 8 (c / 4) + 4 m + c % 4 of the block, rank rows 32 ks + 8 g .. + 7
                    bfrag[q][m][ks] = lds_read_transposed_16x32(bs + 32 * q + 4 * m, kPitch, 8);
            wave_sync();  // the slab is rewritten by the next chunk
        };
        chunk(std::integral_constant<int, 0>{});
        if constexpr (KSTEPS > 1) chunk(std::integral_constant<int, 1>{});
        if constexpr (KSTEPS > 2) chunk(std::integral_constant<int, 2>{});
        if constexpr (KSTEPS > 3) chunk(std::integral_constant<int, 3>{});
        static_assert(KSTEPS <= 4, "the chunks of a block are listed by name");
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            u32x4 h_hi[KSTEPS], h_lo[KSTEPS];
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                h_hi[ks] = hf[((t * KSTEPS + ks) * 2 + 0) * kWave + lane];
                h_lo[ks] = hf[((t * KSTEPS + ks) * 2 + 1) * kWave + lane];
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KSTEPS; ++ks) {
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bfrag[q][m][ks]), as_bf16x8(h_lo[ks]), d, 0, 0, 0);
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bfrag[q][m][ks]), as_bf16x8(h_hi[ks]), d, 0, 0, 0);
                    }
                    // row c of the tile, columns 32 q + 8 g + 4 m .. + 3 = 16-byte chunk 8 q + 2 g + m (swizzled with the row)
                    *reinterpret_cast<f32x4*>(ds + c * 64 + (((8 * q + 2 * g + m) ^ c) & 15) * 4) = d;
                }
            wave_sync();
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int i = 2 * t + jj, rt = 8 * jj + r8;  // load instruction i of the block = row rt of tile t
                const f32x4 d0 = *reinterpret_cast<const f32x4*>(ds + rt * 64 + (((2 * piece) ^ rt) & 15) * 4);
                const f32x4 d1 = *reinterpret_cast<const f32x4*>(ds + rt * 64 + (((2 * piece + 1) ^ rt) & 15) * 4);
                if (live_block && row[i] >= 0 && t * 16 + rt < u.len && n_c < pj.d_out) {
                    float yf[8];
                    unpack8(yv[J][i], yf);
                    u32x4 o;
                    o.x = pack_bf16x2(yf[0] + d0[0], yf[1] + d0[1]);
                    o.y = pack_bf16x2(yf[2] + d0[2], yf[3] + d0[3]);
                    o.z = pack_bf16x2(yf[4] + d1[0], yf[5] + d1[1]);
                    o.w = pack_bf16x2(yf[6] + d1[2], yf[7] + d1[3]);
                    store_once<STREAM>(pj.y + (long long)row[i] * pj.ldy + n_c, o);
                }
            }
            wave_sync();  // the slab is rewritten by the next tile
        }
        __builtin_amdgcn_sched_barrier(0);
        y_load(j + 2, yv[J]);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int j = 0; j < n_mine; j += 2) {
        block(j, std::integral_constant<int, 0>{}, true);
        block(j + 1, std::integral_constant<int, 1>{}, j + 1 < n_mine);
    }
}


// =================================================================================================
// phase 1 of one pass and the sum over the 8 waves in a fixed order: every wave parks its accumulators in its own
// share of the LDS ([register][lane]); after one barrier the 512 threads share the (register, lane) values, add the
// eight partial sums as a balanced tree and hand every live element to emit(projection q of the pass (as an
// integral constant), row i of the unit, rank j, sum).  work: kWaves x kWaveBytes of LDS.  Ends without a barrier.
// =================================================================================================
template <int NT, int NP, int MTM, bool ZERO_X, class PP, class Emit>
__device__ __forceinline__ void slab_shrink_sum(const PP& p, const Unit& u0, const SegInfo (&s)[NP], const int* lds_row,
                                                unsigned char* work, Emit&& emit)
{
    constexpr int REGS = NP * MTM * NT * 4;  // accumulator registers of a wave
    static_assert((size_t)REGS * kWave * sizeof(float) <= kWaveBytes, "a wave's accumulators fit its share of the LDS");
    static_assert((size_t)3 * kChunk * sizeof(u16) <= kWaveBytes, "a wave's slabs fit its share of the LDS");
    const int lane = lane_id(), w = uniform((int)threadIdx.x / kWave);
    const int rank = s[0].rank;
    f32x4 acc[NP][MTM][NT];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int mt = 0; mt < MTM; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[q][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    u16* slab = reinterpret_cast<u16*>(work + (size_t)w * kWaveBytes);
    if (u0.len <= 16) slab_shrink<NT, NP, 1, MTM, ZERO_X>(p, u0, s, lds_row, slab, acc);  // workgroup uniform
    else if (MTM <= 2 || u0.len <= 32) slab_shrink<NT, NP, 2, MTM, ZERO_X>(p, u0, s, lds_row, slab, acc);
    else if (u0.len <= 48) slab_shrink<NT, NP, (MTM > 2 ? 3 : 2), MTM, ZERO_X>(p, u0, s, lds_row, slab, acc);
    else slab_shrink<NT, NP, (MTM > 2 ? 4 : 2), MTM, ZERO_X>(p, u0, s, lds_row, slab, acc);
    {
        float* mine = reinterpret_cast<float*>(slab) + lane;
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int mt = 0; mt < MTM; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) mine[(((q * MTM + mt) * NT + nt) * 4 + v) * kWave] = acc[q][mt][nt][v];
    }
    __syncthreads();
    // thread (wave w, lane) takes register 8 it + w of lane `lane`: NP * NT * MTM / 2 iterations, PQ of them per projection
    constexpr int PQ = NT * MTM / 2;
    auto one = [&](auto index) {
        constexpr int it = decltype(index)::value;
        constexpr int PER_WAVE = (int)(kWaveBytes / sizeof(float));
        constexpr int q = it / PQ;
        const int r = 8 * (it % PQ) + w;  // register within the projection: (mt * NT + nt) * 4 + v
        const int v = r & 3, nt = (r >> 2) % NT, mt = (r >> 2) / NT;
        const float* at = reinterpret_cast<const float*>(work) + (q * MTM * NT * 4 + r) * kWave + lane;
        float t[kWaves];
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) t[ww] = at[ww * PER_WAVE];
        const float sum = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        const int i = mt * 16 + (lane >> 4) * 4 + v, j = nt * 16 + (lane & 15);
        if (i < u0.len && j < rank) emit(std::integral_constant<int, q>{}, i, j, sum);
    };
    static_assert(NP * PQ <= 8, "the iterations are listed by name");
    one(std::integral_constant<int, 0>{});
    if constexpr (NP * PQ > 1) one(std::integral_constant<int, 1>{});
    if constexpr (NP * PQ > 2) one(std::integral_constant<int, 2>{});
    if constexpr (NP * PQ > 3) one(std::integral_constant<int, 3>{});
    if constexpr (NP * PQ > 4) one(std::integral_constant<int, 4>{});
    if constexpr (NP * PQ > 5) one(std::integral_constant<int, 5>{});
    if constexpr (NP * PQ > 6) one(std::integral_constant<int, 6>{});
    if constexpr (NP * PQ > 7) one(std::integral_constant<int, 7>{});
}

// the unit's row indices (rows[0 .. 64): -1 beyond the unit and for an invalid table entry) and, behind them, the
// rows' scales: the adapter's, or the tokens' own (dynamic scaling, Section 3.3).  The caller adds the barrier.
template <class PP>
__device__ __forceinline__ void slab_unit_rows(const PP& p, const Unit& u, const SegInfo& s0, int* rows)
{
    if ((int)threadIdx.x < kSlabRows) {
        const int i = (int)threadIdx.x;
        const int row = i < u.len ? row_of(p, u.pos + i) : -1;
        rows[i] = row;
        reinterpret_cast<float*>(rows + kSlabRows)[i] = p.token_scales ? p.token_scales[max(row, 0)] : s0.scale;
    }
}

__device__ __forceinline__ void store_frag(u16* frag, long long at, float v)
{
    unsigned int hi, lo;
    split_value(v, hi, lo);
    frag[at] = (u16)hi;
    frag[at + kWave * 8] = (u16)lo;
}

// Backward: the unit's rows of the saved h as operands of the weight gradients, with their own scales where the call has
// them.  One thread per (row, rank); run by the waves as they leave phase 2.
template <class PP>
__device__ __forceinline__ void slab_frag_h(const PP& p, const Unit& u, int rank, const float* lds_scale)
{
    if (!p.frag.dB_ptrs || !p.frag.dB_ptrs[u.ad]) return;  // no dB wanted: the caller need not keep that adapter's h
    const float* src = p.frag.h_saved + p.h_offsets[u.seg] + (long long)(u.pos - u.first) * rank;
    const int n = u.len * rank;
    for (int e0 = (int)threadIdx.x; e0 < n; e0 += 4 * kThreads) {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = src[min(e0 + k * kThreads, n - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = e0 + k * kThreads;
            if (e >= n) break;
            const int i = small_div(e, rank), j = e - i * rank;
            store_frag(p.frag.h, frag_at(u.pos + i, j, p.frag.tiles), p.token_scales ? v[k] * lds_scale[i] : v[k]);
        }
    }
}

// the adapters of the pass's projections; false (workgroup uniform, error bit set) if one of them is unusable
template <int NP, class PP>
__device__ __forceinline__ bool slab_adapters(const PP& p, const Unit& u0, const SegInfo& s0, int pi0, SegInfo (&s)[NP])
{
    bool ok = true;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        if (pi0 + q == 0) {
            s[q] = s0;
        } else {
            Unit uq = u0;
            uq.pi = pi0 + q;
            s[q] = load_adapter(p, uq);
        }
        ok = ok && s[q].ok;
    }
    return ok;
}

// How the batch is cut into units: every segment into even chunks of rows, and, where the chunks are few, every chunk into
// column parts (each part repeats phase 1 and takes its share of the columns in phase 2).
//   Chunks of at most 16 rows where they fit one round of the grid, in as many parts (up to kMaxParts) as fit too.
//   Else the smallest chunks, up to `most` rows, that fit one round, or, for longer batches, as few rounds as `most` rows
// take.  A unit costs what its compute unit has to pull: its rows and its adapter's matrices.  So that the units end
// together, a segment of lower rank than the launch's gets more rows per chunk, for 0.8 of the bytes that its matrices are
// smaller by: 8192 rows of ranks 8 to 64 in Zipf lengths, 4096 -> 11008 124 us with equal rows, 118 / 115 / 111 us with 0.25,
// 0.5 and 0.8 of the difference, 11008 -> 4096 101, 95, 89, 89 us; equal ranks are not touched.
//   Wide layers get taller chunks in column parts: n parts of n times as tall chunks re-read a part of B per unit instead of
// all of it, but x once per part; n^2 = rank x columns x grid / (rows x d_in) would balance the two, 0.3 of that is what
// measures best, and only where B is large (from 300000 elements) and n at least twice what there is room for with 16-row
// chunks: 3000 rows, us without and with: rank 64, 2048 -> 28672 148 and 113, 4096 -> 14336 86 and 72 to 75, rank 32,
// 2048 -> 28672 110 and 99, 4096 -> 11008 53 and 50; smaller B lose, 4096 -> 4096, 2500 rows of rank 32, 20.3 and 22 to 26, 1024 ->
// 4096, 1500 rows of rank 64, 17.5 and 20 to 22, and so does one row more than 16 (4096 -> 14336, 700 rows of rank 64, 31.5 and 35).
struct SlabPlan {
    ClassScan cc;  // chunks of the cached segments (prefix sums), of all segments (total)
    int per;       // rows per chunk of the segments beyond the cached ones
    int parts;
};

// (The kernel's start is bound by the instructions it runs once, from a cold instruction cache: so the usual case, 16-row
// chunks, comes first and needs no division.)
template <class PP>
__device__ __forceinline__ SlabPlan slab_plan(const PP& p, const Segs<PP>& sg, int most)
{
    SlabPlan pl;
    ClassScan& cc = pl.cc;
    const int grid = (int)gridDim.x;
    static_assert(kCachedBatches == 2, "the batches are handled by name");
    const bool second = sg.n_seg > kWave;  // wave uniform: most batches have at most 64 segments
    const int len0 = (p.kinds >> sg.c[0].kd) & 1 ? sg.c[0].en - sg.c[0].st : 0;
    const int len1 = (p.kinds >> sg.c[1].kd) & 1 ? sg.c[1].en - sg.c[1].st : 0;
    auto scan = [&](int nch0, int nch1) {
        cc.nch[0] = nch0;
        cc.incl[0] = wave_inclusive_scan(nch0);
        cc.tot0 = lane_value(cc.incl[0], kWave - 1);
        cc.nch[1] = cc.incl[1] = 0;
        if (second) {
            cc.nch[1] = nch1;
            cc.incl[1] = wave_inclusive_scan(nch1);
        }
        cc.total = cc.tot_cached = cc.tot0 + lane_value(cc.incl[1], kWave - 1);
    };
    // column parts there is room for (the parts go by the count padded to the 8 XCDs, see slab_kernel.  By the chunks themselves,
    // 36 of them in 7 parts were 280 ids for a grid of 256: a second round for a few units.  4096 -> 2 x 11008, 512 rows of rank
    // 16 in 12 segments: 35.2 -> 22.7 us.)
    auto parts_for = [&](int n) {
        return 2 * n <= grid ? min(kMaxParts, max(1, (int)((float)grid * __builtin_amdgcn_rcpf((float)(max(n, 1) + 7 & ~7)) + 0.001f))) : 1;
    };
    pl.per = 16;
    scan((len0 + 15) >> 4, (len1 + 15) >> 4);
    pl.parts = parts_for(cc.total);
    if (cc.total <= grid && sg.n_seg <= kCachedBatches * kWave && !(p.slab_parts > 0.f && 2 * pl.parts <= kMaxParts)) return pl;

    int w = 16, bonus0 = 0, bonus1 = 0;
    auto chunks = [&](int len, int rows) {
        const int per = min(most, max(16, rows));
        return small_div(len + per - 1, per);
    };
    auto count = [&](int w) { return wave_sum(chunks(len0, w + bonus0) + (second ? chunks(len1, w + bonus1) : 0)); };
    if (sg.n_seg <= kCachedBatches * kWave) {
        const int live = wave_sum(len0 + len1);
        int parts = 1;
        while (parts < kMaxParts && ((float)parts + 0.5f) * ((float)parts + 0.5f) * (float)live < p.slab_parts) ++parts;
        if (cc.total <= grid && parts < 2 * pl.parts) return pl;
        const int n_live = (int)__popcll(__ballot(len0 > 0)) + (int)__popcll(__ballot(len1 > 0));
        int target = grid;
        if (parts > 1 || live > (grid - n_live) * most) {  // (sum of ceil(len / most) <= live / most + segments)
            const int n_most = count(most);
            while (parts > 1 && ((n_most + 7) >> 3) * 8 * parts > grid) --parts;
            target = parts > 1 ? small_div(grid, 8 * parts) * 8 : max(1, small_div(n_most + grid - 1, grid)) * grid;
        }
        auto bonus_of = [&](int ad) {
            const int lo = __shfl(sg.a[0].rank, ad & (kWave - 1), kWave), hi = __shfl(sg.a[1].rank, ad & (kWave - 1), kWave);
            const int rank = ad >= 0 && ad < kWave ? lo : ad >= kWave && ad < 2 * kWave ? hi : p.max_rank;
            return (int)((float)(p.max_rank - min(max(rank, 0), p.max_rank)) * p.slab_rows_per_rank);
        };
        int spread = 0;
        if (__any(sg.a[0].rank < p.max_rank || sg.a[1].rank < p.max_rank)) {  // (lanes beyond the adapters repeat the last one)
            const int b0 = bonus_of(sg.c[0].ad), b1 = second ? bonus_of(sg.c[1].ad) : 0;
            // only where the batch's own adapters differ: a table may hold others
            const unsigned long long in0 = __ballot(len0 > 0), in1 = __ballot(len1 > 0);
            const int some = in0 ? lane_value(b0, uniform(__ffsll((long long)in0) - 1)) : lane_value(b1, uniform(__ffsll((long long)(in1 | 1ull << 63)) - 1));
            if (__any((len0 > 0 && b0 != some) || (len1 > 0 && b1 != some))) {
                bonus0 = b0;
                bonus1 = b1;
                spread = (int)((float)p.max_rank * p.slab_rows_per_rank);
            }
        }
        // the smallest w with at most `target` chunks: of max(16, w + bonus) rows, at most `most`
        int lo = small_div(live, target) - 1 - spread;  // too many: sum of ceil(len / per) >= live / per
        int hi = target > n_live ? min(most, max(16, small_div(live, target - n_live) + 1)) : most;  // few enough: <= live / per + segments
        // (equal ranks in the batch: hi itself.  The smallest w fits more, shorter units into the round, each with its own A and B to
        // read: 4000 Zipf rows of rank 16 in 110 segments, 4096 -> 4096, 27.6 us instead of 24.9.  From 33 to 48 rows it takes a row tile
        // less more often than not: 46 calls of equal or Zipf lengths 0.99 on average, 0.89 to 1.02, beyond 1.00 with equal lengths, 0.96 to 1.05)
        const bool smallest = spread > 0 || (hi > 32 && hi <= 48);
        while (smallest && hi - lo > 1) {
            const int mid = lo + ((hi - lo) >> 1);
            if (count(mid) > target) lo = mid;
            else hi = mid;
        }
        w = hi;
    } else {
        // (the segments beyond the cached ones are not counted: every segment is charged a whole chunk more than its rows make)
        const int live = min(max(uniform(p.seg_starts[sg.n_seg]), 0), p.n_tokens), slots = grid - sg.n_seg;
        w = slots > 0 ? min(most, max(16, small_div(live + slots - 1, slots))) : most;
    }
    pl.per = w;
    scan(chunks(len0, w + bonus0), chunks(len1, w + bonus1));
    const LenClass all{1, kSlabBig, p.kinds, true};
    for (int s0 = kCachedBatches * kWave; s0 < sg.n_seg; s0 += kWave) {
        const SegLane c = load_seg_lane(p, sg.n_seg, s0 + lane_id());
        cc.total += wave_sum(chunks_in(c.en - c.st, c.kd, w, all));
    }
    pl.parts = parts_for(cc.total);
    return pl;
}

// the id-th unit and its adapter; false (and the error bit set) if the segment is unusable
template <class PP>
__device__ __forceinline__ bool slab_find(const PP& p, const Segs<PP>& sg, const ClassScan& cc, int per, int id, Unit& u, SegInfo& s)
{
    if (id >= cc.tot_cached) return find_unit(p, sg, cc, id, per, LenClass{1, kSlabBig, p.kinds, true}, u, s);
    const bool hi = id >= cc.tot0;  // wave uniform
    const int base = hi ? cc.tot0 : 0;
    const int incl = hi ? cc.incl[1] : cc.incl[0], nch = hi ? cc.nch[1] : cc.nch[0];
    const SegLane& c = hi ? sg.c[1] : sg.c[0];
    const int l = uniform(__ffsll((long long)__ballot(base + incl > id)) - 1);
    const int n = lane_value(nch, l), local = id - base - (lane_value(incl, l) - n);
    u.seg = (hi ? kWave : 0) + l;
    u.first = lane_value(c.st, l);
    u.seg_len = lane_value(c.en, l) - u.first;
    const int each = small_div(u.seg_len + n - 1, n);
    u.pos = u.first + local * each;
    u.len = min(each, u.seg_len - local * each);
    u.ad = lane_value(c.ad, l);
    u.kd = lane_value(c.kd, l);
    s = cached_adapter(p, sg, u);
    return s.ok;
}

// While a unit runs, the tables and chunk counts that every wave holds in registers (one segment and one adapter per
// lane) wait in LDS: the unit needs the registers, the search for the next unit needs the tables.  All waves hold
// the same values; wave 0 writes them, a workgroup barrier later every wave reads them back.
constexpr int kStashInts = 24;
constexpr size_t kStashBytes = (size_t)kStashInts * kWave * sizeof(int);
template <class PP>
__device__ __forceinline__ void stash_tables(const Segs<PP>& sg, const ClassScan& cc, int* stash_base)
{
    if ((int)threadIdx.x >= kWave) return;
    int* stash = stash_base + lane_id();
#pragma unroll
    for (int b = 0; b < kCachedBatches; ++b) {
        int* at = stash + b * 12 * kWave;
        at[0 * kWave] = sg.c[b].st; at[1 * kWave] = sg.c[b].en; at[2 * kWave] = sg.c[b].ad; at[3 * kWave] = sg.c[b].kd;
        at[4 * kWave] = (int)sg.a[b].a_lo; at[5 * kWave] = (int)sg.a[b].a_hi;
        at[6 * kWave] = (int)sg.a[b].b_lo; at[7 * kWave] = (int)sg.a[b].b_hi;
        at[8 * kWave] = sg.a[b].rank; at[9 * kWave] = __float_as_int(sg.a[b].scale);
        at[10 * kWave] = cc.nch[b]; at[11 * kWave] = cc.incl[b];
    }
}
template <class PP>
__device__ __forceinline__ void unstash_tables(Segs<PP>& sg, ClassScan& cc, const int* stash_base)
{
    const int* stash = stash_base + lane_id();
#pragma unroll
    for (int b = 0; b < kCachedBatches; ++b) {
        const int* at = stash + b * 12 * kWave;
        sg.c[b].st = at[0 * kWave]; sg.c[b].en = at[1 * kWave]; sg.c[b].ad = at[2 * kWave]; sg.c[b].kd = at[3 * kWave];
        sg.a[b].a_lo = (unsigned int)at[4 * kWave]; sg.a[b].a_hi = (unsigned int)at[5 * kWave];
        sg.a[b].b_lo = (unsigned int)at[6 * kWave]; sg.a[b].b_hi = (unsigned int)at[7 * kWave];
        sg.a[b].rank = at[8 * kWave]; sg.a[b].scale = __int_as_float(at[9 * kWave]);
        cc.nch[b] = at[10 * kWave]; cc.incl[b] = at[11 * kWave];
    }
}

}  // namespace
}  // namespace lq
