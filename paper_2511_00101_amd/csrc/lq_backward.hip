// Backward of the segmented LoRA update for fine-tune segments.  The paper leaves this to autograd, one
// call per LoRA linear, and names a dedicated kernel as future work (Section 4.2, Appendix A); this is
// the exact gradient of the forward defined in lqlora.h, with g = dy B^T:
//     dx += s g A            dB += s h^T dy            dA += s g^T x
// g = dy B^T is the forward's shrink with the roles (x, A, d_in) := (dy, B, d_out), and dx += s g A is
// the forward's expand with (y, B, d_out) := (dx, A, d_in); both reuse those kernels, restricted to
// fine-tune segments.  The two weight gradients are contractions over the TOKEN axis, which is the
// strided axis of every operand, so they get a kernel of their own:
//   (Small and medium batches behind the slab kernel run in units of whole segments instead, without a reduction: see
//   whole_unit and whole_segments_win.)
//   weight-gradient unit : 512 rows of a fine-tune segment x 256 columns of dy (for dB, with h) or of x
//                          (for dA, with g).  32 rows at a time are staged in LDS with coalesced loads
//                          (four steps in flight in registers, two LDS buffers) and read back
//                          transposed into 16x16x32 bf16 MFMA fragments; h and g are split into bf16
//                          high and low parts.  A segment of up to 512 rows is one unit per column block,
//                          which adds its [rank x 256] result straight into dA / dB; a longer segment is
//                          cut into row chunks whose units store their partials to the workspace.
//   reduce unit          : one cut segment x 512 columns x 8 ranks: adds the segment's partials in chunk
//                          order, applies the scale and accumulates into dA / dB.  Fixed order, so
//                          reproducible.
// (Tried: the unit that stores the last partial of a (segment, column block) adds the partials up, so that no
// reduction launch is needed.  The partials then have to be stored and read with device-scope accesses, and
// every unit ends with a wait for its stores, an arrival and, for the last one, a round of loads: the
// weight-gradient launch went from 28 to 44 us on the layer stack, against 8 us for the reduction launch.)
#include "lq_internal.h"
#include <hip/amd_detail/amd_hip_unsafe_atomics.h>
#include <type_traits>
#include <utility>

namespace lq {
namespace {

constexpr int kWgRows = 512;    // token rows per weight-gradient unit (where those are more than a round of the grid: twice as many)
constexpr int kWgCols = 256;    // columns per unit (8 waves x 32)
constexpr int kWgTiles = kWgCols / (8 * 16);  // 16-column MFMA tiles per wave

constexpr int kStepRows = 32;   // token rows per MFMA k step
constexpr int kBig = 0x7fffffff;

struct BwdParams {
    const u16* x; long long ldx;
    const u16* dy; long long lddy;
    int d_in, d_out;
    float* const* dA_ptrs; float* const* dB_ptrs;
    const void* const* A_ptrs; const void* const* B_ptrs;  // only for the table helpers
    const int32_t* ranks; const float* scales; int n_adapters; int max_rank;
    const float* token_scales;  // per token row; when given it replaces scales[adapter] and moves inside the sums over tokens
    const int32_t* perm; int n_tokens;
    const int32_t* seg_starts; const int32_t* seg_adapter; const uint8_t* seg_kind;
    const int32_t* n_segments; int max_segments;
    const float* h_saved; const long long* h_offsets;
    const float* g;      // g = dy B^T of the fine-tune rows, laid out like h_saved
    int rstride;
    const u16* frag_g; const u16* frag_h;  // g and h as MFMA operands (see frag_at); frag_tiles 16-rank tiles per step
    int frag_tiles;
    int wg_slots;        // > 0: units of 1024 rows where those of 512 rows are more than wg_slots, see unit_rows
    float* wpart;        // [chunk of a segment with more than wg_rows rows][rstride][d_out + d_in] partial weight gradients
    int* err;
};

template <int NT, int ROWS = kWgRows>
struct WgCfg {
    static constexpr int YPITCH = kWgCols + 8;                 // u16 elements per staged activation row
    static constexpr int HPITCH = 16 * NT + 8;                 // u16 elements per staged row of h / g (high or low parts)
    static constexpr size_t Y_BYTES = (size_t)kStepRows * YPITCH * sizeof(u16);
    static constexpr size_t H_BYTES = ((size_t)2 * kStepRows * HPITCH * sizeof(u16) + 15) / 16 * 16;  // high, then low
    static constexpr size_t BUF_BYTES = Y_BYTES + H_BYTES;
    static constexpr size_t LDS_BYTES = 2 * BUF_BYTES + ROWS * sizeof(int);
};

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ...: a loop over register slots that have to be
// indexed with constants
template <int... Js, class F>
__device__ __forceinline__ void for_each_slot(std::integer_sequence<int, Js...>, F&& f)
{
    (f(std::integral_constant<int, Js>{}), ...);
}

// D[rank][col] = sum_t H[t][rank] Y[t][col] over the unit's rows; H = h_saved (for dB, Y = dy) or g (for
// dA, Y = x).  MFMA: lane (c = lane % 16, kg = lane / 16) supplies H[8 kg ..][rank c] and Y[8 kg ..][col c]
// of a 32-row step and receives D[rank 4 kg + v][col c].
// chunk_id < 0: the unit covers its whole segment and accumulates into dA / dB (times scale); else it stores its
// partial to slot chunk_id of wpart
template <int NT, int ROWS>
__device__ __forceinline__ void wgrad_unit(const BwdParams& p, const Unit& u, int rank, float scale, int chunk_id, bool for_b,
                                           int col_block, unsigned char* lds)
{
    using C = WgCfg<NT, ROWS>;
    constexpr int YQ = kWgCols / 128;  // 16-byte pieces of a staged activation row per thread
    const int lane = lane_id(), w = uniform((int)threadIdx.x / kWave), c = lane & 15, kg = lane >> 4;
    const u16* Y = for_b ? p.dy : p.x;
    const long long ldy = for_b ? p.lddy : p.ldx;
    const int d = for_b ? p.d_out : p.d_in;
    const int n0 = col_block * kWgCols;
    int* lds_row = reinterpret_cast<int*>(lds + 2 * C::BUF_BYTES);

    __syncthreads();  // the previous unit's LDS reads are done
    for (int i = (int)threadIdx.x; i < ROWS; i += kThreads) lds_row[i] = i < u.len ? row_of(p, u.pos + i) : -1;
    __syncthreads();
    const int safe_row = max(lds_row[0], 0);

    // staging assignment: 16 threads cover 128 columns (256 bytes) of one row per pass
    const int y_row = (int)threadIdx.x / 16, y_piece = (int)threadIdx.x % 16;
    // the unit's rows of h_saved (for dB) or of g (for dA); both are [row][rank] per segment
    const float* hsrc = (for_b ? p.h_saved : p.g) + p.h_offsets[u.seg] + (long long)(u.pos - u.first) * rank;
    constexpr int DEPTH = NT == 1 ? 4 : NT == 2 ? 3 : NT == 4 ? 2 : 1;  // steps in flight (as many as the registers allow)
    u32x4 gy[DEPTH][YQ];
    float gh[DEPTH][NT + 1];  // [NT]: the row's own scale (1 when the scale is the adapter's, applied by the reduction)
    // all loads are unconditional (clamped addresses), so the number in flight is static; what lies
    // outside the unit is zeroed when it is stored to LDS
    auto stage_load = [&](int step, u32x4 (&y)[YQ], float (&h)[NT + 1]) {
        const int i = step * kStepRows + y_row;
        const int row = lds_row[min(i, ROWS - 1)];
        const u16* yrow = Y + (long long)(row >= 0 ? row : safe_row) * ldy;
#pragma unroll
        for (int q = 0; q < YQ; ++q) y[q] = *reinterpret_cast<const u32x4*>(yrow + min(n0 + (y_piece + 16 * q) * 8, d - 8));
        const float* hrow = hsrc + (long long)min(i, u.len - 1) * rank;
#pragma unroll
        for (int q = 0; q < NT; ++q) h[q] = hrow[min(y_piece + 16 * q, rank - 1)];
        h[NT] = p.token_scales ? p.token_scales[max(row, 0)] : 1.f;
    };
    auto stage_store = [&](int step, int buf, const u32x4 (&y)[YQ], const float (&h)[NT + 1]) {
        u16* ly = reinterpret_cast<u16*>(lds + buf * C::BUF_BYTES);
        u16* lh = reinterpret_cast<u16*>(lds + buf * C::BUF_BYTES + C::Y_BYTES);
        const int i = step * kStepRows + y_row;
        const bool row_live = i < u.len && lds_row[min(i, ROWS - 1)] >= 0;
#pragma unroll
        for (int q = 0; q < YQ; ++q) {
            const bool live = row_live && n0 + (y_piece + 16 * q) * 8 < d;
            *reinterpret_cast<u32x4*>(ly + y_row * C::YPITCH + (y_piece + 16 * q) * 8) = live ? y[q] : u32x4{0u, 0u, 0u, 0u};
        }
        // h / g as bf16 high and low parts (together ~16 mantissa bits), split here once instead of in every wave
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const float v = (i < u.len && y_piece + 16 * q < rank) ? h[q] * h[NT] : 0.f;
            unsigned int hi, lo;
            split_value(v, hi, lo);
            lh[y_row * C::HPITCH + y_piece + 16 * q] = (u16)hi;
            lh[(kStepRows + y_row) * C::HPITCH + y_piece + 16 * q] = (u16)lo;
        }
    };

    f32x4 acc[NT][kWgTiles];
#pragma unroll
    for (int jt = 0; jt < NT; ++jt)
#pragma unroll
        for (int nt = 0; nt < kWgTiles; ++nt) acc[jt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int buf) {
        const u16* ly = reinterpret_cast<const u16*>(lds + buf * C::BUF_BYTES);
        const u16* lh = reinterpret_cast<const u16*>(lds + buf * C::BUF_BYTES + C::Y_BYTES);
        // the staged rows are the MFMA's k axis: both operands are read back transposed
        u32x4 yf[kWgTiles];
#pragma unroll
        for (int nt = 0; nt < kWgTiles; ++nt) yf[nt] = lds_read_transposed_16x32(ly + w * (16 * kWgTiles) + nt * 16, C::YPITCH);
#pragma unroll
        for (int jt = 0; jt < NT; ++jt) {
            const u32x4 hi = lds_read_transposed_16x32(lh + jt * 16, C::HPITCH);
            const u32x4 lo = lds_read_transposed_16x32(lh + kStepRows * C::HPITCH + jt * 16, C::HPITCH);
#pragma unroll
            for (int nt = 0; nt < kWgTiles; ++nt) {
                acc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(lo), as_bf16x8(yf[nt]), acc[jt][nt], 0, 0, 0);
                acc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(hi), as_bf16x8(yf[nt]), acc[jt][nt], 0, 0, 0);
            }
        }
    };

    // Pipeline: the loads of the next DEPTH steps are in flight in registers; a step is stored to one of
    // two LDS buffers (one barrier per step: the buffer written now was last read two steps ago), its
    // register slot is refilled with the step DEPTH ahead, and the step is multiplied out of LDS.
    const int n_steps = (u.len + kStepRows - 1) / kStepRows;
#pragma unroll
    for (int dd = 0; dd < DEPTH; ++dd) stage_load(min(dd, n_steps - 1), gy[dd], gh[dd]);
    auto step_fn = [&](int step, auto slot) {
        constexpr int J = decltype(slot)::value;
        stage_store(step, step & 1, gy[J], gh[J]);
        stage_load(min(step + DEPTH, n_steps - 1), gy[J], gh[J]);  // unconditional; past the end it re-reads
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        compute(step & 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int step = 0; step < n_steps; step += DEPTH)
        for_each_slot(std::make_integer_sequence<int, DEPTH>{}, [&](auto slot) {
            if (step + decltype(slot)::value < n_steps) step_fn(step + decltype(slot)::value, slot);
        });

    if (chunk_id < 0) {
        // Accumulation with the hardware's fp32 addition in memory: every element receives exactly one addition per
        // segment, so the result does not depend on timing as long as an adapter has one fine-tune segment (always
        // true of the builder's tables); two segments of one adapter are both added, in either order.
        float* dst = for_b ? p.dB_ptrs[u.ad] : p.dA_ptrs[u.ad];
#pragma unroll
        for (int jt = 0; jt < NT; ++jt)
#pragma unroll
            for (int nt = 0; nt < kWgTiles; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int j = jt * 16 + 4 * kg + v, n = n0 + w * (16 * kWgTiles) + nt * 16 + c;
                    if (j < rank && n < d) unsafeAtomicAdd(dst + (long long)j * d + n, scale * acc[jt][nt][v]);
                }
        return;
    }
    const int dsum = p.d_out + p.d_in;
    float* out = p.wpart + (long long)chunk_id * p.rstride * dsum + (for_b ? 0 : p.d_out);
#pragma unroll
    for (int jt = 0; jt < NT; ++jt)
#pragma unroll
        for (int nt = 0; nt < kWgTiles; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = jt * 16 + 4 * kg + v, n = n0 + w * (16 * kWgTiles) + nt * 16 + c;
                if (j < rank && n < d) out[(long long)j * dsum + n] = acc[jt][nt][v];
            }
}

// =================================================================================================
// Whole segments: behind the slab kernel, which leaves g and h as ready-made operands (frag_at), a unit takes ALL rows of
// a segment x 64 to 512 columns, so that there are no partials and no reduction launch.  The 8, 4, 2 or 1 waves that share 64
// columns take alternate 32-position steps: the step's rows of dy or x (8 rows x 128 bytes per instruction) go through LDS of the wave's own and come back
// transposed, the operands of h or g come straight from memory (L2: every unit of a segment reads them).  No workgroup
// barrier in the loop; the results of the waves that share columns are added up at the end in a fixed order.
// What bounds it: a unit's fixed part (tables, adapter, first loads, the sum over the waves, about 5 us) and, in long segments,
// the column walk; so two steps in flight per wave and few registers do better than four (2048 + 2048 rows of rank 32,
// 4096 -> 4096: 20.5 us instead of 24; with h as 32-bit rows that every unit splits for itself 21.4, with 144 columns per unit
// 22.1).  2 x 1024 rows of rank 8: 13.1 + 4.1 us with chunks and reduction, 9.7 whole (3.5 TB/s).
//   Columns per unit: a compute unit holds one workgroup (192 registers at rank 32), so more 64-column units than compute units are
// a second round, whose fixed parts several short segments do not repay.  So 128, 256 or 512 columns, the fewest that fit one
// round: us of the backward call with chunks, with 64 columns, and now, rank 32, 4096 -> 4096: 4 segments of 62 rows 20.3, 22.5, 20.7, 16
// of 31 rows 31.2, 42.5, 31.3, 40 of 25 rows 54.5, 85.3, 53.3, 4 of 500 rows 36.4, 33.4, 31.2; 4096 -> 11008, 4 of 125 rows 34.6,
// 40.6, 34.3; rank 8, 4096 -> 14336, 16 of 12 rows 29.6, 63.2, 33.0 (the worst); 490 calls: 0.90 of the time with chunks on average.
// =================================================================================================
constexpr int kWholeCols = 64;  // columns of a unit: a 128-byte line of a row
constexpr int kWholeTiles = kWholeCols / 16;
constexpr int kWholePitch = kWholeCols + 8;  // u16 elements per staged row

template <int NT>
struct WholeCfg {
    static constexpr int DEPTH = 2;                           // steps in flight
    static constexpr int RED = NT * 16 < 32 ? NT * 16 : 32;      // accumulator registers that the waves add up at a time
};
constexpr size_t kWholeWaveBytes = 32 * kWave * sizeof(float);   // LDS of a wave: its rows, later its share of the sum
static_assert((size_t)kStepRows * kWholePitch * sizeof(u16) <= kWholeWaveBytes, "a step's rows fit");
constexpr size_t kWholeLdsBytes = kWaves * kWholeWaveBytes;

// NT: 16-rank tiles of this unit, from rank j0 on; SHARE: so many waves share 64 columns, in alternate steps; the unit has
// kWaves / SHARE x 64 columns
template <int NT, int SHARE>
__device__ __forceinline__ void whole_unit(const BwdParams& p, int begin, int end, int rank, float scale, bool for_b, int col_block,
                                           int j0, float* dst, unsigned char* lds)
{
    using C = WholeCfg<NT>;
    constexpr int D = C::DEPTH, NJ = kStepRows / 8;
    const int lane = lane_id(), w = uniform((int)threadIdx.x / kWave), c = lane & 15, kg = lane >> 4;
    const int r8 = lane >> 3, piece = lane & 7;  // an instruction covers 8 rows x 128 bytes
    const u16* Y = for_b ? p.dy : p.x;
    const long long ldy = for_b ? p.lddy : p.ldx;
    const int d = for_b ? p.d_out : p.d_in;
    const int group = w / SHARE, member = w % SHARE, n0 = (col_block * (kWaves / SHARE) + group) * kWholeCols;
    const bool col_live = n0 + piece * 8 < d;
    const u16* ycol = Y + min(n0 + piece * 8, d - 8);
    typedef const __attribute__((address_space(1))) u32x4* gfrag;
    const gfrag frag = (gfrag)reinterpret_cast<const u32x4*>(for_b ? p.frag_h : p.frag_g) + (j0 >> 4) * 2 * kWave + lane;
    u16* ly = reinterpret_cast<u16*>(lds + (size_t)w * kWholeWaveBytes);

    const int s0 = (begin >> 5) + member, total = ((end + 31) >> 5) - (begin >> 5);
    const int n_mine = member < total && n0 < d ? (total - member + SHARE - 1) / SHARE : 0;  // steps member, member + SHARE, ...
    auto step_at = [&](int j) { return s0 + SHARE * min(j, n_mine - 1); };  // (past the end: the last step again)

    f32x4 acc[NT][kWholeTiles];
#pragma unroll
    for (int jt = 0; jt < NT; ++jt)
#pragma unroll
        for (int nt = 0; nt < kWholeTiles; ++nt) acc[jt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (n_mine > 0) {  // wave uniform
        u32x4 gy[D][NJ], gf[D][NT][2];
        int row_in[D];  // row index of position lane % 32 of the step, as loaded
        int rows[2];    // the same, a step or two ahead of the loads that need it
        // All loads are unconditional (clamped addresses), so the number in flight is static.  The table's entry is kept as
        // it is: checking it where it is loaded would wait for it, and with it for everything in flight.
        const int32_t* tab = p.perm ? p.perm : p.seg_starts;
        auto position = [&](int j) { return min(max(step_at(j) * 32 + (lane & 31), begin), end - 1); };
        auto row_load = [&](int j) { return tab[p.perm ? position(j) : 0]; };
        auto load = [&](int j, int raw, u32x4 (&y)[NJ], u32x4 (&f)[NT][2], int& row) {
            row = p.perm ? raw : position(j);
            const int safe = (unsigned)row < (unsigned)p.n_tokens ? row : 0;
#pragma unroll
            for (int i = 0; i < NJ; ++i) y[i] = *reinterpret_cast<const u32x4*>(ycol + (long long)__shfl(safe, r8 + 8 * i, kWave) * ldy);
            const long long at = (long long)step_at(j) * p.frag_tiles * 2 * kWave;
#pragma unroll
            for (int jt = 0; jt < NT; ++jt)
#pragma unroll
                for (int part = 0; part < 2; ++part) f[jt][part] = frag[at + (jt * 2 + part) * kWave];
        };
        auto step = [&](int j, auto slot) {
            constexpr int J = decltype(slot)::value, S = J % D;
            const int first = step_at(j) * 32;
            const bool inside = first >= begin && first + 32 <= end;  // wave uniform
            if (!inside || !__all(col_live && (unsigned)row_in[S] < (unsigned)p.n_tokens)) {
                // positions outside the segment belong to other segments: nothing of them may reach the sums, not even a NaN
#pragma unroll
                for (int i = 0; i < NJ; ++i) {
                    const int pos = first + r8 + 8 * i;
                    const bool live = col_live && pos >= begin && pos < end && (unsigned)__shfl(row_in[S], r8 + 8 * i, kWave) < (unsigned)p.n_tokens;
                    gy[S][i] = live ? gy[S][i] : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int pos = first + 8 * kg + 2 * e;
                    const unsigned int keep = (pos >= begin && pos < end ? 0xffffu : 0u) | (pos + 1 >= begin && pos + 1 < end ? 0xffff0000u : 0u);
#pragma unroll
                    for (int jt = 0; jt < NT; ++jt)
#pragma unroll
                        for (int part = 0; part < 2; ++part) gf[S][jt][part][e] &= keep;
                }
            }
#pragma unroll
            for (int i = 0; i < NJ; ++i) *reinterpret_cast<u32x4*>(ly + (r8 + 8 * i) * kWholePitch + piece * 8) = gy[S][i];
            u32x4 f[NT][2];
#pragma unroll
            for (int jt = 0; jt < NT; ++jt)
#pragma unroll
                for (int part = 0; part < 2; ++part) f[jt][part] = gf[S][jt][part];
            load(j + D, rows[J & 1], gy[S], gf[S], row_in[S]);  // the registers are free: the step D ahead
            rows[J & 1] = row_load(j + D + 2);
            __builtin_amdgcn_sched_barrier(0);
            wave_sync();
            // the staged rows are the MFMA's k axis: read back transposed
#pragma unroll
            for (int nt = 0; nt < kWholeTiles; ++nt) {
                const u32x4 yf = lds_read_transposed_16x32(ly + nt * 16, kWholePitch);
#pragma unroll
                for (int jt = 0; jt < NT; ++jt) {
                    acc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f[jt][1]), as_bf16x8(yf), acc[jt][nt], 0, 0, 0);
                    acc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f[jt][0]), as_bf16x8(yf), acc[jt][nt], 0, 0, 0);
                }
            }
            wave_sync();  // the rows are overwritten by the next step
        };
        {
            int r[D];
#pragma unroll
            for (int dd = 0; dd < D; ++dd) r[dd] = row_load(dd);
            rows[0] = row_load(D);  // step j takes rows[j & 1] for step j + D
            rows[1] = row_load(D + 1);
#pragma unroll
            for (int dd = 0; dd < D; ++dd) load(dd, r[dd], gy[dd], gf[dd], row_in[dd]);
        }
        constexpr int U = D > 2 ? D : 2;
        for (int j = 0; j < n_mine; j += U)
            for_each_slot(std::make_integer_sequence<int, U>{}, [&](auto slot) {
                if (j + decltype(slot)::value < n_mine) step(j + decltype(slot)::value, slot);
            });
    }

    auto add = [&](int reg, float sum) {
        const int jj = j0 + (reg >> 4) * 16 + 4 * kg + (reg & 3), n = n0 + ((reg >> 2) & 3) * 16 + c;
        if (jj < rank && n < d) unsafeAtomicAdd(dst + (long long)jj * d + n, scale * sum);  // (one addition per segment, see wgrad_unit)
    };
    if constexpr (SHARE == 1) {
#pragma unroll
        for (int reg = 0; reg < NT * 16; ++reg) add(reg, acc[reg >> 4][(reg >> 2) & 3][reg & 3]);
    } else {
        // the sum over the waves that share columns, RED accumulator registers at a time: every wave parks its own, then thread (w,
        // lane) adds its group's partial sums of registers member, member + SHARE, ... of lane `lane` as a balanced tree
        float* red = reinterpret_cast<float*>(lds);
        constexpr int PER_WAVE = C::RED * kWave;
#pragma unroll
        for (int part = 0; part < NT * 16 / C::RED; ++part) {
            __syncthreads();  // the rows (or the previous part's sums) have been read
#pragma unroll
            for (int r = 0; r < C::RED; ++r) {
                const int reg = part * C::RED + r;
                red[w * PER_WAVE + r * kWave + lane] = acc[reg >> 4][(reg >> 2) & 3][reg & 3];
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < C::RED / SHARE; ++it) {
                const int r = it * SHARE + member;
                float t[SHARE];
#pragma unroll
                for (int ww = 0; ww < SHARE; ++ww) t[ww] = red[(group * SHARE + ww) * PER_WAVE + r * kWave + lane];
#pragma unroll
                for (int half = SHARE / 2; half > 0; half /= 2)
#pragma unroll
                    for (int ww = 0; ww < half; ++ww) t[ww] = t[2 * ww] + t[2 * ww + 1];
                add(part * C::RED + r, t[0]);
            }
        }
    }
    __syncthreads();  // before the next unit's rows
}

// segments of a unit by length, the long ones first, so that a launch ends evenly
__device__ __forceinline__ LenClass whole_segments(bool is_long)
{
    return is_long ? LenClass{257, kBig, 1 << LQ_SEG_FINETUNE} : LenClass{1, 257, 1 << LQ_SEG_FINETUNE};
}

// NT: 16-rank tiles of the launch; every unit runs with its own adapter's.  Ranks above 64 are two units of up to 64 ranks
// (eight tiles' accumulators and operands do not fit the registers: 175 spilled).
template <int NT>
__global__ __launch_bounds__(kThreads, 2) void wgrad_whole_kernel(BwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    constexpr int kWhole = 1 << 30;  // rows per unit: no segment is cut
    int n_seg;
    const SegCache c0 = load_seg_cache(p, n_seg);
    constexpr int HALVES = NT >= 8 ? 2 : 1;
    const int segs_long = count_chunks(p, n_seg, c0, kWhole, whole_segments(true));
    const int segs = segs_long + count_chunks(p, n_seg, c0, kWhole, whole_segments(false));
    // columns per unit: 64 where the units fit one round of the grid, else the fewest up to 512 that do
    int cols_log2 = 6, blocks_b, per_seg;
    for (;; ++cols_log2) {
        const int round_up = (1 << cols_log2) - 1;
        blocks_b = (p.d_out + round_up) >> cols_log2;
        per_seg = (blocks_b + ((p.d_in + round_up) >> cols_log2)) * HALVES;
        if (cols_log2 == 9 || segs * per_seg <= (int)gridDim.x) break;
    }
    const int n_long = segs_long * per_seg, n_units = segs * per_seg;
    for (int id = (int)blockIdx.x; id < n_units; id += (int)gridDim.x) {
        Unit u;
        const int base = id < n_long ? 0 : n_long, seg = small_div(id - base, per_seg), at = id - base - seg * per_seg;
        const int cb = at / HALVES, j0 = HALVES > 1 ? (at & 1) * 64 : 0;
        if (!find_chunk(p, n_seg, c0, seg, kWhole, whole_segments(id < n_long), u)) continue;
        if (u.ad < 0 || u.ad >= p.n_adapters) continue;  // flagged by the forward kernels already
        const bool for_b = cb < blocks_b;
        // (requested together: one round trip)
        const int rank = p.ranks[u.ad];
        const float adapter_scale = p.scales[u.ad];
        float* const* const ptrs = for_b ? p.dB_ptrs : p.dA_ptrs;
        float* const dst = ptrs ? ptrs[u.ad] : nullptr;
        if (rank < 1 || rank > p.max_rank || j0 >= rank || !dst) continue;
        const float scale = p.token_scales ? 1.f : adapter_scale;  // (per-token scales are in the operands)
        const int end = u.first + u.seg_len, block = for_b ? cb : cb - blocks_b;
        const int left = rank - j0;  // > 0
        auto run = [&](auto tiles) {  // (all of this is workgroup uniform)
            constexpr int N = decltype(tiles)::value;
            if (cols_log2 == 6) whole_unit<N, 8>(p, u.first, end, rank, scale, for_b, block, j0, dst, lds_raw);
            else if (cols_log2 == 7) whole_unit<N, 4>(p, u.first, end, rank, scale, for_b, block, j0, dst, lds_raw);
            else if (cols_log2 == 8) whole_unit<N, 2>(p, u.first, end, rank, scale, for_b, block, j0, dst, lds_raw);
            else whole_unit<N, 1>(p, u.first, end, rank, scale, for_b, block, j0, dst, lds_raw);
        };
        if (NT >= 4 && left > 32) run(std::integral_constant<int, (NT >= 4 ? 4 : NT)>{});
        else if (NT >= 2 && left > 16) run(std::integral_constant<int, (NT >= 2 ? 2 : NT)>{});
        else run(std::integral_constant<int, 1>{});
    }
}

// the fine-tune segments with more rows than a unit are cut into chunks (partials, then the reduction); the shorter
// ones are one unit per column block
__device__ __forceinline__ LenClass cut_class(int rows) { return LenClass{rows + 1, kBig, 1 << LQ_SEG_FINETUNE}; }
__device__ __forceinline__ LenClass whole_class(int rows) { return LenClass{1, rows + 1, 1 << LQ_SEG_FINETUNE}; }

// Token rows per unit, from the fine-tune rows that the tables hold (the batch's tokens are no measure of them).  1024 where units of 512 rows are
// more than one round of the grid (ranks up to 32: two workgroups per compute unit, 512 units): half the partials.  us of the units
// and of the reduction, 512 and 1024 rows, rank 32: 4096 -> 14336, 4096 rows (576 units) 50.2 and 48.1, 6144 rows (864) 61.4 and 54.5,
// 8192 (1152) 82.8 and 86.3, 12000 (1728) 114.7 and 109.9; 4096 -> 11008, 6144 rows (708) 50.3 and 49.9, 8192 (944) 67.3 and 60.7; below,
// the machine is not full: 4096 -> 4096, 2048 rows (128) 19.4 and 29.1, 4096 (256) 24.2 and 32.8, 4096 -> 11008, 4096 rows (472) 36.7 and 36.8.
__device__ __forceinline__ int unit_rows(const BwdParams& p, int n_seg, const SegCache& c0)
{
    if (p.wg_slots == 0) return kWgRows;
    const int per_chunk = (p.d_out + kWgCols - 1) / kWgCols + (p.d_in + kWgCols - 1) / kWgCols;
    const int chunks = count_chunks(p, n_seg, c0, kWgRows, LenClass{1, kBig, 1 << LQ_SEG_FINETUNE});
    return chunks * per_chunk > p.wg_slots ? 2 * kWgRows : kWgRows;
}

template <int NT, int ROWS>
__device__ __forceinline__ void wgrad_units(const BwdParams& p, int n_seg, const SegCache& c0, unsigned char* lds)
{
    const LenClass cut = cut_class(ROWS), whole = whole_class(ROWS);
    const int blocks_b = (p.d_out + kWgCols - 1) / kWgCols, blocks_a = (p.d_in + kWgCols - 1) / kWgCols;
    const int per_chunk = blocks_b + blocks_a;
    const int n_cut = count_chunks(p, n_seg, c0, ROWS, cut) * per_chunk;  // the (larger) chunks first
    const int n_units = n_cut + count_chunks(p, n_seg, c0, ROWS, whole) * per_chunk;
    for (int id = (int)blockIdx.x; id < n_units; id += (int)gridDim.x) {
        Unit u;
        const bool is_cut = id < n_cut;
        const int chunk_id = small_div(is_cut ? id : id - n_cut, per_chunk), cb = (is_cut ? id : id - n_cut) - chunk_id * per_chunk;
        if (!(is_cut ? find_chunk(p, n_seg, c0, chunk_id, ROWS, cut, u) : find_chunk(p, n_seg, c0, chunk_id, ROWS, whole, u)))
            continue;
        if (u.ad < 0 || u.ad >= p.n_adapters) continue;  // flagged by the forward kernels already
        const int rank = p.ranks[u.ad];
        if (rank < 1 || rank > p.max_rank) continue;
        const bool for_b = cb < blocks_b;
        if (for_b ? (p.dB_ptrs == nullptr || p.dB_ptrs[u.ad] == nullptr) : (p.dA_ptrs == nullptr || p.dA_ptrs[u.ad] == nullptr))
            continue;
        const float scale = p.token_scales ? 1.f : p.scales[u.ad];  // (per-token scales were applied row by row)
        wgrad_unit<NT, ROWS>(p, u, rank, scale, is_cut ? chunk_id : -1, for_b, for_b ? cb : cb - blocks_b, lds);
    }
}

// (ranks up to 32: at most 128 registers, so that two workgroups share a compute unit and one's loads
// overlap the other's barriers)
// EITHER: units of 512 or 1024 rows.  (A number of rows known at run time only slowed the units down: backward of a decoder layer
// 512 -> 526 us.  Spilled at rank 32: 6 registers, 14 with both heights, of which either path pays its own.)
template <int NT, bool EITHER>
__global__ __launch_bounds__(kThreads, NT <= 2 ? 4 : 2) void wgrad_kernel(BwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    int n_seg;
    const SegCache c0 = load_seg_cache(p, n_seg);
    if (EITHER && unit_rows(p, n_seg, c0) > kWgRows) wgrad_units<NT, (EITHER ? 2 * kWgRows : kWgRows)>(p, n_seg, c0, lds_raw);  // grid uniform
    else wgrad_units<NT, kWgRows>(p, n_seg, c0, lds_raw);
}

// dA / dB += scale * (sum of a cut segment's chunk partials, in chunk order).  One unit = the first chunk of
// a segment x 512 columns of [dB | dA] x 8 ranks; a thread owns one column and keeps the 8 sums in
// registers, so the loads of a chunk's partials are independent of each other.  The accumulation is the
// hardware's fp32 addition in memory, one per element and segment (see wgrad_unit).
constexpr int kRedRanks = 8;
__global__ __launch_bounds__(kThreads) void wreduce_kernel(BwdParams p)
{
    int n_seg;
    const SegCache c0 = load_seg_cache(p, n_seg);
    const int rows = unit_rows(p, n_seg, c0);
    const LenClass cut = cut_class(rows);
    const int dsum = p.d_out + p.d_in;
    const int col_blocks = (dsum + kThreads - 1) / kThreads;
    const int rank_groups = (p.max_rank + kRedRanks - 1) / kRedRanks;
    const int per_chunk = col_blocks * rank_groups;
    const int n_units = count_chunks(p, n_seg, c0, rows, cut) * per_chunk;
    for (int id = (int)blockIdx.x; id < n_units; id += (int)gridDim.x) {
        Unit u;
        const int chunk_id = small_div(id, per_chunk), sub = id - chunk_id * per_chunk;
        if (!find_chunk(p, n_seg, c0, chunk_id, rows, cut, u)) continue;
        if (u.pos != u.first) continue;  // only the segment's first chunk adds up the segment
        if (u.ad < 0 || u.ad >= p.n_adapters) continue;
        const int n_chunks = (u.seg_len + rows - 1) / rows;
        const int j0 = (sub / col_blocks) * kRedRanks;
        const int col = (sub % col_blocks) * kThreads + (int)threadIdx.x;
        if (col >= dsum) continue;
        const float* __restrict__ part = p.wpart + ((long long)chunk_id * p.rstride + j0) * dsum + col;
        // Four chunks' partials are requested together (a chunk that does not exist re-reads the last one and is not
        // added): one round trip for the segments of the layer stack instead of one per chunk; the additions keep
        // the chunk order.  The first four go out before the adapter's rank, scale and pointer are asked for: where
        // the partials lie depends on the tables alone (rows beyond the rank lie inside the rstride rows of a partial).
        float v[4][kRedRanks];
        auto request = [&](int cc) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int jj = 0; jj < kRedRanks; ++jj) v[k][jj] = part[((long long)min(cc + k, n_chunks - 1) * p.rstride + jj) * dsum];
        };
        request(0);
        __builtin_amdgcn_sched_barrier(0);
        const int rank = p.ranks[u.ad];
        const float scale = p.token_scales ? 1.f : p.scales[u.ad];  // (per-token scales were applied row by row)
        const bool for_b = col < p.d_out;
        float* __restrict__ dst = for_b ? (p.dB_ptrs ? p.dB_ptrs[u.ad] : nullptr) : (p.dA_ptrs ? p.dA_ptrs[u.ad] : nullptr);
        if (rank < 1 || rank > p.max_rank || j0 >= rank || !dst) continue;
        const int d = for_b ? p.d_out : p.d_in, n = for_b ? col : col - p.d_out;
        float sum[kRedRanks];
#pragma unroll
        for (int jj = 0; jj < kRedRanks; ++jj) sum[jj] = 0.f;
        for (int cc = 0; cc < n_chunks; cc += 4) {
            if (cc > 0) request(cc);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int jj = 0; jj < kRedRanks; ++jj) sum[jj] = cc + k < n_chunks ? sum[jj] + v[k][jj] : sum[jj];
        }
#pragma unroll
        for (int jj = 0; jj < kRedRanks; ++jj)
            if (j0 + jj < rank) unsafeAtomicAdd(dst + (long long)(j0 + jj) * d + n, scale * sum[jj]);
    }
}

// Whole segments or 512-row chunks, by the host's arguments.  Measured on the backward call (g / dx, weight gradients and,
// with chunks of batches above 512 tokens, their reduction) on three sets of operands in turn, us with chunks and whole, fine-tune
// rows only, in one segment and in four:
//   rank 32, 4096 -> 4096, 500 rows 27.1 and 20.7, 23.1 and 22.7, 2000 37.8 and 31.4, 36.4 and 31.2, 3500 51.5 and 45.7, 52.8 and 44.6;
//   5632 67.8 and 70.0 (one segment); 4096 -> 1024, 3500 rows 39.7 and 36.4, 40.7 and 31.5, 5632 52.7 and 53.4 (one); 1024 -> 1024, 2000
//   rows 29.5 and 22.6, 26.3 and 18.3; 4096 -> 14336, 1500 rows 49.0 and 49.0 (one), 2500 77.4 and 81.8 (one).
//   rank 64, 4096 -> 4096, 2000 rows 48.3 and 41.0, 49.1 and 41.4; 4096 -> 1024, 4500 59.2 and 61.0 (one).
//   rank 128, 4096 -> 4096, 500 rows 52.6 and 37.8, 48.2 and 48.6, 2000 67.8 and 51.4, 71.4 and 61.3; 16 segments of 31 rows 82.6 and 84.6.
// Large batches lose because a unit walks down 64 columns, a line of every row, which streams slower from memory than 256
// columns do; narrow layers of one long segment because there are too few units (512 -> 512, rank 32, 5632 rows 32.2 and 35.7).
bool whole_segments_win(int n_tokens, int max_rank, int d_in, int d_out)
{
    const long long width = (long long)d_in + d_out;
    return (n_tokens <= 2048 || width >= 5120) && n_tokens * width <= (max_rank <= 32 ? 29000000 : 18000000);
}

// finished g of the fine-tune rows: at most n_tokens x max_rank floats (a multiple of 16 bytes)
size_t gsum_bytes(int n_tokens, int max_rank) { return ((size_t)n_tokens * (size_t)max_rank * sizeof(float) + 15) / 16 * 16; }

// Only segments with more rows than a unit (512, or 1024, which makes fewer chunks) keep partials: n segments of more than 512
// have at most n_tokens / 512 + n chunks and n <= n_tokens / 513, whatever tables the caller passes.
size_t wpart_bytes(int n_tokens, int max_rank, int d_in, int d_out)
{
    const size_t chunks = 2 * ((size_t)(n_tokens + kWgRows - 1) / kWgRows);
    return chunks * (size_t)rstride_for(max_rank) * ((size_t)d_in + d_out) * sizeof(float);
}

template <int NT, bool EITHER>
int wgrad_grid()
{
    static DeviceGrid cache;
    return cache.get([] { return resident_grid(wgrad_kernel<NT, EITHER>, WgCfg<NT, EITHER ? 2 * kWgRows : kWgRows>::LDS_BYTES); });
}
template <int NT, bool EITHER>
hipError_t launch_wgrad(BwdParams& p, hipStream_t st)
{
    constexpr size_t lds = WgCfg<NT, EITHER ? 2 * kWgRows : kWgRows>::LDS_BYTES;
    const int grid = wgrad_grid<NT, EITHER>();
    p.wg_slots = EITHER ? grid : 0;
    return launch_kernel(kKernelWgrad, wgrad_kernel<NT, EITHER>, dim3(grid), dim3(kThreads), lds, st, p);
}

template <int NT>
hipError_t launch_whole(const BwdParams& p, hipStream_t st)
{
    static DeviceGrid cache;
    const int grid = cache.get([] { return resident_grid(wgrad_whole_kernel<NT>, kWholeLdsBytes); });
    return launch_kernel(kKernelWgrad, wgrad_whole_kernel<NT>, dim3(grid), dim3(kThreads), kWholeLdsBytes, st, p);
}

}  // namespace
}  // namespace lq

// workspace: [header 4096 B][g slices: like the forward's partial h][finished g][partial weight gradients]
extern "C" size_t lora_backward_workspace_bytes(int32_t n_tokens, int32_t n_adapters, int32_t max_rank, int32_t d_in,
                                                int32_t d_out)
{
    (void)n_adapters;
    if (n_tokens < 0 || max_rank < 1 || d_in < 0 || d_out < 0) return lq::kWsHeaderBytes;
    return (size_t)lq::kWsHeaderBytes + lq::h_slices_bytes(n_tokens, max_rank) + lq::gsum_bytes(n_tokens, max_rank) +
           lq::wpart_bytes(n_tokens, max_rank, d_in, d_out);
}

extern "C" lq_status lora_segmented_backward(const void* x, int64_t ldx, const void* dy, int64_t lddy, void* dx,
                                             int64_t lddx, int32_t d_in, int32_t d_out,
                                             const void* const* A_ptrs, const void* const* B_ptrs,
                                             float* const* dA_ptrs, float* const* dB_ptrs,
                                             const int32_t* ranks, const float* scales, const float* token_scales,
                                             int32_t n_adapters, int32_t max_rank, const int32_t* perm, int32_t n_tokens,
                                             const int32_t* seg_starts, const int32_t* seg_adapter,
                                             const uint8_t* seg_kind, const int32_t* n_segments, int32_t max_segments,
                                             const float* h_saved, const int64_t* h_offsets,
                                             int32_t variant, void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace lq;
    if (n_tokens < 0 || d_in <= 0 || d_out <= 0 || n_adapters <= 0 || max_segments < 0 || max_rank < 1)
        return LQ_ERR_INVALID_ARG;
    if (variant != LQ_VARIANT_SPLIT && variant != LQ_VARIANT_FUSED && variant != LQ_VARIANT_SLAB && variant != LQ_VARIANT_AUTO)
        return LQ_ERR_INVALID_ARG;
    if (variant == LQ_VARIANT_AUTO) variant = auto_variant(max_rank, n_tokens, false, 1, d_out, d_in);  // (reads dy, writes dx, of the fine-tune rows)
    if (variant == LQ_VARIANT_SLAB && !(slab_reaches(max_rank, d_in) && slab_reaches(max_rank, d_out))) variant = LQ_VARIANT_SPLIT;
    if (!A_ptrs || !B_ptrs || !ranks || !scales || !seg_starts || !seg_adapter || !seg_kind || !n_segments)
        return LQ_ERR_INVALID_ARG;
    if (n_tokens > 0 && (!x || !dy || !dx)) return LQ_ERR_INVALID_ARG;
    if ((dA_ptrs || dB_ptrs) && n_tokens > 0 && (!h_saved || !h_offsets)) return LQ_ERR_INVALID_ARG;
    if (ldx < d_in || lddx < d_in || lddy < d_out) return LQ_ERR_INVALID_ARG;
    if (x && (x == dx || dy == dx)) return LQ_ERR_INVALID_ARG;
    if (max_rank > LQ_MAX_RANK || n_adapters > LQ_MAX_ADAPTERS) return LQ_ERR_UNSUPPORTED;
    if ((d_in % 8) || (d_out % 8) || (ldx % 8) || (lddx % 8) || (lddy % 8) || !aligned16(x) || !aligned16(dy) || !aligned16(dx))
        return LQ_ERR_UNSUPPORTED;
    if (!workspace || !aligned16(workspace) ||
        workspace_bytes < lora_backward_workspace_bytes(n_tokens, n_adapters, max_rank, d_in, d_out))
        return LQ_ERR_WORKSPACE;
    if (n_tokens == 0 || max_segments == 0) return LQ_OK;

    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);

    // 1. g = dy B^T on fine-tune rows: the forward's shrink over d_out against B
    FwdParams s1;
    s1.x = static_cast<const u16*>(dy); s1.ldx = lddy;
    s1.d_in = d_out;
    Proj q;
    q.y = static_cast<u16*>(dx); q.ldy = lddx; q.d_out = d_in;
    q.A_ptrs = B_ptrs; q.B_ptrs = A_ptrs;
    s1.ranks = ranks; s1.scales = scales;
    s1.n_adapters = n_adapters; s1.max_rank = max_rank;
    s1.token_scales = token_scales;
    s1.perm = perm; s1.n_tokens = n_tokens;
    s1.seg_starts = seg_starts; s1.seg_adapter = seg_adapter; s1.seg_kind = seg_kind;
    s1.n_segments = n_segments; s1.max_segments = max_segments;
    // the finished g goes where the forward would save h: [segment offset + row x rank + j], for the weight gradients
    float* gsum = reinterpret_cast<float*>(ws + kWsHeaderBytes + h_slices_bytes(n_tokens, max_rank));
    const bool want_w = dA_ptrs || dB_ptrs;
    q.h_out = want_w ? gsum : nullptr; s1.h_offsets = want_w ? reinterpret_cast<const long long*>(h_offsets) : nullptr;
    s1.n_proj = 1;
    s1.proj0 = q;
    for (int k = 1; k < kMaxProj; ++k) s1.more[k - 1] = q;
    s1.hpart = reinterpret_cast<float*>(ws + kWsHeaderBytes);
    s1.hproj = 0;
    s1.ksplit = 1; s1.rstride = rstride_for(max_rank);
    s1.header = s1.err = reinterpret_cast<int*>(ws); s1.tickets = reinterpret_cast<int*>(ws) + 4;
    s1.ksplit_hint = 0; s1.kinds = kFinetuneOnly;
    // whole segments' weight gradients behind the slab kernel: the operands lie in the g slices' region, which that kernel leaves free
    const bool slabs = variant == LQ_VARIANT_SLAB || (variant == LQ_VARIANT_FUSED && slab_form(s1));
    const int tiles = nt_for(max_rank);
    const size_t frag = (frag_bytes(n_tokens, tiles) + 255) / 256 * 256;
    const bool whole = want_w && slabs && 2 * frag <= h_slices_bytes(n_tokens, max_rank) && whole_segments_win(n_tokens, max_rank, d_in, d_out);
    const SlabFrag operands = {reinterpret_cast<u16*>(ws + kWsHeaderBytes), reinterpret_cast<u16*>(ws + kWsHeaderBytes + frag), h_saved, dB_ptrs, tiles};
    const SlabFrag* const leave = whole ? &operands : nullptr;
    // 2. dx += s g A on fine-tune rows: the forward's expand over d_in against A.  LQ_VARIANT_FUSED: both in a
    // single launch when its buffer descriptor can address the slices; else two launches with the same k split.
    // Whichever phase finishes g (the shrink without a split, the expand with one) also stores it to gsum.
    const bool one_launch = variant == LQ_VARIANT_FUSED && h_slices_bytes(n_tokens, max_rank) <= 0x7fffffffull;
    s1.coherent = one_launch; s1.hpart_bytes = one_launch ? (unsigned int)h_slices_bytes(n_tokens, max_rank) : 0;
    if (variant == LQ_VARIANT_SLAB) {
        if (run_slab(s1, st, leave) != hipSuccess) return LQ_ERR_HIP;
    } else if (one_launch) {
        if (run_shrink_expand(s1, LQ_VARIANT_FUSED, st, leave) != hipSuccess) return LQ_ERR_HIP;
    } else {
        if (run_shrink_expand(s1, LQ_VARIANT_SHRINK_ONLY, st) != hipSuccess) return LQ_ERR_HIP;
        s1.ksplit_hint = s1.ksplit;
        if (run_shrink_expand(s1, LQ_VARIANT_EXPAND_ONLY, st) != hipSuccess) return LQ_ERR_HIP;
    }

    // 3. partial weight gradients (from x, dy, the saved h and the finished g), then their reduction into dA / dB
    if (dA_ptrs || dB_ptrs) {
        BwdParams b;
        b.x = static_cast<const u16*>(x); b.ldx = ldx;
        b.dy = static_cast<const u16*>(dy); b.lddy = lddy;
        b.d_in = d_in; b.d_out = d_out;
        b.dA_ptrs = dA_ptrs; b.dB_ptrs = dB_ptrs; b.A_ptrs = A_ptrs; b.B_ptrs = B_ptrs;
        b.ranks = ranks; b.scales = scales; b.n_adapters = n_adapters; b.max_rank = max_rank;
        b.token_scales = token_scales;
        b.perm = perm; b.n_tokens = n_tokens;
        b.seg_starts = seg_starts; b.seg_adapter = seg_adapter; b.seg_kind = seg_kind;
        b.n_segments = n_segments; b.max_segments = max_segments;
        b.h_saved = h_saved; b.h_offsets = reinterpret_cast<const long long*>(h_offsets);
        b.g = gsum; b.rstride = s1.rstride;
        b.frag_g = operands.g; b.frag_h = operands.h; b.frag_tiles = tiles;
        b.wpart = reinterpret_cast<float*>(ws + kWsHeaderBytes + h_slices_bytes(n_tokens, max_rank) + gsum_bytes(n_tokens, max_rank));
        b.err = reinterpret_cast<int*>(ws);
        if (whole) {
            const hipError_t e = tiles == 1 ? launch_whole<1>(b, st) : tiles == 2 ? launch_whole<2>(b, st)
                               : tiles == 4 ? launch_whole<4>(b, st) : launch_whole<8>(b, st);
            return e == hipSuccess ? LQ_OK : LQ_ERR_HIP;
        }
        // (the tokens bound the fine-tune rows; the kernel that can do both starts 0.5 to 1 us later)
        const long long most_units = (n_tokens + kWgRows - 1ll) / kWgRows * (((long long)d_in + d_out) / kWgCols);
        const bool either = max_rank <= 32 && most_units > (max_rank <= 16 ? wgrad_grid<1, true>() : wgrad_grid<2, true>());
        const hipError_t e = max_rank <= 16   ? either ? launch_wgrad<1, true>(b, st) : launch_wgrad<1, false>(b, st)
                             : max_rank <= 32 ? either ? launch_wgrad<2, true>(b, st) : launch_wgrad<2, false>(b, st)
                             : max_rank <= 64 ? launch_wgrad<4, false>(b, st) : launch_wgrad<8, false>(b, st);
        if (e != hipSuccess) return LQ_ERR_HIP;
        // (no segment of a batch of up to 512 tokens is cut into chunks: nothing to reduce)
        if (n_tokens > kWgRows && launch_kernel(kKernelWreduce, wreduce_kernel, dim3(512), dim3(kThreads), 0, st, b) != hipSuccess)
            return LQ_ERR_HIP;
    }
    return LQ_OK;
}
