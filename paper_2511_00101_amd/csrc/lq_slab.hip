// Row-slab variant of the segmented multi-adapter LoRA forward (Section 3.3): one launch in which a
// workgroup takes a slab of at most 64 rows of one segment through BOTH products, so that h never leaves the
// compute unit: no partial-h buffer, no device-wide wait, and both phases are spread over the machine the same
// way.  The price is that every slab re-reads its adapter's matrices; they come from the L2 cache (slabs of
// one segment run side by side), which the measured access pattern bears: 256 workgroups that each stream 22
// rows of x and y and re-read 512 KB of A and B run at 4.3 TB/s of algorithmic bytes, against 4.9 TB/s without
// the re-reads.  A long batch takes taller slabs, which re-read less and fill one round of the grid: 32 -> 64 rows at most,
// 16384 rows of rank 64, 4096 -> 4096 104 -> 94 us (4.3 TB/s of algorithmic bytes), 8192 rows of rank 16 67 -> 47, of rank 64 87 ->
// 60, 8000 -> 11008 of rank 16 133 -> 96.  Time stamps of the 16384 rows: tables, plan and rows 7 us, phase 1 31 to 34, phase 2 41
// to 45, the last of 256 units 5 us after the median: the phases run at the HBM's rate.
#include "lq_slab.h"

namespace lq {
namespace {

constexpr size_t kHfragBytes = 16384;  // [projection of the pass][row tile][k step][high | low][lane] x 16 B
// LDS of the kernel: the h fragments, the waves' shares, the unit's row indices and scales, the stashed tables
constexpr size_t kWorkOffset = kHfragBytes;
constexpr size_t kRowsOffset = kWorkOffset + kWaves * kWaveBytes;
constexpr size_t kStashOffset = kRowsOffset + 2 * kSlabRows * sizeof(int);
constexpr size_t kSlabLdsBytes = kStashOffset + kStashBytes;

template <class PP> constexpr bool kFrag = std::is_same_v<PP, FwdFrag>;  // a backward call that leaves g and h as operands

// =================================================================================================
// one pass of a unit: NP projections (pi0 ..) through phase 1, the sum over the waves, and phase 2 (STREAM: y non-temporal, see
// streams_y; ZERO_X: see slab_shrink)
// =================================================================================================
template <int NT, int NP, int MTM, bool STREAM, bool ZERO_X, class PP>
__device__ __forceinline__ void slab_pass(const PP& p, const Unit& u0, const SegInfo& s0, int pi0, int part, int parts,
                                          unsigned char* lds)
{
    constexpr int KSTEPS = (NT + 1) / 2;
    static_assert((size_t)NP * MTM * KSTEPS * 2 * kWave * 16 <= kHfragBytes, "the pass's h fragments fit");
    u32x4* hfrag = reinterpret_cast<u32x4*>(lds);
    unsigned char* work = lds + kWorkOffset;
    const int* lds_row = reinterpret_cast<const int*>(lds + kRowsOffset);
    const float* lds_scale = reinterpret_cast<const float*>(lds_row + kSlabRows);
    const int w = uniform((int)threadIdx.x / kWave);

    SegInfo s[NP];
    if (!slab_adapters(p, u0, s0, pi0, s)) return;  // workgroup uniform; the error bit is set
    const int rank = s[0].rank;

    // the fragments start as zeros: rows and ranks beyond the live ones stay that way
    {
        constexpr u32x4 zero = {0u, 0u, 0u, 0u};
        static_assert(kHfragBytes == (size_t)2 * kThreads * 16, "two 16-byte stores per thread");
        hfrag[threadIdx.x] = zero;
        hfrag[threadIdx.x + kThreads] = zero;
    }
    // phase 1; every finished h element goes to h_out (fine-tune segments) and, scaled and split into a bf16 high and
    // low part, into the fragments phase 2 reads
    u16* hf16 = reinterpret_cast<u16*>(hfrag);
    const bool save = u0.kd == LQ_SEG_FINETUNE && p.h_offsets && part == 0;
    slab_shrink_sum<NT, NP, MTM, ZERO_X>(p, u0, s, lds_row, work, [&](auto qc, int i, int j, float sum) {
        constexpr int q = decltype(qc)::value;
        if (!kFrag<PP> && save) {
            float* h_out = proj_of(p, pi0 + q).h_out;
            if (h_out) h_out[p.h_offsets[u0.seg] + (long long)(u0.pos - u0.first + i) * rank + j] = sum;
        }
        const float scaled = sum * lds_scale[i];
        unsigned int hi, lo;
        split_value(scaled, hi, lo);
        if constexpr (kFrag<PP>)
            if (part == 0) store_frag(p.frag.g, frag_at(u0.pos + i, j, p.frag.tiles), p.token_scales ? scaled : sum);
        // fragment (projection q, row tile i / 16, k step j / 32): lane (j % 32 / 8) * 16 + i % 16 holds ranks 8 (j / 8) .. + 7
        const int slot = ((q * MTM + (i >> 4)) * KSTEPS + (j >> 5)) * 2;
        const int ln = ((j >> 3) & 3) * 16 + (i & 15);
        hf16[((slot + 0) * kWave + ln) * 8 + (j & 7)] = (u16)hi;
        hf16[((slot + 1) * kWave + ln) * 8 + (j & 7)] = (u16)lo;
    });
    __syncthreads();

    u16* bs = reinterpret_cast<u16*>(work + (size_t)w * kWaveBytes);
    float* ds = reinterpret_cast<float*>(bs + kChunk);
    static_assert(kChunk * sizeof(u16) % 16 == 0, "the D slab is 16-byte aligned");
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const Proj pj = proj_of(p, pi0 + q);
        const int nblk = (pj.d_out + kKB - 1) / kKB;
        const int begin = small_div(part * nblk, parts), end = small_div((part + 1) * nblk, parts);
        const u32x4* hf = hfrag + q * MTM * KSTEPS * 2 * kWave;
        if (u0.len <= 16) slab_expand<NT, 1, STREAM>(p, u0, s[q], pj, lds_row, hf, bs, ds, begin, end);  // workgroup uniform
        else if (MTM <= 2 || u0.len <= 32) slab_expand<NT, 2, STREAM>(p, u0, s[q], pj, lds_row, hf, bs, ds, begin, end);
        else if (u0.len <= 48) slab_expand<NT, (MTM > 2 ? 3 : 2), STREAM>(p, u0, s[q], pj, lds_row, hf, bs, ds, begin, end);
        else slab_expand<NT, (MTM > 2 ? 4 : 2), STREAM>(p, u0, s[q], pj, lds_row, hf, bs, ds, begin, end);
    }
    if constexpr (kFrag<PP>)
        if (part == 0) slab_frag_h(p, u0, rank, lds_scale);
    __syncthreads();  // before the next pass or unit reuses the LDS
}

template <int NT, int MTM, bool STREAM, class PP>
__device__ __forceinline__ void slab_unit(const PP& p, const Unit& u, const SegInfo& s0, int part, int parts, unsigned char* lds)
{
    slab_unit_rows(p, u, s0, reinterpret_cast<int*>(lds + kRowsOffset));
    __syncthreads();
    constexpr bool GROUP = std::is_same_v<PP, FwdParams>;
    const int n_proj = n_proj_of(p);
    if constexpr (NT >= 4 && !(GROUP && NT >= 8)) {
        // a launch with adapters of different ranks: every unit runs with as many 16-rank tiles as its own adapter needs.
        // (Not the groups above rank 64: eight tiles spill already, and the other passes beside them took the spills from
        // 40 to 61 registers: 4096 -> 4096, 1024, 1024, 1024 rows of rank 96: 61.5 -> 69.1 us, of mixed ranks 64.4 -> 68.8.)
        for (int pi = 0; pi < n_proj; ++pi) {
            if (NT >= 8 && s0.rank > 64) slab_pass<NT, 1, MTM, STREAM, true>(p, u, s0, pi, part, parts, lds);  // workgroup uniform
            else if (s0.rank > 32) slab_pass<4, 1, MTM, STREAM, true>(p, u, s0, pi, part, parts, lds);
            else if (s0.rank > 16) slab_pass<2, 1, MTM, STREAM, true>(p, u, s0, pi, part, parts, lds);
            else slab_pass<1, 1, MTM, STREAM, true>(p, u, s0, pi, part, parts, lds);
        }
        return;
    }
    constexpr int NPP = GROUP ? pass_projections<NT>() : 1;
    for (int pi0 = 0; pi0 < n_proj; pi0 += NPP) {
        const int np = min(NPP, n_proj - pi0);  // workgroup uniform
        if (NPP >= 4 && np == 4) slab_pass<NT, (NPP >= 4 ? 4 : 1), MTM, STREAM, (NT >= 4 || MTM > 2)>(p, u, s0, pi0, part, parts, lds);
        else if (NPP >= 3 && np == 3) slab_pass<NT, (NPP >= 3 ? 3 : 1), MTM, STREAM, (NT >= 4 || MTM > 2)>(p, u, s0, pi0, part, parts, lds);
        else if (NPP >= 2 && np == 2) slab_pass<NT, (NPP >= 2 ? 2 : 1), MTM, STREAM, (NT >= 4 || MTM > 2)>(p, u, s0, pi0, part, parts, lds);
        else slab_pass<NT, 1, MTM, STREAM, (NT >= 4 || MTM > 2)>(p, u, s0, pi0, part, parts, lds);
    }
}

// NT: 16-rank tiles of the launch (ranks up to 16 NT); MTM: 16-row tiles of its tallest unit.  (Spilled registers: four rank tiles with four
// row tiles 16, or 19 where g and h are left as operands; eight rank tiles 26 in groups, 35 else; the others none.)
template <int NT, int MTM, bool STREAM, class PP>
__global__ __launch_bounds__(kThreads) void slab_kernel(PP p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    __shared__ int s_slot[2];
    auto sg = load_segs(p);
    const SlabPlan pl = slab_plan(p, sg, 16 * MTM);
    ClassScan cc = pl.cc;
    // Workgroups are dealt to the 8 XCDs in turn (workgroup i runs on XCD i % 8), and every XCD has its own L2.  The
    // chunks are numbered segment by segment, so XCD x takes the x-th eighth of them: the slabs of one segment then
    // sit on one XCD (or two) and find their adapter's matrices in its L2, instead of every XCD fetching every adapter.
    // A batch with few chunks is also cut by columns: every part of a chunk repeats phase 1 and takes its share of
    // the column blocks in phase 2; the parts of one chunk get ids r, r + 8, ..., the same XCD again.
    const int n8 = (cc.total + 7) >> 3;  // chunks per XCD
    const int parts = pl.parts;
    const int n_units = 8 * n8 * parts;
    int* stash = reinterpret_cast<int*>(lds_raw + kStashOffset);
    for_each_unit(p.tickets + 0, n_units, s_slot, [&](int gid, int) {
        int slot = gid, part = 0;
        if (parts > 1) {
            const int blk = small_div(gid, 8 * parts), r = gid - blk * 8 * parts;
            part = r >> 3;
            slot = blk * 8 + (r & 7);
        }
        const int chunk = (slot & 7) * n8 + (slot >> 3);
        if (chunk >= cc.total) return;  // (padding)
        Unit u;
        SegInfo s;
        u.pi = 0;
        if (!slab_find(p, sg, cc, pl.per, chunk, u, s)) return;
        stash_tables(sg, cc, stash);
        slab_unit<NT, MTM, STREAM>(p, u, s, part, parts, lds_raw);  // (has a workgroup barrier after its first step)
        unstash_tables(sg, cc, stash);
    });
}

constexpr float kPartsFromB = 300000.f;  // elements of B (of all layers) from which a wide layer is cut into parts, see slab_plan

template <int NT, int MTM, bool STREAM, class PP>
int slab_grid()
{
    static DeviceGrid cache;
    return cache.get([] { return resident_grid(slab_kernel<NT, MTM, STREAM, PP>, kSlabLdsBytes); });
}

template <int NT, int MTM, bool STREAM, class PP>
hipError_t launch_slab(PP p, float columns, hipStream_t st)
{
    const int grid = slab_grid<NT, MTM, STREAM, PP>();
    const float b = (float)p.max_rank * columns, x_passes = NT >= 4 ? (float)p.n_proj : 1.f;
    p.slab_parts = b >= kPartsFromB ? 0.3f * b * (float)grid / ((float)p.d_in * x_passes) : 0.f;
    p.slab_rows_per_rank = 0.8f * ((float)p.d_in * (float)p.n_proj + columns) / ((float)p.d_in + 2.f * columns);
    return launch_kernel(kKernelSlab, slab_kernel<NT, MTM, STREAM, PP>, dim3(grid), dim3(kThreads), kSlabLdsBytes, st, p);
}

template <class PP>
bool wide_layer(const PP& p, float columns) { return (float)p.max_rank * columns >= kPartsFromB; }

// Four row tiles where a unit can get more than 32 rows (single calls up to rank 64).  A batch of ranks up to 32 whose segments'
// 32-row chunks fit one round of the grid (sum of ceil(rows / 32) <= tokens / 32 + segments) has none to speak of, and the kernel of
// two tiles has half the accumulators to add up and starts sooner: 4864 rows of rank 16, 4096 -> 4096, 28.6 us with four tiles and
// 28.4 with two; where it does not fit, 9000 rows, 44.9 and 47.8.  (Up to rank 64 two tiles gain as little, 40.9 and 40.8 us for 4864
// rows, and adapters of lower rank lose their taller units: 7413 rows of ranks 8 to 64, 14336 -> 4096, 76.8 and 81.9.  A batch of
// up to 4096 rows that does not fit has more than 128 segments; its units were never taller.)
//   By itself two tiles are at most 0.2 us slower for 4864 to 6824 rows of ranks 16 and 32 in nine widths, and up to 0.7 us faster.  Behind gate and
// up as single calls, every layer on operands of its own, `down` of 5632 rows takes 70 us; 66 where every such call had four tiles and non-temporal y, but 70
// again with either alone.
//   Wide layers take taller units in column parts, see slab_plan: not before their 16-row chunks leave room for fewer than
// five parts, with 49 chunks, since the plan wants at least twice as many parts as there is room for: 16 rows of rank 32, 4096 ->
// 14336, 12.5 and 12.0 us, 4000 of rank 64 75.5 and 86.
template <int NT, class PP>
bool tall_units(const PP& p, float columns)
{
    const int segments = p.max_segments < p.n_tokens ? p.max_segments : p.n_tokens;
    if (wide_layer(p, columns) && p.n_tokens / 16 + segments >= 49) return true;
    return p.n_tokens > 4096 && (NT > 2 || p.n_tokens / 32 + segments > slab_grid<NT, 2, false, PP>());
}

// y (dx) non-temporal in long batches, wide layers and groups, from 42 million elements of x and y on (84 MB).  Below, x and y of a few
// calls stay in the 256 MB cache and the policy only takes them from whoever reads them next; above, it keeps y from displacing
// what is used again.  Non-temporal over plain, 260 random calls of such shapes on three sets of operands in turn, mean by million elements: 28
// to 36 1.08 to 1.20, 36 to 42 1.03 to 1.10, 42 to 46 0.93 to 1.02, 46 to 58 0.94 to 1.02 (single calls from 0.81 to 1.5: it depends on where the operands
// lie).  us plain and non-temporal: rank 32, q+k+v of 2048 rows (21 M) 31.4 and 38.4, 4096 -> 14336 of 1500 (28 M) 27.8 and 33.6,
// 1024 -> 4096 of 5632 (29 M) 25.2 and 28.4, q+k+v of 4000 (41 M) 46.0 and 47.6; 4096 -> 14336 of 3000 (55 M) 56.4 and 52.5, q+k+v of 5632
// (58 M) 59.5 and 56.7, 8192 Zipf rows, 4096 -> 11008 (124 M), 110 and 99.  A shorter call with much y loses more than the others
// gain, hence the batch's length: 2097 rows of rank 16, 4096 -> 14336 (39 M), 33.4 and 43.2.
//   A backward call touches x too, behind this launch (42 million of dy, dx and x): 260 random calls, 0.98 to 1.02 from 42 to 60 million, 0.97 to 1.00
// where most rows are fine-tune rows, below 1.02 to 1.08; 5632 rows of rank 32, 4096 -> 1024, among the calls of a decoder layer 5 us less.
//   As in a model, with the base product that writes y in front and a reader of y behind, the sum of the three differs less, and
// either way: 4096 -> 4096 of rank 32, 5632 rows 1.4 us less than plain, 8192 rows 3.9 more, 16384 2.7 more (rank 16 5.1 more);
// q+k+v, 4096 rows 1.7 less, 5632 0.9 more, 16384 4.7 less.
//   (The same for x gains as much alone, nothing on top, and loses what the weight gradients find of dy in the cache: 41 -> 49 us.)
//   Only rows of whole 128-byte lines: 260 random calls, widths multiples of 64 0.92 to 0.99 of the plain policy from 42 million on, multiples
// of 32 0.96 to 1.06 (but with a writer in front and a reader behind 3 to 37 % of the call more), other widths 1.14 to 1.75.
bool streams_y(const FwdParams& p, float columns)
{
    return (p.n_tokens > 4096 || p.n_proj > 1 || wide_layer(p, columns)) && y_traffic(p) >= 42e6f && whole_lines(p);
}

template <int NT, class PP>
hipError_t launch_rank(const PP& p, float columns, bool stream, hipStream_t st)
{
    if constexpr (NT < 8 && !std::is_same_v<PP, FwdParams>)
        if (tall_units<NT>(p, columns)) return stream ? launch_slab<NT, 4, true>(p, columns, st) : launch_slab<NT, 4, false>(p, columns, st);
    return stream ? launch_slab<NT, 2, true>(p, columns, st) : launch_slab<NT, 2, false>(p, columns, st);
}

template <class PP>
hipError_t launch_any(const PP& p, float columns, bool stream, hipStream_t st)
{
    const int nt = nt_for(p.max_rank);
    return nt == 1 ? launch_rank<1>(p, columns, stream, st) : nt == 2 ? launch_rank<2>(p, columns, stream, st)
         : nt == 4 ? launch_rank<4>(p, columns, stream, st) : launch_rank<8>(p, columns, stream, st);
}

}  // namespace

hipError_t run_slab(const FwdParams& p, hipStream_t st, const SlabFrag* frag)
{
    const float columns = all_columns(p);
    const bool stream = streams_y(p, columns);
    if (p.n_proj > 1) return launch_any(p, columns, stream, st);
    if (!frag) return launch_any(static_cast<const FwdCore&>(p), columns, stream, st);
    FwdFrag q;
    static_cast<FwdCore&>(q) = p;
    q.frag = *frag;
    return launch_any(q, columns, stream, st);
}

}  // namespace lq
