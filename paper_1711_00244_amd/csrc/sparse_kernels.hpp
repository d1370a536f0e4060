// decode_layer kernel and the small-batch path: fused decode + sparse multiply, and its finishing kernel.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

// ------------------------------------------------------------------------- //
// decode_layer: symbols and (optionally) the dense matrix
// ------------------------------------------------------------------------- //
// For layers with blocks above 128 x 128, blocks that decode_blocks_kernel gains nothing by (small ones:
// decode_by_blocks) and layers without the chunk slots it reads: a wavefront per chunk, eight to a
// workgroup, after fill_kernel has cleared the dense matrix.
__global__ __launch_bounds__(kThreads) void decode_kernel(LayerDev L, uint8_t *val_out, uint8_t *idx_out, float *dense)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const Smem s = carve(smem_raw, L);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const uint32_t c = blockIdx.x * kWaves + (uint32_t)wave;
    const bool have = c < L.n_chunks;
    ChunkHead h{};
    LaneRecord rec{};
    if (have) {
        h = load_head(L, c);
        rec = load_record(L, h, lane);
    }
    store_tables(s, L, fetch_tables(L));
    __syncthreads();
    if (!have) return;
    const Symbols y = decode_record(rec, s.T);
    const LaneStart st = lane_starts(y, h.m.pos0);
    const BlockGeom g = block_geom(L, h.m.blk);
    const uint32_t e0 = h.m.sym_off + st.entry;
    for_each_entry(y, st.sum, [&](uint32_t j, uint32_t v, uint32_t z, uint32_t pos) {
        if (val_out) val_out[e0 + j] = (uint8_t)v;
        if (idx_out) idx_out[e0 + j] = (uint8_t)z;
        if (dense && v != 0 && pos < (uint32_t)g.bhp * (uint32_t)g.bwp) {
            uint32_t r, cc;
            split_pos(pos, g, r, cc);
            dense[(size_t)(g.row_id + (int)r) * L.K + (size_t)(g.col_id + (int)cc)] = s.T.cb[v];
        }
    });
}

// The same for the other layers, whose blocks are at most 128 x 128, everything in one launch: a workgroup
// takes block after block.  A wavefront decodes a chunk of the block and leaves its symbols in
// LDS - value and relative indices in entry order, and the value index once more in a byte
// tile of the block, at its position; then the workgroup writes the block out, dense rows (zeros
// with the rest) and symbols in whole 16-byte pieces, having asked for the next block's
// records first.  Bound by the bytes written: every byte of the outputs is written once, in
// whole lines where the rows of a block begin on one.  The dense matrix goes through the caches: stores that leave it no
// room there take the call itself from 37 to 34 us for 151 MB written to a buffer that was not used just before, but from
// 30 to 34 for one that was, and what reads the matrix next then waits for memory (us for the call and a product
// with one vector, through the caches / past them: 101 MB 42-47 / 54-58, 151 MB in one buffer 59 / 78).
constexpr int kDecodeThreads = 256, kDecodeTile = 128 * 128;

__global__ __launch_bounds__(kDecodeThreads) void decode_blocks_kernel(LayerDev L, const uint32_t *block_ptr, int blocks, uint8_t *val_out, uint8_t *idx_out,
                                                                       uint32_t *ptr_out, float *dense, int stage_bytes)
{
    constexpr int NW = kDecodeThreads / 64;
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const Smem s = carve(smem_raw, L);
    uint8_t *tile = (uint8_t *)s.extra;                     // value index of every position of the block
    uint8_t *stage[2] = {tile + kDecodeTile, tile + kDecodeTile + stage_bytes};        // value, relative indices
    uint8_t *const out[2] = {val_out, idx_out};
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // what a wavefront decodes next: chunk `wave` of a block, by its slot
    ChunkSlot ch{};
    uint64_t rec = 0;
    uint32_t e0 = 0, e1 = 0, first = 0;                     // the block's entries; the chunk's first one
    auto fetch_chunk = [&](int b, int i) {
        ch = L.slot[(size_t)b * (uint32_t)L.block_slots + (uint32_t)i];
        if (ch.nrec == 0) return;
        first = L.meta[L.block_chunk[b] + (uint32_t)i].sym_off;
        rec = (uint32_t)lane < ch.nrec ? L.records[(size_t)ch.rec_off + lane] : 0ull;
    };
    auto fetch_block = [&](int b) {
        ch.nrec = 0;
        if (b >= blocks) return;
        e0 = block_ptr[b];
        e1 = block_ptr[b + 1];
        if (wave < L.block_slots) fetch_chunk(b, wave);
    };

    fetch_block((int)blockIdx.x);
    for (int i = tid; i < L.table_rows; i += kDecodeThreads) s.tables[i] = L.tables[i];
    for (int i = tid; i < kDecodeTile / 16; i += kDecodeThreads) ((u4 *)tile)[i] = u4{0, 0, 0, 0};
    if (ptr_out && blockIdx.x == 0 && tid == 0) ptr_out[blocks] = block_ptr[blocks];
    __syncthreads();
    for (int b = (int)blockIdx.x; b < blocks; b += (int)gridDim.x) {
        const uint32_t at0 = e0, n = e1 - e0;
        // the stages begin where their first 16-byte piece does in memory
        const uint32_t mis[2] = {val_out ? (uint32_t)(uintptr_t)(val_out + at0) & 15u : 0u, idx_out ? (uint32_t)(uintptr_t)(idx_out + at0) & 15u : 0u};
        for (int i = wave; ch.nrec != 0;) {
            const Symbols y = decode_record(split_record(rec, (uint32_t)rec & 15u), s.T);
            const LaneStart st = lane_starts(y, ch.pos0);
            const uint32_t at = first - at0 + st.entry;
            for_each_entry(y, st.sum, [&](uint32_t j, uint32_t v, uint32_t z, uint32_t pos) {
                stage[0][mis[0] + at + j] = (uint8_t)v;
                stage[1][mis[1] + at + j] = (uint8_t)z;
                tile[pos] = (uint8_t)v;                     // (padding: zero, at a position of its own)
            });
            i += NW;
            if (i >= L.block_slots) break;
            fetch_chunk(b, i);
        }
        __syncthreads();
        fetch_block(b + (int)gridDim.x);
        if (ptr_out && tid == 0) ptr_out[b] = at0;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (!out[a]) continue;
            uint8_t *dst = out[a] + at0 - mis[a];
            for (uint32_t p = 16u * (uint32_t)tid; p < mis[a] + n; p += 16u * kDecodeThreads) {
                if (p >= mis[a] && p + 16u <= mis[a] + n) *(u4 *)(dst + p) = *(const u4 *)(stage[a] + p);
                else
                    for (uint32_t q = max(p, mis[a]); q < min(p + 16u, mis[a] + n); ++q) dst[q] = stage[a][q];
            }
        }
        // the dense rows; what has been read of the tile is cleared for the next block
        const BlockGeom g = block_geom(L, (uint32_t)b);
        if (!dense) {
            for (int i = tid; i < (g.bhp * g.bwp + 15) / 16; i += kDecodeThreads) ((u4 *)tile)[i] = u4{0, 0, 0, 0};
        } else if (((L.K | L.bw | g.bwp) & 3) == 0 && ((uintptr_t)dense & 15u) == 0) {
            const int c = (tid & 31) * 4;
            float *dst = dense + (size_t)g.row_id * L.K + g.col_id + c;
            if (c < g.bwp) {
#pragma unroll 4
                for (int r = tid >> 5; r < g.bhp; r += kDecodeThreads / 32) {
                    uint32_t *t = (uint32_t *)(tile + r * g.bwp + c);
                    const uint32_t v = *t;
                    *t = 0u;
                    *(f4 *)(dst + (size_t)r * L.K) = f4{s.T.cb[v & 255u], s.T.cb[(v >> 8) & 255u], s.T.cb[(v >> 16) & 255u], s.T.cb[v >> 24]};
                }
            }
        } else {
            const int c = tid & 127;
            if (c < g.bwp)
                for (int r = tid >> 7; r < g.bhp; r += kDecodeThreads / 128) {
                    const uint8_t v = tile[r * g.bwp + c];
                    tile[r * g.bwp + c] = 0;
                    dense[(size_t)(g.row_id + r) * L.K + g.col_id + c] = s.T.cb[v];
                }
        }
        __syncthreads();
    }
}

__global__ void fill_kernel(float *p, size_t n, float v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// ------------------------------------------------------------------------- //
// fused decode + sparse multiply (small batches)
// ------------------------------------------------------------------------- //
// Workgroup j of block row p takes chunks [8 j, 8 j + 8) of that block row, one per
// wavefront, and accumulates w * x into an LDS tile of the bh x BT outputs of the
// block row (Algorithm 2 step 12, b[row_id : row_id + bh, :] += block * a[col_id :
// col_id + bw, :]); the tile then goes to the workgroup's slot of `part`, and a
// second kernel adds the slots of a block row up.  A lane's entries run along a
// row of the block, so it sums w * x in registers and touches the tile only when
// the row changes.  The activation columns of the blocks the workgroup's chunks
// belong to are staged in LDS first when they fit xcap columns; otherwise they are
// read from global memory.  A padding entry carries codebook value 0 and adds 0.
// Where a layer's input comes from when the layer before it ran on this path too and
// its finishing kernel is left out (a stack of layers at one image, where a launch costs
// as much as the work in it): the partial tiles of that layer's
// workgroups, part[block row][slot][image][row], to be added up in slot order, plus its
// bias, through its activation (Eq. 1) - what fc_reduce_kernel would have written as
// X[image][k], taken by each workgroup for the columns of its own slab only.
struct PrevSlots {
    const float *part;              // null: the input is X
    const uint32_t *panel_chunk;    // of the layer before: how many slots each of its block rows filled
    const float *bias;              // of the layer before, or null
    Divisor bh;
    int wg_per_panel, part_b, relu;
};

// Where fc_sparse_whole_kernel's outputs go.
struct WholeOut {
    const float *bias;              // or null
    float *Y;                       // of the first image of the batch tile
    int relu;
};

// Threads of fc_reduce_body's workgroups, and slices they form beside each other for a block row of `rows` rows.
constexpr int kRedThreads = 512;
__host__ __device__ constexpr int reduce_slices(int rows) { return kRedThreads / (rows < kRedThreads ? (rows + 63) / 64 * 64 : kRedThreads); }

// Up to this batch tile, and for block rows of up to 256 rows, every wavefront of the small-
// batch kernel has an output tile of its own in LDS and writes each row sum once, with a
// plain store (see fc_sparse_body); above, the workgroup shares one tile through float atomics
// (8 x bh x BT floats would crowd the CU, and those batch sizes belong to the tile kernels).
constexpr int kPrivateTileBT = 8;
__host__ __device__ constexpr bool private_tiles(int bh, int bt) { return bt <= kPrivateTileBT && bh <= kPrivateTileRows; }

// Where a column's BT images lie in the LDS slab: as 16-byte groups of four, and for BT > 4 the
// groups of a column rotated by the column number.  Lanes that read group g of 64 arbitrary
// columns then spread over all 32 banks; unrotated, a column stride of 32 or 64 bytes would put
// them on half or a quarter of the banks.
template <int BT> __device__ __forceinline__ int x_group(int col, int g)
{
    if constexpr (BT == 8) return (g + (col >> 2)) & 1;
    else if constexpr (BT == 16) return (g + (col >> 1)) & 3;
    else return g;
}

// Inclusive sums over the lanes of a wavefront in segments: a lane with `start` begins a
// segment.  (value, started) pairs combine as (b.started ? b.value : a.value + b.value,
// a.started | b.started), which is associative, so the usual doubling steps apply.
template <int BT>
__device__ __forceinline__ void wave_segmented_sums(float (&v)[BT], bool start)
{
    uint32_t f = start ? 1u : 0u;
#define CL_SEG_STEP(CTRL, ROWS)                                                                              \
    {                                                                                                        \
        const uint32_t tf = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, CTRL, ROWS, 0xf, false);        \
        _Pragma("unroll") for (int b = 0; b < BT; ++b)                                                       \
        {                                                                                                    \
            const float tv = __builtin_bit_cast(                                                             \
                float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[b]), CTRL, ROWS, 0xf, false)); \
            v[b] = f ? v[b] : v[b] + tv;                                                                     \
        }                                                                                                    \
        f |= tf;                                                                                             \
    }
    CL_SEG_STEP(0x111, 0xf)   // row_shr:1
    CL_SEG_STEP(0x112, 0xf)   // row_shr:2
    CL_SEG_STEP(0x114, 0xf)   // row_shr:4
    CL_SEG_STEP(0x118, 0xf)   // row_shr:8
    CL_SEG_STEP(0x142, 0xa)   // row_bcast:15 into rows 1, 3
    CL_SEG_STEP(0x143, 0xc)   // row_bcast:31 into rows 2, 3
#undef CL_SEG_STEP
}

// An entry of a record on its way to its row's sum: looked up, not yet waited for.
template <int BT> struct Pending {
    float w, x[BT];
    uint32_t row;
};

// A record decoded and used in one pass: entry after entry, both codeword streams side by side.  The position of an
// entry is where the record starts (a table, counted when the layer was loaded) plus what the entries before
// it advance, so an entry is looked up - its weight, its column's activations - as soon as it is
// decoded, and used one entry later, while the next one's table reads are on their way.
// at: the position of the entry before (the record's start less one); in SHIFTED form it is in the bits from 8 up:
// a table entry has its symbol in the second byte and its length below, and added up as they are, with 256 per
// entry, they move the position on (fifteen lengths of at most twelve bits do not reach bit 8).  Every lane goes on
// to the wavefront's longest record; use(entry number, entry) is for the lane's own entries to heed.
template <int BT, bool SHIFTED, class Look, class Use>
__device__ __forceinline__ void entries_in_one_pass(LaneRecord &rec, const Tables &T, uint32_t nmax, uint32_t at, Look look, Use use)
{
    auto next = [&](Pending<BT> &e) {
        const uint32_t ez = next_entry(rec.ibuf, T.ibase, T.imask);
        const uint32_t ev = next_entry(rec.vbuf, T.vbase, T.vmask);
        at += SHIFTED ? ez + 256u : (ez >> 8) + 1u;
        look(at, ev, e);
    };
    Pending<BT> a, b;                                       // (two take turns: nothing is moved)
    uint32_t j = 0;
    next(a);
#pragma unroll 1
    for (; j + 2 < nmax; j += 2) {                          // uniform
        next(b);
        use(j, a);
        next(a);
        use(j + 1, b);
    }
    if (j + 1 < nmax) {
        next(b);
        use(j, a);
        use(j + 1, b);
    } else use(j, a);
}

// (wg: the workgroup's number within the layer's share of the grid; nb <= BT: images that X
// holds - the tile's other images are zeros; FOLD: the input may be the partial tiles of the
// layer before - an instantiation of its own, so that the code for it does not weigh on the
// registers of the others; ONE_PASS: see entries_private; WHOLE: the workgroup, of NW wavefronts with R chunks each, has all
// chunks of the block row and finishes the output itself, see fc_sparse_whole_kernel)
template <int BT, bool FOLD, bool ONE_PASS, bool WHOLE = false, int NW = kWaves, int R = kSparseChunksPerWave>
__device__ __forceinline__ void fc_sparse_body(const LayerDev &L, const float *__restrict__ X, float *part, const Divisor &wg_per_panel,
                                               int xcap, const PrevSlots &prev, uint32_t wg, int nb, const WholeOut &whole = WholeOut{nullptr, nullptr, 0})
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const Smem s = carve(smem_raw, L);
    // Everything the prologue waits for is requested before anything of it is touched: the table image, which needs nothing,
    // then chunk heads, records and their positions, then activations.  (Many layers in one grid gain
    // by it, one layer's launch 1 %: its other workgroups fill the time.)
    TableRegs tr;
    const bool copies = NW == kWaves || threadIdx.x < kThreads;         // the table image is copied by kThreads threads
    if (copies) tr = fetch_tables(L);
    const int p = (int)wg_per_panel.quotient(wg), j = (int)(wg - (uint32_t)p * wg_per_panel.d);
    const uint32_t pc1 = L.panel_chunk[p + 1];
    const uint32_t my0 = L.panel_chunk[p] + (uint32_t)j * (NW * R);
    if (!WHOLE && my0 >= pc1) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    // activation columns of the blocks this workgroup's chunks belong to
    const uint32_t pb0 = (uint32_t)p * (uint32_t)L.nbw;
    const uint32_t blk_a = WHOLE ? 0 : L.meta[my0].blk, blk_b = WHOLE ? 0 : L.meta[min(pc1, my0 + (uint32_t)(NW * R)) - 1u].blk;
    // wavefront w takes chunks my0 + w, my0 + 8 + w, ...
    bool have[R];
    ChunkHead h[R];
    uint64_t word[R];                                                   // the lane's records, as they are stored
    uint32_t rec_pos[R];
    const bool priv = private_tiles(L.bh, BT);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t c = my0 + (uint32_t)(i * NW + wave);
        have[i] = c < pc1;
        h[i] = ChunkHead{};
        word[i] = 0;
        rec_pos[i] = 0;
        // (a chunk past the block row's last: that one's head, so that heads are asked for without a branch; a block row always has one but where
        // a workgroup has the whole of it)
        if (!WHOLE || have[i]) h[i] = load_head(L, WHOLE ? c : min(c, pc1 - 1u));
        if (have[i]) {
            if ((uint32_t)lane < h[i].nrec) {
                const size_t r = (size_t)h[i].m.rec_off + lane;
                word[i] = L.records[r];
                if (priv) rec_pos[i] = L.pos32 ? ((const uint32_t *)L.rec_pos)[r] : ((const uint16_t *)L.rec_pos)[r];
            }
        }
    }
    const int n_tiles = WHOLE ? (int)((pc1 - my0 + kWaves - 1) / kWaves * kWaves) : priv ? kWaves : 1;
    float *ytile = s.extra;                  // [n_tiles][BT][bh]
    float *xs = ytile + (size_t)n_tiles * L.bh * BT;   // [xcap][BT]: a column's BT images side by side, one LDS read per entry
    const int col_a = WHOLE ? 0 : (int)(blk_a - pb0) * L.bw;
    const int col_b = WHOLE ? L.K : min(L.K, (int)(blk_b - pb0 + 1u) * L.bw);
    const int width = col_b - col_a;
    const bool slab = WHOLE || width <= xcap;
    const bool fold = FOLD && slab && prev.part;
    float x0[BT];                                                       // the thread's first column of the slab
#pragma unroll
    for (int b = 0; b < BT; ++b) x0[b] = 0.0f;
    if (slab && !fold && (int)threadIdx.x < width) {
#pragma unroll
        for (int b = 0; b < BT; ++b)
            if (b < nb) x0[b] = X[(size_t)b * L.K + col_a + threadIdx.x];
    }
    if (fold) {
        // (the host takes this form only for layers whose every workgroup has a slab)
        constexpr uint32_t kPerWg = kWaves * kSparseChunksPerWave;
        for (int t = threadIdx.x; t < width; t += blockDim.x) {
            const uint32_t k = (uint32_t)(col_a + t), pp = prev.bh.quotient(k), r = k - pp * prev.bh.d;
            const int active = (int)((prev.panel_chunk[pp + 1] - prev.panel_chunk[pp] + kPerWg - 1) / kPerWg);
            const float *src = prev.part + (size_t)pp * prev.wg_per_panel * prev.part_b * prev.bh.d + r;
            const size_t step = (size_t)prev.part_b * prev.bh.d;
            const float bv = prev.bias ? prev.bias[k] : 0.0f;
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                float acc = 0.0f;
                for (int j = 0; j < active; j += 12) {      // twelve loads in flight, added in slot order
                    float a[12];
#pragma unroll
                    for (int u = 0; u < 12; ++u) a[u] = src[(size_t)(j + u < active ? j + u : j) * step + (size_t)b * prev.bh.d];
#pragma unroll
                    for (int u = 0; u < 12; ++u)
                        if (j + u < active) acc += a[u];
                }
                acc += bv;
                xs[t * BT + b] = prev.relu ? fmaxf(acc, 0.0f) : acc;
            }
        }
    }
    // (16 bytes at a time, and four outputs per thread at the end, pay from four images on -
    // measured; below, they cost a microsecond of a step)
    if (BT >= 4) {
        const int n = n_tiles * L.bh * BT;          // a multiple of 4
        float4 *z4 = (float4 *)ytile;
        for (int t = threadIdx.x; t < n / 4; t += blockDim.x) z4[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        for (int t = threadIdx.x; t < n_tiles * L.bh * BT; t += blockDim.x) ytile[t] = 0.0f;
    }
    if (copies) store_tables(s, L, tr);
    if (slab && !fold) {
        // a column's images are stored together
        auto store_column = [&](int t, const float (&v)[BT]) {
            constexpr int kW = BT < 4 ? BT : 4;
#pragma unroll
            for (int q = 0; q < BT / kW; ++q) store_floats<kW>(xs + t * BT + x_group<BT>(t, q) * kW, v + q * kW);
        };
        if ((int)threadIdx.x < width) store_column((int)threadIdx.x, x0);
        for (int t = threadIdx.x + blockDim.x; t < width; t += blockDim.x) {
            float v[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) v[b] = b < nb ? X[(size_t)b * L.K + col_a + t] : 0.0f;
            store_column(t, v);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (!have[i]) continue;
        const BlockGeom g = block_geom(L, p, (int)(h[i].m.blk - pb0));
        LaneRecord rec = split_record(word[i], (uint32_t)word[i] & 15u);
        // The entries of the record in order, in every lane up to the wavefront's longest
        // record: a lane past its own entries multiplies codebook entry 0 with a column
        // of the block.  The instantiations differ in where the activations come from
        // (LDS stays LDS: no generic pointers) and in how a position splits into row and
        // column (shift and mask for a power-of-two block width).
        auto entries_shared = [&](auto load_x, auto split) {
            // (a count of its own: what the decode makes of it would otherwise be worked out ahead of every form)
            asm volatile("" : "+v"(rec.n));
            const Symbols y = decode_record(rec, s.T);
            const LaneStart st = lane_starts(y, h[i].m.pos0);
            uint32_t cur = 0;
            float acc[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) acc[b] = 0.0f;
            for_each_entry<true>(y, st.sum, [&](uint32_t, uint32_t v, uint32_t, uint32_t pos) {
                uint32_t r, cc;
                split(pos, r, cc);
                if (r != cur) {
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        atomicAdd(ytile + b * L.bh + cur, acc[b]);
                        acc[b] = 0.0f;
                    }
                    cur = r;
                }
                const float w = s.T.cb[v];
                float x[BT];
                load_x((int)cc, x);
#pragma unroll
                for (int b = 0; b < BT; ++b) acc[b] += w * x[b];
            });
#pragma unroll
            for (int b = 0; b < BT; ++b) atomicAdd(ytile + b * L.bh + cur, acc[b]);
        };
        // The same into the wavefront's own tile, without atomics (an LDS float atomic costs about
        // three cycles per lane here: half of the kernel at four images).  The chunk's entries
        // run row by row across the lanes, so a row's terms sit in one lane or in a run of
        // neighbouring lanes: a row that begins and ends inside a lane is stored by that lane; a
        // lane's first row may continue the previous lane's last one, and the run of lanes that
        // have nothing but that row is summed with a segmented scan - the row is then stored
        // once, by the lane where it ends.  No two lanes store the same row, and the tile
        // receives this chunk only, so plain stores do.
        auto entries_private = [&](auto shifted, auto load_x, auto split) {
            constexpr uint32_t kNone = 0xffffffffu;
            float *tile = ytile + (size_t)(i * NW + wave) * L.bh * BT;     // (one chunk to a tile: plain stores)
            uint32_t first_row = kNone, cur = kNone;    // the rows of the lane's first entry and of its last so far (kNone: no record)
            float acc[BT], head[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) acc[b] = head[b] = 0.0f;
            // A change of row: the sum so far is stored, except the first one, which is kept - the
            // first row may have begun in the lanes before.  For one and two images that
            // distinction costs more than it saves: every sum is stored, the first row's too, and
            // that one is read back after the loop and written over with the sum over all its
            // lanes (one image: 33.9 -> 32.5 us per step of the
            // AlexNet-shaped stack; four images: 42.2 -> 43.2, so not there).
            auto use = [&](const Pending<BT> &e) {
                if (e.row != cur) {
                    const bool several = cur != first_row;          // the lane had left its first row before
                    if (BT <= 2 || several) {
#pragma unroll
                        for (int b = 0; b < BT; ++b) tile[b * L.bh + cur] = acc[b];
                    }
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        if (BT > 2) head[b] = several ? head[b] : acc[b];
                        acc[b] = 0.0f;
                    }
                    cur = e.row;
                }
#pragma unroll
                for (int b = 0; b < BT; ++b) acc[b] += e.w * e.x[b];
            };
            // In one pass, but for a layer of its own at eight images: there a wavefront's time is the latency of its reads, of
            // which one entry at a time (32 bytes of activations) is not enough to hide it, and a pass that decodes and one that
            // takes three entries at a time are a little shorter; where many layers share the grid, instructions bound
            // it (us a call, before / one pass / two passes: FC 4096 x 9216 at eight images 23.5 / 24.7 / 23.1, AlexNet-shaped
            // stack at eight 49.9 / 51.9 / 49.7, at four 41.0 / 37.0 / -, at one 31.5 / 28.6 / -; sixteen layers of
            // 4096 x 4096 in one grid at one image 59.7 / 50.2 / -, at four 80.3 / 66.2 / -, at eight 124.1 / 121.3 / 129.8).
            if constexpr (ONE_PASS) {
                const uint32_t n = rec.n;
                bool first = true;                          // no entry looked up yet
                auto look = [&](uint32_t at, uint32_t ev, Pending<BT> &e) {
                    uint32_t cc;
                    split(at, e.row, cc);
                    e.w = *(const float *)((const char *)s.T.cb + (ev >> 6));       // (lengths are below 64: the symbol's word)
                    if (first) first_row = cur = n > 0 ? e.row : kNone;
                    first = false;
                    load_x((int)cc, e.x);
                };
                Tables V = s.T;                             // (the masks in vector registers: an and-or takes one scalar operand)
                asm("" : "+v"(V.vmask), "+v"(V.imask));
                entries_in_one_pass<BT, shifted>(rec, V, wave_max(n), (rec_pos[i] - 1u) << (shifted ? 8 : 0), look,
                                                 [&](uint32_t j, const Pending<BT> &e) { if (j < n) use(e); });
            } else {
                const Symbols y = decode_symbols(rec, s.T);
                auto split_at = [&](uint32_t pos, uint32_t &r, uint32_t &cc) { split(shifted ? pos << 8 : pos, r, cc); };
                if (y.n > 0) {
                    uint32_t unused;
                    split_at(rec_pos[i] + (y.z[0] & 0xffu), first_row, unused);
                    cur = first_row;
                }
                // the codebook and activation reads of three entries go out together: the row logic
                // is all branches, behind which the compiler leaves each read where it is used
                constexpr int G = 3;
                Pending<BT> e[G];
                for_each_entry_grouped<G>(y, rec_pos[i], [&](int u, uint32_t v, uint32_t pos) {
                    uint32_t cc;
                    split_at(pos, e[u].row, cc);
                    e[u].w = s.T.cb[v];
                    load_x((int)cc, e[u].x);
                }, [&](int u) { use(e[u]); });
            }
            // cur: the lane's last row (kNone for a lane without a record), acc its sum so far
            const bool several = cur != first_row;
            // (every lane takes part in the exchange: a lane that sat it out would hand its
            // neighbour a zero)
            const uint32_t from_prev = (uint32_t)__shfl_up((int)cur, 1), from_next = (uint32_t)__shfl_down((int)first_row, 1);
            const uint32_t prev_last = lane == 0 ? kNone : from_prev;
            const uint32_t next_first = lane == 63 ? kNone : from_next;
            const bool joins = first_row != kNone && first_row == prev_last;
            wave_segmented_sums<BT>(acc, !(joins && !several));
            float before[BT];                           // the run that ends in the lane before
#pragma unroll
            for (int b = 0; b < BT; ++b) before[b] = __shfl_up(acc[b], 1);
            if (several) {
#pragma unroll
                for (int b = 0; b < BT; ++b) {
                    if (BT <= 2) head[b] = tile[b * L.bh + first_row];       // (stored in the loop, by this lane)
                    tile[b * L.bh + first_row] = joins ? head[b] + before[b] : head[b];
                }
            }
            if (cur != kNone && next_first != cur) {
#pragma unroll
                for (int b = 0; b < BT; ++b) tile[b * L.bh + cur] = acc[b];
            }
        };
        auto with_split = [&](auto load_x) {
            const uint32_t sh = (uint32_t)g.shift, cmask = (uint32_t)g.bwp - 1u, rmax = (uint32_t)g.bhp - 1u;
            // (rows are used for a lane's own entries only in one pass, and those lie inside the block: checked when the
            // layer was loaded)
            if (WHOLE && !L.pos32 && g.shift >= 0)
                entries_private(std::true_type{}, load_x, [&](uint32_t at, uint32_t &r, uint32_t &cc) { r = at >> (8u + sh); cc = __builtin_amdgcn_ubfe(at, 8u, sh); });
            else if (WHOLE) entries_private(std::false_type{}, load_x, [&](uint32_t pos, uint32_t &r, uint32_t &cc) { split_pos(pos, g, r, cc); });
            else if (priv && L.pos32) entries_private(std::false_type{}, load_x, [&](uint32_t pos, uint32_t &r, uint32_t &cc) { split_pos(pos, g, r, cc); });
            else if (priv && g.shift >= 0)
                entries_private(std::true_type{}, load_x, [&](uint32_t at, uint32_t &r, uint32_t &cc) { r = at >> (8u + sh); cc = __builtin_amdgcn_ubfe(at, 8u, sh); });
            else if (priv) entries_private(std::true_type{}, load_x, [&](uint32_t at, uint32_t &r, uint32_t &cc) { split_pos(at >> 8, g, r, cc); });
            else if (g.shift >= 0) entries_shared(load_x, [&](uint32_t pos, uint32_t &r, uint32_t &cc) { r = min(pos >> sh, rmax); cc = pos & cmask; });
            else entries_shared(load_x, [&](uint32_t pos, uint32_t &r, uint32_t &cc) { split_pos(pos, g, r, cc); });
        };
        if (slab) {
            const int xoff = g.col_id - col_a;
            with_split([&](int cc, float (&x)[BT]) {
                constexpr int kW = BT < 4 ? BT : 4;
#pragma unroll
                for (int q = 0; q < BT / kW; ++q) load_floats<kW>(xs + (xoff + cc) * BT + x_group<BT>(xoff + cc, q) * kW, x + q * kW);
            });
        } else {
            const float *xg = X + g.col_id;
            with_split([&](int cc, float (&x)[BT]) {
#pragma unroll
                for (int b = 0; b < BT; ++b) x[b] = b < nb ? xg[(size_t)b * L.K + cc] : 0.0f;
            });
        }
    }
    __syncthreads();
    if constexpr (WHOLE) {
        // the tiles eight by eight, then these sums as fc_reduce_body adds the workgroups' tiles up: to the last bit what
        // the two launches give
        const int slots = n_tiles / kWaves, slices = reduce_slices(min(L.bh, L.M - p * L.bh)), row_id = p * L.bh;
        for (int t = threadIdx.x; t < L.bh * nb; t += blockDim.x) {
            const int b = t / L.bh, m = row_id + t - b * L.bh;
            if (m >= L.M) continue;
            float y = 0.0f;
            for (int sl = 0; sl < min(slices, max(slots, 1)); ++sl) {
                float acc = 0.0f;
                for (int k = sl; k < slots; k += slices) {
                    const float *tile = ytile + (size_t)k * kWaves * L.bh * BT + t;
                    float sum = tile[0];
#pragma unroll
                    for (int w = 1; w < kWaves; ++w) sum += tile[(size_t)w * L.bh * BT];
                    acc += sum;
                }
                y = sl == 0 ? acc : y + acc;
            }
            if (whole.bias) y += whole.bias[m];
            whole.Y[(size_t)b * L.M + m] = whole.relu ? fmaxf(y, 0.0f) : y;
        }
        return;
    }
    float *mine = part + (size_t)wg * L.bh * BT;
    // (tiles added in wavefront order: the same every run; four outputs per thread where a tile's size allows)
    const int per_tile = L.bh * BT;
    if (BT >= 4) {
        for (int t = threadIdx.x; t < per_tile / 4; t += blockDim.x) {
            float4 v[kWaves];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v[w] = w < n_tiles ? ((const float4 *)(ytile + (size_t)w * per_tile))[t] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float4 sum = v[0];
#pragma unroll
            for (int w = 1; w < kWaves; ++w)
                if (w < n_tiles) { sum.x += v[w].x; sum.y += v[w].y; sum.z += v[w].z; sum.w += v[w].w; }
            ((float4 *)mine)[t] = sum;
        }
    } else {
        for (int t = threadIdx.x; t < per_tile; t += blockDim.x) {
            float sum = ytile[t];
            for (int w = 1; w < n_tiles; ++w) sum += ytile[(size_t)w * per_tile + t];
            mine[t] = sum;
        }
    }
}

template <int BT, bool FOLD>
__global__ __launch_bounds__(kThreads) void fc_sparse_kernel(LayerDev L, const float *__restrict__ X, float *part,
                                                             Divisor wg_per_panel, int xcap, PrevSlots prev, int nb)
{
    constexpr bool kOnePass = BT <= 4;
    fc_sparse_body<BT, FOLD, kOnePass>(L, X, part, wg_per_panel, xcap, prev, blockIdx.x, nb);
}

// A small layer in one launch: a workgroup of sixteen wavefronts takes a whole block row, up to three chunks a wavefront, each
// into a tile of its own, stages all activations, and finishes the output, so that there are no partial tiles and
// nothing to add up in a second launch.  Bound by the latencies of a chunk, one after the other.  With a chunk to a wavefront it
// is shorter on the GPU than the two launches (us, one image: 256 x 256 at 20 % 4.9 / 7.0, 1024 x 384 at 10 %, 15 chunks to a block row, 5.0 / 6.8);
// with two it is about as long, with three longer (1024 x 1024 at 10 %, 40 chunks to a block row, 8.5 / 7.1), and gains only where the
// host's work for its launches bounds the calls (that layer, call behind call from Python: 11.7 -> 9.1): whole_extra decides.
constexpr int kWholeWaves = 16, kWholeRounds = 3, kWholeBT = 4;

template <int BT>
__global__ __launch_bounds__(kWholeWaves * 64) void fc_sparse_whole_kernel(LayerDev L, const float *__restrict__ X, WholeOut out, int nb)
{
    fc_sparse_body<BT, false, true, true, kWholeWaves, kWholeRounds>(L, X, nullptr, Divisor{1, 0, 0, 1}, 0, PrevSlots{},
                                                                    blockIdx.x, nb, out);
}

// Several layers of one shape in one grid (the same layer of several models, or layers
// whose inputs do not depend on each other): workgroups wgs_per_layer i ..
// wgs_per_layer (i + 1) - 1 do layer i's share of Algorithm 2, from its own input
// (x_stride floats apart; 0: one input for all) into its own partial tiles.  Bound by vector issue, so what every lane need not work out
// for itself weighs: with the layer's pointers as they come from `table` (in_global) chunk heads and block geometry were vector values,
// and each load waited for the one before (sixteen layers of 4096 x 4096 at 9 %, one image: 49.9 -> 43.6 us a call).
template <int BT>
__global__ __launch_bounds__(kThreads) void fc_sparse_group_kernel(const LayerDev *__restrict__ table, Divisor wgs_per_layer,
                                                                   const float *__restrict__ X, size_t x_stride, float *part,
                                                                   size_t part_stride, Divisor wg_per_panel, int xcap)
{
    const uint32_t job = wgs_per_layer.quotient(blockIdx.x), wg = blockIdx.x - job * wgs_per_layer.d;
    const LayerDev L = in_global(table[job]);
    fc_sparse_body<BT, false, true>(L, X + job * x_stride, part + job * part_stride, wg_per_panel, xcap,
                       PrevSlots{}, wg, BT);
}

// Finishes the sparse path: adds up the partial tiles of each block row in a fixed
// order, then bias and activation (Eq. 1): Y[b][row] = act(sum_j part[p][j][b][r] + v[row]).
// One workgroup per (block row, image).  The kernel is a chain of memory latencies and
// nothing else, so it is laid out to have few links: the threads form as many groups
// (slices) as fit next to one pass over the rows, slice s adds slots s, s + slices, ...
// with twelve loads in flight, LDS adds the slices in order.
__device__ __forceinline__ void fc_reduce_body(const LayerDev &L, const float *__restrict__ part, const float *__restrict__ bias,
                                               float *Y, int B, int part_b, int wg_per_panel, int relu, int wg)
{
    __shared__ float slice_sum[kRedThreads];
    const int p = __builtin_amdgcn_readfirstlane(wg / B), b = wg - p * B;       // (uniform: said so, or its table entries come by vector loads)
    const int row_id = p * L.bh;
    const int bhp = min(L.bh, L.M - row_id);
    // the sparse kernel fills one slot per workgroup's worth of chunks of the block row
    constexpr uint32_t kPerWg = kWaves * kSparseChunksPerWave;
    const int active = (int)((L.panel_chunk[p + 1] - L.panel_chunk[p] + kPerWg - 1) / kPerWg);
    const int rows = min(kRedThreads, (bhp + 63) / 64 * 64);        // rows per pass: whole wavefronts
    const int slices = kRedThreads / rows;
    const int sl = (int)threadIdx.x / rows, rl = (int)threadIdx.x - sl * rows;
    // part[p][j][image (part_b of them)][bh]
    const float *src = part + ((size_t)p * wg_per_panel * part_b + b) * L.bh;
    const size_t step = (size_t)part_b * L.bh;
    for (int r0 = 0; r0 < bhp; r0 += rows) {
        const int r = r0 + rl;
        float acc = 0.0f;
        if (r < bhp && sl < slices) {
            // twelve slots per round, all loads issued before the first add (a slot past
            // the last one reads slot sl again and is not added)
            for (int j = sl; j < active; j += 12 * slices) {
                float a[12];
#pragma unroll
                for (int u = 0; u < 12; ++u) {
                    const int jj = j + u * slices;
                    a[u] = src[(size_t)(jj < active ? jj : sl) * step + r];
                }
#pragma unroll
                for (int u = 0; u < 12; ++u)
                    if (j + u * slices < active) acc += a[u];
            }
        }
        if (slices > 1) {
            slice_sum[threadIdx.x] = acc;
            __syncthreads();
            if (sl == 0 && r < bhp)
                for (int k = 1; k < slices; ++k) acc += slice_sum[k * rows + rl];
            __syncthreads();
        }
        if (sl == 0 && r < bhp) {
            if (bias) acc += bias[row_id + r];
            Y[(size_t)b * L.M + row_id + r] = relu ? fmaxf(acc, 0.0f) : acc;
        }
    }
}

__global__ __launch_bounds__(kRedThreads) void fc_reduce_kernel(LayerDev L, const float *__restrict__ part,
                                                                const float *__restrict__ bias, float *Y, int B,
                                                                int part_b, int wg_per_panel, int relu)
{
    fc_reduce_body(L, part, bias, Y, B, part_b, wg_per_panel, relu, (int)blockIdx.x);
}

// The finishing kernel for fc_sparse_group_kernel: layer i's outputs at Y + i * y_stride,
// its bias (if any) at bias + i * bias_stride.
__global__ __launch_bounds__(kRedThreads) void fc_reduce_group_kernel(const LayerDev *__restrict__ table, int wgs_per_layer,
                                                                      const float *__restrict__ part, size_t part_stride,
                                                                      const float *__restrict__ bias, size_t bias_stride, float *Y,
                                                                      size_t y_stride, int B, int wg_per_panel, int relu)
{
    const int job = __builtin_amdgcn_readfirstlane((int)blockIdx.x / wgs_per_layer), wg = (int)blockIdx.x - job * wgs_per_layer;
    const LayerDev L = in_global(table[job]);
    fc_reduce_body(L, part + job * part_stride, bias ? bias + job * bias_stride : nullptr, Y + job * y_stride, B, B, wg_per_panel, relu,
                   wg);
}
