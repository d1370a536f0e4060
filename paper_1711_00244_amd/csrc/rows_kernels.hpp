// Batches of a few up to some dozens of images: decode to entry lists in LDS, multiply row by
// row, the images across a few lanes.  fc_rows_kernel.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

constexpr int kRowsThreads = 1024;
constexpr int kXsColumns = kTile + 1;                   // columns of an activation slab; column 128 holds zeros
constexpr int kListSlack = 16;                          // list entries past a block's last: read by idle lanes, the final one written by them

// The value of lane K of each quarter wavefront, in all its lanes.
template <int K> __device__ __forceinline__ uint32_t row_bcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xf, 0xf, true);        // row_newbcast:K
}

// Eight of the sixteen entries a quarter wavefront holds, one per lane (byte offset of the
// entry's column in the activations, and its weight), K .. K + 7: every quarter multiplies
// its k-th entry with its sixteen times IPL (2 or 4) images.  The reads of all eight (or, of N = 4, four) go out together;
// the multiply-adds take the weight from lane k of the quarter themselves (written out: the
// compiler keeps the move apart).
template <int IPL, int K, int N>
__device__ __forceinline__ void rows_read(float (&x)[N][IPL], uint32_t off, uint32_t xbase)
{
    typedef typename WideVec<IPL>::type vec_t;
    typedef const __attribute__((address_space(3))) vec_t *lds_vec;
    uint32_t at[N];
    at[0] = row_bcast<K>(off) + xbase, at[1] = row_bcast<K + 1>(off) + xbase, at[2] = row_bcast<K + 2>(off) + xbase, at[3] = row_bcast<K + 3>(off) + xbase;
    if constexpr (N == 8)
        at[4] = row_bcast<K + 4>(off) + xbase, at[5] = row_bcast<K + 5>(off) + xbase, at[6] = row_bcast<K + 6>(off) + xbase, at[7] = row_bcast<K + 7>(off) + xbase;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const vec_t v = *(lds_vec)(uintptr_t)at[u];
#pragma unroll
        for (int m = 0; m < IPL; ++m) x[u][m] = v[m];
    }
}

template <int IPL, int K, int N>
__device__ __forceinline__ void rows_add(float (&acc)[IPL], const float (&x)[N][IPL], float w)
{
    // (s_nop: two wait states between a vector write of w and its use as another lane's operand)
#pragma unroll
    for (int m = 0; m < IPL; ++m) {
        if constexpr (N == 8)
            asm("s_nop 1\n"
                "v_fmac_f32_dpp %0, %1, %2 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %3 row_newbcast:%10+1 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %4 row_newbcast:%10+2 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %5 row_newbcast:%10+3 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %6 row_newbcast:%10+4 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %7 row_newbcast:%10+5 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %8 row_newbcast:%10+6 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %9 row_newbcast:%10+7 row_mask:0xf bank_mask:0xf"
                : "+v"(acc[m])
                : "v"(w), "v"(x[0][m]), "v"(x[1][m]), "v"(x[2][m]), "v"(x[3][m]), "v"(x[4][m]), "v"(x[5][m]), "v"(x[6][m]), "v"(x[7][m]), "n"(K));
        else
            asm("s_nop 1\n"
                "v_fmac_f32_dpp %0, %1, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %3 row_newbcast:%6+1 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %4 row_newbcast:%6+2 row_mask:0xf bank_mask:0xf\n"
                "v_fmac_f32_dpp %0, %1, %5 row_newbcast:%6+3 row_mask:0xf bank_mask:0xf"
                : "+v"(acc[m])
                : "v"(w), "v"(x[0][m]), "v"(x[1][m]), "v"(x[2][m]), "v"(x[3][m]), "n"(K));
    }
}

// The value of lane K of each group of four lanes, in all four.
template <int K> __device__ __forceinline__ uint32_t quad_bcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, K * 0x55, 0xf, 0xf, true);          // quad_perm:[K,K,K,K]
}

// Four entries of a row, held by its four lanes one each (byte offset of the entry's column in the activations, and its weight),
// times the lane's four images: 4 t .. 4 t + 3 of lane t.
constexpr int kQuadImages = 4;

__device__ __forceinline__ void quad_read(float (&x)[4][kQuadImages], uint32_t off, uint32_t xbase)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(3))) f4 *lds_f4;
    const uint32_t at[4] = {quad_bcast<0>(off) + xbase, quad_bcast<1>(off) + xbase, quad_bcast<2>(off) + xbase, quad_bcast<3>(off) + xbase};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f4 v = *(lds_f4)(uintptr_t)at[u];
#pragma unroll
        for (int m = 0; m < kQuadImages; ++m) x[u][m] = v[m];
    }
}

__device__ __forceinline__ void quad_add(float (&acc)[kQuadImages], const float (&x)[4][kQuadImages], float w)
{
    // (s_nop: two wait states between a vector write of w and its use as another lane's operand)
#pragma unroll
    for (int m = 0; m < kQuadImages; ++m)
        asm("s_nop 1\n"
            "v_fmac_f32_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n"
            "v_fmac_f32_dpp %0, %1, %3 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n"
            "v_fmac_f32_dpp %0, %1, %4 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n"
            "v_fmac_f32_dpp %0, %1, %5 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf"
            : "+v"(acc[m])
            : "v"(w), "v"(x[0][m]), "v"(x[1][m]), "v"(x[2][m]), "v"(x[3][m]));
}

// Bytes of v that are not zero, added to n.
__device__ __forceinline__ uint32_t add_nonzero_bytes(uint32_t v, uint32_t n)
{
    return n + (uint32_t)__builtin_popcount((((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u);
}

// The surviving weights of a record put into a list, two bytes each (value index << 8 |
// column): `at` is the LDS address of the first one's place, `before` the sum of z over the
// block's entries before the record plus its entry count (the position of the record's first
// entry, less its own z).  No branches: what is not a surviving weight - padding, and entries
// the record does not have, whose value index reads 0 - goes to the list's last place, which
// nobody reads.
typedef __attribute__((address_space(3))) uint16_t *lds_u16;

template <int J, class Col>
__device__ __forceinline__ void list_from(const Symbols &y, uint32_t pos, uint32_t at, uint32_t trash, Col &col)
{
    if constexpr (J < kMaxEntries) {
        if ((uint32_t)J >= y.nmax) return;                                  // uniform
        constexpr int w = J / 4, b = J % 4;
        pos += (y.z[w] >> (8 * b)) & 0xffu;
        const uint32_t e = __builtin_amdgcn_perm(y.v[w], col(pos + (uint32_t)J), 0x0c0c0000u | (uint32_t)(4 + b) << 8);
        const bool live = ((y.v[w] >> (8 * b)) & 0xffu) != 0u;
        *(lds_u16)(uintptr_t)(live ? at : trash) = (uint16_t)e;
        list_from<J + 1>(y, pos, live ? at + 2u : at, trash, col);
    }
}

// Workgroup (image tile of 16 IPL images, block row p, split j of its blocks) of sixteen
// wavefronts, one to a CU.  The blocks are taken G at a time.  While a group is multiplied the
// next one is decoded, by the same wavefronts: each decodes its chunk of the next group (one
// record per lane), puts the surviving weights of the chunk in block order into that block's
// list in LDS and then multiplies its rows of the present group.  A row's sum stays in a register from the first block to the last, and
// nothing is added in memory.  Where a row's entries start in a block's list was counted when the layer was loaded (row_ptr).
//   From 17 images on (IPL 2 and 4) a quarter wavefront has two rows, one after the other: it takes sixteen entries of a
//   row, one per lane, and goes through them with row broadcasts, sixteen images, IPL to a lane, across its lanes.
//   Up to 16 images four lanes have a row, four images each: they take four entries, one per lane, and go through them with quad
//   broadcasts.  So a wavefront has sixteen rows at a time, an address and a read serve sixteen entries and not four, and the reads are of
//   16 bytes; a step is as long as the longest of sixteen rows, not of four.  Eight wavefronts have a block's rows; the
//   other eight have the next block's, and the two halves' sums are added at the end.  (us a call at 16 images, two rows to a quarter and
//   this: 4096 x 9216 at 9 % 25.6 and 22.8, 4096 x 25088 at 4 % 42.6 and 31.6, 4096 x 16384 at 3 / 16 / 30 % 32.3 / 53.3 / 80.5 and 22.7 / 38.1 /
//   58.1.  At 32 images, eight to a lane, 28.6 and 29.8, 46.9 and 44.5 for the first two: left as it was.)
// Bound by vector issue (decode and multiply-adds; at 64 images of the VGG-shaped fc6 53 % of the cycles, LDS 37 %) and by what is left of a group's
// turn, which is why small tiles take several blocks to a group.  At 16 images of the AlexNet-shaped fc6, two rows to a quarter, leaving out
// the products took 24 us to 13, leaving out the decode to 21, the activations nothing.  Nothing in a turn waits for loads it has just requested: the decode, which the
// barrier waits for, comes first; ranges stay as loaded; a slot is asked for before the products and its record after
// them (a turn of the VGG-shaped fc6 at 64 images 7.7 k -> 6.5 k cycles).  us per
// layer call at 32 / 64 images: AlexNet-shaped fc6 28 / 41, dense tiles 42 / 60; VGG-shaped fc6 47 / 70, dense tiles 92 / 139.
// (A turn that decodes the symbols of the group after next and places the next group's - half the chain each - 0 to 2 % slower up to 32
// images, 2 % faster at 64 at 4 %, nothing at 9 %.)
template <int IPL, int G>
__global__ __launch_bounds__(kRowsThreads) void fc_rows_kernel(LayerDev L, const float *__restrict__ X, float *__restrict__ part, int B,
                                                               int panels, int splits, int Bp, int list_cap)
{
    constexpr int NW = kRowsThreads / 64, kImages = 16 * IPL, kSlab = kXsColumns * kImages, RQ = kTile / NW / 4;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const Smem s = carve(smem_raw, L);
    float *slabs = s.extra;                                             // [2][G][kXsColumns][kImages]
    uint16_t *lists = (uint16_t *)(slabs + 2 * G * kSlab);              // [2][G][list_cap]
    const int j = (int)blockIdx.x % splits, rest = (int)blockIdx.x / splits;
    const int p = rest % panels, img0 = (rest / panels) * kImages;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63), l16 = lane & 15;
    const int blk_lo = (int)(((int64_t)L.nbw * j) / splits), blk_hi = (int)(((int64_t)L.nbw * (j + 1)) / splits);
    const uint32_t pb0 = (uint32_t)p * (uint32_t)L.nbw;
    const int phases = (blk_hi - blk_lo + G - 1) / G;

    // ---- the chunks: a group's chunks are counted off slot by slot of its blocks (slot_at), wavefront w
    // takes the ones congruent to w + 4 ph.  What a chunk is stands in one table entry, so
    // only the record's load waits for another one.
    const int slots = L.block_slots;
    ChunkSlot ch{};
    uint64_t rec = 0;
    int ch_blk = 0, ch_i = 0;                   // the chunk's block (of the block row) and its number within the group
    auto slot_of = [&](int ph, int i) {
        const int b0 = blk_lo + ph * G;
        int g = 0;
#pragma unroll
        for (int q = 1; q < G; ++q) g += i >= q * slots ? 1 : 0;
        ch_blk = b0 + g;
        return L.slot[(size_t)(pb0 + (uint32_t)b0) * (uint32_t)slots + (uint32_t)i];
    };
    auto slots_of = [&](int ph) { return ph < phases ? min(G, blk_hi - (blk_lo + ph * G)) * slots : 0; };
    auto fetch_chunk = [&](int ph) {            // the next chunk with records from ch_i on, if any
        const int n = slots_of(ph);
        ch.nrec = 0;
        for (; ch_i < n; ch_i += NW) {
            ch = slot_of(ph, ch_i);
            if (ch.nrec != 0) break;
        }
        if (ch.nrec != 0) rec = (uint32_t)lane < ch.nrec ? L.records[(size_t)ch.rec_off + lane] : 0ull;
    };
    // The first chunk of a group is asked for in two steps, so that neither waits: its slot, and
    // some thousand cycles later (the products of a group) its record.
    auto first_slot = [&](int ph) {
        ch_i = (wave + 4 * ph) & (NW - 1);
        ch.nrec = 0;
        if (ch_i < slots_of(ph)) ch = slot_of(ph, ch_i);
    };
    auto first_record = [&](int ph) {
        if (ch.nrec != 0) rec = (uint32_t)lane < ch.nrec ? L.records[(size_t)ch.rec_off + lane] : 0ull;
        else if (ch_i < slots_of(ph)) {
            ch_i += NW;
            fetch_chunk(ph);
        }
    };
    auto decode = [&](int ph) {
        const Symbols y = decode_record(split_record(rec, (uint32_t)rec & 15u), s.T);
        uint32_t weights = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if ((uint32_t)(4 * w) < y.nmax) weights = add_nonzero_bytes(y.v[w], weights);
        // lane counts (<= 15, 960 per chunk) and advances in one scan
        const uint32_t mine = weights | (y.adv << 10);
        const uint32_t excl = wave_incl_scan(mine) - mine;
        const uint16_t *list = lists + ((ph & 1) * G + ch_blk - (blk_lo + ph * G)) * list_cap;
        const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint16_t *)list;
        const uint32_t at = base + 2u * (ch.at + (excl & 1023u)), trash = base + 2u * (uint32_t)(list_cap - 1);
        const uint32_t before = ch.pos0 + (excl >> 10);
        const uint32_t bwp = (uint32_t)min(L.bw, L.K - ch_blk * L.bw);
        if ((bwp & (bwp - 1u)) == 0u) {
            auto col = [&](uint32_t pos) { return pos & (bwp - 1u); };
            list_from<0>(y, before, at, trash, col);
        } else {
            // (a magic multiplier instead of a division: exact for positions below 2^14 and
            // widths up to 128)
            const uint32_t inv = (0x400000u + bwp - 1u) / bwp;
            auto col = [&](uint32_t pos) { return pos - ((pos * inv) >> 22) * bwp; };
            list_from<0>(y, before, at, trash, col);
        }
    };
    auto decode_group = [&](int ph) {
        // (more chunks in a group than wavefronts: the rest is fetched where it is needed)
        while (ch.nrec != 0) {
            decode(ph);
            ch_i += NW;
            fetch_chunk(ph);
        }
    };

    // ---- the activations of a group, X[image][column] in memory, [column][image] in LDS: what a
    // quarter reads of a column is contiguous, so that its reads never conflict with each other.
    // Four lanes fetch 64 bytes of an image, sixteen images side by side.
    constexpr int kPieces = (G * kImages * (kTile / 4) + kRowsThreads - 1) / kRowsThreads;
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    f4 stage[kPieces];
    auto piece = [&](int i, int &g, int &img, int &col) {
        const int t = (wave + i * NW) * 4;                              // four 16-byte columns, sixteen images per wavefront
        const int c = t & (kTile / 4 - 1), q = t / (kTile / 4);
        col = (c + (lane >> 4)) * 4;
        img = (q % (kImages / 16)) * 16 + (lane & 15);
        g = q / (kImages / 16);
    };
    // (images past the batch read the last one: their sums are dropped; columns a block does not
    // have read the next block's or the row's last: no list names them)
    // Where a lane's pieces lie does not change from group to group but for the first column, which all lanes share:
    // a load takes that as its scalar offset, and a lane's own one, in bytes, is worked out here once.
    const bool near = (uint64_t)kImages * (uint64_t)L.K < (uint64_t)1 << 29;        // a tile's images within a buffer's offsets
    const __amdgpu_buffer_rsrc_t images = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(X + (size_t)img0 * L.K), 0, near ? (int)((uint32_t)min(kImages, B - img0) * (uint32_t)L.K * (uint32_t)sizeof(float)) : 0, 0x00020000);
    uint32_t piece_off[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        int g, img, col;
        piece(i, g, img, col);
        piece_off[i] = ((uint32_t)(min(img0 + img, B - 1) - img0) * (uint32_t)L.K + (uint32_t)(min(g, G - 1) * L.bw + col)) * (uint32_t)sizeof(float);
    }
    auto slab_fetch = [&](int ph) {
        const int k0 = (blk_lo + ph * G) * L.bw;                        // uniform
        if (near && k0 + (G - 1) * L.bw + kTile <= L.K) {
#pragma unroll
            for (int i = 0; i < kPieces; ++i)
                stage[i] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(images, (int)piece_off[i], k0 * (int)sizeof(float), 0));
            return;
        }
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            int g, img, col;
            piece(i, g, img, col);
            const int k = min(blk_lo + ph * G + g, L.nbw - 1) * L.bw + col;
            const float *row = X + (size_t)min(img0 + img, B - 1) * L.K;
            if (k + 4 <= L.K) stage[i] = *(const f4u *)(row + k);
            else {
#pragma unroll
                for (int u = 0; u < 4; ++u) stage[i][u] = row[min(k + u, L.K - 1)];
            }
        }
    };
    auto slab_store = [&](int ph) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            int g, img, col;
            piece(i, g, img, col);
            if (g >= G) continue;
            float *dst = slabs + ((ph & 1) * G + g) * kSlab + col * kImages + img;
#pragma unroll
            for (int u = 0; u < 4; ++u) dst[u * kImages] = stage[i][u];
        }
    };

    // ---- where the lane's rows start in the lists of a group of blocks, and where the last ends ----
    // (rows the blocks do not have start and end where the last row ends: the table's last two entries)
    // (QUADS: up to 16 images, four lanes to a row)
    constexpr bool QUADS = IPL == 1;
    constexpr int GW = QUADS ? (G + 1) / 2 : G;             // blocks of a group to a wavefront
    const int g_first = QUADS ? wave >> 3 : 0;              // the first of them
    constexpr int g_step = QUADS ? 2 : 1;
    const int row0 = QUADS ? (wave & 7) * 16 + (lane >> 2) : wave * (kTile / NW) + (lane >> 4) * RQ;
    static_assert(RQ == 2, "a quarter's two rows are one word of row_ptr and the half after it");
    const int row_at = min(row0, L.row_ptrs - 2), row_end = min(row0 + (QUADS ? 1 : RQ), L.row_ptrs - 1);
    // (as they are loaded, and taken apart where they are used: a group's turn would otherwise begin with waiting for them)
    struct RowRange {
        uint32_t starts, end;
        __device__ __forceinline__ uint32_t at(int i) const { return i == 0 ? starts & 0xffffu : i == 1 ? starts >> 16 : end; }
    };
    auto ranges_fetch = [&](int ph, RowRange (&r)[GW]) {
#pragma unroll
        for (int i = 0; i < GW; ++i) {
            const int g = g_first + i * g_step;
            // (a block past the last: the last one's again, which multiply leaves out - a register set to zero here would have
            // every load before it waited for)
            const int blk = min(blk_lo + ph * G + g, blk_hi - 1);
            const uint16_t *rp = L.row_ptr + (size_t)(pb0 + (uint32_t)blk) * (uint32_t)L.row_ptrs;
            r[i] = QUADS ? RowRange{rp[row_at], rp[row_end]} : RowRange{*(const uint32_t *)(rp + row_at), rp[row_end]};
        }
    };

    constexpr int AR = QUADS ? 1 : RQ, AI = QUADS ? kQuadImages : IPL;  // rows and images of a lane
    float acc[AR][AI];
#pragma unroll
    for (int i = 0; i < AR; ++i)
#pragma unroll
        for (int m = 0; m < AI; ++m) acc[i][m] = 0.0f;

    auto multiply_quads = [&](int ph, const RowRange (&r)[GW]) {
        if constexpr (QUADS) {
            // The first sixteen entries of the wavefront's rows of all its blocks, four to a lane, then their weights: requested together
            // (past a row's last entry: codebook entry 0 and the column of zeros).  The activations of four entries of each row are
            // requested while the four before them are multiplied.
            const uint32_t t = (uint32_t)lane & 3u;
            auto entry = [&](uint32_t at, int left) { return (int)t < left ? (uint32_t)*(lds_u16)(uintptr_t)at : (uint32_t)kTile; };
            uint32_t ent[GW][4], at[GW];
            int left[GW];
            float w[GW][4];
#pragma unroll
            for (int i = 0; i < GW; ++i) {
                const int g = g_first + i * g_step;
                left[i] = g < G && blk_lo + ph * G + g < blk_hi ? (int)(r[i].end - r[i].starts) : 0;
                at[i] = (uint32_t)(uintptr_t)(lds_u16)(lists + ((ph & 1) * G + min(g, G - 1)) * list_cap) + 2u * (r[i].starts + t);
#pragma unroll
                for (int q = 0; q < 4; ++q) ent[i][q] = entry(at[i] + 8u * q, left[i] - 4 * q);
            }
#pragma unroll
            for (int i = 0; i < GW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) w[i][q] = s.T.cb[ent[i][q] >> 8];
#pragma unroll
            for (int i = 0; i < GW; ++i) {
                const uint32_t xbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float *)(slabs + ((ph & 1) * G + min(g_first + i * g_step, G - 1)) * kSlab) + 16u * t;
                auto off = [&](uint32_t e) { return (e & 255u) * (uint32_t)(kImages * 4); };
                if (!__any(left[i] > 0)) continue;                          // (all conditions here are uniform)
                for (;;) {
                    float x0[4][kQuadImages], x1[4][kQuadImages];
                    const bool two = __any(left[i] > 4), three = __any(left[i] > 8), four = __any(left[i] > 12), more = __any(left[i] > 16);
                    quad_read(x0, off(ent[i][0]), xbase);
                    if (two) quad_read(x1, off(ent[i][1]), xbase);
                    quad_add(acc[0], x0, w[i][0]);
                    if (two) {
                        if (three) quad_read(x0, off(ent[i][2]), xbase);
                        quad_add(acc[0], x1, w[i][1]);
                        if (three) {
                            if (four) quad_read(x1, off(ent[i][3]), xbase);
                            quad_add(acc[0], x0, w[i][2]);
                            if (four) quad_add(acc[0], x1, w[i][3]);
                        }
                    }
                    if (!more) break;
                    left[i] -= 16;
                    at[i] += 32u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) ent[i][q] = entry(at[i] + 8u * q, left[i] - 4 * q);
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[i][q] = s.T.cb[ent[i][q] >> 8];
                }
            }
        }
    };
    auto multiply_rows = [&](int ph, const RowRange (&r)[GW]) {
        if constexpr (!QUADS) {
            // the first sixteen entries of all the rows, then their weights: requested together
            // (past a row's last entry: codebook entry 0 and the column of zeros)
            auto entry = [&](uint32_t at, int left) { return l16 < left ? (uint32_t)*(lds_u16)(uintptr_t)at : (uint32_t)kTile; };
            auto list_at = [&](int g, int i) { return (uint32_t)(uintptr_t)(lds_u16)(lists + ((ph & 1) * G + g) * list_cap) + 2u * (r[g].at(i) + (uint32_t)l16); };
            auto count = [&](int g, int i) { return blk_lo + ph * G + g < blk_hi ? (int)(r[g].at(i + 1) - r[g].at(i)) : 0; };
            uint32_t ent[G][RQ];
            float w[G][RQ];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < RQ; ++i) ent[g][i] = entry(list_at(g, i), count(g, i));
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < RQ; ++i) w[g][i] = s.T.cb[ent[g][i] >> 8];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint32_t xbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float *)(slabs + ((ph & 1) * G + g) * kSlab) +
                                       (uint32_t)(l16 * IPL * 4);
#pragma unroll
                for (int i = 0; i < RQ; ++i) {
                    int left = count(g, i);
                    uint32_t at = list_at(g, i);
                    for (;;) {
                        const uint32_t off = (ent[g][i] & 255u) * (uint32_t)(kImages * 4);
                        const bool half = __any(left > 8), more = __any(left > 16);      // uniform
                        float x0[8][IPL], x1[IPL == 4 ? 4 : 8][IPL];
                        rows_read<IPL, 0>(x0, off, xbase);
                        if (half) rows_read<IPL, 8>(x1, off, xbase);
                        const float wv = w[g][i];
                        // (with four images a lane the eight behind the first eight go four at a time: rows differ, and it is these lanes'
                        // multiply-adds and reads that count.  With fewer, the wait for the last four does.)
                        const bool rest = IPL == 4 && __any(left > 12);
                        if (more) ent[g][i] = entry(at += 32u, left -= 16);
                        rows_add<IPL, 0>(acc[i], x0, wv);
                        if (more) w[g][i] = s.T.cb[ent[g][i] >> 8];
                        if (half) {
                            float x2[4][IPL];
                            if (rest) rows_read<IPL, 12>(x2, off, xbase);
                            rows_add<IPL, 8>(acc[i], x1, wv);
                            if (rest) rows_add<IPL, 12>(acc[i], x2, wv);
                        }
                        if (!more) break;
                    }
                }
            }
        }
    };

    auto multiply = [&](int ph, const RowRange (&r)[GW]) {
        multiply_quads(ph, r);
        multiply_rows(ph, r);
    };

    if (phases > 0) {
        RowRange now[GW], next[GW];
        for (int i = (int)threadIdx.x; i < L.table_rows; i += kRowsThreads) s.tables[i] = L.tables[i];
        first_slot(0);
        first_record(0);
        slab_fetch(0);
        ranges_fetch(0, now);
        for (int i = (int)threadIdx.x; i < 2 * G * kImages; i += kRowsThreads) slabs[(i / kImages) * kSlab + kTile * kImages + i % kImages] = 0.0f;
        __syncthreads();
        decode_group(0);
        first_slot(1);
        slab_store(0);
        first_record(1);
        __syncthreads();
        for (int ph = 0; ph < phases; ++ph) {
            const bool more = ph + 1 < phases;
            if (more) {
                // (a wavefront with a chunk has the longest way to the barrier: the others' products wait for it.  It decodes
                // first: behind the loads that follow it would wait for them as well)
                __builtin_amdgcn_s_setprio(3);
                decode_group(ph + 1);
                __builtin_amdgcn_s_setprio(0);
                slab_fetch(ph + 1);
                ranges_fetch(ph + 1, next);
                first_slot(ph + 2);
            }
            multiply(ph, now);
            if (more) {
                first_record(ph + 2);
                slab_store(ph + 1);
#pragma unroll
                for (int g = 0; g < GW; ++g) now[g] = next[g];
            }
            __syncthreads();
        }
    }
    // the wavefront's rows of the workgroup's partial tile, part[block row][split][row][Bp]
    float *to = part + (((size_t)p * splits + j) * kTile + row0) * (size_t)Bp + img0;
    if constexpr (QUADS) {
        // (the two halves of the workgroup have every second block's sums each; every wavefront has passed its last barrier)
        float *sums = slabs + (wave & 7) * (64 * kQuadImages) + lane * kQuadImages;
        if (G > 1 && wave >= 8) store_floats<4>(sums, acc[0]);
        if (G > 1) __syncthreads();
        if (wave >= 8) return;
        float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (G > 1) load_floats<4>(sums, y);
#pragma unroll
        for (int m = 0; m < kQuadImages; ++m) y[m] += acc[0][m];
        store_floats<4>(to + 4 * (lane & 3), y);
    } else {
#pragma unroll
        for (int i = 0; i < RQ; ++i) store_floats<IPL>(to + (size_t)i * Bp + l16 * IPL, acc[i]);
    }
}

// Finishes fc_rows_kernel: Y[image][row] = act(sum over the splits + bias) from part[block row][split][row][Bp].  The
// partial tiles are small and the splits many, so it is bound by the latency of its loads, not by bytes: a
// thread takes four images of a row and a quarter of the splits, all its loads (up to eight at a time) in flight together, and
// the quarters are added in order.  (wide_reduce_kernel, whose threads take all splits of two rows, left a 1000-row
// layer 32 workgroups and took 9.8 us for 64 images.  AlexNet-shaped
// stack at 16 images 64.5 -> 54.1 us, VGG-16-shaped at 64 131.5 -> 123.4.)
constexpr int kRowsRedParts = 4, kRowsRedPieces = 64;      // quarters; (row, four images) pieces of a workgroup

__host__ __device__ constexpr int rows_reduce_quads(int Bp) { return Bp >= 64 ? 16 : Bp / 4; }     // pieces of a row in a workgroup

__global__ __launch_bounds__(kRowsRedParts * kRowsRedPieces) void rows_reduce_kernel(LayerDev L, const float *__restrict__ part, const float *__restrict__ bias,
                                                                                     float *Y, int batch, int Bp, int splits, int relu)
{
    __shared__ float sums[kRowsRedParts - 1][kRowsRedPieces][4];
    const int quads = rows_reduce_quads(Bp), image_tiles = Bp / (4 * quads);
    const int piece = (int)threadIdx.x & (kRowsRedPieces - 1);
    const int jp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kRowsRedPieces);
    const int m = (int)(blockIdx.x / (unsigned)image_tiles) * (kRowsRedPieces / quads) + piece / quads;
    const int c = (int)(blockIdx.x % (unsigned)image_tiles) * (4 * quads) + 4 * (piece % quads);
    const bool live = m < L.M && c < batch;
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (live) {
        const int p = m / L.bh, r = m - p * L.bh;
        const int lo = splits * jp / kRowsRedParts, hi = splits * (jp + 1) / kRowsRedParts;
        const size_t stride = (size_t)kTile * Bp;
        const float *src = part + ((size_t)p * splits * kTile + r) * (size_t)Bp + c;
        for (int j = lo; j < hi; j += 8) {
            float a[8][4];
#pragma unroll
            for (int u = 0; u < 8; ++u) load_floats<4>(src + (size_t)(j + u < hi ? j + u : j) * stride, a[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (j + u < hi) t[k] += a[u][k];
        }
        if (jp > 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sums[jp - 1][piece][k] = t[k];
        }
    }
    __syncthreads();
    if (jp > 0 || !live) return;
    const float b = bias ? bias[m] : 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int q = 0; q < kRowsRedParts - 1; ++q) t[k] += sums[q][piece][k];
        t[k] += b;
        if (c + k < batch) Y[(size_t)(c + k) * L.M + m] = relu ? fmaxf(t[k], 0.0f) : t[k];
    }
}
