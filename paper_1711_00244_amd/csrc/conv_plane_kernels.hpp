// Convolution as a matrix product over operands laid out beforehand in bf16 terms:
// conv_prepare_kernel, conv_plane_kernel.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

// (The third form of a convolution, for long calls; the launcher says when.)
// conv_mfma_kernel gathers and splits each activation anew for every filter tap, block row and tile of
// columns.  Here a launch (conv_prepare_kernel; one for each group of images, the weights with the first) splits weights and activations once into the terms
// that the matrix cores multiply, and writes both so that the multiply kernel's operands are
// plain 16-byte pieces, eight k side by side:
//   activations: planes of pixels, eight channels of a pixel to a piece, term by term, with the image's
//   zero border written out, so that a filter tap is one offset for every pixel and no tap is ever tested;
//   weights: the rows of a tile side by side, in the order in which the walk over k takes them.
// k runs in units of eight: (channel group cg, tap r, tap s) with the eight channels 8 cg .. 8 cg + 7 inside, so
// that the taps of a plane follow each other and find its lines in the caches.  Where a filter has
// at most four channels (px4) a pixel is four channels, a unit two neighbouring taps of a filter row; of
// an odd number of taps the last unit takes the last two again, and the one that then is in two units has half its
// weight in each (exact, and an infinity or a NaN gives what it gives once).
struct PlaneGeom {
    int C, Cg, H, W, Hp, Wp;      // channels, channels of a filter group, image, image with its border
    int R, S, pad;
    int px4;                      // four channels to a pixel, not eight
    int CG, SU;                   // channel groups of a filter group; units of a filter row
    int units, steps;             // units of k, pairs of them
    int groups, OCg, tile_rows, ppg;      // filter groups, filters of one, rows of a tile, tiles of a group
    uint32_t pieces;              // 16-byte pieces of a term of the activations
    Divisor per_plane, per_row, planes;   // pieces of a plane, of a row of it; planes (of eight channels, of four) of an image
    Divisor per_s;                // taps of a filter row
    Divisor per_group;            // units of a channel group, or (px4) of a filter row
};

constexpr int kPrepThreads = 1024;
constexpr int kPrepCells = 64;                             // rows x blocks of a workgroup: 64 x 1 to 8 x 8
constexpr int kPrepBlocks = 8;
// LDS of a workgroup's weights: its rows, each the columns of its blocks and a zero
constexpr size_t prep_tile_bytes(int blocks) { return (size_t)(kPrepCells / blocks) * (blocks * kTile + 1) * sizeof(uint2); }

// Unit u's first channel, and the tap (r S + s) of its first slot.
struct Unit {
    int c, tap;
};
__device__ __forceinline__ Unit unit_at(const PlaneGeom &g, int u)
{
    const int q = (int)g.per_group.quotient((uint32_t)u), i = u - q * (int)g.per_group.d;
    return g.px4 ? Unit{0, q * g.S + min(2 * i, g.S - 2)} : Unit{8 * q, i};
}

// A workgroup for each 64 rows of a block of the layer: the rows decoded into LDS as in decode_tiles_kernel, split
// into NP terms (split_weights) and written to wt[tile of rows][step][term][unit % 2][row][8 k].  A block's columns
// rarely end where a unit ends: where a block has only some of a unit's slots it writes those alone.  The slots
// behind a group's last channel, and the second unit of the last step where there is none, are zero (an
// activation times what is not written could be a NaN); rows behind a group's last filter stay as they are, and so do
// the outputs that they reach, which nobody reads.
// The workgroups behind the layer's blocks (no strips: all of them) split the activations (split8), xs[term][image][plane][pixel][8 or 4 channels].
// unit_off[u]: bytes from a receptive field's corner to unit u's piece, 0xffffffff for the second unit of a last step that has
// none.
// A workgroup takes kPrepCells / `blocks` rows of `blocks` neighbouring blocks, finds the chunks that reach into them by the chunks' position
// carries, and splits the codebook once, so that a weight's terms are looked up.  Strips that are fewer than the CUs are decoded by
// several workgroups, each of which writes some of the units.
// Bound by what is written, 6 bytes a weight and an activation (AlexNet's five convolutions at 64 images 17, 17, 14, 14 and 12 us of a call less the multiply launch, 24, 20, 16, 18 and 18 in a
// trace, wavefronts waiting 57-60 % of their time, vector issue 31-40 %; conv1 80 MB written)
// and, for a small call, by the chain carries -> record -> decode -> terms -> stores (VGG-16 conv4_2 at one image 19 us, of which decoding 8 and
// storing 14 MB of weights 7).  With whole blocks of 128 x 128, split as they were stored slot by slot, these six were 40, 31, 21, 19, 22 and 20 us.
template <int NP>
__global__ __launch_bounds__(kPrepThreads) void conv_prepare_kernel(LayerDev L, PlaneGeom g, const float *__restrict__ X, uint4 *wt, uint4 *xs,
                                                                    uint32_t *unit_off, int n_strips, int parts, int blocks)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const int rs = g.R * g.S;
    const uint32_t n_decode = (uint32_t)(n_strips * parts);
    if (blockIdx.x >= n_decode) {
        const uint32_t step = (gridDim.x - n_decode) * kPrepThreads;
        const int hw = g.H * g.W;
        for (uint32_t i = (blockIdx.x - n_decode) * kPrepThreads + threadIdx.x; i < g.pieces; i += step) {
            const uint32_t pl = g.per_plane.quotient(i), o = i - pl * g.per_plane.d;
            const uint32_t y = g.per_row.quotient(o), x = o - y * g.per_row.d;
            const uint32_t img = g.planes.quotient(pl), gc = pl - img * g.planes.d;   // plane of the image: filter group, channel group
            float v[8];
            if (g.px4) {
                const int iy = (int)y - g.pad;
                const float *src = X + (size_t)img * g.C * hw + (size_t)gc * g.Cg * hw;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int ix = 2 * (int)x + (j >> 2) - g.pad, c = j & 3;
                    const bool in = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W && c < g.Cg;
                    v[j] = in ? src[c * hw + iy * g.W + ix] : 0.0f;
                }
            } else {
                const int iy = (int)y - g.pad, ix = (int)x - g.pad;
                const uint32_t grp = gc / (uint32_t)g.CG;
                const int cg = (int)(gc - grp * (uint32_t)g.CG);
                const bool in = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
                const float *src = X + ((size_t)img * g.C + (size_t)grp * g.Cg + 8 * cg) * hw + iy * g.W + ix;
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = in && 8 * cg + j < g.Cg ? src[(size_t)j * hw] : 0.0f;
            }
            uint4 terms[NP];
            split8<NP>(v, terms);
#pragma unroll
            for (int t = 0; t < NP; ++t) xs[(size_t)t * g.pieces + i] = terms[t];
        }
        return;
    }
    {
        const int u = (int)(blockIdx.x * kPrepThreads + threadIdx.x);
        if (u < 2 * g.steps) {
            uint32_t off = 0xffffffffu;
            if (u < g.units) {
                const Unit n = unit_at(g, u);
                const int r = n.tap / g.S, s = n.tap - r * g.S;
                off = g.px4 ? (uint32_t)(r * g.Wp + s) * 8u : (uint32_t)((n.c / 8) * (g.Hp * g.Wp) + r * g.Wp + s) * 16u;
            }
            unit_off[u] = off;
        }
    }
    const Smem s = carve(smem_raw, L);
    const int rows = kPrepCells / blocks, stride = blocks * L.bw + 1;
    uint2 *tile = (uint2 *)s.extra;                         // [rows][stride]: a weight's terms, sixteen bits each; the last column is zero
    uint2 *code = tile + rows * stride;                     // the codebook's terms, then (px4, odd S) those of half its values
    const bool shared = g.px4 && (g.S & 1);
    // Each die takes a run of strips, in which the blocks of a block row follow each other: two blocks' shares of a unit, and so of a
    // line of wt, meet in one L2.
    int brow, bcol, row0, part;
    {
        const uint32_t die = blockIdx.x % 8u, strips = (uint32_t)((L.bh + rows - 1) / rows), runs = (uint32_t)((L.nbw + blocks - 1) / blocks);
        uint32_t at = die * (n_decode / 8u) + min(die, n_decode % 8u) + blockIdx.x / 8u;
        part = __builtin_amdgcn_readfirstlane((int)(at % (uint32_t)parts));
        at /= (uint32_t)parts;
        const uint32_t line = at / runs;
        bcol = __builtin_amdgcn_readfirstlane((int)(at - line * runs)) * blocks;
        brow = __builtin_amdgcn_readfirstlane((int)(line / strips));
        row0 = __builtin_amdgcn_readfirstlane((int)(line % strips)) * rows;
    }
    TableRegs tr;
    if (threadIdx.x < kThreads) tr = fetch_tables(L);
    const int n_blocks = min(blocks, L.nbw - bcol);
    // The chunks that reach into the workgroup's rows: a chunk's entries lie at positions from its own carry up to the next one's.
    uint32_t first[kPrepBlocks], count[kPrepBlocks];
    {
        const uint32_t *chunk = L.block_chunk + (uint32_t)brow * (uint32_t)L.nbw + (uint32_t)bcol;
#pragma unroll
        for (int i = 0; i < kPrepBlocks; ++i) {
            first[i] = count[i] = 0;
            if (i < n_blocks) {
                const uint32_t c0 = chunk[i], c1 = chunk[i + 1], bwp = (uint32_t)min(L.bw, L.K - (bcol + i) * L.bw);
                const uint32_t lo = (uint32_t)row0 * bwp, hi = lo + (uint32_t)rows * bwp;
                uint32_t before = 0, upto = 0;
                for (uint32_t c = c0; c < c1; c += 64) {
                    const uint32_t pos = c + (uint32_t)lane < c1 ? L.meta[c + (uint32_t)lane].pos0 : 0xffffffffu;
                    upto += (uint32_t)__builtin_popcountll(__ballot(pos < hi));
                    before += (uint32_t)__builtin_popcountll(__ballot(pos <= lo));
                }
                const uint32_t skip = before > 0 ? before - 1 : 0;           // (up to the last that starts at or before the rows)
                first[i] = c0 + skip;
                count[i] = upto - min(skip, upto);
            }
        }
    }
    // A wavefront takes every sixteenth of them, the next one's record on its way while one is decoded.
    int q = wave, block = 0, next_block = 0;
    ChunkHead head{};
    LaneRecord rec{};
    auto fetch = [&]() {                                    // chunk q of the workgroup's, if there is one
        uint32_t left = (uint32_t)q, c = 0xffffffffu;
#pragma unroll
        for (int i = 0; i < kPrepBlocks; ++i) {
            if (c == 0xffffffffu) {
                if (left < count[i]) {
                    c = first[i] + left;
                    next_block = i;
                } else left -= count[i];
            }
        }
        if (c == 0xffffffffu) return false;
        head = load_head(L, c);
        rec = load_record(L, head, lane);
        q += kPrepThreads / 64;
        return true;
    };
    bool more = fetch();
    for (int t = threadIdx.x; t < rows * stride; t += kPrepThreads) tile[t] = make_uint2(0u, 0u);
    if (threadIdx.x < kThreads) store_tables(s, L, tr);
    for (int t = threadIdx.x; t < 2 * L.ncode; t += kPrepThreads) {
        if (t >= L.ncode && !shared) break;
        uint32_t w[NP];
        split_weights<NP>(L.codebook[t & (L.ncode - 1)] * (t < L.ncode ? 1.0f : 0.5f), 0.0f, w);
        code[t] = make_uint2((w[0] & 0xffffu) | w[1] << 16, NP == 3 ? w[NP - 1] & 0xffffu : 0u);
    }
    __syncthreads();
    while (more) {
        const LaneRecord now = rec;
        const uint32_t pos0 = head.m.pos0;
        block = next_block;
        more = fetch();
        const BlockGeom bg = block_geom(L, brow, bcol + block);
        const Symbols y = decode_record(now, s.T);
        const LaneStart st = lane_starts(y, pos0);
        for_each_entry(y, st.sum, [&](uint32_t, uint32_t v, uint32_t, uint32_t pos) {
            uint32_t r, cc;
            split_pos(pos, bg, r, cc);
            r -= (uint32_t)row0;
            uint32_t at = v;
            if (shared) {                                   // (the last tap but one of a filter row)
                const uint32_t k = (uint32_t)bg.col_id + cc;
                if (k - g.per_s.quotient(k) * g.per_s.d == (uint32_t)(g.S - 2)) at += (uint32_t)L.ncode;
            }
            if (v != 0 && r < (uint32_t)rows && cc < (uint32_t)L.bw) tile[r * (uint32_t)stride + (uint32_t)(block * L.bw) + cc] = code[at];
        });
    }
    __syncthreads();
    // `blocks` units to a wavefront, the rows of one in neighbouring lanes
    const int k0 = bcol * L.bw, k1 = min(L.K, (bcol + n_blocks) * L.bw);
    int u_lo = 0, u_hi = g.units;
    if (!g.px4) {
        u_lo = (int)g.per_group.quotient((uint32_t)k0) / 8 * rs;
        u_hi = ((int)g.per_group.quotient((uint32_t)(k1 - 1)) / 8 + 1) * rs;
    }
    const int row = lane & (rows - 1);
    const int m = brow * L.bh + row0 + row;
    if (row0 + row >= L.bh || m >= L.M) return;
    const int grp = m / g.OCg, r = m - grp * g.OCg;
    const int p = grp * g.ppg + r / g.tile_rows;
    // 16-byte pieces from the start: the row's piece of step 0, term 0, unit 0
    uint4 *to = wt + (size_t)p * g.steps * (NP * 2) * g.tile_rows + (r - r / g.tile_rows * g.tile_rows);
    const uint2 *from = tile + row * stride;
    for (int u = u_lo + (part * (kPrepThreads / 64) + wave) * blocks + lane / rows; u < u_hi; u += parts * (kPrepThreads / 64) * blocks) {
        // (every slot is read, the row's zero where the blocks have none: nothing is waited for in between)
        const Unit n = unit_at(g, u);
        uint32_t have = 0;
        uint2 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int c = g.px4 ? j & 3 : n.c + j;
            const int k = min(c, g.Cg - 1) * rs + n.tap + (g.px4 ? j >> 2 : 0);
            const bool in = k >= k0 && k < k1;
            have |= (in ? 1u : 0u) << j;
            v[j] = from[in && c < g.Cg ? k - k0 : stride - 1];
        }
        uint32_t t[3][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            t[0][j] = __builtin_amdgcn_perm(v[2 * j + 1].x, v[2 * j].x, 0x05040100u);
            t[1][j] = __builtin_amdgcn_perm(v[2 * j + 1].x, v[2 * j].x, 0x07060302u);
            t[2][j] = __builtin_amdgcn_perm(v[2 * j + 1].y, v[2 * j].y, 0x05040100u);
        }
        uint4 *dst = to + (size_t)((u >> 1) * (NP * 2) + (u & 1)) * g.tile_rows;
        if (have == 0xffu) {
#pragma unroll
            for (int i = 0; i < NP; ++i) dst[(size_t)(2 * i) * g.tile_rows] = uint4{t[i][0], t[i][1], t[i][2], t[i][3]};
            continue;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t two = have >> (2 * h) & 3u;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                uint32_t *d = (uint32_t *)(dst + (size_t)(2 * i) * g.tile_rows) + h;
                if (two == 3u) *d = t[i][h];
                else if (two == 1u) *(uint16_t *)d = (uint16_t)t[i][h];
                else if (two == 2u) ((uint16_t *)d)[1] = (uint16_t)(t[i][h] >> 16);
            }
        }
    }
    if ((g.units & 1) && k1 == L.K && part == 0 && wave == 0 && lane < rows) {
#pragma unroll
        for (int i = 0; i < NP; ++i) to[(size_t)((g.steps - 1) * (NP * 2) + 2 * i + 1) * g.tile_rows] = uint4{0, 0, 0, 0};
    }
}

// What the multiply launch needs beside the operands.
struct PlaneConv {
    int steps, splits, panels, ppg, tiles;     // pairs of units, splits of them, tiles of rows, those of a filter group, tiles of columns
    int n_cols, Np, pq, Q, stride, Wp, px_bytes;
    uint32_t image_bytes, group_bytes, term_bytes;
    int M, OCg;
    float *Y;                                  // the finished output, or null: partial tiles
    const float *bias;
    int relu;
};

// Workgroup = (tile of 32 RT WR filter rows, tile of 32 CT WC columns = image x output pixel, split of the steps), four
// wavefronts of RT x CT accumulators of 32 x 32 each.  A step is two units, sixteen k.  Both operands of a step go from memory into one of
// three LDS buffers without passing through registers (1 KB to a load: 64 rows of a unit, or 64 pixels of one), requested two steps
// before they are read; a wavefront's pieces of the next step are read into registers while the present one is multiplied.
// So a step has one barrier, and next to its multiplies nothing but LDS reads, loads with a scalar offset each, and scalar
// arithmetic.  Two workgroups to a CU: one's barrier, start and end are the other's multiplies.
// Bound by the multiplies: of AlexNet's convolutions at 64 images they are 74 (conv1), 82, 84, 81 and 75 % of the launch's busy cycles (vector issue 13-20 %, LDS
// 14-23 %, no bank conflicts; with one workgroup to a CU a step of 32 of them, 1024 cycles, took 1101 by stamps in a copy, 1627 with reads and requests in a bunch
// behind the barrier and two buffers), and with the chip full the clock gives way: a loop of nothing but these
// multiplies on random operands reaches 1.6-1.9 PFLOP/s here, on zeros 2.45.  conv1 to conv5, 64 images, us of this launch in the network (conv_mfma_kernel's):
// 114 (163), 148 (187), 95 (114), 75 (125), 54 (71), of preparing 24, 20, 16, 18, 18 (of decoding 7-8); VGG-16 conv4_2 at one image 29.7 (36.6).
template <int NP, int RT, int CT, int WR, int WC>
__global__ __launch_bounds__(256, 2) void conv_plane_kernel(const uint4 *__restrict__ wt, const uint4 *__restrict__ xs, const uint32_t *__restrict__ unit_off,
                                                            float *part, PlaneConv g)
{
    constexpr int TR = 32 * RT * WR, TC = 32 * CT * WC;
    static_assert(WR * WC == 4 && TC == 128, "");
    constexpr int kA = NP * 2 * TR, kB = NP * 2 * TC;       // pieces of a step
    constexpr int kLoads = (kA / 64 + 3) / 4 + kB / 256;    // of a wavefront and step
    constexpr int kWaitLds = 0xc07f, kWaitLoads = 0xf70;    // s_waitcnt: no LDS access left; no load left, or-ed with n < 16: n left
    static_assert(2 * kLoads < 16, "");
    __shared__ uint4 lds0[kA + kB], lds1[kA + kB], lds2[kA + kB];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    // Workgroups go to the eight dies in turn: each die takes a run of items, in which the tiles of rows come first,
    // then those of columns, then the splits, so that what a die has in flight shares steps and operands.
    const int items = g.panels * g.tiles * g.splits;
    int item = (int)blockIdx.x;
    {
        const int per = items / 8, more = items % 8, die = item % 8, i = item / 8;
        item = die * per + min(die, more) + i;
    }
    const int p = item % g.panels;
    const int nb = (item / g.panels) % g.tiles;
    const int j = item / (g.panels * g.tiles);
    const int t0 = (int)(((int64_t)g.steps * j) / g.splits), t1 = (int)(((int64_t)g.steps * (j + 1)) / g.splits);

    // a wavefront fetches 64 columns of one of the step's units
    const int cq = wave >> 1, unit = wave & 1;
    uint32_t at;
    {
        const int n = min(nb * TC + 64 * cq + lane, g.n_cols - 1);
        const int img = n / g.pq, o = n - img * g.pq, oy = o / g.Q, ox = o - oy * g.Q;
        at = (uint32_t)img * g.image_bytes + (uint32_t)(p / g.ppg) * g.group_bytes + (uint32_t)((oy * g.Wp + ox) * g.stride * g.px_bytes);
    }
    const __amdgpu_buffer_rsrc_t xb = __builtin_amdgcn_make_buffer_rsrc((void *)xs, 0, (int)(NP * g.term_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t wb =
        __builtin_amdgcn_make_buffer_rsrc((void *)(wt + (size_t)p * g.steps * kA), 0, g.steps * (kA * 16), 0x00020000);
    // where the wavefront's unit of the step to be requested sits, and that of the step after it
    uint32_t off = unit_off[2 * t0 + unit], off_next = 0;
    auto next_off = [&](int t) {
        off = off_next;
        off_next = unit_off[2 * min(t, g.steps - 1) + unit];
    };
    // load i of the wavefront's kLoads of step t
    constexpr int kLoadsA = (kA / 64 + 3) / 4;
    auto request_one = [&](int t, uint4 *buf, int i) {
        if (i < kLoadsA) {
            // (every wavefront the same number: some of the last pieces twice)
            const int q = min(4 * i + wave, kA / 64 - 1);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wb, (lds_ptr)(buf + 64 * q), 16, 16 * lane, t * (kA * 16) + 1024 * q, 0, 0);
        } else {
            const int k = i - kLoadsA;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (lds_ptr)(buf + kA + (2 * k + unit) * TC + 64 * cq), 16, (int)at, (int)((uint32_t)k * g.term_bytes + off), 0, 0);
        }
    };
    // all of them, also of a step whose second unit does not exist
    auto request = [&](int t, uint4 *buf) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            if (i < kLoadsA || off != 0xffffffffu) request_one(t, buf, i);
            else buf[kA + (2 * (i - kLoadsA) + unit) * TC + 64 * cq + lane] = uint4{0, 0, 0, 0};
        }
    };

    const int wr = wave / WC, wc = wave % WC;
    const int kl = lane >> 5, m = lane & 31;
    // the products formed, smallest first: term of the activation, term of the weight
    constexpr int kProducts = NP == 3 ? 8 : 3;
    constexpr int kTermX[8] = {NP == 3 ? 2 : 1, NP == 3 ? 1 : 0, NP == 3 ? 2 : 0, 0, 1, 1, 0, 0};
    constexpr int kTermW[8] = {NP == 3 ? 1 : 0, NP == 3 ? 2 : 1, 0, 2, 1, 0, 1, 0};
    struct Frags {
        uint4 w[RT][NP], x[CT][NP];
    };
    constexpr int kReads = NP * (RT + CT);
    auto read_one = [&](const uint4 *buf, Frags &f, int n) {
        const int i = n / (RT + CT), q = n % (RT + CT);
        if (q < RT) f.w[q][i] = buf[(2 * i + kl) * TR + 32 * (RT * wr + q) + m];
        else f.x[q - RT][i] = buf[kA + (2 * i + kl) * TC + 32 * (CT * wc + q - RT) + m];
    };
    auto read = [&](const uint4 *buf, Frags &f) {
#pragma unroll
        for (int n = 0; n < kReads; ++n) read_one(buf, f, n);
    };
    floatx16 acc[RT][CT], lo[NP == 3 ? RT : 1][NP == 3 ? CT : 1];
#pragma unroll
    for (auto &a : acc)
#pragma unroll
        for (auto &b : a) b = floatx16{0};
#pragma unroll
    for (auto &a : lo)
#pragma unroll
        for (auto &b : a) b = floatx16{0};
    constexpr int kMfmas = kProducts * RT * CT;
    auto multiply_one = [&](const Frags &f, int n) {
        const int pr = n / (RT * CT), r = n % (RT * CT) / CT, c = n % CT;
        floatx16 &sum = NP == 3 && pr + 1 < kProducts ? lo[r][c] : acc[r][c];
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.w[r][kTermW[pr]]), __builtin_bit_cast(bf16x8, f.x[c][kTermX[pr]]), sum, 0,
                                                      0, 0);
    };

    Frags f0, f1;
    // Step t, whose pieces are in `now`: step t + 1 is read from `from`, step t + 3 requested into `to`, which step t was read
    // from.  At its start step t + 1 has arrived (the wavefront's loads of t + 2 may be on their way) and step t is read.
    auto meet = [&](bool more) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        if (more) __builtin_amdgcn_s_waitcnt(kWaitLoads | kLoads);
        else __builtin_amdgcn_s_waitcnt(kWaitLoads);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // Reads and requests go out between the multiplies, in program order (scheduling barriers): in one bunch behind
    // the barrier they would fill the LDS's and the loads' queues, and the multiplies would wait for a place behind them.
    auto step = [&](int t, const Frags &now, Frags &next, const uint4 *__restrict__ from, uint4 *__restrict__ to) {
        meet(true);
        next_off(t + 4);
        constexpr int kActions = kReads + kLoads, kOver = kMfmas * 3 / 4;
#pragma unroll
        for (int n = 0; n < kMfmas; ++n) {
#pragma unroll
            for (int k = 0; k < kActions; ++k)
                if (k * kOver / kActions == n) {
                    if (k < kReads) read_one(from, next, k);
                    else request_one(t + 3, to, k - kReads);
                    __builtin_amdgcn_sched_barrier(0);
                }
            multiply_one(now, n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto last_step = [&](int t, const Frags &now, Frags &next, const uint4 *__restrict__ from, uint4 *__restrict__ to) {
        meet(t + 3 < t1);
        next_off(t + 4);
        if (t + 1 < t1) read(from, next);
        if (t + 3 < t1) request(t + 3, to);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < kMfmas; ++n) multiply_one(now, n);
        __builtin_amdgcn_sched_barrier(0);
    };
    off_next = unit_off[2 * min(t0 + 1, g.steps - 1) + unit];
    request(t0, lds0);
    next_off(t0 + 2);
    if (t0 + 1 < t1) request(t0 + 1, lds1);
    next_off(t0 + 3);
    if (t0 + 2 < t1) request(t0 + 2, lds2);
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    if (t0 + 3 < t1) __builtin_amdgcn_s_waitcnt(kWaitLoads | 2 * kLoads);
    else __builtin_amdgcn_s_waitcnt(kWaitLoads);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read(lds0, f0);
    // (six steps: buffers by threes, registers by twos.  The steps whose requests might be for the last one go the other way.)
    int t = t0;
    for (; t + 9 < t1; t += 6) {
        step(t, f0, f1, lds1, lds0);
        step(t + 1, f1, f0, lds2, lds1);
        step(t + 2, f0, f1, lds0, lds2);
        step(t + 3, f1, f0, lds1, lds0);
        step(t + 4, f0, f1, lds2, lds1);
        step(t + 5, f1, f0, lds0, lds2);
    }
    for (; t < t1; t += 6) {
        last_step(t, f0, f1, lds1, lds0);
        if (t + 1 >= t1) break;
        last_step(t + 1, f1, f0, lds2, lds1);
        if (t + 2 >= t1) break;
        last_step(t + 2, f0, f1, lds0, lds2);
        if (t + 3 >= t1) break;
        last_step(t + 3, f1, f0, lds1, lds0);
        if (t + 4 >= t1) break;
        last_step(t + 4, f0, f1, lds2, lds1);
        if (t + 5 >= t1) break;
        last_step(t + 5, f1, f0, lds0, lds2);
    }
    if constexpr (NP == 3) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[r][c] += lo[r][c];
    }

    // element e of lane (kl, m): row 8 (e / 4) + 4 kl + e % 4 of the accumulator, column m: 32 lanes have 32
    // consecutive columns of a row, as the output has them
    const int grp = p / g.ppg, row0 = (p - grp * g.ppg) * TR;              // first filter of the tile, in its group
    const int rows = min(TR, g.OCg - row0);
    const int step_floats = g.Y ? g.pq : g.Np;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int base = 32 * (RT * wr + r) + 4 * kl;
        float b[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) b[e] = 0.0f;
        if (g.Y && g.bias) {
#pragma unroll
            for (int e = 0; e < 16; ++e) b[e] = g.bias[grp * g.OCg + row0 + min(base + 8 * (e / 4) + (e & 3), rows - 1)];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int n = nb * TC + 32 * (CT * wc + c) + m;
            if (g.Y && n >= g.n_cols) continue;
            float *to = g.Y ? g.Y + ((size_t)(n / g.pq) * g.M + grp * g.OCg + row0) * g.pq + n % g.pq : part + (size_t)(p * g.splits + j) * TR * g.Np + n;
            to += (size_t)(uint32_t)(base * step_floats);
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (base + 8 * e4 + e < rows) {
                        const float y = acc[r][c][4 * e4 + e] + b[4 * e4 + e];
                        *to = g.Y && g.relu ? fmaxf(y, 0.0f) : y;
                    }
                    to += step_floats;
                }
                to += 4 * step_floats;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}
