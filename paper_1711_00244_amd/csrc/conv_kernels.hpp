// Convolution as a matrix product without the column matrix in memory (Sec. III-A builds
// it; here the receptive fields are gathered straight into LDS): conv_mfma_kernel.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

// The products run on the bf16 matrix cores, sixteen times the fp32 ones' rate.  With NP = 3
// (the fp32 path) a weight and an activation are each split into three bf16 terms, w = w1 + w2 +
// w3 and x = x1 + x2 + x3 (split8): together they are the 24 bits of an fp32 value, nothing is
// rounded away.  Six of the nine products are formed - x1 w1, x1 w2, x2 w1, x2 w2, x1 w3, x3 w1 -,
// all exact, and added in fp32; what is left out is below 2^-24 |w x|, an fp32 product's own rounding.
// With NP = 2 (the bf16 path) three of two terms' four, as in fc_mfma_bf16_kernel.
//
// Workgroup = (block row p of the filters, split j of its blocks, tile of 128 columns =
// image x output pixel) of wavefronts in two roles that meet at one barrier per phase, a
// phase being half a block (64 of its columns):
//   Gatherers (wavefronts 4-11) build, one phase ahead, the 64 x 128 piece of the
//   column matrix that the next phase multiplies - row kk is (c, r, s) of the block's
//   column kk, column n an output pixel - in one of two LDS buffers, split, reading the NCHW
//   input directly (zero outside the image, past the last column and for rows the block
//   does not have).  A row is uniform per wavefront, a lane owns two columns (l and l + 64:
//   the 64 lanes of a load read neighbouring pixels) for the workgroup's whole life, so
//   where its pixels sit in the input, and which filter taps
//   fall outside the image there, is worked out once (COMBINED: one bit per tap, for
//   filters of at most 32 taps; else one bit per filter row and one per filter column).
//   What a row is - its offset from a receptive field's corner, its tap - comes from the
//   table that decode_tiles_kernel writes (`rows`), read with uniform loads.  A lane's eight
//   rows of a column are the eight k of a matrix operand: one 16-byte LDS store per plane.
//   Multipliers (wavefronts 0-3, one per SIMD): wavefront w owns filter rows 32w..32w+31
//   and all 128 columns in four 32 x 32 accumulators (other divisions for lower blocks,
//   below).  Weights come from device memory (every block decoded
//   once per call by decode_tiles_kernel; 32 lanes' pieces are contiguous) and are split on the
//   way, in the shadow of the multiplies; activations from LDS (a piece of 32 columns x 8 k is
//   512 contiguous bytes).
// (On the fp32 matrix cores, at nine tenths of their rate, VGG-16 conv4_2 took 45.7 us for one
// image and AlexNet's conv2 to conv5 185 us on average for 64; now 29.5 and 107.)
constexpr int conv_gatherers(int planes) { return planes == 3 ? 4 : 8; }   // wavefronts (eight leave too few registers for two sums)
constexpr int conv_threads(int planes) { return (4 + conv_gatherers(planes)) * 64; }
constexpr int kConvColumns = kTile;                        // columns per workgroup
constexpr int kConvPhase = 64;                             // rows of the column matrix per phase
constexpr int kConvSteps = kConvPhase / 16;                // matrix-multiply steps of a phase
constexpr int kConvPlane = kConvPhase / 8 * kConvColumns;  // 16-byte pieces of a phase, per plane
// halves of a block that have columns
__host__ __device__ constexpr int conv_halves(int bw) { return bw > kConvPhase ? 2 : 1; }
// (at the end the multipliers turn their four pieces of the output there)
constexpr int conv_lds_bytes(int planes)
{
    const int buffers = 2 * planes * kConvPlane * 16, turned = 4 * 32 * (kTile + 1) * 4;
    return buffers > turned ? buffers : turned;
}

// Eight fp32 values as NP (2 or 3) bf16 terms each, largest first: each term is what is left of
// the value, rounded to the nearest bf16.  Three terms are the value itself (8 + 8 + 8 bits; below
// 2^-110 the last ones run into bf16's smallest numbers), two leave less than 2^-16 of it.
// terms[i] holds term i of all eight, in order.  An infinity or NaN becomes the last term
// alone, the one that is multiplied with the other side's first term only: it meets every weight once,
// and so gives what it gives in fp32.
template <int NP> __device__ __forceinline__ void split8(const float (&v)[8], uint4 (&terms)[NP])
{
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    uint32_t t[NP][4];
    float odd = 0.0f;                                       // not finite where a value or its first term is not
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = v[2 * j], b = v[2 * j + 1];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            t[i][j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf2));
            if (i + 1 == NP) break;
            a -= __uint_as_float(t[i][j] << 16);
            b -= __uint_as_float(t[i][j] & 0xffff0000u);
            if (i == 0) odd += a + b;
        }
    }
    if (!(__builtin_fabsf(odd) < __builtin_inff())) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t u = __float_as_uint(v[j]), put = 16 * (j & 1), keep = 0xffffu << (16 - put);
            const bool finite = (u & 0x7f800000u) != 0x7f800000u;
            // (the first term cut off, not rounded: it cannot overflow)
            float a = v[j];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                uint32_t term;
                if (!finite) term = i + 1 < NP ? 0u : (u >> 16) | ((u & 0x7fffffu) ? 0x40u : 0u);
                else if (i == 0) term = u >> 16;
                else term = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, a}), bf2)) & 0xffffu;
                t[i][j / 2] = (t[i][j / 2] & keep) | term << put;
                a -= __uint_as_float(term << 16);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) terms[i] = uint4{t[i][0], t[i][1], t[i][2], t[i][3]};
}

// Two weights (finite) as NP bf16 terms each, a pair to a word.  Of three terms the first is cut
// off, not rounded, so that it cannot overflow; of two it is rounded, which leaves less.
template <int NP> __device__ __forceinline__ void split_weights(float a, float b, uint32_t (&t)[NP])
{
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (NP == 3 && i == 0) t[i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
        else t[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf2));
        if (i + 1 == NP) break;
        a -= __uint_as_float(t[i] << 16);
        b -= __uint_as_float(t[i] & 0xffff0000u);
    }
}

template <bool COMBINED, int S, int Q, int NP>
__global__ __launch_bounds__(conv_threads(NP)) void conv_mfma_kernel(LayerDev L, const float *__restrict__ X, const float *__restrict__ wt,
                                                                 const uint2 *__restrict__ rows, float *part, ConvGeom cg, int n_cols,
                                                                 int Np, int splits, int panels_per_group, DirectOut out)
{
    extern __shared__ __attribute__((aligned(16))) uint4 act[];        // [2][NP][8][128 columns], eight k to a piece
    const int nbt = Np / kConvColumns;
    const int nb = (int)blockIdx.x % nbt;
    const int pj = (int)blockIdx.x / nbt;
    const int p = pj / splits, j = pj % splits;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const int blk_lo = (int)(((int64_t)L.nbw * j) / splits), blk_hi = (int)(((int64_t)L.nbw * (j + 1)) / splits);
    const uint32_t pb0 = (uint32_t)p * (uint32_t)L.nbw;
    // a ragged last block may do without its second half
    const int nh = conv_halves(L.bw);
    const int phases = (blk_hi - blk_lo) * nh - (blk_hi == L.nbw ? nh - conv_halves(L.K - (L.nbw - 1) * L.bw) : 0);

    if (wave >= 4) {
        const int d = wave - 4;
        const int pq = cg.P * cg.Q, plane = cg.H * cg.W;
        const int c0 = (p / panels_per_group) * cg.Cg;              // the filter group's input channels
        // The input is read through a buffer descriptor that starts at the tile's first
        // image, channel c0, moved back by the padding so that a receptive field's corner
        // has a non-negative offset (the launcher keeps 129 images under 2^29 elements, so
        // byte offsets stay below 2^31), and ends with the input: a load past its end returns
        // zero.  That is also how an element outside the image is read - its offset is turned
        // into 0xffffffff - so a gathered element costs a bit test, an add, an or and a load,
        // with no branch.  (Word 3 of the descriptor: 32-bit elements, plain addressing.)
        const int img0 = nb * kConvColumns / pq;
        const int n_img = (n_cols + pq - 1) / pq;
        const int64_t back = (int64_t)cg.pad * cg.W + cg.pad;
        const int64_t span = (((int64_t)(n_img - img0) * cg.C - c0) * plane + back) * (int64_t)sizeof(float);
        const __amdgpu_buffer_rsrc_t xb = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(X + ((int64_t)img0 * cg.C + c0) * plane - back), 0, (int)std::min<int64_t>(span, 0x7fffffff), 0x00020000);
        // The lane's two columns: byte offset of the corner of each pixel's receptive field,
        // and which (r, s) fall outside the image - one bit per (r, s) when the filter has
        // at most 32 taps, else one per r and one per s.  Columns past the last are all outside.
        uint32_t at[2], bad[2], bad_s[2];
        {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int n = nb * kConvColumns + lane + 64 * i;
                const int img = n / pq;
                const int o = n - img * pq;
                const int oy = o / cg.Q, ox = o - oy * cg.Q;
                const int y0 = oy * cg.stride - cg.pad, x0 = ox * cg.stride - cg.pad;
                at[i] = (uint32_t)((img - img0) * cg.C * plane + oy * cg.stride * cg.W + ox * cg.stride) * (uint32_t)sizeof(float);
                uint32_t rb = 0, sb = 0;
                for (int r = 0; r < cg.R; ++r) rb |= (uint32_t)((unsigned)(y0 + r) >= (unsigned)cg.H) << r;
                for (int sx = 0; sx < cg.S; ++sx) sb |= (uint32_t)((unsigned)(x0 + sx) >= (unsigned)cg.W) << sx;
                if (n >= n_cols) rb = sb = 0xffffffffu;
                if (COMBINED) {
                    const uint32_t all_s = cg.S >= 32 ? 0xffffffffu : (1u << cg.S) - 1u;
                    uint32_t both = 0;
                    for (int r = 0; r < cg.R; ++r) both |= ((rb >> r) & 1u ? all_s : (sb & all_s)) << (r * cg.S);
                    rb = both;
                }
                bad[i] = rb;
                bad_s[i] = sb;
            }
        }
        // Wavefront d gathers groups kGroups d .. kGroups (d + 1) - 1 of eight rows of a piece; what
        // a row is comes from the table (uniform loads), so a row costs no arithmetic of its own.
        constexpr int kGroups = kConvPhase / 8 / conv_gatherers(NP);
        float v[kGroups][2][8];
        auto fetch = [&](int ph) {
            const uint2 *rp = rows + ((blk_lo + ph / nh) * kTile + (ph % nh) * kConvPhase + 8 * kGroups * d);
#pragma unroll
            for (int jj = 0; jj < 8 * kGroups; ++jj) {
                const uint2 e = rp[jj];
                const uint32_t no_row = (uint32_t)((int)e.y >> 31);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t out = COMBINED ? (uint32_t)__builtin_amdgcn_sbfe(bad[i], e.y & 0xffu, 1)
                                                  : (uint32_t)(__builtin_amdgcn_sbfe(bad[i], e.y & 0xffu, 1) |
                                                               __builtin_amdgcn_sbfe(bad_s[i], (e.y >> 8) & 0xffu, 1));
                    v[jj / 8][i][jj % 8] =
                        __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xb, (int)((at[i] + e.x) | out | no_row), 0, 0));
                }
            }
        };
        // (the loads of a piece are in flight across the barrier before the one it is for)
        if (phases > 0) fetch(0);
        for (int ph = 0; ph < phases; ++ph) {
            uint4 *dst = act + (ph & 1) * (NP * kConvPlane) + kGroups * d * kConvColumns + lane;
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    uint4 terms[NP];
                    split8<NP>(v[g][i], terms);
#pragma unroll
                    for (int t = 0; t < NP; ++t) dst[t * kConvPlane + g * kConvColumns + 64 * i] = terms[t];
                }
            if (ph + 1 < phases) fetch(ph + 1);
            __syncthreads();
        }
        __syncthreads();
        return;
    }

    // S x Q accumulators of 32 filter rows x 32 columns per multiplying wavefront w, by the
    // height of the layer's blocks:
    //   up to 128 rows (S = 1, Q = 4): rows 32 w .. 32 w + 31, all 128 columns;
    //   up to  96 rows (S = 3, Q = 1): all 96 rows, columns 32 w .. 32 w + 31;
    //   up to  64 rows (S = 1, Q = 2): rows 32 (w % 2) .., columns 64 (w / 2) .. + 63;
    // so that no wavefront multiplies rows that no block has.  Accumulator (s, q) holds,
    // for element e of lane (kl, m), filter row 32 (sbase + s) + m and column
    // cbase + 32 q + i of the tile, i = 8 (e / 4) + 4 kl + e % 4.
    const int sbase = S == 3 ? 0 : (Q == 4 ? wave : wave & 1);
    const int cbase = S == 3 ? 32 * wave : (Q == 4 ? 0 : 64 * (wave >> 1));
    floatx16 acc[S][Q];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[s][q] = floatx16{0};
    // With three terms the products other than x1 w1 have sums of their own, added at the end: in one
    // sum with it each of six additions per step would round at its size (error against 64 bits,
    // 201 channels of 3 x 3: 3.2e-7, with two sums
    // 1.0e-7, on the fp32 matrix cores 2.5e-7)
    floatx16 lo[NP == 3 ? S : 1][NP == 3 ? Q : 1];
#pragma unroll
    for (auto &ls : lo)
#pragma unroll
        for (auto &l : ls) l = floatx16{0};
    const int kl = lane >> 5, m = lane & 31;
    // A unit is a step of one strip: its eight weights per lane, in two 16-byte pieces (a piece:
    // four columns of a row; 128 rows, then the next four columns).  Unit u is multiplied while
    // u + 1 is split and the kRaw after that are on their way.
    constexpr int kUnits = S * kConvSteps;                  // of a phase
    constexpr int kRaw = S == 3 ? 6 : Q == 4 ? 2 : 4;
    static_assert(kUnits % kRaw == 0 && kUnits % 2 == 0, "a unit's registers are the same in every phase");
    const int last_step = phases * kConvSteps - 1;
    const float4 *wf = (const float4 *)wt + ((size_t)(pb0 + (uint32_t)blk_lo) * (kTile / 4) + 2 * kl) * kTile + 32 * sbase + m;
    float raw[kRaw][8];
    uint32_t w[2][NP][4];
    auto load_unit = [&](int t, int s, float (&dst)[8]) {
        // (past the last step: the last one's again, never multiplied)
        t = min(t, last_step);
        const float4 *src = wf + (size_t)(nh == 2 ? t : t + (t & ~(kConvSteps - 1))) * (4 * kTile) + 32 * s;
        load_floats<4>((const float *)src, dst);
        load_floats<4>((const float *)(src + kTile), dst + 4);
    };
    auto split_pair = [&](const float (&v)[8], int j, uint32_t (&dst)[NP][4]) {
        uint32_t t[NP];
        split_weights<NP>(v[2 * j], v[2 * j + 1], t);
#pragma unroll
        for (int i = 0; i < NP; ++i) dst[i][j] = t[i];
    };
    if (phases > 0) {
        float first[8];
        load_unit(0, 0, first);
#pragma unroll
        for (int u = 1; u <= kRaw; ++u) load_unit(u / S, u % S, raw[u % kRaw]);
#pragma unroll
        for (int j = 0; j < 4; ++j) split_pair(first, j, w[0]);
    }
    // the products formed, smallest first: term of the activation, term of the weight
    constexpr int kProducts = NP == 3 ? 6 : 3;
    constexpr int kTermX[6] = {NP == 3 ? 2 : 1, 0, NP == 3 ? 1 : 0, 1, 0, 0}, kTermW[6] = {0, NP == 3 ? 2 : 1, NP == 3 ? 1 : 0, 0, 1, 0};
    constexpr int QB = Q > 1 ? 2 : 1;                       // accumulators multiplied in turn: their chains hide each other's latency
    for (int ph = 0; ph < phases; ++ph) {
        __syncthreads();                                    // this piece gathered
        const uint4 *ap = act + (ph & 1) * (NP * kConvPlane) + kl * kConvColumns + cbase + m;
        uint4 x[2][QB][NP];
        auto load_x = [&](int idx, uint4 (&dst)[QB][NP]) {  // idx = step * (Q / QB) + group of QB accumulators
            const uint4 *src = ap + (idx / (Q / QB)) * (2 * kConvColumns) + (idx % (Q / QB)) * (32 * QB);
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int i = 0; i < NP; ++i) dst[q][i] = src[i * kConvPlane + 32 * q];
        };
        load_x(0, x[0]);
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int st = u / S, s = u % S;
            constexpr int kSlots = kProducts * (Q / QB), kPairs = (4 + kSlots - 1) / kSlots;
            float (&next)[8] = raw[(u + 1) % kRaw];
#pragma unroll
            for (int qb = 0; qb < Q / QB; ++qb) {
                const int idx = st * (Q / QB) + qb;
                // program order is pinned (scheduling barriers): left alone, the compiler sinks the
                // loads to just before their use and their latency lands in front of the multiplies
                __builtin_amdgcn_sched_barrier(0);
                if (s == 0 && idx + 1 < kConvSteps * (Q / QB)) load_x(idx + 1, x[(idx + 1) & 1]);
#pragma unroll
                for (int pr = 0; pr < kProducts; ++pr) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < QB; ++q) {
                        const uint32_t (&ww)[4] = w[u & 1][kTermW[pr]];
                        floatx16 &sum = NP == 3 && pr + 1 < kProducts ? lo[s][qb * QB + q] : acc[s][qb * QB + q];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[idx & 1][q][kTermX[pr]]),
                                                                      __builtin_bit_cast(bf16x8, (uint4{ww[0], ww[1], ww[2], ww[3]})), sum, 0, 0, 0);
                    }
                    // the next unit's split, a pair or two behind each multiply
                    const int slot = qb * kProducts + pr;
#pragma unroll
                    for (int j = slot * kPairs; j < min((slot + 1) * kPairs, 4); ++j) split_pair(next, j, w[(u + 1) & 1]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            load_unit(ph * kConvSteps + (u + 1 + kRaw) / S, (u + 1 + kRaw) % S, next);
        }
    }
    __syncthreads();                                        // done with the last piece
    if constexpr (NP == 3) {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int q = 0; q < Q; ++q) acc[s][q] += lo[s][q];
    }

    const int row_id = p * L.bh;
    const int block_rows = min(L.bh, L.M - row_id);
    if (!out.Y) {
        // the workgroup's partial tile for the finishing kernel: 32 lanes write 32 consecutive rows of a column
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (32 * (sbase + s) + m >= block_rows) continue;
            float *mine = part + ((size_t)pj * Np + (size_t)nb * kConvColumns + cbase) * L.bh + 32 * (sbase + s) + m;
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int q = 0; q < Q; ++q) mine[(size_t)(32 * q + 8 * (e / 4) + 4 * kl + (e & 3)) * L.bh] = acc[s][q][e];
        }
        return;
    }
    // The finished output (block rows that are not split).  The output runs along the
    // columns, the accumulators along the rows: the wavefront turns its 32 S x 32 Q piece in
    // its own part of LDS (the tiles are free: the last barrier was every wavefront's last
    // use of them), then writes each filter row's columns as one run - two rows at a time
    // where a row has 32 columns - bias (lane l holds that of row l % 32 of each strip) and
    // activation on the way.
    constexpr int kCols = 32 * Q, kStride = kCols + 1;
    constexpr int kPerLane = kCols > 64 ? kCols / 64 : 1;       // columns of a row per lane
    constexpr int kRowsAtOnce = kCols < 64 ? 64 / kCols : 1;    // rows per pass of the wavefront
    float *t = (float *)act + wave * (32 * S) * kStride;
    static_assert(4 * 32 * S * kStride * 4 <= conv_lds_bytes(NP), "the pieces fit where the activations were");
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int e = 0; e < 16; ++e)
#pragma unroll
            for (int q = 0; q < Q; ++q) t[(32 * s + m) * kStride + 32 * q + 8 * (e / 4) + 4 * kl + (e & 3)] = acc[s][q][e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int my_col = kRowsAtOnce > 1 ? lane % kCols : lane, my_row = kRowsAtOnce > 1 ? lane / kCols : 0;
    size_t y_at[kPerLane];
    bool live[kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
        const int c = nb * kConvColumns + cbase + my_col + 64 * i;
        live[i] = c < out.ncols;
        y_at[i] = ((size_t)(c / out.pq) * L.M + row_id) * out.pq + (c % out.pq);
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int first = 32 * (sbase + s);                       // the strip's first row in the block
        const int n_rows = min(32, block_rows - first);
        const float bias_l = out.bias && m < n_rows ? out.bias[row_id + first + m] : 0.0f;
        for (int r0 = 0; r0 < n_rows; r0 += 8 * kRowsAtOnce) {
            float y[8][kPerLane];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int ru = min(r0 + kRowsAtOnce * u, 31);     // uniform; this lane's row is ru + my_row
                const float b0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, bias_l), ru));
                const float b1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, bias_l), min(ru + 1, 31)));
                const int rr = min(ru + my_row, 31);
#pragma unroll
                for (int i = 0; i < kPerLane; ++i) y[u][i] = t[(32 * s + rr) * kStride + my_col + 64 * i] + (my_row ? b1 : b0);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int rr = r0 + kRowsAtOnce * u + my_row;
                if (rr >= n_rows) continue;
#pragma unroll
                for (int i = 0; i < kPerLane; ++i)
                    if (live[i]) out.Y[y_at[i] + (size_t)(first + rr) * out.pq] = out.relu ? fmaxf(y[u][i], 0.0f) : y[u][i];
            }
        }
    }
}
