// Convolution as a matrix product without the column matrix in memory (Sec. III-A builds
// it; here the receptive fields are gathered straight into LDS): conv_mfma_kernel.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

// The products run on the bf16 matrix cores, sixteen times the fp32 ones' rate.  With NP = 3
// (the fp32 path) a weight and an activation are each split into three bf16 terms, w = w1 + w2 +
// w3 and x = x1 + x2 + x3 (split8): together they are the 24 bits of an fp32 value, nothing is
// rounded away.  Eight of the nine products are formed, all but x3 w3, which is below 2^-32 |w x|; they
// are exact and added in fp32, so that an output with a single surviving weight is rounded once,
// as an fp32 multiply-add rounds it.  (Without x2 w3 and x3 w2, up to 1.95 * 2^-24 |w x|, such an output was
// off by up to 1.4e-7 instead of 6e-8; VGG-16 conv4_2 at one image took 41.4 us, now 44.7, AlexNet at 64
// images 767, now 828.)
// With NP = 2 (the bf16 path) three of two terms' four, as in fc_mfma_bf16_kernel.
//
// Workgroup = (block row p of the filters, split j of its blocks, tile of 128 columns =
// image x output pixel) of wavefronts in two roles that meet at one barrier per phase, a
// phase being half a block (64 of its columns):
//   Gatherers (wavefronts 4 on) build, two phases ahead, 64 x 128 pieces of the
//   column matrix - row kk is (c, r, s) of the block's
//   column kk, column n an output pixel - in one of three LDS buffers, split, reading the NCHW
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
// A workgroup per CU takes item after item (block row, split, tile of columns): the gatherers are
// at the next one's first piece while the multipliers write the last one's output.
// Bound by the instructions issued: a vector instruction adds its four cycles to the multiplies' time here, and
// there are some 600 of them per phase and SIMD, gathering and splitting, to 128 multiplies of 32 cycles.
// (AlexNet conv1 to conv5, 64 images, us: 156, 182, 111, 118, 68, with six products 149, 155, 96, 105, 60; on
// the fp32 matrix cores, at nine tenths of their rate, 202, 240, 150, 149, 95.  A workgroup per item instead
// of per CU, six products: conv1 178 for 151.)
constexpr int conv_gatherers(int planes) { return planes == 3 ? 4 : 8; }   // wavefronts (eight leave too few registers for two sums)
constexpr int conv_threads(int planes) { return (4 + conv_gatherers(planes)) * 64; }
constexpr int kConvColumns = kTile;                        // columns per workgroup
constexpr int kConvPhase = 64;                             // rows of the column matrix per phase
constexpr int kConvSteps = kConvPhase / 16;                // matrix-multiply steps of a phase
constexpr int kConvPlane = kConvPhase / 8 * kConvColumns;  // 16-byte pieces of a phase, per plane
// halves of a block that have columns
__host__ __device__ constexpr int conv_halves(int bw) { return bw > kConvPhase ? 2 : 1; }
constexpr int kConvBuffers = 3;
constexpr int conv_lds_bytes(int planes) { return kConvBuffers * planes * kConvPlane * 16; }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two values rounded to the nearest bf16
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf16x2));
}

// What is left of two values without their terms.  (v_dot2_f32_bf16 would take one instruction a value, not
// two, and is exact here, but VGG-16 conv4_2 took 34.2 us with it and 30.5 without.)
__device__ __forceinline__ void bf16_rest(uint32_t t, float &a, float &b)
{
    a -= __uint_as_float(t << 16);
    b -= __uint_as_float(t & 0xffff0000u);
}

// Eight fp32 values as NP (2 or 3) bf16 terms each, largest first: each term is what is left of
// the value, rounded to the nearest bf16.  Three terms are the value itself (8 + 8 + 8 bits; below
// 2^-110 the last one can be smaller than bf16's smallest number, 2^-133, and is rounded to a multiple of
// it), two leave less than 2^-16 of it.
// terms[i] holds term i of all eight, in order.  An infinity becomes the last term
// alone, the one that is multiplied with the other side's first two terms only, which have the
// weight's sign or, for a weight of zero, are zero (split_weights): so it gives what it gives in fp32.
template <int NP> __device__ __forceinline__ void split8(const float (&v)[8], uint4 (&terms)[NP])
{
    uint32_t t[NP][4];
    float most = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = v[2 * j], b = v[2 * j + 1];
        most = fmaxf(fmaxf(most, __builtin_fabsf(a)), __builtin_fabsf(b));
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            t[i][j] = bf16_pair(a, b);
            if (i + 1 < NP) bf16_rest(t[i][j], a, b);
        }
    }
    if (most >= 3.3895e38f) {                               // (the largest bf16 and half a step: 0x7f7f8000 is 3.39615e38)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // (the others as they are: whoever sees them and not this one gets what it would without it)
            if (__builtin_fabsf(v[j]) < 3.3895e38f) continue;
            const uint32_t u = __float_as_uint(v[j]), put = 16 * (j & 1), keep = 0xffffu << (16 - put);
            const bool finite = (u & 0x7f800000u) != 0x7f800000u;
            // (the first term cut off, not rounded: it cannot overflow)
            float a = v[j];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                uint32_t term;
                if (!finite) term = i + 1 < NP ? 0u : (u >> 16) | ((u & 0x7fffffu) ? 0x40u : 0u);
                else if (i == 0) term = u >> 16;
                else term = bf16_pair(a, a) & 0xffffu;
                t[i][j / 2] = (t[i][j / 2] & keep) | term << put;
                a -= __uint_as_float(term << 16);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) terms[i] = uint4{t[i][0], t[i][1], t[i][2], t[i][3]};
}

// Two weights (finite) as NP bf16 terms each, a pair to a word.  Of three terms the first is the
// largest bf16 whose magnitude is below the weight's: it cannot overflow, and what it leaves has the
// weight's sign and is zero for a zero only (split8; the subtraction saturates, so that +0 stays +0; the
// launcher keeps -0 and values below 2^-110 away).  Of two it is rounded, which leaves less.
template <int NP> __device__ __forceinline__ void split_weights(float a, float b, uint32_t (&t)[NP])
{
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (NP == 3 && i == 0)
            t[i] = __builtin_amdgcn_perm(__builtin_elementwise_sub_sat(__float_as_uint(b), 1u), __builtin_elementwise_sub_sat(__float_as_uint(a), 1u), 0x07060302u);
        else t[i] = bf16_pair(a, b);
        if (i + 1 < NP) bf16_rest(t[i], a, b);
    }
}

template <bool COMBINED, int Q, int NP>
__global__ __launch_bounds__(conv_threads(NP)) void conv_mfma_kernel(LayerDev L, const float *__restrict__ X, const float *__restrict__ wt,
                                                                 const uint2 *__restrict__ rows, float *part, ConvGeom cg, int n_cols,
                                                                 int Np, int splits, int panels_per_group, int items, DirectOut out)
{
    extern __shared__ __attribute__((aligned(16))) uint4 act[];        // [kConvBuffers][NP][8][128 columns], eight k to a piece
    const int nbt = Np / kConvColumns;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const int nh = conv_halves(L.bw);
    // item -> tile of columns, block row, its blocks blk_lo .. blk_hi - 1 and their phases (a
    // ragged last block may do without its second half)
    struct Item {
        int nb, pj, p, blk_lo, phases;
    };
    auto item_at = [&](int i) {
        Item t;
        t.nb = i % nbt;
        t.pj = i / nbt;
        t.p = t.pj / splits;
        const int j = t.pj % splits;
        t.blk_lo = (int)(((int64_t)L.nbw * j) / splits);
        const int blk_hi = (int)(((int64_t)L.nbw * (j + 1)) / splits);
        t.phases = (blk_hi - t.blk_lo) * nh - (blk_hi == L.nbw ? nh - conv_halves(L.K - (L.nbw - 1) * L.bw) : 0);
        return t;
    };

    if (wave >= 4) {
        const int d = wave - 4;
        const int pq = cg.P * cg.Q, plane = cg.H * cg.W;
        const int n_img = (n_cols + pq - 1) / pq;
        const int64_t back = (int64_t)cg.pad * cg.W + cg.pad;
        __amdgpu_buffer_rsrc_t xb;
        uint32_t at[2], bad[2], bad_s[2];
        Item it;
        auto begin = [&](int i) {
            it = item_at(i);
            const int nb = it.nb, c0 = (it.p / panels_per_group) * cg.Cg;              // the filter group's input channels
            // The input is read through a buffer descriptor that starts at the tile's first
            // image, channel c0, moved back by the padding so that a receptive field's corner
            // has a non-negative offset (the launcher keeps 129 images under 2^29 elements, so
            // byte offsets stay below 2^31), and ends with the input: a load past its end returns
            // zero.  That is also how an element outside the image is read - its lane's offset is turned
            // into 0xffffffff - so a gathered element costs a bit test, an or and a load (the row's offset
            // is the load's scalar one), with no branch.  (Word 3 of the descriptor: 32-bit elements, plain addressing.)
            const int img0 = nb * kConvColumns / pq;
            const int64_t span = (((int64_t)(n_img - img0) * cg.C - c0) * plane + back) * (int64_t)sizeof(float);
            xb = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(X + ((int64_t)img0 * cg.C + c0) * plane - back), 0, (int)std::min<int64_t>(span, 0x7fffffff), 0x00020000);
            // The lane's two columns: byte offset of the corner of each pixel's receptive field,
            // and which (r, s) fall outside the image - one bit per (r, s) when the filter has
            // at most 32 taps, else one per r and one per s.  Columns past the last are all outside.
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
        };
        // Wavefront d gathers groups kGroups d .. kGroups (d + 1) - 1 of eight rows of a piece; what
        // a row is comes from the table (uniform loads), so a row costs no arithmetic of its own.
        constexpr int kGroups = kConvPhase / 8 / conv_gatherers(NP);
        float va[kGroups][2][8], vb[kGroups][2][8];
        auto fetch = [&](int ph, float (&v)[kGroups][2][8]) {
            const uint2 *rp = rows + ((it.blk_lo + ph / nh) * kTile + (ph % nh) * kConvPhase + 8 * kGroups * d);
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
                        __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xb, (int)(at[i] | out | no_row), (int)e.x, 0));
                }
            }
        };
        // Piece after piece, item after item: the next piece is requested, then the present one, requested
        // a barrier earlier, is split and stored.  Piece n is stored before barrier n - 1, into the
        // buffer that the multipliers have left before barrier n - 2.
        int i = (int)blockIdx.x, ph = 0, buffer = 0;
        bool first = true;
        auto turn = [&](const float (&now)[kGroups][2][8], float (&next)[kGroups][2][8]) {
            bool more = true;
            if (++ph == it.phases) {
                i += (int)gridDim.x;
                ph = 0;
                more = i < items;
                if (more) begin(i);
            }
            if (more) fetch(ph, next);
            uint4 *dst = act + buffer * (NP * kConvPlane) + kGroups * d * kConvColumns + lane;
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    uint4 terms[NP];
                    split8<NP>(now[g][i], terms);
#pragma unroll
                    for (int t = 0; t < NP; ++t) dst[t * kConvPlane + g * kConvColumns + 64 * i] = terms[t];
                }
            buffer = buffer + 1 == kConvBuffers ? 0 : buffer + 1;
            if (!first) __syncthreads();
            first = false;
            return more;
        };
        begin(i);
        fetch(0, va);
        while (turn(va, vb) && turn(vb, va)) {}
        __syncthreads();
        return;
    }

    // Q accumulators of 32 filter rows x 32 columns per multiplying wavefront w, by the
    // height of the layer's blocks:
    //   up to 128 rows (Q = 4): rows 32 w .. 32 w + 31, all 128 columns;
    //   up to  64 rows (Q = 2): rows 32 (w % 2) .., columns 64 (w / 2) .. + 63.
    // Accumulator q holds, for element e of lane (kl, m), filter row 32 strip + 8 (e / 4) + 4 kl + e % 4 and column
    // cbase + 32 q + m of the tile: 32 lanes have 32 consecutive columns of a row, as the output has them.
    // (Blocks of 96 rows leave the fourth wavefront without multiplies, but sharing the columns out, so
    // that each wavefront takes all three strips, splits every weight four times: the vector instructions
    // add to the multiplies' time here: AlexNet conv4, 64 images, 125 us so, 105 this way.)
    const int strip = Q == 4 ? wave : wave & 1;
    const int cbase = Q == 4 ? 0 : 64 * (wave >> 1);
    if (32 * strip >= L.bh) {                               // no rows: the barriers only
        for (int i = (int)blockIdx.x; i < items; i += (int)gridDim.x)
            for (int n = item_at(i).phases; n > 0; --n) __syncthreads();
        return;
    }
    const int kl = lane >> 5, m = lane & 31;
    constexpr int QB = 2;                                   // accumulators multiplied in turn: their chains hide each other's latency
    constexpr int kTurns = Q / QB;                          // of them per step
    constexpr int kRaw = Q == 4 ? 2 : 4;                    // steps of weights on their way
    static_assert(kConvSteps % kRaw == 0 && kConvSteps % 2 == 0, "a step's registers are the same in every phase");
    // the products formed, smallest first: term of the activation, term of the weight
    constexpr int kProducts = NP == 3 ? 8 : 3;
    constexpr int kTermX[8] = {NP == 3 ? 2 : 1, NP == 3 ? 1 : 0, NP == 3 ? 2 : 0, 0, 1, 1, 0, 0};
    constexpr int kTermW[8] = {NP == 3 ? 1 : 0, NP == 3 ? 2 : 1, 0, 2, 1, 0, 1, 0};

    uint4 x[2][QB][NP];
    auto load_x = [&](int buffer, int idx, uint4 (&dst)[QB][NP]) {      // idx = step * kTurns + turn
        const uint4 *src = act + buffer * (NP * kConvPlane) + kl * kConvColumns + cbase + m + (idx / kTurns) * (2 * kConvColumns) + (idx % kTurns) * (32 * QB);
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int i = 0; i < NP; ++i) dst[q][i] = src[i * kConvPlane + 32 * q];
    };
    auto split_pair = [&](const float (&v)[8], int j, uint32_t (&dst)[NP][4]) {
        uint32_t t[NP];
        split_weights<NP>(v[2 * j], v[2 * j + 1], t);
#pragma unroll
        for (int i = 0; i < NP; ++i) dst[i][j] = t[i];
    };
    // (the gatherers' instructions wait for the multipliers', not the other way round)
    __builtin_amdgcn_s_setprio(3);
    __syncthreads();                                        // two pieces gathered
    load_x(0, 0, x[0]);
    int buffer = 0;
    bool first = true;
    for (int i = (int)blockIdx.x; i < items; i += (int)gridDim.x) {
        const Item it = item_at(i);
        floatx16 acc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] = floatx16{0};
        // With three terms the products other than x1 w1 have sums of their own, added at the end: in one
        // sum with it each of six additions per step would round at its size (error against 64 bits,
        // 201 channels of 3 x 3: 3.2e-7, with two sums 1.0e-7, on the fp32 matrix cores 2.5e-7).
        floatx16 lo[NP == 3 ? Q : 1];
#pragma unroll
        for (auto &l : lo) l = floatx16{0};
        // A lane's eight weights of a step: two 16-byte pieces (four columns of a row; 128 rows, then
        // the next four columns).  Step t is multiplied while t + 1 is split and the kRaw after that
        // are on their way.
        const int last_step = it.phases * kConvSteps - 1;
        const float4 *wf = (const float4 *)wt + (((size_t)it.p * L.nbw + it.blk_lo) * (kTile / 4) + 2 * kl) * kTile + 32 * strip + m;
        auto load_step = [&](int t, float (&dst)[8]) {
            // (past the last step: the last one's again, never multiplied)
            t = min(t, last_step);
            const float4 *src = wf + (size_t)(nh == 2 ? t : t + (t & ~(kConvSteps - 1))) * (4 * kTile);
            load_floats<4>((const float *)src, dst);
            load_floats<4>((const float *)(src + kTile), dst + 4);
        };
        float raw[kRaw][8];
        uint32_t w[2][NP][4];
        {
            // (in the order in which the loop waits for them: any other, and its first wait in a phase
            // would be for the last of them)
            float step0[8];
            load_step(0, step0);
#pragma unroll
            for (int t = 1; t <= kRaw; ++t) {
                __builtin_amdgcn_sched_barrier(0);
                load_step(t, raw[t % kRaw]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) split_pair(step0, j, w[0]);
        }
        for (int ph = 0; ph < it.phases; ++ph) {
            if (!first) __syncthreads();                    // the piece after this one gathered
            first = false;
            const int next_buffer = buffer + 1 == kConvBuffers ? 0 : buffer + 1;
#pragma unroll
            for (int st = 0; st < kConvSteps; ++st) {
                constexpr int kPairs = (4 + kProducts * kTurns - 1) / (kProducts * kTurns);      // of weights split behind a product
                float (&next)[8] = raw[(st + 1) % kRaw];
#pragma unroll
                for (int turn = 0; turn < kTurns; ++turn) {
                    const int idx = st * kTurns + turn;
                    // program order is pinned (scheduling barriers): left alone, the compiler sinks the
                    // loads to just before their use and their latency lands in front of the multiplies
                    __builtin_amdgcn_sched_barrier(0);
                    // (after the last of a piece the first of the next, also the next item's)
                    if (idx + 1 < kConvSteps * kTurns) load_x(buffer, idx + 1, x[(idx + 1) & 1]);
                    else load_x(next_buffer, 0, x[0]);
#pragma unroll
                    for (int pr = 0; pr < kProducts; ++pr) {
                        __builtin_amdgcn_sched_barrier(0);
                        const uint32_t (&ww)[4] = w[st & 1][kTermW[pr]];
#pragma unroll
                        for (int q = 0; q < QB; ++q) {
                            floatx16 &sum = NP == 3 && pr + 1 < kProducts ? lo[turn * QB + q] : acc[turn * QB + q];
                            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, (uint4{ww[0], ww[1], ww[2], ww[3]})),
                                                                          __builtin_bit_cast(bf16x8, x[idx & 1][q][kTermX[pr]]), sum, 0, 0, 0);
                        }
#pragma unroll
                        for (int j = (turn * kProducts + pr) * kPairs; j < min((turn * kProducts + pr + 1) * kPairs, 4); ++j)
                            split_pair(next, j, w[(st + 1) & 1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                load_step(ph * kConvSteps + st + 1 + kRaw, next);
            }
            buffer = next_buffer;
        }
        if constexpr (NP == 3) {
#pragma unroll
            for (int q = 0; q < Q; ++q) acc[q] += lo[q];
        }

        // the finished output, or (block rows that are split) a partial tile for conv_reduce_kernel, laid
        // out [row][column]
        const int row_id = it.p * L.bh;
        const int block_rows = min(L.bh, L.M - row_id);
        const int step = out.Y ? out.pq : Np;               // floats from row to row
        // (the biases before the first store: waiting for one would wait for the stores before it too)
        __builtin_amdgcn_sched_barrier(0);
        float b[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) b[e] = 0.0f;
        if (out.bias) {
#pragma unroll
            for (int e = 0; e < 16; ++e) b[e] = out.bias[row_id + min(32 * strip + 8 * (e / 4) + 4 * kl + (e & 3), block_rows - 1)];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int c = it.nb * kConvColumns + cbase + 32 * q + m;
            if (out.Y && c >= out.ncols) continue;
            float *to = out.Y ? out.Y + ((size_t)(c / out.pq) * L.M + row_id) * out.pq + c % out.pq : part + (size_t)it.pj * L.bh * Np + c;
            to += (size_t)(uint32_t)((32 * strip + 4 * kl) * step);
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (32 * strip + 8 * e4 + 4 * kl + e < block_rows) {
                        const float y = acc[q][4 * e4 + e] + b[4 * e4 + e];
                        *to = out.relu ? fmaxf(y, 0.0f) : y;
                    }
                    to += step;
                }
                to += 4 * step;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// Adds the partial tiles of split block rows (part[block row][split][row][column], in that order), bias and
// activation, to Y[image][row][pixel].  A workgroup takes 1024 columns of one row, four to a
// thread; bound by the partial tiles, which are read once, in whole lines.  (The dense-tile
// path's finishing kernel, which turns tiles laid out [column][row] in LDS, took 8.5 us for VGG-16
// conv4_2 at one image; this one 5.0.)
constexpr int kConvRedThreads = 256, kConvRedColumns = 4 * kConvRedThreads;

__global__ __launch_bounds__(kConvRedThreads) void conv_reduce_kernel(const float *__restrict__ part, const float *__restrict__ bias, float *Y, int M, int OCg,
                                                                      int panels_per_group, int panel_rows, int ncols, int Np, int splits, int relu, int pq)
{
    const int chunks = (ncols + kConvRedColumns - 1) / kConvRedColumns;
    const int m = (int)blockIdx.x / chunks, c = ((int)blockIdx.x % chunks) * kConvRedColumns + 4 * (int)threadIdx.x;
    const int grp = m / OCg, in_grp = m - grp * OCg, panel = in_grp / panel_rows, r = in_grp - panel * panel_rows;
    if (c >= ncols) return;
    const size_t stride = (size_t)panel_rows * Np;
    const float *src = part + ((size_t)(grp * panels_per_group + panel) * splits * panel_rows + r) * Np + c;
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int j = 0; j < splits; j += 8) {                   // eight loads in flight, added in order
        float a[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u) load_floats<4>(src + (size_t)(j + u < splits ? j + u : j) * stride, a[u]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (j + u < splits) t[k] += a[u][k];
    }
    const float b = bias ? bias[m] : 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t[k] += b;
        if (relu) t[k] = fmaxf(t[k], 0.0f);
    }
    float *dst = Y + ((size_t)(c / pq) * M + m) * pq + c % pq;
    if ((pq & 3) == 0 && ((uintptr_t)Y & 15u) == 0) store_floats<4>(dst, t);     // (four pixels of one image)
    else {
        int o = c % pq;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (c + k < ncols) *dst = t[k];
            ++dst;
            if (++o == pq) {
                o = 0;
                dst += (size_t)(M - 1) * pq;
            }
        }
    }
}
