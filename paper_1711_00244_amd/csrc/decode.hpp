// Wavefront primitives, lane records, the decoding and placement passes (Algorithm 2 steps 5-9), block geometry and the LDS image of the decode tables.
// Part of the device translation unit: included by device.hip inside namespace cl,
// in the order given there.
#pragma once

// ------------------------------------------------------------------------- //
// wavefront primitives
// ------------------------------------------------------------------------- //
// Inclusive add-scan over the 64 lanes (all lanes must be active): four shifts
// inside each row of 16 lanes, then the row totals are carried across rows.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1,3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2,3
    return v;
}

// Largest value over the 64 lanes (all lanes must be active), the same in every lane
// and known to be uniform.
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// n / d for a divisor known on the host, in five scalar instructions (a division of uniform values the compiler
// works out in vector registers, and takes what follows from it for different in every lane).  Granlund and
// Montgomery's round-up method, exact for every 32-bit n.
struct Divisor {
    uint32_t mul, shift1, shift2, d;
    __device__ __forceinline__ uint32_t quotient(uint32_t n) const
    {
        const uint32_t t = __umulhi(n, mul);
        return (t + ((n - t) >> shift1)) >> shift2;
    }
};

static Divisor divisor(uint32_t d)
{
    uint32_t s = 0;
    while (s < 32 && (1ull << s) < d) ++s;
    return Divisor{(uint32_t)((((1ull << s) - d) << 32) / d + 1), s > 0 ? 1u : 0u, s > 0 ? s - 1 : 0u, d};
}

// W consecutive floats (W * 4-byte aligned) with one load.
template <int W> __device__ __forceinline__ void load_floats(const float *p, float *dst)
{
    typedef float vec_t __attribute__((ext_vector_type(W)));
    const vec_t v = *(const vec_t *)p;
#pragma unroll
    for (int i = 0; i < W; ++i) dst[i] = v[i];
}

template <> __device__ __forceinline__ void load_floats<1>(const float *p, float *dst) { dst[0] = *p; }

// and the store
template <int W> __device__ __forceinline__ void store_floats(float *p, const float *src)
{
    typedef float vec_t __attribute__((ext_vector_type(W)));
    vec_t v;
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = src[i];
    *(vec_t *)p = v;
}

template <> __device__ __forceinline__ void store_floats<1>(float *p, const float *src) { *p = src[0]; }

// Decode tables and codebook in LDS.  A table entry is two bytes and the streams are kept one
// bit up, so the masked stream bits are a byte offset; each table starts at a multiple of its
// size, so the offset or-ed to its place is the address.
typedef const __attribute__((address_space(3))) lut_t *lds_lut;
struct Tables {
    const float *cb;
    uint32_t vbase, ibase;     // LDS addresses
    uint32_t vmask, imask;     // of a byte offset
};

// A lane's record, split into its two spans.
struct LaneRecord {
    uint32_t vbuf[2];  // value-index codewords, low word first, next codeword at bit 1
    uint32_t ibuf[2];  // relative-index codewords, the same
    uint32_t n;        // entries in the record (0 for lanes beyond the chunk)
};

// n: entries of the record to decode (its own count, or 0)
__device__ __forceinline__ LaneRecord split_record(uint64_t w, uint32_t n)
{
    const uint64_t v = w >> (kCountBits - 1), i = __builtin_bitreverse64(w) << 1;
    return LaneRecord{{(uint32_t)v, (uint32_t)(v >> 32)}, {(uint32_t)i, (uint32_t)(i >> 32)}, n};
}

// A layer's description read from memory: the compiler takes its pointers for ones that could point anywhere (flat loads, which wait
// for LDS as well, and values that differ from lane to lane), unless it is told that they point to device memory.  (By way of a number: a cast there and back is taken for nothing.)
template <class T> __device__ __forceinline__ const T *in_global(const T *p) { return (const T *)(const __attribute__((address_space(1))) T *)(uintptr_t)p; }

__device__ __forceinline__ LayerDev in_global(LayerDev L)
{
    L.records = in_global(L.records);
    L.meta = in_global(L.meta);
    L.panel_chunk = in_global(L.panel_chunk);
    L.rec_pos = in_global((const uint16_t *)L.rec_pos);
    L.tables = in_global(L.tables);
    return L;
}

struct ChunkHead {
    cl_chunk_meta m;
    uint32_t nrec;
};

__device__ __forceinline__ ChunkHead load_head(const LayerDev &L, uint32_t c)
{
    // (as constant memory, which a launch never writes: one scalar load where c is the same in all lanes, whatever the kernel stores before)
    typedef const __attribute__((address_space(4))) cl_chunk_meta *const_meta;
    const const_meta m = (const_meta)(uintptr_t)L.meta + c;
    ChunkHead h;
    h.m.sym_off = m->sym_off;
    h.m.rec_off = m->rec_off;
    h.m.blk = m->blk;
    h.m.pos0 = m->pos0;
    h.nrec = m[1].rec_off - h.m.rec_off;
    return h;
}

__device__ __forceinline__ LaneRecord load_record(const LayerDev &L, const ChunkHead &h, int lane)
{
    const uint64_t w = (uint32_t)lane < h.nrec ? L.records[(size_t)h.m.rec_off + lane] : 0ull;
    return split_record(w, (uint32_t)w & 15u);
}

// One table lookup: the entry for the codeword at the head of the stream (symbol in its second
// byte); the stream moves on to the next codeword.  The entry itself is the shift amount
// (length in its low bits, the shifters look at the low five), which keeps the loop-carried
// chain at and-or, read, shift.
// (Two 32-bit shifts, which take as long as a 64-bit one: a layer at one image took the same time, to
// three digits, with either.  A 64-bit shift by an amount in the last vector register of a wavefront's
// allocation is a known fault of gfx90a, which the compiler works around there and not here; whether this
// chip has it was not established.)
__device__ __forceinline__ uint32_t next_entry(uint32_t (&buf)[2], uint32_t base, uint32_t mask)
{
    const uint32_t e = *(lds_lut)(uintptr_t)((buf[0] & mask) | base);
    buf[0] = __builtin_amdgcn_alignbit(buf[1], buf[0], e);
    buf[1] >>= (e & 31u);
    return e;
}

constexpr int kMaxEntries = 15;        // a record's count field is four bits

// A lane's record with both codeword streams decoded: eight bits per entry, entry j in
// byte j % 4 of word j / 4; the bytes of entries the record does not have are zero.
struct Symbols {
    uint32_t z[4];     // relative indices
    uint32_t v[4];     // value indices
    uint32_t n;        // entries
    uint32_t nmax;     // largest n of the wavefront (uniform)
    uint32_t adv;      // sum of (z + 1): how far the record moves the position
};

// One step of the decoding pass: entry J of both streams.  Every lane looks up (the
// masked table index is always inside the table) and stores the symbol, also a lane
// that has no entry J: what it stored is cleared after the pass, so the pass has no
// divergent branch and no per-lane test.
template <int J>
__device__ __forceinline__ void decode_from(LaneRecord &rec, const Tables &T, Symbols &y)
{
    if constexpr (J < kMaxEntries) {
        if ((uint32_t)J >= y.nmax) return;                                  // uniform
        constexpr int at = J % 4;
        // identity selector with 5 at byte `at`: the symbol byte of the table entry goes there
        constexpr uint32_t put = (0x03020100u & ~(0xffu << (8 * at))) | (5u << (8 * at));
        const uint32_t ez = next_entry(rec.ibuf, T.ibase, T.imask);
        const uint32_t ev = next_entry(rec.vbuf, T.vbase, T.vmask);
        y.z[J / 4] = __builtin_amdgcn_perm(ez, y.z[J / 4], put);
        y.v[J / 4] = __builtin_amdgcn_perm(ev, y.v[J / 4], put);
        decode_from<J + 1>(rec, T, y);
    }
}

// Algorithm 2 step 6 for one record: both streams are decoded in one pass - two
// independent table chains per lane, so one lookup's latency hides behind the
// other's - and kept in registers; positions and weights follow from them without
// touching the tables again.  The pass is written out for the fifteen possible entries
// (it ends after the wavefront's longest record), so every byte position is a constant.
// All lanes of the wavefront must be active.
// (decode_symbols leaves what lies past a lane's own entries, and their sum, open: for a caller that
// heeds only its own and knows where the record starts.)
__device__ __forceinline__ Symbols decode_symbols(LaneRecord rec, const Tables &T)
{
    Symbols y{{0, 0, 0, 0}, {0, 0, 0, 0}, rec.n, wave_max(rec.n), 0};
    // (the masks in vector registers: an and-or takes one scalar operand)
    Tables V = T;
    asm("" : "+v"(V.vmask), "+v"(V.imask));
    decode_from<0>(rec, V, y);
    return y;
}

__device__ __forceinline__ Symbols decode_record(LaneRecord rec, const Tables &T)
{
    Symbols y = decode_symbols(rec, T);
    // clear the bytes of entries a lane does not have: word w keeps its first
    // clamp(n - 4 w, 0, 4) bytes (the shift by 8 bits per byte is done in two halves,
    // so that four bytes shift everything out)
    const uint32_t n4 = 4u * y.n;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if ((uint32_t)(4 * w) >= y.nmax) break;                             // uniform
        const uint32_t half = (uint32_t)min(max((int)n4 - 16 * w, 0), 16);
        const uint32_t drop = (0xffffffffu << half) << half;
        y.z[w] &= ~drop;
        y.v[w] &= ~drop;
    }
    // absent entries are zero bytes: the byte sums of the four words are the sum of z
    uint32_t adv = y.n;
#pragma unroll
    for (int w = 0; w < 4; ++w) adv = __builtin_amdgcn_sad_u8(y.z[w], 0u, adv);
    y.adv = adv;
    return y;
}

struct LaneStart {
    uint32_t entry;    // index, inside the chunk, of the lane's first entry
    uint32_t sum;      // sum of (z + 1) over the block's entries before the lane's first entry
};

// Algorithm 2 step 7: the prefix sum across the wavefront.  Lane counts (<= 15, 960
// per chunk: 10 bits) and lane advances (<= 15 * 256) travel in one scan.
__device__ __forceinline__ LaneStart lane_starts(const Symbols &y, uint32_t pos0)
{
    const uint32_t mine = y.n | (y.adv << 10);
    const uint32_t excl = wave_incl_scan(mine) - mine;
    LaneStart s;
    s.entry = excl & 1023u;
    s.sum = pos0 + (excl >> 10);
    return s;
}

// Calls f(j, v, z, position) for the record's entries in order; sum starts as the
// lane's LaneStart::sum.  Written out like the decoding pass.  With ALL the call is
// made in every lane up to the wavefront's longest record: a lane past its own last
// entry sees v = 0, z = 0 and a position that moves on by one per call (for callers
// to whom a zero weight at such a position does no harm); without, only for the
// lane's own entries.
template <bool ALL, int J, class F>
__device__ __forceinline__ void entries_from(const Symbols &y, uint32_t pos, F &f)
{
    if constexpr (J < kMaxEntries) {
        if ((uint32_t)J >= y.nmax) return;                                  // uniform
        const uint32_t z = (y.z[J / 4] >> (8 * (J % 4))) & 0xffu, v = (y.v[J / 4] >> (8 * (J % 4))) & 0xffu;
        pos += z + 1u;
        if (ALL || (uint32_t)J < y.n) f((uint32_t)J, v, z, pos);
        entries_from<ALL, J + 1>(y, pos, f);
    }
}

template <bool ALL = false, class F>
__device__ __forceinline__ void for_each_entry(const Symbols &y, uint32_t sum, F f)
{
    entries_from<ALL, 0>(y, sum - 1u, f);
}

// The same walk over a record's entries for callers that look a value up per entry and
// then store it: the entries are taken four at a time, the four look-ups (made in every
// lane, value index 0 for entries a lane does not have) go out together and are waited
// for once, then put(position, looked-up value) is called for the lane's own entries.
template <int J, class Look, class Put>
__device__ __forceinline__ void place_from(const Symbols &y, uint32_t pos, Look &look, Put &put)
{
    if constexpr (J < kMaxEntries) {
        if ((uint32_t)J >= y.nmax) return;                                  // uniform, once per four entries
        constexpr int G = kMaxEntries - J < 4 ? kMaxEntries - J : 4;
        uint32_t at[G];
        decltype(look(0u)) w[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const uint32_t z = (y.z[J / 4] >> (8 * u)) & 0xffu, v = (y.v[J / 4] >> (8 * u)) & 0xffu;
            pos += z + 1u;
            at[u] = pos;
            w[u] = look(v);
        }
#pragma unroll
        for (int u = 0; u < G; ++u)
            if ((uint32_t)(J + u) < y.n) put(at[u], w[u]);
        place_from<J + G>(y, pos, look, put);
    }
}

template <class Look, class Put>
__device__ __forceinline__ void place_entries(const Symbols &y, uint32_t sum, Look look, Put put)
{
    place_from<0>(y, sum - 1u, look, put);
}

// The walk for callers that fetch something per entry and then work on it in order: the
// entries are taken G at a time, fetch(u, v, position) is called for the G of them first (in
// every lane, value index 0 and a position one further for entries a lane does not have),
// so that what it loads is in flight together and waited for once; then use(u) for the
// lane's own entries, in order.  fetch and use share their storage through the slot number
// u < G.  Entries past the wavefront's longest record are skipped.
template <int G, int J, class Fetch, class Use>
__device__ __forceinline__ void groups_from(const Symbols &y, uint32_t pos, Fetch &fetch, Use &use)
{
    if constexpr (J < kMaxEntries) {
        if ((uint32_t)J >= y.nmax) return;                                  // uniform, once per group
        constexpr int N = kMaxEntries - J < G ? kMaxEntries - J : G;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if ((uint32_t)(J + u) < y.nmax) {                               // uniform
                const uint32_t z = (y.z[(J + u) / 4] >> (8 * ((J + u) % 4))) & 0xffu, v = (y.v[(J + u) / 4] >> (8 * ((J + u) % 4))) & 0xffu;
                pos += z + 1u;
                fetch(u, v, pos);
            }
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
            if ((uint32_t)(J + u) < y.n) use(u);
        groups_from<G, J + N>(y, pos, fetch, use);
    }
}

template <int G, class Fetch, class Use>
__device__ __forceinline__ void for_each_entry_grouped(const Symbols &y, uint32_t sum, Fetch fetch, Use use)
{
    groups_from<G, 0>(y, sum - 1u, fetch, use);
}

struct BlockGeom {
    int row_id, col_id, bhp, bwp;
    int shift;        // log2(bwp) when bwp is a power of two, else -1
};

// block `bcol` of block row `brow`
__device__ __forceinline__ BlockGeom block_geom(const LayerDev &L, int brow, int bcol)
{
    BlockGeom g;
    g.row_id = brow * L.bh;
    g.col_id = bcol * L.bw;
    g.bhp = min(L.bh, L.M - g.row_id);
    g.bwp = min(L.bw, L.K - g.col_id);
    g.shift = (g.bwp & (g.bwp - 1)) == 0 ? (31 - __builtin_clz((uint32_t)g.bwp)) : -1;
    return g;
}

// (b the same in all lanes.  A division is vector arithmetic, and what follows from its result would be one value per
// lane to the compiler: the shape of the block, and every branch on it)
__device__ __forceinline__ BlockGeom block_geom(const LayerDev &L, uint32_t b)
{
    const int brow = __builtin_amdgcn_readfirstlane((int)(b / (uint32_t)L.nbw));
    return block_geom(L, brow, (int)(b - (uint32_t)brow * (uint32_t)L.nbw));
}

// Position inside a block -> (row, column) offsets; a block is flattened row by
// row (Algorithm 2 step 9, "arrange as bh x bw block").  The row is clamped so that
// a position beyond the block cannot index outside it.
__device__ __forceinline__ void split_pos(uint32_t pos, const BlockGeom &g, uint32_t &r, uint32_t &c)
{
    if (g.shift >= 0) { r = pos >> g.shift; c = pos & ((uint32_t)g.bwp - 1u); }
    else { r = pos / (uint32_t)g.bwp; c = pos - r * (uint32_t)g.bwp; }
    r = min(r, (uint32_t)g.bhp - 1u);
}

// LDS carve-up shared by the chunk kernels: value table, index table, codebook,
// then kernel-specific space.
struct Smem {
    Tables T;
    uint4 *tables;     // where the table image goes
    float *extra;
};

static size_t smem_fixed_bytes(int vbits, int ibits, int ncode) { return table_image_bytes(vbits, ibits, ncode); }

__device__ __forceinline__ Smem carve(uint8_t *base, const LayerDev &L)
{
    Smem s;
    // the larger table first: each starts at a multiple of its size
    const bool values_first = L.val_bits >= L.idx_bits;
    lut_t *v = (lut_t *)base + (values_first ? 0 : 1 << L.idx_bits);
    lut_t *i = (lut_t *)base + (values_first ? 1 << L.val_bits : 0);
    // both tables have at least two entries, so they end 4-byte aligned; round up to 16
    // (base is where the dynamic LDS starts: at 0, in kernels that have no other - as all that call this
    // must be, which tests/test_kernel_lds.py checks in the built library)
    const size_t tb = (((size_t)1 << L.val_bits) + ((size_t)1 << L.idx_bits)) * sizeof(lut_t);
    float *cb = (float *)(base + ((tb + 15) & ~(size_t)15));
    s.T.vbase = (uint32_t)(uintptr_t)(lds_lut)v;
    s.T.ibase = (uint32_t)(uintptr_t)(lds_lut)i;
    s.T.cb = cb;
    s.tables = (uint4 *)base;
    s.T.vmask = (2u << L.val_bits) - 2u;
    s.T.imask = (2u << L.idx_bits) - 2u;
    s.extra = cb + ((L.ncode + 3) & ~3);
    return s;
}

// The decode tables and the codebook sit in device memory exactly as they sit in
// LDS (value table, index table, padding to 16 bytes, codebook, padding to 16
// bytes), so a workgroup copies them as 16-byte rows: all loads are issued first,
// the LDS stores follow once the rest of the prologue is under way.
constexpr int kTableRows = 3;            // 16-byte rows per thread: 3 * 512 * 16 B covers two 12-bit tables + codebook

struct TableRegs {
    uint4 row[kTableRows];
};

__device__ __forceinline__ TableRegs fetch_tables(const LayerDev &L)
{
    TableRegs t;
    const uint4 *g = L.tables;
#pragma unroll
    // (past the last row: that one again, not stored)
    for (int k = 0; k < kTableRows; ++k) t.row[k] = g[min((int)threadIdx.x + k * kThreads, L.table_rows - 1)];
    return t;
}

__device__ __forceinline__ void store_tables(const Smem &s, const LayerDev &L, const TableRegs &t)
{
    uint4 *d = s.tables;
#pragma unroll
    for (int k = 0; k < kTableRows; ++k) {
        const int i = (int)threadIdx.x + k * kThreads;
        if (i < L.table_rows) d[i] = t.row[k];
    }
}
