// Host side of the library: builds the compressed form of a pruned weight matrix
// (Sec. III-B pipeline, block-contiguous as in Sec. IV-A), validates it, and
// converts it to and from a relocatable byte image.  No HIP calls here.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <memory>
#include <new>

#include <emmintrin.h>

#include "layer.hpp"
#include "team.hpp"

namespace cl {

// (of fixed size: reporting that there is no memory takes none)
static thread_local char g_error[512];

int32_t fail(int32_t code, const char *fmt, ...) noexcept
{
    char buf[sizeof g_error];                   // (an argument may be the message before)
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    std::memcpy(g_error, buf, sizeof buf);
    return code;
}

void clear_error() noexcept { g_error[0] = 0; }

int32_t fail_with_exception() noexcept
{
    try {
        throw;
    } catch (const std::bad_alloc &) {
        return fail(CL_ENOMEM, "out of memory");
    } catch (const std::exception &e) {
        return fail(CL_ENOMEM, "out of a host resource: %s", e.what());
    } catch (...) {
        return fail(CL_ENOMEM, "out of a host resource");
    }
}

namespace {

struct Geometry {
    int M, K, bh, bw;
    int nbh, nbw;
    int64_t n_blocks;
    explicit Geometry(const cl_layer_desc &d)
        : M(d.M), K(d.K), bh(d.block_h), bw(d.block_w), nbh((d.M + d.block_h - 1) / d.block_h),
          nbw((d.K + d.block_w - 1) / d.block_w), n_blocks((int64_t)nbh * nbw) {}
    // Algorithm 2: block i starts at row (i / nbw) * bh and column (i % nbw) * bw.
    void block(int64_t i, int &row_id, int &col_id, int &bhp, int &bwp) const
    {
        row_id = (int)(i / nbw) * bh;
        col_id = (int)(i % nbw) * bw;
        bhp = std::min(bh, M - row_id);
        bwp = std::min(bw, K - col_id);
    }
};

int32_t check_desc(cl_layer_desc &d)
{
    if (d.M < 1 || d.K < 1) return fail(CL_EINVAL, "M and K must be positive (got %d x %d)", d.M, d.K);
    if ((int64_t)d.M * d.K > std::numeric_limits<int32_t>::max()) return fail(CL_EINVAL, "M*K exceeds 2^31-1");
    if (d.weight_bits < 1 || d.weight_bits > 8) return fail(CL_EINVAL, "weight_bits must be in 1..8 (got %d)", d.weight_bits);
    if (d.index_bits < 1 || d.index_bits > 8) return fail(CL_EINVAL, "index_bits must be in 1..8 (got %d)", d.index_bits);
    if (d.block_h < 1 || d.block_w < 1) return fail(CL_EINVAL, "block_h and block_w must be positive");
    if (d.block_h > d.M) d.block_h = d.M;
    if (d.block_w > d.K) d.block_w = d.K;
    if (d.chunk_bits == 0) d.chunk_bits = CL_CHUNK_BITS;
    if (d.chunk_bits != CL_CHUNK_BITS) return fail(CL_EINVAL, "chunk_bits must be %d", CL_CHUNK_BITS);
    if (d.max_code_len == 0) d.max_code_len = CL_MAX_CODE_LEN;
    if (d.max_code_len > CL_MAX_CODE_LEN || d.max_code_len < std::max(d.weight_bits, d.index_bits))
        return fail(CL_EINVAL, "max_code_len must be in max(weight_bits,index_bits)..%d", CL_MAX_CODE_LEN);
    return CL_OK;
}

inline uint64_t bit_reverse64(uint64_t x)
{
    x = ((x >> 1) & 0x5555555555555555ull) | ((x & 0x5555555555555555ull) << 1);
    x = ((x >> 2) & 0x3333333333333333ull) | ((x & 0x3333333333333333ull) << 2);
    x = ((x >> 4) & 0x0f0f0f0f0f0f0f0full) | ((x & 0x0f0f0f0f0f0f0f0full) << 4);
    return __builtin_bswap64(x);
}

// Units of work a thread is started for: about a tenth of a millisecond each, several times
// what starting it costs.
constexpr int64_t kWeightsPerThread = 1 << 18, kRecordsPerThread = 1 << 13, kBytesPerThread = 1 << 17;

// The decode tables with what a check of an entry asks for worked out per slot, so that
// the walk over the records only gathers flags: bits 0-5 codeword length, bits 8-15 symbol,
// bit 16 a surviving weight (value table), bit 30 a value symbol 0 / a relative index that
// padding may not have (the two meet in one entry: malformed padding), bit 31 a slot
// no codeword leads to.
constexpr uint32_t kSlotWeight = 1u << 16, kSlotPad = 1u << 30, kSlotBad = 1u << 31;

std::vector<uint32_t> check_table(const std::vector<lut_t> &lut, const std::vector<uint8_t> &len, bool values, int filler)
{
    std::vector<uint32_t> t(lut.size());
    for (size_t i = 0; i < lut.size(); ++i) {
        const int sym = lut_sym(lut[i]), l = lut_len(lut[i]);
        uint32_t e = (uint32_t)l | ((uint32_t)sym << 8);
        if (len[sym] != l) e |= kSlotBad;
        if (values && sym) e |= kSlotWeight;
        if (values ? sym == 0 : sym != filler) e |= kSlotPad;
        t[i] = e;
    }
    return t;
}

// What one chunk holds, and where in its block.
struct ChunkScan {
    uint64_t advance = 0;              // sum of (z + 1)
    uint32_t entries = 0, weights = 0; // weights: entries that are not padding
    uint32_t right = 0;                // of them, in the block's columns 64 and up
    uint32_t vbits = 0, ibits = 0;
    int64_t bad_record = -1;           // first record that fails a check
};

struct Scanner {
    const cl_layer *L;
    std::vector<uint32_t> vt, it;
    uint32_t vmask, imask;
    uint16_t *pos16;                   // where the records' first positions go (one of the two, or neither)
    uint32_t *pos32;

    // Decodes chunk c (records r0 .. r1 - 1, first position pos0 of a block of bwp columns and np
    // cells).  With cnt, surviving weights are counted per half and row (128 rows a half).
    template <bool COUNT>
    ChunkScan chunk(uint64_t r0, uint64_t r1, uint64_t pos0, uint32_t bwp, uint64_t np, uint16_t *cnt) const
    {
        ChunkScan s;
        const int shift = (bwp & (bwp - 1)) == 0 ? __builtin_ctz(bwp) : -1;
        uint64_t pos = pos0;
        for (uint64_t r = r0; r < r1; ++r) {
            const uint64_t w = L->records[r];
            const int n = (int)(w & 15u);
            if (pos16) pos16[r] = (uint16_t)pos;
            else if (pos32) pos32[r] = (uint32_t)pos;
            uint64_t vbuf = w >> kCountBits, ibuf = bit_reverse64(w);
            uint32_t vused = 0, iused = 0, flags = n < 1 ? kSlotBad : 0;
            for (int j = 0; j < n; ++j) {
                const uint32_t ev = vt[(uint32_t)vbuf & vmask], ei = it[(uint32_t)ibuf & imask];
                vbuf >>= ev & 63u;
                ibuf >>= ei & 63u;
                vused += ev & 63u;
                iused += ei & 63u;
                flags |= ((ev | ei) & kSlotBad) | (ev & ei & kSlotPad);
                pos += ((ei >> 8) & 255u) + 1u;
                if (pos > np) { flags |= kSlotBad; break; }
                if (!(ev & kSlotWeight)) continue;
                ++s.weights;
                if (COUNT) {
                    const uint32_t at = (uint32_t)(pos - 1);
                    const uint32_t row = shift >= 0 ? at >> shift : at / bwp, col = at - row * bwp;
                    const uint32_t h = col >= 64u;
                    s.right += h;
                    ++cnt[h * 128u + row];
                }
            }
            // the bits between the two spans must be zero
            const int gap = CL_RECORD_BITS - kCountBits - (int)(vused + iused);
            if (gap < 0) flags |= kSlotBad;
            else if (gap > 0 && ((w >> (kCountBits + vused)) & ((1ull << gap) - 1ull))) flags |= kSlotBad;
            if (flags) {
                s.bad_record = (int64_t)r;
                return s;
            }
            s.vbits += vused;
            s.ibits += iused;
            s.entries += (uint32_t)n;
        }
        s.advance = pos - pos0;
        return s;
    }
};

// The same checks on one record that failed them, one by one, for the message.
int32_t describe_bad_record(const cl_layer *L, int64_t r)
{
    const uint32_t vmask = (1u << L->val_lut_bits) - 1u, imask = (1u << L->idx_lut_bits) - 1u;
    const uint32_t filler_z = (1u << L->desc.index_bits) - 1u;
    const uint64_t w = L->records[(size_t)r];
    const int n = (int)(w & 15u);
    if (n < 1) return fail(CL_ECORRUPT, "record %lld is empty", (long long)r);
    uint64_t vbuf = w >> kCountBits, ibuf = bit_reverse64(w);
    int used = 0;
    for (int j = 0; j < n; ++j) {
        const lut_t ev = L->val_lut[(uint32_t)vbuf & vmask], ei = L->idx_lut[(uint32_t)ibuf & imask];
        const int v = lut_sym(ev), lv = lut_len(ev), z = lut_sym(ei), li = lut_len(ei);
        if (L->val_len[v] != lv || L->idx_len[z] != li) return fail(CL_ECORRUPT, "record %lld: bit pattern is not a codeword", (long long)r);
        vbuf >>= lv;
        ibuf >>= li;
        used += lv + li;
        if (kCountBits + used > CL_RECORD_BITS) return fail(CL_ECORRUPT, "record %lld overflows", (long long)r);
        if (!v && (uint32_t)z != filler_z) return fail(CL_ECORRUPT, "padding entry with a short gap");
    }
    return fail(CL_ECORRUPT, "record %lld: a position leaves its block, or stray bits between its spans", (long long)r);
}

}  // namespace

// --------------------------------------------------------------------------- //
// Everything that can be derived from the stored sections is derived here, and
// every record is decoded and every table entry compared with what the decode
// finds.  Used after compression (self-check) and after deserialisation.
//
// The tables are checked against each other first, one after the other; then the blocks,
// which do not depend on each other, are decoded by the team's threads, each record
// once: the same walk checks it and counts what the derived tables need.  (One thread
// and two walks: 56 ms for AlexNet's fc6, 4.4 M entries; now 2.)
// --------------------------------------------------------------------------- //
int32_t finalize_and_validate(cl_layer *L, Team &team)
{
    cl_layer_desc d = L->desc;
    if (int32_t rc = check_desc(d)) return rc;
    if (d.block_h != L->desc.block_h || d.block_w != L->desc.block_w || d.chunk_bits != L->desc.chunk_bits ||
        d.max_code_len != L->desc.max_code_len)
        return fail(CL_ECORRUPT, "descriptor is not in normal form");
    const Geometry g(d);
    const int nval = 1 << d.weight_bits, nidx = 1 << d.index_bits;
    L->n_blocks = g.n_blocks;
    L->n_panels = g.nbh;
    L->nbw = g.nbw;
    if ((int)L->codebook.size() != nval || (int)L->val_len.size() != nval || (int)L->idx_len.size() != nidx)
        return fail(CL_ECORRUPT, "codebook / code length tables have the wrong size");
    if (L->codebook[0] != 0.0f) return fail(CL_ECORRUPT, "codebook[0] must be 0");
    for (float c : L->codebook)
        if (!std::isfinite(c)) return fail(CL_ECORRUPT, "non-finite codebook entry");
    if (!canonical_codes(L->val_len, L->val_code, &L->val_lut_bits) ||
        !canonical_codes(L->idx_len, L->idx_code, &L->idx_lut_bits))
        return fail(CL_ECORRUPT, "code lengths are not a prefix code within the length limit");
    if (L->val_lut_bits > d.max_code_len || L->idx_lut_bits > d.max_code_len)
        return fail(CL_ECORRUPT, "code lengths exceed max_code_len");
    L->val_lut_bits = std::max(1, L->val_lut_bits);
    L->idx_lut_bits = std::max(1, L->idx_lut_bits);
    build_lut(L->val_len, L->val_code, L->val_lut_bits, L->val_lut);
    build_lut(L->idx_len, L->idx_code, L->idx_lut_bits, L->idx_lut);

    if ((int64_t)L->block_ptr.size() != g.n_blocks + 1) return fail(CL_ECORRUPT, "block_ptr has the wrong size");
    if ((int64_t)L->panel_chunk.size() != (int64_t)g.nbh + 1) return fail(CL_ECORRUPT, "panel table has the wrong size");
    if (L->meta.empty()) return fail(CL_ECORRUPT, "chunk table is empty");
    L->n_chunks = (int64_t)L->meta.size() - 1;
    L->n_records = (int64_t)L->records.size();
    L->entries = L->meta[L->n_chunks].sym_off;
    if (L->meta[L->n_chunks].rec_off != L->n_records) return fail(CL_ECORRUPT, "chunk table does not span the records");
    if (L->block_ptr[0] != 0 || L->block_ptr[g.n_blocks] != L->entries) return fail(CL_ECORRUPT, "block_ptr does not span the entries");
    for (int64_t b = 0; b < g.n_blocks; ++b)
        if (L->block_ptr[b] > L->block_ptr[b + 1]) return fail(CL_ECORRUPT, "block_ptr is not monotone");
    if (L->panel_chunk[0] != 0 || L->panel_chunk[g.nbh] != L->n_chunks) return fail(CL_ECORRUPT, "panel table does not span the chunks");
    L->max_panel_chunks = 0;
    for (int p = 0; p < g.nbh; ++p) {
        if (L->panel_chunk[p] > L->panel_chunk[p + 1]) return fail(CL_ECORRUPT, "panel table is not monotone");
        L->max_panel_chunks = std::max<int64_t>(L->max_panel_chunks, (int64_t)L->panel_chunk[p + 1] - L->panel_chunk[p]);
    }

    // ---- the chunk table against itself, block_ptr and the panel table ----
    if (L->n_chunks == 0 && L->entries != 0) return fail(CL_ECORRUPT, "records do not add up to the entry count");
    uint64_t next_rec = 0;
    int64_t cur_blk = -1;
    int panel = 0;
    for (int64_t c = 0; c < L->n_chunks; ++c) {
        const cl_chunk_meta &m = L->meta[c], &m1 = L->meta[c + 1];
        const uint64_t r0 = m.rec_off, r1 = m1.rec_off;
        if (r0 != next_rec || r1 <= r0 || r1 - r0 > (uint64_t)kLanes || r1 > (uint64_t)L->n_records)
            return fail(CL_ECORRUPT, "chunk %lld: bad record range", (long long)c);
        // every record holds an entry: with this a block without entries has no chunk, and every
        // chunk lies in its block's range of block_chunk, where the walk below finds it
        if (m.sym_off >= m1.sym_off) return fail(CL_ECORRUPT, "chunk %lld has no entries", (long long)c);
        if (m.blk >= (uint64_t)g.n_blocks || (int64_t)m.blk < cur_blk) return fail(CL_ECORRUPT, "chunk %lld: bad block", (long long)c);
        if ((int64_t)m.blk != cur_blk) {
            if (m.sym_off != L->block_ptr[m.blk] || (c == 0 && m.sym_off != 0)) return fail(CL_ECORRUPT, "chunk %lld does not start its block", (long long)c);
            if (m.pos0 != 0) return fail(CL_ECORRUPT, "chunk %lld: position carry is wrong", (long long)c);
            cur_blk = m.blk;
        }
        // every non-empty block must be covered in full
        if ((c + 1 == L->n_chunks || m1.blk != m.blk) && m1.sym_off != L->block_ptr[m.blk + 1])
            return fail(CL_ECORRUPT, "block %u is not covered by its chunks", m.blk);
        while (panel < g.nbh && (int64_t)L->panel_chunk[panel + 1] <= c) ++panel;
        if ((int64_t)m.blk / g.nbw != panel) return fail(CL_ECORRUPT, "chunk %lld is not inside its block row", (long long)c);
        next_rec = r1;
    }
    // first chunk of every block (blocks without entries get an empty range)
    L->block_chunk.assign((size_t)g.n_blocks + 1, (uint32_t)L->n_chunks);
    for (int64_t c = L->n_chunks - 1; c >= 0; --c) L->block_chunk[L->meta[c].blk] = (uint32_t)c;
    for (int64_t b = g.n_blocks - 1; b >= 0; --b)
        if (L->block_ptr[b] == L->block_ptr[b + 1]) L->block_chunk[b] = L->block_chunk[b + 1];

    // ---- the records, block by block ----
    L->rec_pos16.clear();
    L->rec_pos32.clear();
    if (d.block_h <= kPrivateTileRows) {
        if ((int64_t)d.block_h * d.block_w <= 1 << 16) L->rec_pos16.resize((size_t)L->n_records);
        else L->rec_pos32.resize((size_t)L->n_records);
    }
    const Scanner scan{L, check_table(L->val_lut, L->val_len, true, 0), check_table(L->idx_lut, L->idx_len, false, nidx - 1),
                       (1u << L->val_lut_bits) - 1u, (1u << L->idx_lut_bits) - 1u,
                       L->rec_pos16.empty() ? nullptr : L->rec_pos16.data(), L->rec_pos32.empty() ? nullptr : L->rec_pos32.data()};
    // the half-by-half order of the wide path (blocks of at most 128 x 128 only): per block, counts
    // first, list positions once the weights of all blocks before it are known
    constexpr int kGroups = 16, kPer = 2 * (kGroups + 1), kRows = 128;
    const bool halves = d.block_h <= 128 && d.block_w <= 128;
    L->chunk_nz.assign((size_t)L->n_chunks + 1, 0u);
    L->slot.clear();
    L->chunk_half.clear();
    L->group_ptr.clear();
    L->row_ptr.clear();
    if (halves) {
        L->chunk_half.assign((size_t)L->n_chunks * 2, 0u);
        L->group_ptr.assign((size_t)g.n_blocks * kPer, 0u);
        L->block_slots = 1;
        L->max_block_entries = 0;
        for (int64_t b = 0; b < g.n_blocks; ++b) {
            L->block_slots = std::max<int32_t>(L->block_slots, (int32_t)(L->block_chunk[b + 1] - L->block_chunk[b]));
            L->max_block_entries = std::max<int64_t>(L->max_block_entries, L->block_ptr[b + 1] - L->block_ptr[b]);
        }
        // Small blocks, and blocks of very different content, would make the lookup tables of some kernels
        // heavier than the layer itself, and gain little by those kernels: a table of more than half
        // the records' size and a mebibyte is left out, and the launches do without the kernels that read it.
        auto in_proportion = [&](size_t bytes) { return bytes <= std::max<size_t>((size_t)L->n_records * 8 / 2, 1 << 20); };
        const size_t slots = (size_t)g.n_blocks * L->block_slots;
        if (in_proportion(slots * sizeof(ChunkSlot))) L->slot.assign(slots, ChunkSlot{});
        L->row_ptrs = (d.block_h + 3) & ~1;
        const size_t starts = (size_t)g.n_blocks * L->row_ptrs;
        if (!L->slot.empty() && in_proportion(starts * 2)) L->row_ptr.assign(starts, 0u);
    }
    std::atomic<int64_t> vbits{0}, ibits{0}, bad_chunk{L->n_chunks};
    auto report = [&](int64_t c) {
        int64_t seen = bad_chunk.load();
        while (c < seen && !bad_chunk.compare_exchange_weak(seen, c)) {}
    };
    const int64_t units = std::min<int64_t>(g.n_blocks, (int64_t)team.size() * 8);
    team.each(units, [&](int64_t u) {
        int64_t my_v = 0, my_i = 0;
        for (int64_t b = g.n_blocks * u / units; b < g.n_blocks * (u + 1) / units; ++b) {
            int row_id, col_id, bhp, bwp;
            g.block(b, row_id, col_id, bhp, bwp);
            uint16_t cnt[2 * kRows] = {0};
            uint32_t left = 0, right = 0;
            for (uint32_t c = L->block_chunk[b]; c < L->block_chunk[b + 1]; ++c) {
                const cl_chunk_meta &m = L->meta[c], &m1 = L->meta[(size_t)c + 1];
                const ChunkScan s = halves ? scan.chunk<true>(m.rec_off, m1.rec_off, m.pos0, (uint32_t)bwp, (uint64_t)bhp * bwp, cnt)
                                           : scan.chunk<false>(m.rec_off, m1.rec_off, m.pos0, (uint32_t)bwp, (uint64_t)bhp * bwp, nullptr);
                const bool last = c + 1 == L->block_chunk[b + 1];
                if (s.bad_record >= 0 || (uint64_t)m.sym_off + s.entries != m1.sym_off || (!last && (uint64_t)m.pos0 + s.advance != m1.pos0)) {
                    report(c);
                    return;
                }
                my_v += s.vbits;
                my_i += s.ibits;
                L->chunk_nz[c] = s.weights;
                if (!L->slot.empty()) L->slot[(size_t)b * L->block_slots + (c - L->block_chunk[b])] = ChunkSlot{m.rec_off, m1.rec_off - m.rec_off, m.pos0, left + right};
                if (halves) {
                    L->chunk_half[2 * (size_t)c] = left;
                    L->chunk_half[2 * (size_t)c + 1] = right;
                }
                left += s.weights - s.right;
                right += s.right;
            }
            if (halves) {
                uint32_t at = 0;
                for (int h = 0; h < 2; ++h) {
                    uint32_t *gp = &L->group_ptr[(size_t)b * kPer + (size_t)h * (kGroups + 1)];
                    for (int q = 0; q < kGroups; ++q) {
                        gp[q] = at;
                        for (int r = q * kRows / kGroups; r < (q + 1) * kRows / kGroups; ++r) at += cnt[h * kRows + r];
                    }
                    gp[kGroups] = at;
                }
                if (!L->row_ptr.empty()) {
                    uint16_t *rp = &L->row_ptr[(size_t)b * L->row_ptrs], row_at = 0;
                    for (int r = 0; r < L->row_ptrs; ++r) {
                        rp[r] = row_at;
                        if (r < d.block_h) row_at = (uint16_t)(row_at + cnt[r] + cnt[kRows + r]);
                    }
                }
            }
        }
        vbits += my_v;
        ibits += my_i;
    });
    if (const int64_t c = bad_chunk.load(); c < L->n_chunks) {
        const cl_chunk_meta &m = L->meta[c], &m1 = L->meta[c + 1];
        int row_id, col_id, bhp, bwp;
        g.block(m.blk, row_id, col_id, bhp, bwp);
        const ChunkScan s = scan.chunk<false>(m.rec_off, m1.rec_off, m.pos0, (uint32_t)bwp, (uint64_t)bhp * bwp, nullptr);
        if (s.bad_record >= 0) return describe_bad_record(L, s.bad_record);
        if ((uint64_t)m.sym_off + s.entries != m1.sym_off) return fail(CL_ECORRUPT, "chunk %lld: symbol offset is wrong", (long long)c + 1);
        return fail(CL_ECORRUPT, "chunk %lld: position carry is wrong", (long long)c + 1);
    }
    uint32_t nnz = 0;
    for (int64_t c = 0; c <= L->n_chunks; ++c) {
        const uint32_t mine = L->chunk_nz[c];
        L->chunk_nz[c] = nnz;
        nnz += mine;
    }
    L->max_block_nnz = 0;
    for (int64_t b = 0; b < g.n_blocks; ++b) {
        const uint32_t c0 = L->block_chunk[b], c1 = L->block_chunk[b + 1], start = L->chunk_nz[c0];
        L->max_block_nnz = std::max<int64_t>(L->max_block_nnz, (int64_t)L->chunk_nz[c1] - start);
        if (!halves) continue;
        uint32_t *gp = &L->group_ptr[(size_t)b * kPer];
        const uint32_t n0 = gp[kGroups];
        for (int q = 0; q < kPer; ++q) gp[q] += start;
        for (uint32_t c = c0; c < c1; ++c) {
            L->chunk_half[2 * (size_t)c] += start;
            L->chunk_half[2 * (size_t)c + 1] += start + n0;
        }
    }
    L->max_group_blocks = 0;
    for (int p = 0; p < g.nbh; ++p)
        for (uint32_t c = L->panel_chunk[p]; c < L->panel_chunk[p + 1]; c += 8) {
            const uint32_t last = std::min<uint32_t>(c + 8, L->panel_chunk[p + 1]) - 1;
            L->max_group_blocks = std::max<int32_t>(L->max_group_blocks, (int32_t)(L->meta[last].blk - L->meta[c].blk) + 1);
        }
    L->nnz = nnz;
    L->padding = L->entries - (int64_t)nnz;
    L->val_bits = vbits;
    L->idx_bits = ibits;
    return CL_OK;
}

}  // namespace cl

using namespace cl;

extern "C" const char *cl_last_error(void) { return g_error; }

namespace {

// Smallest and largest surviving weight of W[i0, i1) (lo > hi: none), and the first element
// that is not finite (-1: none).  A pass over the matrix at memory speed.
struct Extent {
    float lo = std::numeric_limits<float>::infinity(), hi = -std::numeric_limits<float>::infinity();
    int64_t bad = -1;
};

Extent extent_of(const float *W, int64_t i0, int64_t i1)
{
    Extent e;
    const __m128 inf = _mm_set1_ps(std::numeric_limits<float>::infinity()), ninf = _mm_set1_ps(-std::numeric_limits<float>::infinity());
    __m128 lo = inf, hi = ninf, odd = _mm_setzero_ps();
    int64_t i = i0;
    for (; i + 4 <= i1; i += 4) {
        const __m128 w = _mm_loadu_ps(W + i), live = _mm_cmpneq_ps(w, _mm_setzero_ps());
        // w - w is 0 for a finite w and NaN otherwise
        odd = _mm_or_ps(odd, _mm_cmpunord_ps(_mm_sub_ps(w, w), w));
        lo = _mm_min_ps(_mm_or_ps(_mm_and_ps(live, w), _mm_andnot_ps(live, inf)), lo);
        hi = _mm_max_ps(_mm_or_ps(_mm_and_ps(live, w), _mm_andnot_ps(live, ninf)), hi);
    }
    float l[4], h[4];
    _mm_storeu_ps(l, lo);
    _mm_storeu_ps(h, hi);
    for (int q = 0; q < 4; ++q) { e.lo = std::min(e.lo, l[q]); e.hi = std::max(e.hi, h[q]); }
    bool any = _mm_movemask_ps(odd) != 0;
    for (; i < i1; ++i) {
        any = any || !std::isfinite(W[i]);
        if (W[i] != 0.0f) { e.lo = std::min(e.lo, W[i]); e.hi = std::max(e.hi, W[i]); }
    }
    if (any)
        for (i = i0; i < i1 && e.bad < 0; ++i)
            if (!std::isfinite(W[i])) e.bad = i;
    return e;
}

// f(column, weight) for the surviving weights of a row piece, in order.
template <class F>
void each_nonzero(const float *w, int n, F f)
{
    int c = 0;
    for (; c + 8 <= n; c += 8) {
        const __m128 z = _mm_setzero_ps();
        unsigned m = (unsigned)_mm_movemask_ps(_mm_cmpneq_ps(_mm_loadu_ps(w + c), z)) |
                     (unsigned)_mm_movemask_ps(_mm_cmpneq_ps(_mm_loadu_ps(w + c + 4), z)) << 4;
        for (; m; m &= m - 1) {
            const int at = c + __builtin_ctz(m);
            f(at, w[at]);
        }
    }
    for (; c < n; ++c)
        if (w[c] != 0.0f) f(c, w[c]);
}

// The index in 1 .. n - 1 of the codebook value nearest to a weight by the distance
// |w - centre| taken in fp64, the lowest index among equals.  The centres are sorted once; a
// weight lies between two neighbours, one of which has the smallest distance (rounding
// is monotone), and every centre at that same distance - duplicates, and centres so close
// together that their distances round alike - lies next to them.
class NearestCentre {
public:
    explicit NearestCentre(const std::vector<float> &codebook)
    {
        const int n = (int)codebook.size() - 1;
        index_.resize(n);
        for (int t = 0; t < n; ++t) index_[t] = t + 1;
        std::stable_sort(index_.begin(), index_.end(), [&](int a, int b) { return codebook[a] < codebook[b]; });
        for (int t : index_) c_.push_back((double)codebook[t]);
        // equally spaced centres: the position follows from the weight, and is put right below
        const double span = c_.back() - c_.front();
        scale_ = span > 0 ? (n - 1) / span : 0.0;
    }

    int operator()(float weight) const
    {
        const double w = (double)weight;
        const int n = (int)c_.size();
        const double guess = (w - c_[0]) * scale_;
        int t = guess > 0 ? (int)std::min(guess, (double)(n - 1)) : 0;
        while (t + 1 < n && c_[t + 1] <= w) ++t;
        while (t > 0 && c_[t] > w) --t;
        // c[t] <= w < c[t + 1], or w is outside the range
        const int below = t, above = t + 1 < n ? t + 1 : t;
        const double best = std::min(std::fabs(w - c_[below]), std::fabs(w - c_[above]));
        int idx = std::numeric_limits<int>::max();
        for (int i = below; i >= 0 && std::fabs(w - c_[i]) == best; --i) idx = std::min(idx, index_[i]);
        for (int i = above; i < n && std::fabs(w - c_[i]) == best; ++i) idx = std::min(idx, index_[i]);
        return idx;
    }

private:
    std::vector<int> index_;
    std::vector<double> c_;
    double scale_;
};

}  // namespace

extern "C" int32_t cl_compress_layer(const cl_layer_desc *desc, const float *W, const float *codebook_or_null,
                                     cl_layer **out)
{
    if (!desc || !W || !out) return fail(CL_EINVAL, "null argument");
    *out = nullptr;
    cl_layer_desc d = *desc;
    if (int32_t rc = check_desc(d)) return rc;
    const Geometry g(d);
    const int nval = 1 << d.weight_bits, nidx = 1 << d.index_bits, nc = nval - 1;
    const int64_t total = (int64_t)d.M * d.K;

    std::unique_ptr<cl_layer> L(new (std::nothrow) cl_layer);
    if (!L) return fail(CL_ENOMEM, "out of memory");
    try {
        Team team(total, kWeightsPerThread);
        L->desc = d;
        // ---- codebook (Sec. III-B: at most 2^r - 1 shared non-zero values plus 0) ----
        L->codebook.assign(nval, 0.0f);
        const int64_t pieces = std::min<int64_t>(total, (int64_t)team.size() * 4);
        std::vector<Extent> extent((size_t)pieces);
        team.each(pieces, [&](int64_t u) { extent[(size_t)u] = extent_of(W, total * u / pieces, total * (u + 1) / pieces); });
        Extent all;
        for (const Extent &e : extent) {
            all.lo = std::min(all.lo, e.lo);
            all.hi = std::max(all.hi, e.hi);
            if (all.bad < 0) all.bad = e.bad;
        }
        if (all.bad >= 0) return fail(CL_EINVAL, "non-finite weight at element %lld", (long long)all.bad);
        const bool have = all.lo <= all.hi;
        const double lo = all.lo, hi = all.hi;
        if (codebook_or_null) {
            if (codebook_or_null[0] != 0.0f) return fail(CL_EINVAL, "codebook[0] must be 0");
            for (int t = 0; t < nval; ++t) {
                if (!std::isfinite(codebook_or_null[t])) return fail(CL_EINVAL, "non-finite codebook entry");
                L->codebook[t] = codebook_or_null[t];
            }
        } else if (have) {
            for (int t = 1; t <= nc; ++t)
                L->codebook[t] = (float)(nc == 1 ? 0.5 * (lo + hi) : lo + (double)(t - 1) * (hi - lo) / (double)(nc - 1));
        }
        // ---- the rest goes by runs of consecutive blocks, which only meet again in the offsets:
        // value index of every surviving weight (nearest centre, ties to the lower index) and
        // the relative-indexed entries, block after block, row by row inside a block ----
        const NearestCentre nearest(L->codebook);
        const int R = 1 << d.index_bits;
        struct Unit {
            int64_t b0 = 0, b1 = 0;                 // its blocks
            std::vector<uint8_t> val, idx;          // their entries
            std::vector<int64_t> vcount, icount;
            std::vector<uint64_t> records;
            std::vector<cl_chunk_meta> meta;
            int64_t entry0 = 0, record0 = 0, chunk0 = 0;
        };
        const int64_t n_units = std::min<int64_t>(g.n_blocks, (int64_t)team.size() * 8);
        std::vector<Unit> units((size_t)n_units);
        L->block_ptr.assign((size_t)g.n_blocks + 1, 0);         // within the unit for now
        team.each(n_units, [&](int64_t i) {
            Unit &u = units[(size_t)i];
            u.b0 = g.n_blocks * i / n_units;
            u.b1 = g.n_blocks * (i + 1) / n_units;
            u.val.reserve((size_t)(total / n_units / 8 + 16));
            u.idx.reserve((size_t)(total / n_units / 8 + 16));
            for (int64_t b = u.b0; b < u.b1; ++b) {
                int row_id, col_id, bhp, bwp;
                g.block(b, row_id, col_id, bhp, bwp);
                L->block_ptr[(size_t)b] = (uint32_t)u.val.size();
                int64_t next = 0;                   // the cell after the last stored one
                for (int r = 0; r < bhp; ++r) {
                    const int64_t cell0 = (int64_t)r * bwp;
                    each_nonzero(W + (size_t)(row_id + r) * d.K + col_id, bwp, [&](int c, float w) {
                        int64_t run = cell0 + c - next;   // zeros since then
                        next = cell0 + c + 1;
                        while (run >= R) { u.val.push_back(0); u.idx.push_back((uint8_t)(R - 1)); run -= R; }
                        u.val.push_back((uint8_t)nearest(w));
                        u.idx.push_back((uint8_t)run);
                    });
                }
            }
            u.vcount.assign(nval, 0);
            u.icount.assign(nidx, 0);
            for (size_t e = 0; e < u.val.size(); ++e) { ++u.vcount[u.val[e]]; ++u.icount[u.idx[e]]; }
        });
        // ---- Huffman codes of the two arrays ----
        std::vector<int64_t> vcount(nval, 0), icount(nidx, 0);
        int64_t n_entries = 0;
        for (Unit &u : units) {
            u.entry0 = n_entries;
            n_entries += (int64_t)u.val.size();
            for (int t = 0; t < nval; ++t) vcount[t] += u.vcount[t];
            for (int t = 0; t < nidx; ++t) icount[t] += u.icount[t];
        }
        if (n_entries > std::numeric_limits<int32_t>::max()) return fail(CL_EINVAL, "more than 2^31-1 entries");
        if (!limited_code_lengths(vcount, d.max_code_len, L->val_len) || !limited_code_lengths(icount, d.max_code_len, L->idx_len))
            return fail(CL_EINVAL, "alphabet does not fit max_code_len");
        L->val_bits_unlimited = unlimited_code_bits(vcount);
        L->idx_bits_unlimited = unlimited_code_bits(icount);
        int dummy;
        if (!canonical_codes(L->val_len, L->val_code, &dummy) || !canonical_codes(L->idx_len, L->idx_code, &dummy))
            return fail(CL_EINVAL, "internal: code construction failed");
        std::vector<uint64_t> idx_top(nidx);                    // the codeword running down from bit 63
        for (int z = 0; z < nidx; ++z) idx_top[z] = bit_reverse64(L->idx_code[z]);
        // ---- lane records and chunks: a record takes as many whole entries as fit its 64 bits,
        // a chunk takes up to 64 records; neither crosses a block ----
        L->panel_chunk.assign((size_t)g.nbh + 1, 0);            // within the unit for now
        team.each(n_units, [&](int64_t i) {
            Unit &u = units[(size_t)i];
            u.records.reserve(u.val.size() / 6 + 16);
            for (int64_t b = u.b0; b < u.b1; ++b) {
                if (b % g.nbw == 0) L->panel_chunk[(size_t)(b / g.nbw)] = (uint32_t)u.meta.size();
                const int64_t be0 = L->block_ptr[(size_t)b], be1 = b + 1 < u.b1 ? L->block_ptr[(size_t)b + 1] : (int64_t)u.val.size();
                uint64_t possum = 0;
                int in_chunk = kLanes;
                for (int64_t e = be0; e < be1;) {
                    if (in_chunk == kLanes) {
                        cl_chunk_meta m;
                        m.sym_off = (uint32_t)(u.entry0 + e);
                        m.rec_off = (uint32_t)u.records.size();
                        m.blk = (uint32_t)b;
                        m.pos0 = (uint32_t)possum;
                        u.meta.push_back(m);
                        in_chunk = 0;
                    }
                    uint64_t rec = 0;
                    int vpos = kCountBits, itop = CL_RECORD_BITS, n = 0;     // value bits go up from vpos, index bits down from itop
                    while (e + n < be1 && n < CL_MAX_RECORD_ENTRIES) {
                        const uint8_t v = u.val[(size_t)(e + n)], z = u.idx[(size_t)(e + n)];
                        const int lv = L->val_len[v], li = L->idx_len[z];
                        if (vpos + lv + li > itop) break;
                        rec |= (uint64_t)L->val_code[v] << vpos;
                        vpos += lv;
                        rec |= idx_top[z] >> (CL_RECORD_BITS - itop);
                        itop -= li;
                        possum += (uint64_t)z + 1;
                        ++n;
                    }
                    rec |= (uint64_t)n;
                    u.records.push_back(rec);
                    e += n;
                    ++in_chunk;
                }
            }
        });
        // ---- the units put together ----
        int64_t n_records = 0, n_chunks = 0;
        for (Unit &u : units) {
            u.record0 = n_records;
            u.chunk0 = n_chunks;
            n_records += (int64_t)u.records.size();
            n_chunks += (int64_t)u.meta.size();
        }
        L->records.resize((size_t)n_records);
        L->meta.resize((size_t)n_chunks + 1);
        team.each(n_units, [&](int64_t i) {
            Unit &u = units[(size_t)i];
            if (!u.records.empty()) std::memcpy(&L->records[(size_t)u.record0], u.records.data(), u.records.size() * 8);
            for (size_t c = 0; c < u.meta.size(); ++c) {
                cl_chunk_meta m = u.meta[c];
                m.rec_off += (uint32_t)u.record0;
                L->meta[(size_t)u.chunk0 + c] = m;
            }
            for (int64_t b = u.b0; b < u.b1; ++b) {
                L->block_ptr[(size_t)b] += (uint32_t)u.entry0;
                if (b % g.nbw == 0) L->panel_chunk[(size_t)(b / g.nbw)] += (uint32_t)u.chunk0;
            }
            u = Unit{};
        });
        L->block_ptr[(size_t)g.n_blocks] = (uint32_t)n_entries;
        L->panel_chunk[(size_t)g.nbh] = (uint32_t)n_chunks;
        cl_chunk_meta sentinel{};
        sentinel.sym_off = (uint32_t)n_entries;
        sentinel.rec_off = (uint32_t)n_records;
        L->meta[(size_t)n_chunks] = sentinel;
        const int64_t vu = L->val_bits_unlimited, iu = L->idx_bits_unlimited;
        if (int32_t rc = finalize_and_validate(L.get(), team)) return fail(rc == CL_ECORRUPT ? CL_EINVAL : rc, "internal: self-check failed: %s", cl_last_error());
        L->val_bits_unlimited = vu;
        L->idx_bits_unlimited = iu;
    } catch (...) {
        return fail_with_exception();
    }
    *out = L.release();
    clear_error();
    return CL_OK;
}

extern "C" int32_t cl_layer_free(cl_layer *layer)
{
    if (!layer) return CL_OK;
    release_device(layer);
    delete layer;
    return CL_OK;
}

extern "C" int32_t cl_layer_stats(const cl_layer *L, cl_stats *s)
{
    if (!L || !s) return fail(CL_EINVAL, "null argument");
    std::memset(s, 0, sizeof *s);
    s->nnz = L->nnz;
    s->padding = L->padding;
    s->entries = L->entries;
    s->n_blocks = L->n_blocks;
    s->n_chunks = L->n_chunks;
    s->val_bits = L->val_bits;
    s->idx_bits = L->idx_bits;
    s->val_bits_unlimited = L->val_bits_unlimited;
    s->idx_bits_unlimited = L->idx_bits_unlimited;
    s->n_records = L->n_records;
    s->payload_bytes = L->n_records * 8;
    s->table_bytes = (int64_t)(L->meta.size() * sizeof(cl_chunk_meta) + L->block_ptr.size() * 4 + L->panel_chunk.size() * 4);
    s->model_bytes = s->payload_bytes + s->table_bytes + (int64_t)(L->codebook.size() * 4 + L->val_len.size() + L->idx_len.size());
    s->lut_bytes = (int64_t)((L->val_lut.size() + L->idx_lut.size()) * sizeof(lut_t));
    s->val_max_len = L->val_lut_bits;
    s->idx_max_len = L->idx_lut_bits;
    return CL_OK;
}

extern "C" int32_t cl_layer_host_view(const cl_layer *L, cl_host_view *v)
{
    if (!L || !v) return fail(CL_EINVAL, "null argument");
    v->desc = L->desc;
    v->codebook = L->codebook.data();
    v->val_len = L->val_len.data();
    v->val_code = L->val_code.data();
    v->idx_len = L->idx_len.data();
    v->idx_code = L->idx_code.data();
    v->block_ptr = L->block_ptr.data();
    v->panel_chunk = L->panel_chunk.data();
    v->chunk_meta = L->meta.data();
    v->chunk_nz = L->chunk_nz.data();
    v->max_block_nnz = L->max_block_nnz;
    v->max_group_blocks = L->max_group_blocks;
    v->chunk_half = L->chunk_half.empty() ? nullptr : L->chunk_half.data();
    v->group_ptr = L->group_ptr.empty() ? nullptr : L->group_ptr.data();
    v->records = L->records.data();
    v->n_blocks = L->n_blocks;
    v->n_chunks = L->n_chunks;
    v->n_records = L->n_records;
    v->n_entries = L->entries;
    v->n_panels = L->n_panels;
    return CL_OK;
}

// --------------------------------------------------------------------------- //
// Byte image: header, then the stored sections back to back (little endian).
// --------------------------------------------------------------------------- //
namespace {
struct ImageHeader {
    char magic[8];          // "CLZLAYER"
    uint32_t version;
    uint32_t header_bytes;
    cl_layer_desc desc;
    int64_t n_blocks, n_chunks, n_records, n_entries;
    int64_t val_bits_unlimited, idx_bits_unlimited;
    uint64_t checksum;      // FNV-1a over every byte after the header
};
constexpr uint64_t kFnvBasis = 1469598103934665603ull, kFnvPrime = 1099511628211ull;

uint64_t fnv1a(const uint8_t *p, size_t n, uint64_t h)
{
    for (size_t i = 0; i < n; ++i) { h ^= p[i]; h *= kFnvPrime; }
    return h;
}

// The same hash by several threads.  A step (h ^ byte) * prime changes only the low eight
// bits of h before it multiplies, and what those become depends on those alone.  So once
// the low byte with which a piece of the data starts is known, the piece can be hashed from
// that byte with zeros above it, and the bits above come in afterwards, multiplied by
// prime^length.  The low bytes at the pieces' starts are found in two walks that follow
// all sixteen values a nibble may have side by side: the low nibble first (its next value
// depends on nothing else), then the high one along the low one now known.
// (One chain of dependent multiplications: 5 ms for a 4.7 MB layer; this way 1.)
uint64_t fnv1a_team(const uint8_t *p, size_t n, Team &team)
{
    constexpr int kLanesPerUnit = 2;               // pieces a thread walks at once: two chains hide each other's latency
    const size_t pieces = (size_t)team.size() * kLanesPerUnit, len = n / pieces;
    if (team.size() == 1 || len < 64) return fnv1a(p, n, kFnvBasis);
    typedef uint8_t nibbles __attribute__((vector_size(16)));
    typedef uint16_t bytes __attribute__((vector_size(32)));
    std::vector<nibbles> low(pieces);
    std::vector<bytes> high(pieces);
    std::vector<uint8_t> start(pieces);
    std::vector<uint64_t> part(pieces);
    const nibbles iota{0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15};
    const bytes tens{0x00, 0x10, 0x20, 0x30, 0x40, 0x50, 0x60, 0x70, 0x80, 0x90, 0xa0, 0xb0, 0xc0, 0xd0, 0xe0, 0xf0};
    constexpr uint8_t kLow = (uint8_t)kFnvPrime;
    team.each(team.size(), [&](int64_t u) {
        const uint8_t *a = p + (size_t)u * 2 * len, *b = a + len;
        nibbles x = iota, y = iota;
        for (size_t i = 0; i < len; ++i) {
            x ^= a[i];
            y ^= b[i];
            x += x + x;                            // times 3: kLow mod 16
            y += y + y;
        }
        low[(size_t)u * 2] = x & (uint8_t)15;
        low[(size_t)u * 2 + 1] = y & (uint8_t)15;
    });
    static_assert((kLow & 15) == 3, "the multiplier of the low nibble");
    start[0] = (uint8_t)(kFnvBasis & 15);
    for (size_t q = 1; q < pieces; ++q) start[q] = low[q - 1][start[q - 1]];
    team.each(team.size(), [&](int64_t u) {
        const uint8_t *a = p + (size_t)u * 2 * len, *b = a + len;
        bytes x = tens | (uint16_t)start[(size_t)u * 2], y = tens | (uint16_t)start[(size_t)u * 2 + 1];
        for (size_t i = 0; i < len; ++i) {
            x = (x ^ (uint16_t)a[i]) * (uint16_t)kLow;
            y = (y ^ (uint16_t)b[i]) * (uint16_t)kLow;
        }
        high[(size_t)u * 2] = x;
        high[(size_t)u * 2 + 1] = y;
    });
    start[0] = (uint8_t)kFnvBasis;
    for (size_t q = 1; q < pieces; ++q) start[q] = (uint8_t)high[q - 1][start[q - 1] >> 4];
    team.each(team.size(), [&](int64_t u) {
        const uint8_t *a = p + (size_t)u * 2 * len, *b = a + len;
        uint64_t x = start[(size_t)u * 2], y = start[(size_t)u * 2 + 1];
        for (size_t i = 0; i < len; ++i) {
            x = (x ^ a[i]) * kFnvPrime;
            y = (y ^ b[i]) * kFnvPrime;
        }
        part[(size_t)u * 2] = x;
        part[(size_t)u * 2 + 1] = y;
    });
    uint64_t power = 1;
    for (size_t e = len, f = kFnvPrime; e; e >>= 1, f *= f)
        if (e & 1) power *= f;
    uint64_t h = kFnvBasis;
    for (size_t q = 0; q < pieces; ++q) h = part[q] + (h - start[q]) * power;
    return fnv1a(p + pieces * len, n - pieces * len, h);
}

const char kMagic[8] = {'C', 'L', 'Z', 'L', 'A', 'Y', 'E', 'R'};

template <class T>
size_t section_bytes(const std::vector<T> &v) { return v.size() * sizeof(T); }
}  // namespace

extern "C" int32_t cl_layer_serialize(const cl_layer *L, void *buf, size_t *bytes)
{
    if (!L || !bytes) return fail(CL_EINVAL, "null argument");
    const size_t need = sizeof(ImageHeader) + section_bytes(L->codebook) + section_bytes(L->val_len) +
                        section_bytes(L->idx_len) + section_bytes(L->block_ptr) + section_bytes(L->panel_chunk) +
                        section_bytes(L->meta) + section_bytes(L->records);
    if (!buf) { *bytes = need; return CL_OK; }
    if (*bytes < need) { *bytes = need; return fail(CL_EINVAL, "buffer too small: need %zu bytes", need); }
    ImageHeader h{};
    std::memcpy(h.magic, kMagic, 8);
    h.version = 2;
    h.header_bytes = sizeof(ImageHeader);
    h.desc = L->desc;
    h.n_blocks = L->n_blocks;
    h.n_chunks = L->n_chunks;
    h.n_records = L->n_records;
    h.n_entries = L->entries;
    h.val_bits_unlimited = L->val_bits_unlimited;
    h.idx_bits_unlimited = L->idx_bits_unlimited;
    char *p = (char *)buf + sizeof h;
    auto put = [&](const void *src, size_t n) { if (n) std::memcpy(p, src, n); p += n; };
    put(L->codebook.data(), section_bytes(L->codebook));
    put(L->val_len.data(), section_bytes(L->val_len));
    put(L->idx_len.data(), section_bytes(L->idx_len));
    put(L->block_ptr.data(), section_bytes(L->block_ptr));
    put(L->panel_chunk.data(), section_bytes(L->panel_chunk));
    put(L->meta.data(), section_bytes(L->meta));
    put(L->records.data(), section_bytes(L->records));
    try {
        Team team((int64_t)need, kBytesPerThread);
        h.checksum = fnv1a_team((const uint8_t *)buf + sizeof h, need - sizeof h, team);
    } catch (...) {
        return fail_with_exception();
    }
    std::memcpy(buf, &h, sizeof h);
    *bytes = need;
    return CL_OK;
}

extern "C" int32_t cl_layer_deserialize(const void *buf, size_t bytes, cl_layer **out)
{
    if (!buf || !out) return fail(CL_EINVAL, "null argument");
    *out = nullptr;
    if (bytes < sizeof(ImageHeader)) return fail(CL_ECORRUPT, "image shorter than its header");
    ImageHeader h;
    std::memcpy(&h, buf, sizeof h);
    if (std::memcmp(h.magic, kMagic, 8) || h.version != 2 || h.header_bytes != sizeof(ImageHeader))
        return fail(CL_ECORRUPT, "not a compressed-layer image");
    cl_layer_desc d = h.desc;
    if (check_desc(d) != CL_OK) return fail(CL_ECORRUPT, "bad descriptor: %s", cl_last_error());
    const Geometry g(d);
    if (h.n_blocks != g.n_blocks || h.n_chunks < 0 || h.n_entries < 0 || h.n_chunks > h.n_records || h.n_records > h.n_entries ||
        h.n_entries > std::numeric_limits<int32_t>::max())
        return fail(CL_ECORRUPT, "inconsistent counts");
    const size_t nval = (size_t)1 << d.weight_bits, nidx = (size_t)1 << d.index_bits;
    const size_t need = sizeof(ImageHeader) + nval * 4 + nval + nidx + ((size_t)g.n_blocks + 1) * 4 + ((size_t)g.nbh + 1) * 4 +
                        ((size_t)h.n_chunks + 1) * sizeof(cl_chunk_meta) + (size_t)h.n_records * 8;
    if (bytes != need) return fail(CL_ECORRUPT, "image size %zu does not match its header (%zu)", bytes, need);
    std::unique_ptr<cl_layer> L(new (std::nothrow) cl_layer);
    if (!L) return fail(CL_ENOMEM, "out of memory");
    try {
        Team team(h.n_records, kRecordsPerThread);
        if (fnv1a_team((const uint8_t *)buf + sizeof h, need - sizeof h, team) != h.checksum) return fail(CL_ECORRUPT, "checksum mismatch");
        L->desc = h.desc;
        const char *p = (const char *)buf + sizeof(ImageHeader);
        auto get = [&](auto &vec, size_t n) {
            vec.resize(n);
            if (n) std::memcpy(vec.data(), p, n * sizeof(vec[0]));
            p += n * sizeof(vec[0]);
        };
        get(L->codebook, nval);
        get(L->val_len, nval);
        get(L->idx_len, nidx);
        get(L->block_ptr, (size_t)g.n_blocks + 1);
        get(L->panel_chunk, (size_t)g.nbh + 1);
        get(L->meta, (size_t)h.n_chunks + 1);
        get(L->records, (size_t)h.n_records);
        if (L->meta[(size_t)h.n_chunks].sym_off != (uint64_t)h.n_entries) return fail(CL_ECORRUPT, "entry count mismatch");
        if (int32_t rc = finalize_and_validate(L.get(), team)) return rc;
    } catch (...) {
        return fail_with_exception();
    }
    L->val_bits_unlimited = h.val_bits_unlimited;
    L->idx_bits_unlimited = h.idx_bits_unlimited;
    *out = L.release();
    clear_error();
    return CL_OK;
}
